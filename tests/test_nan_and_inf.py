"""What NaN and infinities become on their way through the attention and the merges.

A part, a chunk or a wavefront is left out only where it is empty (lse = -inf, no token): a NaN among its
scores reaches the rows it belongs to, however the launch divides the range, and no other row.
"""

import math

import numpy as np
import pytest
import torch

from paper_2510_13223_amd import bana

pytestmark = pytest.mark.gpu


def _merge(outs, lses):
    n, B, Hq, _ = outs.shape
    out, lse = torch.zeros(B, Hq, 128, device="cuda"), torch.zeros(B, Hq, device="cuda")
    bana.bana_merge_partials(outs.cuda(), lses.cuda(), out, lse)
    return out.cpu(), lse.cpu()


# One part count per kernel and thread-group count, few rows and many.
MERGES = [(1, 9, 4), (2, 9, 4), (4, 9, 4), (5, 9, 4), (8, 9, 4), (9, 9, 4), (17, 9, 4), (33, 9, 4), (96, 9, 4),
          (5, 1025, 4), (17, 1025, 8), (40, 1025, 8)]


@pytest.mark.parametrize("n,B,Hq", MERGES)
def test_merge_of_rows_with_only_nan_and_empty_parts(n, B, Hq):
    """Row b: 0 no live part, 1 one NaN part, 2 all parts NaN, 3 the last part NaN and one finite, 4 one finite."""
    lses = torch.full((n, B, Hq), -math.inf)
    for kind in range(5):
        rows = torch.arange(kind, B, 5)
        if kind == 1:
            lses[n // 2, rows] = math.nan
        elif kind == 2:
            lses[:, rows] = math.nan
        elif kind >= 3:
            lses[0, rows] = 2.0
            if kind == 3:
                lses[n - 1, rows] = math.nan  # n = 1: the only part
    outs = torch.ones(n, B, Hq, 128)
    outs[lses == -math.inf] = math.nan  # rows of empty parts never enter a sum
    out, lse = _merge(outs, lses)
    kind = torch.arange(B) % 5
    assert (out[kind == 0] == 0).all() and (lse[kind == 0] == -math.inf).all()
    bad = (kind >= 1) & (kind <= 3)
    assert torch.isnan(out[bad]).all() and torch.isnan(lse[bad]).all()
    assert (out[kind == 4] == 1).all() and (lse[kind == 4] == 2).all()


# (hints, workspace): the library's choice, whole ranges on 1, 4 and 8 wavefronts, chunks of each, the balanced launch.
PLANS = [{}, {"range_hints": False}, {"use_workspace": False}, {"plan_hint": 2},
         *({"waves_hint": w, "chunks_hint": c} for w, c in ((1, 1), (4, 1), (8, 1), (1, 3), (4, 3), (8, 5), (2, 40)))]


@pytest.mark.parametrize("kw", PLANS, ids=lambda kw: "-".join(f"{k}{v}" for k, v in kw.items()) or "chosen")
def test_nan_scores_reach_their_rows_in_every_launch_shape(kw):
    """A NaN query head poisons its rows, a block of NaN keys (alone in its wavefront's walk or chunk, or beside
    others) the rows of its kv head, in every partition that covers them; empty ranges stay empty and all other
    rows keep their bits."""
    from paper_2510_13223_amd import workloads as W
    from paper_2510_13223_amd.runner import DeviceWorkload

    lens = [700, 16, 1333, 33, 5]
    ranges = [[(0, 500), (0, 16), (0, 1300), (0, 17), (0, 0)], [(500, 700), (16, 16), (1300, 1333), (17, 33), (0, 5)]]
    w = W.make_custom(61, 5, 8, 2, lens, ranges, q_scale=1 / math.sqrt(128))
    dw = DeviceWorkload(w, **kw)

    def results():
        dw.run_checked()
        torch.cuda.synchronize()
        return [t.clone() for t in (dw.out_partials, dw.lses, dw.out, dw.lse_out, dw.fused_out, dw.fused_lse)]

    clean = results()
    assert all(not torch.isnan(t).any() for t in clean)
    bad = torch.zeros(5, 8, dtype=torch.bool, device="cuda")
    bad[0, 3] = bad[3, 7] = bad[4, 0] = True  # query heads
    for b, h in bad.nonzero().tolist():
        dw.q[b, h] = math.nan
    part_bad = torch.stack([bad, bad])
    for b, j, g in ((1, 0, 1), (2, 82, 0), (2, 40, 1)):  # the keys of one block of one kv head
        dw.k_cache[dw.block_table[b, j].long(), g] = math.nan
        bad[b, 4 * g:4 * g + 4] = True
        part_bad[1 if (b, j) == (2, 82) else 0, b, 4 * g:4 * g + 4] = True
    part_bad &= (dw.kv_end > dw.kv_begin)[:, :, None]
    for got, want, rows in zip(results(), clean, (part_bad, part_bad, bad, bad, bad, bad)):
        assert torch.isnan(got[rows]).all()
        assert torch.equal(got[~rows], want[~rows])


@pytest.mark.parametrize("n,B,Hq", [m for m in MERGES if m[0] > 4])
def test_merge_leaves_out_infinite_rows_of_vanishing_weight(n, B, Hq):
    """A part whose weight beside the row's largest underflows to 0 leaves no 0 x inf behind, also where its
    weight within a thread group, or the group's within the row, does not underflow."""
    g = torch.Generator().manual_seed(n)
    outs = torch.randn(n, B, Hq, 128, generator=g)
    lses = torch.rand(n, B, Hq, generator=g)
    far = torch.arange(n) % 4  # 0 near the row's largest, 1 out of fp32's range, 2 and 3 in two steps of half of it
    lses -= torch.tensor([0.0, 300.0, 120.0, 60.0])[far][:, None, None]
    outs[(far == 1) | (far == 2)] = math.inf
    out, lse = _merge(outs, lses)
    w = torch.softmax(lses.double(), 0)[..., None]
    want = (w * torch.where(w > 1e-40, outs.double(), 0.0)).sum(0)
    assert torch.isfinite(out).all()
    # fp32: the weights, their products and n sums of values up to top, rounded to 2^-24 each
    top = outs[torch.isfinite(outs)].abs().max().item()
    np.testing.assert_allclose(out.double().numpy(), want.numpy(), rtol=0, atol=(n + 8) * 2.0**-24 * top)
    np.testing.assert_allclose(lse.double().numpy(), torch.logsumexp(lses.double(), 0).numpy(), rtol=0, atol=1e-5)
