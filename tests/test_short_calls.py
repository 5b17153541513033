"""Launch shapes of calls with few (sequence, kv head) pairs: where a range starts to be cut, where the
number of workgroups per CU changes, and the limits of the chunk partials.

GPU cases are held to the fp64 oracle (max-abs 2e-3, rel-L2 1e-3, |dlse| 1e-4, the library's stated bar)
per partition, merged and fused; the plans are checked on the host through the workspace they ask for.
"""

import ctypes
import math

import pytest

from paper_2510_13223_amd import bana, workloads as W

ROW_BYTES = 129 * 4  # a chunk's output row and lse


def _chunks(B, Hq, Hkv, longest, total, **kw):
    d = bana.make_dims(B, Hq, Hkv, 8192, 100000, max_range_tokens=longest, total_range_tokens=total, **kw)
    ws = bana.lib().bana_decode_attn_workspace_bytes(ctypes.byref(d))
    return max(1, round(ws / (B * Hq * ROW_BYTES))), ws


def test_short_ranges_are_not_cut():
    for B, Hkv in ((1, 1), (1, 8), (8, 2), (31, 8)):
        assert _chunks(B, 4 * Hkv, Hkv, 448, 448 * B) == (1, 0)
        assert _chunks(B, 4 * Hkv, Hkv, 464, 464 * B)[0] == (8 if B * Hkv <= 16 else 1)
    # up to 64 blocks (128 without hints) only where that spares a wavefront enough of them
    assert _chunks(16, 32, 8, 800, 16 * 800)[0] == 1
    assert _chunks(8, 32, 8, 800, 8 * 800)[0] == 4
    assert _chunks(51, 28, 4, 1024, 0) == (1, 0) and _chunks(1, 32, 8, 2048, 0)[0] > 1


def test_without_hints_chunks_stay_below_a_bound():
    for B, G, Hkv, blocks, want in ((40, 4, 8, 505, 8), (23, 4, 8, 2799, 15), (60, 4, 8, 129, 3), (63, 4, 8, 384, 6),
                                    (1, 4, 8, 3750, 64), (28, 16, 2, 1875, 9), (28, 16, 2, 8192, 32)):
        assert _chunks(B, G * Hkv, Hkv, 16 * blocks, 0, plan_hint=1)[0] == want, (B, Hkv, blocks)


def test_wide_tables_without_hints_take_the_balanced_launch():
    """From 960 blocks on, where the pairs leave too few chunks to bound them otherwise and the workspace fits."""
    from test_library_abi import _balanced_bytes

    balanced = lambda B, Hq, Hkv, blocks, **kw: (
        _chunks(B, Hq, Hkv, 16 * blocks, 0, **kw)[1] == _balanced_bytes(B, Hq, Hkv))
    for B, Hq, Hkv in ((23, 32, 8), (100, 32, 2), (63, 64, 8), (500, 4, 1)):
        assert balanced(B, Hq, Hkv, 960) and balanced(B, Hq, Hkv, 8192) and not balanced(B, Hq, Hkv, 959)
        assert not balanced(B, Hq, Hkv, 8192, plan_hint=1)
    assert not balanced(1, 32, 8, 8192) and not balanced(39, 4, 1, 8192) and balanced(40, 4, 1, 8192)
    assert not balanced(64, 64, 8, 8192)  # 512 pairs
    assert not balanced(500, 16, 1, 8192, waves_hint=4) and balanced(500, 8, 1, 8192)


def test_planning_a_wide_table_takes_no_longer():
    """The chunk count is chosen among those that can be launched (at most 256), whatever the table's width."""
    import time

    wide = bana.make_dims(1, 32, 8, 1 << 26, 100000)
    ws = bana.lib().bana_decode_attn_workspace_bytes
    t0 = time.perf_counter()
    for _ in range(2000):
        ws(ctypes.byref(wide))
    assert time.perf_counter() - t0 < 1.0  # some 2 us each; a search over the width's chunks took 2 ms
    # One pair, chunks of 192 blocks: from 256 chunks' worth on, all 256.
    assert [_chunks(1, 4, 1, 16 * blocks, 0)[0] for blocks in (49152, 60000, 100000, 131071)] == [256] * 4


def test_even_ranges_get_one_workgroup_per_cu():
    for B, Hkv in ((1, 2), (3, 8), (16, 8), (32, 8), (33, 8), (100, 8)):
        n, _ = _chunks(B, 4 * Hkv, Hkv, 100000, 100000 * B)
        assert n == max(1, 256 // (B * Hkv)), (B, Hkv)


def test_few_active_ranges_of_a_large_batch_are_cut():
    """With a workspace the plan does not depend on the static scratch: few long ranges among empty ones take the
    balanced launch, and where that is not wanted or possible as many chunks as their merge pays for.  (That the
    no-allocation call accepts them all is checked by tests/c/sanitize_host.cpp.)"""
    from test_library_abi import _balanced_bytes

    for B, Hq, Hkv, active, longest, chunks in (
            (2048, 32, 8, 4, 120000, 8), (2000, 64, 8, 1, 131072, 6), (1000, 64, 8, 1, 131072, 9),
            (500, 64, 8, 2, 120000, 12), (256, 64, 8, 1, 65536, 12), (2048, 32, 8, 16, 30000, 3),
            (4096, 32, 8, 16, 65536, 3), (20000, 8, 2, 1, 120000, 5), (1520, 64, 4, 20, 8000, 1)):
        for spread in (1, 4):  # even ranges, and one long one
            total = longest * active if spread == 1 else longest + longest * (active - 1) // 8
            got, ws = _chunks(B, Hq, Hkv, longest, total, nonempty_ranges=active)
            if B <= 2048 and longest > 8000:
                assert ws == _balanced_bytes(B, Hq, Hkv), (B, active, spread)
            got, ws = _chunks(B, Hq, Hkv, longest, total, nonempty_ranges=active, plan_hint=1)
            assert got == chunks or (spread == 4 and got >= chunks), (B, active, spread, got)
    # without a hint of the total, too
    d = bana.make_dims(2048, 32, 8, 8192, 100000, nonempty_ranges=2)
    assert bana.lib().bana_decode_attn_workspace_bytes(ctypes.byref(d)) == _balanced_bytes(2048, 32, 8)


def test_short_balanced_launches_fit_the_static_scratch():
    """A short call of uneven ranges takes the balanced launch only where its whole workspace (piece rows, their lse,
    the prefix sums and the alignment between them) fits, so the no-allocation call keeps accepting it."""
    from test_library_abi import _balanced_bytes

    for Hq, Hkv, longest, total in ((64, 4, 8000, 8950), (64, 8, 3200, 3700)):
        need = {B: _chunks(B, Hq, Hkv, longest, total, nonempty_ranges=min(B, 20))[1] for B in range(1, 2049)}
        assert max(need.values()) <= bana.STATIC_SCRATCH_BYTES, (Hq, Hkv)
        assert any(ws == _balanced_bytes(B, Hq, Hkv) for B, ws in need.items())


GPU_CASES = [
    # B, Hq, Hkv, lengths (cycled), parts
    (1, 4, 1, [256], 1),          # a whole range per workgroup: 16 blocks, 4 wavefronts
    (1, 16, 1, [257], 1),         # 17 blocks, 8 wavefronts
    (3, 8, 2, [448, 447, 440], 1),
    (3, 8, 2, [449, 450, 464], 2),  # 29 blocks: cut, one block per wavefront
    (1, 2, 2, [5000], 2),         # 128 chunks allowed, 79 used
    (17, 32, 16, [700], 1),       # 272 pairs: one chunk
    (16, 32, 16, [700, 690], 1),  # 256 pairs
    (5, 8, 4, [4000, 2500, 2600, 2500, 2500], 2),   # longest below twice the mean
    (6, 32, 8, [6000, 900, 1200, 800, 1, 900], 1),  # up to four times
    (9, 16, 1, [9000, 300, 17, 40, 200, 600, 5, 90, 333], 3),  # beyond, group of 16
    (65, 8, 4, [2064, 1, 255, 256, 257, 15], 1),  # 129 blocks wide: without hints 3 chunks, of 16 blocks at least
    (65, 16, 1, [6200, 30, 1025, 1040], 2),       # likewise 388 blocks, group of 16
    (40, 4, 2, [16000, 40, 900, 17], 2),          # 1000 blocks wide: without hints balanced, or 7 chunks of 64 at least
    (300, 8, 2, [4000] + [1] * 74, 2),            # first partition: 4 even ranges among 296 empty ones, in 5 chunks
    (300, 32, 8, [9000] + [1] * 299, 2),          # one longer one: balanced
    (5000, 16, 2, [9000] + [1] * 2499, 2),        # 2 in a batch beyond the balanced launch: uncut
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(GPU_CASES)))
def test_short_call_shapes_match_the_oracle(case):
    from test_gpu_parity import _full_parity

    B, Hq, Hkv, cycle, parts = GPU_CASES[case]
    lens = [cycle[b % len(cycle)] for b in range(B)]
    # Cuts at any token; the ranges cover the sequence, as the helper expects; parts of short ones are empty.
    ranges = [[(L * p // parts, L * (p + 1) // parts) for L in lens] for p in range(parts)]
    w = W.make_custom(900 + case, B, Hq, Hkv, lens, ranges, q_scale=1 / math.sqrt(128))
    for kw in ({}, {"range_hints": False}, {"range_hints": False, "plan_hint": 1}, {"order_hints": False, "plan_hint": 1},
               {"use_workspace": False}):
        _full_parity(w, **kw)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [5, 8, 16, 17, 33, 96])
def test_merge_of_few_rows_at_its_edges(n):
    from test_gpu_parity import test_merge_matches_oracle_merge

    test_merge_matches_oracle_merge(n, 3, 8)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [5, 8, 16, 17, 33, 96])
def test_merge_of_few_rows_keeps_a_nan_lse(n):
    """Row r: part r % n has a NaN lse, the next part a finite one, the others are empty."""
    import torch

    lses = torch.full((n, n, 4), -math.inf)
    for b in range(n):
        lses[b, b] = math.nan
        lses[(b + 1) % n, b] = 1.0
    out, lse = torch.zeros(n, 4, 128, device="cuda"), torch.zeros(n, 4, device="cuda")
    bana.bana_merge_partials(torch.ones(n, n, 4, 128, device="cuda"), lses.cuda(), out, lse)
    assert torch.isnan(out).all() and torch.isnan(lse).all()
