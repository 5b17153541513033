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
