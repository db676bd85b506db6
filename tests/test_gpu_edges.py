"""Kernels at the edges of their blocks and at the sizes where a dispatch rule
changes the path, against plain torch in FP64 or against the general path."""
from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 15, 17, 255, 1023, 1024, 1025, 5000])
@pytest.mark.parametrize("offset", [0, 1, 3])
def test_feature_stats_block_edges(n, offset):
    """Column means and 1/std around the 1024-row blocks, also for a matrix
    that starts 4 or 12 bytes past a 16-byte boundary.  FP64 sums rounded once
    to float32: 2^-24 of the value, and the variance's cancellation (its
    relative error is at most 64 n 2^-53 (mean^2 + var) / var, below 1e-9 for
    these columns)."""
    from paper_2607_02721_amd import learned
    g = torch.Generator(device="cuda").manual_seed(n)
    buf = torch.randn(n * 64 + 4, generator=g, device="cuda") * 2.0 + 1.0
    feat = buf[offset:offset + n * 64].view(n, 64)
    feat[:, 5] = 0.25       # a constant column: 1/std reads 1
    norm = learned.feature_stats(feat).double()
    x = feat.double()
    mean, std = x.mean(0), x.std(0, unbiased=False)
    inv = torch.where(std > 1e-9, 1 / std.clamp_min(1e-30), torch.ones_like(std))
    assert torch.all((norm[0] - mean).abs() <= 2.0 ** -24 * mean.abs() + 1e-12)
    assert torch.all((norm[1] - inv).abs() <= 1.0e-7 * inv)
