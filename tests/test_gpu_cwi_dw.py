"""Kernel gradients of the cross-window interaction where dy is not finite: a tap
without a neighbour contributes nothing, also for a row whose dy is infinite or
NaN, and such a row spoils its own channel only.  One to four pieces of channels,
several slices of taps, blocks that end inside a step of 32 rows."""
from __future__ import annotations

import numpy as np
import pytest

from tests.gpu_util import to_dev
from tests.test_gpu_parity import sla  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,kx,ky,n,gz", [(32, 3, 17, 33, 2), (64, 13, 13, 700, 3), (128, 5, 1, 300, 1), (256, 3, 3, 64, 1),
                                          (128, 3, 5, 500, 3)])   # the last: k_cwi_dw
def test_dw_not_finite(sla, C, kx, ky, n, gz):  # noqa: F811
    import torch

    rng = np.random.default_rng([81, C, n])
    grid, c = (40, 23, gz), C // 4
    cells = np.sort(rng.choice(grid[0] * grid[1] * gz, size=n, replace=False))
    coords = np.stack([cells % 40, cells // 40 % 23, cells // (40 * 23)], axis=1).astype(np.int32)
    x = rng.standard_normal((n, C)).astype(np.float16)
    dy = rng.standard_normal((n, C)).astype(np.float16)
    bad = {(n - 1, 0): np.inf, (n // 2, c + 1): np.nan, (0, 2 * c + 3): -np.inf}   # (row, channel)
    for (r, ch), v in bad.items():
        dy[r, ch] = v
    w = [(rng.standard_normal((k, c)) / 4).astype(np.float16) for k in (kx, ky, 27)]
    cc = to_dev(coords)
    m, conflicts = sla.cwi_build_map(cc, grid)
    got = sla.cwi_backward(m, grid, cc, to_dev(x), *(to_dev(t) for t in w), to_dev(dy))[1:]
    torch.cuda.synchronize()
    assert int(conflicts.cpu()[0]) == 0
    at = {tuple(p): r for r, p in enumerate(coords.tolist())}
    x64, dy64 = x.astype(np.float64), dy.astype(np.float64)
    for b, (k, t) in enumerate(zip((kx, ky, 27), got)):
        ref, mag = np.zeros((k, c)), np.zeros((k, c))
        for tap in range(k):
            h = tap - k // 2
            d = ((h, 0, 0), (0, h, 0), (tap % 3 - 1, tap // 3 % 3 - 1, tap // 9 - 1))[b]
            pairs = [(r, at[q]) for r, p in enumerate(coords.tolist())
                     if (q := (p[0] + d[0], p[1] + d[1], p[2] + d[2])) in at]
            if pairs:
                rows, nbs = np.array(pairs).T
                with np.errstate(invalid="ignore"):
                    prod = dy64[rows, b * c:(b + 1) * c] * x64[nbs, b * c:(b + 1) * c]
                    ref[tap], mag[tap] = prod.sum(0), np.abs(prod).sum(0)
        g = t.cpu().numpy().astype(np.float64)
        assert np.array_equal(np.isnan(g), np.isnan(ref)) and np.array_equal(np.isinf(g), np.isinf(ref))
        fine = np.isfinite(ref)
        # fp32 sums of n terms (2^-24 n of their magnitudes), rounded once to fp16
        tol = 2.0 ** -11 * np.abs(ref[fine]) + 2.0 ** -24 * n * mag[fine] + 1e-7
        assert np.all(np.abs(g[fine] - ref[fine]) <= tol)
