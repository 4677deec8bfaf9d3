"""XCA at the edges of its values.  An infinity or NaN in q, k or dout reaches the
outputs and gradients that the definition carries it to and no others, in every
storage type and on both sides of the line between the vector-unit and the
matrix-core kernels (fp32, 28 rows per window slot)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads
from tests.gpu_util import TOL, to_dev, to_host64
from tests.test_gpu_parity import GRAD_TOL, sla  # noqa: F401

pytestmark = pytest.mark.gpu

WINDOWS = np.array([40, 64, 33, 300, 28, 50, 90], dtype=np.int64)   # 86 rows per slot: the matrix-core kernels
THIN = np.concatenate([WINDOWS, np.ones(40, dtype=np.int64)])        # 13 per slot: fp32 on the vector units


def run_xca(S, ids, W, tensors, tau, dtype):
    """o, dq, dk, dv (float64) and dtau, and the same from the oracle."""
    import torch

    tq, tk, tv, tdo = (to_dev(a, dtype) for a in tensors)
    tau = np.asarray(tau, dtype=np.float32)
    ttau = torch.from_numpy(tau).cuda()
    plan = S.build_segments(to_dev(ids.astype(np.int32)), num_windows=W)
    o = S.forward_xca(plan, tq, tk, tv, ttau)
    g = S.backward_xca(plan, tq, tk, tv, ttau, tdo)
    torch.cuda.synchronize()
    got = [to_host64(t, dtype) for t in (o, *g[:3])] + [g[3].cpu().numpy().astype(np.float64)]
    perm, off, _ = oracle.segments_ref(ids, W)
    q, k, v, do = (oracle.widen(a, dtype) for a in tensors)
    tau = tau.astype(np.float64)
    with np.errstate(all="ignore"):
        ref = [oracle.xca_forward_ref(q, k, v, tau, off, perm), *oracle.xca_backward_ref(q, k, v, tau, do, off, perm)]
    return got, ref


def _bits(dtype, x):
    return workloads.cast_values(np.float32(x).reshape(1), dtype)[0]


@pytest.mark.parametrize("dtype,thin", [("f32", False), ("f32", True), ("f16", False), ("bf16", False)])
@pytest.mark.parametrize("name", ["q", "k", "dout"])
@pytest.mark.parametrize("value", ["nan", "inf"])
@pytest.mark.parametrize("H,d", [(5, 32), (6, 16)])
def test_not_finite(sla, name, value, H, d, dtype, thin):  # noqa: F811
    rng = np.random.default_rng([91, H, d, len(dtype), thin])
    lengths = THIN if thin else WINDOWS
    ids = workloads.ids_from_lengths(lengths, rng)
    t = dict(zip(("q", "k", "v", "dout"), (workloads.normal_values(rng, ids.size, H, d, dtype) for _ in range(4))))
    for w, h, e in ((2, 1, d - 1), (3, 0, 4)):   # a window of one chunk, and a long one
        t[name][np.flatnonzero(ids == w)[-2], h, e] = _bits(dtype, float(value))
    got, ref = run_xca(sla, ids, lengths.size, t.values(), np.linspace(0.5, 3.0, H), dtype)
    for label, x, r in zip(("o", "dq", "dk", "dv", "dtau"), got, ref):
        assert np.array_equal(~np.isfinite(x), ~np.isfinite(r)), f"{label}: not finite in other places"
        fine = np.isfinite(r)
        tol = TOL[dtype] if label == "o" else GRAD_TOL[dtype]
        assert np.abs(x[fine] - r[fine]).max() <= tol * np.abs(r[fine]).max(), label
