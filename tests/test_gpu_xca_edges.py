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


def _with_magnitudes(q, k, v, do, tau):
    """One window and head in float64: (o, dv, dqh / nq) and, beside each, the sum of the
    magnitudes of the terms it is made of."""
    nq, nk = (np.maximum(np.sqrt((x * x).sum(0)), 1e-12) for x in (q, k))
    g = tau * ((q / nq).T @ (k / nk))
    a = np.exp(g - g.max(1, keepdims=True))
    a /= a.sum(1, keepdims=True)
    da, da_mag = do.T @ v, np.abs(do).T @ np.abs(v)
    dg = a * (da - (a * da).sum(1, keepdims=True))
    dg_mag = a * (da_mag + (a * da_mag).sum(1, keepdims=True))
    b, b_mag = tau * dg / nk / nq[:, None], abs(tau) * dg_mag / nk / nq[:, None]
    return ((v @ a.T, np.abs(v) @ a.T), (do @ a, np.abs(do) @ a), (k @ b.T, np.abs(k) @ b_mag.T))


@pytest.mark.parametrize("dtype,half_ulp", [("f16", 2.0 ** -11), ("bf16", 2.0 ** -8)])
def test_narrow_heads_in_fp32(sla, dtype, half_ulp):  # noqa: F811
    # at d = 16 the weights A and the matrices of the gradients are fp32: where terms
    # cancel, or a row is far smaller than its column's norm, an output is off by its own
    # rounding and what fp32 leaves, and not by a rounding of A, B or the row to 16 bits
    rng = np.random.default_rng([92, len(dtype)])
    lengths, H, d = rng.integers(4, 9, size=60).astype(np.int64), 6, 16
    ids = workloads.ids_from_lengths(lengths, rng)
    f32 = [rng.standard_normal((ids.size, H, d)).astype(np.float32) for _ in range(4)]
    f32[3] *= 1e3   # (dq of the rows below stays above fp16's subnormals)
    zero = np.zeros(ids.size, dtype=bool)
    for w in range(lengths.size):
        rows = np.flatnonzero(ids == w)
        f32[1][rows[0]] *= 1e3     # the norm of every k column
        f32[1][rows[1:]] *= 1e-3   # and rows far below it,
        f32[0][rows[1::2]] = 0     # whose dq, where q is zero, is dqh / nq alone
        zero[rows[1::2]] = True
    t = [workloads.cast_values(x, dtype) for x in f32]
    tau = np.linspace(-1.0, 3.0, H).astype(np.float32)
    got, _ = run_xca(sla, ids, lengths.size, t, tau, dtype)
    q, k, v, do = (oracle.widen(x, dtype) for x in t)
    for w in range(lengths.size):
        rows = ids == w
        for h in range(H):
            o, dv, dq = _with_magnitudes(*(x[rows, h] for x in (q, k, v, do)), float(tau[h]))
            for label, x, (r, mag), which in (("o", got[0], o, rows[rows]), ("dv", got[3], dv, rows[rows]),
                                              ("dq", got[1], dq, zero[rows])):
                # sums over at most 8 rows, 16 columns and their use in a logit up to 3,
                # an exponential, divisions: 128 roundings of 2^-24 at most; the storage
                # type's subnormals
                tol = half_ulp * np.abs(r) + 128 * 2.0 ** -24 * mag + 2.0 ** -25
                bad = np.abs(x[rows, h] - r)[which] > tol[which]
                assert not bad.any(), (label, w, h, int(bad.sum()))


@pytest.mark.parametrize("H,d", [(4, 32), (8, 16)])
def test_fp32_error_on_either_side(sla, H, d):  # noqa: F811
    # the same windows with and without empty slots beside them: on the vector units and on
    # the matrix cores; neither o nor dv is further from float64 there
    rng = np.random.default_rng([93, H, d])
    lengths = rng.integers(10, 120, size=80).astype(np.int64)
    ids = workloads.ids_from_lengths(lengths, rng)
    t = [workloads.normal_values(rng, ids.size, H, d, "f32") for _ in range(4)]
    err = {}
    for W in (80, 80 + ids.size // 28):
        got, ref = run_xca(sla, ids, W, t, np.linspace(0.5, 3.0, H), "f32")
        err[W > 80] = [float(np.linalg.norm(got[m] - ref[m]) / np.linalg.norm(ref[m])) for m in (0, 3)]
    # (errors of 160k values: their ratio scatters by well under a percent)
    assert all(a <= 1.05 * b for a, b in zip(err[False], err[True])), err


@pytest.mark.parametrize("dtype,thin", [("f32", False), ("f32", True), ("bf16", False)])
@pytest.mark.parametrize("d", [16, 32])
def test_norms_beyond_fp32(sla, d, dtype, thin):  # noqa: F811
    # a q column whose squares overflow fp32 divides to zero: a uniform softmax row, zero
    # dq, no NaN anywhere; and a gradient through a floored norm that passes the largest
    # fp32 value is infinite, of the exact value's sign
    rng = np.random.default_rng([94, d, len(dtype), thin])
    H, lengths = 2, THIN if thin else WINDOWS
    ids = workloads.ids_from_lengths(lengths, rng)
    f32 = [rng.standard_normal((ids.size, H, d)).astype(np.float32) for _ in range(4)]
    f32[0][:, 0, 3] = np.float32(1e25) * np.sign(f32[0][:, 0, 3])
    f32[0][:, 1, 5] = 0
    f32[2][:, 1], f32[3][:, 1] = f32[2][:, 1] * 1e16, f32[3][:, 1] * 1e16
    t = [workloads.cast_values(x, dtype) for x in f32]
    got, ref = run_xca(sla, ids, lengths.size, t, np.array([1.0, 1.0]), dtype)
    v, live = oracle.widen(t[2], dtype), np.isin(ids, np.flatnonzero(lengths > 1))
    assert all(np.isfinite(x[:, 0]).all() for x in got[:4])
    assert (got[1][:, 0, 3] == 0).all()
    assert np.abs(got[0][:, 0, 3] - v[:, 0].mean(1)).max() <= TOL[dtype] * np.abs(v[:, 0]).max()
    big = np.abs(ref[1][:, 1, 5]) > 3.5e38
    assert big[live].mean() > 0.5
    assert np.array_equal(got[1][big, 1, 5], np.sign(ref[1][big, 1, 5]) * np.inf)
    assert not np.isnan(got[1][:, 1]).any()
