"""XCA at the edges of its values, on each of its three sets of kernels: a workgroup per
(window, head) with the long-window passes (few pairs), without (more pairs of thin
windows), and work items (many pairs; about 31 rows a slot, so that chunks are split
into parts).  An infinity or NaN in q, k or dout reaches the outputs and gradients that
the definition carries it to and no others; zero columns, norms beyond fp32, one-row
windows; the precision of each."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads
from tests.gpu_util import TOL, to_dev, to_host64
from tests.test_gpu_parity import GRAD_TOL, sla, xca_backward_parity, xca_parity  # noqa: F401

pytestmark = pytest.mark.gpu

# the windows looked at, and what stands beside them: with 6 heads 42, 1,980 and 1,980
# pairs, at 86, 4 and 31 rows per slot
WINDOWS = np.array([40, 64, 33, 300, 28, 50, 90], dtype=np.int64)
BESIDE = {"long": np.zeros(0, dtype=np.int64), "plain": np.arange(323) % 4, "items": 26 + np.arange(323) % 10}


def scene(layout, windows=WINDOWS):
    return np.concatenate([windows, BESIDE[layout]]).astype(np.int64)


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


@pytest.mark.parametrize("layout,value", [("long", "nan"), ("long", "inf"), ("plain", "nan"), ("items", "nan")])
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("name", ["q", "k", "dout"])
@pytest.mark.parametrize("H,d", [(6, 32), (6, 16)])
def test_not_finite(sla, name, value, H, d, dtype, layout):  # noqa: F811
    rng = np.random.default_rng([91, H, d, len(dtype), len(layout)])
    lengths = scene(layout)
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
@pytest.mark.parametrize("windows", [60, 640])   # the kernels of few pairs, and work items
def test_narrow_heads_in_fp32(sla, dtype, half_ulp, windows):  # noqa: F811
    # at d = 16 the weights A and the matrices of the gradients are fp32: where terms
    # cancel, or a row is far smaller than its column's norm, an output is off by its own
    # rounding and what fp32 leaves, and not by a rounding of A, B or the row to 16 bits
    rng = np.random.default_rng([92, len(dtype)])
    lengths, H, d = rng.integers(4, 9, size=windows).astype(np.int64), 6, 16
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
    lengths = rng.integers(10, 120, size=400).astype(np.int64)
    ids = workloads.ids_from_lengths(lengths, rng)
    t = [workloads.normal_values(rng, ids.size, H, d, "f32") for _ in range(4)]
    err = {}
    for W in (400, 400 + ids.size // 28):
        got, ref = run_xca(sla, ids, W, t, np.linspace(0.5, 3.0, H), "f32")
        err[W > 400] = [float(np.linalg.norm(got[m] - ref[m]) / np.linalg.norm(ref[m])) for m in (0, 3)]
    # (errors of 3 million values: their ratio scatters by well under a percent)
    assert all(a <= 1.05 * b for a, b in zip(err[False], err[True])), err


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("layout", sorted(BESIDE))
@pytest.mark.parametrize("d", [16, 32])
def test_norms_beyond_fp32(sla, d, layout, dtype):  # noqa: F811
    # a q column whose squares overflow fp32 divides to zero: a uniform softmax row, zero
    # dq, no NaN anywhere; and a gradient through a floored norm that passes the largest
    # fp32 value is infinite, of the exact value's sign
    rng = np.random.default_rng([94, d, len(dtype), len(layout)])
    H, lengths = 6, scene(layout)
    ids = workloads.ids_from_lengths(lengths, rng)
    f32 = [rng.standard_normal((ids.size, H, d)).astype(np.float32) for _ in range(4)]
    f32[0][:, 0, 3] = np.float32(1e25) * np.sign(f32[0][:, 0, 3])
    f32[0][:, 1, 5] = 0
    f32[2][:, 1], f32[3][:, 1] = f32[2][:, 1] * 1e16, f32[3][:, 1] * 1e16
    t = [workloads.cast_values(x, dtype) for x in f32]
    got, ref = run_xca(sla, ids, lengths.size, t, np.ones(H), dtype)
    v, live = oracle.widen(t[2], dtype), np.isin(ids, np.flatnonzero(lengths > 1))
    assert all(np.isfinite(x[:, 0]).all() for x in got[:4])
    assert (got[1][:, 0, 3] == 0).all()
    assert np.abs(got[0][:, 0, 3] - v[:, 0].mean(1)).max() <= TOL[dtype] * np.abs(v[:, 0]).max()
    big = np.abs(ref[1][:, 1, 5]) > 3.5e38
    assert big[live].mean() > 0.5
    assert np.array_equal(got[1][big, 1, 5], np.sign(ref[1][big, 1, 5]) * np.inf)
    assert not np.isnan(got[1][:, 1]).any()


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("layout", ["plain", "items"])
@pytest.mark.parametrize("d", [16, 32])
def test_degenerate(sla, d, layout, dtype):  # noqa: F811
    # a zero q column and a zero k column (their norms take the floor), tau = 0, a sharp
    # softmax, one- and two-row windows with small columns (whose dq and dk are 0 for one
    # row): as the tests of few windows, on the kernels of more
    rng = np.random.default_rng([95, d, len(dtype), len(layout)])
    H = 6
    lengths = scene(layout, np.array([5, 1, 70, 0, 33, 2, 1, 2, 1, 300]))
    ids = workloads.ids_from_lengths(lengths, rng)
    n, W = ids.size, lengths.size
    q, k, v, do = (workloads.normal_values(rng, n, H, d, dtype) for _ in range(4))
    # (zero columns in the first ten windows only: of a gradient through a floored norm fp32
    # leaves 2^-24 of its terms / 1e-12, some 1e4, so that among many the rare one below
    # fp16's range would be all rounding; in the others it is infinite on both sides)
    first = ids < 10
    q[first, 1, 7] = 0
    k[first, 2, d - 2] = 0
    small = np.isin(ids, np.flatnonzero(lengths[:10] <= 2))
    for x in (q, k):
        x32 = oracle.widen(x, dtype)
        x32[small, 3, :] *= 1e-3
        x[...] = workloads.cast_values(x32.astype(np.float32), dtype)
    label = f"degenerate {layout} d{d}"
    xca_parity(sla, ids, None, n, W, q, k, v, np.array([0.0, 40.0, 1.0, -3.0, 0.5, 2.0]), dtype, label=label)
    xca_backward_parity(sla, ids, None, n, W, q, k, v, do, np.array([0.0, 2.0, 1.0, -3.0, 0.5, 2.0]), dtype, label=label)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("d", [16, 32])
def test_thin_windows_on_items(sla, d, dtype):  # noqa: F811
    # many slots, few of them with a row or three: work items whose chunks span pages of 64
    # slots and are split into parts
    rng = np.random.default_rng([96, d, len(dtype)])
    lengths = (rng.random(4000) < 0.1) * rng.integers(1, 4, size=4000)
    ids = workloads.ids_from_lengths(lengths.astype(np.int64), rng)
    n, W, H = ids.size, lengths.size, 2
    q, k, v, do = (workloads.normal_values(rng, n, H, d, dtype) for _ in range(4))
    tau = np.array([-1.5, 4.0])
    xca_parity(sla, ids, None, n, W, q, k, v, tau, dtype, label=f"thin d{d}")
    xca_backward_parity(sla, ids, None, n, W, q, k, v, do, tau, dtype, label=f"thin d{d}")
