"""Scenes whose work items do not fill the GPU split their chunks into parts, each
of which takes a share of the chunk's non-empty windows: windows of a few rows
(up to 16 parts), chunks that span more window slots than one page of 64, long
windows beside them, and window lengths at the edges of the four-row groups of
the fp32 products."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads
from tests.test_gpu_parity import (_xca_tau, backward_parity, forward_parity, sla, xca_backward_parity,  # noqa: F401
                                   xca_parity)

pytestmark = pytest.mark.gpu

SCENES = {
    "thin": lambda rng: rng.integers(0, 4, size=400),
    "empty-slots": lambda rng: (rng.random(5000) < 0.05) * rng.integers(1, 3, size=5000),
    "long-beside": lambda rng: np.concatenate([rng.integers(0, 3, size=300), [65, 128, 129, 257, 300],
                                               rng.integers(0, 3, size=100)]),
    "groups-of-four": lambda rng: np.array([1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64] * 2),
    "one-row": lambda rng: np.array([0, 0, 1, 0]),
}


@pytest.mark.parametrize("dtype,H,d", [("f32", 2, 32), ("f32", 5, 16), ("f16", 4, 32), ("bf16", 3, 32),
                                       ("f16", 1, 16)])
@pytest.mark.parametrize("scene", sorted(SCENES))
def test_parts(sla, scene, dtype, H, d):  # noqa: F811
    rng = np.random.default_rng([71, sorted(SCENES).index(scene), H, d])
    lengths = SCENES[scene](rng).astype(np.int64)
    ids = workloads.ids_from_lengths(lengths, rng)
    n, W = ids.size, lengths.size
    q, k, v, do = (workloads.normal_values(rng, n, H, d, dtype) for _ in range(4))
    label = f"{scene} H{H} d{d}"
    forward_parity(sla, ids, None, n, W, q, k, v, dtype, label=label)
    xca_parity(sla, ids, None, n, W, q, k, v, _xca_tau(H), dtype, label=label)
    if scene != "one-row":
        backward_parity(sla, ids, None, n, W, q, k, v, do, dtype, label=label)
    else:
        one_row_backward(sla, ids, W, q, k, v, do, dtype)
    # (so few pairs of windows and heads run the kernels with a workgroup each, without parts)
    # dtau sums the shares of windows of a few rows, of either sign: against their magnitudes
    xca_backward_parity(sla, ids, None, n, W, q, k, v, do, _xca_tau(H), dtype, label=label,
                        dtau_scale=dtau_magnitude(ids, W, H, *(oracle.widen(x, dtype) for x in (q, k, v, do))))


def dtau_magnitude(ids, W, H, q, k, v, do):
    """The least over the heads of sum |dG N| over windows and entries (tau as in _xca_tau)."""
    tau, mag = _xca_tau(H), np.zeros(H)
    for w in range(W):
        rows = ids == w
        if rows.any():
            for h in range(H):
                qh, kh = (x[rows, h] / np.maximum(np.sqrt((x[rows, h] ** 2).sum(0)), 1e-12) for x in (q, k))
                nn = qh.T @ kh
                a = np.exp(tau[h] * nn - (tau[h] * nn).max(1, keepdims=True))
                a /= a.sum(1, keepdims=True)
                da = do[rows, h].T @ v[rows, h]
                mag[h] += np.abs(a * (da - (a * da).sum(1, keepdims=True)) * nn).sum()
    return mag.min()


def one_row_backward(S, ids, W, q, k, v, do, dtype):
    """Alone in its window a row has dv = dout and dq = dk = 0: what is left is the rounding
    of two cancelling sums of d terms up to max|dout| max|v| each (phi'(q) phi(k) / (phi(q).
    phi(k)) <= 1), whose operands are rounded once or twice to the storage type, which the
    error measure of the others (a relative one) does not fit."""
    from tests.gpu_util import TOL, to_dev, to_host64

    plan = S.build_segments(to_dev(ids.astype(np.int32)), num_windows=W)
    got = [to_host64(t, dtype) for t in S.backward(plan, *(to_dev(x, dtype) for x in (q, k, v, do)))]
    v64, do64 = (oracle.widen(x, dtype) for x in (v, do))
    unit = {"f32": 2.0 ** -24, "f16": 2.0 ** -11, "bf16": 2.0 ** -8}[dtype]
    left = 4 * unit * q.shape[2] * np.abs(do64).max() * np.abs(v64).max()
    assert np.abs(got[0]).max() <= left and np.abs(got[1]).max() <= left
    assert np.abs(got[2] - do64).max() <= TOL[dtype] * np.abs(do64).max()


@pytest.mark.parametrize("n,W", [(60000, 2049), (60001, 2049), (160000, 2048), (160001, 2048), (160001, 7), (130000, 2048),
                                 (130001, 2048), (75000, 2049), (75001, 2049), (40000, 3201), (40001, 3201),
                                 (10000, 5001), (10001, 5001), (440000, 1023), (440001, 1023), (130001, 1024)])
def test_builder_either_side_of_the_totals(sla, n, W):  # noqa: F811
    # the builder sums its window counts with atomics up to a number of counts, and over
    # the blocks' prefix rows above it: out-of-range ids, long windows and empty ones on
    # both sides, the plan bit for bit, a buffer used twice
    from tests.test_gpu_parity import check_plan
    from tests.gpu_util import to_dev

    rng = np.random.default_rng([72, n, W])
    ids = np.minimum(rng.geometric(3.0 / W, size=n) - 1, W - 1).astype(np.int32)   # uneven: long windows first
    ids[rng.random(n) < 0.01] = W + 5
    ids[rng.random(n) < 0.01] = -1
    plan = sla.build_segments(to_dev(ids), num_windows=W)
    check_plan(sla, plan, ids, W, 0)
    ids = ids[::-1].copy()
    plan = sla.build_segments(to_dev(ids), num_windows=W, plan_buf=plan.buf)
    check_plan(sla, plan, ids, W, 0)


@pytest.mark.parametrize("rows,per", [(60, 37), (2003, 37), (70001, 37), (500, 3), (3001, 5)])
@pytest.mark.parametrize("H,d", [(2, 32), (8, 32)])
def test_saved_qkv_beside_idle_waves(sla, rows, per, H, d):  # noqa: F811
    # the last chunk items leave waves without rows: with parts (few rows) and without
    # (many), they store nothing into the saved q, k, v; rows of no window keep what
    # the buffer held, the others hold the projection; windows of a few rows: a job that
    # several parts project is saved by one of them
    import torch
    from tests.gpu_util import to_dev

    rng = np.random.default_rng([73, rows, H, d])
    ids = rng.integers(0, max(1, rows // per), size=rows).astype(np.int32)
    ids[rng.random(rows) < 0.02] = -1
    C = H * d
    plan = sla.build_segments(to_dev(ids), num_windows=max(1, rows // per))
    gen = torch.Generator(device="cuda").manual_seed(73)
    rand = lambda *s: torch.randn(s, device="cuda", generator=gen)  # noqa: E731
    x, wq, bq = (t.bfloat16() for t in (rand(rows, C), rand(3 * C, C) / C**0.5, 1.0 + rand(3 * C)))
    wo = (rand(C, C) / C**0.5).bfloat16()
    ref = torch.addmm(bq.float(), x.float(), wq.float().t()).reshape(rows, 3, C).transpose(0, 1)
    inside = torch.from_numpy(ids >= 0).cuda()
    for _ in range(3):
        qkv = torch.full((3, rows, C), 7.0, dtype=torch.bfloat16, device="cuda")
        sla.forward_projected(plan, x, wq, wo, H, bq, qkv_out=qkv)
        assert torch.equal(qkv[:, ~inside], torch.full_like(qkv[:, ~inside], 7.0))
        # half a bf16 step of the value, and fp32 sums of up to 256 products
        assert (qkv.float() - ref).abs()[:, inside].le(ref.abs()[:, inside] * 2.0**-8 + 1e-4).all()
