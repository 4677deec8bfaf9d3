"""Performance cases: the calls a program that uses this library makes, over the
sizes, types and options it makes them at.

    listed()              the named cases
    draw(rng)             one more case of the same ranges
    prepare(case, seed)   inputs (and the plan, weights, cell table) on the GPU
    run(state)            one pass through paper_2401_00912_amd.sla
    exact(case, seed)     the same outputs in float64, plain torch on the CPU
    work(case)            bytes and operations one pass cannot do without
    tolerance(case)       how far another correct implementation may be off

A case is a dict of
    kind          "forward"      attention on a plan in hand (rows already window-sorted)
                  "infer"        segment build and attention
                  "train"        segment build, attention and its gradients
                  "block_infer"  projections fused with the attention, plan in hand
                  "block_train"  the same with the gradients of the input and the weights
                  "cwi_train"    cross-window interaction and its gradients, cell table in hand
                  "xca_train"    cross-covariance attention and its gradients, plan in hand
    scene         "frame": pillars of LiDAR-like frames (density ~ 1 / range) on a
                  468 x 468 grid, cut into side x side windows;
                  "sparse": windows of log-normal length (median 20, up to 1,024 and
                  some empty);
                  "short": windows of 1 .. 60 rows.
                  Rows come in random order, window-sorted for "forward"
    rows          voxels in all frames together
    frames        frames in the batch ("frame")
    side          window side in pillars ("frame")
    heads, head_dim, dtype
    relu          ReLU feature map with eps = 1e-6 in place of elu + 1
    saved         "block_train": the forward keeps q, k, v for the backward
    taps, depth   "cwi_train": taps of the axis branches, cells of the grid along z

Values are what the modules see in a network: N(0, 1) rows (after a normalisation
layer), projection weights ~ N(0, 1 / C), convolution weights ~ N(0, 1 / taps).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2401_00912_amd import sla

GRID = 468
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


def _case(name, kind, scene, rows, heads, head_dim, dtype, *, frames=1, side=12, relu=False, saved=False,
          taps=13, depth=1):
    c = dict(kind=kind, scene=scene, rows=rows, frames=frames, side=side, heads=heads, head_dim=head_dim,
             dtype=dtype, relu=relu, saved=saved, taps=taps, depth=depth)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # a crop of a scene, already window-sorted: the smallest call, where latency counts
        _case("tiny_forward_f32", "forward", "short", 1894, 2, 32, "f32"),
        # the training step of one Waymo-like frame, as configured in the paper (C = 128, 4 heads)
        _case("frame_train_f16", "train", "frame", 59837, 4, 32, "f16"),
        # inference on a large scene with very uneven windows
        _case("sparse_infer_bf16", "infer", "sparse", 200000, 8, 16, "bf16"),
        # a batch of four frames on one GPU, wide channels
        _case("batch_train_bf16", "train", "frame", 240011, 8, 32, "bf16", frames=4),
        # the same training step in single precision
        _case("frame_train_f32", "train", "frame", 59837, 4, 32, "f32"),
        # the ReLU linear-attention variant, narrow heads, a thinner frame
        _case("frame_relu_train_bf16", "train", "frame", 41003, 8, 16, "bf16", relu=True),
        # a block's attention with its projections: inference on one frame
        _case("block_infer_f16", "block_infer", "frame", 59837, 4, 32, "f16"),
        # the same block in training
        _case("block_train_bf16", "block_train", "frame", 59837, 4, 32, "bf16"),
        # and in training on a batch with wide channels: the largest call
        _case("block_batch_train_bf16", "block_train", "frame", 240011, 8, 32, "bf16", frames=4),
        # cross-window interaction on pillars
        _case("cwi_pillars_train_f16", "cwi_train", "frame", 59837, 4, 32, "f16"),
        # cross-window interaction on voxels: the 3 x 3 x 3 branch sees all its taps
        _case("cwi_voxels_train_bf16", "cwi_train", "frame", 80021, 4, 16, "bf16", depth=8),
        # the XCA variant in training on one frame
        _case("xca_train_f16", "xca_train", "frame", 59837, 4, 32, "f16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forward", "infer", "train", "train", "train", "block_infer", "block_train", "block_train",
                       "cwi_train", "cwi_train", "xca_train"])
    dtype = rng.choice(["f16", "bf16", "f32"])
    head_dim = rng.choice([32, 32, 16])
    relu, saved, depth, taps = False, False, 1, 13
    if kind in ("block_infer", "block_train"):
        dtype = rng.choice(["f16", "bf16"])
        channels = rng.choice([64, 128, 128, 256])
        saved = kind == "block_train" and rng.random() < 0.3
    elif kind == "cwi_train":
        channels = rng.choice([64, 128, 128, 256])
        depth = rng.choice([1, 1, 5, 8])
        taps = rng.choice([9, 11, 13, 13, 15])
    else:
        channels = rng.choice([64, 128, 128, 192, 256])
        relu = kind in ("infer", "train") and rng.random() < 0.25
    scene = rng.choice(["frame", "frame", "frame", "sparse"])
    if kind == "cwi_train":
        scene = "frame"
    if kind == "forward":
        scene = rng.choice(["short", "short", "frame"])
    side = rng.choice([8, 10, 12, 12, 16])
    frames = 1
    # the largest: four frames of 60k pillars at C = 256 in 16 bits; the fp32, XCA and
    # 3-D convolution paths stop at a quarter of that
    most = 240000 * 256 // channels
    if dtype == "f32" or kind == "xca_train" or depth > 1:
        most //= 4
    most = min(most, 240000)
    rows = _log_int(rng, 1500, most)
    if scene == "frame" and kind != "cwi_train":
        frames = min(4, max(1, -(-rows // 75000)))
    elif kind == "cwi_train":
        rows = min(rows, 120000)
    elif scene == "short":
        rows = min(rows, 30000)
    return _case(None, kind, scene, rows, channels // head_dim, head_dim, dtype, frames=frames, side=side, relu=relu,
                 saved=saved, taps=taps, depth=depth)


# ------------------------------------------------------------------- geometry
_logp = {}


def _cell_logp(depth):
    """log occupancy weight of every cell of the grid (x fastest, then y, then z)."""
    if depth not in _logp:
        c = np.arange(GRID) + 0.5 - GRID / 2
        r = np.sqrt(c[None, :] ** 2 + c[:, None] ** 2)
        # min(1, 1 / range) inside the sensor range; points gather near the ground
        lp = np.where(r <= GRID / 2, -np.log(np.maximum(r, 12.0)), -np.inf)
        _logp[depth] = np.concatenate([(lp - 0.5 * z).ravel() for z in range(depth)]).astype(np.float32)
    return _logp[depth]


def _pillars(rng, rows, depth=1):
    """x, y, z of `rows` distinct cells, drawn without replacement by their weights, in raster order."""
    lp = _cell_logp(depth)
    key = lp - np.log(rng.standard_exponential(lp.size, dtype=np.float32))   # Gumbel top-k
    cells = np.sort(np.argpartition(-key, rows - 1)[:rows])
    return cells % GRID, cells // GRID % GRID, cells // (GRID * GRID)


def _windows(case):
    if case["scene"] == "frame":
        return case["frames"] * (-(-GRID // case["side"])) ** 2
    if case["scene"] == "sparse":
        return max(8, case["rows"] // 49)
    return max(4, case["rows"] // 30)


def _ids(case, seed):
    """Window id of every row."""
    rng = np.random.default_rng([1, seed])
    n, W = case["rows"], _windows(case)
    if case["scene"] == "frame":
        f, side = case["frames"], case["side"]
        per = -(-GRID // side)
        parts = []
        for i in range(f):
            x, y, _ = _pillars(rng, n * (i + 1) // f - n * i // f)
            parts.append((y // side) * per + x // side + i * per * per)
        ids = np.concatenate(parts)
    elif case["scene"] == "sparse":
        weight = np.minimum(rng.lognormal(math.log(20.0), 1.34, size=W), 1024.0)
        ids = np.repeat(np.arange(W), rng.multinomial(n, weight / weight.sum()))
    else:
        lengths = rng.integers(1, 61, size=W)
        ids = np.repeat(np.arange(W), rng.multinomial(n, lengths / lengths.sum()))
    ids = np.sort(ids) if case["kind"] == "forward" else ids[rng.permutation(n)]
    return ids.astype(np.int32)


# --------------------------------------------------------------------- inputs
def _shape(case):
    return case["rows"], case["heads"], case["head_dim"]


def _variant(case):
    return dict(feature_map="relu", eps=1e-6) if case["relu"] else {}


def _inputs(case, seed):
    """Inputs of the pass as torch tensors: geometry on the CPU, values on the GPU."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1_000_003 * int(seed) + 17)
    dt = DTYPES[case["dtype"]]
    n, H, d = _shape(case)
    C = H * d
    rand = lambda *shape, scale=1.0: (torch.randn(*shape, device="cuda", generator=gen) * scale).to(dt)  # noqa: E731
    s = {}
    if case["kind"] == "cwi_train":
        rng = np.random.default_rng([1, seed])
        x, y, z = _pillars(rng, n, case["depth"])
        s["coords"] = torch.from_numpy(np.stack([x, y, z], axis=1).astype(np.int32))
        c, k = C // 4, case["taps"]
        s.update(x=rand(n, C), w_x=rand(k, c, scale=k ** -0.5), w_y=rand(k, c, scale=k ** -0.5),
                 w_3=rand(27, c, scale=27 ** -0.5), dy=rand(n, C))
        return s
    s["ids"] = torch.from_numpy(_ids(case, seed))
    if case["kind"] in ("block_infer", "block_train"):
        s.update(x=rand(n, C), w_qkv=rand(3 * C, C, scale=C ** -0.5), b_qkv=rand(3 * C, scale=0.1),
                 w_o=rand(C, C, scale=C ** -0.5), b_o=rand(C, scale=0.1))
        if case["kind"] == "block_train":
            s["dy"] = rand(n, C)
        return s
    s.update(q=rand(n, H, d), k=rand(n, H, d), v=rand(n, H, d))
    if case["kind"] in ("train", "xca_train"):
        s["dout"] = rand(n, H, d)
    if case["kind"] == "xca_train":
        s["tau"] = torch.linspace(0.5, 3.0, H, device="cuda")
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    if case["kind"] == "cwi_train":
        s["coords"] = s["coords"].cuda()
        s["grid"] = (GRID, GRID, case["depth"])
        s["map"], _ = sla.cwi_build_map(s["coords"], s["grid"])
        return s
    n, W = case["rows"], _windows(case)
    ids = s["ids"]
    s["ids"] = ids.cuda()
    if case["kind"] == "forward":
        off = torch.zeros(W + 1, dtype=torch.int32)
        off[1:] = torch.cumsum(torch.bincount(ids.long(), minlength=W), 0)
        s["plan"] = sla.build_segments(num_windows=W, offsets=off.cuda(), n=n)
    elif case["kind"] in ("infer", "train"):
        s["plan_buf"] = sla.new_plan_buffer(n, W, "cuda")
    else:
        s["plan"] = sla.build_segments(s["ids"], W)
    return s


# ----------------------------------------------------------------------- pass
def run(s):
    case = s["case"]
    kind, H, var = case["kind"], case["heads"], _variant(case)
    if kind == "forward":
        return {"o": sla.forward(s["plan"], s["q"], s["k"], s["v"], **var)}
    if kind in ("infer", "train"):
        plan = sla.build_segments(s["ids"], _windows(case), plan_buf=s["plan_buf"])
        out = {"perm": plan.perm, "offsets": plan.offsets, "o": sla.forward(plan, s["q"], s["k"], s["v"], **var)}
        if kind == "train":
            out["dq"], out["dk"], out["dv"] = sla.backward(plan, s["q"], s["k"], s["v"], s["dout"], **var)
        return out
    if kind in ("block_infer", "block_train"):
        w = (s["x"], s["w_qkv"], s["w_o"])
        qkv = torch.empty((3, *s["x"].shape), dtype=s["x"].dtype, device="cuda") if case["saved"] else None
        o, y = sla.forward_projected(s["plan"], *w, H, b_qkv=s["b_qkv"], b_o=s["b_o"], qkv_out=qkv)
        out = {"o": o, "y": y}
        if kind == "block_train":
            g = sla.backward_projected(s["plan"], *w, o, s["dy"], H, b_qkv=s["b_qkv"], qkv=qkv)
            out.update(zip(("dx", "dw_qkv", "db_qkv", "dw_o", "db_o"), g))
        return out
    if kind == "cwi_train":
        args = (s["map"], s["grid"], s["coords"], s["x"], s["w_x"], s["w_y"], s["w_3"])
        y = sla.cwi_forward(*args)
        return dict(zip(("y", "dx", "dw_x", "dw_y", "dw_3"), (y, *sla.cwi_backward(*args, s["dy"]))))
    o = sla.forward_xca(s["plan"], s["q"], s["k"], s["v"], s["tau"])
    g = sla.backward_xca(s["plan"], s["q"], s["k"], s["v"], s["tau"], s["dout"])
    return dict(zip(("o", "dq", "dk", "dv", "dtau"), (o, *g)))


# ------------------------------------------------------------- float64 results
def _window_batches(ids, limit=1 << 16):
    """Row indices [windows, longest] and a mask, windows of like length together."""
    order = torch.argsort(ids, stable=True)
    lens = torch.bincount(ids)
    start = torch.cumsum(lens, 0) - lens
    by_len = [int(w) for w in torch.argsort(lens, descending=True) if lens[w] > 0]
    i = 0
    while i < len(by_len):
        longest = int(lens[by_len[i]])
        take = by_len[i:i + max(1, limit // longest)]
        w = torch.tensor(take)
        pos = torch.arange(longest)
        mask = pos[None, :] < lens[w][:, None]
        yield order[torch.where(mask, start[w][:, None] + pos, start[w][:, None])], mask
        i += len(take)


def _per_window(fn, ids, *xs):
    """fn on [windows, heads, rows, d] batches of xs [n, H, d]; rows back in place."""
    outs, rows = [], []
    for idx, mask in _window_batches(ids):
        m = mask[:, None, :, None].to(torch.float64)
        o = fn(m, *(x[idx].transpose(1, 2) for x in xs))
        outs.append(o.transpose(1, 2)[mask])
        rows.append(idx[mask])
    back = torch.empty(ids.numel(), dtype=torch.long)
    back[torch.cat(rows)] = torch.arange(ids.numel())
    return torch.cat(outs)[back]


def _attend(relu):
    def fn(m, q, k, v):
        phi = (lambda t: torch.relu(t)) if relu else (lambda t: torch.nn.functional.elu(t) + 1)  # noqa: E731
        fq, fk = phi(q), phi(k) * m
        num = fq @ (fk.transpose(-1, -2) @ v)
        return num / ((fq * fk.sum(-2, keepdim=True)).sum(-1, keepdim=True) + (1e-6 if relu else 0.0))
    return fn


def _xca(tau):
    def fn(m, q, k, v):
        def unit(t):
            return t / torch.sqrt((t * t).sum(-2, keepdim=True)).clamp_min(1e-12)
        a = torch.softmax(tau[None, :, None, None] * (unit(q * m).transpose(-1, -2) @ unit(k * m)), dim=-1)
        return v @ a.transpose(-1, -2)
    return fn


def _cwi(coords, depth, x, w_x, w_y, w_3):
    n, C = x.shape
    c = C // 4
    cell = torch.full((depth + 2, GRID + 64, GRID + 64), n, dtype=torch.long)
    cx, cy, cz = (coords[:, i].long() for i in range(3))
    cell[cz + 1, cy + 32, cx + 32] = torch.arange(n)
    xp = torch.cat([x, torch.zeros(1, C, dtype=x.dtype)])
    ys = []
    for b, w in enumerate((w_x, w_y, w_3)):
        xb, acc = xp[:, b * c:(b + 1) * c], 0.0
        for t in range(w.shape[0]):
            h = t - w.shape[0] // 2
            dx, dy, dz = ((h, 0, 0), (0, h, 0), (t % 3 - 1, t // 3 % 3 - 1, t // 9 - 1))[b]
            if b == 2 and depth == 1 and dz != 0:
                continue
            acc = acc + w[t] * xb[cell[cz + 1 + dz, cy + 32 + dy, cx + 32 + dx]]
        ys.append(acc)
    return torch.cat([*ys, x[:, 3 * c:]], dim=1)


def exact(case, seed):
    s = _inputs(case, seed)
    kind, relu = case["kind"], case["relu"]
    wide = lambda *names: [s[k].detach().cpu().double().requires_grad_() for k in names]  # noqa: E731
    if kind == "cwi_train":
        a = wide("x", "w_x", "w_y", "w_3")
        y = _cwi(s["coords"], case["depth"], *a)
        g = torch.autograd.grad(y, a, s["dy"].cpu().double(), allow_unused=True)
        return dict(zip(("y", "dx", "dw_x", "dw_y", "dw_3"), (y.detach(), *g)))
    ids = s["ids"].long()
    if kind in ("block_infer", "block_train"):
        n, H, d = _shape(case)
        x, w, b, w_o, b_o = a = wide("x", "w_qkv", "b_qkv", "w_o", "b_o")
        q, k, v = ((x @ w.T + b).reshape(n, 3, H, d)).unbind(1)
        o = _per_window(_attend(relu), ids, q, k, v)
        y = o.reshape(n, H * d) @ w_o.T + b_o
        out = {"o": o.detach(), "y": y.detach()}
        if kind == "block_train":
            out.update(zip(("dx", "dw_qkv", "db_qkv", "dw_o", "db_o"),
                           torch.autograd.grad(y, a, s["dy"].cpu().double())))
        return out
    if kind == "xca_train":
        a = wide("q", "k", "v", "tau")
        o = _per_window(_xca(a[3]), ids, *a[:3])
        g = torch.autograd.grad(o, a, s["dout"].cpu().double())
        return dict(zip(("o", "dq", "dk", "dv", "dtau"), (o.detach(), *g)))
    a = wide("q", "k", "v")
    o = _per_window(_attend(relu), ids, *a)
    out = {"o": o.detach()}
    if kind != "forward":
        out.update(perm=None, offsets=None)
    if kind == "train":
        out.update(zip(("dq", "dk", "dv"), torch.autograd.grad(o, a, s["dout"].cpu().double())))
    return out


# -------------------------------------------------------------- work, tolerance
def work(case):
    n, H, d = _shape(case)
    C, kind = H * d, case["kind"]
    t = n * C * (4 if case["dtype"] == "f32" else 2)     # one [n, C] tensor
    if kind == "cwi_train":
        vol = 27 if case["depth"] > 1 else 9
        pairs = n * (C // 4) * (2 * case["taps"] + vol)   # (row, channel, tap), were every neighbour there
        # forward: x, y, coords; backward: x, dy, dx, coords
        return {"bytes": 5 * t + 2 * 12 * n, "flops": 3 * 2 * pairs}
    if kind in ("block_infer", "block_train"):
        weights = 4 * C * C
        b, f = 3 * t + 2 * weights + 4 * n, 8 * n * C * C + 4 * n * C * d        # x; o, y
        if kind == "block_train":                                                # x, o, dy; dx
            b += 4 * t + 2 * weights + 4 * weights + 4 * n
            f += 16 * n * C * C + 10 * n * C * d
        return {"bytes": b, "flops": f}
    if kind == "forward":
        return {"bytes": 4 * t, "flops": 4 * n * C * d}
    b, f = 4 * t + 4 * n, 4 * n * C * d                   # q, k, v; o; the permutation
    if kind in ("train", "xca_train"):
        b, f = b + 7 * t + 4 * n, f + 10 * n * C * d      # q, k, v, dout; dq, dk, dv
    if kind in ("infer", "train"):
        b += 8 * n + 4 * _windows(case)                   # window ids in, permutation and offsets out
    return {"bytes": b, "flops": f}


def tolerance(case):
    # 16 bits: four times the largest relative error against exact() over the listed
    # cases and drawn ones (7.2e-4 and 3.8e-3, both in dq, whose terms cancel);
    # fp32: sums over windows and rows in another order
    return {"f32": {"rel": 1e-5}, "f16": {"rel": 3e-3}, "bf16": {"rel": 1.5e-2}}[case["dtype"]]
