"""The calls whose speed matters to a program that uses this library.

Every case is one pass through the public binding on device tensors: a forward call, a training
step (the forward call that keeps its intermediates, then the gradients from them), or the dense
baseline.  Shapes are those of a video diffusion transformer's self-attention: latent grids of
30 x 52 (480p) and 45 x 80 (720p), chunks of three frames, 21 latent frames, heads of 128 or 64.

`exact` states the same results in 64 bits with plain torch, one query tile at a time.
"""
import math

import torch

from paper_2602_12271_amd import binding

_DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(op, grid, heads, blocks, *, f_kv=None, tile=0, iters=1, chunk=0, offset=0, dtype="bf16", dim=128,
          batch=1, assign="fh_w", **named):
    f, h, w = grid
    return dict(named, op=op, batch=batch, heads=heads, dim=dim, f_q=f, f_kv=f if f_kv is None else f_kv, h=h, w=w,
                b1=blocks[0], b2=blocks[1], tile=tile, iters=iters, chunk=chunk, offset=offset, dtype=dtype,
                assign=assign)


def listed():
    return [
        # the smallest call: one head of one small frame in fp32, two launches; latency is all there is
        _case("forward", (1, 24, 24), 1, (24, 24), dtype="f32", dim=64, name="tiny-f32"),
        # a small model's layer on an odd grid, heads of 64, batch of two (conditional / unconditional)
        _case("forward", (2, 17, 23), 4, (34, 23), iters=2, dim=64, batch=2, name="small-odd-d64"),
        # one autoregressive 480p chunk attending to itself: the ordinary call
        _case("forward", (3, 30, 52), 12, (90, 52), iters=2, name="chunk-480p"),
        # the same chunk with (frame, width) x height blocks: block rows beyond a multiple of 16 (156)
        _case("forward", (3, 30, 52), 12, (156, 30), iters=2, assign="fw_h", name="chunk-480p-fw_h"),
        # the same chunk in fp32 storage and arithmetic, as quality studies run it
        _case("forward", (3, 30, 52), 12, (90, 52), iters=2, dtype="f32", name="chunk-480p-f32"),
        # decoding step: the last chunk against the cached keys of the whole clip, half-width tiles
        _case("forward", (3, 30, 52), 12, (90, 26), f_kv=21, tile=1, iters=2, chunk=3, offset=18, name="cache-480p"),
        # decoding step at 720p with one-frame tiles (the denser setting)
        _case("forward", (3, 45, 80), 12, (45, 80), f_kv=21, tile=1, iters=1, chunk=3, offset=18,
              name="cache-720p-frames"),
        # the largest call: decoding step of a 40-head model at 720p, three refinements
        _case("forward", (3, 45, 80), 40, (135, 40), f_kv=21, tile=1, iters=3, chunk=3, offset=18,
              name="cache-720p-40h"),
        # prefill: a whole bidirectional 480p clip at once
        _case("forward", (21, 30, 52), 12, (90, 52), tile=1, iters=1, name="clip-480p"),
        # training step (forward + gradients) on one chunk
        _case("train", (3, 30, 52), 12, (90, 52), iters=2, name="train-chunk-480p"),
        # training step on a whole clip under the block-causal mask
        _case("train", (21, 30, 52), 12, (90, 52), tile=1, iters=1, chunk=3, name="train-clip-480p"),
        # a layer kept dense, on one chunk
        _case("dense", (3, 30, 52), 12, (0, 0), iters=0, name="dense-chunk-480p"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def _candidate(rng):
    kind = rng.choice(["chunk", "chunk", "cache", "cache", "clip", "train", "dense", "f32"])
    dim = rng.choice([64, 128, 128, 128])
    h, w = _log_int(rng, 12, 45), _log_int(rng, 16, 80)
    heads, batch = _log_int(rng, 1, 40), rng.choice([1, 1, 2])
    width = w // 2 if w % 2 == 0 and rng.random() < 0.5 else w
    if kind in ("chunk", "f32"):
        f = rng.randint(1, max(1, min(4, 180 // h)))
        iters, dtype = rng.randint(1, 3), "f32" if kind == "f32" else "bf16"
        if kind == "chunk" and rng.random() < 0.25:
            f = min(f, 180 // w)
            return _case("forward", (f, h, w), heads, (f * w, h), iters=iters, dim=dim, batch=batch, assign="fw_h")
        if kind == "f32":
            f = min(f, max(1, 96 // h))
        return _case("forward", (f, h, w), heads, (f * h, width), tile=int(width != w), iters=iters, dim=dim,
                     batch=batch, dtype=dtype)
    chunks = rng.randint(2, 7)
    f_kv = 3 * chunks
    rows = 3 * h if rng.random() < 0.5 else h
    if kind == "cache":
        return _case("forward", (3, h, w), heads, (rows, width), f_kv=f_kv, tile=1, iters=rng.randint(1, 3), chunk=3,
                     offset=f_kv - 3, dim=dim, batch=batch)
    if kind == "clip":
        return _case("forward", (f_kv, h, w), heads, (rows, width), tile=1, iters=rng.randint(1, 2), dim=dim,
                     batch=batch)
    if kind == "train":
        rows = rows if rows <= 96 else h
        if rng.random() < 0.5:
            f = max(1, min(3, 96 // h))
            return _case("train", (f, h, w), heads, (f * h, w), iters=rng.randint(1, 2), dim=dim, batch=batch)
        return _case("train", (f_kv, h, w), heads, (rows, width), tile=1, iters=1, chunk=3, dim=dim, batch=batch)
    return _case("dense", (3, h, w), heads, (0, 0), f_kv=3 * min(chunks, 4), iters=0, chunk=3,
                 offset=3 * min(chunks, 4) - 3, dim=dim, batch=batch)


def _pairs(c):
    """(query tile, visible key tile) pairs of one head."""
    _, _, rows_q, _, cols = _sides(c)
    return sum(len(_visible(c, a)) for a in range(rows_q // c["b1"])) * (cols // c["b2"]) ** 2


def _cost(c):
    """A rough time in seconds, to keep drawn cases below the largest listed one."""
    w = work(c)
    rate = 2e13 if c["dtype"] == "f32" else 3e14
    if c["op"] == "dense":
        return w["flops"] / (2 * rate)
    passes = (2 * c["iters"] + 1) * (4 if c["op"] == "train" else 1)
    moved = c["batch"] * c["heads"] * _pairs(c) * c["b1"] * c["b2"] * c["dim"] * 2 * passes
    return w["flops"] / rate + moved / 4e12


def draw(rng):
    most = 0.9 * max(_cost(c) for c in listed())
    while True:
        c = _candidate(rng)
        if _cost(c) <= most:
            return c


def _rope(c, frames, device):
    """cos, sin [tokens, dim / 2]: rotary pairs shared out over (frame, height, width)."""
    pairs = c["dim"] // 2
    ph = pw = pairs // 3

    def angles(pos, n):
        inv = 10000.0 ** (-torch.arange(n, dtype=torch.float64, device=device) / n)
        return pos.to(torch.float64)[:, None] * inv[None]

    grid = torch.cartesian_prod(frames.to(device), torch.arange(c["h"], device=device),
                                torch.arange(c["w"], device=device))
    ang = torch.cat([angles(grid[:, 0], pairs - ph - pw), angles(grid[:, 1], ph), angles(grid[:, 2], pw)], 1)
    return ang.cos().float(), ang.sin().float()


def _inputs(c, seed):
    """Q, K (unit normal content under a 3-D rotary encoding), V and, for training, dO."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)
    dt = _DTYPES[c["dtype"]]

    def normal(frames, rope=None):
        x = torch.empty(c["batch"], c["heads"], frames * c["h"] * c["w"], c["dim"], dtype=dt, device=dev)
        for one in x:                        # one batch entry at a time: the fp32 draw stays small
            v = torch.randn(one.shape, generator=gen, device=dev)
            if rope is not None:
                cos, sin = rope
                even, odd = v[..., 0::2], v[..., 1::2]
                v = torch.stack([even * cos - odd * sin, even * sin + odd * cos], -1).flatten(-2)
            one.copy_(v)
        return x

    q = normal(c["f_q"], _rope(c, c["offset"] + torch.arange(c["f_q"]), dev))
    k = normal(c["f_kv"], _rope(c, torch.arange(c["f_kv"]), dev))
    v = normal(c["f_kv"])
    return (q, k, v, normal(c["f_q"])) if c["op"] == "train" else (q, k, v)


def _arguments(c):
    geometry = dict(f_q=c["f_q"], f_kv=c["f_kv"], h=c["h"], w=c["w"], causal_chunk=c["chunk"],
                    q_frame_offset=c["offset"], scale=_scale(c))
    if c["op"] == "dense":
        return geometry
    return dict(geometry, b1=c["b1"], b2=c["b2"], tile=c["tile"], iters=c["iters"], assign=c["assign"])


def _scale(c):
    return 1.0 / math.sqrt(c["dim"])


def prepare(case, seed):
    c = case
    tensors = _inputs(c, seed)
    state = {"case": c, "tensors": tensors, "args": _arguments(c)}
    if c["op"] != "train":
        state["args"]["out"] = torch.empty_like(tensors[0])
    if c["op"] == "forward":
        # a serving program keeps one workspace for its layers
        problem = binding.make_problem(batch=c["batch"], heads=c["heads"], head_dim=c["dim"], f_q=c["f_q"],
                                       f_kv=c["f_kv"], h=c["h"], w=c["w"], q_frame_offset=c["offset"],
                                       dtype=binding.MRT_F32 if c["dtype"] == "f32" else binding.MRT_BF16,
                                       scale=_scale(c), assign=c["assign"])
        nbytes = binding.monarch_attn_workspace_bytes(problem, c["b1"], c["b2"], c["tile"], c["iters"])
        state["args"]["workspace"] = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    return state


def run(state):
    args = state["args"]
    if state["case"]["op"] == "forward":
        return binding.monarch_attn_fwd(*state["tensors"], **args)
    if state["case"]["op"] == "dense":
        return binding.dense_attn_fwd(*state["tensors"], **args)
    q, k, v, do = state["tensors"]
    o, saved = binding.monarch_attn_fwd_save(q, k, v, **args)
    dq, dk, dv = binding.monarch_attn_bwd_saved(q, k, v, do, saved, **args)
    return {"O": o, "dQ": dq, "dK": dk, "dV": dv}


def work(case):
    c = case
    size = {"bf16": 2, "f32": 4}[c["dtype"]]
    bh, hw = c["batch"] * c["heads"], c["h"] * c["w"]
    nq, nkv = c["f_q"] * hw, c["f_kv"] * hw
    moved = bh * c["dim"] * size * (2 * nq + 2 * nkv)                     # Q, O, K, V
    if c["op"] == "dense":
        seen = sum(len(_visible_frames(c, f)) for f in range(c["f_q"])) * hw * hw
        return {"bytes": moved, "flops": 4 * bh * seen * c["dim"]}
    # per pair of visible tiles: logits and weighted keys of R and logits and weighted rows of L in
    # every iteration, plus the weighted values of R once
    nt, t = c["b1"] * c["b2"], c["iters"]
    flops = 2 * bh * _pairs(c) * nt * c["dim"] * ((2 * t + 1) * c["b2"] + 2 * t * c["b1"])
    if c["op"] == "train":
        # the gradients form about five products where the forward pass formed two
        return {"bytes": moved + bh * c["dim"] * (nq * size + 4 * nq + 8 * nkv), "flops": int(3.5 * flops)}
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    # Four times the largest distance from `exact` measured over the listed cases and 60 drawn ones
    # (forward 3.7e-3, dense 2.4e-3, training step 3.9e-3, fp32 5.5e-7).  bf16 operands are rounded
    # to 2^-9 at every stage, so this is what another correct order of the same roundings shows.
    if case["dtype"] == "f32":
        return {"rel": 2.5e-6}
    return {"rel": {"forward": 1.5e-2, "dense": 1e-2, "train": 1.6e-2}[case["op"]]}


# ---- the same results in 64 bits ---------------------------------------------------------------
def _sides(c):
    """Axis order of the tokens, block-grid rows per frame, rows of the query and key side, columns."""
    if c["assign"] == "fw_h":
        return (0, 2, 1), c["w"], c["f_q"] * c["w"], c["f_kv"] * c["w"], c["h"]
    return (0, 1, 2), c["h"], c["f_q"] * c["h"], c["f_kv"] * c["h"], c["w"]


def _tiles(c, x, frames):
    """[tokens, dim] -> [tile row, tile column, b1, b2, dim]."""
    order, _, _, _, cols = _sides(c)
    x = x.view(frames, c["h"], c["w"], c["dim"]).permute(*order, 3)
    x = x.reshape(-1, c["b1"], cols // c["b2"], c["b2"], c["dim"])
    return x.permute(0, 2, 1, 3, 4).contiguous()


def _tokens(c, x, frames):
    """The inverse of _tiles."""
    order, _, _, _, _ = _sides(c)
    sizes = [(frames, c["h"], c["w"])[i] for i in order]
    x = x.permute(0, 2, 1, 3, 4).reshape(*sizes, c["dim"])
    return x.permute(*order, 3).reshape(-1, c["dim"])       # both orders are their own inverses


def _visible_frames(c, f):
    if c["chunk"] == 0:
        return range(c["f_kv"])
    return range(min(c["f_kv"], ((f + c["offset"]) // c["chunk"] + 1) * c["chunk"]))


def _visible(c, a):
    """Key tile rows that query tile row a sees (a tile never straddles a chunk)."""
    _, per_frame, _, rows_k, _ = _sides(c)
    n = rows_k // c["b1"]
    if c["chunk"] == 0 or c["tile"] == 0:
        return range(n)
    return range(min(n, len(_visible_frames(c, a * c["b1"] // per_frame)) * per_frame // c["b1"]))


def _attend(c, q, k, v):
    """One query tile q [b1, b2, d] over key tiles k, v [n, b1, b2, d]."""
    n, b1, b2, d = k.shape
    k, v = k.reshape(n * b1, b2, d), v.reshape(n * b1, b2, d)
    columns = q.transpose(0, 1).contiguous()                                # [j, l, d]
    abar = q.repeat(n, 1, 1)                                                # [nk, j, d]
    for t in range(1, c["iters"] + 1):
        logr = torch.log_softmax(_scale(c) * torch.matmul(abar, k.transpose(1, 2).contiguous()), -1)
        r = logr.exp()                                                      # [nk, j, i]
        alpha = torch.matmul(r, k).transpose(0, 1).contiguous()             # [j, nk, d]
        entropy = (r * logr).sum(-1).transpose(0, 1)                        # [j, nk]
        z = _scale(c) * torch.matmul(columns, alpha.transpose(1, 2).contiguous()) - entropy[:, None, :]
        logl = torch.log_softmax(z, -1)                                     # [j, l, nk]
        if t < c["iters"]:
            weights = torch.softmax(logl, 1).transpose(1, 2).contiguous()   # [j, nk, l]
            abar = torch.matmul(weights, columns).transpose(0, 1).contiguous()
    y = torch.matmul(r, v).transpose(0, 1).contiguous()
    return torch.matmul(logl.exp(), y).transpose(0, 1)                      # [l, j, d]


def _exact_head(c, q, k, v, do):
    q, k, v = q.double(), k.double(), v.double()
    qt, kt, vt = _tiles(c, q, c["f_q"]), _tiles(c, k, c["f_kv"]), _tiles(c, v, c["f_kv"])
    if do is None:
        out = torch.empty_like(qt)
        for a in range(qt.shape[0]):
            n = len(_visible(c, a))
            for b in range(qt.shape[1]):
                out[a, b] = _attend(c, qt[a, b], kt[:n].flatten(0, 1), vt[:n].flatten(0, 1))
        return (_tokens(c, out, c["f_q"]),)
    out, grads = torch.empty_like(qt), [torch.zeros_like(x) for x in (qt, kt, vt)]
    dt = _tiles(c, do.double(), c["f_q"])
    for a in range(qt.shape[0]):
        n = len(_visible(c, a))
        for b in range(qt.shape[1]):
            leaf = [x.clone().requires_grad_(True) for x in (qt[a, b], kt[:n], vt[:n])]
            o = _attend(c, leaf[0], leaf[1].flatten(0, 1), leaf[2].flatten(0, 1))
            dq, dk, dv = torch.autograd.grad(o, leaf, dt[a, b])
            out[a, b] = o.detach()
            grads[0][a, b] = dq
            grads[1][:n] += dk
            grads[2][:n] += dv
    frames = (c["f_q"], c["f_q"], c["f_kv"], c["f_kv"])
    return tuple(_tokens(c, x, f) for x, f in zip([out] + grads, frames))


def _exact_dense(c, q, k, v):
    q, k, v = q.double(), k.double(), v.double()
    hw, out = c["h"] * c["w"], torch.empty_like(q)
    for f in range(c["f_q"]):
        n = len(_visible_frames(c, f)) * hw
        p = torch.softmax(_scale(c) * torch.matmul(q[f * hw:(f + 1) * hw], k[:n].t().contiguous()), -1)
        out[f * hw:(f + 1) * hw] = torch.matmul(p, v[:n])
    return (out,)


def exact(case, seed):
    c = case
    q, k, v, *do = _inputs(c, seed)
    heads = []
    for b in range(c["batch"]):
        for h in range(c["heads"]):
            if c["op"] == "dense":
                heads.append(_exact_dense(c, q[b, h], k[b, h], v[b, h]))
            else:
                heads.append(_exact_head(c, q[b, h], k[b, h], v[b, h], do[0][b, h] if do else None))
    outs = [torch.stack(x).unflatten(0, (c["batch"], c["heads"])) for x in zip(*heads)]
    return dict(zip(("O", "dQ", "dK", "dV"), outs)) if c["op"] == "train" else outs[0]
