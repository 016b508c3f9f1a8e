"""What a user of this library has it do, as cases that can be timed and compared: the batch-1
product of a decoder (single calls, the launches of a token, the whole pass, with adapters), the
batched product from a few columns to a prefill, dense reconstruction, the one-time re-layout and
one EM iteration of the quantiser.  Shapes are those of the Llama-7B decoder layer that the
benchmark uses and random ones below them; formats are the ones the library lists.

A case is a dict of plain values.  `prepare` makes what a program holds before the call (packed
weights, activations, output buffers) from the seed alone, `run` makes one pass through the
public entry points, `exact` gives the same outputs in 64 bits from plain torch.
"""
from __future__ import annotations

import math

import torch

import paper_2402_15319_amd as vq

DEV = "cuda:0"

# name: (d, k, index bits, codebook dtype, group heights the library takes)
FORMATS = {
    "k16": (2, 16, 4, vq.VQ_F16, (8,)),                      # 2.25 bits per value
    "k256": (2, 256, 8, vq.VQ_F16, (8,)),                    # 8.0
    "k64_i8": (2, 64, 6, vq.VQ_I8, (32, 8, 16)),             # 3.125 at 32 rows: the deployed format
    "k16_i8": (2, 16, 4, vq.VQ_I8, (8, 4)),                  # 2.125
    "k32_i8": (2, 32, 5, vq.VQ_I8, (8,)),                    # 2.75
    "k256_i8": (2, 256, 8, vq.VQ_I8, (128, 64, 256)),        # 4.125 at 128 rows
    "k64_bn": (2, 64, 6, vq.VQ_I8_BN, (32, 8, 16)),          # 3.28
    "k16_bn": (2, 16, 4, vq.VQ_I8_BN, (8,)),                 # 2.38
    "k256_bn": (2, 256, 8, vq.VQ_I8_BN, (128, 64, 256)),     # 4.26
    "d1_k16": (1, 16, 4, vq.VQ_F16, (8,)),                   # 4.125
    "d1_k8": (1, 8, 3, vq.VQ_I8, (32, 8, 16)),               # 3.01
    "d1_k8_bn": (1, 8, 3, vq.VQ_I8_BN, (32, 8, 16)),         # 3.17
    "d1_k4": (1, 4, 2, vq.VQ_I8, (1,)),                      # 2.19
    "d4": (4, 256, 8, vq.VQ_I8, (256, 64, 128)),             # 2.125 at 256 rows
    "d4_f16": (4, 256, 8, vq.VQ_F16, (256, 64, 128)),        # 2.25
    "d4_bn": (4, 256, 8, vq.VQ_I8_BN, (256, 64, 128)),       # 2.25 with int8 tables and block scales
}
INDEX_BITS = {4: 2, 8: 3, 16: 4, 32: 5, 64: 6, 256: 8}

# The launches of one decoder layer in the order its data dependencies allow.
LAYER = (((4096, 4096), (4096, 4096), (4096, 4096)),   # q, k, v
         ((4096, 4096),),                              # o
         ((11008, 4096), (11008, 4096)),               # gate, up
         ((4096, 11008),))                             # down


# ------------------------------------------------------------------------------------ the cases
def listed():
    return [
        # one projection on its own, the smallest call: launch latency
        dict(name="gemv_attn_k16", kind="gemv", fmt="k16", rows=8, out=4096, inp=4096, count=1, f32=False),
        # a token through 8 decoder layers, 4 dependent launches each, replayed from a HIP graph as a
        # serving loop does it; the deployed format (6-bit indices, int8 tables, 32 x 256 groups)
        dict(name="token_k64_graph", kind="layers", fmt="k64_i8", rows=32, layers=8, one_launch=False, graph=True, rank=0, f32=False),
        # 4 layers with rank-16 adapters next to every matrix (2.125 bits per value), eager calls
        dict(name="layers_lora_k16i8", kind="layers", fmt="k16_i8", rows=8, layers=4, one_launch=False, graph=False, rank=16, f32=False),
        # the whole weight pass of a 7B decoder, 224 products in one launch: HBM-bound
        dict(name="pass_k16", kind="layers", fmt="k16", rows=8, layers=32, one_launch=True, graph=False, rank=0, f32=False),
        # 8 layers in the 4D format (one table per 256 rows), fp32 results
        dict(name="pass_d4_f32", kind="layers", fmt="d4", rows=256, layers=8, one_launch=True, graph=False, rank=0, f32=True),
        # 16 sequences decoded together: bandwidth-bound batched product
        dict(name="gemm_b16_k64", kind="gemm", fmt="k64_i8", rows=32, out=4096, inp=11008, batch=16, pad=0, f32=False),
        # a short prompt of odd length in the 4.125 bits per value format, fp32 results
        dict(name="gemm_b203_k256i8", kind="gemm", fmt="k256_i8", rows=128, out=11008, inp=4096, batch=203, pad=0, f32=True),
        # prefill: compute-bound
        dict(name="gemm_b2048_k256", kind="gemm", fmt="k256", rows=8, out=11008, inp=4096, batch=2048, pad=0, f32=False),
        # dense reconstruction of a layer
        dict(name="decode_k256", kind="decode", fmt="k256", rows=8, out=11008, inp=4096),
        # loading a layer: interchange format -> device layout, with an odd number of column blocks
        dict(name="pack_k64bn", kind="pack", fmt="k64_bn", rows=32, out=4096, inp=11008),
        # one EM iteration (E- and M-step) of the quantiser on an attention matrix, small groups
        dict(name="em_k16", kind="em", d=2, k=16, rows=8, out=4096, inp=4096),
        # ... and on an MLP matrix in the 4D setting: 256 centroids shared by 256 rows
        dict(name="em_d4_k256", kind="em", d=4, k=256, rows=256, out=11008, inp=4096),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(("gemv", "gemv", "lora", "gemm", "gemm", "gemm", "decode", "pack", "em", "em"))
    if kind == "em":
        d = rng.choice((1, 2, 2, 4, 4))
        k = rng.choice((8, 16, 64)) if d == 1 else rng.choice((16, 32, 64, 256)) if d == 2 else rng.choice((64, 256))
        rows = rng.choice((8, 32)) if d == 1 else rng.choice((8, 8, 32, 128)) if d == 2 else rng.choice((64, 128, 256))
    else:
        fmt = rng.choice(sorted(FORMATS))
        rows = rng.choice(FORMATS[fmt][4])
    step = max(rows, 8)
    out = max(1, round(_log_uniform(rng, 256, 11008) / step)) * step
    inp = max(1, round(_log_uniform(rng, 256, 11008) / 256)) * 256
    if out * inp > 11008 * 4096:
        inp = 11008 * 4096 // out // 256 * 256
    size = dict(rows=rows, out=out, inp=inp)
    if kind == "em":
        return dict(kind="em", d=d, k=k, **size)
    if kind == "gemm":
        return dict(kind="gemm", fmt=fmt, batch=round(_log_uniform(rng, 1, 2048)), pad=rng.choice((0, 0, 8, 40)),
                    f32=rng.random() < 0.3, **size)
    if kind == "gemv":
        return dict(kind="gemv", fmt=fmt, count=rng.choice((1, 1, 2, 3, 16)), f32=rng.random() < 0.3, **size)
    if kind == "lora":
        return dict(kind="lora", fmt=fmt, count=rng.choice((1, 2, 3)), rank=rng.choice((8, 16, 64)),
                    f32=rng.random() < 0.3, **size)
    return dict(kind=kind, fmt=fmt, **size)


# ------------------------------------------------------------------------------------ inputs
def _generator(seed, salt=0):
    return torch.Generator(DEV).manual_seed(seed * 1000003 + salt)


def _canonical(fmt, rows, out, inp, gen):
    """Random weights in the interchange format: uniform indices; centroids ~ N(0, 0.02) (fp16), or
    uniform int8 entries with a scale per group; block levels on a log grid, uniform codes."""
    d, k, bits, dtype, _ = FORMATS[fmt]
    groups = (out // rows) * (inp // 256)
    idx = torch.randint(0, 256, (groups * (rows * 256 // d * bits // 8),), dtype=torch.uint8, device=DEV, generator=gen)
    if dtype == vq.VQ_F16:
        cb = (torch.randn(groups * k * d, device=DEV, generator=gen) * 0.02).half().view(torch.uint8)
        return idx, cb
    q = torch.randint(-127, 128, (groups * k * d,), dtype=torch.int8, device=DEV, generator=gen).view(torch.uint8)
    scale = (0.06 / 127 * torch.exp2(torch.rand(groups, device=DEV, generator=gen) - 0.5)).half().view(torch.uint8)

    def padded(t):
        return torch.cat([t, t.new_zeros(-t.numel() % 16)])

    if dtype == vq.VQ_I8:
        return idx, torch.cat([padded(q), scale])
    a = 0.1 + 0.2 * torch.rand((groups, 1), device=DEV, generator=gen)
    s0 = -1.5 + torch.rand((groups, 1), device=DEV, generator=gen)
    levels = torch.exp2(a * torch.arange(16, device=DEV) + s0).half().view(torch.uint8).reshape(-1)
    codes = torch.randint(0, 256, (out * (inp // 32) // 2,), dtype=torch.uint8, device=DEV, generator=gen)
    return idx, torch.cat([padded(q), padded(scale), levels, codes])


def _desc(fmt, rows, out, inp):
    d, k, bits, dtype, _ = FORMATS[fmt]
    return vq.make_desc(out, inp, k, bits, rows, 256, d, dtype)


def _packed(fmt, rows, out, inp, gen):
    desc = _desc(fmt, rows, out, inp)
    idx, cb = _canonical(fmt, rows, out, inp, gen)
    n_idx, n_cb = vq.vq_layout_bytes(desc)
    idx_d = torch.zeros(n_idx, dtype=torch.uint8, device=DEV)
    cb_d = torch.zeros(n_cb, dtype=torch.uint8, device=DEV)
    vq.vq_pack_layout(desc, idx, cb, idx_d, cb_d)
    return desc, idx_d, cb_d


def _launches(case):
    """The (out, in) shapes of the products, launch by launch."""
    if case["kind"] != "layers":
        return [[(case["out"], case["inp"])] * case["count"]]
    launches = [list(group) for _ in range(case["layers"]) for group in LAYER]
    return [[s for group in launches for s in group]] if case["one_launch"] else launches


def _dtype(case):
    return torch.float32 if case.get("f32") else torch.float16


def _randn_half(shape, gen, scale=1.0):
    return (torch.randn(shape, device=DEV, generator=gen) * scale).half()


def _vector_inputs(case, shapes, gen):
    """Per product of a launch: x (shared by equal widths, as q, k and v share it), A and B."""
    rank = case.get("rank", 0)
    xs = {n: _randn_half(n, gen) for n in sorted({n for _, n in shapes})}
    adapters = [(_randn_half((rank, n), gen, n ** -0.5), _randn_half((m, rank), gen, 0.02)) if rank else None
                for m, n in shapes]
    return [xs[n] for _, n in shapes], adapters


def _em_inputs(case, seed):
    """Weights ~ N(0, 0.02), column weights 1 / [H^-1]_cc over a factor of 25, a starting codebook of k
    vectors of each group."""
    gen = _generator(seed, 7)
    d, k, rows, out, inp = (case[n] for n in ("d", "k", "rows", "out", "inp"))
    W = torch.randn((out, inp), device=DEV, generator=gen) * 0.02
    h = 0.2 + 4.8 * torch.rand(inp, device=DEV, generator=gen)
    gr, gc = out // rows, inp // 256
    vecs = W.view(gr, rows, gc, 256 // d, d)
    shape = (gr, gc, k)
    r = torch.randint(0, rows, shape, device=DEV, generator=gen)
    v = torch.randint(0, 256 // d, shape, device=DEV, generator=gen)
    gi = torch.arange(gr, device=DEV)[:, None, None]
    ci = torch.arange(gc, device=DEV)[None, :, None]
    cb = vecs[gi, r, ci, v].contiguous()
    return W, h, cb


def prepare(case, seed):
    kind = case["kind"]
    if kind == "em":
        W, h, cb = _em_inputs(case, seed)
        desc = vq.make_desc(case["out"], case["inp"], case["k"], INDEX_BITS[case["k"]], case["rows"], 256, case["d"])
        assign = torch.zeros((case["out"], case["inp"] // case["d"]), dtype=torch.uint8, device=DEV)
        return dict(kind=kind, desc=desc, W=W, h=h, cb=cb, assign=assign, cb_out=torch.zeros_like(cb))
    if kind in ("gemm", "decode", "pack"):
        gen = _generator(seed)
        if kind == "pack":
            desc = _desc(case["fmt"], case["rows"], case["out"], case["inp"])
            idx, cb = _canonical(case["fmt"], case["rows"], case["out"], case["inp"], gen)
            n_idx, n_cb = vq.vq_layout_bytes(desc)
            return dict(kind=kind, desc=desc, idx=idx, cb=cb, idx_d=torch.zeros(n_idx, dtype=torch.uint8, device=DEV),
                        cb_d=torch.zeros(n_cb, dtype=torch.uint8, device=DEV))
        desc, idx_d, cb_d = _packed(case["fmt"], case["rows"], case["out"], case["inp"], gen)
        state = dict(kind=kind, desc=desc, idx_d=idx_d, cb_d=cb_d)
        if kind == "decode":
            state["W"] = torch.empty((case["out"], case["inp"]), dtype=torch.float16, device=DEV)
            return state
        ld = (case["batch"] + 7) // 8 * 8 + case["pad"]
        state["X"] = _randn_half((case["inp"], ld), _generator(seed, 1))
        state["Y"] = torch.zeros((case["out"], ld), dtype=_dtype(case), device=DEV)
        state.update(B=case["batch"], ld=ld, y_dtype=vq.VQ_F32 if case["f32"] else vq.VQ_F16)
        return state

    launches, outputs = [], []
    item = 0
    for li, shapes in enumerate(_launches(case)):
        xs, adapters = _vector_inputs(case, shapes, _generator(seed, 500000 + li))
        # the results of a launch lie behind one another (row counts are multiples of 8: 16-byte pieces)
        y = torch.zeros(sum(m for m, _ in shapes), dtype=_dtype(case), device=DEV)
        outputs.append(y)
        ys, at, weights = [], 0, []
        for m, n in shapes:
            ys.append(y[at:at + m])
            at += m
            weights.append(_packed(case["fmt"], case["rows"], m, n, _generator(seed, 1000 + item)))
            item += 1
        launches.append((vq.GemvMultiArgs([w[0] for w in weights], [w[1] for w in weights], [w[2] for w in weights], xs, ys),
                         adapters, weights, xs, ys))
    state = dict(kind=kind, launches=launches, outputs=outputs, rank=case.get("rank", 0), count=case.get("count", 0),
                 y_dtype=vq.VQ_F32 if case["f32"] else vq.VQ_F16)
    if state["rank"]:
        most = max(len(shapes) for shapes in _launches(case))
        state["workspace"] = torch.zeros(vq.vq_lora_workspace_bytes(most), dtype=torch.uint8, device=DEV)
    if case.get("graph"):
        torch.cuda.synchronize()
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            _run_launches(state)
        torch.cuda.synchronize()
    return state


# ------------------------------------------------------------------------------------ one pass
def _run_launches(state):
    for args, adapters, weights, xs, ys in state["launches"]:
        if state["rank"]:
            vq.vq_gemv_lora_multi(args, [a for a, _ in adapters], [b for _, b in adapters], [state["rank"]] * len(adapters),
                                  state["workspace"], state["y_dtype"])
        elif state["count"] == 1:
            desc, idx_d, cb_d = weights[0]
            vq.vq_gemv(desc, idx_d, cb_d, xs[0], ys[0], state["y_dtype"])
        else:
            vq.vq_gemv_multi(args, y_dtype=state["y_dtype"])


def run(state):
    kind = state["kind"]
    if kind == "em":
        vq.vq_em_assign(state["desc"], state["W"], state["h"], state["cb"], state["assign"])
        vq.vq_em_update(state["desc"], state["W"], state["h"], state["assign"], state["cb_out"])
        return [state["assign"], state["cb_out"]]
    if kind == "pack":
        vq.vq_pack_layout(state["desc"], state["idx"], state["cb"], state["idx_d"], state["cb_d"])
        return [state["idx_d"], state["cb_d"]]
    if kind == "decode":
        vq.vq_decode_dense(state["desc"], state["idx_d"], state["cb_d"], state["W"])
        return state["W"]
    if kind == "gemm":
        vq.vq_gemm_batched(state["desc"], state["idx_d"], state["cb_d"], state["X"], state["B"], state["ld"],
                           state["Y"], state["ld"], state["y_dtype"])
        return state["Y"][:, :state["B"]]
    if "graph" in state:
        state["graph"].replay()
    else:
        _run_launches(state)
    return state["outputs"]


# ------------------------------------------------------------------------------------ what a pass costs
def _weight_bytes(fmt, rows, out, inp):
    """Indices and tables of one matrix, without padding."""
    d, k, bits, dtype, _ = FORMATS[fmt]
    groups = (out // rows) * (inp // 256)
    table = k * d * 2 if dtype == vq.VQ_F16 else k * d + 2
    extra = groups * 32 + out * (inp // 32) // 2 if dtype == vq.VQ_I8_BN else 0
    return out * inp // d * bits // 8 + groups * table + extra


def work(case):
    kind = case["kind"]
    y_bytes = 4 if case.get("f32") else 2
    if kind == "em":
        out, inp, d, k = (case[n] for n in ("out", "inp", "d", "k"))
        groups = (out // case["rows"]) * (inp // 256)
        # the weights once for each step (the steps are two calls), both codebooks, the assignment out and in
        nbytes = 2 * (4 * out * inp + 4 * inp) + 2 * 4 * groups * k * d + 2 * out * inp // d
        # subtract, square, weigh, add per coordinate and centroid; two sums per coordinate
        return {"bytes": nbytes, "flops": out * inp * (4 * k + 3)}
    if kind in ("pack", "decode", "gemm"):
        w = _weight_bytes(case["fmt"], case["rows"], case["out"], case["inp"])
        if kind == "pack":
            return {"bytes": 2 * w, "flops": 0}
        if kind == "decode":
            return {"bytes": w + 2 * case["out"] * case["inp"], "flops": 0}
        b = case["batch"]
        return {"bytes": w + 2 * case["inp"] * b + y_bytes * case["out"] * b, "flops": 2 * case["out"] * case["inp"] * b}
    nbytes = flops = 0
    for shapes in _launches(case):
        nbytes += sum(2 * n for n in {n for _, n in shapes})
        for m, n in shapes:
            rank = case.get("rank", 0)
            nbytes += _weight_bytes(case["fmt"], case["rows"], m, n) + y_bytes * m + 2 * rank * (m + n)
            flops += 2 * m * n + 2 * rank * (m + n)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    kind = case["kind"]
    if kind in ("pack", "decode"):
        return "exact"                     # copies of bit patterns
    if kind == "em":
        return {"rel": 1e-6}               # assignments exact; 32-bit sums of a cluster's members
    if case.get("f32"):
        return {"rel": 2e-6}               # 32-bit sums of fp16 products
    return {"rel": 8e-4, "max": 4e-3}      # one rounding to fp16 on top


# ------------------------------------------------------------------------------------ 64 bits
def _indices(idx, bits, groups):
    b = idx.view(groups, -1)
    if bits == 8:
        return b.long()
    words = b.view(groups, -1, bits).long()              # `bits` bytes hold 8 indices
    word = sum(words[..., i] << (8 * i) for i in range(bits))
    return torch.stack([(word >> (bits * j)) & ((1 << bits) - 1) for j in range(8)], -1).view(groups, -1)


def _dense(fmt, rows, out, inp, gen):
    """W[out, in] in float64, from the interchange format."""
    d, k, bits, dtype, _ = FORMATS[fmt]
    idx, cb = _canonical(fmt, rows, out, inp, gen)
    gr, gc = out // rows, inp // 256
    groups = gr * gc
    nq = groups * k * d
    if dtype == vq.VQ_F16:
        table = cb.view(torch.float16).view(groups, k, d)
    else:
        at = (nq + 15) // 16 * 16
        q = cb[:nq].view(torch.int8).float().view(groups, k, d)
        scale = cb[at:at + 2 * groups].view(torch.float16).float()
        table = (q * scale[:, None, None]).half()        # exact product, one rounding
    sel = _indices(idx, bits, groups)
    W = torch.gather(table, 1, sel[..., None].expand(-1, -1, d))
    W = W.view(gr, gc, rows, 256).permute(0, 2, 1, 3).reshape(out, inp)
    if dtype == vq.VQ_I8_BN:
        at = (at + 2 * groups + 15) // 16 * 16
        levels = cb[at:at + 32 * groups].view(torch.float16).view(gr, 1, gc, 1, 16)
        packed = cb[at + 32 * groups:].view(out, inp // 64)
        codes = torch.stack([packed & 15, packed >> 4], -1).view(gr, rows, gc, 8).long()
        s = torch.gather(levels.expand(gr, rows, gc, 8, 16), 4, codes[..., None])
        W = (W.view(gr, rows, gc, 8, 32).float() * s.float()).half().reshape(out, inp)
    return W.double()


def _em_exact(case, seed):
    """The centroids in 64 bits for the assignment of the E-step, whose arithmetic is defined in
    binary32 (subtract, square, weigh, add, each rounded; the lowest index wins a tie)."""
    W, h, cb = _em_inputs(case, seed)
    d, k, rows, out, inp = (case[n] for n in ("d", "k", "rows", "out", "inp"))
    gr, gc = out // rows, inp // 256
    x = [W.view(gr, rows, gc, 256 // d, d)[..., t].contiguous() for t in range(d)]
    hv = [h.view(1, 1, gc, 256 // d, d)[..., t].contiguous() for t in range(d)]
    best = torch.full_like(x[0], math.inf)
    arg = torch.zeros(best.shape, dtype=torch.long, device=DEV)
    for m in range(k):
        dist = None
        for t in range(d):
            e = x[t] - cb[:, :, m, t].view(gr, 1, gc, 1)
            term = hv[t] * (e * e)
            dist = term if dist is None else dist + term
        closer = dist < best
        best = torch.where(closer, dist, best)
        arg.masked_fill_(closer, m)
    group = torch.arange(gr * gc, device=DEV).view(gr, 1, gc, 1)
    slot = (group * k + arg).reshape(-1)
    new = torch.zeros((gr * gc * k, d), dtype=torch.float64, device=DEV)
    for t in range(d):
        weight = hv[t].double().expand(x[t].shape)
        num = torch.zeros(gr * gc * k, dtype=torch.float64, device=DEV).index_add_(0, slot, (weight * x[t].double()).reshape(-1))
        den = torch.zeros_like(num).index_add_(0, slot, weight.reshape(-1))
        new[:, t] = torch.where(den != 0, num / den, torch.zeros_like(num))
    return [None, new.view(gr, gc, k, d)]


def exact(case, seed):
    kind = case["kind"]
    if kind == "pack":
        return None                        # a permutation of bytes
    if kind == "em":
        return _em_exact(case, seed)
    if kind in ("gemm", "decode"):
        W = _dense(case["fmt"], case["rows"], case["out"], case["inp"], _generator(seed))
        if kind == "decode":
            return W
        ld = (case["batch"] + 7) // 8 * 8 + case["pad"]
        return W @ _randn_half((case["inp"], ld), _generator(seed, 1))[:, :case["batch"]].double()
    outputs, item = [], 0
    for li, shapes in enumerate(_launches(case)):
        xs, adapters = _vector_inputs(case, shapes, _generator(seed, 500000 + li))
        parts = []
        for (m, n), x, ab in zip(shapes, xs, adapters):
            y = _dense(case["fmt"], case["rows"], m, n, _generator(seed, 1000 + item)) @ x.double()
            item += 1
            parts.append(y + ab[1].double() @ (ab[0].double() @ x.double()) if ab else y)
        outputs.append(torch.cat(parts))
    return outputs
