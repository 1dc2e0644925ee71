"""The work that a program built on this library has it do, as cases that can be timed and checked.

Five kinds of case:
  fwd     one layer's forward, called on its own: a short prompt, a small layer, a batch of a few tokens
  decode  the linear layers of a few decoder blocks for the next token of M sequences, the launches kept in a HIP graph as
          a decode loop keeps them (q/k/v and gate/up through the group call)
  tune    one layer's fine-tuning step: forward, then input gradient and weak-block gradient
  out     the attention output projection, whose weak columns stay at their own channels: forward, input gradient, weak
          gradient from the gathered weak activations
  search  the quantizer's grid search over one layer, run once per layer when a model is converted
Layers are stored from seeded draws: weights N(0, 0.02), min-max quantized here in groups of 128, activations N(0, 1) with the weak
channels 20 times as large, output gradients N(0, 0.01).
"""
import math

import torch

from paper_2410_08661_amd import binding as B

G = 128
# (hidden, feed-forward, key/value width) of the decoder blocks
MODELS = {"7b": (4096, 11008, 4096), "13b": (5120, 13824, 5120), "70b": (8192, 28672, 1024)}
N_GRID, STEP = 80, 0.01


def listed():
    return [
        # the smallest call: one token through a layer of the small test configuration
        dict(name="fwd-512", kind="fwd", oc=512, ic=512, k=8, bits=4, dense=False, m=1),
        # the next token of one sequence, 7B blocks: the headline
        dict(name="decode-7b", kind="decode", model="7b", k=128, bits=4, dense=False, m=1, blocks=8),
        # the same for eight sequences served together
        dict(name="decode-7b-8", kind="decode", model="7b", k=128, bits=4, dense=False, m=8, blocks=8),
        # the next token with 3-bit weights
        dict(name="decode-13b-w3", kind="decode", model="13b", k=128, bits=3, dense=False, m=1, blocks=4),
        # forty sequences served together, or as many draft tokens verified at once
        dict(name="decode-7b-40", kind="decode", model="7b", k=128, bits=4, dense=False, m=40, blocks=4),
        # a prompt of a few hundred tokens through an up projection
        dict(name="prompt-13b", kind="fwd", oc=13824, ic=5120, k=128, bits=4, dense=False, m=333),
        # fine-tuning at batch 1, input length 512
        dict(name="tune-7b-512", kind="tune", oc=4096, ic=4096, k=128, bits=4, dense=False, m=512),
        # the output projection of a short sequence
        dict(name="out-7b", kind="out", oc=4096, ic=4096, k=128, bits=4, dense=False, m=777),
        # fine-tuning, 4096 tokens, a down projection
        dict(name="tune-7b", kind="tune", oc=4096, ic=11008, k=128, bits=4, dense=False, m=4096),
        # fine-tuning a 3-bit model at an odd length
        dict(name="tune-13b-w3", kind="tune", oc=5120, ic=5120, k=128, bits=3, dense=True, m=1000),
        # the largest: the 70B down projection
        dict(name="tune-70b", kind="tune", oc=8192, ic=28672, k=256, bits=4, dense=False, m=2048),
        # converting a model
        dict(name="search-7b", kind="search", oc=4096, ic=4096, k=128, bits=4, dense=False, m=0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng):
    """A layer of the three models, or one of any size whose sides are multiples of 8."""
    if rng.random() < 0.6:
        h, f, kv = MODELS[rng.choice(("7b", "13b", "70b"))]
        return rng.choice(((h, h), (kv, h), (f, h), (h, f)))
    step = rng.choice((8, 64, 128, 128))
    return tuple(max(512, _log(rng, 512, 16384) // step * step) for _ in range(2))


def _bits(rng):
    return rng.choice(((4, False), (4, False), (4, False), (3, False), (3, True)))


def draw(rng):
    kind = rng.choice(("fwd", "fwd", "fwd", "decode", "decode", "tune", "tune", "out", "search"))
    bits, dense = _bits(rng)
    k = rng.choice((8, 16, 64, 128, 128, 128, 256))
    if kind == "decode":
        model = rng.choice(("7b", "7b", "13b", "70b"))
        m = rng.choice((1, _log(rng, 1, 64 if bits == 4 else 16), _log(rng, 1, 64 if bits == 4 else 16)))
        blocks = rng.randint(3, 8) * MODELS["7b"][1] // MODELS[model][1] if m <= 16 else 3
        return dict(kind=kind, model=model, k=k, bits=bits, dense=dense, m=m, blocks=max(1, blocks))
    oc, ic = _shape(rng)
    if kind == "fwd":
        m = min(_log(rng, 1, 2048), int(1e12 / (2 * oc * ic)))
    elif kind == "search":
        return dict(kind=kind, oc=oc, ic=max(1024, ic // G * G), k=rng.choice((64, 128, 256)), bits=bits, dense=dense, m=0)
    else:
        if kind == "out":
            oc, bits, dense = ic, 4, False
        m = min(_log(rng, 64, 4096), int(1e12 / (4 * oc * ic)))
    return dict(kind=kind, oc=oc, ic=ic, k=k, bits=bits, dense=dense, m=max(1, m))


# ---- the layers of a case ------------------------------------------------------------------------------------------


def _layers(case):
    """(oc, ic) of the case's layers, and for decode the groups of them that share an input."""
    if case["kind"] != "decode":
        return [(case["oc"], case["ic"])], [[0]]
    h, f, kv = MODELS[case["model"]]
    block = [(h, h), (kv, h), (kv, h), (h, h), (f, h), (f, h), (h, f)]
    groups = [[0, 1, 2], [3], [4, 5], [6]]
    n = case["blocks"]
    return block * n, [[7 * b + i for i in g] for b in range(n) for g in groups]


def _gen(seed, what):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 1009 + what)


def _normal(gen, rows, cols, std):
    return (torch.randn((rows, cols), generator=gen, device="cuda", dtype=torch.float32) * std).half()


def _quantize(w, bits):
    """Min-max round-to-nearest codes, scales and zero-points of w (fp16 [OC][Kq]) in groups of 128, in fp32."""
    oc, kq = w.shape
    ng, qmax = -(-kq // G), float(2 ** bits - 1)
    p = torch.zeros((oc, ng * G), dtype=torch.float32, device=w.device)
    p[:, :kq] = w.float()
    p = p.view(oc, ng, G)
    lo, hi = p.amin(2).clamp(max=0.0), p.amax(2).clamp(min=0.0)
    s = ((hi - lo) / qmax).half()
    s = torch.where(s > 0, s, torch.ones_like(s))
    z = (-lo / s.float()).round().clamp(0, qmax)
    q = ((p / s.float()[..., None]).round() + z[..., None]).clamp(0, qmax).to(torch.uint8)
    return q.view(oc, ng * G)[:, :kq].contiguous(), s, z.half()


def _components(case, seed, i, oc, ic):
    k, bits = case["k"], case["bits"]
    w = _normal(_gen(seed, 100 + i), oc, ic, 0.02)
    return (*_quantize(w[:, : ic - k], bits), w[:, ic - k:].contiguous())


def _desc(case, oc, ic):
    return B.make_desc(oc, ic, case["k"], case["bits"], G, B.QEFT_LAYOUT_DENSE3 if case["dense"] else B.QEFT_LAYOUT_CANONICAL)


def _store(case, seed, i, oc, ic):
    d = _desc(case, oc, ic)
    return d, B.qeft_pack_codes(d, *_components(case, seed, i, oc, ic))


def _x(case, seed, i, ic):
    x = _normal(_gen(seed, 10000 + i), case["m"], ic, 1.0)
    x[:, ic - case["k"]:] *= 20
    return x


def _dy(case, seed, oc):
    return _normal(_gen(seed, 20000), case["m"], oc, 0.01)


def _perm(case, seed, ic):
    """Stored column -> original channel: the other channels in ascending order, then the weak ones."""
    order = torch.randperm(ic, generator=_gen(seed, 30000), device="cuda")
    weak = order[: case["k"]].sort().values
    keep = torch.ones(ic, dtype=torch.bool, device="cuda")
    keep[weak] = False
    return torch.cat([torch.arange(ic, device="cuda")[keep], weak]).int()


def _rows(m, cols, dtype=torch.float16):
    return torch.empty((m, -(-cols // 8) * 8), dtype=dtype, device="cuda")[:, :cols]


def _ws(d, op, m):
    n = B.qeft_workspace_bytes(d, op, m)
    return torch.empty(n, dtype=torch.uint8, device="cuda") if n else False


# ---- prepare, run ----------------------------------------------------------------------------------------------------


def _decode_once(st):
    for grp, x, group, ws in st["calls"]:
        if group is not None:
            B.qeft_linear_fwd_group(None, None, x, group=group)
        else:
            d, w = st["layers"][grp[0]]
            B.qeft_linear_fwd(d, w, x, st["ys"][grp[0]], ws=ws)


def prepare(case, seed):
    m, kind = case["m"], case["kind"]
    shapes, groups = _layers(case)
    if kind == "search":
        oc, ic = shapes[0]
        d = _desc(case, oc, ic)
        return dict(kind=kind, d=d, w=_normal(_gen(seed, 100), oc, ic, 0.02), out=B.Weight(d))
    layers = [_store(case, seed, i, oc, ic) for i, (oc, ic) in enumerate(shapes)]
    st = dict(kind=kind, layers=layers)
    if kind == "decode":
        st["ys"] = [_rows(m, oc) for oc, _ in shapes]
        st["calls"] = []
        for n, grp in enumerate(groups):
            x = _x(case, seed, n, shapes[grp[0]][1])
            group = B.Group([layers[i][0] for i in grp], [layers[i][1] for i in grp], [st["ys"][i] for i in grp]) if len(grp) > 1 else None
            st["calls"].append((grp, x, group, False if group else _ws(layers[grp[0]][0], B.QEFT_OP_FWD, m)))
        _decode_once(st)                       # the kernels' first launch is not part of a capture
        torch.cuda.synchronize()
        st["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(st["graph"]):
            _decode_once(st)
        return st
    d, w = layers[0]
    oc, ic = shapes[0]
    st.update(d=d, w=w, x=_x(case, seed, 0, ic), y=_rows(m, oc))
    if kind == "out":
        perm = _perm(case, seed, ic)
        x = torch.empty_like(st["x"])
        x[:, perm.long()] = st["x"]            # the weak channels are the large ones, where they lie
        st.update(x=x, perm=perm, weak_at=perm[ic - case["k"]:].long(), dy=_dy(case, seed, oc), dx=_rows(m, ic),
                  dw=torch.empty((oc, case["k"]), dtype=torch.float32, device="cuda"),
                  ws_f=_ws(d, B.QEFT_OP_FWD_IRREGULAR, m), ws_b=_ws(d, B.QEFT_OP_BWD_DX_IRREGULAR, m), ws_w=_ws(d, B.QEFT_OP_WEAK_GRAD, m))
    else:
        st["ws_f"] = _ws(d, B.QEFT_OP_FWD, m)
        if kind == "tune":
            st.update(xw=st["x"][:, ic - case["k"]:], dy=_dy(case, seed, oc), dx=_rows(m, ic),
                      dw=torch.empty((oc, case["k"]), dtype=torch.float32, device="cuda"), ws_b=_ws(d, B.QEFT_OP_BWD, m))
    return st


def run(st):
    kind = st["kind"]
    if kind == "decode":
        st["graph"].replay()
        return st["ys"]
    if kind == "search":
        w = B.qeft_pack_search(st["d"], st["w"], N_GRID, STEP, out=st["out"])
        return {"qweight": w.qweight, "scales": w.scales, "zeros": w.zeros, "weak": w.weak}
    d, w = st["d"], st["w"]
    if kind == "fwd":
        return B.qeft_linear_fwd(d, w, st["x"], st["y"], ws=st["ws_f"])
    if kind == "tune":
        y = B.qeft_linear_fwd(d, w, st["x"], st["y"], ws=st["ws_f"])
        dx, dw = B.qeft_linear_bwd(d, w, st["dy"], st["xw"], st["dx"], st["dw"], ws=st["ws_b"] if st["ws_b"] is not False else None)
        return {"y": y, "dx": dx, "dw": dw}
    y = B.qeft_linear_fwd_irregular(d, w, st["perm"], st["x"], st["y"], ws=st["ws_f"])
    dx = B.qeft_linear_bwd_dx_irregular(d, w, st["perm"], st["dy"], st["dx"], ws=st["ws_b"])
    xw = st["x"].index_select(1, st["weak_at"])
    dw = B.qeft_weak_grad(d, st["dy"], xw, st["dw"], ws=st["ws_w"] if st["ws_w"] is not False else None)
    return {"y": y, "dx": dx, "dw": dw}


# ---- work, tolerance, exact --------------------------------------------------------------------------------------------


def _stored_bytes(case, oc, ic):
    kq = ic - case["k"]
    return oc * (kq * case["bits"] / 8 + 4 * -(-kq // G) + 2 * case["k"])


def work(case):
    m, k = case["m"], case["k"]
    shapes, groups = _layers(case)
    if case["kind"] == "search":
        oc, ic = shapes[0]
        # a candidate's code and error of a weight: quotient, rounding, zero-point, difference, product, square and sum
        return {"bytes": 2 * oc * ic + _stored_bytes(case, oc, ic), "flops": 7 * N_GRID * oc * (ic - k)}
    stored = sum(_stored_bytes(case, oc, ic) for oc, ic in shapes)
    xs = sum(2 * m * shapes[g[0]][1] for g in groups)
    ys = sum(2 * m * oc for oc, _ in shapes)
    mac = sum(oc * ic for oc, ic in shapes)
    if case["kind"] in ("fwd", "decode"):
        return {"bytes": stored + xs + ys, "flops": 2 * m * mac}
    oc, ic = shapes[0]
    return {"bytes": stored + 2 * (xs + ys) + 4 * oc * k + (4 * ic if case["kind"] == "out" else 0), "flops": 4 * m * mac + 2 * m * oc * k}


def tolerance(case):
    if case["kind"] == "search":
        # the search scores in fp32: where two candidates are closer than its rounding either is kept
        return {"rel": 1e-3, "max": 0.9, "differ": 1e-3}
    # fp16 results (2e-4 by themselves), weights rounded to fp16 once in the tiled kernels, split sums in fp16: 2.0e-4 to
    # 3.6e-4 from the 64-bit result, so up to 5e-4 between two implementations
    return {"rel": 1.5e-3, "max": 0.02}


def _dequantize(codes, scales, zeros, weak):
    oc, kq = codes.shape
    w = torch.empty((oc, kq + weak.shape[1]), dtype=torch.float64, device="cuda")
    w[:, kq:] = weak.double()
    for c in range(0, kq, G):
        w[:, c: min(kq, c + G)] = (codes[:, c: c + G].double() - zeros[:, c // G, None].double()) * scales[:, c // G, None].double()
    return w


def _search_exact(case, seed):
    """Scales and zero-points of the best of the candidates p = 1 - i * step of every group; the decisions in fp32, the error in 64 bits."""
    oc, ic = case["oc"], case["ic"]
    k, qmax = case["k"], float(2 ** case["bits"] - 1)
    kq = ic - k
    w = _normal(_gen(seed, 100), oc, ic, 0.02)
    ng = -(-kq // G)
    p = torch.zeros((oc, ng * G), dtype=torch.float32, device="cuda")
    p[:, :kq] = w[:, :kq].float()
    p = p.view(oc, ng, G)
    lo, hi = p.amin(2).clamp(max=0.0), p.amax(2).clamp(min=0.0)
    best = torch.full((oc, ng), float("inf"), dtype=torch.float64, device="cuda")
    bs, bz = torch.ones_like(lo), torch.zeros_like(lo)
    step = torch.tensor(STEP, dtype=torch.float32, device="cuda")
    for i in range(N_GRID):
        f = 1.0 - float(i) * step
        l, h = f * lo, f * hi
        s = ((h - l) / qmax).half().float()
        s = torch.where(s > 0, s, torch.ones_like(s))
        z = (-l / s).round().clamp(0, qmax)
        q = ((p / s[..., None]).round() + z[..., None]).clamp(0, qmax)
        e = (p.double() - s.double()[..., None] * (q - z[..., None]).double()).square().sum(2)
        take = e < best
        best = torch.where(take, e, best)
        bs, bz = torch.where(take, s, bs), torch.where(take, z, bz)
    lay = B.qeft_layout(_desc(case, oc, ic))
    out = [torch.zeros((oc, lay.group_stride), dtype=torch.float64, device="cuda") for _ in range(2)]
    out[0][:, :ng], out[1][:, :ng] = bs.double(), bz.double()
    return {"qweight": None, "scales": out[0], "zeros": out[1], "weak": w[:, kq:].double()}


def exact(case, seed):
    if case["kind"] == "search":
        return _search_exact(case, seed)
    shapes, groups = _layers(case)
    if case["kind"] == "decode":
        ys = [None] * len(shapes)
        for n, grp in enumerate(groups):
            x = _x(case, seed, n, shapes[grp[0]][1]).double()
            for i in grp:
                ys[i] = x @ _dequantize(*_components(case, seed, i, *shapes[i])).t()
        return ys
    oc, ic = shapes[0]
    kq = ic - case["k"]
    w = _dequantize(*_components(case, seed, 0, oc, ic))
    x = _x(case, seed, 0, ic).double()
    y = x @ w.t()
    if case["kind"] == "fwd":
        return y
    dy = _dy(case, seed, oc).double()
    dx = dy @ w
    dw = dy.t() @ x[:, kq:]
    if case["kind"] == "out":
        perm = _perm(case, seed, ic).long()
        at = torch.empty_like(dx)
        at[:, perm] = dx
        dx = at
    return {"y": y, "dx": dx, "dw": dw}
