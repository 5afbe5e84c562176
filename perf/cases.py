"""The work that users of this library have it do, as measurable cases.

A case is one pass of one operation through the public entry points (the Python binding, a call per
layer, every layer with its own capsule, caches and parameters, one workspace for all):

  decode    one decode step: kvc_reconstruct_attend_decode for each layer
  ragged    the same for a batch of sequences with their own image and text counts
  static    one decode step of the variant without reconstruction: kvc_static_attend_decode
  full      one decode step over the uncompressed cache: kvc_attend_full_decode
  compress  the prefill's pass: kvc_compress for each layer
  hidden    the first layer of the two-layer key reconstructor: kvc_mlp_hidden, once per prefill
  layer     a layer from start to end: kvc_compress, then one decode step on the capsule it made

Names of the sizes: B batch, Hq / Hkv query / KV heads, d head dimension, n vision tokens of an image
block, I image blocks, c compression rate, t text rows in the cache.  The listed sizes are those of the
benchmark's workloads (paper_2605_16439_amd/synth.py), and for the calls that those leave out generic ones.
"""
import random

import torch

from paper_2605_16439_amd import kvcapsule as kv

DEV = "cuda:0"


def listed():
    def case(name, op, B, Hq, Hkv, d, n, I, c, t, layers, dtype="bf16", mix=0):
        return dict(name=name, op=op, B=B, Hq=Hq, Hkv=Hkv, d=d, n=n, I=I, c=c, t=t, layers=layers, dtype=dtype, mix=mix)

    return [
        # the smallest work: one layer in fp32, compressed and attended once (checks, calibration)
        case("layer_f32_576x1", "layer", 1, 8, 2, 64, 576, 1, 0.6, 64, 1, dtype="f32"),
        # one image per sequence, multi-head attention: the common single-image chat
        case("decode_576x1", "decode", 8, 32, 32, 128, 576, 1, 0.6, 128, 8),
        # a high-resolution image as five tiles, large batch: the most bytes per call
        case("decode_576x5", "decode", 16, 32, 32, 128, 576, 5, 0.6, 256, 4),
        # several images per sequence, grouped-query attention: a token through all 28 layers
        case("decode_1024x8", "decode", 4, 28, 4, 128, 1024, 8, 0.6, 512, 28),
        # a long video: many short image blocks, long text
        case("decode_256x64", "decode", 8, 28, 4, 128, 256, 64, 0.6, 1024, 4),
        # continuous batching: sequences with their own numbers of images and text rows
        case("ragged_1024x8", "ragged", 4, 28, 4, 128, 1024, 8, 0.6, 512, 8, mix=3),
        # one user, images whose token count follows their resolution (27 x 27 patches): odd n
        case("decode_729x3", "decode", 1, 28, 4, 128, 729, 3, 0.6, 200, 4),
        # prefill of the headline workload, and of the odd-sized images
        case("compress_1024x8", "compress", 4, 28, 4, 128, 1024, 8, 0.6, 0, 4),
        case("compress_729x3", "compress", 1, 28, 4, 128, 729, 3, 0.6, 0, 2),
        # the ablation without reconstruction
        case("static_1024x8", "static", 4, 28, 4, 128, 1024, 8, 0.6, 512, 4),
        # the two-layer reconstructor's share of the prefill
        case("hidden_1024x8", "hidden", 4, 28, 4, 128, 1024, 8, 0.6, 0, 1),
        # plain attention over the uncompressed cache, which every capsule figure is compared with
        case("full_1024x8", "full", 4, 28, 4, 128, 1024, 8, 0.0, 512, 8),
    ]


# (query heads, KV heads) of the models that the benchmark and the tests shape their layers after
HEADS = [(32, 32), (28, 4), (32, 8), (16, 2), (12, 2), (14, 2), (16, 8), (8, 2)]


def _log(rng, lo, hi):
    return min(hi, max(lo, round(lo * (hi / lo) ** rng.random())))


# largest multiply-adds of a drawn case (the matrix-core calls reach further than the others)
MACS = {"decode": 4.0e9, "ragged": 4.0e9, "static": 2.0e9, "full": 2.0e9, "compress": 8.0e9, "hidden": 2.8e9, "layer": 2.0e8}


def draw(rng):
    """One more case.  Image blocks of 64 to 1024 tokens: half of the draws a multiple of 64 (square
    grids, merged patches), half any number; fp32 in whole-layer cases only, as in the listed ones."""
    while True:
        op = rng.choice(["decode", "decode", "decode", "ragged", "static", "full", "compress", "compress", "hidden", "layer"])
        Hq, Hkv = rng.choice(HEADS)
        n = rng.choice([256, 576, 1024, 64 * rng.randint(1, 16)]) if rng.random() < 0.5 else _log(rng, 64, 1024)
        c = dict(op=op, B=_log(rng, 1, 16), Hq=Hq, Hkv=Hkv, d=128, n=n, I=_log(rng, 1, 64),
                 c=round(rng.uniform(0.3, 0.85), 2), t=_log(rng, 1, 1500), layers=rng.choice([1, 2, 4]), dtype="bf16",
                 mix=rng.randint(1, 1000))
        if op == "layer":
            c.update(B=rng.randint(1, 2), I=rng.randint(1, 4), d=rng.choice([64, 128]), layers=1, dtype=rng.choice(["f32", "f32", "bf16"]))
            c["Hq"], c["Hkv"] = rng.choice([(8, 2), (4, 4), (16, 2), (14, 2)])
        if op == "hidden":
            c["layers"] = 1
        if op == "full":
            c["c"] = 0.0
        w = work(c)
        if w["flops"] / 2 <= MACS[op] and w["bytes"] <= 1.4e9:
            return c


PER_LAYER = ("params", "K", "V", "Kc", "Vc", "W1", "H", "Kt", "Vt", "q", "kn", "vn", "out")
WRITTEN = {"compress": ("Kc", "Vc"), "decode": ("out", "Kt", "Vt"), "ragged": ("out", "Kt", "Vt"), "static": ("out", "Kt", "Vt"),
           "full": ("out", "K", "V"), "hidden": ("H",), "layer": ("Kc", "Vc", "out", "Kt", "Vt")}


def _counts(case):
    """Image blocks and text rows of each sequence of a ragged batch, the same for every seed."""
    r = random.Random(case["mix"])
    return ([r.randint(0, case["I"]) for _ in range(case["B"])], [r.randint(0, case["t"]) for _ in range(case["B"])])


def _m(case):
    return kv.kvc_compressed_len(case["n"], case["c"])


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def prepare(case, seed):
    """Tensors of the laws that the benchmark uses: keys, values and queries N(0, 1), each key channel
    scaled by U(0.5, 4); parameters N(0, 1 / fan-in); compressed values N(0, 1), as a projection of
    N(0, 1) values with such a U has them.  theta and U are packed once, where the library has a packed
    form for the shape."""
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * (seed + 1))
    B, Hq, Hkv, d, n, I, L, t = (case[k] for k in ("B", "Hq", "Hkv", "d", "n", "I", "layers", "t"))
    op, m, dt = case["op"], _m(case), _dtype(case)
    cap = t + 64
    shape = kv.make_shape(B, Hq, Hkv, d, n, I, m, dt)

    def normal(*size, scale=1.0):
        x = torch.randn(size, generator=g, device=DEV)
        return (x * scale if scale != 1.0 else x).to(dt)

    def keys(*size):
        x = torch.randn(size, generator=g, device=DEV)
        x *= 0.5 + 3.5 * torch.rand((1, Hkv) + (1,) * (len(size) - 3) + (d,), generator=g, device=DEV)
        return x.to(dt)

    def layers(draw_one, *size):
        """One tensor for all layers, its first index the layer."""
        x = torch.zeros((L,) + size, dtype=dt, device=DEV)
        if draw_one is not None:
            for y in x:
                y.copy_(draw_one(*size))
        return x

    st = dict(case=case, shape=shape, cap=cap)
    if op == "full":
        st["kv_len"] = I * n + t
        st["ws"] = torch.empty(kv.kvc_attend_full_workspace_bytes(B, Hq, Hkv, d, dt, I * n + cap) + 256, dtype=torch.uint8, device=DEV)
    else:
        st["ws"] = kv.new_workspace(shape, cap, DEV)
    if op == "ragged":
        st["n_img"], st["t_len"] = (torch.tensor(x, dtype=torch.int32, device=DEV) for x in _counts(case))
    if op in ("decode", "ragged", "compress", "layer"):
        st["keep"], st["params"] = [], []
        for _ in range(L):
            idx = torch.sort(torch.randperm(n, generator=g, device=DEV)[:m]).values.to(torch.int32)
            theta, U = normal(Hkv, m, n, scale=m ** -0.5), normal(Hkv, m, n, scale=n ** -0.5)
            p = [idx, theta, U, normal(Hkv, d, scale=d ** -0.5)]
            if op in ("decode", "ragged") and n % 8 == 0:
                p += [kv.kvc_pack_theta(shape, theta), kv.kvc_pack_u(shape, U)]
            st["keep"].append(p)
            st["params"].append(kv.make_params(*p))
    if op in ("compress", "layer"):             # a prompt in front of the images and room behind them, as a backbone's cache has
        st["pre"] = 35
        st["K"], st["V"] = (layers(f, B, Hkv, 35 + I * n + cap, d) for f in (keys, normal))
    if op == "full":
        st["K"], st["V"] = (layers(f, B, Hkv, I * n + cap, d) for f in (keys, normal))
    if op != "full":
        made = op in ("compress", "layer")      # by the pass itself
        st["Kc"], st["Vc"] = (layers(None if made else f, B, Hkv, I, m, d) for f in (keys, normal))
    if op == "hidden":
        st["W1"], st["H"] = normal(L, Hkv, m, m, scale=m ** -0.5), layers(None, B, Hkv, I, m, d)
    if op in ("decode", "ragged", "static", "layer"):
        st["Kt"], st["Vt"] = (layers(f, B, Hkv, cap, d) for f in (keys, normal))
    if op not in ("compress", "hidden"):
        st["q"], st["kn"], st["vn"] = layers(normal, B, Hq, d), layers(keys, B, Hkv, d), layers(normal, B, Hkv, d)
        st["out"] = layers(None, B, Hq, d)
    st["of_layer"] = [{k: v[i] for k, v in st.items() if k in PER_LAYER} for i in range(L)]
    return st


def run(st):
    """One pass; its outputs, with the caches and capsules that it wrote to."""
    op, shape, cap, ws, t = st["case"]["op"], st["shape"], st["cap"], st["ws"], st["case"]["t"]
    for i in range(st["case"]["layers"]):
        a = st["of_layer"][i]
        if op in ("compress", "layer"):
            kv.kvc_compress(shape, a["params"], a["K"], a["V"], st["pre"], a["Kc"], a["Vc"], ws)
        if op in ("decode", "layer"):
            kv.kvc_reconstruct_attend_decode(shape, a["params"], a["q"], a["Kc"], a["Vc"], a["Kt"], a["Vt"], t, cap,
                                             a["kn"], a["vn"], 0.0, a["out"], None, ws)
        elif op == "ragged":
            kv.kvc_reconstruct_attend_decode_ragged(shape, a["params"], a["q"], a["Kc"], a["Vc"], a["Kt"], a["Vt"], st["n_img"],
                                                    st["t_len"], cap, a["kn"], a["vn"], 0.0, a["out"], None, ws)
        elif op == "static":
            kv.kvc_static_attend_decode(shape, a["q"], a["Kc"], a["Vc"], a["Kt"], a["Vt"], t, cap, a["kn"], a["vn"], 0.0,
                                        a["out"], None, ws)
        elif op == "full":
            kv.kvc_attend_full_decode(a["q"], a["K"], a["V"], st["kv_len"], a["kn"], a["vn"], 0.0, a["out"], None, ws)
        elif op == "hidden":
            kv.kvc_mlp_hidden(shape, a["W1"], kv.KVC_ACT_GELU, a["Kc"], a["H"])
    return [st[k] for k in WRITTEN[op]]


def work(case):
    """What a pass cannot do without: each tensor row it needs read once, each result written once;
    multiply-adds of the score-space order (two operations each)."""
    B, Hq, Hkv, d, n, I, L, t = (case[k] for k in ("B", "Hq", "Hkv", "d", "n", "I", "layers", "t"))
    op, m, es = case["op"], _m(case), 4 if case["dtype"] == "f32" else 2
    blocks, rows = B * I, B * (t + 1)                                 # image blocks and text rows, per KV head
    if op == "ragged":
        ni, tl = _counts(case)
        blocks, rows = sum(ni), sum(tl) + B
    elems = macs = 0
    if op in ("compress", "layer"):
        elems += blocks * Hkv * (n + 3 * m) * d + Hkv * (m * n + d)   # V, kept rows of K, the capsule; U, mu
        macs += blocks * Hkv * m * n * d
    if op in ("decode", "ragged", "layer"):
        elems += Hkv * (2 * m * n + d) + 2 * Hkv * (blocks * m + rows) * d + 2 * B * Hq * d
        macs += Hq * (blocks * (2 * m * n + 2 * m * d) + 2 * rows * d)
    if op == "static":
        elems += 2 * Hkv * (blocks * m + rows) * d + 2 * B * Hq * d
        macs += Hq * (blocks * m + rows) * 2 * d
    if op == "full":
        elems += 2 * Hkv * (blocks * n + rows) * d + 2 * B * Hq * d
        macs += Hq * (blocks * n + rows) * 2 * d
    if op == "hidden":
        elems += 2 * blocks * Hkv * m * d + Hkv * m * m
        macs += blocks * Hkv * m * m * d
    return {"bytes": L * elems * es, "flops": 2 * L * macs}


def tolerance(case):
    """Four times what was measured: in fp32 the output against float64 (1.3e-6); of a bf16 projection what
    another order of the sums changes (4e-5: a few results round the other way); of a bf16 attention against
    float64 1.7e-3 (the rounding of the result) where the intermediate scores and weights are fp32, and
    3.9e-3 where they are bf16, which is how the sizes below are computed."""
    if case["dtype"] == "f32":
        return {"rel": 5e-6}
    if case["op"] in ("compress", "hidden"):
        return {"rel": 2e-4}
    if case["op"] in ("decode", "ragged", "layer") and case["d"] == 128 and case["n"] in (256, 576, 1024):
        return {"rel": 1.6e-2}
    return {"rel": 7e-3}
