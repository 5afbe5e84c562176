"""Matrix-core kernels at shapes that do not divide into their tiles, against the CPU oracle through the C ABI.

Results that are one rounding of a float32 sum (compressed values, hidden rows) are compared with the oracle's
one rounding of the exact sum: they differ only where the float32 error (about sqrt(n) 2^-24 of the sum) moves a
value across a rounding boundary, fewer than one value in a thousand, by one bf16 step (2^-8 relative), which is
1.2e-4 of a block's norm; the bar is 1e-3.
"""
import numpy as np
import pytest
import torch

from oracle import kvc_oracle as orc
from paper_2605_16439_amd import kvcapsule as kv
from paper_2605_16439_amd import synth

from helpers import block_rel_err, decode_plan, f64, store_code, unpack_vc
from test_gpu_parity import Layer

pytestmark = pytest.mark.gpu
DEV = "cuda"
ONE_ROUNDING = 1e-3


def wl(n, I, B=1, hq=4, hkv=2, t=4, steps=1):
    return synth.Workload(f"any_n{n}", 92, 1, B, hq, hkv, 128, "bf16", n, I, 0.6, t, steps)


# n around the 8-column piece of a row of U and the 64-position tile, odd values included; m around 16 and 256 rows
@pytest.mark.parametrize("n,m", [(8, 8), (9, 5), (15, 3), (63, 17), (65, 65), (71, 16), (127, 40), (129, 129), (193, 150),
                                 (329, 257), (729, 292), (1023, 410)])
def test_compress_any_block_length(n, m):
    w = wl(n, 2)
    L = Layer(w, m, pre=3, post=1)
    L.gKc.fill_(float("nan"))
    L.gVc.fill_(float("nan"))
    print(f"[any] compress n={n} m={m}", flush=True)
    L.compress()
    Kc_ref, Vc_ref = orc.compress(f64(L.K), f64(L.V), L.p["key_idx"].numpy(), f64(L.p["U"]), f64(L.p["mu"]), n, 2, 3, store_code(w))
    assert np.array_equal(f64(L.gKc), Kc_ref)
    assert block_rel_err(unpack_vc(L.gVc, m, 128), Vc_ref) <= ONE_ROUNDING


@pytest.mark.parametrize("act", [kv.KVC_ACT_IDENTITY, kv.KVC_ACT_RELU, kv.KVC_ACT_GELU])
@pytest.mark.parametrize("m", [7, 8, 9, 63, 64, 65, 103, 128, 129, 257, 410])
def test_hidden_rows_any_length(m, act):
    B, hkv, I = 1, 2, 2
    g = torch.Generator().manual_seed(m)
    Kc = torch.randn((B, hkv, I, m, 128), generator=g).to(torch.bfloat16)
    W1 = (torch.randn((hkv, m, m), generator=g) * m ** -0.5).to(torch.bfloat16)
    H = torch.full((B, hkv, I, m, 128), float("nan"), dtype=torch.bfloat16, device=DEV)
    print(f"[any] hidden m={m} act={act}", flush=True)
    kv.kvc_mlp_hidden(kv.make_shape(B, 4, hkv, 128, 1024, I, m, torch.bfloat16), W1.to(DEV), act, Kc.to(DEV), H)
    torch.cuda.synchronize()
    assert block_rel_err(f64(H), orc.mlp_hidden(f64(Kc), f64(W1), act, orc.STORE_BF16)) <= ONE_ROUNDING


# GELU over its range: with W1 = I a hidden row is the activation of a key row, rounded once (2^-8 of the value at most;
# 1e-5 for the float32 evaluation and for results below bf16's smallest normal number, which are left out)
def test_gelu_over_its_range():
    m, d = 128, 128
    mag = torch.logspace(-6, 2, m * d // 2, dtype=torch.float64)
    x = torch.cat([mag, -mag]).to(torch.bfloat16).reshape(1, 1, 1, m, d)
    x[0, 0, 0, 0, :2] = torch.tensor([0.0, -0.0])
    H = torch.full_like(x, float("nan")).to(DEV)
    kv.kvc_mlp_hidden(kv.make_shape(1, 1, 1, d, 1024, 1, m, torch.bfloat16), torch.eye(m, dtype=torch.bfloat16)[None].to(DEV), kv.KVC_ACT_GELU,
                      x.to(DEV), H)
    ref = x.double() * 0.5 * torch.special.erfc(-x.double() / 2 ** 0.5)
    got = H.cpu().double()
    assert torch.isfinite(got).all()
    assert ((got - ref).abs() <= (2.0 ** -8 + 1e-5) * ref.abs() + 2.0 ** -126).all()


# Attention results whose scores, weights and sums are float32 differ from the exact result by the rounding of the
# output alone.  bf16 keeps 8 significant bits: neighbours are 2^-7 apart at 1.0, so rounding to nearest moves a value
# by at most 2^-8 of itself, and a row by at most 2^-8 of its norm; float32 adds about 1e-5.
OUT_ROUNDING = 2.0 ** -8 + 1e-4


def check_rows(out, ref):
    assert np.all(np.isfinite(out))
    e = np.linalg.norm(out - ref, axis=-1) / np.maximum(np.linalg.norm(ref, axis=-1), 1e-30)
    print(f"[any]   row rel err {e.max():.3e}", flush=True)
    assert e.max() <= OUT_ROUNDING


# m around the 8-row block and the 32-row step (record shorter than a block included), text around the 128-row
# workgroup step, runs of several steps, every kind of group size, no image, no text
@pytest.mark.parametrize("hq,hkv,I,m,t", [(4, 4, 1, 1, 0), (7, 1, 2, 7, 1), (6, 2, 3, 8, 127), (24, 2, 1, 31, 128), (16, 1, 3, 33, 129),
                                          (14, 2, 5, 41, 300), (8, 8, 70, 64, 5), (2, 2, 0, 20, 260), (28, 4, 64, 103, 40)])
def test_static_variant_any_shape(hq, hkv, I, m, t):
    w = wl(128, I, B=2, hq=hq, hkv=hkv, t=t)
    L = Layer(w, m)
    g = torch.Generator().manual_seed(m)
    L.gKc = torch.randn(L.gKc.shape, generator=g).to(torch.bfloat16).to(DEV)
    L.gVc = torch.randn(L.gVc.shape, generator=g).to(torch.bfloat16).to(DEV)
    q, kn, vn = synth.make_step_inputs(w, 0, 0)
    print(f"[any] static hq={hq} hkv={hkv} I={I} m={m} t={t}", flush=True)
    kv.kvc_static_attend_decode(L.shape, q.to(DEV), L.gKc, L.gVc, L.gKt, L.gVt, t, w.text_cap, kn.to(DEV), vn.to(DEV), 0.0, L.out,
                                L.lse, L.ws)
    torch.cuda.synchronize()
    Kt, Vt = f64(L.Kt).copy(), f64(L.Vt).copy()
    ref, lref = orc.static_attend_decode(f64(q), f64(L.gKc), unpack_vc(L.gVc, m, 128), Kt, Vt, t, f64(kn), f64(vn))
    check_rows(f64(L.out), ref)
    assert np.abs(f64(L.lse) - lref).max() <= 1e-4
    assert np.array_equal(f64(L.gKt), Kt) and np.array_equal(f64(L.gVt), Vt)


def decode_case(w, m, ragged=None, packed=False):
    """One step on random capsules against the oracle; ragged: (image counts, text counts) with NaNs in the capsule
    slots and text rows that a sequence does not own."""
    L = Layer(w, m)
    g = torch.Generator().manual_seed(m)
    L.gKc = torch.randn(L.gKc.shape, generator=g).to(torch.bfloat16).to(DEV)
    L.gVc = torch.randn(L.gVc.shape, generator=g).to(torch.bfloat16).to(DEV)
    if packed:
        thp, up = kv.kvc_pack_theta(L.shape, L.g["theta"]), kv.kvc_pack_u(L.shape, L.g["U"])
        L.params = kv.make_params(L.g["key_idx"], L.g["theta"], L.g["U"], L.g["mu"], thp, up)
    q, kn, vn = synth.make_step_inputs(w, 0, 0)
    th, U, mu = f64(L.p["theta"]), f64(L.p["U"]), f64(L.p["mu"])
    Kt, Vt = f64(L.Kt).copy(), f64(L.Vt).copy()
    Kc, Vc = f64(L.gKc), unpack_vc(L.gVc, m, 128)
    print(f"[any] decode {w.n_q_heads}/{w.n_kv_heads} n={w.n_img_tokens} m={m} I={w.n_images} t={w.text_len} packed={packed} {ragged}", flush=True)
    if ragged is None:
        out, lse = L.decode(q.to(DEV), w.text_len, kn.to(DEV), vn.to(DEV))
        ref, lref = orc.reconstruct_attend_decode(f64(q), Kc, Vc, th, U, mu, w.n_img_tokens, Kt, Vt, w.text_len, f64(kn), f64(vn))
        assert np.array_equal(f64(L.gKt), Kt) and np.array_equal(f64(L.gVt), Vt)
    else:
        ni, tl = ragged
        for b in range(w.batch):
            L.gKc[b, :, ni[b]:] = float("nan")
            L.gVc[b, :, ni[b]:] = float("nan")
            L.gKt[b, :, tl[b] + 1:] = float("nan")
            L.gVt[b, :, tl[b] + 1:] = float("nan")
        dev = [torch.tensor(x, dtype=torch.int32, device=DEV) for x in ragged]
        kv.kvc_reconstruct_attend_decode_ragged(L.shape, L.params, q.to(DEV), L.gKc, L.gVc, L.gKt, L.gVt, *dev, w.text_cap, kn.to(DEV),
                                                vn.to(DEV), 0.0, L.out, L.lse, L.ws)
        torch.cuda.synchronize()
        out, lse = f64(L.out), f64(L.lse)
        ref, lref = orc.reconstruct_attend_decode_ragged(f64(q), Kc, Vc, th, U, mu, w.n_img_tokens, ni, tl, Kt, Vt, f64(kn), f64(vn))
    check_rows(out, ref)
    assert np.abs(lse - lref).max() <= 1e-4


# n around the 8-column piece and the slices of 128 / 256 / 512 positions; m around 8, 16 and 32 rows; tiles with fewer
# image blocks than they hold; group sizes without a tuned kernel; batches that select each slice width
@pytest.mark.parametrize("hq,hkv,B,I,n,m,t", [
    (4, 4, 1, 1, 8, 3, 0), (7, 1, 1, 3, 9, 9, 1), (6, 2, 2, 1, 127, 8, 5), (3, 1, 1, 5, 128, 128, 127), (14, 2, 1, 2, 129, 31, 128),
    (28, 4, 1, 3, 729, 292, 200), (16, 1, 1, 2, 333, 33, 130), (5, 1, 2, 7, 257, 103, 300), (12, 1, 1, 4, 511, 64, 20),
    (9, 1, 1, 1, 1023, 640, 3), (4, 2, 2, 9, 100, 41, 2500), (64, 32, 8, 3, 200, 40, 10), (32, 8, 16, 2, 300, 90, 33),
    (32, 32, 8, 17, 65, 17, 4), (2, 1, 1, 64, 515, 65, 9), (8, 8, 32, 3, 520, 40, 7), (2, 2, 1, 0, 50, 20, 40),
    (10, 2, 1, 2, 1024, 1024, 6)])
def test_decode_any_shape(hq, hkv, B, I, n, m, t):
    decode_case(wl(n, I, B=B, hq=hq, hkv=hkv, t=t), m)


@pytest.mark.parametrize("hq,hkv,B,I,n,m,t", [(4, 4, 1, 1, 8, 3, 0), (14, 2, 1, 3, 136, 29, 9), (28, 4, 1, 3, 728, 292, 200),
                                              (64, 32, 8, 3, 200, 43, 10), (32, 8, 16, 2, 304, 90, 33), (8, 8, 32, 3, 520, 47, 7)])
def test_decode_any_shape_packed_parameters(hq, hkv, B, I, n, m, t):
    decode_case(wl(n, I, B=B, hq=hq, hkv=hkv, t=t), m, packed=True)


# Several tiles per workgroup, the last workgroup with fewer of them, the last tile partly filled: state carried from tile
# to tile, LDS used again.  Every slice width, both forms of the parameters; ragged batches whose sequences end inside the
# first, a middle and the last tile of a workgroup, before the first and behind the last.
@pytest.mark.parametrize("hq,hkv,B,I,n,m,t,ps,tiles,packed", [s + (packed,) for s in [
    (7, 1, 1, 99, 40, 17, 9, 128, 2), (7, 1, 2, 61, 136, 33, 140, 128, 2), (7, 1, 1, 99, 136, 41, 0, 128, 3), (28, 4, 1, 33, 729, 70, 30, 128, 3),
    (96, 6, 1, 25, 304, 20, 5, 256, 2), (96, 6, 1, 25, 600, 33, 5, 512, 2)] for packed in (False, True) if not packed or s[4] % 8 == 0])
def test_decode_several_tiles_per_workgroup(hq, hkv, B, I, n, m, t, ps, tiles, packed):
    plan = decode_plan(hq, hkv, B, I, n, m, t + 1, t + 1)
    assert (plan[0], plan[2]) == (ps, tiles)
    calls = kv.lib().kvc_dev_any_calls()
    decode_case(wl(n, I, B=B, hq=hq, hkv=hkv, t=t), m, packed=packed)
    assert kv.lib().kvc_dev_any_calls() == calls + 1


# Partial logits of plain parameters in LDS of their own up to m = 768, 640 and 384 (slices of 128, 256 and 512 positions), in the
# place of the scores beyond: both sides of each line, and several tiles per workgroup on both sides
@pytest.mark.parametrize("hq,hkv,B,I,n,m,ps,tiles", [
    (4, 2, 1, 2, 1023, 768, 128, 1), (4, 2, 1, 2, 1023, 769, 128, 1), (7, 1, 1, 60, 1023, 769, 128, 5), (7, 1, 1, 60, 1023, 736, 128, 5),
    (8, 8, 8, 2, 1023, 640, 256, 1), (8, 8, 8, 2, 1023, 641, 256, 1), (8, 8, 16, 2, 1023, 384, 512, 1), (8, 8, 16, 2, 1023, 385, 512, 1)])
def test_decode_partial_logits_in_both_places(hq, hkv, B, I, n, m, ps, tiles):
    plan = decode_plan(hq, hkv, B, I, n, m, 6, 6)
    assert (plan[0], plan[2]) == (ps, tiles)
    decode_case(wl(n, I, B=B, hq=hq, hkv=hkv, t=5), m)


@pytest.mark.parametrize("hq,hkv,I,n,m,ni,ps,tiles", [
    (7, 1, 99, 136, 41, [1, 4, 99, 50, 0], 128, 3), (16, 1, 25, 304, 20, [25, 1, 0, 24, 13, 2], 256, 2), (16, 1, 25, 600, 33, [25, 1, 0, 24, 13, 2], 512, 2),
    (32, 8, 2, 304, 40, [2, 1, 0, 2] * 4, 256, 1), (8, 8, 3, 520, 40, [3, 0, 1, 2] * 8, 512, 1)])
@pytest.mark.parametrize("packed", [False, True])
def test_ragged_batch_of_every_slice_width_and_several_tiles(hq, hkv, I, n, m, ni, ps, tiles, packed):
    B, t = len(ni), 130
    plan = decode_plan(hq, hkv, B, I, n, m, t + 1, t + 1)
    assert (plan[0], plan[2]) == (ps, tiles)
    calls = kv.lib().kvc_dev_any_calls()
    decode_case(wl(n, I, B=B, hq=hq, hkv=hkv, t=t), m, ragged=(ni, [(37 * b + 5) % (t + 1) for b in range(B)]), packed=packed)
    assert kv.lib().kvc_dev_any_calls() == calls + 1


# small calls at block lengths that have tuned kernels too: inside and just beyond the limits of 10 steps of 32 rows, 256
# vision workgroups and 512 with the text's that send them to the one-pass kernel
@pytest.mark.parametrize("hq,hkv,B,I,n,m,t", [(28, 4, 1, 16, 256, 103, 200), (28, 4, 1, 32, 256, 154, 1), (32, 32, 1, 1, 576, 320, 0),
                                              (14, 2, 1, 12, 576, 160, 700), (4, 1, 1, 1, 1024, 320, 5), (2, 2, 8, 7, 256, 31, 9),
                                              (32, 8, 1, 2, 1024, 160, 129), (8, 8, 2, 3, 576, 97, 257)])
def test_small_calls_of_tuned_block_lengths(hq, hkv, B, I, n, m, t):
    before, calls = kv.lib().kvc_dev_stream_calls(), kv.lib().kvc_dev_any_calls()
    decode_case(wl(n, I, B=B, hq=hq, hkv=hkv, t=t), m, packed=True)
    assert kv.lib().kvc_dev_stream_calls() == before and kv.lib().kvc_dev_any_calls() == calls + 1


@pytest.mark.parametrize("hq,hkv,B,I,n,m,t", [(32, 32, 1, 1, 576, 321, 0), (14, 2, 16, 1, 256, 103, 1800), (28, 4, 1, 50, 256, 154, 1), (28, 4, 1, 2, 256, 103, 8192)])
def test_calls_just_beyond_the_small_ones_take_the_tuned_kernels(hq, hkv, B, I, n, m, t):
    calls = kv.lib().kvc_dev_any_calls()
    L = layer_of(hq, hkv, B, I, n, m, t, packed=True)
    step_of(L, L.ws)
    assert kv.lib().kvc_dev_any_calls() == calls and torch.isfinite(L.out).all()
    L.params = kv.make_params(L.g["key_idx"], L.g["theta"], L.g["U"], L.g["mu"])       # plain parameters: the same kernels, the same result
    out = L.out.clone()
    step_of(L, L.ws)
    assert kv.lib().kvc_dev_any_calls() == calls
    if n != 1024:
        assert torch.equal(out, L.out)


def test_small_ragged_batch_of_a_tuned_block_length():
    decode_case(wl(256, 5, B=5, hq=14, hkv=2, t=140), 103, ragged=([5, 0, 1, 3, 4], [139, 0, 5, 128, 127]), packed=True)


@pytest.mark.parametrize("n,m,packed", [(137, 41, False), (136, 41, True), (600, 100, False), (600, 100, True)])
def test_ragged_batch_any_shape(n, m, packed):
    decode_case(wl(n, 5, B=5, hq=14, hkv=2, t=140), m, ragged=([5, 0, 1, 3, 4], [139, 0, 5, 128, 127]), packed=packed)


# fp32, and bf16 with other head dimensions: d around the 16-channel tile, n around 4 and the slices of 64 and 256
# positions, m around 16 and 32 rows, text around the 128-row step, few and many image blocks
FLOAT_CASES = [(2, 1, 1, 1, 4, 1, 0, 8), (8, 2, 1, 1, 576, 231, 64, 64), (3, 3, 2, 3, 63, 15, 127, 24), (16, 1, 1, 2, 65, 16, 128, 72),
               (14, 2, 2, 5, 130, 33, 300, 128), (4, 4, 2, 3, 257, 129, 1, 136), (10, 2, 1, 4, 1023, 410, 9, 256),
               (32, 32, 16, 2, 260, 17, 5, 40), (1, 1, 1, 0, 10, 4, 2500, 64), (6, 2, 1, 60, 300, 70, 3, 64)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("hq,hkv,B,I,n,m,t,d", FLOAT_CASES)
def test_layer_on_the_fp32_matrix_instruction(hq, hkv, B, I, n, m, t, d, dtype):
    w = synth.Workload(f"float_n{n}", 93, 1, B, hq, hkv, d, dtype, n, I, 0.6, t, 1)
    L = Layer(w, m, pre=3, post=2)
    print(f"[float] {dtype} {hq}/{hkv} B={B} I={I} n={n} m={m} t={t} d={d}", flush=True)
    th, U, mu = f64(L.p["theta"]), f64(L.p["U"]), f64(L.p["mu"])
    if I > 0:
        L.compress()
        Kc_ref, Vc_ref = orc.compress(f64(L.K), f64(L.V), L.p["key_idx"].numpy(), U, mu, n, I, 3, store_code(w))
        assert np.array_equal(f64(L.gKc), Kc_ref)
        assert block_rel_err(unpack_vc(L.gVc, m, d), Vc_ref) <= (1e-5 if dtype == "f32" else ONE_ROUNDING)
    q, kn, vn = synth.make_step_inputs(w, 0, 0)
    Kt, Vt = f64(L.Kt).copy(), f64(L.Vt).copy()
    out, lse = L.decode(q.to(DEV), t, kn.to(DEV), vn.to(DEV))
    ref, lref = orc.reconstruct_attend_decode(f64(q), f64(L.gKc), unpack_vc(L.gVc, m, d), th, U, mu, n, Kt, Vt, t, f64(kn), f64(vn))
    assert np.array_equal(f64(L.gKt), Kt) and np.array_equal(f64(L.gVt), Vt)
    if dtype == "f32":
        e = np.linalg.norm(out - ref, axis=-1) / np.linalg.norm(ref, axis=-1)
        print(f"[float]   row rel err {e.max():.3e}", flush=True)
        assert e.max() <= 1e-5
    else:
        check_rows(out, ref)
    assert np.abs(lse - lref).max() <= 1e-4


@pytest.mark.parametrize("d", [64, 128])
def test_ragged_batch_fp32(d):
    w = synth.Workload("float_ragged", 94, 1, 4, 14, 2, d, "f32", 150, 5, 0.6, 140, 1)
    m = 41
    L = Layer(w, m)
    g = torch.Generator().manual_seed(m)
    L.gKc, L.gVc = (torch.randn(L.gKc.shape, generator=g).to(DEV) for _ in range(2))
    ni, tl = [5, 0, 1, 3], [139, 0, 5, 128]
    Kc, Vc, Kt, Vt = f64(L.gKc), unpack_vc(L.gVc, m, d), f64(L.Kt).copy(), f64(L.Vt).copy()
    for b in range(w.batch):
        L.gKc[b, :, ni[b]:], L.gVc[b, :, ni[b]:], L.gKt[b, :, tl[b] + 1:], L.gVt[b, :, tl[b] + 1:] = (float("nan"),) * 4
    q, kn, vn = synth.make_step_inputs(w, 0, 0)
    dev = [torch.tensor(x, dtype=torch.int32, device=DEV) for x in (ni, tl)]
    kv.kvc_reconstruct_attend_decode_ragged(L.shape, L.params, q.to(DEV), L.gKc, L.gVc, L.gKt, L.gVt, *dev, w.text_cap, kn.to(DEV),
                                            vn.to(DEV), 0.0, L.out, L.lse, L.ws)
    torch.cuda.synchronize()
    ref, lref = orc.reconstruct_attend_decode_ragged(f64(q), Kc, Vc, f64(L.p["theta"]), f64(L.p["U"]), f64(L.p["mu"]), 150, ni, tl, Kt, Vt,
                                                     f64(kn), f64(vn))
    e = np.linalg.norm(f64(L.out) - ref, axis=-1) / np.linalg.norm(ref, axis=-1)
    assert e.max() <= 1e-5 and np.abs(f64(L.lse) - lref).max() <= 1e-4


# A ragged batch plans for the text cache's capacity, as the uniform call does: small calls that would take other kernels,
# tiles of other sizes and text runs of another length if the rows in the cache decided
@pytest.mark.parametrize("hq,hkv,B,I,n,m,t,cap,dtype,d", [
    (14, 2, 16, 1, 256, 103, 100, 2000, "bf16", 128), (14, 2, 5, 5, 137, 41, 100, 2000, "bf16", 128), (28, 4, 1, 3, 256, 60, 30, 500, "bf16", 128),
    (14, 2, 2, 3, 137, 41, 1500, 5000, "bf16", 128), (8, 2, 2, 2, 150, 33, 1500, 5000, "f32", 64), (8, 2, 2, 0, 150, 33, 700, 2100, "f32", 64)])
def test_uniform_batch_through_the_ragged_entry_point(hq, hkv, B, I, n, m, t, cap, dtype, d):
    w = synth.Workload("rag_eq", 95, 1, B, hq, hkv, d, dtype, n, I, 0.6, t, cap - t)
    assert w.text_cap == cap
    res = []
    for ragged in (False, True):
        L = Layer(w, m)
        g = torch.Generator().manual_seed(m)
        L.gKc, L.gVc = (torch.randn(L.gKc.shape, generator=g).to(L.gKc.dtype).to(DEV) for _ in range(2))
        if n % 8 == 0:
            L.params = kv.make_params(L.g["key_idx"], L.g["theta"], L.g["U"], L.g["mu"], kv.kvc_pack_theta(L.shape, L.g["theta"]),
                                      kv.kvc_pack_u(L.shape, L.g["U"]))
        q, kn, vn = (x.to(DEV) for x in synth.make_step_inputs(w, 0, 0))
        print(f"[any] uniform call, ragged={ragged}: {hq}/{hkv} B={B} n={n} m={m} I={I} t={t} cap={cap} {dtype}", flush=True)
        if ragged:
            counts = [torch.full((B,), x, dtype=torch.int32, device=DEV) for x in (I, t)]
            kv.kvc_reconstruct_attend_decode_ragged(L.shape, L.params, q, L.gKc, L.gVc, L.gKt, L.gVt, *counts, cap, kn, vn, 0.0, L.out,
                                                    L.lse, L.ws)
            torch.cuda.synchronize()
            res.append((f64(L.out), f64(L.lse)))
        else:
            res.append(L.decode(q, t, kn, vn))
    assert np.array_equal(res[0][0], res[1][0]) and np.array_equal(res[0][1], res[1][1])


# The first 64 KB of a workspace belong to the arrival counters of the tuned kernels: what another kernel leaves there
# makes their next call wait out its limit in every workgroup
def layer_of(hq, hkv, B, I, n, m, t, dtype="bf16", d=128, packed=False):
    L = Layer(synth.Workload("ctr", 96, 1, B, hq, hkv, d, dtype, n, I, 0.6, t, 2), m)
    g = torch.Generator().manual_seed(m)
    L.gKc, L.gVc = (torch.randn(L.gKc.shape, generator=g).to(L.gKc.dtype).to(DEV) for _ in range(2))
    if packed:
        L.packed = kv.kvc_pack_theta(L.shape, L.g["theta"]), kv.kvc_pack_u(L.shape, L.g["U"])
        L.params = kv.make_params(L.g["key_idx"], L.g["theta"], L.g["U"], L.g["mu"], *L.packed)
    return L


def step_of(L, ws, static=False):
    q, kn, vn = (x.to(DEV) for x in synth.make_step_inputs(L.w, 0, 0))
    tail = (q, L.gKc, L.gVc, L.gKt, L.gVt, L.w.text_len, L.w.text_cap, kn, vn, 0.0, L.out, L.lse, ws)
    if static:
        kv.kvc_static_attend_decode(L.shape, *tail)
    else:
        kv.kvc_reconstruct_attend_decode(L.shape, L.params, *tail)
    torch.cuda.synchronize()


@pytest.mark.parametrize("hq,hkv,B,I,n,m,t,dtype,d,packed,static", [
    (28, 4, 1, 1, 1024, 256, 100, "bf16", 128, True, False), (28, 4, 1, 3, 729, 292, 100, "bf16", 128, False, False),
    (28, 4, 4, 8, 1024, 410, 100, "bf16", 128, False, True), (8, 2, 1, 2, 576, 231, 64, "f32", 64, False, False)])
def test_arrival_counters_are_left_alone(hq, hkv, B, I, n, m, t, dtype, d, packed, static):
    L = layer_of(hq, hkv, B, I, n, m, t, dtype, d, packed)
    ws = torch.full((kv.kvc_workspace_bytes(L.shape, L.w.text_cap) + 256,), 0x5A, dtype=torch.uint8, device=DEV)
    print(f"[any] counters {hq}/{hkv} n={n} {dtype} static={static}", flush=True)
    step_of(L, ws, static)
    head = ws[(-ws.data_ptr()) % 256:][:65536]
    assert (head == 0x5A).all()


def test_large_calls_after_small_ones_do_not_wait():
    small = layer_of(28, 4, 1, 1, 1024, 256, 100, packed=True)
    large = [layer_of(28, 4, 4, 8, 1024, 410, 300, packed=True), layer_of(8, 8, 8, 1, 576, 231, 128)]
    size = max(kv.kvc_workspace_bytes(L.shape, L.w.text_cap) for L in [small] + large)
    ws = torch.zeros(size + 256, dtype=torch.uint8, device=DEV)
    calls = kv.lib().kvc_dev_any_calls()
    for L in large:
        step_of(L, ws)
        alone = kv.lib().kvc_dev_decode_fallbacks()
        step_of(small, ws)
        step_of(small, ws, static=True)
        step_of(L, ws)
        assert kv.lib().kvc_dev_decode_fallbacks() == alone
    assert kv.lib().kvc_dev_any_calls() == calls + 2


# A workspace that is enough for the scalar kernels only (no more than the counters of the others): they serve the call
@pytest.mark.parametrize("dtype,d,static", [("bf16", 128, False), ("bf16", 128, True), ("f32", 64, False), ("bf16", 64, False)])
def test_smallest_accepted_workspace(dtype, d, static):
    hq, B, I, n, m, t = 16, 1, 20, 8, 3, 5
    L = layer_of(hq, 1, B, I, n, m, t, dtype, d)
    need = sum(-(-4 * B * hq * x // 256) * 256 for x in (I * m, L.w.text_cap, I * n, 4, I * m))
    assert need < 65536
    calls = kv.lib().kvc_dev_any_calls()
    res = []
    for ws in (torch.zeros(need + 512, dtype=torch.uint8, device=DEV), L.ws):
        ws = ws[(-ws.data_ptr()) % 256:]
        L.out.zero_()
        step_of(L, ws[:need] if ws.numel() < 65536 else ws, static)
        res.append(f64(L.out))
    assert kv.lib().kvc_dev_any_calls() == calls + (1 if d == 128 and not static else 0)
    e = np.linalg.norm(res[0] - res[1], axis=-1) / np.linalg.norm(res[1], axis=-1)
    print(f"[any] smallest workspace {dtype} d={d} static={static}: {e.max():.3e}", flush=True)
    assert e.max() <= (1e-5 if dtype == "f32" else OUT_ROUNDING * 2)          # two roundings of nearly the same value


# Many very short blocks: either side of the rules that leave them to the scalar kernels
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 256)])
@pytest.mark.parametrize("n,m,I", [(8, 3, 1), (8, 3, 9), (9, 9, 66), (15, 7, 66), (16, 8, 66), (24, 8, 66)])
def test_compress_many_short_blocks(n, m, I, dtype, d):
    w = synth.Workload("short", 97, 1, 4, 4, 2, d, dtype, n, I, 0.6, 1, 1)
    L = Layer(w, m, pre=1, post=1)
    print(f"[any] compress n={n} m={m} I={I} {dtype} d={d}", flush=True)
    L.compress()
    Kc_ref, Vc_ref = orc.compress(f64(L.K), f64(L.V), L.p["key_idx"].numpy(), f64(L.p["U"]), f64(L.p["mu"]), n, I, 1, store_code(w))
    assert np.array_equal(f64(L.gKc), Kc_ref)
    assert block_rel_err(unpack_vc(L.gVc, m, d), Vc_ref) <= (1e-5 if dtype == "f32" else ONE_ROUNDING)


@pytest.mark.parametrize("m,I", [(8, 32), (8, 33), (9, 33)])
def test_hidden_rows_of_many_short_blocks(m, I):
    B, hkv, d = 4, 2, 128
    g = torch.Generator().manual_seed(m)
    Kc = torch.randn((B, hkv, I, m, d), generator=g).to(torch.bfloat16)
    W1 = (torch.randn((hkv, m, m), generator=g) * m ** -0.5).to(torch.bfloat16)
    H = torch.full_like(Kc, float("nan")).to(DEV)
    kv.kvc_mlp_hidden(kv.make_shape(B, 4, hkv, d, 64, I, m, torch.bfloat16), W1.to(DEV), kv.KVC_ACT_GELU, Kc.to(DEV), H)
    torch.cuda.synchronize()
    assert block_rel_err(f64(H), orc.mlp_hidden(f64(Kc), f64(W1), kv.KVC_ACT_GELU, orc.STORE_BF16)) <= ONE_ROUNDING
