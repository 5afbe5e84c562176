"""Infinities and NaNs stay where they belong: a non-finite input reaches exactly the results that depend on it.

The calls are compared with themselves on clean inputs (results that do not depend on the non-finite value: bit for
bit) and with the CPU oracle or the scalar kernels (results that do: the same infinities, the same NaNs, and finite
values within the bar of the kernel).
"""
import numpy as np
import pytest
import torch

from oracle import kvc_oracle as orc
from paper_2605_16439_amd import kvcapsule as kv

from helpers import f64, unpack_vc

pytestmark = pytest.mark.gpu
DEV = "cuda"
NAN, INF = float("nan"), float("inf")


def normal(seed, *size, dtype=torch.bfloat16):
    g = torch.Generator().manual_seed(seed)
    return torch.randn(size, generator=g).to(dtype).to(DEV)


# No vision parts: the centre mu is no part of the result, and what stands in its place (the query tensor, whose first
# H_kv rows a merge kernel would read as mu) must not reach other sequences or heads.
@pytest.mark.parametrize("bad", [NAN, INF])
@pytest.mark.parametrize("what,dtype,d", [("static", torch.bfloat16, 128), ("static", torch.float32, 64), ("full", torch.bfloat16, 128),
                                          ("full", torch.float32, 64), ("text only", torch.bfloat16, 128), ("text only", torch.float32, 64),
                                          ("decode", torch.bfloat16, 128), ("decode", torch.float32, 64), ("tuned", torch.bfloat16, 128),
                                          ("packed", torch.bfloat16, 128)])
def test_non_finite_query_stays_in_its_own_head(what, dtype, d, bad):
    B, hq, hkv, I, m, t = 3, 14, 2, 2, 41, 70
    I = 0 if what == "text only" else I
    cap = t + 1
    n = 256 if what in ("tuned", "packed") else 100
    shape = kv.make_shape(B, hq, hkv, d, n, I, m, dtype)
    # text only: a centre that no vision row refers to
    mu = torch.full((hkv, d), bad if what == "text only" else 0.5, dtype=dtype, device=DEV)
    par = [normal(1, hkv, m, n, dtype=dtype), normal(2, hkv, m, n, dtype=dtype)]
    packed = [kv.kvc_pack_theta(shape, par[0]), kv.kvc_pack_u(shape, par[1])] if what == "packed" else []
    params = kv.make_params(torch.arange(m, dtype=torch.int32, device=DEV), *par, mu, *packed)
    Kc, Vc = normal(3, B, hkv, max(I, 1), m, d, dtype=dtype), normal(4, B, hkv, max(I, 1), m, d, dtype=dtype)
    kn, vn = normal(5, B, hkv, d, dtype=dtype), normal(6, B, hkv, d, dtype=dtype)
    if what == "full":
        ws = torch.empty(kv.kvc_attend_full_workspace_bytes(B, hq, hkv, d, dtype, cap) + 256, dtype=torch.uint8, device=DEV)
    else:
        ws = kv.new_workspace(shape, cap)

    def run(q):
        Kt, Vt = normal(7, B, hkv, cap, d, dtype=dtype), normal(8, B, hkv, cap, d, dtype=dtype)
        out, lse = torch.full((B, hq, d), 7.0, dtype=dtype, device=DEV), torch.zeros((B, hq), dtype=torch.float32, device=DEV)
        if what == "static":
            kv.kvc_static_attend_decode(shape, q, Kc, Vc, Kt, Vt, t, cap, kn, vn, 0.0, out, lse, ws)
        elif what == "full":
            kv.kvc_attend_full_decode(q, Kt, Vt, t, kn, vn, 0.0, out, lse, ws)
        else:
            kv.kvc_reconstruct_attend_decode(shape, params, q, Kc, Vc, Kt, Vt, t, cap, kn, vn, 0.0, out, lse, ws)
        torch.cuda.synchronize()
        return out.float().cpu(), lse.cpu()

    q = normal(9, B, hq, d, dtype=dtype)
    print(f"[nonfinite] {what} {dtype} d={d} {bad}", flush=True)
    clean, clean_lse = run(q)
    assert torch.isfinite(clean).all() and torch.isfinite(clean_lse).all()
    q[0, 0, 5] = q[0, 1, 3] = bad
    out, lse = run(q)
    assert not torch.isfinite(out[0, :2]).any()
    keep = torch.ones((B, hq), dtype=torch.bool)
    keep[0, :2] = False
    assert torch.equal(out[keep], clean[keep]) and torch.equal(lse[keep], clean_lse[keep])


def check_same_kind(got, ref, bar):
    """The same NaNs and infinities; finite values within `bar` of the reference's norm, per row of the last axis."""
    assert np.array_equal(np.isnan(got), np.isnan(ref)), (np.isnan(got).sum(), np.isnan(ref).sum())
    assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and np.array_equal(np.isneginf(got), np.isneginf(ref))
    fin = np.isfinite(ref)
    g, r = np.where(fin, got, 0.0), np.where(fin, ref, 0.0)
    e = np.linalg.norm(g - r, axis=-1) / np.maximum(np.linalg.norm(r, axis=-1), 1e-30)
    assert e.max() <= bar, e.max()


# Rows past the end of a block fill the last tile of positions: they are zeros, not the last row again, whose infinity
# would meet the zeros of U or W1.  n and m around the tiles of 64 (bf16, d = 128) and 16 (fp32) positions.
@pytest.mark.parametrize("n,m,dtype,d", [(65, 33, torch.bfloat16, 128), (71, 20, torch.bfloat16, 128), (126, 126, torch.bfloat16, 128),
                                         (729, 292, torch.bfloat16, 128), (64, 20, torch.bfloat16, 128), (9, 4, torch.bfloat16, 128),
                                         (65, 33, torch.float32, 64), (30, 7, torch.float32, 128), (100, 40, torch.bfloat16, 72)])
def test_infinite_value_rows_of_compress(n, m, dtype, d):
    B, hkv, I, pre = 1, 2, 3, 5
    shape = kv.make_shape(B, 4, hkv, d, n, I, m, dtype)
    idx = torch.arange(m, dtype=torch.int32, device=DEV)
    U, mu = normal(1, hkv, m, n, dtype=dtype) * n ** -0.5, normal(2, hkv, d, dtype=dtype)
    K, V = normal(3, B, hkv, pre + I * n + 2, d, dtype=dtype), normal(4, B, hkv, pre + I * n + 2, d, dtype=dtype)
    V[0, 0, pre + n - 1, 3] = INF               # last row of the first block
    V[0, 0, pre + n - 1, 4] = -INF
    V[0, 1, pre + 3 * n - 1, 7] = INF           # last row of the last block
    V[0, 1, pre + 3 * n - 1, 8] = NAN
    V[0, 1, pre + n, 9] = INF                   # first row of the second block
    V[0, 1, pre + 3 * n, 10] = NAN              # behind the last block: nobody's
    Kc, Vc = (torch.zeros((B, hkv, I, m, d), dtype=dtype, device=DEV) for _ in range(2))
    print(f"[nonfinite] compress n={n} m={m} {dtype} d={d}", flush=True)
    kv.kvc_compress(shape, kv.make_params(idx, U, U, mu), K, V, pre, Kc, Vc, kv.new_workspace(shape, 1))
    torch.cuda.synchronize()
    code = orc.STORE_F32 if dtype == torch.float32 else orc.STORE_BF16
    Kc_ref, Vc_ref = orc.compress(f64(K), f64(V), idx.cpu().numpy(), f64(U), f64(mu), n, I, pre, code)
    assert np.array_equal(f64(Kc), Kc_ref)
    check_same_kind(unpack_vc(Vc, m, d), Vc_ref, 1e-5 if dtype == torch.float32 else 3e-3)


@pytest.mark.parametrize("act", [kv.KVC_ACT_IDENTITY, kv.KVC_ACT_RELU, kv.KVC_ACT_GELU])
@pytest.mark.parametrize("m", [9, 63, 64, 65, 103, 410])
def test_infinite_key_rows_of_the_hidden_layer(m, act):
    B, hkv, I, d = 1, 2, 2, 128
    Kc, W1 = normal(5, B, hkv, I, m, d), normal(6, hkv, m, m) * m ** -0.5
    Kc[0, 0, 0, m - 1, 3], Kc[0, 0, 0, m - 1, 4], Kc[0, 1, 1, m - 1, 5], Kc[0, 1, 0, 0, 6] = INF, -INF, NAN, INF
    H = torch.zeros_like(Kc)
    print(f"[nonfinite] hidden m={m} act={act}", flush=True)
    kv.kvc_mlp_hidden(kv.make_shape(B, 4, hkv, d, 1024, I, m, torch.bfloat16), W1, act, Kc, H)
    torch.cuda.synchronize()
    check_same_kind(f64(H), orc.mlp_hidden(f64(Kc), f64(W1), act, orc.STORE_BF16), 3e-3)


# Infinite values reach their own channel of their own (sequence, KV head) only.  Text values and the rows of the static
# variant, whose weights are positive, stay infinities; a compressed value's weights have either sign in the parts that a
# decode kernel adds up, so its channel is infinite or NaN there.  m around the blocks of 8 rows and the steps of 16 and 32,
# several image blocks per tile, text around the step of 128.
def poisoned(dtype, d, B, hkv, I, m, t):
    Kc, Vc = normal(11, B, hkv, max(I, 1), m, d, dtype=dtype), normal(12, B, hkv, max(I, 1), m, d, dtype=dtype)
    Kt, Vt = normal(13, B, hkv, t + 1, d, dtype=dtype), normal(14, B, hkv, t + 1, d, dtype=dtype)
    vc = lambda j, c: kv.lib().kvc_capsule_value_offset(j, c, m, d)
    flat = Vc.view(B, hkv, max(I, 1), m * d)
    if I > 0:
        flat[0, 0, I - 1, vc(m - 1, 3)] = INF                # last row of the last block
        flat[0, 0, 0, vc(0, 7)] = -INF                       # first row of the first one
        flat[B - 1, hkv - 1, I // 2, vc(m // 2, 12)] = INF
        flat[B - 1, hkv - 1, I // 2, vc(m - 1, 20)] = NAN
    kn, vn = normal(15, B, hkv, d, dtype=dtype), normal(16, B, hkv, d, dtype=dtype)
    if t > 0:
        Vt[0, 0, t - 1, 30] = INF                            # last row but the new one
        Vt[B - 1, hkv - 1, 0, 31] = -INF
    vn[0, 0, 40] = INF                                       # the new row, which the rows past the end repeat
    return Kc, Vc, Kt, Vt, kn, vn


@pytest.mark.parametrize("hq,hkv,B,I,n,m,t,dtype,d,packed", [
    (14, 2, 2, 5, 130, 41, 70, torch.bfloat16, 128, False), (8, 8, 1, 3, 136, 64, 128, torch.bfloat16, 128, True), (7, 1, 1, 2, 9, 5, 3, torch.bfloat16, 128, False),
    (4, 1, 1, 9, 600, 33, 300, torch.bfloat16, 128, False), (28, 4, 1, 2, 256, 103, 200, torch.bfloat16, 128, True), (14, 2, 1, 33, 200, 40, 9, torch.bfloat16, 128, False),
    (2, 2, 2, 0, 50, 20, 260, torch.bfloat16, 128, False), (14, 2, 2, 5, 130, 41, 70, torch.float32, 64, False), (8, 2, 1, 3, 300, 33, 127, torch.float32, 128, False),
    (16, 2, 1, 2, 65, 16, 130, torch.bfloat16, 72, False), (4, 4, 1, 2, 40, 7, 0, torch.float32, 256, False)])
def test_infinite_values_in_decode(hq, hkv, B, I, n, m, t, dtype, d, packed):
    shape = kv.make_shape(B, hq, hkv, d, n, I, m, dtype)
    U = normal(17, hkv, m, n, dtype=dtype) * n ** -0.5
    par = [torch.arange(m, dtype=torch.int32, device=DEV), normal(18, hkv, m, n, dtype=dtype) * m ** -0.5, U, normal(19, hkv, d, dtype=dtype)]
    if packed:
        par += [kv.kvc_pack_theta(shape, par[1]), kv.kvc_pack_u(shape, U)]
    params, q, ws = kv.make_params(*par), normal(20, B, hq, d, dtype=dtype) * 0.25, kv.new_workspace(shape, t + 1)
    res = []
    for generic in (False, True):
        Kc, Vc, Kt, Vt, kn, vn = poisoned(dtype, d, B, hkv, I, m, t)
        out = torch.zeros((B, hq, d), dtype=dtype, device=DEV)
        print(f"[nonfinite] decode {hq}/{hkv} B={B} I={I} n={n} m={m} t={t} {dtype} d={d} generic={generic}", flush=True)
        kv.kvc_reconstruct_attend_decode(shape, params, q, Kc, Vc, Kt, Vt, t, t + 1, kn, vn, 0.0, out, None, ws, generic=generic)
        torch.cuda.synchronize()
        res.append(f64(out))
    assert not np.isfinite(res[1]).all()
    vision = [3, 7, 12, 20] if I > 0 else []
    assert np.array_equal(np.isfinite(res[0]), np.isfinite(res[1]))
    rest = [c for c in range(d) if c not in vision]
    check_same_kind(res[0][..., rest], res[1][..., rest], 1e-5 if dtype == torch.float32 else 2 * (2.0 ** -8 + 1e-4))


@pytest.mark.parametrize("hq,hkv,B,I,m,t", [(14, 2, 2, 5, 41, 70), (7, 1, 1, 2, 7, 1), (8, 8, 1, 3, 64, 128), (28, 4, 1, 64, 103, 40), (6, 2, 1, 3, 8, 127),
                                            (2, 2, 1, 0, 20, 260)])
def test_infinite_values_in_the_static_variant(hq, hkv, B, I, m, t):
    d, dtype = 128, torch.bfloat16
    shape = kv.make_shape(B, hq, hkv, d, max(m, 64), I, m, dtype)
    q = normal(21, B, hq, d) * 0.25
    Kc, Vc, Kt, Vt, kn, vn = poisoned(dtype, d, B, hkv, I, m, t)
    out = torch.zeros((B, hq, d), dtype=dtype, device=DEV)
    dense, Kth, Vth = unpack_vc(Vc, m, d)[:, :, :I], f64(Kt).copy(), f64(Vt).copy()
    print(f"[nonfinite] static {hq}/{hkv} B={B} I={I} m={m} t={t}", flush=True)
    kv.kvc_static_attend_decode(shape, q, Kc, Vc, Kt, Vt, t, t + 1, kn, vn, 0.0, out, None, kv.new_workspace(shape, t + 1))
    torch.cuda.synchronize()
    ref, _ = orc.static_attend_decode(f64(q), f64(Kc)[:, :, :I], dense, Kth, Vth, t, f64(kn), f64(vn))
    assert not np.isfinite(ref).all()
    check_same_kind(f64(out), ref, 2.0 ** -8 + 1e-4)
