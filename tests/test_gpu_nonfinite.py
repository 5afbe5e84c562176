"""Infinities and NaNs stay where they belong: a non-finite input reaches exactly the results that depend on it.

The calls are compared with themselves on clean inputs (results that do not depend on the non-finite value: bit for
bit) and with the CPU oracle or the scalar kernels (results that do: the same infinities, the same NaNs, and finite
values within the bar of the kernel).
"""
import numpy as np
import pytest
import torch

from paper_2605_16439_amd import kvcapsule as kv

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
                                          ("full", torch.float32, 64), ("text only", torch.bfloat16, 128), ("text only", torch.float32, 64)])
def test_non_finite_query_stays_in_its_own_head(what, dtype, d, bad):
    B, hq, hkv, I, m, t = 3, 14, 2, 2, 41, 70
    I = 0 if what == "text only" else I
    cap = t + 1
    shape = kv.make_shape(B, hq, hkv, d, 100, I, m, dtype)
    mu = torch.full((hkv, d), bad, dtype=dtype, device=DEV)      # text only: a centre that no vision row refers to
    par = [normal(1, hkv, m, 100, dtype=dtype), normal(2, hkv, m, 100, dtype=dtype)]
    params = kv.make_params(torch.arange(m, dtype=torch.int32, device=DEV), *par, mu)
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
