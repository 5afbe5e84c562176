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

from helpers import block_rel_err, f64, store_code, unpack_vc
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
