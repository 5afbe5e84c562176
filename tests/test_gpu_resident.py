"""The decode kernel that keeps theta and U in registers (n = 256, packed parameters, m <= 128) against the CPU oracle through the
C ABI, forced by kvc_dev_resident_decode(1) so that small shapes take it too.  Bars as in tests/test_gpu_parity.py (bf16)."""
import numpy as np
import pytest
import torch

from oracle import kvc_oracle as orc
from paper_2605_16439_amd import kvcapsule as kv
from paper_2605_16439_amd import synth

from helpers import elem_rel_err, f64, row_rel_err, tol, unpack_vc
from test_gpu_parity import DEV
from test_gpu_stream import _packed_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _force():
    kv.lib().kvc_dev_resident_decode(1)
    yield
    kv.lib().kvc_dev_resident_decode(-1)


def wl(I, t, B=2, hq=14, hkv=2, steps=1):
    return synth.Workload("res", 95, 1, B, hq, hkv, 128, "bf16", 256, I, 0.6, t, steps)


def run(w, m, ragged=None, append=True, lse_tol=5e-2):
    """One step against the oracle; a ragged batch with NaNs wherever a sequence has nothing."""
    L = _packed_layer(w, m)
    L.ws.fill_(0xFF)
    gKc, gVc = L.gKc.clone(), L.gVc.clone()
    Kc_h, Vc_h = f64(gKc), unpack_vc(gVc, m, 128)
    n_images, text_len = ragged or ([w.n_images] * w.batch, [w.text_len] * w.batch)
    Kt, Vt = f64(L.Kt).copy(), f64(L.Vt).copy()
    for b in range(w.batch):
        rows = text_len[b] + (1 if append else 0)
        gKc[b, :, n_images[b]:] = float("nan")
        gVc[b, :, n_images[b]:] = float("nan")
        L.gKt[b, :, rows:] = float("nan")
        L.gVt[b, :, rows:] = float("nan")
    q, kn, vn = synth.make_step_inputs(w, 0, 0)
    new = (kn.to(DEV), vn.to(DEV)) if append else (None, None)
    taken = kv.lib().kvc_dev_resident_calls()
    if ragged:
        ni, tl = (torch.tensor(x, dtype=torch.int32, device=DEV) for x in ragged)
        kv.kvc_reconstruct_attend_decode_ragged(L.shape, L.params, q.to(DEV), gKc, gVc, L.gKt, L.gVt, ni, tl, w.text_cap, *new, 0.0,
                                                L.out, L.lse, L.ws)
    else:
        kv.kvc_reconstruct_attend_decode(L.shape, L.params, q.to(DEV), gKc, gVc, L.gKt, L.gVt, w.text_len, w.text_cap, *new, 0.0,
                                         L.out, L.lse, L.ws)
    torch.cuda.synchronize()
    assert kv.lib().kvc_dev_resident_calls() == taken + 1
    ref, lref = orc.reconstruct_attend_decode_ragged(f64(q), Kc_h, Vc_h, f64(L.p["theta"]), f64(L.p["U"]), f64(L.p["mu"]), 256,
                                                     n_images, text_len, Kt, Vt, f64(kn) if append else None,
                                                     f64(vn) if append else None)
    out, lse = f64(L.out), f64(L.lse)
    e, ex, el = row_rel_err(out, ref), elem_rel_err(out, ref), np.abs(lse - lref).max()
    print(f"[resident] m={m} {w}: row {e:.3e} element {ex:.3e} lse {el:.3e}", flush=True)
    assert np.all(np.isfinite(out)) and e <= tol(w) and ex <= 4 * tol(w) and el <= lse_tol
    if append:
        for b in range(w.batch):
            assert np.array_equal(f64(L.gKt)[b, :, text_len[b]], f64(kn)[b])
            assert np.array_equal(f64(L.gVt)[b, :, text_len[b]], f64(vn)[b])
    return out, lse


# every number of 32-row steps, with and without a short last block of 8 rows, a last 16-row tile that is missing
@pytest.mark.parametrize("m", [1, 7, 8, 9, 16, 31, 32, 33, 63, 64, 65, 90, 96, 97, 103, 127, 128])
def test_compressed_lengths(m):
    run(wl(5, 40), m, lse_tol=5e-2 if m > 8 else 2e-1)       # (few rows: logits of +-30 carry one rounded score each)


# one and two tiles of blocks per run and a last tile that is not full; 4 blocks per tile up to 4 heads and m = 64, else 2
@pytest.mark.parametrize("hq,hkv,m", [(2, 2, 60), (4, 2, 64), (8, 2, 33), (8, 2, 70), (12, 2, 40), (14, 2, 103), (16, 2, 128)])
@pytest.mark.parametrize("I", [1, 2, 3, 9])
def test_group_sizes_and_tiles(hq, hkv, m, I):
    run(wl(I, 17, hq=hq, hkv=hkv), m)


def test_many_tiles_per_workgroup():
    run(wl(70, 300, B=1), 103)
    run(wl(37, 30, B=20), 52)


@pytest.mark.parametrize("t,append", [(0, True), (0, False), (1, False), (31, True), (32, True), (33, False), (255, True), (256, True),
                                      (700, True)])
def test_text_lengths(t, append):
    run(wl(3, t), 50, append=append)


@pytest.mark.parametrize("n_images,text_len", [([9, 0, 1, 4], [300, 0, 129, 17]), ([0, 5, 9, 2], [31, 302, 0, 64])])
@pytest.mark.parametrize("m", [41, 103])
def test_ragged_batch(n_images, text_len, m):
    run(wl(9, 302, B=4), m, ragged=(n_images, text_len))


def test_ragged_uniform_batch_equals_the_uniform_call():
    w = wl(11, 200)
    a, la = run(w, 103)
    b, lb = run(w, 103, ragged=([11, 11], [200, 200]))
    assert np.array_equal(a, b) and np.array_equal(la, lb)


def test_rule_and_small_workspace():
    """Without the knob: many blocks take this kernel, few blocks or a long text cache do not, and neither does a workspace that
    only the other kernels' needs fill."""
    kv.lib().kvc_dev_resident_decode(-1)
    for w, m, takes in ((wl(80, 100, B=1), 103, 1), (wl(80, 100, B=1), 140, 0), (wl(40, 9000, B=4), 40, 0), (wl(3, 10, B=1), 103, 0)):
        L = _packed_layer(w, m)
        q, kn, vn = synth.make_step_inputs(w, 0, 0)
        taken = kv.lib().kvc_dev_resident_calls()
        L.decode(q.to(DEV), w.text_len, kn.to(DEV), vn.to(DEV))
        assert kv.lib().kvc_dev_resident_calls() == taken + takes


def test_replayed_from_a_hip_graph():
    w = wl(9, 90)
    L = _packed_layer(w, 103)
    q, kn, vn = synth.make_step_inputs(w, 0, 0)
    gq, gkn, gvn = q.to(DEV), kn.to(DEV), vn.to(DEV)
    eager, _ = L.decode(gq, w.text_len, gkn, gvn)
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            kv.kvc_reconstruct_attend_decode(L.shape, L.params, gq, L.gKc, L.gVc, L.gKt, L.gVt, w.text_len, w.text_cap, gkn, gvn, 0.0,
                                             L.out, L.lse, L.ws, stream=s)
    for rep in range(3):
        L.out.zero_()
        L.ws.fill_(0x5A)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(f64(L.out), eager), f"replay {rep}"
