// Static variant (the paper's ablation without reconstruction, "Static Compression vs.
// Reconstruction-before-Attention") on the matrix cores of gfx950: bf16 storage, head_dim 128, at most 16 query
// heads per KV head.  One new query token attends the I m compressed rows and the t text rows as they are:
//
//   static_split   one workgroup per (batch element, KV head, run of rows); a run lies in the compressed rows or
//                  in the text rows.  Each of its four wavefronts takes every fourth 32-row step of the run with
//                  an online softmax of its own and the four merge through LDS into one part record.
//   finalize       the merge kernel of the other decode paths (a lane per part).
//
// Bound: HBM, 2 B H_kv (I m + t) d 2 bytes read once.  What the layout gives for free: the compressed values are
// stored as 16-byte pieces of 8 consecutive rows of one channel, which is the operand of P V when a lane holds
// the probabilities of 8 consecutive rows -- so the rows of a score tile are numbered such that it does (tile tt
// of a step, row i: key row 8 (i / 4) + 4 tt + i % 4), and values go from memory into the matrix cores without
// LDS.  Text values are row-major and are transposed by the reads of a wavefront-private LDS tile.
//
// The weights are not rounded to bf16: p = p1 + p2 + p3 with three bf16 terms (24 bits, what a float holds), one
// matrix instruction each; the matrix cores idle otherwise (32 instructions of 16 cycles per 16 KB and
// wavefront: 20 times the rate at which memory delivers).
//
// Headline capsule (B = 4, 28 / 4 heads, 8 blocks of m = 410, 513 text rows, 31 MB): 595 us on the scalar
// kernels (output kernel 472 us: a workgroup per query head), 11.0 us here -- this kernel 8 to 9 us, the merge 2 to 3
// (15.0 us while every wavefront also requested the step behind its run; runs of two steps instead of one 13.3; 12.0 while the
// text values were packed into pairs of rows on their way to LDS).
#include "kvc_rows_dev.h"

#include <algorithm>

namespace kvc {

using namespace rows;

namespace {

struct StPlan : Rows {
    int Hq, Hkv, G;
    int NV, NP;                       // runs of compressed rows, all runs
    int t_in, cap, rec;
    unsigned qNP, qHkv;
    float *Ypart;
};

__global__ __launch_bounds__(64 * kSW, 2) void static_split(const uint16_t *__restrict__ q, const uint16_t *__restrict__ Kc,
                                                         const uint16_t *__restrict__ Vc, uint16_t *__restrict__ Kt,
                                                         uint16_t *__restrict__ Vt, const uint16_t *__restrict__ k_new,
                                                         const uint16_t *__restrict__ v_new, StPlan p)
{
    __shared__ __align__(256) char sVt[kSW * kWalkLds];
    __shared__ float sM[kSW][16], sL[kSW][16];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r16 = lane & 15, kg = lane >> 4;
    const int bh = quot(blockIdx.x, p.qNP), pt = blockIdx.x - bh * p.NP;
    const int b = quot(bh, p.qHkv), h = bh - b * p.Hkv;
    u32x4 qf[4];
    {
        const u32x4 *qp = reinterpret_cast<const u32x4 *>(q + (static_cast<size_t>(b) * p.Hq + h * p.G + min(r16, p.G - 1)) * D) + kg;
#pragma unroll
        for (int k = 0; k < 4; ++k) qf[k] = qp[4 * k];
    }
    const bool fresh = k_new != nullptr;
    const uint16_t *kn = fresh ? k_new + static_cast<size_t>(bh) * D : q, *vn = fresh ? v_new + static_cast<size_t>(bh) * D : q;
    uint16_t *Ktb = Kt + static_cast<size_t>(bh) * p.cap * D, *Vtb = Vt + static_cast<size_t>(bh) * p.cap * D;

    // online softmax state of head r16 (columns beyond the group repeat head G - 1), the same in the four
    // lanes kg of a head except for the partial sum
    float m_run = -INFINITY, l_run = 0.f;
    f32x4 acc[8];
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) acc[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bool text = pt >= p.NV;
    const int s0 = (text ? pt - p.NV : pt) * p.cs * kSW;
    if (text)
        walk<true>(p, Ktb, Vtb, kn, vn, fresh ? p.t_in : -1, qf, s0, sVt + wave * kWalkLds, m_run, l_run, acc);
    else
        walk<false>(p, Kc + static_cast<size_t>(bh) * p.I * p.m * D, Vc + static_cast<size_t>(bh) * p.I * p.m * D, kn, vn, -1, qf, s0,
                    sVt + wave * kWalkLds, m_run, l_run, acc);

    merge_waves<kSW>(sVt, sM, sL, m_run, l_run, acc, p.G, p.Ypart + (static_cast<size_t>(bh) * p.NP + pt) * p.rec);
    // the cache grows as in the backbone: the run that owns row t_in stores the new token
    if (fresh && text && p.t_in >= kSR * s0 && p.t_in < kSR * (s0 + kSW * p.cs) && threadIdx.x < 32) {
        const int half = threadIdx.x >> 4, piece = threadIdx.x & 15;
        uint16_t *dst = (half ? Vtb : Ktb) + static_cast<size_t>(p.t_in) * D;
        *(reinterpret_cast<u32x4 *>(dst) + piece) = *(reinterpret_cast<const u32x4 *>(half ? vn : kn) + piece);
    }
}

constexpr int kTargetWg = 512;        // two workgroups per compute unit

bool make_st_plan(StPlan &p, const kvc_shape &s, int t, int t_in, int cap)
{
    p.Hq = s.n_q_heads; p.Hkv = s.n_kv_heads; p.G = p.Hq / p.Hkv;
    p.I = s.n_images; p.m = s.m; p.KS = (s.m + kSR - 1) / kSR;
    p.t = t; p.t_in = t_in; p.cap = cap;
    if (static_cast<long>(p.I) * p.KS > (1 << 24)) return false;
    p.SV = p.I * p.KS;
    const long bh = static_cast<long>(s.batch) * p.Hkv;
    const int wv = (p.SV + kSW - 1) / kSW, wt = (t + kSR * kSW - 1) / (kSR * kSW);      // steps of a whole workgroup
    // runs as long as they have to be for about two workgroups per compute unit, and at most 64 parts per
    // (batch element, KV head), one lane each in the merge
    const int want = static_cast<int>(std::max(1L, kTargetWg / bh));
    p.cs = std::max(1, (wv + wt + want - 1) / want);
    while ((wv + p.cs - 1) / p.cs + (wt + p.cs - 1) / p.cs > 64) ++p.cs;
    p.NV = (wv + p.cs - 1) / p.cs;
    p.NP = p.NV + (wt + p.cs - 1) / p.cs;
    p.rec = static_cast<int>(align_up(p.G * D + 2 * p.G, 4));
    p.ws = 1; p.st = kSW; p.qst = quot_multiplier(kSW);
    p.qNP = quot_multiplier(p.NP); p.qHkv = quot_multiplier(p.Hkv); p.qKS = quot_multiplier(p.KS);
    // quot(): dividends below 2^32 / divisor
    return p.NP > 0 && bh * p.NP * std::max(p.NP, p.Hkv) < (1ll << 32) && static_cast<long>(p.SV) * p.KS < (1ll << 32);
}

}  // namespace

bool fast_static_supported(const kvc_shape &s)
{
    return s.dtype == KVC_BF16 && s.head_dim == D && s.n_q_heads / s.n_kv_heads <= 16;
}

// parts: at most the target number of workgroups and two more per (batch element, KV head)
size_t fast_static_ws_bytes(const kvc_shape &s)
{
    const int G = s.n_q_heads / s.n_kv_heads;
    const size_t bh = static_cast<size_t>(s.batch) * s.n_kv_heads;
    return kCounterBytes + (kTargetWg + 2 * bh) * align_up(G * D + 2 * G, 4) * sizeof(float);
}

kvc_status fast_static_decode(const DecodeCall &c)
{
    StPlan p;
    if (!make_st_plan(p, c.s, c.t, c.t_in, c.cap)) return generic_decode(c);
    if (fast_static_ws_bytes(c.s) > c.ws_bytes) return generic_decode(c);
    p.scale = c.scale;
    p.Ypart = reinterpret_cast<float *>(static_cast<char *>(c.ws) + kCounterBytes);
    static_split<<<c.s.batch * p.Hkv * p.NP, 64 * kSW, 0, c.stream>>>(
        static_cast<const uint16_t *>(c.q), static_cast<const uint16_t *>(c.Kc), static_cast<const uint16_t *>(c.Vc),
        static_cast<uint16_t *>(c.Kt), static_cast<uint16_t *>(c.Vt), static_cast<const uint16_t *>(c.k_new),
        static_cast<const uint16_t *>(c.v_new), p);
    if (hipGetLastError() != hipSuccess) return KVC_ERR_HIP;
    // no vision parts: mu is not read (q stands in for it)
    return finalize_parts(p.Ypart, p.NP, 0, p.rec, c.s.batch, p.Hq, p.Hkv, c.q, c.out, c.lse, c.stream);
}

}  // namespace kvc
