// Decode step with the parameters resident in registers: bf16, head_dim 128, image blocks of 256 tokens (a video's frames),
// compressed lengths up to 128, at most 8 query heads per KV head, packed parameters.
//
// theta and U of a KV head are 2 x 52 KB at m = 103: the eight wavefronts of a workgroup hold both as matrix-core operands (32
// positions of theta and 16 rows of U each), so a workgroup walks tiles of UP image blocks (UP G <= 16 query rows) of one (batch
// element, KV head) through all of Alg. 1 and reads nothing but the blocks' keys and values, each byte once:
//     S = q Kc^T                         (step 1; scores, unscaled, bf16 in LDS)
//     L = sigma S theta, P = exp(L - row maximum), W = P U^T, Y += W Vc      (steps 2 to 4)
// with a running maximum and sum per query row, the next tile's keys requested behind step 1 and its values behind step 4.  A
// workgroup also attends its share of the text rows (walk(), float32 weights) while its first keys are on their way.  One part
// record for the blocks, one for the text; the merge is the other decode paths'.  Scores, weights and W are rounded to bf16
// between the steps, as in the four-kernel form that served these calls.
//
// Bound: HBM, at its rate minus a start of two latencies and the merge.  B = 8, 28/4 heads, 64 blocks, m = 103, 1024 text rows
// (125 MB): 40.5 us in the four-kernel form, 30.8 here (28 in this kernel, 4.5 TB/s); the same at m = 52 28.4 / 20.1.
#include "kvc_rows_dev.h"

#include <algorithm>
#include <atomic>

namespace kvc {

using namespace rows;

namespace {

constexpr int kN = 256;               // positions of an image block
constexpr int kRW = 8;                // wavefronts
constexpr int kMaxKS = 4;             // 32-row steps of the compressed axis

struct RPlan {
    int B, Hq, Hkv, G, I, m;
    int NUT, R, per;                  // tiles of a run, runs per (batch element, KV head), workgroups per XCD
    int t, t_in, cap, rec;
    unsigned qR, qB, qst;
    float scale;
    float *Ypart;
    const int32_t *n_img, *tlen;      // ragged batch: per-sequence counts; I, t and t_in are then the largest
};

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// blocked record ([rows / 8] blocks of [X][w], w = 8 or rows % 8 in the last): where lane (x, kg) finds its operand of the last
// k-step, in bytes, and by how many bytes the 16-byte window is to be shifted
__device__ __forceinline__ uint32_t last_operand(int rows, int X, int x, int kg, int KS, int &sh)
{
    const int nfull = rows >> 3, wt = rows & 7, to = x * 2 * wt, a0 = max(min(to & ~3, X * 2 * wt - 16), 0);
    const int jb = 4 * (KS - 1) + kg;
    const bool mine = wt != 0 && (jb == nfull || nfull == 0);
    sh = mine ? to - a0 : 0;
    return mine ? static_cast<uint32_t>(nfull * 8 * X * 2 + a0) : static_cast<uint32_t>(max(min(jb, nfull - 1), 0) * 8 * X * 2 + x * 16);
}

constexpr size_t resident_lds(int KS)
{
    return std::max(static_cast<size_t>(2 * 16 * (32 * KS + 16) + 16 * (kN + 16)) * 2 + 2 * 16 * kRW * 4 + kRW * 16 * D * 2,
                    static_cast<size_t>(kRW) * (kWalkLds + 2 * 16 * 4));
}

template <int KS, int UP>
__global__ __launch_bounds__(64 * kRW) void fr_pass(const uint16_t *__restrict__ q, const uint16_t *__restrict__ Kc,
                                                    const uint16_t *__restrict__ thp, const uint16_t *__restrict__ Up,
                                                    const uint16_t *__restrict__ Vc, uint16_t *__restrict__ Kt,
                                                    uint16_t *__restrict__ Vt, const uint16_t *__restrict__ k_new,
                                                    const uint16_t *__restrict__ v_new, RPlan p)
{
    constexpr int T = 2 * KS, MP = 32 * KS, LDM = MP + 16, LDP = kN + 16;
    constexpr int NI = UP * T, NR = (NI + kRW - 1) / kRW;        // key tiles of a tile of blocks, rounds over the wavefronts
    constexpr int KP = kN / 32;
    static_assert(KS <= kMaxKS && T <= kRW, "a tile of U per wavefront");
    extern __shared__ __align__(16) uint16_t dyn[];
    uint16_t *sS = dyn, *sW = sS + 16 * LDM, *sP = sW + 16 * LDM;
    float *sRed = reinterpret_cast<float *>(sP + 16 * LDP);      // row maxima [16][kRW], row sums [16][kRW]
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int r16 = lane & 15, kg = lane >> 4;
    char *sTile = reinterpret_cast<char *>(sRed + 2 * 16 * kRW) + wave * (16 * D * 2);       // this wavefront's staging tile

    // an XCD takes a contiguous run of workgroups in (head, batch element, run) order: a head's parameters reach few L2s
    const int id = (blockIdx.x & 7) * p.per + (blockIdx.x >> 3);
    if (id >= p.Hkv * p.B * p.R) return;
    const int hb = quot(id, p.qR), r = id - hb * p.R;
    const int h = quot(hb, p.qB), b = hb - h * p.B, bh = b * p.Hkv + h;
    const int G = p.G, m = p.m;
    int n_img = p.I, t_in = p.t_in, t = p.t;
    const bool fresh = k_new != nullptr;
    if (p.tlen) {
        n_img = min(max(p.n_img[b], 0), p.I);
        const int tlb = max(p.tlen[b], 0);
        t_in = min(tlb, p.t_in);
        t = fresh ? t_in + 1 : min(tlb, p.t);
    }
    u32x4 qf[4];
    {
        const u32x4 *qp = reinterpret_cast<const u32x4 *>(q + (static_cast<size_t>(b) * p.Hq + h * G + min(r16, G - 1)) * D) + kg;
#pragma unroll
        for (int k = 0; k < 4; ++k) qf[k] = qp[4 * k];
    }

    // ---- requests: theta (positions 32 wave + 16 i + r16), the first tile's keys
    const char *th_b = reinterpret_cast<const char *>(thp + static_cast<size_t>(h) * m * kN);
    u32x4 tf[2][KS];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int pos = 32 * wave + 16 * i + r16;
        int sh;
        const uint32_t last = last_operand(m, kN, pos, kg, KS, sh);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            tf[i][ks] = *reinterpret_cast<const u32x4_a4 *>(th_b + (ks < KS - 1 ? static_cast<uint32_t>(((4 * ks + kg) * kN + pos) * 16) : last));
    }
    const int i_lo = r * p.NUT * UP, i_hi = min(i_lo + p.NUT * UP, n_img);        // this run's image blocks
    const char *kc_b = reinterpret_cast<const char *>(Kc + (static_cast<size_t>(bh) * p.I + i_lo) * m * D);
    const char *vc_b = reinterpret_cast<const char *>(Vc + (static_cast<size_t>(bh) * p.I + i_lo) * m * D);
    const int blk = m * D * 2;                                   // bytes of a block
    const int krow = kg, kpc = r16;
    // key tile it of the tile of blocks that starts at i_lo + i0; rows and blocks past the end repeat valid ones
    auto load_k = [&](int i0, int it, u32x4 (&dst)[4]) __attribute__((always_inline)) {
        const int u = it / T, jt = it - u * T;
        const char *tile = kc_b + static_cast<size_t>(max(min(i0 + u, i_hi - i_lo - 1), 0)) * blk + jt * (16 * D * 2);
        const int left = m - 1 - 16 * jt;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            dst[i] = *reinterpret_cast<const u32x4 *>(tile + static_cast<ptrdiff_t>(min(4 * i + krow, left)) * 256 + kpc * 16);
    };
    u32x4 kf[NR][4];
#pragma unroll
    for (int x = 0; x < NR; ++x) load_k(0, min(wave + kRW * x, NI - 1), kf[x]);

    // ---- the run's share of the text rows: 32-row steps r + R (wave + 8 k), so that which run and wavefront a row belongs to
    // does not depend on how many rows there are
    {
        const uint16_t *kn = fresh ? k_new + static_cast<size_t>(bh) * D : q, *vn = fresh ? v_new + static_cast<size_t>(bh) * D : q;
        uint16_t *Ktb = Kt + static_cast<size_t>(bh) * p.cap * D, *Vtb = Vt + static_cast<size_t>(bh) * p.cap * D;
        char *const sw = reinterpret_cast<char *>(dyn);
        float (*sM)[16] = reinterpret_cast<float (*)[16]>(sw + kRW * kWalkLds), (*sL)[16] = sM + kRW;
        float m_t = -INFINITY, l_t = 0.f;
        f32x4 acc[8];
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) acc[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (kSR * r < t) {                                       // the same for the whole workgroup
            Rows rw;
            rw.I = 0; rw.m = 8; rw.KS = 1; rw.SV = 0; rw.qKS = 0; rw.t = t; rw.cs = 1 << 30; rw.ws = p.R; rw.st = kRW * p.R; rw.qst = p.qst;
            rw.scale = p.scale;
            walk<true, 1>(rw, Ktb, Vtb, kn, vn, fresh ? t_in : -1, qf, r, sw + wave * kWalkLds, m_t, l_t, acc);
        }
        merge_waves<kRW>(sw, sM, sL, m_t, l_t, acc, G, p.Ypart + (static_cast<size_t>(bh) * 2 * p.R + p.R + r) * p.rec);
        // Sec. 3.2: the text cache keeps growing as in the backbone -- store the new token's k, v
        const int own = t_in / kSR;
        if (fresh && own - quot(own, p.qR) * p.R == r && threadIdx.x < 32) {
            const int half = threadIdx.x >> 4, piece = threadIdx.x & 15;
            uint16_t *dst = (half ? Vtb : Ktb) + static_cast<size_t>(t_in) * D;
            *(reinterpret_cast<u32x4 *>(dst) + piece) = *(reinterpret_cast<const u32x4 *>(half ? vn : kn) + piece);
        }
    }

    // ---- U (rows 16 wave + r16, all positions), the first tile's values
    const char *u_b = reinterpret_cast<const char *>(Up + static_cast<size_t>(h) * m * kN);
    u32x4 uf[KP];
    {
        const int row = min(16 * wave + r16, m - 1);
#pragma unroll
        for (int ks = 0; ks < KP; ++ks) uf[ks] = *reinterpret_cast<const u32x4 *>(u_b + static_cast<uint32_t>(((4 * ks + kg) * m + row) * 16));
    }
    const int cch = 16 * wave + r16;                             // this lane's channel in step 4
    int vsh;
    const uint32_t v_last = last_operand(m, D, cch, kg, KS, vsh);
    u32x4 vf[KS][UP];
    auto load_v = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < UP; ++u) {
            const char *rec = vc_b + static_cast<size_t>(max(min(i0 + u, i_hi - i_lo - 1), 0)) * blk;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                vf[ks][u] = *reinterpret_cast<const u32x4_a4 *>(rec + (ks < KS - 1 ? static_cast<uint32_t>(((4 * ks + kg) * D + cch) * 16) : v_last));
        }
    };
    load_v(0);
    // theta's last k-step, shifted into place once
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        int sh;
        last_operand(m, kN, 32 * wave + 16 * i + r16, kg, KS, sh);
        tf[i][KS - 1] = shift_window(tf[i][KS - 1], sh >> 2, (sh & 2) * 8u);
    }
    lds_barrier();                                               // the text's LDS is free
    // zeros in the rows of the score tile that no block fills: they feed the matrix cores too
    for (int x = threadIdx.x; x < 16 * LDM / 2; x += 64 * kRW) reinterpret_cast<uint32_t *>(sS)[x] = 0u;
    lds_barrier();

    float m_run = -INFINITY, l_run = 0.f;
    f32x4 y = {0.f, 0.f, 0.f, 0.f};
    const int un = r16 / G;                                      // image block (of the tile) of query row r16
    for (int i0 = 0; i0 < i_hi - i_lo; i0 += UP) {
        const bool more = i0 + UP < i_hi - i_lo;
        // ---- step 1: rows of keys -> operands through this wavefront's staging tile (16-byte piece of row x at piece ^ x)
#pragma unroll
        for (int x = 0; x < NR; ++x) {
            const int it = wave + kRW * x, u = it / T, jt = it - u * T;
            const uint32_t kst = static_cast<uint32_t>(krow * 256 + (kpc ^ krow) * 16);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<u32x4 *>(sTile + (kst ^ static_cast<uint32_t>(i * 64)) + 1024 * i) = kf[x][i];
            f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const bf16x8 ko = *reinterpret_cast<const bf16x8 *>(sTile + r16 * 256 + (((4 * ks + kg) ^ r16) & 15) * 16);
                a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ko, as_bf16x8(qf[ks]), a, 0, 0, 0);
            }
            const int j = 16 * jt + 4 * kg;
            uint32_t w[2];
#pragma unroll
            for (int e = 0; e < 4; e += 2) {
                const uint32_t lo = (j + e < m) ? f32_to_bf16_bits(a[e]) : 0u, hi = (j + e + 1 < m) ? f32_to_bf16_bits(a[e + 1]) : 0u;
                w[e >> 1] = lo | (hi << 16);
            }
            if (r16 < G && it < NI) *reinterpret_cast<u32x2 *>(sS + (u * G + r16) * LDM + j) = u32x2_mk(w[0], w[1]);
        }
        if (more) {
#pragma unroll
            for (int x = 0; x < NR; ++x) load_k(i0 + UP, min(wave + kRW * x, NI - 1), kf[x]);
        }
        lds_barrier();

        // ---- step 2
        f32x4 aL[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 sf = *reinterpret_cast<const bf16x8 *>(sS + r16 * LDM + 32 * ks + 8 * kg);
#pragma unroll
            for (int i = 0; i < 2; ++i) aL[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(tf[i][ks]), sf, aL[i], 0, 0, 0);
        }
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                aL[i][e] *= p.scale;
                mx = fmaxf(mx, aL[i][e]);
            }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        if (kg == 0) sRed[r16 * kRW + wave] = mx;
        lds_barrier();
        {
            const f32x4 a = *reinterpret_cast<const f32x4 *>(sRed + r16 * kRW), c = *reinterpret_cast<const f32x4 *>(sRed + r16 * kRW + 4);
            mx = fmaxf(fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3])), fmaxf(fmaxf(c[0], c[1]), fmaxf(c[2], c[3])));
        }
        float sm = 0.f;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            uint32_t eb[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                eb[e] = f32_to_bf16_bits(__expf(aL[i][e] - mx));
                sm += __uint_as_float(eb[e] << 16);
            }
            *reinterpret_cast<u32x2 *>(sP + r16 * LDP + 32 * wave + 16 * i + 4 * kg) = u32x2_mk(eb[0] | (eb[1] << 16), eb[2] | (eb[3] << 16));
        }
        sm += __shfl_xor(sm, 16, 64);
        sm += __shfl_xor(sm, 32, 64);
        if (kg == 0) sRed[16 * kRW + r16 * kRW + wave] = sm;
        lds_barrier();

        // ---- step 3
        if (wave < T) {                                          // uniform, no loads from memory inside
            f32x4 aw[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int ks = 0; ks < KP; ++ks) {
                const bf16x8 pf = *reinterpret_cast<const bf16x8 *>(sP + r16 * LDP + 32 * ks + 8 * kg);
                aw[ks & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(uf[ks]), pf, aw[ks & 1], 0, 0, 0);
            }
            const int j = 16 * wave + 4 * kg;
            uint32_t w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = j + e < m ? f32_to_bf16_bits(aw[0][e] + aw[1][e]) : 0u;
            *reinterpret_cast<u32x2 *>(sW + r16 * LDM + j) = u32x2_mk(w[0] | (w[1] << 16), w[2] | (w[3] << 16));
        }
        {
            const f32x4 a = *reinterpret_cast<const f32x4 *>(sRed + 16 * kRW + r16 * kRW), c = *reinterpret_cast<const f32x4 *>(sRed + 16 * kRW + r16 * kRW + 4);
            sm = ((a[0] + a[1]) + (a[2] + a[3])) + ((c[0] + c[1]) + (c[2] + c[3]));
        }
        lds_barrier();

        // ---- step 4: wavefront w owns channels 16 w ...; the blocks' products are selected by query row
        f32x4 o[UP];
#pragma unroll
        for (int u = 0; u < UP; ++u) o[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 wf = *reinterpret_cast<const bf16x8 *>(sW + r16 * LDM + 32 * ks + 8 * kg);
#pragma unroll
            for (int u = 0; u < UP; ++u) {
                u32x4 a = vf[ks][u];
                if (ks == KS - 1) a = shift_window(a, vsh >> 2, (vsh & 2) * 8u);
                o[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a), wf, o[u], 0, 0, 0);
            }
        }
        if (more) load_v(i0 + UP);
        if (un < UP && i0 + un < i_hi - i_lo) {                  // rows without a block keep their state
            f32x4 om = o[0];
#pragma unroll
            for (int u = 1; u < UP; ++u)
                if (un == u) om = o[u];
            const float mn = fmaxf(m_run, mx), ca = __expf(m_run - mn), cb = __expf(mx - mn);
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = y[e] * ca + om[e] * cb;
            l_run = l_run * ca + sm * cb;
            m_run = mn;
        }
    }

    // ---- the query heads' rows u G + g into one record
    float gm = -INFINITY;
#pragma unroll
    for (int u = 0; u < UP; ++u) gm = fmaxf(gm, __shfl(m_run, (lane & 48) | min(u * G + r16, 15), 64));
    const float mref = gm == -INFINITY ? 0.f : gm;               // nothing at all (ragged batch): a record without mass
    f32x4 yo = {0.f, 0.f, 0.f, 0.f};
    float lo = 0.f;
#pragma unroll
    for (int u = 0; u < UP; ++u) {
        const int src = (lane & 48) | min(u * G + r16, 15);
        const float w = __expf(__shfl(m_run, src, 64) - mref);
#pragma unroll
        for (int e = 0; e < 4; ++e) yo[e] += w * __shfl(y[e], src, 64);
        lo += w * __shfl(l_run, src, 64);
    }
    if (r16 < G) {
        float *yp = p.Ypart + (static_cast<size_t>(bh) * 2 * p.R + r) * p.rec;
        *reinterpret_cast<f32x4 *>(yp + r16 * D + 16 * wave + 4 * kg) = yo;
        if (wave == 0 && kg == 0) {
            yp[G * D + r16] = gm;
            yp[G * D + G + r16] = lo;
        }
    }
}

constexpr int kTargetRuns = 256;      // workgroups: a compute unit each
std::atomic<long> g_calls{0};         // debug counter (kvc_dev_resident_calls)
int g_mode = -1;                      // developer knob: -1 built-in rule, 0 never, 1 wherever an instance exists

// image blocks of a tile: more than two would not leave registers for the requests in flight beyond m = 64
int blocks_per_tile(int G, int m) { return G <= 4 && m <= 64 ? 4 : 2; }

bool make_rplan(RPlan &p, const DecodeCall &c)
{
    const kvc_shape &s = c.s;
    p.B = s.batch; p.Hq = s.n_q_heads; p.Hkv = s.n_kv_heads; p.G = p.Hq / p.Hkv; p.I = s.n_images; p.m = s.m;
    p.t = c.t; p.t_in = c.t_in; p.cap = c.cap; p.scale = c.scale;
    const long bh = static_cast<long>(p.B) * p.Hkv;
    const int UP = blocks_per_tile(p.G, p.m), tiles = (p.I + UP - 1) / UP;
    // one round of workgroups; at most 32 runs, whose vision and text parts are the 64 lanes of the merge
    p.R = static_cast<int>(std::min<long>(std::min<long>(32, tiles), std::max<long>(1, kTargetRuns / bh)));
    p.NUT = (tiles + p.R - 1) / p.R;
    p.R = (tiles + p.NUT - 1) / p.NUT;
    p.rec = static_cast<int>(align_up(p.G * D + 2 * p.G, 4));
    if (bh * p.R >= 1 << 24) return false;
    const int total = static_cast<int>(bh * p.R);
    p.per = (total + 7) / 8;
    p.qR = quot_multiplier(p.R); p.qB = quot_multiplier(p.B); p.qst = quot_multiplier(kRW * p.R);
    p.n_img = c.n_images_dev; p.tlen = c.text_len_dev;
    p.Ypart = reinterpret_cast<float *>(static_cast<char *>(c.ws) + kCounterBytes);
    // quot(): dividends below 2^32 / divisor
    return static_cast<long>(8) * p.per * std::max(p.R, p.B) < (1l << 31) && static_cast<long>(p.cap + kSR) * kRW * p.R < (1l << 31);
}

template <int KS, int UP> bool launch_r(const RPlan &p, const DecodeCall &c)
{
    static bool attr_set[kMaxDevices] = {};
    constexpr size_t lds = resident_lds(KS);
    if (!allow_lds(reinterpret_cast<const void *>(fr_pass<KS, UP>), lds, attr_set)) return false;
    fr_pass<KS, UP><<<8 * p.per, 64 * kRW, lds, c.stream>>>(
        static_cast<const uint16_t *>(c.q), static_cast<const uint16_t *>(c.Kc), static_cast<const uint16_t *>(c.theta_packed),
        static_cast<const uint16_t *>(c.U_packed), static_cast<const uint16_t *>(c.Vc), static_cast<uint16_t *>(c.Kt),
        static_cast<uint16_t *>(c.Vt), static_cast<const uint16_t *>(c.k_new), static_cast<const uint16_t *>(c.v_new), p);
    return true;
}

template <int UP> bool launch_up(const RPlan &p, const DecodeCall &c)
{
    switch ((p.m + 31) / 32) {
    case 1: return launch_r<1, UP>(p, c);
    case 2: return launch_r<2, UP>(p, c);
    default: break;
    }
    if constexpr (UP == 2) return (p.m + 31) / 32 == 3 ? launch_r<3, UP>(p, c) : launch_r<4, UP>(p, c);
    return false;
}

}  // namespace

void resident_decode_knob(int mode) { g_mode = mode; }
bool resident_decode_default() { return g_mode < 0; }
long resident_decode_calls() { return g_calls.load(); }

bool resident_decode(const DecodeCall &c, kvc_status *st)
{
    const kvc_shape &s = c.s;
    if (g_mode == 0 || c.static_variant || !c.theta_packed || !c.U_packed || s.n_img_tokens != kN || s.m > 32 * kMaxKS || s.n_images < 1 ||
        !fast_decode_supported(s))
        return false;
    if ((c.n_images_dev == nullptr) != (c.text_len_dev == nullptr)) return false;
    RPlan p;
    if (!make_rplan(p, c)) return false;
    const size_t bytes = kCounterBytes + static_cast<size_t>(p.B) * p.Hkv * 2 * p.R * p.rec * sizeof(float);
    if (bytes > c.ws_bytes) return false;
    // Built-in rule, for calls that small_call() in kvc_any_decode.hip leaves: a block for every fourth compute unit, and a text
    // cache that holds no more rows than about twice the compressed ones -- one workgroup, or a few, attend all the text of a
    // (batch element, KV head) here.  us per call, four-kernel form / here: B = 12, 32/32 heads, 4 blocks, m = 24, 1400 text rows
    // 62.4 / 68.4; B = 4, one block, m = 36, 900 rows 21.6 / 21.7; B = 5, 4 blocks, m = 126, 770 rows 29.1 / 25.1; without long
    // texts B = 1, 16/2 heads, 49 blocks, m = 47 14.8 / 10.8; B = 14, 12/2, 16 blocks 13.7 / 10.3; B = 4, 32/32, 5 blocks, m = 112
    // 23.1 / 15.9.
    if (g_mode < 0 && (static_cast<long>(p.B) * p.Hkv * p.I < 64 || p.cap > 2l * p.I * p.m + 128)) return false;
    const bool ok = blocks_per_tile(p.G, p.m) == 4 ? launch_up<4>(p, c) : launch_up<2>(p, c);
    if (ok) ++g_calls;
    *st = ok && hipGetLastError() == hipSuccess
              ? finalize_parts(p.Ypart, 2 * p.R, p.R, p.rec, p.B, p.Hq, p.Hkv, c.mu, c.out, c.lse, c.stream)
              : KVC_ERR_HIP;
    return true;
}

}  // namespace kvc
