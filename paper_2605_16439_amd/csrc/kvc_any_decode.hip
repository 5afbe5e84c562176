// Decode step for the shapes that the tuned kernels are not compiled for, and for small calls of the others
// (small_call): bf16 storage, head_dim 128, 8 to 6144 tokens per image block (48 slices of 128), compressed lengths up to
// 1152 (LDS), at most 16 query heads per KV head.  One launch in the score-space order of Alg. 1, then the merge of the
// part records:
//
//   ga_pass   a vision workgroup owns a slice of PS positions of one (batch element, KV head) and walks tiles of
//             UP image blocks (UP G <= 16 query rows, one matrix-core tile):
//                 S = q Kc^T                (step 1, every slice computes all of it: no hand-over)
//                 L = sigma S theta[:, slice], P = exp(L - slice max)      (step 2)
//                 W = P U[:, slice]^T       (step 3, this slice's part of the sum over positions)
//                 Y += W Vc                 (step 4; by linearity the slices may be multiplied separately)
//             with a running maximum and sum per query row, and writes one part record.  Text workgroups behind
//             them attend 128 rows of the text cache per step.
//
// Precision is that of the scalar kernels, which these shapes ran before: scores, weights and W are float32.  In
// front of the matrix cores a float is three bf16 terms (exact), one instruction each; the other operand is bf16
// already.  The matrix cores have that to spare: 3 x 0.4 GFLOP per layer at the shape below.
//
// What bounds it: like fs_stream (kvc_stream_decode.hip) the latency of the four dependent phases for a few
// workgroups, and for many the bytes pulled through the L1s -- every slice reads the blocks' keys and values, and
// every tile of rows its slices of theta and U.  So a slice is as wide as leaves a workgroup per compute unit
// (make_gplan).  theta and U come in the packed forms where the caller has them (PK); from the plain form both are read
// in 16-byte pieces of rows at element alignment (at odd n rows start at odd elements).  theta's rows are the contraction
// index: its pieces are turned into operands in registers, 8 rows by 8 positions per lane; U's through LDS.
//
// n = 729, m = 292, 3 blocks, B = 1, 28/4 heads, 201 text rows: 205 us per layer on the scalar
// kernels (six launches; their output step alone 135 us), 16.3 us here -- 14.0 us in this kernel at best, 14.9 on average
// (kernel trace; keys, theta, softmax, U and values about 3 : 1.5 : 1.5 : 2 : 2), the rest the merge.
#include "kvc_rows_dev.h"

#include <algorithm>
#include <atomic>

namespace kvc {

using namespace rows;

namespace {

typedef u32x4 u32x4_a2 __attribute__((aligned(2)));     // a 16-byte access at an element-aligned address

constexpr int kGW = 8;                // wavefronts
constexpr int kMaxVisParts = 48, kMaxTextParts = 16;   // part records per (batch element, KV head): a lane each in the merge
constexpr int kTextStep = kSR * kSW;  // text rows of a workgroup's step

struct GPlan {
    int B, Hq, Hkv, G, I, n, m, KS;
    int PS, UP, NUT, NUG, F;          // positions per slice, image blocks per tile, tiles per workgroup, unit groups per sequence, slices
    int NGR, chunk, nvis;             // (head, sequence, unit group) groups, groups per XCD, vision workgroups
    int NTX, NTC, nparts, rec;        // text runs per (batch element, KV head), those of a cache filled to its capacity:
                                      // run r takes the steps r, r + NTC, r + 2 NTC, ...
    int own;                          // plain theta: the partial logits have LDS of their own
    int t, t_in, cap;
    unsigned qF, qBU, qNUG, qT, qNTX, qHkv, qKS, qNTC, qst;
    float scale;
    float *Ypart;
    const int32_t *n_img, *tlen;      // ragged batch (RAG): per-sequence counts; I, t and t_in are then the largest
#if defined(KVC_TIMELINE)
    unsigned long long *tl;           // timeline slots, see TS()
#endif
};

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// four consecutive values of a row of an LDS matrix in three planes of bf16 terms
__device__ __forceinline__ void store_planes(uint16_t *dst, int plane, const float (&x)[4])
{
    float r[4] = {x[0], x[1], x[2], x[3]};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        uint32_t b[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            b[e] = f32_to_bf16_bits(r[e]);
            r[e] -= __uint_as_float(b[e] << 16);
        }
        *reinterpret_cast<u32x2 *>(dst + k * plane) = u32x2_mk(b[0] | (b[1] << 16), b[2] | (b[3] << 16));
    }
}

// acc += A (b1 + b2 + b3), the small terms first
__device__ __forceinline__ f32x4 mfma3(bf16x8 a, const bf16x8 (&b)[3], f32x4 acc)
{
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[2], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[1], acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[0], acc, 0, 0, 0);
}
// the same with an accumulator per term: three short dependency chains where a wavefront has one tile only
struct Acc3 {
    f32x4 v[3];
    __device__ __forceinline__ Acc3()
    {
#pragma unroll
        for (int k = 0; k < 3; ++k) v[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void add(bf16x8 a, const bf16x8 (&b)[3])
    {
#pragma unroll
        for (int k = 0; k < 3; ++k) v[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[k], v[k], 0, 0, 0);
    }
    __device__ __forceinline__ f32x4 sum() const { return v[0] + (v[1] + v[2]); }
};

// maximum / sum over the 32 lanes of half a wavefront, in every lane: exchanges within 16 lanes by DPP (a few
// cycles each; __shfl_xor goes through LDS), one exchange of 16 lanes
template <int CTRL> __device__ __forceinline__ float dpp(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
template <class F> __device__ __forceinline__ float half_reduce(float x, F f)
{
    x = f(x, dpp<0xB1>(x));       // quad_perm 1 0 3 2
    x = f(x, dpp<0x4E>(x));       // quad_perm 2 3 0 1
    x = f(x, dpp<0x141>(x));      // row_half_mirror
    x = f(x, dpp<0x140>(x));      // row_mirror
    return f(x, __shfl_xor(x, 16, 64));
}

// N batches through two register buffers, batches 0 and 1 requested by the caller.  No load in the loop is under a test
// (the compiler would wait for everything in flight behind it), and none is issued past the end: at the sizes this
// kernel serves the batches that nobody needs would be as many as the others.
template <int C, class Step, class Load>
__device__ __forceinline__ void pipe2(int N, Step step, Load load, u32x4 (&b0)[C], u32x4 (&b1)[C])
{
    if (N < 1) return;
    for (int r = 0; r + 2 < N; ++r) {
        step(r, b0);
#pragma unroll
        for (int c = 0; c < C; ++c) b0[c] = b1[c];
        load(r + 2, b1);
    }
    step(max(N - 2, 0), b0);
    if (N > 1) step(N - 1, b1);
}

// LDS of a vision workgroup: three planes of S (then W), three planes of P, staging tiles of the wavefronts (keys in
// step 1; rows of U in step 3 where U is plain), row statistics.  Rows are 32 mod 64 bytes apart: operand reads
// without bank conflicts.  Where theta is plain the partial logits of the wavefronts lie over the staging tiles between
// step 2 and the softmax where the LDS has room for them behind S and P (GPlan::own: two barriers less), else over all of it.
constexpr size_t kStage = kGW * 16 * D * 2;
constexpr int kLDL = 132;             // floats per row of a wavefront's partial logits [16][128]
constexpr size_t kPartial = kGW * 16 * kLDL * sizeof(float);
__host__ __device__ constexpr size_t planes_p(int PS) { return static_cast<size_t>(3) * 16 * (PS + 16) * 2; }
size_t pass_lds(int m, int PS, bool packed, bool own)
{
    const size_t s = 3 * 16 * (align_up(m, 32) + 16) * 2;
    const size_t vis = (own ? s + planes_p(PS) + kPartial : std::max(s + planes_p(PS) + kStage, packed ? size_t(0) : kPartial)) +
                       2 * 16 * kGW * sizeof(float);
    const size_t txt = kSW * (kWalkLds + 2 * 16 * sizeof(float));
    return std::max(vis, txt);
}

template <int NPW, bool PK, bool RAG>
__global__ __launch_bounds__(64 * kGW) void ga_pass(const uint16_t *__restrict__ q, const uint16_t *__restrict__ Kc,
                                                    const uint16_t *__restrict__ th, const uint16_t *__restrict__ U,
                                                    const uint16_t *__restrict__ Vc, uint16_t *__restrict__ Kt,
                                                    uint16_t *__restrict__ Vt, const uint16_t *__restrict__ k_new,
                                                    const uint16_t *__restrict__ v_new, GPlan p)
{
    constexpr int PS = 16 * kGW * NPW, KP = PS / 32;     // positions of a slice, k-steps over them
    constexpr int LDP = PS + 16, PLP = 16 * LDP;         // row and plane of P in LDS
    constexpr int CK = 4 / NPW;                          // packed theta: k-steps per batch of loads
    constexpr int KQ = kGW / NPW;                        // plain theta: wavefronts that share the k-steps of 128 positions
    constexpr int NC4 = KP / 4;                          // batches of four k-steps of U
    extern __shared__ __align__(16) uint16_t dyn[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int r16 = lane & 15, kg = lane >> 4;
    const int G = p.G, m = p.m, n = p.n, KS = p.KS;
    TS(5, 0);

    // ---- text workgroups: a run of the text rows of one (batch element, KV head) -----------------------------
    if (static_cast<int>(blockIdx.x) >= p.nvis) {
        const int id = blockIdx.x - p.nvis;
        const int bh = quot(id, p.qNTX), tc = id - bh * p.NTX;
        const int b = quot(bh, p.qHkv), h = bh - b * p.Hkv;
        char *const sVt = reinterpret_cast<char *>(dyn);
        float (*sM)[16] = reinterpret_cast<float (*)[16]>(sVt + kSW * kWalkLds), (*sL)[16] = sM + kSW;
        const bool fresh = k_new != nullptr;
        int t_in = p.t_in, t = p.t;
        if constexpr (RAG) {
            const int tlb = max(p.tlen[b], 0);
            t_in = min(tlb, p.t_in);
            t = fresh ? t_in + 1 : min(tlb, p.t);
        }
        const int s0 = tc * kSW;
        float m_run = -INFINITY, l_run = 0.f;
        f32x4 acc[8];
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) acc[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
        const uint16_t *kn = fresh ? k_new + static_cast<size_t>(bh) * D : q, *vn = fresh ? v_new + static_cast<size_t>(bh) * D : q;
        uint16_t *Ktb = Kt + static_cast<size_t>(bh) * p.cap * D, *Vtb = Vt + static_cast<size_t>(bh) * p.cap * D;
        // (a run that a shorter sequence of a ragged batch does not have reads nothing and writes a record without mass)
        if (wave < kSW && kSR * s0 < t) {
            u32x4 qf[4];
            const u32x4 *qp = reinterpret_cast<const u32x4 *>(q + (static_cast<size_t>(b) * p.Hq + h * G + min(r16, G - 1)) * D) + kg;
#pragma unroll
            for (int k = 0; k < 4; ++k) qf[k] = qp[4 * k];
            Rows rw;
            rw.I = 0; rw.m = 8; rw.KS = 1; rw.SV = 0; rw.qKS = 0; rw.t = t; rw.cs = 1 << 30; rw.ws = 1; rw.st = kSW * p.NTC; rw.qst = p.qst; rw.scale = p.scale;
            walk<true>(rw, Ktb, Vtb, kn, vn, fresh ? t_in : -1, qf, s0, sVt + wave * kWalkLds, m_run, l_run, acc);
        }
        merge_waves<kSW>(sVt, sM, sL, m_run, l_run, acc, G,
                    p.Ypart + (static_cast<size_t>(bh) * p.nparts + p.NUG * p.F + tc) * p.rec);
        // Sec. 3.2: the text cache keeps growing as in the backbone -- store the new token's k, v
        const int own = t_in / kTextStep;
        if (fresh && own - quot(own, p.qNTC) * p.NTC == tc && threadIdx.x < 32) {
            const int half = threadIdx.x >> 4, piece = threadIdx.x & 15;
            uint16_t *dst = (half ? Vtb : Ktb) + static_cast<size_t>(t_in) * D;
            *(reinterpret_cast<u32x4 *>(dst) + piece) = *(reinterpret_cast<const u32x4 *>(half ? vn : kn) + piece);
        }
        return;
    }

    // ---- vision workgroup -> (KV head, batch element, unit group, slice): ids are dealt round-robin over the 8
    // XCDs; an XCD takes a contiguous run of groups in that order, all slices of a group with it, so a group's
    // capsule is fetched into one L2 and a head's theta and U into as few as possible
    const int kk = blockIdx.x >> 3;
    const int gl = quot(kk, p.qF), s = kk - gl * p.F;
    const int gk = (blockIdx.x & 7) * p.chunk + gl;
    if (gl >= p.chunk || gk >= p.NGR) return;
    const int h = quot(gk, p.qBU), bu = gk - h * (p.B * p.NUG);
    const int b = quot(bu, p.qNUG), ug = bu - b * p.NUG;
    const int bh = b * p.Hkv + h, p0 = s * PS;
    const int MP = 32 * KS, LDM = MP + 16, PLM = 16 * LDM, T = 2 * KS;
    uint16_t *sS = dyn, *sP = dyn + 3 * PLM;              // W takes the place of S
    char *sTile = reinterpret_cast<char *>(sP) + planes_p(PS) + wave * (16 * D * 2);     // this wavefront's staging tile
    // row statistics behind everything else: maxima, sums per wavefront [16][kGW] (packed), per row [16] (plain)
    const uint32_t part_at = !PK && p.own ? static_cast<uint32_t>(3 * PLM * 2 + planes_p(PS)) : 0u;
    float *sRed = reinterpret_cast<float *>(reinterpret_cast<char *>(dyn) +
                                            max(static_cast<uint32_t>(3 * PLM * 2 + planes_p(PS) + kStage), PK ? 0u : static_cast<uint32_t>(part_at + kPartial)));
    int n_img = p.I;
    if constexpr (RAG) n_img = min(max(p.n_img[b], 0), p.I);

    u32x4 qf[4];
    {
        const u32x4 *qp = reinterpret_cast<const u32x4 *>(q + (static_cast<size_t>(b) * p.Hq + h * G + min(r16, G - 1)) * D) + kg;
#pragma unroll
        for (int k = 0; k < 4; ++k) qf[k] = qp[4 * k];
    }
    // running maximum, sum and un-normalised output of query row r16 (image block r16 / G of a tile)
    float m_run = -INFINITY, l_run = 0.f;
    f32x4 y = {0.f, 0.f, 0.f, 0.f};

    for (int ut = 0; ut < p.NUT; ++ut) {
        const int i0 = (ug * p.NUT + ut) * p.UP, nu = min(p.UP, n_img - i0);
        if (nu <= 0) break;                              // the same for the whole workgroup
        const char *kc_b = reinterpret_cast<const char *>(Kc + (static_cast<size_t>(bh) * p.I + i0) * m * D);
        const char *vc_b = reinterpret_cast<const char *>(Vc + (static_cast<size_t>(bh) * p.I + i0) * m * D);
        // (what follows depends on the lane only, not on the tile: kept from being moved in front of the loop, where
        // some hundred registers of addresses would live through it)
        int lane_l = lane;
        asm volatile("" : "+v"(lane_l));
        const int r16 = lane_l & 15, kg = lane_l >> 4;
        // a record of [rows][X] in blocks of 8 rows, the last one w = rows % 8 wide: how the lane (x, kg) reads its operand
        // of the last k-step (an aligned window around its values, shifted into place afterwards)
        const int nfull = m >> 3, wt = m & 7;
        auto last_off = [&](int X, int x, int &sh) __attribute__((always_inline)) -> uint32_t {
            const int to = x * 2 * wt, a0 = max(min(to & ~3, X * 2 * wt - 16), 0);
            const int jb = 4 * (KS - 1) + kg;
            const bool mine = wt != 0 && (jb == nfull || nfull == 0);
            sh = mine ? to - a0 : 0;
            return mine ? static_cast<uint32_t>(nfull * 8 * X * 2 + a0) : static_cast<uint32_t>(max(min(jb, nfull - 1), 0) * 8 * X * 2 + x * 16);
        };
        // theta, packed form: the operand of 16 positions and 8 rows j per lane is one load
        const char *th_b = reinterpret_cast<const char *>(th + static_cast<size_t>(h) * m * n);
        uint32_t th_off[NPW], th_last[NPW];
        int th_sh[NPW];
        if constexpr (PK) {
#pragma unroll
            for (int i = 0; i < NPW; ++i) {
                const int pos = min(p0 + 16 * (wave + kGW * i) + r16, n - 1);
                th_off[i] = static_cast<uint32_t>((kg * n + pos) * 16);
                th_last[i] = last_off(n, pos, th_sh[i]);
            }
        }
        auto load_thp = [&](int ks0, int i) __attribute__((always_inline)) -> u32x4 {
            const int ks = min(ks0, KS - 1);
            return *reinterpret_cast<const u32x4_a4 *>(th_b + (ks < KS - 1 ? static_cast<uint32_t>(ks) * 64u * n + th_off[i] : th_last[i]));
        };
        // theta, plain form: whole rows of 128 positions (16 lanes, 8 positions each), 8 rows j per lane; the turn to
        // operands is made in registers.  Wavefront -> positions p0 + 128 wq ..., k-steps kq, kq + KQ, ...
        const int wq = wave & (NPW - 1), kq = wave / NPW;
        const int tpos = p0 + 128 * wq + 8 * r16, tcol = min(tpos, n - 8);
        auto load_thr = [&](int ks, u32x4 (&x)[8]) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                x[e] = *reinterpret_cast<const u32x4_a2 *>(th_b + (static_cast<uint32_t>(min(32 * min(ks, KS - 1) + 8 * kg + e, m - 1)) * n + tcol) * 2u);
        };
        // U, packed form: operand of row 16 jt + r16, positions p0 + 32 ks + 8 kg ... (past n: zeros of P meet a valid load)
        const char *u_b = reinterpret_cast<const char *>(U + static_cast<size_t>(h) * m * n);
        auto load_up = [&](int jt, int ks) __attribute__((always_inline)) -> u32x4 {
            const int row = min(16 * jt + r16, m - 1), pos = p0 + 32 * ks + 8 * kg;
            return *reinterpret_cast<const u32x4 *>(u_b + (static_cast<uint32_t>(min(pos, n - 8) >> 3) * m + row) * 16u);
        };
        // plain form: 128 positions of four rows per load, as the keys; turned through the staging tile
        const int krow = kg, kpc = r16;
        auto load_ur = [&](int jt, int c, u32x4 (&x)[4]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                x[i] = *reinterpret_cast<const u32x4_a2 *>(u_b + (static_cast<uint32_t>(min(16 * jt + 4 * i + krow, m - 1)) * n +
                                                                 min(p0 + 128 * c + 8 * kpc, n - 8)) * 2u);
        };
        // 16 rows x 256 bytes in registers -> this wavefront's staging tile -> operands (16-byte piece of row r at
        // piece ^ r: no bank conflicts either way)
        const uint32_t kst = static_cast<uint32_t>(krow * 256 + (kpc ^ krow) * 16);
        auto turn = [&](const u32x4 (&src)[4], bf16x8 (&dst)[4]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<u32x4 *>(sTile + (kst ^ static_cast<uint32_t>(i * 64)) + 1024 * i) = src[i];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                dst[ks] = *reinterpret_cast<const bf16x8 *>(sTile + r16 * 256 + (((4 * ks + kg) ^ r16) & 15) * 16);
        };
        const int cch = 16 * wave + r16;                     // this lane's channel in step 4
        int vc_sh;
        const uint32_t vc_off = static_cast<uint32_t>((kg * D + cch) * 16), vc_last = last_off(D, cch, vc_sh);

        // ---- step 1: rows of keys are loaded whole (16 lanes per 256-byte row)
        const int NI = nu * T;
        auto load_k = [&](int it, u32x4 (&dst)[4]) __attribute__((always_inline)) {
            const int itc = min(it, NI - 1), u = quot(itc, p.qT), jt = itc - u * T;
            const char *tile = kc_b + (static_cast<size_t>(u) * m + 16 * jt) * (D * 2);
            const int left = m - 1 - 16 * jt;            // may be negative (padding tile): row m - 1 then
#pragma unroll
            for (int i = 0; i < 4; ++i)
                dst[i] = *reinterpret_cast<const u32x4 *>(tile + static_cast<ptrdiff_t>(min(4 * i + krow, left)) * 256 + kpc * 16);
        };
        auto score = [&](const u32x4 (&src)[4], int it) __attribute__((always_inline)) {
            bf16x8 ko[4];
            turn(src, ko);
            f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ko[ks], as_bf16x8(qf[ks]), a, 0, 0, 0);
            const int u = quot(min(it, NI - 1), p.qT), j = 16 * (it - u * T) + 4 * kg;
            float x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = j + e < m ? a[e] : 0.f;
            if (r16 < G && it < NI) store_planes(sS + (u * G + r16) * LDM + j, PLM, x);
        };
        const int NF = nu * KS;
        auto load_v = [&](int f) __attribute__((always_inline)) -> u32x4 {
            const int fc = min(f, NF - 1), u = quot(fc, p.qKS), ks = fc - u * KS;
            const char *rec = vc_b + static_cast<size_t>(u) * m * (D * 2);
            return *reinterpret_cast<const u32x4_a4 *>(rec + (ks < KS - 1 ? static_cast<uint32_t>(ks) * (64 * D) + vc_off : vc_last));
        };
        // requested in the order they are needed: four tiles of keys, the first k-steps of theta
        // (zeros in what a short case does not request: a value left open would be carried from tile to tile)
        u32x4 ka[4][4] = {}, ua0[4] = {}, ua1[4] = {}, va0[4] = {}, va1[4] = {}, tr0[8] = {}, tr1[8] = {};
        const int NK = NI > wave ? (NI - wave + kGW - 1) / kGW : 0;      // tiles of this wavefront
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < NK) load_k(wave + kGW * i, ka[i]);
        const int NTH = KS > kq ? (KS - kq + KQ - 1) / KQ : 0;            // plain theta: k-steps of this wavefront
        auto load_t = [&](int r, u32x4 (&b)[8]) __attribute__((always_inline)) { load_thr(kq + KQ * r, b); };
        if constexpr (!PK) {
            if (NTH > 0) load_t(0, tr0);
            if (NTH > 1) load_t(1, tr1);
        }
        // one word of each 128-byte line of this slice's share of the blocks' values: they are in the L2 when step 4
        // asks for them (beyond 1024 lines per slice: not, there are enough workgroups then to hide it)
        uint32_t touch[2];
#pragma unroll
        for (int k = 0; k < 2; ++k)
            touch[k] = *reinterpret_cast<const uint32_t *>(
                vc_b + static_cast<size_t>(min((static_cast<int>(threadIdx.x) + 64 * kGW * k) * p.F + s, 2 * nu * m - 1)) * 128);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < NK) score(ka[i], wave + kGW * i);
        if (NK > 4) {
            auto load_k4 = [&](int r, u32x4 (&b)[4]) __attribute__((always_inline)) { load_k(wave + kGW * (r + 4), b); };
            load_k4(0, ka[0]);
            if (NK > 5) load_k4(1, ka[1]);
            pipe2(NK - 4, [&](int r, u32x4 (&b)[4]) __attribute__((always_inline)) { score(b, wave + kGW * (r + 4)); }, load_k4, ka[0], ka[1]);
        }
        TS(5, 1);
        // batch x = (tile, 128 positions) of this wavefront, two in flight (step 3)
        const int NX = T > wave ? NC4 * ((T - wave + kGW - 1) / kGW) : 0;
        auto load_u = [&](int x, u32x4 (&b)[4]) __attribute__((always_inline)) {
            const int jt = wave + kGW * (x / NC4), c4 = x % NC4;
            if constexpr (PK) {
#pragma unroll
                for (int c = 0; c < 4; ++c) b[c] = load_up(jt, 4 * c4 + c);
            } else {
                load_ur(jt, c4, b);
            }
        };
        float mx, sm;                                    // slice maximum and sum of query row r16
        if constexpr (PK) {
            // batch r: CK k-steps x NPW tiles
            auto load_b = [&](int r, u32x4 (&b)[4]) __attribute__((always_inline)) {
#pragma unroll
                for (int c = 0; c < CK; ++c)
#pragma unroll
                    for (int i = 0; i < NPW; ++i) b[c * NPW + i] = load_thp(CK * r + c, i);
            };
            const int NB = (KS + CK - 1) / CK;
            u32x4 tb0[4] = {}, tb1[4] = {};
            load_b(0, tb0);
            if (NB > 1) load_b(1, tb1);
            lds_barrier();

            // ---- step 2: L^T[pos][row] = sum_j theta[j][pos] S[row][j] for this wavefront's position tiles
            Acc3 aL[NPW];
            pipe2(NB, [&](int r, u32x4 (&b)[4]) __attribute__((always_inline)) {
#pragma unroll
                for (int c = 0; c < CK; ++c) {
                    const int ks = CK * r + c;
                    if (ks < KS) {                       // uniform; no loads from memory inside
                        bf16x8 sf[3];
#pragma unroll
                        for (int k = 0; k < 3; ++k) sf[k] = *reinterpret_cast<const bf16x8 *>(sS + k * PLM + r16 * LDM + 32 * ks + 8 * kg);
#pragma unroll
                        for (int i = 0; i < NPW; ++i) {
                            u32x4 a = b[c * NPW + i];
                            if (ks == KS - 1 && wt) a = shift_window(a, th_sh[i] >> 2, (th_sh[i] & 2) * 8u);
                            aL[i].add(as_bf16x8(a), sf);
                        }
                    }
                }
            }, load_b, tb0, tb1);
            if (NX > 0) load_u(0, ua0);
            if (NX > 1) load_u(1, ua1);
            f32x4 accL[NPW];
#pragma unroll
            for (int i = 0; i < NPW; ++i) accL[i] = aL[i].sum();
            mx = -INFINITY;
#pragma unroll
            for (int i = 0; i < NPW; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    accL[i][e] = p0 + 16 * (wave + kGW * i) + 4 * kg + e < n ? accL[i][e] * p.scale : -INFINITY;
                    mx = fmaxf(mx, accL[i][e]);
                }
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            if (kg == 0) sRed[r16 * kGW + wave] = mx;
            lds_barrier();
            {
                const f32x4 a = *reinterpret_cast<const f32x4 *>(sRed + r16 * kGW), c = *reinterpret_cast<const f32x4 *>(sRed + r16 * kGW + 4);
                mx = fmaxf(fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3])), fmaxf(fmaxf(c[0], c[1]), fmaxf(c[2], c[3])));
            }
            sm = 0.f;
#pragma unroll
            for (int i = 0; i < NPW; ++i) {
                float x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[e] = __expf(accL[i][e] - mx);
                    sm += x[e];
                }
                store_planes(sP + r16 * LDP + 16 * (wave + kGW * i) + 4 * kg, PLP, x);
            }
            sm += __shfl_xor(sm, 16, 64);
            sm += __shfl_xor(sm, 32, 64);
            if (kg == 0) sRed[16 * kGW + r16 * kGW + wave] = sm;
            lds_barrier();
            {
                const f32x4 a = *reinterpret_cast<const f32x4 *>(sRed + 16 * kGW + r16 * kGW), c = *reinterpret_cast<const f32x4 *>(sRed + 16 * kGW + r16 * kGW + 4);
                sm = ((a[0] + a[1]) + (a[2] + a[3])) + ((c[0] + c[1]) + (c[2] + c[3]));
            }
        } else {
            // ---- step 2: the wavefront's k-steps for 128 positions: tile i of eight holds the positions 8 x + i
            lds_barrier();
            f32x4 accL[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) accL[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            auto th_step = [&](int r, u32x4 (&b)[8]) __attribute__((always_inline)) {
                const int ks = kq + KQ * r;
                u32x4 (&ta)[8] = b;
                bf16x8 sf[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) sf[k] = *reinterpret_cast<const bf16x8 *>(sS + k * PLM + r16 * LDM + 32 * ks + 8 * kg);
                if (p0 + 128 * wq + 128 > n) {           // uniform; registers only
#pragma unroll
                    for (int e = 0; e < 8; ++e) ta[e] = drop_elems(ta[e], min(tpos - tcol, 8));
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const uint32_t sel = i & 1 ? 0x07060302u : 0x05040100u;      // high or low halves of two words
                    const u32x4 a = u32x4_mk(__builtin_amdgcn_perm(ta[1][i >> 1], ta[0][i >> 1], sel), __builtin_amdgcn_perm(ta[3][i >> 1], ta[2][i >> 1], sel),
                                             __builtin_amdgcn_perm(ta[5][i >> 1], ta[4][i >> 1], sel), __builtin_amdgcn_perm(ta[7][i >> 1], ta[6][i >> 1], sel));
                    accL[i] = mfma3(as_bf16x8(a), sf, accL[i]);
                }
            };
            pipe2(NTH, th_step, load_t, tr0, tr1);
            TS(5, 2);
            if (NX > 0) load_u(0, ua0);
            if (NX > 1) load_u(1, ua1);
            if (!p.own) lds_barrier();                   // uniform.  S has been read: partial logits in its place
            float *sL = reinterpret_cast<float *>(reinterpret_cast<char *>(dyn) + part_at);
#pragma unroll
            for (int e = 0; e < 4; ++e) {                // lane: positions 8 (4 kg + e) + i of query row r16
                float *dst = sL + (wave * 16 + r16) * kLDL + 8 * (4 * kg + e);
                *reinterpret_cast<f32x4 *>(dst) = f32x4_mk(accL[0][e], accL[1][e], accL[2][e], accL[3][e]);
                *reinterpret_cast<f32x4 *>(dst + 4) = f32x4_mk(accL[4][e], accL[5][e], accL[6][e], accL[7][e]);
            }
            lds_barrier();
            // half a wavefront per query row: four positions per lane and window of 128
            const int row = threadIdx.x >> 5, pl = 4 * (threadIdx.x & 31);
            float x[NPW][4], rmx = -INFINITY, rsm = 0.f;
#pragma unroll
            for (int i = 0; i < NPW; ++i) {
                f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < KQ; ++k) a += *reinterpret_cast<const f32x4 *>(sL + ((k * NPW + i) * 16 + row) * kLDL + pl);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[i][e] = p0 + 128 * i + pl + e < n ? a[e] * p.scale : -INFINITY;
                    rmx = fmaxf(rmx, x[i][e]);
                }
            }
            rmx = half_reduce(rmx, [](float a, float b) { return fmaxf(a, b); });
#pragma unroll
            for (int i = 0; i < NPW; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[i][e] = __expf(x[i][e] - rmx);
                    rsm += x[i][e];
                }
            rsm = half_reduce(rsm, [](float a, float b) { return a + b; });
            if ((threadIdx.x & 31) == 0) { sRed[row] = rmx; sRed[16 + row] = rsm; }
            if (!p.own) lds_barrier();                   // the partial logits have been read
#pragma unroll
            for (int i = 0; i < NPW; ++i) store_planes(sP + row * LDP + 128 * i + pl, PLP, x[i]);
            lds_barrier();
            mx = sRed[r16];
            sm = sRed[16 + r16];
        }

        TS(5, 3);
        // ---- step 3: W^T[j][row] = sum_pos U[j][pos] P[row][pos] for tiles of 16 rows of U, eight apart
        Acc3 aw;
        bf16x8 pr[NC4 == 1 ? 4 : 1][3];                  // a slice of 128 positions: P stays in registers
        if constexpr (NC4 == 1) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int k = 0; k < 3; ++k) pr[c][k] = *reinterpret_cast<const bf16x8 *>(sP + k * PLP + r16 * LDP + 32 * c + 8 * kg);
        }
        auto fold = [&](int x, u32x4 (&b)[4]) __attribute__((always_inline)) {
            u32x4 (&ua)[4] = b;
            const int jt = wave + kGW * (x / NC4), c4 = x % NC4;
            bf16x8 uo[4];
            if constexpr (PK) {
#pragma unroll
                for (int c = 0; c < 4; ++c) uo[c] = as_bf16x8(ua[c]);
            } else {
                if (p0 + 128 * c4 + 128 > n) {           // uniform; registers only
                    const int pos = p0 + 128 * c4 + 8 * kpc;
#pragma unroll
                    for (int i = 0; i < 4; ++i) ua[i] = drop_elems(ua[i], min(pos - min(pos, n - 8), 8));
                }
                turn(ua, uo);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                bf16x8 pf[3];
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    pf[k] = NC4 == 1 ? pr[NC4 == 1 ? c : 0][k]
                                     : *reinterpret_cast<const bf16x8 *>(sP + k * PLP + r16 * LDP + 128 * c4 + 32 * c + 8 * kg);
                aw.add(uo[c], pf);
            }
            if (c4 == NC4 - 1) {
                const f32x4 a = aw.sum();
                aw = Acc3();
                const int j = 16 * jt + 4 * kg;
                float w[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = j + e < m ? a[e] : 0.f;
                store_planes(sS + r16 * LDM + j, PLM, w);
            }
        };
        // values of step 4, four k-steps a batch
        const int NV = (NF + 3) / 4;
        auto load_v4 = [&](int r, u32x4 (&b)[4]) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < 4; ++c) b[c] = load_v(4 * r + c);
        };
        load_v4(0, va0);
        if (NV > 1) load_v4(1, va1);
        asm volatile("" ::"v"(touch[0]), "v"(touch[1]));
        pipe2(NX, fold, load_u, ua0, ua1);

        // ---- step 4: Y^T[c][row] = sum_j Vc^T[c][j] W[row][j]: k-steps of all image blocks of the tile in one
        // row; the weights of other blocks' rows are selected to zero.  (An infinite value makes its own channel of the head
        // infinite or NaN, as the slices' weights for it have either sign.)
        lds_barrier();
        TS(5, 4);
        Acc3 ao;
        // (what lies behind the lane's values in the short last block belongs to the next channel)
        const u32x4 vtail = keep_elems(u32x4_mk(0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu), m - 32 * (KS - 1) - 8 * kg);
        auto out_step = [&](int f, u32x4 v) __attribute__((always_inline)) {
            const int u = quot(f, p.qKS), ks = f - u * KS;
            if (wt && ks == KS - 1) {
                v = shift_window(v, vc_sh >> 2, (vc_sh & 2) * 8u);
                v = u32x4_mk(v.x & vtail.x, v.y & vtail.y, v.z & vtail.z, v.w & vtail.w);
            }
            const uint32_t keep = r16 >= u * G && r16 < (u + 1) * G ? 0xffffffffu : 0u;
            bf16x8 wf[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const u32x4 w = *reinterpret_cast<const u32x4 *>(sS + k * PLM + r16 * LDM + 32 * ks + 8 * kg);
                wf[k] = as_bf16x8(u32x4_mk(w.x & keep, w.y & keep, w.z & keep, w.w & keep));
            }
            ao.add(as_bf16x8(v), wf);
        };
        pipe2(NV, [&](int r, u32x4 (&b)[4]) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (c == 0 || 4 * r + c < NF) out_step(4 * r + c, b[c]);      // uniform; no loads from memory inside
        }, load_v4, va0, va1);
        const f32x4 o = ao.sum();
        TS(5, 5);
        // rows of the tile that hold no image block keep their state
        if (r16 < nu * G) {
            const float mn = fmaxf(m_run, mx), ca = __expf(m_run - mn), cb = __expf(mx - mn);
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = y[e] * ca + o[e] * cb;
            l_run = l_run * ca + sm * cb;
            m_run = mn;
        }
        if (ut + 1 < p.NUT) lds_barrier();               // W has been read
    }

    // ---- the image blocks of a query head, rows u G + g of the tile, into one record
    float gm = -INFINITY;
    for (int u = 0; u < p.UP; ++u) gm = fmaxf(gm, __shfl(m_run, (lane & 48) | min(u * G + r16, 15), 64));
    const float mref = gm == -INFINITY ? 0.f : gm;       // nothing at all (ragged batch): a record without mass
    f32x4 yo = {0.f, 0.f, 0.f, 0.f};
    float lo = 0.f;
    for (int u = 0; u < p.UP; ++u) {
        const int src = (lane & 48) | min(u * G + r16, 15);
        const float w = __expf(__shfl(m_run, src, 64) - mref);
#pragma unroll
        for (int e = 0; e < 4; ++e) yo[e] += w * __shfl(y[e], src, 64);
        lo += w * __shfl(l_run, src, 64);
    }
    if (r16 < G) {
        float *yp = p.Ypart + (static_cast<size_t>(bh) * p.nparts + ug * p.F + s) * p.rec;
        *reinterpret_cast<f32x4 *>(yp + r16 * D + 16 * wave + 4 * kg) = yo;
        if (wave == 0 && kg == 0) {
            yp[G * D + r16] = gm;
            yp[G * D + G + r16] = lo;
        }
    }
    TS(5, 6);
}

constexpr size_t kPassLds = 156 * 1024;
constexpr int kOneEach = 256;         // workgroups that find a compute unit each (MI355X has 256)
std::atomic<long> g_any_calls{0};     // debug counter (kvc_dev_any_calls)

// false: no plan (slices or LDS beyond what the kernel holds).  What decides the order of the sums -- slices, tiles, the
// text run that a row belongs to -- follows from the shape and the capacity of the text cache, not from the rows that it
// holds: a ragged batch, whose row counts the host does not know, computes what the uniform call computes, bit for bit
// (runs without a row add zeros), and a generation keeps one order from its first token to its last.
bool make_gplan(GPlan &p, const kvc_shape &s, int t, int t_in, int cap)
{
    p.B = s.batch; p.Hq = s.n_q_heads; p.Hkv = s.n_kv_heads; p.G = p.Hq / p.Hkv;
    p.I = s.n_images; p.n = s.n_img_tokens; p.m = s.m; p.KS = (s.m + 31) / 32;
    p.t = t; p.t_in = t_in; p.cap = cap;
    const long bh = static_cast<long>(p.B) * p.Hkv;
    // Slice and tile.  A workgroup's fixed cost is one latency per phase; beyond that it reads its slice of theta
    // and U per tile and the blocks' keys and values once per slice.  Wide slices and full tiles read least, so
    // they are taken as long as one workgroup per compute unit remains; with fewer, narrow slices and then
    // smaller tiles spread the work.
    const int up_max = std::max(1, std::min(16 / p.G, p.I));
    auto groups = [&](int up) { return bh * ((p.I + up - 1) / up); };
    int ps = 128;
    p.UP = up_max;
    for (int w : {512, 256})
        if (p.n > w / 2 && groups(up_max) * ((p.n + w - 1) / w) >= 256 && pass_lds(p.m, w, false, false) <= kPassLds) { ps = w; break; }
    p.PS = ps;
    p.F = (p.n + ps - 1) / ps;
    if (p.F > kMaxVisParts || pass_lds(p.m, ps, false, false) > kPassLds) return false;
    // (as many runs as give every one the same number of steps in a full cache: the chip is full of workgroups where the
    // text is long, and takes 12 runs of two steps in less time than 16 of one or two)
    auto steps = [](int rows) { return (rows + kTextStep - 1) / kTextStep; };
    const int each = std::max(1, (steps(cap) + kMaxTextParts - 1) / kMaxTextParts);
    p.NTC = std::max(1, (steps(cap) + each - 1) / each);
    p.NTX = std::min(steps(t), p.NTC);
    // Smaller tiles as long as every workgroup, those of a full text cache with them, still has a compute unit to itself and
    // one tile: 12 blocks of n = 576, m = 346, B = 1, 12/2 heads, two tiles per workgroup 24.6 us, one twice as full 20.5.
    // Where the text's workgroups would come behind, in a second round of some 3 us, only if that saves 16 steps of 32
    // compressed rows (a second round against full tiles: 8/8 heads, B = 2, 3 blocks of n = 600, m = 97, 300 text rows, 4
    // steps saved 14.2 / 12.0 us; 16/8, B = 2, 12 blocks of n = 379, m = 178, 2000 rows, 24 steps saved 22.1 / 33.1).
    if (ps == 128)
        for (int up = (p.UP + 1) / 2; p.UP > 1 && groups(up) * p.F <= kOneEach && (p.I + up - 1) / up * p.F <= kMaxVisParts &&
                                      (groups(up) * p.F + bh * p.NTC <= kOneEach || (p.UP - up) * p.KS >= 16);
             up = (p.UP + 1) / 2)
            p.UP = up;
    const int tiles = (p.I + p.UP - 1) / p.UP, ug_max = kMaxVisParts / p.F;
    p.NUT = p.I > 0 ? (tiles + ug_max - 1) / ug_max : 1;
    p.NUG = p.I > 0 ? (tiles + p.NUT - 1) / p.NUT : 0;
    p.NGR = p.Hkv * p.B * p.NUG;
    p.chunk = (p.NGR + 7) / 8;
    p.nvis = 8 * p.chunk * p.F;
    p.nparts = p.NUG * p.F + p.NTX;
    p.rec = static_cast<int>(align_up(p.G * D + 2 * p.G, 4));
    p.qF = quot_multiplier(p.F); p.qBU = quot_multiplier(p.B * p.NUG); p.qNUG = quot_multiplier(p.NUG);
    p.qT = quot_multiplier(2 * p.KS); p.qNTX = quot_multiplier(p.NTX); p.qHkv = quot_multiplier(p.Hkv); p.qKS = quot_multiplier(p.KS);
    p.qNTC = quot_multiplier(p.NTC); p.qst = quot_multiplier(kSW * p.NTC);
    // (the registers allow one workgroup per compute unit anyway: none is kept out by the LDS that this takes.  Two barriers
    // less: 28/4 heads, n = 729, 3 blocks of m = 292, B = 1 16.55 -> 16.35 us per call, B = 8 36.9 -> 36.1; 8/8 heads, 6 blocks
    // of n = 99 9.49 -> 9.29.  Beyond m = 768, 640 and 384 for slices of 128, 256 and 512 positions there is no room.)
    p.own = pass_lds(p.m, p.PS, false, true) <= kPassLds;
    p.n_img = p.tlen = nullptr;
    // quot(): dividends below 2^32 / divisor; 32-bit offsets into a head's theta and U
    const long lim = 1l << 31;
    return p.nparts >= 1 && static_cast<long>(p.nvis) * std::max(p.F, p.B * std::max(p.NUG, 1)) < lim &&
           bh * p.NTC * std::max(std::max(p.NTC, 1), p.Hkv) < lim && static_cast<long>(16) * 2 * p.KS * 2 * p.KS < lim &&
           static_cast<long>(p.KS) * 64 * p.n < lim;
}

template <int NPW, bool PK, bool RAG> bool launch_g3(const GPlan &p, const DecodeCall &c)
{
    static bool attr_set[kMaxDevices] = {};
    if (!allow_lds(reinterpret_cast<const void *>(ga_pass<NPW, PK, RAG>), kPassLds, attr_set)) return false;
    const int grid = p.nvis + p.B * p.Hkv * p.NTX;
    ga_pass<NPW, PK, RAG><<<grid, 64 * kGW, pass_lds(p.m, p.PS, PK, !PK && p.own), c.stream>>>(
        static_cast<const uint16_t *>(c.q), static_cast<const uint16_t *>(c.Kc),
        static_cast<const uint16_t *>(PK ? c.theta_packed : c.theta), static_cast<const uint16_t *>(PK ? c.U_packed : c.U),
        static_cast<const uint16_t *>(c.Vc), static_cast<uint16_t *>(c.Kt), static_cast<uint16_t *>(c.Vt),
        static_cast<const uint16_t *>(c.k_new), static_cast<const uint16_t *>(c.v_new), p);
    return true;
}

template <int NPW> bool launch_g(const GPlan &p, const DecodeCall &c)
{
    const bool pk = c.theta_packed && c.U_packed && p.n % 8 == 0;      // (kvc_pack_u makes no other)
    if (p.n_img) return pk ? launch_g3<NPW, true, true>(p, c) : launch_g3<NPW, false, true>(p, c);
    return pk ? launch_g3<NPW, true, false>(p, c) : launch_g3<NPW, false, false>(p, c);
}

}  // namespace

static bool any_shape(const kvc_shape &s)
{
    return s.dtype == KVC_BF16 && s.head_dim == D && s.n_q_heads / s.n_kv_heads <= 16 && s.n_img_tokens >= 8;
}

// Calls of shapes with tuned kernels that take less time here: a compute unit for every vision workgroup, at most 10 steps of
// 32 compressed rows in each, whose chains are its time, at most 512 workgroups with one for every 128 rows of a full text
// cache, and text runs of at most 4 steps.  us per layer, tuned kernels against this pass: n = 256, m = 154, 16 blocks, 28/4
// heads 16.5 / 11.5, 32 blocks (10 steps) 16.6 / 14.0; n = 576, m = 144, 5 blocks 14.9 / 12.0, 12 blocks (10 steps) 14.9 / 13.1;
// n = 1024, m = 256, one block 14.6 / 12.6, 8 blocks (16 steps) 13.3 / 16.5; m = 615 (20 steps) 19.5 / 21.4.  Workgroups, at
// n = 576, m = 200, one block, B = 4, 16/8 heads: 448 (1000 text rows) 17.3 / 16.2, 704 19.8 / 20.6, 1216 25.6 / 31.6; at n = 256,
// m = 103, one block, B = 16, 14/2 heads: 320 16.6 / 13.1, 576 18.9 / 19.6.  Text rows at n = 256, m = 103, 2 blocks, 28/4 heads,
// B = 1: 4000 16.0 / 12.0, 8000 (4 steps per run) 18.5 / 17.7, 16000 20.7 / 27.2, 28000 26.7 / 41.3: the tuned kernels give every
// 128 rows a workgroup.
static bool small_call(const GPlan &p)
{
    const long vision = static_cast<long>(p.NGR) * p.F, text = static_cast<long>(p.B) * p.Hkv * ((p.cap + kTextStep - 1) / kTextStep);
    return p.I > 0 && p.NUT == 1 && p.UP * p.KS <= 10 && vision <= kOneEach && vision + text <= 2 * kOneEach &&
           p.cap <= 4 * kMaxTextParts * kTextStep;
}

bool any_decode_supported(const kvc_shape &s)
{
    GPlan p;
    return any_shape(s) && make_gplan(p, s, 1, 0, 1);
}

size_t any_decode_ws_bytes(const kvc_shape &s, int32_t max_text)
{
    GPlan p;
    if (!make_gplan(p, s, s.n_images > 0 ? 0 : 1, 0, std::max(max_text, 1))) return 0;
    const int ntx = std::min((std::max(max_text, 1) + kTextStep - 1) / kTextStep, kMaxTextParts);
    return kCounterBytes + static_cast<size_t>(p.B) * p.Hkv * (p.NUG * p.F + ntx) * p.rec * sizeof(float) + kTimelineBytes;
}

bool any_decode_plan(const kvc_shape &s, int t, int cap, int32_t *plan)
{
    GPlan p;
    if (!any_shape(s) || !make_gplan(p, s, t, t, cap)) return false;
    const int32_t v[8] = {p.PS, p.UP, p.NUT, p.F, p.NGR * p.F, p.NTX, (cap + kMaxTextParts * kTextStep - 1) / (kMaxTextParts * kTextStep), small_call(p)};
    std::copy(v, v + 8, plan);
    return true;
}

long any_decode_calls() { return g_any_calls.load(); }

bool any_decode(const DecodeCall &c, kvc_status *st, bool small_only)
{
    if (c.static_variant || !any_shape(c.s)) return false;
    if ((c.n_images_dev == nullptr) != (c.text_len_dev == nullptr)) return false;
    GPlan p;
    if (!make_gplan(p, c.s, c.t, c.t_in, c.cap)) return false;
    if (small_only && !(c.theta_packed && c.U_packed && small_call(p))) return false;
    if (kCounterBytes + static_cast<size_t>(p.B) * p.Hkv * p.nparts * p.rec * sizeof(float) > c.ws_bytes) return false;
    p.scale = c.scale;
    p.Ypart = reinterpret_cast<float *>(static_cast<char *>(c.ws) + kCounterBytes);
    p.n_img = c.n_images_dev; p.tlen = c.text_len_dev;
#if defined(KVC_TIMELINE)
    p.tl = reinterpret_cast<unsigned long long *>(static_cast<char *>(c.ws) + ((c.ws_bytes - kTimelineBytes) & ~size_t(255)));
#endif
    const bool ok = p.PS == 512 ? launch_g<4>(p, c) : p.PS == 256 ? launch_g<2>(p, c) : launch_g<1>(p, c);
    if (ok) ++g_any_calls;
    *st = ok && hipGetLastError() == hipSuccess
              ? finalize_parts(p.Ypart, p.nparts, p.NUG * p.F, p.rec, p.B, p.Hq, p.Hkv, c.mu, c.out, c.lse, c.stream)
              : KVC_ERR_HIP;
    return true;
}

}  // namespace kvc
