// fp32 storage, and bf16 storage with a head_dim other than 128: compression and decode on the fp32 matrix
// instruction of gfx950 (v_mfma_f32_16x16x4_f32: fp32 operands and sums), head_dim up to 256.  Compression: any n >= 4,
// any m.  Decode: n from 4 to 12288 (48 slices of 256), m up to 1952 (LDS), at most 16 query heads per KV head; also bf16
// with head_dim 128 beyond the limits of ga_pass.  bf16 values are widened where they are loaded.
//
//   gx_project  Vc = U (V - 1 mu^T) for 16 rows of U of one image block: eight wavefronts share the positions and add
//               up through LDS.  The workgroup's key rows are copied by the way.
//   gx_pass     the decode step of ga_pass (kvc_any_decode.hip) in this arithmetic: a vision workgroup owns a slice
//               of positions of one (batch element, KV head), walks tiles of image blocks through the four products
//               of Alg. 1 and writes one part record; text workgroups attend runs of 128 text rows.
//   gx_merge    joint softmax over the part records, "+ (sum P_vis) mu", output and log-sum-exp.
//
// Bound: at the sizes that run in fp32 (checks, calibration: one layer, a few sequences) launches and the latency of
// the dependent phases; the scalar kernels that these replace spent it in serial loops over n or m with one load per
// multiply-add, in 58 (projection) and 8 (output) workgroups.  One layer, B = 1, 8/2 heads, d = 64, n = 576, m = 231:
// compression 244 -> 8 us, decode step about 80 us in six launches -> 14.5 us in two; both with their gaps 335 -> 24 us.  (What
// gx_pass spends beyond latency is instructions: 64-bit addresses per load, moved in front of the loop over tiles, took 120
// registers and 0.9 us more, d = 256 three.  The first share of every phase's loads requested at the start: no gain, and 1.6 us
// lost at n = 9.)
#include "kvc_decode_dev.h"

#include <algorithm>

namespace kvc {

using dd::f32x2;
using dd::f32x4;
using dd::f32x4_mk;
using dd::quot;
using dd::quot_multiplier;
using dd::u32x4;

namespace {

constexpr int kXW = 8;                // wavefronts
constexpr int kVisParts = 48, kTextParts = 16;     // part records per (batch element, KV head): a lane each in the merge
constexpr int kTR = 16 * kXW;         // text rows per step; run r of NTC takes the steps r, r + NTC, r + 2 NTC, ...

// four consecutive elements at any element-aligned address
template <class T> struct Vec4;
template <> struct Vec4<float> {
    typedef f32x4 __attribute__((aligned(4))) raw;
    static __device__ __forceinline__ f32x4 wide(raw v) { return v; }
};
template <> struct Vec4<bf16_t> {
    typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
    typedef u16x4 __attribute__((aligned(2))) raw;
    static __device__ __forceinline__ f32x4 wide(raw v)
    {
        return f32x4_mk(__uint_as_float(static_cast<uint32_t>(v[0]) << 16), __uint_as_float(static_cast<uint32_t>(v[1]) << 16),
                        __uint_as_float(static_cast<uint32_t>(v[2]) << 16), __uint_as_float(static_cast<uint32_t>(v[3]) << 16));
    }
};
template <class T> using raw4 = typename Vec4<T>::raw;
// element i of a matrix whose bytes 32 bits count: a scalar base and a 32-bit offset per lane
template <class T> __device__ __forceinline__ const T *at(const T *base, uint32_t i)
{
    return reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + i * static_cast<uint32_t>(sizeof(T)));
}
template <class T> __device__ __forceinline__ raw4<T> load4_raw(const T *p) { return *reinterpret_cast<const raw4<T> *>(p); }
template <class T> __device__ __forceinline__ f32x4 load4(const T *p) { return Vec4<T>::wide(*reinterpret_cast<const typename Vec4<T>::raw *>(p)); }
// elements c .. c + 3 of a row of len >= 4: past the end zeros, and no load past the end
__device__ __forceinline__ f32x4 past_end(f32x4 v, int c, int len)
{
    const int sh = c - min(c, len - 4);
    f32x4 r;
    r[0] = sh == 0 ? v[0] : sh == 1 ? v[1] : sh == 2 ? v[2] : sh == 3 ? v[3] : 0.f;
    r[1] = sh == 0 ? v[1] : sh == 1 ? v[2] : sh == 2 ? v[3] : 0.f;
    r[2] = sh == 0 ? v[2] : sh == 1 ? v[3] : 0.f;
    r[3] = sh == 0 ? v[3] : 0.f;
    return r;
}
template <class T> __device__ __forceinline__ f32x4 load4_in(const T *row, int c, int len) { return past_end(load4(row + min(c, len - 4)), c, len); }
// LDS barrier that leaves loads from memory in flight
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
// acc += sum over e of A[., 4 kg + e] B[4 kg + e, .]: sixteen steps of the contraction
__device__ __forceinline__ f32x4 mfma16(f32x4 a, f32x4 b, f32x4 acc)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], acc, 0, 0, 0);
    return acc;
}

// ---- compression -----------------------------------------------------------------------------------------------
struct XProj {
    int Hkv, n, m, I, d, vis0, JT;
    int64_t sb, sh, ss;
};

// (bf16, d <= 64: four workgroups per CU instead of three, which 72 registers would leave)
template <class T, int DT>
__global__ __launch_bounds__(64 * kXW, DT == 4 && sizeof(T) == 2 ? 8 : 2) void gx_project(const T *__restrict__ K, const T *__restrict__ V, const int32_t *__restrict__ idx,
                                                       const T *__restrict__ U, const T *__restrict__ mu, T *__restrict__ Kc,
                                                       T *__restrict__ Vc, XProj p)
{
    extern __shared__ __align__(16) float sAcc[];        // [wavefront][16 rows][16 DT + 4]
    constexpr int LDA = 16 * DT + 4;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r16 = lane & 15, kg = lane >> 4;
    const int u = blockIdx.x / p.JT, j0 = 16 * (blockIdx.x - u * p.JT);
    const int bh = u / p.I, i = u - bh * p.I, b = bh / p.Hkv, h = bh - b * p.Hkv;
    const int d = p.d, n = p.n, m = p.m;
    const int64_t blk = b * p.sb + h * p.sh + (static_cast<int64_t>(p.vis0) + static_cast<int64_t>(i) * n) * p.ss;
    const T *Vb = V + blk, *Ub = U + (static_cast<size_t>(h) * m + min(j0 + r16, m - 1)) * n;
    int ch[DT];
    float muc[DT];
#pragma unroll
    for (int ct = 0; ct < DT; ++ct) {
        ch[ct] = min(16 * ct + r16, d - 1);
        muc[ct] = to_f(mu[static_cast<size_t>(h) * d + ch[ct]]);
    }
    f32x4 acc[DT];
#pragma unroll
    for (int ct = 0; ct < DT; ++ct) acc[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    // 16 positions per step; past the end the centre stands in for a row of V: its zero meets zeros of U
    const T *muh = mu + static_cast<size_t>(h) * d;
    for (int s = wave; 16 * s < n; s += kXW) {
        const f32x4 a = load4_in(Ub, 16 * s + 4 * kg, n);
        float v[4][DT];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int pos = 16 * s + 4 * kg + e;
            const T *row = pos < n ? Vb + static_cast<int64_t>(pos) * p.ss : muh;
#pragma unroll
            for (int ct = 0; ct < DT; ++ct) v[e][ct] = to_f(row[ch[ct]]);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int ct = 0; ct < DT; ++ct) acc[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], v[e][ct] - muc[ct], acc[ct], 0, 0, 0);
    }
    // keys: 16-byte pieces of this workgroup's rows (an index outside the block must not leave it)
    {
        const int pieces = d * static_cast<int>(sizeof(T)) / 16, rows = min(16, m - j0);
        for (int x = threadIdx.x; x < rows * pieces; x += 64 * kXW) {
            const int r = x / pieces, pc = x - r * pieces;
            const int row = min(max(idx[j0 + r], 0), n - 1);
            reinterpret_cast<u32x4 *>(Kc + (static_cast<size_t>(u) * m + j0 + r) * d)[pc] =
                reinterpret_cast<const u32x4 *>(K + blk + static_cast<int64_t>(row) * p.ss)[pc];
        }
    }
#pragma unroll
    for (int ct = 0; ct < DT; ++ct)
#pragma unroll
        for (int e = 0; e < 4; ++e) sAcc[(wave * 16 + 4 * kg + e) * LDA + 16 * ct + r16] = acc[ct][e];
    __syncthreads();
    // two 8-row blocks of the record, channel-major
    T *out = Vc + static_cast<size_t>(u) * m * d;
    for (int x = threadIdx.x; x < 16 * d; x += 64 * kXW) {
        const int r = x & 7, q = x >> 3, jb = q / d, c = q - jb * d, j = j0 + 8 * jb + r;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < kXW; ++w) sum += sAcc[(w * 16 + 8 * jb + r) * LDA + c];
        if (j < m) out[vc_offset(j, c, m, d)] = from_f<T>(sum);
    }
}

// ---- decode ----------------------------------------------------------------------------------------------------
struct XPlan {
    int B, Hq, Hkv, G, I, n, m, d, KB;                  // KB: 32-row steps of the compressed axis
    int UP, NUT, NUG, F, NP;                            // image blocks per tile, tiles per workgroup, unit groups, slices, position tiles per wavefront
    int NTX, NTC, nparts, rec, nvis;
    int t, t_in, cap;
    unsigned qF, qNUG, qHkv, qNTX, qT, qNTC;
    float scale;
    float *Ypart;
    const int32_t *n_img, *tlen;
};

// row stride (floats) of S / W in LDS: 4 or 36 mod 64, so that the 16 rows x 4 columns of an operand hit 64 banks
__host__ __device__ constexpr int ld_rows(int k32) { return 32 * k32 + 4; }
size_t x_lds(int m, int NP)
{
    return (static_cast<size_t>(16) * ld_rows((m + 31) / 32) + 16 * (64 * NP + 4) + 4 * NP * 64 * 4 + 2 * 16 * kXW) * sizeof(float);
}
size_t x_lds_text() { return (static_cast<size_t>(16) * (kTR + 4) + 2 * 16 * kXW + 4 * 64 * 4) * sizeof(float); }

template <class T, int DT, int NP>
__global__ __launch_bounds__(64 * kXW) void gx_pass(const T *__restrict__ q, const T *__restrict__ Kc, const T *__restrict__ th,
                                                    const T *__restrict__ U, const T *__restrict__ Vc, T *__restrict__ Kt,
                                                    T *__restrict__ Vt, const T *__restrict__ k_new, const T *__restrict__ v_new, XPlan p)
{
    constexpr int PS = 64 * NP, LDP = PS + 4;
    constexpr int KH = DT == 4 ? 2 : 1, CW = DT == 16 ? 2 : 1;     // step 4: wavefronts per channel tile, channel tiles per wavefront
    extern __shared__ __align__(16) float lds[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int r16 = lane & 15, kg = lane >> 4;
    const int G = p.G, d = p.d, n = p.n, m = p.m;
    const bool text = static_cast<int>(blockIdx.x) >= p.nvis;
    int bh, ug = 0, s = 0, tc = 0;
    if (text) {
        const int id = blockIdx.x - p.nvis;
        bh = quot(id, p.qNTX);
        tc = id - bh * p.NTX;
    } else {
        const int g = quot(blockIdx.x, p.qF);
        s = blockIdx.x - g * p.F;
        bh = quot(g, p.qNUG);
        ug = g - bh * p.NUG;
    }
    const int b = quot(bh, p.qHkv), h = bh - b * p.Hkv;
    // step 4 roles
    const int kh4 = KH == 2 ? wave >> 2 : 0, ct4 = KH == 2 ? wave & 3 : wave;

    f32x4 qf[DT];
#pragma unroll
    for (int s4 = 0; s4 < DT; ++s4) {
        const int c = 16 * s4 + 4 * kg;
        const f32x4 v = load4(q + (static_cast<size_t>(b) * p.Hq + h * G + min(r16, G - 1)) * d + min(c, d - 4));
        qf[s4] = c < d ? v : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // scores of 16 key rows (lane: row r16, channels 16 s4 + 4 kg ...): D[row][head], unscaled
    auto product = [&](const raw4<T> (&xr)[DT]) __attribute__((always_inline)) {
        f32x4 x[DT];
#pragma unroll
        for (int s4 = 0; s4 < DT; ++s4) x[s4] = Vec4<T>::wide(xr[s4]);
        f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s4 = 0; s4 < DT; ++s4) a = mfma16(x[s4], qf[s4], a);
        return a;
    };
    auto score = [&](const T *row) __attribute__((always_inline)) {
        raw4<T> x[DT];
#pragma unroll
        for (int s4 = 0; s4 < DT; ++s4) x[s4] = load4_raw(row + min(16 * s4 + 4 * kg, d - 4));
        return product(x);
    };
    // running maximum, sum and un-normalised output of row r16: image block r16 / G of a tile, or a text run's head r16
    float m_run = -INFINITY, l_run = 0.f;
    f32x4 y[CW];
#pragma unroll
    for (int c = 0; c < CW; ++c) y[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto advance = [&](float mx, float sm, const f32x4 (&o)[CW]) __attribute__((always_inline)) {
        const float mn = fmaxf(m_run, mx), mref = mn == -INFINITY ? 0.f : mn, ca = __expf(m_run - mref), cb = __expf(mx - mref);
#pragma unroll
        for (int c = 0; c < CW; ++c) y[c] = y[c] * ca + o[c] * cb;
        l_run = l_run * ca + sm * cb;
        m_run = mn;
    };

    if (text) {
        float *sP = lds;                                  // weights [16 heads][kTR + 4]
        float *sRed = lds + 16 * (kTR + 4);               // maxima, sums [16][kXW]
        const bool fresh = k_new != nullptr;
        int t_in = p.t_in, t = p.t;
        if (p.tlen) {
            const int tlb = max(p.tlen[b], 0);
            t_in = min(tlb, p.t_in);
            t = fresh ? t_in + 1 : min(tlb, p.t);
        }
        const T *kn = fresh ? k_new + static_cast<size_t>(bh) * d : q, *vn = fresh ? v_new + static_cast<size_t>(bh) * d : q;
        T *Ktb = Kt + static_cast<size_t>(bh) * p.cap * d, *Vtb = Vt + static_cast<size_t>(bh) * p.cap * d;
        const int t_new = fresh ? t_in : -1;
        for (int x0 = tc * kTR; x0 < t; x0 += kTR * p.NTC) {       // (a run that a shorter sequence does not have: nothing)
            const int xr = min(x0 + 16 * wave + r16, t - 1);
            const f32x4 a = score(xr == t_new ? kn : Ktb + static_cast<size_t>(xr) * d);
            f32x4 l;
            float mx = -INFINITY;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                l[e] = x0 + 16 * wave + 4 * kg + e < t ? a[e] * p.scale : -INFINITY;
                mx = fmaxf(mx, l[e]);
            }
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            if (kg == 0) sRed[r16 * kXW + wave] = mx;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < kXW; ++w) mx = fmaxf(mx, sRed[r16 * kXW + w]);      // finite: the step has a row
            float sm = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                l[e] = __expf(l[e] - mx);
                sm += l[e];
            }
            *reinterpret_cast<f32x4 *>(sP + r16 * (kTR + 4) + 16 * wave + 4 * kg) = l;
            sm += __shfl_xor(sm, 16, 64);
            sm += __shfl_xor(sm, 32, 64);
            if (kg == 0) sRed[16 * kXW + r16 * kXW + wave] = sm;
            __syncthreads();
            sm = 0.f;
#pragma unroll
            for (int w = 0; w < kXW; ++w) sm += sRed[16 * kXW + r16 * kXW + w];
            f32x4 o[CW];
#pragma unroll
            for (int c = 0; c < CW; ++c) o[c] = f32x4{0.f, 0.f, 0.f, 0.f};
            const int steps = (min(t - x0, kTR) + 15) / 16;
            for (int k = kh4; k < steps; k += KH) {
                const f32x4 w = *reinterpret_cast<const f32x4 *>(sP + r16 * (kTR + 4) + 16 * k + 4 * kg);
#pragma unroll
                for (int c = 0; c < CW; ++c) {
                    const int cc = min(16 * (ct4 + kXW * c) + r16, d - 1);
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int x = min(x0 + 16 * k + 4 * kg + e, t - 1);
                        v[e] = to_f((x == t_new ? vn : Vtb + static_cast<size_t>(x) * d)[cc]);
                        v[e] = x0 + 16 * k + 4 * kg + e < t ? v[e] : 0.f;
                    }
                    o[c] = mfma16(v, w, o[c]);
                }
            }
            advance(mx, sm, o);
            __syncthreads();                              // the weights have been read
        }
        // Sec. 3.2: the text cache keeps growing as in the backbone -- store the new token's k, v
        const int own = t_in / kTR;
        if (fresh && own - quot(own, p.qNTC) * p.NTC == tc)
            for (int c = threadIdx.x; c < d; c += 64 * kXW) {
                Ktb[static_cast<size_t>(t_in) * d + c] = kn[c];
                Vtb[static_cast<size_t>(t_in) * d + c] = vn[c];
            }
    } else {
        const int LDM = ld_rows(p.KB), TT = 2 * p.KB, p0 = s * PS;
        float *sS = lds, *sP = sS + 16 * LDM, *sX = sP + 16 * LDP, *sRed = sX + 4 * NP * 64 * 4;     // W takes the place of S
        const T *th_b = th + static_cast<size_t>(h) * m * n, *u_b = U + static_cast<size_t>(h) * m * n;
        const int n_img = p.n_img ? min(max(p.n_img[b], 0), p.I) : p.I;
        for (int ut = 0; ut < p.NUT; ++ut) {
            const int i0 = (ug * p.NUT + ut) * p.UP, nu = min(p.UP, n_img - i0);
            if (nu <= 0) break;                           // the same for the whole workgroup
            const T *kc_b = Kc + (static_cast<size_t>(bh) * p.I + i0) * m * d, *vc_b = Vc + (static_cast<size_t>(bh) * p.I + i0) * m * d;
            // (what follows depends on the lane, not on the tile: kept from being moved in front of the loop, where its
            // addresses would take up registers throughout)
            int lane_l = lane;
            asm volatile("" : "+v"(lane_l));
            const int r16 = lane_l & 15, kg = lane_l >> 4;
            const int tg = wave & 3, kh = wave >> 2;      // step 2: position tiles tg + 4 i, every other 32 rows j
            int pos[NP];
#pragma unroll
            for (int i = 0; i < NP; ++i) pos[i] = min(p0 + 16 * (tg + 4 * i) + r16, n - 1);
            auto load_tile = [&](int it, raw4<T> (&x)[DT]) __attribute__((always_inline)) {
                const int u = quot(it, p.qT), jt = it - u * TT;
                const T *base = kc_b + static_cast<size_t>(u) * m * d;
#pragma unroll
                for (int s4 = 0; s4 < DT; ++s4) x[s4] = load4_raw(at(base, static_cast<uint32_t>(min(16 * jt + r16, m - 1) * d + min(16 * s4 + 4 * kg, d - 4))));
            };
            auto load_theta = [&](int k, T (&x)[8][NP]) __attribute__((always_inline)) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
#pragma unroll
                    for (int i = 0; i < NP; ++i) x[e][i] = *at(th_b, static_cast<uint32_t>(min(32 * k + 4 * e + kg, m - 1) * n + pos[i]));
            };
            auto load_u = [&](int jt, raw4<T> (&x)[PS / 16]) __attribute__((always_inline)) {
#pragma unroll
                for (int k = 0; k < PS / 16; ++k)
                    x[k] = load4_raw(at(u_b, static_cast<uint32_t>(min(16 * jt + r16, m - 1) * n + min(p0 + 16 * k + 4 * kg, n - 4))));
            };
            const int sfull = m >> 4, send = (m + 15) >> 4;      // step 4: 16-row steps inside full 8-row blocks, all steps
            auto value = [&](const T *rec, int k, int c) __attribute__((always_inline)) {
                const int cc = min(16 * (ct4 + kXW * c) + r16, d - 1);
                return at(rec, static_cast<uint32_t>((2 * k + (kg >> 1)) * 8 * d + cc * 8 + 4 * (kg & 1)));
            };
            // ---- step 1: S = q Kc^T
            auto store_scores = [&](int it, f32x4 a) __attribute__((always_inline)) {
                const int u = quot(it, p.qT), jt = it - u * TT, j = 16 * jt + 4 * kg;
#pragma unroll
                for (int e = 0; e < 4; ++e) a[e] = j + e < m ? a[e] : 0.f;
                if (r16 < G) *reinterpret_cast<f32x4 *>(sS + (u * G + r16) * LDM + j) = a;
            };
            for (int it = wave; it < nu * TT; it += kXW) {
                raw4<T> x[DT];
                load_tile(it, x);
                store_scores(it, product(x));
            }
            lds_barrier();
            // ---- step 2: L^T[pos][row] = sum_j theta[j][pos] S[row][j]
            f32x4 aL[NP];
#pragma unroll
            for (int i = 0; i < NP; ++i) aL[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            auto theta_step = [&](int k, const T (&x)[8][NP]) __attribute__((always_inline)) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float sv = sS[r16 * LDM + 32 * k + 4 * e + kg];
#pragma unroll
                    for (int i = 0; i < NP; ++i) aL[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(to_f(x[e][i]), sv, aL[i], 0, 0, 0);
                }
            };
            for (int k = kh; k < p.KB; k += 2) {
                T x[8][NP];
                load_theta(k, x);
                theta_step(k, x);
            }
            if (kh == 1) {
#pragma unroll
                for (int i = 0; i < NP; ++i) *reinterpret_cast<f32x4 *>(sX + ((tg + 4 * i) * 64 + lane) * 4) = aL[i];
            }
            lds_barrier();
            float mx = -INFINITY;
            if (kh == 0) {
#pragma unroll
                for (int i = 0; i < NP; ++i) {
                    aL[i] += *reinterpret_cast<const f32x4 *>(sX + ((tg + 4 * i) * 64 + lane) * 4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        aL[i][e] = p0 + 16 * (tg + 4 * i) + 4 * kg + e < n ? aL[i][e] * p.scale : -INFINITY;
                        mx = fmaxf(mx, aL[i][e]);
                    }
                }
                mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
                mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
                if (kg == 0) sRed[r16 * kXW + tg] = mx;
            }
            lds_barrier();
            {
                const f32x4 a = *reinterpret_cast<const f32x4 *>(sRed + r16 * kXW);
                mx = fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3]));
            }
            if (kh == 0) {
                float sm = 0.f;
#pragma unroll
                for (int i = 0; i < NP; ++i) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        aL[i][e] = __expf(aL[i][e] - mx);
                        sm += aL[i][e];
                    }
                    *reinterpret_cast<f32x4 *>(sP + r16 * LDP + 16 * (tg + 4 * i) + 4 * kg) = aL[i];
                }
                sm += __shfl_xor(sm, 16, 64);
                sm += __shfl_xor(sm, 32, 64);
                if (kg == 0) sRed[16 * kXW + r16 * kXW + tg] = sm;
            }
            lds_barrier();
            float sm;
            {
                const f32x4 a = *reinterpret_cast<const f32x4 *>(sRed + 16 * kXW + r16 * kXW);
                sm = (a[0] + a[1]) + (a[2] + a[3]);
            }
            // ---- step 3: W^T[j][row] = sum_pos U[j][pos] P[row][pos]
            auto u_tile = [&](int jt, const raw4<T> (&x)[PS / 16]) __attribute__((always_inline)) {
                f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < PS / 16; ++k)
                    a = mfma16(past_end(Vec4<T>::wide(x[k]), p0 + 16 * k + 4 * kg, n),
                               *reinterpret_cast<const f32x4 *>(sP + r16 * LDP + 16 * k + 4 * kg), a);
                const int j = 16 * jt + 4 * kg;
#pragma unroll
                for (int e = 0; e < 4; ++e) a[e] = j + e < m ? a[e] : 0.f;
                *reinterpret_cast<f32x4 *>(sS + r16 * LDM + j) = a;
            };
            for (int jt = wave; jt < TT; jt += kXW) {
                raw4<T> x[PS / 16];
                load_u(jt, x);
                u_tile(jt, x);
            }
            lds_barrier();
            // ---- step 4: Y^T[c][row] = sum_j Vc^T[c][j] W[row][j]; of a block's product the rows of that block are taken
            f32x4 o[CW], yu[CW];
#pragma unroll
            for (int c = 0; c < CW; ++c) o[c] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int u = 0; u < nu; ++u) {
                const bool mine = r16 >= u * G && r16 < (u + 1) * G;
                const T *rec = vc_b + static_cast<size_t>(u) * m * d;
                auto weights = [&](int k) __attribute__((always_inline)) { return *reinterpret_cast<const f32x4 *>(sS + r16 * LDM + 16 * k + 4 * kg); };
#pragma unroll
                for (int c = 0; c < CW; ++c) yu[c] = f32x4{0.f, 0.f, 0.f, 0.f};
                int k = kh4;
                // (four steps at a time: their loads together)
                for (; k + 3 * KH < sfull; k += 4 * KH) {
                    raw4<T> x[4][CW];
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int c = 0; c < CW; ++c) x[r][c] = load4_raw(value(rec, k + KH * r, c));
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const f32x4 w = weights(k + KH * r);
#pragma unroll
                        for (int c = 0; c < CW; ++c) yu[c] = mfma16(Vec4<T>::wide(x[r][c]), w, yu[c]);
                    }
                }
                for (; k < sfull; k += KH) {
                    const f32x4 w = weights(k);
#pragma unroll
                    for (int c = 0; c < CW; ++c) yu[c] = mfma16(load4(value(rec, k, c)), w, yu[c]);
                }
                if (sfull < send && (KH == 1 || (sfull & 1) == kh4)) {
                    const f32x4 w = weights(sfull);
#pragma unroll
                    for (int c = 0; c < CW; ++c) {
                        const int cc = min(16 * (ct4 + kXW * c) + r16, d - 1);
                        f32x4 v;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int j = 16 * sfull + 4 * kg + e;
                            v[e] = j < m ? to_f(rec[vc_offset(min(j, m - 1), cc, m, d)]) : 0.f;
                        }
                        yu[c] = mfma16(v, w, yu[c]);
                    }
                }
#pragma unroll
                for (int c = 0; c < CW; ++c)
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[c][e] = mine ? yu[c][e] : o[c][e];
            }
            if (r16 < nu * G) advance(mx, sm, o);         // rows of the tile that hold no image block keep their state
            lds_barrier();                              // W and P have been read
        }
    }

    // ---- one record: the rows u G + g of a query head together, the two halves of the contraction too
    const int NU = text ? 1 : p.UP;
    float gm = -INFINITY;
    for (int u = 0; u < NU; ++u) gm = fmaxf(gm, __shfl(m_run, (lane & 48) | min(u * G + r16, 15), 64));
    const float mref = gm == -INFINITY ? 0.f : gm;        // nothing at all: a record without mass
    f32x4 yo[CW];
    float lo = 0.f;
#pragma unroll
    for (int c = 0; c < CW; ++c) yo[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int u = 0; u < NU; ++u) {
        const int src = (lane & 48) | min(u * G + r16, 15);
        const float w = __expf(__shfl(m_run, src, 64) - mref);
#pragma unroll
        for (int c = 0; c < CW; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) yo[c][e] += w * __shfl(y[c][e], src, 64);
        lo += w * __shfl(l_run, src, 64);
    }
    if constexpr (KH == 2) {
        float *sY = lds;                                  // nothing else is live
        if (kh4 == 1) *reinterpret_cast<f32x4 *>(sY + (ct4 * 64 + lane) * 4) = yo[0];
        __syncthreads();
        if (kh4 == 1) return;
        yo[0] += *reinterpret_cast<const f32x4 *>(sY + (ct4 * 64 + lane) * 4);
    }
    if (r16 < G) {
        float *yp = p.Ypart + (static_cast<size_t>(bh) * p.nparts + (text ? p.NUG * p.F + tc : ug * p.F + s)) * p.rec;
#pragma unroll
        for (int c = 0; c < CW; ++c) {
            const int c0 = 16 * (ct4 + kXW * c) + 4 * kg;
            if (c0 < d) *reinterpret_cast<f32x4 *>(yp + r16 * d + c0) = yo[c];
        }
        if (wave == 0 && kg == 0) {
            yp[G * d + r16] = gm;
            yp[G * d + G + r16] = lo;
        }
    }
}

// joint softmax over the part records of one (batch element, query head); a lane per part
template <class T>
__global__ __launch_bounds__(256) void gx_merge(const float *__restrict__ Ypart, const T *__restrict__ mu, T *__restrict__ out,
                                                float *__restrict__ lse, int Hkv, int G, int d, int np, int nvp, int rec)
{
    __shared__ float sY[256];
    const int Hq = Hkv * G, bg = blockIdx.x, b = bg / Hq, hq = bg - b * Hq, h = hq / G, g = hq - h * G;
    const int lane = threadIdx.x & 63;
    const float *yb = Ypart + static_cast<size_t>(b * Hkv + h) * np * rec;
    const int pl = min(lane, np - 1);
    float ml = yb[static_cast<size_t>(pl) * rec + G * d + g], sl = yb[static_cast<size_t>(pl) * rec + G * d + G + g];
    if (lane >= np) { ml = -INFINITY; sl = 0.f; }
    const float mx = wave_max(ml), a = __expf(ml - mx);   // zero beyond the last part
    const float z = wave_sum(sl * a), zv = wave_sum(lane < nvp ? sl * a : 0.f), rz = 1.f / z, wgt = a * rz;
    // threads: channel, and a share of the parts where the channels leave some over
    const int SL = 256 / d, c = threadIdx.x % d, sh = threadIdx.x / d;
    float y = 0.f;
    for (int k0 = 0; k0 < np; k0 += SL) {
        const int k = k0 + sh;                            // (every lane takes part in the exchange)
        const float w = __shfl(wgt, min(k, np - 1), 64);
        if (k < np && sh < SL) y += w * yb[static_cast<size_t>(k) * rec + g * d + c];
    }
    sY[threadIdx.x] = y;
    __syncthreads();
    if (static_cast<int>(threadIdx.x) < d) {
        for (int k = 1; k < SL; ++k) y += sY[k * d + c];
        if (nvp > 0) y += (zv * rz) * to_f(mu[static_cast<size_t>(h) * d + c]);
        out[static_cast<size_t>(bg) * d + c] = from_f<T>(y);
    }
    if (threadIdx.x == 0 && lse) lse[bg] = mx + __logf(z);
}

constexpr size_t kXLds = 156 * 1024;

// What decides the order of the sums follows from the shape and the capacity of the text cache, not from the rows that it
// holds: a ragged batch equals the uniform call bit for bit.
bool make_xplan(XPlan &p, const kvc_shape &s, int t, int t_in, int cap)
{
    p.B = s.batch; p.Hq = s.n_q_heads; p.Hkv = s.n_kv_heads; p.G = p.Hq / p.Hkv;
    p.I = s.n_images; p.n = s.n_img_tokens; p.m = s.m; p.d = s.head_dim; p.KB = (s.m + 31) / 32;
    p.t = t; p.t_in = t_in; p.cap = cap;
    if (p.G > 16 || p.n < 4) return false;
    const long bh = static_cast<long>(p.B) * p.Hkv;
    // narrow slices spread a small call over the chip; wide ones read the keys and values less often, taken as soon
    // as they leave two workgroups per compute unit.  Smaller tiles spread it further, as long as every workgroup keeps one
    // tile: beyond the part records that the merge takes they would follow each other in the same workgroups (us per layer,
    // B = 1, d = 64: 8/2 heads, 16 blocks of n = 576 one tile of four 36.7, four of one 51.6; 14/2, 4 of 1024 34.9 / 43.0).
    p.UP = std::max(1, std::min(16 / p.G, p.I));
    auto groups = [&](int up) { return bh * ((p.I + up - 1) / up); };
    p.NP = groups(p.UP) * ((p.n + 255) / 256) >= 512 ? 4 : 1;
    if ((p.n + 63) / 64 > kVisParts) p.NP = 4;
    if (p.NP == 1)
        for (int up = (p.UP + 1) / 2; p.UP > 1 && groups(p.UP) * ((p.n + 63) / 64) < 256 && (p.I + up - 1) / up * ((p.n + 63) / 64) <= kVisParts;
             up = (p.UP + 1) / 2)
            p.UP = up;
    p.F = (p.n + 64 * p.NP - 1) / (64 * p.NP);
    if (p.F > kVisParts || x_lds(p.m, p.NP) > kXLds) return false;
    const int tiles = (p.I + p.UP - 1) / p.UP, ug_max = kVisParts / p.F;
    p.NUT = p.I > 0 ? (tiles + ug_max - 1) / ug_max : 1;
    p.NUG = p.I > 0 ? (tiles + p.NUT - 1) / p.NUT : 0;
    p.nvis = static_cast<int>(std::min(bh * p.NUG * p.F, 1l << 30));
    const int full = (cap + kTR - 1) / kTR, each = std::max(1, (full + kTextParts - 1) / kTextParts);
    p.NTC = std::max(1, (full + each - 1) / each);
    p.NTX = std::min((t + kTR - 1) / kTR, p.NTC);
    p.qNTC = quot_multiplier(p.NTC);
    p.nparts = p.NUG * p.F + p.NTX;
    p.rec = static_cast<int>(align_up(p.G * p.d + 2 * p.G, 4));
    p.qF = quot_multiplier(p.F); p.qNUG = quot_multiplier(p.NUG); p.qHkv = quot_multiplier(p.Hkv);
    p.qNTX = quot_multiplier(p.NTX); p.qT = quot_multiplier(2 * p.KB);
    p.n_img = p.tlen = nullptr;
    // quot(): dividends below 2^32 / divisor
    const long lim = 1l << 31;
    return p.nparts >= 1 && bh * std::max(p.NUG, 1) * p.F * std::max({p.F, p.NUG, p.Hkv}) < lim &&
           bh * std::max(p.NTX, 1) * std::max(p.NTX, p.Hkv) < lim && static_cast<long>(16) * 2 * p.KB * 2 * p.KB < lim;
}

template <class T, int DT, int NP> bool launch_x2(const XPlan &p, const DecodeCall &c)
{
    static bool attr_set[kMaxDevices] = {};
    if (!allow_lds(reinterpret_cast<const void *>(gx_pass<T, DT, NP>), kXLds, attr_set)) return false;
    gx_pass<T, DT, NP><<<p.nvis + p.B * p.Hkv * p.NTX, 64 * kXW, std::max(x_lds(p.m, NP), x_lds_text()), c.stream>>>(
        static_cast<const T *>(c.q), static_cast<const T *>(c.Kc), static_cast<const T *>(c.theta), static_cast<const T *>(c.U),
        static_cast<const T *>(c.Vc), static_cast<T *>(c.Kt), static_cast<T *>(c.Vt), static_cast<const T *>(c.k_new),
        static_cast<const T *>(c.v_new), p);
    return true;
}
template <class T> bool launch_x(const XPlan &p, const DecodeCall &c)
{
    if (p.d <= 64) return p.NP == 4 ? launch_x2<T, 4, 4>(p, c) : launch_x2<T, 4, 1>(p, c);
    if (p.d <= 128) return p.NP == 4 ? launch_x2<T, 8, 4>(p, c) : launch_x2<T, 8, 1>(p, c);
    return p.NP == 4 ? launch_x2<T, 16, 4>(p, c) : launch_x2<T, 16, 1>(p, c);
}

template <class T, int DT> bool launch_p(const XProj &p, const CompressCall &c, int grid)
{
    constexpr size_t lds = static_cast<size_t>(kXW) * 16 * (16 * DT + 4) * sizeof(float);
    static bool attr_set[kMaxDevices] = {};
    if (!allow_lds(reinterpret_cast<const void *>(gx_project<T, DT>), lds, attr_set)) return false;
    gx_project<T, DT><<<grid, 64 * kXW, lds, c.stream>>>(static_cast<const T *>(c.K), static_cast<const T *>(c.V), c.key_idx,
                                                         static_cast<const T *>(c.U), static_cast<const T *>(c.mu),
                                                         static_cast<T *>(c.Kc), static_cast<T *>(c.Vc), p);
    return true;
}
template <class T> bool launch_project(const XProj &p, const CompressCall &c, int grid)
{
    return p.d <= 64 ? launch_p<T, 4>(p, c, grid) : p.d <= 128 ? launch_p<T, 8>(p, c, grid) : launch_p<T, 16>(p, c, grid);
}

}  // namespace

bool float_compress(const CompressCall &c, kvc_status *st)
{
    const kvc_shape &s = c.s;
    if (s.n_img_tokens < 4 || s.n_images == 0) return false;
    // Many very short blocks stay on the scalar kernel: a workgroup here costs the same for them, and the more LDS its sums
    // take the fewer of them a compute unit holds (4, 2, 1).  us per call, scalar against this, 5120 blocks: d = 64, n = 8, m = 2
    // 13.8 / 23.0, n = 16, m = 5 27.4 / 22.8; d = 128 39.6 / 41.6 there, n = 24, m = 8 70.7 / 56.5; d = 256, n = 24 102 / 139,
    // n = 32, m = 10 168 / 166; 576 blocks (2.3 rounds at d = 256) n = 17 16.0 / 18.3, n = 24 24.8 / 18.9; 8 blocks, d = 256,
    // n = 8 5.6 / 6.0, n = 16 9.1 / 5.8.
    {
        const long wgs = static_cast<long>(s.batch) * s.n_kv_heads * s.n_images * ((s.m + 15) / 16);
        const long round = 256 * (s.head_dim <= 64 ? 4 : s.head_dim <= 128 ? 2 : 1);
        const int chain = scalar_chain(s.n_img_tokens, s.m);
        const int least = s.head_dim <= 64 ? 16 : s.head_dim <= 128 ? (wgs > 8 * round ? 20 : 16) : wgs > 8 * round ? 48 : 24;
        if (chain < (wgs > round ? least : s.head_dim > 128 ? 12 : 0)) return false;
    }
    XProj p;
    p.Hkv = s.n_kv_heads; p.n = s.n_img_tokens; p.m = s.m; p.I = s.n_images; p.d = s.head_dim; p.vis0 = c.vis_start;
    p.sb = c.stride_b; p.sh = c.stride_h; p.ss = c.stride_s;
    p.JT = (p.m + 15) / 16;
    const long grid = static_cast<long>(s.batch) * p.Hkv * p.I * p.JT;
    if (grid > 0x7fffffffl) return false;
    const bool ok = s.dtype == KVC_F32 ? launch_project<float>(p, c, static_cast<int>(grid)) : launch_project<bf16_t>(p, c, static_cast<int>(grid));
    *st = ok && hipGetLastError() == hipSuccess ? KVC_OK : KVC_ERR_HIP;
    return true;
}

// the largest number of part records a call of this shape writes
size_t float_decode_ws_bytes(const kvc_shape &s, int32_t max_text)
{
    XPlan p;
    if (!make_xplan(p, s, std::max(max_text, 1), 0, std::max(max_text, 1))) return 0;
    const int ntx = std::min((std::max(max_text, 1) + kTR - 1) / kTR, kTextParts);
    return dd::kCounterBytes + static_cast<size_t>(p.B) * p.Hkv * (p.NUG * p.F + ntx) * p.rec * sizeof(float);
}

bool float_decode_plan(const kvc_shape &s, int t, int cap, int32_t *plan)
{
    XPlan p;
    if (!make_xplan(p, s, t, t, cap)) return false;
    const int32_t v[8] = {64 * p.NP, p.UP, p.NUT, p.F, p.nvis, p.NTX, (cap + kTR * kTextParts - 1) / (kTR * kTextParts), 0};
    std::copy(v, v + 8, plan);
    return true;
}

bool float_decode(const DecodeCall &c, kvc_status *st)
{
    if (c.static_variant || (c.n_images_dev == nullptr) != (c.text_len_dev == nullptr)) return false;
    XPlan p;
    if (!make_xplan(p, c.s, c.t, c.t_in, c.cap)) return false;
    if (dd::kCounterBytes + static_cast<size_t>(p.B) * p.Hkv * p.nparts * p.rec * sizeof(float) > c.ws_bytes) return false;
    p.scale = c.scale;
    p.Ypart = reinterpret_cast<float *>(static_cast<char *>(c.ws) + dd::kCounterBytes);
    p.n_img = c.n_images_dev; p.tlen = c.text_len_dev;
    const bool f32 = c.s.dtype == KVC_F32;
    if (!(f32 ? launch_x<float>(p, c) : launch_x<bf16_t>(p, c)) || hipGetLastError() != hipSuccess) { *st = KVC_ERR_HIP; return true; }
    if (f32)
        gx_merge<float><<<p.B * p.Hq, 256, 0, c.stream>>>(p.Ypart, static_cast<const float *>(c.mu), static_cast<float *>(c.out), c.lse,
                                                         p.Hkv, p.G, p.d, p.nparts, p.NUG * p.F, p.rec);
    else
        gx_merge<bf16_t><<<p.B * p.Hq, 256, 0, c.stream>>>(p.Ypart, static_cast<const bf16_t *>(c.mu), static_cast<bf16_t *>(c.out),
                                                          c.lse, p.Hkv, p.G, p.d, p.nparts, p.NUG * p.F, p.rec);
    *st = hipGetLastError() == hipSuccess ? KVC_OK : KVC_ERR_HIP;
    return true;
}

}  // namespace kvc
