// Device code shared by the decode kernels that keep scores and weights at float32 precision
// (kvc_static_decode.hip, kvc_any_decode.hip): a float as three bf16 terms, and one wavefront's pass over rows
// that are attended as they are -- compressed rows or rows of the text cache.
#pragma once
#include "kvc_decode_dev.h"

namespace kvc {
namespace rows {

using namespace dd;

constexpr int kSW = 4;                // wavefronts
constexpr int kSR = 32;               // rows per wavefront and step
constexpr int kLDO = D + 4;           // floats per head row of a wavefront's output in LDS
constexpr int kWalkLds = 16 * kLDO * 4;       // a wavefront's LDS: its tile of 32 rows of values, then its output rows
static_assert(kWalkLds >= kSR * D * 2 && kWalkLds % 256 == 0, "32 rows of 256 bytes, whole passes over the banks");

// what walk() needs to know of a sequence's rows
struct Rows {
    int I, m, KS, SV;                 // compressed rows: blocks of m rows, KS 32-row steps each, SV = I KS steps
    int t;                            // rows of the text cache
    int cs, ws, st;                   // steps per wavefront and run, at most; distance between wavefronts' first steps; between steps
    unsigned qKS, qst;
    float scale;
};

// p = p1 + p2 + p3, each a bf16: the high parts are exact remainders
struct Split3 {
    bf16x8 a, b, c;
};
__device__ __forceinline__ Split3 split3(const float (&p)[8])
{
    uint32_t w[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float x0 = p[2 * i], x1 = p[2 * i + 1];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const uint32_t h0 = f32_to_bf16_bits(x0), h1 = f32_to_bf16_bits(x1);
            w[k][i] = h0 | (h1 << 16);
            x0 -= __uint_as_float(h0 << 16);
            x1 -= __uint_as_float(h1 << 16);
        }
    }
    Split3 r;
    r.a = as_bf16x8(u32x4_mk(w[0][0], w[0][1], w[0][2], w[0][3]));
    r.b = as_bf16x8(u32x4_mk(w[1][0], w[1][1], w[1][2], w[1][3]));
    r.c = as_bf16x8(u32x4_mk(w[2][0], w[2][1], w[2][2], w[2][3]));
    return r;
}

// the first n of 8 elements (n from below 0 to above 8), zeros behind
__device__ __forceinline__ u32x4 keep_elems(u32x4 v, int n)
{
    auto mask = [&](int i) { return n >= 2 * i + 2 ? 0xffffffffu : n == 2 * i + 1 ? 0xffffu : 0u; };
    return u32x4_mk(v.x & mask(0), v.y & mask(1), v.z & mask(2), v.w & mask(3));
}
// Infinities and NaNs become the largest finite value of their sign.  For the products with the second and third term of a
// weight: these may be zero or of the other sign, and 0 * Inf or Inf - Inf would make a NaN of what is an infinity; the
// product with the first term has the value itself.
__device__ __forceinline__ u32x4 finite_elems(u32x4 v)
{
    typedef short s16x2 __attribute__((ext_vector_type(2)));
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    auto one = [](uint32_t w) {
        const s16x2 a = __builtin_elementwise_min(__builtin_bit_cast(s16x2, w), s16x2{0x7f7f, 0x7f7f});      // bits of +max
        const u16x2 b = __builtin_elementwise_min(__builtin_bit_cast(u16x2, a), u16x2{0xff7f, 0xff7f});      // of -max
        return __builtin_bit_cast(uint32_t, b);
    };
    return u32x4_mk(one(v.x), one(v.y), one(v.z), one(v.w));
}

// One wavefront's pass over its steps of a run: s0 + wave p.ws, then every p.st-th.  TEXT: rows of the text cache, else compressed
// rows.  GUARD: infinities among the values stay infinities (see walk()).  NB: steps in flight, 2 or (half the registers) 1.
template <bool TEXT, bool GUARD, int NB>
__device__ __forceinline__ void walk_once(const Rows &p, const uint16_t *__restrict__ Kb, const uint16_t *__restrict__ Vb,
                                     const uint16_t *__restrict__ kn, const uint16_t *__restrict__ vn, int t_new,
                                     const u32x4 (&qf)[4], int s0, char *vt, float &m_run, float &l_run, f32x4 (&acc)[8])
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r16 = lane & 15, kg = lane >> 4;
    const int nfull = p.m >> 3, wt = p.m & 7;
    // Key rows of a tile are permuted: tile tt, row i holds key row 8 (i / 4) + 4 tt + i % 4 of the step.  A lane's
    // probabilities are then those of 8 consecutive rows, and a 16-byte piece of the compressed values (8 consecutive
    // rows of one channel) is the other operand as it lies in memory.
    const int krow = 8 * (r16 >> 2) + (r16 & 3);

    // step s: first row, and how many rows from there on exist (at most 32 count)
    auto rows_of = [&](int s, int &base, int &left, int &i, int &ks) {
        if constexpr (TEXT) {
            i = 0; ks = s;
            base = kSR * s; left = p.t - base;
        } else {
            const int sc = min(s, p.SV - 1);
            i = quot(sc, p.qKS); ks = sc - i * p.KS;
            base = i * p.m + kSR * ks; left = s < p.SV ? p.m - kSR * ks : 0;
        }
    };
    // loads of step s; a step past the end reads valid rows again and is masked
    auto load = [&](int s, u32x4 (&kf)[2][4], u32x4 (&vf)[8]) {
        int base, left, i, ks;
        rows_of(s, base, left, i, ks);
        const int last = TEXT ? max(p.t - 1, 0) : (i + 1) * p.m - 1;
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            const int x = min(base + krow + 4 * tt, last);
            const u32x4 *kp = reinterpret_cast<const u32x4 *>((TEXT && x == t_new) ? kn : Kb + static_cast<size_t>(x) * D) + kg;
#pragma unroll
            for (int k = 0; k < 4; ++k) kf[tt][k] = kp[4 * k];
        }
        if constexpr (TEXT) {
            // rows base + 4 k + kg, 16 lanes per row
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int x = min(base + 4 * k + kg, last);
                vf[k] = *(reinterpret_cast<const u32x4 *>(x == t_new ? vn : Vb + static_cast<size_t>(x) * D) + r16);
            }
        } else {
            // 8-row block 4 ks + kg of the record; the record's shorter last block [D][wt] is read as a dword-aligned
            // window around the lane's values (shifted into place in compute()), a block past it reads a valid one
            const char *rec = reinterpret_cast<const char *>(Vb + static_cast<size_t>(i) * p.m * D);
            const int jb = 4 * ks + kg;
            const bool tail = wt != 0 && jb == nfull;
            const uint32_t full = static_cast<uint32_t>(max(min(jb, nfull - 1), 0) * (8 * D * 2));
#pragma unroll
            for (int ct = 0; ct < 8; ++ct) {
                const int c = 16 * ct + r16;
                const uint32_t a0 = static_cast<uint32_t>(max(min(c * 2 * wt & ~3, D * 2 * wt - 16), 0));
                const uint32_t off = tail ? static_cast<uint32_t>(nfull * 8 * D * 2) + a0 : nfull ? full + c * 16 : 0u;
                vf[ct] = *reinterpret_cast<const u32x4_a4 *>(rec + off);
            }
        }
    };
    auto compute = [&](int s, const u32x4 (&kf)[2][4], u32x4 (&vf)[8]) {
        int base, left, i, ks;
        rows_of(s, base, left, i, ks);
        if constexpr (TEXT) {
            if (GUARD && left < kSR) {                           // uniform, registers only: rows past the end are zeros
#pragma unroll
                for (int k = 0; k < 8; ++k) vf[k] = keep_elems(vf[k], 4 * k + kg < left ? 8 : 0);
            }
            // rows as they lie in memory, their 32-byte pieces at piece ^ (row bits 0, 1, 3): the transposed reads of 32 lanes
            // below cover every bank once.  (Against pairs of rows packed into 32-bit words, 64 stores instead of 8: 6000 text
            // rows, 16 (batch element, KV head) pairs, 18.7 -> 14.8 us per call.)
#pragma unroll
            for (int k = 0; k < 8; ++k)
                *reinterpret_cast<u32x4 *>(vt + 1024 * k + ((kg * 256 + r16 * 16) ^ ((kg | ((k & 2) << 1)) << 5))) = vf[k];
        }
        // logits of rows base + 8 kg + 4 tt + e for head r16
        float sc[8];
#pragma unroll
        for (int tt = 0; tt < 2; ++tt) {
            f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < 4; ++k)
                a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(kf[tt][k]), as_bf16x8(qf[k]), a, 0, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) sc[4 * tt + e] = 8 * kg + 4 * tt + e < left ? a[e] * p.scale : -INFINITY;
        }
        float mx = fmaxf(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])), fmaxf(fmaxf(sc[4], sc[5]), fmaxf(sc[6], sc[7])));
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m_run, mx);
        const float mref = m_new == -INFINITY ? 0.f : m_new;     // nothing valid so far: exp(-inf - 0) = 0
        const float alpha = __expf(m_run - mref);
        m_run = m_new;
        float pr[8], ls = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            pr[e] = __expf(sc[e] - mref);
            ls += pr[e];
        }
        l_run = l_run * alpha + ls;
        const Split3 pf = split3(pr);
        if constexpr (TEXT) {
            // the wavefront reads back what its own lanes stored: LDS works through its requests in order
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_wave_barrier();
        }
        const bool tail = !TEXT && wt != 0 && 4 * ks + kg == nfull;
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) {
            u32x4 v;
            if constexpr (TEXT) {
                const char *x = vt + (8 * kg + (r16 >> 2)) * 256 + ((((r16 >> 2) | ((kg & 1) << 2)) ^ ct) << 5) + (r16 & 3) * 8;
                const u32x2 a = read_tr(x), c2 = read_tr(x + 4 * 256);
                v = u32x4_mk(a.x, a.y, c2.x, c2.y);
            } else {
                v = vf[ct];
                if (GUARD ? left < kSR : wt != 0 && ks == p.KS - 1) {        // uniform, registers only
                    const int to = (16 * ct + r16) * 2 * wt, sh = tail ? to - max(min(to & ~3, D * 2 * wt - 16), 0) : 0;
                    v = shift_window(v, sh >> 2, (sh & 2) * 8u);
                    if constexpr (GUARD) v = keep_elems(v, left - 8 * kg);
                }
            }
            f32x4 o = acc[ct];
            o[0] *= alpha; o[1] *= alpha; o[2] *= alpha; o[3] *= alpha;
            const bf16x8 f = as_bf16x8(GUARD ? finite_elems(v) : v);
            o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, pf.c, o, 0, 0, 0);
            o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, pf.b, o, 0, 0, 0);
            acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(v), pf.a, o, 0, 0, 0);
        }
        if constexpr (TEXT) __builtin_amdgcn_wave_barrier();
    };

    // Two steps in flight in two register sets.  No step is requested that the run does not have: with runs of one or
    // two steps a request ahead of the end would double what the kernel reads.
    const int all = TEXT ? (p.t + kSR - 1) / kSR : p.SV;
    const int sw = s0 + wave * p.ws;
    const int ST = p.st, left_w = all - sw, N = left_w > 0 ? min(quot(left_w + ST - 1, p.qst), p.cs) : 0;
    if (N == 0) return;
    u32x4 kA[2][4], vA[8];
    load(sw, kA, vA);
    if constexpr (NB == 1) {
        for (int it = 0; it < N; ++it) {
            compute(sw + ST * it, kA, vA);
            if (it + 1 < N) load(sw + ST * (it + 1), kA, vA);
        }
        return;
    }
    u32x4 kB[2][4] = {}, vB[8] = {};
    if (N > 1) load(sw + ST, kB, vB);
    int it = 0;
    for (; it + 2 < N; it += 2) {
        compute(sw + ST * it, kA, vA);
        load(sw + ST * (it + 2), kA, vA);
        compute(sw + ST * (it + 1), kB, vB);
        load(sw + ST * min(it + 3, N - 1), kB, vB);
    }
    compute(sw + ST * it, kA, vA);
    if (it + 1 < N) compute(sw + ST * (it + 1), kB, vB);
}

// The pass, from the state of an empty run.  Zero weights (rows past the end of a run repeat its last row, or its neighbour
// channel) and the lower terms of the others make NaNs of infinities among the values.  Such values are not expected, so the
// sums are looked at once, behind the pass, and where they hold a NaN the pass is repeated with the values guarded: guarding
// every step costs 5 %, the look 1.5 % (B = 16, 32/8 heads, 5 blocks of m = 231, 256 text rows: 23.9, 25.1 and 24.2 us).
template <bool TEXT, int NB = 2>
__device__ __forceinline__ void walk(const Rows &p, const uint16_t *__restrict__ Kb, const uint16_t *__restrict__ Vb,
                                     const uint16_t *__restrict__ kn, const uint16_t *__restrict__ vn, int t_new,
                                     const u32x4 (&qf)[4], int s0, char *vt, float &m_run, float &l_run, f32x4 (&acc)[8])
{
    auto start = [&]() {
        m_run = -INFINITY;
        l_run = 0.f;
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) acc[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    start();
    walk_once<TEXT, false, NB>(p, Kb, Vb, kn, vn, t_new, qf, s0, vt, m_run, l_run, acc);
    f32x4 sum = acc[0];
#pragma unroll
    for (int ct = 1; ct < 8; ++ct) sum += acc[ct];
    const float x = (sum[0] + sum[1]) + (sum[2] + sum[3]);
    if (__any(x != x)) {
        start();
        walk_once<TEXT, true, NB>(p, Kb, Vb, kn, vn, t_new, qf, s0, vt, m_run, l_run, acc);
    }
}

// The NW wavefronts of a run merge into one part record: [G][D] un-normalised output, [G] maxima, [G] sums.  sVt: kWalkLds bytes
// per wavefront.  Every thread of the workgroup calls this; those beyond the NW wavefronts only meet the barrier.
template <int NW>
__device__ __forceinline__ void merge_waves(char *sVt, float (*sM)[16], float (*sL)[16], float m_run, float l_run,
                                            const f32x4 (&acc)[8], int G, float *yp)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r16 = lane & 15, kg = lane >> 4;
    if (wave < NW) {
        l_run += __shfl_xor(l_run, 16, 64);
        l_run += __shfl_xor(l_run, 32, 64);
        float *fo = reinterpret_cast<float *>(sVt + wave * kWalkLds);     // [16 heads][kLDO]
#pragma unroll
        for (int ct = 0; ct < 8; ++ct) *reinterpret_cast<f32x4 *>(fo + r16 * kLDO + 16 * ct + 4 * kg) = acc[ct];
        if (kg == 0) { sM[wave][r16] = m_run; sL[wave][r16] = l_run; }
    }
    __syncthreads();
    if (wave >= NW) return;
    for (int idx = threadIdx.x; idx < G * (D / 4); idx += 64 * NW) {
        const int g = idx / (D / 4), c4 = (idx - g * (D / 4)) * 4;
        float M = sM[0][g];
#pragma unroll
        for (int w = 1; w < NW; ++w) M = fmaxf(M, sM[w][g]);
        const float mref = M == -INFINITY ? 0.f : M;
        f32x4 y = {0.f, 0.f, 0.f, 0.f};
        float l = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float a = __expf(sM[w][g] - mref);
            const f32x4 o = *reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(sVt + w * kWalkLds) + g * kLDO + c4);
            y[0] += a * o[0]; y[1] += a * o[1]; y[2] += a * o[2]; y[3] += a * o[3];
            l += a * sL[w][g];
        }
        *reinterpret_cast<f32x4 *>(yp + g * D + c4) = y;
        if (c4 == 0) {
            yp[G * D + g] = M;
            yp[G * D + G + g] = l;
        }
    }
}

}  // namespace rows
}  // namespace kvc
