// Row-wise GEMM + TopK with the score tile resident in registers, for gfx950
// and key heads of up to 4096 chunks (RouteRelay, arXiv 2609.07306).
//
// Callers: MODE_FULL (Eq. (1)-(2)), MODE_ANCHOR (full routing plus the ledger
// build of Sec. 3.1) and MODE_RELAY (the whole relay layer of Sec. 3.2 in one
// launch: rescoring, trigger, and the routing of the flagged rows).
//
// A workgroup of NW waves owns 32 query rows of one head.  The padded key
// range is cut into 2 NW segments of 16 nb keys; at stage st wave w multiplies
// the 32-key tile made of keys 16 st .. 16 st + 15 of segments 2w and 2w+1
// (A = keys, B = queries), so that lane (row, hh) ends with 16 consecutive
// scores of segment 2w + hh.  All nb <= KT stages keep their accumulators:
// the tile's scores stay in registers (16 KT per lane, the 512 KB register
// file of a compute unit holds two tiles of 32 x 1024), so the threshold, the
// collection and a relay's rescoring read them there and every product is
// formed once.  (A tile that sweeps the keys twice spends more on the second
// sweep's barriers and stores than on its products.)  A wave's keys are its
// own: they go global -> registers a stage ahead and registers -> the wave's
// own LDS rows, with no workgroup barrier in the sweep.
//
// More than 2048 keys are swept in panels (P = 3, of up to 1536 keys on eight
// waves of six stages): after each panel the row's bound is raised over the
// panel's group maxima and the candidates so far, and the list is rewritten from
// both, so what follows sees one list.  A relay's trigger is known after the last
// panel only; before it every row keeps a list.  The LDS holds key rows and lists
// side by side then, with the staging in the key rows' place after the last
// sweep.  Six stages and one stage in flight instead of eight and two, because a
// register spilled in the sweep is reloaded behind the keys in flight and waits
// for them (two panels of eight stages: 7100 cycles a stage, three of six: 3400).
// Long-context schedule (32 heads x 4096, causal, bf16, T = 96): 2653 us with the
// two-sweep tiles, 2024 us.
//
// Selecting the T = k + m best of a row:
//   1. bound: per lane and register slot the maximum over the stages, so a
//      row has 32 NW group maxima.  Any v with at least T maxima >= v is at
//      most the T-th score; a few bisection steps over the maxima, 2 NW
//      adjacent lanes per row (DPP reductions), give a v that few more than T
//      scores reach.
//   2. collection: a lane counts its scores >= v, takes its place in the row's
//      list by one LDS add, and appends (score, id) in any order.  A row with
//      more candidates than its list holds raises v by bisection on the
//      order-preserving integer image of the scores, then cuts its ties by id:
//      counts over registers, every wave following all 32 rows.
//   3. selection, 2 NW adjacent lanes per row, the row's lanes in one wave
//      (no barrier from here on): a bitonic network over the lanes sorts the
//      candidates' scores for the k-th and T-th; R and N become bitmaps over
//      the keys, whose prefix counts give each chosen id its place in
//      ascending order.
//   4. the random sentinels, a row's slots hashed in parallel: every slot
//      proposes its first probe outside the bitmaps, and a slot whose chunk an
//      earlier slot proposes too moves to its next probe, until none does.
//      Earlier slots never yield to later ones, so this ends at the draws of
//      the slots decided one by one.
// The results leave through LDS staging in whole 16-byte pieces per row.
//
// Any float is a score that a row may have: infinities rank as what they are, a
// NaN with -inf, and the bound's overshoots (an uncut range, a rounding) only
// cost repair steps, for each row's count is checked before its list is used.
#pragma once

#include <float.h>
#include <limits.h>
#include <math.h>

#include "rr_device.hpp"
#include "rr_internal.hpp"
#include "rr_route_impl.hpp"

namespace rr {
namespace resident {

using route_detail::kMaxFixIters;
using route_detail::merge_desc;
using route_detail::sort_desc;
using route_detail::static_for;
using route_detail::transposed_row;

constexpr int kBoundRounds = 3;  // times the bound's range is cut into levels, at most
constexpr float kLeastSpan = 0x1p-100f, kMostSpan = 0x1p120f;  // widths of a range that is cut into levels
constexpr float kLowest = -FLT_MAX;  // threshold that admits every score but -inf (which masked keys hold, too)
// What th_s holds in place of a threshold's bits.  Every float is a threshold
// that a row may have, +inf too, so these are bits of NaN, and as such they are
// only compared as integers.
constexpr uint32_t kNotRouted = 0xFFFFFFFFu;  // the row is not routed by this launch
constexpr uint32_t kStopped = 0xFFFFFFFEu;    // it stopped at the sweep cap in an earlier panel: no candidate
constexpr uint32_t kNoScore = 0x7FC00000u;    // a threshold (NaN) that v_cmp_ge finds no score to reach

template <typename DT, int D, int NW, int KT, int P>
struct Shape {
    static constexpr int NT = 64 * NW, BM = 32, NSEG = 2 * NW;
    static constexpr int ROWB = D * (int)sizeof(DT);
    // a stage moves in SUB parts of at most 256 bytes per key row; part q holds
    // bytes [q RB/2, (q+1) RB/2) of each half of the row
    static constexpr int SUB = ROWB > 256 ? ROWB / 256 : 1;
    static constexpr int RB = ROWB / SUB;
    static constexpr int PR = RB / 16;        // 16-byte pieces of a row part
    static constexpr int PT = 32 * PR / 64;   // ... per lane
    static constexpr int LS = RB + 16;        // LDS row stride: an odd number of 16-byte bank groups
    static constexpr int KSTR = 36;           // row stride of the kept maxima (floats)
    static constexpr int WST = (32 * LS > 32 * KSTR * 4) ? 32 * LS : 32 * KSTR * 4;  // a wave's LDS rows
    static constexpr int LPR = NSEG;          // lanes per row after the sweep
    static constexpr int RPW = 64 / LPR;      // rows per wave
    static constexpr int CPL = P > 1 ? 12 : 16, CAP = CPL * LPR;  // candidates per lane and row
    static constexpr int LSTR = CAP * 8 + 64;        // row stride of the candidate lists (bytes)
    static constexpr int NET = 8 * LPR;              // scores the sorting network holds
    static constexpr int NWD = P > 1 ? 128 : KT * NW;  // words of a bitmap over the padded keys
    static constexpr int BW = NWD + 1;               // its row stride in word pairs
    static constexpr int WPL = NWD / LPR;            // words per lane
    // LDS of one panel: key rows or candidate lists, bitmaps, prefix counts, staging
    static constexpr int R0 = (NW * WST > BM * LSTR) ? NW * WST : BM * LSTR;
    static constexpr int OFF_BM = R0, OFF_PRE = OFF_BM + BM * BW * 8, OFF_STG = OFF_PRE + BM * NWD * 4;
    // ... of several: the lists outlive a panel, so the prefix counts and the
    // staging (needed after the last sweep) share the key rows' region instead
    __host__ __device__ static constexpr int region(int staged) { return NW * WST > BM * NWD * 4 + staged ? NW * WST : BM * NWD * 4 + staged; }
    static_assert(NWD % LPR == 0 && WPL >= 1 && PT >= 1 && OFF_STG % 16 == 0, "layout");
};

// The row's lanes read what others of them wrote to LDS: they are in one wave,
// whose LDS operations execute in order, so only the compiler must keep it.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int CTRL>
__device__ __forceinline__ int dpp(int x)
{
    return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ float dpp(float x)
{
    return __int_as_float(dpp<CTRL>(__float_as_int(x)));
}

// All-reduce over LPR (8 or 16) adjacent lanes: after the quad permutations
// the four lanes agree, so the half-row and row mirrors pair whole groups.
template <int LPR, typename T, class F>
__device__ __forceinline__ T row_all(T x, F f)
{
    x = f(x, dpp<0xB1>(x));
    x = f(x, dpp<0x4E>(x));
    x = f(x, dpp<0x141>(x));
    if (LPR == 16) x = f(x, dpp<0x140>(x));
    return x;
}
template <int LPR>
__device__ __forceinline__ int row_sum(int x)
{
    return row_all<LPR>(x, [](int a, int b) { return a + b; });
}
template <int LPR>
__device__ __forceinline__ float row_max(float x)
{
    return row_all<LPR>(x, [](float a, float b) { return fmaxf(a, b); });
}
template <int LPR>
__device__ __forceinline__ float row_min(float x)
{
    return row_all<LPR>(x, [](float a, float b) { return fminf(a, b); });
}

// Exclusive prefix sum over the row's lanes.
template <int LPR>
__device__ __forceinline__ int row_before(int x, int part)
{
    int s = x, y;
    y = dpp<0x111>(s);
    s += part >= 1 ? y : 0;
    y = dpp<0x112>(s);
    s += part >= 2 ? y : 0;
    y = dpp<0x114>(s);
    s += part >= 4 ? y : 0;
    if (LPR == 16) {
        y = dpp<0x118>(s);
        s += part >= 8 ? y : 0;
    }
    return s - x;
}

// Sorted-run merges over the row's lanes (8 scores per lane, descending, lane
// order).  keep(x, p, hi): the larger of the pair in the upper lanes (hi =
// +inf), the smaller in the lower (hi = -inf).
__device__ __forceinline__ float keep(float x, float p, float hi) { return __builtin_amdgcn_fmed3f(x, p, hi); }

template <int CTRL>
__device__ __forceinline__ void split_mirror(float (&v)[8], float hi)
{
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float x = v[q], y = v[7 - q];
        const float px = dpp<CTRL>(x), py = dpp<CTRL>(y);
        v[q] = keep(x, py, hi);
        v[7 - q] = keep(y, px, hi);
    }
}
template <int XM>
__device__ __forceinline__ float lane_xor(float x)
{
    if constexpr (XM == 1) return dpp<0xB1>(x);
    if constexpr (XM == 2) return dpp<0x4E>(x);
    return dpp<0x1B>(dpp<0x141>(x));  // 7 - lane, then reversed within the quad: lane ^ 4
}
template <int XM>
__device__ __forceinline__ void split_straight(float (&v)[8], float hi)
{
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = keep(v[q], lane_xor<XM>(v[q]), hi);
}

template <int LPR>
__device__ __forceinline__ void sort_row(float (&v)[8], int part)
{
    sort_desc<8>(v);
    const float h1 = (part & 1) ? -INFINITY : INFINITY;
    const float h2 = (part & 2) ? -INFINITY : INFINITY;
    const float h4 = (part & 4) ? -INFINITY : INFINITY;
    split_mirror<0xB1>(v, h1);
    merge_desc<8>(v);
    split_mirror<0x1B>(v, h2);
    split_straight<1>(v, h1);
    merge_desc<8>(v);
    split_mirror<0x141>(v, h4);
    split_straight<2>(v, h2);
    split_straight<1>(v, h1);
    merge_desc<8>(v);
    if constexpr (LPR == 16) {
        const float h8 = (part & 8) ? -INFINITY : INFINITY;
        split_mirror<0x140>(v, h8);
        split_straight<4>(v, h4);
        split_straight<2>(v, h2);
        split_straight<1>(v, h1);
        merge_desc<8>(v);
    }
}

// One part of a key stage as MFMA operands: lane (l32, hh) holds bytes
// [hh RB/2, (hh+1) RB/2) of LDS row l32, and the matching part of the query
// fragment follows in d order.
template <typename DT, int D, int SUB>
struct KeyPart;

template <int D, int SUB>
struct KeyPart<bf16_t, D, SUB> {
    static constexpr int NS = D / 16 / SUB;
    __device__ static __forceinline__ f32x16_t mma(const unsigned char *row, const Frag<bf16_t, D> &fq, int q, f32x16_t c)
    {
        const bf16x8_t *p = reinterpret_cast<const bf16x8_t *>(row);
        bf16x8_t f[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) f[s] = p[s];
#pragma unroll
        for (int s = 0; s < NS; ++s) c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[s], fq.v[q * NS + s], c, 0, 0, 0);
        return c;
    }
};
template <int D, int SUB>
struct KeyPart<float, D, SUB> {
    static constexpr int NS = D / 2 / SUB;
    __device__ static __forceinline__ f32x16_t mma(const unsigned char *row, const Frag<float, D> &fq, int q, f32x16_t c)
    {
        const float4 *p = reinterpret_cast<const float4 *>(row);
        float4 f[NS / 4];
#pragma unroll
        for (int s = 0; s < NS / 4; ++s) f[s] = p[s];
#pragma unroll
        for (int s = 0; s < NS / 4; ++s) {
            c = __builtin_amdgcn_mfma_f32_32x32x2f32(f[s].x, fq.v[q * NS + 4 * s], c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_32x32x2f32(f[s].y, fq.v[q * NS + 4 * s + 1], c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_32x32x2f32(f[s].z, fq.v[q * NS + 4 * s + 2], c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_32x32x2f32(f[s].w, fq.v[q * NS + 4 * s + 3], c, 0, 0, 0);
        }
        return c;
    }
};

__device__ __forceinline__ uint32_t lds_offset(const void *p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p;
}

// Those of a lane's scores that reach th (a float's bits), by the compare instruction that
// append16 admits by: the count sizes the place a lane takes in its row's list,
// so the two agree on every pair of floats.  (The sign of s - th, also two
// operations a score, does not: -0 - +0 is -0, and a NaN has either sign.)
// Four compares go to scalar masks before the first is read, as a carry; each
// of the four adds to a count of its own.
struct Count4 {
    int n[4] = {0, 0, 0, 0};
    template <int N = 16, class X>
    __device__ __forceinline__ void add(const X &s, uint32_t th)
    {
        static_assert(N % 4 == 0, "groups of four");
#define RR_CMP(m) "v_cmp_ge_f32_e64 %[m" #m "], %[x" #m "], %[th]\n\t"
#define RR_ADD(m) "v_addc_co_u32_e64 %[n" #m "], %[m" #m "], 0, %[n" #m "], %[m" #m "]\n\t"
#pragma unroll
        for (int b = 0; b < N; b += 4) {
            uint64_t m0, m1, m2, m3;
            asm(RR_CMP(0) RR_CMP(1) RR_CMP(2) RR_CMP(3) RR_ADD(0) RR_ADD(1) RR_ADD(2) RR_ADD(3)
                : [n0] "+v"(n[0]), [n1] "+v"(n[1]), [n2] "+v"(n[2]), [n3] "+v"(n[3]), [m0] "=&s"(m0), [m1] "=&s"(m1),
                  [m2] "=&s"(m2), [m3] "=&s"(m3)
                : [x0] "v"(s[b]), [x1] "v"(s[b + 1]), [x2] "v"(s[b + 2]), [x3] "v"(s[b + 3]), [th] "v"(th));
        }
#undef RR_ADD
#undef RR_CMP
    }
    __device__ __forceinline__ int sum() const { return n[0] + n[1] + n[2] + n[3]; }
};

// -inf for a NaN.  (Ties are cut by compares that the compiler may turn round:
// to it scores are no NaN.)
__device__ __forceinline__ float no_nan(float x)
{
    asm("v_max_f32_e32 %0, 0xff800000, %0" : "+v"(x));
    return x;
}

// Appends those of a lane's 16 scores that reach th to LDS as (score, id)
// pairs from byte `at`, with the id of score i = id + i.  The compares of
// eight scores go to scalar masks first; then a score takes its mask as the
// execution mask for one write of both words and two adds (left to the
// compiler each store becomes a branch of its own: 86 cycles a score; a
// compare straight into the execution mask waits for it: 58).  Every lane of
// the wave is active.  The writes are complete only after a wait on the LDS
// counter, which is the caller's.
__device__ __forceinline__ void append16(const f32x16_t &s, uint32_t th, uint32_t &at, uint32_t id)
{
#define RR_CMP(m, x) "v_cmp_ge_f32_e64 %[m" #m "], %[x" #m "], %[th]\n\t"
#define RR_APP(m, i) \
    "s_mov_b64 exec, %[m" #m "]\n\t" \
    "v_add_u32_e32 %[t], " #i ", %[id]\n\t" \
    "ds_write2_b32 %[at], %[x" #m "], %[t] offset0:0 offset1:1\n\t" \
    "v_add_u32_e32 %[at], 8, %[at]\n\t"
#define RR_APPEND8(b, i0, i1, i2, i3, i4, i5, i6, i7) \
    { \
        uint64_t sv, m0, m1, m2, m3, m4, m5, m6, m7; \
        uint32_t t; \
        asm volatile("s_mov_b64 %[sv], exec\n\t" RR_CMP(0, 0) RR_CMP(1, 1) RR_CMP(2, 2) RR_CMP(3, 3) RR_CMP(4, 4) \
                         RR_CMP(5, 5) RR_CMP(6, 6) RR_CMP(7, 7) RR_APP(0, i0) RR_APP(1, i1) RR_APP(2, i2) RR_APP(3, i3) \
                             RR_APP(4, i4) RR_APP(5, i5) RR_APP(6, i6) RR_APP(7, i7) "s_mov_b64 exec, %[sv]\n\t" \
                     : [at] "+v"(at), [t] "=&v"(t), [sv] "=&s"(sv), [m0] "=&s"(m0), [m1] "=&s"(m1), [m2] "=&s"(m2), \
                       [m3] "=&s"(m3), [m4] "=&s"(m4), [m5] "=&s"(m5), [m6] "=&s"(m6), [m7] "=&s"(m7) \
                     : [x0] "v"(s[b + 0]), [x1] "v"(s[b + 1]), [x2] "v"(s[b + 2]), [x3] "v"(s[b + 3]), \
                       [x4] "v"(s[b + 4]), [x5] "v"(s[b + 5]), [x6] "v"(s[b + 6]), [x7] "v"(s[b + 7]), [th] "v"(th), \
                       [id] "v"(id) \
                     : "memory"); \
    }
    RR_APPEND8(0, 0, 1, 2, 3, 4, 5, 6, 7)
    RR_APPEND8(8, 8, 9, 10, 11, 12, 13, 14, 15)
#undef RR_APPEND8
#undef RR_APP
#undef RR_CMP
}

// The same for N (a multiple of four) scores with an id each.
template <int N>
__device__ __forceinline__ void append_listed(const float (&x)[N], const uint32_t (&id)[N], uint32_t th, uint32_t &at)
{
    static_assert(N % 4 == 0, "groups of four");
#define RR_CMP(m) "v_cmp_ge_f32_e64 %[m" #m "], %[x" #m "], %[th]\n\t"
#define RR_APP(m) \
    "s_mov_b64 exec, %[m" #m "]\n\t" \
    "ds_write2_b32 %[at], %[x" #m "], %[i" #m "] offset0:0 offset1:1\n\t" \
    "v_add_u32_e32 %[at], 8, %[at]\n\t"
#pragma unroll
    for (int b = 0; b < N; b += 4) {
        uint64_t sv, m0, m1, m2, m3;
        asm volatile("s_mov_b64 %[sv], exec\n\t" RR_CMP(0) RR_CMP(1) RR_CMP(2) RR_CMP(3) RR_APP(0) RR_APP(1) RR_APP(2)
                         RR_APP(3) "s_mov_b64 exec, %[sv]\n\t"
                     : [at] "+v"(at), [sv] "=&s"(sv), [m0] "=&s"(m0), [m1] "=&s"(m1), [m2] "=&s"(m2), [m3] "=&s"(m3)
                     : [x0] "v"(x[b]), [x1] "v"(x[b + 1]), [x2] "v"(x[b + 2]), [x3] "v"(x[b + 3]), [i0] "v"(id[b]),
                       [i1] "v"(id[b + 1]), [i2] "v"(id[b + 2]), [i3] "v"(id[b + 3]), [th] "v"(th)
                     : "memory");
    }
#undef RR_APP
#undef RR_CMP
}

// Waves per SIMD the registers should allow: the accumulators take 16 KT, the
// query fragment and a stage in flight ROWB / 8 and RB / 8 each.
template <typename DT, int D, int NW, int KT>
constexpr int min_waves()
{
    using S = Shape<DT, D, NW, KT, 1>;
    const int regs = 16 * KT + S::ROWB / 8 + S::RB / 4 + 40;
    return regs <= 168 ? 3 : (regs <= 264 ? 2 : 1);
}

template <int MODE, typename DT, int D, int NW, int KT, int P>
__global__ __attribute__((amdgpu_flat_work_group_size(1, 64 * NW), amdgpu_waves_per_eu(min_waves<DT, D, NW, KT>())))
void resident_kernel(RouteArgs a)
{
    using S = Shape<DT, D, NW, KT, P>;
    constexpr int LPR = S::LPR, RPW = S::RPW, CAP = S::CAP;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t th_s[32];
    __shared__ float rmax_s[32];
    __shared__ int32_t row_cnt[3][32], row_c[32];
    __shared__ float2 ab_s[NW][32];
    __shared__ unsigned long long s_pairs;
    __shared__ int32_t s_rows;

    int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int hh = lane >> 5, l32 = lane & 31;
    const int group = a.n_heads / a.n_kv_heads;
    const int n_mand = a.n_sink + a.n_recent, c_sent = a.m + a.r + n_mand;
    // LDS strides of the staged rows (int32), multiples of four
    const int k4 = (a.k + 3) & ~3, c4 = (c_sent + 3) & ~3, r4 = (a.r + 3) & ~3;
    unsigned char *const lists = smem + (P > 1 ? a.lds_region0 : 0);  // [32][LSTR] candidates
    // [32][BW] (R, N or ledger R, C) words
    uint2 *bm = reinterpret_cast<uint2 *>(P > 1 ? lists + S::BM * S::LSTR : smem + S::OFF_BM);
    // [32][NWD] counts before a word: R | N << 16
    uint32_t *pre = reinterpret_cast<uint32_t *>(smem + (P > 1 ? 0 : S::OFF_PRE));
    int32_t *stgR = reinterpret_cast<int32_t *>(smem + (P > 1 ? S::BM * S::NWD * 4 : S::OFF_STG));  // [32][k4]
    int32_t *stgS = stgR + 32 * k4;                                  // [32][c4]; full routing: slot scores [32][k4]
    int32_t *dra = stgS + 32 * c4;                                   // [32][r4] random draws

    if ((MODE == MODE_FULL || MODE == MODE_ANCHOR) && a.pairs_out && blockIdx.x == 0 && tid == 0)
        *a.pairs_out = a.pairs_value;

    int h, t;
    tile_of_block(blockIdx.x, a.n_heads, a.n_kv_heads, a.tiles_per_head, h, t);
    if (a.causal) t = a.tiles_per_head - 1 - t;  // the longest tiles first
    const int i0 = 32 * t;
    const int nrows = min(32, a.n_q - i0);
    const int64_t g0 = (int64_t)h * a.n_q + i0;
    const int ncols = a.causal ? min(i0 + nrows, a.n_k) : a.n_k;
    const int nbt = (ncols + 32 * NW - 1) / (32 * NW);  // stages, <= P KT
    const int np = P > 1 ? (nbt + KT - 1) / KT : 1;     // panels
    int nb = P > 1 ? (nbt + np - 1) / np : nbt;         // stages of the panel, <= KT
    int seg = 16 * nb, kp = 0;                          // its segments' length and its first key
    const unsigned char *Kg = reinterpret_cast<const unsigned char *>(a.K) + (int64_t)(h / group) * a.n_k * S::ROWB;

    // ---- after the sweep, lane (rl, part) of wave w serves row sr
    int part = lane & (LPR - 1), sr = w * RPW + lane / LPR;
    int64_t grow = g0 + min(sr, nrows - 1);  // (rows past the tile's last repeat it and write nothing)

    // ------------------------------------------------------ requests, set-up
    // global -> registers: this lane's pieces of part q of stage st (keys past
    // the last repeat it; their scores are masked)
    constexpr int NF = P > 1 ? 1 : 2;  // stage parts in flight (one: the panel loop needs the registers)
    u32x4_t breg[NF][S::PT];
    const bool whole = (2 * w + 2) * seg <= a.n_k;  // every key of the wave's segments exists
    uint32_t lrow = lane / S::PR, lcol = lane % S::PR;
    const __amdgpu_buffer_rsrc_t keys =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char *>(Kg), 0, a.n_k * S::ROWB, 0x00020000);
    auto gload = [&](u32x4_t (&breg)[S::PT], int st, int q) __attribute__((always_inline)) {
        const uint32_t coff = (lcol / (S::PR / 2)) * (S::ROWB / 2) + q * (S::RB / 2) + (lcol % (S::PR / 2)) * 16;
        constexpr int RS = 64 / S::PR;  // key rows a wave loads at a time
        if constexpr (P > 1) {
            // (bounded by the key head: keys past the last read as zero)
#pragma unroll
            for (int u = 0; u < S::PT; ++u) {
                const int tr = u * RS;
                const uint32_t key = kp + (2 * w + tr / 16) * seg + 16 * st + tr % 16;
                breg[u] = __builtin_amdgcn_raw_buffer_load_b128(keys, lrow * S::ROWB + coff + key * S::ROWB, 0, 0);
            }
        } else if (whole) {
            const uint32_t voff = lrow * S::ROWB + coff;
#pragma unroll
            for (int u = 0; u < S::PT; ++u) {
                const int tr = u * RS;  // (RS divides 16)
                const unsigned char *base = Kg + (int64_t)(kp + (2 * w + tr / 16) * seg + 16 * st + tr % 16) * S::ROWB;
                breg[u] = *reinterpret_cast<const u32x4_t *>(base + voff);
            }
        } else {
#pragma unroll
            for (int u = 0; u < S::PT; ++u) {
                const int tr = u * RS + (int)lrow;
                const int key = min(kp + (2 * w + (tr >> 4)) * seg + 16 * st + (tr & 15), a.n_k - 1);
                breg[u] = *reinterpret_cast<const u32x4_t *>(Kg + (uint32_t)key * S::ROWB + coff);
            }
        }
    };
    unsigned char *const wst = smem + w * S::WST;
    // registers -> the wave's LDS rows; key row t lies where the lane that
    // multiplies it reads (transposed_row)
    auto lstore = [&](const u32x4_t (&breg)[S::PT]) __attribute__((always_inline)) {
        constexpr int RS = 64 / S::PR;
#pragma unroll
        for (int u = 0; u < S::PT; ++u) {
            const int tr = u * RS + (int)lrow;
            const int pos = ((tr & 15) >> 2) * 8 + (tr >> 4) * 4 + (tr & 3);
            *reinterpret_cast<u32x4_t *>(wst + pos * S::LS + lcol * 16) = breg[u];
        }
    };
    // (the query fragment first: loads complete in order, so the wait for the
    // first stage covers it and no later product waits for younger loads)
    Frag<DT, D> fq;
    const DT *const Qrow = reinterpret_cast<const DT *>(a.Q) + (g0 + min(l32, nrows - 1)) * D;
    fq.load(Qrow, hh);
    auto gload_first = [&]() __attribute__((always_inline)) {
        gload(breg[0], 0, 0);
        if constexpr (NF > 1) {
            if (S::SUB > 1 || nb > 1) gload(breg[NF - 1], S::SUB > 1 ? 0 : 1, S::SUB > 1 ? 1 : 0);
        }
    };
    gload_first();

    // relay: the wave's rows' ledger ids -> bitmaps.  The first 16 bytes per
    // lane of R and of C are requested here and marked under the sweep.
    int led_nc = 0, led_ns = 0;  // the row's ledger counts |R|, |C|
    int4 led_r = make_int4(-1, -1, -1, -1), led_c = led_r;
    const int32_t *const lr_row = a.led_routes + grow * a.k, *const ls_row = a.led_sent + grow * c_sent;
    const bool vr = (a.k & 3) == 0 && a.vec, vs = (c_sent & 3) == 0 && a.vec;
    if constexpr (MODE == MODE_RELAY) {
        if (vr && 4 * part < a.k) led_r = reinterpret_cast<const int4 *>(lr_row)[part];
        if (vs && 4 * part < c_sent) led_c = reinterpret_cast<const int4 *>(ls_row)[part];
        for (int j = lane; j < RPW * S::BW; j += 64) bm[w * RPW * S::BW + j] = make_uint2(0u, 0u);
        if (tid == 0) {
            s_pairs = 0ull;
            s_rows = 0;
        }
    }
    auto mark_ledger = [&]() __attribute__((always_inline)) {
        uint32_t *bw = reinterpret_cast<uint32_t *>(bm + sr * S::BW);
        auto mark = [&](int id, int which, int &n) __attribute__((always_inline)) {
            if ((id >= 0) & (id < a.n_k) & (sr < nrows)) {
                atomicOr(&bw[2 * (id >> 5) + which], 1u << (id & 31));
                ++n;
            }
        };
        auto mark4 = [&](const int4 &v, int which, int &n) __attribute__((always_inline)) {
            mark(v.x, which, n);
            mark(v.y, which, n);
            mark(v.z, which, n);
            mark(v.w, which, n);
        };
        auto mark_rest = [&](const int32_t *src, int wd, bool vec, int which, int &n) __attribute__((always_inline)) {
            if (vec) {
                for (int j = part + LPR; j < wd >> 2; j += LPR) mark4(reinterpret_cast<const int4 *>(src)[j], which, n);
            } else {
                for (int j = part; j < wd; j += LPR) mark(src[j], which, n);
            }
        };
        wave_sync();
        mark4(led_r, 0, led_nc);
        mark4(led_c, 1, led_ns);
        mark_rest(lr_row, a.k, vr, 0, led_nc);
        mark_rest(ls_row, c_sent, vs, 1, led_ns);
        led_nc = row_sum<LPR>(led_nc);
        led_ns = row_sum<LPR>(led_ns);
        lds_barrier();  // the bitmaps are read by every wave
    };
    if (tid < 96) row_cnt[tid >> 5][tid & 31] = 0;

    // ------------------------------------------------------------- the sweep
    const int myn = l32 < nrows ? (a.causal ? min(i0 + l32 + 1, a.n_k) : a.n_k) : 0;  // valid keys of the lane's row
    int kbase = (2 * w + hh) * seg;                                                   // first key of its segment
    const int minn = a.causal ? i0 + 1 : a.n_k;                                       // least over the tile's rows
    f32x16_t acc[KT];
    float amin = INFINITY, bmax = -INFINITY;
    // (several panels: a stage's limits are formed where they are used, not kept for
    // every stage of the panel loop)
    auto finish = [&](f32x16_t &x, int st) __attribute__((always_inline)) {
        if (kp + (2 * w + 1) * seg + 16 * st + 16 > minn) {  // (wave-uniform) some key is invalid for some row
            int my = myn;
            if (P > 1) asm volatile("" : "+v"(my));
            const int vlim = my - (kbase + 16 * st);
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = (i < vlim) ? x[i] : -INFINITY;
        }
        if constexpr (MODE == MODE_RELAY) {
            // alpha = min over R, beta = max over C, by bit-select from the
            // ledger's bitmaps
            int k0 = kbase + 16 * st;
            if (P > 1) asm volatile("" : "+v"(k0));
            const uint2 wv = bm[l32 * S::BW + (k0 >> 5)];
            const uint32_t sh = (uint32_t)(k0 & 16);
            const uint32_t mr = wv.x >> sh, mc = wv.y >> sh;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const uint32_t xb = __float_as_uint(x[i]);
                const uint32_t nr = (uint32_t)((int32_t)(mr << (31 - i)) >> 31);
                const uint32_t nc = (uint32_t)((int32_t)(mc << (31 - i)) >> 31);
                amin = fminf(amin, __uint_as_float((xb & nr) | (0x7F800000u & ~nr)));
                bmax = fmaxf(bmax, __uint_as_float((xb & nc) | (0xFF800000u & ~nc)));
            }
        }
    };
    bool on = sr < nrows, routed = false;  // row sr, row l32: routed by this launch
    unsigned long long pub = 0;  // relay: what the launch's pair total was before this tile's
    unsigned long long fin = 0;  // relay: tiles finished before this one << 32 | their flagged rows
    if constexpr (P > 1 && MODE == MODE_RELAY) mark_ledger();
    for (int p = 0;; ++p) {
        const bool last = P == 1 || p == np - 1;
        if constexpr (P > 1) {
            // (opaque: values derived from the lane are formed again in each panel
            // instead of being kept in registers across the sweeps)
            asm volatile("" : "+v"(tid));
            lane = tid & 63;
            hh = lane >> 5;
            l32 = lane & 31;
            lrow = lane / S::PR;
            lcol = lane % S::PR;
        }
        if (P > 1 && p > 0) {
            kp += 32 * NW * nb;
            nb = min(nb, nbt - p * nb);
            seg = 16 * nb;
            kbase = kp + (2 * w + hh) * seg;
            if (tid < 96) row_cnt[tid >> 5][tid & 31] = 0;
            fq.load(Qrow, hh);  // (loaded again: kept, it would cost the collection its registers)
            gload_first();
        }
        const unsigned char *const lp = wst + l32 * S::LS + hh * (S::RB / 2);
        // relay: the ledger's marks (and their barrier) come under stage `mst`
        // (several panels: before the first)
        const int mst = P > 1 ? -1 : min(KT > 2 ? 2 : 0, nb - 1);
        static_for<KT>([&](auto sc) __attribute__((always_inline)) {
            constexpr int st = decltype(sc)::value;
            if (st < nb) {
                f32x16_t c = f32x16_t{};
                static_for<S::SUB>([&](auto qc) __attribute__((always_inline)) {
                    constexpr int q = decltype(qc)::value, x = st * S::SUB + q;  // x: the part's number
                    constexpr int nst = (x + NF) / S::SUB, nq = (x + NF) % S::SUB;
                    lstore(breg[x % NF]);
                    if (nst < nb) gload(breg[x % NF], nst, nq);
                    wave_sync();
                    c = KeyPart<DT, D, S::SUB>::mma(lp, fq, q, c);
                    if (q == S::SUB - 1) {
                        acc[st] = c;
                        if constexpr (st > 0) {
                            if (MODE != MODE_RELAY || st > mst) finish(acc[st > 0 ? st - 1 : 0], st - 1);
                        }
                    }
                    wave_sync();
                });
                if constexpr (P == 1 && MODE == MODE_RELAY && st <= (KT > 2 ? 2 : 0)) {
                    if (st == mst) {
                        mark_ledger();
                        static_for<st>([&](auto jc) __attribute__((always_inline)) { finish(acc[decltype(jc)::value], decltype(jc)::value); });
                    }
                }
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[st][i] = -INFINITY;
            }
        });
        static_for<KT>([&](auto sc) __attribute__((always_inline)) {
            constexpr int st = decltype(sc)::value;
            if (st == nb - 1) finish(acc[st], st);
        });

        // kept maxima -> the wave's LDS rows (the key tile there is consumed)
        {
            float *const kept = reinterpret_cast<float *>(wst) + l32 * S::KSTR + hh * 16;
            float gm[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                gm[i] = acc[0][i];
#pragma unroll
                for (int st = 1; st < KT; ++st) gm[i] = fmaxf(gm[i], acc[st][i]);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                reinterpret_cast<float4 *>(kept)[q] = make_float4(gm[4 * q], gm[4 * q + 1], gm[4 * q + 2], gm[4 * q + 3]);
            if (MODE == MODE_RELAY && last) {
                amin = fminf(amin, __shfl_xor(amin, 32, 64));
                bmax = fmaxf(bmax, __shfl_xor(bmax, 32, 64));
                if (hh == 0) ab_s[w][l32] = make_float2(amin, bmax);
            }
        }
        lds_barrier();

        // ------------------------------------------------- trigger, bound per row
        if constexpr (P > 1) {
            asm volatile("" : "+v"(tid));
            part = tid & (LPR - 1);
            sr = w * RPW + (tid & 63) / LPR;
            grow = g0 + min(sr, nrows - 1);
        }
        // (before the last panel every row counts as routed)
        if (MODE == MODE_RELAY && last) {
            const float2 x = ab_s[part & (NW - 1)][sr];
            const float al = row_min<LPR>(x.x), be = row_max<LPR>(x.y);
            int flagged = 0;
            if (on && part == 0) {
                const bool flag = relay_trigger(led_ns, al, be, a.gamma, a.gamma_rows, grow, a.layer,
                                                a.min_reuse > 0 ? a.led_build[grow] : 0, a.min_reuse);
                a.flags[grow] = flag ? 1 : 0;
                if (a.mask_out) a.mask_out[grow] = flag ? 1 : 0;
                a.alpha_out[grow] = al;
                a.beta_out[grow] = be;
                if (!flag) a.led_age[grow] = a.layer - a.led_build[grow];
                flagged = flag ? 1 : 0;
                const int ni = a.causal ? min(i0 + sr + 1, a.n_k) : a.n_k;
                atomicAdd(&s_pairs, (unsigned long long)(led_nc + led_ns + (flag ? ni : 0)));
                if (flag) atomicAdd(&s_rows, 1);
            }
            on = row_sum<LPR>(flagged) != 0;
        }
        {
            const float4 *const kept = reinterpret_cast<const float4 *>(smem + (part >> 1) * S::WST) + sr * (S::KSTR / 4) + (part & 1) * 4;
            // a later panel takes the candidates so far as well
            constexpr int NU = P > 1 ? 16 + S::CPL : 16;
            const int c1 = (P > 1 && p > 0) ? row_c[sr] : 0;
            const bool dead = P > 1 && p > 0 && c1 == 0;  // stopped at the sweep cap: keeps no candidate
            float u[NU];
            if constexpr (P > 1) {
                const uint2 *lst = reinterpret_cast<const uint2 *>(lists + sr * S::LSTR);
#pragma unroll
                for (int j = 0; j < S::CPL; ++j) {
                    u[16 + j] = -INFINITY;
                    if (part + LPR * j < c1) u[16 + j] = __uint_as_float(lst[part + LPR * j].x);
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 x = kept[q];
                u[4 * q] = x.x;
                u[4 * q + 1] = x.y;
                u[4 * q + 2] = x.z;
                u[4 * q + 3] = x.w;
            }
            float rmax = u[0], umin = INFINITY;
            int nfin = 0;
#pragma unroll
            for (int q = 0; q < NU; ++q) {
                const bool fin = u[q] > -INFINITY;
                rmax = fmaxf(rmax, u[q]);
                umin = fminf(umin, fin ? u[q] : INFINITY);
                nfin += fin ? 1 : 0;
            }
            rmax = row_max<LPR>(rmax);
            umin = row_min<LPR>(umin);
            nfin = row_sum<LPR>(nfin);
            const int T = a.k + a.m;
            // The T-th maximum to one of 127 levels of [lo, hi]: the maxima become
            // bytes, four to a word, and a level's count takes three operations a
            // word (subtract, top bits, population count); seven steps give the
            // highest level that T of them reach.  A level holds the maxima within
            // half a step of it however the conversion rounds, so its bound lies
            // 0.51 steps below.  Where much of the row falls into one level (an
            // outlier stretches the range) that level is cut again.  A range whose
            // width or its reciprocal leaves the normal floats is not cut: its
            // levels would come out as infinities and NaN.  lo then stays where it
            // is, a lower bound still, and the collection raises it.
            float lo = nfin >= T ? umin : kLowest, hi = rmax;
            if (P > 1 && p > 0) {
                const uint32_t before = th_s[sr];
                if (before < kStopped) lo = fmaxf(lo, __uint_as_float(before));
            }
            int clo = nfin;
            for (int it = 0; it < kBoundRounds; ++it) {
                const float span = hi - lo;
                const bool go = on & (nfin >= T) & (clo > T + (T >> 3)) & (span > kLeastSpan) & (span < kMostSpan);
                if (__ballot(go) == 0ull) break;
                const float step = span * (1.0f / 127.0f), inv = 127.0f * __builtin_amdgcn_rcpf(span);
                uint32_t x[NU / 4];
#pragma unroll
                for (int q = 0; q < NU / 4; ++q) {
                    uint32_t b = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        b = __builtin_amdgcn_cvt_pk_u8_f32(fminf((u[4 * q + e] - lo) * inv, 127.0f), e, b);
                    x[q] = b | 0x80808080u;
                }
                uint32_t lev = 0;  // the level in every byte
                int cl = clo;
#pragma unroll
                for (uint32_t b = 0x40404040u; b >= 0x01010101u; b >>= 1) {
                    const uint32_t p = lev | b;
                    int n = 0;
#pragma unroll
                    for (int q = 0; q < NU / 4; ++q) n += __popc((x[q] - p) & 0x80808080u);
                    n = row_sum<LPR>(n);
                    lev = n >= T ? p : lev;
                    cl = n >= T ? n : cl;
                }
                const float L = (float)(lev & 0x7Fu);
                if (go) {
                    hi = lo + (L + 0.51f) * step;
                    if (lev != 0u) lo = lo + (L - 0.51f) * step;
                    clo = (lev == 0u && it > 0) ? T : cl;
                }
            }
            if (part == 0) {
                th_s[sr] = on ? (dead ? kStopped : __float_as_uint(lo)) : kNotRouted;
                rmax_s[sr] = rmax;
            }
        }
        lds_barrier();
        if (MODE == MODE_RELAY && last) {
            if (tid == 0)
                pub = __hip_atomic_fetch_add(reinterpret_cast<unsigned long long *>(a.done) + 1, s_pairs, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        }

        // ------------------------------------------- collection into row lists
        // (every wave follows all 32 rows: lane (l32, hh) holds row l32's state)
        // (the threshold is kept as bits: kNoScore must not meet float arithmetic)
        uint32_t th = th_s[l32];
        bool live = th < kStopped;  // the row collects
        routed = th != kNotRouted;
        th = live ? th : kNoScore;
        const int nv = last ? myn : min(myn, kp + 32 * NW * nb);  // the row's valid keys so far
        int base = 0, cnt = 0;
        {
            int th_id = INT_MAX, state = 0, id_lo = -1, id_hi = 0;  // state 1: cutting ties at th by id
            uint32_t lk = float_order(__uint_as_float(th)), hk = float_order(rmax_s[l32]) + 1u;
            bool settled = true, ties = false;
            int total = 0;
            // the candidates so far, rewritten with this panel's: every 2 NW-th is this lane's
            constexpr int NX = P > 1 ? S::CPL : 1;
            float xs[NX];
            uint32_t xi[NX];
            const bool more_lists = P > 1 && p > 0;
            if constexpr (P > 1) {
                const int c1 = p > 0 ? row_c[l32] : 0;
                const uint2 *lst = reinterpret_cast<const uint2 *>(lists + l32 * S::LSTR);
#pragma unroll
                for (int j = 0; j < NX; ++j) {
                    const int e = 2 * w + hh + LPR * j;
                    xs[j] = -INFINITY;
                    xi[j] = INT_MAX;  // (past every id cut)
                    if (e < c1) {
                        const uint2 x = lst[e];
                        xs[j] = __uint_as_float(x.x);
                        xi[j] = x.y;
                    }
                }
            }
            // ties: a score is admitted above tf, or at it by its id (none of a row that does not collect)
            auto tie_score = [&]() { return __uint_as_float(live ? th : 0x7F800000u); };
            auto tie_cut = [&]() { return live ? th_id : -1; };
            for (int it = 0;; ++it) {
                cnt = 0;
                if (!ties) {
                    Count4 c4;
                    if constexpr (P > 1) {
                        if (more_lists) c4.template add<NX>(xs, th);
                    }
#pragma unroll
                    for (int st = 0; st < KT; ++st) {
                        if (st < nb) c4.add(acc[st], th);  // (masked scores are -inf, th is above)
                    }
                    cnt += c4.sum();
                } else {
                    const float tf = tie_score();
                    const int tid_cut = tie_cut();
                    if (more_lists) {
#pragma unroll
                        for (int j = 0; j < NX; ++j) cnt += ((xs[j] > tf) | ((xs[j] == tf) & ((int)xi[j] <= tid_cut))) ? 1 : 0;
                    }
#pragma unroll
                    for (int st = 0; st < KT; ++st) {
                        if (st < nb) {
                            const int lim = tid_cut - (kbase + 16 * st);
#pragma unroll
                            for (int i = 0; i < 16; ++i) {
                                const float x = no_nan(acc[st][i]);
                                cnt += ((x > tf) | ((x == tf) & (i <= lim))) ? 1 : 0;
                            }
                        }
                    }
                }
                const int slot = it % 3;
                if (cnt > 0) base = atomicAdd(&row_cnt[slot][l32], cnt);
                if (it > 0 && tid < 32) row_cnt[(it + 1) % 3][tid] = 0;
                lds_barrier();
                total = row_cnt[slot][l32];
                bool again = false;
                // the row's least admissible count (T_i <= T; rows not routed admit nothing)
                bool few = false;
                if (it == 0) {
                    few = live & (total < min(a.k + a.m, nv));
                    if (__ballot((total > CAP) | few) == 0ull) break;  // the usual case
                    // the bound's rounding overshot, or the row has fewer finite scores
                    // than it takes
                    if (few) lk = float_order(-INFINITY);
                }
                if (live) {
                    const int ki = a.k_rows ? min(max(a.k_rows[g0 + min(l32, nrows - 1)], 1), a.k) : a.k;
                    const int Ti = ki + a.m, need = min(Ti, nv);
                    if (state == 1) {
                        const int mid = th_id;
                        if (total >= need)
                            id_hi = mid;
                        else
                            id_lo = mid;
                        if (id_hi - id_lo > 1) {
                            th_id = id_lo + ((id_hi - id_lo) >> 1);
                            again = true;
                        } else if (mid != id_hi) {
                            th_id = id_hi;
                            again = true;
                        }
                    } else if (total < need) {
                        hk = float_order(__uint_as_float(th));
                        again = true;
                    } else if (total > CAP) {
                        lk = float_order(__uint_as_float(th));
                        again = true;
                    }
                    if (state == 0 && again) {
                        if (hk - lk > 1u) {
                            th = few ? __float_as_uint(kLowest) : __float_as_uint(order_float(lk + ((hk - lk) >> 1)));
                        } else {
                            // lk is the T_i-th score: the chunks above it and the
                            // lowest ids of its ties; bisect the id cut.  (Ties at
                            // -inf: the masked keys' ids lie past the valid ones.)
                            state = 1;
                            th = __float_as_uint(order_float(lk));
                            id_lo = -1;
                            id_hi = nv - 1;
                            th_id = -1 + (nv >> 1);
                        }
                    }
                }
                const uint64_t more = __ballot(again);
                if (more == 0ull) break;
                if (it + 1 >= a.sweep_cap) {
                    // stopped at the cap: the row keeps no candidate
                    settled = !again;
                    if (again) {
                        live = false;
                        th = kNoScore;
                        cnt = 0;
                        total = 0;
                    }
                    break;
                }
                ties = __ballot(state == 1) != 0ull;
            }
            if (w == 0 && hh == 0) {
                row_c[l32] = total;
                if (!settled && a.unconverged) atomicAdd(a.unconverged, 1ull);
            }
            if (!ties) {
                uint32_t at = (uint32_t)(l32 * S::LSTR + base * 8) + lds_offset(lists);
                if constexpr (P > 1) {
                    if (p > 0) append_listed<NX>(xs, xi, th, at);
                }
                static_for<KT>([&](auto sc) __attribute__((always_inline)) {
                    constexpr int st = decltype(sc)::value;
                    if (st < nb) append16(acc[st], th, at, (uint32_t)(kbase + 16 * st));
                });
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            } else {
                uint2 *lst = reinterpret_cast<uint2 *>(lists + l32 * S::LSTR) + base;
                const float tf = tie_score();
                const int tid_cut = tie_cut();
                if (more_lists) {
#pragma unroll
                    for (int j = 0; j < NX; ++j) {
                        if ((xs[j] > tf) | ((xs[j] == tf) & ((int)xi[j] <= tid_cut))) {
                            *lst = make_uint2(__float_as_uint(xs[j]), xi[j]);
                            ++lst;
                        }
                    }
                }
#pragma unroll
                for (int st = 0; st < KT; ++st) {
                    if (st < nb) {
                        const int lim = tid_cut - (kbase + 16 * st);
#pragma unroll
                        for (int i = 0; i < 16; ++i) {
                            const float x = no_nan(acc[st][i]);
                            if ((x > tf) | ((x == tf) & (i <= lim))) {
                                *lst = make_uint2(__float_as_uint(x), (uint32_t)(kbase + 16 * st + i));
                                ++lst;
                            }
                        }
                    }
                }
            }
        }
        if (MODE == MODE_RELAY && last) {
            // published after the pair total has been added (pub has returned)
            if (tid == 0) {
                asm volatile("" : "+v"(pub)::"memory");
                fin = __hip_atomic_fetch_add(reinterpret_cast<unsigned long long *>(a.done),
                                             (1ull << 32) + (unsigned long long)(uint32_t)s_rows, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        lds_barrier();
        if (last) break;
    }

    // -------------------------------------------- selection (row's own lanes)
    // Slot `slot` of the tile (staging, bitmaps) serves row `row`.  A relay's
    // routed rows are packed into the first slots, so that waves without one
    // skip the rest.
    const int slot = sr;
    int row = sr;
    bool act = on;
    if constexpr (MODE == MODE_RELAY) {
        const uint32_t mask = (uint32_t)__ballot(routed);  // (every lane (l32, hh) holds row l32's)
        act = slot < __popc(mask);
        row = act ? select_bit(mask, slot) : 0;
    }
    auto put_row = [&](void *dst, const void *src, int wd) __attribute__((always_inline)) {
        if ((wd & 3) == 0 && a.vec) {
            for (int j = part; j < wd >> 2; j += LPR)
                reinterpret_cast<u32x4_t *>(dst)[j] = reinterpret_cast<const u32x4_t *>(src)[j];
        } else {
            for (int j = part; j < wd; j += LPR)
                reinterpret_cast<uint32_t *>(dst)[j] = reinterpret_cast<const uint32_t *>(src)[j];
        }
    };
    if (MODE == MODE_RELAY && !on && sr < nrows && a.routes_out) {  // a kept route
        if (P == 1 && vr && a.k <= 4 * LPR) {
            if (4 * part < a.k) reinterpret_cast<int4 *>(a.routes_out + grow * a.k)[part] = led_r;
        } else {
            put_row(a.routes_out + grow * a.k, a.led_routes + grow * a.k, a.k);
        }
    }
    if (__ballot(act) != 0ull) {
        const int64_t orow = g0 + min(row, nrows - 1);
        const int ni = act ? (a.causal ? min(i0 + row + 1, a.n_k) : a.n_k) : 0;
        const uint2 *lst = reinterpret_cast<const uint2 *>(lists + row * S::LSTR);
        const int c = act ? row_c[row] : 0;
        const int ki = a.k_rows ? min(max(a.k_rows[orow], 1), a.k) : a.k;
        const int ke = min(ki, c), Te = min(ki + a.m, c);
        uint2 *const bmr = bm + slot * S::BW;
        uint32_t *const bw = reinterpret_cast<uint32_t *>(bmr), *const prr = pre + slot * S::NWD;
        int32_t *const sR = stgR + slot * k4, *const sS = stgS + slot * c4;
        float *const sF = reinterpret_cast<float *>(stgS) + slot * k4;
        for (int j = lane; j < RPW * S::BW; j += 64) bm[w * RPW * S::BW + j] = make_uint2(0u, 0u);
        int cmax = c;
#pragma unroll
        for (int off = LPR; off < 64; off <<= 1) cmax = max(cmax, __shfl_xor(cmax, off, 64));
        cmax = __builtin_amdgcn_readfirstlane(cmax);
        // candidate part + LPR j: the first eight per lane in registers, any
        // more stay in the list (j < jmax <= CPL)
        const int jmax = (cmax + LPR - 1) / LPR;
        float sc[8], vk, vT;
        uint32_t id[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int e = part + LPR * j;
            const uint2 x = lst[e];
            sc[j] = (e < c) ? __uint_as_float(x.x) : -INFINITY;
            id[j] = x.y;
        }
        {
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = sc[j];
            sort_row<LPR>(v, part);
            for (int e = S::NET; e < cmax; ++e) {
                // keep the NET largest: lane part inserts the smaller of x and
                // the last entry of lane part - 1 (which that lane evicts)
                const float x = (e < c) ? __uint_as_float(lst[e].x) : -INFINITY;
                const float pl = dpp<0x111>(v[7]);
                const float xe = part > 0 ? fminf(x, pl) : x;
                float prev = v[0];
                v[0] = fmaxf(prev, xe);
#pragma unroll
                for (int j = 1; j < 8; ++j) {
                    const float cur = v[j];
                    v[j] = __builtin_amdgcn_fmed3f(prev, cur, xe);
                    prev = cur;
                }
            }
            auto at_pos = [&](int g) {
                g = max(g, 0);
                const float x0 = (g & 1) ? v[1] : v[0], x1 = (g & 1) ? v[3] : v[2];
                const float x2 = (g & 1) ? v[5] : v[4], x3 = (g & 1) ? v[7] : v[6];
                const float y0 = (g & 2) ? x1 : x0, y1 = (g & 2) ? x3 : x2;
                return __shfl((g & 4) ? y1 : y0, (lane & ~(LPR - 1)) + min(g >> 3, LPR - 1), 64);
            };
            vk = at_pos(ke - 1);
            vT = at_pos(Te - 1);
        }
        // members: R = ranks < ke, N = ranks in [ke, Te); bit j of a mask is
        // candidate part + LPR j
        uint32_t mR = 0, mT = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool in = part + LPR * j < c;
            mR |= (in & (sc[j] >= vk)) ? 1u << j : 0u;
            mT |= (in & (sc[j] >= vT)) ? 1u << j : 0u;
        }
        for (int j = 8; j < jmax; ++j) {
            const int e = part + LPR * j;
            const float s = __uint_as_float(lst[e].x);
            mR |= ((e < c) & (s >= vk)) ? 1u << j : 0u;
            mT |= ((e < c) & (s >= vT)) ? 1u << j : 0u;
        }
        const int gR = row_sum<LPR>(__popc(mR)), gT = row_sum<LPR>(__popc(mT));
        if (__ballot((gR != ke) | (gT != Te)) != 0ull) {
            // equal scores at a boundary rank the lower id first: those of them
            // past the boundary leave the set
            if ((gR != ke) | (gT != Te)) {
                for (int j = 0; j < jmax; ++j) {
                    const uint2 x = lst[part + LPR * j];
                    const float s = __uint_as_float(x.x);
                    if (!((mT >> j) & 1u) | !((s == vk) | (s == vT))) continue;
                    int rank = 0;
#pragma unroll 4
                    for (int e = 0; e < c; ++e) {
                        const uint2 y = lst[e];
                        const float s2 = __uint_as_float(y.x);
                        rank += ((s2 > s) | ((s2 == s) & (y.y < x.y))) ? 1 : 0;
                    }
                    if (rank >= ke) mR &= ~(1u << j);
                    if (rank >= Te) mT &= ~(1u << j);
                }
            }
        }
        wave_sync();
        auto set_bit = [&](uint32_t x, int j) __attribute__((always_inline)) {
            if ((mT >> j) & 1u) atomicOr(&bw[2 * (x >> 5) + (((mR >> j) & 1u) ? 0 : 1)], 1u << (x & 31));
        };
#pragma unroll
        for (int j = 0; j < 8; ++j) set_bit(id[j], j);
        for (int j = 8; j < jmax; ++j) set_bit(lst[part + LPR * j].y, j);
        wave_sync();
        // counts before each word, then every member's place
        {
            uint2 wd[S::WPL];
            int n = 0;
#pragma unroll
            for (int q = 0; q < S::WPL; ++q) {
                wd[q] = bmr[part * S::WPL + q];
                n += __popc(wd[q].x) + (__popc(wd[q].y) << 16);
            }
            int at = row_before<LPR>(n, part);
#pragma unroll
            for (int q = 0; q < S::WPL; ++q) {
                prr[part * S::WPL + q] = (uint32_t)at;
                at += __popc(wd[q].x) + (__popc(wd[q].y) << 16);
            }
        }
        wave_sync();
        auto place = [&](float s, uint32_t x, int j) __attribute__((always_inline)) {
            // (ids of no candidate are stale: their word is clamped, nothing is stored)
            const uint32_t q = min(x >> 5, (uint32_t)(S::NWD - 1)), bits = (1u << (x & 31)) - 1u;
            const uint2 wd = bmr[q];
            const uint32_t p = prr[q];
            const bool r = (mR >> j) & 1u, t = (mT >> j) & 1u;
            const int pos = r ? (int)(p & 0xFFFFu) + __popc(wd.x & bits) : (int)(p >> 16) + __popc(wd.y & bits);
            int32_t *const dst = r ? sR : sS;
            if (MODE == MODE_FULL ? r : t) dst[pos] = (int32_t)x;
            if (MODE == MODE_FULL && a.scores_out && r) sF[pos] = s;
        };
#pragma unroll
        for (int j = 0; j < 8; ++j) place(sc[j], id[j], j);
        for (int j = 8; j < jmax; ++j) {
            const uint2 x = lst[part + LPR * j];
            place(__uint_as_float(x.x), x.y, j);
        }
        const int nR = min(ke, gR), nN = min(Te, gT) - nR;
        for (int j = nR + part; j < a.k; j += LPR) {
            sR[j] = -1;
            if (MODE == MODE_FULL && a.scores_out) sF[j] = -INFINITY;
        }

        // --------------------------------------------------------- sentinels
        if constexpr (MODE != MODE_FULL) {
            for (int j = nN + part; j < a.m; j += LPR) sS[j] = -1;
            auto marked = [&](int x) __attribute__((always_inline)) {
                const uint2 wd = bmr[x >> 5];
                return (((wd.x | wd.y) >> (x & 31)) & 1u) != 0u;
            };
            auto mark = [&](int x) __attribute__((always_inline)) {
                if (x >= 0) atomicOr(&bw[2 * (x >> 5) + 1], 1u << (x & 31));
            };
            int nM = 0;
            if (n_mand > 0) {
                // mandatory sentinels (Sec. 3.1, item 3): the valid sink chunks
                // and the n_recent valid chunks up to the row's position, less R
                // and N, ascending; marked, so that the draws leave them out
                if (act && part == 0) {
                    int32_t *mout = sS + a.m + a.r;
                    int pos = (a.n_q == a.n_k) ? i0 + row : a.n_k - 1;
                    pos = min(pos, ni - 1);
                    const int sink_end = min(a.n_sink, ni);
                    const int rec_lo = (a.n_recent > 0) ? max(pos - a.n_recent + 1, sink_end) : pos + 1;
                    auto take = [&](int x) {
                        if (!marked(x)) {
                            mout[nM++] = x;
                            mark(x);
                        }
                    };
                    for (int x = 0; x < sink_end; ++x) take(x);
                    for (int x = rec_lo; x <= pos; ++x) take(x);
                    for (int q = nM; q < n_mand; ++q) mout[q] = -1;
                }
                nM = __shfl(nM, lane & ~(LPR - 1), 64);
                wave_sync();
            }
            if (a.r > 0) {
                const int pool = ni - (nR + nN + nM);
                int32_t *const dr = dra + slot * r4;
                const uint64_t h0 = sm64(sm64(sm64(a.seed) ^ (uint64_t)(uint32_t)a.layer) ^ (uint64_t)orow);
                // regimes of a row: the whole pool; ranks of a pool of at most
                // half the valid chunks; probes of a larger one
                const bool all = act & (pool <= a.r), ranks = act & !all & (2 * pool <= ni), probes = act & !all & !ranks;
                bool serial = false;
                if (__ballot(probes) != 0ull) {
                    // x mod n_i by Barrett reduction: hi64(x M) with M =
                    // floor((2^64 - 1) / n_i) undershoots the quotient by at most
                    // 1.  (Without the causal mask n_i = n_k, and M comes from
                    // the host.)
                    const uint64_t nn = (uint64_t)(a.causal ? (probes ? ni : 1) : a.n_k);
                    const uint64_t M = a.causal ? max_u64_div_small((uint32_t)nn) : a.barrett;
                    auto mod_ni = [&](uint64_t x) __attribute__((always_inline)) {
                        uint64_t rm = x - __umul64hi(x, M) * nn;
                        rm = (rm >= nn) ? rm - nn : rm;
                        rm = (rm >= nn) ? rm - nn : rm;
                        return (int)rm;
                    };
                    constexpr int SPL = 8;  // slots per lane, at most
                    serial = probes & (a.r > SPL * LPR);
                    const bool go = probes & !serial;
                    auto probe = [&](int s, int tt) __attribute__((always_inline)) {
                        return mod_ni(sm64(sm64(h0 ^ (uint64_t)s) ^ (uint64_t)tt));
                    };
                    // The row's claims: a byte per chunk, in the row's candidate list
                    // (consumed by now), holds the slot that last proposed the chunk.
                    // A slot writes its number at the chunk it proposes and reads it
                    // back: its own number, or that of a later slot (it writes again,
                    // and the later slot will see it), or that of an earlier one (it
                    // is rejected).  A claim is never read before it was written.
                    // Bit j of `pend`: slot part + LPR j has no proposal; byte j of
                    // `tried`: its attempts so far.  Few slots need a second attempt,
                    // so after the first a lane retries one slot at a time.
                    // (Several panels: the list is shorter than the chunks, and a slot compares
                    // its proposal with the earlier slots' instead.)
                    uint8_t *const claim = lists + row * S::LSTR;
                    uint32_t pend = 0;
                    uint64_t tried = 0x0101010101010101ull;
                    bool out = false;  // a slot ran out of attempts
                    // many rejections (short causal rows): some row of the wave has
                    // more than a quarter of its chunks marked
                    const bool dense = __ballot(go & (4 * pool < 3 * ni)) != 0ull;
                    for (int j = 0; LPR * j < a.r; ++j) {  // (uniform)
                        const int s = part + LPR * j;
                        if (go & (s < a.r)) {
                            const int z = probe(s, 0);
                            if (marked(z)) {
                                pend |= 1u << j;
                                if (P > 1) dr[s] = -1;
                            } else {
                                dr[s] = z;
                                if (P == 1) claim[z] = (uint8_t)s;
                            }
                        }
                    }
                    for (;;) {
                        wave_sync();
                        bool again = false;
                        if constexpr (P > 1) {
                            int z[SPL];
                            uint32_t hit = 0;
#pragma unroll
                            for (int j = 0; j < SPL; ++j) {
                                const int s = part + LPR * j;
                                z[j] = (go & (s < a.r) & (((pend >> j) & 1u) == 0u)) ? dr[s] : -2;
                            }
                            for (int t = 0; t < min(a.r, SPL * LPR); t += 4) {
                                const int4 y = *reinterpret_cast<const int4 *>(dr + t);
#pragma unroll
                                for (int j = 0; j < SPL; ++j) {
                                    if (LPR * j < a.r) {  // (uniform)
                                        const int n = part + LPR * j - t;  // earlier slots among the four
                                        const bool x = ((y.x == z[j]) & (n > 0)) | ((y.y == z[j]) & (n > 1)) |
                                                       ((y.z == z[j]) & (n > 2)) | ((y.w == z[j]) & (n > 3));
                                        hit |= x ? 1u << j : 0u;
                                    }
                                }
                            }
                            pend |= hit;
                        } else {
                            for (int j = 0; LPR * j < a.r; ++j) {  // (uniform)
                                const int s = part + LPR * j;
                                if (go & (s < a.r) & (((pend >> j) & 1u) == 0u)) {
                                    const int z = dr[s], v = claim[z];
                                    if (v < s) pend |= 1u << j;
                                    if (v > s) claim[z] = (uint8_t)s;
                                    again |= v > s;
                                }
                            }
                        }
                        if (out) pend = 0u;
                        if (__ballot((pend != 0u) | again) == 0ull) break;
                        if (pend != 0u) {
                            const int j = __ffs(pend) - 1, s = part + LPR * j;
                            const int tt = (int)(tried >> (8 * j)) & 0xFF;
                            int z = -1, used = 1;
                            if (dense) {
                                // four attempts at a time, the first unmarked counts
                                const uint64_t hs = sm64(h0 ^ (uint64_t)s);
                                int zz[4];
                                bool ok[4];
#pragma unroll
                                for (int u = 0; u < 4; ++u) zz[u] = mod_ni(sm64(hs ^ (uint64_t)(tt + u)));
#pragma unroll
                                for (int u = 0; u < 4; ++u) ok[u] = (tt + u < 64) & !marked(zz[u]);
                                z = ok[0] ? zz[0] : (ok[1] ? zz[1] : (ok[2] ? zz[2] : (ok[3] ? zz[3] : -1)));
                                used = ok[0] ? 1 : (ok[1] ? 2 : (ok[2] ? 3 : 4));
                            } else if (tt < 64) {
                                z = probe(s, tt);
                                z = marked(z) ? -1 : z;
                            }
                            if (z >= 0) {
                                dr[s] = z;
                                if (P == 1) claim[z] = (uint8_t)s;
                                pend &= pend - 1u;
                            }
                            out = tt >= 64;
                            tried += (uint64_t)used << (8 * j);
                        }
                    }
                    // (a slot that ran out: the row is decided slot by slot)
                    serial |= go & (row_sum<LPR>(out ? 1 : 0) != 0);
                }
                if (__ballot(all | ranks | serial) != 0ull) {
                    if (__ballot(ranks) != 0ull) {
                        // rank draws: the slots' ranks, hashed in parallel, then slot
                        // by slot the lane whose words hold the rank takes its bit
                        if (ranks) {
                            for (int s = part; s < a.r; s += LPR)
                                dr[s] = (int)mod_u64_small(sm64(sm64(h0 ^ (uint64_t)s)), (uint32_t)(pool - s));
                        }
                        wave_sync();
                        uint32_t fw[S::WPL];  // the lane's words of free chunks
                        int n = 0;
#pragma unroll
                        for (int q = 0; q < S::WPL; ++q) {
                            const uint2 wd = bmr[part * S::WPL + q];
                            const int lim = ni - (part * S::WPL + q) * 32;
                            fw[q] = ranks ? ~(wd.x | wd.y) & (lim >= 32 ? ~0u : (lim <= 0 ? 0u : (1u << lim) - 1u)) : 0u;
                            n += __popc(fw[q]);
                        }
                        for (int s = 0; s < a.r; ++s) {
                            int y = (ranks ? dr[s] : 0) - row_before<LPR>(n, part);
                            if (ranks & (y >= 0) & (y < n)) {
#pragma unroll
                                for (int q = 0; q < S::WPL; ++q) {
                                    const int pc = __popc(fw[q]);
                                    if ((y >= 0) & (y < pc)) {
                                        const int b = select_bit(fw[q], y);
                                        fw[q] &= ~(1u << b);
                                        dr[s] = (part * S::WPL + q) * 32 + b;
                                        y = -1;
                                    } else {
                                        y -= pc;
                                    }
                                }
                                --n;
                            }
                        }
                    }
                    if ((all | serial) & (part == 0)) {
                        auto free_word = [&](int q) {
                            const uint2 wd = bmr[q];
                            uint32_t z = ~(wd.x | wd.y);
                            const int lim = ni - q * 32;
                            return lim < 32 ? z & ((1u << lim) - 1u) : z;
                        };
                        auto nth_free = [&](int y) {
                            for (int q = 0; q * 32 < ni; ++q) {
                                const uint32_t z = free_word(q);
                                const int pc = __popc(z);
                                if (y < pc) return q * 32 + select_bit(z, y);
                                y -= pc;
                            }
                            return -1;
                        };
                        if (all) {
                            int s = 0;
                            for (int q = 0; q * 32 < ni; ++q)
                                for (uint32_t z = free_word(q); z != 0u && s < a.r; z &= z - 1u)
                                    dr[s++] = q * 32 + __ffs(z) - 1;
                            for (; s < a.r; ++s) dr[s] = -1;
                        } else {
                            for (int s = 0; s < a.r; ++s) {
                                const uint64_t hs = sm64(h0 ^ (uint64_t)s);
                                int x = -1;
                                for (int tt = 0; x < 0 && tt < 64; ++tt) {
                                    const int z = (int)mod_u64_small(sm64(hs ^ (uint64_t)tt), (uint32_t)ni);
                                    if (!marked(z)) x = z;
                                }
                                // 64 rejections: the y-th remaining pool chunk, ascending
                                if (x < 0) x = nth_free((int)mod_u64_small(sm64(hs ^ 64ull), (uint32_t)(pool - s)));
                                mark(x);
                                dr[s] = x;
                            }
                        }
                    }
                }
                wave_sync();
                for (int s = part; s < a.r; s += LPR) sS[a.m + s] = dr[s];
            }
        }
        wave_sync();

        // ---------------------------------------------------------- copy-out
        if (act) {
            if (MODE != MODE_FULL) put_row(a.led_routes + orow * a.k, sR, a.k);
            if (a.routes_out) put_row(a.routes_out + orow * a.k, sR, a.k);
            if (MODE == MODE_FULL && a.scores_out) put_row(a.scores_out + orow * a.k, sF, a.k);
            if (MODE != MODE_FULL) {
                if (c_sent > 0) put_row(a.led_sent + orow * c_sent, sS, c_sent);
                if (part == 0) {
                    a.led_build[orow] = a.layer;
                    a.led_age[orow] = 0;
                }
            }
        }
    }
    if constexpr (MODE == MODE_RELAY) {
        // the launch's totals, by the tile that published last; the sums are
        // reset for the next launch
        if (tid == 0 && (uint32_t)(fin >> 32) == gridDim.x - 1) {
            const int32_t rows = (int32_t)((uint32_t)fin + (uint32_t)s_rows);
            const unsigned long long pairs =
                __hip_atomic_exchange(reinterpret_cast<unsigned long long *>(a.done) + 1, 0ull, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(reinterpret_cast<unsigned long long *>(a.done), 0ull, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            *a.stat_pairs = (int64_t)pairs;
            *a.stat_nrr = rows;
            if (a.pairs_out) *a.pairs_out = (int64_t)pairs;
            if (a.nrr_out) *a.nrr_out = rows;
        }
    }
}

template <int MODE, typename DT, int D, int NW, int KT, int P = 1>
hipError_t launch_t(RouteArgs a, hipStream_t stream)
{
    using S = Shape<DT, D, NW, KT, P>;
    const int c_sent = MODE == MODE_FULL ? 0 : a.m + a.r + a.n_sink + a.n_recent;
    const int k4 = (a.k + 3) & ~3, c4 = (c_sent + 3) & ~3, r4 = (a.r + 3) & ~3;
    const int second = MODE == MODE_FULL ? (a.scores_out ? k4 : 0) : c4 + r4;
    const int staged = 32 * 4 * (k4 + second);
    a.lds_region0 = P > 1 ? S::region(staged) : 0;
    const size_t lds = P > 1 ? (size_t)a.lds_region0 + S::BM * (S::LSTR + S::BW * 8) : (size_t)S::OFF_STG + staged;
    if (a.n_k > (P > 1 ? 32 * S::NWD : 32 * NW * KT) || a.k + a.m > S::NET) return hipErrorInvalidValue;
    const void *fn = reinterpret_cast<const void *>(&resident_kernel<MODE, DT, D, NW, KT, P>);
    static LdsLimit seen;
    hipError_t e = raise_lds_limit(fn, lds, seen);
    if (e != hipSuccess) return e;
    if (a.sweep_cap < 1) a.sweep_cap = kMaxFixIters;
    a.tiles_per_head = (a.n_q + S::BM - 1) / S::BM;
    a.barrett = max_u64_div_small((uint32_t)a.n_k);  // (n_k <= 4096)
    const auto al = [](const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
    a.vec = al(a.led_routes) && al(a.led_sent) && al(a.routes_out) && al(a.scores_out);
    hipLaunchKernelGGL((resident_kernel<MODE, DT, D, NW, KT, P>), dim3(a.n_heads * a.tiles_per_head), dim3(64 * NW), lds,
                       stream, a);
    return hipGetLastError();
}

template <int MODE, typename DT, int D>
hipError_t launch_d(const RouteArgs &a, hipStream_t stream)
{
    const bool led = MODE != MODE_FULL;
    switch (resident_shape(a.n_k, a.k, a.m, led ? a.r : 0, led ? a.n_sink + a.n_recent : 0)) {
    case 42: return launch_t<MODE, DT, D, 4, 2>(a, stream);
    case 44: return launch_t<MODE, DT, D, 4, 4>(a, stream);
    case 48: return launch_t<MODE, DT, D, 4, 8>(a, stream);
    case 82: return launch_t<MODE, DT, D, 8, 2>(a, stream);
    case 84: return launch_t<MODE, DT, D, 8, 4>(a, stream);
    case 88: return launch_t<MODE, DT, D, 8, 8>(a, stream);
    case 386: return launch_t<MODE, DT, D, 8, 6, 3>(a, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace resident
}  // namespace rr
