// One row of any length solved by T threads with C contiguous samples (and duals) each: the mapping
// of rows to threads, the exchanges between the threads of a row, and the projected Newton solver
// that the long-row kernels (tv_long.hpp) and the plane-per-workgroup kernels (tv_plane2d.hpp) share.
//
// T = 8 .. 64 keep a row inside one wavefront; T >= 128 spread it over several, up to a whole
// workgroup.  The row, its dual and the Newton direction stay in registers for the entire solve.
//
// Thread mapping: ROWS (unit element stride): tid = row_in_group * T + t, so a wave reads
// one row's consecutive chunks; COLS (strided samples, e.g. image columns): tid = t * G +
// row_in_group, so adjacent lanes read adjacent columns and global accesses coalesce.
#pragma once
#include "tv_common.hpp"
#include "tv_dispatch.hpp"

namespace tvk {

template <int T, int G, bool COLS>
struct LongMap {
    static constexpr int NT = T * G;
    static constexpr int NW = NT / 64;
    static constexpr int RG = COLS ? G : 1;            // rows interleaved inside a wave
    static constexpr int WPR = COLS ? NW : (T + 63) / 64;   // waves holding parts of one row
    static constexpr int LANES = T < 64 ? T : 64;      // ROWS mapping: lanes of a wave on one row
    // A row that lives in exactly one wave (which holds nothing else) never has to wait for
    // the other waves of its workgroup: its LDS slices are its own, every barrier becomes a
    // wave-level fence and every workgroup vote a wave vote, and the wave leaves when its
    // row is done.
    static constexpr bool PRIVATE = !COLS && T <= 64;
    __device__ static __forceinline__ int row_of(int tid) { return G == 1 ? 0 : (COLS ? tid % G : tid / T); }
    __device__ static __forceinline__ int t_of(int tid) { return G == 1 ? tid : (COLS ? tid / G : tid % T); }
    // orders LDS writes before later LDS reads among the threads that share rows
    __device__ static __forceinline__ void sync()
    {
        if (PRIVATE) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        } else {
            __syncthreads();
        }
    }
};

// v of the lane that a row-local DPP pattern names (0xB1 / 0x4E: quad_perm [1,0,3,2] / [2,3,0,1];
// 0x141 / 0x140: mirror within 8 / 16 lanes).
template <int CTRL>
__device__ __forceinline__ float long_dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

// Rows of at most 16 threads lie inside one 16-lane DPP row (ROWS mapping: consecutive lanes are
// consecutive threads of a row; two rows share a DPP row when T = 8): a thread then gets the
// value of thread t - S / t + S of its own row from a row shift that rides on the reading
// instruction, instead of a write to LDS, a fence and a read.  Beyond the ends of the row: 0.
// Every lane of the wave must take part: a shift reads 0 from a lane that a branch has switched off.
template <int T, int S>
__device__ __forceinline__ float from_left(float v, int t)
{
    static_assert(T <= 16 && S >= 1 && S < 16, "row shifts stay inside a 16-lane row");
    const float r = long_dpp<0x110 + S>(v);                    // row_shr:S
    return (T < 16 && t < S) ? 0.f : r;
}
template <int T, int S>
__device__ __forceinline__ float from_right(float v, int t)
{
    static_assert(T <= 16 && S >= 1 && S < 16, "row shifts stay inside a 16-lane row");
    const float r = long_dpp<0x100 + S>(v);                    // row_shl:S
    return (T < 16 && t + S >= T) ? 0.f : r;
}
// (Rows of 32 and 64 threads could fetch their direct neighbours by a shift of the whole wave
// (wave_shr:1); measured, that changes nothing for them: their time goes into the scan steps at
// distances that no single shift covers.)

// OR over the T <= 16 lanes of a row (rows are aligned groups of T lanes), the result in all of them.
template <int T>
__device__ __forceinline__ uint32_t row_or_all(uint32_t v)
{
    static_assert(T == 8 || T == 16, "butterflies inside a 16-lane DPP row");
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true);     // quad_perm [1,0,3,2]
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, true);     // quad_perm [2,3,0,1]
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true);    // mirror within 8
    if (T > 8) v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, true);   // within 16
    return v;
}

// Segment code of a row of at most 32 samples (FwdParams::seg) from its output, which is bit-constant
// inside a segment: bit k of .x = x jumps behind sample k, of .y = it rises there.  xs: the thread's
// chunk; every lane of the wave calls, all lanes of the row get the code.
template <int T, int C>
__device__ __forceinline__ uint2 row_segment_code(const float (&xs)[C], int n, int t)
{
    const float xnext0 = from_right<T, 1>(xs[0], t);
    uint32_t jm = 0, up = 0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int k = t * C + c;
        const float xn = (c + 1 < C) ? xs[c + 1] : xnext0;
        if (k < n - 1) {
            if (xn != xs[c]) jm |= 1u << k;
            if (xn > xs[c]) up |= 1u << k;
        }
    }
    return make_uint2(row_or_all<T>(jm), row_or_all<T>(up));
}

// Sum over the 64 lanes of a wave, the same total in every lane, in a fixed order: four
// exchanges inside the 16-lane rows ride on the adds themselves (DPP), two swaps cross the rows.
template <int LANES = 64>
__device__ __forceinline__ float wave_sum_all(float v)
{
    v += long_dpp<0xB1>(v);
    v += long_dpp<0x4E>(v);
    v += long_dpp<0x141>(v);
    if (LANES > 8) v += long_dpp<0x140>(v);
    if (LANES > 16) {                                 // LANES = 16: four rows per wave, kept apart
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    if (LANES > 32) {                                 // LANES = 32: two rows per wave
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    return v;
}

// Sums NV values over the T threads of each row; every thread of the row gets the totals.
// Deterministic: fixed shuffle tree inside a wave, then a fixed-order sum over waves.
template <int T, int G, bool COLS, int NV>
__device__ __forceinline__ void row_sum(float (&v)[NV], float *red, int j, int tid)
{
    using Mp = LongMap<T, G, COLS>;
    if constexpr (Mp::RG == 1) {
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] = wave_sum_all<Mp::LANES>(v[q]);
    } else {
#pragma unroll
        for (int off = 32; off >= Mp::RG; off >>= 1) {
#pragma unroll
            for (int q = 0; q < NV; ++q) v[q] += __shfl_xor(v[q], off);
        }
    }
    if (Mp::WPR == 1) return;
    const int wave = tid >> 6, lane = tid & 63;
    __syncthreads();
    if (lane < Mp::RG) {
#pragma unroll
        for (int q = 0; q < NV; ++q) red[(q * Mp::NW + wave) * Mp::RG + (COLS ? j : 0)] = v[q];
    }
    __syncthreads();
    const int w0 = COLS ? 0 : j * Mp::WPR;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        float s = 0.f;
        for (int w = 0; w < Mp::WPR; ++w) s += red[(q * Mp::NW + w0 + w) * Mp::RG + (COLS ? j : 0)];
        v[q] = s;
    }
}

// The same with ONE barrier: consecutive calls alternate between two halves of `red`
// (par = 0, 1, 0, ...), so the writes of a call cannot overtake the reads of the one before.
template <int T, int G, bool COLS, int NV>
__device__ __forceinline__ void row_sum_alt(float (&v)[NV], float *red, int j, int tid, int par)
{
    using Mp = LongMap<T, G, COLS>;
    if constexpr (Mp::RG == 1) {
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] = wave_sum_all<Mp::LANES>(v[q]);
    } else {
#pragma unroll
        for (int off = 32; off >= Mp::RG; off >>= 1) {
#pragma unroll
            for (int q = 0; q < NV; ++q) v[q] += __shfl_xor(v[q], off);
        }
    }
    if (Mp::WPR == 1) return;
    float *r = red + par * (4 * Mp::NW * Mp::RG);
    const int wave = tid >> 6, lane = tid & 63;
    if (lane < Mp::RG) {
#pragma unroll
        for (int q = 0; q < NV; ++q) r[(q * Mp::NW + wave) * Mp::RG + (COLS ? j : 0)] = v[q];
    }
    __syncthreads();
    const int w0 = COLS ? 0 : j * Mp::WPR;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        float s = 0.f;
        for (int w = 0; w < Mp::WPR; ++w) s += r[(q * Mp::NW + w0 + w) * Mp::RG + (COLS ? j : 0)];
        v[q] = s;
    }
}

// Maximum of one non-negative value over the T threads of each row.
template <int T, int G, bool COLS>
__device__ __forceinline__ void row_max(float (&v)[1], float *red, int j, int tid)
{
    using Mp = LongMap<T, G, COLS>;
    if constexpr (Mp::RG == 1) {
        v[0] = fmaxf(v[0], long_dpp<0xB1>(v[0]));
        v[0] = fmaxf(v[0], long_dpp<0x4E>(v[0]));
        v[0] = fmaxf(v[0], long_dpp<0x141>(v[0]));
        if (Mp::LANES > 8) v[0] = fmaxf(v[0], long_dpp<0x140>(v[0]));
        if (Mp::LANES > 16) {
            const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[0]), __float_as_uint(v[0]), false, false);
            v[0] = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
        }
        if (Mp::LANES > 32) {
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[0]), __float_as_uint(v[0]), false, false);
            v[0] = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
        }
    } else {
#pragma unroll
        for (int off = 32; off >= Mp::RG; off >>= 1) v[0] = fmaxf(v[0], __shfl_xor(v[0], off));
    }
    if (Mp::WPR == 1) return;
    const int wave = tid >> 6, lane = tid & 63;
    __syncthreads();
    if (lane < Mp::RG) red[wave * Mp::RG + (COLS ? j : 0)] = v[0];
    __syncthreads();
    const int w0 = COLS ? 0 : j * Mp::WPR;
    float s = 0.f;
    for (int w = 0; w < Mp::WPR; ++w) s = fmaxf(s, red[(w0 + w) * Mp::RG + (COLS ? j : 0)]);
    v[0] = s;
}

// Segmented exclusive scan over the T threads of a row, from t = 0 upwards (DIR = +1) or
// from t = T-1 downwards (DIR = -1).  Each thread contributes (closed, s, n): `closed`
// says its chunk holds a segment boundary, and (s, n) describe the part of the chunk
// beyond its last boundary in scan direction (the whole chunk if there is none).
// ADD: open parts accumulate (sums and counts).  !ADD: the value of the nearest closed
// chunk is copied forward.  Returns what arrives at this thread from the scan's origin
// side; zero at the origin.  buf: [2][3][G][T] floats.
template <int T, int G, bool COLS, int DIR, bool ADD>
__device__ __forceinline__ void seg_scan(bool closed, float s, float n, float *buf, int j, int t,
                                         float &cs, float &cn)
{
    using Mp = LongMap<T, G, COLS>;
    if constexpr (Mp::RG == 1) {
        // A wave holds 64 consecutive threads of one row: scan inside the wave with lane
        // shuffles (no LDS, no barrier), then combine the waves' totals, which takes one
        // barrier.  combine(A earlier, B later) = B if B is closed, else A with B's open part
        // added (ADD) or A unchanged (copy).
        constexpr int LN = Mp::LANES;                     // lanes of the wave that hold this row
        const int lane = t & (LN - 1);
        float f = closed ? 1.f : 0.f;
#pragma unroll
        for (int d = 1; d < LN; d <<= 1) {
            const float of = DIR > 0 ? __shfl_up(f, d, LN) : __shfl_down(f, d, LN);
            const float os = DIR > 0 ? __shfl_up(s, d, LN) : __shfl_down(s, d, LN);
            const float on = DIR > 0 ? __shfl_up(n, d, LN) : __shfl_down(n, d, LN);
            const bool has = DIR > 0 ? (lane >= d) : (lane + d < LN);
            if (has && f == 0.f) {
                if (ADD) { s += os; n += on; } else { s = os; n = on; }
                f = of;
            }
        }
        // what arrives at this lane from inside its wave: the inclusive value of the lane before
        float ef = DIR > 0 ? __shfl_up(f, 1, LN) : __shfl_down(f, 1, LN);
        float es = DIR > 0 ? __shfl_up(s, 1, LN) : __shfl_down(s, 1, LN);
        float en = DIR > 0 ? __shfl_up(n, 1, LN) : __shfl_down(n, 1, LN);
        const bool edge = DIR > 0 ? (lane == 0) : (lane == LN - 1);
        if (edge) { ef = 0.f; es = 0.f; en = 0.f; }
        if constexpr (T > 64) {
            constexpr int NWR = T / 64;                       // waves per row
            float *tot = buf + (DIR > 0 ? 0 : 3 * G * NWR);   // the two directions never share
            const int w = t >> 6;
            const bool lastlane = DIR > 0 ? (lane == LN - 1) : (lane == 0);
            if (lastlane) {
                tot[(0 * G + j) * NWR + w] = f; tot[(1 * G + j) * NWR + w] = s; tot[(2 * G + j) * NWR + w] = n;
            }
            __syncthreads();
            // Exclusive scan over the waves' totals, done by every wave for itself: lane q (< NWR)
            // takes the totals of the q-th wave in scan order, a segmented inclusive scan runs
            // over those lanes (row-shift DPP: NWR <= 16 lanes lie in one DPP row), and the wave
            // picks the lane before its own position (a uniform index).
            static_assert(NWR <= 16, "the waves' totals must fit one 16-lane DPP row");
            const int wl = t & 63;
            float bf = 0.f, bs = 0.f, bn = 0.f;
            if (wl < NWR) {
                const int ww = DIR > 0 ? wl : NWR - 1 - wl;
                bf = tot[(0 * G + j) * NWR + ww]; bs = tot[(1 * G + j) * NWR + ww]; bn = tot[(2 * G + j) * NWR + ww];
            }
#define TV_SHR(v, D) __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x110 + (D), 0xf, 0xf, true))
#define TV_STEP(D)                                                                         \
            if constexpr ((D) < NWR) {                                                     \
                const float of = TV_SHR(bf, D), os = TV_SHR(bs, D), on = TV_SHR(bn, D);    \
                if (wl >= (D) && bf == 0.f) {                                              \
                    if (ADD) { bs += os; bn += on; } else { bs = os; bn = on; }            \
                    bf = of;                                                               \
                }                                                                          \
            }
            TV_STEP(1) TV_STEP(2) TV_STEP(4) TV_STEP(8)
#undef TV_STEP
#undef TV_SHR
            const int qme = DIR > 0 ? w : NWR - 1 - w;                 // this wave's position in scan order
            const int src = __builtin_amdgcn_readfirstlane(qme > 0 ? qme - 1 : 0);
            float af = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bf), src));
            float as = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bs), src));
            float an = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bn), src));
            if (qme == 0 || (!ADD && af == 0.f)) { as = 0.f; an = 0.f; }
            // combine(waves before, lanes before)
            if (ef == 0.f) {
                if (ADD) { es += as; en += an; } else { es = as; en = an; }
            }
        }
        cs = es; cn = en;
        return;
    } else {
#define TV_B(c, q, tt) buf[(((c) * 3 + (q)) * G + j) * T + (tt)]
    float f = closed ? 1.f : 0.f;
    int cur = 0;
    for (int d = 1; d < T; d <<= 1) {
        TV_B(cur, 0, t) = f; TV_B(cur, 1, t) = s; TV_B(cur, 2, t) = n;
        Mp::sync();
        const int o = t - DIR * d;
        if (o >= 0 && o < T && f == 0.f) {
            const float of = TV_B(cur, 0, o), os = TV_B(cur, 1, o), on = TV_B(cur, 2, o);
            if (ADD) { s += os; n += on; } else { s = os; n = on; }
            f = of;
        }
        cur ^= 1;
    }
    TV_B(cur, 1, t) = s; TV_B(cur, 2, t) = n;
    Mp::sync();
    const int o = t - DIR;
    cs = 0.f; cn = 0.f;
    if (o >= 0 && o < T) { cs = TV_B(cur, 1, o); cn = TV_B(cur, 2, o); }
    Mp::sync();
#undef TV_B
    }
}

// ---------------------------------------------------------------------------------
// The solver: projected Newton on the dual of one row (paper Eq. 3-4), T threads per row.
// ---------------------------------------------------------------------------------
//
// The Newton direction without a tridiagonal solve.  Between two held duals (and the ends of the
// row) the masked system of Eq. 4 asks for the free duals that make the gradient x_k - x_{k+1}
// vanish, that is, for an x that is constant on the block of samples between them; the block's
// sum is fixed by the two held duals, so that constant is the block's mean of the current x.
// Hence d_k = sum over the block's samples up to k of (x_i - mean), and the Newton decrement
// g^T d is the sum of the (x_i - mean)^2.  A step is thus one segmented sum over the row's threads
// and one mean fetched back from the thread in which a block ends.
//
// Sums that span threads are taken relative to a sample of the block itself (the first one in the
// thread where it begins): near the solution x is constant on a block up to rounding, so the
// differences are exact and so small that neither the length of the block nor its level costs
// digits.  That reference travels with the sum; all threads of a block see the same reference
// and the same mean, which makes the block's output value bit-identical in all of them.

// Votes: the lanes that pass, as a mask in scalar registers (the comparison's own result).
__device__ __forceinline__ uint64_t lanes_with(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ bool wave_any(bool p) { return lanes_with(p) != 0; }

// The lanes of one row inside one wave.
template <int T, int G, bool COLS>
struct RowWave {
    using Mp = LongMap<T, G, COLS>;
    static constexpr int RG = Mp::RG;                                    // lanes between neighbouring threads
    static constexpr int TW = RG == 1 ? (T < 64 ? T : 64) : 64 / RG;     // threads of the row in this wave
    static constexpr int NWR = Mp::WPR;                                  // waves of the row
    static constexpr bool MULTI = NWR > 1;
    static constexpr bool HALF = RG == 1 && TW <= 32;                    // the row's lanes lie in one half of the wave
    int lane, tw, home, wave;                    // home: lane of the row's first thread in this wave
    uint64_t before, after, first, last;         // the row's lanes below / above this one, its first, its last
    uint32_t before32, after32, first32, last32; // HALF: the same within the half

    __device__ __forceinline__ RowWave(int t)
    {
        lane = threadIdx.x & 63;
        if constexpr (RG == 1) { home = lane & ~(TW - 1); tw = lane & (TW - 1); }
        else { home = lane % RG; tw = lane / RG; }
        wave = MULTI ? (RG == 1 ? __builtin_amdgcn_readfirstlane(t >> 6) : (int)(threadIdx.x >> 6)) : 0;
        before = after = first = last = 0;
        before32 = after32 = first32 = last32 = 0;
        if constexpr (HALF) {
            const uint32_t row = (TW == 32 ? ~0u : (1u << (TW & 31)) - 1u) << (home & 31);
            const uint32_t me = 1u << (lane & 31);
            before32 = row & (me - 1u);
            after32 = row & ~before32 & ~me;
            first32 = 1u << (home & 31);
            last32 = first32 << (TW - 1);
        } else {
            uint64_t row = 0;
#pragma unroll
            for (int q = 0; q < TW; ++q) row |= 1ull << (q * RG);
            row <<= home;
            const uint64_t me = 1ull << lane;
            before = row & (me - 1ull);
            after = row & ~before & ~me;
            first = 1ull << home;
            last = first << ((TW - 1) * RG);
        }
    }
    __device__ __forceinline__ uint32_t half(uint64_t m) const { return (lane & 32) ? (uint32_t)(m >> 32) : (uint32_t)m; }
    // nearest lane of the row below this one whose bit is set in m, else the row's first lane
    __device__ __forceinline__ int last_before(uint64_t m) const
    {
        if constexpr (HALF) return 31 - __builtin_clz((half(m) & before32) | first32) + (lane & 32);
        else return 63 - __builtin_clzll((m & before) | first);
    }
    // ... above this one, else the row's last lane
    __device__ __forceinline__ int first_after(uint64_t m) const
    {
        if constexpr (HALF) return __builtin_ctz((half(m) & after32) | last32) + (lane & 32);
        else return __builtin_ctzll((m & after) | last);
    }
    __device__ __forceinline__ bool some_before(uint64_t m) const { return (m & before) != 0; }      // (not HALF)
    __device__ __forceinline__ bool some_after(uint64_t m) const { return (m & after) != 0; }
    // does any thread of the row in this wave pass `pred`?
    __device__ __forceinline__ bool any(bool pred) const
    {
        const uint64_t m = lanes_with(pred);
        if constexpr (RG == 1 && TW == 64) return m != 0;
        else if constexpr (HALF) return (half(m) & (before32 | after32 | (1u << (lane & 31)))) != 0;
        else return (m & (before | after | (1ull << lane))) != 0;
    }
    // v of the thread before / after this one in the row, inside the wave (0 at the wave's ends)
    __device__ __forceinline__ float prev(float v) const
    {
        if constexpr (RG > 1) { const float r = __shfl_up(v, RG); return tw == 0 ? 0.f : r; }
        else if constexpr (TW <= 16) return from_left<TW, 1>(v, tw);
        else { const float r = long_dpp<0x138>(v); return (TW < 64 && tw == 0) ? 0.f : r; }         // wave_shr:1
    }
    __device__ __forceinline__ float next(float v) const
    {
        if constexpr (RG > 1) { const float r = __shfl_down(v, RG); return tw == TW - 1 ? 0.f : r; }
        else if constexpr (TW <= 16) return from_right<TW, 1>(v, tw);
        else { const float r = long_dpp<0x130>(v); return (TW < 64 && tw == TW - 1) ? 0.f : r; }    // wave_shl:1
    }
    __device__ static __forceinline__ float at(float v, int from)
    {
        return __int_as_float(__builtin_amdgcn_ds_bpermute(from << 2, __float_as_int(v)));
    }
    // Segmented sum: v of this thread and of the `dist` threads before it (in this wave).  Row
    // shifts inside the 16-lane rows, broadcasts of a row's last lane across them; a step that no
    // lane needs is skipped.  (Selects, not masks: a neighbouring row's NaN stays out.)
    __device__ __forceinline__ float open_sum(float v, int dist) const
    {
        if constexpr (RG > 1) {
#pragma unroll
            for (int s = 1; s < TW; s <<= 1) {
                const float o = __shfl_up(v, s * RG);
                if (dist >= s) v += o;
            }
            return v;
        } else {
#define TV_STEP(S)                                                                  \
            if constexpr ((S) < TW) {                                               \
                if (wave_any(dist >= (S))) {                                   \
                    const float o = long_dpp<0x110 + ((S) & 15)>(v);                \
                    v += dist >= (S) ? o : 0.f;                                     \
                }                                                                   \
            }
            TV_STEP(1) TV_STEP(2) TV_STEP(4) TV_STEP(8)
#undef TV_STEP
            if constexpr (TW > 16) {
                const bool take = dist > (lane & 15);                     // row_bcast:15 into the odd 16-lane rows
                if (wave_any(take)) {
                    const float o = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x142, 0xa, 0xf, false));
                    v += take ? o : 0.f;
                }
            }
            if constexpr (TW > 32) {
                const bool take = dist > (lane & 31);                     // row_bcast:31 into the upper half
                if (wave_any(take)) {
                    const float o = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x143, 0xc, 0xf, false));
                    v += take ? o : 0.f;
                }
            }
            return v;
        }
    }
};

template <int T, int C, int G, bool COLS>
struct RowSmem {
    using Mp = LongMap<T, G, COLS>;
    using Rw = RowWave<T, G, COLS>;
    static constexpr bool M = Rw::MULTI;
    // The input is read once per Newton step, for the x of the trial point: with 8 samples per thread
    // and more it waits in LDS (each thread its own chunk, 16 bytes at a time, consecutive lanes in
    // consecutive slots), not in registers.
    static constexpr bool PARK = C >= 8;
    float4 y[PARK ? C / 4 : 1][PARK ? T * G : 1];
    float rtab[C + 1];                                 // rtab[m] = 1 / m
    // rows that span waves: the open block at the end of every wave (closed?, reference, sum, count);
    // its votes (flags, decrement, first and last block value, dual held at its end); the mean of the
    // block that ends first in a wave; chunk edges; partial sums
    float tot[M ? 4 : 1][M ? G : 1][M ? Mp::WPR : 1];
    float vote[M ? 5 : 1][M ? G : 1][M ? Mp::WPR : 1];
    float head[M ? G : 1][M ? Mp::WPR : 1];
    float edge[M ? 2 : 1][2][M ? G : 1][M ? Mp::WPR + 1 : 1];
    float red[M ? 2 * 4 * Mp::NW * Mp::RG : 1];
    float buf[!M ? 1 : (Mp::RG == 1 ? 2 * 3 * G * Mp::WPR : 2 * 3 * G * T)];      // seg_scan
    __device__ __forceinline__ void init(int tid)
    {
        if (tid <= C) rtab[tid] = tid > 0 ? 1.0f / (float)tid : 0.f;
    }
    // 1 / m from 4 m
    __device__ __forceinline__ float reciprocal(uint32_t at) const
    {
        return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(rtab) + at);
    }
    __device__ __forceinline__ void park(int tid, const float (&v)[C])
    {
        if constexpr (PARK) {
#pragma unroll
            for (int q = 0; q < C / 4; ++q) y[q][tid] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
        }
    }
    // The thread's chunk again (without PARK it is `kept`).  The memory clobber makes the compiler
    // load it here instead of keeping it from the last time.
    __device__ __forceinline__ void fetch(int tid, const float (&kept)[C], float (&v)[C]) const
    {
        if constexpr (!PARK) {
#pragma unroll
            for (int i = 0; i < C; ++i) v[i] = kept[i];
        } else {
            asm volatile("" ::: "memory");
#pragma unroll
            for (int q = 0; q < C / 4; ++q) {
                const float4 w = y[q][tid];
                v[4 * q] = w.x; v[4 * q + 1] = w.y; v[4 * q + 2] = w.z; v[4 * q + 3] = w.w;
            }
        }
    }
};

// Sum of f over a row that spans waves, and the OR of a flag, with one barrier (consecutive calls
// alternate between two halves of the buffer).
template <int T, int C, int G, bool COLS>
__device__ __forceinline__ void row_totals(const RowWave<T, G, COLS> &rw, RowSmem<T, C, G, COLS> &sm, int j, int tid,
                                           int &par, float &f, bool &ch)
{
    using Rw = RowWave<T, G, COLS>;
    using Mp = LongMap<T, G, COLS>;
    if constexpr (Rw::RG == 1) {
        f = wave_sum_all<Mp::LANES>(f);
        ch = rw.any(ch);
        float *r = sm.red + par * (2 * Mp::NW);
        par ^= 1;
        if (rw.lane == 0) { r[rw.wave] = f; r[Mp::NW + rw.wave] = ch ? 1.f : 0.f; }
        __syncthreads();
        const int e = rw.lane & 15;
        const float v = r[e < Rw::NWR ? e : 0], c = r[Mp::NW + (e < Rw::NWR ? e : 0)];
        f = wave_sum_all<16>(e < Rw::NWR ? v : 0.f);
        ch = wave_any(c != 0.f);
    } else {
        float v[2] = {f, ch ? 1.f : 0.f};
        row_sum_alt<T, G, COLS, 2>(v, sm.red, j, tid, par);
        par ^= 1;
        f = v[0];
        ch = v[1] != 0.f;
    }
}

// One row solved by the T threads that hold it.  y: the thread's chunk of the row (zero past the
// end, n samples in the row); every thread of the workgroup calls, rows that do not exist with
// valid = false.  xs receives the chunk of the minimiser, u the final dual (DUAL; and sm.fetch has y
// again, which frees its registers during the solve).  Returns the step count and flags of
// FwdParams::info.
//   WARM 0: from the bounds the local differences point to.  1: from the dual whose negated running
//   sums inside the chunk are in u on entry (wsum: the chunk's total).  2: as 0, or, where cu is
//   given, from the dual cu (coarse_n entries) of the row averaged in groups of kMlFactor.
//   3: as 0, or from the constant row's dual (see there).
//   POLISH: a clipped trial point is polished by two Gauss-Seidel sweeps.  DEBUG: rec, if not null, receives the row's step record.
//   DUAL: the caller wants u (coarse levels, whose rows have unit stride); else it is left where the row landed.
template <int T, int C, int G, bool COLS, int WARM, bool POLISH, bool DEBUG, bool DUAL>
__device__ __forceinline__ int row_solve(const float (&y)[C], float (&u)[C], float wsum, float lam, int n, int j,
                                         int t, bool valid, RowSmem<T, C, G, COLS> &sm, const float *cu,
                                         int coarse_n, float *rec, float (&xs)[C])
{
    using Mp = LongMap<T, G, COLS>;
    using Rw = RowWave<T, G, COLS>;
    constexpr bool MULTI = Rw::MULTI;
    constexpr bool SHARED = MULTI ? G > 1 : Rw::TW < 64;       // rows share a wave
    constexpr bool KEEP = DUAL && SHARED;
    static_assert(!POLISH || !MULTI, "rows inside one wave");
    // (the flags of FwdParams::info, shifted into the range of inline constants)
    constexpr int kConverged = kInfoConverged >> 16, kStalled = kInfoStalled >> 16, kCapped = kInfoCapped >> 16,
                  kPlain = kInfoPlain >> 16;
    const Rw rw(t);
    const int tid = threadIdx.x;
    const int k0 = t * C, M = n - 1;
    int par = 0, epar = 0;

    // value `last` of the thread before this one and `first` of the one after it (0 beyond the row)
    auto edges = [&](float first, float last, float &left, float &right) {
        left = rw.prev(last);
        right = rw.next(first);
        if constexpr (MULTI) {
            auto &ed = sm.edge[epar];
            epar ^= 1;
            if (rw.tw == Rw::TW - 1) ed[0][j][rw.wave + 1] = last;
            if (rw.tw == 0) ed[1][j][rw.wave] = first;
            __syncthreads();
            if (rw.tw == 0) left = rw.wave > 0 ? ed[0][j][rw.wave] : 0.f;
            if (rw.tw == Rw::TW - 1) right = rw.wave + 1 < Rw::NWR ? ed[1][j][rw.wave + 1] : 0.f;
        }
    };

    // rounding floor of a difference of two x values (|x| <= max|y|, |u| <= lam)
    float gtol;
    {
        float ym[1] = {0.f};
#pragma unroll
        for (int i = 0; i < C; ++i) ym[0] = fmaxf(ym[0], fabsf(y[i]));
        row_max<T, G, COLS>(ym, sm.red, j, tid);
        // lam_max = max_k |sum_{i<=k} (mean(y) - y_i)| = max_k |(k / n) sum_{i>k} y_i -
        // ((n - k) / n) sum_{i<=k} y_i| <= 2 k (n - k) / n max|y| <= n / 2 max|y|, and every lambda from
        // lam_max on gives the same minimiser (the row's mean): a lambda beyond that bound is
        // replaced by it, which keeps the dual box, and with it the rounding errors of
        // x = y - D^T u, at the scale of the data.  The cold start needs it (it puts the duals on
        // the bounds), and so does a start from a coarser level's dual, whose stopping tolerance
        // scales with lambda; a pass that starts from the dual an addend encodes is left alone.
        if constexpr (WARM != 1) lam = fminf(lam, 0.51f * (float)n * ym[0]);
        gtol = kGradNoise * (ym[0] + lam);
    }

    // duals past the end of the row are held at 0 and never move
    const int nvd = min(max(M - k0, 0), C);            // duals of this chunk inside the row
    // (where a row spans several waves the comparison is redone from an opaque copy of nvd in
    // every phase: as a loop invariant the compiler keeps all C results in scalar register pairs
    // for the whole solve, and those kernels then spill scalar registers by the hundred; the
    // wave-per-row kernels have the registers to spare and are faster with the invariant)
    int nv = nvd;
#define TV_NV_REFRESH() do { if constexpr (MULTI) { nv = nvd; asm volatile("" : "+v"(nv)); } } while (0)
#define TV_LK(i) (((i) < nv) ? lam : 0.0f)
    TV_NV_REFRESH();

    float ynext0, unused;
    edges(y[0], 0.f, unused, ynext0);

    // ---- starting point: every dual at the bound its local difference points to, or the dual
    //      the addend encodes, brought into the box (duals within rounding distance of a bound onto it)
    if constexpr (WARM == 1) {
        float before;
        if constexpr (MULTI) {
            seg_scan<T, G, COLS, +1, true>(false, wsum, 0.f, sm.buf, j, t, before, unused);
        } else {
            before = rw.prev(rw.open_sum(wsum, rw.tw));
        }
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const float l = TV_LK(i);
            u[i] = __builtin_amdgcn_fmed3f((u[i] + before) * kWarmSnap, -l, l);
        }
    } else {
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const float l = TV_LK(i);
            const float dy = ((i + 1 < C) ? y[i + 1] : ynext0) - y[i];
            u[i] = __builtin_amdgcn_fmed3f(dy * 1e30f, -l, l);
        }
    }
    if constexpr (WARM == 3) {
        // The other candidate: the dual of the constant row, u_k = sum_{i <= k} (mean(y) -
        // y_i), clipped into the box.  It is the solution whenever lam >= lam_max =
        // max_k |u_k|, and from lam_max / 4 on it is the better start by far (few segments:
        // from the bounds every Newton step frees only a few more duals, and random-walk
        // rows of 5000-16 384 samples with lambda from 0.3 lam_max on were still moving
        // after 128 steps; from here they take a handful).  Below lam_max / 4 the bounds
        // win.  Three more row-wide reductions: only the long rows that cannot take the
        // multilevel start pay for it (5-15 % of a cold call).
        int ns = min(max(n - k0, 0), C);               // samples of this chunk inside the row
        asm volatile("" : "+v"(ns));
        float tot[1] = {0.f};
#pragma unroll
        for (int i = 0; i < C; ++i) tot[0] += (i < ns) ? y[i] : 0.f;
        row_sum<T, G, COLS, 1>(tot, sm.red, j, tid);
        const float mean = tot[0] / (float)n;
        float mine = 0.f;
#pragma unroll
        for (int i = 0; i < C; ++i) mine += (i < ns) ? mean - y[i] : 0.f;
        float before;
        seg_scan<T, G, COLS, +1, true>(false, mine, 0.f, sm.buf, j, t, before, unused);
        float run = before;
        float am[1] = {0.f};
#pragma unroll
        for (int i = 0; i < C; ++i) {
            run += mean - y[i];
            if (i < nv) am[0] = fmaxf(am[0], fabsf(run));
        }
        row_max<T, G, COLS>(am, sm.red, j, tid);
        if (lam >= 0.25f * am[0]) {                    // (never with a NaN or Inf in the row)
            run = before;
#pragma unroll
            for (int i = 0; i < C; ++i) {
                const float l = TV_LK(i);
                run += mean - y[i];
                u[i] = __builtin_amdgcn_fmed3f(run, -l, l);
            }
        }
    }
    if constexpr (WARM == 2) {
        // Prolongation of the coarse dual.  The coarse row is this row with every group of
        // kMlFactor samples replaced by its mean, and its dual uc solves the same problem
        // restricted to rows that are constant on the groups (lambda / kMlFactor there).
        // At the knot behind a group the fine dual is kMlFactor * uc (exact for a power of
        // two, so bound coarse duals give bound fine duals); inside a group it follows
        // u_k = u_{k-1} + (x_group - y_k) with the group's coarse x, clipped into the box.
        static_assert(WARM != 2 || C % kMlFactor == 0, "groups must not straddle chunks");
        if (cu) {
            constexpr int F = kMlFactor;
            const int j0 = k0 / F;
            float ucl = (j0 > 0 && j0 - 1 < coarse_n) ? cu[j0 - 1] : 0.f;
#pragma unroll
            for (int c = 0; c < C / F; ++c) {
                const float ucr = (j0 + c < coarse_n) ? cu[j0 + c] : 0.f;
                float sum = 0.f, cnt = 0.f;
#pragma unroll
                for (int r = 0; r < F; ++r)
                    if (k0 + c * F + r < n) { sum += y[c * F + r]; cnt += 1.f; }
                const float xg = (cnt > 0.f ? sum / cnt : 0.f) + ucr - ucl;
                float run = (float)F * ucl;
#pragma unroll
                for (int r = 0; r < F - 1; ++r) {
                    const float l = TV_LK(c * F + r);
                    run += xg - y[c * F + r];
                    u[c * F + r] = __builtin_amdgcn_fmed3f(run, -l, l);
                }
                const float l = TV_LK(c * F + F - 1);
                u[c * F + F - 1] = __builtin_amdgcn_fmed3f((float)F * ucr, -l, l);
                ucl = ucr;
            }
        }
    }

    // x(u) of the thread's chunk, the first sample of the next one, and half the row's squared norm
    float x[C], xnext0, uleft, fcur;
    {
        float uright;
        edges(u[0], u[C - 1], uleft, uright);
        float acc = 0.f;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            x[i] = y[i] + u[i] - (i > 0 ? u[i - 1] : uleft);
            acc = fmaf(x[i], x[i], acc);
        }
        xnext0 = rw.next(x[0]);
        if (MULTI && rw.tw == Rw::TW - 1) xnext0 = ynext0 + uright - u[C - 1];
        if constexpr (MULTI) {
            bool none = false;
            row_totals(rw, sm, j, tid, par, acc, none);
        } else {
            acc = wave_sum_all<Mp::LANES>(acc);
        }
        fcur = 0.5f * acc;
    }

    // (the data's scale, taken back out of gtol)
    const float scale = 1.f + fmaxf(gtol * (1.0f / kGradNoise) - lam, 0.f);
    sm.park(tid, y);
    // n samples moved by 2 ulp of max|y| + lam each.  (It is 0, as gtol^2 is, where such squares underflow:
    // the tests against both are strict, or every clipped point of a row of 1e-24 would pass for the end.)
    const float noise = (float)n * gtol * gtol * (1.f / 64.f);
    // A row that has landed is done: it ends on the block means of the x it landed from, whatever the rows
    // that share its wave or workgroup still do.  While they go on, its dual stays where it landed from
    // and every trip forms the same means from it.  (DUAL forms the landing step anew in every trip, so that
    // the last one has it; formed once more at the end instead, the three arrays it takes were 4-9 registers
    // spilled in the kernels of 8 and 12 samples a thread.)
    bool active = valid, done = false;
    int steps = 0, flags = 0, quiet = 0;
    if constexpr (DEBUG) {
        if (rec && t == 0) { rec[0] = 0.f; rec[1] = lam; rec[kRecF] = fcur; }
    }

    // what the primal recovery needs of the last iteration: the held duals, and the values of the
    // blocks that end at the first one and begin behind the last one
    uint32_t held;
    float head_x, tail_x, uc[C];
    for (int it = 0;; ++it) {
        TV_NV_REFRESH();
        // ---- gradient and bound set (Bertsekas' sign test with exact comparisons: a clipped dual
        //      is bit-equal to +-lam); f[i] = 0 where dual i is held, which ends a block
        bool bnd[C], closed = false;
        float f[C];
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const float up = ((i + 1 < C) ? x[i + 1] : xnext0) - x[i];             // minus the gradient
            bnd[i] = (i >= nv) | (u[i] == copysignf(lam, up));
            f[i] = bnd[i] ? 0.f : 1.f;
            closed |= bnd[i];
        }
        // ---- sums of the thread's pieces, relative to its first sample: tail, behind its last held
        //      dual (the whole chunk if it has none), head, up to its first one, and the means m[i]
        //      of the blocks that end in it at dual i, as if they had begun in it too
        const float x0 = x[0];
        const float xlast = bnd[C - 1] ? xnext0 : x[C - 1];     // a sample of the block open at the chunk's end
        float m[C];
        float tail_s, tail_n, head_s, head_n;
        {
            float s = 0.f;
            uint32_t at = 4;                                   // 4 x the samples of the piece so far
            x[0] = 0.f;
            m[0] = 0.f;
#pragma unroll
            for (int i = 1; i < C; ++i) {
                x[i] -= x0;
                s = i > 1 ? fmaf(f[i - 1], s, x[i]) : x[i];
                at = bnd[i - 1] ? 4u : at + 4u;
                asm volatile("" : "+v"(at));                   // a select, not a branch around a table load
                m[i] = s * sm.reciprocal(at);
            }
            tail_s = bnd[C - 1] ? 0.f : s;
            tail_n = bnd[C - 1] ? 0.f : 0.25f * (float)at;
            head_s = C > 1 ? x[C - 1] : 0.f;
            head_n = 1.f;
#pragma unroll
            for (int i = C - 2; i >= 0; --i) {
                head_s = i > 0 ? fmaf(f[i], head_s, x[i]) : f[i] * head_s;
                head_n = fmaf(f[i], head_n, 1.f);
            }
        }
        // ---- the block that is open at the chunk's start: begun in thread L, the last one before
        //      this with a held dual.  ref: its reference; left_s, left_n: sum and count of its samples
        //      in the threads before this one
        const uint64_t cmask = lanes_with(closed);
        const int L = rw.last_before(cmask);                   // (or the row's first thread in this wave)
        float ref = Rw::at(closed ? xlast : x0, L);
        float left_n = Rw::at(tail_n, L);
        const int apart = (rw.lane - L) / Rw::RG;              // threads of the row since L
        left_n += (float)(apart * C - C);
        if (rw.tw == 0) { ref = x0; left_n = 0.f; }
        // what this thread adds to the block open at its end
        const float mine = closed ? fmaf(-tail_n, xlast - x0, tail_s) : fmaf((float)C, x0 - ref, tail_s);
        const float upto = rw.open_sum(mine, closed ? 0 : apart);
        float left_s = rw.prev(upto);

        uint32_t wmask = 0;                                    // MULTI, RG == 1: the row's waves with a held dual
        bool none_before = false;
        if constexpr (MULTI) {
            // hand the block open at the wave's end over to the waves behind it
            const bool wclosed = rw.any(closed);
            if (rw.tw == Rw::TW - 1) {
                sm.tot[0][j][rw.wave] = wclosed ? 1.f : 0.f;
                sm.tot[1][j][rw.wave] = closed ? xlast : ref;
                sm.tot[2][j][rw.wave] = upto;
                sm.tot[3][j][rw.wave] = closed ? tail_n : left_n + (float)C;
            }
            __syncthreads();
            float cref, cs = 0.f, cn = 0.f;
            if constexpr (Rw::RG == 1) {
                static_assert(Rw::NWR <= 16, "the waves' entries must fit one 16-lane DPP row");
                const int e = rw.lane < Rw::NWR ? rw.lane : 0;
                const float tr = sm.tot[1][j][e], ts = sm.tot[2][j][e], tn = sm.tot[3][j][e];
                wmask = (uint32_t)lanes_with(rw.lane < Rw::NWR && sm.tot[0][j][e] != 0.f);
                const uint32_t bw = wmask & ((1u << rw.wave) - 1u);
                const int W = bw ? 31 - __builtin_clz(bw) : 0;
                cref = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(tr), W));
                const bool in = rw.lane >= W && rw.lane < rw.wave;
                cs = wave_sum_all<16>(in ? fmaf(tn, tr - cref, ts) : 0.f);
                cn = wave_sum_all<16>(in ? tn : 0.f);
                cs = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(cs)));
                cn = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(cn)));
            } else {
                int W = 0;
                for (int w = 0; w < rw.wave; ++w)
                    if (sm.tot[0][j][w] != 0.f) W = w;
                cref = sm.tot[1][j][W];
                for (int w = W; w < rw.wave; ++w) {
                    cs += fmaf(sm.tot[3][j][w], sm.tot[1][j][w] - cref, sm.tot[2][j][w]);
                    cn += sm.tot[3][j][w];
                }
            }
            none_before = !rw.some_before(cmask);              // the block comes from an earlier wave
            if (none_before && rw.wave > 0) {
                left_s = cs + fmaf(left_n, ref - cref, left_s);
                left_n += cn;
                ref = cref;
            }
        }
        // ---- the thread in which the block ends knows its mean; the others fetch it
        const float head_m = fmaf(head_n, x0 - ref, left_s + head_s) * __builtin_amdgcn_rcpf(left_n + head_n);
        //      (the row's last thread always holds one; a wave's last thread need not)
        float tail_m = Rw::at(head_m, rw.first_after(cmask));
        if constexpr (MULTI) {
            const bool none_after = !rw.some_after(cmask);     // the block goes on in the next wave
            if (closed && none_before) sm.head[j][rw.wave] = head_m;
            __syncthreads();
            if constexpr (Rw::RG == 1) {
                const uint32_t aw = wmask >> (rw.wave + 1);
                const float far = sm.head[j][aw ? rw.wave + 1 + __builtin_ctz(aw) : rw.wave];
                if (none_after) tail_m = far;
            } else if (none_after) {
                int w = rw.wave + 1;
                while (w < Rw::NWR - 1 && sm.tot[0][j][w] == 0.f) ++w;
                tail_m = sm.head[j][w < Rw::NWR ? w : rw.wave];
            }
        }
        const float tail_ref = closed ? xlast : ref;
        const float open_m = closed ? head_m : tail_m;         // mean of the block open at the chunk's start
        const float head_v = open_m + (ref - x0);              // the same relative to x0, and of the block
        const float tail_v = tail_m + (tail_ref - x0);         // open at the chunk's end
        bool seen[C];                                          // a held dual before dual i in this chunk
        seen[0] = false;
#pragma unroll
        for (int i = 1; i < C; ++i) seen[i] = seen[i - 1] | bnd[i - 1];

        if (active && it >= kMaxNewtonSteps) { active = false; flags = kCapped; }
        bool go = wave_any(active);      // (a row's flag is the same in all its threads)

        // ---- Newton direction: running sum of x - mean, 0 on the held duals; decrement
        float d[C], decp = 0.f;
        {
            float v = tail_v;
#pragma unroll
            for (int i = C - 1; i >= 0; --i) {
                if (bnd[i]) v = seen[i] ? m[i] : head_v;
                x[i] -= v;
            }
            float run = fmaf(-left_n, open_m, left_s);
#pragma unroll
            for (int i = 0; i < C; ++i) {
                decp = fmaf(x[i], x[i], decp);
                run = f[i] * (run + x[i]);
                d[i] = run;
            }
        }
        if constexpr (DEBUG) {
            if (rec && it == 0) {
#pragma unroll
                for (int i = 0; i < C; ++i)
                    if (i < nvd) {
                        rec[kRecU + k0 + i] = u[i];
                        rec[kRecU + n + k0 + i] = d[i];
                        rec[kRecU + 2 * n + k0 + i] = bnd[i] ? 1.f : 0.f;
                    }
            }
        }
        // ---- the step, projected
        float alpha = active || (KEEP && done) ? 1.f : 0.f;
        float ucleft, ucright, dec;
        bool clipped = false;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const float tt = fmaf(-alpha, d[i], u[i]);
            uc[i] = __builtin_amdgcn_fmed3f(tt, -lam, lam);
            clipped |= (uc[i] != tt);
        }
        // ---- optimality, looked at before the step is taken: it lands on the block means (nothing
        //      clipped), and there no held dual is pushed inwards by more than the rounding floor.
        //      (That floor follows lambda.  A start from a coarser level's dual can land in its first or
        //      second step, and where lambda is large against the data, a step that moved x by more
        //      than 2 % of the data's scale, in the 2-norm, does not end the solve: the next, small
        //      one takes back what the floor let pass.)
        //      POLISH, WARM = 3 (TINY): or, with the same signs, the decrement, the squared length of the
        //      move of x, is below the floor of a difference of two x values, squared: no sample would
        //      move.  (A polished point and the Newton step from it can swap a last ulp for ever; the
        //      constant row's dual can leave a dual exactly on its bound with a gradient that is
        //      rounding noise, lambda = lam_max being the extreme case, which changes sides with every
        //      step.  For the others the floor, which follows lambda, is too coarse an end.)
        //      All: or, with the same signs, this is the third step that moves x by no more than its own
        //      rounding: a free dual that touches its bound without a jump is clipped by noise every time.
        //      A held dual that is pushed inwards by less than the floor has no jump to stand for: the row
        //      is done, but its blocks are those of the bound set behind the step (`soft`: one more
        //      look at x, without a step).
        bool soft = false;
        auto pushed = [&](float vnext) {                       // vnext: relative to x0, behind the chunk
            bool p = false;
            float vr = vnext, v = tail_v;
#pragma unroll
            for (int i = C - 1; i >= 0; --i) {
                if (bnd[i]) v = seen[i] ? m[i] : head_v;
                const float g = v - vr;
                const bool in = bnd[i] & (u[i] == copysignf(lam, g));
                p |= in & (fabsf(g) > gtol);
                soft |= in & (g != 0.f);
                vr = v;
            }
            return p;
        };
        constexpr bool TINY = POLISH || WARM == 3;
        bool landed;
        //      Rows that share a wave: a last step that moves the samples by more than max|y| / 16 (root of
        //      the mean square) comes from an x of large duals, lambda >> the data as a rule, whose
        //      rounding is in its block means, so that one gets another look as well.  (Rows of 20, 0/1
        //      samples, lambda 10^U(-2, 1): relative error 2.7e-8, without it 1.9e-7.  A look behind every
        //      last step is hardly closer, 4.41e-8 against 4.44e-8 on N(0, 1), and 9 % slower on planes of 64 x 64.)
        auto far = [&]() {
            const float ym = gtol * (1.0f / kGradNoise) - lam;
            return SHARED && dec > (1.f / 256.f) * (float)n * ym * ym;
        };
        if constexpr (MULTI) {
            // the votes ride on the exchange of the trial's chunk edges
            const float vfirst = x0 + head_v;
            float vn = rw.next(vfirst);
            const bool last = rw.tw == Rw::TW - 1;
            bool p = pushed(last ? (bnd[C - 1] ? (seen[C - 1] ? m[C - 1] : head_v) : tail_v) : vn - x0);
            const float vlast = x0 + (bnd[C - 1] ? (seen[C - 1] ? m[C - 1] : head_v) : tail_v);
            p = rw.any(p);
            soft = rw.any(soft);
            clipped = rw.any(clipped);
            float ds = decp;
            if constexpr (Rw::RG == 1) ds = wave_sum_all<64>(ds);
            else {
#pragma unroll
                for (int o = 32; o >= Rw::RG; o >>= 1) ds += __shfl_xor(ds, o);
            }
            if (rw.tw == 0) {
                sm.vote[0][j][rw.wave] = __int_as_float((p ? 1 : 0) | (clipped ? 2 : 0) | (soft ? 4 : 0));
                sm.vote[1][j][rw.wave] = ds;
                sm.vote[2][j][rw.wave] = vfirst;
            }
            if (last) {
                sm.vote[3][j][rw.wave] = vlast;
                sm.vote[4][j][rw.wave] = bnd[C - 1] ? u[C - 1] : 0.f;
            }
            edges(uc[0], uc[C - 1], ucleft, ucright);
            p = false; clipped = false; soft = false; dec = 0.f;
            auto look = [&](int w) {
                const int v = __float_as_int(sm.vote[0][j][w]);
                const float g = sm.vote[3][j][w] - sm.vote[2][j][w + 1 < Rw::NWR ? w + 1 : w];
                const float ul = sm.vote[4][j][w];
                const bool in = ul != 0.f && ul == copysignf(lam, g);
                p |= (v & 1) != 0 || (in && fabsf(g) > gtol);
                clipped |= (v & 2) != 0;
                soft |= (v & 4) != 0 || (in && g != 0.f);
                return sm.vote[1][j][w];
            };
            if constexpr (Rw::RG == 1) {
                const int e = rw.lane & 15;
                const float one = look(e < Rw::NWR ? e : 0);
                p = wave_any(p);
                soft = wave_any(soft);
                clipped = wave_any(clipped);
                dec = wave_sum_all<16>(e < Rw::NWR ? one : 0.f);
            } else {
                for (int w = 0; w < Rw::NWR; ++w) dec += look(w);
            }
            quiet += dec < noise ? 1 : 0;
            landed = (!clipped || (TINY && dec < gtol * gtol) || quiet > 2) && !p;
            soft |= far();
        } else {
            clipped = rw.any(clipped);
            dec = wave_sum_all<Mp::LANES>(decp);
            landed = false;
            quiet += dec < noise ? 1 : 0;
            const bool may = active && (!clipped || (TINY && dec < gtol * gtol) || quiet > 2);
            if (wave_any(may)) {
                landed = may & !rw.any(pushed(rw.next(x0 + head_v) - x0));
                soft = rw.any(soft) || far();
            }
        }
        if (WARM == 2 && lam > 0.25f * scale && !(dec <= fmaxf(gtol * gtol, 4e-4f * scale * scale))) landed = false;
        const bool look_again = active && landed && soft;
        if constexpr (DEBUG) {                                 // the objective behind the last step
            if (wave_any(active && landed)) {                  // (uniform in the workgroup: one row, or a row per wave)
                if constexpr (!MULTI) edges(uc[0], uc[C - 1], ucleft, ucright);
                float yl[C], acc = 0.f;
                sm.fetch(tid, y, yl);
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    const float xi = yl[i] + uc[i] - (i > 0 ? uc[i - 1] : ucleft);
                    acc = fmaf(xi, xi, acc);
                }
                bool none = false;
                if constexpr (MULTI) row_totals(rw, sm, j, tid, par, acc, none);
                else acc = wave_sum_all<Mp::LANES>(acc);
                if (rec && t == 0 && active && landed) {
                    const int c = (int)rec[0] + 1;
                    if (c < kRecMaxF) { rec[kRecF + c] = 0.5f * acc; rec[0] = (float)c; }
                }
            }
        }
        bool landed_now = false;
        if (active && landed) { active = false; flags = kConverged; ++steps; landed_now = !soft; }
        done |= landed_now;
        if (go) go = wave_any(active || look_again);

        if (!go) {                                             // every row of the wave (workgroup) has stopped
            held = 0;
#pragma unroll
            for (int i = 0; i < C; ++i) held |= bnd[i] ? 1u << i : 0u;
            head_x = ref + head_m;
            tail_x = tail_ref + tail_m;
            break;
        }
        if constexpr (SHARED) {
            const bool freeze = KEEP ? done : landed_now;
            if (wave_any(freeze)) {                            // (uniform in the workgroup where rows span waves)
                if (freeze) {
#pragma unroll
                    for (int i = 0; i < C; ++i) uc[i] = u[i];
                }
                if constexpr (MULTI) edges(uc[0], uc[C - 1], ucleft, ucright);
            }
        }

        // ---- the trial point, its x and its objective; Armijo test with quadratic interpolation
        float xc[C], fc, xcnext0;
        bool changed = true;
        {
            if constexpr (!MULTI) edges(uc[0], uc[C - 1], ucleft, ucright);
            float yl[C];
            sm.fetch(tid, y, yl);
            if constexpr (POLISH) {
                // A clipped trial point is polished by two Gauss-Seidel sweeps (exact minimisation
                // of the dual objective over one dual at a time, inside the box), each thread over
                // its own chunk with its neighbours' trial values held: the duals that the clip
                // stopped at a bound let go of the ones next to them, which Newton's direction for
                // the old bound set could not know.  The result goes through the Armijo test like
                // any clipped step.  (CPU prototype, 32 x 32 feature maps: 14 % fewer trips of the
                // slowest row of a pass, and hardly any backtracking.)
                if (wave_any(clipped && active)) {
                    if (clipped && active) {            // (in place: no lane of another row takes part)
#pragma unroll
                        for (int i = 0; i < C; ++i) {
                            const float l = TV_LK(i);
                            const float hd = 0.5f * (((i + 1 < C) ? yl[i + 1] : ynext0) - yl[i]);
                            const float nb = (i > 0 ? uc[i - 1] : ucleft) + (i + 1 < C ? uc[i + 1] : ucright);
                            uc[i] = __builtin_amdgcn_fmed3f(fmaf(0.5f, nb, hd), -l, l);
                        }
#pragma unroll
                        for (int i = C - 1; i >= 0; --i) {
                            const float l = TV_LK(i);
                            const float hd = 0.5f * (((i + 1 < C) ? yl[i + 1] : ynext0) - yl[i]);
                            const float nb = (i > 0 ? uc[i - 1] : ucleft) + (i + 1 < C ? uc[i + 1] : ucright);
                            uc[i] = __builtin_amdgcn_fmed3f(fmaf(0.5f, nb, hd), -l, l);
                        }
                    }
                    edges(uc[0], uc[C - 1], ucleft, ucright);
                }
            }
            float acc = 0.f;
#pragma unroll
            for (int i = 0; i < C; ++i) {
                xc[i] = yl[i] + uc[i] - (i > 0 ? uc[i - 1] : ucleft);
                acc = fmaf(xc[i], xc[i], acc);
            }
            xcnext0 = rw.next(xc[0]);
            if (MULTI && rw.tw == Rw::TW - 1) xcnext0 = ynext0 + ucright - uc[C - 1];
            if constexpr (MULTI) {
                bool ch = false;
#pragma unroll
                for (int i = 0; i < C; ++i) ch |= (uc[i] != u[i]);
                row_totals(rw, sm, j, tid, par, acc, ch);
                changed = ch;
            } else {
                acc = wave_sum_all<Mp::LANES>(acc);
            }
            fc = 0.5f * acc;
        }
        // a row with NaN in it stops here and keeps x = y - D^T u as it stands
        if (active && fc != fc) { active = false; flags = kStalled | kPlain; }
        bool ok = !active || !clipped || fc <= fcur - kArmijoSigma * dec + kArmijoSlackEps * fabsf(fcur);
        if (wave_any(!ok)) {                                   // (uniform in the workgroup: see go)
            // rows that fail try shorter steps along the same direction; the others keep their trial point
            for (int ls = 0;; ++ls) {
                if (!ok) {
                    const float den = 2.f * (fc - fcur + dec * alpha);
                    const float an = den > 0.f ? dec * alpha * alpha / den : 0.5f * alpha;
                    alpha = ls >= kMaxBacktracks ? 0.f : fminf(fmaxf(an, 0.1f * alpha), 0.5f * alpha);
#pragma unroll
                    for (int i = 0; i < C; ++i) uc[i] = __builtin_amdgcn_fmed3f(fmaf(-alpha, d[i], u[i]), -lam, lam);
                }
                edges(uc[0], uc[C - 1], ucleft, ucright);
                float yl[C], acc = 0.f;
                sm.fetch(tid, y, yl);
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    xc[i] = yl[i] + uc[i] - (i > 0 ? uc[i - 1] : ucleft);
                    acc = fmaf(xc[i], xc[i], acc);
                }
                if constexpr (MULTI) {
                    bool ch = false;
#pragma unroll
                    for (int i = 0; i < C; ++i) ch |= (uc[i] != u[i]);
                    row_totals(rw, sm, j, tid, par, acc, ch);
                    changed = ch;
                } else {
                    acc = wave_sum_all<Mp::LANES>(acc);
                }
                fc = 0.5f * acc;
                if (!ok) ok = alpha == 0.f || fc <= fcur - kArmijoSigma * alpha * dec + kArmijoSlackEps * fabsf(fcur);
                if (!wave_any(!ok)) break;
            }
            xcnext0 = rw.next(xc[0]);
            if (MULTI && rw.tw == Rw::TW - 1) xcnext0 = ynext0 + ucright - uc[C - 1];
        }
        steps += active ? 1 : 0;
        if constexpr (!MULTI) {
            // (a step that leaves the dual bit-identical also leaves f so)
            if (wave_any(active && !(fc < fcur))) {
                bool ch = false;
#pragma unroll
                for (int i = 0; i < C; ++i) ch |= (uc[i] != u[i]);
                changed = rw.any(ch);
            }
        }
        if (active && !changed) { active = false; flags = kStalled; }
#pragma unroll
        for (int i = 0; i < C; ++i) { u[i] = uc[i]; x[i] = xc[i]; }
        uleft = ucleft;
        xnext0 = xcnext0;
        if (active) fcur = fc;
        if constexpr (DEBUG) {
            if (rec && t == 0 && active && alpha > 0.f) {
                const int c = (int)rec[0] + 1;
                if (c < kRecMaxF) { rec[kRecF + c] = fc; rec[0] = (float)c; }
            }
        }
    }
    // ---- primal recovery: every sample takes the value of its block, the mean of x = y - D^T u
    //      between two held duals, and constant runs are bit-identical
    float yl[C];
    sm.fetch(tid, y, yl);
    {
        float first = 0.f, s = 0.f, ul = uleft;
        uint32_t at = 0;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const float xi = yl[i] + u[i] - ul;
            ul = u[i];
            const bool begin = i == 0 || ((held >> (i > 0 ? i - 1 : 0)) & 1u);
            first = begin ? xi : first;
            s = begin ? 0.f : s + (xi - first);
            at = begin ? 4u : at + 4u;
            if (i > 0) asm volatile("" : "+v"(at));
            xs[i] = fmaf(s, sm.reciprocal(at), first);
        }
    }
    {
        float v = tail_x;
        const uint32_t lowest = held & (0u - held);            // the first held dual
#pragma unroll
        for (int i = C - 1; i >= 0; --i) {
            if ((held >> i) & 1u) v = ((lowest >> i) & 1u) ? head_x : xs[i];
            xs[i] = v;
        }
    }
    // A row that did not get to a KKT point keeps the plain x = y - D^T u, unless the blocks
    // are where it is: within 2e-5 of the data, but not below four rounding floors of a
    // difference of two x values (the floor follows the row's largest sample, and next to one
    // large sample a converged row's small segments still carry that much noise).  A NaN counts
    // as a deviation, so that a row's output shows the NaN of its input; an infinite sample
    // makes the floor infinite, and such a row keeps its plain output, which shows it.
    if (wave_any(flags != kConverged && valid)) {
        float dv[1] = {0.f};
        float ul = uleft;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const float xi = yl[i] + u[i] - ul;
            ul = u[i];
            if (!(fabsf(xs[i] - xi) <= fmaxf(2e-5f * (1.f + fabsf(yl[i]) + lam), 4.f * gtol))) dv[0] += 1.f;
        }
        row_sum<T, G, COLS, 1>(dv, sm.red, j, tid);
        if (flags != kConverged && ((flags & (kCapped | kPlain)) || dv[0] != 0.f || !(gtol <= 3.0e38f))) {
            ul = uleft;
#pragma unroll
            for (int i = 0; i < C; ++i) {
                xs[i] = yl[i] + u[i] - ul;
                ul = u[i];
            }
            flags |= kPlain;
        }
    }
#pragma unroll
    for (int i = 0; i < C; ++i) u[i] = uc[i];
#undef TV_LK
#undef TV_NV_REFRESH
    return steps | (flags << 16);
}

}  // namespace tvk
