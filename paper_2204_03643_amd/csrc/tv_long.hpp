// Kernels for rows longer than 32 samples: T threads share one row, C contiguous samples
// (and duals) per thread, G rows per workgroup; the solver is in tv_rowsolve.hpp.
#pragma once
#include "tv_rowsolve.hpp"

namespace tvk {

// Which group of G rows a workgroup of a strided launch works on.  Workgroups go to the 8 XCDs
// round-robin in launch order, and each XCD has its own L2.  The G adjacent columns of a
// workgroup are 4 G bytes of every image row, a part of a 128-byte line (half of it for G = 16);
// with the identity mapping the other parts belong to the next workgroups, which run on other
// XCDs, so several L2s fetch the whole line (measured with G = 16: twice the algorithmic bytes on
// the read side).  Here the SH = 32 / G workgroups b, b + 8, ..., which the same XCD starts one
// after the other, take the SH neighbouring groups that share a line.
template <int G>
__device__ __forceinline__ uint32_t xcd_grouped(uint32_t b, uint32_t n_groups)
{
    constexpr uint32_t SH = G >= 32 ? 1u : 32u / (uint32_t)G;     // groups per 128-byte line
    if (SH == 1u) return b;
    const uint32_t base = b - b % (8u * SH);
    if (base + 8u * SH > n_groups) return b;        // the ragged end keeps the launch order
    const uint32_t x = b & 7u, s = (b >> 3) % SH;
    return base + SH * x + s;
}

// A thread's C contiguous samples k0 .. k0 + C - 1 of a row (zero past the end) move four at a time where the
// samples lie side by side: a wave then touches every cache line of its 64 * C samples C / 4 times instead of C
// times.  Global memory takes 16-byte accesses at any address that is a multiple of four, which is all that
// the rows of an odd length have; the type says so.  (Word by word, as such rows moved before: 8M samples in rows of 127 / 481 / 3001 / 16 001,
// backward 43 / 37 / 50 / 95 us, now 21 / 23 / 23 / 36; forward 61 / 69 / 106 / 189, now 55 / 66 / 96 / 149.  Rows on
// 16-byte boundaries take the same time as with a type that asks for one.)
template <int C>
__device__ __forceinline__ bool chunk_vec_ok(const void *base, int64_t es)
{
    return C % 4 == 0 && es == 1 && ((uintptr_t)base & 3u) == 0;
}

typedef float tv_long_v4f __attribute__((ext_vector_type(4), aligned(4)));

// Chunk codes: what the reverse sweep of a 2D call reads of a pass on sides of 65-768 samples, a word per
// thread of the pass kernel.  Two bits a sample, sample k0 + i at 2i: x changes after it; x rises there (duals
// past the row's end: anything).  An eighth of the bytes of x and no transpose, and the
// passes then share two output tensors, which stay in the last-level cache, instead of filling 2K.
template <int T, int C>
constexpr bool chunk_coded() { return T <= 64 && C <= 16 && T * C > 64 && T * C <= 768; }

// Rows of 33-64 samples, a thread's samples a part of a row mask (tv_small2d.hpp).
template <int T, int C>
constexpr bool row_masked() { return T * C == 64; }

// The bits of samples k0 .. k0 + C - 1 in a row mask's jumps and rises.
template <int C>
__device__ __forceinline__ void mask_bits(const uint32_t *__restrict__ masks, size_t row, int k0, uint32_t &jump, uint32_t &up)
{
    const uint4 m = *reinterpret_cast<const uint4 *>(masks + row * 4);
    constexpr uint32_t low = (1u << C) - 1u;                // (C divides 32: a chunk lies in one word)
    jump = ((k0 < 32 ? m.x : m.y) >> (k0 & 31)) & low;
    up = ((k0 < 32 ? m.z : m.w) >> (k0 & 31)) & low;
}

// code <- 16 code + 8 (x2 > x1) + 4 (x2 != x1) + 2 (x1 > x0) + (x1 != x0): a comparison a bit and an addition that takes
// it as its carry.  (The comparisons themselves, as where the segments are read off x: the bits of a difference
// call -0 beside +0 a fall, and say nothing next to an infinity.)
// A carry may be read in the third instruction after the comparison that writes it at the earliest, and nothing but
// the order of the block sees to that: the compiler puts no waits inside.  So four comparisons come before the four
// additions, which also spares the two idle slots a bit that it would put between each two of its own.
__device__ __forceinline__ uint32_t shift_in_two(uint32_t code, float x0, float x1, float x2)
{
    uint64_t c0, c1, c2;
    asm("v_cmp_gt_f32 %1, %6, %5\n\t"
        "v_cmp_neq_f32 %2, %6, %5\n\t"
        "v_cmp_gt_f32 %3, %5, %4\n\t"
        "v_cmp_neq_f32 vcc, %5, %4\n\t"
        "v_addc_co_u32 %0, %1, %0, %0, %1\n\t"
        "v_addc_co_u32 %0, %2, %0, %0, %2\n\t"
        "v_addc_co_u32 %0, %3, %0, %0, %3\n\t"
        "v_addc_co_u32 %0, vcc, %0, %0, vcc"
        : "+v"(code), "=&s"(c0), "=&s"(c1), "=&s"(c2) : "v"(x0), "v"(x1), "v"(x2) : "vcc");
    return code;
}

template <int T, int C>
__device__ __forceinline__ uint32_t chunk_code(const float (&xs)[C])
{
    static_assert(C % 2 == 0, "two samples at a time");
    const float xnext0 = __shfl_down(xs[0], 1, T);
    uint32_t code = 0;
#pragma unroll
    for (int i = C - 2; i >= 0; i -= 2) code = shift_in_two(code, xs[i], xs[i + 1], (i + 2 < C) ? xs[i + 2] : xnext0);
    return code;
}

// Every other bit of v, the lowest first.
__device__ __forceinline__ uint32_t even_bits(uint32_t v)
{
    v &= 0x55555555u;
    v = (v | v >> 1) & 0x33333333u;
    v = (v | v >> 2) & 0x0f0f0f0fu;
    v = (v | v >> 4) & 0x00ff00ffu;
    return (v | v >> 8) & 0x0000ffffu;
}

// stream: the tensor is far larger than the last-level cache and touched once per call;
// non-temporal accesses keep such streams from evicting each other.
template <int C>
__device__ __forceinline__ void chunk_load(const float *__restrict__ base, int64_t off, int64_t es,
                                           int k0, int n, bool rvalid, float (&v)[C], bool stream = false)
{
    if (rvalid && chunk_vec_ok<C>(base, es)) {
#pragma unroll
        for (int i = 0; i < C; i += 4) {
            if (k0 + i + 3 < n) {
                tv_long_v4f q;
                if (stream) q = __builtin_nontemporal_load(reinterpret_cast<const tv_long_v4f *>(base + off + k0 + i));
                else q = *reinterpret_cast<const tv_long_v4f *>(base + off + k0 + i);
                v[i] = q.x; v[i + 1] = q.y; v[i + 2] = q.z; v[i + 3] = q.w;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[i + e] = (k0 + i + e < n) ? base[off + k0 + i + e] : 0.f;
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < C; ++i) v[i] = (rvalid && k0 + i < n) ? base[off + (int64_t)(k0 + i) * es] : 0.f;
}

template <int C>
__device__ __forceinline__ void chunk_store(float *__restrict__ base, int64_t off, int64_t es, int k0,
                                            int n, bool rvalid, const float (&v)[C], bool stream = false)
{
    if (!rvalid) return;
    if (chunk_vec_ok<C>(base, es)) {
#pragma unroll
        for (int i = 0; i < C; i += 4) {
            if (k0 + i + 3 < n) {
                tv_long_v4f q;
                q.x = v[i]; q.y = v[i + 1]; q.z = v[i + 2]; q.w = v[i + 3];
                if (stream) __builtin_nontemporal_store(q, reinterpret_cast<tv_long_v4f *>(base + off + k0 + i));
                else *reinterpret_cast<tv_long_v4f *>(base + off + k0 + i) = q;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (k0 + i + e < n) base[off + k0 + i + e] = v[i + e];
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < C; ++i)
        if (k0 + i < n) base[off + (int64_t)(k0 + i) * es] = v[i];
}

// Pitch of the tile through which the transposing kernels turn G strided rows: T chunks of C
// samples with a pad word each (a wave's chunk accesses t * (C + 1) + i then hit 32 different
// banks per half wave with any pitch), rounded up so that consecutive rows start 32 / G banks
// apart: the transposing accesses of half a wave are G rows x 32 / G neighbouring samples, which
// then cover the 32 banks exactly once.  (With an odd pitch, which serves only G = 32, 9 % of
// the LDS cycles of the sixteen-row forward kernels were bank conflicts, 31 % of the backward
// kernels' and 49 % of the eight-row forward kernels'.)
template <int T, int C, int G>
constexpr int xpose_tile_pitch()
{
    constexpr int base = T * (C + 1);
    constexpr int want = G >= 32 ? 1 : 32 / G;
    return base + ((want - base % 32) + 32) % 32;
}

// The backward kernel exchanges two values per thread and scans through LDS only where a row
// spans several waves: a smaller footprint lets more workgroups share a CU.
template <int T, int C, int G, bool COLS>
struct LongSmemBwd {
    using Mp = LongMap<T, G, COLS>;
    static constexpr int TP = T + 2;
    float ex[2][G][TP];
    float buf[COLS ? 2 * 3 * G * T : (T > 64 ? 2 * 3 * G * (T / 64) : 1)];
    float red[2 * 4 * Mp::NW * Mp::RG];
};

// ---------------------------------------------------------------------------------
// Forward: projected Newton on the dual (paper Eq. 3-4), one row per T threads.
// ---------------------------------------------------------------------------------
//
// XPOSE (strided samples, T <= 64): global memory is accessed as in the COLS mapping (adjacent
// lanes <-> adjacent rows, so that the accesses coalesce), but the G rows of the workgroup
// are transposed through an LDS tile on the way in and out, and the solve itself runs in the
// ROWS mapping with one row per wave, i.e. without any workgroup barrier.
// WARM = 1: p.addend is given and the solve starts from the dual it encodes.
// WARM = 3: the cold start picks between two candidates (see there); for long rows that cannot
// take the multilevel start.
// WARM = 2 (unit-stride rows, C a multiple of kMlFactor): rows flagged in p.ml_flag start from
// the dual of the same row averaged in groups of kMlFactor samples (p.coarse_u), which a launch
// on the averaged rows with lambda / kMlFactor left behind (p.dual_out of that launch).
// WARM = 4: that launch, cold, where it forms the averages itself (average_groups); it leaves nothing but the duals.
// DEBUG: the first p.debug_rows rows leave a step record in p.debug (see step_record_floats).

// Waves per SIMD that the forward kernel asks the register allocator for (the second argument
// of __launch_bounds__; 1 = no request).  Left alone, the kernels with 8 samples per thread take
// 77-89 VGPRs and those with 12 take 102-116: a few registers above the step to one more
// resident wave (80 for six, 96 for five).  These kernels wait much of their time (barriers,
// LDS exchanges, the drain of a launch in partly filled rounds), so the extra wave pays although
// the cold-start kernels spill 5-17 registers for it: without the request, 8M samples in rows of
// 520 (64 threads x 12 samples), random walks, 80.8 us instead of 76.9, 144 (16 x 12) 75.4 / 72.4,
// 300 (32 x 12) 74.2 / 71.3, 768 59.5 / 58.0; 12 288 columns of 512 samples 57 -> 52 (three
// 512-thread workgroups per CU, two rounds instead of three).  Not requested for 128 threads x 12
// samples and the transposing kernel with 32 x 12, which ran 2-3 % slower with it.
template <int T, int C, int G, bool COLS, bool XPOSE>
constexpr int fwd_waves_per_simd()
{
    if (T * G == 512 && !COLS) return 4;        // at most 128 VGPRs: a CU holds two such workgroups
    if (XPOSE && C <= 4) return 8;
    if (C == 8 && (T * G <= 256 || (XPOSE && T * G == 512))) return 6;
    if (C == 12 && T * G <= 256 && T != 128 && !(XPOSE && T == 32)) return 5;
    // (64 threads x 16 samples from an addend's dual: 130 VGPRs left alone, 128 and a fourth wave
    // on request; six images of 1024 x 1024, K = 3: 434 -> 418 us)
    if (C == 16 && T * G <= 256) return 4;
    return 1;
}

// The multilevel start's first look at a row (WARM = 4): whether lambda is large enough against the variation of its
// first kMlProbeGroups groups of kMlFactor samples for the start to pay (p.ml_flag), and if so the means of all its groups, the
// thread's chunk of them in y.  Threads read neighbouring groups, 16 bytes each, and the means change
// hands through the room in LDS where the solver parks its input.  Every thread of the workgroup calls; false: the row takes no part.
// (As a kernel of its own, this read the rows and wrote the means for the coarse launch to read.
// Forward, 4096 rows of 16 384: 685 -> 648 us; 2999 of 3001: 96 -> 86; 8M samples in rows of 1001 / 2048 / 4096 / 8001:
// 83 -> 70, 80 -> 74, 92 -> 89, 110 -> 99.)
template <int T, int C, int G>
__device__ __forceinline__ bool average_groups(const FwdParams &p, uint32_t row, int64_t off, bool rvalid,
                                               RowSmem<T, C, G, false> &sm, int j, int t, float (&y)[C])
{
    using Mp = LongMap<T, G, false>;
    static_assert(kMlFactor == 4 && RowSmem<T, C, G, false>::PARK, "groups of 16 bytes; the parked input's room");
    static_assert(Mp::PRIVATE || G == 1, "a row that stays out must not leave others of its workgroup behind");
    constexpr int PROBE = kMlProbeGroups / T < C ? kMlProbeGroups / T : C;      // groups of a thread that are judged
    const int n = p.L.n, n_in = p.fine_n;
    const float *src = p.y + off;
    float *means = reinterpret_cast<float *>(sm.y);
    tv_long_v4f q[C];
    auto load = [&](int i, bool go) {                           // group i T + t, zero past the end of the row
        const int k = (i * T + t) * kMlFactor;
        q[i] = tv_long_v4f{0.f, 0.f, 0.f, 0.f};
        if (go && k + 3 < n_in) q[i] = *reinterpret_cast<const tv_long_v4f *>(src + k);
        else if (go && k < n_in) {
            q[i].x = src[k];
            if (k + 1 < n_in) q[i].y = src[k + 1];
            if (k + 2 < n_in) q[i].z = src[k + 2];
        }
    };
    auto put = [&](int i) {
        const int g = i * T + t, e = g % C;
        const int have = min(n_in - g * kMlFactor, kMlFactor);
        float sum = 0.f;
        sum += q[i].x; sum += q[i].y; sum += q[i].z; sum += q[i].w;
        const float mean = have == kMlFactor ? sum * (1.f / kMlFactor) : sum / (float)max(have, 1);
        means[((e >> 2) * (T * G) + j * T + g / C) * 4 + (e & 3)] = g < n ? mean : 0.f;
    };
#pragma unroll
    for (int i = 0; i < PROBE; ++i) load(i, rvalid);
    float var[1] = {0.f};
#pragma unroll
    for (int i = 0; i < PROBE; ++i) {
        const int k = (i * T + t) * kMlFactor;
        if (k + 1 < n_in) var[0] += fabsf(q[i].y - q[i].x);
        if (k + 2 < n_in) var[0] += fabsf(q[i].z - q[i].y);
        if (k + 3 < n_in) var[0] += fabsf(q[i].w - q[i].z);
        put(i);
    }
    row_sum<T, G, false, 1>(var, sm.red, j, (int)threadIdx.x);
    // differences counted: kMlFactor - 1 of every kMlFactor neighbouring pairs of the probed samples
    const int last = min(kMlProbeGroups * kMlFactor, n_in);
    const float pairs = (float)(last - 1) * (float)(kMlFactor - 1) / (float)kMlFactor;
    const bool flagged = rvalid && load_lambda(p.lam, p.L, row) * pairs >= kMlLambdaRatio * var[0];
    if (rvalid && t == 0) p.ml_flag[(size_t)row * p.flag_pitch] = flagged ? 1u : 0u;
    if (!__any(flagged)) return false;          // (rows that span waves: the same in all of them)
#pragma unroll
    for (int i = PROBE; i < C; ++i) load(i, flagged);
#pragma unroll
    for (int i = PROBE; i < C; ++i) put(i);
    Mp::sync();
    sm.fetch((int)threadIdx.x, y, y);
    return flagged;
}

template <int T, int C, int G, bool COLS, bool XPOSE = false, int WARM = 0, bool DEBUG = false>
__global__ __launch_bounds__(T *G, (fwd_waves_per_simd<T, C, G, COLS, XPOSE>())) void tv1d_fwd_long_kernel(FwdParams p)
{
    static_assert(!XPOSE || (COLS && T <= 64), "the transposing variant is for strided rows inside one wave");
    constexpr bool MCOLS = COLS && !XPOSE;             // mapping used by the solve
    using Mp = LongMap<T, G, MCOLS>;
    __shared__ RowSmem<T, C, G, MCOLS> sm;
    // tile[row][k + k / C]: the pad after every chunk makes a wave's chunk reads conflict-free,
    // the pitch does the same for the transposing accesses (xpose_tile_pitch)
    constexpr int TILE_PITCH = xpose_tile_pitch<T, C, G>();
    __shared__ float tile[XPOSE ? G * TILE_PITCH : 1];
    const int tid = threadIdx.x;
    const int j = Mp::row_of(tid), t = Mp::t_of(tid);

    if constexpr (!DEBUG && !COLS && row_masked<T, C>() && WARM != 1) {
        if (blockIdx.x == 0 && tid == 0 && p.codes_tag) *p.codes_tag = 0u;     // (pass by pass, such sides leave no masks)
    }
    const uint32_t group = COLS ? xcd_grouped<G>(blockIdx.x, gridDim.x) : blockIdx.x;
    const uint32_t row = group * G + j;
    bool rvalid = row < p.L.n_rows;
    bool from_coarse = false;
    if (WARM != 4 && p.ml_flag && rvalid) {
        const bool flagged = p.ml_flag[(size_t)row * p.flag_pitch] != 0;
        if (p.ml_skip) rvalid = flagged;            // a coarse level: only rows that asked for it
        else from_coarse = WARM == 2 && flagged;
    }
    const int n = p.L.n;
    const int k0 = t * C;

    sm.init(tid);
    if (Mp::PRIVATE) __syncthreads();       // the table of reciprocals is the one thing the waves share

    const int64_t off = rvalid ? row_offset(p.L, row) : 0;
    const int64_t es = p.L.elem_stride;
    const float lam = rvalid ? load_lambda(p.lam, p.L, row) * p.lam_scale : 0.f;
    float y[C];
    // transposing variant: thread tid moves samples k = tid / G, tid / G + T, ... of row tid % G
    const int xj = tid % G, xk0 = tid / G;
    const uint32_t xrow = group * G + xj;
    const int64_t xoff = (XPOSE && xrow < p.L.n_rows) ? row_offset(p.L, xrow) : 0;
    // Warm start: the addend is D^T u of an earlier solve of nearly the same rows, so
    // u_k = -(addend_0 + .. + addend_k): u takes the negated running sums inside the chunk, the
    // solver adds the chunks before this one.
    constexpr bool warm = WARM == 1;
    float u[C];
    float wsum = 0.f;                                  // negated sum of the chunk's addend
    if constexpr (WARM == 4) {
        rvalid = average_groups<T, C, G>(p, row, off, rvalid, sm, j, t, y);
        if (!__any(rvalid)) return;
    } else if constexpr (XPOSE) {
        // every global load is issued before the first trip through the tile
        const bool xvalid = xrow < p.L.n_rows;
        float ry[C], ra[C];
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const int k = xk0 + i * T;
            ry[i] = (xvalid && k < n) ? p.y[xoff + (int64_t)k * es] : 0.f;
        }
        if (warm || p.addend) {
#pragma unroll
            for (int i = 0; i < C; ++i) {
                const int k = xk0 + i * T;
                ra[i] = (xvalid && k < n) ? p.addend[xoff + (int64_t)k * es] : 0.f;
            }
            if constexpr (warm) {
                // the addend alone goes through the tile first
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    const int k = xk0 + i * T;
                    tile[xj * TILE_PITCH + k + k / C] = ra[i];
                }
                __syncthreads();
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    wsum -= tile[j * TILE_PITCH + t * (C + 1) + i];
                    u[i] = wsum;
                }
                __syncthreads();
            }
#pragma unroll
            for (int i = 0; i < C; ++i) ry[i] += ra[i];
        }
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const int k = xk0 + i * T;
            tile[xj * TILE_PITCH + k + k / C] = ry[i];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < C; ++i) y[i] = tile[j * TILE_PITCH + t * (C + 1) + i];
    } else {
        chunk_load<C>(p.y, off, es, k0, n, rvalid, y);
        if (warm || p.addend) {
            float ad[C];
            chunk_load<C>(p.addend, off, es, k0, n, rvalid, ad);
#pragma unroll
            for (int i = 0; i < C; ++i) {
                y[i] += ad[i];
                if (warm) { wsum -= ad[i]; u[i] = wsum; }
            }
        }
    }

    float *rec = nullptr;
    if constexpr (DEBUG) {
        if (rvalid && row < p.debug_rows) rec = p.debug + (size_t)row * step_record_floats(n);
    }
    const float *cu = from_coarse ? p.coarse_u + (size_t)row * p.coarse_pitch : nullptr;
    // Polished trial points pay where the solve starts cold and has five or six steps to go (6M samples,
    // rows of 64 / 256 / 512 with lambda = 2 on unit noise: 46 / 47 / 45 -> 40 / 41 / 42 us; columns of
    // 256 / 512, lambda = 0.1 on images: 42 / 42 -> 38 / 40), not where it starts from a good dual
    // (workload 4, K = 10, warm passes with them: 700 -> 740 us; rows of 900 from the coarse level:
    // 120 -> 123).  Rows that span waves would need one more exchange through a barrier for them.
    constexpr bool POLISH = Mp::PRIVATE && (WARM == 0 || WARM == 3 || WARM == 4);
    constexpr bool DUAL = !COLS && (WARM == 0 || WARM == 2 || WARM == 4);
    float xs[C];
    const int info = row_solve<T, C, G, MCOLS, WARM == 4 ? 0 : WARM, POLISH, DEBUG, DUAL>(y, u, wsum, lam, n, j, t, rvalid, sm, cu,
                                                                   p.coarse_n, rec, xs);

    // (rows of at most 32 samples, small batches: the segment code comes from the registers; a kernel
    // that read it off x again, a thread per row, took 6.8 of the 21 us of 8192 x 32 forward + backward)
    if constexpr (T * C <= 32) {
        if (p.seg) {
            const uint2 code = row_segment_code<T, C>(xs, n, t);
            if (rvalid && t == 0) p.seg[row] = code;
        }
    }
    if (DUAL && (WARM == 4 || p.dual_out)) chunk_store<C>(p.dual_out, (int64_t)row * p.dual_pitch, 1, k0, n, rvalid, u);
    if constexpr (WARM == 4) return;

    if constexpr (XPOSE) {
        // a wave writes only its own row of the tile; the barrier then hands the tile over
#pragma unroll
        for (int i = 0; i < C; ++i) tile[j * TILE_PITCH + t * (C + 1) + i] = xs[i];
        __syncthreads();
        for (int k = xk0; k < T * C; k += T)
            if (xrow < p.L.n_rows && k < n) {
                const float v = tile[xj * TILE_PITCH + k + k / C];
                p.x[xoff + (int64_t)k * es] = v;
                if (p.x2) p.x2[xoff + (int64_t)k * es] = v;
            }
        if (p.resid) {
            float yl[C];
            sm.fetch(tid, y, yl);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < C; ++i) tile[j * TILE_PITCH + t * (C + 1) + i] = yl[i] - xs[i];
            __syncthreads();
            for (int k = xk0; k < T * C; k += T)
                if (xrow < p.L.n_rows && k < n)
                    p.resid[xoff + (int64_t)k * es] = tile[xj * TILE_PITCH + k + k / C];
        }
    } else {
        if (p.x) chunk_store<C>(p.x, off, es, k0, n, rvalid, xs);
        if (p.x2) chunk_store<C>(p.x2, off, es, k0, n, rvalid, xs);
        if (p.resid) {
            float yl[C];
            sm.fetch(tid, y, yl);
#pragma unroll
            for (int i = 0; i < C; ++i) yl[i] -= xs[i];
            chunk_store<C>(p.resid, off, es, k0, n, rvalid, yl);
        }
    }
    // (last, behind the stores that the wave waits for at its end anyway)
    if constexpr (!DEBUG && chunk_coded<T, C>() && WARM <= 2) {
        if (p.chunk_codes) {
            const uint32_t code = chunk_code<T, C>(xs);
            if (rvalid) p.chunk_codes[(size_t)row * T + t] = code;
        }
        if (p.codes_tag && blockIdx.x == 0 && tid == 0) *p.codes_tag = p.chunk_codes ? 1u : 0u;
    }
    if (p.info && rvalid && t == 0) p.info[row] = info;
    if constexpr (DEBUG) {
        if (rec && t == 0) rec[2] = (float)info;
    }
}

// ---------------------------------------------------------------------------------
// Backward (paper Eq. 5-6 as segment averaging), one row per T threads.
// ---------------------------------------------------------------------------------
// Unit-stride rows, and strided ones of more than 1024 samples (shorter ones: tv_cols.hpp).
// HAS_SUB: p.sub is given (the reverse sweep of the 2D operator).
// Workgroups of 1024 threads ask for 8 waves per SIMD (at most 64 VGPRs), so that a CU holds two of
// them and one's loads overlap the other's scans.
// CODES: where the forward pass left chunk codes (p.codes_tag says whether it did) they are read, not x.
template <int T, int C, int G, bool COLS, bool HAS_SUB = false, bool CODES = false>
__global__ __launch_bounds__(T *G, (T * G == 1024 && !COLS && !HAS_SUB) ? 8 : 1) void tv1d_bwd_long_kernel(BwdParams p)
{
    static_assert(!CODES || chunk_coded<T, C>() || row_masked<T, C>(), "chunk codes are for rows inside one wave");
    using Mp = LongMap<T, G, COLS>;
    __shared__ LongSmemBwd<T, C, G, COLS> sm;
    const int tid = threadIdx.x;
    const int j = Mp::row_of(tid), t = Mp::t_of(tid);
#define TV_EX(q, tt) sm.ex[q][j][(tt) + 1]
    const uint32_t group = COLS ? xcd_grouped<G>(blockIdx.x, gridDim.x) : blockIdx.x;
    const uint32_t row = group * G + j;
    const bool rvalid = row < p.L.n_rows;
    const int n = p.L.n;
    const int k0 = t * C;
    if (t == 0) {
#pragma unroll
        for (int q = 0; q < 2; ++q) { sm.ex[q][j][0] = 0.f; sm.ex[q][j][T + 1] = 0.f; }
    }
    const int64_t off = rvalid ? row_offset(p.L, row) : 0;
    const int64_t es = p.L.elem_stride;

    // g becomes the averaged quantity, then the segment means, then the output; of x only two
    // bits per sample are kept (is there a jump behind it, and does x rise there)
    float g[C], sb[HAS_SUB ? C : 1];
    uint32_t jmask = 0, upmask = 0;
    // duals of this chunk that lie inside the row (dual i sits behind sample k0 + i)
    const int nv = min(max(n - 1 - k0, 0), C);
    const uint32_t inrow = (1u << nv) - 1u;
    bool coded = false;
    if constexpr (CODES) coded = *p.codes_tag == 1u;
    if (CODES && coded) {
        const uint32_t code = !row_masked<T, C>() && rvalid ? p.chunk_codes[(size_t)row * T + t] : 0u;
        chunk_load<C>(p.g, off, es, k0, n, rvalid, g, p.L.stream);
        if constexpr (HAS_SUB) chunk_load<C>(p.sub, off, es, k0, n, rvalid, sb, p.L.stream);
        if constexpr (row_masked<T, C>()) {
            if (rvalid) mask_bits<C>(p.chunk_codes, row, k0, jmask, upmask);
        } else {
            jmask = even_bits(code);
            upmask = even_bits(code >> 1);
        }
    } else {
        float x[C];
        chunk_load<C>(p.x, off, es, k0, n, rvalid, x, p.L.stream);
        chunk_load<C>(p.g, off, es, k0, n, rvalid, g, p.L.stream);
        if constexpr (HAS_SUB) chunk_load<C>(p.sub, off, es, k0, n, rvalid, sb, p.L.stream);
        TV_EX(0, t) = x[0];
        Mp::sync();
        const float xnext0 = TV_EX(0, t + 1);
        // jump after sample i (always at the end of the row; samples past the end are their
        // own segments and contribute nothing)
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const float xn = (i + 1 < C) ? x[i + 1] : xnext0;
            if (xn != x[i]) jmask |= 1u << i;
            if (xn > x[i]) upmask |= 1u << i;
        }
    }
    const uint32_t gmask = jmask & inrow;      // jumps that count for dL/dlam
    jmask |= ~inrow;
    if constexpr (HAS_SUB) {
#pragma unroll
        for (int i = 0; i < C; ++i) g[i] -= sb[i];
    }
#define TV_JUMP(i) ((jmask >> (i)) & 1u)
    // chunk-local pieces: head = samples up to and including the first jump, tail = samples
    // after the last jump; both are the whole chunk when it holds no jump
    bool any = false;
    float head_s = 0.f, head_n = 0.f, tail_s = 0.f, tail_n = 0.f;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        if (!any) { head_s += g[i]; head_n += 1.f; }
        tail_s += g[i]; tail_n += 1.f;
        if (TV_JUMP(i)) { any = true; tail_s = 0.f; tail_n = 0.f; }
    }
    float ls, ln, rs, rn;
    seg_scan<T, G, COLS, +1, true>(any, tail_s, tail_n, sm.buf, j, t, ls, ln);   // open part on the left
    seg_scan<T, G, COLS, -1, true>(any, head_s, head_n, sm.buf, j, t, rs, rn);   // open part on the right

    // per-sample means: forward pass accumulates, backward pass broadcasts
    float (&mean)[C] = g;
    {
        float s = ls, c = ln;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            s += g[i]; c += 1.f;
            mean[i] = 0.f;
            if (TV_JUMP(i)) { mean[i] = s * __builtin_amdgcn_rcpf(c); s = 0.f; c = 0.f; }
        }
        // trailing open part continues into the next chunks
        const float open_mean = (c > 0.f) ? (s + rs) * __builtin_amdgcn_rcpf(c + rn) : 0.f;
        float carry = open_mean;
#pragma unroll
        for (int i = C - 1; i >= 0; --i) {
            if (TV_JUMP(i)) carry = mean[i];
            mean[i] = carry;
        }
    }
    // a head piece that is closed inside this chunk still needs nothing from the right; a
    // head piece open to the left got (ls, ln) above.  dL/dlam needs the next chunk's first mean.
    TV_EX(1, t) = mean[0];
    Mp::sync();
    const float mnext0 = TV_EX(1, t + 1);
    float gl[1] = {0.f};
#pragma unroll
    for (int i = 0; i < C; ++i) {
        if ((gmask >> i) & 1u) {
            const float mn = (i + 1 < C) ? mean[i + 1] : mnext0;
            const float sg = ((upmask >> i) & 1u) ? 1.f : -1.f;
            gl[0] = fmaf(sg, mean[i] - mn, gl[0]);
        }
    }
    if constexpr (HAS_SUB) {
#pragma unroll
        for (int i = 0; i < C; ++i) mean[i] += sb[i];
    }
    chunk_store<C>(p.gy, off, es, k0, n, rvalid, mean, p.L.stream);
    if (p.partial) {
        row_sum<T, G, COLS, 1>(gl, sm.red, j, tid);
        if (rvalid && t == 0) p.partial[row] = gl[0];
    }
#undef TV_EX
#undef TV_JUMP
}

// ---------------------------------------------------------------------------------
// Launchers: pick threads-per-row T and samples-per-thread C from the row length.
// ---------------------------------------------------------------------------------
template <int T, int C, int G, bool COLS>
inline hipError_t launch_fwd_long_t(const FwdParams &p, hipStream_t s)
{
    const dim3 grid((p.L.n_rows + G - 1) / G), block(T * G);
    constexpr bool XP = COLS && T <= 64;
    if (p.warm == 2) {
        if constexpr (!COLS && C % kMlFactor == 0)
            hipLaunchKernelGGL((tv1d_fwd_long_kernel<T, C, G, COLS, XP, 2>), grid, block, 0, s, p);
        else
            return hipErrorInvalidValue;
    } else if (p.warm == 3 && T * C > 768) {
        // (cold, with the constant row's dual as a second candidate: rows of 769 samples and more)
        if constexpr (T * C > 768)
            hipLaunchKernelGGL((tv1d_fwd_long_kernel<T, C, G, COLS, XP, 3>), grid, block, 0, s, p);
    } else if (p.warm == 1)
        hipLaunchKernelGGL((tv1d_fwd_long_kernel<T, C, G, COLS, XP, 1>), grid, block, 0, s, p);
    else
        hipLaunchKernelGGL((tv1d_fwd_long_kernel<T, C, G, COLS, XP, 0>), grid, block, 0, s, p);
    return hipGetLastError();
}

template <int T, int C, int G, bool COLS>
inline hipError_t launch_bwd_long_t(const BwdParams &p, hipStream_t s)
{
    const dim3 grid((p.L.n_rows + G - 1) / G), block(T * G);
    if constexpr (chunk_coded<T, C>() || row_masked<T, C>()) {
        if (p.chunk_codes) {
            if (p.sub)
                hipLaunchKernelGGL((tv1d_bwd_long_kernel<T, C, G, COLS, true, true>), grid, block, 0, s, p);
            else
                hipLaunchKernelGGL((tv1d_bwd_long_kernel<T, C, G, COLS, false, true>), grid, block, 0, s, p);
            return hipGetLastError();
        }
    }
    if (p.sub)
        hipLaunchKernelGGL((tv1d_bwd_long_kernel<T, C, G, COLS, true>), grid, block, 0, s, p);
    else
        hipLaunchKernelGGL((tv1d_bwd_long_kernel<T, C, G, COLS, false>), grid, block, 0, s, p);
    return hipGetLastError();
}

// Threads of the mappings below per row of 65-768 samples (the same for rows and columns, and for the
// elimination kernels of tv_long_tri.hpp): the words a row's chunk codes take.
inline int chunk_threads(int64_t n)
{
    return n <= 96 ? 8 : n <= 192 ? 16 : n <= 384 ? 32 : 64;
}

// Unit-stride rows of more than 32 samples.
#define TV_LONG_ROWS(FN, n, p, s)                                                         \
    do {                                                                                  \
        if (n <= 64) return FN<8, 8, 32, false>(p, s);                                    \
        if (n <= 96) return FN<8, 12, 32, false>(p, s);                                   \
        if (n <= 128) return FN<16, 8, 16, false>(p, s);                                  \
        if (n <= 192) return FN<16, 12, 16, false>(p, s);                                 \
        if (n <= 256) return FN<32, 8, 8, false>(p, s);                                   \
        if (n <= 384) return FN<32, 12, 8, false>(p, s);                                  \
        if (n <= 512) return FN<64, 8, 4, false>(p, s);                                   \
        if (n <= 768) return FN<64, 12, 4, false>(p, s);                                  \
        if (n <= 1024) return FN<64, 16, 4, false>(p, s);                                 \
        if (n <= 1536) return FN<128, 12, 1, false>(p, s);                                \
        if (n <= 2048) return FN<256, 8, 1, false>(p, s);                                 \
        if (n <= 3072) return FN<256, 12, 1, false>(p, s);                                \
        if (n <= 4096) return FN<256, 16, 1, false>(p, s);                                \
        if (n <= 6144) return FN<512, 12, 1, false>(p, s);                                \
        if (n <= 8192) return FN<512, 16, 1, false>(p, s);                                \
        if (n <= 12288) return FN<1024, 12, 1, false>(p, s);                              \
        return FN<1024, 16, 1, false>(p, s);                                              \
    } while (0)

// Strided rows of more than 1024 samples.
#define TV_LONG_COLS(FN, n, p, s)                                                         \
    do {                                                                                  \
        if (n <= 1536) return FN<128, 12, 8, true>(p, s);                                 \
        if (n <= 2048) return FN<128, 16, 8, true>(p, s);                                 \
        if (n <= 3072) return FN<256, 12, 4, true>(p, s);                                 \
        if (n <= 4096) return FN<256, 16, 4, true>(p, s);                                 \
        if (n <= 8192) return FN<1024, 8, 1, true>(p, s);                                 \
        if (n <= 12288) return FN<1024, 12, 1, true>(p, s);                               \
        return FN<1024, 16, 1, true>(p, s);                                               \
    } while (0)

inline hipError_t launch_fwd_long(const FwdParams &p, hipStream_t s)
{
    const int n = p.L.n;
    const bool wide = (int64_t)p.L.n_rows <= tvd::get(tvd::kThreadPerSampleWideRows);
    if (p.L.elem_stride == 1) {
        if (n <= 32) return wide ? launch_fwd_long_t<16, 2, 16, false>(p, s) : launch_fwd_long_t<8, 4, 32, false>(p, s);
        TV_LONG_ROWS(launch_fwd_long_t, n, p, s);
    }
    // through an LDS tile up to 1024 samples.  Rows a workgroup, of 193-768 samples: 8.  A
    // workgroup of 512 threads (at most 128 registers each) leaves room for a second one on the CU,
    // whose loads and transposes then overlap the first one's solve (with 16 rows, 1024 threads, a CU
    // holds one workgroup and every phase waits for the slowest wave; 24 images of 512 x 512: column
    // pass 61 -> 57 us, K = 4 forward 313 -> 295; 12 of 768 x 768: 48 -> 42, 372 -> 344; columns of
    // 769-1024 samples need 139 registers that way and are slower, 44 -> 48).
    if (n <= 32) return wide ? launch_fwd_long_t<16, 2, 16, true>(p, s) : launch_fwd_long_t<8, 4, 16, true>(p, s);
    if (n <= 64) return launch_fwd_long_t<8, 8, 16, true>(p, s);
    if (n <= 96) return launch_fwd_long_t<8, 12, 16, true>(p, s);
    if (n <= 128) return launch_fwd_long_t<16, 8, 16, true>(p, s);
    if (n <= 192) return launch_fwd_long_t<16, 12, 16, true>(p, s);
    if (n <= 256) return launch_fwd_long_t<32, 8, 8, true>(p, s);
    if (n <= 384) return launch_fwd_long_t<32, 12, 8, true>(p, s);
    if (n <= 512) return launch_fwd_long_t<64, 8, 8, true>(p, s);
    if (n <= 768) return launch_fwd_long_t<64, 12, 8, true>(p, s);
    if (n <= 1024) return launch_fwd_long_t<64, 16, 16, true>(p, s);
    TV_LONG_COLS(launch_fwd_long_t, n, p, s);
}

// The coarse level that forms its averages itself, for the lengths that ml_min_length's default leaves it
// (193 groups and more), in the mappings of TV_LONG_ROWS.
inline bool averages_itself(int64_t groups) { return groups > 192 && groups <= 4096; }

template <int T, int C, int G>
inline hipError_t launch_fwd_averaged_t(const FwdParams &p, hipStream_t s)
{
    hipLaunchKernelGGL((tv1d_fwd_long_kernel<T, C, G, false, false, 4>), dim3((p.L.n_rows + G - 1) / G), dim3(T * G), 0, s, p);
    return hipGetLastError();
}

inline hipError_t launch_fwd_averaged(const FwdParams &p, hipStream_t s)
{
    const int n = p.L.n;
    if (n <= 256) return launch_fwd_averaged_t<32, 8, 8>(p, s);
    if (n <= 384) return launch_fwd_averaged_t<32, 12, 8>(p, s);
    if (n <= 512) return launch_fwd_averaged_t<64, 8, 4>(p, s);
    if (n <= 768) return launch_fwd_averaged_t<64, 12, 4>(p, s);
    if (n <= 1024) return launch_fwd_averaged_t<64, 16, 4>(p, s);
    if (n <= 1536) return launch_fwd_averaged_t<128, 12, 1>(p, s);
    if (n <= 2048) return launch_fwd_averaged_t<256, 8, 1>(p, s);
    if (n <= 3072) return launch_fwd_averaged_t<256, 12, 1>(p, s);
    return launch_fwd_averaged_t<256, 16, 1>(p, s);
}

// Small batches of unit-stride rows of 65-256 samples (wave_per_row_rows in tv_dispatch.hpp): four samples per
// thread instead of eight or twelve, cold start.  A lone wave per SIMD is bound by its chains, which follow
// the samples per thread.
inline hipError_t launch_fwd_long_few(const FwdParams &p, hipStream_t s)
{
    if (p.L.n <= 128)
        hipLaunchKernelGGL((tv1d_fwd_long_kernel<32, 4, 2, false, false, 0>), dim3((p.L.n_rows + 1) / 2), dim3(64), 0, s, p);
    else
        hipLaunchKernelGGL((tv1d_fwd_long_kernel<64, 4, 1, false, false, 0>), dim3(p.L.n_rows), dim3(64), 0, s, p);
    return hipGetLastError();
}

// The forward launch with step records (cold start, unit-stride rows): one mapping of each kind
// -- rows inside a wave (wave-level fences, scans inside the wave), and a workgroup per
// row with 256 and with 1024 threads (workgroup barriers, the waves' totals through LDS).
inline hipError_t launch_fwd_long_debug(const FwdParams &p, hipStream_t s)
{
    const int n = p.L.n;
    if (n <= 512)
        hipLaunchKernelGGL((tv1d_fwd_long_kernel<64, 8, 4, false, false, 0, true>), dim3((p.L.n_rows + 3) / 4),
                           dim3(256), 0, s, p);
    else if (n <= 4096)
        hipLaunchKernelGGL((tv1d_fwd_long_kernel<256, 16, 1, false, false, 0, true>), dim3(p.L.n_rows), dim3(256), 0,
                           s, p);
    else
        hipLaunchKernelGGL((tv1d_fwd_long_kernel<1024, 16, 1, false, false, 0, true>), dim3(p.L.n_rows), dim3(1024),
                           0, s, p);
    return hipGetLastError();
}

inline hipError_t launch_bwd_long(const BwdParams &p, hipStream_t s)
{
    const int n = p.L.n;
    if (p.L.elem_stride == 1) TV_LONG_ROWS(launch_bwd_long_t, n, p, s);
    TV_LONG_COLS(launch_bwd_long_t, n, p, s);
}

}  // namespace tvk
