// The 2D operator (paper Alg. 1) and its reverse sweep (Sec. 3.2) for planes of at most 32 x 32,
// all 2K passes of a call in one launch; planes of at most 16 x 16 or 8 x 8 are packed four or
// eight to a wave.  Forward kernel: at the end of this file.
//
// Reverse sweep.
// The backward pass of a 1D prox is segment averaging (paper Eq. 5-6) and moves 12 bytes per
// sample for a few dozen instructions, so the pass-by-pass reverse sweep is bound by memory:
// 2K passes read and write the two adjoint state tensors again and again.  Here a wave keeps the
// state of its planes (two of up to 32 x 32, four of up to 16 x 16, eight of up to 8 x 8) in LDS for the whole sweep: the upstream gradient is read once, grad_y is
// written once, and per pass only the rows' 8-byte segment codes come from memory.  Both views of
// a plane (a row per lane, a column per lane) read the same tile of odd pitch without bank
// conflicts, so no transpose is needed between the row and the column passes.
#pragma once
#include "tv_short.hpp"

namespace tvk {

// ---- bf16 storage of the planes (fp32 everywhere inside): the wave's planes between memory (bf16
//      bit patterns, plane after plane) and an LDS tile of fp32 rows at pitch P.
// FULL planes (S x S, 16-byte aligned block): eight samples per 16-byte access.
template <int S>
__device__ __forceinline__ void planes16_into_tile(const uint16_t *__restrict__ src, int n_here, int lane,
                                                   float *tile, bool stream)
{
    constexpr int P = S + 1;
#pragma unroll
    for (int i = 0; i < S / 8; ++i) {
        const int e = (i * 64 + lane) * 8;                 // sample index inside the wave's block
        float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
        if (e / (S * S) < n_here) q = load16(reinterpret_cast<const float *>(src + e), stream);
        const uint32_t w[4] = {__float_as_uint(q.x), __float_as_uint(q.y), __float_as_uint(q.z), __float_as_uint(q.w)};
        float *d = tile + (e / S) * P + (e % S);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            d[2 * j] = __uint_as_float(w[j] << 16);
            d[2 * j + 1] = __uint_as_float(w[j] & 0xffff0000u);
        }
    }
}
template <int S>
__device__ __forceinline__ void tile_into_planes16(const float *tile, uint16_t *__restrict__ dst, int n_here,
                                                   int lane, bool stream)
{
    constexpr int P = S + 1;
#pragma unroll
    for (int i = 0; i < S / 8; ++i) {
        const int e = (i * 64 + lane) * 8;
        const float *sp = tile + (e / S) * P + (e % S);
        uint32_t w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = f32x2_to_bf16x2(sp[2 * j], sp[2 * j + 1]);
        if (e / (S * S) < n_here)
            store16(reinterpret_cast<float *>(dst + e),
                    make_float4(__uint_as_float(w[0]), __uint_as_float(w[1]), __uint_as_float(w[2]), __uint_as_float(w[3])),
                    stream);
    }
}
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float v) { return (uint16_t)(f32x2_to_bf16x2(v, 0.f) & 0xffffu); }

struct Small2dBwdParams {
    const float *g_up;
    float       *gy;
    const uint2 *codes;        // pass i (row pass of sweep k: 2k, column pass: 2k + 1) at codes + i * code_stride
    size_t       code_stride;  // in uint2
    const float *saved;        // planes of 33-64 samples a side (unless tag says that codes are there): the output of pass i,
    size_t       saved_stride; // at saved + i * saved_stride (floats), is read instead
    float       *partial;      // optional: one dL/dlam term per plane (all passes summed)
    int32_t      planes, H, W, sweeps;
    uint32_t     stream;       // tensors too large to stay in cache: non-temporal accesses
    const uint32_t *tag;       // sides of 33-64, where the workspace may hold row masks (below): 1 if it does; null otherwise
};                             // (IO16 kernels: g_up and gy point to bf16 bit patterns)

// Row masks: what the reverse sweep reads of a pass on planes with both sides of 33-64 samples, 16 bytes a row where its output
// takes 132-256.  Bit k of .x (low) and .y (high): the row jumps behind sample k < n - 1; of .z and .w: it rises
// there.
__device__ __forceinline__ uint64_t mask64(uint32_t lo, uint32_t hi) { return (uint64_t)hi << 32 | lo; }

// Bit k of a row's segment code: x = jump bits, y = direction bits.
template <int K>
__device__ __forceinline__ bool code_jump(const uint2 &c) { return (c.x & (1u << K)) != 0u; }
template <int K>
__device__ __forceinline__ bool code_up(const uint2 &c) { return (c.y & (1u << K)) != 0u; }

// Segment means of g[0 .. n-1] in place, segments given by the code's jump bits; returns the
// row's dL/dlam term  sum over jumps k of sign(x[k+1] - x[k]) (mean_left - mean_right).
// FULL: n = S at compile time.
template <int S, bool FULL, int K = 0>
__device__ __forceinline__ void small2d_means_up(float (&g)[S], const uint2 &code, int n, const float *rtab,
                                                 float &s, int &c4)
{
    if constexpr (K < S) {
        s += g[K];
        c4 += 4;
        const bool last = FULL ? (K == S - 1) : (K >= n - 1);
        bool end = last;
        if constexpr (K + 1 < S) end = end || code_jump<K>(code);
        g[K] = s * *reinterpret_cast<const float *>(reinterpret_cast<const char *>(rtab) + c4);
        if (end) { s = 0.f; c4 = 0; }
        small2d_means_up<S, FULL, K + 1>(g, code, n, rtab, s, c4);
    }
}
template <int S, bool FULL, int K = S - 1>
__device__ __forceinline__ void small2d_means_down(float (&g)[S], const uint2 &code, int n, float &carry,
                                                   float &glam)
{
    if constexpr (K >= 0) {
        const float right = carry;
        const bool last = FULL ? (K == S - 1) : (K >= n - 1);
        bool end = last;
        if constexpr (K + 1 < S) end = end || code_jump<K>(code);
        carry = end ? g[K] : carry;
        g[K] = carry;
        if constexpr (K + 1 < S) {
            if (FULL || K < n - 1) {
                const float d = carry - right;
                glam += code_up<K>(code) ? d : -d;
            }
        }
        small2d_means_down<S, FULL, K - 1>(g, code, n, carry, glam);
    }
}
template <int S, bool FULL>
__device__ __forceinline__ float small2d_segment_means(float (&g)[S], const uint2 &code, int n, const float *rtab)
{
    float s = 0.f, carry = 0.f, glam = 0.f;
    int c4 = 0;
    // the row length in a vector register: as a wave-uniform value every "k is past the end"
    // predicate of the unrolled loops would be kept in scalar registers, 2 S pairs of them
    if (!FULL) asm volatile("" : "+v"(n));
    small2d_means_up<S, FULL>(g, code, n, rtab, s, c4);
    small2d_means_down<S, FULL>(g, code, n, carry, glam);
    return glam;
}
// S = 8, 16 or 32: the side of the square a plane is padded to; a wave holds 64 / S planes,
// one row or column per lane.  FULL: planes of exactly S x S.
// IO16: the upstream gradient and grad_y are bf16 in memory (fp32 in the tiles and in all arithmetic).
template <int S, bool FULL, bool IO16 = false>
__global__ __launch_bounds__(64) void tv2d_bwd_small_kernel(Small2dBwdParams p)
{
    constexpr int P = S + 1;                        // tile pitch
    constexpr int PP = 64 / S;                      // planes per wave
    __shared__ float A[64 * P], B[64 * P], rtab[S + 2];
    const int lane = threadIdx.x;
    for (int i = lane; i <= S; i += 64) rtab[i] = i > 0 ? 1.0f / (float)i : 0.0f;
    const int h = lane / S, idx = lane % S;         // which of the wave's planes; row or column
    const int H = FULL ? S : p.H, W = FULL ? S : p.W, HW = H * W;
    const int64_t plane0 = (int64_t)blockIdx.x * PP;
    const int64_t plane = plane0 + h;
    const bool pvalid = plane < p.planes;
    const int n_here = (int)((p.planes - plane0 < PP) ? (p.planes - plane0) : PP);

    // the upstream gradient of the wave's planes -> A
    if constexpr (IO16) {
        const uint16_t *src = reinterpret_cast<const uint16_t *>(p.g_up) + plane0 * HW;
        if (FULL && ((uintptr_t)src % 16) == 0) {
            planes16_into_tile<S>(src, n_here, lane, A, p.stream != 0);
        } else if (pvalid && idx < W) {
            const uint16_t *col = src + h * HW + idx;
            for (int r = 0; r < H; ++r) A[(h * S + r) * P + idx] = bf16_bits_to_f32(col[r * W]);
        }
    } else {
        const float *src = p.g_up + plane0 * HW;
        if (FULL && ((uintptr_t)src % 16) == 0) {
#pragma unroll
            for (int i = 0; i < S / 4; ++i) {
                const int e = (i * 64 + lane) * 4;              // 0 .. 64 S - 1
                float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
                if (e / (S * S) < n_here) q = load16(src + e, p.stream != 0);
                float *d = A + (e / S) * P + (e % S);
                d[0] = q.x; d[1] = q.y; d[2] = q.z; d[3] = q.w;
            }
        } else {
            // lane (h, idx) moves column idx of its plane: W contiguous floats per memory row
            if (pvalid && idx < W) {
                const float *col = src + h * HW + idx;
                for (int r = 0; r < H; ++r) A[(h * S + r) * P + idx] = col[r * W];
            }
        }
    }
    wave_lds_sync();

    float glam = 0.f;
    float v[S];
    // the segment code of a pass is fetched one pass ahead, so that its latency hides behind
    // the pass before
    const bool cvalid = pvalid && (FULL || idx < W), rvalid = pvalid && (FULL || idx < H);
    auto fetch_code = [&](int pass) -> uint2 {
        if (pass < 0) return make_uint2(0u, 0u);
        const bool col = (pass & 1) != 0;
        if (!(col ? cvalid : rvalid)) return make_uint2(0u, 0u);
        return p.codes[(size_t)pass * p.code_stride + (size_t)plane * (col ? W : H) + idx];
    };
    uint2 code_next = fetch_code(2 * p.sweeps - 1);
    for (int k = p.sweeps - 1; k >= 0; --k) {
        const bool first = (k == p.sweeps - 1);
        // ---- adjoint of the column pass: B <- C^T(A - B) + B  (B = 0 in the first reverse step);
        //      a lane holds column idx of its plane
        {
            const bool valid = cvalid;
            const uint2 code = code_next;
            code_next = fetch_code(2 * k);
            const float *a = A + (h * S) * P + idx;
            float *b = B + (h * S) * P + idx;
            // (tile entries outside H x W, and the tile half of a plane that does not exist, hold
            // garbage that stays where it is: a segment never extends past the row's end)
            if (first) {
#pragma unroll
                for (int r = 0; r < S; ++r) v[r] = a[r * P];
            } else {
#pragma unroll
                for (int r = 0; r < S; ++r) v[r] = a[r * P] - b[r * P];
            }
            const float t = small2d_segment_means<S, FULL>(v, code, H, rtab);
            if (valid) glam += t;
            if (first) {
#pragma unroll
                for (int r = 0; r < S; ++r) b[r * P] = v[r];
            } else {
#pragma unroll
                for (int r = 0; r < S; ++r) b[r * P] += v[r];
            }
        }
        wave_lds_sync();
        // ---- adjoint of the row pass: A <- R^T(B - A) + A  (without A in the first reverse step);
        //      a lane holds row idx of its plane
        {
            const bool valid = rvalid;
            const uint2 code = code_next;
            code_next = fetch_code(2 * k - 1);
            float *a = A + (h * S + idx) * P;
            const float *b = B + (h * S + idx) * P;
            if (first) {
#pragma unroll
                for (int c = 0; c < S; ++c) v[c] = b[c];
            } else {
#pragma unroll
                for (int c = 0; c < S; ++c) v[c] = b[c] - a[c];
            }
            const float t = small2d_segment_means<S, FULL>(v, code, W, rtab);
            if (valid) glam += t;
            if (first) {
#pragma unroll
                for (int c = 0; c < S; ++c) a[c] = v[c];
            } else {
#pragma unroll
                for (int c = 0; c < S; ++c) a[c] += v[c];
            }
        }
        wave_lds_sync();
    }

    // grad_y = A
    if constexpr (IO16) {
        uint16_t *dst = reinterpret_cast<uint16_t *>(p.gy) + plane0 * HW;
        if (FULL && ((uintptr_t)dst % 16) == 0) {
            tile_into_planes16<S>(A, dst, n_here, lane, p.stream != 0);
        } else if (pvalid && idx < W) {
            uint16_t *col = dst + h * HW + idx;
            for (int r = 0; r < H; ++r) col[r * W] = f32_to_bf16_bits(A[(h * S + r) * P + idx]);
        }
    } else {
        float *dst = p.gy + plane0 * HW;
        if (FULL && ((uintptr_t)dst % 16) == 0) {
#pragma unroll
            for (int i = 0; i < S / 4; ++i) {
                const int e = (i * 64 + lane) * 4;
                const float *s = A + (e / S) * P + (e % S);
                if (e / (S * S) < n_here) store16(dst + e, make_float4(s[0], s[1], s[2], s[3]), p.stream != 0);
            }
        } else {
            if (pvalid && idx < W) {
                float *col = dst + h * HW + idx;
                for (int r = 0; r < H; ++r) col[r * W] = A[(h * S + r) * P + idx];
            }
        }
    }
    if (p.partial) {
        // sum over the S lanes of each plane, in a fixed order
        float s = glam;
#pragma unroll
        for (int d = 1; d < S; d <<= 1) s += __shfl_xor(s, d);
        if (pvalid && idx == 0) p.partial[plane] = s;
    }
}

// ---------------------------------------------------------------------------------
// Forward: K sweeps of paper Alg. 1 on planes of at most 16 x 16 in one launch.  (17-32 a side: two lanes
// a row, tv_pair.hpp.)
//
// A wave owns its planes (four or eight, as in the reverse sweep) for the whole call.  A row pass gives each lane a row of its plane, a
// column pass a column; either way the lane solves its 1D problem exactly as the short-row
// kernel does (same RowSolver, row in registers).  Between passes the plane changes hands
// through one LDS tile of odd pitch (side + 1), which both views read and write without bank conflicts.
// The correction terms P (rows) and Q (columns) are only ever touched by the lane that owns
// the row or column, so they live in a lane-private LDS column; one such column suffices,
// because P is consumed (A = Y + P) just before the new Q has to be put away and the other way
// round.  From the second sweep on a pass starts from the dual its correction term encodes
// (P = D^T u of the row pass one sweep earlier, likewise Q).
//
// Memory traffic: y is read once; every pass writes its output (the reverse sweep's tests and
// the caller's workspace contract want them) and one 8-byte segment code per row or column.
// ---------------------------------------------------------------------------------
struct Small2dFwdParams {
    const float *y;
    float       *x;
    float       *saved;        // output of pass i at saved + i * saved_stride (floats)
    size_t       saved_stride;
    uint32_t     keep_passes;  // planes of at most 32 x 32: 0 = write the codes only, not the pass outputs
    uint2       *codes;        // as in Small2dBwdParams (sides of 33-64: null where the pass outputs are kept)
    size_t       code_stride;
    const float *lam;          // plane p uses lam[p % lam_count]
    int64_t      lam_count;
    int32_t      planes, H, W, sweeps;
    uint32_t     stream;
    uint32_t    *tag;          // sides of 33-64: receives whether codes were written
};

// S, FULL: as in the reverse sweep (a wave holds 64 / S planes), S <= 16.
// IO16: y and x are bf16 in memory; the saved pass outputs stay fp32.
// (Planes of 17-64 samples a side: tv_plane2d.hpp and tv_pair.hpp.  A row of 64 samples per lane would take four
// arrays of 64 registers, the whole register file of a SIMD lane, for one wave per SIMD.)
// Waves per SIMD asked of the register allocator: two at least; six for planes of 8 x 8, which fit
// 64-73 registers.  Planes of 16 x 16 take 104 registers, four waves; planes of 9-15 a side 129, one
// too many: the variant DENSE asks for 128 (16 384 planes of 14 x 14, K = 4: 101 -> 78 us), and the
// dispatch takes it wherever a fourth wave has something to do.
// What set these counts: every pass solves inside the loop over passes, and whatever the loop or the
// solver's own loop could leave early kept arrays alive through the half it skips (see
// RowSolver::solve, and below).  Without that, and with predicates that are formed where they are
// used, 16 x 16 (16 384, K = 4) went from 95 to 71 us, 14 x 14 (65 536, K = 2) from 258 to 147.
template <int S, bool FULL, bool IO16 = false, bool DENSE = false>
__global__ __launch_bounds__(64, (S == 8 ? 6 : ((S == 16 && DENSE) ? 4 : 2))) void tv2d_fwd_small_kernel(Small2dFwdParams p)
{
    static_assert(S <= 16, "a row or column per lane: planes of at most 16 x 16");
    constexpr int P = S + 1;
    constexpr int PP = 64 / S;
    __shared__ float T1[64 * P], T2[64 * S], gtab[S + 2], rtab[S + 2];
    const int lane = threadIdx.x;
    fill_tables<S>(gtab, rtab);
    const int h = lane / S, idx = lane % S;
    const int H = FULL ? S : p.H, W = FULL ? S : p.W, HW = H * W;
    const int64_t plane0 = (int64_t)blockIdx.x * PP;
    const int64_t plane = plane0 + h;
    const bool pvalid = plane < p.planes;
    const int n_here = (int)((p.planes - plane0 < PP) ? (p.planes - plane0) : PP);
    float lam = 0.f;
    if (pvalid) lam = fmaxf(p.lam[plane % p.lam_count], 0.f);

    // row idx of the lane's plane: T1 + (h * S + idx) * P, unit step; column idx: T1 + (h * S) * P + idx, step P
    auto opaque = [](int at) { asm volatile("" : "+v"(at)); return at; };
    float *park = T1 + lane;                    // the solver's read-only copy of its input, step 64
    float *mine = T2 + lane;                    // lane-private: the correction term, step 64

    // the wave's planes -> T1 (memory rows at pitch P)
    if constexpr (IO16) {
        const uint16_t *src = reinterpret_cast<const uint16_t *>(p.y) + plane0 * HW;
        if (FULL && ((uintptr_t)src % 16) == 0) {
            planes16_into_tile<S>(src, n_here, lane, T1, p.stream != 0);
        } else if (pvalid && idx < W) {
            const uint16_t *col = src + h * HW + idx;
            for (int r = 0; r < H; ++r) T1[(h * S + r) * P + idx] = bf16_bits_to_f32(col[r * W]);
        }
    } else {
        const float *src = p.y + plane0 * HW;
        if (FULL && ((uintptr_t)src % 16) == 0) {
#pragma unroll
            for (int i = 0; i < S / 4; ++i) {
                const int e = (i * 64 + lane) * 4;
                float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
                if (e / (S * S) < n_here) q = load16(src + e, p.stream != 0);
                float *d = T1 + (e / S) * P + (e % S);
                d[0] = q.x; d[1] = q.y; d[2] = q.z; d[3] = q.w;
            }
        } else {
            // lane (h, idx) moves column idx of its plane: W contiguous floats per memory row
            if (pvalid && idx < W) {
                const float *col = src + h * HW + idx;
                for (int r = 0; r < H; ++r) T1[(h * S + r) * P + idx] = col[r * W];
            }
        }
    }
    wave_lds_sync();

    // a pass's output, T1 -> memory in plane order
    auto put_planes = [&](float *dst) {
        if (FULL && ((uintptr_t)dst % 16) == 0) {
            int own = lane;
            asm volatile("" : "+v"(own));       // (addresses formed here, not kept through the solves)
#pragma unroll
            for (int i = 0; i < S / 4; ++i) {
                const int e = (i * 64 + own) * 4;
                const float *s = T1 + (e / S) * P + (e % S);
                if (e / (S * S) < n_here) store16(dst + e, make_float4(s[0], s[1], s[2], s[3]), p.stream != 0);
            }
        } else {
            if (pvalid && idx < W) {
                float *col = dst + h * HW + idx;
                for (int r = 0; r < H; ++r) col[r * W] = T1[(h * S + r) * P + idx];
            }
        }
    };

    // a row (step 1) or column (step P) of the tile, zero past its n samples.  (Lanes that hold none
    // read what is there: they take no part in the solve.  n through an opaque copy: as loop
    // invariants the S comparisons fill the scalar registers, 215 of which were spilled.)
    auto take = [&](const float *from, int step, int n, float (&t)[S]) {
        int nn = n;
        if (!FULL) asm volatile("" : "+s"(nn));
#pragma unroll
        for (int k = 0; k < S; ++k) {
            t[k] = from[k * step];
            if (!FULL) t[k] = k < nn ? t[k] : 0.f;
        }
    };
    float v[S], u0[S];                          // a pass's input, and the dual it starts from
    bool valid = pvalid && (FULL || idx < H);   // first pass: rows, of W samples
    int n = W;
    take(T1 + opaque((h * S + idx) * P), 1, n, v);
#pragma unroll
    for (int k = 0; k < S; ++k) u0[k] = 0.f;

    const int n_pass = 2 * p.sweeps;
    for (int i = 0; i < n_pass; ++i) {
        const bool col = (i & 1) != 0;
        wave_lds_sync();                        // every lane has taken its input out of T1
#pragma unroll
        for (int k = 0; k < S; ++k) park[k * 64] = v[k];
        wave_lds_sync();

        RowSolver<S, FULL> sv;
        float xs[S];
        sv.yl = park; sv.gtab = gtab; sv.lam = lam; sv.m = n - 1;
        sv.alpha_try = 1.f; sv.steps = 0; sv.flags = 0; sv.nfail = 0;
        sv.active = valid; sv.prev_unclipped = false;
        if (i < 2) sv.start(v, rtab[n]);        // first sweep: no correction term yet
        else {
#pragma unroll
            for (int k = 0; k < S - 1; ++k) sv.u[k] = u0[k];
            sv.start_warm(v);
        }
        sv.solve();
        sv.recover(xs);

        {   // segment code of the row / column (as the short-row kernel builds it)
            uint32_t jm = 0, up = 0;
#pragma unroll
            for (int k = S - 2; k >= 0; --k) {
                const float d = xs[k] - xs[k + 1];
                up = __builtin_amdgcn_alignbit(up, __float_as_uint(d), 31);
                jm = __builtin_amdgcn_alignbit(jm, __float_as_uint(0.0f - fabsf(d)), 31);
            }
            if (!FULL) {
                const uint32_t in = n > 1 ? (0xffffffffu >> (33 - n)) : 0u;
                jm &= in; up &= in;
            }
            if (valid) p.codes[(size_t)i * p.code_stride + (size_t)plane * (col ? W : H) + idx] = make_uint2(jm, up);
        }

        // the pass's new correction term (input - output); needed by the same direction's pass
        // of the next sweep
        const bool keep = i + 2 < n_pass;
        float corr[S];                          // (formed always: conditionally it would tie up v during the solve)
#pragma unroll
        for (int k = 0; k < S; ++k) corr[k] = park[k * 64] - xs[k];
        wave_lds_sync();                        // the parked inputs have been read
        // (each view through its own opaque address: merged, the two would be S selected addresses)
        if (col) {
            float *to = T1 + opaque((h * S) * P + idx);
#pragma unroll
            for (int k = 0; k < S; ++k) to[k * P] = xs[k];
        } else {
            float *to = T1 + opaque((h * S + idx) * P);
#pragma unroll
            for (int k = 0; k < S; ++k) to[k] = xs[k];
        }
        wave_lds_sync();
        // (planes of at most 32 x 32: the reverse sweep reads the codes written above)
        if (p.keep_passes) put_planes(p.saved + (size_t)i * p.saved_stride + plane0 * HW);
        // input of the next pass: this output seen the other way, plus that direction's
        // correction term, whose negated running sum is the dual to start from
        // (formed behind the last pass too: leaving the loop before it would tie up registers for
        // this state during every solve)
        valid = pvalid && (FULL || idx < (col ? H : W));
        n = col ? W : H;
        float t[S];
        if (col) take(T1 + opaque((h * S + idx) * P), 1, n, t);
        else take(T1 + opaque((h * S) * P + idx), P, n, t);
        if (i >= 1) {
            float run = 0.f;
#pragma unroll
            for (int k = 0; k < S; ++k) {
                const float c = mine[k * 64];
                t[k] += c;
                run -= c;
                u0[k] = run;
            }
        } else {
#pragma unroll
            for (int k = 0; k < S; ++k) u0[k] = 0.f;
        }
        if (keep) {
#pragma unroll
            for (int k = 0; k < S; ++k) mine[k * 64] = corr[k];
        }
#pragma unroll
        for (int k = 0; k < S; ++k) v[k] = t[k];
    }
    if constexpr (IO16) {
        uint16_t *dst = reinterpret_cast<uint16_t *>(p.x) + plane0 * HW;
        if (FULL && ((uintptr_t)dst % 16) == 0) {
            tile_into_planes16<S>(T1, dst, n_here, lane, p.stream != 0);
        } else if (pvalid && idx < W) {
            uint16_t *colo = dst + h * HW + idx;
            for (int r = 0; r < H; ++r) colo[r * W] = f32_to_bf16_bits(T1[(h * S + r) * P + idx]);
        }
    } else {
        put_planes(p.x + plane0 * HW);
    }
}

}  // namespace tvk
