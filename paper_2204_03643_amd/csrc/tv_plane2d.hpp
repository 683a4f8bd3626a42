// The 2D operator (paper Alg. 1) and its reverse sweep (Sec. 3.2) for small batches of planes of
// at most 64 x 64: one plane per workgroup, resident in LDS for all 2K passes of a call, each row
// (or column) of a pass handled by T neighbouring lanes with C samples each.  Forward kernel
// first, reverse sweep at the end of the file.
//
// With a few hundred planes the row-per-lane kernels of tv_small2d.hpp fill a fraction of the
// chip with long dependent chains (one wave per one or two planes), and the pass-by-pass route
// pays a launch and a trip through memory per pass for a few microseconds of arithmetic.  Here a
// workgroup of 512 threads holds the plane; the row and the column view read the same tile of
// odd pitch, a thread touches the same tile elements going in and coming out of a pass, so one
// barrier per pass is all the synchronisation there is, and the correction terms of paper Alg. 1
// (P for the rows, Q for the columns) never leave the registers of the threads that own them.
//
// The solve is tv_rowsolve.hpp's with rows inside one 16-lane DPP row: every exchange between the
// threads of a row is a row shift, a butterfly or a permutation inside the wave, and nothing but
// the table of reciprocals and, with 8 samples a thread, its own parked input is read from LDS
// during a solve.
#pragma once
#include "tv_long.hpp"
#include "tv_small2d.hpp"

namespace tvk {

// T threads per row, C samples per thread: planes of at most S x S, S = T * C (16 x 2: up to
// 32 x 32, with segment codes for the reverse sweep; 8 x 8: up to 64 x 64, with row masks where both sides are
// longer than 32 and the passes are not asked for, pass outputs otherwise).  With masks, 256 planes of
// 64 x 64, K = 4: forward 73 -> 68 us, reverse sweep 33 -> 19.  One plane per workgroup of S * T = 512 threads.
// (32 x 32 with 8 threads x 4 samples, 256 threads: 256 planes, K = 4, 52 us against 38 with
// 16 x 2, whose chains are shorter; from 1500 planes on 8 x 4 is 5-10 % ahead, where the
// row-per-lane kernels take over anyway.)
// IO16: y and x are bf16 in memory (fp32 in the tile and in all arithmetic; the saved pass outputs
// stay fp32).
// MASKS: row masks are written, not pass outputs (S > 32), and p.tag says so.  (Of its own: with both in one kernel 300 planes of
// 32 x 40, K = 1, took 24.8 us against 23.4 before there were masks, now 22.9; of 33 x 40 26.1 against 24.7, now 24.2.)
template <int T, int C, bool IO16 = false, bool MASKS = false>
__global__ __launch_bounds__(T * T * C, C <= 4 ? 8 : 4) void tv2d_fwd_plane_kernel(Small2dFwdParams p)
{
    constexpr int S = T * C, P = S + 1, NT = S * T;
    static_assert(NT % 64 == 0 && NT <= 1024, "whole waves");
    __shared__ float X[S * P];
    __shared__ RowSmem<T, C, S, false> sm;
    const int tid = threadIdx.x;
    const int j = tid / T, t = tid % T, k0 = t * C;
    const int H = p.H, W = p.W, HW = H * W;
    const int64_t plane = blockIdx.x;
    if (MASKS && blockIdx.x == 0 && tid == 0) *p.tag = 1u;         // (here, not at the end, where its address is waited for)
    sm.init(tid);
    const float lam = fmaxf(p.lam[plane % p.lam_count], 0.f);
    if constexpr (IO16) {
        const uint16_t *src = reinterpret_cast<const uint16_t *>(p.y) + plane * HW;
        for (int e = tid; e < HW; e += NT) X[(e / W) * P + e % W] = bf16_bits_to_f32(src[e]);
    } else {
        const float *src = p.y + plane * HW;
        for (int e = tid; e < HW; e += NT) X[(e / W) * P + e % W] = src[e];
    }
    __syncthreads();
    auto put_plane = [&](float *dst) {
        for (int e = tid; e < HW; e += NT) dst[e] = X[(e / W) * P + e % W];
    };

    // the correction terms of the thread's row chunk and of its column chunk (paper Alg. 1)
    float corr_r[C], corr_c[C];
    const int n_pass = 2 * p.sweeps;
    for (int i = 0; i < n_pass; ++i) {
        const bool col = (i & 1) != 0;
        const int n = col ? H : W, rows = col ? W : H;
        const bool valid = j < rows;
        // sample k of the thread's row: X[j][k] in a row pass, X[k][j] in a column pass
        const int base = col ? j : j * P, step = col ? P : 1;
        float y[C], u[C], xs[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            y[c] = (valid && k0 + c < n) ? X[base + (k0 + c) * step] : 0.f;
            u[c] = 0.f;
        }
        int info;
        if (i < 2) {
            info = row_solve<T, C, S, false, 0, true, false, false>(y, u, 0.f, lam, n, j, t, valid, sm, nullptr, 0, nullptr, xs);
        } else {
            // input = the other direction's output plus this direction's correction term, which
            // is D^T u of this direction's pass one sweep earlier: start from that dual
            float wsum = 0.f;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float cr = col ? corr_c[c] : corr_r[c];
                y[c] += cr;
                wsum -= cr;
                u[c] = wsum;
            }
            info = row_solve<T, C, S, false, 1, true, false, false>(y, u, wsum, lam, n, j, t, valid, sm, nullptr, 0, nullptr, xs);
        }
        (void)info;
        if (i + 2 < n_pass) {
            float yl[C];
            sm.fetch(tid, y, yl);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                if (col) corr_c[c] = yl[c] - xs[c];
                else corr_r[c] = yl[c] - xs[c];
            }
        }
#pragma unroll
        for (int c = 0; c < C; ++c)
            if (valid && k0 + c < n) X[base + (k0 + c) * step] = xs[c];

        if constexpr (S <= 32) {
            const uint2 code = row_segment_code<T, C>(xs, n, t);
            if (valid && t == 0)
                p.codes[(size_t)i * p.code_stride + (size_t)plane * rows + j] = code;
        } else if constexpr (MASKS) {
            // row masks, a byte of eight samples a thread
            static_assert(S <= 32 || C == 8, "");
            const float xnext0 = from_right<T, 1>(xs[0], t);
            uint32_t jm = 0, up = 0;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float xn = (c + 1 < C) ? xs[c + 1] : xnext0;
                if (k0 + c < n - 1) {
                    if (xn != xs[c]) jm |= 1u << c;
                    if (xn > xs[c]) up |= 1u << c;
                }
            }
            if (valid) {
                uint8_t *to = reinterpret_cast<uint8_t *>(p.codes + (size_t)i * p.code_stride + ((size_t)plane * rows + j) * 2);
                to[t] = (uint8_t)jm;
                to[8 + t] = (uint8_t)up;
            }
        }
        __syncthreads();
        // (planes of at most 32 x 32: the reverse sweep reads the codes written above)
        if (S > 32 ? !MASKS : p.keep_passes != 0u) {
            put_plane(p.saved + (size_t)i * p.saved_stride + plane * HW);
            if (i + 1 < n_pass) __syncthreads();      // the next pass writes into the tile
        }
    }
    if constexpr (IO16) {
        uint16_t *dst = reinterpret_cast<uint16_t *>(p.x) + plane * HW;
        for (int e = tid; e < HW; e += NT) dst[e] = f32_to_bf16_bits(X[(e / W) * P + e % W]);
    } else {
        put_plane(p.x + plane * HW);
    }
}

// ---------------------------------------------------------------------------------
// Reverse sweep through paper Alg. 1 (Sec. 3.2) for small batches: one plane per workgroup, the
// two adjoint state tensors resident in LDS for all 2K passes, T threads x C samples per row.
// ---------------------------------------------------------------------------------

// Segmented exclusive sums over the T threads of a row, from thread 0 upwards (DIR = +1) or from
// thread T - 1 downwards (DIR = -1), by row shifts: each thread contributes (closed, s, n) as in
// seg_scan of tv_rowsolve.hpp (closed: its chunk holds a segment boundary; (s, n): sum and count of
// the part of its chunk beyond the last boundary in scan direction) and gets the sum and count
// of the open part that arrives at it (zero at the origin).
template <int T, int DIR>
__device__ __forceinline__ void row_open_part_before(bool closed, float s, float n, int t, float &cs, float &cn)
{
    float f = closed ? 1.f : 0.f;
#define TV_STEP(D)                                                                                  \
    if constexpr ((D) < T) {                                                                        \
        constexpr int DD = (D) < T ? (D) : 1;                                                       \
        const float of = DIR > 0 ? from_left<T, DD>(f, t) : from_right<T, DD>(f, t);                \
        const float os = DIR > 0 ? from_left<T, DD>(s, t) : from_right<T, DD>(s, t);                \
        const float on = DIR > 0 ? from_left<T, DD>(n, t) : from_right<T, DD>(n, t);                \
        const bool has = DIR > 0 ? (t >= (D)) : (t + (D) < T);                                      \
        if (has && f == 0.f) { s += os; n += on; f = of; }                                          \
    }
    TV_STEP(1) TV_STEP(2) TV_STEP(4) TV_STEP(8)
#undef TV_STEP
    cs = DIR > 0 ? from_left<T, 1>(s, t) : from_right<T, 1>(s, t);
    cn = DIR > 0 ? from_left<T, 1>(n, t) : from_right<T, 1>(n, t);
}

// Segment means of one row held by T threads (paper Eq. 5-6 as segment averaging): g is the
// thread's chunk of the averaged quantity on entry (zero past the end of the row) and of the
// means on return.  Bit i of jm: the row's output jumps behind sample k0 + i; of up: it rises
// there (only duals inside the row are looked at).  Returns the thread's part of the row's
// dL/dlam term  sum over jumps of sign(x[k+1] - x[k]) (mean_left - mean_right).
template <int T, int C>
__device__ __forceinline__ float lanes_segment_means(float (&g)[C], uint32_t jm, uint32_t up, int n, int t)
{
    const int k0 = t * C;
    const int nv = min(max(n - 1 - k0, 0), C);             // duals of this chunk inside the row
    const uint32_t inrow = (1u << nv) - 1u;
    const uint32_t gmask = jm & inrow;                      // jumps that count for dL/dlam
    // the end of the row closes a segment, and samples past it are segments of their own
    const uint32_t jmask = (jm & inrow) | ~inrow;
#define TV_JUMP(i) ((jmask >> (i)) & 1u)
    bool any = false;
    float head_s = 0.f, head_n = 0.f, tail_s = 0.f, tail_n = 0.f;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        if (!any) { head_s += g[i]; head_n += 1.f; }
        tail_s += g[i]; tail_n += 1.f;
        if (TV_JUMP(i)) { any = true; tail_s = 0.f; tail_n = 0.f; }
    }
    float ls, ln, rs, rn;
    row_open_part_before<T, +1>(any, tail_s, tail_n, t, ls, ln);       // open part on the left
    row_open_part_before<T, -1>(any, head_s, head_n, t, rs, rn);       // open part on the right
    {
        float s = ls, c = ln;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            s += g[i]; c += 1.f;
            g[i] = 0.f;
            if (TV_JUMP(i)) { g[i] = s * __builtin_amdgcn_rcpf(c); s = 0.f; c = 0.f; }
        }
        // the trailing open part continues into the next chunks
        float carry = (c > 0.f) ? (s + rs) * __builtin_amdgcn_rcpf(c + rn) : 0.f;
#pragma unroll
        for (int i = C - 1; i >= 0; --i) {
            if (TV_JUMP(i)) carry = g[i];
            g[i] = carry;
        }
    }
#undef TV_JUMP
    const float mnext0 = from_right<T, 1>(g[0], t);
    float gl = 0.f;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        if ((gmask >> i) & 1u) {
            const float mn = (i + 1 < C) ? g[i + 1] : mnext0;
            const float d = g[i] - mn;
            gl += ((up >> i) & 1u) ? d : -d;
        }
    }
    return gl;
}

// T, C as in the forward kernel.  Planes of at most 32 x 32 read the segments of a pass from its
// 8-byte codes, larger ones from their row masks (MASKS, where p.tag says so) or its saved output.  p.partial gets one dL/dlam term per plane.
// IO16: the upstream gradient and grad_y are bf16 in memory.  MASKS: the workspace may hold row masks.
template <int T, int C, bool IO16 = false, bool MASKS = false>
__global__ __launch_bounds__(T * T * C, C <= 4 ? 8 : 4) void tv2d_bwd_plane_kernel(Small2dBwdParams p)
{
    constexpr int S = T * C, P = S + 1, NT = S * T, NW = NT / 64;
    static_assert(NT % 64 == 0 && NT <= 1024, "whole waves");
    __shared__ float A[S * P], B[S * P], part[NW];
    const int tid = threadIdx.x;
    const int j = tid / T, t = tid % T, k0 = t * C;
    const int H = p.H, W = p.W, HW = H * W;
    const int64_t plane = blockIdx.x;
    if constexpr (IO16) {
        const uint16_t *src = reinterpret_cast<const uint16_t *>(p.g_up) + plane * HW;
        for (int e = tid; e < HW; e += NT) A[(e / W) * P + e % W] = bf16_bits_to_f32(src[e]);
    } else {
        const float *src = p.g_up + plane * HW;
        for (int e = tid; e < HW; e += NT) A[(e / W) * P + e % W] = src[e];
    }

    // Segments of pass `pass` for the thread's chunk of its row (row pass) or column (column
    // pass); fetched one pass ahead, so that the latency hides behind the pass before.
    const bool coded = MASKS && *p.tag == 1u;
    auto fetch = [&](int pass, uint32_t &jm, uint32_t &up) {
        jm = 0u; up = 0u;
        if (pass < 0) return;
        const bool col = (pass & 1) != 0;
        const int n = col ? H : W, rows = col ? W : H;
        const bool valid = j < rows;
        if constexpr (S <= 32) {
            if (valid) {
                const uint2 c = p.codes[(size_t)pass * p.code_stride + (size_t)plane * rows + j];
                jm = (c.x >> k0) & ((1u << C) - 1u);
                up = (c.y >> k0) & ((1u << C) - 1u);
            }
        } else if (coded) {
            if (valid) {
                const uint8_t *from = reinterpret_cast<const uint8_t *>(p.codes + (size_t)pass * p.code_stride + ((size_t)plane * rows + j) * 2);
                jm = from[t];
                up = from[8 + t];
            }
        } else {
            const float *xs = p.saved + (size_t)pass * p.saved_stride + (size_t)plane * HW;
            float x[C];
#pragma unroll
            for (int c = 0; c < C; ++c)
                x[c] = (valid && k0 + c < n) ? (col ? xs[(k0 + c) * W + j] : xs[j * W + k0 + c]) : 0.f;
            const float xnext0 = from_right<T, 1>(x[0], t);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float xn = (c + 1 < C) ? x[c + 1] : xnext0;
                if (xn != x[c]) jm |= 1u << c;
                if (xn > x[c]) up |= 1u << c;
            }
        }
    };

    float glam = 0.f;
    uint32_t jm_next, up_next;
    fetch(2 * p.sweeps - 1, jm_next, up_next);
    __syncthreads();
    // Adjoint of one sweep (A = Y + P, Z = R(A), P' = A - Z, B = Z + Q, Y' = C(B), Q' = B - Y'):
    //   Bbar = Qbar' + C^T(Ybar' - Qbar'),   Abar = Pbar' + R^T(Bbar - Pbar'),   Ybar = Pbar = Abar;
    // tile A carries Ybar = Pbar, tile B carries Qbar = Bbar.  A thread reads and writes only its
    // own tile elements in a pass, so one barrier per pass suffices.
    for (int k = p.sweeps - 1; k >= 0; --k) {
        const bool first = (k == p.sweeps - 1);
#pragma unroll
        for (int dir = 1; dir >= 0; --dir) {
            const bool col = dir != 0;
            const int n = col ? H : W, rows = col ? W : H;
            const bool valid = j < rows;
            const int base = col ? j : j * P, step = col ? P : 1;
            const uint32_t jm = jm_next, up = up_next;
            fetch(2 * k + dir - 1, jm_next, up_next);
            float *dst = col ? B : A;                    // column pass: B <- C^T(A - B) + B
            const float *src = col ? A : B;              // row pass:    A <- R^T(B - A) + A
            float v[C], old[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const bool in = valid && k0 + c < n;
                const int e = base + (k0 + c) * step;
                old[c] = (in && !first) ? dst[e] : 0.f;
                v[c] = in ? src[e] - old[c] : 0.f;
            }
            const float gl = lanes_segment_means<T, C>(v, jm, up, n, t);
            if (valid) glam += gl;
#pragma unroll
            for (int c = 0; c < C; ++c)
                if (valid && k0 + c < n) dst[base + (k0 + c) * step] = old[c] + v[c];
            __syncthreads();
        }
    }
    if constexpr (IO16) {
        uint16_t *dst = reinterpret_cast<uint16_t *>(p.gy) + plane * HW;
        for (int e = tid; e < HW; e += NT) dst[e] = f32_to_bf16_bits(A[(e / W) * P + e % W]);
    } else {
        float *dst = p.gy + plane * HW;
        for (int e = tid; e < HW; e += NT) dst[e] = A[(e / W) * P + e % W];
    }
    if (p.partial) {
        // the plane's term: waves in a fixed order
        const float s = wave_sum_all<64>(glam);
        if ((tid & 63) == 0) part[tid >> 6] = s;
        __syncthreads();
        if (tid == 0) {
            float tot = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) tot += part[w];
            p.partial[plane] = tot;
        }
    }
}

}  // namespace tvk
