// Backward kernel for strided rows (the columns of images) of 33-1024 samples: nothing is transposed.
#pragma once
#include <type_traits>

#include "tv_long.hpp"

namespace tvk {

// Which group of columns a workgroup works on: runs of 1 << lg neighbouring groups on one XCD (see xcd_grouped), which has
// its own L2.
__device__ __forceinline__ uint32_t xcd_together(uint32_t b, uint32_t n_groups, uint32_t lg)
{
    const uint32_t base = b & ~((8u << lg) - 1u);
    if (base + (8u << lg) > n_groups) return b;     // the ragged end keeps the launch order
    return base + ((b & 7u) << lg) + ((b >> 3) & ((1u << lg) - 1u));
}

// The value of `v` in the lane that a DPP control word or a permutation names, for 64-bit values.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ double dpp64(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWS, 0xf, true);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double lane64(double v, int from)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(from << 2, (int)(uint32_t)u);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(from << 2, (int)(uint32_t)(u >> 32));
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
// s / n, to 2^-45 or so
__device__ __forceinline__ double mean64(double s, float n)
{
    const double r = (double)__builtin_amdgcn_rcpf(n);
    return s * fma(fma(-(double)n, r, 1.0), r, r);
}
// RowWave::open_sum in 64 bits: v of this lane and of the `dist` lanes before it, TW lanes a row, at most 64.
template <int TW>
__device__ __forceinline__ double open_sum64(double v, int dist, int lane)
{
#define TV_STEP(S)                                        \
    if constexpr ((S) < TW) {                             \
        const double o = dpp64<0x110 + ((S) & 15)>(v);    \
        v += dist >= (S) ? o : 0.0;                       \
    }
    TV_STEP(1) TV_STEP(2) TV_STEP(4) TV_STEP(8)
#undef TV_STEP
    if constexpr (TW > 16) {
        const double o = lane64(v, (lane & ~15) - 1);     // the last lane of the 16 before
        v += (lane & 16) && dist > (lane & 15) ? o : 0.0;
    }
    if constexpr (TW > 32) {
        const double o = lane64(v, 31);
        v += (lane & 32) && dist > (lane & 31) ? o : 0.0;
    }
    return v;
}

// T threads a column with C contiguous samples each, G adjacent columns a workgroup, thread = t * G + column: every load and
// store of a wave covers 4 G contiguous bytes of 64 / G image rows, and a thread's samples stay in its registers from
// the load to the store.  Between the threads of a column travel only the pieces of the segments that cross from one
// chunk to the next (paper Eq. 5-6 as segment averaging): the sum and count of a chunk's samples up to its
// first jump and behind its last one.  They lie in LDS as [t][column]; with columns and threads exchanged (T
// neighbouring lanes take the T pieces of one column) a segmented sum over lanes and one fetch of a mean from the
// lane where a segment ends turn them into the two means that each chunk needs: that of the segment open at its
// start and that of the one open at its end.
// Bound by memory, and by the vector ALUs on columns of at most 64 samples: 24 planes of 512 x 512, backward with its
// lambda sum, 26.9 -> 19.1 us (75 MB); 8M samples in planes of 33 / 64 / 100 / 200 / 481 / 900 a side
// 128 / 71 / 67 / 45 / 45 / 47 -> 35 / 25 / 26 / 25 / 26 / 27.  (Before, every tensor crossed an LDS tile that turned columns into
// rows and back.)  Error against 64 bits, thirty calls: grad_y 6.3e-8 -> 2.5e-8, dL/dlam 3.1e-7 -> 4.0e-8; with
// sums and means in 32 bits and dL/dlam in 64, 4.8e-8 and 2.4e-7, at 19.0 us where 64 bits then took 20.5: one lambda's gradient cancels, and was
// further off than before in one call of ten.
// G: 32 columns, a line, where that leaves workgroups of at most 512 threads, 16 beyond (512 a side, with sub: 18.5 us, with 32
// columns 21.6; 768, no sub, 64 threads of 12 samples 19.8, 32 threads of 24 and 32 columns 23.8).
// HAS_SUB: p.sub is given (the reverse sweep of the 2D operator).  CODES: where the forward pass left chunk codes
// (p.codes_tag says whether it did) they are read, not x: CW words of C / CW samples a thread, in the forward kernel's
// order (word t of its row); CW = -2: a word for two threads; row masks where columns have 33-64 samples.
// SUMS: p.partial is given.  (Of its own on columns of at most 64 samples, where the instructions count: 260 000 columns of 44 without
// dL/dlam, 33.9 us in a kernel that forms it all the same, 30.6 here.)
template <int T, int C, int G, int CW, bool HAS_SUB, bool CODES, bool SUMS = true>
__global__ __launch_bounds__(T *G) void tv1d_bwd_cols_kernel(BwdParams p)
{
    static_assert(T <= 64 && C <= 32 && (CW == -2 || C % CW == 0) && G <= 64, "a column's threads inside one wave when exchanged");
    using Rw = RowWave<T, G, false>;
    constexpr int P = G + 1;                     // (both [t][column] accesses are then free of bank conflicts)
    __shared__ double first[T * P], last[T * P]; // sums of the pieces, then the two means
    __shared__ uint32_t sizes[T * P];            // their counts and whether the chunk holds a jump, then dL/dlam terms
    const int tid = threadIdx.x;
    const int col = tid % G, t = tid / G;
    const uint32_t group = xcd_together(blockIdx.x, gridDim.x, p.near_lg);
    const uint32_t row = group * G + col;
    const bool rvalid = row < p.L.n_rows;
    const uint32_t arow = rvalid ? row : p.L.n_rows - 1u;      // (what is read for a column that does not exist)
    const int n = p.L.n, k0 = t * C;
    const int64_t es = p.L.elem_stride;
    const int64_t at0 = row_offset(p.L, arow) + (int64_t)k0 * es;
    const bool whole = k0 + C <= n;
    // A chunk that the column's end cuts is read with a branch a sample, or, where more than half of it is there and instructions count,
    // without: past the end its last sample (260 000 columns of 44 without dL/dlam 30.6 -> 27.7 us, 600 000 of 60
    // 97 -> 86; 250 000 of 50, two samples of sixteen, 28.2 -> 29.9 that way).
    const bool clamp = T * C == 64 && n % C > C / 2 && !__all(whole);
    const int64_t last0 = at0 - (int64_t)max(k0 - (n - 1), 0) * es;
    auto fetch = [&](const float *__restrict__ src, float (&v)[C]) {
        if (clamp) {
            const float *from = src + last0;
#pragma unroll
            for (int i = 0; i < C; ++i) {
                v[i] = *from;
                from += k0 + i + 1 < n ? es : 0;
            }
#pragma unroll
            for (int i = 0; i < C; ++i) v[i] = k0 + i < n ? v[i] : 0.f;
            return;
        }
        const float *at = src + at0;
        if (whole) {
#pragma unroll
            for (int i = 0; i < C; ++i) v[i] = at[i * es];
        } else {
#pragma unroll
            for (int i = 0; i < C; ++i) v[i] = k0 + i < n ? at[i * es] : 0.f;
        }
    };

    float g[C], sb[HAS_SUB ? C : 1];
    uint32_t jmask = 0, upmask = 0;
    // duals of this chunk that lie inside the row (dual i sits behind sample k0 + i)
    const int nv = min(max(n - 1 - k0, 0), C);
    const uint32_t inrow = nv == 32 ? ~0u : (1u << nv) - 1u;
    bool coded = false;
    if constexpr (CODES) coded = *p.codes_tag == 1u;
    fetch(p.g, g);
    if constexpr (HAS_SUB) fetch(p.sub, sb);
    if (CODES && coded) {
        if constexpr (row_masked<T, C>()) {
            mask_bits<C>(p.chunk_codes, arow, k0, jmask, upmask);
        } else if constexpr (CW == -2) {
            const uint32_t code = p.chunk_codes[(size_t)arow * (T / 2) + t / 2] >> (t & 1) * 2 * C;
            jmask = even_bits(code) & ((1u << C) - 1u);
            upmask = even_bits(code >> 1) & ((1u << C) - 1u);
        } else {
            const uint32_t *words = p.chunk_codes + ((size_t)arow * T + t) * CW;
#pragma unroll
            for (int w = 0; w < CW; ++w) {
                const uint32_t code = words[w];
                jmask |= even_bits(code) << (w * (C / CW));
                upmask |= even_bits(code >> 1) << (w * (C / CW));
            }
        }
    } else {
        float x[C];
        fetch(p.x, x);
        const float xnext0 = k0 + C < n ? p.x[at0 + C * es] : 0.f;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const float xn = (i + 1 < C) ? x[i + 1] : xnext0;
            if (xn != x[i]) jmask |= 1u << i;
            if (xn > x[i]) upmask |= 1u << i;
        }
    }
    const uint32_t gmask = jmask & inrow;      // jumps that count for dL/dlam
    const uint32_t end = nv < C ? 1u << nv : 0u;       // the end of the row ends a segment (what lies past it counts for nothing)
    const uint32_t jumps = gmask | end, lowest = jumps & (0u - jumps);
    if constexpr (HAS_SUB) {
#pragma unroll
        for (int i = 0; i < C; ++i) g[i] -= sb[i];
    }
#define TV_JUMP(i) ((jumps >> (i)) & 1u)
    // Segments that lie inside the chunk are done at once.  Sums and means in 64 bits: dL/dlam sees only differences of
    // means, each once at either end of its segment, with the signs of the jumps there, and those of a slot cancel.
    // A mean's weight is 2 or -2 where the row turns at the segment's end, and 0 where it goes on rising or falling (an infinite mean or NaN
    // shows there too): the signs of all jumps of a chunk and of the jumps before them come from a few operations on its masks, a carry
    // taking the sign of a jump to the next one.
    const uint32_t up = upmask & gmask, up_before = ((up << 1) + ~jumps) & jumps;
    const uint32_t turns = (up ^ up_before) & gmask, falls = turns & ~up;
    double gl = 0.0;
    bool any = false;
    {
        double s = 0.0, head_s = 0.0, m = 0.0;
        float c = 0.f;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            s += (double)g[i]; c += 1.f;
            if (TV_JUMP(i)) {
                if (any) {
                    m = mean64(s, c);
                    if (SUMS) {
                        constexpr int TWO = 30;                  // (the bit of a double's upper half that makes it 2)
                        const uint32_t two = i <= TWO ? turns << (TWO - i & 31) : turns >> (i - TWO & 31);
                        const uint32_t w = (two & 1u << TWO) | (falls << (31 - i) & 1u << 31);
                        gl = fma(__builtin_bit_cast(double, (uint64_t)w << 32), m, gl);
                    }
                    g[i] = (float)m;
                } else {
                    head_s = s;
                }
                any = true;
                s = 0.0; c = 0.f;
            }
        }
        if (SUMS && (end & ~lowest) != 0u) gl += (up_before & end) != 0u ? -m : m;       // the row's last segment has a sign at one end only
        const double tail_s = s;
        if (!any) head_s = s;
        const uint32_t head_n = any ? (uint32_t)__builtin_ctz(jumps | 0x80000000u) + 1u : (uint32_t)C;
        const uint32_t tail_n = (uint32_t)c;
        first[t * P + col] = head_s;
        last[t * P + col] = tail_s;
        sizes[t * P + col] = head_n | tail_n << 8 | (any ? 1u << 16 : 0u);
    }
    __syncthreads();
    {
        const int at = (tid % T) * P + tid / T;
        const double head_s = first[at], tail_s = last[at];
        const uint32_t sz = sizes[at];
        const float head_n = (float)(sz & 0xffu), tail_n = (float)(sz >> 8 & 0xffu);
        const bool closed = (sz >> 16) != 0u;
        const Rw rw(tid % T);
        const uint64_t cmask = lanes_with(closed);
        const int L = rw.last_before(cmask);
        const int apart = rw.lane - L;
        const double upto = open_sum64<T>(tail_s, closed ? 0 : apart, rw.lane);
        double left_s = lane64(upto, rw.lane - 1);
        float left_n = Rw::at(tail_n, L) + (float)(apart * C - C);
        if (rw.tw == 0) { left_s = 0.0; left_n = 0.f; }
        // the lane in which a segment ends knows its mean; the others fetch it (the last one always holds an end)
        const double head_m = mean64(left_s + head_s, left_n + head_n);
        const double tail_m = lane64(head_m, rw.first_after(cmask));
        first[at] = closed ? head_m : tail_m;
        last[at] = tail_m;
    }
    __syncthreads();
    {
        const double head_m = first[t * P + col], tail_m = last[t * P + col];
        if (SUMS && (lowest & gmask) != 0u) gl += (up & lowest) != 0u ? head_m : -head_m;
        const uint32_t highest = 0x80000000u >> __builtin_clz(jumps | 1u);
        if (SUMS && (highest & gmask) != 0u) gl += (up & highest) != 0u ? -tail_m : tail_m;
        const float head = (float)head_m;
        float carry = (float)tail_m;
#pragma unroll
        for (int i = C - 1; i >= 0; --i) {
            if (TV_JUMP(i)) carry = (lowest >> i) & 1u ? head : g[i];
            g[i] = carry;
        }
    }
    if constexpr (HAS_SUB) {
#pragma unroll
        for (int i = 0; i < C; ++i) g[i] += sb[i];
    }
    if (rvalid) {
        float *at = p.gy + at0;
        if (whole) {
#pragma unroll
            for (int i = 0; i < C; ++i) at[i * es] = g[i];
        } else {
#pragma unroll
            for (int i = 0; i < C; ++i)
                if (k0 + i < n) at[i * es] = g[i];
        }
    }
#undef TV_JUMP
    if (SUMS && p.partial) {
        float *terms = reinterpret_cast<float *>(sizes);
        terms[t * P + col] = rvalid ? (float)gl : 0.f;
        __syncthreads();
        if (tid < G) {
            double sum = 0.0;                    // (64 bits from here on)
#pragma unroll 8
            for (int q = 0; q < T; ++q) sum += (double)terms[q * P + tid];
            // neighbouring columns that share a slot leave as one term, in two floats (the second says nothing beside an infinity)
            for (uint32_t d = 0; d < p.part_lg; ++d) sum += __shfl_xor(sum, 1 << d);
            if (rvalid && (tid & ((1 << p.part_lg) - 1)) == 0) {
                const float hi = (float)sum;
                const float lo = isfinite(hi) ? (float)(sum - (double)hi) : 0.f;
                if (p.part_lg) *reinterpret_cast<float2 *>(p.partial + 2 * (size_t)(row >> p.part_lg)) = make_float2(hi, lo);
                else p.partial[row] = hi;
            }
        }
    }
}

// Runs of neighbouring groups on one XCD: a 128-byte line at least.  Where image rows are no whole number of
// lines every group shares one with each of its neighbours, in every image row: runs of 512 columns there, or as many as
// leave three rounds of eight runs.  (8M samples, runs of 32 / 128 / 512 columns: 33 a side 32.0 / 22.6 / 21.0 us, 200
// 28.7 / 24.5 / 22.6, 481 32.6 / 26.0 / 23.6, 900 30.1 / 24.6 / 23.0; whole lines, 512 a side, 18.7 / 18.7 / 18.2, a third fewer
// images 14.8 / 15.5 / 15.7.)
template <int G>
inline uint32_t bwd_cols_near_lg(const BwdParams &p, uint32_t groups)
{
    const bool lines = p.L.elem_stride % 32 == 0 && p.L.n_inner % 32 == 0 && ((uintptr_t)p.g | (uintptr_t)p.gy) % 128 == 0;
    uint32_t lg = 0;
    while ((G << lg) < (lines ? 32 : 512) && (48u << lg) <= groups) ++lg;
    return lg;
}

// Strided rows that go this way; and the columns of a workgroup, whose dL/dlam terms can leave as one.
inline bool bwd_cols_apply(int64_t n, int64_t elem_stride) { return n > 32 && n <= 1024 && elem_stride != 1; }
// (16 of them at least, 32 in larger calls on shorter columns; groups of 16 leave as one in both.)
constexpr int kBwdColsGroupLg = 4;

template <int T, int C, int CW, int G = (T <= 16 ? 32 : 16)>
inline hipError_t launch_bwd_cols_t(BwdParams p, hipStream_t s)
{
    const dim3 grid((p.L.n_rows + G - 1) / G), block(T * G);
    p.near_lg = bwd_cols_near_lg<G>(p, grid.x);
    auto launch = [&](auto sums) {
        constexpr bool SUMS = decltype(sums)::value;
        if constexpr (CW != 0) {
            if (p.chunk_codes) {
                if (p.sub) hipLaunchKernelGGL((tv1d_bwd_cols_kernel<T, C, G, CW, true, true, SUMS>), grid, block, 0, s, p);
                else hipLaunchKernelGGL((tv1d_bwd_cols_kernel<T, C, G, CW, false, true, SUMS>), grid, block, 0, s, p);
                return hipGetLastError();
            }
        }
        if (p.sub) hipLaunchKernelGGL((tv1d_bwd_cols_kernel<T, C, G, 1, true, false, SUMS>), grid, block, 0, s, p);
        else hipLaunchKernelGGL((tv1d_bwd_cols_kernel<T, C, G, 1, false, false, SUMS>), grid, block, 0, s, p);
        return hipGetLastError();
    };
    if constexpr (T * C == 64)
        if (!p.partial) return launch(std::false_type{});
    return launch(std::true_type{});
}

// CW: the words of chunk_threads(n) that a thread's C samples are (1 where it reads a row mask, -2 for half a word), 0 where there are none.
inline hipError_t launch_bwd_cols(const BwdParams &p, hipStream_t s)
{
    const int n = p.L.n;
    if ((int64_t)p.L.n_rows <= tvd::get(tvd::kBwdFewColumns)) {
        if (n <= 64) return launch_bwd_cols_t<16, 4, 1, 16>(p, s);
        if (n <= 96) return launch_bwd_cols_t<16, 6, -2, 16>(p, s);
        if (n <= 128) return launch_bwd_cols_t<16, 8, 1, 16>(p, s);
        if (n <= 192) return launch_bwd_cols_t<32, 6, -2, 16>(p, s);
        if (n <= 256) return launch_bwd_cols_t<32, 8, 1, 16>(p, s);
    }
    if (n <= 64) return launch_bwd_cols_t<4, 16, 1>(p, s);
    if (n <= 96) return launch_bwd_cols_t<8, 12, 1>(p, s);
    if (n <= 128) return launch_bwd_cols_t<8, 16, 2>(p, s);
    if (n <= 192) return launch_bwd_cols_t<16, 12, 1>(p, s);
    if (n <= 256) return launch_bwd_cols_t<16, 16, 2>(p, s);
    if (n <= 384) return launch_bwd_cols_t<32, 12, 1>(p, s);
    if (n <= 512) return launch_bwd_cols_t<32, 16, 2>(p, s);
    if (n <= 768) return launch_bwd_cols_t<64, 12, 1>(p, s);
    // (with sub 64 threads of 16 samples take 72 registers, and a CU holds one workgroup: 900 a side 36 us against 32)
    return p.sub ? launch_bwd_cols_t<32, 32, 0>(p, s) : launch_bwd_cols_t<64, 16, 0>(p, s);
}

}  // namespace tvk
