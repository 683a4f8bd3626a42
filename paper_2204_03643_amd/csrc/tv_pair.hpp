// Two neighbouring lanes per row, one from each end: projected Newton on the dual (paper Eq. 3-4) of
// a row of at most 2 C samples, and the kernels built on it: the one-launch 2D forward on planes of 17-64
// samples a side, and the forward on large batches of rows of 17-64 samples.
//
// A row-per-lane solve (RowSolver, tv_short.hpp) keeps four arrays of a row's length in registers and
// walks chains of that length.  Here the row is cut in the middle: the left lane holds samples 0 .. C-1,
// the right lane samples 2C-1 .. C, outermost first.  Seen from its own end each half is the same
// problem (a row reversed has the reversed x and the reversed, negated dual), so both lanes run the
// same instructions on C registers a array and chains of C steps, and meet in the dual between the
// halves, which both hold, with opposite signs, and form from symmetric expressions, so that the
// copies stay exact mirrors of one another.  Half the registers make twice the waves, each wave is
// done when the slowest of 32 rows is (not of 64), and rounding errors run through chains half as long.
#pragma once
#include "tv_small2d.hpp"

namespace tvk {

// v of the other lane of the pair (rides on the instruction that reads it)
__device__ __forceinline__ float pair_other(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xf, 0xf, true));     // quad_perm [1,0,3,2]
}
__device__ __forceinline__ uint32_t pair_other(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true);
}
// v of the pair's left / right lane, in both
__device__ __forceinline__ float pair_left(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xA0, 0xf, 0xf, true));     // [0,0,2,2]
}
__device__ __forceinline__ float pair_right(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xF5, 0xf, 0xf, true));     // [1,1,3,3]
}
// p or the other lane's p (in scalar registers)
__device__ __forceinline__ bool pair_either(bool p)
{
    const uint64_t even = 0x5555555555555555ull;
    const uint64_t m = __builtin_amdgcn_ballot_w64(p);
    return __builtin_amdgcn_inverse_ballot_w64(m | ((m >> 1) & even) | ((m & even) << 1));
}

template <int PADS>
__device__ __forceinline__ float pair_masked(float v, uint32_t have, int k)
{
    return k >= PADS ? v : __uint_as_float(__float_as_uint(v) & (uint32_t)__builtin_amdgcn_sbfe((int)have, k, 1));
}

// Local sample i of a lane is sample i of its row (left lane) or 2C-1-i (right lane); local dual i lies
// behind local sample i, towards the middle, and dual C-1 is the shared one.  Rows of fewer than 2C
// samples: those past the end are 0, the dual behind the last one (`cut`, a local index, none if negative)
// is held at 0, and bit i of `live` says that local dual i lies inside the row.  All that concerns local
// indices below PADS only: PADS = 0, rows of exactly 2C samples; PADS = C, any.
// STRIDE: between the parked samples of a lane (the threads of the workgroup).
template <int C, int PADS, int STRIDE = 64>
struct PairSolver {
    static constexpr bool FULL = PADS == 0;
    float X[C];         // x(u) for the current dual
    float u[C];         // the dual
    float D[C];         // g, then gamma * w, then the Newton direction
    float G[C];         // pivots gamma (0 exactly at bound duals; G[C-1]: 0 or 1), then the previous dual
    const float *yl, *gtab;       // the parked input (sample i at yl[STRIDE i]), gtab[j] = j / (j + 1)
    float lam, fcur, alpha_try, gtol;
    uint32_t live;
    int cut, steps, flags, nfail;
    bool active, prev_unclipped;

    // (inside: `live`, made opaque in every loop: as loop invariants the C boxes would be kept in registers)
    __device__ __forceinline__ uint32_t inside() const
    {
        uint32_t l = live;
        if (!FULL) asm volatile("" : "+v"(l));
        return l;
    }
    __device__ __forceinline__ float box(uint32_t inside, int k) const
    {
        if (k >= PADS) return lam;
        return __uint_as_float(__float_as_uint(lam) & (uint32_t)__builtin_amdgcn_sbfe((int)inside, k, 1));
    }
    __device__ __forceinline__ float yk(int k) const { return yl[k * STRIDE]; }
    static __device__ __forceinline__ void reread() { asm volatile("" ::: "memory"); }

    // Two Gauss-Seidel sweeps on the dual, u_k <- clip((u_{k-1} + u_{k+1} + y_{k+1} - y_k) / 2): from both ends
    // to the middle, and back.  D holds half the differences of y.
    __device__ __forceinline__ void sweep_in_and_out()
    {
        uint32_t in = inside();
        float up = 0.f;
#pragma unroll
        for (int k = 0; k < C - 1; ++k) {
            const float l = box(in, k);
            up = __builtin_amdgcn_fmed3f(fmaf(0.5f, up + u[k + 1], D[k]), -l, l);
            u[k] = up;
        }
        float un;
        {
            const float l = box(in, C - 1);
            un = __builtin_amdgcn_fmed3f(fmaf(0.5f, up - pair_other(up), D[C - 1]), -l, l);
            u[C - 1] = un;
        }
        in = inside();
#pragma unroll
        for (int k = C - 2; k >= 0; --k) {
            const float l = box(in, k);
            const float ul = k > 0 ? u[k - 1] : 0.f;
            un = __builtin_amdgcn_fmed3f(fmaf(0.5f, ul + un, D[k]), -l, l);
            u[k] = un;
        }
    }

    // x(u) and the dual objective of the starting dual
    __device__ __forceinline__ void primal_of_start(const float (&y)[C])
    {
        float acc = 0.f, prev = 0.f;
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const float xc = y[k] + u[k] - prev;
            acc = fmaf(xc, xc, acc);
            X[k] = xc; prev = u[k];
        }
        fcur = 0.5f * (acc + pair_other(acc));
    }
    __device__ __forceinline__ void set_gtol(const float (&y)[C])
    {
        float ymax = 0.f;
#pragma unroll
        for (int k = 0; k < C; ++k) ymax = fmaxf(ymax, fabsf(y[k]));
        ymax = fmaxf(ymax, pair_other(ymax));
        // (lambda = 0: every dual sits on both of its bounds, no gradient may count as pointing inwards)
        gtol = lam > 0.f ? kGradNoise * (ymax + lam) : __builtin_inff();
    }

    // Cold start: the two candidates and the choice of RowSolver::start, then two Gauss-Seidel sweeps.
    // have: bit i = local sample i exists.
    __device__ __forceinline__ void start(const float (&y)[C], float inv_n, uint32_t have)
    {
        float sum = 0.f;
#pragma unroll
        for (int k = 0; k < C; ++k) {
            sum -= y[k];
            X[k] = sum;
        }
        set_gtol(y);
        const float ybar = -(sum + pair_other(sum)) * inv_n;
        float run = 0.f, rmax = 0.f, past = 0.f;
#pragma unroll
        for (int k = 0; k < C; ++k) {
            if (PADS == 0) run = fmaf(ybar, (float)(k + 1), X[k]);      // sum over i <= k of ybar - y_i
            else {
                past += pair_masked<PADS>(ybar, have, k);
                run = past + X[k];
            }
            X[k] = run;
            rmax = fmaxf(rmax, fabsf(run));
        }
        X[C - 1] = 0.5f * (run - pair_other(run));
        rmax = fmaxf(rmax, pair_other(rmax));
        const bool free_row = lam >= 0.25f * rmax;
        const uint32_t in = inside();
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const float l = box(in, k);
            const float yn = k + 1 < C ? y[k + 1] : pair_other(y[C - 1]);
            const float hd = 0.5f * (yn - y[k]);
            u[k] = __builtin_amdgcn_fmed3f(free_row ? X[k] : hd * 1e30f, -l, l);
            D[k] = hd;
        }
        sweep_in_and_out();
        primal_of_start(y);
    }

    // Warm start: u holds the negated running sums, from the lane's own end, of the correction term
    // that the input carries (see RowSolver::start_warm).
    __device__ __forceinline__ void start_warm(const float (&y)[C])
    {
        set_gtol(y);
        u[C - 1] = 0.5f * (u[C - 1] - pair_other(u[C - 1]));
        const uint32_t in = inside();
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const float l = box(in, k);
            u[k] = __builtin_amdgcn_fmed3f(u[k] * kWarmSnap, -l, l);
        }
        primal_of_start(y);
    }

    // Gradient, bound set, elimination and optimality test; true when every row of the wave has stopped.
    __device__ __forceinline__ bool look(int it, bool &vio, float &dec)
    {
        vio = false;
        uint32_t pos4 = 0, mid4 = 0;                // 4 * position inside the free run
        {
            int c = cut;
            if (!FULL) asm volatile("" : "+v"(c));
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const float g = X[k] - (k + 1 < C ? X[k + 1] : pair_other(X[C - 1]));
                const float s = copysignf(lam, g);
                bool bnd = (u[k] == -s) || (k < PADS && k == c);
                // (the middle: +0 has the same sign in both lanes, where -s would say different things)
                if (k == C - 1) bnd |= g == 0.f && fabsf(u[k]) == lam;
                vio |= (u[k] == s) && (fabsf(g) > gtol);
                D[k] = g;
                if (k < C - 1) {
                    pos4 = bnd ? 0u : pos4 + 4u;
                    G[k] = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(gtab) + pos4);
                    mid4 = pos4;
                } else {
                    G[k] = bnd ? 0.f : 1.f;
                }
            }
        }
        vio = pair_either(vio);
        // (rows that landed on the minimiser of their free subspace need no elimination to see that they are done)
        if (active && !vio && prev_unclipped) { active = false; flags = kInfoConverged; }
        if (!__any(active)) { dec = 0.f; return true; }
        // from both ends: w_k = g_k + gamma_{k-1} w_{k-1}, kept as t_k = gamma_k w_k
        float t = 0.f;
        dec = 0.f;
#pragma unroll
        for (int k = 0; k < C - 1; ++k) {
            const float w = D[k] + t;
            t = G[k] * w;
            dec = fmaf(t, w, dec);
            D[k] = t;
        }
        asm volatile("" : "+v"(dec));
        // the middle: the runs of a - 1 and b - 1 free duals that end on either side of it leave the pivot
        // 2 - (a - 1) / a - (b - 1) / b = (a + b) / (a b)
        {
            const float a = fmaf(0.25f, (float)mid4, 1.f), b = pair_other(a);
            const float w = D[C - 1] + (t - pair_other(t));
            const float d = G[C - 1] * w * (a * b) * __builtin_amdgcn_rcpf(a + b);
            dec = fmaf(w, d, dec + pair_other(dec));
            D[C - 1] = d;
        }
        const float small = C > 16 ? gtol * gtol : fmaxf(kDecNoise * fcur, gtol * gtol);
        if (active && !vio && (C > 16 ? dec < small : dec <= small)) {
            active = false; flags = kInfoConverged;
        }
        if (active && it >= kMaxNewtonSteps) { active = false; flags = kInfoCapped; }
        return !__any(active);
    }

    // Direction, projected step, line search (RowSolver::iterate has the reasons for every rule).
    __device__ __forceinline__ void step(bool vio, float dec)
    {
        steps += active ? 1 : 0;
        reread();
#pragma unroll
        for (int k = 0; k < C; ++k) X[k] = yk(k);
        float dn = D[C - 1];
#pragma unroll
        for (int k = C - 2; k >= 0; --k) {
            dn = fmaf(G[k], dn, D[k]);
            D[k] = dn;
        }
        const float alpha = active ? alpha_try : 0.f;
        float tmax = 0.f;
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const float uo = u[k];
            const float t = fmaf(-alpha, D[k], uo);
            tmax = fmaxf(tmax, fabsf(t));
            G[k] = uo;
            u[k] = __builtin_amdgcn_fmed3f(t, -lam, lam);
        }
        const bool clipped = fmaxf(tmax, pair_other(tmax)) > lam;
        const bool polish = clipped && active;
        if (__any(polish)) {
            float half = 0.5f;
            asm volatile("" : "+v"(half));
#pragma unroll
            for (int k = 0; k < C; ++k) D[k] = half * ((k + 1 < C ? X[k + 1] : pair_other(X[C - 1])) - X[k]);
            if (polish) sweep_in_and_out();         // (both lanes of a row or neither)
        }
        float acc = 0.f, prev = 0.f;
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const float c = u[k];
            const float xc = X[k] + c - prev;
            acc = fmaf(xc, xc, acc);
            X[k] = xc; prev = c;
        }
        const float fc = 0.5f * (acc + pair_other(acc));
        bool changed = true;
        if (__any(active && fc == fcur)) {          // (a step that leaves the dual bit-identical also leaves f so)
            changed = false;
#pragma unroll
            for (int k = 0; k < C; ++k) changed |= (u[k] != G[k]);
            changed = pair_either(changed);
        }
        if (active && fc != fc) { active = false; flags = kInfoStalled | kInfoPlain; }      // NaN in the row
        const bool ok = !active || (alpha == 1.f && !clipped) ||
                        (fc <= fcur - kArmijoSigma * alpha * dec + kArmijoSlackEps * fabsf(fcur));
        if (__any(!ok)) {
            reread();
            float pv = 0.f;
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const float c = ok ? u[k] : G[k];
                u[k] = c;
                X[k] = yk(k) + c - pv;
                pv = c;
            }
            if (!ok) {
                const float den = 2.f * (fc - fcur + dec * alpha);
                const float an = den > 0.f ? dec * alpha * alpha / den : 0.5f * alpha;
                alpha_try = fminf(fmaxf(an, 0.1f * alpha), 0.5f * alpha);
                prev_unclipped = false;
                if (++nfail > kMaxBacktracks) { active = false; flags = kInfoStalled | kInfoPlain; }
            }
        }
        if (ok && active) {
            fcur = fc;
            prev_unclipped = (alpha == 1.f) && !clipped;
            alpha_try = 1.f;
            nfail = 0;
            if (!changed) {
                active = false;
                flags = kInfoStalled | ((alpha == 1.f && (!vio || polish)) ? 0 : kInfoPlain);
            }
        }
    }
    __device__ __forceinline__ void solve(bool valid)
    {
        alpha_try = 1.f; steps = 0; flags = 0; nfail = 0;
        active = valid; prev_unclipped = false;
        bool vio;
        float dec;
        bool done = look(0, vio, dec);
        for (int it = 0; !done; ++it) {
            step(vio, dec);
            done = look(it + 1, vio, dec);
        }
    }

    // Primal recovery: between two bound duals every sample takes the mean of the block's x.  The running
    // mean of a block needs no count: behind j free duals it takes 1 / (j + 1) of the new sample, and the
    // pivot in G is j / (j + 1) (0 where a block begins, whose first sample is then taken as it is).  It is kept
    // as its distance from the sample, off: x is constant on a block up to rounding, so those distances are
    // exact and small, and the mean is rounded once.
    // (Instead of the value of one sample: planes of 32 x 32, N(0, 1), K = 3, error against 64 bits 3.1e-7 ->
    // 9e-8.  A running mean that is rounded at every sample, two instructions a sample less, is 8-30 % further
    // off on rows of a few long blocks.)
    __device__ __forceinline__ void recover(float (&xs)[C])
    {
        // (made opaque: the differences below are those of the last look, and the compiler would keep them, C
        // more registers, through everything in between)
#pragma unroll
        for (int k = 0; k < C; ++k) asm volatile("" : "+v"(X[k]));
        float off = 0.f;
        xs[0] = X[0];
#pragma unroll
        for (int k = 1; k < C; ++k) {
            off = G[k - 1] * (off + (X[k - 1] - X[k]));
            xs[k] = X[k] + off;
        }
        // the block around the middle: both lanes form the mean of its parts from the left lane's side
        float mean;
        {
            const float part = C > 1 ? 1.f - G[C - 2] : 1.f;            // 1 / samples of the lane's part
            const float xl = pair_left(X[C - 1]), ol = pair_left(off), pl = pair_left(part);
            const float xr = pair_right(X[C - 1]), orr = pair_right(off), pr = pair_right(part);
            const float apart = (xr - xl) + (orr - ol);
            const float both = xl + fmaf(apart, pl * __builtin_amdgcn_rcpf(pl + pr), ol);
            mean = G[C - 1] == 0.f ? xs[C - 1] : both;
        }
        xs[C - 1] = mean;
#pragma unroll
        for (int k = C - 2; k >= 0; --k) {
            mean = (G[k] == 0.f) ? xs[k] : mean;
            xs[k] = mean;
        }
        const bool plain = (flags & (kInfoCapped | kInfoPlain)) != 0;
        if (__any(plain)) {
#pragma unroll
            for (int k = 0; k < C; ++k) xs[k] = plain ? X[k] : xs[k];
        }
    }
};

// Segment code (FwdParams::seg) of a pair's row of n samples, in both lanes; right: this is the right lane.
template <int C, bool FULL>
__device__ __forceinline__ uint2 pair_segment_code(const float (&xs)[C], int n, bool right)
{
    // bit i: local dual i (the middle one counts in both lanes); rises: x increases behind that dual, seen from the lane's end
    uint32_t jm = 0, rises = 0;
    {
        const float d = xs[C - 1] - pair_other(xs[C - 1]);
        rises = __float_as_uint(d) >> 31;
        jm = __float_as_uint(0.0f - fabsf(d)) >> 31;
    }
#pragma unroll
    for (int k = C - 2; k >= 0; --k) {
        const float d = xs[k] - xs[k + 1];
        rises = __builtin_amdgcn_alignbit(rises, __float_as_uint(d), 31);
        jm = __builtin_amdgcn_alignbit(jm, __float_as_uint(0.0f - fabsf(d)), 31);
    }
    // local dual i of the right lane is dual 2C-2-i of the row, and there the row rises where the lane falls
    const uint32_t turned_jm = __builtin_bitreverse32(jm) >> (33 - 2 * C);
    const uint32_t turned_up = __builtin_bitreverse32(jm & ~rises) >> (33 - 2 * C);
    jm = right ? turned_jm : jm;
    rises = right ? turned_up : rises;
    jm |= pair_other(jm);
    rises |= pair_other(rises);
    if (!FULL) {
        const uint32_t in = n > 1 ? (0xffffffffu >> (33 - n)) : 0u;
        jm &= in; rises &= in;
    }
    return make_uint2(jm, rises);
}

// The half of a pair's row mask (tv_small2d.hpp) that the lane leaves: the left lane the jumps, the right one the rises.
// From the signs of differences, as in pair_segment_code, which say nothing next to an infinity or NaN: where a wave
// has one, its masks come from the comparisons that readers of pass outputs make.  (From comparisons alone:
// 1024 planes of 64 x 64, K = 4, forward, 131.7 -> 137.6 us.)
template <int C, bool FULL>
__device__ __forceinline__ uint2 pair_row_mask(const float (&xs)[C], int n, bool right)
{
    uint32_t jump, rises;                       // local duals, as in pair_segment_code
    const float across = pair_other(xs[C - 1]);
    float before = xs[C - 1] - across, check = 0.f;     // check: finite where every difference is, and not huge
    rises = __float_as_uint(before) >> 31;
    jump = __float_as_uint(0.0f - fabsf(before)) >> 31;
#pragma unroll
    for (int k = C - 2; k >= 0; --k) {
        const float d = xs[k] - xs[k + 1];
        rises = __builtin_amdgcn_alignbit(rises, __float_as_uint(d), 31);
        jump = __builtin_amdgcn_alignbit(jump, __float_as_uint(0.0f - fabsf(d)), 31);
        if (k % 2 == 0) check = fmaf(d, before, check);
        before = d;
    }
    if (__any(!(fabsf(check) < INFINITY))) {
        rises = across > xs[C - 1] ? 1u : 0u;
        jump = across != xs[C - 1] ? 1u : 0u;
#pragma unroll
        for (int k = C - 2; k >= 0; --k) {
            rises = rises << 1 | ((right ? !(xs[k] > xs[k + 1]) : xs[k + 1] > xs[k]) ? 1u : 0u);
            jump = jump << 1 | (xs[k + 1] != xs[k] ? 1u : 0u);
        }
    }
    // left: duals 0 .. C-1 as they are.  Right: its duals 0 .. C-2 are 2C-2 .. C of the row, which rises where the lane falls
    const uint32_t turned_jump = __builtin_bitreverse32(jump) >> (33 - C);
    const uint32_t turned_rises = __builtin_bitreverse32(jump & ~rises) >> (33 - C);
    jump = right ? turned_jump : jump;
    rises = right ? turned_rises : rises;
    const uint32_t other = pair_other(right ? jump : rises);
    uint64_t mask = right ? other | (uint64_t)rises << C : jump | (uint64_t)other << C;
    if (!FULL) mask &= (1ull << (n - 1)) - 1ull;
    return make_uint2((uint32_t)mask, (uint32_t)(mask >> 32));
}

// The tile in LDS: samples 0 .. C-1 of a row in order, the others from the row's end, HALF places on, so
// that either lane of a pair finds its half at offsets known at compile time.  With HALF = 16 the 16 rows
// that half a wave works on cover 16 banks, and their other halves the other 16.  (HALF = 32: two by two
// the same; the tile is crossed twice a pass, the solve in between reads lane-private columns.)
template <int C>
struct PairTile {
    static constexpr int HALF = C <= 16 ? 16 : 32, PITCH = 2 * HALF + 1;
    static_assert(C >= 2 && C <= 32, "rows of at most 64 samples");
    __device__ static __forceinline__ int place(int k) { return k < C ? k : HALF + 2 * C - 1 - k; }
    // step between neighbouring samples from sample k on (groups of four that the middle does not split)
    __device__ static __forceinline__ int step(int k) { return k < C ? 1 : -1; }
};

// gtab: pivots j / (j + 1) of a free run, from memory (a division a wave is 2 % of a short solve)
struct PairPivots {
    float g[34];
    constexpr PairPivots() : g()
    {
        for (int j = 0; j < 34; ++j) g[j] = (float)j / (float)(j + 1);
    }
};
static __device__ const PairPivots pair_pivots;
template <int C>
__device__ __forceinline__ void pair_fill_table(float *gtab, int tid)
{
    static_assert(C < 34, "");
    if (tid <= C) gtab[tid] = pair_pivots.g[tid];
}

// Which of a lane's samples exist in a row of n (bit i: local sample i), the local index of the dual
// behind the row's last sample, and the duals inside the row (PairSolver::live).
template <int C>
__device__ __forceinline__ uint32_t pair_samples(int n, bool right)
{
    const int pads = 2 * C - n;                 // (the right lane's from its end, then the left lane's from the middle)
    if (right) return pads < C ? ~0u << pads : 0u;
    return n < C ? (1u << n) - 1u : ~0u;
}
template <int C>
__device__ __forceinline__ int pair_cut(int n, bool right) { return right ? 2 * C - 1 - n : n - 1; }
__device__ __forceinline__ uint32_t pair_live(int cut, bool right)
{
    if (right) return cut < 31 ? ~0u << (cut + 1) : 0u;
    return cut < 32 ? (1u << cut) - 1u : ~0u;
}

// ---------------------------------------------------------------------------------
// Forward: K sweeps of paper Alg. 1 in one launch, a plane of at most 2C x 2C per wave (C <= 16) or per
// workgroup of two waves.
//
// A row pass gives a pair of lanes a row of the plane, a column pass a column.  The plane changes hands
// between passes through one LDS tile, whose rows and columns both lie as PairTile has them.  As in
// tv2d_fwd_small_kernel the tile also parks the solver's input, and the correction term that is not in
// use lives in a lane-private LDS column.  Planes of at most 32 x 32 leave segment codes for the reverse
// sweep, larger ones row masks (1024 planes of 64 x 64, K = 4, forward + reverse sweep 184 -> 173 us,
// 2000 of 47 x 47, K = 3, 312 -> 260) or, where those are asked for, their pass outputs.
// Registers: four waves a SIMD up to 32 x 32 (a fifth, at 96 registers, spills and is 10 % slower), two beyond,
// where LDS holds no more (33 KB a plane).
// ---------------------------------------------------------------------------------
template <int C, int PADS, bool IO16 = false>
__global__ __launch_bounds__(C > 16 ? 128 : 64, C > 16 ? 2 : 4) void tv2d_fwd_pair_kernel(Small2dFwdParams p)
{
    using Tile = PairTile<C>;
    constexpr bool FULL = PADS == 0;
    constexpr int HO = Tile::HALF, P = Tile::PITCH, S = 2 * C, NT = 4 * HO;
    static_assert(!IO16 || C <= 16, "bf16 storage: planes of at most 32 x 32");
    __shared__ float T1[2 * HO * P], T2[NT * C], gtab[C + 2];
    static_assert(NT * C <= 2 * HO * P, "the parked input fits the tile");
    const int tid = threadIdx.x;
    pair_fill_table<C>(gtab, tid);
    const int H = FULL ? S : p.H, W = FULL ? S : p.W, HW = H * W;
    const int64_t plane = blockIdx.x;
    const float lam = fmaxf(p.lam[plane % p.lam_count], 0.f);
    auto sync = []() { if (C > 16) __syncthreads(); else wave_lds_sync(); };

    auto place = [](int k) { return Tile::place(k); };          // of row or column k in the tile
    const int at = tid >> 1;                        // the pair's row or column, by place
    const bool right = (tid & 1) != 0;
    const int idx = at < HO ? at : HO + S - 1 - at;
    const bool in_half = (at & (HO - 1)) < C;
    float *by_row = T1 + at * P + (right ? HO : 0);             // step 1
    float *by_col = T1 + (right ? HO : 0) * P + at;             // step P
    float *park = T1 + tid, *mine = T2 + tid;                   // step NT

    // memory <-> tile: sample e = tid, tid + NT, ... of the plane
    auto each_sample = [&](auto &&f) {
        int r = tid / W, c = tid - r * W;
        const int dq = NT / W, dr = NT - dq * W;
        for (int e = tid; e < HW; e += NT) {
            f(e, T1 + place(r) * P + place(c));
            r += dq; c += dr;
            if (c >= W) { c -= W; r += 1; }
        }
    };
    auto plane_in = [&](auto &&load) {
        constexpr int N = (S * S + NT - 1) / NT;
        float q[N];                                 // every load is issued before the first is waited for
#pragma unroll
        for (int i = 0; i < N; ++i) q[i] = i * NT + tid < HW ? load(i * NT + tid) : 0.f;
        int r = tid / W, c = tid - r * W;
        const int dq = NT / W, dr = NT - dq * W;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if (i * NT + tid < HW) T1[place(r) * P + place(c)] = q[i];
            r += dq; c += dr;
            if (c >= W) { c -= W; r += 1; }
        }
    };
    // four samples of a row from sample e of the plane on, e a multiple of 4
    auto four = [&](int e) { return T1 + place(e / S) * P + place(e % S); };
    constexpr bool QUADS = FULL && C == HO;
    constexpr int N4 = S * S / 4 / NT;
    if constexpr (IO16) {
        const uint16_t *src = reinterpret_cast<const uint16_t *>(p.y) + plane * HW;
        plane_in([&](int e) { return bf16_bits_to_f32(src[e]); });
    } else {
        const float *src = p.y + plane * HW;
        if (QUADS && ((uintptr_t)src % 16) == 0) {
            float4 q[N4];
#pragma unroll
            for (int i = 0; i < N4; ++i) q[i] = load16(src + (i * NT + tid) * 4, p.stream != 0);
#pragma unroll
            for (int i = 0; i < N4; ++i) {
                const int e = (i * NT + tid) * 4;
                float *d = four(e);
                const int s = Tile::step(e % S);
                d[0] = q[i].x; d[s] = q[i].y; d[2 * s] = q[i].z; d[3 * s] = q[i].w;
            }
        } else {
            plane_in([&](int e) { return src[e]; });
        }
    }
    auto put_plane = [&](float *dst) {
        if (QUADS && ((uintptr_t)dst % 16) == 0) {
            int own = tid;
            asm volatile("" : "+v"(own));           // (addresses formed here, not kept through the solves)
#pragma unroll
            for (int i = 0; i < N4; ++i) {
                const int e = (i * NT + own) * 4;
                const float *d = four(e);
                const int s = Tile::step(e % S);
                store16(dst + e, make_float4(d[0], d[s], d[2 * s], d[3 * s]), p.stream != 0);
            }
        } else {
            each_sample([&](int e, const float *d) { dst[e] = *d; });
        }
    };
    sync();

    auto samples = [&](int n) -> uint32_t { return FULL ? ~0u : pair_samples<C>(n, right); };
    auto masked = [](float v, uint32_t have, int k) { return pair_masked<PADS>(v, have, k); };

    float v[C], u0[C];                              // a pass's input, and the dual it starts from
    bool valid = in_half && (FULL || idx < H);      // first pass: rows, of W samples
    int n = W;
    uint32_t have = samples(n);
#pragma unroll
    for (int k = 0; k < C; ++k) { v[k] = masked(by_row[k], have, k); u0[k] = 0.f; }

    const int n_pass = 2 * p.sweeps;
    for (int i = 0; i < n_pass; ++i) {
        const bool col = (i & 1) != 0;
        sync();                            // every lane has taken its input out of the tile
#pragma unroll
        for (int k = 0; k < C; ++k) park[k * NT] = v[k];
        sync();

        PairSolver<C, PADS, NT> sv;
        float xs[C];
        sv.yl = park; sv.gtab = gtab; sv.lam = lam;
        if constexpr (!FULL) {
            sv.cut = pair_cut<C>(n, right);
            sv.live = pair_live(sv.cut, right);
        }
        if (i < 2) sv.start(v, __builtin_amdgcn_rcpf((float)n), have);
        else {
#pragma unroll
            for (int k = 0; k < C; ++k) sv.u[k] = u0[k];
            sv.start_warm(v);
        }
        sv.solve(valid);
        sv.recover(xs);

        if constexpr (C <= 16) {
            const uint2 code = pair_segment_code<C, FULL>(xs, n, right);
            if (valid) {
                uint32_t *to = reinterpret_cast<uint32_t *>(p.codes + (size_t)i * p.code_stride + (size_t)plane * (col ? W : H) + idx);
                to[right ? 1 : 0] = right ? code.y : code.x;
            }
        } else if (p.codes) {
            const uint2 mask = pair_row_mask<C, FULL>(xs, n, right);
            if (valid) p.codes[(size_t)i * p.code_stride + ((size_t)plane * (col ? W : H) + idx) * 2 + (right ? 1 : 0)] = mask;
        }

        const bool keep = i + 2 < n_pass;
        float corr[C];
#pragma unroll
        for (int k = 0; k < C; ++k) corr[k] = park[k * NT] - xs[k];
        sync();
        if (col) {
#pragma unroll
            for (int k = 0; k < C; ++k) by_col[k * P] = xs[k];
        } else {
#pragma unroll
            for (int k = 0; k < C; ++k) by_row[k] = xs[k];
        }
        sync();
        if (C > 16 ? p.codes == nullptr : p.keep_passes != 0u) put_plane(p.saved + (size_t)i * p.saved_stride + plane * HW);
        // input of the next pass: this output seen the other way plus that direction's correction
        // term, whose negated running sum is the dual to start from
        valid = in_half && (FULL || idx < (col ? H : W));
        n = col ? W : H;
        have = samples(n);
        float t[C];
        if (col) {
#pragma unroll
            for (int k = 0; k < C; ++k) t[k] = masked(by_row[k], have, k);
        } else {
#pragma unroll
            for (int k = 0; k < C; ++k) t[k] = masked(by_col[k * P], have, k);
        }
        if (i >= 1) {
            float run = 0.f;
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const float c = mine[k * NT];
                t[k] += c;
                run -= c;
                u0[k] = run;
            }
        } else {
#pragma unroll
            for (int k = 0; k < C; ++k) u0[k] = 0.f;
        }
        if (keep) {
#pragma unroll
            for (int k = 0; k < C; ++k) mine[k * NT] = corr[k];
        }
#pragma unroll
        for (int k = 0; k < C; ++k) v[k] = t[k];
    }
    if constexpr (IO16) {
        uint16_t *dst = reinterpret_cast<uint16_t *>(p.x) + plane * HW;
        each_sample([&](int e, const float *d) { dst[e] = f32_to_bf16_bits(*d); });
    } else {
        put_plane(p.x + plane * HW);
    }
    if (C > 16 && p.tag && blockIdx.x == 0 && tid == 0) *p.tag = p.codes ? 1u : 0u;
}

// ---------------------------------------------------------------------------------
// Forward on a batch of rows, 32 to a wave: plain calls (input y, output x, optionally info words and
// segment codes).  Grid and tiles: TileMap with tiles of 32 rows.
// MODE: how the rows lie in memory.  kPairPacked: row r starts n r samples after the base; a wave's rows are
// moved through the tile as one block.  kPairPacked4: the same for multiples of 8 samples, 16-byte aligned,
// whose rows start on a quarter of the banks or less: the tile has the rows by place (rows of 56, most of them
// done at once, 103 -> 79 us).  kPairPlane: the rows are the columns of contiguous 32 x 32
// planes, a plane a wave.  kPairStrided: anything else, read and written sample by sample.  (PADS < C:
// n > 2C - 1 - PADS.)
// IO16: y and x are bf16 (packed rows of 32).
// ---------------------------------------------------------------------------------
constexpr int kPairStrided = 0, kPairPacked = 1, kPairPlane = 2, kPairPacked4 = 3;

template <int C, int PADS, int MODE, bool IO16 = false>
__global__ __launch_bounds__(64, C > 16 ? 3 : 4) void tv1d_fwd_pair_kernel(FwdParams p)
{
    using Tile = PairTile<C>;
    constexpr int P = Tile::PITCH, HO = Tile::HALF;
    constexpr bool FULL = PADS == 0;
    constexpr bool WHOLE = FULL && C == 16;         // rows of exactly 32
    static_assert(MODE != kPairPlane || WHOLE, "plane columns: 32 x 32 planes");
    static_assert(!IO16 || (WHOLE && MODE == kPairPacked4), "bf16 storage: packed rows of 32");
    static_assert(MODE != kPairPacked4 || (FULL && C % 4 == 0), "the middle splits no group of four");
    __shared__ __align__(16) float tile[MODE == kPairStrided ? 64 * C : 32 * P];
    __shared__ float gtab[C + 2];
    const int lane = threadIdx.x;
    pair_fill_table<C>(gtab, lane);
    // (the row pass of a 2D call with one sweep on sides of 33-64: this route leaves no masks)
    if (C > 16 && p.codes_tag && blockIdx.x == 0 && blockIdx.y == 0 && lane == 0) *p.codes_tag = 0u;

    const uint32_t slot = p.order ? min(p.order[blockIdx.y], gridDim.y - 1u) : blockIdx.y;
    const uint32_t r0 = p.tm.first<32>(__builtin_amdgcn_readfirstlane(blockIdx.x), slot);
    const int at = lane >> 1;
    const bool right = (lane & 1) != 0;
    // (plane columns lie in the tile by place, like the planes' rows)
    const uint32_t row = p.tm.row(r0, (uint32_t)(MODE == kPairPlane ? PairTile<16>::place(at) : at));
    const bool valid = row < p.L.n_rows;
    const int n = FULL ? 2 * C : p.L.n;
    float lam = 0.f;
    if (p.tm.grouped) lam = fmaxf(p.lam[slot], 0.f);            // one slot per tile
    else if (valid) lam = load_lambda(p.lam, p.L, row);
    const uint32_t have = FULL ? ~0u : pair_samples<C>(n, right);
    const bool stream = p.L.stream != 0;

    // the lane's samples in the tile (kPairPacked: the right lane's backwards from place 2C - 1 of its row)
    float *half = MODE == kPairPlane    ? tile + (right ? HO * P : 0) + at
                  : MODE == kPairPacked ? tile + at * n + (right ? 2 * C - 1 : 0)
                                        : tile + at * P + (right ? HO : 0);
    const int half_step = MODE == kPairPlane ? P : (MODE == kPairPacked && right ? -1 : 1);
    float *park = tile + lane;

    // kPairPacked4: four samples at a time, group c of the wave's row r.  (Past the last group, and past the
    // last row, the last one again: nothing is read out of bounds, and a tile entry gets the same value twice.)
    auto move_fours = [&](auto &&f) {
        int own = lane;
        asm volatile("" : "+v"(own));               // (addresses formed here, not kept through the solve)
        const int per = n / 4;                      // groups a row
        int r = own / per, c = own - r * per;
        const int dq = 64 / per, dr = 64 - dq * per;
#pragma unroll
        for (int i = 0; i < (C + 3) / 4; ++i) {     // (32 rows of at most 2C samples)
            const int rr = min(r, 31);
            const uint32_t g = min(p.tm.row(r0, (uint32_t)rr), p.L.n_rows - 1u);
            f(i, (size_t)g * n + c * 4, rr, c * 4);
            r += dq; c += dr;
            if (c >= per) { c -= per; r += 1; }
        }
    };
    const bool all_there = p.tm.row(r0, 31u) < p.L.n_rows;
    // (rows of 32 or 64: an access of the wave covers RP whole rows, which lie together where a lambda's rows do)
    constexpr int RP = 128 / C, LR = C / 2;         // rows an access, lanes a row
    const bool whole_rows = FULL && (C == 16 || C == 32) && all_there && (1u << p.tm.lg) >= (uint32_t)RP;
    auto rows_at = [&](int i) { return (size_t)__builtin_amdgcn_readfirstlane(p.tm.row(r0, (uint32_t)(i * RP))) * (2 * C); };
    // kPairPacked: the wave's rows lie in the tile as in memory, one block of samples
    const int total = MODE == kPairPacked ? (int)min(32u, p.L.n_rows - r0) * n : 0;
    const bool aligned = MODE == kPairPacked && all_there && ((uintptr_t)p.y | (uintptr_t)p.x) % 16 == 0;
    auto put4 = [&](int r, int c, const float4 &q) {
        float *d = tile + r * P + Tile::place(c);
        const int s = Tile::step(c);
        d[0] = q.x; d[s] = q.y; d[2 * s] = q.z; d[3 * s] = q.w;
    };
    auto get4 = [&](int r, int c) {
        const float *d = tile + r * P + Tile::place(c);
        const int s = Tile::step(c);
        return make_float4(d[0], d[s], d[2 * s], d[3 * s]);
    };
    // plane columns: the plane's samples 4 (i * 64 + lane) ..
    const int64_t plane_at = MODE == kPairPlane ? (int64_t)(r0 >> 5) * p.L.outer_stride : 0;
    const bool plane_there = MODE == kPairPlane && r0 < p.L.n_rows;
    const int64_t off = MODE == kPairStrided && valid ? row_offset(p.L, row) + (right ? (int64_t)(2 * C - 1) * p.L.elem_stride : 0) : 0;
    const int64_t step = right ? -p.L.elem_stride : p.L.elem_stride;

    float y[C];
    if constexpr (MODE == kPairStrided) {
#pragma unroll
        for (int k = 0; k < C; ++k) y[k] = valid && ((have >> k) & 1u) ? p.y[off + k * step] : 0.f;
    } else {
        if constexpr (MODE == kPairPlane) {
            float4 q[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                q[i] = plane_there ? load16(p.y + plane_at + (i * 64 + lane) * 4, stream) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = (i * 64 + lane) * 4;
                put4(PairTile<16>::place(e >> 5), e & 31, q[i]);
            }
        } else if constexpr (IO16) {
            const uint16_t *src = reinterpret_cast<const uint16_t *>(p.y);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int e = (i * 64 + lane) * 8;
                const uint32_t g = p.tm.row(r0, (uint32_t)e >> 5);
                if (g >= p.L.n_rows) continue;
                const float4 q = load16(reinterpret_cast<const float *>(src + (size_t)g * 32 + (e & 31)), stream);
                const uint32_t w[4] = {__float_as_uint(q.x), __float_as_uint(q.y), __float_as_uint(q.z), __float_as_uint(q.w)};
                float *d = tile + (e >> 5) * P + Tile::place(e & 31);
                const int s = Tile::step(e & 31);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    d[2 * j * s] = __uint_as_float(w[j] << 16);
                    d[(2 * j + 1) * s] = __uint_as_float(w[j] & 0xffff0000u);
                }
            }
        } else if constexpr (MODE == kPairPacked4) {
            float4 q[(C + 3) / 4];                  // (every load is issued before the first is waited for)
            if (whole_rows) {
#pragma unroll
                for (int i = 0; i < C / 4; ++i) q[i] = load16(p.y + rows_at(i) + lane * 4, stream);
#pragma unroll
                for (int i = 0; i < C / 4; ++i) put4(i * RP + lane / LR, lane % LR * 4, q[i]);
            } else {
                move_fours([&](int i, size_t a, int, int) { q[i] = load16(p.y + a, stream); });
                move_fours([&](int i, size_t, int r, int c) { put4(r, c, q[i]); });
            }
        } else {
            const float *blk = p.y + (size_t)r0 * n;
            if (aligned) {
                float4 q[(C + 3) / 4];
#pragma unroll
                for (int i = 0; i < (C + 3) / 4; ++i) {
                    const int e = (i * 64 + lane) * 4;
                    q[i] = e < total ? load16(blk + e, stream) : make_float4(0.f, 0.f, 0.f, 0.f);
                }
#pragma unroll
                for (int i = 0; i < (C + 3) / 4; ++i) {
                    const int e = (i * 64 + lane) * 4;
                    if (e < total) *reinterpret_cast<float4 *>(tile + e) = q[i];
                }
            } else {
#pragma unroll 4
                for (int e = lane; e < total; e += 64) tile[e] = blk[e];
            }
        }
        wave_lds_sync();
#pragma unroll
        for (int k = 0; k < C; ++k) y[k] = pair_masked<PADS>(half[k * half_step], have, k);
        if (!valid) {                               // (its part of the tile was not written)
#pragma unroll
            for (int k = 0; k < C; ++k) y[k] = 0.f;
        }
        wave_lds_sync();
    }
#pragma unroll
    for (int k = 0; k < C; ++k) park[k * 64] = y[k];
    wave_lds_sync();

    PairSolver<C, PADS> sv;
    sv.yl = park; sv.gtab = gtab; sv.lam = lam;
    if constexpr (!FULL) {
        sv.cut = pair_cut<C>(n, right);
        sv.live = pair_live(sv.cut, right);
    }
    sv.start(y, __builtin_amdgcn_rcpf((float)n), have);
    sv.solve(valid);
    float xs[C];
    sv.recover(xs);

    if (p.info && valid && !right) p.info[row] = sv.steps | sv.flags;
    if constexpr (C <= 16) if (p.seg) {
        const uint2 code = pair_segment_code<C, FULL>(xs, n, right);
        if (valid) reinterpret_cast<uint32_t *>(p.seg + row)[right ? 1 : 0] = right ? code.y : code.x;
    }
    if constexpr (MODE == kPairStrided) {
#pragma unroll
        for (int k = 0; k < C; ++k)
            if (valid && ((have >> k) & 1u)) p.x[off + k * step] = xs[k];
        return;
    }
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < C; ++k)
        if (MODE != kPairPacked || k >= PADS || ((have >> k) & 1u)) half[k * half_step] = xs[k];
    wave_lds_sync();
    if constexpr (MODE == kPairPlane) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int own = lane;
            asm volatile("" : "+v"(own));
            const int e = (i * 64 + own) * 4;
            const float4 q = get4(PairTile<16>::place(e >> 5), e & 31);
            if (plane_there) store16(p.x + plane_at + e, q, stream);
        }
    } else if constexpr (IO16) {
        uint16_t *dst = reinterpret_cast<uint16_t *>(p.x);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int e = (i * 64 + lane) * 8;
            const uint32_t g = p.tm.row(r0, (uint32_t)e >> 5);
            if (g >= p.L.n_rows) continue;
            const float *d = tile + (e >> 5) * P + Tile::place(e & 31);
            const int s = Tile::step(e & 31);
            uint32_t w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = f32x2_to_bf16x2(d[2 * j * s], d[(2 * j + 1) * s]);
            store16(reinterpret_cast<float *>(dst + (size_t)g * 32 + (e & 31)),
                    make_float4(__uint_as_float(w[0]), __uint_as_float(w[1]), __uint_as_float(w[2]), __uint_as_float(w[3])), stream);
        }
    } else if constexpr (MODE == kPairPacked4) {
        if (whole_rows) {
            int own = lane;
            asm volatile("" : "+v"(own));
#pragma unroll
            for (int i = 0; i < C / 4; ++i)
                store16(p.x + rows_at(i) + own * 4, get4(i * RP + own / LR, own % LR * 4), stream);
        } else if (all_there) move_fours([&](int, size_t a, int r, int c) { store16(p.x + a, get4(r, c), stream); });
        else move_fours([&](int, size_t a, int r, int c) {
            if (p.tm.row(r0, (uint32_t)r) < p.L.n_rows) store16(p.x + a, get4(r, c), stream);
        });
    } else {
        float *blk = p.x + (size_t)r0 * n;
        int own = lane;
        asm volatile("" : "+v"(own));
        if (aligned) {
#pragma unroll
            for (int i = 0; i < (C + 3) / 4; ++i) {
                const int e = (i * 64 + own) * 4;
                if (e < total) store16(blk + e, *reinterpret_cast<const float4 *>(tile + e), stream);
            }
        } else {
            for (int e = own; e < total; e += 64) blk[e] = tile[e];
        }
    }
}

// ---------------------------------------------------------------------------------
// Reverse sweep on planes of 33-64 samples a side in one launch, two lanes a row, two waves a plane.
//
// Bound by the chains of its segment sums: with a row per lane a plane is one wave, 1024 planes are one wave
// per SIMD, and each walks 64 samples twice a pass (VALU busy a third of the time).  Halves make twice the
// waves and chains of 32.  Both adjoint state tensors of the plane lie in LDS as PairTile has them; of
// a pass's output a lane reads its half row one pass ahead, rows in 16-byte pieces, columns in rows of 32
// neighbouring columns, and keeps a jump and a direction bit a sample.
// Row masks in place of pass outputs (p.tag): 1024 planes of 64 x 64, K = 4, with the lambda sum 48 -> 38 us.
// Reverse sweep of 1024 planes of 64 x 64, K = 4, a row per lane / two lanes: 69 / 48 us, 8192 planes, K = 2: 290 / 180;
// 1024 planes of 40 x 40, K = 4, a plane per workgroup / two lanes: 56 / 31.
// At most 2C / 5 samples short of 2C.
// MASKS: the workspace may hold row masks.  QUADS: rows of a multiple of four samples, read in 16-byte pieces from pass outputs.
// (A kernel for every case: with both ways of reading rows in one, 6000 planes of 32 x 40, K = 4, take 12 % longer,
// 4200 of 60 x 60, K = 1, 18 %.)
// ---------------------------------------------------------------------------------
template <int C, bool FULL, bool QUADS, bool MASKS>
__global__ __launch_bounds__(128, 2) void tv2d_bwd_pair_kernel(Small2dBwdParams p)
{
    static_assert(C > 16 && C <= 32 && C % 4 == 0, "planes of 33-64 samples a side");
    static_assert(QUADS || !FULL, "2C is a multiple of four");
    using Tile = PairTile<C>;
    constexpr int HO = Tile::HALF, P = Tile::PITCH, S = 2 * C, NT = 4 * HO;
    __shared__ float A[2 * HO * P], B[2 * HO * P], rtab[S + 2], wave_term[2];
    const int tid = threadIdx.x;
    for (int i = tid; i <= S; i += NT) rtab[i] = i > 0 ? 1.0f / (float)i : 0.0f;
    const int H = FULL ? S : p.H, W = FULL ? S : p.W, HW = H * W;
    const int64_t plane = blockIdx.x;
    const int at = tid >> 1;                        // the pair's row or column, by place
    const bool right = (tid & 1) != 0;
    const int idx = at < HO ? at : HO + S - 1 - at;
    const bool in_half = (at & (HO - 1)) < C;
    const bool cvalid = in_half && (FULL || idx < W), rvalid = in_half && (FULL || idx < H);
    const int row_at = at * P + (right ? HO : 0);               // half row in a tile, step 1
    const int col_at = (right ? HO : 0) * P + at;               // half column, step P

    // memory <-> tile: sample e = tid, tid + NT, ... of the plane
    auto each_sample = [&](auto &&f) {
        int r = tid / W, c = tid - r * W;
        const int dq = NT / W, dr = NT - dq * W;
        for (int e = tid; e < HW; e += NT) {
            f(e, Tile::place(r) * P + Tile::place(c));
            r += dq; c += dr;
            if (c >= W) { c -= W; r += 1; }
        }
    };
    {
        const float *src = p.g_up + plane * HW;
        constexpr int N = (S * S + NT - 1) / NT;
        float q[N];                                 // every load is issued before the first is waited for
#pragma unroll
        for (int i = 0; i < N; ++i) q[i] = i * NT + tid < HW ? src[i * NT + tid] : 0.f;
        int r = tid / W, c = tid - r * W;
        const int dq = NT / W, dr = NT - dq * W;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if (i * NT + tid < HW) A[Tile::place(r) * P + Tile::place(c)] = q[i];
            r += dq; c += dr;
            if (c >= W) { c -= W; r += 1; }
        }
    }

    // The lane's half of its row or column of a pass's output, in the order of memory: samples 0 .. C-1, or
    // C .. n-1 and beyond (lanes without a row, and samples past the end, read inside the plane all the same:
    // no branch a load).
    const int row_in = FULL ? idx : min(idx, H - 1), col_in = FULL ? idx : min(idx, W - 1);
    // Or, where the forward call left row masks, the row's mask.
    const bool coded = MASKS && *p.tag == 1u;
    uint4 mask = make_uint4(0u, 0u, 0u, 0u);
    auto fetch = [&](int pass, float (&xv)[C]) {
        if (pass < 0) return;
        if (coded) {
            const size_t row = (size_t)plane * ((pass & 1) ? W : H) + ((pass & 1) ? col_in : row_in);
            mask = *reinterpret_cast<const uint4 *>(p.codes + (size_t)pass * p.code_stride + row * 2);
            return;
        }
        const float *xs = p.saved + (size_t)pass * p.saved_stride + (size_t)plane * HW;
        if (pass & 1) {
            const int r0 = right ? C : 0;
#pragma unroll
            for (int r = 0; r < C; ++r) xv[r] = xs[(FULL ? r0 + r : min(r0 + r, H - 1)) * W + col_in];
        } else {
            const int c0 = right ? C : 0;
            const float *from = xs + row_in * W;
            if constexpr (QUADS) {
#pragma unroll
                for (int c = 0; c < C; c += 4) {
                    const float4 q = *reinterpret_cast<const float4 *>(from + (FULL ? c0 + c : min(c0 + c, W - 4)));
                    xv[c] = q.x; xv[c + 1] = q.y; xv[c + 2] = q.z; xv[c + 3] = q.w;
                }
            } else {
#pragma unroll
                for (int c = 0; c < C; ++c) xv[c] = from[min(c0 + c, W - 1)];
            }
        }
    };
    // Jump and direction bits of the lane's local duals: bit i behind local sample i, towards the middle; up: x rises there,
    // seen from the lane's end.  The sign of x[k] - x[k+1] says "rises", that of -|.| "differs".
    auto bits_of = [&](const float (&xv)[C], uint32_t &jump, uint32_t &up) {
        if (coded) {
            const uint64_t j = mask64(mask.x, mask.y), u = mask64(mask.z, mask.w);
            const uint32_t middle = (uint32_t)(j >> (C - 1)) & 1u;
            const uint32_t rj = (uint32_t)(j >> C), ru = (uint32_t)(u >> C);
            constexpr uint32_t half = C == 32 ? ~0u : (1u << (C & 31)) - 1u;
            jump = right ? __builtin_bitreverse32(rj) >> (33 - C) | middle << (C - 1) : (uint32_t)j & half;
            up = right ? __builtin_bitreverse32(rj & ~ru) >> (33 - C) : (uint32_t)u & half;
            return;
        }
        jump = 0; up = 0;
#pragma unroll
        for (int k = C - 2; k >= 0; --k) {
            const float d = xv[k] - xv[k + 1];
            up = __builtin_amdgcn_alignbit(up, __float_as_uint(d), 31);
            jump = __builtin_amdgcn_alignbit(jump, __float_as_uint(0.0f - fabsf(d)), 31);
        }
        // (the right lane's duals the other way round: C - 1 bits turned; there x rises where it falls in memory)
        const uint32_t turned_jump = __builtin_bitreverse32(jump) >> (33 - C);
        const uint32_t turned_up = __builtin_bitreverse32(jump & ~up) >> (33 - C);
        jump = right ? turned_jump : jump;
        up = right ? turned_up : up;
        const float near = right ? xv[0] : xv[C - 1];           // the sample at the middle
        const float d = near - pair_other(near);
        up |= (__float_as_uint(d) >> 31) << (C - 1);
        jump |= (__float_as_uint(0.0f - fabsf(d)) >> 31) << (C - 1);
    };
    // Segment means of the pair's row of n samples in place; returns the lane's part of the row's dL/dlam term.
    auto means = [&](float (&g)[C], uint32_t jump, uint32_t up, int n) -> float {
        // local samples past the row's end, outermost (at most 2C / 5 of them: the shorter side fills four fifths)
        const int pads = FULL ? 0 : (right ? S - n : 0);
        if (!FULL && pads > 0) jump |= 1u << (pads - 1);
        float s = 0.f;
        int c4 = 0;
        auto inverse = [&](int bytes) { return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(rtab) + bytes); };
#pragma unroll
        for (int k = 0; k < C; ++k) {
            s += g[k];
            c4 += 4;
            if (k < C - 1) {
                g[k] = s * inverse(c4);
                if (jump & (1u << k)) { s = 0.f; c4 = 0; }
            }
        }
        const bool mid = (jump & (1u << (C - 1))) != 0u;
        const float s2 = pair_other(s);
        const int c2 = (int)pair_other((uint32_t)c4);
        if (!mid) { s += s2; c4 += c2; }
        float carry = s * inverse(c4), term = 0.f;
        {
            const float d = carry - pair_other(carry);          // (0 where the middle is no jump)
            term = right ? 0.f : ((up & (1u << (C - 1))) ? d : -d);
        }
        g[C - 1] = carry;
#pragma unroll
        for (int k = C - 2; k >= 0; --k) {
            const float inner = carry;
            carry = (jump & (1u << k)) ? g[k] : carry;
            g[k] = carry;
            const float d = carry - inner;
            if (FULL || k >= 2 * C / 5 || k >= pads) term += (up & (1u << k)) ? d : -d;
        }
        return term;
    };
    float glam = 0.f;
    float v[C], xv[C];
    fetch(2 * p.sweeps - 1, xv);
    __syncthreads();
    for (int k = p.sweeps - 1; k >= 0; --k) {
        const bool first = (k == p.sweeps - 1);
        uint32_t jump, up;
        // ---- adjoint of the column pass: B <- C^T(A - B) + B  (B = 0 in the first reverse step)
        bits_of(xv, jump, up);
        fetch(2 * k, xv);
        {
            const float *a = A + col_at;
            float *b = B + col_at;
#pragma unroll
            for (int r = 0; r < C; ++r) v[r] = first ? a[r * P] : a[r * P] - b[r * P];
            const float t = means(v, jump, up, H);
            if (cvalid) glam += t;
#pragma unroll
            for (int r = 0; r < C; ++r) b[r * P] = first ? v[r] : b[r * P] + v[r];
        }
        __syncthreads();
        // ---- adjoint of the row pass: A <- R^T(B - A) + A  (without A in the first reverse step)
        bits_of(xv, jump, up);
        fetch(2 * k - 1, xv);
        {
            float *a = A + row_at;
            const float *b = B + row_at;
#pragma unroll
            for (int c = 0; c < C; ++c) v[c] = first ? b[c] : b[c] - a[c];
            const float t = means(v, jump, up, W);
            if (rvalid) glam += t;
#pragma unroll
            for (int c = 0; c < C; ++c) a[c] = first ? v[c] : a[c] + v[c];
        }
        __syncthreads();
    }

    float *dst = p.gy + plane * HW;
    each_sample([&](int e, int place) { dst[e] = A[place]; });
    if (p.partial) {
        // sum over the plane's lanes, in a fixed order
        float s = glam;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) s += __shfl_xor(s, d);
        if ((tid & 63) == 0) wave_term[tid >> 6] = s;
        __syncthreads();
        if (tid == 0) p.partial[plane] = wave_term[0] + wave_term[1];
    }
}

}  // namespace tvk
