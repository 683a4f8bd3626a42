// Forward kernel for rows of 33-768 samples inside one wave that finds the Newton direction by
// solving the masked tridiagonal system of paper Eq. 4: every thread eliminates its chunk (Thomas,
// pivots from a table: they depend only on the position inside a free run), the chunks' last duals
// obey a tridiagonal Schur complement whose entries follow from that and from the closed-form
// corner entries of the inverse of tridiag(-1,2,-1), (A^-1)_11 = m/(m+1), (A^-1)_1m = 1/(m+1), which is
// solved by parallel cyclic reduction, and every thread substitutes back.
//
// tv_rowsolve.hpp does the same in fewer instructions.  What is left here are the passes of 2D calls
// with one lambda for all planes and three sweeps or more (one_lambda_tri_side in tv_dispatch.hpp).  From sweep to sweep the jumps inside
// flat regions of an image shrink towards zero (24 images of 512 x 512: two rows in the first sweep,
// some three hundred in the tenth have one that is as small as the last bit of x, and rounding
// decides whether it is there), each such jump is a term of the lambda gradient, and one signed sum
// over all of them, with one lambda, cancels to a few of its terms: another rounding moves it by up to
// 5 % (three of ten inputs beyond 1 %).  These calls keep the rounding they had.
#pragma once
#include "tv_long.hpp"

namespace tvk {

template <int T, int C, int G>
struct TriSmem {
    static constexpr int TP = T + 2;                   // one zero sentinel on either side
    float gtab[C + 2];
    float rtab[C + 2];                                 // rtab[m] = 1 / (m + 1) = 1 - gtab[m]
    float ex[5][G][TP];
    float buf[2 * 3 * G * T];
};

template <class Mp>
__device__ __forceinline__ bool tri_sync_any(bool pred)
{
    Mp::sync();
    return __any(pred ? 1 : 0) != 0;
}

template <int T, int C, int G, bool XPOSE, int WARM>
__global__ __launch_bounds__(T *G, (fwd_waves_per_simd<T, C, G, XPOSE, XPOSE>())) void tv1d_fwd_tri_kernel(FwdParams p)
{
    static_assert(T <= 64, "rows inside one wave");
    using Mp = LongMap<T, G, false>;
    // a row inside one 16-lane DPP row: neighbours' values by row shifts, not through LDS (from_left)
    constexpr bool DPPX = T <= 16;
    __shared__ TriSmem<T, C, G> sm;
    // tile[row][k + k / C]: the pad after every chunk makes a wave's chunk reads conflict-free,
    // the pitch does the same for the transposing accesses (xpose_tile_pitch)
    constexpr int TILE_PITCH = xpose_tile_pitch<T, C, G>();
    // The tile is in use before the solve and after it, the exchange and PCR buffers during it:
    // where it fits it lies on top of them (two barriers more), which is what lets a second
    // workgroup share the CU's LDS.
    constexpr bool TILE_ALIAS = XPOSE && (size_t)G * TILE_PITCH * sizeof(float) <= sizeof(sm.ex) + sizeof(sm.buf);
    using Smem = TriSmem<T, C, G>;
    static_assert(__builtin_offsetof(Smem, buf) == __builtin_offsetof(Smem, ex) + sizeof(sm.ex),
                  "ex and buf must be adjacent");
    __shared__ float tile_own[(XPOSE && !TILE_ALIAS) ? G * TILE_PITCH : 1];
    float *tile = TILE_ALIAS ? &sm.ex[0][0][0] : tile_own;
    const int tid = threadIdx.x;
    const int j = Mp::row_of(tid), t = Mp::t_of(tid);
#define TV_EX(q, tt) sm.ex[q][j][(tt) + 1]
#define TV_PB(c, q, tt) sm.buf[(((c) * 3 + (q)) * G + j) * T + (tt)]

    const uint32_t group = XPOSE ? xcd_grouped<G>(blockIdx.x, gridDim.x) : blockIdx.x;
    const uint32_t row = group * G + j;
    const bool rvalid = row < p.L.n_rows;
    const int n = p.L.n, M = n - 1;
    const int k0 = t * C;

    if (tid <= C) {
        sm.gtab[tid] = (float)tid / (float)(tid + 1);
        sm.rtab[tid] = 1.0f / (float)(tid + 1);
    }
    if (!TILE_ALIAS && t == 0) {
#pragma unroll
        for (int q = 0; q < 5; ++q) { sm.ex[q][j][0] = 0.f; sm.ex[q][j][T + 1] = 0.f; }
    }
    __syncthreads();                        // the pivot table is the one thing the waves share

    const int64_t off = rvalid ? row_offset(p.L, row) : 0;
    const int64_t es = p.L.elem_stride;
    float lam = rvalid ? load_lambda(p.lam, p.L, row) : 0.f;
    float y[C];
    // transposing variant: thread tid moves samples k = tid / G, tid / G + T, ... of row tid % G
    const int xj = tid % G, xk0 = tid / G;
    const uint32_t xrow = group * G + xj;
    const int64_t xoff = (XPOSE && xrow < p.L.n_rows) ? row_offset(p.L, xrow) : 0;
    // Warm start: the addend is D^T u of an earlier solve of nearly the same rows, so
    // u_k = -(addend_0 + .. + addend_k).  u first takes the negated running sums inside the
    // chunk; the chunks before this one are added further down.
    constexpr bool warm = WARM == 1;
    float u[C];
    float wsum = 0.f;                                  // negated sum of the chunk's addend
    if constexpr (XPOSE) {
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
        if constexpr (TILE_ALIAS) {
            __syncthreads();                // everyone has left the tile: its memory turns into ex / buf
            if (t == 0) {
#pragma unroll
                for (int q = 0; q < 5; ++q) { sm.ex[q][j][0] = 0.f; sm.ex[q][j][T + 1] = 0.f; }
            }
        }
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
    // rounding floor of a difference of two x values (|x| <= max|y|, |u| <= lam)
    float gtol;
    {
        float ym[1] = {0.f};
#pragma unroll
        for (int i = 0; i < C; ++i) ym[0] = fmaxf(ym[0], fabsf(y[i]));
        row_max<T, G, false>(ym, nullptr, j, tid);
        // lam_max = max_k |sum_{i<=k} (mean(y) - y_i)| = max_k |(k / n) sum_{i>k} y_i -
        // ((n - k) / n) sum_{i<=k} y_i| <= 2 k (n - k) / n max|y| <= n / 2 max|y|, and every lambda from
        // lam_max on gives the same minimiser (the row's mean): a lambda beyond that bound is
        // replaced by it, which keeps the dual box, and with it the rounding errors of
        // x = y - D^T u, at the scale of the data.  The cold start needs it (it puts the duals on
        // the bounds), and so does a start from a coarser level's dual, whose stopping tolerance
        // scales with lambda; a pass that starts from the dual an addend encodes is left alone,
        // where the extra dependency cost 3 % of the 2D operator's time.
        if constexpr (WARM != 1) lam = fminf(lam, 0.51f * (float)n * ym[0]);
        gtol = kGradNoise * (ym[0] + lam);
        Mp::sync();
    }

    // duals past the end of the row get an empty box and never move
    const int nv = min(max(M - k0, 0), C);             // duals of this chunk inside the row
#define TV_LK(i) (((i) < nv) ? lam : 0.0f)

    float ynext0;
    if constexpr (DPPX) {
        ynext0 = from_right<T, 1>(y[0], t);
    } else {
        TV_EX(0, t) = y[0];
        Mp::sync();
        ynext0 = TV_EX(0, t + 1);
        Mp::sync();
    }
    // ---- starting point: every dual at the bound its local difference points to, or the
    //      dual the addend encodes, brought into the box (duals within rounding distance of a
    //      bound onto it)
    float fcur;
    float edge_l, edge_r;     // the neighbours' duals next to this chunk, carried between steps
    {
        if (warm) {
            float before, unused;
            seg_scan<T, G, false, +1, true>(false, wsum, 0.f, sm.buf, j, t, before, unused);
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
        float uleft;
        if constexpr (DPPX) {
            uleft = from_left<T, 1>(u[C - 1], t);
            edge_r = from_right<T, 1>(u[0], t);
        } else {
            TV_EX(0, t) = u[C - 1];
            TV_EX(1, t) = u[0];
            Mp::sync();
            uleft = TV_EX(0, t - 1);
            edge_r = TV_EX(1, t + 1);
        }
        edge_l = uleft;
        float acc[1] = {0.f};
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const float xi = y[i] + u[i] - (i > 0 ? u[i - 1] : uleft);
            acc[0] = fmaf(xi, xi, acc[0]);
        }
        row_sum<T, G, false, 1>(acc, nullptr, j, tid);
        fcur = 0.5f * acc[0];
        Mp::sync();
    }

    bool active = rvalid;
    bool prev_unclipped = false;
    int flags = 0;
    for (int it = 0;; ++it) {
            // ---- chunk edges of the dual: exchanged by the accepted trial of the step before
        const float uleft = edge_l;
        const float unext0 = edge_r;

        // ---- gradient, bound set, optimality test, interior elimination (Thomas, pass 1)
        float g[C], gam[C], w[C];
        bool bsep;
        int pos = 0, a = 0;
        bool seen_bound = false;
        float viof[1] = {0.f};
        {
            float wprev = 0.f, gprev = 0.f;
            float xi = y[0] + u[0] - uleft;
#pragma unroll
            for (int i = 0; i < C; ++i) {
                const float xn = (i + 1 < C) ? (y[i + 1] + u[i + 1] - u[i])
                                             : (ynext0 + unext0 - u[C - 1]);
                const float gi = xi - xn;
                g[i] = gi;
                const float s = copysignf(TV_LK(i), gi);
                const bool bnd = (u[i] == -s);
                if (i < nv && u[i] == s && fabsf(gi) > gtol) viof[0] += 1.f;
                if (i < C - 1) {
                    pos = bnd ? 0 : pos + 1;
                    const float gm = sm.gtab[pos];
                    const float wi = fmaf(gprev, wprev, gi);
                    gam[i] = gm; w[i] = wi;
                    wprev = wi; gprev = gm;
                    if (!seen_bound) { if (bnd) seen_bound = true; else a += 1; }
                } else {
                    bsep = bnd;
                }
                xi = xn;
            }
        }
        float p0, pl;
        {
            float pn = 0.f;
            pl = 0.f;
#pragma unroll
            for (int i = C - 2; i >= 0; --i) {
                pn = gam[i] * (w[i] + pn);
                if (i == C - 2) pl = pn;
            }
            p0 = pn;
        }
        // The separator's diagonal is 2 - (A^-1)_{last,last} of this chunk's interior block -
        // (A^-1)_{first,first} of the next one's, with (A^-1)_{first,first} = a / (a + 1) for a
        // leading free duals (likewise at the other end).  Inside a long free run that is
        // 2 - 2 (C - 1) / C: formed from the rounded fractions it loses all but a few bits
        // unless C is a power of two, so the exchange carries 1 - a / (a + 1) = 1 / (a + 1).
        const float c_alpha = sm.rtab[a];                       // 1 - (A^-1)_{first,first}
        const float c_delta = sm.rtab[pos];                     // 1 - (A^-1)_{last,last}
        const float c_beta = (a == C - 1) ? (1.0f / (float)C) : 0.f;  // (A^-1)_{first,last}
        if constexpr (!DPPX) {
            TV_EX(2, t) = p0;
            TV_EX(3, t) = c_alpha;
            TV_EX(4, t) = c_beta;
        }
        bool vio;
        row_sum<T, G, false, 1>(viof, nullptr, j, tid);
        vio = viof[0] != 0.f;
        Mp::sync();
        float p0n, alphan, betan;
        if constexpr (DPPX) {
            p0n = from_right<T, 1>(p0, t); alphan = from_right<T, 1>(c_alpha, t); betan = from_right<T, 1>(c_beta, t);
        } else {
            p0n = TV_EX(2, t + 1); alphan = TV_EX(3, t + 1); betan = TV_EX(4, t + 1);
        }

        if (active && prev_unclipped && !vio) { active = false; flags = kInfoConverged; }
        if (active && it >= kMaxNewtonSteps) { active = false; flags = kInfoCapped; }
        if (!tri_sync_any<Mp>(active)) break;

        // ---- separator system (normalised to unit diagonal) and PCR
        float ea = 0.f, ec = 0.f, er = 0.f;
        if (!bsep) {
            const float inv = __builtin_amdgcn_rcpf(c_delta + alphan);
            ea = -c_beta * inv;
            ec = -betan * inv;
            er = (g[C - 1] + pl + p0n) * inv;
        }
        float sleft;
        if constexpr (DPPX) {
            // the same reduction with the neighbours' equations fetched by row shifts
#define TV_PCR_STEP(S)                                                                              \
            if constexpr ((S) < T) {                                                                \
                if (going && (going = __any((ea != 0.f || ec != 0.f) ? 1 : 0) != 0)) {             \
                    const float la = from_left<T, (S) < T ? (S) : 1>(ea, t), lc = from_left<T, (S) < T ? (S) : 1>(ec, t),      \
                                lr = from_left<T, (S) < T ? (S) : 1>(er, t);                        \
                    const float ra = from_right<T, (S) < T ? (S) : 1>(ea, t), rc = from_right<T, (S) < T ? (S) : 1>(ec, t),    \
                                rr = from_right<T, (S) < T ? (S) : 1>(er, t);                       \
                    const float inv = __builtin_amdgcn_rcpf(1.0f - ea * lc - ec * ra);              \
                    er = (er - ea * lr - ec * rr) * inv;                                            \
                    const float na = -ea * la * inv, nc = -ec * rc * inv;                           \
                    ea = na; ec = nc;                                                               \
                }                                                                                   \
            }
            bool going = true;
            TV_PCR_STEP(1) TV_PCR_STEP(2) TV_PCR_STEP(4) TV_PCR_STEP(8)
#undef TV_PCR_STEP
            sleft = from_left<T, 1>(er, t);
        } else {
            int cur = 0;
            bool published = false;
            for (int s = 1; s < T; s <<= 1) {
                TV_PB(cur, 0, t) = ea; TV_PB(cur, 1, t) = ec; TV_PB(cur, 2, t) = er;
                // every equation decoupled: the right-hand sides just published are the solution
                if (!tri_sync_any<Mp>(ea != 0.f || ec != 0.f)) { published = true; break; }
                float la = 0.f, lc = 0.f, lr = 0.f, ra = 0.f, rc = 0.f, rr = 0.f;
                if (t - s >= 0) { la = TV_PB(cur, 0, t - s); lc = TV_PB(cur, 1, t - s); lr = TV_PB(cur, 2, t - s); }
                if (t + s < T) { ra = TV_PB(cur, 0, t + s); rc = TV_PB(cur, 1, t + s); rr = TV_PB(cur, 2, t + s); }
                const float inv = __builtin_amdgcn_rcpf(1.0f - ea * lc - ec * ra);
                er = (er - ea * lr - ec * rr) * inv;
                const float na = -ea * la * inv, nc = -ec * rc * inv;
                ea = na; ec = nc;
                cur ^= 1;
            }
            if (!published) {
                TV_PB(cur, 2, t) = er;
                Mp::sync();
            }
            sleft = t > 0 ? TV_PB(cur, 2, t - 1) : 0.f;
        }
        const float sigma = er;

        // ---- interior back-substitution with the separators as boundary terms (pass 2);
        //      w becomes the Newton direction d
        float decp = 0.f;
        {
            float wprev = 0.f, gprev = 0.f;
#pragma unroll
            for (int i = 0; i < C - 1; ++i) {
                float rhs = g[i];
                if (i == 0) rhs += sleft;
                if (i == C - 2) rhs += sigma;
                const float wi = fmaf(gprev, wprev, rhs);
                w[i] = wi; wprev = wi; gprev = gam[i];
            }
            float dn = 0.f;
#pragma unroll
            for (int i = C - 2; i >= 0; --i) {
                dn = gam[i] * (w[i] + dn);
                w[i] = dn;
                decp = fmaf(g[i], dn, decp);
            }
            w[C - 1] = sigma;
            decp = fmaf(g[C - 1], sigma, decp);
        }

        // ---- projected step with Armijo backtracking (quadratic interpolation)
        float alpha = active ? 1.f : 0.f;
        float uc[C];
        float fc = 0.f, dec = 0.f;
        bool clipped = false, changed = false;
        for (int ls = 0;; ++ls) {
            float v[4] = {0.f, decp, 0.f, 0.f};
            bool cl = false, ch = false;
#pragma unroll
            for (int i = 0; i < C; ++i) {
                const float l = TV_LK(i);
                const float tt = fmaf(-alpha, w[i], u[i]);
                const float cc = __builtin_amdgcn_fmed3f(tt, -l, l);
                cl |= (cc != tt);
                ch |= (cc != u[i]);
                uc[i] = cc;
            }
            float ucleft;
            if constexpr (DPPX) {
                ucleft = from_left<T, 1>(uc[C - 1], t);
                edge_r = from_right<T, 1>(uc[0], t);
            } else {
                TV_EX(0, t) = uc[C - 1];
                TV_EX(1, t) = uc[0];
                Mp::sync();
                ucleft = TV_EX(0, t - 1);
                edge_r = TV_EX(1, t + 1);
            }
            edge_l = ucleft;
#pragma unroll
            for (int i = 0; i < C; ++i) {
                const float xc = y[i] + uc[i] - (i > 0 ? uc[i - 1] : ucleft);
                v[0] = fmaf(xc, xc, v[0]);
            }
            v[2] = cl ? 1.f : 0.f;
            v[3] = ch ? 1.f : 0.f;
            row_sum<T, G, false, 4>(v, nullptr, j, tid);
            fc = 0.5f * v[0]; dec = v[1]; clipped = v[2] > 0.f; changed = v[3] > 0.f;
            const bool ok = !active || alpha == 0.f || (alpha == 1.f && !clipped) ||
                            (fc <= fcur - kArmijoSigma * alpha * dec + kArmijoSlackEps * fabsf(fcur));
            if (!tri_sync_any<Mp>(!ok)) break;
            if (!ok) {
                if (ls >= kMaxBacktracks) {
                    alpha = 0.f;
                } else {
                    const float den = 2.f * (fc - fcur + dec * alpha);
                    const float an = den > 0.f ? dec * alpha * alpha / den : 0.5f * alpha;
                    alpha = fminf(fmaxf(an, 0.1f * alpha), 0.5f * alpha);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < C; ++i) u[i] = uc[i];
        prev_unclipped = (alpha == 1.f) && !clipped;
        if (active) fcur = fc;
        if (active && !changed) { active = false; flags = kInfoStalled; }
        if (!tri_sync_any<Mp>(active)) break;
    }

    // ---- primal recovery x = y - D^T u, then every block between two bound duals takes
    //      the value of its first sample, so that constant runs are bit-identical
    float xs[C];
    {
            float uleft, unext0;
        if constexpr (DPPX) {
            uleft = from_left<T, 1>(u[C - 1], t);
            unext0 = from_right<T, 1>(u[0], t);
        } else {
            TV_EX(0, t) = u[C - 1];
            TV_EX(1, t) = u[0];
            Mp::sync();
            uleft = TV_EX(0, t - 1);
            unext0 = TV_EX(1, t + 1);
        }
        bool bnd[C];
        float xi = y[0] + u[0] - uleft;
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const float xn = (i + 1 < C) ? (y[i + 1] + u[i + 1] - u[i]) : (ynext0 + unext0 - u[C - 1]);
            const float gi = xi - xn;
            bnd[i] = (u[i] == -copysignf(TV_LK(i), gi));
            xs[i] = xi;
            xi = xn;
        }
        // a sample starts a block when the dual on its left is bound; chunk-local pass first
        bool start0;
        if constexpr (DPPX) {
            // (fetched by all lanes before any of them branches: a row shift reads 0 from a lane that is switched off)
            const float left_bound = from_left<T, 1>(bnd[C - 1] ? 1.f : 0.f, t);
            start0 = (t == 0) || (left_bound != 0.f);
        } else {
            TV_EX(2, t) = bnd[C - 1] ? 1.f : 0.f;
            Mp::sync();
            start0 = (t == 0) || (TV_EX(2, t - 1) != 0.f);
        }
        bool closed = start0;
        float last = xs[0];
#pragma unroll
        for (int i = 1; i < C; ++i)
            if (bnd[i - 1]) { closed = true; last = xs[i]; }
        // `last` = first sample of the chunk's last block (valid when closed)
        float cv, cdummy;
        seg_scan<T, G, false, +1, false>(closed, last, 0.f, sm.buf, j, t, cv, cdummy);
        float val = start0 ? xs[0] : cv;
        float dev[1] = {0.f};
#pragma unroll
        for (int i = 0; i < C; ++i) {
            if (i > 0 && bnd[i - 1]) val = xs[i];
            // (not below four rounding floors of a difference of two x values: the floor follows
            // the row's largest sample, and next to one large sample a converged row's small
            // segments still carry that much noise)
            if (fabsf(val - xs[i]) > fmaxf(2e-5f * (1.f + fabsf(y[i]) + lam), 4.f * gtol)) dev[0] += 1.f;
            u[i] = val;       // u is dead from here on: reuse it for the block values
        }
        row_sum<T, G, false, 1>(dev, nullptr, j, tid);
        // (an infinite sample makes the floor infinite: such a row keeps its plain output, which shows it)
        const bool use_blocks = !(flags & kInfoCapped) && dev[0] == 0.f && gtol <= 3.0e38f;
        if (use_blocks) {
#pragma unroll
            for (int i = 0; i < C; ++i) xs[i] = u[i];
        }
    }

    if constexpr (XPOSE) {
        // a wave writes only its own row of the tile; the barrier then hands the tile over
        if constexpr (TILE_ALIAS) __syncthreads();      // every wave is done with ex / buf
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
            __syncthreads();
#pragma unroll
            for (int i = 0; i < C; ++i) tile[j * TILE_PITCH + t * (C + 1) + i] = y[i] - xs[i];
            __syncthreads();
            for (int k = xk0; k < T * C; k += T)
                if (xrow < p.L.n_rows && k < n)
                    p.resid[xoff + (int64_t)k * es] = tile[xj * TILE_PITCH + k + k / C];
        }
    } else {
        if (p.x) chunk_store<C>(p.x, off, es, k0, n, rvalid, xs);
        if (p.x2) chunk_store<C>(p.x2, off, es, k0, n, rvalid, xs);
        if (p.resid) {
#pragma unroll
            for (int i = 0; i < C; ++i) y[i] -= xs[i];
            chunk_store<C>(p.resid, off, es, k0, n, rvalid, y);
        }
    }
    if constexpr (chunk_coded<T, C>()) {
        if (p.chunk_codes) {
            const uint32_t code = chunk_code<T, C>(xs);
            if (rvalid) p.chunk_codes[(size_t)row * T + t] = code;
        }
        if (p.codes_tag && blockIdx.x == 0 && tid == 0) *p.codes_tag = p.chunk_codes ? 1u : 0u;
    }
#undef TV_EX
#undef TV_PB
#undef TV_LK
}

template <int T, int C, int G>
inline hipError_t launch_fwd_tri_t(const FwdParams &p, hipStream_t s)
{
    const dim3 grid((p.L.n_rows + G - 1) / G), block(T * G);
    const bool cols = p.L.elem_stride != 1;
    if (p.warm) {
        if (cols) hipLaunchKernelGGL((tv1d_fwd_tri_kernel<T, C, G, true, 1>), grid, block, 0, s, p);
        else hipLaunchKernelGGL((tv1d_fwd_tri_kernel<T, C, G, false, 1>), grid, block, 0, s, p);
    } else {
        if (cols) hipLaunchKernelGGL((tv1d_fwd_tri_kernel<T, C, G, true, 0>), grid, block, 0, s, p);
        else hipLaunchKernelGGL((tv1d_fwd_tri_kernel<T, C, G, false, 0>), grid, block, 0, s, p);
    }
    return hipGetLastError();
}

inline hipError_t launch_fwd_tri(const FwdParams &p, hipStream_t s)
{
    const int n = p.L.n;
    if (p.L.elem_stride != 1) {
        if (n <= 64) return launch_fwd_tri_t<8, 8, 16>(p, s);
        if (n <= 96) return launch_fwd_tri_t<8, 12, 16>(p, s);
        if (n <= 128) return launch_fwd_tri_t<16, 8, 16>(p, s);
        if (n <= 192) return launch_fwd_tri_t<16, 12, 16>(p, s);
        if (n <= 256) return launch_fwd_tri_t<32, 8, 8>(p, s);
        if (n <= 384) return launch_fwd_tri_t<32, 12, 8>(p, s);
        if (n <= 512) return launch_fwd_tri_t<64, 8, 8>(p, s);
        return launch_fwd_tri_t<64, 12, 8>(p, s);
    }
    if (n <= 64) return launch_fwd_tri_t<8, 8, 32>(p, s);
    if (n <= 96) return launch_fwd_tri_t<8, 12, 32>(p, s);
    if (n <= 128) return launch_fwd_tri_t<16, 8, 16>(p, s);
    if (n <= 192) return launch_fwd_tri_t<16, 12, 16>(p, s);
    if (n <= 256) return launch_fwd_tri_t<32, 8, 8>(p, s);
    if (n <= 384) return launch_fwd_tri_t<32, 12, 8>(p, s);
    if (n <= 512) return launch_fwd_tri_t<64, 8, 4>(p, s);
    return launch_fwd_tri_t<64, 12, 4>(p, s);
}

}  // namespace tvk
