// hh_idr_kernels.hpp -- IDR(s) passes (right preconditioned, x-space form of
// the prototype algorithm of Sonneveld & van Gijzen, with the
// minimal-residual omega), one step = one matvec (V-cycle + H apply):
//
//   P1  k_idr_v   start-up: v = r;  cycle step: q = -sum_j dR_j c_j, v = r + q
//   --  V-cycle   w = V(v)
//   P3  k_idr_t   start-up / k = 0: t = H w, partials (t, v), (t, t)
//                 k >= 1: dX_old = om w - sum_j dX_j c_j
//   fin           omega = (t, v) / (t, t)   (start-up and k = 0)
//   P4  k_idr_up  start-up: dX_k = om w, dR_k = -om t
//                 k = 0:    dR_old = q - om t, dX_old = om w - sum_j dX_j c_j
//                 k >= 1:   dR_old = -H dX_old
//                 then r += dR, x += dX; partials ||r||^2, P^H dR (and P^H r
//                 at start-up)
//   fin           residual check, G(:, old) = P^H dR, m += P^H dR, next c
//                 from the s x s LU solve G c = m
//
// Sums over columns run j = 0..s-1 left to right; the small solve uses LU
// with partial pivoting (first maximum of |re| + |im|) -- the same order as
// the CPU oracle, so FP64 iterates agree value for value.
#pragma once
#include "hh_kernels.hpp"

namespace hh {

// s x s complex LU solve G c = m (G row major), same algorithm as the host
// setup's dense LU.  Returns false for an exactly singular pivot.  One thread,
// in LDS; for s <= 4 in registers (S = s, rows swapped by selects), where it
// takes about 2 us instead of waiting for LDS between dependent steps.
__device__ inline bool small_solve_lds(const double2 *Gin, int s, const double2 *m, double2 *c)
{
    __shared__ double2 A[HH_MAX_S * HH_MAX_S];   // thread 0 only (keeps the solve out of scratch memory)
    __shared__ int perm[HH_MAX_S];
    for (int i = 0; i < s * s; ++i) A[i] = Gin[i];
    for (int i = 0; i < s; ++i) perm[i] = i;
    for (int k = 0; k < s; ++k) {
        int p = k;
        double best = fabs(A[k * s + k].x) + fabs(A[k * s + k].y);
        for (int i = k + 1; i < s; ++i) {
            double v = fabs(A[i * s + k].x) + fabs(A[i * s + k].y);
            if (v > best) {
                best = v;
                p = i;
            }
        }
        if (best == 0.0) return false;
        if (p != k) {
            for (int j = 0; j < s; ++j) {
                double2 t = A[k * s + j];
                A[k * s + j] = A[p * s + j];
                A[p * s + j] = t;
            }
            int t = perm[k];
            perm[k] = perm[p];
            perm[p] = t;
        }
        const double2 piv = A[k * s + k];
        for (int i = k + 1; i < s; ++i) {
            double2 l = cdiv<double>(A[i * s + k], piv);
            A[i * s + k] = l;
            for (int j = k + 1; j < s; ++j) A[i * s + j] = csub<double>(A[i * s + j], cmul<double>(l, A[k * s + j]));
        }
    }
    for (int i = 0; i < s; ++i) {
        double2 v = m[perm[i]];
        for (int j = 0; j < i; ++j) v = csub<double>(v, cmul<double>(A[i * s + j], c[j]));
        c[i] = v;
    }
    for (int i = s - 1; i >= 0; --i) {
        double2 v = c[i];
        for (int j = i + 1; j < s; ++j) v = csub<double>(v, cmul<double>(A[i * s + j], c[j]));
        c[i] = cdiv<double>(v, A[i * s + i]);
    }
    return true;
}
template <int S> __device__ inline bool small_solve_reg(const double2 *Gin, const double2 *min, double2 *cout)
{
    double2 A[S][S], m[S], c[S];
#pragma unroll
    for (int i = 0; i < S; ++i) {
#pragma unroll
        for (int j = 0; j < S; ++j) A[i][j] = Gin[i * S + j];
        m[i] = min[i];
    }
#pragma unroll
    for (int k = 0; k < S; ++k) {
        int p = k;
        double best = fabs(A[k][k].x) + fabs(A[k][k].y);
#pragma unroll
        for (int i = k + 1; i < S; ++i) {
            const double v = fabs(A[i][k].x) + fabs(A[i][k].y);
            if (v > best) {
                best = v;
                p = i;
            }
        }
        if (best == 0.0) return false;
#pragma unroll
        for (int i = k + 1; i < S; ++i) {
            const bool sw = p == i;
#pragma unroll
            for (int j = 0; j <= S; ++j) {       // column S: the right-hand side
                double2 &a = j < S ? A[k][j < S ? j : 0] : m[k], &b = j < S ? A[i][j < S ? j : 0] : m[i];
                const double2 t = a;
                a = cmk<double>(sw ? b.x : t.x, sw ? b.y : t.y);
                b = cmk<double>(sw ? t.x : b.x, sw ? t.y : b.y);
            }
        }
#pragma unroll
        for (int i = k + 1; i < S; ++i) {
            const double2 l = cdiv<double>(A[i][k], A[k][k]);
            A[i][k] = l;
#pragma unroll
            for (int j = k + 1; j < S; ++j) A[i][j] = csub<double>(A[i][j], cmul<double>(l, A[k][j]));
        }
    }
#pragma unroll
    for (int i = 0; i < S; ++i) {
        double2 v = m[i];
#pragma unroll
        for (int j = 0; j < i; ++j) v = csub<double>(v, cmul<double>(A[i][j], c[j]));
        c[i] = v;
    }
#pragma unroll
    for (int i = S - 1; i >= 0; --i) {
        double2 v = c[i];
#pragma unroll
        for (int j = i + 1; j < S; ++j) v = csub<double>(v, cmul<double>(A[i][j], c[j]));
        c[i] = cdiv<double>(v, A[i][i]);
    }
#pragma unroll
    for (int i = 0; i < S; ++i) cout[i] = c[i];
    return true;
}
__device__ inline bool small_solve(const double2 *G, int s, const double2 *m, double2 *c)
{
    switch (s) {
    case 1: return small_solve_reg<1>(G, m, c);
    case 2: return small_solve_reg<2>(G, m, c);
    case 3: return small_solve_reg<3>(G, m, c);
    case 4: return small_solve_reg<4>(G, m, c);
    default: return small_solve_lds(G, s, m, c);
    }
}

// scalar state after a pass (one thread; st in LDS, v the pass's sums)
__device__ inline void idr_advance(const ProbDev *pd, SolveState *st, int kind, const double *v)
{
    const int s = st->s;
    if (kind == FIN_IDR_INIT) {
        st->phase = PH_RUN;
        st->reason = RS_NONE;
        st->startup = 0;
        st->kstep = 0;
        st->oldest = 0;
        st->om_idr = cmk<double>(1.0, 0.0);
        st->best_rel = INFINITY;
        st->best_mv = st->mv;
        return;
    }
    const int mode = st->startup >= 0 ? 0 : (st->kstep == 0 ? 1 : 2);
    if (kind == FIN_IDR_OMEGA) {
        st->mv += 1;
        double2 tv = cmk<double>(v[0], v[1]);
        double tt = v[2];
        if (!cfin(tv) || !isfinite(tt)) { stop(st, RS_NONFIN); return; }
        if (tt == 0.0) { stop(st, RS_BREAK); return; }
        st->om_idr = cmk<double>(tv.x / tt, tv.y / tt);
        return;
    }
    // FIN_IDR_STEP
    if (mode == 2) st->mv += 1;
    if (mode != 0) st->it += 1;
    const double rel = sqrt(v[0]) / st->bnorm;
    record(pd, st, rel);
    if (!isfinite(rel)) { stop(st, RS_NONFIN); return; }
    if (rel < st->tol) { stop(st, RS_CONV); return; }
    if (st->mv >= st->max_mv) { stop(st, RS_MAXMV); return; }
    if (st->guard && drift(rel, st->mv, st->best_rel, st->best_mv, st->drift_grow, st->drift_stall)) { stop(st, RS_DRIFT); return; }
    const int col = mode == 0 ? st->startup : st->oldest;
    for (int i = 0; i < s; ++i) {
        double2 dm = cmk<double>(v[1 + 2 * i], v[2 + 2 * i]);
        st->G[i * s + col] = dm;
        if (mode != 0) st->m[i] = cadd<double>(st->m[i], dm);
    }
    if (mode == 0) {
        st->startup += 1;
        if (st->startup < s) return;
        st->startup = -1;
        st->oldest = 0;
        st->kstep = 0;
        for (int i = 0; i < s; ++i) st->m[i] = cmk<double>(v[1 + 2 * HH_MAX_S + 2 * i], v[2 + 2 * HH_MAX_S + 2 * i]);
    } else {
        st->oldest = st->oldest + 1 == s ? 0 : st->oldest + 1;
        st->kstep = st->kstep + 1 == s + 1 ? 0 : st->kstep + 1;
    }
    if (!small_solve(st->G, s, st->m, st->c)) stop(st, RS_BREAK);
}

// Finaliser of the IDR passes: the state block is copied to LDS by all
// threads, advanced there by one, and copied back (a chain of dependent
// global accesses by one thread cost more than the sums).  Passes that reduce
// nothing in the current mode (omega in steps k >= 1) return after the copy.
__device__ void idr_finalize(const ProbDev *pd, int kind, bool gate)
{
    constexpr int SW = sizeof(SolveState) / 4, CW = sizeof(Ctrl) / 4;
    static_assert(sizeof(SolveState) % 4 == 0 && sizeof(Ctrl) % 4 == 0 && SW <= HH_FIN_WG && CW <= HH_FIN_WG, "one word per thread");
    __shared__ SolveState st;
    __shared__ Ctrl ct;
    __shared__ double res[4 * HH_MAX_S + 4];
    const int t = threadIdx.x;
    if (t < SW) ((uint32_t *)&st)[t] = ((const HH_GLOBAL uint32_t *)pd->st)[t];
    __syncthreads();
    if (kind != FIN_IDR_INIT && st.phase != PH_RUN) return;
    const int mode = st.startup >= 0 ? 0 : (st.kstep == 0 ? 1 : 2);
    if (kind == FIN_IDR_OMEGA) {
        if (mode == 2) return;
        reduce_partials(pd->part, pd->ngroup, 0, 3, res);
    } else if (kind == FIN_IDR_STEP) {
        reduce_partials(pd->part, pd->ngroup, 0, 1 + 2 * st.s, res);
        if (mode == 0) reduce_partials(pd->part, pd->ngroup, 1 + 2 * HH_MAX_S, 2 * st.s, res + 1 + 2 * HH_MAX_S);
    }
    if (t == 0) {
        idr_advance(pd, &st, kind, res);
        mirror(ct, st);
    }
    __syncthreads();
    if (t < SW) ((HH_GLOBAL uint32_t *)pd->st)[t] = ((const uint32_t *)&st)[t];
    if (pd->ctrl && t < CW) ((HH_GLOBAL uint32_t *)pd->ctrl)[t] = ((const uint32_t *)&ct)[t];
}

// NS (4 or 8): the columns the passes are built for, at least every problem's
// s.  With 8, IDR(4) held and reduced twice the values it has: the update
// pass took 95 us at 128^3, 3.5 TB/s.

// P1: v = r (start-up) or q = -sum_j dR_j c_j, v = r + q
template <int NS>
__global__ __launch_bounds__(HH_VWG) void k_idr_v(Ctx cx)
{
    const Tile tl = tile_of(cx);
    const Ctrl ct = ctrl_of(cx, tl.prob);
    if (ct.phase != PH_RUN) return;
    const ProbDev *pd = cx.P + tl.prob;
    const int64_t N = pd->N, base = (int64_t)tl.idx * HH_SPAN;
    const double2 *__restrict__ r = (const double2 *)pd->vec[VS_R];
    double2 *__restrict__ v = (double2 *)pd->vec[VS_V];
    double2 *__restrict__ q = (double2 *)pd->vec[VS_Q];
    if (ct.mode == 0) {
        double2 rr[HH_PER_SLOT];
#pragma unroll
        for (int e = 0; e < HH_PER_SLOT; ++e)
            if (CHUNK_P(e) < N) rr[e] = ldg(r, CHUNK_P(e));
#pragma unroll
        for (int e = 0; e < HH_PER_SLOT; ++e)
            if (CHUNK_P(e) < N) stg(v, CHUNK_P(e), rr[e]);
        return;
    }
    const int ns = pd->nidr;
    const double2 *__restrict__ dR = pd->dR;
#pragma unroll
    for (int e = 0; e < HH_PER_SLOT; ++e) {
        const int64_t p = CHUNK_P(e);
        if (p < N) {
            double2 col[NS];
#pragma unroll
            for (int j = 0; j < NS; ++j)
                if (j < ns) col[j] = ldg(dR, (int64_t)j * N + p);
            const double2 rv = ldg(r, p);
            double2 acc = cmul<double>(col[0], ct.c[0]);
#pragma unroll
            for (int j = 1; j < NS; ++j)
                if (j < ns) acc = cadd<double>(acc, cmul<double>(col[j], ct.c[j]));
            const double2 qv = cmk<double>(-acc.x, -acc.y);
            stg(v, p, cadd<double>(rv, qv));
            if (ct.mode == 1) stg(q, p, qv);
        }
    }
}

// P3: t = H w with partials (t, v), (t, t)   (start-up, k = 0)
//     dX_old = om w - sum_j dX_j c_j          (k >= 1)
template <int DIM, typename SW, int NS>
__global__ __launch_bounds__(HH_VWG) void k_idr_t(Ctx cx)
{
    const Tile tl = tile_of(cx);
    const Ctrl ct = ctrl_of(cx, tl.prob);
    if (ct.phase != PH_RUN) return;
    const ProbDev *pd = cx.P + tl.prob;
    const SW *__restrict__ w = (const SW *)pd->vec[VS_W];
    const int64_t base = (int64_t)tl.idx * HH_SPAN;
    if (ct.mode == 2) {
        const int64_t N = pd->N;
        const int ns = pd->nidr;
        double2 *__restrict__ dX = pd->dX;
#pragma unroll
        for (int e = 0; e < HH_PER_SLOT; ++e) {
            const int64_t p = CHUNK_P(e);
            if (p < N) {
                double2 col[NS];
#pragma unroll
                for (int j = 0; j < NS; ++j)
                    if (j < ns) col[j] = ldg(dX, (int64_t)j * N + p);
                const double2 wv = ld64(w, p);
                double2 acc = cmul<double>(col[0], ct.c[0]);
#pragma unroll
                for (int j = 1; j < NS; ++j)
                    if (j < ns) acc = cadd<double>(acc, cmul<double>(col[j], ct.c[j]));
                stg(dX, (int64_t)ct.old * N + p, csub<double>(cmul<double>(ct.om_idr, wv), acc));
            }
        }
        return;
    }
    const HView h = hview(pd);
    double2 *__restrict__ t = (double2 *)pd->vec[VS_T];
    const double2 *__restrict__ vv = (const double2 *)pd->vec[VS_V];
    double2 y[HH_PER_SLOT], b[HH_PER_SLOT];
#pragma unroll
    for (int e = 0; e < HH_PER_SLOT; ++e) {
        const int64_t p = CHUNK_P(e);
        if (p < h.N) {
            int i, j, k;
            split(p, h.nx, h.ny, h.fx, h.fxy, i, j, k);
            y[e] = stencil<DIM, double>(h, w, i, j, k, p);
            b[e] = ldg(vv, p);
        }
    }
    double acc[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int e = 0; e < HH_PER_SLOT; ++e) {
        const int64_t p = CHUNK_P(e);
        if (p < h.N) {
            stg(t, p, y[e]);
            acc[0] = acc[0] + (y[e].x * b[e].x + y[e].y * b[e].y);
            acc[1] = acc[1] + (y[e].x * b[e].y - y[e].y * b[e].x);
            acc[2] = acc[2] + (y[e].x * y[e].x + y[e].y * y[e].y);
        }
    }
    group_finish<3>(pd, tl.idx, acc);
}

// P4: the dR/dX column of this step, r += dR, x += dX; partials ||r||^2,
// P^H dR (and P^H r during start-up).  All loads of a point are issued before
// its first store.
template <int DIM, typename SW, int NS>
__global__ __launch_bounds__(HH_VWG) void k_idr_up(Ctx cx)
{
    const Tile tl = tile_of(cx);
    const Ctrl ct = ctrl_of(cx, tl.prob);
    if (ct.phase != PH_RUN) return;
    const ProbDev *pd = cx.P + tl.prob;
    const HView h = hview(pd);
    const int64_t N = h.N, p = (int64_t)tl.idx * HH_SPAN + threadIdx.x;
    const int ns = pd->nidr, mode = ct.mode;
    const double2 om = ct.om_idr;
    const SW *__restrict__ w = (const SW *)pd->vec[VS_W];
    double2 *__restrict__ x = (double2 *)pd->vec[VS_X];
    double2 *__restrict__ r = (double2 *)pd->vec[VS_R];
    const double2 *__restrict__ t = (const double2 *)pd->vec[VS_T];
    const double2 *__restrict__ q = (const double2 *)pd->vec[VS_Q];
    double2 *__restrict__ dR = pd->dR;
    double2 *__restrict__ dX = pd->dX;
    const double2 *__restrict__ Pm = pd->P;
    double2 *__restrict__ dRo = dR + (int64_t)ct.old * N;
    double2 *__restrict__ dXo = dX + (int64_t)ct.old * N;
    static_assert(HH_PER_SLOT == 1, "one unknown per thread");
    double acc[1 + 2 * NS], acr[2 * NS];
#pragma unroll
    for (int k = 0; k < 1 + 2 * NS; ++k) acc[k] = 0.0;
#pragma unroll
    for (int k = 0; k < 2 * NS; ++k) acr[k] = 0.0;
    if (p < N) {
        double2 dr, dx, pv[NS];
#pragma unroll
        for (int i = 0; i < NS; ++i)
            if (i < ns) pv[i] = ldg(Pm, (int64_t)i * N + p);
        const double2 r0 = ldg(r, p), x0 = ldg(x, p);
        if (mode == 0) {
            const double2 ot = cmul<double>(om, ldg(t, p));
            dx = cmul<double>(om, ld64(w, p));
            dr = cmk<double>(-ot.x, -ot.y);
        } else if (mode == 1) {
            double2 col[NS];
#pragma unroll
            for (int j = 0; j < NS; ++j)
                if (j < ns) col[j] = ldg(dX, (int64_t)j * N + p);
            const double2 tv = ldg(t, p), qv = ldg(q, p), wv = ld64(w, p);
            double2 ax = cmul<double>(col[0], ct.c[0]);
#pragma unroll
            for (int j = 1; j < NS; ++j)
                if (j < ns) ax = cadd<double>(ax, cmul<double>(col[j], ct.c[j]));
            dr = csub<double>(qv, cmul<double>(om, tv));
            dx = csub<double>(cmul<double>(om, wv), ax);
        } else {
            int i, j, k;
            split(p, h.nx, h.ny, h.fx, h.fxy, i, j, k);
            const double2 hv = stencil<DIM, double>(h, dXo, i, j, k, p);
            dr = cmk<double>(-hv.x, -hv.y);
            dx = ldg(dXo, p);
        }
        if (mode != 2) stg(dXo, p, dx);
        stg(dRo, p, dr);
        const double2 rn = cadd<double>(r0, dr);
        stg(r, p, rn);
        stg(x, p, cadd<double>(x0, dx));
        acc[0] = acc[0] + (rn.x * rn.x + rn.y * rn.y);
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            if (i < ns) {
                acc[1 + 2 * i] = acc[1 + 2 * i] + (pv[i].x * dr.x + pv[i].y * dr.y);
                acc[2 + 2 * i] = acc[2 + 2 * i] + (pv[i].x * dr.y - pv[i].y * dr.x);
                if (mode == 0) {
                    acr[2 * i] = acr[2 * i] + (pv[i].x * rn.x + pv[i].y * rn.y);
                    acr[1 + 2 * i] = acr[1 + 2 * i] + (pv[i].x * rn.y - pv[i].y * rn.x);
                }
            }
        }
    }
    group_finish<1 + 2 * NS>(pd, tl.idx, acc);
    if (mode == 0) {
        __syncthreads();
        group_finish<2 * NS>(pd, tl.idx, acr, 1 + 2 * HH_MAX_S);
    }
}

} // namespace hh
