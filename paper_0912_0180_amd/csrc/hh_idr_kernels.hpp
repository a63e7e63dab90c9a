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

// s x s complex LU solve G c = m (G row major, in LDS), same algorithm and
// order per value as the host setup's dense LU, by one wave: lane 8 i + j holds
// entry (i, j) and, in every lane of a row, that row's right-hand side.  The
// pivot, row and column values come from their lanes, a lane known to the whole
// wave by v_readlane.  Returns false for an exactly singular pivot.  c: LDS.
__device__ inline double2 lane_get(double2 v, int l) { return cmk<double>(__shfl(v.x, l), __shfl(v.y, l)); }
__device__ inline double2 lane_one(double2 v, int l) { return cmk<double>(lane_value(v.x, l), lane_value(v.y, l)); }   // l uniform
__device__ __forceinline__ bool small_solve(const double2 *G, int s, const double2 *m, double2 *c)
{
    const int lane = threadIdx.x & 63, i = lane >> 3, j = lane & 7;
    const bool in = i < s && j < s;
    double2 a = in ? G[i * s + j] : cmk<double>(0.0, 0.0);
    double2 v = i < s ? m[i] : cmk<double>(0.0, 0.0);
    for (int k = 0; k < s; ++k) {
        // first maximum of |re| + |im| in column k from row k
        const double ab = fabs(a.x) + fabs(a.y);
        int p = k;
        double best = lane_value(ab, 9 * k);
        for (int r = k + 1; r < s; ++r) {
            const double w = lane_value(ab, 8 * r + k);
            if (w > best) {
                best = w;
                p = r;
            }
        }
        if (best == 0.0) return false;   // uniform over the wave, as p
        p = __builtin_amdgcn_readfirstlane(p);
        if (p != k) {
            const int from = i == k ? p : i == p ? k : i;
            a = lane_get(a, 8 * from + j);
            v = lane_get(v, 8 * from);
        }
        const double2 l = cdiv<double>(lane_get(a, 8 * i + k), lane_one(a, 9 * k));
        const double2 u = lane_get(a, 8 * k + j);
        if (i > k) a = j == k ? l : j > k ? csub<double>(a, cmul<double>(l, u)) : a;
    }
    // forward: row i takes the terms of columns 0 .. i - 1 in order
    for (int k = 0; k + 1 < s; ++k) {
        const double2 ck = lane_one(v, 8 * k), l = lane_get(a, 8 * i + k);
        if (i > k) v = csub<double>(v, cmul<double>(l, ck));
    }
    // backward: row r, columns r + 1 .. s - 1 in order, each c in its row's lanes
    for (int r = s - 1; r >= 0; --r) {
        double2 w = lane_one(v, 8 * r);
        for (int k = r + 1; k < s; ++k) w = csub<double>(w, cmul<double>(lane_one(a, 8 * r + k), lane_one(v, 8 * k)));
        w = cdiv<double>(w, lane_one(a, 9 * r));
        if (i == r) v = w;
    }
    if (j == 0 && i < s) c[i] = v;
    return true;
}

// Finaliser of the IDR passes.  The state block is copied to LDS by all
// threads, advanced there by the first wave (every lane the same scalars, row i
// of G and m in lane i) and copied back: a chain of dependent global accesses
// by one thread cost more than the sums.  Passes that reduce nothing in the
// current mode (omega in steps k >= 1) return after the copy.
__device__ __forceinline__ void idr_finalize(const ProbDev *pd, int kind, int ng)
{
    constexpr int SW = sizeof(SolveState) / 4, CW = sizeof(Ctrl) / 4;
    static_assert(sizeof(SolveState) % 4 == 0 && sizeof(Ctrl) % 4 == 0 && SW <= HH_FIN_WG && CW <= HH_FIN_WG, "one word per thread");
    __shared__ SolveState st;
    __shared__ Ctrl ct;
    __shared__ double res[4 * HH_MAX_S + 4];
    const int t = threadIdx.x;
    if (t < SW) ((uint32_t *)&st)[t] = ((const HH_GLOBAL uint32_t *)pd->st)[t];
    __syncthreads();
    const int s = st.s, max_mv = st.max_mv, hist_len = st.hist_len, guard = st.guard, stall = st.drift_stall;
    const double tol = st.tol, bnorm = st.bnorm, grow = st.drift_grow;
    double rel = st.rel, best_rel = st.best_rel;
    int phase = st.phase, reason = st.reason, mv = st.mv, it = st.it, best_mv = st.best_mv, startup = st.startup, kstep = st.kstep,
        oldest = st.oldest;
    double2 om = st.om_idr;
    if (kind != FIN_IDR_INIT && phase != PH_RUN) return;
    const int mode = startup >= 0 ? 0 : (kstep == 0 ? 1 : 2);
    if (kind == FIN_IDR_OMEGA) {
        if (mode == 2) return;
        reduce_partials<HH_FIN_WG / 64>(pd->part, pd->ngroup, ng, 0, 3, res);
    } else if (kind == FIN_IDR_STEP) {
        reduce_partials<HH_FIN_WG / 64>(pd->part, pd->ngroup, ng, 0, 1 + 2 * s, res);
        if (mode == 0) reduce_partials<HH_FIN_WG / 64>(pd->part, pd->ngroup, ng, 1 + 2 * HH_MAX_S, 2 * s, res + 1 + 2 * HH_MAX_S);
    }
    if (t < 64) {
        auto halt = [&](int why) {
            phase = PH_STOP;
            reason = why;
        };
        auto step = [&]() {
            if (kind == FIN_IDR_INIT) {
                phase = PH_RUN;
                reason = RS_NONE;
                startup = kstep = oldest = 0;
                om = cmk<double>(1.0, 0.0);
                best_rel = INFINITY;
                best_mv = mv;
                return;
            }
            if (kind == FIN_IDR_OMEGA) {
                mv += 1;
                const double2 tv = cmk<double>(res[0], res[1]);
                const double tt = res[2];
                if (!cfin(tv) || !isfinite(tt)) return halt(RS_NONFIN);
                if (tt == 0.0) return halt(RS_BREAK);
                om = cmk<double>(tv.x / tt, tv.y / tt);
                return;
            }
            // FIN_IDR_STEP
            if (mode == 2) mv += 1;
            if (mode != 0) it += 1;
            rel = sqrt(res[0]) / bnorm;
            if (t == 0 && pd->hist && mv - 1 < hist_len && mv >= 1) pd->hist[mv - 1] = rel;
            if (!isfinite(rel)) return halt(RS_NONFIN);
            if (rel < tol) return halt(RS_CONV);
            if (mv >= max_mv) return halt(RS_MAXMV);
            if (guard && drift(rel, mv, best_rel, best_mv, grow, stall)) return halt(RS_DRIFT);
            const int col = mode == 0 ? startup : oldest;
            const bool last = mode == 0 && startup + 1 == s;     // the start-up's m = P^H r
            if (t < s) {
                const double2 dm = cmk<double>(res[1 + 2 * t], res[2 + 2 * t]);
                st.G[t * s + col] = dm;
                if (mode != 0) st.m[t] = cadd<double>(st.m[t], dm);
                else if (last) st.m[t] = cmk<double>(res[1 + 2 * HH_MAX_S + 2 * t], res[2 + 2 * HH_MAX_S + 2 * t]);
            }
            if (mode == 0) {
                startup += 1;
                if (!last) return;
                startup = -1;
                oldest = kstep = 0;
            } else {
                oldest = oldest + 1 == s ? 0 : oldest + 1;
                kstep = kstep + 1 == s + 1 ? 0 : kstep + 1;
            }
            wave_order();           // G and m, a row per lane, to the lanes of the solve
            if (!small_solve(st.G, s, st.m, st.c)) halt(RS_BREAK);
        };
        step();
        wave_order();               // c, a row per lane, to the lane that mirrors it
        if (t == 0) {
            st.phase = phase;
            st.reason = reason;
            st.mv = mv;
            st.it = it;
            st.rel = rel;
            st.best_rel = best_rel;
            st.best_mv = best_mv;
            st.startup = startup;
            st.kstep = kstep;
            st.oldest = oldest;
            st.om_idr = om;
            mirror(ct, st);
        }
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
    double acc[1 + 2 * NS];
#pragma unroll
    for (int k = 0; k < 1 + 2 * NS; ++k) acc[k] = 0.0;
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
            }
        }
    }
    group_finish<1 + 2 * NS>(pd, tl.idx, acc);
    if (mode == 0) {
        // P^H r, from this thread's own r and P again: the s start-up steps
        // read them twice so that the other steps hold fewer registers
        double acr[2 * NS];
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            acr[2 * i] = acr[1 + 2 * i] = 0.0;
            if (i < ns && p < N) {
                const double2 pv = ldg(Pm, (int64_t)i * N + p), rn = ldg(r, p);
                acr[2 * i] = acr[2 * i] + (pv.x * rn.x + pv.y * rn.y);
                acr[1 + 2 * i] = acr[1 + 2 * i] + (pv.x * rn.y - pv.y * rn.x);
            }
        }
        group_finish<2 * NS>(pd, tl.idx, acr, 1 + 2 * HH_MAX_S);
    }
}

} // namespace hh
