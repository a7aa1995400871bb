// The V-cycle on mid-size 1-D and 2-D levels in two launches per level: one on
// the way down (pre-smoothing, defect, restriction of the iterate and of the
// defect, coarse right-hand side) and one on the way up (prolongation,
// post-smoothing), FP64 and FP32, with the per-node arithmetic of the launched
// kernels.
//
// What bounds these levels: the chain of dependent launches.  A colour pass over
// 65^2 .. 513^2 nodes takes 4 to 5 us as a launch of its own, of which the solve
// is under one; the level needs 2 (nu1 + nu2) of them and four more for defect
// and transfers.  Here a work-group loads its tile with a halo into LDS once and
// makes all the passes there with barriers (a pass of about 1000 cycles), every
// thread keeping its nodes in registers as in cycle_wg.h.  The halo nodes are
// recomputed by each tile that needs them: after k colour passes the values k
// nodes inside the rim of the loaded box are those of the whole-level sweep, so
// the results do not depend on the tiling.  A pass writes another array than it
// reads (tiles of one launch run in any order): down reads x and writes y, up
// reads y and writes x.
#pragma once

#include "cycle_wg.h"

namespace rs {

// One node per thread and colour: boxes of up to 33^2 nodes, in 2-D 16^2 owned
// for V(2,2) going down and 24^2 going up.  (Two nodes per thread and boxes of
// 47^2 spilled: 53 us for the finest level of the 513^2 vGM slice going down
// against 2 x 15 here.)
constexpr int kTileThreads = 576;

template <typename T>
struct TileArgs {
    WgGeo g;              // the level (patch range of the level)
    int dim;
    int own[2], halo;     // owned nodes per tile and axis (even), halo (even)
    int tiles0;           // tiles along axis 0
    int ns;               // sweeps
    const T *x;           // iterate in
    T *y;                 // iterate out
    const T *rhs, *K, *pb;
    const double *beta;
    const unsigned char *soil;
    double lambdaU;
    // next coarser level: restricted iterate, right-hand side, first iterate
    // (down); corrected iterate (up: xc - bar is interpolated)
    T *bar, *rhsc, *xc;
    const T *Kc, *pbc;
    const double *betac;
    const unsigned char *soilc;
    unsigned long long *norm;   // max-norm of the defect over the level (or null)
};

// Tile phases: sweeps only, down, up.
enum : int { kTileSweep = 0, kTileDown = 1, kTileUp = 2 };

// One tile (blockIdx.x).
template <class Op>
__device__ __forceinline__ void tile_run(const TileArgs<typename Op::T> &A, int phase,
                                         const typename Op::Env &e, typename Op::T *lds)
{
    typedef typename Op::T T;
    constexpr int DIM = Op::DIM, NQ = 2 * DIM;
    const WgGeo &g = A.g;
    const WgLevel<DIM> v = wg_level<DIM>(g, 0), vc = wg_level<DIM>(g, 1);
    const int tid = threadIdx.x;
    constexpr int nthreads = kTileThreads;
    // owned range and loaded box of the tile (even origins, odd box extents:
    // the box's lexicographic parity is the colour)
    int a0[3] = {0, 0, 0}, b0[3] = {0, 0, 0}, o[3] = {0, 0, 0}, oe[3] = {0, 0, 0};
    WgLevel<DIM> w = v;   // shape of the box
    {
        int t[2];
        t[1] = DIM > 1 ? (int)blockIdx.x / A.tiles0 : 0;
        t[0] = DIM > 1 ? (int)blockIdx.x - t[1] * A.tiles0 : (int)blockIdx.x;
        w.N = 1;
#pragma unroll
        for (int l = 0; l < DIM; ++l) {
            a0[l] = t[l] * A.own[l];
            b0[l] = a0[l] + A.own[l] >= v.n[l] - 1 ? v.n[l] : a0[l] + A.own[l];
            o[l] = max(a0[l] - A.halo, 0);
            oe[l] = min(a0[l] + A.own[l] + A.halo, v.n[l] - 1);
            w.n[l] = oe[l] - o[l] + 1;
            w.N *= w.n[l];
        }
        w.s[1] = w.n[0] + 1;
        w.s[2] = 0;
        w.base = 1 + (DIM > 1 ? w.s[1] : 0);
        w.size = 2 * w.base + (w.n[0] - 1) + (DIM > 1 ? (w.n[1] - 1) * w.s[1] : 0);
        w.r0 = 1.0f / (float)w.n[0];
    }
    T *lx = lds, *lk = lds + w.size;   // iterate; K*, later the defect
    // coarse box: nodes o/2 .. oe/2 (the box origin is even), one unused column
    const int cn0 = ((oe[0] - o[0]) >> 1) + 1, cn1 = DIM > 1 ? ((oe[1] - o[1]) >> 1) + 1 : 1;
    const int cs1 = cn0 + 1, cbase = 1 + (DIM > 1 ? cs1 : 0);
    T *lc = lk + w.size;               // restricted iterate / coarse correction
    int so[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) so[q] = (q & 1) ? w.s[q >> 1] : -w.s[q >> 1];

    typename Op::Node nd[2];
    bool on[2], has[2], mine[2];
    int c[2][3];
    // the coarse node this thread evaluates (down): owned coarse nodes
    const int q0 = a0[0] >> 1, q1 = DIM > 1 ? a0[1] >> 1 : 0;
    const int m0 = ((b0[0] - 1) >> 1) - q0 + 1, m1 = DIM > 1 ? ((b0[1] - 1) >> 1) - q1 + 1 : 1;
    {
        T Kn[2][NQ], Kc[2];
#pragma unroll
        for (int col = 0; col < 2; ++col) {
            typename Op::Node &q = nd[col];
            const int lin = 2 * tid + col;
            has[col] = lin < w.N;
            int *cc = c[col];
            wg_ijk<DIM>(w, has[col] ? lin : 0, cc);
            q.p = wg_pos<DIM>(w, cc);
            bool rim = false, own = has[col];
#pragma unroll
            for (int l = 0; l < DIM; ++l) {
                const int i = cc[l] + o[l];
                rim = rim | (cc[l] == 0 && i > 0) | (i == oe[l] && i < v.n[l] - 1);
                own = own & (i >= a0[l]) & (i < b0[l]);
                cc[l] = i;
            }
            mine[col] = own;
            on[col] = has[col] & !rim;
            const int at = wg_mem<DIM>(g, v, cc);
            Kc[col] = A.K[at];
            q.x = A.x[at];
            q.g = A.rhs[at];
            q.b = Op::SINK ? (T)A.beta[cc[DIM - 1]] : T(0);
            if constexpr (sizeof(T) == 8) {
                q.soil = 0;
                if constexpr (Op::MODEL == kMulti) q.soil = A.soil[at];
            } else {
                q.base.psi = A.pb[at];
            }
        }
        if (phase == kTileUp) {
            for (int t = tid; t < cn0 * cn1; t += nthreads) {
                const int j = DIM > 1 ? (int)(((float)t + 0.5f) / (float)cn0) : 0;
                const int i = t - j * cn0;
                const int cc[3] = {(o[0] >> 1) + i, DIM > 1 ? (o[1] >> 1) + j : 0, 0};
                const int at = wg_mem<DIM>(g, vc, cc);
                lc[cbase + i + j * cs1] = A.xc[at] - A.bar[at];
            }
        }
        // unused columns and rows hold zeros (read under zero coefficients)
        for (int t = tid; t < 2 * w.size; t += nthreads) lds[t] = T(0);
        __syncthreads();
#pragma unroll
        for (int col = 0; col < 2; ++col)
            if (has[col]) {
                lx[nd[col].p] = nd[col].x;
                lk[nd[col].p] = Kc[col];
            }
        __syncthreads();
#pragma unroll
        for (int col = 0; col < 2; ++col)
#pragma unroll
            for (int t = 0; t < NQ; ++t) Kn[col][t] = lk[nd[col].p + so[t]];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int col = 0; col < 2; ++col) {
            typename Op::Node &q = nd[col];
            const int *cc = c[col];
            on[col] = on[col] && !wg_dirichlet<DIM>(g, v, cc);
            T mii = T(0);
#pragma unroll
            for (int l = 0; l < DIM; ++l) {
                const bool lo = cc[l] == 0, hi = cc[l] == v.n[l] - 1;
                const double cf = (lo || hi ? 1.0 : 0.5) * g.ih2[l];
                const T cl = lo ? T(0) : (T)cf, ch = hi ? T(0) : (T)cf;
                const T kl = Kc[col] + Kn[col][2 * l], kh = Kc[col] + Kn[col][2 * l + 1];
                q.m[2 * l] = cl * kl;
                q.m[2 * l + 1] = ch * kh;
                mii = fma(cl, kl, mii);   // as the launched kernels' sum contracts
                mii = fma(ch, kh, mii);
            }
            if (e.L.kappa_rule == kKappaConst) q.kap = (T)e.L.kappa;
            else if (e.L.kappa_rule == kKappaRel) q.kap = (T)e.L.kappa * mii;
            else q.kap = wg_remark<DIM, T>(g, v, cc, col, (T)A.lambdaU, q.m);
            if constexpr (sizeof(T) == 4) {
                q.base = base_of<Op::MODEL>(e.L, q.base.psi);
                base_room<Op::MODEL>(e.L, q.base, q.up, q.down);
                q.ab = Op::SINK ? feddes_value32(e.L, q.base.psi) : 0.0f;
            }
            Op::coefficients(e, q, mii);
        }
        if (phase == kTileUp) {
#pragma unroll
            for (int col = 0; col < 2; ++col) {
                typename Op::Node &q = nd[col];
                int oc[2][2] = {{0, 0}, {0, 0}};
                T wt[2][2];
#pragma unroll
                for (int l = 0; l < DIM; ++l) {
                    const int i = c[col][l] - o[l];
                    const bool odd = i & 1;
                    oc[l][0] = (i >> 1) * (l ? cs1 : 1);
                    oc[l][1] = ((i + 1) >> 1) * (l ? cs1 : 1);
                    wt[l][0] = odd ? T(0.5) : T(1);
                    wt[l][1] = odd ? T(0.5) : T(0);
                }
                T sum = T(0);
#pragma unroll
                for (int t1 = 0; t1 < (DIM > 1 ? 2 : 1); ++t1)
#pragma unroll
                    for (int t0 = 0; t0 < 2; ++t0)
                        sum += wt[0][t0] * (DIM > 1 ? wt[1][t1] : T(1)) *
                               lc[cbase + oc[0][t0] + (DIM > 1 ? oc[1][t1] : 0)];
                // the rim takes the correction too: its neighbours read it
                if (has[col] && !wg_dirichlet<DIM>(g, v, c[col])) {
                    q.x += sum;
                    lx[q.p] = q.x;
                }
            }
            __syncthreads();
        }
    }
    for (int sw = 0; sw < A.ns; ++sw) {
#pragma unroll
        for (int col = 0; col < 2; ++col) {
            typename Op::Node &q = nd[col];
            if (on[col]) {
                T f = q.g;
#pragma unroll
                for (int t = 0; t < NQ; ++t) f += q.m[t] * lx[q.p + so[t]];
                f += q.kap * q.x;
                q.x = Op::solve(e, q, f);
                lx[q.p] = q.x;
            }
            __syncthreads();
        }
    }
#pragma unroll
    for (int col = 0; col < 2; ++col)
        if (mine[col]) A.y[wg_mem<DIM>(g, v, c[col])] = nd[col].x;
    if (phase != kTileDown) return;

    // the coarse node of this thread: its K* (and neighbours'), loaded ahead
    const int ncoarse = m0 * m1;
    const bool eval = tid < ncoarse;   // at most (own / 2 + 1)^DIM < nthreads nodes
    typename Op::Node qc;
    int ccl[3] = {0, 0, 0}, atc = 0;
    T Kcc = T(0), Kcn[NQ];
    if (eval) {
        const int j = DIM > 1 ? (int)(((float)tid + 0.5f) / (float)m0) : 0;
        ccl[0] = q0 + tid - j * m0;
        if (DIM > 1) ccl[1] = q1 + j;
        atc = wg_mem<DIM>(g, vc, ccl);
        Kcc = A.Kc[atc];
#pragma unroll
        for (int t = 0; t < NQ; ++t) {
            int d[3] = {ccl[0], ccl[1], ccl[2]};
            d[t >> 1] += (t & 1) ? 1 : -1;
            const bool in = d[t >> 1] >= 0 && d[t >> 1] < vc.n[t >> 1];
            Kcn[t] = A.Kc[in ? wg_mem<DIM>(g, vc, d) : atc];
        }
        qc.b = Op::SINK ? (T)A.betac[ccl[DIM - 1]] : T(0);
        if constexpr (sizeof(T) == 8) {
            qc.soil = 0;
            if constexpr (Op::MODEL == kMulti) qc.soil = A.soilc[atc];
        } else {
            qc.base = base_of<Op::MODEL>(e.L, A.pbc[atc]);
        }
    }
    // defect (0 at Dirichlet nodes) into the K* box
    double nrm = 0.0;
#pragma unroll
    for (int col = 0; col < 2; ++col) {
        typename Op::Node &q = nd[col];
        T md = T(0);
#pragma unroll
        for (int t = 0; t < NQ; ++t) md += q.m[t] * (q.x - lx[q.p + so[t]]);
        const T r = on[col] ? q.g - Op::template apply<true>(e, q, q.x, md) : T(0);
        if (has[col]) lk[q.p] = r;
        if (mine[col]) {
            const double ar = fabs((double)r);
            nrm = (ar > nrm || ar != ar) ? ar : nrm;
        }
    }
    __syncthreads();
    if (A.norm) {
        const double m = block_max(nrm);
        if (tid == 0) {
            const unsigned long long bits = (unsigned long long)__double_as_longlong(m);
            if (bits > __hip_atomic_load(A.norm, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                atomicMax(A.norm, bits);
        }
    }
    // full weighting on the owned coarse nodes and one ring around them: the
    // iterate's into lc, the defect's into ld
    T *ld = lc + 2 * cbase + (cn0 - 1) + (DIM > 1 ? (cn1 - 1) * cs1 : 0);
    const int r0a = max(q0 - 1, 0), r0b = min(q0 + m0, vc.n[0] - 1);
    const int r1a = DIM > 1 ? max(q1 - 1, 0) : 0, r1b = DIM > 1 ? min(q1 + m1, vc.n[1] - 1) : 0;
    const int rn0 = r0b - r0a + 1, rn = rn0 * (r1b - r1a + 1);
    for (int t = tid; t < 2 * rn; t += nthreads) {
        const bool def = t >= rn;
        const int t1 = def ? t - rn : t;
        const int j = DIM > 1 ? (int)(((float)t1 + 0.5f) / (float)rn0) : 0;
        const int cc[3] = {r0a + t1 - j * rn0, DIM > 1 ? r1a + j : 0, 0};
        const T *src = def ? lk : lx;
        int of[2][3];
#pragma unroll
        for (int l = 0; l < DIM; ++l) {
            const int F = (2 * cc[l] - o[l]) * w.s[l];
            of[l][0] = F + (cc[l] == 0 ? w.s[l] : -w.s[l]);
            of[l][1] = F;
            of[l][2] = F + (2 * cc[l] == v.n[l] - 1 ? -w.s[l] : w.s[l]);
        }
        constexpr int N1 = DIM > 1 ? 3 : 1;
        T tap[N1][3];
#pragma unroll
        for (int o1 = 0; o1 < N1; ++o1)
#pragma unroll
            for (int o0 = 0; o0 < 3; ++o0)
                tap[o1][o0] = src[w.base + of[0][o0] + (DIM > 1 ? of[DIM > 1 ? 1 : 0][o1] : 0)];
        __builtin_amdgcn_sched_barrier(0);
        const T wt[3] = {T(0.25), T(0.5), T(0.25)};
        T sum = T(0);
#pragma unroll
        for (int o1 = 0; o1 < N1; ++o1)
#pragma unroll
            for (int o0 = 0; o0 < 3; ++o0) sum += wt[o0] * (DIM > 1 ? wt[o1] : T(1)) * tap[o1][o0];
        if (wg_dirichlet<DIM>(g, vc, cc)) sum = def ? T(0) : tap[N1 / 2][1];
        (def ? ld : lc)[cbase + cc[0] - (o[0] >> 1) + (DIM > 1 ? (cc[1] - (o[1] >> 1)) * cs1 : 0)] =
            sum;
    }
    __syncthreads();
    if (eval) {
        const int p = cbase + ccl[0] - (o[0] >> 1) + (DIM > 1 ? (ccl[1] - (o[1] >> 1)) * cs1 : 0);
        const T xb = lc[p];
        T gc = ld[p];
        if (!wg_dirichlet<DIM>(g, vc, ccl)) {
            T md = T(0);
#pragma unroll
            for (int l = 0; l < DIM; ++l) {
                const bool lo = ccl[l] == 0, hi = ccl[l] == vc.n[l] - 1;
                const double cf = (lo || hi ? 1.0 : 0.5) * ldexp(g.ih2[l], -2);
                const int st = l ? cs1 : 1;
                const T ml = lo ? T(0) : (T)cf * (Kcc + Kcn[2 * l]);
                const T mh = hi ? T(0) : (T)cf * (Kcc + Kcn[2 * l + 1]);
                md += ml * (xb - (lo ? xb : lc[p - st]));
                md += mh * (xb - (hi ? xb : lc[p + st]));
            }
            gc = Op::template apply<true>(e, qc, xb, md) + gc;
        }
        A.bar[atc] = xb;
        A.rhsc[atc] = gc;
        A.xc[atc] = xb;
    }
}

// Tile shape of a level for a phase with the given halo: the loaded box has at
// most 2 kTileThreads - 1 nodes, near-square; false if the halo leaves too little.
inline bool tile_shape(const Geo &g, int halo, int own[2], int tiles[2])
{
    const int room = 2 * kTileThreads - 1;
    if (g.dim == 1) {
        int e = room;
        if (e % 2 == 0) --e;
        own[0] = (e - 1 - 2 * halo) & ~1;
        own[1] = 1;
        if (own[0] < 2) return false;
        own[0] = own[0] < g.n[0] - 1 ? own[0] : g.n[0] - 1;
        tiles[0] = (g.n[0] - 1 + own[0] - 1) / own[0];
        tiles[1] = 1;
        return true;
    }
    int side = 1;
    while ((side + 2) * (side + 2) <= room) side += 2;
    int e[2] = {side, side};
    for (int l = 0; l < 2; ++l)
        if (g.n[l] < e[l]) {   // a short axis is loaded whole, the other one longer
            e[l] = g.n[l];
            int o = room / e[l];
            if (o % 2 == 0) --o;
            e[1 - l] = o;
            break;
        }
    for (int l = 0; l < 2; ++l) {
        own[l] = e[l] >= g.n[l] ? g.n[l] - 1 : e[l] - 1 - 2 * halo;
        if (own[l] < 2) return false;
        tiles[l] = (g.n[l] - 1 + own[l] - 1) / own[l];
    }
    // one owned coarse node per thread (long boxes on short axes)
    return (own[0] / 2 + 1) * (own[1] / 2 + 1) <= kTileThreads;
}

// LDS words of a tile: two boxes and two coarse boxes of the largest extents.
inline size_t tile_lds_words(int dim, const Geo &g, int halo, const int own[2])
{
    size_t e[2] = {1, 1};
    for (int l = 0; l < dim; ++l) {
        e[l] = (size_t)own[l] + 2 * (size_t)halo + 1;
        if (e[l] > (size_t)g.n[l]) e[l] = (size_t)g.n[l];
    }
    const size_t box = (e[0] + 1) * (e[1] + (dim > 1 ? 2 : 0)) + 4;
    const size_t c0 = (e[0] - 1) / 2 + 1, c1 = (e[1] - 1) / 2 + 1;
    return 2 * box + 2 * ((c0 + 1) * (c1 + (dim > 1 ? 2 : 0)) + 4);
}

void launch_tile(const TileArgs<double> &A, int phase, int blocks, size_t words,
                 const Law &law, double a, hipStream_t s);
void launch_tile32(const TileArgs<float> &A, int phase, int blocks, size_t words,
                   const Law32 &law, float a, hipStream_t s);

}  // namespace rs
