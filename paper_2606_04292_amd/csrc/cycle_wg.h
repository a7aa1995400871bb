// The V-cycle on the small levels of a grid in one work-group, FP64 (the full
// variable) and FP32 (the correction equation), with the per-node arithmetic
// of the launched kernels.
//
// What bounds it: a chain of dependent phases (colour passes, defect,
// transfers), each as long as one pointwise solve plus a barrier; on a few
// hundred nodes no unit of the chip is busy.  So the phases are made short:
//  - every level lives in LDS as a box with one unused column and row between
//    rows and planes (zeros), so a node's neighbours are at fixed distances
//    and a missing one reads any finite value under a zero coefficient;
//  - a thread owns the same red and black nodes for a whole visit of a level
//    and keeps their face coefficients, diagonal and its reciprocal,
//    right-hand side and own value in registers: a colour pass reads 2 DIM
//    neighbour values, solves and writes one value.  Power terms of the law are
//    not carried from solve to solve: scaled on from one to the next, their
//    roundings would add up over a solve's history, and a sweep's result would
//    depend on it (they save 12 % of a 257-node column's step);
//  - nodes of one colour are the even (odd) positions of the lexicographic
//    order (all axes have an odd node count), so slots map to nodes without
//    padding; levels of at most 64 nodes per colour run on one wave without
//    barriers (LDS operations of a wave complete in order).
// One wave issues an instruction every 6 to 7 cycles (dependent or not, FP64
// or FP32; measured with chains of multiply-adds), a barrier of nine waves
// takes 76 cycles and an LDS round trip about 70, so a colour pass of 1000
// cycles is the instruction count of its solve.  Steps against the same cycle
// on generic pointers with every coefficient formed anew in each pass: 257-node
// vGM column (three Newton steps per solve) 3.39 -> 2.36 ms for two steps,
// 2049-node Haverkamp column V(5,5) 7.8 -> 4.8 ms for three, 65^3 block (its
// 9^3 level and below) 8.75 -> 7.35 ms for two.
#pragma once

#include "rs_internal.h"
#include "soil_device.h"
#include "soil_mp.h"
#include "grid_device.h"

namespace rs {

constexpr int kWgMaxLev = 12;        // levels of one cycle (2049 nodes on the shortest axis)
// Cycles of one launch of the whole-grid solve at most, and sweeps (on all levels;
// one cycle at least): a sweep takes 2 to 5 us with three Newton steps, so a launch
// some 40 ms at most unless one cycle alone is longer.
constexpr int kWgSolveCycles = 60;
constexpr int kWgSolveSweeps = 8192;
// Three waves per SIMD, so a lane may hold 168 registers (2-D and most 3-D levels
// take one node per thread and colour; with two the 3-D kernels spill).
constexpr int kWgMaxThreads = 768;

// The geometry of the cycle's top level that the kernels read (few scalars).
struct WgGeo {
    int n[3];
    int xs;          // Geo::xs of every level
    int dmask;       // bit f: face f is Dirichlet
    int pface;       // patch face or -1, and its range
    int plo[2], phi[2];
    double ih2[3];
};

inline WgGeo wg_geo(const Geo &g)
{
    WgGeo w;
    w.xs = g.xs;
    w.dmask = 0;
    for (int f = 0; f < 2 * g.dim; ++f) w.dmask |= (g.bc[f] == kBcDirichlet ? 1 : 0) << f;
    w.pface = g.pface;
    for (int t = 0; t < 2; ++t) {
        w.plo[t] = g.plo[t];
        w.phi[t] = g.phi[t];
    }
    for (int l = 0; l < 3; ++l) {
        w.n[l] = g.n[l];
        w.ih2[l] = g.ih2[l];
    }
    return w;
}

// A level of the cycle and its LDS box.
template <int DIM>
struct WgLevel {
    int n[3], N;
    int s[3];        // distances along the axes: 1, n0 + 1, (n0 + 1)(n1 + 1)
    int base, size;  // box position of node (0, 0, 0), positions of the box
    int lev;
    float r0, r1;    // 1 / n0, 1 / n1
};

// Level top + s of a cycle whose top level is g (coarsening halves every axis).
template <int DIM>
__host__ __device__ __forceinline__ WgLevel<DIM> wg_level(const WgGeo &g, int s)
{
    WgLevel<DIM> v;
    v.lev = s;
    v.N = 1;
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        v.n[l] = l < DIM ? ((g.n[l] - 1) >> s) + 1 : 1;
        v.N *= v.n[l];
    }
    v.s[0] = 1;
    v.s[1] = v.n[0] + 1;
    v.s[2] = (v.n[0] + 1) * (v.n[1] + 1);
    v.base = 1 + (DIM > 1 ? v.s[1] : 0) + (DIM > 2 ? v.s[2] : 0);
    v.size = 2 * v.base + (v.n[0] - 1) + (DIM > 1 ? (v.n[1] - 1) * v.s[1] : 0) +
             (DIM > 2 ? (v.n[2] - 1) * v.s[2] : 0);
    v.r0 = 1.0f / (float)v.n[0];
    v.r1 = 1.0f / (float)v.n[1];
    return v;
}

// (i, j, k) of position lin < 2^12 of the lexicographic order (the quotient of
// lin + 1/2 by n < 2^12 is at least 1/(2n) away from an integer, far more than
// the rounding of the product).
template <int DIM>
__device__ __forceinline__ void wg_ijk(const WgLevel<DIM> &v, int lin, int c[3])
{
    c[0] = lin;
    c[1] = c[2] = 0;
    if (DIM > 1) {
        const int row = (int)(((float)lin + 0.5f) * v.r0);
        c[0] = lin - row * v.n[0];
        c[1] = row;
        if (DIM > 2) {
            c[2] = (int)(((float)row + 0.5f) * v.r1);
            c[1] = row - c[2] * v.n[1];
        }
    }
}

template <int DIM>
__device__ __forceinline__ int wg_pos(const WgLevel<DIM> &v, const int c[3])
{
    return v.base + c[0] + (DIM > 1 ? c[1] * v.s[1] : 0) + (DIM > 2 ? c[2] * v.s[2] : 0);
}

// Position of node c in a level's row layout in memory.
template <int DIM>
__device__ __forceinline__ int wg_mem(const WgGeo &g, const WgLevel<DIM> &v, const int c[3])
{
    const int x = g.xs ? (c[0] >> 1) + (c[0] & 1) * ((v.n[0] + 1) >> 1) : c[0];
    return x + v.n[0] * (c[1] + v.n[1] * c[2]);
}

template <int DIM>
__device__ __forceinline__ bool wg_dirichlet(const WgGeo &g, const WgLevel<DIM> &v,
                                             const int c[3])
{
    bool dir = false;
#pragma unroll
    for (int l = 0; l < DIM; ++l)
        dir = dir | ((c[l] == 0) & ((g.dmask >> (2 * l)) & 1)) |
              ((c[l] == v.n[l] - 1) & ((g.dmask >> (2 * l + 1)) & 1));
    if (DIM > 1 && g.pface >= 0) {
        const int ax = g.pface >> 1, m = (1 << v.lev) - 1;
        const int cp = ax == 0 ? c[0] : (ax == 1 ? c[1] : c[2]);
        const int t0 = ax == 0 ? c[1] : c[0];
        const int t1 = ax == 2 ? c[1] : c[2];
        const int at = (g.pface & 1) ? (ax == 0 ? v.n[0] : (ax == 1 ? v.n[1] : v.n[2])) - 1 : 0;
        bool in = (cp == at) & (t0 >= ((g.plo[0] + m) >> v.lev)) & (t0 <= (g.phi[0] >> v.lev));
        if (DIM == 3) in = in & (t1 >= ((g.plo[1] + m) >> v.lev)) & (t1 <= (g.phi[1] >> v.lev));
        dir = dir | in;
    }
    return dir;
}

// Diagonal shift of an unknown by the Remark's rule: lambda minus the row sum
// of U over unknown neighbours (every neighbour of a red node), lambda at
// black nodes.
template <int DIM, typename T>
__device__ __forceinline__ T wg_remark(const WgGeo &g, const WgLevel<DIM> &v, const int c[3],
                                       int colour, T lambdaU, const T *m)
{
    T usum = T(0);
    if (colour == 0) {
#pragma unroll
        for (int q = 0; q < 2 * DIM; ++q) {
            int d[3] = {c[0], c[1], c[2]};
            d[q >> 1] += (q & 1) ? 1 : -1;
            if (d[q >> 1] >= 0 && d[q >> 1] < v.n[q >> 1] && !wg_dirichlet<DIM>(g, v, d))
                usum += m[q];
        }
    }
    return lambdaU - usum;
}

// FP64 operations of a node: the step system N(psi) = g.
template <int MODEL_, bool SINK_, int DIM_>
struct WgOp64 {
    static constexpr int MODEL = MODEL_, DIM = DIM_;
    static constexpr bool SINK = SINK_;
    typedef double T;
    struct Env {
        const Law &L;
        const Law *soils;   // kMulti: the soil table (LDS)
        double a;
    };
    struct Node {
        T m[2 * DIM], c, ic, kap, x, g, b;
        int p, soil;
    };
    static __device__ __forceinline__ void coefficients(const Env &e, Node &nd, T mii)
    {
        nd.c = e.L.xi + nd.kap + mii;
        nd.ic = MODEL == kLinear ? 0.0 : rcp_nr(nd.c);
    }
    // N_i(psi) = a theta(x) + sink + (xi x + md), md = sum_j m_ij (x - psi_j), with
    // the roundings apply_N_t has in the launched kernels (LAUNCHED: tiles, norms)
    // and had in the one-work-group cycle (its last sum contracts differently there)
    template <bool LAUNCHED = false>
    static __device__ __forceinline__ T apply(const Env &e, const Node &nd, T x, T md)
    {
#pragma clang fp contract(off)
        T th;
        if constexpr (MODEL == kMulti) th = theta_only(e.soils[nd.soil], x);
        else th = theta_only_t<MODEL>(e.L, x);
        const T rest = fma(e.L.xi, x, md);
        if (SINK) {
            T fa, dfa;
            feddes(e.L, x, fa, dfa);
            return fma(e.a, th, nd.b * fa) + rest;
        }
        if (LAUNCHED || MODEL == kMulti) return fma(e.a, th, rest);
        return e.a * th + rest;
    }
    static __device__ __forceinline__ T solve(const Env &e, Node &nd, T f)
    {
        if constexpr (MODEL == kMulti) {
            const Law &Ls = e.soils[nd.soil];
            return local_solve_soil_ic<SINK, 0>(Ls, e.a, nd.b, nd.c, nd.ic, f, nd.x);
        } else {
            return local_solve_ic<MODEL, SINK, 0>(e.L, e.a, nd.b, nd.c, nd.ic, f, nd.x);
        }
    }
    // moved by more than 4 ulp
    static __device__ __forceinline__ bool moved(T x1, T x0)
    {
        return fabs(x1 - x0) > 8.8817841970012523e-16 * fabs(x0);   // 4 ulp (2^-50 |x0|)
    }
};

// FP32 operations of a node: the correction equation about psi_b.
template <int MODEL_, bool SINK_, int DIM_>
struct WgOp32 {
    static constexpr int MODEL = MODEL_, DIM = DIM_;
    static constexpr bool SINK = SINK_;
    typedef float T;
    struct Env {
        const Law32 &L;
        float a;
    };
    struct Node {
        T m[2 * DIM], c, ic, kap, x, g, b;
        Base base;
        T up, down, ab;
        int p;
    };
    static __device__ __forceinline__ void coefficients(const Env &e, Node &nd, T mii)
    {
        nd.c = e.L.xi + nd.kap + mii;
        nd.ic = f_rcp(nd.c);
    }
    template <bool LAUNCHED = false>
    static __device__ __forceinline__ T apply(const Env &e, const Node &nd, T x, T md)
    {
        T dth, slope;
        dtheta32<MODEL>(e.L, nd.base, x, dth, slope);
        T s = e.a * dth;
        if (SINK) {
            T da, ds;
            dfeddes32(e.L, nd.base.psi, x, da, ds);
            s += nd.b * da;
        }
        return s + (e.L.xi * x + md);
    }
    static __device__ __forceinline__ T solve(const Env &e, Node &nd, T f)
    {
        return local_solve32_ic<MODEL, SINK>(e.L, e.a, nd.b, nd.c, nd.ic, f, nd.base, nd.up,
                                             nd.down, nd.ab, nd.x);
    }
    static __device__ __forceinline__ bool moved(T x1, T x0)
    {
        return !(fabsf(x1 - x0) <= 4.0f * 1.1920929e-7f * fabsf(x1));
    }
};

// Memory of one level: K* and, FP32, the base state; root density, soil index.
template <typename T>
struct WgMem {
    const T *K, *pb;
    const double *beta;
    const unsigned char *soil;
    double lambdaU;
};

// The cycle: levels from the top one (geometry g) down, smoothing counts, the
// top level's iterate (in and out) and right-hand side in memory.
template <typename T>
struct WgCycle {
    WgGeo g;
    int levels, nu1, nu2, nuc;
    T *x;
    const T *rhs;
    // the coarsest level takes all its sweeps, also once no value moves (the
    // sweeps of one level on their own, levels = 1)
    int all;
};

// Level memory as kernel arguments.
template <typename T>
struct WgMems {
    WgMem<T> lv[kWgMaxLev];
    __device__ __forceinline__ const WgMem<T> &operator()(int s) const { return lv[s]; }
};

// LDS of the cycle: per level the iterate, K*, right-hand side, restricted
// iterate (then the correction) and, FP32, the base state; one defect box of the
// top level's size.
template <typename T, int DIM>
__host__ __device__ __forceinline__ int wg_words(const WgGeo &g, int s)
{
    return wg_level<DIM>(g, s).size * (sizeof(T) == 4 ? 5 : 4);
}

// At most 148 KB (FP64, a 2049-node column) of 160.
template <typename T, int DIM>
inline size_t wg_lds_bytes(const WgGeo &g, int levels)
{
    size_t w = 0;
    for (int s = 0; s < levels; ++s) w += (size_t)wg_words<T, DIM>(g, s);
    return sizeof(T) * (w + (size_t)wg_level<DIM>(g, 0).size);
}

template <typename T, int DIM>
struct WgBox {
    T *x, *K, *g, *bar;
    T *pb;   // FP32: base state
};

template <typename T, int DIM>
__device__ __forceinline__ WgBox<T, DIM> wg_box(T *lds, int off, const WgLevel<DIM> &v)
{
    WgBox<T, DIM> b;
    T *q = lds + off;
    b.x = q;
    b.K = q + v.size;
    b.g = q + 2 * v.size;
    b.bar = q + 3 * v.size;
    b.pb = q + 4 * v.size;
    return b;
}

template <bool WAVE>
__device__ __forceinline__ void wg_sync()
{
    if (WAVE) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    } else {
        __syncthreads();
    }
}

// One visit of level s of the cycle by nthreads threads (S nodes per colour
// and thread).  Down (up = false): right-hand side (levels below the top),
// sweeps, defect and its restriction to level s + 1; the coarsest level has
// only the sweeps.  Up: the coarser level's correction, sweeps.  A level that
// is left for good holds its correction x - bar in bar (the top level's x
// goes back to memory unless the cycle repeats, and with norm set its defect's
// max-norm into *norm).  norm_only: just that norm, of the top level's iterate
// as it is.  The LDS reads of a step are issued together, ahead of
// its arithmetic (a read takes about 70 cycles: waited for one by one, the 54
// taps of a 3-D restriction took 6000).
template <class Op, int S, bool WAVE>
__device__ __forceinline__ void wg_visit(const WgCycle<typename Op::T> &A,
                                         const WgMem<typename Op::T> &M,
                                         const typename Op::Env &e, int s, bool up, int nthreads,
                                         typename Op::T *lds, int off, typename Op::T *dbox,
                                         double *norm = nullptr, bool norm_only = false)
{
    typedef typename Op::T T;
    constexpr int DIM = Op::DIM, NQ = 2 * DIM;
    const WgGeo &g = A.g;
    const WgLevel<DIM> v = wg_level<DIM>(g, s);
    const WgBox<T, DIM> B = wg_box<T, DIM>(lds, off, v);
    const WgLevel<DIM> vc = wg_level<DIM>(g, s + 1);
    const int noff = off + wg_words<T, DIM>(g, s);
    const WgBox<T, DIM> C = wg_box<T, DIM>(lds, noff, vc);
    const bool last = s == A.levels - 1;
    const int tid = threadIdx.x;
    int so[NQ];
    double ih[DIM];   // 1/h^2: h doubles exactly from level to level
#pragma unroll
    for (int q = 0; q < NQ; ++q) so[q] = (q & 1) ? v.s[q >> 1] : -v.s[q >> 1];
#pragma unroll
    for (int l = 0; l < DIM; ++l) ih[l] = ldexp(g.ih2[l], -2 * s);

    typename Op::Node nd[2][S];
    bool on[2][S], has[2][S];
    {
        int c[2][S][3];
        T Kc[2][S], Kn[2][S][NQ];
#pragma unroll
        for (int col = 0; col < 2; ++col)
#pragma unroll
            for (int u = 0; u < S; ++u) {
                typename Op::Node &q = nd[col][u];
                const int lin = 2 * (tid + u * nthreads) + col;
                has[col][u] = lin < v.N;
                wg_ijk<DIM>(v, has[col][u] ? lin : 0, c[col][u]);
                q.p = wg_pos<DIM>(v, c[col][u]);
                Kc[col][u] = B.K[q.p];
#pragma unroll
                for (int t = 0; t < NQ; ++t) Kn[col][u][t] = B.K[q.p + so[t]];
                q.x = B.x[q.p];
                q.g = B.g[q.p];
                q.b = Op::SINK ? (T)M.beta[c[col][u][DIM - 1]] : T(0);
                if constexpr (sizeof(T) == 8) {
                    q.soil = 0;
                    if constexpr (Op::MODEL == kMulti) q.soil = M.soil[wg_mem<DIM>(g, v, c[col][u])];
                } else {
                    q.base.psi = B.pb[q.p];
                }
            }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int col = 0; col < 2; ++col)
#pragma unroll
            for (int u = 0; u < S; ++u) {
                typename Op::Node &q = nd[col][u];
                const int *cc = c[col][u];
                on[col][u] = has[col][u] && !wg_dirichlet<DIM>(g, v, cc);
                // face coefficients m_ij = (K_i + K_j) / (2 w h^2), 0 without a neighbour
                T mii = T(0);
#pragma unroll
                for (int l = 0; l < DIM; ++l) {
                    const bool lo = cc[l] == 0, hi = cc[l] == v.n[l] - 1;
                    const double cf = (lo || hi ? 1.0 : 0.5) * ih[l];
                    const T cl = lo ? T(0) : (T)cf, ch = hi ? T(0) : (T)cf;
                    const T kl = Kc[col][u] + Kn[col][u][2 * l], kh = Kc[col][u] + Kn[col][u][2 * l + 1];
                    q.m[2 * l] = cl * kl;
                    q.m[2 * l + 1] = ch * kh;
                    mii = fma(cl, kl, mii);   // as the launched kernels' sum contracts
                    mii = fma(ch, kh, mii);
                }
                if (e.L.kappa_rule == kKappaConst) q.kap = (T)e.L.kappa;
                else if (e.L.kappa_rule == kKappaRel) q.kap = (T)e.L.kappa * mii;
                else q.kap = wg_remark<DIM, T>(g, v, cc, col, (T)M.lambdaU, q.m);
                if constexpr (sizeof(T) == 4) {
                    q.base = base_of<Op::MODEL>(e.L, q.base.psi);
                    base_room<Op::MODEL>(e.L, q.base, q.up, q.down);
                    q.ab = Op::SINK ? feddes_value32(e.L, q.base.psi) : 0.0f;
                }
                Op::coefficients(e, q, mii);
            }
        if (up) {
            // tensor interpolation of the correction: two taps per axis, the
            // second of weight 0 at an even index
            constexpr int N2 = DIM > 2 ? 2 : 1, N1 = DIM > 1 ? 2 : 1, NT = 2 * N1 * N2;
            T tap[2][S][NT];
#pragma unroll
            for (int col = 0; col < 2; ++col)
#pragma unroll
                for (int u = 0; u < S; ++u) {
                    int o[3][2];
#pragma unroll
                    for (int l = 0; l < 3; ++l) {
                        o[l][0] = (c[col][u][l] >> 1) * vc.s[l];
                        o[l][1] = ((c[col][u][l] + 1) >> 1) * vc.s[l];
                    }
#pragma unroll
                    for (int q = 0; q < NT; ++q)
                        tap[col][u][q] = C.bar[vc.base + o[0][q & 1] +
                                               (DIM > 1 ? o[1][(q >> 1) & 1] : 0) +
                                               (DIM > 2 ? o[2][q >> 2] : 0)];
                }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int col = 0; col < 2; ++col)
#pragma unroll
                for (int u = 0; u < S; ++u) {
                    typename Op::Node &q = nd[col][u];
                    T w[3][2];
#pragma unroll
                    for (int l = 0; l < 3; ++l) {
                        const bool odd = c[col][u][l] & 1;
                        w[l][0] = odd ? T(0.5) : T(1);
                        w[l][1] = odd ? T(0.5) : T(0);
                    }
                    T sum = T(0);
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        sum += w[0][t & 1] * (DIM > 1 ? w[1][(t >> 1) & 1] : T(1)) *
                               (DIM > 2 ? w[2][t >> 2] : T(1)) * tap[col][u][t];
                    if (on[col][u]) {
                        q.x += sum;
                        B.x[q.p] = q.x;
                    }
                }
        } else if (s > 0) {
            // FAS right-hand side N(bar) + restricted defect (g holds it)
            T bn[2][S][NQ];
#pragma unroll
            for (int col = 0; col < 2; ++col)
#pragma unroll
                for (int u = 0; u < S; ++u)
#pragma unroll
                    for (int t = 0; t < NQ; ++t) bn[col][u][t] = B.bar[nd[col][u].p + so[t]];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int col = 0; col < 2; ++col)
#pragma unroll
                for (int u = 0; u < S; ++u) {
                    typename Op::Node &q = nd[col][u];
                    T md = T(0);
#pragma unroll
                    for (int t = 0; t < NQ; ++t) md += q.m[t] * (q.x - bn[col][u][t]);
                    if (on[col][u]) {
                        q.g = Op::apply(e, q, q.x, md) + q.g;
                        B.g[q.p] = q.g;
                    }
                }
        }
    }
    if (up) wg_sync<WAVE>();
    const int n = norm_only ? 0 : (last ? A.nuc : (up ? A.nu2 : A.nu1));
    for (int sw = 0; sw < n; ++sw) {
        bool changed = false;
#pragma unroll
        for (int col = 0; col < 2; ++col) {
#pragma unroll
            for (int u = 0; u < S; ++u) {
                typename Op::Node &q = nd[col][u];
                if (on[col][u]) {
                    T f = q.g;
#pragma unroll
                    for (int t = 0; t < NQ; ++t) f += q.m[t] * B.x[q.p + so[t]];
                    f += q.kap * q.x;
                    const T x1 = Op::solve(e, q, f);
                    if (last) changed |= Op::moved(x1, q.x);
                    q.x = x1;
                    B.x[q.p] = x1;
                }
            }
            if (col == 0 || !last) wg_sync<WAVE>();
        }
        // the coarsest problem is solved to rounding after a sweep that moved
        // no value by more than 4 ulp
        if (last) {
            if (WAVE) {
                wg_sync<true>();
                if (!A.all && !__any(changed)) break;
            } else if (!__syncthreads_or(changed) && !A.all) {
                break;
            }
        }
    }
    if (!up && !last && !norm_only) {
        // defect (0 at Dirichlet nodes), then its full weighting and the iterate's
        {
            T xn[2][S][NQ];
#pragma unroll
            for (int col = 0; col < 2; ++col)
#pragma unroll
                for (int u = 0; u < S; ++u)
#pragma unroll
                    for (int t = 0; t < NQ; ++t) xn[col][u][t] = B.x[nd[col][u].p + so[t]];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int col = 0; col < 2; ++col)
#pragma unroll
                for (int u = 0; u < S; ++u) {
                    typename Op::Node &q = nd[col][u];
                    T md = T(0);
#pragma unroll
                    for (int t = 0; t < NQ; ++t) md += q.m[t] * (q.x - xn[col][u][t]);
                    if (has[col][u]) dbox[q.p] = on[col][u] ? q.g - Op::apply(e, q, q.x, md) : T(0);
                }
        }
        wg_sync<WAVE>();
        // one coarse value per thread: the iterate's for the first N_c, the
        // defect's for the rest
        for (int t = tid; t < 2 * vc.N; t += nthreads) {
            const bool def = t >= vc.N;
            int c[3];
            wg_ijk<DIM>(vc, def ? t - vc.N : t, c);
            const int pc = wg_pos<DIM>(vc, c);
            const T *src = def ? dbox : B.x;
            int o[3][3];
#pragma unroll
            for (int l = 0; l < 3; ++l) {
                const int F = 2 * c[l] * v.s[l];
                o[l][0] = F + (c[l] == 0 ? v.s[l] : -v.s[l]);
                o[l][1] = F;
                o[l][2] = F + (2 * c[l] == v.n[l] - 1 ? -v.s[l] : v.s[l]);
            }
            constexpr int N2 = DIM > 2 ? 3 : 1, N1 = DIM > 1 ? 3 : 1;
            T tap[N2][N1][3];
#pragma unroll
            for (int o2 = 0; o2 < N2; ++o2)
#pragma unroll
                for (int o1 = 0; o1 < N1; ++o1)
#pragma unroll
                    for (int o0 = 0; o0 < 3; ++o0)
                        tap[o2][o1][o0] = src[v.base + o[0][o0] + (DIM > 1 ? o[1][o1] : 0) +
                                              (DIM > 2 ? o[2][o2] : 0)];
            __builtin_amdgcn_sched_barrier(0);
            const T wt[3] = {T(0.25), T(0.5), T(0.25)};
            T sum = T(0);
#pragma unroll
            for (int o2 = 0; o2 < N2; ++o2)
#pragma unroll
                for (int o1 = 0; o1 < N1; ++o1)
#pragma unroll
                    for (int o0 = 0; o0 < 3; ++o0)
                        sum += wt[o0] * (DIM > 1 ? wt[o1] : T(1)) * (DIM > 2 ? wt[o2] : T(1)) *
                               tap[o2][o1][o0];
            if (wg_dirichlet<DIM>(g, vc, c)) sum = def ? T(0) : tap[N2 / 2][N1 / 2][1];
            if (def) {
                C.g[pc] = sum;
            } else {
                C.bar[pc] = sum;
                C.x[pc] = sum;
            }
        }
        wg_sync<WAVE>();
        return;
    }
    if (s > 0) {
        // the correction the finer level interpolates
#pragma unroll
        for (int col = 0; col < 2; ++col)
#pragma unroll
            for (int u = 0; u < S; ++u)
                if (has[col][u])
                    B.bar[nd[col][u].p] = nd[col][u].x - B.bar[nd[col][u].p];
        wg_sync<WAVE>();
    } else if (norm) {
        double m = 0.0;
#pragma unroll
        for (int col = 0; col < 2; ++col)
#pragma unroll
            for (int u = 0; u < S; ++u) {
                typename Op::Node &q = nd[col][u];
                T md = T(0);
#pragma unroll
                for (int t = 0; t < NQ; ++t) md += q.m[t] * (q.x - B.x[q.p + so[t]]);
                const double r = on[col][u] ? fabs((double)(q.g - Op::template apply<true>(e, q, q.x, md))) : 0.0;
                m = (r > m || r != r) ? r : m;
            }
        if (WAVE) {
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) {
                const double o = __shfl_xor(m, d);
                m = (o > m || o != o) ? o : m;
            }
        } else {
            m = block_max(m);
        }
        if (tid == 0) *norm = m;
    } else {
#pragma unroll
        for (int col = 0; col < 2; ++col)
#pragma unroll
            for (int u = 0; u < S; ++u)
                if (on[col][u]) {
                    int c[3];
                    wg_ijk<DIM>(v, 2 * (tid + u * nthreads) + col, c);
                    A.x[wg_mem<DIM>(g, v, c)] = nd[col][u].x;
                }
    }
}

// The levels' LDS boxes from memory; returns the defect box.
template <class Op, class Mem>
__device__ __forceinline__ typename Op::T *wg_load(const WgCycle<typename Op::T> &A,
                                                   const Mem &mem, typename Op::T *lds)
{
    typedef typename Op::T T;
    constexpr int DIM = Op::DIM;
    const int nthreads = blockDim.x, tid = threadIdx.x;
    // every level's K* (and base state), the top level's iterate and
    // right-hand side; zeros elsewhere (the sweeps of one level read three boxes).
    // The loads of all levels that a pass of the work-group covers are in flight
    // together, the iterate's and right-hand side's among them (behind the barrier
    // they cost one more memory latency: a sweep of 9x9x3 nodes 7.4 -> 6.7 us).
    int total = 0;
    for (int s = 0; s < A.levels; ++s) total += wg_words<T, DIM>(A.g, s);
    T *dbox = lds + total;
    const int top = wg_level<DIM>(A.g, 0).size;
    const int all = A.levels == 1 ? 3 * top : total + top;
    const WgLevel<DIM> v0 = wg_level<DIM>(A.g, 0);
    T x0 = T(0), g0 = T(0);
    if (tid < v0.N) {
        int c[3];
        wg_ijk<DIM>(v0, tid, c);
        x0 = A.x[wg_mem<DIM>(A.g, v0, c)];
        g0 = A.rhs[wg_mem<DIM>(A.g, v0, c)];
    }
    T k0[kWgMaxLev], p0[kWgMaxLev];
#pragma unroll
    for (int s = 0; s < kWgMaxLev; ++s)
        if (s < A.levels) {
            const WgLevel<DIM> v = wg_level<DIM>(A.g, s);
            if (tid < v.N) {
                int c[3];
                wg_ijk<DIM>(v, tid, c);
                k0[s] = mem(s).K[wg_mem<DIM>(A.g, v, c)];
                if (sizeof(T) == 4) p0[s] = mem(s).pb[wg_mem<DIM>(A.g, v, c)];
            }
        }
    for (int t = tid; t < all; t += nthreads) lds[t] = T(0);
    __syncthreads();
    int off = 0;
#pragma unroll
    for (int s = 0; s < kWgMaxLev; ++s)
        if (s < A.levels) {
            const WgLevel<DIM> v = wg_level<DIM>(A.g, s);
            const WgBox<T, DIM> B = wg_box<T, DIM>(lds, off, v);
            if (tid < v.N) {
                int c[3];
                wg_ijk<DIM>(v, tid, c);
                B.K[wg_pos<DIM>(v, c)] = k0[s];
                if (sizeof(T) == 4) B.pb[wg_pos<DIM>(v, c)] = p0[s];
                if (s == 0) {
                    B.x[wg_pos<DIM>(v, c)] = x0;
                    B.g[wg_pos<DIM>(v, c)] = g0;
                }
            }
            off += wg_words<T, DIM>(A.g, s);
        }
    off = 0;
    for (int s = 0; s < A.levels; ++s) {
        const WgLevel<DIM> v = wg_level<DIM>(A.g, s);
        if (v.N <= nthreads) break;
        const WgBox<T, DIM> B = wg_box<T, DIM>(lds, off, v);
#pragma unroll 2
        for (int t = tid + nthreads; t < v.N; t += nthreads) {
            int c[3];
            wg_ijk<DIM>(v, t, c);
            const int at = wg_mem<DIM>(A.g, v, c);
            const int p = wg_pos<DIM>(v, c);
            B.K[p] = mem(s).K[at];
            if (sizeof(T) == 4) B.pb[p] = mem(s).pb[at];
            if (s == 0) {
                B.x[p] = A.x[at];
                B.g[p] = A.rhs[at];
            }
        }
        off += wg_words<T, DIM>(A.g, s);
    }
    __syncthreads();
    return dbox;
}

// One visit, in the mode of its level: two nodes per thread and colour on levels
// of more nodes per colour than threads (TWO), one wave from the first level of
// at most 64 nodes per colour (wave: the last visit was of that kind).
template <class Op, bool TWO, class Mem>
__device__ __forceinline__ void wg_visit_mode(const WgCycle<typename Op::T> &A, const Mem &mem,
                                              const typename Op::Env &e, int s, bool up,
                                              bool &wave, typename Op::T *lds, int off,
                                              typename Op::T *dbox, double *norm, bool norm_only)
{
    constexpr int DIM = Op::DIM;
    const int nthreads = blockDim.x;
    const int slots = (wg_level<DIM>(A.g, s).N + 1) / 2;
    if (slots <= 64) {
        wave = true;
        if (threadIdx.x < 64)
            wg_visit<Op, 1, true>(A, mem(s), e, s, up, 64, lds, off, dbox, norm, norm_only);
        return;
    }
    if (wave) __syncthreads();   // the other waves join again
    wave = false;
    if (slots <= nthreads)
        wg_visit<Op, 1, false>(A, mem(s), e, s, up, nthreads, lds, off, dbox, norm, norm_only);
    else if constexpr (TWO)
        wg_visit<Op, 2, false>(A, mem(s), e, s, up, nthreads, lds, off, dbox, norm, norm_only);
}

// The cycle: down and up over the levels.
template <class Op, bool TWO = Op::DIM == 1, class Mem>
__device__ __forceinline__ void wg_cycle(const WgCycle<typename Op::T> &A, const Mem &mem,
                                         const typename Op::Env &e, typename Op::T *lds)
{
    typedef typename Op::T T;
    constexpr int DIM = Op::DIM;
    T *dbox = wg_load<Op>(A, mem, lds);
    int off = 0;
    const int visits = 2 * A.levels - 1;
    bool wave = false;
    for (int q = 0; q < visits; ++q) {
        const bool up = q >= A.levels;
        const int s = up ? visits - 1 - q : q;
        const int words = wg_words<T, DIM>(A.g, s);
        if (up) off -= words;
        wg_visit_mode<Op, TWO>(A, mem, e, s, up, wave, lds, off, dbox, nullptr, false);
        if (!up && s + 1 < A.levels) off += words;
    }
}

// Cycles of a whole grid in one work-group until the step's stopping test ends
// them (the test of rs_bdf_step: the norm after each cycle at most tol, not
// finite, or two cycles in a row without a new minimum), at most `most` of
// them, with the iterate in LDS throughout.
struct WgSolve {
    double tol, best;
    int slow, stagnation, most;
    int first;    // 1: the norm of the iterate as it is comes first (hist[0])
};

// What it reports: the norm after each cycle, behind the first norm.
struct WgSolveOut {
    double r, best;
    int cycles, slow, stagnated, pad;
    double hist[kWgSolveCycles + 1];
};

template <class Op, class Mem>
__device__ __forceinline__ void wg_solve(const WgCycle<typename Op::T> &A, const Mem &mem,
                                         const typename Op::Env &e, typename Op::T *lds,
                                         const WgSolve &S, WgSolveOut *out)
{
    typedef typename Op::T T;
    constexpr int DIM = Op::DIM;
    __shared__ double norm;
    T *dbox = wg_load<Op>(A, mem, lds);
    const int visits = 2 * A.levels - 1;
    bool wave = false, stagnated = false;
    double best = S.best, r = 0.0;
    int slow = S.slow, cycles = 0, off = 0;
    // one loop over all visits (the visit's code appears once per mode): q = -1
    // is the norm of the iterate as it is
    int q = S.first ? -1 : 0;
    while (true) {
        const bool up = q >= A.levels;
        const int s = q < 0 ? 0 : (up ? visits - 1 - q : q);
        const int words = wg_words<T, DIM>(A.g, s);
        if (up) off -= words;
        const bool end = q < 0 || q == visits - 1;
        wg_visit_mode<Op, DIM == 1>(A, mem, e, s, up, wave, lds, off, dbox, end ? &norm : nullptr,
                                    q < 0);
        if (!end) {
            if (!up && s + 1 < A.levels) off += words;
            ++q;
            continue;
        }
        __syncthreads();
        wave = false;
        r = norm;
        const bool finite = fabs(r) <= 1.7976931348623157e308;
        if (q < 0) {
            best = r;
            if (threadIdx.x == 0) out->hist[0] = r;
        } else {
            ++cycles;
            if (threadIdx.x == 0) out->hist[cycles] = r;
            if (S.stagnation) {
                if (r < best) {
                    best = r;
                    slow = 0;
                } else if (++slow >= 2) {
                    stagnated = true;
                }
            }
        }
        if (stagnated || !(finite && r > S.tol) || cycles >= S.most) break;
        q = 0;
        off = 0;
        __syncthreads();
    }
    // the iterate back to memory
    const WgLevel<DIM> v = wg_level<DIM>(A.g, 0);
    const WgBox<T, DIM> B = wg_box<T, DIM>(lds, 0, v);
    for (int t = threadIdx.x; t < v.N; t += blockDim.x) {
        int c[3];
        wg_ijk<DIM>(v, t, c);
        A.x[wg_mem<DIM>(A.g, v, c)] = B.x[wg_pos<DIM>(v, c)];
    }
    if (threadIdx.x == 0) {
        out->r = r;
        out->best = best;
        out->cycles = cycles;
        out->slow = slow;
        out->stagnated = stagnated ? 1 : 0;
        __threadfence_system();
    }
}

// Levels that fit the work-group, with two nodes per thread and colour in 1-D only.
inline bool wg_level_fits(const Geo &g)
{
    return g.N <= (g.dim == 1 ? kTailNodes : 2LL * kWgMaxThreads);
}

// Levels of a grid's V-cycles that run in it: also the 3-D ones up to kTailNodes
// nodes (5x5x65 and its like), two nodes per thread and colour, in a kernel of
// their own (in the others' it would cost registers).  A V(2,2) cycle of 5x5x65
// nodes, launches per colour and transfer against this: 104 us (vGM) and 99
// (Haverkamp) against 47 and 90, in mixed precision 207 and 234 against 100 and 95.
inline bool wg_cycle_level(const Geo &g)
{
    return wg_level_fits(g) || (g.dim == 3 && g.N <= kTailNodes);
}

// Work-group size: one node per thread and colour on the top level where that
// fits, else two.
inline int wg_threads(const WgGeo &g, int dim)
{
    const int slots = (g.n[0] * g.n[1] * g.n[2] + 1) / 2;
    int t = slots <= kWgMaxThreads ? slots : (slots + 1) / 2;
    if (dim == 2) {   // one pass over the coarse values (2 N_c, just above the slots)
        const int nc = 2 * ((g.n[0] + 1) / 2) * ((g.n[1] + 1) / 2);
        if (nc > t && nc <= kWgMaxThreads) t = nc;
    }
    return (t + 63) / 64 * 64;
}

// Launchers (kernels_cycle.hip, kernels_cycle32.hip): one cycle, or the cycles
// of a step, as one work-group.
void launch_solve_wg(const WgCycle<double> &A, const WgMems<double> &M, const Law &law, double a,
                     int dim, const WgSolve &S, WgSolveOut *out, hipStream_t s);
void launch_cycle_wg(const WgCycle<double> &A, const WgMems<double> &M, const Law &law, double a,
                     int dim, hipStream_t s);
void launch_sweeps_wg(const WgCycle<double> &A, const WgMems<double> &M, const Law &law, double a,
                      int dim, hipStream_t s);
void launch_cycle_wg32(const WgCycle<float> &A, const WgMems<float> &M, const Law32 &law, float a,
                       int dim, hipStream_t s);

}  // namespace rs
