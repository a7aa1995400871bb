// FP64 V-cycles of the small levels in one work-group (cycle_wg.h) and of the
// mid-size 1-D and 2-D levels in tiles (cycle_tile.h).
#include "rs_internal.h"
#include "soil_device.h"
#include "grid_device.h"
#include "cycle_wg.h"
#include "cycle_tile.h"

namespace rs {

namespace {

// The soil table of a layered medium, staged in LDS; null for one law.
template <int MODEL>
__device__ __forceinline__ const Law *stage_soils(const Law &L)
{
    if constexpr (MODEL == kMulti) {
        __shared__ Law tab[kMaxSoils];
        const int *src = (const int *)L.soils;
        for (int t = threadIdx.x; t < (int)(sizeof(Law) / sizeof(int)) * kMaxSoils;
             t += blockDim.x)
            ((int *)tab)[t] = src[t];
        return tab;   // read after the first barrier of the cycle
    }
    return nullptr;
}

// The V-cycle from a level of at most kTailNodes nodes down and back in one
// work-group (cycle_wg.h).
template <int MODEL, bool SINK, int DIM, bool TWO>
__global__ __launch_bounds__(kWgMaxThreads) void k_cycle_wg(WgCycle<double> A, WgMems<double> M,
                                                            Law L, double a)
{
    extern __shared__ double lds64[];
    const Law *soils = stage_soils<MODEL>(L);
    typedef WgOp64<MODEL, SINK, DIM> Op;
    wg_cycle<Op, TWO>(A, M, typename Op::Env{L, soils, a}, lds64);
}

// The cycles of a step on a grid whose finest level fits one work-group.
template <int MODEL, bool SINK, int DIM>
__global__ __launch_bounds__(kWgMaxThreads) void k_solve_wg(WgCycle<double> A, WgMems<double> M,
                                                            Law L, double a, WgSolve S,
                                                            WgSolveOut *out)
{
    extern __shared__ double lds64[];
    const Law *soils = stage_soils<MODEL>(L);
    typedef WgOp64<MODEL, SINK, DIM> Op;
    wg_solve<Op>(A, M, typename Op::Env{L, soils, a}, lds64, S, out);
}

// A.nuc sweeps of one level: the visit of the cycle's coarsest one, with no sweep
// left out.  Bound by the chain of barriers and solves of one work-group, so the
// level is loaded once and its nodes and face coefficients stay in registers.
// Against one launch per colour, two and twenty sweeps: 1025 nodes 19.2 -> 9.4 and
// 169 -> 60 us, 33^2 21.2 -> 11.0 and 181 -> 70, 9x9x17 21.3 -> 12.2 and 181 -> 72
// (vGM).  Against a work-group on global memory, which suits a single sweep of a
// few hundred nodes: 9x9x3 nodes, one sweep 6.0 -> 6.7, two 9.6 -> 8.4, six 24.4 ->
// 16.4.
template <int MODEL, bool SINK, int DIM>
__global__ __launch_bounds__(kWgMaxThreads) void k_sweeps_wg(WgCycle<double> A, WgMems<double> M,
                                                             Law L, double a)
{
    extern __shared__ double lds64[];
    const Law *soils = stage_soils<MODEL>(L);
    typedef WgOp64<MODEL, SINK, DIM> Op;
    const typename Op::Env e{L, soils, a};
    A.levels = 1;   // known here: the transfers drop out of the visit's code
    A.all = 1;
    double *dbox = wg_load<Op>(A, M, lds64);
    bool wave = false;
    wg_visit_mode<Op, DIM == 1>(A, M, e, 0, false, wave, lds64, 0, dbox, nullptr, false);
}

// One tile of a phase of a level (cycle_tile.h).
template <int MODEL, bool SINK, int DIM>
__global__ __launch_bounds__(kTileThreads) void k_cycle_tile(TileArgs<double> A, int phase, Law L,
                                                             double a)
{
    extern __shared__ double lds64[];
    const Law *soils = stage_soils<MODEL>(L);
    typedef WgOp64<MODEL, SINK, DIM> Op;
    tile_run<Op>(A, phase, typename Op::Env{L, soils, a}, lds64);
}

struct CycleWgLaunch {
    const WgCycle<double> &A; const WgMems<double> &M; const Law &law; double a; hipStream_t s;
    template <int MO, bool S, int D, bool TWO>
    void run()
    {
        const size_t bytes = wg_lds_bytes<double, D>(A.g, A.levels);
        if (bytes > 64 * 1024)
            (void)hipFuncSetAttribute((const void *)k_cycle_wg<MO, S, D, TWO>,
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        hipLaunchKernelGGL((k_cycle_wg<MO, S, D, TWO>), dim3(1), dim3(wg_threads(A.g, D)), bytes, s, A,
                           M, law, a);
    }
    template <int MO, bool S, int D>
    void go()
    {
        if constexpr (D == 3)
            if (A.g.n[0] * A.g.n[1] * A.g.n[2] > 2 * kWgMaxThreads) return run<MO, S, D, true>();
        run<MO, S, D, D == 1>();
    }
};

struct SweepsWgLaunch {
    const WgCycle<double> &A; const WgMems<double> &M; const Law &law; double a; hipStream_t s;
    template <int MO, bool S, int D>
    void go()
    {
        const size_t bytes = wg_lds_bytes<double, D>(A.g, 1);
        if (bytes > 64 * 1024)
            (void)hipFuncSetAttribute((const void *)k_sweeps_wg<MO, S, D>,
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        hipLaunchKernelGGL((k_sweeps_wg<MO, S, D>), dim3(1), dim3(wg_threads(A.g, D)), bytes, s, A,
                           M, law, a);
    }
};

struct SolveWgLaunch {
    const WgCycle<double> &A; const WgMems<double> &M; const Law &law; double a; const WgSolve &S;
    WgSolveOut *out; hipStream_t s;
    template <int MO, bool SK, int D>
    void go()
    {
        const size_t bytes = wg_lds_bytes<double, D>(A.g, A.levels);
        if (bytes > 64 * 1024)
            (void)hipFuncSetAttribute((const void *)k_solve_wg<MO, SK, D>,
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        hipLaunchKernelGGL((k_solve_wg<MO, SK, D>), dim3(1), dim3(wg_threads(A.g, D)), bytes, s, A,
                           M, law, a, S, out);
    }
};

struct TileLaunch {
    const TileArgs<double> &A; int phase, blocks; size_t words; const Law &law; double a;
    hipStream_t s;
    template <int MO, bool SK, int D>
    void go()
    {
        const size_t bytes = sizeof(double) * words;
        if constexpr (D < 3)
            hipLaunchKernelGGL((k_cycle_tile<MO, SK, D>), dim3(blocks), dim3(kTileThreads), bytes,
                               s, A, phase, law, a);
    }
};

}  // namespace

void launch_tile(const TileArgs<double> &A, int phase, int blocks, size_t words,
                 const Law &law, double a, hipStream_t s)
{
    dispatch<true>(law, A.dim, TileLaunch{A, phase, blocks, words, law, a, s});
}

void launch_solve_wg(const WgCycle<double> &A, const WgMems<double> &M, const Law &law, double a,
                     int dim, const WgSolve &S, WgSolveOut *out, hipStream_t s)
{
    dispatch<true>(law, dim, SolveWgLaunch{A, M, law, a, S, out, s});
}

void launch_sweeps_wg(const WgCycle<double> &A, const WgMems<double> &M, const Law &law, double a,
                      int dim, hipStream_t s)
{
    dispatch<true>(law, dim, SweepsWgLaunch{A, M, law, a, s});
}

void launch_cycle_wg(const WgCycle<double> &A, const WgMems<double> &M, const Law &law, double a,
                     int dim, hipStream_t s)
{
    dispatch<true>(law, dim, CycleWgLaunch{A, M, law, a, s});
}

}  // namespace rs
