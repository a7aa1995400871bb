// FP32 correction cycles of the small levels in one work-group (cycle_wg.h) and
// of the mid-size 1-D and 2-D levels in tiles (cycle_tile.h).
#include "rs_internal.h"
#include "soil_device.h"
#include "grid_device.h"
#include "mp_internal.h"
#include "cycle_wg.h"
#include "cycle_tile.h"

namespace rs {

namespace {

// The FP32 correction cycle from a level of at most kTailNodes nodes down and
// back in one work-group (cycle_wg.h).
template <int MODEL, bool SINK, int DIM, bool TWO>
__global__ __launch_bounds__(kWgMaxThreads) void k_cycle_wg32(WgCycle<float> A, WgMems<float> M,
                                                              Law32 L, float a)
{
    extern __shared__ float lds32[];
    typedef WgOp32<MODEL, SINK, DIM> Op;
    wg_cycle<Op, TWO>(A, M, typename Op::Env{L, a}, lds32);
}

// One tile of a phase of a level (cycle_tile.h).
template <int MODEL, bool SINK, int DIM>
__global__ __launch_bounds__(kTileThreads) void k_cycle_tile32(TileArgs<float> A, int phase,
                                                               Law32 L, float a)
{
    extern __shared__ float lds32[];
    typedef WgOp32<MODEL, SINK, DIM> Op;
    tile_run<Op>(A, phase, typename Op::Env{L, a}, lds32);
}

struct CycleWg32Launch {
    const WgCycle<float> &A; const WgMems<float> &M; const Law32 &law; float a; hipStream_t s;
    template <int MO, bool S, int D, bool TWO>
    void run()
    {
        const size_t bytes = wg_lds_bytes<float, D>(A.g, A.levels);
        if (bytes > 64 * 1024)
            (void)hipFuncSetAttribute((const void *)k_cycle_wg32<MO, S, D, TWO>,
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        hipLaunchKernelGGL((k_cycle_wg32<MO, S, D, TWO>), dim3(1), dim3(wg_threads(A.g, D)), bytes, s, A,
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

struct Tile32Launch {
    const TileArgs<float> &A; int phase, blocks; size_t words; const Law32 &law; float a;
    hipStream_t s;
    template <int MO, bool SK, int D>
    void go()
    {
        const size_t bytes = sizeof(float) * words;
        if constexpr (D < 3)
            hipLaunchKernelGGL((k_cycle_tile32<MO, SK, D>), dim3(blocks), dim3(kTileThreads), bytes,
                               s, A, phase, law, a);
    }
};

}  // namespace

void launch_tile32(const TileArgs<float> &A, int phase, int blocks, size_t words,
                   const Law32 &law, float a, hipStream_t s)
{
    dispatch(dispatch_key(law), A.dim, Tile32Launch{A, phase, blocks, words, law, a, s});
}

void launch_cycle_wg32(const WgCycle<float> &A, const WgMems<float> &M, const Law32 &law, float a,
                       int dim, hipStream_t s)
{
    dispatch(dispatch_key(law), dim, CycleWg32Launch{A, M, law, a, s});
}

}  // namespace rs
