// BOOST with its two sums on two units (boost_pieces.h): the wide kernel in that form, and its launch.
#include "mmlike_valu_impl.h"

#ifndef AMULET_MMLIKE_BOOST_IMPL_H
#define AMULET_MMLIKE_BOOST_IMPL_H

namespace amulet {

// A tile by pieces, or, if it holds what they do not take, by the wide kernel's own arithmetic.
template <int TF, int TRANS>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4)))
mmlike_boost_kernel(const MmlikeArgs args)
{
    constexpr bool BPRE = (TRANS & 1) == 0;
    extern __shared__ __attribute__((aligned(16))) char boost_smem[];
    BoostLds &L = *(BoostLds *)boost_smem;
    auto &no_a = *(float (*)[1][1][4])L.s;
    const unsigned wave = own_wave();
    if (valu_tile<TASK_BOOST, TF, TRANS, 4, 1, 8, BOOST_BK, 4, false, false, BPRE, true, false, false>(args, threadIdx.x, L.b, no_a)) return;
    unsigned tid;
    const auto &again = opaque_args<MmlikeArgs>(wave, tid);
    valu_tile<TASK_BOOST, TF, TRANS, 4, 1, 8, BOOST_BK, 4, false, false, BPRE, false, false, false>(again, tid, L.b, no_a);
}

template <int TF, int TRANS>
static hipError_t launch_boost(MmlikeArgs &b, int64_t blocks, int splits, hipStream_t s)
{
    static hipError_t granted = hipFuncSetAttribute(reinterpret_cast<const void *>(&mmlike_boost_kernel<TF, TRANS>),
                                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(BoostLds));
    if (granted != hipSuccess) return granted;
    return launch_row_of_blocks(b, blocks, 512, [&](unsigned n) {
        hipLaunchKernelGGL((mmlike_boost_kernel<TF, TRANS>), dim3(n, (unsigned)splits), dim3(512), sizeof(BoostLds), s, b);
    });
}

template <int TF>
hipError_t launch_mmlike_boost(const MmlikeArgs &args, hipStream_t s)
{
    MmlikeArgs b = args;
    const int64_t tiles_m = ((int64_t)b.M + BOOST_ROWS - 1) / BOOST_ROWS, tiles_n = ((int64_t)b.N + BOOST_COLS - 1) / BOOST_COLS;
    int64_t blocks = xcd_grid(tiles_m, tiles_n);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    // K in the parts of the wide kernel: every tile's where tiles are few, else the last round's
    const int64_t chunk = wide_k_range(tiles_m * tiles_n * 8, b.K);
    b.kchunk = (int)chunk;
    const int splits = (int)((b.K + chunk - 1) / chunk);
    b.tail_base = 0; b.tail_blocks = 0; b.tail_splits = 1;
    TailSplit t;
    if (splits == 1 && choose_tail_split(tiles_m * tiles_n, blocks, (int64_t)compute_units() * 2, b.K, 64, t)) {
        b.tail_base = (int)t.base;
        b.tail_blocks = (int)t.blocks;
        b.tail_splits = t.splits;
        b.kchunk = t.chunk;
        blocks = t.grid;
    }
    switch ((b.transA ? 1 : 0) | (b.transB ? 2 : 0)) {
    case 0: return launch_boost<TF, 0>(b, blocks, splits, s);
    case 1: return launch_boost<TF, 1>(b, blocks, splits, s);
    case 2: return launch_boost<TF, 2>(b, blocks, splits, s);
    default: return launch_boost<TF, 3>(b, blocks, splits, s);
    }
}

}  // namespace amulet
#endif
