// The two column passes of the direct form (direct.hip), templated on the
// butterfly arithmetic (direct_mf.hip instantiates the split MFMA forms).
#pragma once

#include "tile.h"

namespace paco {

struct DirectArgs {
    const float2 *src;
    float2 *dst;
    const float2 *stw;
    TopRoots top;
    int32_t l1, l2;
    int32_t conj_in;
    float out_scale;
};

// the split MFMA forms' passes (direct_mf.hip)
hipError_t direct_pass_mf(int prec, bool b, int l, int lcols, const DirectArgs &a, hipStream_t s);

namespace {

template <int L, int PREC>
__global__ __launch_bounds__(tile_threads(L, tile_cols(L, PREC != kPrecFP32), tile_groups(L))) void direct_a_kernel(DirectArgs P)
{
    constexpr int LT = tile_cols(L, PREC != kPrecFP32);
    __shared__ float2 smem[tile_lds(L, LT, tile_groups(L))];
    pass_a_tile<L, LT, tile_groups(L), false, PREC>(P.src, P.dst, P.l2, tile_cols(P.l2, PREC != kPrecFP32),
                                               uint32_t(tile_order(blockIdx.x, gridDim.x)) << LT, P.stw, smem,
                                               threadIdx.x, P.conj_in != 0);
}

template <int L, int PREC>
__global__ __launch_bounds__(tile_threads(L, tile_cols(L, PREC != kPrecFP32), tile_groups(L))) void direct_b_kernel(DirectArgs P)
{
    constexpr int LT = tile_cols(L, PREC != kPrecFP32);
    __shared__ float2 smem[tile_lds(L, LT, tile_groups(L))];
    pass_b_tile<L, LT, tile_groups(L), PREC>(P.src, P.dst, P.l1, uint32_t(tile_order(blockIdx.x, gridDim.x)) << LT, P.top,
                                        P.stw, smem, threadIdx.x, P.out_scale);
}

template <int L, int PREC>
void launch_pass(bool b, int lcols, const DirectArgs &a, hipStream_t s)
{
    constexpr int LT = tile_cols(L, PREC != kPrecFP32);
    const dim3 tiles(1u << (lcols - LT)), threads(tile_threads(L, LT, tile_groups(L)));
    if constexpr (L < 12) {  // 4096 points: pass A only
        if (b) {
            hipLaunchKernelGGL((direct_b_kernel<L, PREC>), tiles, threads, 0, s, a);
            return;
        }
    }
    hipLaunchKernelGGL((direct_a_kernel<L, PREC>), tiles, threads, 0, s, a);
}

// one pass of 2^l points over 2^lcols columns
template <int PREC>
hipError_t direct_pass_t(bool b, int l, int lcols, const DirectArgs &a, hipStream_t s)
{
    switch (l) {
    case 7: launch_pass<7, PREC>(b, lcols, a, s); break;
    case 8: launch_pass<8, PREC>(b, lcols, a, s); break;
    case 9: launch_pass<9, PREC>(b, lcols, a, s); break;
    case 10: launch_pass<10, PREC>(b, lcols, a, s); break;
    case 11: launch_pass<11, PREC>(b, lcols, a, s); break;
    case 12:
        // split butterflies at 4096 points spilled and took 209 us at 2048 x 4096, the three-pass form 175
        if (PREC != kPrecFP32 || b) return hipErrorInvalidValue;
        if constexpr (PREC == kPrecFP32) launch_pass<12, PREC>(false, lcols, a, s);
        break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace
}  // namespace paco
