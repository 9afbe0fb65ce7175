// The direct form of a single FP32 transform of at most 2^23 items: one
// workgroup up to 2^14 items, two column passes above (tile.h).
//
// At these sizes a call is launches and latency, not bytes: the phases' three
// dependent launches took 14.2 us at 2^12, 16.7 at 2^16, 24.2 at 2^20 and 53 at
// 2^22 (calls back to back), where a copy of the data takes 0.01, 0.2, 3.2 and
// 13 us.  Lemma 1 holds for any digit-aligned split of N, so the form takes the
// one with the fewest launches: 5.1, 8.4, 14.7 and 32 us.  Calls back to back, one
// workgroup takes 10.2 us at 2^14 (its kernel in a trace 4.5 us at 2^12, 6.6 at
// 2^13 and 11.2 at 2^14), where the two launches of 2^15 take 7.9: two passes
// would be 2 us faster there; the batched kernel, which has to give the same bits,
// moves 5.3 TB/s at 2^14 in one workgroup and would move half of it in two passes.
#include "direct_kernels.h"

namespace paco {
namespace {

template <int L>
__global__ __launch_bounds__(tile_threads(L, 0, 1)) void direct_chip_kernel(DirectArgs P)
{
    __shared__ float2 smem[tile_lds(L, 0, 1)];
    chip_tile<L, 0>(P.src, P.dst, [](int) { return int64_t(0); }, P.stw, smem, threadIdx.x, P.conj_in != 0, P.out_scale);
}

__global__ __launch_bounds__(1024) void direct_chip14_kernel(DirectArgs P)
{
    __shared__ float2 smem[tile_lds(13, 1, 1)];
    chip14_wide_tile(P.src, P.dst, P.stw, P.top.hi, P.top.lo, smem, threadIdx.x, P.conj_in != 0, P.out_scale);
}

template <int L>
void chip(const DirectArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(direct_chip_kernel<L>, dim3(1), dim3(tile_threads(L, 0, 1)), 0, s, a);
}

}  // namespace

DirectForm direct_form(int l1, int l2)
{
    DirectForm f{};
    f.log2N = l1 + l2;
    if (f.log2N <= kDirectChipLog2) return f;
    f.l1 = direct_l1(l1, l2);
    f.l2 = f.log2N - f.l1;
    return f;
}

hipError_t launch_direct(const DirectForm &f, const float2 *in, float2 *out, float2 *ws, bool inverse, hipStream_t s)
{
    DirectArgs a{};
    a.top = {f.hi, f.lo, f.cw, f.log2N, f.log2Lo};
    a.l1 = f.l1;
    a.l2 = f.l2;
    const float scale = inverse ? 1.0f / float(int64_t(1) << f.log2N) : 0.f;  // 2^-log2 N: exact
    a.src = in;
    a.stw = f.stw1;
    a.conj_in = inverse ? 1 : 0;
    if (f.l1 == 0) {
        a.dst = out;
        a.out_scale = scale;
        switch (f.log2N) {
        case 2: chip<2>(a, s); break;
        case 3: chip<3>(a, s); break;
        case 4: chip<4>(a, s); break;
        case 5: chip<5>(a, s); break;
        case 6: chip<6>(a, s); break;
        case 7: chip<7>(a, s); break;
        case 8: chip<8>(a, s); break;
        case 9: chip<9>(a, s); break;
        case 10: chip<10>(a, s); break;
        case 11: chip<11>(a, s); break;
        case 12: chip<12>(a, s); break;
        case 13: chip<13>(a, s); break;
        case 14: hipLaunchKernelGGL(direct_chip14_kernel, dim3(1), dim3(1024), 0, s, a); break;
        default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    a.dst = ws;
    const auto pass = [&](bool b, int l, int lcols) {
        return f.prec == kPrecFP32 ? direct_pass_t<kPrecFP32>(b, l, lcols, a, s) : direct_pass_mf(f.prec, b, l, lcols, a, s);
    };
    hipError_t e = pass(false, f.l1, f.l2);
    if (e != hipSuccess) return e;
    a.src = ws;
    a.dst = out;
    a.stw = f.stw2;
    a.conj_in = 0;
    a.out_scale = scale;
    return pass(true, f.l2, f.l1);
}

}  // namespace paco
