// bf16 products of operands that no kernel can load straight into LDS: odd leading dimensions, tiles or contractions that are no
// multiples of 8.  Such products ran on the register-staged kernel, whose loads are in flight for one k-step of 32 and whose
// macro-tiles end at every tile's edge: 130 to 220 TFLOP/s.  Here a first kernel lays both operands out afresh (gemm_pack.hip), in one piece each and
// padded, and the direct-load kernels run on that, with macro-tiles on one grid over all of C, so that neither the tiles'
// edges nor their alignment cost anything in the loop.  Their result path sorts the results into C's tiles.
// The copy moves 4 bytes per element of A and B; the three products of a layer of 1333 x 2001 over 2068 tokens on tiles of 500, copies
// included: 79 -> 54, 81 -> 48 and 55 -> 43 us, the layer 172 -> 93.
#include "gemm_bf16_dl_body.hpp"

namespace nnt {
namespace {

// ------------------------------------------------------------------ products
template <typename TO, bool AKF, bool BKF>
__global__ void __launch_bounds__(256) gemm_bf16_span_kernel(const GemmArgs g) {
    __shared__ __attribute__((aligned(16))) char lds[DlShape<4>::kLdsBytes];
    dl_body<TO, AKF, BKF, 4, false, 2, true>(g, lds);
}
template <typename TO, bool AKF, bool BKF>
__global__ void __launch_bounds__(256, 2) gemm_bf16_span_tall_kernel(const GemmArgs g) {
    __shared__ __attribute__((aligned(16))) char lds[DlShape<2>::kLdsBytes];
    dl_body<TO, AKF, BKF, 2, false, 2, true>(g, lds);
}
template <typename TO, bool AKF, bool BKF>
__global__ void __launch_bounds__(256, 2) gemm_bf16_span_wide_kernel(const GemmArgs g) {
    __shared__ __attribute__((aligned(16))) char lds[DlShape<1, 1>::kLdsBytes];
    dl_body<TO, AKF, BKF, 1, false, 1, true>(g, lds);
}

using KernelFn = void (*)(const GemmArgs);

template <typename TO, bool AKF, bool BKF>
KernelFn kernel_of(int cfg) {
    return cfg == kCfgSquare ? gemm_bf16_span_kernel<TO, AKF, BKF> : cfg == kCfgTall ? gemm_bf16_span_tall_kernel<TO, AKF, BKF> : gemm_bf16_span_wide_kernel<TO, AKF, BKF>;
}
template <typename TO>
KernelFn kernel_of(int akf, int bkf, int cfg) {
    return akf ? kernel_of<TO, true, true>(cfg) : bkf ? kernel_of<TO, false, true>(cfg) : kernel_of<TO, false, false>(cfg);
}

}  // namespace

int32_t launch_gemm_bf16_span(hipStream_t st, int out_is_f32, int akf, int bkf, int cfg, const GemmArgs& g, int64_t nwg) {
    if ((cfg != kCfgSquare && cfg != kCfgTall && cfg != kCfgWide) || (akf && !bkf)) return NNT_EINVAL;
    hipLaunchKernelGGL(out_is_f32 ? kernel_of<float>(akf, bkf, cfg) : kernel_of<uint16_t>(akf, bkf, cfg), dim3((unsigned)nwg), dim3(256), 0, st, g);
    return hipGetLastError() == hipSuccess ? NNT_OK : NNT_EHIP;
}

}  // namespace nnt
