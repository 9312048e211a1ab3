// bf16 product kernels on the tiles of C: direct-load kernels for aligned operands (the loop is in gemm_bf16_dl_body.hpp).
#include "gemm_bf16_dl_body.hpp"

namespace nnt {
namespace {

template <typename TO, bool AKF, bool BKF>
__global__ void __launch_bounds__(256) gemm_bf16_dl_kernel(const GemmArgs g) {
    __shared__ __attribute__((aligned(16))) char lds[DlShape<4>::kLdsBytes];
    dl_body<TO, AKF, BKF, 4>(g, lds);
}

// two workgroups per compute unit: at most 256 registers per lane
template <typename TO, bool AKF, bool BKF, bool RAG>
__global__ void __launch_bounds__(256, 2) gemm_bf16_dl_tall_kernel(const GemmArgs g) {
    __shared__ __attribute__((aligned(16))) char lds[DlShape<2>::kLdsBytes];
    dl_body<TO, AKF, BKF, 2, RAG>(g, lds);
}

// 128 x 128 macro-tiles for products with few rows (m = head size: the other operand is the score-shaped one and
// the kernel streams it): the four waves side by side, 128 rows x 32 columns each, five stages of 16 KB so that
// the loads of four k-steps are in flight, two workgroups per compute unit.  Always the ragged variant (m = 64
// is half a macro-tile; sequence tiles need not be multiples of 128).
template <typename TO, bool AKF, bool BKF>
__global__ void __launch_bounds__(256, 2) gemm_bf16_dl_wide_kernel(const GemmArgs g) {
    __shared__ __attribute__((aligned(16))) char lds[DlShape<1, 1>::kLdsBytes];
    dl_body<TO, AKF, BKF, 1, true, 1>(g, lds);
}

using KernelFn = void (*)(const GemmArgs);

template <typename TO>
KernelFn wide_kernel_of(int akf, int bkf) {
    if (akf) return bkf ? gemm_bf16_dl_wide_kernel<TO, true, true> : gemm_bf16_dl_wide_kernel<TO, true, false>;
    return bkf ? gemm_bf16_dl_wide_kernel<TO, false, true> : gemm_bf16_dl_wide_kernel<TO, false, false>;
}

template <typename TO, bool RAG>
KernelFn tall_kernel_of(int akf, int bkf) {
    if (akf) return bkf ? gemm_bf16_dl_tall_kernel<TO, true, true, RAG> : gemm_bf16_dl_tall_kernel<TO, true, false, RAG>;
    return bkf ? gemm_bf16_dl_tall_kernel<TO, false, true, RAG> : gemm_bf16_dl_tall_kernel<TO, false, false, RAG>;
}

template <typename TO>
KernelFn kernel_of(int akf, int bkf, bool tall, bool ragged) {
    if (tall) return ragged ? tall_kernel_of<TO, true>(akf, bkf) : tall_kernel_of<TO, false>(akf, bkf);
    if (akf) return bkf ? gemm_bf16_dl_kernel<TO, true, true> : gemm_bf16_dl_kernel<TO, true, false>;
    return bkf ? gemm_bf16_dl_kernel<TO, false, true> : gemm_bf16_dl_kernel<TO, false, false>;
}

KernelFn kernel_of(int out_is_f32, int akf, int bkf, int cfg, bool ragged) {
    if (cfg == kCfgWide) return out_is_f32 ? wide_kernel_of<float>(akf, bkf) : wide_kernel_of<uint16_t>(akf, bkf);
    return out_is_f32 ? kernel_of<float>(akf, bkf, cfg == kCfgTall, ragged) : kernel_of<uint16_t>(akf, bkf, cfg == kCfgTall, ragged);
}

}  // namespace

int32_t launch_gemm_bf16_dl(hipStream_t st, int out_is_f32, int akf, int bkf, int cfg, bool ragged, const GemmArgs& g, int64_t nwg) {
    if (nwg <= 0) return NNT_OK;
    if (ragged && cfg != kCfgTall && cfg != kCfgWide) return NNT_EINVAL;
    hipLaunchKernelGGL(kernel_of(out_is_f32, akf, bkf, cfg, ragged), dim3((unsigned)nwg), dim3(256), 0, st, g);
    return hipGetLastError() == hipSuccess ? NNT_OK : NNT_EHIP;
}


}  // namespace nnt
