// bf16 products of operands that no kernel can load straight into LDS: odd leading dimensions, tiles or contractions that are no
// multiples of 8.  Such products ran on the register-staged kernel, whose loads are in flight for one k-step of 32 and whose
// macro-tiles end at every tile's edge: 130 to 220 TFLOP/s.  Here a first kernel lays both operands out afresh (pack_kernel), in one piece each and
// padded, and the direct-load kernels run on that, with macro-tiles on one grid over all of C, so that neither the tiles'
// edges nor their alignment cost anything in the loop.  Their result path sorts the results into C's tiles.
// The copy moves 4 bytes per element of A and B; the three products of a layer of 1333 x 2001 over 2068 tokens on tiles of 500, copies
// included: 81 -> 53, 76 -> 44 and 51 -> 42 us, the layer 168 -> 92.
#include "gemm_bf16_dl_body.hpp"

#include <algorithm>

namespace nnt {
namespace {

// ------------------------------------------------------------------ operands laid out afresh
typedef uint32_t u32x4_any2 __attribute__((ext_vector_type(4), aligned(2)));

constexpr int kPackVecs = 4;       // vectors per thread, their loads in flight together

// Bound by memory: every thread fetches four vectors of 8 elements, each at any alignment, and writes them to aligned places.
__global__ void __launch_bounds__(256) pack_kernel(PackOperand oa, PackOperand ob) {
    const PackOperand o = blockIdx.y ? ob : oa;
    const uint32_t nvec = (uint32_t)o.pitch / 8;
    const int64_t total = (int64_t)nvec * o.all_lines;
    // the four vectors step by step together: places, tiles, tile pointers, data
    const uint32_t v0 = blockIdx.x * (kPackVecs * 256) + threadIdx.x;          // (vector numbers fit 31 bits: see the plan)
    int line[kPackVecs], e[kPackVecs], first[kPackVecs], j[kPackVecs], i[kPackVecs], r[kPackVecs], ext[kPackVecs];
#pragma unroll
    for (int u = 0; u < kPackVecs; u++) {
        const uint32_t v = v0 + 256u * u;
        line[u] = (int)(v / nvec);
        e[u] = (int)(v - (uint32_t)line[u] * nvec) * 8;
        first[u] = j[u] = 0;
        i[u] = (int)((uint32_t)e[u] / (uint32_t)o.base);
        r[u] = e[u] - i[u] * o.base;
        ext[u] = min(o.base, o.contig - i[u] * o.base);
    }
    for (int q = 1; q < o.ntl; q++) {
        const int s = o.line0[q];
#pragma unroll
        for (int u = 0; u < kPackVecs; u++)
            if (line[u] >= s) { first[u] = s; j[u] = q; }
    }
    const uint16_t* p[kPackVecs];
    uint4 x[kPackVecs];
#pragma unroll
    for (int u = 0; u < kPackVecs; u++) {
        x[u] = make_uint4(0u, 0u, 0u, 0u);
        p[u] = nullptr;
        if (line[u] < o.lines && e[u] < o.contig) p[u] = global_as<const uint16_t>(o.tiles[i[u] + o.ntc * j[u]]) + (int64_t)(line[u] - first[u]) * ext[u] + r[u];
    }
#pragma unroll
    for (int u = 0; u < kPackVecs; u++)
        if (p[u] && r[u] + 8 <= ext[u]) {
            const u32x4_any2 y = *reinterpret_cast<const u32x4_any2*>(p[u]);
            x[u] = make_uint4(y[0], y[1], y[2], y[3]);
        }
#pragma unroll
    for (int u = 0; u < kPackVecs; u++)
        if (p[u] && r[u] + 8 > ext[u]) {
            // across the edge of a tile, or the end of the line
            uint32_t w[4] = {0u, 0u, 0u, 0u};
            const int room = ext[u] - r[u], left = min(8, o.contig - e[u]);
            if (o.base >= 8) {
                // the elements one by one, from this tile and the next
                const uint16_t* q = p[u];
                if (left > room) q = global_as<const uint16_t>(o.tiles[i[u] + 1 + o.ntc * j[u]]) + (int64_t)(line[u] - first[u]) * min(o.base, o.contig - (i[u] + 1) * o.base) - room;
                uint32_t h[8];
#pragma unroll
                for (int k = 0; k < 8; k++) h[k] = k < left ? (uint32_t)*((k < room ? p[u] : q) + k) : 0u;
#pragma unroll
                for (int k = 0; k < 8; k++) w[k >> 1] |= h[k] << (16 * (k & 1));
            } else {
                for (int k = 0; k < left; k++) {          // (tiles narrower than a vector)
                    const int ee = e[u] + k, ii = ee / o.base;
                    const uint16_t* q = global_as<const uint16_t>(o.tiles[ii + o.ntc * j[u]]) + (int64_t)(line[u] - first[u]) * min(o.base, o.contig - ii * o.base) + (ee - ii * o.base);
                    const uint32_t hv = (uint32_t)*q << (16 * (k & 1));
                    if (k < 2) w[0] |= hv; else if (k < 4) w[1] |= hv; else if (k < 6) w[2] |= hv; else w[3] |= hv;
                }
            }
            x[u] = make_uint4(w[0], w[1], w[2], w[3]);
        }
#pragma unroll
    for (int u = 0; u < kPackVecs; u++)
        if ((int64_t)v0 + 256 * u < total) reinterpret_cast<uint4*>(o.dst)[v0 + 256u * u] = x[u];
}

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

int32_t pack_operands(hipStream_t st, const PackOperand& a, const PackOperand& b) {
    const int64_t most = std::max((int64_t)a.pitch / 8 * a.all_lines, (int64_t)b.pitch / 8 * b.all_lines);
    hipLaunchKernelGGL(pack_kernel, dim3((unsigned)((most + 256 * kPackVecs - 1) / (256 * kPackVecs)), 2), dim3(256), 0, st, a, b);
    return hipGetLastError() == hipSuccess ? NNT_OK : NNT_EHIP;
}

}  // namespace nnt
