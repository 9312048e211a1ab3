// Operands of products laid out afresh: in one piece, padded with zeros, for the kernels that load straight from global memory into LDS.
#include "gemm_common.hpp"
#include "nntile_mi.h"

#include <algorithm>

namespace nnt {
namespace {

template <typename T> struct Any;          // 16 bytes at any address of an element
template <> struct Any<uint16_t> { typedef uint32_t V __attribute__((ext_vector_type(4), aligned(2))); };
template <> struct Any<uint32_t> { typedef uint32_t V __attribute__((ext_vector_type(4), aligned(4))); };

constexpr int kPackVecs = 4;       // vectors per thread, their loads in flight together

// Bound by memory: every thread fetches four vectors of 16 bytes, each at any alignment, and writes them to aligned places.
template <typename T>
__global__ void __launch_bounds__(256) pack_kernel(PackOperand oa, PackOperand ob) {
    const PackOperand o = blockIdx.y ? ob : oa;
    constexpr int V = 16 / (int)sizeof(T);
    const uint32_t nvec = (uint32_t)o.pitch / V;
    const int64_t total = (int64_t)nvec * o.all_lines;
    // the four vectors step by step together: places, tiles, tile pointers, data
    const uint32_t v0 = blockIdx.x * (kPackVecs * 256) + threadIdx.x;          // (vector numbers fit 31 bits: see the plan)
    int line[kPackVecs], e[kPackVecs], first[kPackVecs], j[kPackVecs], i[kPackVecs], r[kPackVecs], ext[kPackVecs];
#pragma unroll
    for (int u = 0; u < kPackVecs; u++) {
        const uint32_t v = v0 + 256u * u;
        line[u] = (int)(v / nvec);
        e[u] = (int)(v - (uint32_t)line[u] * nvec) * V;
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
    const T* p[kPackVecs];
    uint4 x[kPackVecs];
#pragma unroll
    for (int u = 0; u < kPackVecs; u++) {
        x[u] = make_uint4(0u, 0u, 0u, 0u);
        p[u] = nullptr;
        if (line[u] < o.lines && e[u] < o.contig) p[u] = global_as<const T>(o.tiles[i[u] + o.ntc * j[u]]) + (int64_t)(line[u] - first[u]) * ext[u] + r[u];
    }
#pragma unroll
    for (int u = 0; u < kPackVecs; u++)
        if (p[u] && r[u] + V <= ext[u]) {
            const typename Any<T>::V y = *reinterpret_cast<const typename Any<T>::V*>(p[u]);
            x[u] = make_uint4(y[0], y[1], y[2], y[3]);
        }
#pragma unroll
    for (int u = 0; u < kPackVecs; u++)
        if (p[u] && r[u] + V > ext[u]) {
            // across the edge of a tile, or the end of the line
            uint32_t w[4] = {0u, 0u, 0u, 0u};
            const int room = ext[u] - r[u], left = min(V, o.contig - e[u]);
            if (o.base >= V) {
                // the elements one by one, from this tile and the next
                const T* q = p[u];
                if (left > room) q = global_as<const T>(o.tiles[i[u] + 1 + o.ntc * j[u]]) + (int64_t)(line[u] - first[u]) * min(o.base, o.contig - (i[u] + 1) * o.base) - room;
                uint32_t h[V];
#pragma unroll
                for (int k = 0; k < V; k++) h[k] = k < left ? (uint32_t)*((k < room ? p[u] : q) + k) : 0u;
#pragma unroll
                for (int k = 0; k < V; k++) w[k * 4 / V] |= V == 4 ? h[k] : h[k] << (16 * (k & 1));
            } else {
                for (int k = 0; k < left; k++) {          // (tiles narrower than a vector)
                    const int ee = e[u] + k, ii = ee / o.base;
                    const T* q = global_as<const T>(o.tiles[ii + o.ntc * j[u]]) + (int64_t)(line[u] - first[u]) * min(o.base, o.contig - ii * o.base) + (ee - ii * o.base);
                    const uint32_t hv = V == 4 ? (uint32_t)*q : (uint32_t)*q << (16 * (k & 1));
                    const int at = k * 4 / V;
                    if (at == 0) w[0] |= hv; else if (at == 1) w[1] |= hv; else if (at == 2) w[2] |= hv; else w[3] |= hv;
                }
            }
            x[u] = make_uint4(w[0], w[1], w[2], w[3]);
        }
#pragma unroll
    for (int u = 0; u < kPackVecs; u++)
        if ((int64_t)v0 + 256 * u < total) reinterpret_cast<uint4*>(o.dst)[v0 + 256u * u] = x[u];
}

}  // namespace

int32_t pack_operands(hipStream_t st, bool bf16, const PackOperand& a, const PackOperand& b) {
    const int V = bf16 ? 8 : 4;
    const int64_t most = std::max((int64_t)a.pitch / V * a.all_lines, (int64_t)b.pitch / V * b.all_lines);
    const dim3 grid((unsigned)((most + 256 * kPackVecs - 1) / (256 * kPackVecs)), 2);
    if (bf16) hipLaunchKernelGGL((pack_kernel<uint16_t>), grid, dim3(256), 0, st, a, b);
    else hipLaunchKernelGGL((pack_kernel<uint32_t>), grid, dim3(256), 0, st, a, b);
    return hipGetLastError() == hipSuccess ? NNT_OK : NNT_EHIP;
}

}  // namespace nnt
