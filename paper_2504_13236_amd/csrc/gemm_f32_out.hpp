// Result path of the fp32 product kernels whose macro-tiles may end inside their C tile.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_common.hpp"
#include "gemm_sums.hpp"
#include "global_ptr.hpp"

namespace nnt {

// Writes one wave's (32 WMB) x (32 WNB) block of C = alpha * acc + bias + beta * C[+ cin_off]: a lane holds row
// m = lane % 32 and columns 8 * (i / 4) + 4 * (lane / 32) + i % 4 of each 32 x 32 block, so a half-wave stores 32
// consecutive rows.  The beta terms of a row block are read before its first store and waited for once: with the loads
// and the tests for the edge in one place the compiler puts a full wait before every single store, and 64 store
// latencies in a row are 7 us of a workgroup's life (what a 128 x 128 macro-tile of 128 k takes in all).
template <int WMB, int WNB>
__device__ __forceinline__ void write_tile_f32(const f32x16 (&acc)[WNB][WMB], float* C, int64_t ldc, int64_t cin_off, const float* bias_ptr,
                                               float alpha, float beta, int m_base, int n_base, int m_lim, int n_lim, int lane) {
    const int r32 = lane & 31, half = lane >> 5;
#pragma unroll
    for (int bm = 0; bm < WMB; bm++) {
        const int gm = m_base + 32 * bm + r32;
        if (gm >= m_lim) continue;
        const float bias = bias_ptr ? bias_ptr[gm] : 0.f;
        float* row = C + gm + (int64_t)(n_base + 4 * half) * ldc;
        float cin[WNB][16];
        if (beta != 0.f) {
#pragma unroll
            for (int bn = 0; bn < WNB; bn++)
#pragma unroll
                for (int i = 0; i < 16; i++) {
                    const int c = 32 * bn + 8 * (i >> 2) + (i & 3);
                    cin[bn][i] = n_base + c + 4 * half < n_lim ? row[(int64_t)c * ldc + cin_off] : 0.f;
                }
        } else {
#pragma unroll
            for (int bn = 0; bn < WNB; bn++)
#pragma unroll
                for (int i = 0; i < 16; i++) cin[bn][i] = 0.f;
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);        // vmcnt(0): no load is pending at the stores below
#pragma unroll
        for (int bn = 0; bn < WNB; bn++) {
            float* p = row + (int64_t)(32 * bn) * ldc;
            float v[16];
#pragma unroll
            for (int i = 0; i < 16; i++) {
                v[i] = alpha * acc[bn][bm][i] + bias;
                if (beta != 0.f) v[i] += beta * cin[bn][i];
            }
            if (n_base + 32 * bn + 32 <= n_lim) {          // uniform: the whole block of columns exists
#pragma unroll
                for (int i = 0; i < 16; i++) p[(int64_t)(8 * (i >> 2) + (i & 3)) * ldc] = v[i];
            } else {
                const int left = n_lim - (n_base + 32 * bn + 4 * half);
#pragma unroll
                for (int i = 0; i < 16; i++)
                    if (8 * (i >> 2) + (i & 3) < left) p[(int64_t)(8 * (i >> 2) + (i & 3)) * ldc] = v[i];
            }
        }
    }
}

// The same for a macro-tile that may cross the edges of C's tiles (GemmSpan).  m_off, n_off: the wave's block within the macro-tile.
template <int WMB, int WNB>
__device__ __forceinline__ void write_span_f32(const f32x16 (&acc)[WNB][WMB], const GemmSpan* span, float alpha, float beta, int m_off, int n_off, int lane) {
    const GemmSpan s = *span;
    const int r32 = lane & 31, half = lane >> 5;
#pragma unroll
    for (int bm = 0; bm < WMB; bm++) {
        const int gm = m_off + 32 * bm + r32;
        if (gm >= s.rows) continue;
        const bool a = gm >= s.sm;
        float* const C0 = in_global(static_cast<float*>(a ? s.C[1] : s.C[0])) + gm;
        float* const C1 = in_global(static_cast<float*>(a ? s.C[3] : s.C[2])) + gm;
        const int64_t ldc = a ? s.ldc[1] : s.ldc[0], cin0 = a ? s.cin[1] : s.cin[0], cin1 = a ? s.cin[3] : s.cin[2];
        const float bias = s.bias[0] ? (a ? in_global(s.bias[1]) : in_global(s.bias[0]))[gm] : 0.f;
#pragma unroll
        for (int bn = 0; bn < WNB; bn++) {
            float cin[16];
#pragma unroll
            for (int i = 0; i < 16; i++) {
                const int gn = n_off + 32 * bn + 8 * (i >> 2) + 4 * half + (i & 3);
                cin[i] = 0.f;
                if (beta != 0.f && gn < s.cols) cin[i] = (gn >= s.sn ? C1 + cin1 : C0 + cin0)[(int64_t)gn * ldc];
            }
            __builtin_amdgcn_s_waitcnt(0x0F70);        // vmcnt(0): no load is pending at the stores below (see write_tile_f32)
#pragma unroll
            for (int i = 0; i < 16; i++) {
                const int gn = n_off + 32 * bn + 8 * (i >> 2) + 4 * half + (i & 3);
                float v = alpha * acc[bn][bm][i] + bias;
                if (beta != 0.f) v += beta * cin[i];
                if (gn < s.cols) (gn >= s.sn ? C1 : C0)[(int64_t)gn * ldc] = v;
            }
        }
    }
}

}  // namespace nnt
