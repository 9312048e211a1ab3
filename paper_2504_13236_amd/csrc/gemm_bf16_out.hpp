// Result path shared by the bf16 product kernels: a wave's block of fp32 accumulators goes
// through LDS and leaves as 16-byte vectors along m, the contiguous index of a C tile.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "gemm_common.hpp"
#include "gemm_sums.hpp"
#include "global_ptr.hpp"

namespace nnt {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// A pointer that is the same in every lane, moved to scalar registers.
template <typename T>
__device__ __forceinline__ const T* uniform_ptr(const T* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return in_global(reinterpret_cast<const T*>(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ void store_out(float* p, float v) { *p = v; }
__device__ __forceinline__ void store_out(uint16_t* p, float v) {
    const __bf16 h = (__bf16)v;
    *p = __builtin_bit_cast(uint16_t, h);
}
__device__ __forceinline__ float load_out(const float* p) { return *p; }
__device__ __forceinline__ float load_out(const uint16_t* p) { return __uint_as_float((uint32_t)*p << 16); }

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));          // at any address of a float
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));       // at any address of a bf16 element

// 16 bytes at a 16-byte aligned address, or (ANY) at any address of an element.
template <bool ANY>
__device__ __forceinline__ uint4 get16(const void* p) {
    if constexpr (ANY) {
        const u32x4_any x = *static_cast<const u32x4_any*>(p);
        return make_uint4(x[0], x[1], x[2], x[3]);
    } else {
        return *static_cast<const uint4*>(p);
    }
}

// Writes one wave's (32 WMB) x (32 WNB) block of C = alpha * acc + bias + beta * C[+ cin_off].  `stage` is
// 32 rows of 32 WMB + 4 floats of LDS owned by the wave; every wave of the workgroup must call
// this (it synchronises the workgroup between the passes).  ANY: the vectors may start at any element (global
// memory takes 16-byte accesses at every multiple of 2 bytes), so tiles of odd leading dimensions
// leave as vectors too, and only the ragged edge goes element by element.  The direct-load kernels, whose tiles
// are nearly always aligned, use the form that tests for alignment: the other makes the compiler spill nine
// more registers of the 256 x 256 kernel with an fp32 result, which then takes 2.22 instead of 2.11 ms for
// 8192 x 32768 over 4096 tokens.
template <typename TO, int WMB, int WNB, bool ANY = false>
__device__ __forceinline__ void write_tile(float* stage, const f32x16 (&acc)[WNB][WMB], TO* C, int64_t ldc,
                                           const float* bias, float alpha, float beta, int m_base, int n_base,
                                           int m_lim, int n_lim, int lane, int64_t cin_off = 0) {
    constexpr int MW = 32 * WMB, ROW = MW + 4;
    constexpr int V = 16 / (int)sizeof(TO);          // elements per 16-byte store
    constexpr int CH = MW / V, RPI = 64 / CH;        // vectors per row, rows per pass of the wave
    static_assert(CH <= 64 && 32 % RPI == 0, "row shape");
    const int r32 = lane & 31, half = lane >> 5;
    // (the beta term comes from C + cin_off: the tile itself, or the tile of a residual input with the same geometry)
    const bool vec_ok = ANY || ((reinterpret_cast<uintptr_t>(C) % 16 == 0) && (ldc % V == 0) && (cin_off % V == 0));
#pragma unroll
    for (int bn = 0; bn < WNB; bn++) {
#pragma unroll
        for (int bm = 0; bm < WMB; bm++)
#pragma unroll
            for (int q = 0; q < 4; q++) {
                f32x4 v;
                v[0] = alpha * acc[bn][bm][4 * q];
                v[1] = alpha * acc[bn][bm][4 * q + 1];
                v[2] = alpha * acc[bn][bm][4 * q + 2];
                v[3] = alpha * acc[bn][bm][4 * q + 3];
                *reinterpret_cast<f32x4*>(&stage[r32 * ROW + bm * 32 + 8 * q + 4 * half]) = v;
            }
        __syncthreads();
        // the beta term (C itself, or a residual input's tile behind cin_off) of every row of this pass is
        // asked for before the pass's first store: a load placed after a store to what may be the same
        // tile waits for that store
        constexpr int NIT = 32 / RPI;
        uint4 cin[NIT];
        if (beta != 0.f && vec_ok) {
#pragma unroll
            for (int it = 0; it < NIT; it++) {
                const int row = it * RPI + lane / CH, mc = (lane % CH) * V;
                const int gn = n_base + bn * 32 + row, gm = m_base + mc;
                cin[it] = make_uint4(0u, 0u, 0u, 0u);
                if (gn < n_lim && gm + V <= m_lim) cin[it] = get16<ANY>(C + gm + (int64_t)gn * ldc + cin_off);
            }
        }
#pragma unroll
        for (int it = 0; it < NIT; it++) {
            const int row = it * RPI + lane / CH, mc = (lane % CH) * V;
            float v[V];
#pragma unroll
            for (int j = 0; j < V; j += 4) {
                const f32x4 x = *reinterpret_cast<const f32x4*>(&stage[row * ROW + mc + j]);
                v[j] = x[0]; v[j + 1] = x[1]; v[j + 2] = x[2]; v[j + 3] = x[3];
            }
            const int gn = n_base + bn * 32 + row, gm = m_base + mc;
            if (gn < n_lim && gm < m_lim) {
                TO* p = C + gm + (int64_t)gn * ldc;
                if (vec_ok && gm + V <= m_lim) {
                    if (bias) {
#pragma unroll
                        for (int j = 0; j < V; j += 4) {
                            const std::conditional_t<ANY, f32x4_any, f32x4> bv = *reinterpret_cast<const std::conditional_t<ANY, f32x4_any, f32x4>*>(bias + gm + j);
                            v[j] += bv[0]; v[j + 1] += bv[1]; v[j + 2] += bv[2]; v[j + 3] += bv[3];
                        }
                    }
                    if constexpr (sizeof(TO) == 4) {
                        if (beta != 0.f) {
                            const uint4 c = cin[it];
                            v[0] += beta * __uint_as_float(c.x); v[1] += beta * __uint_as_float(c.y);
                            v[2] += beta * __uint_as_float(c.z); v[3] += beta * __uint_as_float(c.w);
                        }
                        f32x4 o = {v[0], v[1], v[2], v[3]};
                        *reinterpret_cast<std::conditional_t<ANY, f32x4_any, f32x4>*>(p) = o;
                    } else {
                        if (beta != 0.f) {
                            const uint4 c = cin[it];
                            const uint32_t w[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
                            for (int j = 0; j < 4; j++) {
                                v[2 * j] += beta * __uint_as_float(w[j] << 16);
                                v[2 * j + 1] += beta * __uint_as_float(w[j] & 0xffff0000u);
                            }
                        }
                        uint32_t w[4];
#pragma unroll
                        for (int j = 0; j < 4; j++) {
                            const __bf16 lo = (__bf16)v[2 * j], hi = (__bf16)v[2 * j + 1];
                            w[j] = (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
                        }
                        if constexpr (ANY) *reinterpret_cast<u32x4_any*>(p) = u32x4_any{w[0], w[1], w[2], w[3]};
                        else *reinterpret_cast<uint4*>(p) = make_uint4(w[0], w[1], w[2], w[3]);
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < V; j++) {
                        if (gm + j < m_lim) {
                            float x = v[j] + (bias ? bias[gm + j] : 0.f);
                            if (beta != 0.f) x += beta * load_out(p + cin_off + j);
                            store_out(p + j, x);
                        }
                    }
                }
            }
        }
        __syncthreads();
    }
}

// The same for a macro-tile that may cross the edges of C's tiles (GemmSpan): every 16-byte vector goes to the part that it lies in, at any
// alignment, and vectors that cross an edge go element by element.  m_off, n_off: the wave's block within the macro-tile.
template <typename TO, int WMB, int WNB>
__device__ __forceinline__ void write_span(float* stage, const f32x16 (&acc)[WNB][WMB], const GemmSpan* span, float alpha, float beta, int m_off, int n_off, int lane) {
    constexpr int MW = 32 * WMB, ROW = MW + 4;
    constexpr int V = 16 / (int)sizeof(TO), CH = MW / V, RPI = 64 / CH, NIT = 32 / RPI;
    static_assert(CH <= 64 && 32 % RPI == 0, "row shape");
    const int r32 = lane & 31, half = lane >> 5;
    const GemmSpan s = *span;
    const int mc = (lane % CH) * V, gm = m_off + mc;
    // the part along m is the lane's for good; vectors that cross an edge are told apart here
    const bool a = gm >= s.sm;
    const bool vec = gm + V <= s.rows && (a || gm + V <= s.sm);
    TO* const C0 = in_global(static_cast<TO*>(a ? s.C[1] : s.C[0]));
    TO* const C1 = in_global(static_cast<TO*>(a ? s.C[3] : s.C[2]));
    const int64_t ldc = a ? s.ldc[1] : s.ldc[0], cin0 = a ? s.cin[1] : s.cin[0], cin1 = a ? s.cin[3] : s.cin[2];
    const float* const bias = in_global(a ? s.bias[1] : s.bias[0]);
    const bool has_bias = s.bias[0] != nullptr;
    float bv[V];
#pragma unroll
    for (int j = 0; j < V; j++) bv[j] = 0.f;
    if (has_bias && vec) {
#pragma unroll
        for (int j = 0; j < V; j += 4) {
            const f32x4_any x = *reinterpret_cast<const f32x4_any*>(bias + gm + j);
            bv[j] = x[0]; bv[j + 1] = x[1]; bv[j + 2] = x[2]; bv[j + 3] = x[3];
        }
    } else if (has_bias && gm < s.rows) {
#pragma unroll
        for (int j = 0; j < V; j++) {
            const int ge = min(gm + j, s.rows - 1);
            bv[j] = (ge >= s.sm ? in_global(s.bias[1]) : in_global(s.bias[0]))[ge];
        }
    }
    const bool edge = __any(!vec && gm < s.rows);          // some lane of the wave has a vector that crosses an edge
#pragma unroll
    for (int bn = 0; bn < WNB; bn++) {
#pragma unroll
        for (int bm = 0; bm < WMB; bm++)
#pragma unroll
            for (int q = 0; q < 4; q++) {
                f32x4 v;
                v[0] = alpha * acc[bn][bm][4 * q];
                v[1] = alpha * acc[bn][bm][4 * q + 1];
                v[2] = alpha * acc[bn][bm][4 * q + 2];
                v[3] = alpha * acc[bn][bm][4 * q + 3];
                *reinterpret_cast<f32x4*>(&stage[r32 * ROW + bm * 32 + 8 * q + 4 * half]) = v;
            }
        __syncthreads();
        uint4 cin[NIT];                  // asked for before the pass's first store (see write_tile)
        if (beta != 0.f) {
#pragma unroll
            for (int it = 0; it < NIT; it++) {
                const int gn = n_off + bn * 32 + it * RPI + lane / CH;
                cin[it] = make_uint4(0u, 0u, 0u, 0u);
                if (gn < s.cols && vec) cin[it] = get16<true>((gn >= s.sn ? C1 + cin1 : C0 + cin0) + gm + (int64_t)gn * ldc);
            }
        }
#pragma unroll
        for (int it = 0; it < NIT; it++) {
            const int row = it * RPI + lane / CH, gn = n_off + bn * 32 + row;
            float v[V];
#pragma unroll
            for (int j = 0; j < V; j += 4) {
                const f32x4 x = *reinterpret_cast<const f32x4*>(&stage[row * ROW + mc + j]);
                v[j] = x[0]; v[j + 1] = x[1]; v[j + 2] = x[2]; v[j + 3] = x[3];
            }
            if (vec && gn < s.cols) {
                TO* p = (gn >= s.sn ? C1 : C0) + gm + (int64_t)gn * ldc;
#pragma unroll
                for (int j = 0; j < V; j++) v[j] += bv[j];
                if constexpr (sizeof(TO) == 4) {
                    if (beta != 0.f) {
                        const uint4 c = cin[it];
                        v[0] += beta * __uint_as_float(c.x); v[1] += beta * __uint_as_float(c.y);
                        v[2] += beta * __uint_as_float(c.z); v[3] += beta * __uint_as_float(c.w);
                    }
                    *reinterpret_cast<f32x4_any*>(p) = f32x4_any{v[0], v[1], v[2], v[3]};
                } else {
                    if (beta != 0.f) {
                        const uint4 c = cin[it];
                        const uint32_t w[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
                        for (int j = 0; j < 4; j++) {
                            v[2 * j] += beta * __uint_as_float(w[j] << 16);
                            v[2 * j + 1] += beta * __uint_as_float(w[j] & 0xffff0000u);
                        }
                    }
                    uint32_t w[4];
#pragma unroll
                    for (int j = 0; j < 4; j++) {
                        const __bf16 lo = (__bf16)v[2 * j], hi = (__bf16)v[2 * j + 1];
                        w[j] = (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
                    }
                    *reinterpret_cast<u32x4_any*>(p) = u32x4_any{w[0], w[1], w[2], w[3]};
                }
            }
        }
        if (edge && !vec && gm < s.rows) {
            // (the passes one after the other: their vectors lie in LDS; straight code for all of them keeps the loop above from being
            // unrolled, and with it the accumulators out of registers)
#pragma unroll 1
            for (int it = 0; it < NIT; it++) {
                const int row = it * RPI + lane / CH, gn = n_off + bn * 32 + row;
                if (gn >= s.cols) break;
                const bool b = gn >= s.sn;
                TO* const P0 = in_global(static_cast<TO*>(b ? s.C[2] : s.C[0])) + (int64_t)gn * s.ldc[0];
                TO* const P1 = in_global(static_cast<TO*>(b ? s.C[3] : s.C[1])) + (int64_t)gn * s.ldc[1];
                const int64_t c0 = b ? s.cin[2] : s.cin[0], c1 = b ? s.cin[3] : s.cin[1];
                float x[V];
#pragma unroll
                for (int j = 0; j < V; j++) {
                    const int ge = gm + j;
                    x[j] = stage[row * ROW + mc + j] + bv[j];
                    if (beta != 0.f && ge < s.rows) x[j] += beta * load_out(ge >= s.sm ? P1 + ge + c1 : P0 + ge + c0);
                }
#pragma unroll
                for (int j = 0; j < V; j++) {
                    const int ge = gm + j;
                    if (ge < s.rows) store_out((ge >= s.sm ? P1 : P0) + ge, x[j]);
                }
            }
        }
        __syncthreads();
    }
}

}  // namespace nnt
