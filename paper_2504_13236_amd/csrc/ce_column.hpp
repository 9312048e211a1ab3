// The cross-entropy loss of a column of logits in one pass (section 3, Cross-Entropy loss; whole-operation launches).
#pragma once
#include "colwise.hpp"
#include "device_util.hpp"

namespace nnt {
namespace {

// Eight bf16 or four fp32 logits as they are in memory, at any address of an element; a tile's last vector may be short
// (`cnt` elements, the rest is not touched).
template <typename T> struct RawVec;
template <> struct RawVec<float> {
    static constexpr int V = 4;
    typedef float vec __attribute__((ext_vector_type(4), aligned(4)));
    vec x;
    __device__ __forceinline__ void load(const float* p, int cnt) {
        if (cnt >= V) {
            x = *reinterpret_cast<const vec*>(p);
        } else {
#pragma unroll
            for (int j = 0; j < V; j++) x[j] = j < cnt ? p[j] : 0.f;
        }
    }
    static constexpr bool kKeeps = true;          // holds fp32 values: the shifted exponentials can take the logits' place
    __device__ __forceinline__ float at(int j) const { return x[j]; }
    __device__ __forceinline__ void set(int j, float f) { x[j] = f; }
    static __device__ __forceinline__ void store(float* p, const float (&f)[V], int cnt) {
        if (cnt >= V) {
            *reinterpret_cast<vec*>(p) = vec{f[0], f[1], f[2], f[3]};
        } else {
#pragma unroll
            for (int j = 0; j < V; j++)
                if (j < cnt) p[j] = f[j];
        }
    }
};
template <> struct RawVec<bf16_t> {
    static constexpr int V = 8;
    typedef uint32_t vec __attribute__((ext_vector_type(4), aligned(2)));
    vec x;
    __device__ __forceinline__ void load(const bf16_t* p, int cnt) {
        if (cnt >= V) {
            x = *reinterpret_cast<const vec*>(p);
        } else {
            x = vec{0u, 0u, 0u, 0u};
#pragma unroll
            for (int j = 0; j < V; j++)
                if (j < cnt) x[j >> 1] |= (uint32_t)p[j] << (16 * (j & 1));
        }
    }
    static constexpr bool kKeeps = false;
    __device__ __forceinline__ void set(int, float) {}
    __device__ __forceinline__ float at(int j) const { return __uint_as_float((j & 1) ? (x[j >> 1] & 0xffff0000u) : (x[j >> 1] << 16)); }
    static __device__ __forceinline__ void store(bf16_t* p, const float (&f)[V], int cnt) {
        if (cnt >= V) {
            vec y;
#pragma unroll
            for (int j = 0; j < 4; j++) y[j] = (uint32_t)f2bf(f[2 * j]) | ((uint32_t)f2bf(f[2 * j + 1]) << 16);
            *reinterpret_cast<vec*>(p) = y;
        } else {
#pragma unroll
            for (int j = 0; j < V; j++)
                if (j < cnt) p[j] = f2bf(f[j]);
        }
    }
};

constexpr int kCeTiles = 64;         // most vocabulary tiles of a column

// One workgroup of NT threads takes one column of logits: it reads the column once into registers (SLOTS vectors per thread),
// finds maximum and sum of shifted exponentials, and writes the gradient (probabilities, minus one at the label) over it,
// the column's statistics and its loss, which comes from the label's logit.  Bound by memory: one read and one write of
// the logits.  bf16 logits stay packed and their exponentials are taken twice: with 28 instead of 56 registers for a
// vocabulary of 50304 a compute unit holds two such workgroups, and one's reads and writes overlap with the other's (the
// 64 registers that leaves make the instances of seven and eight vectors spill 16 and 24 bytes).  The vectors of all
// vocabulary tiles are numbered through, `vt` to a tile and `nvec` in all; the addresses of the column's tiles lie in LDS,
// so that no store waits for a look-up in the tile table.
template <typename T, int SLOTS, int NT>
__global__ void __launch_bounds__(NT, (sizeof(T) == 2 && NT == 1024) ? 8 : 1) ce_column_kernel(const int32_t* labels, TiledView X, TiledView S, float* losses, int vt, int nvec) {
    constexpr int V = RawVec<T>::V, NW = NT / 64;
    __shared__ uint64_t base_of[kCeTiles];
    __shared__ float red[2][NW];
    const int tid = threadIdx.x, wave = tid >> 6;
    const int64_t col = blockIdx.x;
    const Column c = column_of(X, col);
    if (tid < X.grid[0]) base_of[tid] = reinterpret_cast<uint64_t>(col_ptr<T>(X, c, tid, ext0_of(X, tid)));
    const int lab = labels[col];
    const bool has = lab >= 0 && lab < X.shape[0];
    const int lab_tile = has ? lab / X.base[0] : 0, lab_e = lab - lab_tile * X.base[0];
    const int lab_f = has ? lab_tile * vt + lab_e / V : -1, lab_j = has ? lab_e % V : 0;
    const float inv_vt = 1.f / (float)vt;
    __syncthreads();
    // vector f: its tile (the half keeps the product away from an integer), first element, elements that exist
    auto place = [&](int f, int& l, int& e, int& cnt) {
        l = (int)(((float)f + 0.5f) * inv_vt);
        e = (f - l * vt) * V;
        cnt = ext0_of(X, l) - e;
    };
    RawVec<T> raw[SLOTS];
#pragma unroll
    for (int it = 0; it < SLOTS; it++) {
        const int f = it * NT + tid;
        if (f < nvec) {
            int l, e, cnt;
            place(f, l, e, cnt);
            raw[it].load(in_global(reinterpret_cast<const T*>(base_of[l])) + e, cnt);
        }
    }
    float mx = -__builtin_huge_valf(), x_label = 0.f;
#pragma unroll
    for (int it = 0; it < SLOTS; it++) {
        const int f = it * NT + tid;
        if (f < nvec) {
            int l, e, cnt;
            place(f, l, e, cnt);
#pragma unroll
            for (int j = 0; j < V; j++)
                if (j < cnt) mx = fmaxf(mx, raw[it].at(j));
            if (f == lab_f) {
#pragma unroll
                for (int j = 0; j < V; j++)
                    if (j == lab_j) x_label = raw[it].at(j);
            }
        }
    }
    mx = wave_max(mx);
    if ((tid & 63) == 0) red[0][wave] = mx;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; w++) mx = fmaxf(mx, red[0][w]);
    auto shifted = [&](float x) { return __builtin_amdgcn_exp2f((x - mx) * 1.4426950408889634f); };
    float sum = 0.f;
#pragma unroll
    for (int it = 0; it < SLOTS; it++) {
        const int f = it * NT + tid;
        if (f < nvec) {
            int l, e, cnt;
            place(f, l, e, cnt);
#pragma unroll
            for (int j = 0; j < V; j++) {
                const float x = shifted(raw[it].at(j));
                if (RawVec<T>::kKeeps) raw[it].set(j, x);
                if (j < cnt) sum += x;
            }
        }
    }
    sum = wave_sum(sum);
    if ((tid & 63) == 0) red[1][wave] = sum;
    __syncthreads();
    sum = 0.f;
#pragma unroll
    for (int w = 0; w < NW; w++) sum += red[1][w];       // the same order in every thread
    const float inv = 1.f / sum;
#pragma unroll
    for (int it = 0; it < SLOTS; it++) {
        const int f = it * NT + tid;
        if (f < nvec) {
            int l, e, cnt;
            place(f, l, e, cnt);
            float y[V];
#pragma unroll
            for (int j = 0; j < V; j++) y[j] = (RawVec<T>::kKeeps ? raw[it].at(j) : shifted(raw[it].at(j))) * inv;
            if (f == lab_f) {
#pragma unroll
                for (int j = 0; j < V; j++)
                    if (j == lab_j) y[j] -= 1.f;
            }
            RawVec<T>::store(in_global(reinterpret_cast<T*>(base_of[l])) + e, y, cnt);
        }
    }
    if (has ? (lab_f % NT == tid) : tid == 0) losses[col] = has ? -(x_label - mx - logf(sum)) : 0.f;
    if (tid == 0) {
        float* s = global_as<float>(S.tiles[c.stat_tile]) + 2 * (int64_t)c.colidx;
        s[0] = mx;
        s[1] = sum;
    }
}

using CeColumnFn = void (*)(const int32_t*, TiledView, TiledView, float*, int, int);
// The instance that holds a column of `nvec` vectors with the fewest registers, its workgroup size in *nt; nullptr: too long.
// Columns of up to 16384 logits (64 registers per thread of one wavefront group of four) take workgroups of 256 threads, of which a
// compute unit holds several; longer ones need all the registers that 1024 threads have.
CeColumnFn ce_column_of(int dtype, int nvec, int* nt) {
    *nt = nvec <= (dtype == NNT_F32 ? 4096 : 2048) ? 256 : 1024;
    const int per = (nvec + *nt - 1) / *nt;
    if (dtype == NNT_F32) {
        if (*nt == 256) return per <= 4 ? ce_column_kernel<float, 4, 256> : ce_column_kernel<float, 16, 256>;
        return per <= 8 ? ce_column_kernel<float, 8, 1024> : per <= 13 ? ce_column_kernel<float, 13, 1024> : per <= 16 ? ce_column_kernel<float, 16, 1024> : nullptr;
    }
    if (*nt == 256) return per <= 2 ? ce_column_kernel<bf16_t, 2, 256> : ce_column_kernel<bf16_t, 8, 256>;
    return per <= 4 ? ce_column_kernel<bf16_t, 4, 1024> : per <= 7 ? ce_column_kernel<bf16_t, 7, 1024> : per <= 8 ? ce_column_kernel<bf16_t, 8, 1024> : nullptr;
}

}  // namespace
}  // namespace nnt
