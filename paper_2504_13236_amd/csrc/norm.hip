// Layer normalisation over the embedding axis (section 3, layer normalization) and
// the column-sum reductions (bias gradient, gain / bias gradients).
//
// Tile form: the paper's steps, one kernel per step and tile -- (1) fold the
// tile's mean and variance into the running statistics, (2)+(3) normalise, scale
// and add the bias.  Tensor form: one wavefront per token walks all embedding
// tiles of that token through the tile-pointer table; the token's values stay in
// registers between the statistics pass and the output pass when they fit, so a
// whole tiled tensor costs one read and one write.  All statistics are fp32; the
// variance is the mean of the squared deviations from the mean (two passes over
// the cached token), never a difference of two large sums.
#include "colwise.hpp"
#include "internal.hpp"

#include <algorithm>
#include <mutex>

namespace nnt {
namespace {

// Visits every V-wide vector of a column: fn(slot, l, e, ext) with l the tile
// along axis 0, e the first row inside it and ext the tile's extent.  With NV > 0
// the loop is fully unrolled and `slot` is a compile-time index into a per-lane
// register cache; with NV == 0 it is a plain loop and slot is 0.
// ANY (only with NV > 0): tiles of any extent and alignment.  A vector that would pass the tile's end is moved back to end there, and
// fn(slot, l, e, ext, own) is told which of its elements are the vector's own (the others belong to its neighbour, or do not exist in tiles shorter
// than a vector).
struct Own { int lo, hi; __device__ __forceinline__ bool operator()(int k) const { return k >= lo && k < hi; } };
template <int V, int NV, int WPT = 1, bool ANY = false, typename Fn>
__device__ __forceinline__ void walk(const TiledView& v, int lane, Fn fn, int w = 0) {
    const int g0 = v.grid[0];
    if constexpr (NV > 0) {
        const int vpt = (v.base[0] + 64 * V - 1) / (64 * V);
        int l = 0, j = 0;                 // slot it is vector j of tile l (counted up: no division per slot)
        if constexpr (WPT > 1) {          // wave w of the WPT that share the column takes every WPT-th vector
            l = w / vpt;
            j = w - l * vpt;
        }
#pragma unroll
        for (int it = 0; it < NV; it++) {
            if (l < g0) {
                const int ext = ext0_of(v, l);
                const int e = (j * 64 + lane) * V;
                if constexpr (ANY) {
                    if (e < ext) {
                        const int at = max(min(e, ext - V), 0);
                        fn(it, l, at, ext, Own{e - at, min(V, ext - at)});
                    }
                } else {
                    if (e < ext) fn(it, l, e, ext, Own{0, V});
                }
            }
            if constexpr (WPT == 1) {
                if (++j == vpt) {
                    j = 0;
                    l++;
                }
            } else {
                j += WPT;
                while (j >= vpt) {
                    j -= vpt;
                    l++;
                }
            }
        }
    } else {
        for (int l = 0; l < g0; l++) {
            const int ext = ext0_of(v, l);
            for (int e = (w * 64 + lane) * V; e < ext; e += 64 * V * WPT) fn(0, l, e, ext, Own{0, V});
        }
    }
}

// V elements at any address of an element; `n` < V of them where a tile is shorter than a vector (the same in every lane of a wave).
typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u4_any __attribute__((ext_vector_type(4), aligned(2)));
template <bool ANY, int V> __device__ __forceinline__ void ldn(const float* p, int n, float (&f)[V]) {
    if constexpr (!ANY || V == 1) {
        ldv<V>(p, f);
    } else if (n >= V) {
#pragma unroll
        for (int i = 0; i < V; i += 4) {
            const f4_any x = *reinterpret_cast<const f4_any*>(p + i);
            f[i] = x[0]; f[i + 1] = x[1]; f[i + 2] = x[2]; f[i + 3] = x[3];
        }
    } else {
#pragma unroll
        for (int i = 0; i < V; i++) f[i] = i < n ? p[i] : 0.f;
    }
}
template <bool ANY, int V> __device__ __forceinline__ void ldn(const bf16_t* p, int n, float (&f)[V]) {
    if constexpr (!ANY || V == 1) {
        ldv<V>(p, f);
    } else if (n >= V) {
        const u4_any x = *reinterpret_cast<const u4_any*>(p);
#pragma unroll
        for (int i = 0; i < 4; i++) { f[2 * i] = __uint_as_float(x[i] << 16); f[2 * i + 1] = __uint_as_float(x[i] & 0xffff0000u); }
    } else {
#pragma unroll
        for (int i = 0; i < V; i++) f[i] = i < n ? bf2f(p[i]) : 0.f;
    }
}
template <bool ANY, int V> __device__ __forceinline__ void stn(float* p, int n, const float (&f)[V]) {
    if constexpr (!ANY || V == 1) {
        stv<V>(p, f);
    } else if (n >= V) {
        *reinterpret_cast<f4_any*>(p) = f4_any{f[0], f[1], f[2], f[3]};
    } else {
#pragma unroll
        for (int i = 0; i < V; i++) if (i < n) p[i] = f[i];
    }
}
template <bool ANY, int V> __device__ __forceinline__ void stn(bf16_t* p, int n, const float (&f)[V]) {
    if constexpr (!ANY || V == 1) {
        stv<V>(p, f);
    } else if (n >= V) {
        u4_any x;
#pragma unroll
        for (int i = 0; i < 4; i++) x[i] = (uint32_t)f2bf(f[2 * i]) | ((uint32_t)f2bf(f[2 * i + 1]) << 16);
        *reinterpret_cast<u4_any*>(p) = x;
    } else {
#pragma unroll
        for (int i = 0; i < V; i++) if (i < n) p[i] = f2bf(f[i]);
    }
}

// Sum over the WPT wavefronts that share a column (all of one workgroup), in wave order.
template <int WPT>
__device__ __forceinline__ float column_sum(float x, float* red, int w, int lane) {
    x = wave_sum(x);
    if constexpr (WPT == 1) return x;
    if (lane == 0) red[w] = x;
    __syncthreads();
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < WPT; i++) s += red[i];
    __syncthreads();
    return s;
}

// WPT = 1: one wavefront per token, four tokens per workgroup.  WPT = 4: the workgroup's four wavefronts share
// one token (long tokens: a quarter of the registers per wave, four times the waves in flight).
template <typename T, int V, int NV, int WPT = 1, bool ANY = false>
__global__ void __launch_bounds__(256) ln_fwd_fused(TiledView X, TiledView Y, TiledView S, TiledView G, TiledView Bt,
                                                     float eps, int64_t ncols) {
    __shared__ float red[4];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);      // wave-uniform: the index arithmetic below runs on the scalar unit
    const int64_t col = WPT == 1 ? (int64_t)blockIdx.x * 4 + wave : (int64_t)blockIdx.x;
    const int w = WPT == 1 ? 0 : wave;
    if (col >= ncols) return;
    const Column c = column_of(X, col);
    const int N = X.shape[0];
    float cache[NV > 0 ? NV : 1][V];
    // Two passes, mean first and then the squared deviations from it (the one-pass forms cancel when one
    // element of the token lies far from the rest).  The second pass runs over the register cache when
    // the token fits there and re-reads the token otherwise (it is still in the L2 of this wave's XCD).
    float s1 = 0.f;
    walk<V, NV, WPT, ANY>(X, lane, [&](int slot, int l, int e, int ext, Own own) {
        float x[V];
        ldn<ANY, V>(col_ptr<const T>(X, c, l, ext) + e, ext, x);
#pragma unroll
        for (int k = 0; k < V; k++) {
            s1 += !ANY || own(k) ? x[k] : 0.f;
            if constexpr (NV > 0) cache[slot][k] = x[k];
        }
    }, w);
    const float mean = column_sum<WPT>(s1, red, w, lane) / (float)N;
    float s2 = 0.f;
    walk<V, NV, WPT, ANY>(X, lane, [&](int slot, int l, int e, int ext, Own own) {
        float x[V];
        if constexpr (NV > 0) {
#pragma unroll
            for (int k = 0; k < V; k++) x[k] = cache[slot][k];
        } else {
            ldn<ANY, V>(col_ptr<const T>(X, c, l, ext) + e, ext, x);
        }
#pragma unroll
        for (int k = 0; k < V; k++) s2 += !ANY || own(k) ? (x[k] - mean) * (x[k] - mean) : 0.f;
    }, w);
    const float var = column_sum<WPT>(s2, red, w, lane) / (float)N;
    const float rstd = 1.f / sqrtf(var + eps);
    walk<V, NV, WPT, ANY>(X, lane, [&](int slot, int l, int e, int ext, Own own) {
        float x[V], g[V], b[V];
        if constexpr (NV > 0) {
#pragma unroll
            for (int k = 0; k < V; k++) x[k] = cache[slot][k];
        } else {
            ldn<ANY, V>(col_ptr<const T>(X, c, l, ext) + e, ext, x);
        }
        ldn<ANY, V>(global_as<const float>(G.tiles[l]) + e, ext, g);
        ldn<ANY, V>(global_as<const float>(Bt.tiles[l]) + e, ext, b);
#pragma unroll
        for (int k = 0; k < V; k++) x[k] = g[k] * ((x[k] - mean) * rstd) + b[k];
        stn<ANY, V>(col_ptr<T>(Y, c, l, ext) + e, ext, x);
    }, w);
    if (lane == 0 && w == 0) {
        float* s = global_as<float>(S.tiles[c.stat_tile]) + 2 * (int64_t)c.colidx;
        s[0] = mean;
        s[1] = rstd;
    }
}

template <typename T, int V, int NV, int WPT = 1>
__global__ void __launch_bounds__(256) ln_bwd_fused(TiledView X, TiledView S, TiledView G, TiledView dY, TiledView dR,
                                                     TiledView dX, int has_res, int64_t ncols) {
    __shared__ float red[4];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);      // wave-uniform: the index arithmetic below runs on the scalar unit
    const int64_t col = WPT == 1 ? (int64_t)blockIdx.x * 4 + wave : (int64_t)blockIdx.x;
    const int w = WPT == 1 ? 0 : wave;
    if (col >= ncols) return;
    const Column c = column_of(X, col);
    const int N = X.shape[0];
    const float* st = global_as<const float>(S.tiles[c.stat_tile]) + 2 * (int64_t)c.colidx;
    const float mean = st[0], rstd = st[1];
    float cg[NV > 0 ? NV : 1][V], ch[NV > 0 ? NV : 1][V];   // g = dy * gamma, xhat
    float a = 0.f, b = 0.f;
    walk<V, NV, WPT>(X, lane, [&](int slot, int l, int e, int ext, Own) {
        float x[V], d[V], g[V];
        ldv<V>(col_ptr<const T>(X, c, l, ext) + e, x);
        ldv<V>(col_ptr<const T>(dY, c, l, ext) + e, d);
        ldv<V>(global_as<const float>(G.tiles[l]) + e, g);
#pragma unroll
        for (int k = 0; k < V; k++) {
            const float gg = d[k] * g[k], xh = (x[k] - mean) * rstd;
            a += gg;
            b += gg * xh;
            if constexpr (NV > 0) { cg[slot][k] = gg; ch[slot][k] = xh; }
        }
    }, w);
    a = column_sum<WPT>(a, red, w, lane) / (float)N;
    b = column_sum<WPT>(b, red, w, lane) / (float)N;
    walk<V, NV, WPT>(X, lane, [&](int slot, int l, int e, int ext, Own) {
        float gg[V], xh[V], r[V];
        if constexpr (NV > 0) {
#pragma unroll
            for (int k = 0; k < V; k++) { gg[k] = cg[slot][k]; xh[k] = ch[slot][k]; }
        } else {
            float x[V], d[V], g[V];
            ldv<V>(col_ptr<const T>(X, c, l, ext) + e, x);
            ldv<V>(col_ptr<const T>(dY, c, l, ext) + e, d);
            ldv<V>(global_as<const float>(G.tiles[l]) + e, g);
#pragma unroll
            for (int k = 0; k < V; k++) { gg[k] = d[k] * g[k]; xh[k] = (x[k] - mean) * rstd; }
        }
#pragma unroll
        for (int k = 0; k < V; k++) r[k] = rstd * (gg[k] - a - xh[k] * b);
        if (has_res) {
            float q[V];
            ldv<V>(col_ptr<const T>(dR, c, l, ext) + e, q);
#pragma unroll
            for (int k = 0; k < V; k++) r[k] += q[k];
        }
        stv<V>(col_ptr<T>(dX, c, l, ext) + e, r);
    }, w);
}

// ------------------------------------------------------------------ tile-form kernels (one wave per token of an m x n tile)
template <typename T, int V>
__global__ void __launch_bounds__(256) ln_stats_tile(const T* x, float* stats, int m, int64_t n, int64_t count_before,
                                                      int64_t finalize_total, float eps) {
    const int lane = threadIdx.x & 63;
    const int64_t col = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);      // wave-uniform: the index arithmetic below runs on the scalar unit
    if (col >= n) return;
    const T* p = x + col * m;
    float s = 0.f;
    for (int e = lane * V; e < m; e += 64 * V) {
        float f[V];
        ldv<V>(p + e, f);
#pragma unroll
        for (int k = 0; k < V; k++) s += f[k];
    }
    const float mean_t = wave_sum(s) / (float)m;
    float q = 0.f;
    for (int e = lane * V; e < m; e += 64 * V) {
        float f[V];
        ldv<V>(p + e, f);
#pragma unroll
        for (int k = 0; k < V; k++) q += (f[k] - mean_t) * (f[k] - mean_t);
    }
    const float m2_t = wave_sum(q);
    if (lane == 0) {
        float mean = mean_t, m2 = m2_t;
        const float na = (float)count_before, nb = (float)m;
        if (count_before > 0) {
            // pairwise update of (count, mean, sum of squared deviations)
            const float mean_a = stats[2 * col], m2_a = stats[2 * col + 1];
            const float delta = mean_t - mean_a;
            mean = mean_a + delta * (nb / (na + nb));
            m2 = m2_a + m2_t + delta * delta * (na * nb / (na + nb));
        }
        if (finalize_total > 0) m2 = 1.f / sqrtf(m2 / (float)finalize_total + eps);
        stats[2 * col] = mean;
        stats[2 * col + 1] = m2;
    }
}

template <typename T, int V>
__global__ void __launch_bounds__(256) ln_apply_tile(const T* x, const float* stats, const float* gamma, const float* beta,
                                                      T* y, int m, int64_t n) {
    const int lane = threadIdx.x & 63;
    const int64_t col = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);      // wave-uniform: the index arithmetic below runs on the scalar unit
    if (col >= n) return;
    const float mean = stats[2 * col], rstd = stats[2 * col + 1];
    for (int e = lane * V; e < m; e += 64 * V) {
        float f[V], g[V], b[V];
        ldv<V>(x + col * m + e, f);
        ldv<V>(gamma + e, g);
        ldv<V>(beta + e, b);
#pragma unroll
        for (int k = 0; k < V; k++) f[k] = g[k] * ((f[k] - mean) * rstd) + b[k];
        stv<V>(y + col * m + e, f);
    }
}

template <typename T, int V>
__global__ void __launch_bounds__(256) ln_bwd_sums_tile(const T* x, const float* stats, const float* gamma, const T* dy,
                                                         float* sums, int init, int m, int64_t n) {
    const int lane = threadIdx.x & 63;
    const int64_t col = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);      // wave-uniform: the index arithmetic below runs on the scalar unit
    if (col >= n) return;
    const float mean = stats[2 * col], rstd = stats[2 * col + 1];
    float a = 0.f, b = 0.f;
    for (int e = lane * V; e < m; e += 64 * V) {
        float f[V], d[V], g[V];
        ldv<V>(x + col * m + e, f);
        ldv<V>(dy + col * m + e, d);
        ldv<V>(gamma + e, g);
#pragma unroll
        for (int k = 0; k < V; k++) {
            const float gg = d[k] * g[k];
            a += gg;
            b += gg * ((f[k] - mean) * rstd);
        }
    }
    a = wave_sum(a);
    b = wave_sum(b);
    if (lane == 0) {
        if (init) { sums[2 * col] = a; sums[2 * col + 1] = b; }
        else { sums[2 * col] += a; sums[2 * col + 1] += b; }
    }
}

template <typename T, int V>
__global__ void __launch_bounds__(256) ln_bwd_dx_tile(const T* x, const float* stats, const float* gamma, const T* dy,
                                                       const float* sums, const T* dres, T* dx, int m, int64_t n, float inv_N) {
    const int lane = threadIdx.x & 63;
    const int64_t col = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);      // wave-uniform: the index arithmetic below runs on the scalar unit
    if (col >= n) return;
    const float mean = stats[2 * col], rstd = stats[2 * col + 1];
    const float a = sums[2 * col] * inv_N, b = sums[2 * col + 1] * inv_N;
    for (int e = lane * V; e < m; e += 64 * V) {
        float f[V], d[V], g[V];
        ldv<V>(x + col * m + e, f);
        ldv<V>(dy + col * m + e, d);
        ldv<V>(gamma + e, g);
#pragma unroll
        for (int k = 0; k < V; k++) f[k] = rstd * (d[k] * g[k] - a - ((f[k] - mean) * rstd) * b);
        if (dres) {
            float q[V];
            ldv<V>(dres + col * m + e, q);
#pragma unroll
            for (int k = 0; k < V; k++) f[k] += q[k];
        }
        stv<V>(dx + col * m + e, f);
    }
}

// ------------------------------------------------------------------ column sums in two stages
// Stage 1: block (bx, by, tile) sums the rows [bx * 64 V, ...) of one tile over the
// columns [by * cpb, (by + 1) * cpb) and stores a partial row; stage 2 adds the
// partials of every row.  MODE 0: sum of dy (bias gradient).  MODE 1: sums of
// dy * xhat and of dy (gain and bias gradients of the layer norm).
struct RowsumGeom {
    TiledView y;            // tiling (tensor form)
    void* const* ytab;      // tile tables (tensor form) ...
    void* const* xtab;
    void* const* stab;
    const void* y1;         // ... or single tiles
    const void* x1;
    const float* s1;
    int32_t m1;             // extents of the single tile
    int64_t n1;
    int32_t tiled;
    int32_t cpb;            // columns per block
    int32_t splits;         // column splits per tile
    int64_t rows_total;     // length of a partial row
    int64_t nslots;         // partial rows per output (the second output of MODE 1 follows the first)
};

// (ANY: rows of any extent and alignment, see walk)
template <typename T, int V, int MODE, bool ANY = false>
__global__ void __launch_bounds__(256) rowsum_stage1(RowsumGeom g, float* part) {
    __shared__ float red[2][4][64 * V];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int tile = blockIdx.z;
    int ext0, row0;
    int64_t ncol, slot;
    const T* y;
    const T* x = nullptr;
    const float* st = nullptr;
    if (g.tiled) {
        int tc[kMaxDim], ext[kMaxDim];
        tile_geometry(g.y, tile, tc, ext);
        ext0 = ext[0];
        ncol = (int64_t)ext[1] * ext[2] * ext[3];
        row0 = tc[0] * g.y.base[0];
        y = global_as<const T>(g.ytab[tile]);
        const int rest = tile / g.y.grid[0];
        if (MODE == 1) {
            x = global_as<const T>(g.xtab[tile]);
            st = global_as<const float>(g.stab[rest]);
        }
        slot = (int64_t)rest * g.splits + blockIdx.y;
    } else {
        ext0 = g.m1;
        ncol = g.n1;
        row0 = 0;
        y = static_cast<const T*>(g.y1);
        if (MODE == 1) { x = static_cast<const T*>(g.x1); st = g.s1; }
        slot = blockIdx.y;
    }
    const int e0 = (blockIdx.x * 64 + lane) * V, e = ANY ? max(min(e0, ext0 - V), 0) : e0;
    const Own own{e0 - e, min(V, ext0 - e)};
    const int64_t c0 = (int64_t)blockIdx.y * g.cpb;
    const int64_t c1 = min(ncol, c0 + g.cpb);
    float a0[V], a1[V];
#pragma unroll
    for (int k = 0; k < V; k++) a0[k] = a1[k] = 0.f;
    if (y && e0 < ext0) {
        // four columns per trip so that four loads per operand are in flight
        for (int64_t cb = c0 + wave; cb < c1; cb += 16) {
            float d[4][V], f[4][V];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int64_t c = cb + 4 * u;
                if (c < c1) {
                    ldn<ANY, V>(y + c * ext0 + e, ext0, d[u]);
                    if (MODE == 1) ldn<ANY, V>(x + c * ext0 + e, ext0, f[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int64_t c = cb + 4 * u;
                if (c < c1) {
                    if (MODE == 1) {
                        const float mean = st[2 * c], rstd = st[2 * c + 1];
#pragma unroll
                        for (int k = 0; k < V; k++) { a0[k] += d[u][k] * ((f[u][k] - mean) * rstd); a1[k] += d[u][k]; }
                    } else {
#pragma unroll
                        for (int k = 0; k < V; k++) a0[k] += d[u][k];
                    }
                }
            }
        }
    }
#pragma unroll
    for (int k = 0; k < V; k++) {
        red[0][wave][lane * V + k] = a0[k];
        if (MODE == 1) red[1][wave][lane * V + k] = a1[k];
    }
    __syncthreads();
    if (wave == 0 && e0 < ext0) {
#pragma unroll
        for (int k = 0; k < V; k++) {
            if (ANY && !own(k)) continue;
            const int i = lane * V + k;
            part[slot * g.rows_total + row0 + e + k] = red[0][0][i] + red[0][1][i] + red[0][2][i] + red[0][3][i];
            if (MODE == 1)
                part[(slot + g.nslots) * g.rows_total + row0 + e + k] =
                    red[1][0][i] + red[1][1][i] + red[1][2][i] + red[1][3][i];
        }
    }
}

// out[r] = (accumulate ? out[r] : 0) + sum_s part[s][r]; the output is a 1-axis tiled tensor or a plain vector.
constexpr int kStage2Rows = 16;

// gridDim.y = 2 reduces a second set of partial rows (right behind the first) into (otab_b, ob)
__global__ void __launch_bounds__(256) rowsum_stage2(const float* part, int64_t nslots, int64_t rows_total,
                                                      void* const* otab, float* o1, int base0, int accumulate,
                                                      void* const* otab_b, float* ob) {
    if (blockIdx.y) {
        part += nslots * rows_total;
        otab = otab_b;
        o1 = ob;
    }
    // 16 rows per block (64-byte runs of a partial row); 16 groups of lanes take every sixteenth partial
    // row, four loads in flight each, then combine through LDS in a fixed order.  The grid is small
    // (rows / 16 blocks), so the kernel is bound by the latency of its load chain: many short chains.
    __shared__ float red[16][17];
    const int rl = threadIdx.x & 15, kg = threadIdx.x >> 4;
    const int64_t r = (int64_t)blockIdx.x * kStage2Rows + rl;
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
    if (r < rows_total) {
        int64_t k = kg;
        for (; k + 48 < nslots; k += 64) {
            s0 += part[k * rows_total + r];
            s1 += part[(k + 16) * rows_total + r];
            s2 += part[(k + 32) * rows_total + r];
            s3 += part[(k + 48) * rows_total + r];
        }
        for (; k < nslots; k += 16) s0 += part[k * rows_total + r];
    }
    red[kg][rl] = (s0 + s1) + (s2 + s3);
    __syncthreads();
    if (kg == 0 && r < rows_total) {
        float s = 0.f;
#pragma unroll
        for (int q = 0; q < 16; q++) s += red[q][rl];
        float* o = otab ? global_as<float>(otab[r / base0]) + (r % base0) : o1 + r;
        *o = accumulate ? *o + s : s;
    }
}

// The whole sum of up to 1024 columns in one or two tiles per row of tiles in one launch: a block owns four vectors of rows, its 256 groups of four
// lanes take the columns in turn and meet in shuffles and LDS.  Latency is all such a call consists of, so the second launch costs
// as much as the first; the tiles come one after the other, each a latency of its own.
constexpr int kSmallThreads = 1024;
template <typename T, int V, bool ANY>
__global__ void __launch_bounds__(kSmallThreads) rowsum_small(TiledView y, void* const* otab) {
    __shared__ float red[kSmallThreads / 64][4][V];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, rv = threadIdx.x & 3, cg = threadIdx.x >> 2;
    constexpr int kGroups = kSmallThreads / 4;
    const int l = blockIdx.y, ext0 = min(y.base[0], y.shape[0] - l * y.base[0]);
    const int e0 = (blockIdx.x * 4 + rv) * V, e = ANY ? max(min(e0, ext0 - V), 0) : e0;
    float a[V];
#pragma unroll
    for (int k = 0; k < V; k++) a[k] = 0.f;
    const int rest_tiles = y.grid[1] * y.grid[2] * y.grid[3];
    for (int rest = 0; rest < rest_tiles; rest++) {
        int tc[kMaxDim], ext[kMaxDim];
        tile_geometry(y, l + y.grid[0] * rest, tc, ext);
        const int ncol = ext[1] * ext[2] * ext[3];
        const T* p = global_as<const T>(y.tiles[l + y.grid[0] * rest]);
        if (e0 >= ext0) continue;
        // four columns per trip, which 1024 of them fill, so that four loads are in flight
        for (int c = cg; c < ncol; c += 4 * kGroups) {
            float d[4][V];
#pragma unroll
            for (int u = 0; u < 4; u++)
                if (c + u * kGroups < ncol) ldn<ANY, V>(p + (int64_t)(c + u * kGroups) * ext0 + e, ext0, d[u]);
#pragma unroll
            for (int u = 0; u < 4; u++)
                if (c + u * kGroups < ncol) {
#pragma unroll
                    for (int k = 0; k < V; k++) a[k] += d[u][k];
                }
        }
    }
#pragma unroll
    for (int k = 0; k < V; k++) {
#pragma unroll
        for (int o = 32; o >= 4; o >>= 1) a[k] += __shfl_xor(a[k], o, 64);
        if (lane < 4) red[wave][lane][k] = a[k];
    }
    __syncthreads();
    if (threadIdx.x < 4 * V) {
        const int r = threadIdx.x / V, k = threadIdx.x % V, first = (blockIdx.x * 4 + r) * V, at = ANY ? max(min(first, ext0 - V), 0) : first;
        const int row = at + k;
        if (first < ext0 && row >= first && row < ext0) {
            float s = 0.f;
#pragma unroll
            for (int q = 0; q < kSmallThreads / 64; q++) s += red[q][r][k];
            global_as<float>(otab[l])[row] = s;
        }
    }
}

// The same for rows in fours: 64 rows per block, 16-byte loads, eight in flight (256 partial rows of 8192, twice: 11.6 -> 4.9 us).
__global__ void __launch_bounds__(256) rowsum_stage2_vec(const float* part, int64_t nslots, int64_t rows_total, void* const* otab, int base0, void* const* otab_b) {
    if (blockIdx.y) {
        part += nslots * rows_total;
        otab = otab_b;
    }
    __shared__ float4 red[16][17];
    const int rl = threadIdx.x & 15, kg = threadIdx.x >> 4;
    const int64_t r = ((int64_t)blockIdx.x * 16 + rl) * 4;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (r < rows_total)
        for (int64_t k = kg; k < nslots; k += 128) {
            float4 x[8];
#pragma unroll
            for (int u = 0; u < 8; u++) x[u] = k + 16 * u < nslots ? *reinterpret_cast<const float4*>(part + (k + 16 * u) * rows_total + r) : make_float4(0.f, 0.f, 0.f, 0.f);
            // (in pairs: a chain of all of them would be the longest in the sum)
#pragma unroll
            for (int d = 1; d < 8; d *= 2)
#pragma unroll
                for (int u = 0; u < 8; u += 2 * d) { x[u].x += x[u + d].x; x[u].y += x[u + d].y; x[u].z += x[u + d].z; x[u].w += x[u + d].w; }
            s.x += x[0].x; s.y += x[0].y; s.z += x[0].z; s.w += x[0].w;
        }
    red[kg][rl] = s;
    __syncthreads();
    if (threadIdx.x < 64) {
        const int q = threadIdx.x >> 2, c = threadIdx.x & 3;
        const int64_t row = (int64_t)blockIdx.x * 64 + threadIdx.x;
        if (row < rows_total) {
            float t[16];
#pragma unroll
            for (int g = 0; g < 16; g++) t[g] = reinterpret_cast<const float*>(&red[g][q])[c];
#pragma unroll
            for (int d = 1; d < 16; d *= 2)
#pragma unroll
                for (int g = 0; g < 16; g += 2 * d) t[g] += t[g + d];
            global_as<float>(otab[row / base0])[row % base0] = t[0];
        }
    }
}

// partial rows to one or two tiled vectors
int32_t launch_stage2(hipStream_t st, const float* part, int64_t nslots, int64_t rows, void* const* o0, void* const* o1, int base0) {
    const unsigned outs = o1 ? 2 : 1;
    if (rows % 4 == 0) hipLaunchKernelGGL(rowsum_stage2_vec, dim3((unsigned)((rows + 63) / 64), outs), dim3(256), 0, st, part, nslots, rows, o0, base0, o1);
    else hipLaunchKernelGGL(rowsum_stage2, dim3((unsigned)((rows + kStage2Rows - 1) / kStage2Rows), outs), dim3(256), 0, st, part, nslots, rows, o0, nullptr, base0, 0, o1, nullptr);
    return hipGetLastError() == hipSuccess ? NNT_OK : NNT_EHIP;
}

constexpr int kColsPerBlock = 128;

int64_t scratch_elems(int64_t m, int64_t n, int mode) { return ((n + kColsPerBlock - 1) / kColsPerBlock) * m * (mode ? 2 : 1); }

// How the first stage reads: whole vectors, vectors at any alignment, or single elements.  On odd extents vectors are the faster form on tiles of more than 64
// rows (fp32 1031 x 4000 on tiles of 129 12.4 -> 9.9 us, 8007 x 8000 61 -> 50), in bf16 from two million elements on (1607 x 4000 on tiles of 201 16.4 -> 11.3, 8007 x
// 8000 57 -> 29).  Tiles of up to 64 rows are one step of a wavefront either way (fp32 295 x 4000 on tiles of 37 8.8 and 9.8, bf16 9.8 and 11.2), and a small bf16 launch
// waits for its few vectors longer than for single elements (201 x 1200 7.5 and 8.8, 1001 x 1200 8.1 and 8.8).
enum SumForm { kSumVec, kSumAny, kSumScalar };
inline SumForm sum_form(bool vec, bool bf16, int64_t ext, int64_t rows, int64_t ncols) {
    return vec ? kSumVec : ext > 64 && (!bf16 || rows * ncols >= 2000000) ? kSumAny : kSumScalar;
}
// (ext: rows of the largest tile)
template <typename T, int MODE>
int32_t launch_rowsum_t(hipStream_t st, const RowsumGeom& g, int64_t ext, int64_t ntiles, SumForm form, float* part) {
    constexpr int V = VecOf<T>::V;
    const int per = 64 * (form == kSumScalar ? 1 : V);
    const dim3 grid((unsigned)((ext + per - 1) / per), g.splits, (unsigned)ntiles), block(256);
    if (form == kSumVec) hipLaunchKernelGGL((rowsum_stage1<T, V, MODE>), grid, block, 0, st, g, part);
    else if (form == kSumAny) hipLaunchKernelGGL((rowsum_stage1<T, V, MODE, true>), grid, block, 0, st, g, part);
    else hipLaunchKernelGGL((rowsum_stage1<T, 1, MODE>), grid, block, 0, st, g, part);
    return hipGetLastError() == hipSuccess ? NNT_OK : NNT_EHIP;
}

// single tile: dY (m x n) -> out0 (and out1 in MODE 1)
int32_t rowsum_single(hipStream_t st, int dtype, int mode, int64_t m, int64_t n, const void* dy, const void* x,
                      const float* stats, float* out0, float* out1, int accumulate, float* scratch) {
    if (m == 0) return NNT_OK;
    RowsumGeom g = {};
    g.tiled = 0;
    g.y1 = dy; g.x1 = x; g.s1 = stats;
    g.m1 = (int32_t)m; g.n1 = n;
    g.cpb = kColsPerBlock;
    g.splits = (int32_t)std::max<int64_t>(1, (n + kColsPerBlock - 1) / kColsPerBlock);
    g.rows_total = m;
    g.nslots = g.splits;
    const int V = dtype == NNT_F32 ? 4 : 8;
    const SumForm form = sum_form(m % V == 0 && aligned16(dy) && (!x || aligned16(x)), dtype == NNT_BF16, m, m, n);
    int32_t rc;
    if (dtype == NNT_F32) rc = mode ? launch_rowsum_t<float, 1>(st, g, m, 1, form, scratch) : launch_rowsum_t<float, 0>(st, g, m, 1, form, scratch);
    else rc = mode ? launch_rowsum_t<bf16_t, 1>(st, g, m, 1, form, scratch) : launch_rowsum_t<bf16_t, 0>(st, g, m, 1, form, scratch);
    if (rc != NNT_OK) return rc;
    const unsigned blocks = (unsigned)((m + kStage2Rows - 1) / kStage2Rows);
    hipLaunchKernelGGL(rowsum_stage2, dim3(blocks, mode ? 2 : 1), dim3(256), 0, st, scratch, (int64_t)g.splits, m, nullptr, out0, 1,
                       accumulate, nullptr, out1);
    return hipGetLastError() == hipSuccess ? NNT_OK : NNT_EHIP;
}

// Columns per block, column splits per tile and partial rows of the two-stage sums over a tensor: fewer columns per block when the tensor would
// otherwise give the chip too few blocks.
struct RowsumSplit { int32_t cpb, splits; int64_t nslots; };
RowsumSplit split_of(const nnt_tensor* dY) {
    int64_t max_cols = 1, rest_tiles = 1;
    for (int a = 1; a < dY->ndim; a++) { max_cols *= dY->base[a]; rest_tiles *= dY->grid[a]; }
    const int V = dY->dtype == NNT_F32 ? 4 : 8;
    const int64_t row_blocks = (dY->base[0] + 64 * V - 1) / (64 * V);
    int cpb = kColsPerBlock;
    while (cpb > 32 && row_blocks * ((max_cols + cpb - 1) / cpb) * dY->ntiles < 1024) cpb /= 2;
    const int32_t splits = (int32_t)((max_cols + cpb - 1) / cpb);
    return RowsumSplit{cpb, splits, rest_tiles * splits};
}

// The scratch that the two-stage sums would take, also where a form without it runs: a later call inside a capture, where nothing can
// be allocated, may need it ("run the operation once first" holds for any call of the operation that is no larger).
int32_t keep_rowsum_scratch(nnt_ctx* ctx, int mode, const nnt_tensor* dY) {
    if (ctx->capturing) return NNT_OK;
    return ensure_scratch(ctx, split_of(dY).nslots * dY->shape[0] * (mode ? 2 : 1));
}

// whole tiled tensor dY [rows, ...] -> out0 / out1: 1-axis tensors tiled like dY's first axis
int32_t rowsum_tensor(nnt_ctx* ctx, int mode, nnt_tensor* dY, nnt_tensor* X, nnt_tensor* S, nnt_tensor* out0, nnt_tensor* out1) {
    const int V = dY->dtype == NNT_F32 ? 4 : 8;
    bool vec = dY->base[0] % V == 0 && dY->shape[0] % V == 0;
    for (void* p : dY->tiles) vec = vec && aligned16(p);
    if (X) for (void* p : X->tiles) vec = vec && aligned16(p);
    // in one launch up to 1024 columns, 13 MB and two tiles along the columns: 4.3 to 6 us where the two launches take 6.5 to 8.1 (fp32 256 x 64: 4.3, 6.8;
    // 768 x 1024: 5.0, 7.4; 3072 x 1024 in two tiles 5.6, 7.7); beyond, its few blocks take longer (fp32 768 x 2048: 7.5, 6.7;
    // 8192 x 512: 9.2, 7.2), and every tile costs another latency: four tiles 6.7 to 9.5 (256 columns 6.9, 7.0; 1024 8.4, 7.4), sixteen 13.7, 7.1, sixty-four 43, 7.3
    const int64_t ncols = n_columns(dY);
    if (mode == 0 && ncols <= 1024 && ncols * dY->shape[0] * dY->elem_size() <= 13000000 && dY->ntiles <= std::min<int64_t>(2 * dY->grid[0], 65535)) {
        const int32_t kept = keep_rowsum_scratch(ctx, mode, dY);
        if (kept != NNT_OK) return kept;
        const TiledView vy = dY->view();
        void* const* ot = out0->d_tiles;
        const int dt = dY->dtype;
        const dim3 grid((unsigned)((dY->base[0] + 4 * V - 1) / (4 * V)), (unsigned)dY->grid[0]);
        return submit(ctx, {dY->all(kRead), out0->all(kWrite)}, [=](hipStream_t st) {
            if (dt == NNT_F32) {
                if (vec) hipLaunchKernelGGL((rowsum_small<float, 4, false>), grid, dim3(kSmallThreads), 0, st, vy, ot);
                else hipLaunchKernelGGL((rowsum_small<float, 4, true>), grid, dim3(kSmallThreads), 0, st, vy, ot);
            } else {
                if (vec) hipLaunchKernelGGL((rowsum_small<bf16_t, 8, false>), grid, dim3(kSmallThreads), 0, st, vy, ot);
                else hipLaunchKernelGGL((rowsum_small<bf16_t, 8, true>), grid, dim3(kSmallThreads), 0, st, vy, ot);
            }
            return hipGetLastError() == hipSuccess ? (int32_t)NNT_OK : (int32_t)NNT_EHIP;
        });
    }
    RowsumGeom g = {};
    g.tiled = 1;
    g.y = dY->view();
    g.ytab = dY->d_tiles;
    g.xtab = X ? X->d_tiles : nullptr;
    g.stab = S ? S->d_tiles : nullptr;
    const RowsumSplit cut = split_of(dY);
    g.cpb = cut.cpb;
    g.splits = cut.splits;
    g.rows_total = dY->shape[0];
    const int64_t nslots = cut.nslots;
    g.nslots = nslots;
    int32_t rc = ensure_scratch(ctx, nslots * g.rows_total * (mode ? 2 : 1));
    if (rc != NNT_OK) return rc;
    if (dY->ntiles > 65535 || g.splits > 65535) return fail(ctx, NNT_EINVAL, "column sum: too many tiles");
    const int64_t ext = dY->base[0];
    const SumForm form = sum_form(vec, dY->dtype == NNT_BF16, ext, dY->shape[0], ncols);
    float* scratch = ctx->red_scratch;
    const int dtype = dY->dtype;
    const int64_t ntiles = dY->ntiles, rows = g.rows_total;
    void* const* o0 = out0->d_tiles;
    void* const* o1 = out1 ? out1->d_tiles : nullptr;
    const int base0 = (int)out0->base[0];
    // (the shared scratch, not the stream's own part: column sums of large tensors side by side with the products of two streams cost
    // the fp32 block 3690 -> 3770 us and a model of four blocks 9170 -> 9340)
    std::vector<Access> acc = {dY->all(kRead), out0->all(kWrite), Access{&ctx->red_dep, 1, kReadWrite}};
    if (X) acc.push_back(X->all(kRead));
    if (S) acc.push_back(S->all(kRead));
    if (out1) acc.push_back(out1->all(kWrite));
    return submit(ctx, acc, [=](hipStream_t st) {
        int32_t r;
        if (dtype == NNT_F32) r = mode ? launch_rowsum_t<float, 1>(st, g, ext, ntiles, form, scratch) : launch_rowsum_t<float, 0>(st, g, ext, ntiles, form, scratch);
        else r = mode ? launch_rowsum_t<bf16_t, 1>(st, g, ext, ntiles, form, scratch) : launch_rowsum_t<bf16_t, 0>(st, g, ext, ntiles, form, scratch);
        if (r != NNT_OK) return r;
        return launch_stage2(st, scratch, nslots, rows, o0, mode ? o1 : nullptr, base0);
    }, 2);
}

bool tensors_vec_ok(std::initializer_list<const nnt_tensor*> ts, int V) {
    for (const nnt_tensor* t : ts) {
        if (!t) continue;
        if (t->base[0] % V != 0 || t->shape[0] % V != 0) return false;
        for (void* p : t->tiles)
            if (p && !aligned16(p)) return false;
    }
    return true;
}

// Whether vectors may be read and written at the tiles' own alignment: every tile begins at an element.
bool any_vec(std::initializer_list<const nnt_tensor*> ts) {
    for (const nnt_tensor* t : ts)
        if (t)
            for (void* p : t->tiles)
                if ((uintptr_t)p % (uintptr_t)t->elem_size() != 0) return false;
    return true;
}

// Tokens of more vectors per lane than this are shared by the four wavefronts of a workgroup (measured: shorter
// tokens lose to the two workgroup barriers, longer ones gain from four times the loads in flight).
constexpr int kLnShareAbove = 4;

template <typename T>
int32_t launch_ln_fwd(hipStream_t st, bool vec, bool any, int nv_needed, const TiledView& X, const TiledView& Y, const TiledView& S,
                      const TiledView& G, const TiledView& B, float eps, int64_t ncols) {
    constexpr int V = VecOf<T>::V;
    // tokens of more than `kLnShareAbove` vectors per lane are shared by the four wavefronts of a workgroup
    // Odd extents: vectors at any alignment where they save enough of the steps in which 64 lanes take 64 single elements of a tile.  Measured on tiles of 5 to
    // 2003, one to eight per token, 100 to 8000 tokens: with a third of the steps or less 1.0 to 4 times faster in fp32, with a quarter or less in bf16 (1.0 to 5.9); with 2 of 5
    // in fp32 where a token has 16 vectors per lane or more (1.2 to 2.2), with half where it has 32 (3000 on tiles of 75 x 4000 tokens 87 -> 80 us).  Tiles of up to 63
    // take as many steps either way, which single elements do faster (bf16 999 on tiles of 37 x 4000 31 us and 88, 320 on tiles of 50 12 and 20).  With few tokens what counts is
    // that four wavefronts come to share one: more than four vectors per lane up to 1200 tokens (1.0 to 1.5 times), up to 256 where
    // that would be many slots of few elements (bf16 255 on tiles of 51 x 1000 7.7 us and 9.0, 1600 on tiles of 25 41 and 49).
    const int vecs = (X.base[0] + 64 * V - 1) / (64 * V), singles = (X.base[0] + 63) / 64;
    const bool fewer_steps = V == 4 ? singles >= 3 * vecs || (nv_needed >= 16 && 2 * singles >= 5 * vecs) || (nv_needed >= 32 && singles >= 2 * vecs) : singles >= 4 * vecs;
    const bool wide_slots = V == 8 ? nv_needed <= 16 && singles > vecs : nv_needed >= 8 || singles > vecs;
    const bool few_tokens = nv_needed > kLnShareAbove && ncols <= (wide_slots ? 1200 : 256);
    any = any && !vec && nv_needed <= 64 && (fewer_steps || few_tokens);
    const bool shared = (vec || any) && nv_needed > kLnShareAbove;
    const dim3 grid((unsigned)(shared ? ncols : (ncols + 3) / 4)), block(256);
    // (odd extents: vectors at any alignment, the last one of a tile moved back to end there)
    if (any && !shared) hipLaunchKernelGGL((ln_fwd_fused<T, V, kLnShareAbove, 1, true>), grid, block, 0, st, X, Y, S, G, B, eps, ncols);
    else if (any && nv_needed <= 16) hipLaunchKernelGGL((ln_fwd_fused<T, V, 4, 4, true>), grid, block, 0, st, X, Y, S, G, B, eps, ncols);
    else if (any) hipLaunchKernelGGL((ln_fwd_fused<T, V, 16, 4, true>), grid, block, 0, st, X, Y, S, G, B, eps, ncols);
    else if (!vec) hipLaunchKernelGGL((ln_fwd_fused<T, 1, 0>), grid, block, 0, st, X, Y, S, G, B, eps, ncols);
    else if (!shared) hipLaunchKernelGGL((ln_fwd_fused<T, V, kLnShareAbove>), grid, block, 0, st, X, Y, S, G, B, eps, ncols);
    else if (nv_needed <= 16) hipLaunchKernelGGL((ln_fwd_fused<T, V, 4, 4>), grid, block, 0, st, X, Y, S, G, B, eps, ncols);
    else if (nv_needed <= 64) hipLaunchKernelGGL((ln_fwd_fused<T, V, 16, 4>), grid, block, 0, st, X, Y, S, G, B, eps, ncols);
    else hipLaunchKernelGGL((ln_fwd_fused<T, V, 0, 4>), grid, block, 0, st, X, Y, S, G, B, eps, ncols);
    return hipGetLastError() == hipSuccess ? NNT_OK : NNT_EHIP;
}

template <typename T>
int32_t launch_ln_bwd(hipStream_t st, bool vec, int nv_needed, const TiledView& X, const TiledView& S, const TiledView& G,
                      const TiledView& dY, const TiledView& dR, const TiledView& dX, int has_res, int64_t ncols) {
    constexpr int V = VecOf<T>::V;
    // (what ln_bwd_onepass does not take: tokens of more than `kLnShareAbove` vectors per lane are shared by the four wavefronts of a workgroup)
    const dim3 quarter((unsigned)((ncols + 3) / 4)), block(256);
    if (!vec) hipLaunchKernelGGL((ln_bwd_fused<T, 1, 0>), quarter, block, 0, st, X, S, G, dY, dR, dX, has_res, ncols);
    else if (nv_needed <= kLnShareAbove) hipLaunchKernelGGL((ln_bwd_fused<T, V, 4>), quarter, block, 0, st, X, S, G, dY, dR, dX, has_res, ncols);
    else if (nv_needed <= 16) hipLaunchKernelGGL((ln_bwd_fused<T, V, 4, 4>), dim3((unsigned)ncols), block, 0, st, X, S, G, dY, dR, dX, has_res, ncols);
    else if (nv_needed <= 32) hipLaunchKernelGGL((ln_bwd_fused<T, V, 8, 4>), dim3((unsigned)ncols), block, 0, st, X, S, G, dY, dR, dX, has_res, ncols);
    else hipLaunchKernelGGL((ln_bwd_fused<T, V, 0, 4>), dim3((unsigned)ncols), block, 0, st, X, S, G, dY, dR, dX, has_res, ncols);
    return hipGetLastError() == hipSuccess ? NNT_OK : NNT_EHIP;
}

// ------------------------------------------------------------------ layer norm backward, all in one pass
// The input gradient and the partial gain / bias gradients from one read of x and dy.  As two kernels (ln_bwd_fused behind
// the column sums) the adjoint reads x and dy twice; its bytes and, for few tokens, its launches are what bounds it.  A workgroup is
// eight waves: WPT of them share a token, the 8 / WPT groups take tokens in turn, and every lane keeps its two sums
// in registers while the vectors of the next token are on their way (all loads of a token in one piece and in every round, tile pointers through
// the scalar memory: pointers out of the vector memory, whose loads come back in order, waited for the next token's data and for the last one's
// stores, three to four memory latencies per token: 2664 x 8168 in fp32 on tiles of 512 129 us, 86 now; 768 x 8192 34 -> 26, bf16 4096 x 8192 75 -> 57).
// At the end the groups' sums meet in LDS and the workgroup leaves one partial row per gradient (at most
// 256 rows, which rowsum_stage2 adds in a fixed order).  Against the two passes, which in a captured graph run side by side on two streams,
// adjoints back to back: fp32 1024 x 8192 37 -> 35 us, 4096 x 8192 140 -> 122, 8192 x 8192 326 -> 235, odd extents (vectors at any alignment instead of single
// elements) 777 x 2664 27 -> 24, 1370 x 1672 35 -> 22; slower where less than half of the lanes have a vector or the longest tokens are few (bf16 768 x 8192
// on tiles of 256 25 -> 27, 8192 x 4096 72 -> 77, fp32 5840 x 387 22 -> 28).  Called one by one, forward and backward, all of these are faster:
// 49 -> 36, 126 -> 104, 49 -> 36; 75 sizes between 128 x 128 and 8192 x 8192: 1.26 times in graphs, 1.56 by calls.
template <typename T, int V> struct RawVec;
template <> struct RawVec<float, 4> { using R = float4; };
template <> struct RawVec<bf16_t, 8> { using R = uint4; };
__device__ __forceinline__ void unpack(const float4& r, float (&f)[4]) { f[0] = r.x; f[1] = r.y; f[2] = r.z; f[3] = r.w; }
__device__ __forceinline__ void unpack(const uint4& r, float (&f)[8]) {
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int i = 0; i < 4; i++) { f[2 * i] = __uint_as_float(w[i] << 16); f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u); }
}

// the compiler takes the value as changed here
__device__ __forceinline__ void keep(float4& r) { asm volatile("" : "+v"(r.x), "+v"(r.y), "+v"(r.z), "+v"(r.w)); }
__device__ __forceinline__ void keep(uint4& r) { asm volatile("" : "+v"(r.x), "+v"(r.y), "+v"(r.z), "+v"(r.w)); }

// the value, or zeros
__device__ __forceinline__ void only_if(bool c, float4& r) { if (!c) r = make_float4(0.f, 0.f, 0.f, 0.f); }
__device__ __forceinline__ void only_if(bool c, uint4& r) { if (!c) r = make_uint4(0u, 0u, 0u, 0u); }

// a vector as it lies in memory
template <bool ANY, typename T, typename R> __device__ __forceinline__ void raw(const T* p, int n, R& r) {
    constexpr int V = (int)(sizeof(R) / sizeof(T));
    if constexpr (!ANY) {
        r = *reinterpret_cast<const R*>(p);
    } else {
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        if (n >= V) {
            if constexpr (V == 4) {
                const f4_any x = *reinterpret_cast<const f4_any*>(p);
                for (int i = 0; i < 4; i++) w[i] = __float_as_uint(x[i]);
            } else {
                const u4_any x = *reinterpret_cast<const u4_any*>(p);
                for (int i = 0; i < 4; i++) w[i] = x[i];
            }
        } else {
#pragma unroll
            for (int i = 0; i < V; i++)
                if (i < n) {
                    if constexpr (V == 4) w[i] = __float_as_uint(p[i]);
                    else w[i / 2] |= (uint32_t)p[i] << (16 * (i & 1));
                }
        }
        if constexpr (V == 4) r = make_float4(__uint_as_float(w[0]), __uint_as_float(w[1]), __uint_as_float(w[2]), __uint_as_float(w[3]));
        else r = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// Entry `i` (wave-uniform) of a table of tile pointers.  Tables do not change while a kernel runs, but behind a store the compiler does not
// know that and would fetch the entry through the vector memory, whose loads come back in order.
template <typename T> __device__ __forceinline__ T* table_entry(void* const* tab, int i) {
    return in_global((T*)(uintptr_t)((const __attribute__((address_space(4))) uint64_t*)(uintptr_t)tab)[i]);
}

constexpr int kOnepassWaves = 8;
// Tokens of a group between two moves of its gradient sums to the partial rows (even).  The sums of one chain over all its tokens would be less
// exact than the column sums' with their chains of 32 (256 tokens, 4096 x 65536: 3.1e-7 instead of 1.4e-7 in the 2-norm; 32 tokens, 4096 x 8192: the same
// 1.4e-7 once the partial rows are added in pairs, 1.5e-7 before).
constexpr unsigned kSumRounds = 32;
constexpr int kOnepassGroups = 256;      // workgroups at most: one per compute unit, which is what the registers allow

template <typename T, int V, int NV, int WPT, bool RES, bool ANY>
__global__ void __launch_bounds__(64 * kOnepassWaves, 2) ln_bwd_onepass(TiledView X, TiledView S, TiledView G, TiledView dY, TiledView dR,
                                                                     TiledView dX, unsigned ncols, unsigned rounds, float* part) {
    using R = typename RawVec<T, V>::R;
    constexpr int GR = kOnepassWaves / WPT, kWave = 64 * NV * V;
    __shared__ float2 red[2][kOnepassWaves];
    __shared__ float sums[kOnepassWaves * kWave];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = wave / WPT, w = wave % WPT;
    const int g0 = X.grid[0], vpt = (X.base[0] + 64 * V - 1) / (64 * V);
    // this wave's vectors of a token: the same for all tokens
    int l[NV], ext[NV];
    unsigned e[NV];
    bool ok[NV];
    Own own[NV];          // (ANY: see walk)
    float ag[NV][V], ab[NV][V];
    // the gain lies in LDS (read twice per token, and again after a move of the sums): registers are what the kernel is short of
    float* const gam = sums + w * kWave + lane * V;
#pragma unroll
    for (int it = 0; it < NV; it++) {
        const int s = w + WPT * it, ll = s / vpt;
        l[it] = min(ll, g0 - 1);
        ext[it] = ext0_of(X, l[it]);
        e[it] = (unsigned)(((s - ll * vpt) * 64 + lane) * V);
        ok[it] = ll < g0 && (int)e[it] < ext[it];
        if constexpr (ANY) {
            const int at = max(min((int)e[it], ext[it] - V), 0);
            own[it] = Own{(int)e[it] - at, min(V, ext[it] - at)};
            if (ok[it]) e[it] = (unsigned)at;
        }
        if (!ok[it]) e[it] = 0;
#pragma unroll
        for (int k = 0; k < V; k++) ag[it][k] = ab[it][k] = 0.f;
    }
    auto load_gain = [&]() {
        if (grp != 0) return;
        float gm[NV][V];
#pragma unroll
        for (int it = 0; it < NV; it++) ldn<ANY, V>(table_entry<const float>(G.tiles, l[it]) + e[it], ext[it], gm[it]);
#pragma unroll
        for (int it = 0; it < NV; it++)
#pragma unroll
            for (int k = 0; k < V; k++) gam[it * 64 * V + k] = ok[it] ? gm[it][k] : 0.f;
    };
    struct Token {
        R x[NV], d[NV], q[RES ? NV : 1];
        float mean, rstd;
        T* o[NV];
        bool real;
    };
    // (lanes without a vector fetch their tile's first, groups without a token the last one: loads behind a condition would be waited for
    // where the ways meet)
    auto fetch = [&](unsigned col, Token& t) {
        t.real = col < ncols;
        const Column c = column_of(X, min(col, ncols - 1));
        const float* st = table_entry<const float>(S.tiles, c.stat_tile) + 2 * (int64_t)c.colidx;
        t.mean = st[0];
        t.rstd = st[1];
#pragma unroll
        for (int it = 0; it < NV; it++) {
            const int64_t at = (int64_t)c.colidx * ext[it];
            t.o[it] = table_entry<T>(dX.tiles, c.tile0 + l[it]) + at;
            raw<ANY>(table_entry<const T>(X.tiles, c.tile0 + l[it]) + at + e[it], ext[it], t.x[it]);
            raw<ANY>(table_entry<const T>(dY.tiles, c.tile0 + l[it]) + at + e[it], ext[it], t.d[it]);
            if constexpr (RES) raw<ANY>(table_entry<const T>(dR.tiles, c.tile0 + l[it]) + at + e[it], ext[it], t.q[it]);
        }
    };
    // (the same number of rounds for every group: the waves of a workgroup meet once per token)
    const unsigned step = gridDim.x * GR, col0 = blockIdx.x * GR + grp;
    auto work_on = [&](Token& t, unsigned r) {
        const float mean = t.real ? t.mean : 0.f, rstd = t.real ? t.rstd : 0.f;
        float a = 0.f, b = 0.f;
#pragma unroll
        for (int it = 0; it < NV; it++) {
            float x[V], d[V], gm[V];
            only_if(t.real && ok[it], t.x[it]);
            only_if(t.real && ok[it], t.d[it]);
            unpack(t.x[it], x);
            unpack(t.d[it], d);
            ldv<V>(gam + it * 64 * V, gm);
#pragma unroll
            for (int k = 0; k < V; k++) {
                if constexpr (ANY) d[k] = own[it](k) ? d[k] : 0.f;
                const float gg = d[k] * gm[k], xh = (x[k] - mean) * rstd;
                a += gg;
                b += gg * xh;
                ag[it][k] += d[k] * xh;
                ab[it][k] += d[k];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        a = wave_sum(a);
        b = wave_sum(b);
        if constexpr (WPT > 1) {
            // (dX may be the residual: a vector that was moved back is stored over elements of the neighbour's, which lie in another
            // wave's registers by the time the waves meet.  x and dy do, being summed; the residual is made to)
            if constexpr (RES && ANY) {
#pragma unroll
                for (int it = 0; it < NV; it++) keep(t.q[it]);
            }
            // two buffers: a wave that is a token ahead writes the other one
            if (lane == 0) red[r & 1][wave] = make_float2(a, b);
            __syncthreads();
            a = b = 0.f;
#pragma unroll
            for (int i = 0; i < WPT; i++) {
                a += red[r & 1][grp * WPT + i].x;
                b += red[r & 1][grp * WPT + i].y;
            }
        }
        a /= (float)X.shape[0];
        b /= (float)X.shape[0];
        // (unpacked again below: the unpacked values held over the sums would take another 32 registers)
#pragma unroll
        for (int it = 0; it < NV; it++) { keep(t.x[it]); keep(t.d[it]); }
        if (t.real) {
#pragma unroll
            for (int it = 0; it < NV; it++)
                if (ok[it]) {
                    float x[V], d[V], gm[V], o[V];
                    unpack(t.x[it], x);
                    unpack(t.d[it], d);
                    ldv<V>(gam + it * 64 * V, gm);
#pragma unroll
                    for (int k = 0; k < V; k++) {
                        // (rounded one by one, as where they are kept over the sums)
#pragma clang fp contract(off)
                        const float gg = d[k] * gm[k], xh = (x[k] - mean) * rstd;
                        const float t0 = gg - a;
                        o[k] = rstd * __builtin_fmaf(-xh, b, t0);
                    }
                    if constexpr (RES) {
                        float q[V];
                        unpack(t.q[it], q);
#pragma unroll
                        for (int k = 0; k < V; k++) o[k] += q[k];
                    }
                    stn<ANY, V>(t.o[it] + e[it], ext[it], o);
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
    };
    // the groups' sums since the last time, gain first, added to the workgroup's partial rows; element r of slot `it` of wave w at [it * 64 V + r]
    const int64_t rows = X.shape[0];
    auto leave_sums = [&](bool first) {
#pragma unroll
        for (int which = 0; which < 2; which++) {
            __syncthreads();
#pragma unroll
            for (int it = 0; it < NV; it++)
#pragma unroll
                for (int k = 0; k < V; k++) {
                    float& s = which ? ab[it][k] : ag[it][k];
                    sums[wave * kWave + it * 64 * V + lane * V + k] = s;
                    s = 0.f;
                }
            __syncthreads();
            float* out = part + ((int64_t)which * gridDim.x + blockIdx.x) * rows;
            for (int p = threadIdx.x; p < WPT * kWave; p += 64 * kOnepassWaves) {
                const int ww = p / kWave, q = p - ww * kWave, it = q / (64 * V);
                const int s = ww + WPT * it, ll = s / vpt;
                int el = (s - ll * vpt) * 64 * V + (q - it * 64 * V);
                if (ll >= g0) continue;
                const int ex = ext0_of(X, ll);
                if constexpr (ANY) {      // (where the vector was moved to, and whether the element is its own)
                    const int k = el % V, first_el = el - k, at = max(min(first_el, ex - V), 0);
                    if (first_el >= ex || k < first_el - at || at + k >= ex) continue;
                    el = at + k;
                } else if (el >= ex) {
                    continue;
                }
                float t = 0.f;
#pragma unroll
                for (int gq = 0; gq < GR; gq++) t += sums[gq * WPT * kWave + p];
                float* const dst = out + (int64_t)ll * X.base[0] + el;
                *dst = first ? t : *dst + t;
            }
        }
    };
    // Two tokens in turn, the next one's loads started before the present one's are waited for.  (A fetch only where a token is left would be
    // waited for where the ways meet.)  Four vectors per lane: in fp32 the next token's registers are copied at the end of a round, where they
    // are waited for; in bf16 one set, which leaves the overlap to the eight waves (two sets spill up to 232 registers, copied ones up to 28: 10001 x 2048 92 us
    // instead of 75, 16384 x 2048 90 and 74).
    constexpr bool kTwoSets = NV <= 2;
    auto sums_so_far = [&](bool first) {
        leave_sums(first);
        __syncthreads();
        load_gain();
        __syncthreads();
    };
    Token t0, t1;
    fetch(col0, t0);
    load_gain();
    __syncthreads();
    unsigned r = 0, moved = 0;
    if constexpr (kTwoSets) {
        while (rounds - r > 2) {
            const unsigned end = min(r + kSumRounds, (rounds - 1) & ~1u);
            for (; r < end; r += 2) {
                fetch(col0 + (r + 1) * step, t1);
                work_on(t0, r);
                fetch(col0 + (r + 2) * step, t0);
                work_on(t1, r + 1);
            }
            if (r - moved == kSumRounds) {
                sums_so_far(moved == 0);
                moved = r;
            }
        }
        if (rounds - r == 2) {
            fetch(col0 + (r + 1) * step, t1);
            work_on(t0, r);
            work_on(t1, r + 1);
        } else {
            work_on(t0, r);
        }
    } else {
        for (;;) {
            for (const unsigned end = min(r + kSumRounds, rounds); r < end; r++) {
                if constexpr (sizeof(T) == 2) {
                    work_on(t0, r);
                    if (r + 1 < rounds) fetch(col0 + (r + 1) * step, t0);
                } else {
                    if (r + 1 < rounds) fetch(col0 + (r + 1) * step, t1);
                    work_on(t0, r);
                    t0 = t1;
                }
            }
            if (r >= rounds) break;
            sums_so_far(moved == 0);
            moved = r;
        }
    }
    leave_sums(moved == 0);
}

// Waves that share a token so that each has at most NV vectors of it per lane; 0: too long for the kernel.
template <int NV>
inline int onepass_wpt(int nv_needed) {
    int wpt = 1;
    while (wpt <= kOnepassWaves && wpt * NV < nv_needed) wpt *= 2;
    return wpt <= kOnepassWaves ? wpt : 0;
}
// (two vectors of 16 bytes per lane: up to 206 registers, the next token's included; sixteen waves per workgroup would have to make do with
// 128, and the spilled ones' reloads wait for the next token's loads: 113 us for 8192 x 4096 with the copied registers of then, 77 now)
// Longer tokens (8192 fp32 elements, 16384 in bf16): all eight waves on one with four vectors per lane, up to 256 registers (two passes and one, fp32
// 8192 x 4096 150 and 135 us, bf16 16384 x 2048 82 and 74; odd extents, fp32 7001 x 1000 125 and 43, bf16 10001 x 2048 173 and 75).  Few of them, or
// on narrow tiles, are slower than two passes that run side by side in a graph (bf16 8200 x 300 19 and 33, fp32 2048 x 1000 on tiles of 64 26 and 36), and about as
// fast as calls (41 and 42, 54 and 47).
constexpr int kOnepassVecs = 2, kOnepassLong = 4;
// 4096 bf16 tokens and more of three or four whole vectors per lane stay with one wave and that form: the sums over a token are then added in the order of the
// two passes, and dx is what they leave bit for bit (single flipped roundings of dx travel through the products behind it).  Two waves are the faster form for
// fewer tokens (1664 x 2319 on tiles of 512, forward and backward, 20 us, one wave 23; 4096 and more: 1600 x 8192 on tiles of 400 32 either way, 768 x 8192 29 and 27, 2048 x 8192 on tiles of
// 512 38 and 42), in fp32, where the last digit is all that changes (1024 x 8192 32 us, one wave 35), and on odd extents, which the two passes take element by element
// (bf16 1120 x 128 on tiles of 300 13 and 17).
inline int onepass_waves(bool bf16_vec, int nv_needed, int64_t ncols) {
    if (bf16_vec && nv_needed > kOnepassVecs && nv_needed <= kOnepassLong && ncols >= 4096) return 1;
    const int w = onepass_wpt<kOnepassVecs>(nv_needed);
    return w ? w : onepass_wpt<kOnepassLong>(nv_needed);
}
inline int64_t onepass_wgs(int wpt, int64_t ncols) { const int64_t gr = kOnepassWaves / wpt; return std::min<int64_t>(kOnepassGroups, (ncols + gr - 1) / gr); }

template <typename T, int NV, int WPT>
int32_t launch_onepass_w(hipStream_t st, bool vec, const TiledView& X, const TiledView& S, const TiledView& G, const TiledView& dY,
                         const TiledView& dR, const TiledView& dX, int has_res, int64_t ncols, float* part) {
    constexpr int V = VecOf<T>::V;
    constexpr bool kAny = !(NV == kOnepassLong && WPT == 1);       // (whole vectors only: see onepass_waves)
    const int64_t wgs = onepass_wgs(WPT, ncols), per = wgs * (kOnepassWaves / WPT);
    const unsigned n = (unsigned)ncols, rounds = (unsigned)((ncols + per - 1) / per);
    const dim3 grid((unsigned)wgs), block(64 * kOnepassWaves);
    if (!vec && !kAny) return NNT_EINVAL;
    if (vec && has_res) hipLaunchKernelGGL((ln_bwd_onepass<T, V, NV, WPT, true, false>), grid, block, 0, st, X, S, G, dY, dR, dX, n, rounds, part);
    else if (vec) hipLaunchKernelGGL((ln_bwd_onepass<T, V, NV, WPT, false, false>), grid, block, 0, st, X, S, G, dY, dR, dX, n, rounds, part);
    if constexpr (kAny) {
        if (!vec && has_res) hipLaunchKernelGGL((ln_bwd_onepass<T, V, NV, WPT, true, true>), grid, block, 0, st, X, S, G, dY, dR, dX, n, rounds, part);
        else if (!vec) hipLaunchKernelGGL((ln_bwd_onepass<T, V, NV, WPT, false, true>), grid, block, 0, st, X, S, G, dY, dR, dX, n, rounds, part);
    }
    return hipGetLastError() == hipSuccess ? NNT_OK : NNT_EHIP;
}
template <typename T>
int32_t launch_onepass(hipStream_t st, bool vec, int wpt, int nv_needed, const TiledView& X, const TiledView& S, const TiledView& G, const TiledView& dY,
                       const TiledView& dR, const TiledView& dX, int has_res, int64_t ncols, float* part) {
    if (wpt * kOnepassVecs < nv_needed) {
        if (wpt == kOnepassWaves) return launch_onepass_w<T, kOnepassLong, kOnepassWaves>(st, vec, X, S, G, dY, dR, dX, has_res, ncols, part);
        if constexpr (sizeof(T) == 2)
            if (wpt == 1) return launch_onepass_w<T, kOnepassLong, 1>(st, vec, X, S, G, dY, dR, dX, has_res, ncols, part);
        return NNT_EINVAL;
    }
    switch (wpt) {
        case 1: return launch_onepass_w<T, kOnepassVecs, 1>(st, vec, X, S, G, dY, dR, dX, has_res, ncols, part);
        case 2: return launch_onepass_w<T, kOnepassVecs, 2>(st, vec, X, S, G, dY, dR, dX, has_res, ncols, part);
        case 4: return launch_onepass_w<T, kOnepassVecs, 4>(st, vec, X, S, G, dY, dR, dX, has_res, ncols, part);
        case 8: return launch_onepass_w<T, kOnepassVecs, 8>(st, vec, X, S, G, dY, dR, dX, has_res, ncols, part);
        default: return NNT_EINVAL;
    }
}

int32_t check_ln_shapes(nnt_ctx* ctx, const nnt_tensor* X, const nnt_tensor* gamma, const nnt_tensor* stats, const char* who) {
    if (X->ndim < 2) return fail(ctx, NNT_EINVAL, std::string(who) + ": X needs at least 2 axes");
    if (gamma->dtype != NNT_F32 || gamma->ndim != 1 || gamma->shape[0] != X->shape[0] || gamma->base[0] != X->base[0])
        return fail(ctx, NNT_EINVAL, std::string(who) + ": gain / bias must be fp32 vectors tiled like X's first axis");
    if (stats->dtype != NNT_F32 || stats->ndim != X->ndim || stats->shape[0] != 2 || stats->base[0] != 2)
        return fail(ctx, NNT_EINVAL, std::string(who) + ": stats must be fp32 [2, ...] with an untiled first axis");
    for (int a = 1; a < X->ndim; a++)
        if (stats->shape[a] != X->shape[a] || stats->base[a] != X->base[a])
            return fail(ctx, NNT_EINVAL, std::string(who) + ": stats must be tiled like X's other axes");
    for (void* p : X->tiles) if (!p) return fail(ctx, NNT_EINVAL, std::string(who) + ": structural-zero tiles not allowed");
    for (void* p : stats->tiles) if (!p) return fail(ctx, NNT_EINVAL, std::string(who) + ": structural-zero tiles not allowed");
    for (void* p : gamma->tiles) if (!p) return fail(ctx, NNT_EINVAL, std::string(who) + ": structural-zero tiles not allowed");
    return NNT_OK;
}

}  // namespace
}  // namespace nnt

using namespace nnt;

#define DT_OK(d) ((d) == NNT_F32 || (d) == NNT_BF16)
// Runs CALL with T = element type and V = vector width (full width when `vec`, else 1).
#define DISPATCH_TV(dtype, vec, CALL)                                           \
    do {                                                                        \
        if ((dtype) == NNT_F32) {                                               \
            typedef float T;                                                    \
            if (vec) { constexpr int V = 4; CALL; } else { constexpr int V = 1; CALL; } \
        } else {                                                                \
            typedef bf16_t T;                                                   \
            if (vec) { constexpr int V = 8; CALL; } else { constexpr int V = 1; CALL; } \
        }                                                                       \
    } while (0)

static inline bool cols_ok(int64_t m, int64_t n) { return m >= 1 && n >= 0 && m <= INT32_MAX && n <= (int64_t)INT32_MAX * 4; }

// ------------------------------------------------------------------ bias gradient without any allocation
// Partial column sums of nnt_tile_bias_grad_static live in this array: one copy per GPU, held until
// the process ends.  In host code the array's name is only a stand-in for the symbol; the device
// address is looked up once per device and kept.
constexpr int64_t kStaticScratchElems = (int64_t)1 << 20;      // 4 MiB of fp32
constexpr int kStaticMaxDevices = 64;
static __device__ __align__(256) float static_scratch[kStaticScratchElems];

namespace {
std::mutex g_static_mu;
float* g_static_ptr[kStaticMaxDevices] = {};

// device address of this GPU's copy of `static_scratch` (current device), or nullptr with *rc set
float* static_scratch_of_current_device(int32_t* rc) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kStaticMaxDevices) { *rc = NNT_EHIP; return nullptr; }
    std::lock_guard<std::mutex> lock(g_static_mu);
    if (!g_static_ptr[dev]) {
        float* ptr = nullptr;
        if (hipGetSymbolAddress((void**)&ptr, HIP_SYMBOL(static_scratch)) != hipSuccess || !ptr) { *rc = NNT_EHIP; return nullptr; }
        g_static_ptr[dev] = ptr;
    }
    *rc = NNT_OK;
    return g_static_ptr[dev];
}
}  // namespace

namespace nnt {
int32_t static_scratch_setup() {
    int32_t rc;
    (void)static_scratch_of_current_device(&rc);
    return rc;
}
}  // namespace nnt

extern "C" {

int32_t nnt_tile_ln_stats(void* stream, int32_t dtype, int64_t m, int64_t n, const void* x, float* stats,
                          int64_t count_before, int64_t finalize_total, float eps) {
    if (!DT_OK(dtype)) return NNT_EDTYPE;
    if (!cols_ok(m, n) || count_before < 0 || (finalize_total > 0 && finalize_total != count_before + m)) return NNT_EINVAL;
    if (n == 0) return NNT_OK;
    if (!x || !stats) return NNT_EINVAL;
    const bool vec = aligned16(x) && m % (dtype == NNT_F32 ? 4 : 8) == 0;
    const dim3 grid((unsigned)((n + 3) / 4)), block(256);
    DISPATCH_TV(dtype, vec, hipLaunchKernelGGL((ln_stats_tile<T, V>), grid, block, 0, (hipStream_t)stream,
                                               (const T*)x, stats, (int)m, n, count_before, finalize_total, eps));
    return hipGetLastError() == hipSuccess ? NNT_OK : NNT_EHIP;
}

int32_t nnt_tile_ln_apply(void* stream, int32_t dtype, int64_t m, int64_t n, const void* x, const float* stats,
                          const float* gamma, const float* beta, void* y) {
    if (!DT_OK(dtype)) return NNT_EDTYPE;
    if (!cols_ok(m, n)) return NNT_EINVAL;
    if (n == 0) return NNT_OK;
    if (!x || !stats || !gamma || !beta || !y) return NNT_EINVAL;
    const bool vec = aligned16(x) && aligned16(y) && aligned16(gamma) && aligned16(beta) && m % (dtype == NNT_F32 ? 4 : 8) == 0;
    const dim3 grid((unsigned)((n + 3) / 4)), block(256);
    DISPATCH_TV(dtype, vec, hipLaunchKernelGGL((ln_apply_tile<T, V>), grid, block, 0, (hipStream_t)stream,
                                               (const T*)x, stats, gamma, beta, (T*)y, (int)m, n));
    return hipGetLastError() == hipSuccess ? NNT_OK : NNT_EHIP;
}

int32_t nnt_tile_ln_bwd_sums(void* stream, int32_t dtype, int64_t m, int64_t n, const void* x, const float* stats,
                             const float* gamma, const void* dy, float* sums, int32_t init) {
    if (!DT_OK(dtype)) return NNT_EDTYPE;
    if (!cols_ok(m, n)) return NNT_EINVAL;
    if (n == 0) return NNT_OK;
    if (!x || !stats || !gamma || !dy || !sums) return NNT_EINVAL;
    const bool vec = aligned16(x) && aligned16(dy) && aligned16(gamma) && m % (dtype == NNT_F32 ? 4 : 8) == 0;
    const dim3 grid((unsigned)((n + 3) / 4)), block(256);
    DISPATCH_TV(dtype, vec, hipLaunchKernelGGL((ln_bwd_sums_tile<T, V>), grid, block, 0, (hipStream_t)stream,
                                               (const T*)x, stats, gamma, (const T*)dy, sums, (int)init, (int)m, n));
    return hipGetLastError() == hipSuccess ? NNT_OK : NNT_EHIP;
}

int32_t nnt_tile_ln_bwd_dx(void* stream, int32_t dtype, int64_t m, int64_t n, int64_t N_e, const void* x,
                           const float* stats, const float* gamma, const void* dy, const float* sums,
                           const void* dres, void* dx) {
    if (!DT_OK(dtype)) return NNT_EDTYPE;
    if (!cols_ok(m, n) || N_e < m) return NNT_EINVAL;
    if (n == 0) return NNT_OK;
    if (!x || !stats || !gamma || !dy || !sums || !dx) return NNT_EINVAL;
    const bool vec = aligned16(x) && aligned16(dy) && aligned16(gamma) && aligned16(dx) && (!dres || aligned16(dres)) &&
                     m % (dtype == NNT_F32 ? 4 : 8) == 0;
    const dim3 grid((unsigned)((n + 3) / 4)), block(256);
    const float inv_N = 1.f / (float)N_e;
    DISPATCH_TV(dtype, vec, hipLaunchKernelGGL((ln_bwd_dx_tile<T, V>), grid, block, 0, (hipStream_t)stream,
                                               (const T*)x, stats, gamma, (const T*)dy, sums, (const T*)dres, (T*)dx, (int)m, n, inv_N));
    return hipGetLastError() == hipSuccess ? NNT_OK : NNT_EHIP;
}

int64_t nnt_tile_ln_bwd_params_scratch(int64_t m, int64_t n) { return m < 0 || n < 0 ? 0 : scratch_elems(m, std::max<int64_t>(n, 1), 1); }
int64_t nnt_tile_bias_grad_scratch(int64_t m, int64_t n) { return m < 0 || n < 0 ? 0 : scratch_elems(m, std::max<int64_t>(n, 1), 0); }

int32_t nnt_tile_ln_bwd_params(void* stream, int32_t dtype, int64_t m, int64_t n, const void* x, const float* stats,
                               const void* dy, float* dgamma, float* dbeta, int32_t accumulate, float* scratch) {
    if (!DT_OK(dtype)) return NNT_EDTYPE;
    if (!cols_ok(m, n)) return NNT_EINVAL;
    if (!x || !stats || !dy || !dgamma || !dbeta || !scratch) return NNT_EINVAL;
    return rowsum_single((hipStream_t)stream, dtype, 1, m, n, dy, x, stats, dgamma, dbeta, accumulate, scratch);
}

int32_t nnt_tile_bias_grad(void* stream, int32_t dtype, int64_t m, int64_t n, const void* dY, float* db,
                           int32_t accumulate, float* scratch) {
    if (!DT_OK(dtype)) return NNT_EDTYPE;
    if (!cols_ok(m, n)) return NNT_EINVAL;
    if (!dY || !db || !scratch) return NNT_EINVAL;
    return rowsum_single((hipStream_t)stream, dtype, 0, m, n, dY, nullptr, nullptr, db, nullptr, accumulate, scratch);
}

// ------------------------------------------------------------------ bias gradient without any allocation
int64_t nnt_tile_bias_grad_static_max(void) { return kStaticScratchElems; }

int32_t nnt_tile_bias_grad_static(void* stream, int32_t dtype, int64_t m, int64_t n, const void* dY, float* db,
                                  int32_t accumulate) {
    if (!DT_OK(dtype)) return NNT_EDTYPE;
    if (!cols_ok(m, n)) return NNT_EINVAL;
    if (!dY || !db) return NNT_EINVAL;
    if (scratch_elems(m, n, 0) > kStaticScratchElems) return NNT_EINVAL;      // partial sums would not fit the static array
    int32_t rc;
    float* part = static_scratch_of_current_device(&rc);
    if (!part) return rc;
    // every partial row that stage 2 reads is written by stage 1 of this call: nothing to clear
    return rowsum_single((hipStream_t)stream, dtype, 0, m, n, dY, nullptr, nullptr, db, nullptr, accumulate, part);
}

// ------------------------------------------------------------------ tensor form
int32_t nnt_bias_grad(nnt_ctx* ctx, nnt_tensor* dY, nnt_tensor* db) {
    NNT_CHECK_CTX(ctx);
    if (!dY || !db) return fail(ctx, NNT_EINVAL, "nnt_bias_grad: null tensor");
    if (db->dtype != NNT_F32 || db->ndim != 1 || db->shape[0] != dY->shape[0] || db->base[0] != dY->base[0])
        return fail(ctx, NNT_EINVAL, "nnt_bias_grad: db must be an fp32 vector tiled like dY's first axis");
    for (void* p : dY->tiles) if (!p) return fail(ctx, NNT_EINVAL, "nnt_bias_grad: structural-zero tiles not allowed");
    for (void* p : db->tiles) if (!p) return fail(ctx, NNT_EINVAL, "nnt_bias_grad: structural-zero tiles not allowed");
    double numel = 1;
    for (int a = 0; a < dY->ndim; a++) numel *= (double)dY->shape[a];
    OpTag tag(ctx, "bias_grad", numel * dY->elem_size(), true);
    if (ctx->granularity == NNT_GRAN_OP) return rowsum_tensor(ctx, 0, dY, nullptr, nullptr, db, nullptr);
    // tile by tile: each dY tile adds its column sums to the db tile of its row range
    std::vector<char> seen(db->ntiles, 0);
    for (int64_t t = 0; t < dY->ntiles; t++) {
        const int64_t c0 = t % dY->grid[0];
        const int64_t m = dY->tile_extent(0, c0), n = dY->tile_numel(t) / m;
        int32_t rc = ensure_scratch(ctx, scratch_elems(m, n, 0));
        if (rc != NNT_OK) return rc;
        const void* yp = dY->tiles[t];
        float* op = static_cast<float*>(db->tiles[c0]);
        float* scratch = ctx->red_scratch;
        const int acc = seen[c0];
        seen[c0] = 1;
        const int dt = dY->dtype;
        rc = submit(ctx, {dY->one(t, kRead), db->one(c0, acc ? kReadWrite : kWrite), Access{&ctx->red_dep, 1, kReadWrite}},
                    [=](hipStream_t st) { return rowsum_single(st, dt, 0, m, n, yp, nullptr, nullptr, op, nullptr, acc, scratch); }, 2);
        if (rc != NNT_OK) return rc;
    }
    return NNT_OK;
}

int32_t nnt_layernorm_fwd(nnt_ctx* ctx, nnt_tensor* X, nnt_tensor* gamma, nnt_tensor* beta, float eps,
                          nnt_tensor* Y, nnt_tensor* stats) {
    NNT_CHECK_CTX(ctx);
    if (!X || !gamma || !beta || !Y || !stats) return fail(ctx, NNT_EINVAL, "nnt_layernorm_fwd: null tensor");
    int32_t rc = check_ln_shapes(ctx, X, gamma, stats, "nnt_layernorm_fwd");
    if (rc != NNT_OK) return rc;
    if (!same_tiling(gamma, beta) || beta->dtype != NNT_F32 || !same_tiling(X, Y) || X->dtype != Y->dtype)
        return fail(ctx, NNT_EINVAL, "nnt_layernorm_fwd: operands tiled or typed differently");
    for (void* p : Y->tiles) if (!p) return fail(ctx, NNT_EINVAL, "nnt_layernorm_fwd: structural-zero tiles not allowed");
    for (void* p : beta->tiles) if (!p) return fail(ctx, NNT_EINVAL, "nnt_layernorm_fwd: structural-zero tiles not allowed");
    const int dtype = X->dtype;
    double numel = 1;
    for (int a = 0; a < X->ndim; a++) numel *= (double)X->shape[a];
    // one wave per token reads x once and writes y once; tile by tile x is read twice
    OpTag tag(ctx, "layernorm_fwd", numel * X->elem_size() * (ctx->granularity == NNT_GRAN_OP ? 2 : 3), true);
    if (ctx->granularity == NNT_GRAN_OP) {
        const int V = dtype == NNT_F32 ? 4 : 8;
        const bool vec = tensors_vec_ok({X, Y, gamma, beta}, V), any = any_vec({X, Y, gamma, beta});
        const int nv = (int)(((X->base[0] + 64 * V - 1) / (64 * V)) * X->grid[0]);
        const TiledView vx = X->view(), vy = Y->view(), vs = stats->view(), vg = gamma->view(), vb = beta->view();
        const int64_t ncols = n_columns(X);
        if (ncols > INT32_MAX) return fail(ctx, NNT_EINVAL, "nnt_layernorm_fwd: tensor too large");
        std::vector<Access> acc = {X->all(kRead), gamma->all(kRead), beta->all(kRead), Y->all(kWrite), stats->all(kWrite)};
        return submit(ctx, acc, [=](hipStream_t st) {
            return dtype == NNT_F32 ? launch_ln_fwd<float>(st, vec, any, nv, vx, vy, vs, vg, vb, eps, ncols)
                                    : launch_ln_fwd<bf16_t>(st, vec, any, nv, vx, vy, vs, vg, vb, eps, ncols);
        });
    }
    // the paper's steps, tile by tile
    const int64_t g0 = X->grid[0], rest = X->ntiles / g0, N_e = X->shape[0];
    for (int64_t r = 0; r < rest; r++) {
        float* sp = static_cast<float*>(stats->tiles[r]);
        int64_t before = 0;
        for (int64_t l = 0; l < g0; l++) {
            const int64_t t = l + g0 * r, m = X->tile_extent(0, l), n = X->tile_numel(t) / m;
            const void* xp = X->tiles[t];
            const int64_t fin = l == g0 - 1 ? N_e : 0;
            rc = submit(ctx, {X->one(t, kRead), stats->one(r, l == 0 ? kWrite : kReadWrite)},
                        [=](hipStream_t st) { return nnt_tile_ln_stats(st, dtype, m, n, xp, sp, before, fin, eps); });
            if (rc != NNT_OK) return rc;
            before += m;
        }
    }
    for (int64_t t = 0; t < X->ntiles; t++) {
        const int64_t l = t % g0, r = t / g0, m = X->tile_extent(0, l), n = X->tile_numel(t) / m;
        const void* xp = X->tiles[t];
        void* yp = Y->tiles[t];
        const float* sp = static_cast<const float*>(stats->tiles[r]);
        const float* gp = static_cast<const float*>(gamma->tiles[l]);
        const float* bp = static_cast<const float*>(beta->tiles[l]);
        rc = submit(ctx, {X->one(t, kRead), stats->one(r, kRead), gamma->one(l, kRead), beta->one(l, kRead), Y->one(t, kWrite)},
                    [=](hipStream_t st) { return nnt_tile_ln_apply(st, dtype, m, n, xp, sp, gp, bp, yp); });
        if (rc != NNT_OK) return rc;
    }
    return NNT_OK;
}

int32_t nnt_layernorm_bwd(nnt_ctx* ctx, nnt_tensor* X, nnt_tensor* stats, nnt_tensor* gamma, nnt_tensor* dY,
                          nnt_tensor* dRes, nnt_tensor* dX, nnt_tensor* dgamma, nnt_tensor* dbeta) {
    NNT_CHECK_CTX(ctx);
    if (!X || !stats || !gamma || !dY || !dX || !dgamma || !dbeta) return fail(ctx, NNT_EINVAL, "nnt_layernorm_bwd: null tensor");
    int32_t rc = check_ln_shapes(ctx, X, gamma, stats, "nnt_layernorm_bwd");
    if (rc != NNT_OK) return rc;
    if (!same_tiling(X, dY) || !same_tiling(X, dX) || (dRes && !same_tiling(X, dRes)) || X->dtype != dY->dtype ||
        X->dtype != dX->dtype || (dRes && dRes->dtype != X->dtype) || !same_tiling(gamma, dgamma) || !same_tiling(gamma, dbeta) ||
        dgamma->dtype != NNT_F32 || dbeta->dtype != NNT_F32)
        return fail(ctx, NNT_EINVAL, "nnt_layernorm_bwd: operands tiled or typed differently");
    for (nnt_tensor* t : {dY, dX, dgamma, dbeta})
        for (void* p : t->tiles) if (!p) return fail(ctx, NNT_EINVAL, "nnt_layernorm_bwd: structural-zero tiles not allowed");
    if (dRes) for (void* p : dRes->tiles) if (!p) return fail(ctx, NNT_EINVAL, "nnt_layernorm_bwd: structural-zero tiles not allowed");
    const int dtype = X->dtype;
    const int64_t g0 = X->grid[0], rest = X->ntiles / g0, N_e = X->shape[0];
    double numel = 1;
    for (int a = 0; a < X->ndim; a++) numel *= (double)X->shape[a];
    // parameter gradients read x and dy; the input gradient reads x, dy (and the residual) and writes dx: in one pass x and dy are read once
    const double bytes = numel * X->elem_size();
    OpTag tag(ctx, "layernorm_bwd", bytes * (5 + (dRes ? 1 : 0)), true);
    if (ctx->granularity == NNT_GRAN_OP) {
        const int V = dtype == NNT_F32 ? 4 : 8;
        const bool vec = tensors_vec_ok({X, dY, dX, dRes, gamma}, V);
        const int nv = (int)(((X->base[0] + 64 * V - 1) / (64 * V)) * X->grid[0]);
        const TiledView vx = X->view(), vs = stats->view(), vg = gamma->view(), vdy = dY->view(), vdx = dX->view();
        const TiledView vr = dRes ? dRes->view() : vdy;
        const int has_res = dRes != nullptr;
        const int64_t ncols = n_columns(X);
        if (ncols > INT32_MAX) return fail(ctx, NNT_EINVAL, "nnt_layernorm_bwd: tensor too large");
        std::vector<Access> acc = {X->all(kRead), stats->all(kRead), gamma->all(kRead), dY->all(kRead), dX->all(kWrite)};
        if (dRes) acc.push_back(dRes->all(kRead));
        // One pass over the tokens wherever the eight waves of a workgroup can hold one (see ln_bwd_onepass for both sides); longer ones take the column
        // sums and the input gradient one after the other.
        // Tiles that fill less than half of a wave's lanes, more than 1024 tokens: two passes as well.  The one pass is the faster call by itself there too,
        // but its 256 large workgroups, most lanes idle, hold up the products of the other stream: 66 blocks and models of 128 to 768 wide on tiles of
        // 64 and 128 with 2048 and 4096 tokens are 1 % faster in two passes on average (0.93 to 1.04), 33 with 1024 tokens 1 % slower.
        // Odd extents: the two passes take them element by element, 64 to a step, which is slower (4097 x 1000 on tiles of 1024 1.8 times) but for tiles of up to 64 rows: more than
        // 1024 tokens, or more than 256 of more than eight vectors per lane (bf16 500 x 4000 on tiles of 50 23 us and 56, 63 x 1000 on tiles of 5 20 and 35, fp32 500 x 4000
        // 25 and 44; with fewer 1.0 to 1.6 times the other way round).
        const int lanes = 64 * V * (int)((X->base[0] + 64 * V - 1) / (64 * V));
        const bool narrow = vec ? 2 * X->base[0] < lanes && ncols > 1024 : X->base[0] <= 64 && (ncols > 1024 || (nv > 8 && ncols > 256));
        const int wpt = !narrow && (vec || any_vec({X, dY, dX, dRes, gamma})) ? onepass_waves(vec && dtype == NNT_BF16, nv, ncols) : 0;
        // (so do calls inside a capture whose partial rows have no room yet)
        const int64_t wgs = wpt > 0 ? onepass_wgs(wpt, ncols) : 0, rows = X->shape[0];
        if (wpt > 0 && ncols > 0 && ncols < INT32_MAX / 2 && X->ntiles <= 65535 && !(ctx->capturing && 2 * wgs * rows > ctx->stream_scratch_elems)) {
            rc = keep_rowsum_scratch(ctx, 1, dY);
            if (rc != NNT_OK) return rc;
            rc = ensure_stream_scratch(ctx, 2 * wgs * rows);
            if (rc != NNT_OK) return rc;
            // (what the records say; for the choice of a stream the operation keeps the weight of two passes, being as long as a pass over that much:
            // 11 to 16 us with its second launch where x, dy, the residual and dx are 10 to 16 MB.  Counted by those bytes it would be a small task: 20
            // blocks and models with such adjoints 0.4 % slower, bf16 768 x 2048 580 -> 595 us, fp32 1024 x 896 3060 -> 3115)
            ctx->cur_work = bytes * (3 + (dRes ? 1 : 0));
            void* const* og = dgamma->d_tiles;
            void* const* ob = dbeta->d_tiles;
            const int base0 = (int)dgamma->base[0];
            acc.push_back(dgamma->all(kWrite));
            acc.push_back(dbeta->all(kWrite));
            return submit(ctx, acc, [=](hipStream_t st) {
                float* part = stream_scratch_of(ctx);
                const int32_t r = dtype == NNT_F32 ? launch_onepass<float>(st, vec, wpt, nv, vx, vs, vg, vdy, vr, vdx, has_res, ncols, part)
                                                   : launch_onepass<bf16_t>(st, vec, wpt, nv, vx, vs, vg, vdy, vr, vdx, has_res, ncols, part);
                if (r != NNT_OK) return r;
                return launch_stage2(st, part, wgs, rows, og, ob, base0);
            }, 2);
        }
        rc = rowsum_tensor(ctx, 1, dY, X, stats, dgamma, dbeta);
        if (rc != NNT_OK) return rc;
        return submit(ctx, acc, [=](hipStream_t st) {
            return dtype == NNT_F32 ? launch_ln_bwd<float>(st, vec, nv, vx, vs, vg, vdy, vr, vdx, has_res, ncols)
                                    : launch_ln_bwd<bf16_t>(st, vec, nv, vx, vs, vg, vdy, vr, vdx, has_res, ncols);
        });
    }
    // tile by tile.  The per-token sums live in the reduction scratch: [2][columns] per group of tiles.
    int64_t max_cols = 1;
    for (int a = 1; a < X->ndim; a++) max_cols *= X->base[a];
    int64_t pmax = 0;
    for (int64_t l = 0; l < g0; l++) pmax = std::max(pmax, scratch_elems(X->tile_extent(0, l), max_cols, 1));
    rc = ensure_scratch(ctx, 2 * max_cols + pmax);
    if (rc != NNT_OK) return rc;
    float* sums = ctx->red_scratch;
    float* pscratch = ctx->red_scratch + 2 * max_cols;
    std::vector<char> seen(gamma->ntiles, 0);
    const Access scr{&ctx->red_dep, 1, kReadWrite};
    for (int64_t r = 0; r < rest; r++) {
        const float* sp = static_cast<const float*>(stats->tiles[r]);
        for (int64_t l = 0; l < g0; l++) {
            const int64_t t = l + g0 * r, m = X->tile_extent(0, l), n = X->tile_numel(t) / m;
            const void* xp = X->tiles[t];
            const void* dyp = dY->tiles[t];
            const float* gp = static_cast<const float*>(gamma->tiles[l]);
            const int init = l == 0;
            rc = submit(ctx, {X->one(t, kRead), dY->one(t, kRead), stats->one(r, kRead), gamma->one(l, kRead), scr},
                        [=](hipStream_t st) { return nnt_tile_ln_bwd_sums(st, dtype, m, n, xp, sp, gp, dyp, sums, init); });
            if (rc != NNT_OK) return rc;
        }
        for (int64_t l = 0; l < g0; l++) {
            const int64_t t = l + g0 * r, m = X->tile_extent(0, l), n = X->tile_numel(t) / m;
            const void* xp = X->tiles[t];
            const void* dyp = dY->tiles[t];
            const void* rp = dRes ? dRes->tiles[t] : nullptr;
            void* dxp = dX->tiles[t];
            const float* gp = static_cast<const float*>(gamma->tiles[l]);
            float* dgp = static_cast<float*>(dgamma->tiles[l]);
            float* dbp = static_cast<float*>(dbeta->tiles[l]);
            const int acc = seen[l];
            seen[l] = 1;
            std::vector<Access> a1 = {X->one(t, kRead), dY->one(t, kRead), stats->one(r, kRead), gamma->one(l, kRead), scr,
                                      dgamma->one(l, acc ? kReadWrite : kWrite), dbeta->one(l, acc ? kReadWrite : kWrite)};
            rc = submit(ctx, a1, [=](hipStream_t st) {
                return rowsum_single(st, dtype, 1, m, n, dyp, xp, sp, dgp, dbp, acc, pscratch);
            }, 2);
            if (rc != NNT_OK) return rc;
            std::vector<Access> a2 = {X->one(t, kRead), dY->one(t, kRead), stats->one(r, kRead), gamma->one(l, kRead), scr,
                                      dX->one(t, kWrite)};
            if (dRes) a2.push_back(dRes->one(t, kRead));
            rc = submit(ctx, a2, [=](hipStream_t st) {
                return nnt_tile_ln_bwd_dx(st, dtype, m, n, N_e, xp, sp, gp, dyp, sums, rp, dxp);
            });
            if (rc != NNT_OK) return rc;
        }
    }
    return NNT_OK;
}

}  // extern "C"
