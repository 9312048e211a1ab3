// fp32 tile-grid product on the gfx950 matrix cores (v_mfma_f32_32x32x2_f32):
// true fp32 inputs, fp32 accumulation.
//
// One workgroup of four wavefronts owns a BM x BN macro-tile of one C tile and
// walks the task's chunks in k-steps of 16.  Both operands are staged through
// LDS in the orientation they have in memory (no transposes): an operand whose
// contracted index is contiguous ("k-fast") is kept as [row][16 + 4 pad], one
// whose row index is contiguous as [k][rows]; the matrix-core fragments are read
// with 128-bit or 32-bit LDS loads accordingly.  Global loads for step i+1 are
// issued before the MFMAs of step i and written to the other LDS buffer after
// them, so each step costs one barrier.
//
// The matrix-core "A" operand carries the columns of C (index n) and the "B"
// operand the rows (index m): a lane then holds 16 values of one row index m =
// lane % 32, and the 32 lanes of a half-wave store 32 consecutive rows, which are
// contiguous in the column-major C tile.
#include "gemm_common.hpp"
#include "gemm_f32_out.hpp"
#include "nntile_mi.h"

namespace nnt {

typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace {

// A pointer that is the same in every lane, moved to scalar registers.
template <typename T>
__device__ __forceinline__ const T* uniform_ptr(const T* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return in_global(reinterpret_cast<const T*>(((uint64_t)hi << 32) | lo));
}

constexpr int BK = 16;
constexpr int kSumSteps = 16;  // k-steps between two moves of the sums (256 k)
constexpr int KP = BK + 4;   // padded k extent of a k-fast LDS row (conflict-free 128-bit reads)

// Four floats at any address that a float may have: global memory takes 16-byte accesses at every multiple of 4 bytes,
// so odd leading dimensions and operands that start anywhere are read with vectors too (read one element at a time,
// an operand of odd extents kept these kernels at 20 to 35 TFLOP/s).
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// Where vector i of this thread lies in a step's block: row r, first k.
template <bool KF, int ROWS>
__device__ __forceinline__ void vec_at(int tid, int i, int& r, int& k) {
    const int idx = tid + 256 * i;
    if (KF) { r = idx >> 2; k = (idx & 3) << 2; }
    else { k = idx / (ROWS / 4); r = (idx % (ROWS / 4)) << 2; }
}

// Interior k-step: no predicates, no branches, so the loads stay in flight across the
// matrix-core work that follows.  `base` points at (row0, k0).
template <bool KF, int ROWS>
__device__ __forceinline__ void gload_fast(f32x4 (&v)[ROWS / 64], const float* base, int ld, int tid) {
#pragma unroll
    for (int i = 0; i < ROWS / 64; i++) {
        int r, k;
        vec_at<KF, ROWS>(tid, i, r, k);
        const float* p = KF ? base + k + (int64_t)r * ld : base + r + (int64_t)k * ld;
        v[i] = *reinterpret_cast<const f32x4u*>(p);
    }
}

// A step that reaches beyond the operand's `nrows` rows or the chunk's `kc` k (both counted from `base`): every lane
// fetches four elements that exist, whole rows (or lines) beyond the edge standing in for the last one, and a vector
// that crosses the edge along its own direction being moved back until it ends there (mend_edge puts its elements in
// place).  Like the interior form it branches only on scalars, so these loads stay in flight as well.  Operands with
// fewer than four elements along the vectors' direction are read one by one.
template <bool KF, int ROWS>
__device__ __forceinline__ void gload_edge(f32x4 (&v)[ROWS / 64], const float* base, int ld, int row0, int nrows, int k0, int kc, int tid) {
    const bool vectors = (KF ? kc : nrows) >= 4;
#pragma unroll
    for (int i = 0; i < ROWS / 64; i++) {
        int r, k;
        vec_at<KF, ROWS>(tid, i, r, k);
        const int gr = row0 + r, gk = k0 + k;
        if (vectors) {
            const float* p = KF ? base + min(gk, kc - 4) + (int64_t)min(gr, nrows - 1) * ld
                                : base + min(gr, nrows - 4) + (int64_t)min(gk, kc - 1) * ld;
            v[i] = *reinterpret_cast<const f32x4u*>(p);
        } else {
            const float* p = KF ? base + gk + (int64_t)gr * ld : base + gr + (int64_t)gk * ld;
            const int cnt = KF ? (gr < nrows ? kc - gk : 0) : (gk < kc ? nrows - gr : 0);
            f32x4 x = {0.f, 0.f, 0.f, 0.f};
            if (cnt > 0) x[0] = p[0];
            if (cnt > 1) x[1] = p[1];
            if (cnt > 2) x[2] = p[2];
            v[i] = x;
        }
    }
}

// What gload_edge left in the registers, put in place once it has arrived: elements of a moved vector shifted back,
// zeros for k beyond the chunk (in both operands: whatever stands for a missing k must not meet an infinity).  Rows
// beyond the edge keep what was fetched for them: it only reaches results that are never stored.  So a step whose k all
// exist needs nothing where k is the contiguous index or the edge falls between two vectors; most steps of a macro-tile on
// an edge are such (the test is the same for every lane).
template <bool KF, int ROWS>
__device__ __forceinline__ void mend_edge(f32x4 (&v)[ROWS / 64], int row0, int nrows, int k0, int kc, int tid) {
    if ((KF ? kc : nrows) < 4) return;
    if (k0 + BK <= kc && (KF || (nrows & 3) == 0 || row0 + ROWS <= nrows)) return;
#pragma unroll
    for (int i = 0; i < ROWS / 64; i++) {
        int r, k;
        vec_at<KF, ROWS>(tid, i, r, k);
        const int over = KF ? k0 + k + 4 - kc : row0 + r + 4 - nrows;      // elements of the vector beyond the edge
        const bool gone = !KF && k0 + k >= kc;
        const f32x4 x = v[i];
        f32x4 y;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            float t = over <= 0 ? x[e] : 0.f;
#pragma unroll
            for (int s = 1; e + s < 4; s++) t = over == s ? x[e + s] : t;
            y[e] = gone ? 0.f : t;
        }
        v[i] = y;
    }
}

template <bool KF, int ROWS>
__device__ __forceinline__ void lstore(float* l, const f32x4 (&v)[ROWS / 64], int tid) {
#pragma unroll
    for (int i = 0; i < ROWS / 64; i++) {
        const int idx = tid + 256 * i;
        if (KF) {
            const int r = idx >> 2, k = (idx & 3) << 2;
            *reinterpret_cast<f32x4*>(&l[r * KP + k]) = v[i];
        } else {
            const int k = idx / (ROWS / 4), r = (idx % (ROWS / 4)) << 2;
            *reinterpret_cast<f32x4*>(&l[k * ROWS + r]) = v[i];
        }
    }
}

// The 8 k-values of this lane's half (k = 8 * half + j) for one 32-row block.
template <bool KF, int ROWS>
__device__ __forceinline__ void lfrag(float (&f)[8], const float* l, int row, int half) {
    if (KF) {
        const f32x4 a = *reinterpret_cast<const f32x4*>(&l[row * KP + half * 8]);
        const f32x4 b = *reinterpret_cast<const f32x4*>(&l[row * KP + half * 8 + 4]);
        f[0] = a[0]; f[1] = a[1]; f[2] = a[2]; f[3] = a[3];
        f[4] = b[0]; f[5] = b[1]; f[6] = b[2]; f[7] = b[3];
    } else {
#pragma unroll
        for (int j = 0; j < 8; j++) f[j] = l[(half * 8 + j) * ROWS + row];
    }
}

// (two workgroups per compute unit asked for: within 256 registers the compiler keeps the matrix accumulators in vector
// registers; otherwise it takes accumulation registers and copies them out and back in every k-step)
template <bool AKF, bool BKF, int WAVES_M, int WAVES_N, int WMB, int WNB>
__global__ void __launch_bounds__(256, 2) gemm_f32_kernel(const GemmArgs g) {
    constexpr int BM = 32 * WMB * WAVES_M, BN = 32 * WNB * WAVES_N;
    constexpr int A_SZ = AKF ? BM * KP : BK * BM;
    constexpr int B_SZ = BKF ? BN * KP : BK * BN;
    __shared__ __attribute__((aligned(16))) float lds[2 * (A_SZ + B_SZ)];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WAVES_M, wn = wave / WAVES_M;
    const int r32 = lane & 31, half = lane >> 5;

    GemmTask task;
    int m0, n0, bat;
    // (the chunk table is only ever addressed through g.chunks, a global pointer with a uniform
    // index, so that the descriptors arrive through scalar loads and the loop control stays scalar)
    const bool table = g.wgs != nullptr;
    if (table) {
        const GemmWg w = g.wgs[blockIdx.x];
        task = g.tasks[w.task];
        m0 = w.m0; n0 = w.n0; bat = w.batch;
    } else {
        task = g.one_task;
        const int b = blockIdx.x;
        m0 = (b % g.grid_m) * BM;
        n0 = ((b / g.grid_m) % g.grid_n) * BN;
        bat = b / (g.grid_m * g.grid_n);
    }
    // (batch members that are pairs: see GemmTask::nb1)
    int bat_lo = bat, bat_hi = 0;
    if (task.nb1 > 0) {
        bat_hi = bat / task.nb1;
        bat_lo = bat - bat_hi * task.nb1;
    }

    f32x16 sum[WNB][WMB];
    clear<WMB, WNB>(sum);

    if (task.nchunk > 0) {
        // Loop state that is the same for every lane is kept in scalar registers on purpose
        // (readfirstlane): the k-loop then branches on the scalar unit and the loads address
        // memory as scalar base + per-lane offset.
        int c = 0, k0 = 0, chk = 0, lda = 0, ldb = 0;
        const float* Ab = nullptr;
        const float* Bb = nullptr;
        auto set_chunk = [&](const GemmChunk& ch) {
            chk = __builtin_amdgcn_readfirstlane(ch.k);
            lda = __builtin_amdgcn_readfirstlane((int)ch.lda);
            ldb = __builtin_amdgcn_readfirstlane((int)ch.ldb);
            Ab = uniform_ptr(static_cast<const float*>(ch.A) + (int64_t)bat_lo * ch.strideA + (int64_t)bat_hi * ch.strideA2);
            Bb = uniform_ptr(static_cast<const float*>(ch.B) + (int64_t)bat_lo * ch.strideB + (int64_t)bat_hi * ch.strideB2);
        };
        set_chunk(table ? g.chunks[task.chunk0] : g.one_chunk);
        f32x4 va[BM / 64], vb[BN / 64];
        // whole macro-tile inside the C tile: k-steps that are also whole need no look at the edges
        const bool inside = m0 + BM <= task.m && n0 + BN <= task.n;
        bool edge = false;              // of the step in the registers: whether it has to be mended, its k0 and chunk length
        int ek0 = 0, ekc = 0;
        auto load_step = [&]() {
            edge = !(inside && k0 + BK <= chk);
            ek0 = k0;
            ekc = chk;
            if (!edge) {
                gload_fast<AKF, BM>(va, AKF ? Ab + k0 + (int64_t)m0 * lda : Ab + m0 + (int64_t)k0 * lda, lda, tid);
                gload_fast<BKF, BN>(vb, BKF ? Bb + k0 + (int64_t)n0 * ldb : Bb + n0 + (int64_t)k0 * ldb, ldb, tid);
            } else {
                gload_edge<AKF, BM>(va, Ab, lda, m0, task.m, k0, chk, tid);
                gload_edge<BKF, BN>(vb, Bb, ldb, n0, task.n, k0, chk, tid);
            }
        };
        auto store_step = [&](float* l) {
            if (edge) {
                mend_edge<AKF, BM>(va, m0, task.m, ek0, ekc, tid);
                mend_edge<BKF, BN>(vb, n0, task.n, ek0, ekc, tid);
            }
            lstore<AKF, BM>(l, va, tid);
            lstore<BKF, BN>(l + A_SZ, vb, tid);
        };
        load_step();
        int cur = 0;
        store_step(lds);
        __syncthreads();
        bool more = true;
        while (more) {
            f32x16 acc[WNB][WMB];
            clear<WMB, WNB>(acc);
            for (int step = 0; more && step < kSumSteps; step++) {
                // advance to the next k-step (possibly the next chunk) and start its loads
                k0 += BK;
                if (k0 >= chk) {
                    c++;
                    k0 = 0;
                    if (c < task.nchunk) set_chunk(g.chunks[task.chunk0 + c]);
                }
                more = c < task.nchunk;
                if (more) load_step();
                const float* lA = lds + cur * (A_SZ + B_SZ);
                const float* lB = lA + A_SZ;
                float pf[WNB][8], qf[WMB][8];
#pragma unroll
                for (int bn = 0; bn < WNB; bn++) lfrag<BKF, BN>(pf[bn], lB, (wn * WNB + bn) * 32 + r32, half);
#pragma unroll
                for (int bm = 0; bm < WMB; bm++) lfrag<AKF, BM>(qf[bm], lA, (wm * WMB + bm) * 32 + r32, half);
#pragma unroll
                for (int j = 0; j < 8; j++)
#pragma unroll
                    for (int bn = 0; bn < WNB; bn++)
#pragma unroll
                        for (int bm = 0; bm < WMB; bm++)
                            acc[bn][bm] = __builtin_amdgcn_mfma_f32_32x32x2f32(pf[bn][j], qf[bm][j], acc[bn][bm], 0, 0, 0);
                if (more) store_step(lds + (cur ^ 1) * (A_SZ + B_SZ));
                __syncthreads();
                cur ^= 1;
            }
            add_sums<WMB, WNB>(acc, sum);
        }
    }

    write_tile_f32<WMB, WNB>(sum, global_as<float>(task.C) + (int64_t)bat_lo * task.strideC + (int64_t)bat_hi * task.strideC2, task.ldc, task.cin_off,
                             in_global(task.bias), task.partial ? 1.f : g.alpha, task.partial ? 0.f : g.beta, m0 + wm * WMB * 32,
                             n0 + wn * WNB * 32, task.m, task.n, lane);
}

using KernelFn = void (*)(const GemmArgs);

template <bool AKF, bool BKF>
KernelFn kernel_of(int cfg) {
    switch (cfg) {
        case kCfgMid:
        case kCfgResident: return gemm_f32_kernel<AKF, BKF, 2, 2, 1, 2>;
        case kCfgSkinny64n128: return gemm_f32_kernel<AKF, BKF, 1, 4, 2, 1>;
        case kCfgSkinny64n64: return gemm_f32_kernel<AKF, BKF, 2, 2, 1, 1>;
        default: return gemm_f32_kernel<AKF, BKF, 2, 2, 2, 2>;
    }
}

KernelFn kernel_of(int akf, int bkf, int cfg) {
    if (akf) return bkf ? kernel_of<true, true>(cfg) : kernel_of<true, false>(cfg);
    return bkf ? kernel_of<false, true>(cfg) : kernel_of<false, false>(cfg);
}

}  // namespace

int32_t launch_gemm_f32(hipStream_t st, int akf, int bkf, int cfg, const GemmArgs& g, int64_t nwg) {
    if (nwg <= 0) return NNT_OK;
    hipLaunchKernelGGL(kernel_of(akf, bkf, cfg), dim3((unsigned)nwg), dim3(256), 0, st, g);
    return hipGetLastError() == hipSuccess ? NNT_OK : NNT_EHIP;
}


}  // namespace nnt
