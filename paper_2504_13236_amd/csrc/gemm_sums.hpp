// Partial sums of the product kernels, beside the accumulators of their matrix instructions.
#pragma once
#include <hip/hip_runtime.h>

namespace nnt {

typedef float f32x16 __attribute__((ext_vector_type(16)));

template <int WMB, int WNB>
__device__ __forceinline__ void clear(f32x16 (&acc)[WNB][WMB]) {
#pragma unroll
    for (int bn = 0; bn < WNB; bn++)
#pragma unroll
        for (int bm = 0; bm < WMB; bm++)
#pragma unroll
            for (int i = 0; i < 16; i++) acc[bn][bm][i] = 0.f;
}

// Adds what the matrix instructions have summed up to the sums so far; the accumulators then start again from zero.  A chain
// of k additions in fp32 is off by about sqrt(k) roundings of its result; cut every 256 k, with the partial sums added up on
// the side, a contraction of 8192 is off by a sixth of that, whether or not it is cut into slices as well.  (At 512 k a tenth
// of 150 random layers were less exact than products cut into more slices had been, 2.9e-7 -> 4.0e-7 at worst; at 256 none, for
// 0.5 % of a four-block model's time.)
// This belongs behind a loop of its own over the 256 k, not behind a test inside the one loop over all of them: there the
// accumulators leave their registers in every step.  And the wait in front is needed: a vector instruction that reads the
// result of a 32x32x2 matrix instruction has to come at least 18 wait states after it (nothing holds it back), the
// compiler counts them along one of the paths that lead here, which need not be the shortest, and left 8 to 11, so that
// the last row of the accumulators was read before it was written.  The build looks for such reads on every path.
template <int WMB, int WNB>
__device__ __forceinline__ void add_sums(const f32x16 (&acc)[WNB][WMB], f32x16 (&sum)[WNB][WMB]) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 1" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int bn = 0; bn < WNB; bn++)
#pragma unroll
        for (int bm = 0; bm < WMB; bm++)
#pragma unroll
            for (int i = 0; i < 16; i++) sum[bn][bm][i] += acc[bn][bm][i];
}

}  // namespace nnt
