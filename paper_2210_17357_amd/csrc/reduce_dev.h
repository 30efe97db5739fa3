// Per-layer sum of the quantization profile's tile partials, shared by the stand-alone reduction
// kernel and the Top-K kernels that resolve the threshold bins (which take the reduction along as extra
// workgroups when both families are profiled in one call).
#pragma once

#include "common.h"

namespace lgreco {

struct ReduceCols {
    int32_t n;
    int32_t col[kMaxQuant];
};

// errors[l][c] = sum of the layer's tile partials (fixed order -> reproducible); one workgroup per layer, of which 256
// threads add up and all meet at the barrier.  All
// columns together: per thread the same strided sums, then a tree inside the wavefront and the four wavefronts' (one barrier; with
// a tree over the workgroup in LDS, eight of them: 5.9 us instead of 3.8 on 16 layers of 7 columns, 6 instead of 4.5 on 62).
__device__ __forceinline__ void reduce_partials_block(const double* __restrict__ partials, int stride,
                                                      const ReduceCols& cols, const DevLayer* __restrict__ layers,
                                                      double* __restrict__ errors, int layer,
                                                      double (*s)[4]) {
    const int tid = threadIdx.x;
    if (tid < 256) {                                     // (whole wavefronts)
        const DevLayer L = layers[layer];
        double a[kMaxQuant];
#pragma unroll
        for (int ci = 0; ci < kMaxQuant; ++ci) a[ci] = 0.0;
        for (int t = L.tile_begin + tid; t < L.tile_end; t += 256) {
#pragma unroll
            for (int ci = 0; ci < kMaxQuant; ++ci)
                if (ci < cols.n) a[ci] += partials[(size_t)t * stride + cols.col[ci]];
        }
#pragma unroll
        for (int ci = 0; ci < kMaxQuant; ++ci) {
            if (ci < cols.n) {
                const double w = wave_sum(a[ci]);
                if ((tid & 63) == 0) s[ci][tid >> 6] = w;
            }
        }
    }
    __syncthreads();
    if (tid < cols.n) errors[(size_t)layer * stride + cols.col[tid]] = (s[tid][0] + s[tid][1]) + (s[tid][2] + s[tid][3]);
}

}  // namespace lgreco
