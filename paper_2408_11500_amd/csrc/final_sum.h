// Final stage of the weight-gradient reductions: partial sums of blocks of rows -> gradients, in fp64 and in a fixed order.  Its own
// launch (dense.hip), or some workgroups of the aggregation that follows (spmm.hip).
#ifndef SLICEGCN_FINAL_SUM_H
#define SLICEGCN_FINAL_SUM_H

#include "common.h"

namespace slicegcn {

struct FinalDst { float *ptr[4]; float *copy; int32_t begin[5]; }; // element ranges [begin[q], begin[q+1]) go to ptr[q], range 3 also to copy
struct FinalWork { // one entry per slice model
    const float *partial[SPMM_BATCH];
    FinalDst dst[SPMM_BATCH];
    int64_t n_blocks;
    int32_t row_stride, stride; // floats per block in memory; elements to sum
};
constexpr int FINAL_ELEMS = 32; // elements per workgroup

// out[e] = sum over row blocks of partial[b][e] for the elements [32 wg, 32 wg + 32) of slice y: 32 runs of blocks per element, then
// the runs in order.  The order is the same for every number of threads.
template <int THREADS>
__device__ inline void final_sum(const FinalWork &f, int64_t wg, int y)
{
    const float *__restrict__ partial = f.partial[y];
    const FinalDst &dst = f.dst[y];
    __shared__ double red[32][33];
    const int el = threadIdx.x % 32;
    const int64_t e = wg * FINAL_ELEMS + el;
    const int64_t per = (f.n_blocks + 31) / 32;
#pragma unroll
    for (int part = threadIdx.x / 32; part < 32; part += THREADS / 32) {
        const int64_t b0 = part * per, b1 = b0 + per < f.n_blocks ? b0 + per : f.n_blocks;
        double acc = 0.0;
        if (e < f.stride) {
            int64_t b = b0;
            for (; b + 8 <= b1; b += 8) { // eight independent loads in flight; the additions stay in block order
                float q[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) q[i] = partial[(b + i) * f.row_stride + e];
#pragma unroll
                for (int i = 0; i < 8; ++i) acc += (double)q[i];
            }
            for (; b < b1; ++b) acc += (double)partial[b * f.row_stride + e];
        }
        red[part][el] = acc;
    }
    __syncthreads();
    if (threadIdx.x < 32 && e < f.stride) {
        double s = 0.0;
        for (int q = 0; q < 32; ++q) s += red[q][el];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (e >= dst.begin[q] && e < dst.begin[q + 1] && dst.ptr[q]) dst.ptr[q][e - dst.begin[q]] = (float)s;
        if (e >= dst.begin[3] && e < dst.begin[4] && dst.copy) dst.copy[e - dst.begin[3]] = (float)s;
    }
}

int launch_final_sum(const FinalWork &f, int batch, hipStream_t stream); // dense.hip

} // namespace slicegcn

#endif
