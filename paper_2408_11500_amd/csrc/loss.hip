// Mean softmax cross-entropy over all nodes and its gradient: the paper's loss equation with every
// node labelled,  loss = -(1/n) sum_v log softmax(logits[v, :])[y_v],
// dlogits[v, j] = (softmax(logits[v, :])[j] - [j == y_v]) / n.
//
// One 16-lane group per row.  Up to 64 classes a row lives in four registers per lane and is read once, four rows of a group at a time;
// wider rows are swept three times (maximum, sum of exponentials, gradient), the second and third time from L1/L2.  Row losses are added
// per workgroup (64 rows) in fp64 in a fixed order, and a single-workgroup kernel adds the workgroup sums in fp64 in a fixed order: no
// floating-point atomics, bitwise reproducible.  A label outside [0, c) cannot be reported to the
// host without a synchronisation, so it poisons the result instead: the loss becomes NaN.
#include "common.h"

namespace slicegcn {

namespace {

constexpr int CE_LPR = 16;                // lanes per row
constexpr int CE_ROWS = 256 / CE_LPR;     // rows per workgroup pass
constexpr int CE_ROWS_PER_BLOCK = 4 * CE_ROWS; // each group handles four rows

// Sum of a workgroup's row losses, in row order
__device__ inline void ce_store_partial(const double *row_loss, double *__restrict__ partial)
{
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
#pragma unroll 16
        for (int i = 0; i < CE_ROWS_PER_BLOCK; ++i) s += row_loss[i];
        partial[blockIdx.x] = s;
    }
}

// logits and dlogits may be the same buffer (gradient in place), so neither is declared restrict: every
// read of a row element, the label's logit included, precedes in program order the store that replaces it.
//
// At most 64 classes.  VEC: rows on 16-byte boundaries, c % 4 == 0: a lane holds columns 4 sub to 4 sub + 3 from one load; else columns
// sub + 16 i.  All loads of a group's four rows are requested before the first is used (rows past the end re-read the last): bound by
// bytes on many rows and by one chain of loads on few.  With the
// final sum, and a kernel that took the rows in turn: 2.4 M rows of 47 218 us (519), 169 k rows of 41 22 (35), 2048 rows of 8 6.9 (9.1).
template <bool VEC, int R>
__global__ __launch_bounds__(256) void softmax_ce_rows_kernel(const float *logits, int64_t ld, int64_t n, int32_t c,
                                                              const int32_t *__restrict__ labels, float *dlogits,
                                                              int64_t ldd, double *__restrict__ partial)
{
    __shared__ double row_loss[CE_ROWS_PER_BLOCK];
    const int grp = threadIdx.x / CE_LPR, sub = threadIdx.x % CE_LPR, lane0 = threadIdx.x & 48; // first lane of the group in its wavefront
    const float inv_n = 1.0f / (float)n;
    auto col = [&](int i) { return VEC ? 4 * sub + i : sub + CE_LPR * i; };
    static_assert(!VEC || R == 4, "a load of four columns");
    float x[4][R];
    int label[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t v = (int64_t)blockIdx.x * CE_ROWS_PER_BLOCK + q * CE_ROWS + grp, row = v < n ? v : n - 1;
        const float *p = logits + row * ld;
        label[q] = labels[row];
        if constexpr (VEC) {
            const float4 w = *reinterpret_cast<const float4 *>(p + (col(0) < c ? col(0) : 0));
            x[q][0] = w.x; x[q][1] = w.y; x[q][2] = w.z; x[q][3] = w.w;
        } else {
#pragma unroll
            for (int i = 0; i < R; ++i) x[q][i] = p[col(i) < c ? col(i) : c - 1];
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int local = q * CE_ROWS + grp;
        const int64_t v = (int64_t)blockIdx.x * CE_ROWS_PER_BLOCK + local;
        const bool bad = label[q] < 0 || label[q] >= c;
        const int y = bad ? 0 : label[q];
        float m = -INFINITY, mine = 0.f, e[R];
#pragma unroll
        for (int i = 0; i < R; ++i) {
            if (col(i) >= c) x[q][i] = -INFINITY;
            m = fmaxf(m, x[q][i]);
            if ((VEC ? y % 4 : y / CE_LPR) == i) mine = x[q][i];
        }
        const float at_label = __shfl(mine, lane0 + (VEC ? y / 4 : y % CE_LPR), 64);
#pragma unroll
        for (int s = 1; s < CE_LPR; s <<= 1) m = fmaxf(m, __shfl_xor(m, s, 64));
#pragma unroll
        for (int i = 0; i < R; ++i) e[i] = col(i) < c ? expf(x[q][i] - m) : 0.f;
        float sum = e[0];
        if constexpr (VEC) {
            sum = (e[0] + e[1]) + (e[2] + e[3]);
        } else {
#pragma unroll
            for (int i = 1; i < R; ++i) sum += e[i];
        }
#pragma unroll
        for (int s = 1; s < CE_LPR; s <<= 1) sum += __shfl_xor(sum, s, 64);
        if (sub == 0) row_loss[local] = v >= n ? 0.0 : bad ? (double)NAN : (double)(m + logf(sum)) - (double)at_label;
        if (dlogits && v < n) {
            float *g = dlogits + v * ldd;
            const float inv_sum = 1.0f / sum;
            float d[R];
#pragma unroll
            for (int i = 0; i < R; ++i) d[i] = (e[i] * inv_sum - (col(i) == y ? 1.f : 0.f)) * inv_n;
            if constexpr (VEC) {
                if (col(0) < c) *reinterpret_cast<float4 *>(g + col(0)) = make_float4(d[0], d[1], d[2], d[3]);
            } else {
#pragma unroll
                for (int i = 0; i < R; ++i)
                    if (col(i) < c) g[col(i)] = d[i];
            }
        }
    }
    ce_store_partial(row_loss, partial);
}

// Any number of classes
__global__ __launch_bounds__(256) void softmax_ce_kernel(const float *logits, int64_t ld, int64_t n, int32_t c,
                                                         const int32_t *__restrict__ labels, float *dlogits,
                                                         int64_t ldd, double *__restrict__ partial)
{
    __shared__ double row_loss[CE_ROWS_PER_BLOCK];
    const int grp = threadIdx.x / CE_LPR, sub = threadIdx.x % CE_LPR;
    const float inv_n = 1.0f / (float)n;
    for (int q = 0; q < 4; ++q) {
        const int local = q * CE_ROWS + grp;
        const int64_t v = (int64_t)blockIdx.x * CE_ROWS_PER_BLOCK + local;
        double loss = 0.0;
        if (v < n) { // uniform within the 16-lane group
            const float *x = logits + v * ld;
            int y = labels[v];
            const bool bad = y < 0 || y >= c;
            if (bad) y = 0;
            float m = -INFINITY;
            for (int j = sub; j < c; j += CE_LPR) m = fmaxf(m, x[j]);
#pragma unroll
            for (int s = 1; s < CE_LPR; s <<= 1) m = fmaxf(m, __shfl_xor(m, s, 64));
            float sum = 0.f;
            for (int j = sub; j < c; j += CE_LPR) sum += expf(x[j] - m);
#pragma unroll
            for (int s = 1; s < CE_LPR; s <<= 1) sum += __shfl_xor(sum, s, 64);
            loss = bad ? (double)NAN : (double)(m + logf(sum)) - (double)x[y];
            if (dlogits) {
                float *g = dlogits + v * ldd;
                const float inv_sum = 1.0f / sum;
                for (int j = sub; j < c; j += CE_LPR) g[j] = (expf(x[j] - m) * inv_sum - (j == y ? 1.f : 0.f)) * inv_n;
            }
        }
        if (sub == 0) row_loss[local] = loss;
    }
    ce_store_partial(row_loss, partial);
}

// loss = (sum of the workgroup sums) / n, fp64, fixed order: thread t adds every 256th sum (eight requested at a time), then
// the sums of the threads that had one are added in thread order.
__global__ __launch_bounds__(256) void ce_final_kernel(const double *__restrict__ partial, int64_t n_blocks, int64_t n,
                                                       float *__restrict__ loss)
{
    __shared__ double red[256];
    double s = 0.0;
    int64_t b = threadIdx.x;
    for (; b + 7 * 256 < n_blocks; b += 8 * 256) {
        double p[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) p[i] = partial[b + i * 256];
#pragma unroll
        for (int i = 0; i < 8; ++i) s += p[i];
    }
    for (; b < n_blocks; b += 256) s += partial[b];
    red[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        const int threads = n_blocks < 256 ? (int)n_blocks : 256;
#pragma unroll 16
        for (int i = 0; i < threads; ++i) t += red[i];
        *loss = (float)(t / (double)n);
    }
}

inline int64_t ce_blocks(int64_t n) { return (n + CE_ROWS_PER_BLOCK - 1) / CE_ROWS_PER_BLOCK; }

} // namespace

} // namespace slicegcn

using namespace slicegcn;

extern "C" size_t slicegcn_softmax_ce_workspace_bytes(int64_t n)
{
    if (n < 1) return 0;
    return (size_t)round_up(ce_blocks(n) * (int64_t)sizeof(double), 256);
}

extern "C" int slicegcn_softmax_ce(const float *logits, int64_t ld, int64_t n, int32_t n_classes, const int32_t *labels,
                                   float *loss, float *dlogits, int64_t ldd, void *ws, size_t ws_bytes, void *stream_)
{
    SG_REQUIRE(logits && labels && loss, SLICEGCN_EINVAL, "softmax_ce: NULL logits, labels or loss");
    SG_REQUIRE(n >= 1 && n_classes >= 1, SLICEGCN_EINVAL, "softmax_ce: sizes must be >= 1");
    SG_REQUIRE(ld >= n_classes && (dlogits == nullptr || ldd >= n_classes), SLICEGCN_EINVAL,
               "softmax_ce: leading dimension smaller than the number of classes");
    const size_t need = slicegcn_softmax_ce_workspace_bytes(n);
    SG_REQUIRE(ws != nullptr && ws_bytes >= need, SLICEGCN_EWORKSPACE, "softmax_ce: workspace of %zu bytes, %zu needed",
               ws_bytes, need);
    SG_REQUIRE((reinterpret_cast<uintptr_t>(ws) & 255u) == 0, SLICEGCN_EINVAL, "softmax_ce: workspace not 256-byte aligned");
    hipStream_t stream = as_stream(stream_);
    const int64_t nb = ce_blocks(n);
    SG_REQUIRE(nb <= INT32_MAX, SLICEGCN_ERANGE, "softmax_ce: too many rows for one launch");
    double *partial = static_cast<double *>(ws);
    ProfScope prof(SLICEGCN_PROF_LOSS, n_classes, stream);
    const bool vec = n_classes % 4 == 0 && ld % 4 == 0 && aligned16(logits) && (dlogits == nullptr || (ldd % 4 == 0 && aligned16(dlogits)));
    if (n_classes > 64) softmax_ce_kernel<<<(unsigned)nb, 256, 0, stream>>>(logits, ld, n, n_classes, labels, dlogits, ldd, partial);
    else if (vec) softmax_ce_rows_kernel<true, 4><<<(unsigned)nb, 256, 0, stream>>>(logits, ld, n, n_classes, labels, dlogits, ldd, partial);
    else if (n_classes <= CE_LPR) softmax_ce_rows_kernel<false, 1><<<(unsigned)nb, 256, 0, stream>>>(logits, ld, n, n_classes, labels, dlogits, ldd, partial);
    else softmax_ce_rows_kernel<false, 4><<<(unsigned)nb, 256, 0, stream>>>(logits, ld, n, n_classes, labels, dlogits, ldd, partial);
    SG_LAUNCH_CHECK();
    ce_final_kernel<<<1, 256, 0, stream>>>(partial, nb, n, loss);
    SG_LAUNCH_CHECK();
    return SLICEGCN_OK;
}
