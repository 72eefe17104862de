// Dense half of a SliceGCN layer (the layer equation's weight products, bias, ReLU and self
// term) and of its backward pass, plus the layer entry points that chain it with the
// aggregation kernels.
//
//   forward :  Hout = act(Z W_agg + b) + Hin W_self + b_self,  mask = [P > 0] bit-packed
//   backward:  dZ = (dHout * mask) W_agg^T,  T = dHout W_self^T            (pair kernel, transposed)
//              dW_agg = Z^T (dHout * mask), dW_self = Hin^T dHout, db, db_self   (reduce kernels)
//
// All products run on v_mfma_f32_32x32x2_f32 tiles (fp32 in, fp32 accumulate), one 32-row strip per wavefront.
// Lane layout of the 32x32x2 fp32 MFMA (64 lanes, l = lane): A operand = A[m = l % 32][k = l / 32],
// B operand = B[k = l / 32][n = l % 32], accumulator register r (0..15) = C[8*(r/4) + 4*(l/32) + r%4][l % 32].
#include "common.h"
#include "final_sum.h"
#include "wide_rules.h"

#include <type_traits>

namespace slicegcn {

namespace {

struct PairArgs {
    const float *A1; int64_t lda1; // forward: Z          backward: dHout (masked on load)
    const float *A2; int64_t lda2; // forward: Hin        backward: dHout           (NULL: no second product)
    const float *B1;               // W_agg  (w_in x w_out row-major)
    const float *B2;               // W_self (same shape) or NULL
    const float *bias1;            // forward only
    const float *bias2;            // forward only
    const float *enc = nullptr;    // forward only: second summand of the outer bias (slice encoding)
    float *O1; int64_t ldo1;       // forward: Hout       backward: dZ
    float *O2; int64_t ldo2;       // backward: T (may be NULL)
    uint32_t *mask; int64_t mask_words; // forward: written (act = ReLU); backward: read
    int64_t n;
    int32_t K;     // reduction length: w_in forward, w_out backward
    int32_t Nout;  // output width:     w_out forward, w_in backward
    int32_t ldw;   // leading dimension of W (= w_out)
    int32_t act;
    // Scaled layout (activations stored as D~^-1/2 H, the operand form the aggregation wants): per-row factors.
    const float *scale2 = nullptr;   // forward: rows of A2 are multiplied by scale2[row] when read (sqrt(d~): undoes the scaling of Hin)
    const float *scale_o1 = nullptr; // rows of O1 are multiplied by scale_o1[row] (forward: on store; backward: dZ rows, folded into dP)
};

// The same products for a batch of slice models (equal shapes and leading dimensions): grid row y works on slice y, with
// the pointers taken from here.  Small graphs need it: their kernels last microseconds and fill a fraction of the chip.
constexpr int BATCH = SPMM_BATCH;
// From so many rows of all slices of a launch on, layers up to 64 wide take a strip kernel (64 -> 64 with self term, strips / pair_rows_kernel:
// four slices of 66 k rows forward 75 / 71 us, backward 69 / 78; of 169 k rows 149 / 157 and 130 / 172).
constexpr int64_t STRIP64_ROWS = 262144;
struct PairPtrs {
    const float *A1, *A2, *B1, *B2, *bias1, *bias2, *enc;
    float *O1, *O2;
    uint32_t *mask;
};
struct PairBatch { PairPtrs p[BATCH]; };
__device__ inline PairArgs slice_of(const PairArgs &common, const PairBatch &b)
{
    PairArgs a = common;
    const PairPtrs &p = b.p[blockIdx.y];
    a.A1 = p.A1; a.A2 = p.A2; a.B1 = p.B1; a.B2 = p.B2; a.bias1 = p.bias1; a.bias2 = p.bias2; a.enc = p.enc;
    a.O1 = p.O1; a.O2 = p.O2; a.mask = p.mask;
    return a;
}
// Biases of output column col: inside the activation, and outside it (the encoding joins the outer one; with a single
// product there is no outer part and it joins the only one)
template <bool TWO> __device__ inline float inner_bias(const PairArgs &a, int col)
{
    return (a.bias1 ? a.bias1[col] : 0.f) + (!TWO && a.enc ? a.enc[col] : 0.f);
}
__device__ inline float outer_bias(const PairArgs &a, int col) { return (a.bias2 ? a.bias2[col] : 0.f) + (a.enc ? a.enc[col] : 0.f); }

__device__ inline void scale4(float4 &v, float s) { v.x *= s; v.y *= s; v.z *= s; v.w *= s; }

// base + count for a base that is the same for the wavefront and count < 2^30, by an access's own 32-bit offset
template <class T> __device__ __forceinline__ const T *plus(const T *base, uint32_t count)
{
    return reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + count * 4u);
}
// The same number, as far as the compiler knows a new one: an offset that does not change in a loop has its extension to 64 bits moved out of
// it, and then every access adds it to its base per lane
__device__ __forceinline__ uint32_t fresh(uint32_t v)
{
    asm volatile("" : "+v"(v));
    return v;
}

typedef float floatx16 __attribute__((ext_vector_type(16)));

// The halves of `bits`, which is the same for the wavefront, into lanes lo and hi (constants) of v.  One instruction each; chosen per lane, with the lanes'
// conditions in scalar registers, it is five and a branch.  (The instructions read a scalar register that a vector compare may have
// just written: two wait states.)
__device__ __forceinline__ void set_lanes(uint32_t &v, unsigned long long bits, int lo, int hi)
{
    asm("s_nop 1\n\tv_writelane_b32 %0, %1, %3\n\tv_writelane_b32 %0, %2, %4" : "+v"(v) : "s"((uint32_t)bits), "s"((uint32_t)(bits >> 32)), "n"(lo), "n"(hi));
}

// Four floats of row `row` starting at column k (k % 4 == 0), zero beyond column K.
__device__ inline float4 load_k4(const float *__restrict__ base, int64_t ld, int64_t row, int k, int K, bool vec_ok)
{
    const float *p = base + row * ld + k;
    if (vec_ok && k + 4 <= K) return *reinterpret_cast<const float4 *>(p);
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (k < K) v.x = p[0];
    if (k + 1 < K) v.y = p[1];
    if (k + 2 < K) v.z = p[2];
    if (k + 3 < K) v.w = p[3];
    return v;
}

__device__ inline float pick(const float4 &v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx4_u __attribute__((ext_vector_type(4), aligned(4))); // 16-byte accesses at any 4-byte boundary

// Workgroup b of a grid of row tiles x column tiles (1-D, 8 row tiles x all column tiles per group of workgroups): the column
// tiles of one row tile run back to back on the same XCD (workgroup b goes to XCD b mod 8), so the rows are fetched from memory
// once and re-read from L2.  The last group of 8 row tiles may be partial.
// (In 32 bits: a 64-bit division is as long as a small layer's loads.)
struct TilePlace { uint32_t row_tile, col_tile; };
__device__ inline TilePlace tile_place(uint32_t b, uint32_t n_col_tiles)
{
    const uint32_t group = b / (8 * n_col_tiles);
    return TilePlace{group * 8 + b % 8, b / 8 - group * n_col_tiles};
}

// Four consecutive columns per lane and register group of a 32-column tile to row `o` (+ 4 * h + 8 * q); `width` columns exist from
// the tile's first one on
__device__ inline void store_tile_row(const floatx16 &c, float *o, int h, int width, float f)
{
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int at = 8 * q + 4 * h, left = width - at;
        if (width >= 32 || left >= 4) { // the first test is the same for the whole workgroup
            floatx4_u v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = c[4 * q + i] * f;
            *reinterpret_cast<floatx4_u *>(o + at) = v;
        } else {
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (i < left) o[at + i] = c[4 * q + i] * f;
        }
    }
}

// Four columns of a row from column c on, `left` of which exist; WHOLE: all four, of a row that exists
template <bool WHOLE> __device__ inline void store_cols4(float *o, const float4 &v, bool row_ok, int left)
{
    if (WHOLE || (row_ok && left >= 4)) {
        const floatx4_u w = {v.x, v.y, v.z, v.w};
        *reinterpret_cast<floatx4_u *>(o) = w;
    } else if (row_ok) {
        if (left > 0) o[0] = v.x;
        if (left > 1) o[1] = v.y;
        if (left > 2) o[2] = v.z;
    }
}

// Products of every layer the strip kernels do not take.  Forward: Hout = act(Z W_agg + b) + Hin W_self + b_self; backward: dZ = (dHout *
// mask) W_agg^T, then T = dHout W_self^T over the same accumulators.  Workgroup = 4 wavefronts; a wavefront owns 32 rows and all
// NT * 32 columns of the workgroup's tile.  A row is used by one wavefront only, so it goes from memory straight into
// registers (a lane loads the k of its row that it feeds to the matrix cores, the next chunk's while the current one is
// multiplied).  The weights are shared and go through LDS: 32 steps of k at a time, two buffers, one barrier per chunk, in units of
// four k of a column, so that a 16-byte read feeds four instructions.  The weights are the A operand and the rows the B operand:
// a lane then holds four consecutive columns of one row in four registers, stores them as 16 bytes and collects the
// activation bits of its row without votes.
// The order is that of the strip kernels: chains over all of k, a step takes k and k + 4, one chain per product (for the row factor of dZ see
// scale_operand there).  Whether an
// activation passes depends on the last bit of its sum where that is near zero (a few in 10^8), and then a row's gradient changes
// by a whole term: every kernel and size gives the same bits for the same operands.  (Operands split into three bf16
// terms on the bf16 matrix cores were as exact against fp64 and faster, 2.4 M rows 256 -> 256 2.16 ms, but rounded differently.)
// Bound by the matrix cores when wide: 2.4 M rows 256 -> 256 2.93 ms = 110 TFLOP/s (a kernel with rows and weights in LDS: 3.71), 169 k rows
// 0.238 (0.288); slice layers 64 -> 64 with self term, 169 k rows: 47 us (61).  A last chunk ends with its steps, in eights (before, all 32 were
// multiplied: input gradients of 169 k rows 256 -> 40 80 -> 68 us, 2.4 M rows 256 -> 47 1.25 -> 1.15 ms; 100 k rows 200 -> 200 131 -> 122 us).
template <int NT, bool TWO, bool BWD>
__device__ __forceinline__ void pair_rows_tile(const PairArgs &a, uint32_t wg, int n_col_tiles)
{
    constexpr int BN = NT * 32, KC = 32, GS = BN + 4; // GS: units per group of four k (padded: conflict-free writes and reads)
    constexpr int TS = 36; // row stride of a wavefront's output tile
    constexpr int POOL = 2 * (KC / 4) * GS > 4 * 32 * TS / 4 ? 2 * (KC / 4) * GS : 4 * 32 * TS / 4;
    __shared__ floatx4 pool[POOL]; // the weights; behind the last chunk the output tiles
    floatx4 (*Bs)[KC / 4][GS] = reinterpret_cast<floatx4 (*)[KC / 4][GS]>(pool);
    __shared__ __attribute__((aligned(16))) float bias_s[2][BN];
    const int tid = threadIdx.x;
    // In a scalar register it leaves four vector registers more, without which three tiles of an input gradient spill two (169 k rows 288 -> 40
    // 69.8 -> 66.8 us, 800 k rows 326 -> 312); with one tile it was slower (20 k rows 32 -> 256 11.1 -> 11.9).
    const int wave = NT == 3 && BWD && !TWO ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6, lane = tid & 63;
    const int m = lane & 31, h = lane >> 5;
    const TilePlace place = tile_place(wg, n_col_tiles);
    const int64_t row_tile = place.row_tile;
    const int col0 = (int)place.col_tile * BN;
    if (row_tile * 128 >= a.n) return; // uniform per workgroup
    const int chunks = (a.K + KC - 1) / KC, total = TWO ? 2 * chunks : chunks;

    // biases of this thread's column: requested here, added and put into LDS behind the first chunk's requests
    float in_b = 0.f, out_b = 0.f, enc_b = 0.f;
    if (!BWD) {
        const int col = col0 + (tid < BN ? tid : 0), c = col < a.Nout ? col : a.Nout - 1;
        in_b = a.bias1 ? a.bias1[c] : 0.f;
        if (TWO) out_b = a.bias2 ? a.bias2[c] : 0.f;
        enc_b = a.enc ? a.enc[c] : 0.f;
    }
    // The row this lane feeds.  Rows past the end and columns past the last one re-read the last: what they give is not
    // stored.  Steps of k past K are zero in both operands.
    const int64_t my_row = row_tile * 128 + wave * 32 + m, row = my_row < a.n ? my_row : a.n - 1;
    const float *in_scale = BWD ? a.scale_o1 : TWO ? a.scale2 : nullptr; // factor on the rows of one of the products:
    const float f_in = in_scale ? in_scale[row] : 1.f;                   // dZ rows; rows of Hin kept scaled
    const uint32_t *src_words = BWD && a.mask ? a.mask + row * a.mask_words : nullptr;

    floatx4 next[KC / 8];
    uint32_t next_word = ~0u; // backward: activation bits of the next chunk
    const float *src = nullptr;
    auto fetch_rows = [&](int cc) {
        const bool second = TWO && cc >= chunks;
        const int c = second ? cc - chunks : cc, k0 = c * KC;
        if (c == 0) src = (second ? a.A2 + row * a.lda2 : a.A1 + row * a.lda1) + 4 * h; // first chunk of a product
        if (k0 + KC <= a.K) {
#pragma unroll
            for (int q = 0; q < KC / 8; ++q) next[q] = *reinterpret_cast<const floatx4_u *>(src + k0 + 8 * q);
        } else {
#pragma unroll
            for (int q = 0; q < KC / 8; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) next[q][i] = k0 + 8 * q + 4 * h + i < a.K ? src[k0 + 8 * q + i] : 0.f;
        }
        if (BWD && src_words) next_word = second ? ~0u : src_words[c];
    };
    // This thread's weights of the next chunk.  Unit u: consecutive threads walk the contiguous axis of W (columns forward, groups of
    // four k backward)
    floatx4 rw[NT];
    auto unit_g = [&](int u) { return BWD ? u & 7 : u / BN; };
    auto unit_c = [&](int u) { return BWD ? u >> 3 : u % BN; };
    auto fetch_weights = [&](int cc) {
        const bool second = TWO && cc >= chunks;
        const int k0 = (second ? cc - chunks : cc) * KC;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int u = tid + 256 * j, c = col0 + unit_c(u), k = k0 + 4 * unit_g(u), col = c < a.Nout ? c : a.Nout - 1;
            const int64_t step = BWD ? 1 : a.ldw;
            const float *p = (second ? a.B2 : a.B1) + (BWD ? (int64_t)col * a.ldw + k : (int64_t)k * a.ldw + col);
            if (k0 + KC <= a.K) {
                if constexpr (BWD) {
                    rw[j] = *reinterpret_cast<const floatx4_u *>(p);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) rw[j][i] = p[i * step];
                }
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) rw[j][i] = k + i < a.K ? p[i * step] : 0.f;
            }
        }
    };
    auto stash_weights = [&](int buf) {
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int u = tid + 256 * j;
            Bs[buf][unit_g(u)][unit_c(u)] = rw[j];
        }
    };

    floatx16 acc[NT], first[TWO && !BWD ? NT : 1]; // first: the activated first product
    auto clear = [&]() {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
    };
    // register r of lane (m, h): column 8 * (r / 4) + 4 * h + r % 4 of tile t
    auto activate = [&](floatx16 &c, int t) { // end of the first forward product: bias, activation and its bits
        uint32_t bits = 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 b1 = *reinterpret_cast<const float4 *>(&bias_s[0][32 * t + 8 * q + 4 * h]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float p = c[4 * q + i] + pick(b1, i);
                if (a.act == SLICEGCN_ACT_RELU) {
                    if (p > 0.f) bits |= 1u << (8 * q + i);
                    else p = 0.f;
                }
                c[4 * q + i] = p;
            }
        }
        if (a.act == SLICEGCN_ACT_RELU) {
            const int left = a.Nout - col0 - 32 * t; // columns of this word
            bits <<= 4 * h;
            bits |= __shfl_xor(bits, 32, 64);
            if (left < 32) bits &= left > 0 ? (1u << left) - 1u : 0u;
            if (h == 0 && my_row < a.n && left > 0) a.mask[row * a.mask_words + ((col0 >> 5) + t)] = bits;
        }
    };
    auto store_all = [&](float *O, int64_t ldo, float f) {
        if (my_row >= a.n) return;
#pragma unroll
        for (int t = 0; t < NT; ++t) store_tile_row(acc[t], O + row * ldo + col0 + 32 * t, h, a.Nout - col0 - 32 * t, f);
    };
    // Behind the last chunk: through LDS, so that a row of a tile goes out as eight 16-byte stores of one instruction (from the accumulators
    // an instruction stores 32 bytes to each of 32 rows, which takes the CU's L1 64 cycles instead of 16: 2.4 M rows 47 -> 256 1.23 -> 1.02 ms,
    // 256 -> 256 3.03 -> 2.93, 169 k rows 40 -> 256 87 -> 68 us).  In a tile that is not full the lane at a row's end stores the row's last
    // four columns, some of them once more, and below four columns a lane stores a row: no branches per lane and store (2.4 M rows 12 -> 44 213 -> 153 us, 256 -> 47
    // 872 -> 830, 70 -> 7 213 -> 191, 160 -> 3 334 -> 317; input gradients 197 -> 143, 848 -> 819, 236 -> 216, 349 -> 335).
    auto store_last = [&](float *O, int64_t ldo, float f) {
        float (*tile)[TS] = reinterpret_cast<float (*)[TS]>(pool) + 32 * wave;
        const int lr = lane >> 3, lc = (lane & 7) * 4;
        const int64_t row0 = row_tile * 128 + wave * 32;
        constexpr bool ROW_PER_LANE = !(NT == 3 && BWD && !TWO); // (it would spill two registers there)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int left = a.Nout - col0 - 32 * t;
            if (left <= 0) break; // uniform
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                floatx4 v;
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = acc[t][4 * q + i] * f;
                *reinterpret_cast<floatx4 *>(&tile[m][8 * q + 4 * h]) = v;
            }
            __builtin_amdgcn_wave_barrier();
            float *o = O + (row0 + lr) * ldo + col0 + 32 * t + lc;
            if (row0 + 32 <= a.n && left >= 32) { // uniform per wavefront
#pragma unroll
                for (int it = 0; it < 4; ++it) store_cols4<true>(o + 8 * it * ldo, *reinterpret_cast<const float4 *>(&tile[lr + 8 * it][lc]), true, 32);
            } else if (row0 + 32 <= a.n && left >= 4) {
                const int back = lc > left - 4 ? lc - (left - 4) : 0;
                if (lc < left) {
#pragma unroll
                    for (int it = 0; it < 4; ++it)
                        *reinterpret_cast<floatx4_u *>(o + 8 * it * ldo - back) = *reinterpret_cast<const floatx4_u *>(&tile[lr + 8 * it][lc - back]);
                }
            } else if (ROW_PER_LANE && left < 4) {
                float *narrow = O + row * ldo + col0 + 32 * t;
#pragma unroll
                for (int c = 0; c < 4; c += 2)
                    if (my_row < a.n && c + h < left) narrow[c + h] = tile[m][c + h];
            } else {
#pragma unroll
                for (int it = 0; it < 4; ++it)
                    store_cols4<false>(o + 8 * it * ldo, *reinterpret_cast<const float4 *>(&tile[lr + 8 * it][lc]), row0 + lr + 8 * it < a.n, left - lc);
            }
            __builtin_amdgcn_wave_barrier();
        }
    };

    clear();
    fetch_weights(0);
    fetch_rows(0);
    if (!BWD && tid < BN) { // inside the activation, and outside it (the encoding joins the outer one; with a single product the only one)
        bias_s[0][tid] = in_b + (TWO ? 0.f : enc_b);
        bias_s[1][tid] = out_b + enc_b;
    }
    stash_weights(0);
    __syncthreads();
    for (int cc = 0; cc < total; ++cc) {
        const bool more = cc + 1 < total;
        if (more) fetch_weights(cc + 1);
        floatx4 x[KC / 8];
#pragma unroll
        for (int q = 0; q < KC / 8; ++q) x[q] = next[q];
        if (BWD && src_words) {
#pragma unroll
            for (int q = 0; q < KC / 8; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (!((next_word >> (8 * q + 4 * h + i)) & 1u)) x[q][i] = 0.f;
        }
        if (in_scale && (BWD ? cc < chunks : cc >= chunks)) {
#pragma unroll
            for (int q = 0; q < KC / 8; ++q) x[q] *= f_in;
        }
        if (more) fetch_rows(cc + 1);
        const int left = a.K - (TWO && cc >= chunks ? cc - chunks : cc) * KC; // steps of the product from this chunk on
        floatx4 w[2][NT]; // the weights of four steps are read while the four before them are multiplied
#pragma unroll
        for (int t = 0; t < NT; ++t) w[0][t] = Bs[cc & 1][h][32 * t + m];
#pragma unroll
        for (int q = 0; q < KC / 8; ++q) {
            // uniform; both operands are zero from here on (not with both products of a backward pass: it costs them 20 registers)
            if (!(TWO && BWD) && q > 0 && 8 * q >= left) break;
            if (q + 1 < KC / 8) {
#pragma unroll
                for (int t = 0; t < NT; ++t) w[(q + 1) & 1][t] = Bs[cc & 1][2 * (q + 1) + h][32 * t + m];
            }
            // (one tile of an input gradient: the compiler's own order is better, 221 k rows 16 <- 93 32.6 / 30.6 us, 2.4 M rows 327 / 318)
            if (!(NT == 1 && BWD && !TWO)) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[q & 1][t][i], x[q][i], acc[t], 0, 0, 0);
        }
        if (more) stash_weights((cc + 1) & 1); // the buffer of the chunk before this one, which every wavefront has left
        __syncthreads();
        if (TWO && cc == chunks - 1) { // end of the first product
            if constexpr (BWD) {
                store_all(a.O1, a.ldo1, 1.f);
            } else {
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    activate(acc[t], t);
                    first[TWO && !BWD ? t : 0] = acc[t];
                }
            }
            clear();
        }
    }
    if constexpr (BWD) {
        if (!TWO) store_last(a.O1, a.ldo1, 1.f);
        else if (a.O2) store_last(a.O2, a.ldo2, 1.f);
    } else {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            if constexpr (TWO) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 b2 = *reinterpret_cast<const float4 *>(&bias_s[1][32 * t + 8 * q + 4 * h]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[t][4 * q + i] = first[t][4 * q + i] + (acc[t][4 * q + i] + pick(b2, i));
                }
            } else {
                activate(acc[t], t);
            }
        }
        store_last(a.O1, a.ldo1, a.scale_o1 ? a.scale_o1[row] : 1.f);
    }
}
template <int NT, bool TWO, bool BWD>
__global__ __launch_bounds__(256, NT == 4 || (TWO && NT == 3) ? 2 : 3) void pair_rows_kernel(const PairArgs common, const PairBatch batch, int n_col_tiles, unsigned first)
{
    pair_rows_tile<NT, TWO, BWD>(slice_of(common, batch), blockIdx.x + first, n_col_tiles);
}

// Products of wide layers on many rows, one at a time.  What bounded pair_rows_kernel there was waiting: fp32 matrix instructions take the vector
// pipe, so nothing but other matrix instructions fills a wait, and a workgroup asked for its next 32 steps of rows and weights when the
// current ones began, 0.9 us ahead.  Here a workgroup stays for the whole launch, one per CU and of eight wavefronts, with all of its columns'
// weights in LDS (up to 128 KB; no barrier behind the first), and a wavefront keeps the next R chunks of its rows in flight
// across the ends of its strips of 32 rows.  No memory access of the loop depends on a branch that another path does not match, so that the
// compiler's waits are for the chunk in turn: past the last row the last one is read and stored again, a product's chunks are padded to
// a multiple of R by reading the last one again (no instruction is issued for these).  The column tiles of a strip are worked on at about the same time on the
// same XCD.  The order of the sums is that of pair_rows_kernel: the same bits.
// Bound by the matrix instructions and, under their load, by a clock of about 2.2 GHz (143 TFLOP/s): 1 M rows 256 -> 256 are 81 % of its cycles, other
// vector instructions 6 %.  rows / wide, forward and input gradients with a mask: 2.4 M rows 256 -> 256 3.09 / 2.73 and 3.17 / 2.69 ms, 256 -> 47
// 846 / 750 and 1087 / 785 us, 800 k 200 -> 200 844 / 725 and 876 / 711, 66 k 512 -> 512 336 / 290 and 327 / 298, 169 k 40 -> 256 67.6 / 57.4; both input
// gradients of two slices of 233 k rows 128 <- 128 355 / 307.
template <int NT, int R, bool RAGGED, bool BWD> // RAGGED: K is no multiple of 32
__global__ __launch_bounds__(64 * WIDE_WAVES, 2) void pair_wide_kernel(const PairArgs common, const PairBatch batch, int n_tiles, int walkers)
{
    constexpr int BN = NT * 32, KC = WIDE_CHUNK, TS = 36;
    __shared__ floatx4 Bs[wide_groups(wide_k(NT))][BN]; // units of four k of a column
    __shared__ __attribute__((aligned(16))) float tiles[WIDE_WAVES][16][TS];
    __shared__ __attribute__((aligned(16))) float bias_s[BN];
    const PairArgs a = slice_of(common, batch);
    const int tid = threadIdx.x, lane = tid & 63, m = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroup b runs on XCD b mod 8: the column tiles of a walker are neighbours there
    const int slot = blockIdx.x / 8, tile = slot % n_tiles, walker = slot / n_tiles * 8 + blockIdx.x % 8;
    const int col0 = tile * BN, K = a.K;
    const int chunks = (K + KC - 1) / KC, padded = (chunks + R - 1) / R * R;
    const int64_t n = a.n, strips = (n + 31) / 32, stride = (int64_t)walkers * WIDE_WAVES;
    const int64_t first = (int64_t)wave * walkers + walker; // a last, partial turn goes to the first wavefronts of many workgroups
    const bool masked = BWD && a.mask != nullptr;
    const uint32_t lda = (uint32_t)a.lda1, ldm = BWD && !masked ? 0 : (uint32_t)a.mask_words;
    const uint32_t *words = masked ? a.mask : reinterpret_cast<const uint32_t *>(a.A1);

    // chunk c of strip s; a lane loads the k of its row that it feeds to the matrix cores: 8 q + 4 h + i
    floatx4 ring[R][KC / 8];
    uint32_t ring_word[R];
    auto load = [&](floatx4 (&x)[KC / 8], uint32_t &word, int64_t s, int c) {
        if (c >= chunks) c = chunks - 1;
        const int64_t row0 = s * 32;
        uint32_t r = m;
        if (row0 + 32 > n) r = (uint32_t)min((int64_t)m, n - 1 - row0); // uniform
        const float *p = a.A1 + row0 * (int64_t)lda;
        const uint32_t off = r * lda + c * KC + 4 * h;
#pragma unroll
        for (int q = 0; q < KC / 8; ++q) { // nothing behind the row is read: moved into place where it is used
            const int over = RAGGED ? max(c * KC + 8 * q + 4 * h + 4 - K, 0) : 0;
            x[q] = *reinterpret_cast<const floatx4_u *>(plus(p, off + 8 * q - over));
        }
        if (BWD) word = *plus(words + row0 * (int64_t)ldm, masked ? r * ldm + c : 0u);
    };
    auto factor_of = [&](int64_t s) { return BWD && a.scale_o1 ? a.scale_o1[min(s * 32 + m, n - 1)] : 1.f; }; // of the row this lane feeds
    float next_f = first < strips ? factor_of(first) : 1.f;
    if (first < strips) {
#pragma unroll
        for (int j = 0; j < R; ++j) load(ring[j], ring_word[j], first, j);
    }

    // Units of four k of a column; zero past K.  Consecutive threads walk the contiguous axis of W (columns forward, groups of four k backward),
    // and eight units of a thread are requested before the first is stored.
    const int groups = (K + 7) / 8 * 2, units = wide_groups(K) * BN;
    for (int u0 = tid; u0 < units; u0 += 8 * 64 * WIDE_WAVES) {
        floatx4 w[8];
        auto group_of = [&](int u) { return BWD ? (u & 7) + u / (8 * BN) * 8 : u / BN; };
        auto column_of = [&](int u) { return BWD ? (u >> 3) % BN : u % BN; };
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int u = u0 + 64 * WIDE_WAVES * j, k = 4 * group_of(u), col = min(col0 + column_of(u), a.Nout - 1);
            const int64_t step = BWD ? 1 : a.ldw;
            const float *p = a.B1 + (BWD ? (int64_t)col * a.ldw : col);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float v = p[min(k + i, K - 1) * step];
                w[j][i] = k + i < K ? v : 0.f;
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int u = u0 + 64 * WIDE_WAVES * j;
            if (group_of(u) < groups) Bs[group_of(u)][column_of(u)] = w[j];
        }
    }
    if (!BWD && tid < BN) bias_s[tid] = inner_bias<false>(a, col0 + tid < a.Nout ? col0 + tid : a.Nout - 1);
    __syncthreads();

    float (*out)[TS] = tiles[wave];
    const int lr = lane >> 3, lc = (lane & 7) * 4;
    const floatx4 *w_first = &Bs[h][m];
    floatx4 w[2][NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) w[0][t] = w_first[32 * t];
    for (int64_t s = first; s < strips; s += stride) {
        const int64_t next = s + stride < strips ? s + stride : s;
        const float f = next_f;
        next_f = factor_of(next);
        floatx16 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
        for (int c0 = 0; c0 < padded; c0 += R) {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int c = c0 + j, left = K - c * KC; // steps from this chunk on
                if (left > 0) { // uniform; no access to memory in here
                    floatx4 (&x)[KC / 8] = ring[j];
                    if (RAGGED && left < KC) {
#pragma unroll
                        for (int q = 0; q < KC / 8; ++q) {
                            const int over = 8 * q + 4 * h + 4 - left; // columns the load was moved back by
                            const bool one = over & 1, two = over & 2, none = over >= 4, any = over > 0;
                            const float y0 = one ? x[q][1] : x[q][0], y1 = one ? x[q][2] : x[q][1], y2 = one ? x[q][3] : x[q][2], y3 = one ? 0.f : x[q][3];
                            const floatx4 z = {two ? y2 : y0, two ? y3 : y1, two ? 0.f : y2, two ? 0.f : y3};
#pragma unroll
                            for (int i = 0; i < 4; ++i) x[q][i] = none ? 0.f : any ? z[i] : x[q][i];
                        }
                    }
                    if (masked) {
                        const int word = (int)(ring_word[j] >> (4 * h));
#pragma unroll
                        for (int q = 0; q < KC / 8; ++q)
#pragma unroll
                            for (int i = 0; i < 4; ++i) // a bit extended to a word
                                x[q][i] = __int_as_float(__float_as_int(x[q][i]) & __builtin_amdgcn_sbfe(word, 8 * q + i, 1));
                    }
                    if (BWD && a.scale_o1) { // uniform
                        asm volatile(""); // (a branch)
#pragma unroll
                        for (int q = 0; q < KC / 8; ++q) x[q] *= f;
                    }
                    const floatx4 *w_at = w_first + c * (KC / 4) * BN;
#pragma unroll
                    for (int q = 0; q < KC / 8; ++q) { // the weights of four steps are read while the four before them are multiplied
                        if (RAGGED && q > 0 && 8 * q >= left) break; // uniform: both operands are zero from here on
                        const floatx4 *w_next = wide_more(left, q) ? w_at + 2 * (q + 1) * BN : w_first;
                        if (!RAGGED || q + 1 < KC / 8 || left >= KC) {
#pragma unroll
                            for (int t = 0; t < NT; ++t) w[(q + 1) & 1][t] = w_next[32 * t];
                        }
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int i = 0; i < 4; ++i)
#pragma unroll
                            for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[q & 1][t][i], x[q][i], acc[t], 0, 0, 0);
                    }
                    if (RAGGED && left < KC) { // the next strip's first
#pragma unroll
                        for (int t = 0; t < NT; ++t) w[0][t] = w_first[32 * t];
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                const bool over = c + R >= padded; // uniform
                load(ring[j], ring_word[j], over ? next : s, over ? c + R - padded : c + R);
                __builtin_amdgcn_sched_barrier(0);
            }
        }

        const int64_t row0 = s * 32;
        const bool full = row0 + 32 <= n; // uniform
        const int most = full ? 31 : (int)(n - 1 - row0); // last row of the strip
        const bool relu = !BWD && a.act == SLICEGCN_ACT_RELU;
        uint32_t bits[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int left = a.Nout - col0 - 32 * t;
            if (!BWD) { // bias, activation and its bits; register r of lane (m, h): column 8 * (r / 4) + 4 * h + r % 4
                float4 bias[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) bias[q] = *reinterpret_cast<const float4 *>(&bias_s[32 * t + 8 * q + 4 * h]);
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[t][r] += pick(bias[r / 4], r % 4);
                if (relu) { // uniform
                    uint32_t b = 0u;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const bool on = acc[t][r] > 0.f;
                        b |= (uint32_t)on << (8 * (r / 4) + r % 4);
                        acc[t][r] = on ? acc[t][r] : 0.f;
                    }
                    b <<= 4 * h;
                    b |= __shfl_xor(b, 32, 64);
                    if (left < 32) b &= left > 0 ? (1u << left) - 1u : 0u;
                    bits[t] = b;
                }
            }
            if (left <= 0) break; // uniform
            // through LDS, half of the rows at a time, so that a row of a tile goes out as eight 16-byte stores of one instruction; in a tile
            // that is not full the lanes at a row's end store its last four columns again
            const int back = left < 32 && lc > left - 4 ? lc - (left - 4) : 0;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                if ((m >> 4) == half) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const floatx4 v = {acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]};
                        *reinterpret_cast<floatx4 *>(&out[m & 15][8 * q + 4 * h]) = v;
                    }
                }
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    const int r = 16 * half + 8 * it + lr;
                    floatx4 v;
                    if (left >= 32) v = *reinterpret_cast<const floatx4 *>(&out[8 * it + lr][lc]); // uniform
                    else v = *reinterpret_cast<const floatx4_u *>(&out[8 * it + lr][lc - back]);
                    float *o = a.O1 + row0 * a.ldo1 + col0 + 32 * t;
                    *reinterpret_cast<floatx4_u *>(o + (int)((uint32_t)min(r, most) * (uint32_t)a.ldo1) + lc - back) = v;
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
        if (relu) {
            uint32_t *word = a.mask + row0 * (int64_t)ldm + (col0 >> 5) + (uint32_t)min(m, most) * ldm;
#pragma unroll
            for (int t = 0; t < NT; ++t)
                if (a.Nout - col0 - 32 * t > 0) word[t] = bits[t]; // both halves of the wavefront the same
        }
    }
}

// Four consecutive floats of an operand row as a strip kernel's lane loads them.  The lane that owns columns [c, c + 4) loads
// from column min(c, K - 4) on, so that nothing outside the row's K columns is read and no load depends on a branch: a loop of such loads
// and of unconditional stores has wait counts the compiler knows, and the next strip's loads and the last one's stores stay in flight (with
// a branch per row it waited for every access at the top of the loop).  What a tail lane loaded is moved into place, and zeroed
// beyond K, where it is used.
// NARROW: rows that may have fewer than four columns, one float at a time.
template <bool NARROW = false> struct LaneCols {
    int at, shift; // first column loaded; columns to drop
    int last;      // NARROW: last column of the row
    __device__ LaneCols(int c, int K) : at(NARROW || c < K - 4 ? c : K - 4), shift(c - at), last(K - 1) {}
    __device__ float4 load(const float *row) const
    {
        if constexpr (NARROW) return make_float4(row[min(at, last)], row[min(at + 1, last)], row[min(at + 2, last)], row[min(at + 3, last)]);
        const floatx4_u v = *reinterpret_cast<const floatx4_u *>(row + at);
        return make_float4(v.x, v.y, v.z, v.w);
    }
    __device__ void place(float4 &v) const
    {
        if constexpr (NARROW) {
            v.x = at <= last ? v.x : 0.f;
            v.y = at + 1 <= last ? v.y : 0.f;
            v.z = at + 2 <= last ? v.z : 0.f;
            v.w = at + 3 <= last ? v.w : 0.f;
            return;
        }
        const bool one = shift & 1, two = shift & 2, none = shift >= 4;
        const float x = one ? v.y : v.x, y = one ? v.z : v.y, z = one ? v.w : v.z, w = one ? 0.f : v.w;
        v.x = none ? 0.f : two ? z : x;
        v.y = none ? 0.f : two ? w : y;
        v.z = none || two ? 0.f : z;
        v.w = none || two ? 0.f : w;
    }
};

// Variant for the narrowest layers (4 <= K <= 32, at most 32 output columns: every layer of the workload
// with slices and hidden width 32).  These layers are HBM bound (about 10 flop per byte), so the kernel
// is built around the memory accesses: a wavefront owns strips of 32 rows; it reads a strip with fully
// coalesced 16-byte loads (eight lanes per 128-byte row), parks it in its own LDS tile, and reads it
// back in the MFMA operand layout (lane = row, four consecutive k per 16-byte LDS read; the row
// stride of 36 floats keeps those reads conflict free).  The next strip's loads are issued before
// the current strip's MFMAs.  The weight operands never change, so every lane keeps its 16 values per
// product in registers.  No workgroup barrier anywhere: a wavefront only touches its own tile, and
// its LDS accesses execute in program order.
template <bool BWD, bool TWO>
__device__ __forceinline__ void pair_strip32(const PairArgs &a, uint32_t wg, uint32_t n_wg) // workgroup wg of n_wg
{
    constexpr int ST = 36;
    constexpr bool PAIR = TWO && !BWD; // two operand strips
    __shared__ __attribute__((aligned(16))) float T1[4][32][ST];
    __shared__ __attribute__((aligned(16))) float T2[PAIR ? 4 : 1][32][ST];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int m = lane & 31, h = lane >> 5;
    const int lr = lane >> 3, lc = (lane & 7) * 4; // coalesced layout: row lr + 8 * it, columns lc..lc+3
    const LaneCols<> cols(lc, a.K);
    const bool place = a.K < 32; // uniform: some lanes' columns have to be moved or zeroed
    float (*t1)[ST] = T1[wave];
    float (*t2)[ST] = T2[PAIR ? wave : 0];

    const int64_t n_full = a.n / 32; // whole strips
    const int64_t first = (int64_t)wg * 4 + wave, step = (int64_t)n_wg * 4;
    if (first * 32 >= a.n) return; // uniform per wavefront
    // what is absent is read from an operand and replaced, so that every strip has the same accesses
    const uint32_t *words = BWD && a.mask ? a.mask : reinterpret_cast<const uint32_t *>(a.A1);
    const int64_t word_ld = BWD && a.mask ? a.mask_words : 0;
    const float *s2 = PAIR && a.scale2 ? a.scale2 : a.A1, *so = a.scale_o1 ? a.scale_o1 : a.A1;
    const int64_t s2_ld = PAIR && a.scale2 ? 1 : 0, so_ld = a.scale_o1 ? 1 : 0;

    float4 p1[4], p2[PAIR ? 4 : 1];
    uint32_t pw = ~0u; // backward: activation word of strip row m (the row this lane feeds to the MFMAs)
    float ps = 1.f;    // backward: scale_o1 of strip row m
    // forward, scaled layout: factors of the rows lr + 8 it this lane loads and stores (only fetched here; they are
    // applied where the strip is consumed, so that the next strip's loads stay in flight behind the MFMAs).  One
    // load per lane and strip handed on by cross-lane reads was measured slower (the LDS pipe carries the tiles).
    float f2[PAIR ? 4 : 1], fo[BWD ? 1 : 4];
    const uint32_t ld1 = (uint32_t)a.lda1, ld2 = (uint32_t)a.lda2;
    auto fetch = [&](int64_t strip, auto whole) {
        const int64_t r0 = strip * 32;
        const int end = whole ? 31 : (int)(a.n - 1 - r0);
        auto row = [&](int i) { return (uint32_t)(whole || i < end ? i : end); }; // rows past the end re-read the last
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int64_t r = r0 + (whole ? 8 * it : 0);
            const uint32_t mine = row(whole ? lr : lr + 8 * it);
            p1[it] = cols.load(plus(a.A1 + r * a.lda1, mine * ld1));
            if (PAIR) {
                p2[it] = cols.load(plus(a.A2 + r * a.lda2, mine * ld2));
                f2[it] = *plus(s2 + r * s2_ld, mine * (uint32_t)s2_ld);
            }
            if (!BWD) fo[it] = *plus(so + r * so_ld, mine * (uint32_t)so_ld);
        }
        if (BWD) {
            pw = *plus(words + r0 * word_ld, row(m) * (uint32_t)word_ld);
            ps = *plus(so + r0 * so_ld, row(m) * (uint32_t)so_ld);
        }
    };
    if (first < n_full) fetch(first, std::true_type());
    else fetch(first, std::false_type());

    float b1[16], b2[16];
    const int mc = m < a.Nout ? m : a.Nout - 1;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int kk = 8 * q + 4 * h + i, kc = kk < a.K ? kk : a.K - 1;
            const int64_t id = BWD ? (int64_t)mc * a.ldw + kc : (int64_t)kc * a.ldw + mc;
            b1[q * 4 + i] = a.B1[id];
            b2[q * 4 + i] = TWO ? a.B2[id] : 0.f;
        }
    const bool col_ok = m < a.Nout;
    const float bias1 = (!BWD && col_ok) ? inner_bias<TWO>(a, m) : 0.f;
    const float bias2 = (PAIR && col_ok) ? outer_bias(a, m) : 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (8 * q + 4 * h + i >= a.K || !col_ok) b1[q * 4 + i] = b2[q * 4 + i] = 0.f;

    // One strip from the registers fetched; `next`: the strip to fetch meanwhile.  WHOLE: 32 rows and 32 columns to store.
    auto strip_step = [&](int64_t strip, int64_t next, auto whole) {
        constexpr bool WHOLE = decltype(whole)::value;
        float out_f[4]; // output factors of the rows lr + 8 it of this strip (the fetch below overwrites fo)
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            if (place) {
                cols.place(p1[it]);
                if (PAIR) cols.place(p2[it]);
            }
            if (PAIR) scale4(p2[it], s2_ld ? f2[it] : 1.f);
            out_f[it] = !BWD && so_ld ? fo[it] : 1.f;
            *reinterpret_cast<float4 *>(&t1[lr + 8 * it][lc]) = p1[it];
            if (PAIR) *reinterpret_cast<float4 *>(&t2[lr + 8 * it][lc]) = p2[it];
        }
        __builtin_amdgcn_wave_barrier();
        float4 a1[4], a2[4];
        const uint32_t word = BWD && a.mask ? pw : ~0u;
        const float scale = BWD && so_ld ? ps : 1.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            a1[q] = *reinterpret_cast<const float4 *>(&t1[m][8 * q + 4 * h]);
            if (PAIR) a2[q] = *reinterpret_cast<const float4 *>(&t2[m][8 * q + 4 * h]);
            if (BWD) { // second product: dHout as it is; first product: dP = dHout * mask (times the row's output factor)
                a2[q] = a1[q];
                const uint32_t bits = word >> (8 * q + 4 * h);
                if (!(bits & 1u)) a1[q].x = 0.f;
                if (!(bits & 2u)) a1[q].y = 0.f;
                if (!(bits & 4u)) a1[q].z = 0.f;
                if (!(bits & 8u)) a1[q].w = 0.f;
                scale4(a1[q], scale);
            }
        }
        __builtin_amdgcn_wave_barrier();
        if (WHOLE) fetch(next, std::true_type()); // flies during the MFMAs and the stores below
        floatx16 acc1, acc2;
#pragma unroll
        for (int r = 0; r < 16; ++r) { acc1[r] = 0.f; acc2[r] = 0.f; }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc1 = __builtin_amdgcn_mfma_f32_32x32x2f32(pick(a1[q], i), b1[q * 4 + i], acc1, 0, 0, 0);
                if (TWO) acc2 = __builtin_amdgcn_mfma_f32_32x32x2f32(pick(a2[q], i), b2[q * 4 + i], acc2, 0, 0, 0);
            }
        const int64_t row0 = strip * 32;
        uint32_t my_word = 0u; // lane L < 32 collects the activation word of strip row L
        float o1[16], o2[16];
        if constexpr (BWD) {
#pragma unroll
            for (int r = 0; r < 16; ++r) { o1[r] = acc1[r]; o2[r] = acc2[r]; }
        } else { // columns past the last have zero weights and biases: not active
#pragma unroll
            for (int r = 0; r < 16; ++r) o1[r] = acc1[r] + bias1;
            if (a.act == SLICEGCN_ACT_RELU) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const bool pos = o1[r] > 0.f;
                    set_lanes(my_word, __ballot(pos), 8 * (r / 4) + r % 4, 8 * (r / 4) + 4 + r % 4);
                    o1[r] = pos ? o1[r] : 0.f;
                }
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) o1[r] += TWO ? acc2[r] + bias2 : 0.f;
        }
        // Outputs leave through the wavefront's tile so that a row goes out as eight 16-byte stores
        // (register r of lane (m, h) is strip row 8*(r/4) + 4*h + r%4, column m).
        // `scaled`: rows take out_f on the way out (forward outputs kept in the scaled layout)
        auto store_tile = [&](const float (&o)[16], float *O, int64_t ldo, bool scaled) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int r = 0; r < 16; ++r) t1[8 * (r / 4) + 4 * h + (r % 4)][m] = o[r];
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int64_t row = row0 + lr + 8 * it;
                float4 v = *reinterpret_cast<const float4 *>(&t1[lr + 8 * it][lc]);
                if (scaled) scale4(v, out_f[it]);
                store_cols4<WHOLE>(O + row * ldo + lc, v, row < a.n, a.Nout - lc);
            }
            __builtin_amdgcn_wave_barrier();
        };
        store_tile(o1, a.O1, a.ldo1, !BWD && so_ld != 0);
        if (BWD && TWO && a.O2) store_tile(o2, a.O2, a.ldo2, false);
        if (!BWD && a.act == SLICEGCN_ACT_RELU && lane < 32 && (WHOLE || row0 + lane < a.n))
            a.mask[(row0 + lane) * a.mask_words] = my_word;
    };
    int64_t strip = first;
    if (a.Nout == 32) {
#pragma unroll 1
        for (; strip < n_full; strip += step) strip_step(strip, strip + step < n_full ? strip + step : strip, std::true_type());
    } else {
#pragma unroll 1
        for (; strip < n_full; strip += step) {
            strip_step(strip, 0, std::false_type());
            if (strip + step < n_full) fetch(strip + step, std::true_type());
        }
    }
    if (strip == n_full && a.n % 32 != 0) { // the rows left
        if (strip != first) fetch(strip, std::false_type());
        strip_step(strip, 0, std::false_type());
    }
}
template <bool BWD, bool TWO>
__global__ __launch_bounds__(256) void pair_strip32_kernel(const PairArgs common, const PairBatch batch)
{
    pair_strip32<BWD, TWO>(slice_of(common, batch), blockIdx.x, gridDim.x);
}

// Layers up to 64 wide (4 <= K <= 32 * KC, at most 32 * NC output columns) on many rows: a wavefront owns strips of 32 rows, reads a strip with
// coalesced 16-byte loads, parks it in its own LDS tile and reads it back in the operand layout of the matrix instruction.  The weights
// do not fit in registers next to the accumulators, so the workgroup keeps them (zero padded, already transposed for the backward
// products) in LDS and every MFMA takes its B operand from there: four consecutive k of a column lie together, so that one 16-byte read
// serves four instructions, and the reads of the next eight k are issued before the instructions of these.  (Left to itself the compiler
// read the weights of two instructions right before them and waited for the LDS each time, and it moved the next strip's loads behind all
// of the instructions; the barriers in `step` hold the order.)  The two operand strips of the forward pass go through the
// wavefront's one tile in turn.  Compiled for two wavefronts per SIMD: one computes while the other moves its strip.  A strip's addresses are a
// base that is the same for the wavefront and a 32-bit offset that is the same for every strip, and activation words are collected by lane writes
// (set_lanes): 85 + 230 vector instructions per strip instead of 172 + 440.  2.4 M rows 64 -> 64 forward 459 -> 401 us, 25 -> 64 295 -> 250, input
// gradients 404 -> 381; four slices of 169 k rows 145 -> 128, 93 -> 76, 131 -> 122.  Without their loads and stores the kernels take 106 us (input
// gradients, four slices), without the matrix instructions 83, which is the rate of a copy.  Strips handed out by a counter per workgroup
// instead of fixed shares: no gain, input gradients 381 -> 399.
template <int KC, int NC, bool BWD, bool TWO>
__global__ __launch_bounds__(256, 2) void pair_strip64_kernel(const PairArgs common, const PairBatch batch)
{
    const PairArgs a = slice_of(common, batch);
    constexpr int KW = 32 * KC, NW = 32 * NC;
    constexpr int ST = (KW > NW ? KW : NW) + 4; // tile row stride: 16-byte reads with lane = row stay conflict free
    constexpr int LK = KW / 4, LN = NW / 4;     // lanes per row, operand strips / output strips
    constexpr int PK = 32 * LK / 64, PN = 32 * LN / 64; // 16-byte accesses per lane and strip
    constexpr int RK = 64 / LK, RN = 64 / LN;   // rows per access
    constexpr int QN = 4 * KC;                  // float4 of the reduction axis per row
    constexpr bool PAIR = TWO && !BWD;          // two operand strips
    __shared__ __attribute__((aligned(16))) float Tl[4][32][ST];
    __shared__ float4 W1s[KW / 4][NW];
    __shared__ float4 W2s[TWO ? KW / 4 : 1][NW];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int m = lane & 31, h = lane >> 5;
    const int rk = lane / LK, rn = lane / LN, cn = (lane % LN) * 4; // coalesced layouts of an operand and of an output strip
    const LaneCols<> cols((lane % LK) * 4, a.K);
    const bool place = a.K < KW; // uniform: some lanes' columns have to be moved or zeroed
    float (*tl)[ST] = Tl[wave];

    const int64_t n_full = a.n / 32; // whole strips
    const int64_t first = (int64_t)blockIdx.x * 4 + wave, step = (int64_t)gridDim.x * 4;
    // what is absent is read from an operand and replaced, so that every strip has the same accesses
    const uint32_t *words = BWD && a.mask ? a.mask : reinterpret_cast<const uint32_t *>(a.A1);
    const int64_t word_ld = BWD && a.mask ? a.mask_words : 0;
    const float *s2 = PAIR && a.scale2 ? a.scale2 : a.A1, *so = a.scale_o1 ? a.scale_o1 : a.A1;
    const int64_t s2_ld = PAIR && a.scale2 ? 1 : 0, so_ld = a.scale_o1 ? 1 : 0;

    // The row factor of dZ: on the operand on fewer rows, as pair_rows_kernel has it, on the result on many.  The two differ in the last bit;
    // a gradient keeps its bits however many slices share a launch.
    const bool scale_operand = BWD && a.n < STRIP64_ROWS;

    float4 p1[PK], p2[PAIR ? PK : 1];
    uint32_t pw[KC];                // backward: activation words of strip row m
    float ps = 1.f;                 // and its row factor
    float f2[PAIR ? PK : 1], fo[PN]; // factors of the rows this lane loads and stores
    const uint32_t ld1 = (uint32_t)a.lda1, ld2 = (uint32_t)a.lda2;
    auto fetch = [&](int64_t strip, auto whole) {
        const int64_t r0 = strip * 32;
        const int end = whole ? 31 : (int)(a.n - 1 - r0);
        auto row = [&](int i) { return (uint32_t)(whole || i < end ? i : end); }; // rows past the end re-read the last
#pragma unroll
        for (int it = 0; it < PK; ++it) {
            const int64_t r = r0 + (whole ? RK * it : 0);
            const uint32_t mine = row(whole ? rk : rk + RK * it);
            p1[it] = cols.load(plus(a.A1 + r * a.lda1, mine * ld1));
            if (PAIR) {
                p2[it] = cols.load(plus(a.A2 + r * a.lda2, mine * ld2));
                f2[it] = *plus(s2 + r * s2_ld, mine * (uint32_t)s2_ld);
            }
        }
        if (BWD) {
            const uint32_t mine = row(m);
#pragma unroll
            for (int w = 0; w < KC; ++w) pw[w] = *plus(words + r0 * word_ld + (32 * w < a.K ? w : 0), mine * (uint32_t)word_ld);
            ps = *plus(so + r0 * so_ld, mine * (uint32_t)so_ld);
        }
#pragma unroll
        for (int it = 0; it < PN; ++it) {
            const int64_t r = r0 + (whole ? RN * it : 0);
            fo[it] = *plus(so + r * so_ld, row(whole ? rn : rn + RN * it) * (uint32_t)so_ld);
        }
    };
    if (first < n_full) fetch(first, std::true_type());

    constexpr int WN = KW * NW / 256; // weights of a thread
    float w1[WN], w2[TWO ? WN : 1];
#pragma unroll
    for (int i = 0; i < WN; ++i) {
        // consecutive threads walk the contiguous axis of W: columns forward, k backward (W^T)
        const int idx = threadIdx.x + 256 * i, kk = BWD ? idx % KW : idx / NW, j = BWD ? idx / KW : idx % NW;
        const int kc = kk < a.K ? kk : a.K - 1, jc = j < a.Nout ? j : a.Nout - 1;
        const int64_t id = BWD ? (int64_t)jc * a.ldw + kc : (int64_t)kc * a.ldw + jc;
        w1[i] = a.B1[id];
        if (TWO) w2[i] = a.B2[id];
    }
#pragma unroll
    for (int i = 0; i < WN; ++i) {
        const int idx = threadIdx.x + 256 * i, kk = BWD ? idx % KW : idx / NW, j = BWD ? idx / KW : idx % NW;
        const bool there = kk < a.K && j < a.Nout;
        reinterpret_cast<float *>(&W1s[kk / 4][j])[kk % 4] = there ? w1[i] : 0.f;
        if (TWO) reinterpret_cast<float *>(&W2s[kk / 4][j])[kk % 4] = there ? w2[i] : 0.f;
    }
    float bias1[NC], bias2[NC];
#pragma unroll
    for (int t = 0; t < NC; ++t) {
        const bool ok = 32 * t + m < a.Nout;
        bias1[t] = (!BWD && ok) ? inner_bias<TWO>(a, 32 * t + m) : 0.f;
        bias2[t] = (PAIR && ok) ? outer_bias(a, 32 * t + m) : 0.f;
    }
    __syncthreads(); // the only workgroup barrier: from here on a wavefront touches its own tile only

    // One strip from the registers fetched; `next`: the strip to fetch meanwhile.  32 rows and NW columns to store (WHOLE), 32 rows and at least four
    // columns (FULL_ROWS), or whatever there is (then nothing is fetched).
    // FULL_ROWS: a lane without four columns of its own stores the row's last four once more, so that no store depends on a branch and the
    // next strip's loads stay in flight as with WHOLE (2.4 M rows, fetched behind stores with a test per lane /
    // here: 25 -> 40 208 / 158 us, 64 -> 47 297 / 255, 40 -> 10 173 / 128; input gradients 190 / 151, 290 / 252, 164 / 135).
    // Not where rows lie apart in more than half of the last-level cache: lines are written in part there, which bounds the kernel, and the last four columns cost one such write more (rows of
    // 64 or 32 floats: 25 -> 40 245 / 272, 40 -> 10 214 / 238, 50 -> 33 324 / 345; but 1 M rows 40 -> 10 80 / 61).
    constexpr int64_t PARTIAL_LINES = (int64_t)128 << 20;
    constexpr std::integral_constant<int, 0> REST;
    constexpr std::integral_constant<int, 1> FULL_ROWS;
    constexpr std::integral_constant<int, 2> WHOLE;
    constexpr bool AHEAD = !TWO || KC == 1; // two products of up to 64 columns leave no registers for it (64 -> 16 with self term 508 / 523 us)
    const int last4 = a.Nout - 4, cs = cn < last4 ? cn : last4; // first column of the four that this lane stores
    auto strip_step = [&](int64_t strip, int64_t next, auto form) {
        constexpr bool ALL_ROWS = form.value >= FULL_ROWS.value;
        float out_f[PN]; // output factors of this strip's rows (the fetch below overwrites fo)
#pragma unroll
        for (int it = 0; it < PN; ++it) out_f[it] = so_ld && !scale_operand ? fo[it] : 1.f;
        const float in_f = BWD && so_ld && scale_operand ? ps : 1.f;
        if (place) {
#pragma unroll
            for (int it = 0; it < PK; ++it) {
                cols.place(p1[it]);
                if (PAIR) cols.place(p2[it]);
            }
        }
#pragma unroll
        for (int it = 0; it < PK; ++it) *reinterpret_cast<float4 *>(&tl[rk + RK * it][(lane % LK) * 4]) = p1[it];
        __builtin_amdgcn_wave_barrier();
        float4 a1[QN];
#pragma unroll
        for (int q = 0; q < QN; ++q) a1[q] = *reinterpret_cast<const float4 *>(&tl[m][8 * q + 4 * h]);
        __builtin_amdgcn_wave_barrier();
        if (PAIR) { // the second operand strip takes the tile while the first product runs from registers
#pragma unroll
            for (int it = 0; it < PK; ++it) {
                scale4(p2[it], s2_ld ? f2[it] : 1.f);
                *reinterpret_cast<float4 *>(&tl[rk + RK * it][(lane % LK) * 4]) = p2[it];
            }
            __builtin_amdgcn_wave_barrier();
        }
        uint32_t word[KC];
#pragma unroll
        for (int w = 0; w < KC; ++w) word[w] = !BWD ? 0u : !a.mask ? ~0u : pw[w];
        __builtin_amdgcn_sched_barrier(0);
        if (ALL_ROWS) fetch(next, std::true_type()); // flies during the MFMAs and the stores below
        floatx16 acc1[NC], acc2[NC];
#pragma unroll
        for (int t = 0; t < NC; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) { acc1[t][r] = 0.f; acc2[t][r] = 0.f; }
        // Steps of eight k, those of the second product behind those of the first.  Backward both read dHout, the first one through the
        // activation bits (dP = dHout * mask); forward a step's operand is replaced by the second strip's when it is done with.
        constexpr int STEPS = TWO ? 2 * QN : QN;
        float4 bw[2][NC];
        auto weights = [&](int s) {
#pragma unroll
            for (int t = 0; t < NC; ++t) bw[s & 1][t] = s < QN ? W1s[2 * s + h][32 * t + m] : W2s[TWO ? 2 * (s - QN) + h : 0][32 * t + m];
        };
        weights(0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) { // step
            const int q = s < QN ? s : s - QN;
            if (s + 1 < STEPS) weights(s + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float x = pick(a1[q], i);
                if (BWD && s < QN) x = (((word[q >> 2] >> (8 * (q & 3) + 4 * h + i)) & 1u) ? x : 0.f) * in_f;
#pragma unroll
                for (int t = 0; t < NC; ++t) {
                    if (s < QN) acc1[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(x, pick(bw[s & 1][t], i), acc1[t], 0, 0, 0);
                    else acc2[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(x, pick(bw[s & 1][t], i), acc2[t], 0, 0, 0);
                }
            }
            if (PAIR && s < QN) a1[q] = *reinterpret_cast<const float4 *>(&tl[m][8 * q + 4 * h]);
            __builtin_amdgcn_sched_barrier(0);
        }
        const int64_t row0 = strip * 32;
        uint32_t my_word[NC]; // lane L < 32 collects the activation words of strip row L
        if (!BWD) { // the forward result replaces the first accumulator (columns past the last have zero weights and biases: not active)
#pragma unroll
            for (int t = 0; t < NC; ++t) {
                my_word[t] = 0u;
#pragma unroll
                for (int r = 0; r < 16; ++r) acc1[t][r] += bias1[t];
                if (a.act == SLICEGCN_ACT_RELU) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const bool pos = acc1[t][r] > 0.f;
                        const unsigned long long bal = __ballot(pos);
                        set_lanes(my_word[t], bal, 8 * (r / 4) + r % 4, 8 * (r / 4) + 4 + r % 4);
                        acc1[t][r] = pos ? acc1[t][r] : 0.f;
                    }
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) acc1[t][r] += TWO ? acc2[t][r] + bias2[t] : 0.f;
            }
        }
        // Outputs leave through the wavefront's tile so that a row goes out as 16-byte stores
        // (register r of lane (m, h) is strip row 8*(r/4) + 4*h + r%4, column 32 t + m).
        // `scaled`: rows take out_f on the way out (outputs kept in the scaled layout)
        auto store_tile = [&](const floatx16 (&o)[NC], float *O, int64_t ldo, bool scaled) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int t = 0; t < NC; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) tl[8 * (r / 4) + 4 * h + (r % 4)][32 * t + m] = o[t][r];
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int it = 0; it < PN; ++it) {
                const int64_t row = row0 + rn + RN * it;
                float4 v;
                if constexpr (form.value == FULL_ROWS.value) {
                    const floatx4_u u = *reinterpret_cast<const floatx4_u *>(&tl[rn + RN * it][cs]);
                    v = make_float4(u.x, u.y, u.z, u.w);
                } else {
                    v = *reinterpret_cast<const float4 *>(&tl[rn + RN * it][cn]);
                }
                if (scaled) scale4(v, out_f[it]);
                store_cols4<ALL_ROWS>(O + row * ldo + (form.value == FULL_ROWS.value ? cs : cn), v, row < a.n, a.Nout - cn);
            }
            __builtin_amdgcn_wave_barrier();
        };
        store_tile(acc1, a.O1, a.ldo1, so_ld != 0 && !scale_operand);
        if constexpr (BWD && TWO) {
            if (a.O2) store_tile(acc2, a.O2, a.ldo2, false);
        }
        if (!BWD && a.act == SLICEGCN_ACT_RELU && lane < 32 && (ALL_ROWS || row0 + lane < a.n)) {
#pragma unroll
            for (int t = 0; t < NC; ++t)
                if (form.value == WHOLE.value || 32 * t < a.Nout) a.mask[(row0 + lane) * a.mask_words + t] = my_word[t];
        }
    };
    int64_t strip = first;
    auto in_turn = [&](auto form) {
#pragma unroll 1
        for (; strip < n_full; strip += step) strip_step(strip, strip + step < n_full ? strip + step : strip, form);
    };
    if (a.Nout == NW) in_turn(WHOLE);
    else if (AHEAD && a.Nout >= 4 && (a.ldo1 < a.Nout + 8 || a.n * a.ldo1 * 4 <= PARTIAL_LINES)) in_turn(FULL_ROWS);
    else {
#pragma unroll 1
        for (; strip < n_full; strip += step) {
            strip_step(strip, 0, REST);
            if (strip + step < n_full) fetch(strip + step, std::true_type());
        }
    }
    if (strip == n_full && a.n % 32 != 0) { // the rows left
        fetch(strip, std::false_type());
        strip_step(strip, 0, REST);
    }
}

template <int KC, int NC, bool BWD>
void launch_strip64(const PairArgs &a, const PairBatch &b, dim3 grid, hipStream_t stream)
{
    if (a.A2 != nullptr && a.B2 != nullptr) pair_strip64_kernel<KC, NC, BWD, true><<<grid, 256, 0, stream>>>(a, b);
    else pair_strip64_kernel<KC, NC, BWD, false><<<grid, 256, 0, stream>>>(a, b);
}

// Products in place: whether output rows are rows of an operand (the leading dimensions agree; the kernels read a row before they
// store it, but another workgroup may still read the row for its own columns)
inline bool same_rows(const float *o, int64_t ldo, int32_t wo, const float *x, int64_t ldx, int32_t wx)
{
    const int64_t d = (reinterpret_cast<intptr_t>(x) - reinterpret_cast<intptr_t>(o)) / (int64_t)sizeof(float);
    return o && x && ldo == ldx && d < wo && -d < wx;
}
inline bool in_place(const PairArgs *list, int batch)
{
    bool any = false;
    for (int i = 0; i < batch; ++i) {
        const PairArgs &a = list[i];
        const float *second = a.B2 ? a.A2 : nullptr;
        any = any || same_rows(a.O1, a.ldo1, a.Nout, a.A1, a.lda1, a.K) || same_rows(a.O1, a.ldo1, a.Nout, second, a.lda2, a.K) ||
              same_rows(a.O2, a.ldo2, a.Nout, a.A1, a.lda1, a.K) || same_rows(a.O2, a.ldo2, a.Nout, second, a.lda2, a.K);
    }
    return any;
}
// Tiles of 32 columns a workgroup of pair_rows_kernel can take (three for two products, and four, have their registers at two workgroups
// per CU; four are compiled for products in place alone)
inline int most_tiles(const PairArgs &a) { return a.A2 != nullptr && a.B2 != nullptr ? 3 : 4; }
int check_in_place(const PairArgs *list, int batch)
{
    const int tiles = (list[0].Nout + 31) / 32, most = most_tiles(list[0]);
    SG_REQUIRE(tiles <= most || !in_place(list, batch), SLICEGCN_EINVAL, "dense product in place: %d output columns, at most %d", list[0].Nout,
               32 * most);
    return SLICEGCN_OK;
}

// Which kernel forms the products, with how many workgroups per slice
struct PairForm {
    enum Kernel { STRIP32, STRIP64, WIDE, ROWS } kernel;
    bool two;
    int64_t blocks;
    int nt, n_col; // ROWS, WIDE: tiles of 32 columns a workgroup takes, workgroups along the columns
};
inline PairForm pair_form(const PairArgs *list, int batch, bool backward, bool wide = true) // wide: may take pair_wide_kernel
{
    const PairArgs &a = list[0];
    const bool two = a.A2 != nullptr && a.B2 != nullptr;
    const int64_t strips = (a.n + 31) / 32, strip_blocks = (strips + 3) / 4;
    // narrowest layers: per-wavefront strips, no barriers; but below STRIP64_ROWS not those whose K is a whole chunk of pair_rows_kernel or no
    // more than its first eight steps, which issues far fewer instructions per row there and keeps more wavefronts on a SIMD.  Strips / rows, 32
    // columns out:
    //     K    with self term, 20 k rows   66 k          169 k         262 k         input gradients, 20 k   169 k
    //     8    6.3 / 6.3 us                11.3 / 8.6    20.7 / 17.0   26.0 / 20.2   5.5 / 3.9               13.2 / 10.9
    //     12   6.3 / 6.3                   11.1 / 8.9    20.8 / 18.2   26.0 / 22.0   4.7 / 4.1               12.3 / 11.3
    //     16   6.3 / 7.3                   11.1 / 11.1   21.4 / 22.9   26.1 / 27.4   5.5 / 4.5               14.1 / 13.9
    //     24   6.3 / 7.9                   11.1 / 13.7   21.0 / 28.3   26.2 / 34.3   5.5 / 5.0               13.9 / 16.2
    //     28   6.3 / 7.3                   11.1 / 12.5   20.9 / 25.9   25.7 / 33.0   4.7 / 4.5               13.1 / 15.4
    //     32   6.1 / 5.9                   10.9 / 9.5    20.8 / 19.5   25.9 / 25.8   5.4 / 4.1               13.5 / 12.2
    // (from there on strips: 2.4 M rows with self term, K = 8 165 / 181, K = 16 166 / 224, K = 32 189 / 198).
    const int64_t resident = 512 / batch; // as many workgroups as the chip holds at once: two per CU
    const bool near = a.lda1 < (1 << 24) && a.lda2 < (1 << 24) && a.mask_words < (1 << 24); // a strip's rows lie within 32-bit offsets
    if (near && a.K >= 4 && a.K <= 32 && a.Nout <= 32 && ((a.K > 8 && a.K < 32) || a.n * batch >= STRIP64_ROWS)) {
        // Each stages the weights once, and a second strip is requested while the first is multiplied (K = 16 with self term, 2048 / 512
        // workgroups: 130 k rows 20.4 / 17.0 us, 169 k 26.0 / 21.3, 262 k 32.8 / 26.1, 800 k 73 / 66; input gradients 130 k 14.0 / 11.8, 262 k
        // 23.5 / 16.8).  More where the launch is long: 2.4 M rows of 8 columns out 217 / 240, input gradients of 12 columns 91 / 96, and
        // beside weight gradients 800 k rows 16 -> 28 73.7 / 76.1.
        const int64_t most = strip_blocks * batch <= (two ? 8192 : 2048) ? resident : 2048;
        return PairForm{PairForm::STRIP32, two, strip_blocks < most ? strip_blocks : most, 0, 0};
    }
    if (near && a.K >= 4 && a.K <= 64 && a.Nout <= 64 && a.n * batch >= STRIP64_ROWS) { // up to 64 wide: strips, weights in LDS
        // (each workgroup stages the weights once: four slices of 169 k rows with 2048 workgroups forward 164 us instead of 149, backward
        // 151 instead of 130)
        return PairForm{PairForm::STRIP64, two, strip_blocks < resident ? strip_blocks : resident, 0, 0};
    }
    const int tiles = (a.Nout + 31) / 32;
    // Tiles of 32 columns a workgroup of pair_rows_kernel takes: two keep three or four workgroups on a CU, where four (two workgroups) take 244 us instead
    // of 238 for 169 k rows 256 -> 256 and 158 instead of 130 for 20 k rows 512 -> 512; three for widths of three tiles, which two would
    // pad to four; one where that would leave fewer than eight workgroups per CU (20 k rows 256 -> 256: 38 us instead of 41,
    // 169 k rows 256 -> 40: 67 instead of 75; 169 k rows 256 -> 256, above the line: 253 instead of 238).
    int nt = tiles % 2 != 0 && tiles % 3 == 0 ? 3 : tiles < 2 ? 1 : 2;
    // Wide single products, and the two input gradients of a slice layer as two of them (forward the sum would have to be read back), where a workgroup per CU
    // that holds its columns' weights has strips enough (wide_even; one slice below and above its line, rows / wide: 66 k rows 128 -> 128, two strips a SIMD,
    // 31.3 / 37.7 us; 100 k 100 -> 96, three, 31.5 / 34.0; 66 k 256 -> 256, four, 98.4 / 93.7, its input gradients 93.6 / 96.8; 169 k 128 -> 128, five,
    // 67.5 / 66.6 and 64.7 / 67.7; 300 k 47 <- 131, nine, 76.4 / 74.2; 169 k 256 -> 256, ten, 221 / 196 and 218 / 197; 400 k 37 -> 70, twelve, 65.5 / 51.0),
    // enough to multiply (wide_long) and no more tiles of padding than pair_rows_kernel (280 k rows 400 -> 96, four tiles for three, 0.83 times as fast).  Not
    // where K is one whole chunk of pair_rows_kernel, which loads it without tests and has nothing to wait for twice (400 k rows 32 -> 128 66 / 68,
    // 128 <- 32 52 / 57).
    const bool form = backward || (!two && !a.scale_o1), columns = tiles >= 2 && (a.Nout % 32 == 0 || a.Nout % 32 >= 4);
    if (wide && near && form && columns && a.K >= 4 && a.K != 32 && a.ldo1 < (1 << 24) && a.ldo2 < (1 << 24) && !in_place(list, batch)) {
        // as few tiles of padding as can be, then as many per workgroup as can be
        const auto padded = [&](int t) { return (tiles + t - 1) / t * t; };
        int wt = 2;
        for (int t = 3; t <= 4; ++t)
            if (padded(t) <= padded(wt) && a.K <= wide_k(t)) wt = t;
        const int n_col = padded(wt) / wt, walkers = wide_walkers(n_col * batch);
        const bool lines = a.ldo1 % 32 == 0 && (!a.O2 || a.ldo2 % 32 == 0), bits = backward ? a.mask != nullptr : a.act == SLICEGCN_ACT_RELU;
        if (padded(wt) <= padded(nt) && a.K <= wide_k(wt) && wide_long(wt, n_col, a.K, lines, bits, two) && wide_even(n_col * batch, strips))
            return PairForm{PairForm::WIDE, two, 8 * (int64_t)walkers * n_col, wt, n_col};
    }
    // everything else: 1-D grid per slice, 8 row tiles x all column tiles per group of workgroups (see the kernel)
    const int64_t row_tiles = (a.n + 127) / 128;
    if (row_tiles * ((tiles + nt - 1) / nt) * batch < 2048) nt = 1;
    if (tiles > nt && in_place(list, batch)) nt = tiles; // whole rows
    const int n_col = (tiles + nt - 1) / nt;
    return PairForm{PairForm::ROWS, two, (row_tiles + 7) / 8 * 8 * n_col, nt, n_col};
}
inline PairBatch pair_batch(const PairArgs *list, int batch)
{
    PairBatch b;
    for (int i = 0; i < BATCH; ++i) {
        const PairArgs &x = list[i < batch ? i : 0];
        b.p[i] = PairPtrs{x.A1, x.A2, x.B1, x.B2, x.bias1, x.bias2, x.enc, x.O1, x.O2, x.mask};
    }
    return b;
}

template <int NT, bool BWD>
void launch_wide(const PairArgs &a, const PairBatch &b, dim3 grid, int n_col, hipStream_t stream)
{
    const int walkers = (int)grid.x / n_col;
    const auto launch = [&](auto r) {
        if (a.K % 32 == 0) pair_wide_kernel<NT, r.value, false, BWD><<<grid, 64 * WIDE_WAVES, 0, stream>>>(a, b, n_col, walkers);
        else pair_wide_kernel<NT, r.value, true, BWD><<<grid, 64 * WIDE_WAVES, 0, stream>>>(a, b, n_col, walkers);
    };
    if (a.K <= 64) launch(std::integral_constant<int, 2>());
    else launch(std::integral_constant<int, 4>());
}
template <bool BWD>
int launch_wide(const PairArgs *list, int batch, const PairForm &f, hipStream_t stream)
{
    const dim3 grid((unsigned)f.blocks, (unsigned)batch);
    const PairBatch b = pair_batch(list, batch);
    if (f.nt == 2) launch_wide<2, BWD>(list[0], b, grid, f.n_col, stream);
    else if (f.nt == 3) launch_wide<3, BWD>(list[0], b, grid, f.n_col, stream);
    else launch_wide<4, BWD>(list[0], b, grid, f.n_col, stream);
    SG_LAUNCH_CHECK();
    if (!BWD || !f.two || !list[0].O2) return SLICEGCN_OK;
    PairArgs second[BATCH]; // of a slice layer's two input-gradient products: no mask, no row factors
    for (int i = 0; i < batch; ++i) {
        PairArgs &p = second[i] = list[i];
        p.A1 = p.A2; p.lda1 = p.lda2; p.B1 = p.B2; p.O1 = p.O2; p.ldo1 = p.ldo2;
        p.mask = nullptr; p.scale_o1 = nullptr; p.O2 = nullptr;
    }
    return launch_wide<BWD>(second, batch, f, stream);
}

// `list`: one entry per slice model of the batch (1 to BATCH, equal but for the pointers)
template <bool BWD>
int launch_pair(const PairArgs *list, int batch, hipStream_t stream)
{
    if (int rc = check_in_place(list, batch)) return rc;
    const PairArgs &a = list[0];
    const PairBatch b = pair_batch(list, batch);
    const PairForm f = pair_form(list, batch, BWD);
    SG_REQUIRE(f.blocks <= INT32_MAX, SLICEGCN_ERANGE, "dense product: grid too large");
    const dim3 grid((unsigned)f.blocks, (unsigned)batch);
    const int n_col = f.n_col;
    switch (f.kernel) {
    case PairForm::STRIP32:
        if (f.two) pair_strip32_kernel<BWD, true><<<grid, 256, 0, stream>>>(a, b);
        else pair_strip32_kernel<BWD, false><<<grid, 256, 0, stream>>>(a, b);
        break;
    case PairForm::STRIP64:
        if (a.K <= 32) launch_strip64<1, 2, BWD>(a, b, grid, stream);
        else if (a.Nout <= 32) launch_strip64<2, 1, BWD>(a, b, grid, stream);
        else launch_strip64<2, 2, BWD>(a, b, grid, stream);
        break;
    case PairForm::WIDE:
        return launch_wide<BWD>(list, batch, f, stream);
    case PairForm::ROWS:
        return launch_parts(f.blocks, [&](unsigned first, unsigned count) { // one to three columns in: any number of rows comes here
            const dim3 grid(count, (unsigned)batch);
            switch (2 * f.nt + (f.two ? 1 : 0)) {
            case 2: pair_rows_kernel<1, false, BWD><<<grid, 256, 0, stream>>>(a, b, n_col, first); break;
            case 3: pair_rows_kernel<1, true, BWD><<<grid, 256, 0, stream>>>(a, b, n_col, first); break;
            case 4: pair_rows_kernel<2, false, BWD><<<grid, 256, 0, stream>>>(a, b, n_col, first); break;
            case 5: pair_rows_kernel<2, true, BWD><<<grid, 256, 0, stream>>>(a, b, n_col, first); break;
            case 6: pair_rows_kernel<3, false, BWD><<<grid, 256, 0, stream>>>(a, b, n_col, first); break;
            case 7: pair_rows_kernel<3, true, BWD><<<grid, 256, 0, stream>>>(a, b, n_col, first); break;
            default: pair_rows_kernel<4, false, BWD><<<grid, 256, 0, stream>>>(a, b, n_col, first); break;
            }
        });
    }
    SG_LAUNCH_CHECK();
    return SLICEGCN_OK;
}

template <bool BWD>
int launch_pair(const PairArgs &a, hipStream_t stream) { return launch_pair<BWD>(&a, 1, stream); }

// ---- weight-gradient reductions over the node axis ----------------------------------------
constexpr int RED_ROWS = 1024; // rows per block: fp32 chains stay this short
constexpr int RED_TILE = 32;   // output tile edge
constexpr int RED_RK = 32;     // rows staged per step

struct ReduceArgs {
    const float *Z; int64_t ldz;
    const float *Hin; int64_t ldi;      // NULL: no self term
    const float *dHout; int64_t ldo;
    const uint32_t *mask; int64_t mask_words; // NULL: all ones
    float *partial;                     // [n_row_blocks][stride]
    int64_t n;
    int32_t w_in, w_out;
    int32_t stride;                     // 2*w_in*w_out + 2*w_out; compact: w_in*w_out + w_out
    int32_t compact;                    // 1: no self term and no slot for it: [Z^T dP | colsum dP]
    int32_t rows_per_block = RED_ROWS;  // tiled kernels: node rows per workgroup (one partial each)
    int32_t j_tiles = 1;                // tiled kernels: output tiles along w_out (grid depth = j_tiles x batch)
    const float *hin_scale = nullptr;   // rows of Hin are multiplied by hin_scale[row] when read (Hin stored as D~^-1/2 Hin)
};

struct ReducePtrs {
    const float *Z, *Hin, *dHout;
    const uint32_t *mask;
    float *partial;
};
struct ReduceBatch { ReducePtrs p[BATCH]; };
__device__ inline ReduceArgs slice_of(const ReduceArgs &common, const ReduceBatch &b, int i)
{
    ReduceArgs r = common;
    const ReducePtrs &p = b.p[i];
    r.Z = p.Z; r.Hin = p.Hin; r.dHout = p.dHout; r.mask = p.mask; r.partial = p.partial;
    return r;
}

// Partial weight gradients of the layers the strip kernels do not take (but see grad_big_mfma_kernel): a workgroup forms a tile of one
// product (Z^T dP or Hin^T dHout, the grid's depth) over rows_per_block node rows.  The node axis is the matrix instruction's k axis, so an operand register
// is 32 consecutive columns of two rows: they come straight from memory, several pairs of rows ahead, with no LDS and no
// barrier in the row loop.  Two forms, which differ in the order of the sums and so are not chosen by speed:
//   WJ = 0  wavefront w takes rows 8 w to 8 w + 7 of every 32 for the whole tile of MI x NJ times 32 x 32; the four sums are added in
//           order at the end (slice layers, and dense layers up to 64 wide)
//   WJ > 0  the four wavefronts own tiles of their own, WJ of them along w_out, over all rows (wider dense layers)
// Column sums (bias gradients) run in row order over the loaded values.
// A kernel that staged 32 x 32 tiles in LDS re-read its operands per tile and waited at two barriers per 32 rows.  Pairs of products:
// two slices of 233 k rows 301 x 128 1.65 -> 1.19 ms (0.75 with scalar bases and 32-bit offsets, 102 TFLOP/s), 800 k rows 64 x 64 338 -> 235, 169 k rows 64 x 64 76 -> 63; dense layers: 2.4 M rows
// 256 x 47 1.93 -> 1.40 ms, 60 k rows 64 x 64 46 -> 22 us.  Bound by the loads, one register of two rows' pieces at a time.  A load's base comes from the
// one before it by an addition: with a product of row and leading dimension each, some 140 scalar multiplications per step, chains of few rows were 2 to 6 % slower than
// with an address per lane, and all of them slower than now: backward passes of layers 7.6 k rows 72 -> 222 39.0 -> 36.3 us, 30 k rows 100 -> 64 46.1 -> 42.1;
// 169 k rows 256 x 40 127 -> 97, 300 k 64 x 200 221 -> 153, 2.4 M 47 x 256 1.26 -> 1.18 ms, without activation bits 1.09 / 1.10 (500 k 40 x 300 421 / 436 us).
// Grid: x = 8 row blocks x all tiles per group of workgroups (a row block's tiles meet on one XCD), y = slice, z = product.
template <int MI, int NJ, int WJ>
__device__ __forceinline__ void grad_rows_tile(const ReduceArgs &a, int64_t wg, bool self, int n_tiles) // self: the product Hin^T dHout
{
    constexpr bool SPLIT = WJ == 0;
    constexpr int WI = SPLIT ? 1 : 4 / (SPLIT ? 1 : WJ);
    constexpr int PAIRS = MI * NJ == 1 ? 8 : 4; // pairs of rows a wavefront loads at a time
    constexpr int ROWS = (SPLIT ? 8 : 2) * PAIRS;                   // rows the workgroup advances by
    __shared__ __attribute__((aligned(16))) float red[SPLIT ? 4 : 1][SPLIT ? 32 * 32 : 1];
    __shared__ float bsum[SPLIT ? 4 : 1][SPLIT ? NJ * 32 : 1];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int m = lane & 31, h = lane >> 5;
    const TilePlace place = tile_place((uint32_t)wg, n_tiles); // (the division is done by vector instructions)
    const int col_tile = __builtin_amdgcn_readfirstlane(place.col_tile);
    const int64_t block = (uint32_t)__builtin_amdgcn_readfirstlane(place.row_tile), r_begin = block * a.rows_per_block;
    if (r_begin >= a.n) return; // uniform per workgroup
    const int64_t r_end = r_begin + a.rows_per_block < a.n ? r_begin + a.rows_per_block : a.n;
    const int i_base = (col_tile / a.j_tiles) * (WI * MI * 32) + (SPLIT ? 0 : wave / (SPLIT ? 1 : WJ) * (MI * 32));
    const int j_base = (col_tile % a.j_tiles) * ((SPLIT ? 1 : WJ) * NJ * 32) + (SPLIT ? 0 : wave % (SPLIT ? 1 : WJ) * (NJ * 32));
    if (!SPLIT && (i_base >= a.w_in || j_base >= a.w_out)) return; // uniform per wavefront; no barriers in this form
    const float *X = self ? a.Hin : a.Z;
    const int64_t ldx = self ? a.ldi : a.ldz;
    const float *x_scale = self ? a.hin_scale : nullptr;
    const uint32_t *mask = self ? nullptr : a.mask;
    const bool sums = i_base == 0; // this workgroup (wavefront) also forms the column sums of its columns

    // This lane's columns of row h of a pair, as offsets from the pair's first row, which is the same for the wavefront.  Columns past the last one
    // re-read the last: what they give is not stored
    int cx[MI], cg[NJ], cw[NJ];
#pragma unroll
    for (int t = 0; t < MI; ++t) cx[t] = i_base + 32 * t + m < a.w_in ? i_base + 32 * t + m : a.w_in - 1;
#pragma unroll
    for (int t = 0; t < NJ; ++t) {
        cg[t] = j_base + 32 * t + m < a.w_out ? j_base + 32 * t + m : a.w_out - 1;
        cw[t] = (j_base + 32 * t < a.w_out ? j_base + 32 * t : a.w_out - 1) >> 5;
    }
    constexpr int64_t FAR = (int64_t)1 << 28; // a row's length in 32 bits of bytes
    const bool near = ldx < FAR && a.ldo < FAR && (!mask || a.mask_words < FAR);
    const uint32_t hx = (uint32_t)(h * ldx), hg = (uint32_t)(h * a.ldo), hw = mask ? (uint32_t)(h * a.mask_words) : 0u;
    float nx[PAIRS][MI], np[PAIRS][NJ], nf[PAIRS];
    uint32_t nw[PAIRS][NJ];
    auto row_of = [&](int64_t r0, int p) { return r0 + (SPLIT ? 32 * (p / 4) + 8 * wave + 2 * (p % 4) : 2 * p); }; // of pair p, and the next one
    // from a pair to the next, and from a wavefront's eight rows to its next eight (opaque, or the compiler makes products of them again)
    int64_t two_x = 2 * ldx, two_g = 2 * a.ldo, two_w = 2 * a.mask_words, far_x = 26 * ldx, far_g = 26 * a.ldo, far_w = 26 * a.mask_words;
    asm("" : "+s"(two_x), "+s"(two_g), "+s"(two_w), "+s"(far_x), "+s"(far_g), "+s"(far_w));
    auto fetch = [&](int64_t r0) {
        if (near && r0 + ROWS <= r_end) {
            int64_t at = row_of(r0, 0);
            asm("" : "+s"(at)); // (or the compiler keeps a 64-bit address per load and lane, steps them all, and spills)
            const float *x = X + at * ldx, *g = a.dHout + at * a.ldo;
            uint32_t ox[MI], og[NJ];
#pragma unroll
            for (int t = 0; t < MI; ++t) ox[t] = fresh(hx + cx[t]);
#pragma unroll
            for (int t = 0; t < NJ; ++t) og[t] = fresh(hg + cg[t]);
#pragma unroll
            for (int p = 0; p < PAIRS; ++p) {
#pragma unroll
                for (int t = 0; t < MI; ++t) nx[p][t] = *plus(x, ox[t]);
#pragma unroll
                for (int t = 0; t < NJ; ++t) np[p][t] = *plus(g, og[t]);
                x += SPLIT && p % 4 == 3 ? far_x : two_x;
                g += SPLIT && p % 4 == 3 ? far_g : two_g;
            }
            if (mask) {
                const uint32_t *w = mask + at * a.mask_words;
                uint32_t ow[NJ];
#pragma unroll
                for (int t = 0; t < NJ; ++t) ow[t] = fresh(hw + cw[t]);
#pragma unroll
                for (int p = 0; p < PAIRS; ++p) {
#pragma unroll
                    for (int t = 0; t < NJ; ++t) nw[p][t] = *plus(w, ow[t]);
                    w += SPLIT && p % 4 == 3 ? far_w : two_w;
                }
            }
            if (x_scale) {
#pragma unroll
                for (int p = 0; p < PAIRS; ++p) nf[p] = *plus(x_scale + at + (row_of(0, p) - row_of(0, 0)), h);
            }
        } else { // rows past the end re-read the last (what they give is zeroed below)
#pragma unroll
            for (int p = 0; p < PAIRS; ++p) {
                const int64_t at = row_of(r0, p) + h < r_end ? row_of(r0, p) + h : r_end - 1;
#pragma unroll
                for (int t = 0; t < MI; ++t) nx[p][t] = X[at * ldx + cx[t]];
#pragma unroll
                for (int t = 0; t < NJ; ++t) np[p][t] = a.dHout[at * a.ldo + cg[t]];
#pragma unroll
                for (int t = 0; t < NJ; ++t) nw[p][t] = mask ? mask[at * a.mask_words + cw[t]] : 0u;
                nf[p] = x_scale ? x_scale[at] : 1.f;
            }
        }
    };

    floatx16 acc[MI][NJ];
    float accb[NJ]; // lanes 0..31: column sums
#pragma unroll
    for (int t = 0; t < NJ; ++t) accb[t] = 0.f;
    fetch(r_begin);
    auto step = [&](int64_t r0) {
        float x[PAIRS][MI], g[PAIRS][NJ];
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) {
#pragma unroll
            for (int t = 0; t < MI; ++t) x[p][t] = nx[p][t];
#pragma unroll
            for (int t = 0; t < NJ; ++t) g[p][t] = np[p][t];
        }
        if (x_scale) {
#pragma unroll
            for (int p = 0; p < PAIRS; ++p)
#pragma unroll
                for (int t = 0; t < MI; ++t) x[p][t] *= nf[p];
        }
        if (mask) { // the lane's bit, extended to a word
#pragma unroll
            for (int p = 0; p < PAIRS; ++p)
#pragma unroll
                for (int t = 0; t < NJ; ++t) g[p][t] = __int_as_float(__float_as_int(g[p][t]) & __builtin_amdgcn_sbfe((int)nw[p][t], m, 1));
        }
        if (r0 + ROWS > r_end) {
#pragma unroll
            for (int p = 0; p < PAIRS; ++p) {
                const bool there = row_of(r0, p) + h < r_end;
#pragma unroll
                for (int t = 0; t < MI; ++t) x[p][t] = there ? x[p][t] : 0.f;
#pragma unroll
                for (int t = 0; t < NJ; ++t) g[p][t] = there ? g[p][t] : 0.f;
            }
        }
        if (r0 + ROWS < r_end) fetch(r0 + ROWS);
#pragma unroll
        for (int p = 0; p < PAIRS; ++p)
#pragma unroll
            for (int ti = 0; ti < MI; ++ti)
#pragma unroll
                for (int tj = 0; tj < NJ; ++tj)
                    acc[ti][tj] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[p][ti], g[p][tj], acc[ti][tj], 0, 0, 0);
        if (sums) {
#pragma unroll
            for (int p = 0; p < PAIRS; ++p)
#pragma unroll
                for (int t = 0; t < NJ; ++t) accb[t] = (accb[t] + g[p][t]) + __shfl_xor(g[p][t], 32, 64); // rows in order
        }
    };
#pragma unroll
    for (int ti = 0; ti < MI; ++ti)
#pragma unroll
        for (int tj = 0; tj < NJ; ++tj) acc[ti][tj] = floatx16(0.f);
#pragma unroll 1
    for (int64_t r0 = r_begin; r0 < r_end; r0 += ROWS) step(r0);

    const int ww = a.w_in * a.w_out;
    float *out = a.partial + block * a.stride, *out_b = out + (a.compact ? ww : 2 * ww + (self ? a.w_out : 0));
    if (self) out += ww;
    if constexpr (SPLIT) {
        if (sums && h == 0) {
#pragma unroll
            for (int t = 0; t < NJ; ++t) bsum[wave][32 * t + m] = accb[t];
        }
#pragma unroll
        for (int ti = 0; ti < MI; ++ti)
#pragma unroll
            for (int tj = 0; tj < NJ; ++tj) {
#pragma unroll
                for (int r = 0; r < 16; ++r) red[wave][(8 * (r / 4) + 4 * h + (r % 4)) * 32 + m] = acc[ti][tj][r];
                __syncthreads();
                const int i = i_base + 32 * ti + (tid >> 3), j = j_base + 32 * tj + 4 * (tid & 7); // four columns of a row per thread
                floatx4 v = *reinterpret_cast<const floatx4 *>(&red[0][4 * tid]);
#pragma unroll
                for (int q = 1; q < 4; ++q) v += *reinterpret_cast<const floatx4 *>(&red[q][4 * tid]);
                if (i < a.w_in) {
                    float *o = out + (int64_t)i * a.w_out + j;
                    if (j + 4 <= a.w_out) *reinterpret_cast<floatx4_u *>(o) = v;
                    else
                        for (int c = 0; c < 3; ++c)
                            if (j + c < a.w_out) o[c] = v[c];
                }
                __syncthreads();
            }
        if (sums && tid < NJ * 32 && j_base + tid < a.w_out) out_b[j_base + tid] = ((bsum[0][tid] + bsum[1][tid]) + bsum[2][tid]) + bsum[3][tid];
    } else {
#pragma unroll
        for (int ti = 0; ti < MI; ++ti)
#pragma unroll
            for (int tj = 0; tj < NJ; ++tj)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int i = i_base + 32 * ti + 8 * (r / 4) + 4 * h + (r % 4), j = j_base + 32 * tj + m;
                    if (i < a.w_in && j < a.w_out) out[(int64_t)i * a.w_out + j] = acc[ti][tj][r];
                }
        if (sums && h == 0) {
#pragma unroll
            for (int t = 0; t < NJ; ++t)
                if (j_base + 32 * t + m < a.w_out) out_b[j_base + 32 * t + m] = accb[t];
        }
    }
}
template <int MI, int NJ, int WJ>
__global__ __launch_bounds__(256, 3) void grad_rows_kernel(const ReduceArgs common, const ReduceBatch batch, int n_tiles)
{
    grad_rows_tile<MI, NJ, WJ>(slice_of(common, batch, blockIdx.y), blockIdx.x, blockIdx.z == 1, n_tiles);
}

// Partial weight gradients of the narrowest layers (w_in, w_out <= 32, large n): every wavefront owns
// its own accumulators and every n_waves-th strip of 32 rows (so that the chip reads one contiguous
// window at a time), reads a strip with coalesced 16-byte loads into wave-private LDS tiles (the
// next strip's loads in flight during the MFMAs), and writes one partial result.  The node axis is the MFMA's k axis (lane (m, h) feeds
// column m of node row 2s + h).  No workgroup barrier; same output layout as grad_rows_kernel,
// one partial per wavefront.
__global__ __launch_bounds__(256) void grad_strip32_kernel(const ReduceArgs common, const ReduceBatch batch, int64_t n_waves)
{
    const ReduceArgs a = slice_of(common, batch, blockIdx.y);
    __shared__ __attribute__((aligned(16))) float Zs[4][32][32];
    __shared__ __attribute__((aligned(16))) float Hs[4][32][32];
    __shared__ __attribute__((aligned(16))) float Gs[4][32][32];
    __shared__ uint32_t Ms[4][32];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int m = lane & 31, h = lane >> 5;
    const int lr = lane >> 3, lc = (lane & 7) * 4;
    const int64_t w_id = (int64_t)blockIdx.x * 4 + wave;
    const int64_t n_strips = (a.n + 31) / 32, r_end = a.n;
    if (w_id >= n_waves) return; // uniform per wavefront; no barriers below (n_waves <= n_strips)
    const bool self = a.Hin != nullptr;
    const bool vz = aligned16(a.Z) && a.ldz % 4 == 0, vh = self && aligned16(a.Hin) && a.ldi % 4 == 0;
    const bool vg = aligned16(a.dHout) && a.ldo % 4 == 0;
    float (*zs)[32] = Zs[wave];
    float (*hs)[32] = Hs[wave];
    float (*gs)[32] = Gs[wave];
    uint32_t *ms = Ms[wave];

    floatx16 accA, accS;
#pragma unroll
    for (int r = 0; r < 16; ++r) { accA[r] = 0.f; accS[r] = 0.f; }
    float sum_p = 0.f, sum_g = 0.f; // column m of dP and of dHout over the node rows 2s + h

    float4 pz[4], ph[4], pg[4];
    float hf[4] = {1.f, 1.f, 1.f, 1.f}; // factors of the rows of Hin this lane loads (scaled layout); applied on the way to LDS
    uint32_t pw = ~0u;
    auto fetch = [&](int64_t r0) {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int64_t row = r0 + lr + 8 * it;
            float4 z = make_float4(0.f, 0.f, 0.f, 0.f), hh = z, g = z;
            if (row < r_end) {
                if (lc < a.w_in) {
                    z = load_k4(a.Z, a.ldz, row, lc, a.w_in, vz);
                    if (self) {
                        hh = load_k4(a.Hin, a.ldi, row, lc, a.w_in, vh);
                        if (a.hin_scale) hf[it] = a.hin_scale[row];
                    }
                }
                if (lc < a.w_out) g = load_k4(a.dHout, a.ldo, row, lc, a.w_out, vg);
            }
            pz[it] = z; ph[it] = hh; pg[it] = g;
        }
        if (a.mask && lane < 32) pw = r0 + lane < r_end ? a.mask[(r0 + lane) * a.mask_words] : 0u;
    };
    fetch(w_id * 32);
    for (int64_t strip = w_id; strip < n_strips; strip += n_waves) { // wavefront w takes strips w, w + n_waves, ...
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            if (a.hin_scale) scale4(ph[it], hf[it]);
            *reinterpret_cast<float4 *>(&zs[lr + 8 * it][lc]) = pz[it];
            *reinterpret_cast<float4 *>(&hs[lr + 8 * it][lc]) = ph[it];
            *reinterpret_cast<float4 *>(&gs[lr + 8 * it][lc]) = pg[it];
        }
        if (lane < 32) ms[lane] = pw;
        __builtin_amdgcn_wave_barrier();
        if (strip + n_waves < n_strips) fetch((strip + n_waves) * 32);
#pragma unroll
        for (int s2 = 0; s2 < 16; ++s2) {
            const int k = 2 * s2 + h;
            const float g = gs[k][m];
            const float p = ((ms[k] >> m) & 1u) ? g : 0.f;
            accA = __builtin_amdgcn_mfma_f32_32x32x2f32(zs[k][m], p, accA, 0, 0, 0);
            if (self) accS = __builtin_amdgcn_mfma_f32_32x32x2f32(hs[k][m], g, accS, 0, 0, 0);
            sum_p += p;
            sum_g += g;
        }
        __builtin_amdgcn_wave_barrier();
    }
    sum_p += __shfl_xor(sum_p, 32, 64);
    sum_g += __shfl_xor(sum_g, 32, 64);
    float *out = a.partial + w_id * a.stride;
    const int ww = a.w_in * a.w_out;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int i = 8 * (r / 4) + 4 * h + (r % 4);
        if (i < a.w_in && m < a.w_out) {
            out[i * a.w_out + m] = accA[r];
            if (!a.compact) out[ww + i * a.w_out + m] = accS[r];
        }
    }
    if (lane < 32 && m < a.w_out) {
        out[(a.compact ? ww : 2 * ww) + m] = sum_p;
        if (!a.compact) out[2 * ww + a.w_out + m] = sum_g;
    }
}

// Backward pass of a narrow layer (w_in, w_out <= 32, self term present, input gradient wanted) in one sweep over the
// node rows: the weight-gradient sums of grad_strip32_kernel and the two input-gradient products of
// pair_strip32_kernel<true, true> from the same wavefront-private tiles, so that dHout (and the mask) are read once
// instead of twice.  Per strip of 32 rows: Z, Hin and dHout go to LDS with coalesced 16-byte loads (the next strip's
// loads in flight behind the MFMAs); the node axis is the k axis of Z^T dP and Hin^T dHout (column reads of the
// tiles), the column axis that of dZ = dP W_agg^T and T = dHout W_self^T (row reads, weights in registers); dZ and T
// leave through the Z and Hin tiles as 16-byte stores.  Partial sums: one per wavefront, layout of
// grad_rows_kernel.  `a` carries the input-gradient half: B1 / B2 = W_agg / W_self (ldw), O1 = dZ (rows
// scaled by scale_o1), O2 = T, K = w_out, Nout = w_in.
__global__ __launch_bounds__(256, 2) void bwd_strip32_kernel(const ReduceArgs rcommon, const ReduceBatch rbatch, const PairArgs pcommon, const PairBatch pbatch,
                                                             int64_t n_waves)
{
    const ReduceArgs r = slice_of(rcommon, rbatch, blockIdx.y);
    const PairArgs a = slice_of(pcommon, pbatch);
    constexpr int ST = 36; // row stride: 16-byte row reads and 4-byte column reads are both conflict free
    __shared__ __attribute__((aligned(16))) float Zs[4][32][ST];
    __shared__ __attribute__((aligned(16))) float Hs[4][32][ST];
    __shared__ __attribute__((aligned(16))) float Gs[4][32][ST];
    __shared__ uint32_t Ms[4][32];
    __shared__ __attribute__((aligned(16))) float W1s[32][ST]; // W_agg and W_self, zero padded to 32 x 32: row i, k contiguous
    __shared__ __attribute__((aligned(16))) float W2s[32][ST];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int m = lane & 31, h = lane >> 5;
    const int lr = lane >> 3, lc = (lane & 7) * 4;
    for (int idx = threadIdx.x; idx < 32 * 32; idx += 256) {
        const int i = idx >> 5, kk = idx & 31;
        const bool ok = i < r.w_in && kk < r.w_out;
        W1s[i][kk] = ok ? a.B1[(int64_t)i * a.ldw + kk] : 0.f;
        W2s[i][kk] = ok ? a.B2[(int64_t)i * a.ldw + kk] : 0.f;
    }
    __syncthreads(); // the only workgroup barrier: before any wavefront leaves
    const int64_t w_id = (int64_t)blockIdx.x * 4 + wave;
    const int64_t n_strips = (r.n + 31) / 32, r_end = r.n;
    if (w_id >= n_waves) return; // uniform per wavefront (n_waves <= n_strips)
    const bool vz = aligned16(r.Z) && r.ldz % 4 == 0, vh = aligned16(r.Hin) && r.ldi % 4 == 0;
    const bool vg = aligned16(r.dHout) && r.ldo % 4 == 0;
    float (*zs)[ST] = Zs[wave];
    float (*hs)[ST] = Hs[wave];
    float (*gs)[ST] = Gs[wave];
    uint32_t *ms = Ms[wave];

    floatx16 accA, accS;
#pragma unroll
    for (int x = 0; x < 16; ++x) { accA[x] = 0.f; accS[x] = 0.f; }
    float sum_p = 0.f, sum_g = 0.f;

    float4 pz[4], ph[4], pg[4];
    float hf[4] = {1.f, 1.f, 1.f, 1.f};
    uint32_t pw = ~0u;
    float ps = 1.f; // scale_o1 of strip row m
    auto fetch = [&](int64_t r0) {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int64_t row = r0 + lr + 8 * it;
            float4 z = make_float4(0.f, 0.f, 0.f, 0.f), hh = z, g = z;
            if (row < r_end) {
                if (lc < r.w_in) {
                    z = load_k4(r.Z, r.ldz, row, lc, r.w_in, vz);
                    hh = load_k4(r.Hin, r.ldi, row, lc, r.w_in, vh);
                    if (r.hin_scale) hf[it] = r.hin_scale[row];
                }
                if (lc < r.w_out) g = load_k4(r.dHout, r.ldo, row, lc, r.w_out, vg);
            }
            pz[it] = z; ph[it] = hh; pg[it] = g;
        }
        if (lane < 32) pw = r0 + lane < r_end ? (r.mask ? r.mask[(r0 + lane) * r.mask_words] : ~0u) : 0u;
        if (a.scale_o1) ps = r0 + m < r_end ? a.scale_o1[r0 + m] : 1.f;
    };
    fetch(w_id * 32);
    for (int64_t strip = w_id; strip < n_strips; strip += n_waves) {
        const int64_t row0 = strip * 32;
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            if (r.hin_scale) scale4(ph[it], hf[it]);
            *reinterpret_cast<float4 *>(&zs[lr + 8 * it][lc]) = pz[it];
            *reinterpret_cast<float4 *>(&hs[lr + 8 * it][lc]) = ph[it];
            *reinterpret_cast<float4 *>(&gs[lr + 8 * it][lc]) = pg[it];
        }
        if (lane < 32) ms[lane] = pw;
        const float so = ps;
        __builtin_amdgcn_wave_barrier();
        if (strip + n_waves < n_strips) fetch((strip + n_waves) * 32); // flies during the MFMAs and the stores below
#pragma unroll 4
        for (int s2 = 0; s2 < 16; ++s2) { // node rows 2 s2 + h: Z^T dP, Hin^T dHout and the bias sums
            const int k = 2 * s2 + h;
            const float g = gs[k][m];
            const float p = ((ms[k] >> m) & 1u) ? g : 0.f;
            accA = __builtin_amdgcn_mfma_f32_32x32x2f32(zs[k][m], p, accA, 0, 0, 0);
            accS = __builtin_amdgcn_mfma_f32_32x32x2f32(hs[k][m], g, accS, 0, 0, 0);
            sum_p += p;
            sum_g += g;
        }
        __builtin_amdgcn_sched_barrier(0); // keep the two halves apart: interleaved they do not fit the register file
        floatx16 acc1, acc2;
#pragma unroll
        for (int x = 0; x < 16; ++x) { acc1[x] = 0.f; acc2[x] = 0.f; }
        const uint32_t word = ms[m];
#pragma unroll
        for (int q = 0; q < 4; ++q) { // columns 8 q + 4 h + i: dZ = dP W_agg^T and T = dHout W_self^T for strip row m
            const float4 g4 = *reinterpret_cast<const float4 *>(&gs[m][8 * q + 4 * h]);
            float4 p4 = g4; // dP = dHout * mask, times the row's output factor
            const uint32_t bits = word >> (8 * q + 4 * h);
            if (!(bits & 1u)) p4.x = 0.f;
            if (!(bits & 2u)) p4.y = 0.f;
            if (!(bits & 4u)) p4.z = 0.f;
            if (!(bits & 8u)) p4.w = 0.f;
            if (a.scale_o1) scale4(p4, so);
            const float4 w1 = *reinterpret_cast<const float4 *>(&W1s[m][8 * q + 4 * h]);
            const float4 w2 = *reinterpret_cast<const float4 *>(&W2s[m][8 * q + 4 * h]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc1 = __builtin_amdgcn_mfma_f32_32x32x2f32(pick(p4, i), pick(w1, i), acc1, 0, 0, 0);
                acc2 = __builtin_amdgcn_mfma_f32_32x32x2f32(pick(g4, i), pick(w2, i), acc2, 0, 0, 0);
            }
        }
        // dZ leaves through the Z tile and T through the Hin tile (register x of lane (m, h) is strip row
        // 8*(x/4) + 4*h + x%4, column m); layouts without 16-byte stores write the registers directly
        auto store_tile = [&](const floatx16 &o, float (*t)[ST], float *O, int64_t ldo, bool vec_ok) {
            if (vec_ok) {
#pragma unroll
                for (int x = 0; x < 16; ++x) t[8 * (x / 4) + 4 * h + (x % 4)][m] = o[x];
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int it = 0; it < 4; ++it) {
                    const int64_t row = row0 + lr + 8 * it;
                    if (row < r_end && lc < r.w_in)
                        *reinterpret_cast<float4 *>(O + row * ldo + lc) = *reinterpret_cast<const float4 *>(&t[lr + 8 * it][lc]);
                }
            } else {
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    const int64_t orow = row0 + 8 * (x / 4) + 4 * h + (x % 4);
                    if (orow < r_end && m < r.w_in) O[orow * ldo + m] = o[x];
                }
            }
        };
        const bool nout4 = r.w_in % 4 == 0;
        __builtin_amdgcn_wave_barrier(); // every lane is done reading the tiles
        store_tile(acc1, zs, a.O1, a.ldo1, nout4 && aligned16(a.O1) && a.ldo1 % 4 == 0);
        store_tile(acc2, hs, a.O2, a.ldo2, nout4 && aligned16(a.O2) && a.ldo2 % 4 == 0);
        __builtin_amdgcn_wave_barrier();
    }
    sum_p += __shfl_xor(sum_p, 32, 64);
    sum_g += __shfl_xor(sum_g, 32, 64);
    float *out = r.partial + w_id * r.stride;
    const int ww = r.w_in * r.w_out;
#pragma unroll
    for (int x = 0; x < 16; ++x) {
        const int i = 8 * (x / 4) + 4 * h + (x % 4);
        if (i < r.w_in && m < r.w_out) {
            out[i * r.w_out + m] = accA[x];
            out[ww + i * r.w_out + m] = accS[x];
        }
    }
    if (lane < 32 && m < r.w_out) {
        out[2 * ww + m] = sum_p;
        out[2 * ww + r.w_out + m] = sum_g;
    }
}

// The same for layers up to 64 wide (w_in <= 32 * MI, w_out <= 32 * NJ, large n): a wavefront owns the
// whole w_in x w_out gradient pair (2 * MI * NJ accumulators), so every operand row is read from
// memory exactly once.  Strips are dealt to the wavefronts round-robin, so at any moment the chip
// reads one contiguous window of the operands.  Short strips (8 node rows; 4, 16 and 32 are no
// faster, nor is keeping two or three strips in flight) keep the staging registers and the
// wave-private LDS tiles small enough for two wavefronts per SIMD beside the 128 accumulator
// registers of the full-width variant, three for the half-width ones.
// BLOCKS: the sums of grad_rows_kernel<.., 0> instead, for fewer rows: a workgroup takes rows_per_block rows, wavefront w the strips w, w + 4, ...
// of them, and the four sums are added in order; column sums in row order.  Both products from one read of dHout, with 16-byte loads:
// four slices of 169 k rows 64 x 64 172 -> 151 us, 32 x 64 107 -> 87.
template <int MI, int NJ, int SR, int WPS, bool SELF, bool NARROW, bool BLOCKS = false> // SR: node rows per strip; WPS: wavefronts per SIMD to compile for
__global__ __launch_bounds__(256, WPS) void grad_strip64_kernel(const ReduceArgs common, const ReduceBatch batch, int64_t n_waves)
{
    const ReduceArgs a = slice_of(common, batch, blockIdx.y);
    constexpr int WI = 32 * MI, WJ = 32 * NJ; // padded widths
    constexpr int LI = WI / 4, LJ = WJ / 4;   // lanes per row (16-byte accesses)
    constexpr int PI = SR * LI / 64, PJ = SR * LJ / 64; // passes over a strip
    __shared__ __attribute__((aligned(16))) float Zs[4][SR][WI];
    __shared__ __attribute__((aligned(16))) float Hs[4][SR][WI];
    __shared__ __attribute__((aligned(16))) float Gs[4][SR][WJ];
    __shared__ uint32_t Ms[4][SR][NJ];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int m = lane & 31, h = lane >> 5;
    const int ri = lane / LI, ci = (lane % LI) * 4; // coalesced layout of the w_in-wide operands
    const int rj = lane / LJ, cj = (lane % LJ) * 4; // and of dHout
    __shared__ __attribute__((aligned(16))) float red[BLOCKS ? 4 : 1][BLOCKS ? 32 * 32 : 1];
    __shared__ float bsum[BLOCKS ? 4 : 1][BLOCKS ? 2 * WJ : 1];
    const int64_t block_strips = a.rows_per_block / SR, left = (a.n + SR - 1) / SR - blockIdx.x * block_strips; // BLOCKS: strips of a block
    const int64_t w_id = BLOCKS ? blockIdx.x * block_strips + wave : (int64_t)blockIdx.x * 4 + wave, hop = BLOCKS ? 4 : n_waves;
    const int64_t past = BLOCKS ? blockIdx.x * block_strips + (left < block_strips ? left : block_strips) : (a.n + SR - 1) / SR; // strips end here
    const int64_t n_full = past * SR <= a.n ? past : past - 1; // whole strips before it
    if (!BLOCKS && w_id >= n_waves) return; // uniform per wavefront; no workgroup barriers in this form (no more wavefronts than strips)
    const LaneCols<NARROW> ic(ci, a.w_in), oc(cj, a.w_out);
    const bool place_i = a.w_in < WI, place_o = a.w_out < WJ; // uniform
    // what is absent is read from an operand and replaced, so that every strip has the same accesses
    const uint32_t *words = a.mask ? a.mask : reinterpret_cast<const uint32_t *>(a.dHout);
    const int64_t word_ld = a.mask ? a.mask_words : 0;
    const float *hs_f = SELF && a.hin_scale ? a.hin_scale : a.Z;
    const int64_t hs_ld = SELF && a.hin_scale ? 1 : 0;
    const int word = lane % NJ; // lane l < SR * NJ: word l % NJ of strip row l / NJ
    float (*zs)[WI] = Zs[wave];
    float (*hs)[WI] = Hs[wave];
    float (*gs)[WJ] = Gs[wave];
    uint32_t (*ms)[NJ] = Ms[wave];

    floatx16 accA[MI][NJ], accS[MI][NJ];
    float sum_p[NJ], sum_g[NJ]; // column 32 j + m of dP and of dHout over the node rows 2 s + h
#pragma unroll
    for (int j = 0; j < NJ; ++j) { sum_p[j] = 0.f; sum_g[j] = 0.f; }

    float4 pz[PI], ph[SELF ? PI : 1], pg[PJ];
    float hf[SELF ? PI : 1]; // factors of the rows of Hin this lane loads (scaled layout); applied on the way to LDS
    uint32_t pw;
    // (32-bit offsets within a strip: as many rows as come here would not fit into memory if eight of them did not lie within 4 GB)
    const uint32_t ldz = (uint32_t)a.ldz, ldi = (uint32_t)a.ldi, ldo = (uint32_t)a.ldo;
    auto fetch = [&](int64_t strip, auto whole) {
        const int64_t r0 = strip * SR;
        const int end = whole ? SR - 1 : (int)(a.n - 1 - r0);
        auto row = [&](int i) { return (uint32_t)(whole || i < end ? i : end); }; // rows past the end re-read the last
        constexpr int RI = 64 / LI, RJ = 64 / LJ;
#pragma unroll
        for (int it = 0; it < PI; ++it) {
            const int64_t r = r0 + (whole ? RI * it : 0);
            const uint32_t mine = row(whole ? ri : ri + RI * it);
            pz[it] = ic.load(plus(a.Z + r * a.ldz, mine * ldz));
            if (SELF) {
                ph[it] = ic.load(plus(a.Hin + r * a.ldi, mine * ldi));
                hf[it] = *plus(hs_f + r * hs_ld, mine * (uint32_t)hs_ld);
            }
        }
#pragma unroll
        for (int it = 0; it < PJ; ++it) pg[it] = oc.load(plus(a.dHout + (r0 + (whole ? RJ * it : 0)) * a.ldo, row(whole ? rj : rj + RJ * it) * ldo));
        pw = *plus(words + r0 * word_ld, row(lane / NJ % SR) * (uint32_t)word_ld + (32 * word < a.w_out && word_ld ? word : 0));
    };
    auto strip_step = [&](int64_t strip, int64_t next, auto whole, auto first) { // first: of the wavefront (the accumulators are the constant zero)
        constexpr bool WHOLE = decltype(whole)::value, FIRST = decltype(first)::value;
#pragma unroll
        for (int it = 0; it < PI; ++it) {
            if (place_i) {
                ic.place(pz[it]);
                if (SELF) ic.place(ph[it]);
            }
            if (SELF) scale4(ph[it], hs_ld ? hf[it] : 1.f);
            if (!WHOLE && strip * SR + ri + (64 / LI) * it >= a.n) {
                pz[it] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (SELF) ph[it] = pz[it];
            }
            *reinterpret_cast<float4 *>(&zs[ri + (64 / LI) * it][ci]) = pz[it];
            if (SELF) *reinterpret_cast<float4 *>(&hs[ri + (64 / LI) * it][ci]) = ph[it];
        }
#pragma unroll
        for (int it = 0; it < PJ; ++it) {
            if (place_o) oc.place(pg[it]);
            if (!WHOLE && strip * SR + rj + (64 / LJ) * it >= a.n) pg[it] = make_float4(0.f, 0.f, 0.f, 0.f);
            *reinterpret_cast<float4 *>(&gs[rj + (64 / LJ) * it][cj]) = pg[it];
        }
        if (lane < SR * NJ) ms[lane / NJ][word] = a.mask ? pw : ~0u;
        __builtin_amdgcn_wave_barrier();
        if (WHOLE) fetch(next, std::true_type());
        // the operands of two node rows are read while the two before them are multiplied
        float rg[2][NJ], rz[2][MI], rh[2][MI];
        uint32_t rw[2][NJ];
        auto read = [&](int s2) {
            const int k = 2 * s2 + h, at = s2 & 1;
#pragma unroll
            for (int j = 0; j < NJ; ++j) { rg[at][j] = gs[k][32 * j + m]; rw[at][j] = ms[k][j]; }
#pragma unroll
            for (int i = 0; i < MI; ++i) { rz[at][i] = zs[k][32 * i + m]; rh[at][i] = SELF ? hs[k][32 * i + m] : 0.f; }
        };
        read(0);
#pragma unroll
        for (int s2 = 0; s2 < SR / 2; ++s2) {
            if (s2 + 1 < SR / 2) read(s2 + 1);
            __builtin_amdgcn_sched_barrier(0);
            const int at = s2 & 1;
            float pp[NJ];
#pragma unroll
            for (int j = 0; j < NJ; ++j) { // the lane's bit of the word, extended to a word
                const float g = rg[at][j];
                pp[j] = __int_as_float(__float_as_int(g) & __builtin_amdgcn_sbfe((int)rw[at][j], m, 1));
                if constexpr (BLOCKS) { // rows in order
                    sum_p[j] = (sum_p[j] + pp[j]) + __shfl_xor(pp[j], 32, 64);
                    if (SELF) sum_g[j] = (sum_g[j] + g) + __shfl_xor(g, 32, 64);
                } else {
                    sum_p[j] += pp[j];
                    sum_g[j] += g;
                }
            }
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    accA[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(rz[at][i], pp[j], FIRST && s2 == 0 ? floatx16(0.f) : accA[i][j], 0, 0, 0);
                    if (SELF) accS[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(rh[at][i], rg[at][j], FIRST && s2 == 0 ? floatx16(0.f) : accS[i][j], 0, 0, 0);
                }
        }
        __builtin_amdgcn_wave_barrier();
    };
    int64_t strip = w_id; // wavefront w takes strips w, w + hop, ...
    auto ahead = [&](int64_t s) { return s + hop < n_full ? s + hop : s; };
    if (strip < n_full) {
        fetch(strip, std::true_type());
        strip_step(strip, ahead(strip), std::true_type(), std::true_type());
        strip += hop;
    } else {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) accA[i][j] = accS[i][j] = floatx16(0.f);
    }
#pragma unroll 1
    for (; strip < n_full; strip += hop) strip_step(strip, ahead(strip), std::true_type(), std::false_type());
    if (strip == n_full && strip < past) { // the rows left
        fetch(strip, std::false_type());
        strip_step(strip, 0, std::false_type(), std::false_type());
    }
    if constexpr (BLOCKS) {
        const int tid = threadIdx.x, ww = a.w_in * a.w_out;
        float *out = a.partial + (int64_t)blockIdx.x * a.stride;
        if (h == 0) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                bsum[wave][32 * j + m] = sum_p[j];
                bsum[wave][WJ + 32 * j + m] = sum_g[j];
            }
        }
#pragma unroll
        for (int s = 0; s < (SELF ? 2 : 1); ++s)
#pragma unroll
            for (int ti = 0; ti < MI; ++ti)
#pragma unroll
                for (int tj = 0; tj < NJ; ++tj) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) red[wave][(8 * (r / 4) + 4 * h + (r % 4)) * 32 + m] = s ? accS[ti][tj][r] : accA[ti][tj][r];
                    __syncthreads();
                    const int i = 32 * ti + (tid >> 3), j = 32 * tj + 4 * (tid & 7); // four columns of a row per thread
                    floatx4 v = *reinterpret_cast<const floatx4 *>(&red[0][4 * tid]);
#pragma unroll
                    for (int q = 1; q < 4; ++q) v += *reinterpret_cast<const floatx4 *>(&red[q][4 * tid]);
                    if (i < a.w_in) store_cols4<false>(out + s * ww + (int64_t)i * a.w_out + j, make_float4(v[0], v[1], v[2], v[3]), true, a.w_out - j);
                    __syncthreads();
                }
        const int q = tid / WJ, col = tid % WJ; // 0: sums of dP, 1: of dHout
        if (q < (SELF ? 2 : 1) && col < a.w_out)
            out[(a.compact ? ww : 2 * ww) + q * a.w_out + col] = ((bsum[0][tid] + bsum[1][tid]) + bsum[2][tid]) + bsum[3][tid];
        return;
    }
    float *out = a.partial + w_id * a.stride;
    const int ww = a.w_in * a.w_out;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = 32 * i + 8 * (r / 4) + 4 * h + (r % 4), col = 32 * j + m;
                if (row < a.w_in && col < a.w_out) {
                    out[row * a.w_out + col] = accA[i][j][r];
                    if (!a.compact) out[ww + row * a.w_out + col] = accS[i][j][r];
                }
            }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const float sp = sum_p[j] + __shfl_xor(sum_p[j], 32, 64);
        const float sg = sum_g[j] + __shfl_xor(sum_g[j], 32, 64);
        const int col = 32 * j + m;
        if (lane < 32 && col < a.w_out) {
            out[(a.compact ? ww : 2 * ww) + col] = sp;
            if (!a.compact) out[2 * ww + a.w_out + col] = sg;
        }
    }
}

// Partial weight gradient of a single product (compact layout: [X^T dP | colsum dP]) for wide
// layers: one workgroup per 128 x 128 output tile and block of rows_per_block rows, each wavefront owning a
// 64 x 64 quarter (four MFMA accumulators).  Per step 32 rows of the X tile and of the dP tile are
// staged in LDS (the next step's loads are issued into registers before this step's MFMAs); the
// node axis is the MFMA's k axis.  32 flop per staged byte instead of 8 for 32 x 32 tiles.  The tiles of a row block run back to back on
// one XCD (grid as in grad_rows_kernel).  Loads are unconditional, in one form per kernel, and columns are moved into place and activation bits applied on
// the way to LDS, each in one branch a step: with two forms of loads behind a test a step of a tile that is not full waited for its own accesses (1 M rows
// 65 x 65 401 -> 320 us, 324 k rows 70 x 280 395 -> 325, 400 k rows 128 x 128 178 -> 161, 169 k rows 256 x 256 240 -> 230; 408 k rows 264 x 84, five workgroups on some
// CUs, 452 -> 426).  Three wavefronts per SIMD (two: 2 % slower), one buffer (two, with half the barriers: 6 %).
constexpr int GB_T = 128;

template <bool NEAR> // a step's rows lie within 32-bit offsets
__global__ __launch_bounds__(256, 3) void grad_big_mfma_kernel(const ReduceArgs common, const ReduceBatch batch, int n_tiles)
{
    const ReduceArgs a = slice_of(common, batch, blockIdx.y);
    const TilePlace place = tile_place(blockIdx.x, n_tiles);
    const int col_tile = __builtin_amdgcn_readfirstlane(place.col_tile);
    const int64_t block = (uint32_t)__builtin_amdgcn_readfirstlane(place.row_tile);
    __shared__ __attribute__((aligned(16))) float Xs[RED_RK][GB_T];
    __shared__ __attribute__((aligned(16))) float Ps[RED_RK][GB_T];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int m = lane & 31, h = lane >> 5;
    const int i_base = col_tile / common.j_tiles * GB_T, j_base = col_tile % common.j_tiles * GB_T;
    const int wi = (wave >> 1) * 64, wj = (wave & 1) * 64;
    const int64_t r_begin = block * a.rows_per_block;
    if (r_begin >= a.n) return; // uniform per workgroup
    const int64_t r_end = r_begin + a.rows_per_block < a.n ? r_begin + a.rows_per_block : a.n;
    const bool bias_wave = i_base == 0 && (wave >> 1) == 0;
    // this thread's four columns of the tiles, of rows tid / 32, tid / 32 + 8, ... of a step
    const int c4 = (tid & 31) * 4, lr = tid >> 5;
    const LaneCols<> xc(i_base + c4, a.w_in), pc(j_base + c4, a.w_out);
    const bool place_x = i_base + GB_T > a.w_in, place_p = j_base + GB_T > a.w_out; // uniform
    const int j = j_base + c4 < a.w_out ? j_base + c4 : a.w_out - 1;
    const uint32_t *words = a.mask ? a.mask : reinterpret_cast<const uint32_t *>(a.dHout); // none: read anything, use all ones
    const int word = a.mask ? j >> 5 : 0;
    const int64_t word_ld = a.mask ? a.mask_words : 0;

    floatx16 acc[2][2];
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int tj = 0; tj < 2; ++tj)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[ti][tj][r] = 0.f;
    float accb = 0.f; // column j_base + wj + lane of dP

    float4 rx[4], rp[4];
    uint32_t rw[4];
    const uint32_t ox = (uint32_t)lr * (uint32_t)a.ldz, op = (uint32_t)lr * (uint32_t)a.ldo, ow = (uint32_t)lr * (uint32_t)word_ld;
    auto fetch = [&](int64_t r0, auto whole) {
        if (whole && NEAR) {
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int64_t r = r0 + 8 * it;
                rx[it] = xc.load(plus(a.Z + r * a.ldz, ox));
                rp[it] = pc.load(plus(a.dHout + r * a.ldo, op));
                rw[it] = *plus(words + r * word_ld, ow + word);
            }
        } else {
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int64_t r = r0 + lr + 8 * it, row = whole || r < r_end ? r : r_end - 1; // rows past the end re-read the last
                rx[it] = xc.load(a.Z + row * a.ldz);
                rp[it] = pc.load(a.dHout + row * a.ldo);
                rw[it] = words[row * word_ld + word];
            }
        }
    };
    // `next`: first row to fetch meanwhile.  The activation bits are applied on the way to LDS, not where they are fetched: the next
    // step's accesses stay in flight behind this one's products.
    auto step = [&](int64_t r0, int64_t next, auto whole, auto more) {
        if (place_x) {
#pragma unroll
            for (int it = 0; it < 4; ++it) xc.place(rx[it]);
        }
        if (place_p) {
#pragma unroll
            for (int it = 0; it < 4; ++it) pc.place(rp[it]);
        }
        if (a.mask) { // a bit of the word, extended to a word
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                auto masked = [&](float v, int c) { return __int_as_float(__float_as_int(v) & __builtin_amdgcn_sbfe((int)rw[it], (j & 31) + c, 1)); };
                rp[it] = make_float4(masked(rp[it].x, 0), masked(rp[it].y, 1), masked(rp[it].z, 2), masked(rp[it].w, 3));
            }
        }
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            if (!whole && r0 + lr + 8 * it >= r_end) rx[it] = rp[it] = make_float4(0.f, 0.f, 0.f, 0.f);
            *reinterpret_cast<float4 *>(&Xs[lr + 8 * it][c4]) = rx[it];
            *reinterpret_cast<float4 *>(&Ps[lr + 8 * it][c4]) = rp[it];
        }
        __syncthreads();
        if constexpr (decltype(more)::value) fetch(next, std::true_type());
        float xs[2][2], ps[2][2]; // the operands of two node rows are read while the two before them are multiplied
        auto read = [&](int kp) {
            const int k = 2 * kp + h;
#pragma unroll
            for (int t = 0; t < 2; ++t) { xs[kp & 1][t] = Xs[k][wi + 32 * t + m]; ps[kp & 1][t] = Ps[k][wj + 32 * t + m]; }
        };
        read(0);
#pragma unroll
        for (int kp = 0; kp < RED_RK / 2; ++kp) {
            if (kp + 1 < RED_RK / 2) read(kp + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ti = 0; ti < 2; ++ti)
#pragma unroll
                for (int tj = 0; tj < 2; ++tj) acc[ti][tj] = __builtin_amdgcn_mfma_f32_32x32x2f32(xs[kp & 1][ti], ps[kp & 1][tj], acc[ti][tj], 0, 0, 0);
        }
        if (bias_wave) {
#pragma unroll
            for (int r = 0; r < RED_RK; ++r) accb += Ps[r][wj + lane];
        }
        __syncthreads();
    };
    int64_t r0 = r_begin;
    if (r0 + RED_RK <= r_end) fetch(r0, std::true_type());
#pragma unroll 1
    for (; r0 + RED_RK <= r_end; r0 += RED_RK) step(r0, r0 + 2 * RED_RK <= r_end ? r0 + RED_RK : r0, std::true_type(), std::true_type());
    if (r0 < r_end) { // the rows left
        fetch(r0, std::false_type());
        step(r0, 0, std::false_type(), std::false_type());
    }

    float *out = a.partial + block * a.stride;
#pragma unroll
    for (int ti = 0; ti < 2; ++ti)
#pragma unroll
        for (int tj = 0; tj < 2; ++tj)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int i = i_base + wi + 32 * ti + 8 * (r / 4) + 4 * h + (r % 4);
                const int j = j_base + wj + 32 * tj + m;
                if (i < a.w_in && j < a.w_out) out[i * a.w_out + j] = acc[ti][tj][r];
            }
    if (bias_wave) {
        const int j = j_base + wj + lane;
        if (j < a.w_out) out[a.w_in * a.w_out + j] = accb;
    }
}

// Column sums of an n x w matrix (slice-encoding gradient): partial[block][w].
__global__ __launch_bounds__(256) void colsum_partial_kernel(const float *__restrict__ M, int64_t ld, int64_t n, int32_t w,
                                                             float *__restrict__ partial)
{
    const int64_t r_begin = (int64_t)blockIdx.x * RED_ROWS;
    const int64_t r_end = r_begin + RED_ROWS < n ? r_begin + RED_ROWS : n;
    // thread t owns column (t % cw) of every (256 / cw)-th row, cw = columns rounded up to a power of two <= 256
    __shared__ float red[256];
    for (int c0 = 0; c0 < w; c0 += 256) {
        const int cols = w - c0 < 256 ? w - c0 : 256;
        int cw = 1;
        while (cw < cols) cw <<= 1;
        const int lanes_r = 256 / cw;
        const int c = threadIdx.x % cw, rr = threadIdx.x / cw;
        float acc = 0.f;
        if (c < cols)
            for (int64_t r = r_begin + rr; r < r_end; r += lanes_r) acc += M[r * ld + c0 + c];
        red[threadIdx.x] = acc;
        __syncthreads();
        if (rr == 0 && c < cols) {
            float s = 0.f;
            for (int q = 0; q < lanes_r; ++q) s += red[q * cw + c];
            partial[(int64_t)blockIdx.x * w + c0 + c] = s;
        }
        __syncthreads();
    }
}

// Same sums with 16-byte loads (aligned base, ld % 4 == 0, w % 4 == 0): thread t owns four
// columns of every (256 / q)-th row, q = float4 per row rounded up to a power of two.
__global__ __launch_bounds__(256) void colsum_partial_vec_kernel(const float *__restrict__ M, int64_t ld, int64_t n, int32_t w,
                                                                 float *__restrict__ partial)
{
    const int64_t r_begin = (int64_t)blockIdx.x * RED_ROWS;
    const int64_t r_end = r_begin + RED_ROWS < n ? r_begin + RED_ROWS : n;
    __shared__ float4 red[256];
    for (int c0 = 0; c0 < w; c0 += 1024) {
        const int cols4 = (w - c0 < 1024 ? w - c0 : 1024) >> 2;
        int q = 1;
        while (q < cols4) q <<= 1;
        const int lanes_r = 256 / q;
        const int c = threadIdx.x % q, rr = threadIdx.x / q;
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        if (c < cols4) {
            const float *p = M + c0 + c * 4;
            int64_t r = r_begin + rr;
            for (; r + 3 * lanes_r < r_end; r += 4 * lanes_r) {
                const float4 v0 = *reinterpret_cast<const float4 *>(p + r * ld);
                const float4 v1 = *reinterpret_cast<const float4 *>(p + (r + lanes_r) * ld);
                const float4 v2 = *reinterpret_cast<const float4 *>(p + (r + 2 * lanes_r) * ld);
                const float4 v3 = *reinterpret_cast<const float4 *>(p + (r + 3 * lanes_r) * ld);
                acc.x += v0.x; acc.y += v0.y; acc.z += v0.z; acc.w += v0.w;
                acc.x += v1.x; acc.y += v1.y; acc.z += v1.z; acc.w += v1.w;
                acc.x += v2.x; acc.y += v2.y; acc.z += v2.z; acc.w += v2.w;
                acc.x += v3.x; acc.y += v3.y; acc.z += v3.z; acc.w += v3.w;
            }
            for (; r < r_end; r += lanes_r) {
                const float4 v = *reinterpret_cast<const float4 *>(p + r * ld);
                acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
            }
        }
        red[threadIdx.x] = acc;
        __syncthreads();
        if (rr == 0 && c < cols4) {
            float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
            for (int k = 0; k < lanes_r; ++k) {
                const float4 v = red[k * q + c];
                s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
            }
            *reinterpret_cast<float4 *>(partial + (int64_t)blockIdx.x * w + c0 + c * 4) = s;
        }
        __syncthreads();
    }
}

// 32 elements x 32 runs of blocks per workgroup
__global__ __launch_bounds__(1024) void reduce_final_kernel(const FinalWork f) { final_sum<1024>(f, blockIdx.x, blockIdx.y); }

inline int64_t red_blocks(int64_t n) { return (n + RED_ROWS - 1) / RED_ROWS; }

// Node rows per partial sum of a slice layer's weight gradients: RED_ROWS, or a quarter of it when that would give fewer than
// 2048 workgroups of one 32 x 32 tile each (a workgroup walks its rows in dependent steps, so on small graphs shorter walks in more
// workgroups finish sooner: cfg2 80 -> 35 us with such tiles).  grad_rows_kernel takes up to 64 x 64 a workgroup; the line stays where
// it is all the same, since the rows of a sum decide a gradient's last bits.
inline int32_t layer_grad_rows(int64_t n, int32_t w_in, int32_t w_out)
{
    const int64_t tiles = (int64_t)((w_in + RED_TILE - 1) / RED_TILE) * ((w_out + RED_TILE - 1) / RED_TILE);
    return red_blocks(n) * tiles < 2048 ? RED_ROWS / 4 : RED_ROWS;
}
inline int64_t layer_grad_blocks(int64_t n, int32_t w_in, int32_t w_out)
{
    const int32_t rows = layer_grad_rows(n, w_in, w_out);
    return (n + rows - 1) / rows;
}

// How the weight gradients of a slice layer are formed: by which kernel, and in how many partial sums.  A function of the
// sizes alone: the rows that go into one fp32 chain, and so the bits of a gradient, do not depend on the launch.
struct GradPlan {
    enum Kind { STRIP32, STRIP64, TILED } kind;
    int64_t partials;
    int32_t rows; // TILED: node rows per workgroup
};
inline GradPlan grad_plan(int64_t n, int32_t w_in, int32_t w_out)
{
    const int64_t nb = layer_grad_blocks(n, w_in, w_out);
    if (w_in <= 32 && w_out <= 32 && n >= 65536) { // one partial sum per wavefront
        const int64_t strips = (n + 31) / 32, waves = nb < 8192 ? nb : 8192;
        return GradPlan{GradPlan::STRIP32, waves < strips ? waves : strips, 0};
    }
    if (w_in <= 64 && w_out <= 64 && n >= ((int64_t)1 << 21)) {
        // whole waves of resident workgroups (256 CUs x 3 workgroups x 4 wavefronts) where there are as many blocks
        const int64_t resident = 3072;
        const int64_t waves = nb >= resident ? nb / resident * resident : nb >= 2048 ? 2048 : nb;
        const int64_t strips = (n + 7) / 8; // strips of 8 rows in every variant launched here
        return GradPlan{GradPlan::STRIP64, waves < strips ? waves : strips, 0};
    }
    return GradPlan{GradPlan::TILED, nb, layer_grad_rows(n, w_in, w_out)};
}

// A dense layer's weight and bias gradients: by grad_rows_kernel or, where both widths are large, in 128 x 128 tiles (`big`: layers
// wider than 64; see grad_form), a partial sum per RED_ROWS node rows.  On few rows that leaves most of the chip idle behind
// chains of RED_ROWS rows, so up to SMALL_LINEAR elements of the wider operand the rows are split until 512 workgroups of one tile are
// there or a workgroup is down to one step, as far as the workspace has room (`capacity` partial sums; the least workspace leaves
// RED_ROWS): the last bits of these gradients depend on it.  Split / in chains of 1024, 96 -> 96: 1000 rows 11 / 57 us, 5000 rows
// 14 / 58, 5461 rows (the line) 14 / 53.
// The line is not where splitting stops paying (8000 rows 17 / 58, 40 000 30 / 58, 160 000 67 / 122; 256 -> 256 from 160 000 rows
// on 256 either way).  Above it the sums keep the order they have with every workspace: an update carries a gradient's last bits
// into the next forward pass, where a few activations in 10^8 lie within rounding of zero and, passing or not, change a whole
// term.  Up to 2^19 elements that is one activation in a hundred passes.
struct LinearGradPlan {
    bool big;
    int32_t rows;
    int64_t partials;
};
constexpr int64_t NO_LIMIT = (int64_t)1 << 40, SMALL_LINEAR = (int64_t)1 << 19;
inline LinearGradPlan linear_grad_plan(int64_t n, int32_t w_in, int32_t w_out, int64_t capacity)
{
    LinearGradPlan p;
    p.big = w_in > 64 || w_out > 64;
    int64_t rows = RED_ROWS;
    if (n * (w_in > w_out ? w_in : w_out) <= SMALL_LINEAR) {
        const int32_t t = p.big ? GB_T : RED_TILE;
        const int64_t tiles = (int64_t)((w_in + t - 1) / t) * ((w_out + t - 1) / t);
        const int64_t fine = round_up(n * tiles / 512 + 1, RED_RK), least = round_up((n + capacity - 1) / capacity, RED_RK);
        if (fine < rows) rows = fine > least ? fine : least;
    }
    p.rows = (int32_t)rows;
    p.partials = (n + rows - 1) / rows;
    return p;
}

// launch(self, narrow) with both as constants; narrow: a row of an operand is too short for 16-byte loads
template <class F> void launch_grad_strip(bool self, bool narrow, F launch)
{
    if (self && narrow) launch(std::true_type(), std::true_type());
    else if (self) launch(std::true_type(), std::false_type());
    else if (narrow) launch(std::false_type(), std::true_type());
    else launch(std::false_type(), std::false_type());
}

// Which kernel forms the partial weight gradients (r.rows_per_block rows a workgroup), with how many workgroups per slice and product
struct GradForm {
    enum Kernel { STRIPS, LDS, ROWS } kernel;
    int64_t blocks;
    int mi, nj, wj;       // ROWS: its template arguments
    int j_tiles, n_tiles; // LDS, ROWS: output tiles along w_out, and in all
};
inline GradForm grad_form(const ReduceArgs &r, int batch, int products, bool big, bool from_lds = true) // from_lds: LDS where it pays alone
{
    int mi = r.w_in > 32 ? 2 : 1, nj = r.w_out > 32 ? 2 : 1;
    const int64_t n_blocks = (r.n + r.rows_per_block - 1) / r.rows_per_block;
    // From enough workgroups on: a workgroup does both products, so there are half as many or fewer (pairs 64 x 64, strips / grad_rows_kernel:
    // 79 workgroups 21.5 / 16.3 us, 157 22.9 / 23.3, 235 24.0 / 30.2, 662 47.3 / 57.5; single products 127 36.3 / 31.8, 977 121 / 147).
    if (!big && r.w_in <= 64 && r.w_out <= 64 && r.w_in >= 4 && r.w_out >= 4 && n_blocks * batch >= (products == 2 ? 160 : 512))
        return GradForm{GradForm::STRIPS, n_blocks, mi, nj, 0, 1, 1};
    auto tiled = [&](GradForm::Kernel kernel, int ti, int tj, int wj) { // output tiles of ti x tj per workgroup
        const int j_tiles = (r.w_out + tj - 1) / tj, n_tiles = (r.w_in + ti - 1) / ti * j_tiles;
        return GradForm{kernel, (n_blocks + 7) / 8 * 8 * n_tiles, mi, nj, wj, j_tiles, n_tiles};
    };
    // both wide: operands are re-read so often that staging them in LDS pays once there are enough 128 x 128 tiles for the chip
    // (from LDS / from registers: 2.4 M rows 256 x 256 2.95 / 5.36 ms; 169 k rows 128 x 128, 166 tiles, 106 / 153 us; 98 tiles 104 / 106;
    // 49 tiles 100 / 65)
    if (from_lds && big && r.w_in > 64 && r.w_out > 64) {
        const GradForm f = tiled(GradForm::LDS, GB_T, GB_T, 0);
        if (n_blocks * f.n_tiles * batch >= 128) return f;
    }
    // Tiles of 64 x 64 per workgroup or wavefront as far as the widths go; 32 x 32, whose operands are loaded twice as often, where
    // those would leave fewer than two workgroups per CU.
    const int64_t tiles = (int64_t)((r.w_in + 32 * mi - 1) / (32 * mi)) * ((r.w_out + 32 * nj - 1) / (32 * nj));
    if (n_blocks * tiles * products * batch < (big ? 4 : 1) * 512) mi = nj = 1;
    if (!big) return tiled(GradForm::ROWS, 32 * mi, 32 * nj, 0);
    // the wavefronts of a workgroup share their operands through L1: along both widths, or along w_in if one covers w_out
    if (r.w_out <= 32 * nj) return tiled(GradForm::ROWS, 128 * mi, 32 * nj, 1);
    return tiled(GradForm::ROWS, 64 * mi, 64 * nj, 2);
}

template <int WJ> void launch_grad_tiles(const GradForm &f, const ReduceArgs &r, const ReduceBatch &b, dim3 grid, hipStream_t stream)
{
    if (f.mi == 1 && f.nj == 1) grad_rows_kernel<1, 1, WJ><<<grid, 256, 0, stream>>>(r, b, f.n_tiles);
    else if (f.mi == 1) grad_rows_kernel<1, 2, WJ><<<grid, 256, 0, stream>>>(r, b, f.n_tiles);
    else if (f.nj == 1) grad_rows_kernel<2, 1, WJ><<<grid, 256, 0, stream>>>(r, b, f.n_tiles);
    else grad_rows_kernel<2, 2, WJ><<<grid, 256, 0, stream>>>(r, b, f.n_tiles);
}
int launch_grad_rows(ReduceArgs r, const ReduceBatch &b, int batch, int products, bool big, hipStream_t stream)
{
    const GradForm f = grad_form(r, batch, products, big);
    SG_REQUIRE(f.blocks <= INT32_MAX, SLICEGCN_ERANGE, "weight gradients: grid too large");
    r.j_tiles = f.j_tiles;
    dim3 grid((unsigned)f.blocks, (unsigned)batch);
    switch (f.kernel) {
    case GradForm::STRIPS:
        launch_grad_strip(products == 2, false, [&](auto s, auto) {
            if (f.mi == 1 && f.nj == 1) grad_strip64_kernel<1, 1, 8, 3, s.value, false, true><<<grid, 256, 0, stream>>>(r, b, 0);
            else if (f.mi == 1) grad_strip64_kernel<1, 2, 8, 3, s.value, false, true><<<grid, 256, 0, stream>>>(r, b, 0);
            else if (f.nj == 1) grad_strip64_kernel<2, 1, 8, 3, s.value, false, true><<<grid, 256, 0, stream>>>(r, b, 0);
            else grad_strip64_kernel<2, 2, 8, 2, s.value, false, true><<<grid, 256, 0, stream>>>(r, b, 0);
        });
        break;
    case GradForm::LDS:
        if (r.ldz < (1 << 24) && r.ldo < (1 << 24) && r.mask_words < (1 << 24)) grad_big_mfma_kernel<true><<<grid, 256, 0, stream>>>(r, b, f.n_tiles);
        else grad_big_mfma_kernel<false><<<grid, 256, 0, stream>>>(r, b, f.n_tiles);
        break;
    case GradForm::ROWS:
        grid.z = (unsigned)products;
        if (f.wj == 0) launch_grad_tiles<0>(f, r, b, grid, stream);
        else if (f.wj == 1) launch_grad_tiles<1>(f, r, b, grid, stream);
        else launch_grad_tiles<2>(f, r, b, grid, stream);
        break;
    }
    SG_LAUNCH_CHECK();
    return SLICEGCN_OK;
}

// Weight gradients and the products of the input gradients read the same dHout and do not depend on each other: on few rows, where
// either is a chain of a few dependent loads in a fraction of the chip, one launch does both.  The first `grads` workgroups of a slice form
// weight gradients (products x grad_x), the others what pair_strip32_kernel or pair_rows_kernel would.  Backward passes of dense
// layers, in two launches / one: 1000 rows 64 -> 8 10.1 / 6.8 us, 2048 rows 64 -> 64 11.9 / 8.8, 20 k rows 64 -> 64 27.2 / 23.1, 60 k rows
// 256 -> 64 99 / 90, 100 k rows 64 -> 64 49.6 / 41.1, 169 k rows 256 -> 40 152 / 145 (with the two
// kinds of workgroups in turn half as long again: the long ones have to start first).  The two products of a slice layer, dZ and T, are workgroups of
// their own (pair_x each): half the chain, and nothing is shared but dHout.  Backward passes of slice layers, two launches / one / one with the
// products apart: 2048 rows 64 -> 32 18.5 / 12.9 / 13.0 us, 30 k rows 64 -> 64 39.5 / 35.9 / 33.6, 5000 rows 64 -> 64 22.3 / 17.8 / 15.7.
template <int WJ, int NT> // NT: tiles of 32 columns, 0 for the strips
__global__ __launch_bounds__(256, 3) void grad_pair_kernel(const ReduceArgs r, const ReduceBatch rb, const PairArgs p, const PairBatch pb,
                                                           uint32_t grad_x, uint32_t grads, int n_tiles, uint32_t pair_x, int n_col)
{
    const uint32_t wg = blockIdx.x;
    if (wg < grads) {
        const bool self = wg >= grad_x;
        grad_rows_tile<1, 1, WJ>(slice_of(r, rb, blockIdx.y), self ? wg - grad_x : wg, self, n_tiles);
        return;
    }
    PairArgs a = slice_of(p, pb);
    uint32_t at = wg - grads;
    if (at >= pair_x) {
        at -= pair_x;
        a.B1 = a.B2; a.O1 = a.O2; a.ldo1 = a.ldo2; a.mask = nullptr; a.scale_o1 = nullptr;
    }
    if constexpr (NT == 0) pair_strip32<true, false>(a, at, pair_x);
    else pair_rows_tile<NT, false, true>(a, at, n_col);
}

// Whether the n x w rows at o, in leading dimension ldo, may share memory with those at x, by the address ranges from first to last element:
// column ranges of one wide matrix count as shared, though nothing overlaps, and are worked on in two launches
inline bool may_share(const void *o, int64_t ldo, int64_t wo, const void *x, int64_t ldx, int64_t wx, int64_t n)
{
    const uintptr_t p = reinterpret_cast<uintptr_t>(o), q = reinterpret_cast<uintptr_t>(x);
    return o && x && p < q + 4 * ((n - 1) * ldx + wx) && q < p + 4 * ((n - 1) * ldo + wo);
}

constexpr int64_t LONG_PRODUCT = 72000000; // elements of the input gradient
// launch_grad_rows, and launch_pair<true> for `list` in the same launch where the gradients take their smallest tiles, which leave the chip
// idle (with larger ones 2.4 M rows 256 -> 47 take 2.86 ms together and 2.64 apart; up to 32 -> 3, where they are the only tiles, one launch is
// faster on any number of rows: 32 -> 2, 169 k rows 31.2 / 24.1 us, 800 k 70 / 55, 2.4 M 196 / 184), and nothing that is stored is read by the other (an
// input gradient may take the place of an operand); `pair_done` says whether it was.  Not where the input gradient alone is
// pair_wide_kernel's and long (together / apart: 262 k rows 128 -> 40 121 / 126 us, 350 k 154 / 158, 450 k 207 / 204, 600 k 265 / 250, 1 M 441 / 398, 233 k 256 -> 41
// 212 / 206, 300 k 264 / 252, 500 k 432 / 394, 200 k 512 -> 40 347 / 335; 700 k 100 -> 36 299 / 306, 1 M 100 -> 64 444 / 442,
// 128 -> 28 356 / 319; but fewer steps 600 k 128 -> 20 194 / 201, 400 k 224 -> 16 without activation bits 233 / 248, and two tiles a workgroup 300 k 310 -> 40 300 / 315).  A layer whose gradients are cut into chains shorter
// than RED_ROWS leaves the LDS form for it (5000 rows 96 -> 96 19.5 / 14.9 us, 2048 rows 256 -> 256 34.7 / 30.3).
int launch_grads_and_pair(const ReduceArgs &r, const ReduceBatch &b, int batch, int products, bool big, const PairArgs *list, bool *pair_done,
                          hipStream_t stream)
{
    *pair_done = false;
    if (!list) return launch_grad_rows(r, b, batch, products, big, stream);
    const GradForm g = grad_form(r, batch, products, big, r.rows_per_block == RED_ROWS);
    const PairForm f = pair_form(list, batch, true, false);
    const PairForm alone = pair_form(list, batch, true);
    const bool apart = alone.kernel == PairForm::WIDE && alone.nt > 2 && list[0].K >= 24 && r.n * batch * list[0].Nout >= LONG_PRODUCT;
    bool merge = !apart && g.kernel == GradForm::ROWS && g.mi == 1 && g.nj == 1 &&
                 (f.kernel == PairForm::STRIP32 || (f.kernel == PairForm::ROWS && (f.nt == 1 || (f.nt == 2 && g.wj != 0)))) &&
                 products * g.blocks + 2 * f.blocks <= MAX_GRID;
    for (int i = 0; merge && i < batch; ++i)
        for (int q = 0; merge && q < batch; ++q)
            for (int o = 0; o < 2; ++o) {
                const float *out = o ? list[i].O2 : list[i].O1;
                const int64_t ldo = o ? list[i].ldo2 : list[i].ldo1;
                auto reads = [&](const void *x, int64_t ldx, int64_t wx) { return may_share(out, ldo, list[i].Nout, x, ldx, wx, r.n); };
                if (reads(b.p[q].Z, r.ldz, r.w_in) || reads(b.p[q].Hin, r.ldi, r.w_in) || reads(b.p[q].dHout, r.ldo, r.w_out) ||
                    reads(b.p[q].mask, r.mask_words, (r.w_out + 31) / 32))
                    merge = false;
            }
    if (!merge) return launch_grad_rows(r, b, batch, products, big, stream);
    ReduceArgs t = r;
    t.j_tiles = g.j_tiles;
    const PairBatch pb = pair_batch(list, batch);
    const uint32_t grad_x = (uint32_t)g.blocks, grads = grad_x * products;
    const uint32_t pair_x = (uint32_t)f.blocks;
    const dim3 grid(grads + pair_x * (f.two && list[0].O2 ? 2 : 1), (unsigned)batch);
    auto launch = [&](auto wj, auto nt) {
        grad_pair_kernel<wj.value, nt.value><<<grid, 256, 0, stream>>>(t, b, list[0], pb, grad_x, grads, g.n_tiles, pair_x, f.n_col);
    };
    const std::integral_constant<int, 0> c0;
    const std::integral_constant<int, 1> c1;
    const std::integral_constant<int, 2> c2;
    switch (3 * g.wj + f.nt) { // wj > 0, layers wider than 64: no strips
    case 0: launch(c0, c0); break;
    case 1: launch(c0, c1); break;
    case 4: launch(c1, c1); break;
    case 5: launch(c1, c2); break;
    case 7: launch(c2, c1); break;
    default: launch(c2, c2); break;
    }
    SG_LAUNCH_CHECK();
    *pair_done = true;
    return SLICEGCN_OK;
}

// ---- pieces of the transform-first layer order -------------------------------------------------
// Hout[v, j] = act(P[v, j] + bias[j]) (+ Hout[v, j] when add), mask bit j of row v = [P + bias > 0].
// One thread per element of the row padded to a multiple of 32 columns, so every half wavefront lies
// inside one mask word of one row and a ballot assembles the word.
struct BiasActBatch {
    const float *P[BATCH], *bias[BATCH];
    float *Hout[BATCH];
    uint32_t *mask[BATCH];
};
__global__ __launch_bounds__(256) void bias_act_add_kernel(const BiasActBatch b, int64_t ldp, int64_t ldo, int add,
                                                           int64_t mask_words, int64_t n, int32_t w_out, int32_t act)
{
    const float *__restrict__ P = b.P[blockIdx.y];
    const float *__restrict__ bias = b.bias[blockIdx.y];
    float *__restrict__ Hout = b.Hout[blockIdx.y];
    uint32_t *__restrict__ mask = b.mask[blockIdx.y];
    const int wpad = (w_out + 31) / 32 * 32;
    const int64_t total = n * (int64_t)wpad;
    const int64_t padded_total = (total + 63) / 64 * 64; // whole wavefronts take part in every ballot
    const int lane = threadIdx.x & 63;
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < padded_total; t += (int64_t)gridDim.x * 256) {
        const int64_t row = t / wpad;
        const int col = (int)(t - row * wpad);
        const bool valid = t < total && col < w_out;
        const float p = valid ? P[row * ldp + col] + (bias ? bias[col] : 0.f) : 0.f;
        const bool pos = valid && p > 0.f;
        const unsigned long long bits = __ballot(pos);
        if (valid) {
            float r = act == SLICEGCN_ACT_RELU ? (pos ? p : 0.f) : p;
            if (add) r += Hout[row * ldo + col];
            Hout[row * ldo + col] = r;
        }
        if (act == SLICEGCN_ACT_RELU && (lane & 31) == 0 && t < total)
            mask[row * mask_words + (col >> 5)] = (uint32_t)(bits >> (lane & 32));
    }
}

// dP[v, j] = dHout[v, j] where the activation passed (all of it when mask == NULL)
struct MaskApplyBatch {
    const float *dHout[BATCH];
    const uint32_t *mask[BATCH];
    float *dP[BATCH];
};
__global__ __launch_bounds__(256) void mask_apply_kernel(const MaskApplyBatch b, int64_t ldo, int64_t mask_words, int64_t ldp, int64_t n,
                                                         int32_t w_out)
{
    const float *__restrict__ dHout = b.dHout[blockIdx.y];
    const uint32_t *__restrict__ mask = b.mask[blockIdx.y];
    float *__restrict__ dP = b.dP[blockIdx.y];
    const int64_t total = n * (int64_t)w_out;
    for (int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x; t < total; t += (int64_t)gridDim.x * 256) {
        const int64_t row = t / w_out;
        const int col = (int)(t - row * w_out);
        float v = dHout[row * ldo + col];
        if (mask && ((mask[row * mask_words + (col >> 5)] >> (col & 31)) & 1u) == 0u) v = 0.f;
        dP[row * ldp + col] = v;
    }
}

// Wt[j][i] = W[i][j] for a rows x cols row-major W (weights are small: one thread per element)
struct TransposeBatch {
    const float *W[2 * BATCH];
    float *Wt[2 * BATCH];
};
__global__ __launch_bounds__(256) void transpose_kernel(const TransposeBatch b, int32_t rows, int32_t cols)
{
    const float *__restrict__ W = b.W[blockIdx.y];
    float *__restrict__ Wt = b.Wt[blockIdx.y];
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= rows * cols) return;
    const int i = t / cols, j = t - i * cols;
    Wt[(int64_t)j * rows + i] = W[t];
}

inline unsigned ew_grid(int64_t total)
{
    const int64_t b = (total + 255) / 256;
    return (unsigned)(b < 1 ? 1 : (b > 262144 ? 262144 : b));
}

// aggregate first: Z = A^ Hin, then the weight products; transform first: T = Hin W_agg, then P = A^ T.
// Equal in exact arithmetic; the second gathers rows of w_out instead of w_in columns.
inline bool transform_first(const slicegcn_layer_desc *d)
{
    if (d->flags & SLICEGCN_LAYER_TRANSFORM_FIRST) return true;
    return (d->flags & SLICEGCN_LAYER_ORDER_AUTO) && d->w_out < d->w_in;
}

int check_layer(const slicegcn_graph *g, const slicegcn_layer_desc *d, const slicegcn_layer_params *p, const char *who)
{
    SG_REQUIRE(g && d && p, SLICEGCN_EINVAL, "%s: NULL graph, desc or params", who);
    SG_REQUIRE(d->w_in >= 1 && d->w_out >= 1, SLICEGCN_EINVAL, "%s: widths must be >= 1", who);
    SG_REQUIRE(d->act == SLICEGCN_ACT_NONE || d->act == SLICEGCN_ACT_RELU, SLICEGCN_EINVAL, "%s: unknown act %d", who, d->act);
    SG_REQUIRE((d->flags & ~(SLICEGCN_LAYER_Z_VALID | SLICEGCN_LAYER_TRANSFORM_FIRST | SLICEGCN_LAYER_ORDER_AUTO |
                             SLICEGCN_LAYER_IN_SCALED | SLICEGCN_LAYER_OUT_SCALED)) == 0, SLICEGCN_EINVAL,
               "%s: unknown flag bits 0x%x", who, d->flags);
    SG_REQUIRE(!((d->flags & (SLICEGCN_LAYER_IN_SCALED | SLICEGCN_LAYER_OUT_SCALED)) && transform_first(d)), SLICEGCN_EINVAL,
               "%s: the scaled layout needs the aggregate-first order", who);
    SG_REQUIRE(!((d->flags & SLICEGCN_LAYER_TRANSFORM_FIRST) && (d->flags & SLICEGCN_LAYER_ORDER_AUTO)), SLICEGCN_EINVAL,
               "%s: TRANSFORM_FIRST and ORDER_AUTO exclude each other", who);
    SG_REQUIRE(!((d->flags & SLICEGCN_LAYER_Z_VALID) && transform_first(d)), SLICEGCN_EINVAL,
               "%s: Z_VALID needs the aggregate-first order (no aggregation of the input is kept by the transform-first order)", who);
    SG_REQUIRE(p->W_agg != nullptr, SLICEGCN_EINVAL, "%s: W_agg is NULL", who);
    SG_REQUIRE(p->W_self != nullptr || p->b_self == nullptr, SLICEGCN_EINVAL, "%s: b_self without W_self", who);
    return SLICEGCN_OK;
}

int check_saved(const slicegcn_layer_desc *d, const slicegcn_layer_saved *s, const char *who)
{
    SG_REQUIRE(s != nullptr, SLICEGCN_EINVAL, "%s: saved is NULL", who);
    if (!transform_first(d)) { // the transform-first order keeps no aggregation: Z is neither written nor read
        SG_REQUIRE(s->Z != nullptr, SLICEGCN_EINVAL, "%s: saved->Z is NULL", who);
        SG_REQUIRE(s->ldz >= d->w_in && s->ldz % 4 == 0 && aligned16(s->Z), SLICEGCN_EINVAL,
                   "%s: saved->Z needs ldz >= w_in, ldz %% 4 == 0 and a 16-byte aligned base", who);
    }
    if (d->act == SLICEGCN_ACT_RELU)
        SG_REQUIRE(s->mask && s->mask_words >= (d->w_out + 31) / 32, SLICEGCN_EINVAL,
                   "%s: mask is NULL or mask_words < ceil(w_out / 32)", who);
    return SLICEGCN_OK;
}

} // namespace

// shared with misc.hip
int launch_colsum_partial(const float *M, int64_t ld, int64_t n, int32_t w, float *ws, hipStream_t stream)
{
    const int64_t nb = red_blocks(n);
    if (aligned16(M) && ld % 4 == 0 && w % 4 == 0)
        colsum_partial_vec_kernel<<<(unsigned)nb, 256, 0, stream>>>(M, ld, n, w, ws);
    else
        colsum_partial_kernel<<<(unsigned)nb, 256, 0, stream>>>(M, ld, n, w, ws);
    SG_LAUNCH_CHECK();
    return SLICEGCN_OK;
}

int launch_final_sum(const FinalWork &f, int batch, hipStream_t stream)
{
    reduce_final_kernel<<<dim3((unsigned)((f.stride + FINAL_ELEMS - 1) / FINAL_ELEMS), (unsigned)batch), 1024, 0, stream>>>(f);
    SG_LAUNCH_CHECK();
    return SLICEGCN_OK;
}

int launch_colsum_final(const float *ws_first, int64_t n, int32_t ws_row, int32_t count, float *out, hipStream_t stream)
{
    FinalWork f;
    f.partial[0] = ws_first;
    f.dst[0] = FinalDst{{out, nullptr, nullptr, nullptr}, nullptr, {0, count, count, count, count}};
    f.n_blocks = red_blocks(n); f.row_stride = ws_row; f.stride = count;
    return launch_final_sum(f, 1, stream);
}

size_t colsum_workspace_bytes(int64_t n, int32_t w) { return (size_t)red_blocks(n) * (size_t)w * sizeof(float); }

} // namespace slicegcn

using namespace slicegcn;

// partial sums of a dense layer's weight and bias gradients: `partials` rows of [w_in*w_out + w_out]
static size_t linear_partial_bytes(int64_t partials, int32_t w_in, int32_t w_out)
{
    const size_t stride = (size_t)w_in * w_out + (size_t)w_out;
    return (size_t)round_up((int64_t)(partials * stride * sizeof(float)), 256);
}
// what the kernels use where the workspace allows it
static size_t linear_full_bytes(int64_t n, int32_t w_in, int32_t w_out)
{
    return linear_partial_bytes(linear_grad_plan(n, w_in, w_out, NO_LIMIT).partials, w_in, w_out);
}

struct LinearGradArgs { // one layer of a batch (equal shapes and leading dimensions)
    const float *X;
    const uint32_t *mask;
    const float *dY;
    float *dW, *db;
    float *db_copy = nullptr;
};

// dW = X^T (dY * mask) (w_in x w_out), db = colsum(dY * mask); NULL outputs are skipped.  ws: ws_each bytes per layer of
// the batch, at least linear_partial_bytes(red_blocks(n)).
static int launch_linear_grads(const LinearGradArgs *list, int batch, int64_t ldx, int64_t n, int32_t w_in, int32_t w_out,
                               int64_t mask_words, int64_t lddy, void *ws, size_t ws_each, hipStream_t stream,
                               const PairArgs *inputs = nullptr, bool *inputs_done = nullptr)
{
    const int ww = w_in * w_out;
    const int32_t stride = ww + w_out;
    const LinearGradPlan plan = linear_grad_plan(n, w_in, w_out, (int64_t)(ws_each / ((size_t)stride * sizeof(float))));
    ReduceArgs r;
    r.Z = nullptr; r.ldz = ldx; r.Hin = nullptr; r.ldi = 0; r.dHout = nullptr; r.ldo = lddy;
    r.mask = nullptr; r.mask_words = mask_words;
    r.partial = nullptr; r.n = n; r.w_in = w_in; r.w_out = w_out; r.stride = stride; r.compact = 1;
    r.rows_per_block = plan.rows;
    ReduceBatch b;
    FinalWork f;
    f.n_blocks = plan.partials; f.row_stride = f.stride = stride;
    for (int i = 0; i < BATCH; ++i) {
        const LinearGradArgs &x = list[i < batch ? i : 0];
        float *partial = reinterpret_cast<float *>(static_cast<char *>(ws) + (i < batch ? i : 0) * ws_each);
        b.p[i] = ReducePtrs{x.X, nullptr, x.dY, x.mask, partial};
        f.partial[i] = partial;
        f.dst[i] = FinalDst{{x.dW, nullptr, nullptr, x.db}, x.db_copy, {0, ww, ww, ww, stride}};
    }
    bool pair_done;
    if (int rc = launch_grads_and_pair(r, b, batch, 1, plan.big, inputs, &pair_done, stream)) return rc;
    if (inputs_done) *inputs_done = pair_done;
    return launch_final_sum(f, batch, stream);
}

// ---- one layer of a batch of slice models --------------------------------------------------
static size_t mat_bytes(int64_t n, int32_t w) { return (size_t)round_up(n * round_up(w, 32) * (int64_t)sizeof(float), 256); }

// Transform-first order:
// forward : T = Hin W_agg;  S = Hin W_self + b_self (stored straight into Hout);  P = A^ T;
//           Hout = act(P + b) + S,  mask = [P + b > 0]
// backward: dP = dHout * mask;  db = colsum dP;  G = A^^T dP;  dW_agg = Hin^T G;
//           dW_self = Hin^T dHout, db_self = colsum dHout;  dHin = G W_agg^T + dHout W_self^T
// Nothing of the forward pass but the mask is kept: the backward pass aggregates dP instead of re-using A^ Hin.
static size_t tf_wt_bytes(const slicegcn_layer_desc *d) { return (size_t)round_up((int64_t)d->w_in * d->w_out * (int64_t)sizeof(float), 256); }
static size_t tf_red_bytes(int64_t n, const slicegcn_layer_desc *d, bool full)
{
    const size_t a = full ? linear_full_bytes(n, d->w_in, d->w_out) : 0, c = linear_partial_bytes(red_blocks(n), d->w_in, d->w_out);
    const size_t b = (size_t)round_up((int64_t)colsum_workspace_bytes(n, d->w_out), 256);
    const size_t m = a > c ? a : c;
    return m > b ? m : b;
}

// Bytes of workspace per slice of a batch.  `full`: with as many partial sums as the reductions would use.
static size_t fwd_bytes(const slicegcn_graph *g, const slicegcn_layer_desc *d)
{
    if (transform_first(d)) return 2 * mat_bytes(g->n, d->w_out) + spmm_workspace_bytes(g->fwd, d->w_out);
    return spmm_workspace_bytes(g->fwd, d->w_in);
}
static size_t bwd_partial_bytes(int64_t n, const slicegcn_layer_desc *d)
{
    const size_t stride = 2 * (size_t)d->w_in * d->w_out + 2 * (size_t)d->w_out;
    return (size_t)round_up((int64_t)(layer_grad_blocks(n, d->w_in, d->w_out) * stride * sizeof(float)), 256);
}
static size_t bwd_bytes(const slicegcn_graph *g, const slicegcn_layer_desc *d, bool need_dHin, bool full)
{
    if (transform_first(d)) // [dP | G | W_agg^T | W_self^T | reduction partials | aggregation workspace]
        return 2 * mat_bytes(g->n, d->w_out) + 2 * tf_wt_bytes(d) + tf_red_bytes(g->n, d, full) + spmm_workspace_bytes(g->tr, d->w_out);
    // [partial weight gradients | dZ (only with dHin) | aggregation workspace (only with dHin)]
    size_t bytes = bwd_partial_bytes(g->n, d);
    if (need_dHin) bytes += mat_bytes(g->n, d->w_in) + spmm_workspace_bytes(g->tr, d->w_in);
    return bytes;
}

// Workspace sections: section q of slice i starts at base + batch * (bytes of the sections before) + i * (bytes of section q)
struct Sections {
    char *base;
    int batch;
    size_t used = 0;
    char *take(size_t bytes) { char *p = base + used; used += bytes * batch; return p; }
};

static int fwd_transform_first(const slicegcn_graph *g, const slicegcn_layer_group *lg, const slicegcn_layer_io *io, int batch, void *ws,
                               hipStream_t stream)
{
    const slicegcn_layer_desc *desc = &lg->desc;
    const int w_in = desc->w_in, w_out = desc->w_out;
    const bool self = io[0].params.W_self != nullptr;
    const int64_t ldt = round_up(w_out, 32);
    const size_t mat = mat_bytes(g->n, w_out), agg = spmm_workspace_bytes(g->fwd, w_out);
    Sections sec{static_cast<char *>(ws), batch};
    char *Ts = sec.take(mat), *Ps = sec.take(mat), *agg_ws = sec.take(agg);
    {
        ProfScope prof(SLICEGCN_PROF_DENSE_FWD, w_out, stream);
        PairArgs list[BATCH];
        for (int i = 0; i < batch; ++i) {
            PairArgs &a = list[i];
            a.A1 = io[i].Hin; a.lda1 = lg->ldi; a.A2 = nullptr; a.lda2 = 0;
            a.B1 = io[i].params.W_agg; a.B2 = nullptr; a.bias1 = a.bias2 = nullptr;
            a.O1 = reinterpret_cast<float *>(Ts + i * mat); a.ldo1 = ldt; a.O2 = nullptr; a.ldo2 = 0;
            a.mask = nullptr; a.mask_words = 0;
            a.n = g->n; a.K = w_in; a.Nout = w_out; a.ldw = w_out; a.act = SLICEGCN_ACT_NONE;
        }
        if (int rc = launch_pair<false>(list, batch, stream)) return rc;
        if (self) { // the self term goes straight to the output; the epilogue below adds the activated part
            for (int i = 0; i < batch; ++i) {
                list[i].B1 = io[i].params.W_self; list[i].bias1 = io[i].params.b_self; list[i].enc = io[i].enc;
                list[i].O1 = io[i].Hout; list[i].ldo1 = lg->ldo;
            }
            if (int rc = launch_pair<false>(list, batch, stream)) return rc;
        }
    }
    SpmmOperands ops[BATCH];
    BiasActBatch b;
    for (int i = 0; i < BATCH; ++i) {
        const int q = i < batch ? i : 0;
        float *P = reinterpret_cast<float *>(Ps + q * mat);
        ops[i] = SpmmOperands{reinterpret_cast<float *>(Ts + q * mat), P, nullptr};
        b.P[i] = P; b.bias[i] = io[q].params.b; b.Hout[i] = io[q].Hout;
        b.mask[i] = desc->act == SLICEGCN_ACT_RELU ? io[q].mask : nullptr;
    }
    if (int rc = launch_spmm(g, g->fwd, ops, batch, ldt, w_out, ldt, 0, agg_ws, agg * batch, stream)) return rc;
    ProfScope prof(SLICEGCN_PROF_DENSE_FWD, w_out, stream);
    const int64_t total = g->n * round_up(w_out, 32);
    bias_act_add_kernel<<<dim3(ew_grid(total), (unsigned)batch), 256, 0, stream>>>(b, ldt, lg->ldo, self, lg->mask_words, g->n, w_out, desc->act);
    SG_LAUNCH_CHECK();
    return SLICEGCN_OK;
}

static int bwd_transform_first(const slicegcn_graph *g, const slicegcn_layer_group *lg, const slicegcn_layer_io *io, int batch, void *ws,
                               bool full, hipStream_t stream)
{
    const slicegcn_layer_desc *desc = &lg->desc;
    const int w_in = desc->w_in, w_out = desc->w_out;
    const int64_t n = g->n, ldp = round_up(w_out, 32);
    const bool relu = desc->act == SLICEGCN_ACT_RELU, self = io[0].params.W_self != nullptr;
    const size_t mat = mat_bytes(n, w_out), wt = tf_wt_bytes(desc), red_each = tf_red_bytes(n, desc, full), agg = spmm_workspace_bytes(g->tr, w_out);
    Sections sec{static_cast<char *>(ws), batch};
    char *dPs = sec.take(mat), *Gs = sec.take(mat), *WaTs = sec.take(wt), *WsTs = sec.take(wt), *red = sec.take(red_each), *agg_ws = sec.take(agg);
    auto dP = [&](int i) { return reinterpret_cast<float *>(dPs + i * mat); };
    auto G = [&](int i) { return reinterpret_cast<float *>(Gs + i * mat); };
    // dHin = G W_agg^T + dHout W_self^T, the last step: one forward-form launch over the transposed weights
    TransposeBatch t;
    int mats = 0;
    PairArgs list[BATCH];
    for (int i = 0; i < batch && io[0].dHin; ++i) {
        float *WaT = reinterpret_cast<float *>(WaTs + i * wt), *WsT = reinterpret_cast<float *>(WsTs + i * wt);
        t.W[mats] = io[i].params.W_agg; t.Wt[mats++] = WaT;
        if (self) { t.W[mats] = io[i].params.W_self; t.Wt[mats++] = WsT; }
        PairArgs &a = list[i];
        a.A1 = G(i); a.lda1 = ldp;
        a.A2 = self ? io[i].dHout : nullptr; a.lda2 = lg->ldgo;
        a.B1 = WaT; a.B2 = self ? WsT : nullptr;
        a.bias1 = a.bias2 = nullptr;
        a.O1 = io[i].dHin; a.ldo1 = lg->ldgi; a.O2 = nullptr; a.ldo2 = 0;
        a.mask = nullptr; a.mask_words = 0;
        a.n = n; a.K = w_out; a.Nout = w_in; a.ldw = w_in; a.act = SLICEGCN_ACT_NONE;
    }
    if (mats > 0)
        if (int rc = check_in_place(list, batch)) return rc; // before anything is launched
    {
        ProfScope prof(SLICEGCN_PROF_DENSE_BWD, w_out, stream);
        MaskApplyBatch b;
        for (int i = 0; i < BATCH; ++i) {
            const int q = i < batch ? i : 0;
            b.dHout[i] = io[q].dHout; b.mask[i] = relu ? io[q].mask : nullptr; b.dP[i] = dP(q);
        }
        mask_apply_kernel<<<dim3(ew_grid(n * w_out), (unsigned)batch), 256, 0, stream>>>(b, lg->ldgo, lg->mask_words, ldp, n, w_out);
        SG_LAUNCH_CHECK();
    }
    SpmmOperands ops[BATCH];
    for (int i = 0; i < batch; ++i) ops[i] = SpmmOperands{dP(i), G(i), nullptr};
    if (int rc = launch_spmm(g, g->tr, ops, batch, ldp, w_out, ldp, 0, agg_ws, agg * batch, stream)) return rc;
    {
        ProfScope prof(SLICEGCN_PROF_GRAD_REDUCE, w_out, stream);
        for (int i = 0; i < batch; ++i)
            if (io[i].grads.db) {
                if (int rc = launch_colsum_partial(dP(i), ldp, n, w_out, reinterpret_cast<float *>(red), stream)) return rc;
                if (int rc = launch_colsum_final(reinterpret_cast<float *>(red), n, w_out, w_out, io[i].grads.db, stream)) return rc;
            }
        LinearGradArgs agg_list[BATCH], self_list[BATCH];
        bool any_agg = false, any_self = false;
        for (int i = 0; i < batch; ++i) {
            const slicegcn_layer_grads &gr = io[i].grads;
            agg_list[i] = LinearGradArgs{io[i].Hin, nullptr, G(i), gr.dW_agg, nullptr};
            self_list[i] = LinearGradArgs{io[i].Hin, nullptr, io[i].dHout, gr.dW_self, gr.db_self, io[i].denc};
            any_agg = any_agg || gr.dW_agg;
            any_self = any_self || (self && (gr.dW_self || gr.db_self || io[i].denc));
        }
        if (any_agg)
            if (int rc = launch_linear_grads(agg_list, batch, lg->ldi, n, w_in, w_out, 0, ldp, red, red_each, stream)) return rc;
        if (any_self)
            if (int rc = launch_linear_grads(self_list, batch, lg->ldi, n, w_in, w_out, 0, lg->ldgo, red, red_each, stream)) return rc;
    }
    if (mats > 0) {
        ProfScope prof(SLICEGCN_PROF_DENSE_BWD, w_in, stream);
        const int count = w_in * w_out;
        transpose_kernel<<<dim3((unsigned)((count + 255) / 256), (unsigned)mats), 256, 0, stream>>>(t, w_in, w_out);
        SG_LAUNCH_CHECK();
        if (int rc = launch_pair<false>(list, batch, stream)) return rc;
    }
    return SLICEGCN_OK;
}

// Forward pass of one layer for `batch` slice models.  ws: batch * fwd_bytes.
static int layers_fwd(const slicegcn_graph *g, const slicegcn_layer_group *lg, const slicegcn_layer_io *io, int batch, void *ws,
                      size_t ws_bytes, hipStream_t stream)
{
    const slicegcn_layer_desc *desc = &lg->desc;
    if (transform_first(desc)) return fwd_transform_first(g, lg, io, batch, ws, stream);
    const bool self = io[0].params.W_self != nullptr;
    if (!(desc->flags & SLICEGCN_LAYER_Z_VALID)) {
        SpmmOperands ops[BATCH];
        for (int i = 0; i < batch; ++i) ops[i] = SpmmOperands{io[i].Hin, io[i].Z, nullptr};
        if (int rc = launch_spmm(g, g->fwd, ops, batch, lg->ldi, desc->w_in, lg->ldz, 0, ws, ws_bytes, stream,
                                 (desc->flags & SLICEGCN_LAYER_IN_SCALED) != 0))
            return rc;
    }
    PairArgs list[BATCH];
    for (int i = 0; i < batch; ++i) {
        PairArgs &a = list[i];
        const slicegcn_layer_params &p = io[i].params;
        a.A1 = io[i].Z; a.lda1 = lg->ldz;
        a.A2 = self ? io[i].Hin : nullptr; a.lda2 = lg->ldi;
        a.B1 = p.W_agg; a.B2 = p.W_self;
        a.bias1 = p.b; a.bias2 = p.b_self; a.enc = io[i].enc;
        a.O1 = io[i].Hout; a.ldo1 = lg->ldo; a.O2 = nullptr; a.ldo2 = 0;
        a.mask = desc->act == SLICEGCN_ACT_RELU ? io[i].mask : nullptr; a.mask_words = lg->mask_words;
        a.n = g->n; a.K = desc->w_in; a.Nout = desc->w_out; a.ldw = desc->w_out; a.act = desc->act;
        a.scale2 = ((desc->flags & SLICEGCN_LAYER_IN_SCALED) && self) ? g->sqrtd : nullptr;
        a.scale_o1 = (desc->flags & SLICEGCN_LAYER_OUT_SCALED) ? g->dinv : nullptr;
    }
    ProfScope prof(SLICEGCN_PROF_DENSE_FWD, desc->w_out, stream);
    return launch_pair<false>(list, batch, stream);
}

// Backward pass of one layer for `batch` slice models.  ws: batch * bwd_bytes(..., full).
static int layers_bwd(const slicegcn_graph *g, const slicegcn_layer_group *lg, const slicegcn_layer_io *io, int batch, void *ws, bool full,
                      hipStream_t stream)
{
    const slicegcn_layer_desc *desc = &lg->desc;
    if (transform_first(desc)) return bwd_transform_first(g, lg, io, batch, ws, full, stream);
    const int w_in = desc->w_in, w_out = desc->w_out;
    const bool self = io[0].params.W_self != nullptr, need_dHin = io[0].dHin != nullptr, relu = desc->act == SLICEGCN_ACT_RELU;
    const size_t part = bwd_partial_bytes(g->n, desc), mat = mat_bytes(g->n, w_in), agg = spmm_workspace_bytes(g->tr, w_in);
    Sections sec{static_cast<char *>(ws), batch};
    char *parts = sec.take(part), *dZs = need_dHin ? sec.take(mat) : nullptr, *agg_ws = need_dHin ? sec.take(agg) : nullptr;

    // ---- input gradient, dense half: dZ = dP W_agg^T (staged, rows scaled by D~^-1/2) and T = dHout W_self^T (into dHin) ----
    const int64_t ldz_in = round_up(w_in, 32); // rows of the gathered operand start on 128-byte boundaries
    PairArgs list[BATCH];
    for (int i = 0; i < batch && need_dHin; ++i) {
        PairArgs &a = list[i];
        a.A1 = io[i].dHout; a.lda1 = lg->ldgo;
        a.A2 = self ? io[i].dHout : nullptr; a.lda2 = lg->ldgo;
        a.B1 = io[i].params.W_agg; a.B2 = io[i].params.W_self;
        a.bias1 = a.bias2 = nullptr;
        a.O1 = reinterpret_cast<float *>(dZs + i * mat); a.ldo1 = ldz_in;
        a.O2 = self ? io[i].dHin : nullptr; a.ldo2 = lg->ldgi;
        a.mask = relu ? io[i].mask : nullptr; a.mask_words = lg->mask_words;
        a.n = g->n; a.K = w_out; a.Nout = w_in; a.ldw = w_out; a.act = desc->act;
        a.scale_o1 = g->dinv; // dZ is staged as D~^-1/2 dZ: its aggregation then skips the stored values
    }
    if (need_dHin)
        if (int rc = check_in_place(list, batch)) return rc; // before anything is launched
    const GradPlan plan = grad_plan(g->n, w_in, w_out);
    // narrow layers with a self term: the kernel that forms the weight gradients also forms dZ and T (one read of dHout)
    const bool fused_inputs = need_dHin && self && plan.kind == GradPlan::STRIP32;
    bool pair_done = fused_inputs; // so does one launch on few rows

    // ---- parameter gradients: per-row-block partial sums, then an fp64 combination ----
    const int32_t stride = 2 * w_in * w_out + 2 * w_out;
    FinalWork sums;
    {
        ProfScope prof(SLICEGCN_PROF_GRAD_REDUCE, w_out, stream);
        ReduceArgs r;
        r.Z = nullptr; r.ldz = lg->ldz; r.Hin = nullptr; r.ldi = lg->ldi; r.dHout = nullptr; r.ldo = lg->ldgo;
        r.mask = nullptr; r.mask_words = lg->mask_words;
        r.partial = nullptr; r.n = g->n; r.w_in = w_in; r.w_out = w_out; r.stride = stride; r.compact = 0;
        r.rows_per_block = plan.rows;
        r.hin_scale = (desc->flags & SLICEGCN_LAYER_IN_SCALED) ? g->sqrtd : nullptr;
        ReduceBatch b;
        sums.n_blocks = plan.partials; sums.row_stride = sums.stride = stride;
        const int ww = w_in * w_out;
        for (int i = 0; i < BATCH; ++i) {
            const slicegcn_layer_io &x = io[i < batch ? i : 0];
            float *partial = reinterpret_cast<float *>(parts + (i < batch ? i : 0) * part);
            b.p[i] = ReducePtrs{x.Z, self ? x.Hin : nullptr, x.dHout, relu ? x.mask : nullptr, partial};
            sums.partial[i] = partial;
            sums.dst[i] = FinalDst{{x.grads.dW_agg, self ? x.grads.dW_self : nullptr, x.grads.db, self ? x.grads.db_self : nullptr},
                                   self ? x.denc : nullptr, {0, ww, 2 * ww, 2 * ww + w_out, stride}};
        }
        const unsigned by = (unsigned)batch, gb = (unsigned)((plan.partials + 3) / 4);
        switch (plan.kind) {
        case GradPlan::STRIP32:
            if (fused_inputs) { // weight gradients and the two input-gradient products in one sweep over the rows
                bwd_strip32_kernel<<<dim3(gb, by), 256, 0, stream>>>(r, b, list[0], pair_batch(list, batch), plan.partials);
            } else {
                grad_strip32_kernel<<<dim3(gb, by), 256, 0, stream>>>(r, b, plan.partials);
            }
            break;
        case GradPlan::STRIP64:
            launch_grad_strip(self, w_in < 4 || w_out < 4, [&](auto s, auto w) {
                if (w_in <= 32) grad_strip64_kernel<1, 2, 8, 3, s.value, w.value><<<dim3(gb, by), 256, 0, stream>>>(r, b, plan.partials);
                else if (w_out <= 32) grad_strip64_kernel<2, 1, 8, 3, s.value, w.value><<<dim3(gb, by), 256, 0, stream>>>(r, b, plan.partials);
                else grad_strip64_kernel<2, 2, 8, 2, s.value, false><<<dim3(gb, by), 256, 0, stream>>>(r, b, plan.partials);
            });
            break;
        case GradPlan::TILED:
            if (int rc = launch_grads_and_pair(r, b, batch, self ? 2 : 1, false, need_dHin ? list : nullptr, &pair_done, stream)) return rc;
            break;
        }
        SG_LAUNCH_CHECK();
        if (!need_dHin)
            if (int rc = launch_final_sum(sums, batch, stream)) return rc;
    }

    // ---- input gradient: dHin = A^^T (dP W_agg^T) + dHout W_self^T ----
    if (need_dHin) {
        if (!pair_done) {
            ProfScope prof(SLICEGCN_PROF_DENSE_BWD, w_in, stream);
            if (int rc = launch_pair<true>(list, batch, stream)) return rc;
        }
        // padding columns of dZ are never read as data: the aggregation masks them on store
        SpmmOperands ops[BATCH];
        for (int i = 0; i < batch; ++i)
            ops[i] = SpmmOperands{reinterpret_cast<float *>(dZs + i * mat), io[i].dHin, self ? io[i].dHin : nullptr};
        if (int rc = launch_spmm(g, g->tr, ops, batch, ldz_in, w_in, lg->ldgi, lg->ldgi, agg_ws, agg * batch, stream, true, &sums)) return rc;
    }
    return SLICEGCN_OK;
}

static slicegcn_layer_group one_layer(const slicegcn_layer_desc *desc, int64_t ldi, int64_t ldo, const slicegcn_layer_saved *saved,
                                      int64_t ldgo, int64_t ldgi)
{
    slicegcn_layer_group lg;
    lg.desc = *desc;
    lg.count = 1;
    lg.ldi = ldi; lg.ldo = ldo; lg.ldz = saved->ldz; lg.mask_words = saved->mask_words; lg.ldgo = ldgo; lg.ldgi = ldgi;
    return lg;
}

extern "C" int slicegcn_layer_fwd(const slicegcn_graph *g, const slicegcn_layer_desc *desc,
                                  const slicegcn_layer_params *params, const float *Hin, int64_t ldi,
                                  float *Hout, int64_t ldo, slicegcn_layer_saved *saved, void *ws, size_t ws_bytes,
                                  void *stream_)
{
    if (int rc = check_layer(g, desc, params, "layer_fwd")) return rc;
    SG_REQUIRE(Hin && Hout, SLICEGCN_EINVAL, "layer_fwd: NULL Hin or Hout");
    SG_REQUIRE(ldi >= desc->w_in && ldo >= desc->w_out, SLICEGCN_EINVAL, "layer_fwd: leading dimension too small");
    if (int rc = check_saved(desc, saved, "layer_fwd")) return rc;
    if (transform_first(desc)) {
        const size_t need = fwd_bytes(g, desc);
        SG_REQUIRE(ws != nullptr && ws_bytes >= need, SLICEGCN_EWORKSPACE, "layer_fwd: workspace of %zu bytes, %zu needed", ws_bytes, need);
        SG_REQUIRE((reinterpret_cast<uintptr_t>(ws) & 255u) == 0, SLICEGCN_EINVAL, "layer_fwd: workspace not 256-byte aligned");
    }
    const slicegcn_layer_group lg = one_layer(desc, ldi, ldo, saved, 0, 0);
    slicegcn_layer_io io{};
    io.params = *params; io.Hin = Hin; io.Hout = Hout; io.Z = saved->Z; io.mask = saved->mask;
    return layers_fwd(g, &lg, &io, 1, ws, ws_bytes, as_stream(stream_));
}

extern "C" size_t slicegcn_layer_fwd_workspace_bytes(const slicegcn_graph *g, const slicegcn_layer_desc *desc)
{
    if (!g || !desc || desc->w_in < 1 || desc->w_out < 1) return 0;
    return fwd_bytes(g, desc);
}

extern "C" size_t slicegcn_layer_bwd_workspace_bytes(const slicegcn_graph *g, const slicegcn_layer_desc *desc, int need_dHin)
{
    if (!g || !desc || desc->w_in < 1 || desc->w_out < 1) return 0;
    return bwd_bytes(g, desc, need_dHin != 0, false);
}

extern "C" int slicegcn_layer_bwd(const slicegcn_graph *g, const slicegcn_layer_desc *desc,
                                  const slicegcn_layer_params *params, const float *Hin, int64_t ldi,
                                  const slicegcn_layer_saved *saved, const float *dHout, int64_t ldo,
                                  float *dHin, int64_t ldgi, slicegcn_layer_grads *grads,
                                  void *ws, size_t ws_bytes, void *stream_)
{
    if (int rc = check_layer(g, desc, params, "layer_bwd")) return rc;
    SG_REQUIRE(Hin && dHout && grads, SLICEGCN_EINVAL, "layer_bwd: NULL Hin, dHout or grads");
    SG_REQUIRE(ldi >= desc->w_in && ldo >= desc->w_out, SLICEGCN_EINVAL, "layer_bwd: leading dimension too small");
    SG_REQUIRE(dHin == nullptr || ldgi >= desc->w_in, SLICEGCN_EINVAL, "layer_bwd: ldgi < w_in");
    if (int rc = check_saved(desc, saved, "layer_bwd")) return rc;
    const size_t need = bwd_bytes(g, desc, dHin != nullptr, false);
    SG_REQUIRE(ws != nullptr && ws_bytes >= need, SLICEGCN_EWORKSPACE, "layer_bwd: workspace of %zu bytes, %zu needed",
               ws_bytes, need);
    SG_REQUIRE((reinterpret_cast<uintptr_t>(ws) & 255u) == 0, SLICEGCN_EINVAL, "layer_bwd: workspace not 256-byte aligned");
    const slicegcn_layer_group lg = one_layer(desc, ldi, 0, saved, ldo, ldgi);
    slicegcn_layer_io io{};
    io.params = *params; io.Hin = Hin; io.Z = saved->Z; io.mask = saved->mask; io.dHout = dHout; io.dHin = dHin; io.grads = *grads;
    return layers_bwd(g, &lg, &io, 1, ws, false, as_stream(stream_));
}

// ---- the same layer of several slice models -------------------------------------------------

static int check_group(const slicegcn_graph *g, const slicegcn_layer_group *lg, const slicegcn_layer_io *io, bool backward, const char *who)
{
    SG_REQUIRE(g && lg && io, SLICEGCN_EINVAL, "%s: NULL graph, group or io", who);
    SG_REQUIRE(lg->count >= 1 && lg->count <= BATCH, SLICEGCN_EINVAL, "%s: count = %d outside [1, %d]", who, lg->count, BATCH);
    const slicegcn_layer_desc *d = &lg->desc;
    for (int i = 0; i < lg->count; ++i) {
        const slicegcn_layer_io &x = io[i];
        if (int rc = check_layer(g, d, &x.params, who)) return rc;
        const slicegcn_layer_saved saved{x.Z, lg->ldz, x.mask, lg->mask_words};
        if (int rc = check_saved(d, &saved, who)) return rc;
        SG_REQUIRE(x.Hin && (backward ? x.dHout != nullptr : x.Hout != nullptr), SLICEGCN_EINVAL, "%s: NULL operand", who);
        SG_REQUIRE((x.params.W_self == nullptr) == (io[0].params.W_self == nullptr) && (x.dHin == nullptr) == (io[0].dHin == nullptr),
                   SLICEGCN_EINVAL, "%s: slices of a group differ in their terms", who);
        SG_REQUIRE(x.params.W_self || (!x.enc && !x.denc), SLICEGCN_EINVAL, "%s: encoding without a self term", who);
    }
    SG_REQUIRE(lg->ldi >= d->w_in, SLICEGCN_EINVAL, "%s: ldi < w_in", who);
    if (backward) SG_REQUIRE(lg->ldgo >= d->w_out && (!io[0].dHin || lg->ldgi >= d->w_in), SLICEGCN_EINVAL, "%s: leading dimension too small", who);
    else SG_REQUIRE(lg->ldo >= d->w_out, SLICEGCN_EINVAL, "%s: ldo < w_out", who);
    return SLICEGCN_OK;
}

extern "C" size_t slicegcn_layers_fwd_workspace_bytes(const slicegcn_graph *g, const slicegcn_layer_desc *desc, int32_t count)
{
    if (!g || !desc || desc->w_in < 1 || desc->w_out < 1 || count < 1) return 0;
    return (size_t)count * fwd_bytes(g, desc);
}

extern "C" size_t slicegcn_layers_bwd_workspace_bytes(const slicegcn_graph *g, const slicegcn_layer_desc *desc, int need_dHin, int32_t count)
{
    if (!g || !desc || desc->w_in < 1 || desc->w_out < 1 || count < 1) return 0;
    return (size_t)count * bwd_bytes(g, desc, need_dHin != 0, true);
}

extern "C" int slicegcn_layers_fwd(const slicegcn_graph *g, const slicegcn_layer_group *group, const slicegcn_layer_io *io,
                                   void *ws, size_t ws_bytes, void *stream_)
{
    if (int rc = check_group(g, group, io, false, "layers_fwd")) return rc;
    const size_t need = group->count * fwd_bytes(g, &group->desc);
    SG_REQUIRE(need == 0 || (ws != nullptr && ws_bytes >= need), SLICEGCN_EWORKSPACE, "layers_fwd: workspace of %zu bytes, %zu needed", ws_bytes, need);
    SG_REQUIRE((reinterpret_cast<uintptr_t>(ws) & 255u) == 0, SLICEGCN_EINVAL, "layers_fwd: workspace not 256-byte aligned");
    return layers_fwd(g, group, io, group->count, ws, ws_bytes, as_stream(stream_));
}

extern "C" int slicegcn_layers_bwd(const slicegcn_graph *g, const slicegcn_layer_group *group, const slicegcn_layer_io *io,
                                   void *ws, size_t ws_bytes, void *stream_)
{
    if (int rc = check_group(g, group, io, true, "layers_bwd")) return rc;
    const size_t need = group->count * bwd_bytes(g, &group->desc, io[0].dHin != nullptr, true);
    SG_REQUIRE(ws != nullptr && ws_bytes >= need, SLICEGCN_EWORKSPACE, "layers_bwd: workspace of %zu bytes, %zu needed", ws_bytes, need);
    SG_REQUIRE((reinterpret_cast<uintptr_t>(ws) & 255u) == 0, SLICEGCN_EINVAL, "layers_bwd: workspace not 256-byte aligned");
    return layers_bwd(g, group, io, group->count, ws, true, as_stream(stream_));
}

// ---- dense layer Y = act(X W + b): the unit of the paper's classifier MLP_CLS and of MLP_FF ----

extern "C" int slicegcn_linear_fwd(const float *X, int64_t ldx, int64_t n, int32_t w_in, int32_t w_out, const float *W,
                                   const float *b, int32_t act, float *Y, int64_t ldy, uint32_t *mask, int64_t mask_words,
                                   void *stream_)
{
    SG_REQUIRE(X && W && Y, SLICEGCN_EINVAL, "linear_fwd: NULL X, W or Y");
    SG_REQUIRE(n >= 1 && w_in >= 1 && w_out >= 1, SLICEGCN_EINVAL, "linear_fwd: sizes must be >= 1");
    SG_REQUIRE(ldx >= w_in && ldy >= w_out, SLICEGCN_EINVAL, "linear_fwd: leading dimension too small");
    SG_REQUIRE(act == SLICEGCN_ACT_NONE || act == SLICEGCN_ACT_RELU, SLICEGCN_EINVAL, "linear_fwd: unknown act %d", act);
    if (act == SLICEGCN_ACT_RELU)
        SG_REQUIRE(mask && mask_words >= (w_out + 31) / 32, SLICEGCN_EINVAL,
                   "linear_fwd: mask is NULL or mask_words < ceil(w_out / 32)");
    hipStream_t stream = as_stream(stream_);
    PairArgs a;
    a.A1 = X; a.lda1 = ldx; a.A2 = nullptr; a.lda2 = 0;
    a.B1 = W; a.B2 = nullptr; a.bias1 = b; a.bias2 = nullptr;
    a.O1 = Y; a.ldo1 = ldy; a.O2 = nullptr; a.ldo2 = 0;
    a.mask = act == SLICEGCN_ACT_RELU ? mask : nullptr; a.mask_words = mask_words;
    a.n = n; a.K = w_in; a.Nout = w_out; a.ldw = w_out; a.act = act;
    ProfScope prof(SLICEGCN_PROF_LINEAR_FWD, w_out, stream);
    return launch_pair<false>(a, stream);
}

extern "C" size_t slicegcn_linear_bwd_workspace_bytes(int64_t n, int32_t w_in, int32_t w_out)
{
    if (n < 1 || w_in < 1 || w_out < 1) return 0;
    return linear_partial_bytes(red_blocks(n), w_in, w_out);
}

extern "C" size_t slicegcn_linear_bwd_full_workspace_bytes(int64_t n, int32_t w_in, int32_t w_out)
{
    if (n < 1 || w_in < 1 || w_out < 1) return 0;
    const size_t a = linear_partial_bytes(red_blocks(n), w_in, w_out), b = linear_full_bytes(n, w_in, w_out);
    return a > b ? a : b;
}

extern "C" int slicegcn_linear_bwd(const float *X, int64_t ldx, int64_t n, int32_t w_in, int32_t w_out, const float *W,
                                   int32_t act, const uint32_t *mask, int64_t mask_words, const float *dY, int64_t lddy,
                                   float *dX, int64_t lddx, float *dW, float *db, void *ws, size_t ws_bytes, void *stream_)
{
    SG_REQUIRE(X && W && dY, SLICEGCN_EINVAL, "linear_bwd: NULL X, W or dY");
    SG_REQUIRE(n >= 1 && w_in >= 1 && w_out >= 1, SLICEGCN_EINVAL, "linear_bwd: sizes must be >= 1");
    SG_REQUIRE(ldx >= w_in && lddy >= w_out && (dX == nullptr || lddx >= w_in), SLICEGCN_EINVAL,
               "linear_bwd: leading dimension too small");
    SG_REQUIRE(act == SLICEGCN_ACT_NONE || act == SLICEGCN_ACT_RELU, SLICEGCN_EINVAL, "linear_bwd: unknown act %d", act);
    if (act == SLICEGCN_ACT_RELU)
        SG_REQUIRE(mask && mask_words >= (w_out + 31) / 32, SLICEGCN_EINVAL,
                   "linear_bwd: mask is NULL or mask_words < ceil(w_out / 32)");
    hipStream_t stream = as_stream(stream_);
    const uint32_t *m = act == SLICEGCN_ACT_RELU ? mask : nullptr;
    PairArgs a;
    a.A1 = dY; a.lda1 = lddy; a.A2 = nullptr; a.lda2 = 0;
    a.B1 = W; a.B2 = nullptr; a.bias1 = a.bias2 = nullptr;
    a.O1 = dX; a.ldo1 = lddx; a.O2 = nullptr; a.ldo2 = 0;
    a.mask = const_cast<uint32_t *>(m); a.mask_words = mask_words;
    a.n = n; a.K = w_out; a.Nout = w_in; a.ldw = w_out; a.act = act;
    if (int rc = check_in_place(&a, 1)) return rc; // before anything is launched
    bool dX_done = false;
    if (dW || db) {
        const size_t need = linear_partial_bytes(red_blocks(n), w_in, w_out);
        SG_REQUIRE(ws != nullptr && ws_bytes >= need, SLICEGCN_EWORKSPACE, "linear_bwd: workspace of %zu bytes, %zu needed",
                   ws_bytes, need);
        SG_REQUIRE((reinterpret_cast<uintptr_t>(ws) & 255u) == 0, SLICEGCN_EINVAL, "linear_bwd: workspace not 256-byte aligned");
        ProfScope prof(SLICEGCN_PROF_LINEAR_GRAD, w_out, stream);
        const LinearGradArgs args{X, m, dY, dW, db};
        if (int rc = launch_linear_grads(&args, 1, ldx, n, w_in, w_out, mask_words, lddy, ws, ws_bytes, stream, dX ? &a : nullptr, &dX_done))
            return rc;
    }
    if (dX && !dX_done) {
        ProfScope prof(SLICEGCN_PROF_LINEAR_BWD, w_in, stream);
        if (int rc = launch_pair<true>(a, stream)) return rc;
    }
    return SLICEGCN_OK;
}
