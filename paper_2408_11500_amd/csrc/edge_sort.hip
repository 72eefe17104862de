// Edge pairs -> distinct entries of the adjacency pattern, by row and ascending column, and each row's number of entries.
//
//   count, distribute   the keys (row, col) are distributed to buckets of consecutive rows, straight from the edge list: one pass over the
//                       keys for up to 512 buckets, two above; each reads them twice, to count and to move.  Runs of a digit are
//                       written in one piece per tile; the order within a bucket is whatever the LDS atomics give;
//   sort                a workgroup sorts a bucket in registers, drops repeats and counts its rows (degrees and their roots included),
//                       so that no later pass looks for row starts;
//   emit                column indices and values, once the row pointers are there (a scan of the degrees).
// Keys within a bucket are the low bits of the row and the column, 32 bits up to 2^25 nodes, so all but the first pass move 4 bytes per
// entry.  The result is a function of the set of pairs alone: integer counters decide only where a key waits to be sorted.
//
// 62 M edges, 2.4 M nodes (126 M keys): 3.7 ms with the schedule, where a device radix sort of 44-bit keys (six passes over 8-byte
// keys), a sweep for repeats and one for the values took 6.6.  Of it: counting and distributing 0.22 + 0.59 and 0.24 + 0.38 (5.5 GB, 3.9 TB/s),
// sorting 0.64 + 0.36 (vector unit and LDS crossbar: about 90 comparisons per key), columns and values 1.06 (gather of dinv[col]).
#include "common.h"

namespace slicegcn {

namespace {

constexpr int TPB = 256;
inline unsigned blocks_for(int64_t n) { return (unsigned)((n + TPB - 1) / TPB); }
// pieces of at most `size` that `count` items fill; counts reach 2^31 - 1, where adding size - 1 first would not fit
__device__ inline int32_t pieces_of(int32_t count, int32_t size) { return count / size + (count % size != 0 ? 1 : 0); }
inline unsigned bits_for(uint64_t v)
{
    unsigned b = 1;
    while ((v >> b) != 0) ++b;
    return b;
}

// ---- edges -> entries by row -------------------------------------------------------------
// How the entries are cut into buckets.  Bucket b holds the entries of the rows [b << row_shift, (b + 1) << row_shift); an entry is a
// key (row within the bucket) << col_bits | col.
//   * enough buckets that one holds about BUCKET_KEYS entries and is sorted by one workgroup in registers (126 M keys, sorting and
//     distributing: 1024 per bucket 2.44 ms, 2048 2.33, 4096 2.36);
//   * no more than 2^MAX_ROW_SHIFT rows in a bucket as far as the bits go (a workgroup counts the rows of its bucket);
//   * 32-bit keys where that takes no more than MAX_BITS bits of bucket number (up to 2^25 nodes), 64-bit keys above;
//   * up to 2^DIGIT_BITS buckets one pass over the edges distributes them, above it two passes by half of the bits each.
constexpr int DIGIT_BITS = 9, MAX_DIGITS = 1 << DIGIT_BITS, MAX_BITS = 2 * DIGIT_BITS;
constexpr int64_t BUCKET_KEYS = 2048;
constexpr int MAX_ROW_SHIFT = 11;
constexpr int PT = 512;           // threads of a distributing workgroup
// edges (two keys each) or diagonal entries a workgroup takes from the edge list: longer runs per digit or more workgroups on a CU (126 M keys,
// distributed: 2048 0.61 ms, 2560 0.60, 3072 0.57, 3584 0.64, 4096 0.62)
constexpr int TILE_ITEMS = 3072;
constexpr int TILE_KEYS = 8192;   // keys a workgroup takes in the second pass
constexpr int SORT_KEYS = 8192;   // most keys one workgroup sorts in registers
constexpr int MOST_KEYS = 16384;  // most a larger workgroup does; buckets of more are cut once more

struct BucketPlan {
    int64_t n_items, max_keys; // edges and diagonal entries; the most keys they can give
    int col_bits, row_shift, bits1, bits2; // digits of the two passes (bits2 = 0: one pass)
    int64_t n_buckets, tiles1, max_tiles2;
    bool wide; // 64-bit keys
    size_t key_bytes() const { return wide ? 8 : 4; }
    int64_t digits1() const { return bits2 ? ((n_buckets - 1) >> bits2) + 1 : n_buckets; }
    int64_t counts1() const { return digits1() * tiles1 + 1; }
    int64_t counts2() const { return bits2 ? (max_tiles2 << bits2) + 1 : 0; }
};
BucketPlan bucket_plan(int64_t n_edges, int64_t n, bool sym, bool loops)
{
    BucketPlan p;
    p.n_items = n_edges + (loops ? n : 0);
    p.max_keys = n_edges * (sym ? 2 : 1) + (loops ? n : 0);
    p.col_bits = (int)bits_for((uint64_t)(n - 1));
    int bits = 0; // of the bucket number
    while (bits < MAX_BITS && bits < p.col_bits && (p.max_keys >> bits) > BUCKET_KEYS) ++bits;
    if (bits < p.col_bits - MAX_ROW_SHIFT) bits = p.col_bits - MAX_ROW_SHIFT < MAX_BITS ? p.col_bits - MAX_ROW_SHIFT : MAX_BITS;
    p.wide = 2 * p.col_bits - MAX_BITS > 32;
    if (!p.wide && bits < 2 * p.col_bits - 32) bits = 2 * p.col_bits - 32;
    p.row_shift = p.col_bits - bits;
    p.n_buckets = ((n - 1) >> p.row_shift) + 1;
    p.bits1 = bits <= DIGIT_BITS ? bits : bits / 2;
    p.bits2 = bits - p.bits1;
    p.tiles1 = (p.n_items + TILE_ITEMS - 1) / TILE_ITEMS;
    p.max_tiles2 = p.max_keys / TILE_KEYS + MAX_DIGITS;
    return p;
}

struct EdgeList {
    const int64_t *row, *col;
    int64_t n_edges, n, n_items;
    int sym;
    int col_bits, shift; // digit of a row = row >> shift
};

// The keys of item i: an edge gives (row, col) and, symmetrised, (col, row); the items behind the edges give the diagonal.  Self pairs
// give nothing, pairs with an id out of range nothing but a count.
template <class F> __device__ inline void for_each_key(const EdgeList &e, int64_t i, int &bad, F f)
{
    if (i < e.n_edges) {
        const int64_t u = e.row[i], v = e.col[i];
        if (u < 0 || u >= e.n || v < 0 || v >= e.n) {
            ++bad;
        } else if (u != v) {
            f(0, (uint32_t)u, (uint32_t)v);
            if (e.sym) f(1, (uint32_t)v, (uint32_t)u);
        }
    } else if (i < e.n_items) {
        f(0, (uint32_t)(i - e.n_edges), (uint32_t)(i - e.n_edges));
    }
}

// counts[digit * tiles + tile]: keys of every digit in a tile of the edge list
__global__ __launch_bounds__(PT) void count_edges_kernel(const EdgeList e, int64_t n_tiles, int n_digits, int32_t *__restrict__ counts, int32_t *__restrict__ n_bad)
{
    __shared__ int32_t cnt[MAX_DIGITS];
    for (int d = threadIdx.x; d < MAX_DIGITS; d += PT) cnt[d] = 0;
    __syncthreads();
    int bad = 0;
    const int64_t first = (int64_t)blockIdx.x * TILE_ITEMS + threadIdx.x;
#pragma unroll
    for (int j = 0; j < TILE_ITEMS / PT; ++j)
        for_each_key(e, first + j * PT, bad, [&](int, uint32_t row, uint32_t) { atomicAdd(&cnt[row >> e.shift], 1); });
    if (bad) atomicAdd(n_bad, bad);
    __syncthreads();
    for (int d = threadIdx.x; d < n_digits; d += PT) counts[(int64_t)d * n_tiles + blockIdx.x] = cnt[d];
}

// off = exclusive prefix sums of the MAX_DIGITS counts, one per thread of the workgroup; returns the total
__device__ inline int scan_digits(const int32_t *cnt, int32_t *off, int32_t *wave_sums)
{
    static_assert(PT == MAX_DIGITS, "one digit per thread");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t mine = cnt[threadIdx.x];
    int32_t sum = mine;
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) {
        const int32_t up = __shfl_up(sum, s, 64);
        if (lane >= s) sum += up;
    }
    if (lane == 63) wave_sums[wave] = sum;
    __syncthreads();
    int32_t before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < PT / 64; ++w) {
        before += w < wave ? wave_sums[w] : 0;
        total += wave_sums[w];
    }
    off[threadIdx.x] = before + sum - mine;
    return total;
}

// Distributes a tile of the edge list: the keys are ranked by digit in LDS (in any order within a digit: they are sorted later), laid out by
// digit there and written as one run per digit.  at[digit * tiles + tile]: where the tile's run of a digit starts.
// BUCKET: the digit is the bucket, the key has the row within it and the column.
// Otherwise there is a second pass.  32-bit keys: row bits within the bucket as well, and the second digit goes to an array of its own
// (6 bytes a key instead of 8, of which the counting reads 2: 126 M keys distributed 0.59 -> 0.57 ms, counted 0.25 -> 0.09, distributed again
// 0.38 -> 0.35); 64-bit keys: the whole row.
template <class K, bool BUCKET>
__global__ __launch_bounds__(PT) void distribute_edges_kernel(const EdgeList e, int64_t n_tiles, int n_digits, const int32_t *__restrict__ at, K *__restrict__ out,
                                                              int bits2, uint16_t *__restrict__ second)
{
    constexpr bool SPLIT = !BUCKET && sizeof(K) == 4;
    __shared__ K keys[2 * TILE_ITEMS];
    __shared__ uint16_t digit[BUCKET || SPLIT ? 2 * TILE_ITEMS : 1], digit2[SPLIT ? 2 * TILE_ITEMS : 1];
    __shared__ int32_t cnt[MAX_DIGITS], off[MAX_DIGITS], wave_sums[PT / 64];
    constexpr int J = TILE_ITEMS / PT;
    cnt[threadIdx.x] = 0;
    __syncthreads();
    uint32_t row[J][2], col[J][2];
    int32_t rank[J][2];
    int bad = 0;
    const int64_t first = (int64_t)blockIdx.x * TILE_ITEMS + threadIdx.x;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        rank[j][0] = rank[j][1] = -1;
        for_each_key(e, first + j * PT, bad, [&](int which, uint32_t r, uint32_t c) {
            row[j][which] = r;
            col[j][which] = c;
            rank[j][which] = atomicAdd(&cnt[r >> e.shift], 1);
        });
    }
    __syncthreads();
    const int total = scan_digits(cnt, off, wave_sums);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int w = 0; w < 2; ++w)
            if (rank[j][w] >= 0) {
                const int within = e.shift - (SPLIT ? bits2 : 0); // row bits within the bucket
                const uint32_t d = row[j][w] >> e.shift, r = BUCKET || SPLIT ? row[j][w] & ((1u << within) - 1u) : row[j][w];
                const int pos = off[d] + rank[j][w];
                keys[pos] = ((K)r << e.col_bits) | (K)col[j][w];
                if (BUCKET || SPLIT) digit[pos] = (uint16_t)d;
                if (SPLIT) digit2[pos] = (uint16_t)((row[j][w] >> within) & ((1u << bits2) - 1u));
            }
    if ((int)threadIdx.x < n_digits) cnt[threadIdx.x] = at[(int64_t)threadIdx.x * n_tiles + blockIdx.x] - off[threadIdx.x]; // the ranks are in registers
    __syncthreads();
    for (int i = threadIdx.x; i < total; i += PT) {
        const K k = keys[i];
        const int64_t to = (int64_t)cnt[BUCKET || SPLIT ? digit[i] : (int)(k >> (e.col_bits + e.shift))] + i;
        out[to] = k;
        if (SPLIT) second[to] = digit2[i];
    }
}

// Tiles of the second pass: the keys of first-pass digit d are cut into tiles of their own, numbered from tile_start[d].
// at1: scanned counts of the first pass; start1 of digit d = at1[d * tiles1]
__global__ __launch_bounds__(PT) void tile_starts_kernel(const int32_t *__restrict__ at1, int64_t tiles1, int n_digits, int32_t *__restrict__ tile_start)
{
    __shared__ int32_t cnt[MAX_DIGITS], off[MAX_DIGITS], wave_sums[PT / 64];
    const int d = threadIdx.x;
    cnt[d] = d < n_digits ? pieces_of(at1[(int64_t)(d + 1) * tiles1] - at1[(int64_t)d * tiles1], TILE_KEYS) : 0;
    __syncthreads();
    const int total = scan_digits(cnt, off, wave_sums);
    if (d < n_digits) tile_start[d] = off[d];
    if (d == 0) tile_start[n_digits] = total;
}

struct SecondPass {
    const void *keys;          // by first-pass digit: keys of the sorting's type and their second digits, or whole 64-bit keys
    const uint16_t *second;
    const int32_t *at1;        // see tile_starts_kernel
    const int32_t *tile_start; // [digits1 + 1]
    int64_t tiles1;
    int digits1, bits2, col_bits, row_shift;
};
struct SecondTile { int d, tile, tiles; int64_t beg, end; };
__device__ inline bool second_tile(const SecondPass &p, int block, SecondTile &t)
{
    if (block >= p.tile_start[p.digits1]) return false;
    int lo = 0, hi = p.digits1 - 1; // last digit whose first tile is at or before this one (digits without tiles share a start)
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (p.tile_start[mid] <= block) lo = mid; else hi = mid - 1;
    }
    t.d = lo;
    t.tile = block - p.tile_start[lo];
    t.tiles = p.tile_start[lo + 1] - p.tile_start[lo];
    t.beg = p.at1[(int64_t)lo * p.tiles1] + (int64_t)t.tile * TILE_KEYS;
    const int64_t end = p.at1[(int64_t)(lo + 1) * p.tiles1];
    t.end = t.beg + TILE_KEYS < end ? t.beg + TILE_KEYS : end;
    return true;
}
// place of (first-pass digit, second digit, tile) in the counts: all tiles of a bucket in a row, buckets in order
__device__ inline int64_t second_count(const SecondPass &p, const SecondTile &t, int d2)
{
    return ((int64_t)p.tile_start[t.d] << p.bits2) + (int64_t)d2 * t.tiles + t.tile;
}

// Key i as it is sorted, and its second digit
template <class K> __device__ inline K low_key(const SecondPass &p, int64_t i)
{
    const K k = static_cast<const K *>(p.keys)[i];
    return sizeof(K) == 4 ? k : k & (K)(((uint64_t)1 << (p.col_bits + p.row_shift)) - 1);
}
template <class K> __device__ inline int second_digit(const SecondPass &p, int64_t i)
{
    if constexpr (sizeof(K) == 4) return p.second[i];
    else return (int)(static_cast<const K *>(p.keys)[i] >> (p.col_bits + p.row_shift)) & ((1 << p.bits2) - 1);
}

template <class K>
__global__ __launch_bounds__(PT) void count_keys_kernel(const SecondPass p, int32_t *__restrict__ counts)
{
    __shared__ int32_t cnt[MAX_DIGITS];
    SecondTile t;
    if (!second_tile(p, blockIdx.x, t)) return; // uniform per workgroup
    cnt[threadIdx.x] = 0;
    __syncthreads();
    constexpr int J = TILE_KEYS / PT;
    int d[J];
#pragma unroll
    for (int j = 0; j < J; ++j) { // every load before the first use
        const int64_t i = t.beg + j * PT + threadIdx.x;
        d[j] = second_digit<K>(p, i < t.end ? i : t.beg);
    }
#pragma unroll
    for (int j = 0; j < J; ++j)
        if (t.beg + j * PT + threadIdx.x < t.end) atomicAdd(&cnt[d[j]], 1);
    __syncthreads();
    if ((int)threadIdx.x < 1 << p.bits2) counts[second_count(p, t, threadIdx.x)] = cnt[threadIdx.x];
}

template <class K>
__global__ __launch_bounds__(PT) void distribute_keys_kernel(const SecondPass p, const int32_t *__restrict__ at, K *__restrict__ out)
{
    __shared__ K keys[TILE_KEYS];
    __shared__ uint16_t digit[TILE_KEYS];
    __shared__ int32_t cnt[MAX_DIGITS], off[MAX_DIGITS], wave_sums[PT / 64];
    constexpr int J = TILE_KEYS / PT;
    SecondTile t;
    if (!second_tile(p, blockIdx.x, t)) return; // uniform per workgroup
    cnt[threadIdx.x] = 0;
    __syncthreads();
    K k[J];
    int d[J];
    int32_t rank[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int64_t i = t.beg + j * PT + threadIdx.x, from = i < t.end ? i : t.beg;
        k[j] = low_key<K>(p, from);
        d[j] = second_digit<K>(p, from);
    }
#pragma unroll
    for (int j = 0; j < J; ++j) rank[j] = t.beg + j * PT + threadIdx.x < t.end ? atomicAdd(&cnt[d[j]], 1) : -1;
    __syncthreads();
    const int total = scan_digits(cnt, off, wave_sums);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < J; ++j)
        if (rank[j] >= 0) {
            const int pos = off[d[j]] + rank[j];
            keys[pos] = k[j];
            digit[pos] = (uint16_t)d[j];
        }
    if ((int)threadIdx.x < 1 << p.bits2) cnt[threadIdx.x] = at[second_count(p, t, threadIdx.x)] - off[threadIdx.x];
    __syncthreads();
    for (int i = threadIdx.x; i < total; i += PT) out[(int64_t)cnt[digit[i]] + i] = keys[i];
}

// start[b] = first key of bucket b, start[n_buckets] = number of keys.  Two passes: at2 = scanned counts of the second one.
__global__ void bucket_starts_kernel(const SecondPass p, const int32_t *__restrict__ at2, int64_t n_buckets, int32_t *__restrict__ start)
{
    const int64_t b = (int64_t)blockIdx.x * TPB + threadIdx.x;
    if (b > n_buckets) return;
    if (p.bits2 == 0) { // digits are buckets
        start[b] = p.at1[b * p.tiles1];
        return;
    }
    const int d = (int)(b >> p.bits2);
    if (b == n_buckets || p.tile_start[d + 1] == p.tile_start[d]) { // the end; digits without keys
        start[b] = p.at1[(int64_t)(b == n_buckets ? p.digits1 : d) * p.tiles1];
        return;
    }
    const SecondTile t{d, 0, p.tile_start[d + 1] - p.tile_start[d], 0, 0};
    start[b] = at2[second_count(p, t, (int)(b & ((1 << p.bits2) - 1)))];
}

// ---- sorting within a workgroup ----------------------------------------------------------
// Value of lane ^ X: within 16 lanes by the data-parallel paths of the vector unit (no LDS), otherwise through the LDS crossbar.
template <int X> __device__ inline uint32_t lane_xor(uint32_t v)
{
    const int i = (int)v;
    if constexpr (X == 1) return (uint32_t)__builtin_amdgcn_mov_dpp(i, 0xB1, 0xF, 0xF, true);         // quad_perm [1,0,3,2]
    else if constexpr (X == 2) return (uint32_t)__builtin_amdgcn_mov_dpp(i, 0x4E, 0xF, 0xF, true);    // quad_perm [2,3,0,1]
    else if constexpr (X == 3) return (uint32_t)__builtin_amdgcn_mov_dpp(i, 0x1B, 0xF, 0xF, true);    // quad_perm [3,2,1,0]
    else if constexpr (X == 7) return (uint32_t)__builtin_amdgcn_mov_dpp(i, 0x141, 0xF, 0xF, true);   // row_half_mirror
    else if constexpr (X == 15) return (uint32_t)__builtin_amdgcn_mov_dpp(i, 0x140, 0xF, 0xF, true);  // row_mirror
    else if constexpr (X == 8) return (uint32_t)__builtin_amdgcn_mov_dpp(i, 0x128, 0xF, 0xF, true);   // row_ror:8
    else if constexpr (X < 32) return (uint32_t)__builtin_amdgcn_ds_swizzle(i, (X << 10) | 0x1F);
    else return (uint32_t)__shfl_xor(i, X, 64);
}
template <int X> __device__ inline uint64_t lane_xor(uint64_t v)
{
    return ((uint64_t)lane_xor<X>((uint32_t)(v >> 32)) << 32) | lane_xor<X>((uint32_t)v);
}

template <class K> __device__ inline void order(K &a, K &b) { const K lo = a < b ? a : b, hi = a < b ? b : a; a = lo; b = hi; }
// the smaller of a and b where `bound` is 0, the larger where it is the type's largest: the middle one of the three
template <class K> __device__ inline K pick_side(K a, K b, K bound)
{
    const K lo = a < b ? a : b, hi = a < b ? b : a, top = hi < bound ? hi : bound;
    return lo > top ? lo : top;
}

// steps of distance D * KPT, D / 2 * KPT, ..., KPT (one element per lane each)
template <class K, int KPT, int D> __device__ inline void lane_steps(K (&k)[KPT], int tid)
{
    if constexpr (D >= 1) {
        const K bound = tid & D ? (K)~(K)0 : (K)0;
#pragma unroll
        for (int r = 0; r < KPT; ++r) k[r] = pick_side(k[r], lane_xor<D>(k[r]), bound);
        lane_steps<K, KPT, D / 2>(k, tid);
    }
}
template <class K, int KPT> __device__ inline void register_steps(K (&k)[KPT])
{
#pragma unroll
    for (int j = KPT / 2; j >= 1; j >>= 1)
#pragma unroll
        for (int i = 0; i < KPT; ++i)
            if (!(i & j)) order(k[i], k[i + j]);
}
// merges sorted runs of T / 2 threads into runs of T threads, T = 2 .. 64
template <class K, int KPT, int T> __device__ inline void lane_stages(K (&k)[KPT], int tid)
{
    if constexpr (T <= 64) {
        const K bound = tid & (T / 2) ? (K)~(K)0 : (K)0;
        K o[KPT];
#pragma unroll
        for (int r = 0; r < KPT; ++r) o[r] = lane_xor<T - 1>(k[KPT - 1 - r]);
#pragma unroll
        for (int r = 0; r < KPT; ++r) k[r] = pick_side(k[r], o[r], bound);
        lane_steps<K, KPT, T / 4>(k, tid);
        register_steps<K, KPT>(k);
        lane_stages<K, KPT, 2 * T>(k, tid);
    }
}

// Sorts the KPT * THREADS keys of a workgroup, element tid * KPT + r in register r of thread tid (bitonic network in the form whose
// first step of a stage pairs an element with its mirror image: every comparison then orders upwards, and side and distance
// are constants or bits of the lane).  Only steps between wavefronts go through LDS (buf: KPT * THREADS keys).
template <class K, int KPT, int THREADS> __device__ inline void sort_keys(K (&k)[KPT], K *buf, int tid)
{
#pragma unroll
    for (int size = 2; size <= KPT; size <<= 1) {
#pragma unroll
        for (int i = 0; i < KPT; ++i)
            if ((i & (size - 1)) < size / 2) order(k[i], k[i ^ (size - 1)]);
#pragma unroll
        for (int j = size / 4; j >= 1; j >>= 1)
#pragma unroll
            for (int i = 0; i < KPT; ++i)
                if (!(i & j)) order(k[i], k[i + j]);
    }
    lane_stages<K, KPT, 2>(k, tid);
    auto across = [&](int partner, bool mirror, bool upper) {
        __syncthreads(); // what was read from buf before
#pragma unroll
        for (int r = 0; r < KPT; ++r) buf[r * THREADS + tid] = k[r];
        __syncthreads();
        const K bound = upper ? (K)~(K)0 : (K)0;
#pragma unroll
        for (int r = 0; r < KPT; ++r) k[r] = pick_side(k[r], buf[(mirror ? KPT - 1 - r : r) * THREADS + partner], bound);
    };
#pragma unroll 1
    for (int t = 128; t <= THREADS; t <<= 1) {
        across(tid ^ (t - 1), true, (tid & (t / 2)) != 0);
#pragma unroll 1
        for (int d = t / 4; d >= 64; d >>= 1) across(tid ^ d, false, (tid & d) != 0);
        lane_steps<K, KPT, 32>(k, tid);
        register_steps<K, KPT>(k);
    }
}

// exclusive prefix sum over the workgroup's threads; sums: THREADS / 64 words.  Synchronises before and after it uses them.
template <int THREADS> __device__ inline int32_t scan_threads(int32_t mine, int32_t *sums, int tid, int32_t &total)
{
    const int lane = tid & 63, wave = tid >> 6;
    int32_t sum = mine;
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) {
        const int32_t up = __shfl_up(sum, s, 64);
        if (lane >= s) sum += up;
    }
    __syncthreads();
    if (lane == 63) sums[wave] = sum;
    __syncthreads();
    int32_t before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) {
        before += w < wave ? sums[w] : 0;
        total += sums[w];
    }
    return before + sum - mine;
}

// Loads cnt <= KPT * THREADS keys, leaves the distinct ones in ascending order in buf and returns how many.  Ends synchronised.
template <class K, int KPT, int THREADS>
__device__ inline int32_t sort_distinct(const K *keys, int32_t cnt, K *buf, K *last, int32_t *sums, int tid)
{
    K k[KPT];
#pragma unroll
    for (int r = 0; r < KPT; ++r) { // any order will do; what is missing sorts to the end
        const int32_t i = r * THREADS + tid;
        k[r] = i < cnt ? keys[i] : (K)~(K)0;
    }
    sort_keys<K, KPT, THREADS>(k, buf, tid);
    last[tid] = k[KPT - 1];
    __syncthreads(); // also: buf has been read
    K prev = tid > 0 ? last[tid - 1] : (K)0;
    bool keep[KPT];
    int32_t mine = 0;
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
        const int32_t e = tid * KPT + r;
        keep[r] = e < cnt && (e == 0 || k[r] != prev);
        mine += keep[r] ? 1 : 0;
        prev = k[r];
    }
    int32_t total;
    int32_t at = scan_threads<THREADS>(mine, sums, tid, total);
#pragma unroll
    for (int r = 0; r < KPT; ++r)
        if (keep[r]) buf[at++] = k[r];
    __syncthreads();
    return total;
}

// What a row's number of entries gives
struct RowOut {
    int32_t *deg;
    float *dinv, *sqrtd; // may be NULL
};
__device__ inline void put_row(const RowOut &o, int64_t row, int32_t d)
{
    o.deg[row] = d;
    if (o.dinv) {
        o.dinv[row] = (float)(1.0 / sqrt((double)(d > 0 ? d : 1)));
        o.sqrtd[row] = (float)sqrt((double)(d > 0 ? d : 1));
    }
}

constexpr int SUB_BITS = 11, SUBS = 1 << SUB_BITS;
struct Buckets {
    const int32_t *start; // [n_buckets + 1]
    int32_t *kept;        // distinct keys of every bucket, from its start on
    int32_t *big;         // buckets of more than SORT_KEYS keys, in no particular order
    int32_t *huge;        // buckets of more than MOST_KEYS keys, likewise; such a bucket is cut by the high bits of its keys into SUBS parts,
    int2 *tiles;          // in tiles of TILE_KEYS keys: (h, tile) of all tiles, for the h-th such bucket
    int32_t *sub_count;   // [h * SUBS + u] keys of part u; at the end the distinct keys of the parts before it
    int32_t *sub_kept;    // [h * SUBS + u] how many keys of the part have been dealt out; then the distinct keys of the group it begins, or 0
    int32_t *sub_start;   // [h * (SUBS + 1) + u] the part's first key
    int2 *groups;         // (h * SUBS + first part, parts) of every group of parts, which are sorted together
    int2 *pieces;         // (bucket, piece) of every piece but the first of the buckets with more than EMIT_PIECE distinct keys, and of all
                          // pieces of groups (-1 - h * SUBS - first part in the bucket's place), in no order
    int32_t *n_big, *n_huge, *n_tiles, *n_groups, *n_pieces;
    int64_t n, n_buckets;
    int col_bits, row_shift;
    __host__ __device__ int sub_shift() const { return row_shift + col_bits > SUB_BITS ? row_shift + col_bits - SUB_BITS : 0; }
    __device__ int rows_of(int64_t b) const
    {
        const int64_t left = n - (b << row_shift);
        return left < ((int64_t)1 << row_shift) ? (int)left : 1 << row_shift;
    }
};

constexpr int EMIT_PIECE = 2048; // entries a workgroup writes
// lists pieces `first` ... of a bucket or part with so many distinct keys
__device__ inline void list_pieces(const Buckets &s, int64_t id, int32_t kept, int32_t first, int tid)
{
    const int32_t more = pieces_of(kept, EMIT_PIECE) - first;
    if (more <= 0) return; // uniform per workgroup
    __shared__ int32_t at;
    if (tid == 0) at = atomicAdd(s.n_pieces, more);
    __syncthreads();
    for (int32_t i = tid; i < more; i += blockDim.x) s.pieces[at + i] = make_int2((int)id, first + i);
}

template <class K> __device__ inline int32_t first_at_or_above(const K *sorted, int32_t count, uint64_t value)
{
    int32_t lo = 0, hi = count;
    while (lo < hi) {
        const int32_t mid = (lo + hi) >> 1;
        if ((uint64_t)sorted[mid] < value) lo = mid + 1; else hi = mid;
    }
    return lo;
}
// the rows of the bucket whose first row is row0, from its distinct keys
template <class K, int THREADS>
__device__ inline void put_rows(const Buckets &s, const RowOut &o, int64_t row0, int rows, const K *sorted, int32_t count, int tid)
{
    for (int r = tid; r < rows; r += THREADS)
        put_row(o, row0 + r, first_at_or_above(sorted, count, (uint64_t)(r + 1) << s.col_bits) - first_at_or_above(sorted, count, (uint64_t)r << s.col_bits));
}

// One workgroup per bucket: sorts its keys in registers, drops repeats, writes them back and counts its rows.  Larger buckets are listed.
template <class K>
__global__ __launch_bounds__(256) void sort_buckets_kernel(const Buckets s, const RowOut o, K *__restrict__ keys)
{
    __shared__ K buf[SORT_KEYS];
    __shared__ K last[256];
    __shared__ int32_t sums[4], place, first_tile;
    const int tid = threadIdx.x;
    const int64_t b = blockIdx.x, row0 = b << s.row_shift;
    const int32_t beg = s.start[b], cnt = s.start[b + 1] - beg;
    if (cnt > MOST_KEYS) { // uniform per workgroup
        const int32_t tiles = pieces_of(cnt, TILE_KEYS);
        if (tid == 0) {
            place = atomicAdd(s.n_huge, 1);
            first_tile = atomicAdd(s.n_tiles, tiles);
            s.huge[place] = (int32_t)b;
            s.kept[b] = 0;
        }
        __syncthreads();
        for (int32_t t = tid; t < tiles; t += 256) s.tiles[first_tile + t] = make_int2(place, t);
        for (int u = tid; u < SUBS; u += 256) s.sub_count[place * SUBS + u] = s.sub_kept[place * SUBS + u] = 0;
        for (int r = tid; r < s.rows_of(b); r += 256) o.deg[row0 + r] = 0; // the groups add to it
        return;
    }
    if (cnt > SORT_KEYS) {
        if (tid == 0) s.big[atomicAdd(s.n_big, 1)] = (int32_t)b;
        return;
    }
    K *mine = keys + beg;
    int32_t m;
    if (cnt <= 1024) m = sort_distinct<K, 4, 256>(mine, cnt, buf, last, sums, tid);
    else if (cnt <= 2048) m = sort_distinct<K, 8, 256>(mine, cnt, buf, last, sums, tid);
    else if (cnt <= 4096) m = sort_distinct<K, 16, 256>(mine, cnt, buf, last, sums, tid);
    else m = sort_distinct<K, 32, 256>(mine, cnt, buf, last, sums, tid);
    for (int32_t i = tid; i < m; i += 256) mine[i] = buf[i];
    put_rows<K, 256>(s, o, row0, s.rows_of(b), buf, m, tid);
    if (tid == 0) s.kept[b] = m;
    list_pieces(s, b, m, 1, tid);
}

// The buckets a hub (or a few) makes so large that one workgroup would be the whole build's last: their keys are counted and dealt by their
// SUB_BITS high bits, in tiles as in the passes before, by many workgroups, and runs of parts that fit a workgroup's registers are
// then sorted each on its own.  (One workgroup per such bucket: 3.3 ms for a star of a million nodes, 7.7 ms for 126 M entries whose hubs
// have neighbouring ids.)
struct HugeTile { int h; int64_t b, beg, end; };
__device__ inline HugeTile huge_tile(const Buckets &s, int at)
{
    const int2 t = s.tiles[at];
    const int64_t b = s.huge[t.x], beg = s.start[b] + (int64_t)t.y * TILE_KEYS, end = s.start[b + 1];
    return HugeTile{t.x, b, beg, beg + TILE_KEYS < end ? beg + TILE_KEYS : end};
}
constexpr int TILE_BLOCKS = 1024; // workgroups that take the tiles in turn
template <class K> __global__ __launch_bounds__(PT) void count_huge_kernel(const Buckets s, const K *__restrict__ keys)
{
    __shared__ int32_t cnt[SUBS];
    const int shift = s.sub_shift(), tid = threadIdx.x, n_tiles = *s.n_tiles;
    for (int at = blockIdx.x; at < n_tiles; at += gridDim.x) {
        const HugeTile t = huge_tile(s, at);
        for (int u = tid; u < SUBS; u += PT) cnt[u] = 0;
        __syncthreads();
        K k[TILE_KEYS / PT];
#pragma unroll
        for (int j = 0; j < TILE_KEYS / PT; ++j) k[j] = keys[t.beg + j * PT + tid < t.end ? t.beg + j * PT + tid : t.beg];
#pragma unroll
        for (int j = 0; j < TILE_KEYS / PT; ++j)
            if (t.beg + j * PT + tid < t.end) atomicAdd(&cnt[k[j] >> shift], 1);
        __syncthreads();
        for (int u = tid; u < SUBS; u += PT)
            if (cnt[u] > 0) atomicAdd(&s.sub_count[t.h * SUBS + u], cnt[u]);
        __syncthreads();
    }
}
// Where the parts of a huge bucket start, and its groups: runs of parts of together at most MOST_KEYS keys, or one part of more.
__global__ __launch_bounds__(PT) void group_huge_kernel(const Buckets s)
{
    constexpr int R = SUBS / PT;
    __shared__ int32_t end[SUBS], sums[PT / 64], n_new, first;
    __shared__ int2 list[SUBS];
    const int tid = threadIdx.x, n_huge = *s.n_huge;
    for (int h = blockIdx.x; h < n_huge; h += gridDim.x) {
        int32_t c[R], sum = 0, total;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            c[q] = s.sub_count[h * SUBS + tid * R + q];
            sum += c[q];
        }
        const int32_t start = s.start[s.huge[h]];
        int32_t from = scan_threads<PT>(sum, sums, tid, total);
#pragma unroll
        for (int q = 0; q < R; ++q) {
            s.sub_start[h * (SUBS + 1) + tid * R + q] = start + from;
            from += c[q];
            end[tid * R + q] = from;
        }
        if (tid == 0) s.sub_start[h * (SUBS + 1) + SUBS] = start + total;
        __syncthreads();
        if (tid == 0) {
            int n = 0;
            for (int u = 0; u < SUBS;) {
                const int32_t before = u > 0 ? end[u - 1] : 0;
                int lo = u + 1, hi = SUBS; // most parts [u, lo) that fit, one at least
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (end[mid - 1] - before <= MOST_KEYS) lo = mid; else hi = mid - 1;
                }
                if (end[lo - 1] > before) list[n++] = make_int2(h * SUBS + u, lo - u);
                u = lo;
            }
            n_new = n;
            first = atomicAdd(s.n_groups, n);
        }
        __syncthreads();
        for (int i = tid; i < n_new; i += PT) s.groups[first + i] = list[i];
        __syncthreads();
    }
}
template <class K> __global__ __launch_bounds__(PT) void deal_huge_kernel(const Buckets s, const K *__restrict__ keys, K *__restrict__ dealt)
{
    __shared__ int32_t cnt[SUBS];
    const int shift = s.sub_shift(), tid = threadIdx.x, n_tiles = *s.n_tiles;
    for (int at = blockIdx.x; at < n_tiles; at += gridDim.x) {
        const HugeTile t = huge_tile(s, at);
        for (int u = tid; u < SUBS; u += PT) cnt[u] = 0;
        __syncthreads();
        K k[TILE_KEYS / PT];
        int32_t rank[TILE_KEYS / PT];
#pragma unroll
        for (int j = 0; j < TILE_KEYS / PT; ++j) k[j] = keys[t.beg + j * PT + tid < t.end ? t.beg + j * PT + tid : t.beg];
#pragma unroll
        for (int j = 0; j < TILE_KEYS / PT; ++j) rank[j] = t.beg + j * PT + tid < t.end ? atomicAdd(&cnt[k[j] >> shift], 1) : -1;
        __syncthreads();
        for (int u = tid; u < SUBS; u += PT)
            if (cnt[u] > 0) cnt[u] = s.sub_start[t.h * (SUBS + 1) + u] + atomicAdd(&s.sub_kept[t.h * SUBS + u], cnt[u]);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < TILE_KEYS / PT; ++j)
            if (rank[j] >= 0) dealt[(int64_t)cnt[k[j] >> shift] + rank[j]] = k[j];
        __syncthreads();
    }
}

// The larger buckets, and the groups of the huge ones.  A part of more keys than fit (repeats, or a row nearly as dense as its columns
// allow) goes through a bitmap of its keys' low bits, BITMAP of them at a time, which drops repeats by itself.
constexpr int BIG_THREADS = 512;
template <class K>
__global__ __launch_bounds__(BIG_THREADS) void sort_big_buckets_kernel(const Buckets s, const RowOut o, K *__restrict__ keys, const K *__restrict__ dealt)
{
    constexpr int WORDS = MOST_KEYS * sizeof(K) / 4, BITMAP = 32 * WORDS, U = 16;
    __shared__ __attribute__((aligned(16))) uint32_t mem[WORDS]; // the keys being sorted, or the bitmap
    __shared__ K last[BIG_THREADS];
    __shared__ int32_t sums[BIG_THREADS / 64];
    K *buf = reinterpret_cast<K *>(mem);
    const int tid = threadIdx.x, shift = s.sub_shift();
    const int n_groups = *s.n_groups, n_big = *s.n_big;
    for (int at = blockIdx.x; at < n_groups + n_big; at += gridDim.x) {
        __syncthreads(); // buf is used again
        if (at >= n_groups) { // uniform per workgroup
            const int64_t b = s.big[at - n_groups], row0 = b << s.row_shift;
            const int32_t beg = s.start[b], cnt = s.start[b + 1] - beg;
            K *mine = keys + beg;
            const int32_t m = sort_distinct<K, MOST_KEYS / BIG_THREADS, BIG_THREADS>(mine, cnt, buf, last, sums, tid);
            for (int32_t i = tid; i < m; i += BIG_THREADS) mine[i] = buf[i];
            put_rows<K, BIG_THREADS>(s, o, row0, s.rows_of(b), buf, m, tid);
            if (tid == 0) s.kept[b] = m;
            list_pieces(s, b, m, 1, tid);
            continue;
        }
        const int2 g = s.groups[at];
        const int h = g.x / SUBS, u = g.x % SUBS;
        const int64_t b = s.huge[h], row0 = b << s.row_shift;
        const int32_t beg = s.sub_start[h * (SUBS + 1) + u], cnt = s.sub_start[h * (SUBS + 1) + u + g.y] - beg;
        const K *from = dealt + beg;
        K *mine = keys + beg;
        int32_t m = 0;
        if (cnt > MOST_KEYS) { // one part
            const K high = (K)u << shift;
            for (int64_t x0 = 0; x0 < ((int64_t)1 << shift); x0 += BITMAP) {
                __syncthreads();
                for (int i = tid; i < WORDS; i += BIG_THREADS) mem[i] = 0u;
                __syncthreads();
                for (int64_t i0 = tid; i0 < cnt; i0 += BIG_THREADS * U) {
                    K k[U];
#pragma unroll
                    for (int q = 0; q < U; ++q) k[q] = from[i0 + q * BIG_THREADS < cnt ? i0 + q * BIG_THREADS : i0]; // repeats do no harm
#pragma unroll
                    for (int q = 0; q < U; ++q) {
                        const int64_t x = (int64_t)(k[q] - high) - x0;
                        if (x >= 0 && x < BITMAP && !(mem[x >> 5] >> (x & 31) & 1u)) atomicOr(&mem[x >> 5], 1u << (x & 31));
                    }
                }
                __syncthreads();
                constexpr int W = WORDS / BIG_THREADS; // words per thread
                int32_t bits = 0, all;
#pragma unroll
                for (int q = 0; q < W; ++q) bits += __popc(mem[tid * W + q]);
                int32_t to = m + scan_threads<BIG_THREADS>(bits, sums, tid, all);
#pragma unroll 1
                for (int q = 0; q < W; ++q)
                    for (uint32_t w = mem[tid * W + q]; w != 0u; w &= w - 1u) mine[to++] = high + (K)(x0 + (tid * W + q) * 32 + __ffs(w) - 1);
                m += all;
            }
            __syncthreads(); // the keys are read back below
        } else {
            m = sort_distinct<K, MOST_KEYS / BIG_THREADS, BIG_THREADS>(from, cnt, buf, last, sums, tid);
            for (int32_t i = tid; i < m; i += BIG_THREADS) mine[i] = buf[i];
        }
        const K *sorted = cnt > MOST_KEYS ? mine : buf;
        const int rows = s.rows_of(b), r0 = (int)(((uint64_t)u << shift) >> s.col_bits), r1 = (int)((((uint64_t)(u + g.y) << shift) - 1) >> s.col_bits);
        for (int r = r0 + tid; r <= r1 && r < rows; r += BIG_THREADS) { // the rows the group's values can lie in
            const int32_t d = first_at_or_above(sorted, m, (uint64_t)(r + 1) << s.col_bits) - first_at_or_above(sorted, m, (uint64_t)r << s.col_bits);
            if (d > 0) atomicAdd(&o.deg[row0 + r], d);
        }
        for (int q = tid; q < g.y; q += BIG_THREADS) s.sub_kept[g.x + q] = q == 0 ? m : 0;
        list_pieces(s, -1 - (int64_t)g.x, m, 0, tid);
    }
}

// where the groups of a huge bucket begin among its distinct keys, and its rows' roots
__global__ __launch_bounds__(PT) void finish_huge_kernel(const Buckets s, const RowOut o)
{
    constexpr int R = SUBS / PT;
    __shared__ int32_t sums[PT / 64];
    const int n_huge = *s.n_huge, tid = threadIdx.x;
    for (int h = blockIdx.x; h < n_huge; h += gridDim.x) {
        int32_t c[R], sum = 0, total;
#pragma unroll
        for (int q = 0; q < R; ++q) {
            c[q] = s.sub_kept[h * SUBS + tid * R + q];
            sum += c[q];
        }
        int32_t from = scan_threads<PT>(sum, sums, tid, total);
#pragma unroll
        for (int q = 0; q < R; ++q) {
            s.sub_count[h * SUBS + tid * R + q] = from;
            from += c[q];
        }
        const int64_t b = s.huge[h], row0 = b << s.row_shift;
        for (int r = tid; r < s.rows_of(b); r += PT) put_row(o, row0 + r, o.deg[row0 + r]);
        __syncthreads();
    }
}

// ---- sorted buckets -> column indices and values -----------------------------------------
struct EmitArgs {
    const int32_t *rowptr;
    int32_t *colidx;
    float *vals;
    const float *dinv;
};
// entries [from, from + EMIT_PIECE) of a bucket or part whose distinct keys are keys[first, first + kept) and the entries from `base` on
template <class K>
__device__ inline void emit_piece(const Buckets &s, const EmitArgs &a, const K *__restrict__ keys, int64_t row0, int64_t first, int64_t base, int32_t kept, int32_t from)
{
    constexpr int U = EMIT_PIECE / 256; // entries of a thread, all in flight
    const int32_t left = kept - from, count = left < EMIT_PIECE ? left : EMIT_PIECE;
    if (count <= 0) return;
    const K col_mask = ((K)1 << s.col_bits) - 1, *mine = keys + first + from;
    K k[U];
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = u * 256 + (int)threadIdx.x;
        k[u] = __builtin_nontemporal_load(mine + (i < count ? i : count - 1));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) { // (at workgroup scope: past L1)
        const float other = __hip_atomic_load(a.dinv + (int32_t)(k[u] & col_mask), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        v[u] = a.dinv[row0 + (int64_t)(k[u] >> s.col_bits)] * other;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = u * 256 + (int)threadIdx.x;
        if (i < count) {
            __builtin_nontemporal_store((int32_t)(k[u] & col_mask), a.colidx + base + from + i);
            __builtin_nontemporal_store(v[u], a.vals + base + from + i);
        }
    }
}
// Workgroup b writes the first EMIT_PIECE entries of bucket b, the workgroups behind those the listed pieces in turn.  What bounds it is the
// gather of dinv[col], 123 G/s at 2.4 M nodes: what streams past is kept out of the way of the gathered lines (1.09 -> 1.06 ms for 126 M
// entries), and the gathers themselves out of L1 (1.02; as non-temporal loads 2.03).  A 16-bit table of degrees in dinv's place, with the
// roots in LDS, fits the L2s but was slower (1.2 to 1.3 ms).
template <class K>
__global__ __launch_bounds__(256) void emit_kernel(const Buckets s, const EmitArgs a, const K *__restrict__ keys)
{
    if (blockIdx.x < s.n_buckets) { // uniform per workgroup
        const int64_t b = blockIdx.x, row0 = b << s.row_shift;
        emit_piece(s, a, keys, row0, s.start[b], a.rowptr[row0], s.kept[b], 0);
        return;
    }
    const int n_pieces = *s.n_pieces;
    for (int64_t at = blockIdx.x - s.n_buckets; at < n_pieces; at += gridDim.x - s.n_buckets) {
        const int2 p = s.pieces[at];
        if (p.x >= 0) {
            const int64_t row0 = (int64_t)p.x << s.row_shift;
            emit_piece(s, a, keys, row0, s.start[p.x], a.rowptr[row0], s.kept[p.x], p.y * EMIT_PIECE);
        } else { // a group of parts of a huge bucket
            const int part = -1 - p.x, h = part / SUBS;
            const int64_t row0 = (int64_t)s.huge[h] << s.row_shift;
            emit_piece(s, a, keys, row0, s.sub_start[h * (SUBS + 1) + part % SUBS], a.rowptr[row0] + (int64_t)s.sub_count[part], s.sub_kept[part], p.y * EMIT_PIECE);
        }
    }
}

constexpr int N_COUNTS = 5; // n_big ... n_pieces
// Workspace: what lives until the entries are emitted, then what the distribution needs
struct Layout {
    BucketPlan p;
    size_t spare_bytes() const { return (size_t)p.max_keys * (p.bits2 ? 8 : p.key_bytes()); }
    int64_t max_big() const { return p.max_keys / SORT_KEYS + 1; }
    int64_t max_huge() const { return p.max_keys / MOST_KEYS + 1; }
    int64_t max_tiles() const { return p.max_keys / TILE_KEYS + max_huge(); }
    // two groups in a row hold more than MOST_KEYS keys, or they would be one
    int64_t max_groups() const { return 2 * (p.max_keys / MOST_KEYS) + max_huge(); }
    int64_t max_pieces() const { return p.max_keys / EMIT_PIECE + 1 + max_groups(); }
    size_t bytes(int64_t n) const
    {
        const auto r = [](int64_t words) { return Arena::rounded((size_t)words * 4); };
        size_t scan = scan_bytes(p.counts1());
        if (p.bits2 && scan_bytes(p.counts2()) > scan) scan = scan_bytes(p.counts2());
        if (scan_bytes(n + 1) > scan) scan = scan_bytes(n + 1);
        return Arena::rounded((size_t)p.max_keys * p.key_bytes()) + Arena::rounded(spare_bytes()) + r(p.n_buckets + 1) + r(p.n_buckets) + r(max_big()) +
               r(max_huge()) + r(2 * max_tiles()) + 2 * r(max_huge() * SUBS) + r(max_huge() * (SUBS + 1)) + r(2 * max_groups()) +
               r(2 * max_pieces()) + r(N_COUNTS) + 2 * r(p.counts1()) +
               2 * r(p.counts2()) + r(MAX_DIGITS + 1) + scan;
    }
};

template <class K>
int sort_rows(const Layout &l, const int64_t *row, const int64_t *col, int64_t n_edges, int64_t n, bool sym, const RowOut &rows, int32_t *rowptr,
              int32_t *n_bad, Arena &ws, EdgeSort *out, hipStream_t stream)
{
    const BucketPlan &p = l.p;
    K *keys = nullptr, *spare = nullptr;
    int32_t *start = nullptr;
    Buckets b{};
    if (int rc = ws.take((size_t)p.max_keys * sizeof(K), &keys)) return rc;
    if (int rc = ws.take(l.spare_bytes(), &spare)) return rc;
    if (int rc = ws.take((size_t)(p.n_buckets + 1) * 4, &start)) return rc;
    if (int rc = ws.take((size_t)p.n_buckets * 4, &b.kept)) return rc;
    if (int rc = ws.take((size_t)l.max_big() * 4, &b.big)) return rc;
    if (int rc = ws.take((size_t)l.max_huge() * 4, &b.huge)) return rc;
    if (int rc = ws.take((size_t)l.max_tiles() * sizeof(int2), &b.tiles)) return rc;
    if (int rc = ws.take((size_t)l.max_huge() * SUBS * 4, &b.sub_count)) return rc;
    if (int rc = ws.take((size_t)l.max_huge() * SUBS * 4, &b.sub_kept)) return rc;
    if (int rc = ws.take((size_t)l.max_huge() * (SUBS + 1) * 4, &b.sub_start)) return rc;
    if (int rc = ws.take((size_t)l.max_groups() * sizeof(int2), &b.groups)) return rc;
    if (int rc = ws.take((size_t)l.max_pieces() * sizeof(int2), &b.pieces)) return rc;
    if (int rc = ws.take(N_COUNTS * 4, &b.n_big)) return rc;
    b.n_huge = b.n_big + 1;
    b.n_tiles = b.n_big + 2;
    b.n_groups = b.n_big + 3;
    b.n_pieces = b.n_big + 4;
    b.start = start;
    b.n = n;
    b.n_buckets = p.n_buckets;
    b.col_bits = p.col_bits;
    b.row_shift = p.row_shift;
    const size_t mark = ws.used;
    SG_HIP(hipMemsetAsync(b.n_big, 0, N_COUNTS * 4, stream));
    if (p.n_items > 0) {
        int32_t *counts = nullptr, *at1 = nullptr;
        if (int rc = ws.take((size_t)p.counts1() * 4, &counts)) return rc;
        if (int rc = ws.take((size_t)p.counts1() * 4, &at1)) return rc;
        const EdgeList e{row, col, n_edges, n, p.n_items, sym ? 1 : 0, p.col_bits, p.row_shift + p.bits2};
        const int digits1 = (int)p.digits1();
        count_edges_kernel<<<(unsigned)p.tiles1, PT, 0, stream>>>(e, p.tiles1, digits1, counts, n_bad);
        SG_LAUNCH_CHECK();
        if (int rc = scan_i32(counts, at1, p.counts1(), ws, stream)) return rc; // the last element is only written: the total
        SecondPass s{nullptr, nullptr, at1, nullptr, p.tiles1, digits1, p.bits2, p.col_bits, p.row_shift};
        int32_t *at2 = nullptr;
        if (p.bits2 == 0) {
            distribute_edges_kernel<K, true><<<(unsigned)p.tiles1, PT, 0, stream>>>(e, p.tiles1, digits1, at1, keys, 0, nullptr);
            SG_LAUNCH_CHECK();
        } else {
            uint16_t *second = sizeof(K) == 4 ? reinterpret_cast<uint16_t *>(spare + p.max_keys) : nullptr; // spare has 8 bytes a key
            int32_t *counts2 = nullptr, *tile_start = nullptr;
            if (int rc = ws.take((size_t)p.counts2() * 4, &counts2)) return rc;
            if (int rc = ws.take((size_t)p.counts2() * 4, &at2)) return rc;
            if (int rc = ws.take((size_t)(MAX_DIGITS + 1) * 4, &tile_start)) return rc;
            s.keys = spare;
            s.second = second;
            s.tile_start = tile_start;
            distribute_edges_kernel<K, false><<<(unsigned)p.tiles1, PT, 0, stream>>>(e, p.tiles1, digits1, at1, spare, p.bits2, second);
            SG_LAUNCH_CHECK();
            tile_starts_kernel<<<1, PT, 0, stream>>>(at1, p.tiles1, digits1, tile_start);
            SG_LAUNCH_CHECK();
            count_keys_kernel<K><<<(unsigned)p.max_tiles2, PT, 0, stream>>>(s, counts2);
            SG_LAUNCH_CHECK();
            if (int rc = scan_i32(counts2, at2, p.counts2(), ws, stream)) return rc; // elements past the last tile's are not used
            distribute_keys_kernel<K><<<(unsigned)p.max_tiles2, PT, 0, stream>>>(s, at2, keys);
            SG_LAUNCH_CHECK();
        }
        bucket_starts_kernel<<<blocks_for(p.n_buckets + 1), TPB, 0, stream>>>(s, at2, p.n_buckets, start);
        SG_LAUNCH_CHECK();
    } else {
        SG_HIP(hipMemsetAsync(start, 0, (size_t)(p.n_buckets + 1) * 4, stream));
    }
    ws.used = mark; // later users are ordered behind these kernels on the stream
    sort_buckets_kernel<K><<<(unsigned)p.n_buckets, 256, 0, stream>>>(b, rows, keys);
    SG_LAUNCH_CHECK();
    const unsigned huge_blocks = (unsigned)(l.max_huge() < 512 ? l.max_huge() : 512), tile_blocks = (unsigned)(l.max_tiles() < TILE_BLOCKS ? l.max_tiles() : TILE_BLOCKS);
    if (p.max_keys > MOST_KEYS) {
        count_huge_kernel<K><<<tile_blocks, PT, 0, stream>>>(b, keys);
        SG_LAUNCH_CHECK();
        group_huge_kernel<<<huge_blocks, PT, 0, stream>>>(b);
        SG_LAUNCH_CHECK();
        deal_huge_kernel<K><<<tile_blocks, PT, 0, stream>>>(b, keys, spare);
        SG_LAUNCH_CHECK();
    }
    if (p.max_keys > SORT_KEYS) { // two workgroups per CU
        sort_big_buckets_kernel<K><<<512, BIG_THREADS, 0, stream>>>(b, rows, keys, spare);
        SG_LAUNCH_CHECK();
    }
    if (p.max_keys > MOST_KEYS) {
        finish_huge_kernel<<<huge_blocks, PT, 0, stream>>>(b, rows);
        SG_LAUNCH_CHECK();
    }
    if (int rc = scan_i32(rows.deg, rowptr, n + 1, ws, stream)) return rc; // deg[n] is read, what it holds is not used
    static_assert(sizeof(Buckets) <= sizeof(out->state), "what the emission needs travels in the caller's struct");
    memcpy(out->state, &b, sizeof(b));
    out->keys = keys;
    out->max_pieces = l.max_pieces();
    out->wide = p.wide;
    return SLICEGCN_OK;
}

template <class K>
int emit(const EdgeSort &e, const int32_t *rowptr, int32_t *colidx, float *vals, const float *dinv, hipStream_t stream)
{
    Buckets b;
    memcpy(&b, e.state, sizeof(b));
    const EmitArgs a{rowptr, colidx, vals, dinv};
    emit_kernel<K><<<(unsigned)(b.n_buckets + (e.max_pieces < 16384 ? e.max_pieces : 16384)), 256, 0, stream>>>(b, a, static_cast<const K *>(e.keys));
    SG_LAUNCH_CHECK();
    return SLICEGCN_OK;
}

} // namespace

size_t edge_sort_bytes(int64_t n_edges, int64_t n, bool sym, bool loops) { return Layout{bucket_plan(n_edges, n, sym, loops)}.bytes(n); }

int edge_sort_rows(const int64_t *row, const int64_t *col, int64_t n_edges, int64_t n, bool sym, bool loops, int32_t *deg, float *dinv, float *sqrtd,
                   int32_t *rowptr, int32_t *n_bad, Arena &ws, EdgeSort *out, hipStream_t stream)
{
    const Layout l{bucket_plan(n_edges, n, sym, loops)};
    SG_REQUIRE(l.p.tiles1 <= INT32_MAX && l.p.max_tiles2 <= INT32_MAX, SLICEGCN_ERANGE, "build_norm_csr: too many edges for one launch");
    const RowOut rows{deg, dinv, sqrtd};
    return l.p.wide ? sort_rows<uint64_t>(l, row, col, n_edges, n, sym, rows, rowptr, n_bad, ws, out, stream)
                    : sort_rows<uint32_t>(l, row, col, n_edges, n, sym, rows, rowptr, n_bad, ws, out, stream);
}

int edge_sort_emit(const EdgeSort &e, const int32_t *rowptr, int32_t *colidx, float *vals, const float *dinv, hipStream_t stream)
{
    return e.wide ? emit<uint64_t>(e, rowptr, colidx, vals, dinv, stream) : emit<uint32_t>(e, rowptr, colidx, vals, dinv, stream);
}

} // namespace slicegcn
