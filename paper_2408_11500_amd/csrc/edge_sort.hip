// Edge pairs -> distinct entries of the adjacency pattern, by row and ascending column, and each row's number of entries.
//
//   count, distribute   the keys (row, col) are distributed to buckets of consecutive rows, straight from the edge list: one pass over the
//                       keys for up to 512 buckets, two above; each reads them twice, to count and to move.  Runs of a digit are
//                       written in one piece per tile; the order within a bucket is whatever the LDS atomics give;
//   sort                a workgroup sorts a bucket in registers, drops repeats and counts its rows (degrees and their roots included),
//                       so that no later pass looks for row starts; larger buckets are cut first;
//   emit                column indices and values, once the row pointers are there (a scan of the degrees).
// Keys within a bucket are the low bits of the row and the column, 32 bits up to 2^25 nodes (see BucketPlan).  Then the first pass writes 6 bytes per key (the
// second digit apart), the second counts from 2 of them, reads 6 and writes 4, and sorting and emission move 4.  The result is a function
// of the set of pairs alone: integer counters decide only where a key waits to be sorted.
//
// 62 M edges, 2.4 M nodes (126 M keys): 3.6 ms with the schedule, where a device radix sort of 44-bit keys (six passes over 8-byte
// keys), a sweep for repeats and one for the values took 6.6.  Of it: counting and distributing 0.23 + 0.57 and 0.09 + 0.35 (4 TB/s in the
// first pass), sorting 0.65 + 0.30 and 0.07 for the cuts (vector unit and LDS crossbar: about 90 comparisons per key), columns and values
// 1.03 (gather of dinv[col]).
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
//     distributing: 1024 per bucket 2.44 ms, 2048 2.33, 4096 2.36), half as many with 64-bit keys, whose comparisons cost more (44 M keys
//     of 40 M nodes, build: 2.97 ms with 2048, 2.87 with 1024);
//   * no more than 2^MAX_ROW_SHIFT rows in a bucket as far as the bits go (a workgroup counts the rows of its bucket);
//   * 32-bit keys where that takes no more than MAX_BITS bits of bucket number (up to 2^25 nodes), 64-bit keys above, and where it takes all of
//     those bits (from 2^24 nodes on) for buckets of fewer than SPARSE_KEYS keys: a workgroup for every few keys costs more than wider ones
//     (30 M nodes, 32 / 64 bits: 8 keys a bucket 1.73 / 0.92 ms, 118 2.34 / 2.01, 145 4.89 / 4.71 for both directions, 152 2.78 / 2.87, 175 2.59 / 2.64);
//   * up to 2^DIGIT_BITS buckets one pass over the edges distributes them, above it two passes by half of the bits each.
constexpr int DIGIT_BITS = 9, MAX_DIGITS = 1 << DIGIT_BITS, MAX_BITS = 2 * DIGIT_BITS;
constexpr int64_t BUCKET_KEYS = 2048, BUCKET_KEYS_64 = 1024;
constexpr int64_t SPARSE_KEYS = 150;
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
    p.wide = 2 * p.col_bits - MAX_BITS > 32 || (2 * p.col_bits - MAX_BITS == 32 && (p.max_keys >> MAX_BITS) < SPARSE_KEYS);
    while (bits < MAX_BITS && bits < p.col_bits && (p.max_keys >> bits) > (p.wide ? BUCKET_KEYS_64 : BUCKET_KEYS)) ++bits;
    if (bits < p.col_bits - MAX_ROW_SHIFT) bits = p.col_bits - MAX_ROW_SHIFT < MAX_BITS ? p.col_bits - MAX_ROW_SHIFT : MAX_BITS;
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

constexpr int MAX_LEVELS = 3;                // see Cut
constexpr int N_COUNTS = 4 + 2 * MAX_LEVELS; // Buckets' n_big ... n_tiles, which the first kernel of a sort clears

// counts[digit * tiles + tile]: keys of every digit in a tile of the edge list
__global__ __launch_bounds__(PT) void count_edges_kernel(const EdgeList e, int64_t n_tiles, int n_digits, int32_t *__restrict__ counts, int32_t *__restrict__ n_bad,
                                                         int32_t *__restrict__ cleared)
{
    __shared__ int32_t cnt[MAX_DIGITS];
    if (blockIdx.x == 0 && threadIdx.x < N_COUNTS) cleared[threadIdx.x] = 0;
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
// BUCKET: the digit is the bucket, the key has the row within it and the column.  at = NULL: there is one tile, which knows where its digits
// start and counts the pairs out of range itself; the buckets' starts go to `start` (no counting, no scan: 300 edges of 100 nodes, build
// 142 -> 109 us).
// Otherwise there is a second pass.  32-bit keys: row bits within the bucket as well, and the second digit goes to an array of its own
// (6 bytes a key instead of 8, of which the counting reads 2: 126 M keys distributed 0.59 -> 0.57 ms, counted 0.25 -> 0.09, distributed again
// 0.38 -> 0.35); 64-bit keys: the whole row.
template <class K, bool BUCKET>
__global__ __launch_bounds__(PT) void distribute_edges_kernel(const EdgeList e, int64_t n_tiles, int n_digits, const int32_t *__restrict__ at, K *__restrict__ out,
                                                              int bits2, uint16_t *__restrict__ second, int32_t *__restrict__ start, int32_t *__restrict__ n_bad,
                                                              int32_t *__restrict__ cleared)
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
    if (BUCKET && !at) { // uniform
        if (bad) atomicAdd(n_bad, bad);
        cnt[threadIdx.x] = 0;
        if ((int)threadIdx.x < n_digits) start[threadIdx.x] = off[threadIdx.x];
        if (threadIdx.x == 0) start[n_digits] = total;
        if (threadIdx.x < N_COUNTS) cleared[threadIdx.x] = 0;
    } else if ((int)threadIdx.x < n_digits) {
        cnt[threadIdx.x] = at[(int64_t)threadIdx.x * n_tiles + blockIdx.x] - off[threadIdx.x]; // the ranks are in registers
    }
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

// 64-bit keys: one comparison and one choice (as above it would be three of each: 44 M keys of 40 M nodes sorted 2.4 ms instead of 1.6)
__device__ inline uint64_t pick_side(uint64_t a, uint64_t b, uint64_t bound) { return (b < a) != (bound != 0) ? b : a; }

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

// Buckets a hub, a few of them or repeats make so large that one workgroup would be the whole build's last are cut by the next SUB_BITS bits of
// their keys, which many workgroups count and deal in tiles as in the passes before; parts of more than MOST_KEYS keys are cut again, up to
// MAX_LEVELS times in all (as many as leave at most SUB_BITS bits), and runs of parts that fit a workgroup's registers are sorted each on
// its own.  What is left of more than MOST_KEYS keys with at most SUB_BITS bits between them (all keys of up to 2^SUB_BITS nodes, in buckets of one
// row) holds repeats: its tiles are marked in a bitmap.
// Builds with one workgroup per part and a bitmap of its values, gone over once per 2^19 of them / cut again (a radix sort of all keys): star
// of a million leaves 0.72 / 0.43 ms (0.48); one pair 20 M times, 1000 nodes 5.5 / 0.87 (0.89), 3 M nodes 5.6 / 1.5 (2.0); a row of
// 100 000 among 2 M edges of 40 M nodes 6.3 / 3.0 (3.0); 40 000 pairs 1250 times each, 200 nodes 1.84 / 0.87 (1.69), 3 M nodes 2.4 / 3.1 (4.5).
constexpr int SUB_BITS = 11, SUBS = 1 << SUB_BITS;
struct Cut {
    int32_t bucket, parent; // parent: the part (its cut * SUBS + its number) that is cut here, -1: the whole bucket
    int32_t beg, end;       // the keys
    int32_t tiles;          // tiles not counted yet; whoever counts the last one groups the parts
    int32_t open;           // groups, parts of repeats and cuts of parts not finished yet
};
struct Buckets {
    const int32_t *start; // [n_buckets + 1]
    int32_t *kept;        // distinct keys of every bucket, from its start on
    int32_t *big;         // buckets of more than SORT_KEYS keys, in no particular order
    Cut *cuts;            // max_cuts per level
    int2 *tiles;          // max_tiles per level: (cut, tile) of all tiles of TILE_KEYS keys
    int32_t *sub_count;   // [cut * SUBS + u] keys of part u; at the end the distinct keys of the parts before it
    int32_t *sub_kept;    // [cut * SUBS + u] how many keys of the part have been dealt out; then its distinct keys, those of a group at its first part
    int32_t *sub_start;   // [cut * (SUBS + 1) + u] the part's first key
    int4 *groups;         // (cut * SUBS + first part, parts, -1, level) of every group of parts, which are sorted together, and
                          // (cut * SUBS + part, r, tile, level) of every tile of MOST_KEYS keys of the r-th part of repeats; level -1: a
                          // bucket of repeats that has never been cut
    int32_t *repeats;     // [r * REPEAT_WORDS] the bitmap of the r-th part of repeats, its last word the number of tiles not marked yet
    int2 *pieces;         // (bucket, piece) of every piece but the first of the buckets with more than EMIT_PIECE distinct keys, and of all
                          // pieces of groups (-1 - cut * SUBS - first part in the bucket's place), in no order
    int32_t *n_big, *n_groups, *n_pieces, *n_repeats, *n_cuts, *n_tiles; // n_cuts, n_tiles: per level
    int64_t n, n_buckets;
    int32_t max_cuts, max_tiles;
    int col_bits, row_shift, levels;
    __host__ __device__ int shift(int level) const // of the part number in a key
    {
        const int s = row_shift + col_bits - SUB_BITS * (level + 1);
        return s > 0 ? s : 0;
    }
    __device__ int rows_of(int64_t b) const
    {
        const int64_t left = n - (b << row_shift);
        return left < ((int64_t)1 << row_shift) ? (int)left : 1 << row_shift;
    }
};
inline int cut_levels(int key_bits)
{
    const int levels = (key_bits + SUB_BITS - 1) / SUB_BITS - 1;
    return levels < 1 ? 1 : levels;
}
template <class K> __device__ inline int part_of(K key, int shift) { return (int)(key >> shift) & (SUBS - 1); }

// another cut of keys [beg, end), in so many tiles; returns its number.  Uniform per workgroup
__device__ inline int32_t new_cut(const Buckets &s, int level, int32_t bucket, int32_t parent, int32_t beg, int32_t end, int32_t tiles, int tid)
{
    __shared__ int32_t place, first_tile;
    __syncthreads(); // of the cut before
    if (tid == 0) {
        place = level * s.max_cuts + atomicAdd(s.n_cuts + level, 1);
        first_tile = level * s.max_tiles + atomicAdd(s.n_tiles + level, tiles);
        s.cuts[place] = Cut{bucket, parent, beg, end, tiles, 0};
    }
    __syncthreads();
    for (int32_t t = tid; t < tiles; t += blockDim.x) s.tiles[first_tile + t] = make_int2(place, t);
    for (int u = tid; u < SUBS; u += blockDim.x) s.sub_count[place * SUBS + u] = s.sub_kept[place * SUBS + u] = 0;
    return place;
}
constexpr int BITMAP_WORDS = SUBS / 32, REPEAT_WORDS = BITMAP_WORDS + 1;
// another part of repeats; uniform per workgroup
__device__ inline void new_repeats(const Buckets &s, int level, int32_t part, int32_t count, int tid)
{
    __shared__ int32_t first, number;
    const int32_t tiles = pieces_of(count, MOST_KEYS);
    __syncthreads(); // of the part before
    if (tid == 0) {
        first = atomicAdd(s.n_groups, tiles);
        number = atomicAdd(s.n_repeats, 1);
    }
    __syncthreads();
    for (int32_t t = tid; t < tiles; t += blockDim.x) s.groups[first + t] = make_int4(part, number, t, level);
    for (int w = tid; w < REPEAT_WORDS; w += blockDim.x) s.repeats[number * REPEAT_WORDS + w] = w < BITMAP_WORDS ? 0 : tiles;
}

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
    const int lane = tid & 63; // two searches per row: 44 M keys of 40 M nodes sorted 1.47 ms instead of 1.33
    for (int r0 = (tid >> 6) * 63; r0 < rows; r0 += THREADS / 64 * 63) { // the next lane's row starts where this one's ends
        const int r = r0 + lane;
        const int32_t beg = first_at_or_above(sorted, count, (uint64_t)r << s.col_bits), end = __shfl_down(beg, 1, 64);
        if (lane < 63 && r < rows) put_row(o, row0 + r, end - beg);
    }
}

// One workgroup per bucket: sorts its keys in registers, drops repeats, writes them back and counts its rows.  Larger buckets are listed.
template <class K>
__global__ __launch_bounds__(256) void sort_buckets_kernel(const Buckets s, const RowOut o, K *__restrict__ keys)
{
    __shared__ K buf[SORT_KEYS];
    __shared__ K last[256];
    __shared__ int32_t sums[4];
    const int tid = threadIdx.x;
    const int64_t b = blockIdx.x, row0 = b << s.row_shift;
    const int32_t beg = s.start[b], cnt = s.start[b + 1] - beg;
    if (cnt > MOST_KEYS) { // uniform per workgroup
        const bool repeats = s.shift(-1) <= SUB_BITS;
        const int32_t h = new_cut(s, 0, (int32_t)b, -1, beg, beg + cnt, repeats ? 0 : pieces_of(cnt, TILE_KEYS), tid);
        if (repeats) { // its first part is the whole bucket
            if (tid < 2) s.sub_start[h * (SUBS + 1) + tid] = beg + tid * cnt;
            if (tid == 0) s.cuts[h].open = 1;
            new_repeats(s, -1, h * SUBS, cnt, tid);
        }
        if (tid == 0) s.kept[b] = 0;
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

// How many keys of this lane's part the workgroup has met before: a counter in LDS, one addition for a wavefront whose keys are all of
// one part, as those of repeats and hubs are (64 additions to one word otherwise).  -1 without a key.
__device__ inline int32_t count_part(int32_t *cnt, int part, bool in)
{
    const unsigned long long lanes = __ballot(in);
    if (lanes == 0) return -1;
    const int leader = __ffsll(lanes) - 1, lane = threadIdx.x & 63, lead = __shfl(part, leader, 64);
    if (__ballot(in && part != lead) != 0) return in ? atomicAdd(&cnt[part], 1) : -1;
    int32_t base = 0;
    if (lane == leader) base = atomicAdd(&cnt[lead], __popcll(lanes));
    base = __shfl(base, leader, 64);
    return in ? base + __popcll(lanes & ((1ull << lane) - 1ull)) : -1;
}
__device__ inline int32_t load_shared(const int32_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); } // written in this launch
// Counts `done` down for the whole workgroup, behind everything it has written; true where nothing is left, and then all that the others
// wrote before is there to be read, by load_shared.  Uniform per workgroup.
// STORES: some of it was written by plain stores, and making those known to the other XCDs takes a write-back of the L2 (100 M keys of
// 40 000 values, one per tile and group: sorting 2.0 ms instead of 0.6); workgroups take runs of groups and count once per run and cut.
// Otherwise all of it are additions at device scope, which are performed in one place for all XCDs, and none is outstanding behind the wait
// (126 M keys of an R-MAT graph, cut buckets counted: 58 us with the write-back, 26 without, grouping included).
template <bool STORES> __device__ inline bool last_of(int32_t *left, int32_t done, int tid)
{
    __shared__ int last;
    __builtin_amdgcn_s_waitcnt(0); // no access of this wavefront is outstanding
    __syncthreads();
    if (tid == 0) {
        last = __hip_atomic_fetch_sub(left, done, STORES ? __ATOMIC_RELEASE : __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == done;
        if (last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    const bool yes = last;
    __syncthreads();
    return yes;
}
// the run of `count` items in order that this workgroup takes
struct Run { int beg, end; };
__device__ inline Run run_of(int count)
{
    const int per = (count + (int)gridDim.x - 1) / (int)gridDim.x, beg = min(per * (int)blockIdx.x, count);
    return Run{beg, min(beg + per, count)};
}

// Where the parts of a cut start, and its groups: runs of parts of together at most MOST_KEYS keys.  Parts of more are cut again or, at the last
// level, listed as repeats.  next: SUBS words
__device__ inline void group_parts(const Buckets &s, int h, int level, int32_t *next, int tid)
{
    constexpr int R = SUBS / PT;
    __shared__ int32_t end[SUBS], sums[PT / 64], n_sorted, n_large, first;
    __shared__ int2 list[SUBS]; // groups from the front, larger parts from the back
    const Cut &cut = s.cuts[h];
    const int32_t start = cut.beg;
    int32_t c[R], sum = 0, total;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        c[q] = load_shared(&s.sub_count[h * SUBS + tid * R + q]);
        sum += c[q];
    }
    int32_t from = scan_threads<PT>(sum, sums, tid, total);
#pragma unroll
    for (int q = 0; q < R; ++q) {
        s.sub_start[h * (SUBS + 1) + tid * R + q] = start + from;
        from += c[q];
        end[tid * R + q] = from;
    }
    if (tid == 0) s.sub_start[h * (SUBS + 1) + SUBS] = start + total;
    __syncthreads();
    for (int u = tid; u < SUBS; u += PT) {
        const int32_t before = u > 0 ? end[u - 1] : 0;
        int lo = u + 1, hi = SUBS; // most parts [u, lo) that fit, one at least
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (end[mid - 1] - before <= MOST_KEYS) lo = mid; else hi = mid - 1;
        }
        next[u] = lo;
    }
    __syncthreads();
    if (tid == 0) {
        int n = 0, large = 0;
        for (int u = 0, v; u < SUBS; u = v) {
            v = next[u];
            const int32_t count = end[v - 1] - (u > 0 ? end[u - 1] : 0);
            if (count > MOST_KEYS) list[SUBS - ++large] = make_int2(u, count);
            else if (count > 0) list[n++] = make_int2(u, v - u);
        }
        n_sorted = n;
        n_large = large;
        s.cuts[h].open = n + large;
        first = atomicAdd(s.n_groups, n);
    }
    __syncthreads();
    for (int i = tid; i < n_sorted; i += PT) s.groups[first + i] = make_int4(h * SUBS + list[i].x, list[i].y, -1, level);
    for (int i = 1; i <= n_large; ++i) {
        const int u = list[SUBS - i].x, part = h * SUBS + u;
        const int32_t count = list[SUBS - i].y, beg = start + end[u] - count;
        if (level + 1 < s.levels) new_cut(s, level + 1, cut.bucket, part, beg, beg + count, pieces_of(count, TILE_KEYS), tid);
        else new_repeats(s, level, part, count, tid);
    }
}

struct CutTile { int h; int64_t beg, end; };
__device__ inline CutTile cut_tile(const Buckets &s, int level, int at)
{
    const int2 t = s.tiles[level * s.max_tiles + at];
    const int64_t beg = s.cuts[t.x].beg + (int64_t)t.y * TILE_KEYS, end = s.cuts[t.x].end;
    return CutTile{t.x, beg, beg + TILE_KEYS < end ? beg + TILE_KEYS : end};
}
constexpr int TILE_BLOCKS = 1024; // workgroups that take the tiles in turn
template <class K> __global__ __launch_bounds__(PT) void count_cuts_kernel(const Buckets s, int level, const K *__restrict__ in)
{
    __shared__ int32_t cnt[SUBS];
    const int shift = s.shift(level), tid = threadIdx.x;
    const Run run = run_of(s.n_tiles[level]);
    int counted = 0; // tiles of the present cut in cnt
    for (int at = run.beg; at < run.end; ++at) {
        const CutTile t = cut_tile(s, level, at);
        if (counted == 0) {
            for (int u = tid; u < SUBS; u += PT) cnt[u] = 0;
            __syncthreads();
        }
        K k[TILE_KEYS / PT];
#pragma unroll
        for (int j = 0; j < TILE_KEYS / PT; ++j) k[j] = in[t.beg + j * PT + tid < t.end ? t.beg + j * PT + tid : t.beg];
#pragma unroll
        for (int j = 0; j < TILE_KEYS / PT; ++j) count_part(cnt, part_of(k[j], shift), t.beg + j * PT + tid < t.end);
        ++counted;
        if (at + 1 < run.end && s.tiles[level * s.max_tiles + at + 1].x == t.h) continue; // uniform
        __syncthreads();
        for (int u = tid; u < SUBS; u += PT)
            if (cnt[u] > 0) atomicAdd(&s.sub_count[t.h * SUBS + u], cnt[u]);
        if (last_of<false>(&s.cuts[t.h].tiles, counted, tid)) group_parts(s, t.h, level, cnt, tid);
        __syncthreads();
        counted = 0;
    }
}
template <class K> __global__ __launch_bounds__(PT) void deal_cuts_kernel(const Buckets s, int level, const K *__restrict__ in, K *__restrict__ out)
{
    __shared__ int32_t cnt[SUBS];
    const int shift = s.shift(level), tid = threadIdx.x, n_tiles = s.n_tiles[level];
    for (int at = blockIdx.x; at < n_tiles; at += gridDim.x) {
        const CutTile t = cut_tile(s, level, at);
        for (int u = tid; u < SUBS; u += PT) cnt[u] = 0;
        __syncthreads();
        K k[TILE_KEYS / PT];
        int32_t rank[TILE_KEYS / PT];
#pragma unroll
        for (int j = 0; j < TILE_KEYS / PT; ++j) k[j] = in[t.beg + j * PT + tid < t.end ? t.beg + j * PT + tid : t.beg];
#pragma unroll
        for (int j = 0; j < TILE_KEYS / PT; ++j) rank[j] = count_part(cnt, part_of(k[j], shift), t.beg + j * PT + tid < t.end);
        __syncthreads();
        for (int u = tid; u < SUBS; u += PT)
            if (cnt[u] > 0) cnt[u] = s.sub_start[t.h * (SUBS + 1) + u] + atomicAdd(&s.sub_kept[t.h * SUBS + u], cnt[u]);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < TILE_KEYS / PT; ++j)
            if (rank[j] >= 0) out[(int64_t)cnt[part_of(k[j], shift)] + rank[j]] = k[j];
        __syncthreads();
    }
}

// The larger buckets, the groups of the cut ones and their parts of repeats.  Whoever finishes a cut's last group adds up the distinct keys
// before each of its parts, and so on up to the bucket, whose rows' roots it writes.
constexpr int BIG_THREADS = 512;
template <class K>
__global__ __launch_bounds__(BIG_THREADS) void sort_big_buckets_kernel(const Buckets s, const RowOut o, K *keys, K *spare)
{
    constexpr int R = SUBS / BIG_THREADS, U = 16;
    __shared__ __attribute__((aligned(16))) K buf[MOST_KEYS];
    __shared__ K last[BIG_THREADS];
    __shared__ int32_t sums[BIG_THREADS / 64], bits[BITMAP_WORDS];
    const int tid = threadIdx.x;
    const int n_groups = *s.n_groups;
    const Run run = run_of(n_groups + *s.n_big);
    const int groups_end = min(run.end, n_groups);
    int marked = 0, finished = 0; // tiles of the present part of repeats in bits; groups and parts of the present cut that are done
    for (int at = run.beg; at < groups_end; ++at) {
        const int4 g = s.groups[at];
        const int level = g.w, u = g.x % SUBS, parts = g.z < 0 ? g.y : 1;
        const int next = at + 1 < groups_end ? s.groups[at + 1].x : -1; // the part of the next item
        int h = g.x / SUBS;
        const int64_t b = s.cuts[h].bucket, row0 = b << s.row_shift;
        const int32_t beg = s.sub_start[h * (SUBS + 1) + u], cnt = s.sub_start[h * (SUBS + 1) + u + parts] - beg;
        const K *from = (level & 1 ? keys : spare) + beg; // where the level's parts were dealt to
        int32_t m = 0;
        if (g.z >= 0) { // a tile of repeats
            const K low = ((K)1 << s.shift(level)) - 1, high = from[0] & ~low;
            const int32_t left = cnt - g.z * MOST_KEYS, count = left < MOST_KEYS ? left : MOST_KEYS;
            const K *tile = from + g.z * (int64_t)MOST_KEYS;
            int32_t *words = s.repeats + g.y * REPEAT_WORDS;
            if (marked == 0) {
                if (tid < BITMAP_WORDS) bits[tid] = 0;
                __syncthreads();
            }
            for (int32_t i0 = tid; i0 < count; i0 += BIG_THREADS * U) {
                K k[U];
#pragma unroll
                for (int q = 0; q < U; ++q) k[q] = tile[i0 + q * BIG_THREADS < count ? i0 + q * BIG_THREADS : i0]; // once more does no harm
#pragma unroll
                for (int q = 0; q < U; ++q) {
                    const int x = (int)(k[q] & low);
                    if (!((uint32_t)bits[x >> 5] >> (x & 31) & 1u)) atomicOr(&bits[x >> 5], (int)(1u << (x & 31)));
                }
            }
            ++marked;
            if (next == g.x) continue; // uniform: the next tile of this part
            __syncthreads();
            if (tid < BITMAP_WORDS && (bits[tid] & ~load_shared(words + tid)) != 0) atomicOr(words + tid, bits[tid]);
            if (last_of<false>(words + BITMAP_WORDS, marked, tid)) { // uniform; the others have nothing to finish
                if (tid < BITMAP_WORDS) bits[tid] = load_shared(words + tid);
                __syncthreads();
                const int x0 = tid * R, four = bits[x0 >> 5] >> (x0 & 31) & 15;
                static_assert(R == 4, "four values of a part per thread");
                int32_t to = scan_threads<BIG_THREADS>(__popc(four), sums, tid, m);
#pragma unroll
                for (int q = 0; q < R; ++q)
                    if (four >> q & 1) buf[to++] = high + (K)(x0 + q);
                __syncthreads();
            }
            marked = 0;
        } else {
            m = sort_distinct<K, MOST_KEYS / BIG_THREADS, BIG_THREADS>(from, cnt, buf, last, sums, tid);
        }
        if (m > 0) {
            K *mine = keys + beg; // from's own keys at odd levels, which are in buf now
            for (int32_t i = tid; i < m; i += BIG_THREADS) mine[i] = buf[i];
            const int r0 = (int)(buf[0] >> s.col_bits), r1 = (int)(buf[m - 1] >> s.col_bits);
            for (int r = r0 + tid; r <= r1; r += BIG_THREADS) {
                const int32_t d = first_at_or_above(buf, m, (uint64_t)(r + 1) << s.col_bits) - first_at_or_above(buf, m, (uint64_t)r << s.col_bits);
                if (d > 0) atomicAdd(&o.deg[row0 + r], d);
            }
            for (int q = tid; q < parts; q += BIG_THREADS) s.sub_kept[g.x + q] = q == 0 ? m : 0;
            list_pieces(s, -1 - (int64_t)g.x, m, 0, tid);
            ++finished;
        }
        __syncthreads(); // buf and bits are used again
        if (finished == 0 || (next >= 0 && next / SUBS == h)) continue; // uniform
        while (last_of<true>(&s.cuts[h].open, finished, tid)) {
            int32_t c[R], sum = 0, total;
#pragma unroll
            for (int q = 0; q < R; ++q) {
                c[q] = load_shared(&s.sub_kept[h * SUBS + tid * R + q]);
                sum += c[q];
            }
            int32_t before = scan_threads<BIG_THREADS>(sum, sums, tid, total);
#pragma unroll
            for (int q = 0; q < R; ++q) {
                s.sub_count[h * SUBS + tid * R + q] = before;
                before += c[q];
            }
            const int32_t parent = s.cuts[h].parent;
            if (parent < 0) {
                for (int r = tid; r < s.rows_of(b); r += BIG_THREADS) put_row(o, row0 + r, load_shared(&o.deg[row0 + r]));
                break;
            }
            if (tid == 0) s.sub_kept[parent] = total;
            h = parent / SUBS;
            finished = 1;
        }
        finished = 0;
    }
    for (int at = max(run.beg, n_groups); at < run.end; ++at) {
        const int64_t b = s.big[at - n_groups], row0 = b << s.row_shift;
        const int32_t beg = s.start[b], cnt = s.start[b + 1] - beg;
        K *mine = keys + beg;
        const int32_t m = sort_distinct<K, MOST_KEYS / BIG_THREADS, BIG_THREADS>(mine, cnt, buf, last, sums, tid);
        for (int32_t i = tid; i < m; i += BIG_THREADS) mine[i] = buf[i];
        put_rows<K, BIG_THREADS>(s, o, row0, s.rows_of(b), buf, m, tid);
        if (tid == 0) s.kept[b] = m;
        list_pieces(s, b, m, 1, tid);
        __syncthreads(); // buf is used again
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
        } else { // a group of parts: behind the distinct keys of the parts before it, in its cut and those around it
            const int part = -1 - p.x;
            int h = part / SUBS;
            const int64_t row0 = (int64_t)s.cuts[h].bucket << s.row_shift;
            const int32_t first = s.sub_start[h * (SUBS + 1) + part % SUBS];
            int64_t base = a.rowptr[row0];
            for (int at_part = part;; h = at_part / SUBS) {
                base += s.sub_count[at_part];
                at_part = s.cuts[h].parent;
                if (at_part < 0) break;
            }
            emit_piece(s, a, keys, row0, first, base, s.sub_kept[part], p.y * EMIT_PIECE);
        }
    }
}

// Workspace: what lives until the entries are emitted, then what the distribution needs
struct Layout {
    BucketPlan p;
    // keys, and behind them first the second digits and then, when those are used up, the tables of the cuts
    size_t keys_bytes() const { return Arena::rounded((size_t)p.max_keys * p.key_bytes()); }
    size_t spare_bytes() const
    {
        const size_t second = p.bits2 && !p.wide ? (size_t)p.max_keys * 2 : 0;
        return keys_bytes() + (second > table_bytes() ? second : table_bytes());
    }
    size_t table_bytes() const
    {
        const size_t cuts = (size_t)(levels() * max_cuts());
        return 2 * Arena::rounded(cuts * SUBS * 4) + Arena::rounded(cuts * (SUBS + 1) * 4);
    }
    int levels() const { return cut_levels(p.row_shift + p.col_bits); }
    int64_t max_big() const { return p.max_keys / SORT_KEYS + 1; }
    int64_t max_cuts() const { return p.max_keys / MOST_KEYS + 1; } // of a level
    int64_t max_tiles() const { return p.max_keys / TILE_KEYS + max_cuts(); }
    // two groups of a cut in a row hold more than MOST_KEYS keys, or they would be one
    int64_t max_groups() const { return levels() * (2 * (p.max_keys / MOST_KEYS) + max_cuts()) + p.max_keys / MOST_KEYS + max_cuts(); }
    int64_t max_pieces() const { return p.max_keys / EMIT_PIECE + 1 + max_groups(); }
    size_t bytes(int64_t n) const
    {
        const auto r = [](int64_t words) { return Arena::rounded((size_t)words * 4); };
        size_t scan = scan_bytes(p.counts1());
        if (p.bits2 && scan_bytes(p.counts2()) > scan) scan = scan_bytes(p.counts2());
        if (scan_bytes(n + 1) > scan) scan = scan_bytes(n + 1);
        return keys_bytes() + Arena::rounded(spare_bytes()) + r(p.n_buckets + 1) + r(p.n_buckets) + r(max_big()) +
               Arena::rounded((size_t)(levels() * max_cuts()) * sizeof(Cut)) + r(2 * levels() * max_tiles()) + r(4 * max_groups()) + r(max_cuts() * REPEAT_WORDS) + r(2 * max_pieces()) + r(N_COUNTS) + 2 * r(p.counts1()) +
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
    const int64_t cuts = l.levels() * l.max_cuts();
    if (int rc = ws.take((size_t)cuts * sizeof(Cut), &b.cuts)) return rc;
    if (int rc = ws.take((size_t)(l.levels() * l.max_tiles()) * sizeof(int2), &b.tiles)) return rc;
    Arena tables{reinterpret_cast<char *>(spare) + l.keys_bytes(), l.table_bytes(), 0}; // used behind the distribution only
    if (int rc = tables.take((size_t)cuts * SUBS * 4, &b.sub_count)) return rc;
    if (int rc = tables.take((size_t)cuts * SUBS * 4, &b.sub_kept)) return rc;
    if (int rc = tables.take((size_t)cuts * (SUBS + 1) * 4, &b.sub_start)) return rc;
    if (int rc = ws.take((size_t)l.max_groups() * sizeof(int4), &b.groups)) return rc;
    if (int rc = ws.take((size_t)l.max_cuts() * REPEAT_WORDS * 4, &b.repeats)) return rc;
    if (int rc = ws.take((size_t)l.max_pieces() * sizeof(int2), &b.pieces)) return rc;
    if (int rc = ws.take(N_COUNTS * 4, &b.n_big)) return rc;
    b.n_groups = b.n_big + 1;
    b.n_pieces = b.n_big + 2;
    b.n_repeats = b.n_big + 3;
    b.n_cuts = b.n_big + 4;
    b.n_tiles = b.n_cuts + MAX_LEVELS;
    b.max_cuts = (int32_t)l.max_cuts();
    b.max_tiles = (int32_t)l.max_tiles();
    b.levels = l.levels();
    b.start = start;
    b.n = n;
    b.n_buckets = p.n_buckets;
    b.col_bits = p.col_bits;
    b.row_shift = p.row_shift;
    const size_t mark = ws.used;
    if (p.tiles1 == 1 && p.bits2 == 0) {
        const EdgeList e{row, col, n_edges, n, p.n_items, sym ? 1 : 0, p.col_bits, p.row_shift};
        if constexpr (sizeof(K) == 4) // 64-bit keys take two passes
            distribute_edges_kernel<K, true><<<1, PT, 0, stream>>>(e, 1, (int)p.n_buckets, nullptr, keys, 0, nullptr, start, n_bad, b.n_big);
        SG_LAUNCH_CHECK();
    } else if (p.n_items > 0) {
        int32_t *counts = nullptr, *at1 = nullptr;
        if (int rc = ws.take((size_t)p.counts1() * 4, &counts)) return rc;
        if (int rc = ws.take((size_t)p.counts1() * 4, &at1)) return rc;
        const EdgeList e{row, col, n_edges, n, p.n_items, sym ? 1 : 0, p.col_bits, p.row_shift + p.bits2};
        const int digits1 = (int)p.digits1();
        count_edges_kernel<<<(unsigned)p.tiles1, PT, 0, stream>>>(e, p.tiles1, digits1, counts, n_bad, b.n_big);
        SG_LAUNCH_CHECK();
        if (int rc = scan_i32(counts, at1, p.counts1(), ws, stream)) return rc; // the last element is only written: the total
        SecondPass s{nullptr, nullptr, at1, nullptr, p.tiles1, digits1, p.bits2, p.col_bits, p.row_shift};
        int32_t *at2 = nullptr;
        if (p.bits2 == 0) {
            if constexpr (sizeof(K) == 4)
                distribute_edges_kernel<K, true><<<(unsigned)p.tiles1, PT, 0, stream>>>(e, p.tiles1, digits1, at1, keys, 0, nullptr, nullptr, nullptr, nullptr);
            SG_LAUNCH_CHECK();
        } else {
            uint16_t *second = sizeof(K) == 4 ? reinterpret_cast<uint16_t *>(tables.base) : nullptr;
            int32_t *counts2 = nullptr, *tile_start = nullptr;
            if (int rc = ws.take((size_t)p.counts2() * 4, &counts2)) return rc;
            if (int rc = ws.take((size_t)p.counts2() * 4, &at2)) return rc;
            if (int rc = ws.take((size_t)(MAX_DIGITS + 1) * 4, &tile_start)) return rc;
            s.keys = spare;
            s.second = second;
            s.tile_start = tile_start;
            distribute_edges_kernel<K, false><<<(unsigned)p.tiles1, PT, 0, stream>>>(e, p.tiles1, digits1, at1, spare, p.bits2, second, nullptr, nullptr, nullptr);
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
        SG_HIP(hipMemsetAsync(b.n_big, 0, N_COUNTS * 4, stream));
        SG_HIP(hipMemsetAsync(start, 0, (size_t)(p.n_buckets + 1) * 4, stream));
    }
    ws.used = mark; // later users are ordered behind these kernels on the stream
    sort_buckets_kernel<K><<<(unsigned)p.n_buckets, 256, 0, stream>>>(b, rows, keys);
    SG_LAUNCH_CHECK();
    if (p.max_keys > MOST_KEYS && p.row_shift + p.col_bits > SUB_BITS) {
        const unsigned tile_blocks = (unsigned)(l.max_tiles() < TILE_BLOCKS ? l.max_tiles() : TILE_BLOCKS);
        for (int level = 0; level < l.levels(); ++level) { // a level's parts lie in the other array
            count_cuts_kernel<K><<<tile_blocks, PT, 0, stream>>>(b, level, level & 1 ? spare : keys);
            SG_LAUNCH_CHECK();
            deal_cuts_kernel<K><<<tile_blocks, PT, 0, stream>>>(b, level, level & 1 ? spare : keys, level & 1 ? keys : spare);
            SG_LAUNCH_CHECK();
        }
    }
    if (p.max_keys > SORT_KEYS) { // two workgroups per CU
        sort_big_buckets_kernel<K><<<512, BIG_THREADS, 0, stream>>>(b, rows, keys, spare);
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
