// Slice aggregation Y = A^ X (+ Add): the neighbour sum of the SliceGCN layer equation.
//
// Work split (fixed per graph when it is built, see the schedule notes in common.h):
//   * rows of at most TINY_ROW stored entries: up to 64 of them, in row order, per wavefront (8-lane groups,
//     narrow slices).  Lane i loads the list's element and the entries of row i; the gather phase
//     then hands row (t * GROUPS + grp) to lane group grp in sub-round t through cross-lane reads,
//     so one wavefront keeps many independent row gathers in flight and the output stream stays
//     nearly contiguous (listed by their number of entries instead, so that no gather is of an absent one, 10 M nodes,
//     32 columns: 422 -> 490 us, as the stores of a list lie apart);
//   * lane-group items (whole rows of up to item_max entries, short class pieces of partitioned
//     rows): one item per lane group, its (column, value) pairs read LPR at a time by the
//     group's lanes and handed out by cross-lane reads;
//   * wavefront items (everything longer, cut at SEG_NNZ entries): the wavefront loads 64
//     (column, value) pairs per coalesced read, the 64/LPR lane groups take them in turn through
//     cross-lane reads with eight gathers in flight per lane, and the groups' sums are combined
//     with cross-lane shuffles;
//   * a row with several items stores per-item partial sums that a fix-up kernel adds in item order.
// Workgroup b serves column class b mod 8, which pins each column class of the
// gathered operand to one XCD's L2 (workgroups are placed round-robin over the XCDs), so the
// eight L2s hold disjoint sets of hot rows instead of eight copies of the same set.  If the
// placement were different the result would be the same, only slower.
// No floating-point atomics anywhere: the summation order is a function of the graph only.
//
// Lanes map to columns: with vector width V (4 floats; 1 for operands of fewer than 4 columns), lane `sub`
// of a group owns columns [V*sub, V*sub + V) of the current column pass; wider operands take several passes.
// The 16-byte loads and stores need 4-byte alignment only (the hardware runs in unaligned mode), so rows may start
// anywhere: a contiguous 25-wide matrix takes the same kernels as a padded one.  Where the last vector of a row
// would reach past the row, its lane loads the row's last four columns instead and shifts its sums into place
// before they are stored, so nothing outside the operand is read.  (One float per lane on the single-class
// schedule, which such operands took before: 93 us per call for 1.6 M entries of 25 columns; 28 us here.)
//
// The partial sums of rows with several items live in a workspace the caller passes in (its size comes
// from spmm_workspace_bytes), so a graph handle is read-only here and calls on different streams
// only have to use different workspaces.
#include "common.h"
#include "final_sum.h"

#include <mutex>
#include <type_traits>

namespace slicegcn {

namespace {

struct SpmmArgs {
    const int32_t *colidx;
    const float *vals;
    const Segment *items;
    const FixRow *fix;
    const TinyRow *tiny;  // the short rows, in schedule order
    const float *dinv;    // factored form only: X rows come pre-scaled by dinv[u], sums are scaled by dinv[row] on store
    float *scratch;
    int64_t scratch_stride; // floats of partial-sum slots per operand of the batch
    int64_t ldx, ldy, ldadd;
    uint32_t ldx_bytes;   // S32 kernels: byte stride of X rows (n * ldx * 4 < 2^32, n and ldx * 4 < 2^24)
    int32_t item_max;     // longest lane-group item of the schedule (ITEM_SHORT or ITEM_LONG)
    int32_t ipw;          // wavefront items per wavefront (1 to 4 in the one-launch kernel, otherwise 1); a workgroup takes 4 * ipw
    int32_t rounds;       // lane-group items per lane group (1 to MAX_RUN in the one-launch kernel, otherwise 1)
    int32_t deal;         // log2 of the chunks of lane-group whole rows a class takes in turn
    int32_t tiny_rounds;  // short rows per lane group (2, 4, 6 or 8)
    int32_t tiny_cnt;     // their number
    int32_t big_blocks;   // workgroups per class in the wavefront-item section
    int32_t small_blocks; // workgroups per class in the lane-group-item section
    int32_t slot_cols;    // floats per partial-sum slot
    int32_t col0;         // first column of this launch
    int32_t col_end;      // one past its last column (<= width)
    int32_t load_max;     // ragged rows (RAG kernels): last column a 16-byte load may start at; 0: rows end on a whole vector
    int32_t big_off[N_CLASSES], big_cnt[N_CLASSES];     // wavefront pieces of class c
    int32_t small_off[N_CLASSES], small_cnt[N_CLASSES]; // lane-group pieces of class c
    int32_t wbig_off, wbig_cnt;     // wavefront items of rows kept whole (dealt to the classes a workgroup's share at a time)
    int32_t wsmall_off, wsmall_cnt; // lane-group whole rows (dealt in stretches of 2^deal workgroups' shares)
};

// The operands of one launch: a batch of slices aggregated over the same graph (workgroups of grid row y work on slice y).
constexpr int MAX_BATCH = SPMM_BATCH;
struct SpmmBatch {
    const float *X[MAX_BATCH];
    float *Y[MAX_BATCH];
    const float *Add[MAX_BATCH];
};

// What a workgroup works on: one slice of the batch and one pass of columns.
struct SpmmIo {
    const float *X;
    float *Y;
    const float *Add;
    float *scratch;
    int32_t col0, col_end; // columns [col0, col_end) of the operand
};
__device__ inline SpmmIo pick_io(const SpmmArgs &a, const SpmmBatch &b)
{
    const int y = blockIdx.y;
    SpmmIo io;
    io.X = b.X[y]; io.Y = b.Y[y]; io.Add = b.Add[y];
    io.scratch = a.scratch + y * a.scratch_stride;
    io.col0 = a.col0 + (int32_t)blockIdx.z * PASS_COLS; // grid depth: passes of PASS_COLS columns in one launch
    io.col_end = io.col0 + PASS_COLS < a.col_end ? io.col0 + PASS_COLS : a.col_end;
    return io;
}

template <int V> struct Acc;
// 16-byte accesses at any 4-byte boundary
typedef float floatx4_u __attribute__((ext_vector_type(4), aligned(4)));
__device__ inline float4 load4(const float *p)
{
    const floatx4_u v = *reinterpret_cast<const floatx4_u *>(p);
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ inline void store4(float *p, const float4 &v)
{
    const floatx4_u o = {v.x, v.y, v.z, v.w};
    *reinterpret_cast<floatx4_u *>(p) = o;
}

template <> struct Acc<4> {
    float4 v;
    __device__ Acc() : v(make_float4(0.f, 0.f, 0.f, 0.f)) {}
    __device__ void fma(float a, const float4 &x) { v.x += a * x.x; v.y += a * x.y; v.z += a * x.z; v.w += a * x.w; }
    __device__ void plus(const float4 &x) { v.x += x.x; v.y += x.y; v.z += x.z; v.w += x.w; }
    __device__ void scale(float a) { v.x *= a; v.y *= a; v.z *= a; v.w *= a; }
    __device__ void add(const Acc &o) { v.x += o.v.x; v.y += o.v.y; v.z += o.v.z; v.w += o.v.w; }
    // drop the first s columns (what moves in from the end is never stored).  In two steps of fixed distance: written as one choice per
    // column the compiler made it an array indexed by s, moved that to LDS, and read the workgroup's size for its address from the
    // dispatch packet, which lies in host memory: every wavefront began with a read across the bus (100 003 nodes, 1.6 M entries,
    // 25 columns: 4 392 workgroups that return at once took 16.9 us with that read, 2.8 us without).
    __device__ void shift(int s)
    {
        const bool one = s & 1, two = s & 2;
        const float x = one ? v.y : v.x, y = one ? v.z : v.y, z = one ? v.w : v.z;
        v.x = two ? z : x;
        v.y = two ? v.w : y;
        v.z = z;
    }
    __device__ float get(int i) const { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }
};
template <> struct Acc<1> {
    float v;
    __device__ Acc() : v(0.f) {}
    __device__ void fma(float a, float x) { v += a * x; }
    __device__ void plus(float x) { v += x; }
    __device__ void scale(float a) { v *= a; }
    __device__ void add(const Acc &o) { v += o.v; }
    __device__ void shift(int) {}
    __device__ float get(int) const { return v; }
};

template <int V> struct Ld;
template <> struct Ld<4> {
    using T = float4;
    static __device__ T zero() { return make_float4(0.f, 0.f, 0.f, 0.f); }
    static __device__ T load(const float *p) { return load4(p); }
};
template <> struct Ld<1> {
    using T = float;
    static __device__ T zero() { return 0.f; }
    static __device__ T load(const float *p) { return *p; }
};

// Address of columns [col, col + V) of row c of the gathered operand.  S32: the whole operand lies
// within 4 GiB of its base and both factors fit 24 bits, so one 24-bit multiply-add gives an
// unsigned 32-bit byte offset from the (wavefront-uniform) base pointer.
template <int V, bool S32>
__device__ inline typename Ld<V>::T load_x(const SpmmArgs &a, const float *X, int c, int col)
{
    if (S32) {
        const uint32_t off = __umul24((uint32_t)c, a.ldx_bytes) + (uint32_t)col * 4u;
        return Ld<V>::load(reinterpret_cast<const float *>(reinterpret_cast<const char *>(X) + off));
    }
    return Ld<V>::load(X + (int64_t)c * a.ldx + col);
}

// Factored form (FACT): the operand rows already carry dinv[u], so every stored entry weighs 1 (the value stream is
// not read, its cross-lane reads vanish and the multiply-adds fold to adds) and the row sum is scaled by dinv[row] on store.
template <bool FACT> __device__ inline float ld_val(const SpmmArgs &a, int idx) { return FACT ? 1.f : a.vals[idx]; }
template <bool FACT> __device__ inline float shfl_val(float v, int src) { return FACT ? 1.f : __shfl(v, src, 64); }

template <int V> __device__ inline Acc<V> shfl_xor_acc(const Acc<V> &a, int mask);
template <> __device__ inline Acc<4> shfl_xor_acc<4>(const Acc<4> &a, int mask)
{
    Acc<4> r;
    r.v.x = __shfl_xor(a.v.x, mask, 64);
    r.v.y = __shfl_xor(a.v.y, mask, 64);
    r.v.z = __shfl_xor(a.v.z, mask, 64);
    r.v.w = __shfl_xor(a.v.w, mask, 64);
    return r;
}
template <> __device__ inline Acc<1> shfl_xor_acc<1>(const Acc<1> &a, int mask)
{
    Acc<1> r;
    r.v = __shfl_xor(a.v, mask, 64);
    return r;
}

// Columns of the operand the lane that owns columns [col, col + V) loads (the lane's own, or the row's last four
// where its own would reach past the row; lanes beyond the pass load what the first lane does and drop it).
template <bool RAG> __device__ inline int load_col(const SpmmArgs &a, const SpmmIo &io, int col)
{
    const int c = col < io.col_end ? col : io.col0;
    return RAG && c > a.load_max ? a.load_max : c;
}

// Store the V columns a lane owns (clipped to col_end), adding `add_row` when present.
template <int V>
__device__ inline void store_cols(const Acc<V> &acc, float *y_row, const float *add_row, int col, int col_end)
{
    if (V == 4 && col + 4 <= col_end) {
        float4 o = make_float4(acc.get(0), acc.get(1), acc.get(2), acc.get(3));
        if (add_row) {
            const float4 a = load4(add_row + col);
            o.x += a.x; o.y += a.y; o.z += a.z; o.w += a.w;
        }
        store4(y_row + col, o);
    } else {
#pragma unroll
        for (int i = 0; i < V; ++i)
            if (col + i < col_end) y_row[col + i] = acc.get(i) + (add_row ? add_row[col + i] : 0.f);
    }
}

// Accumulate one chunk of a wavefront item: lane i holds the (column, value) pair of the chunk's
// entry i (lanes past the chunk hold a valid column).  Sub-step t hands entry t * G + grp to lane
// group grp through cross-lane reads, eight sub-steps (eight gathers per lane) at a time.  A
// full chunk (cnt >= 64) and the whole eights of a shorter one run without any per-entry test; the sub-steps behind them make no access
// without an entry (a 16-byte gather takes the CU's L1 16 cycles however many of its lanes are wanted).  With a test per sub-step in the
// eights as well: 61 k nodes, 7.3 M entries, 79 columns 310 -> 380 us.  Every lane of the wavefront must call
// this (lanes past the last column pass a valid `col` and drop their result).
template <int LPR, int V, bool S32, bool FACT>
__device__ inline void gather_chunk(Acc<V> &acc, const SpmmArgs &a, const SpmmIo &io, int c_l, float v_l, int cnt, int grp, int col)
{
    constexpr int G = 64 / LPR; // lane groups = entries per sub-step
    constexpr int U = 8;        // gathers in flight per lane
    using L = Ld<V>;
    // sub-steps t to t + U of the chunk, `left` of which have an entry (ALL: every lane of all of them)
    auto sub_steps = [&](int t, int left, auto all) {
        constexpr bool ALL = decltype(all)::value;
        int c[U];
        float v[U];
        typename L::T x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int src = ALL ? (t + u) * G + grp : ((t + u) * G + grp) & 63;
            c[u] = __shfl(c_l, src, 64);
            v[u] = shfl_val<FACT>(v_l, src);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (ALL || u < left) x[u] = load_x<V, S32>(a, io.X, c[u], col);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (ALL || (t + u) * G + grp < cnt) acc.fma(v[u], x[u]);
    };
    // not unrolled: with 16 or more lanes per row the unrolled loop holds the shuffled pairs of the whole chunk and
    // halves the wavefronts per SIMD (60 registers against 81-97), which costs 1.5 % at 301 columns
    const int full = cnt >= 64 ? LPR : cnt / G / U * U; // sub-steps of whole eights
#pragma unroll 1
    for (int t = 0; t < full; t += U) sub_steps(t, U, std::true_type());
    if (full * G < cnt && full < LPR) sub_steps(full, (cnt - full * G + G - 1) / G, std::false_type());
}

// Write an item's (or a row's) sum: to the output row, or to its partial-sum slot.
template <int V, bool RAG>
__device__ inline void store_result(Acc<V> acc, const SpmmArgs &a, const SpmmIo &io, int row, int dst, int col)
{
    if (RAG) acc.shift(col - load_col<RAG>(a, io, col));
    if (dst >= 0) {
        if (a.dinv) acc.scale(a.dinv[row]); // factored form: the row's own factor (partial sums stay unscaled)
        store_cols<V>(acc, io.Y + (int64_t)row * a.ldy, io.Add ? io.Add + (int64_t)row * a.ldadd : nullptr, col, io.col_end);
    } else {
        float *p = io.scratch + (int64_t)(-(dst + 1)) * a.slot_cols - a.col0;
        store_cols<V>(acc, p, nullptr, col, io.col_end);
    }
}

constexpr int NO_UNIT = INT32_MIN;

// Which chunk of the whole-row lane-group items the q-th workgroup of class c takes: 2^deal consecutive chunks per class in
// turn, so that with a row order that puts rows with common neighbours side by side (breadth first) an XCD works on a
// stretch of some thousand rows at a time and their gathers meet in its L2, while every class still gets its share of
// each part of the list.  2^deal = 1 / 8 / 16 / 32 / 64 / 512, 2 M nodes in communities in breadth-first order, 32 columns:
// 1.29 / 1.11 / 1.09 / 1.08 / 1.08 / 1.09 ms (64 columns 2.53 / 2.17 / 2.15 / 2.14 / 2.14 / 2.17); R-MAT and uniform
// random graphs of 0.3 to 2.4 M nodes, any order: no difference above 1 %.  Shorter lists are dealt in smaller stretches,
// eight turns per class or single chunks, so that no class runs dry.
constexpr int MAX_DEAL = 5;
__device__ inline int64_t dealt(int q, int c, int deal) { return ((((int64_t)(q >> deal) * N_CLASSES + c) << deal) + (q & ((1 << deal) - 1))); }
constexpr int MAX_RUN = 8; // items per lane group, RUNS
constexpr int64_t SMALL_GRID = 1024; // workgroups of one kind a cache-resident graph is cut into before runs grow

// One gather phase of the tiny-row path: sub-round t hands unit (t * GROUPS + grp) of the wavefront
// to lane group grp.  c_l / v_l hold, per lane, four (column, value) pairs of the unit that lane
// owns (column -1 = no entry).  Two sub-rounds (eight gathers per lane) are in flight at a time.
template <int LPR, int V, bool S32, bool FACT>
__device__ inline void batch_gather(Acc<V> (&acc)[8], const SpmmArgs &a, const SpmmIo &io, const int (&c_l)[4], const float (&v_l)[4],
                                    int grp, int colc)
{
    constexpr int G = 64 / LPR;
    using L = Ld<V>;
#pragma unroll
    for (int t0 = 0; t0 < 8; t0 += 2) {
        if (t0 >= a.tiny_rounds) break; // uniform
        int cc[2][4];
        float vv[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                cc[u][i] = __shfl(c_l[i], (t0 + u) * G + grp, 64);
                vv[u][i] = shfl_val<FACT>(v_l[i], (t0 + u) * G + grp);
            }
        typename L::T x[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int c = cc[u][i] >= 0 ? cc[u][i] : 0; // an absent entry re-reads row 0 and is not accumulated
                x[u][i] = load_x<V, S32>(a, io.X, c, colc);
            }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (cc[u][i] >= 0) acc[t0 + u].fma(vv[u][i], x[u][i]);
    }
}

// Rows of at most TINY_ROW (= 4) entries: tiny_rounds * GROUPS rows per wavefront.  Lane i owns row i
// (entries [beg_l, end_l), destination dst_l, NO_UNIT = nothing) and loads its entries; the gather
// phase hands them to the lane groups.  Every lane of the wavefront must call this.
template <int LPR, int V, bool S32, bool FACT, bool RAG>
__device__ inline void batch_units(const SpmmArgs &a, const SpmmIo &io, int beg_l, int end_l, int row_l, int dst_l, int lane)
{
    constexpr int G = 64 / LPR;
    const int grp = lane / LPR, sub = lane % LPR;
    const int col = io.col0 + sub * V;
    const bool col_ok = col < io.col_end;
    const int colc = load_col<RAG>(a, io, col);
    Acc<V> acc[8];
    int c_l[4];
    float v_l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int idx = beg_l + i;
        const bool ok = idx < end_l;
        c_l[i] = ok ? a.colidx[idx] : -1;
        v_l[i] = ok ? ld_val<FACT>(a, idx) : 0.f;
    }
    batch_gather<LPR, V, S32, FACT>(acc, a, io, c_l, v_l, grp, colc);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        if (t >= a.tiny_rounds) break; // uniform
        const int d = __shfl(dst_l, t * G + grp, 64);
        const int r = __shfl(row_l, t * G + grp, 64);
        if (d != NO_UNIT && col_ok) store_result<V, RAG>(acc[t], a, io, r, d, col);
    }
}

// Wavefront items: workgroup b serves class b mod 8, four items per workgroup: first the
// class's own pieces, then every eighth group of four whole-row items.  An item's
// entries are read 64 (column, value) pairs at a time with one coalesced load each, lane i holding
// entry base + i, and the next 64 are requested before the current ones are consumed.  (Giving a
// wavefront several items and prefetching across them was measured and changes nothing: the
// kernel is bound by the traffic of the gathers, not by the latency of its index loads.)
// The XCDs' fabric serves 7.2 TB/s of 128-byte rows that miss the L2s, wherever they lie, and the L1s deliver 28 TB/s of rows that hit;
// a loop over the same column indices in one list per class, without items, gathers 24.8 TB/s (233 k nodes, 106 M entries, 128 columns) and
// 18.1 (2.4 M nodes, 94 M entries, 32 and 64 columns).  Long rows' pieces in ranges of length, no access without an entry and descriptors
// through the scalar cache: this kernel 2.28 -> 2.19 ms (128 columns of the former graph), 745 -> 706 us and 1.48 -> 1.43 ms (of the latter).
template <int LPR, int V, bool S32, bool FACT, bool RAG>
__device__ __forceinline__ void wave_items_body(const SpmmArgs &a, const SpmmIo &io, int block)
{
    // told to be the same for a wavefront: its item's descriptor comes through the scalar cache
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int cls = block % N_CLASSES, j = block / N_CLASSES;
    const int piece_blocks = (a.big_cnt[cls] + 3) >> 2;
    int64_t item;
    if (j < piece_blocks) { // uniform per workgroup
        item = j * 4 + wave;
        if (item >= a.big_cnt[cls]) return;
        item += a.big_off[cls];
    } else {
        item = ((int64_t)(j - piece_blocks) * N_CLASSES + cls) * 4 + wave;
        if (item >= a.wbig_cnt) return;
        item += a.wbig_off;
    }
    const int4 s = *reinterpret_cast<const int4 *>(a.items + item);
    const int grp = lane / LPR, sub = lane % LPR;
    const int col = io.col0 + sub * V;
    const bool active = col < io.col_end;
    const int colc = load_col<RAG>(a, io, col);
    const int beg = s.y, end = s.z;
    Acc<V> acc;
    int idx = beg + lane;
    int c_l = a.colidx[idx < end ? idx : beg];
    float v_l = ld_val<FACT>(a, idx < end ? idx : beg);
    for (int base = beg; base < end; base += 64) {
        int c_n = 0;
        float v_n = 0.f;
        if (base + 64 < end) { // wavefront-uniform
            idx = base + 64 + lane;
            c_n = a.colidx[idx < end ? idx : beg];
            v_n = ld_val<FACT>(a, idx < end ? idx : beg);
        }
        gather_chunk<LPR, V, S32, FACT>(acc, a, io, c_l, v_l, end - base, grp, colc);
        c_l = c_n;
        v_l = v_n;
    }
#pragma unroll
    for (int m = LPR; m < 64; m <<= 1) acc.add(shfl_xor_acc<V>(acc, m));
    if (grp == 0 && active) store_result<V, RAG>(acc, a, io, s.x, s.w, col);
}

// The same for graphs that stay in cache (the one-launch kernel below): a workgroup takes 4 * ipw consecutive items,
// wavefront w the items w, w + 4, ... of them; the next item's descriptor is requested when an item starts and its first
// entries during the item's last chunk.  There a call lasts tens of microseconds and is made of chains of dependent loads
// (descriptor -> entries -> gathers), which this overlaps across items: 0.049 -> 0.043 ms per call at 2.5 M entries.  On
// graphs that stream from memory it changes nothing and its eight extra registers cost 2 %, so they keep one item per wavefront.
template <int LPR, int V, bool S32, bool FACT, bool RAG>
__device__ __forceinline__ void wave_items_run_body(const SpmmArgs &a, const SpmmIo &io, int block)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int cls = block % N_CLASSES, j = block / N_CLASSES;
    const int ipb = 4 * a.ipw; // items per workgroup
    const int piece_blocks = (a.big_cnt[cls] + ipb - 1) / ipb;
    int64_t first, left;
    if (j < piece_blocks) { // uniform per workgroup
        first = (int64_t)j * ipb;
        left = a.big_cnt[cls] - first;
        first += a.big_off[cls];
    } else {
        first = ((int64_t)(j - piece_blocks) * N_CLASSES + cls) * ipb;
        left = a.wbig_cnt - first;
        first += a.wbig_off;
    }
    const int cnt = left < ipb ? (int)left : ipb;
    int t = wave; // this wavefront takes items wave, wave + 4, ... of the workgroup's run
    if (t >= cnt) return;
    const int grp = lane / LPR, sub = lane % LPR;
    const int col = io.col0 + sub * V;
    const bool active = col < io.col_end;
    const int colc = load_col<RAG>(a, io, col);
    int4 s = *reinterpret_cast<const int4 *>(a.items + first + t);
    int idx = s.y + lane;
    int c_l = a.colidx[idx < s.z ? idx : s.y];
    float v_l = ld_val<FACT>(a, idx < s.z ? idx : s.y);
    for (;;) {
        const bool more = t + 4 < cnt; // wavefront-uniform
        // the next item's descriptor is requested now and its first entries during this item's last chunk, so
        // that a short item does not expose the whole chain descriptor -> entries -> gathers
        int4 sn = s;
        if (more) sn = *reinterpret_cast<const int4 *>(a.items + first + t + 4);
        const int beg = s.y, end = s.z;
        Acc<V> acc;
        for (int base = beg; base < end; base += 64) {
            int c_n = 0;
            float v_n = 0.f;
            if (base + 64 < end) { // wavefront-uniform
                idx = base + 64 + lane;
                c_n = a.colidx[idx < end ? idx : beg];
                v_n = ld_val<FACT>(a, idx < end ? idx : beg);
            } else if (more) {
                idx = sn.y + lane;
                c_n = a.colidx[idx < sn.z ? idx : sn.y];
                v_n = ld_val<FACT>(a, idx < sn.z ? idx : sn.y);
            }
            gather_chunk<LPR, V, S32, FACT>(acc, a, io, c_l, v_l, end - base, grp, colc);
            c_l = c_n;
            v_l = v_n;
        }
#pragma unroll
        for (int m = LPR; m < 64; m <<= 1) acc.add(shfl_xor_acc<V>(acc, m));
        if (grp == 0 && active) store_result<V, RAG>(acc, a, io, s.x, s.w, col);
        if (!more) break;
        s = sn;
        t += 4;
    }
}

// Lane-group items (whole rows and class pieces of 5..GI_MAX entries, GI_MAX = the schedule's item_max):
// workgroup b serves class b mod 8 and takes 4 * G consecutive items of its list (first the class's own pieces, then its
// share of the whole rows; RUNS: a.rounds times as many), lane group grp of wavefront w the item w * G + grp of them.  The group reads the item's
// (column, value) pairs with one read per LPR entries (lane `sub` holds entries sub, sub + LPR, ...), and each gather takes
// its pair from the holding lane by a cross-lane read, eight gathers in flight.
// One item per lane group, not a run of several: what is in flight together on an XCD is then a short stretch of rows
// (with a row order its gathers meet in the L2), the last workgroups end together, and the registers that held the next
// item's pairs are free.  Runs of 8 / 4 / 2 / 1 items per lane group: 6.3 M entries, 300 k nodes 70 / 64 / 63 / 63 us;
// 41 M entries, 1 M nodes 0.422 / 0.410 / 0.406 / 0.404 ms; 126 M entries 1.246 / 1.237 / 1.232 / 1.229 ms; 2 M nodes in
// communities, breadth-first order 1.55 / 1.53 / 1.42 / 1.29 ms (all 32 columns).
// RUNS, where a graph stays in cache and a row's columns lie close together (meshes, bands, rows that all point at a few nodes): gathers return at once there,
// the chain descriptor, pairs, gathers, store bounds a wavefront, and runs overlap it (the next round's pairs are requested behind the
// first gathers).  1 M nodes, 1 / 8 items per lane group: 5 entries a row 64 columns 217 / 168 us, 128 columns 422 / 309, 7 entries 64 columns
// 222 / 177, 9 entries 273 / 242, 17 entries 327 / 309; 885 k nodes, 12 entries a row in the columns below 885, 16 columns 106 / 93; but uniform
// random graphs of 7 entries a row 235 / 247, 128 columns 461 / 487.
// On graphs that stay in cache the compiler is kept from moving a set's first gather into the branch that adds it (the entry may be absent), behind all others,
// where the wavefront waits for memory a second time: 2 k nodes, 11 k edges, 64 columns 4.05 -> 3.70 us, 15 k nodes, 64 k edges, 100 columns 10.3 -> 9.7,
// from some 100 k nodes on level; streamed graphs are 0.5 % slower with it (2 M nodes in communities, inference 10.84 -> 10.89 ms).
template <int LPR, int V, bool S32, int GI_MAX, bool FACT, bool RAG, bool RUNS>
__device__ __forceinline__ void group_items_body(const SpmmArgs &a, const SpmmIo &io, int block)
{
    constexpr int G = 64 / LPR;                 // items in flight per wavefront
    constexpr int K = LPR >= GI_MAX ? 1 : GI_MAX / LPR; // index registers per lane (K * LPR >= GI_MAX entries)
    constexpr int U = 8;
    constexpr int ROUND = 4 * G;                // items a workgroup has in flight
    using L = Ld<V>;
    const int run = RUNS ? ROUND * a.rounds : ROUND; // items per workgroup
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int cls = block % N_CLASSES, blk = block / N_CLASSES;
    const int piece_blocks = (a.small_cnt[cls] + run - 1) / run;
    const int grp = lane / LPR, sub = lane % LPR, gbase = lane - sub;
    const bool pieces = blk < piece_blocks; // uniform per workgroup
    const int64_t at = (pieces ? blk : dealt(blk - piece_blocks, cls, a.deal)) * run;
    const int64_t left = (pieces ? a.small_cnt[cls] : a.wsmall_cnt) - at - wave * G; // from this wavefront's first item on
    const int4 *items = reinterpret_cast<const int4 *>(a.items) + (pieces ? a.small_off[cls] : a.wsmall_off) + at + wave * G;
    if (RUNS && left <= 0) return; // uniform per wavefront
    // Round r works on the ROUND consecutive items from r * ROUND on.  RUNS: lane r * G + g holds the descriptor of round r, group g.
    int4 d = make_int4(0, 0, 0, NO_UNIT);
    static_assert(MAX_RUN * G <= 64, "one descriptor per lane");
    const int q = RUNS ? lane / G * ROUND + lane % G : grp;
    if ((!RUNS || lane < a.rounds * G) && q < left) d = items[q];
    const int rounds = !RUNS ? 1 : left < run ? (int)(left + ROUND - 1) / ROUND : a.rounds;
    const int col = io.col0 + sub * V;
    const bool col_ok = col < io.col_end;
    const int colc = load_col<RAG>(a, io, col);
    auto of_round = [&](int x, int r) { return RUNS ? __shfl(x, r * G + grp, 64) : x; };
    int beg = of_round(d.y, 0), end = of_round(d.z, 0);
    int c_k[K];
    float v_k[K];
    auto pairs = [&](int (&c)[K], float (&v)[K], int from, int to) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int e = from + sub + LPR * k;
            const bool ok = e < to;
            c[k] = ok ? a.colidx[e] : 0;
            v[k] = ok ? ld_val<FACT>(a, e) : 0.f;
        }
    };
    pairs(c_k, v_k, beg, end);
    for (int r = 0; r < rounds; ++r) {
        const int row = of_round(d.x, r), dst = of_round(d.w, r), len = end - beg;
        int c_n[K];
        float v_n[K];
        if (RUNS) {
            const int next = r + 1 < rounds ? r + 1 : 0;
            beg = of_round(d.y, next);
            end = next ? of_round(d.z, next) : beg;
        }
        Acc<V> acc;
#pragma unroll
        for (int j0 = 0; j0 < GI_MAX; j0 += U) {
            if (!__any(j0 < len)) break; // wavefront-uniform
            int c[U];
            float v[U];
            typename L::T x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int jj = j0 + u;
                const int cc = __shfl(c_k[jj / LPR < K ? jj / LPR : 0], gbase + jj % LPR, 64);
                v[u] = shfl_val<FACT>(v_k[jj / LPR < K ? jj / LPR : 0], gbase + jj % LPR);
                c[u] = jj < len ? cc : 0; // an absent entry re-reads row 0 and is not accumulated
            }
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = load_x<V, S32>(a, io.X, c[u], colc);
            if (GI_MAX == ITEM_SHORT) asm volatile("" ::: "memory"); // all gathers are requested before one is used (see above)
            if (RUNS && j0 == 0) pairs(c_n, v_n, beg, end); // the next round's, behind the first gathers (none behind the last round)
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (j0 + u < len) acc.fma(v[u], x[u]);
        }
        if (dst != NO_UNIT && col_ok) store_result<V, RAG>(acc, a, io, row, dst, col);
        if (RUNS) {
#pragma unroll
            for (int k = 0; k < K; ++k) { c_k[k] = c_n[k]; v_k[k] = v_n[k]; }
        }
    }
}

// Rows of at most TINY_ROW entries, up to 64 consecutive ones of their list per wavefront.
template <int LPR, int V, bool S32, bool FACT, bool RAG>
__device__ __forceinline__ void tiny_rows_body(const SpmmArgs &a, const SpmmIo &io, int block)
{
    const int units = a.tiny_rounds * (64 / LPR); // rows per wavefront
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t first = ((int64_t)block * 4 + wave) * units;
    if (first >= a.tiny_cnt) return; // uniform per wavefront
    int beg_l = 0, end_l = 0, row_l = 0, dst_l = NO_UNIT;
    if (lane < units && first + lane < a.tiny_cnt) {
        const TinyRow r = a.tiny[first + lane];
        row_l = dst_l = (int)(r.row & NO_ENTRIES);
        if (r.beg != NO_ENTRIES) {
            beg_l = (int)(r.beg & NO_ENTRIES);
            end_l = beg_l + 1 + (int)(r.row >> 31 | r.beg >> 31 << 1);
        }
    }
    batch_units<LPR, V, S32, FACT, RAG>(a, io, beg_l, end_l, row_l, dst_l, lane);
}

template <int LPR, int V, bool S32, bool FACT, bool RAG>
__global__ __launch_bounds__(256) void spmm_wave_items_kernel(const SpmmArgs a, const SpmmBatch b, unsigned first) { const SpmmIo io = pick_io(a, b); wave_items_body<LPR, V, S32, FACT, RAG>(a, io, blockIdx.x + first); }

template <int LPR, int V, bool S32, int GI_MAX, bool FACT, bool RAG>
__global__ __launch_bounds__(256) void spmm_group_items_kernel(const SpmmArgs a, const SpmmBatch b, unsigned first) { const SpmmIo io = pick_io(a, b); group_items_body<LPR, V, S32, GI_MAX, FACT, RAG, false>(a, io, blockIdx.x + first); }

template <int LPR, int V, bool S32, bool FACT, bool RAG>
__global__ __launch_bounds__(256) void spmm_tiny_rows_kernel(const SpmmArgs a, const SpmmBatch b, unsigned first) { const SpmmIo io = pick_io(a, b); tiny_rows_body<LPR, V, S32, FACT, RAG>(a, io, blockIdx.x + first); }

// All three item kinds in one launch: workgroups [0, g1) take wavefront items, [g1, g1 + g2)
// lane-group items, the rest tiny rows (g1 and g2 are multiples of 8, so workgroup b still
// serves class b mod 8).  For graphs that stay in cache a call takes tens of microseconds and
// each of three launches would pay its own ramp-up and its own chain of dependent loads; in one launch
// they overlap (cfg2: 0.075 -> 0.056 ms per call).  Large graphs keep the three launches: there the
// class pieces must have the L2s to themselves before the whole rows start (merged: cfg5 4.09 -> 4.30 ms).
template <int LPR, int V, bool S32, bool FACT, bool RAG, bool RUNS>
__global__ __launch_bounds__(256) void spmm_merged_kernel(const SpmmArgs a, const SpmmBatch batch, int g1, int g2, unsigned first)
{
    const SpmmIo io = pick_io(a, batch);
    const int b = blockIdx.x + first; // uniform per workgroup
    if (b < g1) wave_items_run_body<LPR, V, S32, FACT, RAG>(a, io, b);
    else if (b < g1 + g2) group_items_body<LPR, V, S32, ITEM_SHORT, FACT, RAG, RUNS>(a, io, b - g1);
    else tiny_rows_body<LPR, V, S32, FACT, RAG>(a, io, b - g1 - g2);
}

// The same behind the first `extra` workgroups (a multiple of 8), which form the final sums of the weight gradients: those are a launch of
// their own otherwise, on a small graph as long as the aggregation itself.  Backward passes of slice layers, sums in their own launch / here:
// 2048 rows 64 -> 32 12.9 / 11.1 us, 5000 rows 200 -> 200 78.9 / 73.6, 60 k rows 32 -> 32 32.9 / 29.9; 169 k rows, four slices: 10 us less.
template <int LPR, bool RUNS>
__global__ __launch_bounds__(256) void spmm_merged_sums_kernel(const SpmmArgs a, const SpmmBatch batch, int g1, int g2, const FinalWork f, int extra)
{
    const int b = (int)blockIdx.x - extra; // uniform per workgroup
    if (b < 0) {
        final_sum<256>(f, blockIdx.x, blockIdx.y);
        return;
    }
    const SpmmIo io = pick_io(a, batch);
    if (b < g1) wave_items_run_body<LPR, 4, true, true, false>(a, io, b);
    else if (b < g1 + g2) group_items_body<LPR, 4, true, ITEM_SHORT, true, false, RUNS>(a, io, b - g1);
    else tiny_rows_body<LPR, 4, true, true, false>(a, io, b - g1 - g2);
}

// Rows with several items: add the partial slots in order.  One thread per (row, column); eight
// independent slot reads are in flight at a time, the additions stay in slot order.
__global__ __launch_bounds__(256) void spmm_fix_kernel(const SpmmArgs a, const SpmmBatch b, int32_t n_fix)
{
    const SpmmIo io = pick_io(a, b);
    const int w = a.col_end - a.col0;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t r = t / w;
    if (r >= n_fix) return;
    const int j = (int)(t - r * w);
    const int4 f = *reinterpret_cast<const int4 *>(a.fix + r);
    const float *p = io.scratch + j;
    float acc = 0.f;
    int s = f.y;
    for (; s + 8 <= f.z; s += 8) {
        float q[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) q[i] = p[(int64_t)(s + i) * a.slot_cols];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc += q[i];
    }
    for (; s < f.z; ++s) acc += p[(int64_t)s * a.slot_cols];
    if (a.dinv) acc *= a.dinv[f.x]; // factored form: the row's own factor
    const int col = a.col0 + j;
    if (io.Add) acc += io.Add[(int64_t)f.x * a.ldadd + col];
    io.Y[(int64_t)f.x * a.ldy + col] = acc;
}

// `batch`: slices aggregated in this launch; `passes`: column passes in this launch (the one-launch kernel only); `sums`: final sums to form in
// the launch (may_join_sums)
template <int LPR, int V, bool S32, bool FACT, bool RAG>
int launch_variant(const SpmmArgs &a, const SpmmBatch &b, int batch, int passes, const FinalWork *sums, hipStream_t stream)
{
    const int64_t units_per_block = 4 * a.tiny_rounds * (64 / LPR);
    const int64_t g1 = (int64_t)N_CLASSES * a.big_blocks;
    const int64_t g2 = (int64_t)N_CLASSES * a.small_blocks;
    const int64_t g3 = (a.tiny_cnt + units_per_block - 1) / units_per_block;
    SG_REQUIRE(g1 + g2 + g3 + N_CLASSES <= INT32_MAX, SLICEGCN_ERANGE, "spmm: grid too large");
    if (a.item_max <= ITEM_SHORT) { // cache-resident graph: one launch (big_blocks counts runs of 4 * ipw items)
        // the grid's first dimension is a multiple of 8, so that a class meets the same XCD in every slice and pass
        const int64_t blocks = round_up(g1 + g2 + g3, N_CLASSES);
        if constexpr (V == 4 && S32 && FACT && !RAG) {
            const int64_t extra = sums ? round_up((sums->stride + FINAL_ELEMS - 1) / FINAL_ELEMS, N_CLASSES) : 0;
            if (sums && blocks + extra <= MAX_GRID) {
                const dim3 grid((unsigned)(blocks + extra), (unsigned)batch, (unsigned)passes);
                if (a.rounds > 1) spmm_merged_sums_kernel<LPR, true><<<grid, 256, 0, stream>>>(a, b, (int)g1, (int)g2, *sums, (int)extra);
                else spmm_merged_sums_kernel<LPR, false><<<grid, 256, 0, stream>>>(a, b, (int)g1, (int)g2, *sums, (int)extra);
                SG_LAUNCH_CHECK();
                return SLICEGCN_OK;
            }
        }
        if (sums)
            if (int rc = launch_final_sum(*sums, batch, stream)) return rc;
        return launch_parts(blocks, [&](unsigned first, unsigned count) {
            const dim3 grid(count, (unsigned)batch, (unsigned)passes);
            if (a.rounds > 1) spmm_merged_kernel<LPR, V, S32, FACT, RAG, true><<<grid, 256, 0, stream>>>(a, b, (int)g1, (int)g2, first);
            else spmm_merged_kernel<LPR, V, S32, FACT, RAG, false><<<grid, 256, 0, stream>>>(a, b, (int)g1, (int)g2, first);
        });
    }
    // a part of a grid starts at a multiple of 8, so that workgroup b still serves class b mod 8
    if (int rc = launch_parts(g1, [&](unsigned first, unsigned count) {
            spmm_wave_items_kernel<LPR, V, S32, FACT, RAG><<<dim3(count, (unsigned)batch), 256, 0, stream>>>(a, b, first);
        }))
        return rc;
    if (int rc = launch_parts(g2, [&](unsigned first, unsigned count) {
            spmm_group_items_kernel<LPR, V, S32, ITEM_LONG, FACT, RAG><<<dim3(count, (unsigned)batch), 256, 0, stream>>>(a, b, first);
        }))
        return rc;
    return launch_parts(g3, [&](unsigned first, unsigned count) {
        spmm_tiny_rows_kernel<LPR, V, S32, FACT, RAG><<<dim3(count, (unsigned)batch), 256, 0, stream>>>(a, b, first);
    });
}

template <int LPR, int V, bool FACT>
int launch_layout(const SpmmArgs &a, const SpmmBatch &b, int batch, int passes, const FinalWork *sums, hipStream_t stream)
{
    if constexpr (V == 1) return launch_variant<LPR, V, false, FACT, false>(a, b, batch, passes, sums, stream);
    else {
        if (a.load_max > 0)
            return a.ldx_bytes != 0 ? launch_variant<LPR, V, true, FACT, true>(a, b, batch, passes, sums, stream)
                                    : launch_variant<LPR, V, false, FACT, true>(a, b, batch, passes, sums, stream);
        return a.ldx_bytes != 0 ? launch_variant<LPR, V, true, FACT, false>(a, b, batch, passes, sums, stream)
                                : launch_variant<LPR, V, false, FACT, false>(a, b, batch, passes, sums, stream);
    }
}

template <int LPR, int V>
int launch_kernels(const SpmmArgs &a, const SpmmBatch &b, int batch, int passes, const FinalWork *sums, hipStream_t stream)
{
    return a.dinv ? launch_layout<LPR, V, true>(a, b, batch, passes, sums, stream) : launch_layout<LPR, V, false>(a, b, batch, passes, sums, stream);
}

int launch_pass(const SpmmArgs &a, const SpmmBatch &b, int batch, int passes, int v, int lpr, const FinalWork *sums, hipStream_t stream)
{
    if (v == 1) return launch_kernels<8, 1>(a, b, batch, passes, sums, stream); // fewer than 4 columns
    switch (lpr) {
    case 8: return launch_kernels<8, 4>(a, b, batch, passes, sums, stream);
    case 16: return launch_kernels<16, 4>(a, b, batch, passes, sums, stream);
    default: return launch_kernels<32, 4>(a, b, batch, passes, sums, stream); // a pass is at most 128 columns
    }
}

// Whether a launch can form final sums beside the aggregation (the form that the input gradients of layers take)
inline bool may_join_sums(const SpmmArgs &a, int v, int passes)
{
    return a.item_max <= ITEM_SHORT && passes == 1 && v == 4 && a.ldx_bytes != 0 && a.dinv != nullptr && a.load_max <= 0;
}

} // namespace

// Bytes of partial-sum workspace an aggregation of `width` columns over pattern `m` needs: one slot per item of
// every row cut into several items, of as many floats as one launch covers columns: all of them (rounded up to 4) on a
// cache-resident graph, at most one pass otherwise or where the caller has no more room (`one_pass`).
size_t spmm_workspace_bytes(const Csr &m, int32_t width, bool one_pass)
{
    const int64_t w4 = round_up(width, 4);
    const bool all = !one_pass && m.sched.item_max <= ITEM_SHORT;
    return (size_t)round_up(m.sched.n_slots * (w4 < PASS_COLS || all ? w4 : PASS_COLS) * (int64_t)sizeof(float), 256);
}

int launch_spmm(const slicegcn_graph *g, const Csr &m, const SpmmOperands *ops, int batch, int64_t ldx, int32_t width,
                int64_t ldy, int64_t ldadd, void *ws, size_t ws_bytes, hipStream_t stream, bool prescaled, const FinalWork *sums)
{
    SG_REQUIRE(batch >= 1 && batch <= MAX_BATCH, SLICEGCN_EINVAL, "aggregation: batch of %d", batch);
    // Operands of 1 to 3 columns: one float per lane, also where their rows have room for a 16-byte gather.  1 column in rows of 4 / 32
    // floats, 126 M entries: 1.07 / 1.28 ms (with 16-byte gathers, which they took before: 1.17 / 1.34); 310 M entries 3.35 / 4.12 (3.48 /
    // 4.15); 2.5 M entries 26 / 29 us (43 / 45, of which the shorter runs on small graphs are the larger part).
    const int V = width >= 4 ? 4 : 1;
    // passes of at most 128 columns (32 lanes per row): narrower ones re-read the index streams more often, wider ones
    // make the set of hot rows of the operand too large for the L2s (301 columns: 7.8 / 7.4 / 7.7 ms for passes of 64 / 128 / 256)
    const Schedule &sc = m.sched;
    const bool resident = sc.item_max <= ITEM_SHORT;
    const bool multi_pass = resident && width > PASS_COLS && ws_bytes >= batch * spmm_workspace_bytes(m, width, false);
    const size_t each = spmm_workspace_bytes(m, width, !multi_pass);
    const size_t need = sc.n_slots > 0 ? batch * each : 0;
    SG_REQUIRE(need == 0 || (ws != nullptr && ws_bytes >= need), SLICEGCN_EWORKSPACE,
               "aggregation: workspace of %zu bytes, %zu needed", ws_bytes, need);
    SG_REQUIRE(need == 0 || (reinterpret_cast<uintptr_t>(ws) & 255u) == 0, SLICEGCN_EINVAL,
               "aggregation: workspace not 256-byte aligned");
    SpmmArgs a;
    SpmmBatch b;
    bool aligned = true, any_add = false;
    for (int i = 0; i < MAX_BATCH; ++i) {
        const SpmmOperands &o = ops[i < batch ? i : 0];
        b.X[i] = o.X; b.Y[i] = o.Y; b.Add[i] = o.Add;
        aligned = aligned && aligned16(o.X);
        any_add = any_add || o.Add;
    }
    a.colidx = m.colidx; a.vals = m.vals; a.items = sc.items; a.fix = sc.fix; a.tiny = sc.tiny;
    a.scratch = static_cast<float *>(ws);
    a.scratch_stride = (int64_t)(each / sizeof(float));
    a.dinv = prescaled ? g->dinv : nullptr;
    a.ldx = ldx; a.ldy = ldy; a.ldadd = ldadd;
    const bool s32 = g->n < (1 << 24) && ldx * 4 < (1 << 24) && (int64_t)g->n * ldx * 4 < ((int64_t)1 << 32);
    a.ldx_bytes = s32 ? (uint32_t)(ldx * 4) : 0u;
    a.item_max = sc.item_max;
    const int64_t w4 = round_up(width, 4);
    a.slot_cols = (int32_t)(multi_pass || w4 < PASS_COLS ? w4 : PASS_COLS);
    // rows whose last vector stays inside the row: a multiple of four columns, or room for the padding up to one
    const bool whole = V == 1 || width % 4 == 0 || (aligned && ldx % 4 == 0);
    a.load_max = whole ? 0 : width - 4;
    a.wbig_off = sc.wbig_off; a.wbig_cnt = sc.wbig_cnt;
    a.wsmall_off = sc.wsmall_off; a.wsmall_cnt = sc.wsmall_cnt;
    a.tiny_cnt = sc.tiny_cnt;
    for (int c = 0; c < N_CLASSES; ++c) {
        a.big_off[c] = sc.big_off[c]; a.big_cnt[c] = sc.big_cnt[c];
        a.small_off[c] = sc.small_off[c]; a.small_cnt[c] = sc.small_cnt[c];
    }
    ProfScope prof(any_add ? SLICEGCN_PROF_SPMM_ADD : SLICEGCN_PROF_SPMM, width, stream);
    const int32_t full_cols = width / PASS_COLS * PASS_COLS; // whole passes share a launch, the rest has lane groups of its own width
    for (int32_t c0 = 0; c0 < width; c0 = a.col_end) {
        a.col0 = c0;
        a.col_end = c0 >= full_cols ? width : multi_pass ? full_cols : c0 + PASS_COLS;
        const int passes = (a.col_end - c0 + PASS_COLS - 1) / PASS_COLS;
        const int pass_cols = passes > 1 ? PASS_COLS : a.col_end - c0;
        int lpr = 8;
        while (lpr < (pass_cols + V - 1) / V) lpr <<= 1; // 8, 16 or 32
        // How much a wavefront works through in turn.  On a large graph long runs amortise the chain of dependent loads
        // (descriptor, entries, gathers) across items; a small graph has too few items to fill the chip with such runs, so
        // they are cut until about SMALL_GRID workgroups of each kind are there (2048 nodes, 64 columns: 11.3 -> 6.5 us).
        const int64_t groups = 4 * (64 / lpr), copies = (int64_t)batch * passes;
        auto turns = [&](int64_t items, int64_t per_turn, int most) {
            const int64_t t = items * copies / (per_turn * SMALL_GRID);
            return (int)(t < 1 ? 1 : t > most ? most : t);
        };
        a.ipw = resident ? turns(sc.wbig_cnt, 4, 4) : 1;
        a.rounds = resident && sc.local ? turns(sc.wsmall_cnt, groups, MAX_RUN) : 1;
        a.tiny_rounds = resident ? 2 * turns(sc.tiny_cnt, 2 * groups, 4) : 8;
        // workgroups per class: the class's own pieces, then its share of the whole-row chunks
        const int64_t ipb = 4 * a.ipw;
        const int64_t wbig_chunks = ((int64_t)sc.wbig_cnt + ipb - 1) / ipb;
        const int64_t run = groups * a.rounds;
        const int64_t wsmall_chunks = ((int64_t)sc.wsmall_cnt + run - 1) / run;
        a.deal = 0;
        while (a.deal < MAX_DEAL && (wsmall_chunks >> (a.deal + 1)) >= 8 * N_CLASSES) ++a.deal;
        const int64_t wsmall_blocks = round_up(wsmall_chunks, N_CLASSES << a.deal) / N_CLASSES;
        int64_t big_blocks = 0, small_blocks = 0;
        for (int c = 0; c < N_CLASSES; ++c) {
            const int64_t x = (sc.big_cnt[c] + ipb - 1) / ipb + (wbig_chunks + N_CLASSES - 1 - c) / N_CLASSES;
            const int64_t y = (sc.small_cnt[c] + run - 1) / run + wsmall_blocks;
            big_blocks = x > big_blocks ? x : big_blocks;
            small_blocks = y > small_blocks ? y : small_blocks;
        }
        SG_REQUIRE(big_blocks * N_CLASSES <= INT32_MAX && small_blocks * N_CLASSES <= INT32_MAX, SLICEGCN_ERANGE, "spmm: grid too large");
        a.big_blocks = (int32_t)big_blocks;
        a.small_blocks = (int32_t)small_blocks;
        const bool join = sums && may_join_sums(a, V, passes);
        if (sums && !join)
            if (int rc = launch_final_sum(*sums, batch, stream)) return rc;
        if (int rc = launch_pass(a, b, batch, passes, V, lpr, join ? sums : nullptr, stream)) return rc;
        sums = nullptr;
        if (sc.n_fix > 0) {
            const int64_t threads = sc.n_fix * (int64_t)(a.col_end - c0);
            spmm_fix_kernel<<<dim3((unsigned)((threads + 255) / 256), (unsigned)batch), 256, 0, stream>>>(a, b, (int32_t)sc.n_fix);
            SG_LAUNCH_CHECK();
        }
    }
    return SLICEGCN_OK;
}

} // namespace slicegcn

using namespace slicegcn;

// ---- aggregation without a caller workspace --------------------------------------------------
// The partial sums go to this fixed array instead (one copy per GPU the library runs on, held until the
// process ends).  In host code `scratch` is only a handle for the symbol: the device address comes from
// hipGetSymbolAddress, once per device, and only that address is ever handed to a kernel.
static __device__ __align__(256) unsigned char scratch[SLICEGCN_STATIC_WS_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[MAX_DEVICES] = {nullptr};

// device address of `scratch` on the current device (looked up on the first call per device)
int static_scratch(void **out)
{
    int dev = -1;
    SG_HIP(hipGetDevice(&dev));
    SG_REQUIRE(dev >= 0 && dev < MAX_DEVICES, SLICEGCN_EUNSUPPORTED, "spmm_slice_static: device index %d not supported", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void *ptr = nullptr;
        SG_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        SG_REQUIRE(ptr != nullptr, SLICEGCN_EHIP, "spmm_slice_static: hipGetSymbolAddress returned NULL");
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return SLICEGCN_OK;
}
} // namespace

extern "C" int slicegcn_spmm_slice_static(const slicegcn_graph *g, int op, const float *X, int64_t ldx,
                                          int32_t width, float *Y, int64_t ldy, void *stream)
{
    SG_REQUIRE(g && X && Y, SLICEGCN_EINVAL, "spmm_slice_static: NULL argument");
    SG_REQUIRE((op & ~(SLICEGCN_SPMM_TRANSPOSE | SLICEGCN_SPMM_PRESCALED)) == 0, SLICEGCN_EINVAL, "spmm_slice_static: unknown op bits 0x%x", op);
    SG_REQUIRE(width >= 1, SLICEGCN_EINVAL, "spmm_slice_static: width = %d < 1", width);
    SG_REQUIRE(ldx >= width && ldy >= width, SLICEGCN_EINVAL, "spmm_slice_static: leading dimension smaller than width");
    const Csr &m = (op & SLICEGCN_SPMM_TRANSPOSE) ? g->tr : g->fwd;
    const size_t need = spmm_workspace_bytes(m, width, true);
    SG_REQUIRE(need <= (size_t)SLICEGCN_STATIC_WS_BYTES, SLICEGCN_EWORKSPACE,
               "spmm_slice_static: this graph and width need %zu bytes of partial sums, the built-in buffer holds %zu; "
               "use slicegcn_spmm_slice with a workspace", need, (size_t)SLICEGCN_STATIC_WS_BYTES);
    void *ptr = nullptr;
    if (need > 0)
        if (int rc = static_scratch(&ptr)) return rc;
    const SpmmOperands o{X, Y, nullptr};
    return launch_spmm(g, m, &o, 1, ldx, width, ldy, 0, ptr, need > 0 ? SLICEGCN_STATIC_WS_BYTES : 0, as_stream(stream),
                       (op & SLICEGCN_SPMM_PRESCALED) != 0);
}

extern "C" size_t slicegcn_spmm_workspace_bytes(const slicegcn_graph *g, int op, int32_t width)
{
    if (!g || width < 1) return 0;
    return spmm_workspace_bytes((op & SLICEGCN_SPMM_TRANSPOSE) ? g->tr : g->fwd, width, false);
}

extern "C" int slicegcn_spmm_slice(const slicegcn_graph *g, int op, const float *X, int64_t ldx,
                                   int32_t width, float *Y, int64_t ldy, void *ws, size_t ws_bytes, void *stream)
{
    SG_REQUIRE(g && X && Y, SLICEGCN_EINVAL, "spmm_slice: NULL argument");
    SG_REQUIRE((op & ~(SLICEGCN_SPMM_TRANSPOSE | SLICEGCN_SPMM_PRESCALED)) == 0, SLICEGCN_EINVAL, "spmm_slice: unknown op bits 0x%x", op);
    SG_REQUIRE(width >= 1, SLICEGCN_EINVAL, "spmm_slice: width = %d < 1", width);
    SG_REQUIRE(ldx >= width && ldy >= width, SLICEGCN_EINVAL, "spmm_slice: leading dimension smaller than width");
    const SpmmOperands o{X, Y, nullptr};
    return launch_spmm(g, (op & SLICEGCN_SPMM_TRANSPOSE) ? g->tr : g->fwd, &o, 1, ldx, width, ldy, 0, ws, ws_bytes,
                       as_stream(stream), (op & SLICEGCN_SPMM_PRESCALED) != 0);
}
