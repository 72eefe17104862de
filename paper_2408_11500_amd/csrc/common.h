// Internal declarations shared by the translation units of libslicegcn (not installed).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <cstring>
#include <vector>

#include "slicegcn.h"
#include "slicegcn_native.h"

namespace slicegcn {

// ---- error plumbing ------------------------------------------------------------------
void set_error(const char *fmt, ...) __attribute__((format(printf, 1, 2)));

#define SG_REQUIRE(cond, code, ...)        \
    do {                                   \
        if (!(cond)) {                     \
            ::slicegcn::set_error(__VA_ARGS__); \
            return (code);                 \
        }                                  \
    } while (0)

#define SG_HIP(call)                                                                       \
    do {                                                                                   \
        hipError_t sg_e_ = (call);                                                         \
        if (sg_e_ != hipSuccess) {                                                         \
            ::slicegcn::set_error("%s failed: %s (%s:%d)", #call, hipGetErrorString(sg_e_), \
                                  __FILE__, __LINE__);                                     \
            return sg_e_ == hipErrorOutOfMemory ? SLICEGCN_ENOMEM : SLICEGCN_EHIP;         \
        }                                                                                  \
    } while (0)

#define SG_LAUNCH_CHECK() SG_HIP(hipGetLastError())

inline hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }
inline int64_t round_up(int64_t v, int64_t m) { return (v + m - 1) / m * m; }

// A grid holds fewer than 2^32 threads along a dimension; one of more wraps and runs a part of its workgroups without an error.  Grids that can
// come near that are launched in parts of so many workgroups (of 256 threads; a multiple of the number of XCDs): launch(first, count)
constexpr int64_t MAX_GRID = (int64_t)1 << 23;
template <class F> inline int launch_parts(int64_t blocks, F launch)
{
    for (int64_t first = 0; first < blocks; first += MAX_GRID) {
        launch((unsigned)first, (unsigned)(blocks - first < MAX_GRID ? blocks - first : MAX_GRID));
        SG_LAUNCH_CHECK();
    }
    return SLICEGCN_OK;
}

__host__ __device__ inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// ---- aggregation schedule -------------------------------------------------------------
// Rows are split by their number of stored entries d:
//   d <= TINY_ROW            : handled whole, up to 64 of them per wavefront, in schedule order;
//   TINY_ROW < d <= item_max : one lane-group item (the whole row);
//   d > item_max             : wavefront items of at most SEG_NNZ entries;
//   d > PART_ROW             : the row is first cut by column class
//       (8 contiguous column ranges holding equal shares of the stored entries; a row's entries of
//       one class are contiguous because columns ascend); a class piece of at most item_max
//       entries is a lane-group item, a longer one is cut into wavefront items.
// item_max is fixed per graph: ITEM_SHORT when the whole working set stays in the last-level cache
// (the kernels are then bound by instruction issue, and shorter lane-group items win), ITEM_LONG when
// the gathers go to memory (fewer, longer items keep more gathers in flight).
// Pieces of class c are executed by workgroups whose index is c modulo 8; with
// the round-robin placement of workgroups over the 8 XCDs, each XCD's L2 only ever sees its
// own class of columns of the gathered operand for the partitioned rows.  Whole-row items form
// two lists of their own (wavefront and lane-group items, in row order) that are dealt to the
// classes in fixed-size chunks, round-robin, and run behind the class's pieces.  A row with
// several items gets one partial-sum slot per item (in a workspace the caller of the aggregation
// provides) and is finished by a fix-up pass that adds the slots in order.
// Where item_max is ITEM_LONG the long rows are taken in ranges of d, longest first (LONG_BINS, bounds doubling from 2 * PART_ROW on):
// wavefronts that run at the same time have pieces of similar length, and no long piece starts when a launch is about to end (figures at
// spmm.hip's wave_items_body).  A resident graph's wavefronts take several pieces of the list in turn, which should not all be long ones.
constexpr int TINY_ROW = 4;
constexpr int ITEM_SHORT = 32;
constexpr int ITEM_LONG = 64;
constexpr int PART_ROW = 256;
constexpr int SEG_NNZ = 2048;
constexpr int N_CLASSES = 8;   // column classes, one per XCD
constexpr int LONG_BINS = 6;   // ranges of rows cut by column class
constexpr int PASS_COLS = 128; // columns per pass of the aggregation (floats per partial-sum slot)

struct Segment { // 16 bytes, read as one int4
    int32_t row;
    int32_t beg;
    int32_t end;
    int32_t dst; // >= 0: final (write the row); < 0: partial slot index -(dst+1)
};

struct FixRow { // a row whose items went to partial slots [slot_beg, slot_end)
    int32_t row;
    int32_t slot_beg;
    int32_t slot_end;
    int32_t pad;
};

// A row of at most TINY_ROW entries in 8 bytes, read as one int2: the row and where its entries begin in 31 bits each, its entries less
// one in the upper bits; a row without entries begins at NO_ENTRIES.
struct TinyRow {
    uint32_t row;
    uint32_t beg;
};
constexpr uint32_t NO_ENTRIES = 0x7fffffffu;

struct Schedule {
    int32_t item_max = ITEM_LONG; // longest lane-group item (whole row or class piece)
    Segment *items = nullptr; // per class its wavefront pieces, then its lane-group pieces; then the whole-row lists
    FixRow *fix = nullptr;
    TinyRow *tiny = nullptr;  // rows of at most TINY_ROW entries, in schedule order
    int32_t tiny_cnt = 0;
    int32_t big_off[N_CLASSES] = {0}, big_cnt[N_CLASSES] = {0};     // wavefront pieces of class c
    int32_t small_off[N_CLASSES] = {0}, small_cnt[N_CLASSES] = {0}; // lane-group pieces of class c
    int32_t wbig_off = 0, wbig_cnt = 0;     // wavefront items of rows kept whole
    int32_t wsmall_off = 0, wsmall_cnt = 0; // lane-group items that are whole rows
    bool local = false; // most rows' columns lie close together, so that gathers mostly meet in the L2s
    int64_t n_items = 0;
    int64_t n_fix = 0;
    int64_t n_slots = 0;
};

struct Csr {
    int32_t *rowptr = nullptr;
    int32_t *colidx = nullptr;
    float *vals = nullptr;
    Schedule sched;
};

} // namespace slicegcn

struct slicegcn_graph {
    int64_t n = 0;
    int64_t nnz = 0;
    int symmetric = 0;
    int device = 0;
    int32_t *deg = nullptr;
    float *dinv = nullptr;
    float *sqrtd = nullptr; // sqrt(max(d~_v, 1)) = 1 / dinv: undoes the row scaling of activations kept as D~^-1/2 H
    int32_t *order = nullptr; // order[p] = row at position p of the aggregation's schedule; NULL = natural order
    slicegcn::Csr fwd;  // A^
    slicegcn::Csr tr;   // A^^T (arrays alias fwd when the pattern is symmetric)
    std::vector<void *> owned; // device blocks to free with the handle (none where the caller's allocator made them)
};

namespace slicegcn {

// spmm.hip: Y[:, 0:width] = M X (+ Add) for each of `batch` operands (at most SPMM_BATCH, all with the same leading
// dimensions), M given by `m`.  Add may alias Y.  ws: 256-byte aligned, at least batch * spmm_workspace_bytes(m, width)
// bytes (partial sums of rows cut into several items; may be NULL when that is 0).
// prescaled: X rows carry dinv[u] already (the value stream is not read)
// sums: final sums of weight gradients that are still due, formed beside the aggregation or before it
constexpr int SPMM_BATCH = 8;
struct FinalWork; // final_sum.h
struct SpmmOperands {
    const float *X;
    float *Y;
    const float *Add; // NULL: nothing is added
};
int launch_spmm(const slicegcn_graph *g, const Csr &m, const SpmmOperands *ops, int batch, int64_t ldx, int32_t width,
                int64_t ldy, int64_t ldadd, void *ws, size_t ws_bytes, hipStream_t stream, bool prescaled = false,
                const FinalWork *sums = nullptr);
size_t spmm_workspace_bytes(const Csr &m, int32_t width, bool one_pass = false);

// dense.hip: column sums of an n x w matrix: fp32 per block of rows into ws[blocks][w], then
// out[j] = sum over blocks of ws[b][first + j] in fp64 (ws_row = floats per ws row)
int launch_colsum_partial(const float *M, int64_t ld, int64_t n, int32_t w, float *ws, hipStream_t stream);
int launch_colsum_final(const float *ws_first, int64_t n, int32_t ws_row, int32_t count, float *out, hipStream_t stream);
size_t colsum_workspace_bytes(int64_t n, int32_t w);

// misc.hip: brackets the launches of its scope with an event pair while profiling is on
struct ProfScope {
    ProfScope(int kind, int width, hipStream_t stream);
    ~ProfScope();
    ProfScope(const ProfScope &) = delete;
    ProfScope &operator=(const ProfScope &) = delete;
    int slot_;
    hipStream_t stream_;
};

// Scratch memory of a graph build, handed out from one workspace.  Passed by value to a phase, it gives back on return
// what the phase took (phases run in order on one stream).
struct Arena {
    char *base;
    size_t size, used;
    static size_t rounded(size_t bytes) { return (bytes + 255) / 256 * 256; }
    template <class T> int take(size_t bytes, T **out)
    {
        SG_REQUIRE(used + rounded(bytes) <= size, SLICEGCN_EWORKSPACE, "build_norm_csr: workspace exhausted (%zu of %zu bytes used, %zu wanted)",
                   used, size, bytes);
        *out = reinterpret_cast<T *>(base + used);
        used += rounded(bytes);
        return SLICEGCN_OK;
    }
};

// Memory that lives as long as a graph handle: from the caller's allocator, or from the device and owned by the handle.
struct Keep {
    const slicegcn_allocator *allocator;
    slicegcn_graph *g;
    template <class T> int take(size_t bytes, T **out)
    {
        if (bytes == 0) bytes = 256;
        if (allocator) {
            *out = static_cast<T *>(allocator->alloc(allocator->ctx, bytes));
            SG_REQUIRE(*out != nullptr, SLICEGCN_ENOMEM, "build_norm_csr: the caller's allocator gave no %zu bytes", bytes);
            SG_REQUIRE((reinterpret_cast<uintptr_t>(*out) & 255u) == 0, SLICEGCN_EINVAL, "build_norm_csr: allocation not 256-byte aligned");
            return SLICEGCN_OK;
        }
        void *p = nullptr;
        const hipError_t e = hipMalloc(&p, bytes);
        SG_REQUIRE(e == hipSuccess, e == hipErrorOutOfMemory ? SLICEGCN_ENOMEM : SLICEGCN_EHIP, "hipMalloc of %zu bytes failed: %s", bytes,
                   hipGetErrorString(e));
        g->owned.push_back(p);
        *out = static_cast<T *>(p);
        return SLICEGCN_OK;
    }
};

// build_csr.hip: exclusive prefix sums (in and out may not overlap) and the scratch they take
int scan_i32(const int32_t *in, int32_t *out, int64_t count, Arena &ws, hipStream_t stream);
size_t scan_bytes(int64_t count);

// edge_sort.hip: the distinct entries of a pattern, sorted in buckets of rows in the workspace, and with them the rows' numbers of entries
// (deg has room for one more element than rows; dinv and sqrtd, from deg, may be NULL) and row pointers.  n_bad is increased by the
// pairs with an id outside [0, n).  Then, with room for rowptr[n] entries, edge_sort_emit writes columns and values.
struct EdgeSort {
    const void *keys;
    int64_t max_pieces;
    bool wide;
    alignas(8) unsigned char state[256]; // pointers into the workspace, for edge_sort.hip alone
};
size_t edge_sort_bytes(int64_t n_edges, int64_t n, bool sym, bool loops);
int edge_sort_rows(const int64_t *row, const int64_t *col, int64_t n_edges, int64_t n, bool sym, bool loops, int32_t *deg, float *dinv, float *sqrtd,
                   int32_t *rowptr, int32_t *n_bad, Arena &ws, EdgeSort *out, hipStream_t stream);
int edge_sort_emit(const EdgeSort &e, const int32_t *rowptr, int32_t *colidx, float *vals, const float *dinv, hipStream_t stream);

// order.hip: order[p] = id of the row at position p (by degree, or breadth first).  counters: two device words.
int build_row_order(int64_t n, const int32_t *rowptr, const int32_t *colidx, bool breadth_first, int32_t *order, Arena ws,
                    int32_t *counters, hipStream_t stream);
size_t row_order_bytes(int64_t n); // scratch it takes

} // namespace slicegcn
