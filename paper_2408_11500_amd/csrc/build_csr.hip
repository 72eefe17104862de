// Normalised-adjacency builder: edge pairs -> canonical CSR of A^ = D~^-1/2 (A + I) D~^-1/2
// (the normalisation 1/c_vu of the paper's GCN layer equation), plus the row schedule the
// aggregation kernels use.  Integer work only, apart from one rsqrt per node and one multiply
// per stored entry.
//
//   entries   edge_sort.hip: edges distributed to buckets of rows, sorted there in registers, repeats dropped, rows counted;
//   schedule  rows sorted into the item lists by ballot; only rows that are cut by column class
//             need per-row tables.
//
// What bounds a build beside the sort is the host: device allocations and synchronisations.  All scratch
// memory is one workspace and the handle's arrays are at most five blocks, both from the caller if it has an
// allocator of its own; the stream is synchronised only where a size has to be known.
#include "common.h"
#include "slicegcn_native.h"

#include <rocprim/rocprim.hpp>

#include <cstdlib>
#include <new>

namespace slicegcn {

namespace {

constexpr int TPB = 256;
inline unsigned blocks_for(int64_t n) { return (unsigned)((n + TPB - 1) / TPB); }

// Device words the host reads back: [0] out-of-range edges, [1] those the transposed pattern's sort counts again, [2] ... the schedule's and the row order's.
constexpr int N_COUNTERS = 64;

// ---- schedule ---------------------------------------------------------------------------
// Column class c holds the columns [first[c], first[c+1]); the boundaries are the eighth-quantiles of the stored
// entries per column, so that the classes carry equal numbers of entries whatever the vertex numbering (with hubs
// numbered first, equal column ranges would put almost half of the entries into the first class).
struct ClassBounds {
    int32_t first[N_CLASSES + 1];
};

// colptr: row pointer of the transposed pattern (entries per column, scanned)
__device__ inline int32_t class_bound(const int32_t *__restrict__ colptr, int64_t n, int c)
{
    if (c == 0) return 0;
    if (c == N_CLASSES) return (int32_t)n;
    const int64_t target = (int64_t)colptr[n] * c / N_CLASSES;
    int64_t lo = 0, hi = n; // smallest column j with colptr[j] >= target
    while (lo < hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        if (colptr[mid] < target) lo = mid + 1; else hi = mid;
    }
    return (int32_t)lo;
}

// Kinds of rows (see common.h): whole rows make one item each, long ones (ranges of their length, the longest first) are cut by
// column class, tiny ones are listed.
constexpr int ROW_WAVE = 0, ROW_GROUP = 1, ROW_LONG = 2, ROW_TINY = ROW_LONG + LONG_BINS, ROW_KINDS = ROW_TINY + 1;
// Kinds that are counted: those of the ranges in use.  The tiny rows are the others (with all kinds in the scan of the counts, 270 k nodes took a second
// launch for it, 750 us a build instead of 742).
inline __host__ __device__ int counted_kinds(int32_t item_max) { return ROW_LONG + (item_max > ITEM_SHORT ? LONG_BINS : 1); }
__device__ inline int row_kind(int32_t d, int32_t item_max)
{
    if (d <= TINY_ROW) return ROW_TINY;
    if (d <= PART_ROW) return d <= item_max ? ROW_GROUP : ROW_WAVE;
    int range = 0; // doublings of 2 * PART_ROW below d
    if (item_max > ITEM_SHORT) {
#pragma unroll
        for (int b = 1; b < LONG_BINS; ++b) range += d > PART_ROW << b;
    }
    return counted_kinds(item_max) - 1 - range;
}

// Thread p handles the row at position p of the schedule (order[p], or p itself in natural order), so that the items
// come out in schedule order.  FILL = false: rows of every kind per workgroup, counts[kind * n_groups + workgroup];
// FILL = true, with the scan of those counts: the items of the whole rows (wavefront items, then lane-group items) and the list of the
// tiny rows, and the list of the long rows, whichever is asked for.
template <bool FILL>
__global__ __launch_bounds__(256) void sched_rows_kernel(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ order,
                                                         int64_t n, int32_t item_max, int32_t *__restrict__ counts, int64_t n_groups,
                                                         Segment *__restrict__ items, TinyRow *__restrict__ tiny, int32_t *__restrict__ long_rows)
{
    __shared__ int32_t per_wave[4][ROW_KINDS];
    __shared__ int32_t before[ROW_TINY]; // rows of every counted kind among the workgroups before
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t p = (int64_t)blockIdx.x * TPB + threadIdx.x;
    int kind = -1;
    int32_t row = 0, beg = 0, end = 0;
    if (p < n) {
        row = order ? order[p] : (int32_t)p;
        beg = rowptr[row];
        end = rowptr[row + 1];
        kind = row_kind(end - beg, item_max);
    }
    int32_t rank = 0;
    const int counted = counted_kinds(item_max);
    // (all kinds at once: one after the other by every thread that needs them, 1.9 M nodes, 7.7 M edges 14.5 instead of 10.9 us)
    if (FILL && tiny && threadIdx.x < counted) before[threadIdx.x] = counts[threadIdx.x * n_groups + blockIdx.x] - counts[threadIdx.x * n_groups];
#pragma unroll
    for (int k = 0; k < ROW_KINDS; ++k) {
        if (k >= counted && k < ROW_TINY) continue; // uniform
        const unsigned long long bits = __ballot(kind == k);
        if (kind == k) rank = __popcll(bits & ((1ull << lane) - 1ull));
        if (lane == 0) per_wave[wave][k] = __popcll(bits);
    }
    __syncthreads();
    if (!FILL) {
        if (threadIdx.x < counted)
            counts[threadIdx.x * n_groups + blockIdx.x] = per_wave[0][threadIdx.x] + per_wave[1][threadIdx.x] +
                                                          per_wave[2][threadIdx.x] + per_wave[3][threadIdx.x];
        return;
    }
    if (kind < 0) return;
    for (int w = 0; w < wave; ++w) rank += per_wave[w][kind];
    if (kind == ROW_TINY) {
        if (!tiny) return;
        int32_t at = (int32_t)blockIdx.x * TPB + rank; // the rows before this one, less those of the other kinds among the workgroups before
        for (int k = 0; k < counted; ++k) at -= before[k];
        const uint32_t more = end > beg ? (uint32_t)(end - beg - 1) : 0u;
        TinyRow r;
        r.row = (uint32_t)row | more << 31;
        r.beg = (end > beg ? (uint32_t)beg : NO_ENTRIES) | more >> 1 << 31;
        tiny[at] = r;
        return;
    }
    const int32_t at = counts[kind * n_groups + blockIdx.x] + rank; // the scan ran over the kinds back to back
    if (kind >= ROW_LONG) {
        if (long_rows) long_rows[at - counts[ROW_LONG * n_groups]] = row;
    } else if (items) {
        Segment sg;
        sg.row = row; sg.beg = beg; sg.end = end; sg.dst = row;
        items[at] = sg;
    }
}

// Counters for the host: rows of every kind, and how many more of SAMPLES rows have all of their columns (but for the diagonal, beside two or more)
// within a LOCAL_SPAN-th of the nodes than have not (one row per thread beside the wavefront that searches the boundaries, which takes longer); the column class boundaries
// stay on the device.
constexpr int SAMPLES = 960, LOCAL_SPAN = 16;
__global__ __launch_bounds__(SAMPLES + 64) void sched_summary_kernel(const int32_t *__restrict__ counts, int64_t n_groups, int counted, const int32_t *__restrict__ colptr, int64_t n,
                                                           const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
                                                           int32_t *__restrict__ summary, ClassBounds *__restrict__ cb)
{
    const int t = threadIdx.x;
    bool near = false, far = false;
    if (t < counted) summary[t] = counts[(t + 1) * n_groups] - counts[t * n_groups];
    if (t <= N_CLASSES) {
        cb->first[t] = class_bound(colptr, n, t);
    } else if (t >= 64) {
        const int64_t row = n * (t - 64) / SAMPLES;
        const int32_t beg = rowptr[row], end = rowptr[row + 1];
        if (end - beg >= 2) {
            const int more = end - beg > 2 ? 1 : 0, first = colidx[beg], last = colidx[end - 1];
            const int lo = first == row ? colidx[beg + more] : first, hi = last == row ? colidx[end - 1 - more] : last;
            near = (int64_t)(hi - lo) * LOCAL_SPAN <= n;
            far = !near;
        }
    }
    const int excess = __syncthreads_count(near) - __syncthreads_count(far);
    if (t == counted) summary[t] = excess;
}

// ---- long rows: cut by column class ------------------------------------------------------
// Tables: 2c = wavefront pieces of class c, 2c + 1 = lane-group pieces of class c, then partial-sum slots and rows with
// several items.  cnt[table * (n_long + 1) + i] for the i-th long row.
constexpr int T_SLOT = 2 * N_CLASSES, T_FIX = T_SLOT + 1, N_TABLES = T_FIX + 1;

__device__ inline int pieces_of(int32_t len) { return (len + SEG_NNZ - 1) / SEG_NNZ; }

// The entries of the classes of long row i, one lane per class (eight lanes per row): [beg, end) of this lane's class.  Per row: the entries
// of column class c are [lower_bound(first[c]), lower_bound(first[c+1])); every lane searches its own start and takes its end from the
// next lane.  The searches read most lines of a row (126 M entries, 98 k long rows: 80 us), so they are done once and the starts kept in
// class_beg for the second kernel.
struct ClassPiece { int32_t row, beg, end; };
template <bool SEARCH>
__device__ inline ClassPiece class_piece(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx, const int32_t *__restrict__ long_rows,
                                         int64_t i, int64_t n_long, const ClassBounds &cb, int c, int32_t *__restrict__ class_beg)
{
    ClassPiece p{0, 0, 0};
    if (i < n_long) {
        p.row = long_rows[i];
        p.end = rowptr[p.row + 1];
        if (SEARCH) {
            p.beg = rowptr[p.row];
            if (c > 0) {
                int32_t hi = p.end;
                const int32_t target = cb.first[c];
                while (p.beg < hi) {
                    const int32_t mid = p.beg + ((hi - p.beg) >> 1);
                    if (colidx[mid] < target) p.beg = mid + 1; else hi = mid;
                }
            }
            class_beg[i * N_CLASSES + c] = p.beg;
        } else {
            p.beg = class_beg[i * N_CLASSES + c];
        }
    }
    const int32_t next = __shfl_down(p.beg, 1, 64);
    if (c + 1 < N_CLASSES) p.end = next;
    return p;
}
// items of a class piece, and whether they are wavefront items
__device__ inline int items_of(int32_t len, int32_t item_max) { return len <= 0 ? 0 : len <= item_max ? 1 : pieces_of(len); }
constexpr int LONG_PER_BLOCK = TPB / N_CLASSES; // rows per workgroup

__global__ __launch_bounds__(TPB) void long_count_kernel(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
                                                         const int32_t *__restrict__ long_rows, int64_t n_long, const ClassBounds *__restrict__ cb,
                                                         int32_t item_max, int32_t *__restrict__ class_beg, int32_t *__restrict__ cnt)
{
    const int64_t i = (int64_t)blockIdx.x * LONG_PER_BLOCK + threadIdx.x / N_CLASSES;
    const int c = threadIdx.x % N_CLASSES;
    const ClassPiece p = class_piece<true>(rowptr, colidx, long_rows, i, n_long, *cb, c, class_beg);
    const int mine = items_of(p.end - p.beg, item_max);
    int total = mine;
#pragma unroll
    for (int s = 1; s < N_CLASSES; s <<= 1) total += __shfl_xor(total, s, 64);
    if (i > n_long) return; // row n_long: the zeros the scan's totals come from
    const int64_t stride = n_long + 1;
    const bool wide = p.end - p.beg > item_max;
    cnt[(2 * c) * stride + i] = wide ? mine : 0;
    cnt[(2 * c + 1) * stride + i] = wide ? 0 : mine;
    if (c == 0) {
        cnt[T_SLOT * stride + i] = total > 1 ? total : 0;
        cnt[T_FIX * stride + i] = total > 1 ? 1 : 0;
    }
}

// starts[t] = first element of table t in the scan over all tables, starts[N_TABLES] = the total
__global__ void long_starts_kernel(const int32_t *__restrict__ off, const int32_t *__restrict__ cnt, int64_t stride, int32_t *__restrict__ starts)
{
    const int t = threadIdx.x;
    if (t < N_TABLES) starts[t] = off[t * stride];
    if (t == N_TABLES) starts[t] = off[N_TABLES * stride - 1] + cnt[N_TABLES * stride - 1];
}

// items of the long rows: slots are handed out in (class, piece) order, a table's pieces of a row are adjacent
__global__ __launch_bounds__(TPB) void long_fill_kernel(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
                                                        const int32_t *__restrict__ long_rows, int64_t n_long, const ClassBounds *__restrict__ cb,
                                                        int32_t item_max, int32_t *__restrict__ class_beg, const int32_t *__restrict__ off, Segment *__restrict__ items, FixRow *__restrict__ fix)
{
    const int64_t i = (int64_t)blockIdx.x * LONG_PER_BLOCK + threadIdx.x / N_CLASSES;
    const int c = threadIdx.x % N_CLASSES;
    const ClassPiece p = class_piece<false>(rowptr, colidx, long_rows, i, n_long, *cb, c, class_beg);
    const int32_t len = p.end - p.beg;
    const int mine = items_of(len, item_max);
    int before = mine; // items of this row up to this class
#pragma unroll
    for (int s = 1; s < N_CLASSES; s <<= 1) {
        const int up = __shfl_up(before, s, N_CLASSES);
        if (c >= s) before += up;
    }
    before -= mine;
    if (i >= n_long) return;
    const int64_t stride = n_long + 1;
    const int32_t *slots = off + T_SLOT * stride, *fixes = off + T_FIX * stride;
    const int32_t slot0 = slots[i] - slots[0], n_slots = slots[i + 1] - slots[i];
    const int table = len > item_max ? 2 * c : 2 * c + 1;
    const int32_t piece = mine > 0 ? (len + mine - 1) / mine : 0; // equal cuts, the last one takes the remainder
    for (int j = 0; j < mine; ++j) {
        Segment sg;
        sg.row = p.row;
        sg.beg = p.beg + j * piece;
        sg.end = min(p.end, p.beg + (j + 1) * piece);
        sg.dst = n_slots == 0 ? p.row : -(slot0 + before + j + 1);
        items[off[table * stride + i] + j] = sg;
    }
    if (n_slots > 0 && c == 0) {
        FixRow f;
        f.row = p.row;
        f.slot_beg = slot0;
        f.slot_end = slot0 + n_slots;
        f.pad = 0;
        fix[fixes[i] - fixes[0]] = f;
    }
}

} // namespace

int scan_i32(const int32_t *in, int32_t *out, int64_t count, Arena &ws, hipStream_t stream)
{
    size_t bytes = 0;
    SG_HIP(rocprim::exclusive_scan(nullptr, bytes, in, out, (int32_t)0, (size_t)count, rocprim::plus<int32_t>(), stream));
    const size_t mark = ws.used;
    void *tmp = nullptr;
    if (int rc = ws.take(bytes, &tmp)) return rc;
    SG_HIP(rocprim::exclusive_scan(tmp, bytes, in, out, (int32_t)0, (size_t)count, rocprim::plus<int32_t>(), stream));
    ws.used = mark; // later users are ordered behind the scan on the stream
    return SLICEGCN_OK;
}
size_t scan_bytes(int64_t count)
{
    size_t bytes = 0;
    (void)rocprim::exclusive_scan(nullptr, bytes, (const int32_t *)nullptr, (int32_t *)nullptr, (int32_t)0, (size_t)count, rocprim::plus<int32_t>(), (hipStream_t)0);
    return Arena::rounded(bytes);
}

namespace {

// ---- host side ---------------------------------------------------------------------------
int64_t candidates(int64_t n_edges, int64_t n, uint32_t flags) // entries the pattern can have
{
    return n_edges * ((flags & SLICEGCN_SYMMETRIZE) ? 2 : 1) + ((flags & SLICEGCN_ADD_SELF_LOOPS) ? n : 0);
}

size_t sched_bytes(int64_t n, int64_t n_keys)
{
    const int64_t groups = ROW_TINY * (int64_t)blocks_for(n) + 1, n_long = n_keys / PART_ROW < n ? n_keys / PART_ROW : n;
    const int64_t tables = N_TABLES * (n_long + 1);
    const size_t a = scan_bytes(groups), b = scan_bytes(tables);
    return 2 * Arena::rounded((size_t)groups * 4) + Arena::rounded((size_t)n_long * 4) + Arena::rounded((size_t)n_long * N_CLASSES * 4) + 2 * Arena::rounded((size_t)tables * 4) +
           Arena::rounded(sizeof(ClassBounds)) + (a > b ? a : b);
}

int read_counters(const int32_t *from, int32_t *to, int count, hipStream_t stream)
{
    SG_HIP(hipMemcpyAsync(to, from, (size_t)count * sizeof(int32_t), hipMemcpyDeviceToHost, stream));
    SG_HIP(hipStreamSynchronize(stream));
    return SLICEGCN_OK;
}

// colptr: row pointer of the transposed pattern.  counters: at least N_TABLES + 1 device words.
int build_schedule(slicegcn_graph *g, const Csr &m, const int32_t *colptr, uint32_t flags, Keep &keep, Arena ws, int32_t *counters,
                   Schedule &out, hipStream_t stream)
{
    const int64_t n = g->n, nnz = g->nnz;
    out = Schedule();
    // entries (8 bytes each) plus one 128-byte operand row per node against the 256 MB last-level cache
    const bool resident = nnz * 8 + n * 128 <= ((int64_t)256 << 20);
    int32_t item_max = resident ? ITEM_SHORT : ITEM_LONG;
    if (flags & SLICEGCN_SCHED_SHORT_ITEMS) item_max = ITEM_SHORT;
    if (flags & SLICEGCN_SCHED_LONG_ITEMS) item_max = ITEM_LONG;
    out.item_max = item_max;
    const int64_t n_groups = blocks_for(n);
    const int counted = counted_kinds(item_max);
    int32_t *counts = nullptr, *offs = nullptr;
    ClassBounds *cb = nullptr;
    if (int rc = ws.take((size_t)(counted * n_groups + 1) * 4, &counts)) return rc;
    if (int rc = ws.take((size_t)(counted * n_groups + 1) * 4, &offs)) return rc;
    if (int rc = ws.take(sizeof(ClassBounds), &cb)) return rc;
    sched_rows_kernel<false><<<(unsigned)n_groups, TPB, 0, stream>>>(m.rowptr, g->order, n, item_max, counts, n_groups, nullptr, nullptr, nullptr);
    SG_LAUNCH_CHECK();
    if (int rc = scan_i32(counts, offs, counted * n_groups + 1, ws, stream)) return rc; // the last element is only written
    sched_summary_kernel<<<1, SAMPLES + 64, 0, stream>>>(offs, n_groups, counted, colptr, n, m.rowptr, m.colidx, counters, cb);
    SG_LAUNCH_CHECK();
    int32_t kinds[ROW_KINDS];
    if (int rc = read_counters(counters, kinds, counted + 1, stream)) return rc;
    out.local = kinds[counted] > 0;
    const int64_t n_group = kinds[ROW_GROUP], n_wave = kinds[ROW_WAVE];
    int64_t n_long = 0;
    for (int k = ROW_LONG; k < counted; ++k) n_long += kinds[k];
    out.tiny_cnt = (int32_t)(n - n_wave - n_group - n_long);

    int32_t *long_rows = nullptr, *class_beg = nullptr, *cnt = nullptr, *off = nullptr;
    int32_t starts[N_TABLES + 1] = {0};
    const int64_t stride = n_long + 1;
    if (n_long > 0) {
        if (int rc = ws.take((size_t)n_long * 4, &long_rows)) return rc;
        if (int rc = ws.take((size_t)n_long * N_CLASSES * 4, &class_beg)) return rc;
        if (int rc = ws.take((size_t)(N_TABLES * stride) * 4, &cnt)) return rc;
        if (int rc = ws.take((size_t)(N_TABLES * stride) * 4, &off)) return rc;
        sched_rows_kernel<true><<<(unsigned)n_groups, TPB, 0, stream>>>(m.rowptr, g->order, n, item_max, offs, n_groups, nullptr, nullptr, long_rows);
        SG_LAUNCH_CHECK();
        long_count_kernel<<<blocks_for(stride * N_CLASSES), TPB, 0, stream>>>(m.rowptr, m.colidx, long_rows, n_long, cb, item_max, class_beg, cnt);
        SG_LAUNCH_CHECK();
        if (int rc = scan_i32(cnt, off, N_TABLES * stride, ws, stream)) return rc;
        long_starts_kernel<<<1, 64, 0, stream>>>(off, cnt, stride, counters);
        SG_LAUNCH_CHECK();
        if (int rc = read_counters(counters, starts, N_TABLES + 1, stream)) return rc;
    }
    // items: whole rows (wavefront, lane-group), then per class its wavefront and its lane-group pieces
    out.wbig_off = 0;
    out.wbig_cnt = (int32_t)n_wave;
    out.wsmall_off = (int32_t)n_wave;
    out.wsmall_cnt = (int32_t)n_group;
    const int32_t base = (int32_t)(n_wave + n_group);
    for (int c = 0; c < N_CLASSES; ++c) {
        out.big_off[c] = base + starts[2 * c];
        out.big_cnt[c] = starts[2 * c + 1] - starts[2 * c];
        out.small_off[c] = base + starts[2 * c + 1];
        out.small_cnt[c] = starts[2 * c + 2] - starts[2 * c + 1];
    }
    out.n_items = base + starts[T_SLOT];
    out.n_slots = starts[T_FIX] - starts[T_SLOT];
    out.n_fix = starts[N_TABLES] - starts[T_FIX];
    const size_t item_bytes = Arena::rounded((size_t)out.n_items * sizeof(Segment)), fix_bytes = Arena::rounded((size_t)out.n_fix * sizeof(FixRow));
    char *block = nullptr;
    if (int rc = keep.take(item_bytes + fix_bytes + (size_t)out.tiny_cnt * sizeof(TinyRow), &block)) return rc;
    out.items = reinterpret_cast<Segment *>(block);
    out.fix = reinterpret_cast<FixRow *>(block + item_bytes);
    out.tiny = reinterpret_cast<TinyRow *>(block + item_bytes + fix_bytes);
    if (base > 0 || out.tiny_cnt > 0) {
        sched_rows_kernel<true><<<(unsigned)n_groups, TPB, 0, stream>>>(m.rowptr, g->order, n, item_max, offs, n_groups, out.items, out.tiny, nullptr);
        SG_LAUNCH_CHECK();
    }
    if (n_long > 0) {
        long_fill_kernel<<<blocks_for(n_long * N_CLASSES), TPB, 0, stream>>>(m.rowptr, m.colidx, long_rows, n_long, cb, item_max, class_beg, off,
                                                                out.items + base, out.fix);
        SG_LAUNCH_CHECK();
    }
    static const bool verbose = getenv("SLICEGCN_VERBOSE") != nullptr;
    if (verbose) {
        fprintf(stderr, "[slicegcn] schedule: whole rows %d wavefront + %d lane-group items, %lld rows with several items, "
                        "%lld partial-sum slots\n", out.wbig_cnt, out.wsmall_cnt, (long long)out.n_fix, (long long)out.n_slots);
        for (int c = 0; c < N_CLASSES; ++c)
            fprintf(stderr, "[slicegcn]   class %d: %d wavefront + %d lane-group pieces\n", c, out.big_cnt[c], out.small_cnt[c]);
    }
    return SLICEGCN_OK;
}

// Column indices and values of a pattern whose rows have been counted; allocates both.
int csr_entries(const EdgeSort &sorted, const slicegcn_graph *g, Csr &m, Keep &keep, hipStream_t stream)
{
    const size_t col_bytes = Arena::rounded((size_t)g->nnz * 4);
    char *block = nullptr;
    if (int rc = keep.take(2 * col_bytes, &block)) return rc;
    m.colidx = reinterpret_cast<int32_t *>(block);
    m.vals = reinterpret_cast<float *>(block + col_bytes);
    return g->nnz > 0 ? edge_sort_emit(sorted, m.rowptr, m.colidx, m.vals, g->dinv, stream) : SLICEGCN_OK;
}

int build_from_edges(const int64_t *src, const int64_t *dst, int64_t n_edges, uint32_t flags, slicegcn_graph *g, Keep &keep, Arena ws, hipStream_t stream)
{
    const int64_t n = g->n;
    const bool sym = (flags & SLICEGCN_SYMMETRIZE) != 0, loops = (flags & SLICEGCN_ADD_SELF_LOOPS) != 0;
    int32_t *counters = nullptr;
    if (int rc = ws.take(N_COUNTERS * sizeof(int32_t), &counters)) return rc;
    {
        // rowptr (both directions of a directed pattern), degrees (one element more than rows) and their roots, row order: one block
        const size_t a = Arena::rounded((size_t)(n + 1) * 4), b = Arena::rounded((size_t)n * 4);
        const bool ordered = (flags & (SLICEGCN_REORDER_DEGREE | SLICEGCN_REORDER_BFS)) != 0;
        char *block = nullptr;
        if (int rc = keep.take(a + (sym ? 1 : 2) * a + (ordered ? 3 : 2) * b, &block)) return rc;
        g->deg = reinterpret_cast<int32_t *>(block);
        g->dinv = reinterpret_cast<float *>(block + a);
        g->sqrtd = reinterpret_cast<float *>(block + a + b);
        g->fwd.rowptr = reinterpret_cast<int32_t *>(block + a + 2 * b);
        if (!sym) g->tr.rowptr = reinterpret_cast<int32_t *>(block + 2 * a + 2 * b);
        if (ordered) g->order = reinterpret_cast<int32_t *>(block + (sym ? 2 : 3) * a + 2 * b);
    }
    SG_HIP(hipMemsetAsync(counters, 0, N_COUNTERS * sizeof(int32_t), stream));
    {
        Arena phase = ws;
        EdgeSort sorted;
        if (int rc = edge_sort_rows(src, dst, n_edges, n, sym, loops, g->deg, g->dinv, g->sqrtd, g->fwd.rowptr, counters, phase, &sorted, stream)) return rc;
        int32_t bad = 0, nnz = 0;
        SG_HIP(hipMemcpyAsync(&bad, counters, sizeof(int32_t), hipMemcpyDeviceToHost, stream));
        SG_HIP(hipMemcpyAsync(&nnz, g->fwd.rowptr + n, sizeof(int32_t), hipMemcpyDeviceToHost, stream));
        SG_HIP(hipStreamSynchronize(stream));
        SG_REQUIRE(bad == 0, SLICEGCN_ERANGE, "build_norm_csr: %d edge(s) name a node outside [0, %lld)", bad, (long long)n);
        g->nnz = nnz;
        if (int rc = csr_entries(sorted, g, g->fwd, keep, stream)) return rc;
    }
    if (g->order)
        if (int rc = build_row_order(n, g->fwd.rowptr, g->fwd.colidx, (flags & SLICEGCN_REORDER_BFS) != 0, g->order, ws, counters + 2, stream)) return rc;

    if (sym) {
        if (int rc = build_schedule(g, g->fwd, g->fwd.rowptr, flags, keep, ws, counters + 2, g->fwd.sched, stream)) return rc;
        g->tr = g->fwd; // A^ is symmetric: the same arrays serve the transposed product
    } else {
        Arena phase = ws;
        EdgeSort sorted;
        int32_t *in_deg = nullptr; // entries of the transposed pattern's rows; its values use the degrees of the pattern itself
        if (int rc = phase.take((size_t)(n + 1) * 4, &in_deg)) return rc;
        if (int rc = edge_sort_rows(dst, src, n_edges, n, false, loops, in_deg, nullptr, nullptr, g->tr.rowptr, counters + 1, phase, &sorted, stream)) return rc;
        if (int rc = csr_entries(sorted, g, g->tr, keep, stream)) return rc;
        if (int rc = build_schedule(g, g->fwd, g->tr.rowptr, flags, keep, ws, counters + 2, g->fwd.sched, stream)) return rc;
        if (int rc = build_schedule(g, g->tr, g->fwd.rowptr, flags, keep, ws, counters + 2, g->tr.sched, stream)) return rc;
    }
    SG_HIP(hipStreamSynchronize(stream));
    return SLICEGCN_OK;
}

size_t build_bytes(int64_t n_edges, int64_t n, uint32_t flags)
{
    const bool sym = (flags & SLICEGCN_SYMMETRIZE) != 0;
    size_t most = edge_sort_bytes(n_edges, n, sym, (flags & SLICEGCN_ADD_SELF_LOOPS) != 0) + (sym ? 0 : Arena::rounded((size_t)(n + 1) * 4));
    const size_t sched = sched_bytes(n, candidates(n_edges, n, flags));
    if (sched > most) most = sched;
    if (flags & (SLICEGCN_REORDER_DEGREE | SLICEGCN_REORDER_BFS)) {
        const size_t order = row_order_bytes(n);
        if (order > most) most = order;
    }
    return Arena::rounded(N_COUNTERS * sizeof(int32_t)) + most;
}

// Checks of what is to be built, for both entry points and the workspace query
int check_sizes(int64_t n_edges, int64_t n_nodes, uint32_t flags)
{
    SG_REQUIRE(n_nodes >= 1, SLICEGCN_EINVAL, "build_norm_csr: n_nodes = %lld < 1", (long long)n_nodes);
    SG_REQUIRE(n_edges >= 0, SLICEGCN_EINVAL, "build_norm_csr: n_edges = %lld < 0", (long long)n_edges);
    SG_REQUIRE((flags & ~(SLICEGCN_SYMMETRIZE | SLICEGCN_ADD_SELF_LOOPS | SLICEGCN_REORDER_DEGREE | SLICEGCN_REORDER_BFS |
                          SLICEGCN_SCHED_SHORT_ITEMS | SLICEGCN_SCHED_LONG_ITEMS)) == 0,
               SLICEGCN_EINVAL, "build_norm_csr: unknown flag bits 0x%x", flags);
    SG_REQUIRE(!((flags & SLICEGCN_REORDER_DEGREE) && (flags & SLICEGCN_REORDER_BFS)), SLICEGCN_EINVAL,
               "build_norm_csr: REORDER_DEGREE and REORDER_BFS exclude each other");
    SG_REQUIRE(!((flags & SLICEGCN_SCHED_SHORT_ITEMS) && (flags & SLICEGCN_SCHED_LONG_ITEMS)), SLICEGCN_EINVAL,
               "build_norm_csr: SCHED_SHORT_ITEMS and SCHED_LONG_ITEMS exclude each other");
    SG_REQUIRE(n_nodes <= INT32_MAX, SLICEGCN_ERANGE, "build_norm_csr: n_nodes exceeds int32");
    SG_REQUIRE(n_edges <= (int64_t)INT32_MAX, SLICEGCN_ERANGE, "build_norm_csr: n_edges exceeds int32");
    const int64_t n_keys = candidates(n_edges, n_nodes, flags);
    SG_REQUIRE(n_keys <= (int64_t)INT32_MAX, SLICEGCN_ERANGE,
               "build_norm_csr: %lld candidate entries exceed int32 indexing", (long long)n_keys);
    return SLICEGCN_OK;
}
int check_build(const int64_t *src, const int64_t *dst, int64_t n_edges, int64_t n_nodes, uint32_t flags, slicegcn_graph **out)
{
    SG_REQUIRE(out != nullptr, SLICEGCN_EINVAL, "build_norm_csr: out is NULL");
    *out = nullptr;
    SG_REQUIRE(n_edges <= 0 || (src && dst), SLICEGCN_EINVAL, "build_norm_csr: NULL edge arrays");
    return check_sizes(n_edges, n_nodes, flags);
}

} // namespace

} // namespace slicegcn

using namespace slicegcn;

extern "C" size_t slicegcn_build_workspace_bytes(int64_t n_edges, int64_t n_nodes, uint32_t flags)
{
    if (check_sizes(n_edges, n_nodes, flags)) return 0;
    return build_bytes(n_edges, n_nodes, flags);
}

extern "C" int slicegcn_build_norm_csr_with(const int64_t *src, const int64_t *dst, int64_t n_edges, int64_t n_nodes, uint32_t flags,
                                            const slicegcn_allocator *allocator, void *ws, size_t ws_bytes, void *stream_,
                                            slicegcn_graph **out)
{
    if (int rc = check_build(src, dst, n_edges, n_nodes, flags, out)) return rc;
    SG_REQUIRE(allocator == nullptr || allocator->alloc != nullptr, SLICEGCN_EINVAL, "build_norm_csr: allocator without a function");
    SG_REQUIRE((reinterpret_cast<uintptr_t>(ws) & 255u) == 0, SLICEGCN_EINVAL, "build_norm_csr: workspace not 256-byte aligned");
    const size_t need = build_bytes(n_edges, n_nodes, flags);
    SG_REQUIRE(ws == nullptr || ws_bytes >= need, SLICEGCN_EWORKSPACE, "build_norm_csr: workspace of %zu bytes, %zu needed", ws_bytes, need);
    hipStream_t stream = as_stream(stream_);

    slicegcn_graph *g = new (std::nothrow) slicegcn_graph();
    SG_REQUIRE(g != nullptr, SLICEGCN_ENOMEM, "build_norm_csr: host allocation failed");
    struct Guard { // destroys the half-built handle on any early return
        slicegcn_graph *g;
        void *own_ws;
        ~Guard() { (void)hipFree(own_ws); if (g) slicegcn_graph_destroy(g); }
    } guard{g, nullptr};
    g->n = n_nodes;
    g->symmetric = (flags & SLICEGCN_SYMMETRIZE) != 0;
    SG_HIP(hipGetDevice(&g->device));
    if (ws == nullptr) {
        const hipError_t e = hipMalloc(&guard.own_ws, need);
        SG_REQUIRE(e == hipSuccess, e == hipErrorOutOfMemory ? SLICEGCN_ENOMEM : SLICEGCN_EHIP, "hipMalloc of %zu bytes failed: %s", need,
                   hipGetErrorString(e));
        ws = guard.own_ws;
        ws_bytes = need;
    }
    Arena arena{static_cast<char *>(ws), ws_bytes, 0};
    Keep keep{allocator, g};
    const int rc = build_from_edges(src, dst, n_edges, flags, g, keep, arena, stream);
    if (rc) {
        (void)hipStreamSynchronize(stream); // nothing may still use the memory given back below
        return rc;
    }
    guard.g = nullptr;
    *out = g;
    return SLICEGCN_OK;
}

extern "C" int slicegcn_build_norm_csr(const int64_t *src, const int64_t *dst, int64_t n_edges,
                                       int64_t n_nodes, uint32_t flags, void *stream, slicegcn_graph **out)
{
    return slicegcn_build_norm_csr_with(src, dst, n_edges, n_nodes, flags, nullptr, nullptr, 0, stream, out);
}

extern "C" int slicegcn_graph_view(const slicegcn_graph *g, slicegcn_csr_view *view)
{
    SG_REQUIRE(g && view, SLICEGCN_EINVAL, "graph_view: NULL argument");
    view->n_nodes = g->n;
    view->nnz = g->nnz;
    view->rowptr = g->fwd.rowptr;
    view->colidx = g->fwd.colidx;
    view->deg = g->deg;
    view->dinv = g->dinv;
    view->vals = g->fwd.vals;
    view->symmetric = g->symmetric;
    view->order = g->order;
    return SLICEGCN_OK;
}

extern "C" int slicegcn_graph_destroy(slicegcn_graph *g)
{
    if (!g) return SLICEGCN_OK;
    for (void *p : g->owned) (void)hipFree(p);
    delete g;
    return SLICEGCN_OK;
}
