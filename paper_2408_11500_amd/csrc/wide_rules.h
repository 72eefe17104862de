// Sizes of pair_wide_kernel that are arithmetic alone: no HIP in here, so that they can be gone through on the host.
#pragma once

namespace slicegcn {

constexpr int WIDE_WAVES = 8, WIDE_WEIGHTS = 32768; // wavefronts of a workgroup; floats of its weights
constexpr int WIDE_CHUNK = 32;                      // steps of k a wavefront takes from its rows at a time
constexpr int wide_k(int nt) { return WIDE_WEIGHTS / (32 * nt) / 8 * 8; } // longest product of a workgroup with nt tiles of columns
// Groups of four k that a product of K steps has room for in LDS: those of whole chunks.  The weights of eight steps are requested while the eight before
// them are multiplied, also where a last chunk ends with those; what lies there is never used and not stored either.  (A test in the loop instead: 400 k
// rows 37 -> 70 56.9 / 58.0 us, 200 -> 200 365 / 370; zeros stored there: 169 k rows 40 -> 256 57.3 / 58.5.)
constexpr int wide_groups(int K) { return (K + WIDE_CHUNK - 1) / WIDE_CHUNK * (WIDE_CHUNK / 4); }
// Whether the eight steps behind the q-th eight of a chunk that has `left` steps to go are requested then (if not, the next strip's first)
constexpr bool wide_more(int left, int q) { return q + 1 < WIDE_CHUNK / 8 || left > WIDE_CHUNK; }

// Workgroups per XCD, of 32 CUs, along the strips of rows: a workgroup takes a CU for the launch, and `per_strip` of them (column tiles times slices) share a
// strip.  0: there is no room for one.
constexpr int WIDE_CUS = 32;
constexpr int wide_walkers(int per_strip) { return WIDE_CUS / per_strip; }
// Whether the launch is even enough for pair_wide_kernel to be faster than pair_rows_kernel, which spreads any number of tiles over the chip: CUs without a
// workgroup cost what the deeper reads give, and staging the weights wants eight strips of rows a SIMD, or twelve beside idle CUs.  Rows / wide,
// products of 256 steps, forward and input gradients, by the CUs of 32 in use:
//     30 (per_strip 10)  26.7 k rows 174 / 158, 177 / 165 us   104.9 k rows 642 / 571, 652 / 585
//     28 (14)            19.1 k 176 / 173, 174 / 182           28.1 k 252 / 239, 252 / 249 (100 steps 123 / 120, 131 / 124)   149.8 k 1263 / 1194
//     27 (9)             29.7 k 175 / 173, 175 / 183           58.3 k 326 / 319, 333 / 330 (100 steps 159 / 161, 174 / 167)
//     26 (13)            20.6 k 177 / 186, 181 / 193           80.7 k 645 / 651, 648 / 668
//     22 (11)            24.3 k 175 / 203, 174 / 216           95.3 k 640 / 762, 647 / 780
//     17 (17)            15.7 k 178 / 263, 179 / 279           61.7 k 646 / 979, 661 / 999
//     32 of 40           eight slices, input gradients 320 <- 320 of 19.7 k rows 693 / 912 (the last workgroups start when the others end)
// With 28 two tiles a workgroup lose at any length (280 k rows 448 columns out of 128 steps 0.94 to 1.01 times as fast, of 192 0.95 to 1.00).
constexpr bool wide_even(int nt, int per_strip, int K, long long strips)
{
    const int used = wide_walkers(per_strip) * per_strip;
    return used >= 30 ? strips * per_strip >= 8192 : used >= 28 && nt >= 3 && K >= 96 && strips * per_strip >= 12288;
}
// Whether products of K steps have enough to multiply, by the tiles of 32 columns a workgroup takes and the workgroups along the columns.  Short ones are bound
// by what is stored, and a row's columns come from n_col workgroups that drift apart: lines that two of them share are written in parts, and the rows
// are read n_col times.  Times as fast as pair_rows_kernel, forward and input gradients of 280 k and 900 k rows, stored in whole lines or not:
//     nt 4, n_col 1 to 4  K 8 0.89 to 1.40   16 0.93 to 1.47   24 1.00 to 1.48   33 0.97 to 1.22   64 0.98 to 1.13   128 1.03 to 1.15
//     nt 4, n_col 5 to 8  K 8 0.69 to 1.38   16 0.74 to 1.49   24 0.84 to 1.43   33 0.98 to 1.17   64 1.03 to 1.12   128 1.04 to 1.18
//     nt 3, n_col 1, 2    K 8 0.89 to 1.14   16 0.99 to 1.21   24 1.03 to 1.30   33 0.99 to 1.23   64 0.96 to 1.23   128 0.99 to 1.17
//     nt 3, n_col 3 to 6  K 8 0.68 to 1.29   16 0.83 to 1.27   24 0.92 to 1.29   33 0.88 to 1.23   64 0.92 to 1.13    96 0.98 to 1.11   128 1.02 to 1.12
//     nt 2, n_col 5       K 8 0.70 to 1.03   16 0.83 to 1.03   33 0.85 to 1.05   64 0.87 to 0.98   96 0.93 to 1.01   128 1.00 to 1.06   192 1.00 to 1.10
//     nt 2, n_col 1       K 65 0.95 to 1.17   96 0.98 to 1.20   128 1.03 to 1.22   192 1.01 to 1.15   (up to 64 a strip kernel's)
// Five chunks are read like eight (nt 2 0.92 to 1.05, nt 3 0.94 to 1.06, nt 4 1.01 to 1.14).
// `lines`: rows begin on lines of 128 bytes.  Where they do not, a product of a single chunk loses as well (1 M rows of 93 columns out of 30 steps 0.88 to 1.04,
// 786 k of 509 out of 25 0.86 to 0.94; in whole lines 24 steps 1.03 to 1.38).
constexpr bool wide_long(int nt, int n_col, int K, bool lines)
{
    if (nt == 4) return K >= (n_col <= 4 && lines ? 24 : 33);
    if ((K + WIDE_CHUNK - 1) / WIDE_CHUNK == 5) return false;
    return nt == 3 ? K >= (n_col > 2 ? 96 : lines ? 24 : 33) : K >= (n_col == 1 ? 65 : 128);
}

} // namespace slicegcn
