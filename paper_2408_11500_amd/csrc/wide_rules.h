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
// (one shape each; over drawn ones, times as fast as pair_rows_kernel, geometric mean: 32 of 32 1.13 to 1.20, 30 1.03 to 1.16, 28 1.01 to 1.06, 27 1.04).
constexpr bool wide_even(int per_strip, long long strips) { return wide_walkers(per_strip) * per_strip >= 27 && strips * per_strip >= 8192; }
// Whether products of K steps have enough to multiply, by the tiles of 32 columns a workgroup takes, the workgroups along the columns, whether rows begin on lines
// of 128 bytes (`lines`) and whether activation bits are read or written (`bits`).  Short ones are bound by what is stored, and a row's columns come from n_col
// workgroups that drift apart: lines that two of them share are written in parts.  Times as fast as pair_rows_kernel, geometric mean (and the
// tenth from below) of 2700 drawn products of 30 k to 1.2 M rows, forward and input gradients, into the same memory (results in memory of their own differ by up
// to a fifth with the place alone):
//     K         nt 4, lines             nt 4                    nt 3, lines             nt 3                    nt 2
//     4 to 7    0.98 (bits 1.08)        0.86 (0.94)             0.97 (1.01)             0.92 (0.99)             0.87 (0.88 to 0.95)
//     8 to 15   1.04 (1.11)             0.95 (1.01)             1.03 (1.05)             0.94 (1.02)             0.90 (0.90 to 0.96)
//     16 to 23  1.15 (1.20)             1.02 (1.08)             1.06 (1.12)             1.10 (1.11)             0.95 to 0.97
//     24 to 31  1.11 to 1.25            1.09 to 1.19            1.08 to 1.22            1.12 to 1.21            1.08
//     33 to 64  1.16 to 1.33 (least tenth 0.98 to 1.23)         1.13 to 1.32 (1.02 to 1.24)                     1.06 (0.92)
//     65 to 128 1.15 to 1.23 (1.05 to 1.13)                     1.11 to 1.23 (1.01 to 1.13)                     1.06 to 1.21 (0.98 to 1.13)
//     to 160, five chunks, read like eight  1.09 to 1.13        1.04 to 1.11                                    1.00 to 1.01 (0.94)
//     above     1.13 to 1.21                                    1.10 to 1.18                                    1.08 to 1.15
// In lines up to 15 steps forward products with five workgroups or more along the columns 0.92 to 0.98.  The two input gradients of a slice layer (`two`), of which
// pair_rows_kernel loads dH_out once: 8 to 15 steps, not in lines, whole backward passes 1.02 to 1.06, up to 7 1.01 to 1.03.
constexpr bool wide_long(int nt, int n_col, int K, bool lines, bool bits, bool two)
{
    return nt == 2 ? K >= 24 : two || K >= 16 || (lines && n_col <= 4 && K >= (bits ? 4 : 8));
}

} // namespace slicegcn
