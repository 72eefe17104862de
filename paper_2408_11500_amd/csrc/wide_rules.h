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
constexpr bool wide_even(int per_strip, long long strips)
{
    const int used = wide_walkers(per_strip) * per_strip;
    return used >= 30 ? strips * per_strip >= 8192 : used >= 28 && strips * per_strip >= 12288;
}

} // namespace slicegcn
