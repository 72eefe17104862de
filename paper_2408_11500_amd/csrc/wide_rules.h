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

} // namespace slicegcn
