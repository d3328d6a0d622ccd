// Rules of dispatch that need nothing but sizes: plain host functions.
#pragma once
#include <algorithm>
#include <cstddef>

namespace ead {

constexpr int kEntMaxChunks = 64;                       // most pieces a row of logits is cut into

// The split of a row into work items depends on (rows, V) alone, so a step's result does not depend on
// how many steps share a launch, nor on which entry point asked for it.  Long chunks (up to 8 vectors
// per thread) amortise the per-workgroup merge; shorter ones only when the rows of one step would
// otherwise give too few workgroups to fill the chip.
inline void entropy_split(int rows, int V, int *chunks_out, int *per_out) {
    const int nvec = V / 8;
    int chunks = std::max(1, (nvec + 2047) / 2048);
    while ((long)chunks * rows < 512 && chunks < kEntMaxChunks && nvec / (chunks * 2) >= 256) chunks *= 2;
    int per = (std::max(nvec, 1) + chunks - 1) / chunks;
    while (per > 8 * 256) { ++chunks; per = (nvec + chunks - 1) / chunks; }
    *chunks_out = chunks; *per_out = per;
}

// Whether ead_entropy_argmax merges a row's chunks in the launch that computes them.  The call is bound by the host where a
// second launch is saved (10.3 -> 7.5 us), as long as the chain behind a row's last chunk stays hidden: its chunks
// arrive one after another at a word of their row, and rows share the words' cache lines, so the time grows about
// as rows x chunks^2 (us in one launch against two: 4 chunks x 128 rows 8.1 / 10.4, 8 x 64 9.2 / 10.2, 16 x 16 9.0 / 10.3, 40 x 3
// 8.9 / 10.3, 64 x 1 7.7 / 10.4; but 16 x 24 11.1 / 10.2, 40 x 6 11.8 / 10.3, 40 x 13 14.8 / 10.6, 64 x 4 12.1 / 10.3).  A workgroup that takes one item
// after another waits for the chain each time (2000 rows of one chunk: 16.8 / 15.2; 800: 10.4 / 10.4).  Above 4 MB the kernel
// itself is the longer part.
inline bool entropy_folds(int rows, int chunks, size_t bytes) {
    return bytes <= ((size_t)4 << 20) && (long)rows * chunks <= 600 && (long)rows * chunks * chunks <= 4800;
}

// Pieces a row is given to workgroups in by k_entropy_rows (1: a workgroup takes whole rows, 2048 vectors at a time), by rows
// and vocabulary alone, so that a step's result does not depend on how many steps share a launch.  One or two rows of
// more than three times 2048 vectors: eight pieces (more where 2048 vectors ask for it), which keep 16 steps of two rows
// at about one workgroup per compute unit
// (2 rows x 151936: one step 19.5 -> 9.9 us, 64 steps 90 -> 58; 37 pieces: 10.4 and 105).  Shorter rows are through
// before a piece's partial and counter are (1 x 32000: whole 7.3 and 45 us, in pieces 9.6 and 50).  From more rows on the pieces'
// merges cost more over 16 steps than the fuller chip gives (8 rows x 151936, 40 steps: 75 whole, 132 in pieces).
inline int entropy_row_parts(int rows, int V) {
    const int nvec = V / 8, least = (nvec + 2047) / 2048;         // at most 8 vectors per thread and piece
    return rows > 2 || nvec <= 3 * 2048 ? 1 : std::max(least, 8);
}

}  // namespace ead
