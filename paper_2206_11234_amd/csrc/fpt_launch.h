// fpt_launch.h -- sizes of the record and training kernels' launches, as plain functions of the work and
// of the number of compute units.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace fpt {

// Paths per wave of a replay: as few of 64, 32, 16 and 8 as leave each SIMD two waves, since a SIMD issues
// an instruction per 5 cycles for one wave and per 2.4 for two or more.
inline uint32_t record_slots(uint64_t n_paths, int cus) {
    uint32_t slots = 64;
    while (slots > 8 && (n_paths + slots / 2 - 1) / (slots / 2) <= 8ull * cus) slots /= 2;
    return slots;
}

// Waves per workgroup of a replay: one while the waves fit the SIMDs once, else one for each SIMD of a CU.
inline uint32_t record_waves_per_group(uint64_t waves, int cus) { return waves <= 4ull * cus ? 1 : 4; }

// Workgroups of the evaluation, 256 records each at a time: those that share the CUs (three waves per SIMD).
constexpr int EVAL_WG_PER_CU = 3;
inline uint32_t eval_groups(uint64_t n_rec, int cus) {
    return static_cast<uint32_t>(std::min<uint64_t>((n_rec + 255) / 256, static_cast<uint64_t>(EVAL_WG_PER_CU) * cus));
}

// The evaluation's results are kept for a piece of the records at a time, whole paths of at most
// EVAL_PIECE records together or one longer path: the end of the piece that starts at path i (off: the
// paths' first records and, last, their number).  The array is 4 B a record beside the records' 16, which
// pieces keep to 64 MiB.
constexpr uint64_t EVAL_PIECE = 1ull << 24;
inline int64_t eval_piece_end(const uint64_t *off, int64_t n_paths, int64_t i, uint64_t piece = EVAL_PIECE) {
    return std::max<int64_t>(i + 1, std::upper_bound(off + i + 1, off + n_paths + 1, off[i] + piece) - off - 1);
}

// Records that the array of one call's evaluation has to hold.
inline uint64_t eval_capacity(const uint64_t *off, int64_t n_paths, uint64_t piece = EVAL_PIECE) {
    uint64_t most = 0;
    for (int64_t i = 0, j; i < n_paths; i = j) {
        j = eval_piece_end(off, n_paths, i, piece);
        most = std::max(most, off[j] - off[i]);
    }
    return most;
}

// Workgroups of the record check, 256 records each at a time: a CU's 2048 threads.  (A launch holds fewer
// than 2^32 threads; a call may hold more records.)
inline uint32_t check_groups(uint64_t n_rec, int cus) {
    return static_cast<uint32_t>(std::min<uint64_t>((n_rec + 255) / 256, 8ull * cus));
}

}  // namespace fpt
