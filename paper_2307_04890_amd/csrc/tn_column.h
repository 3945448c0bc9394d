// The row-OR stream of networks whose word columns fit in LDS (Sec. 3.1
// Algorithm 1 in reverse time, Sec. 3.4), and of many such networks in one
// launch (the hashed proxies, Sec. 4.3).
#pragma once

#include "tn_internal.h"

namespace tn {

// The column form of an op schedule: ops in level order as {a | b << 16,
// d1 | d2 << 16}, their rows in the column (the real rows, then the scratch
// rows in use; d2 = d1 where there is no second target), in blocks of 64.
// kColumnFlag is set in the first word of the last op of each level, and in the
// second word of op i < 32 of a block where bit i of the level of the block's
// first op is.  Ops that pad the last block act on the row past the scratch rows.
constexpr uint32_t kColumnRow = 0x7fffu;
constexpr uint32_t kColumnFlag = 0x80000000u;
// One network of a launch (persist nullable: the layout of
// launch_rowor_global's with one-word slices).
struct ColumnNet {
    const uint2 *ops;  // device
    uint32_t blocks, levels;
    uint64_t *C;
    int64_t ld;
    uint32_t *persist;
};
// Whether n real rows, scratch_rows in use and the padding's row fit.
inline bool rowor_column_fits(uint32_t n, uint32_t scratch_rows) {
    return (uint64_t)n + scratch_rows < kColumnRows;
}
// ... in a column of half words: ids of 15 bits, and 127 rows a lane of 256 (the
// counters of the sizes).
inline bool rowor_half_column_fits(uint32_t n, uint32_t scratch_rows) {
    return n <= 127 * 256 && (uint64_t)n + scratch_rows <= kColumnRow;
}
// Rounds of word columns, one a compute unit, that cover n nodes: a launch takes
// about as long for each whatever its ops, as it reads or writes all of C.
inline uint32_t rowor_column_rounds(uint32_t n) { return ((n + 63) / 64 + 255) / 256; }
// Whether a stream whose first batch's largest chunk has so many events takes
// one-word slices, so that chunks may run on word columns.  A second round of
// columns only pays for larger chunks, and small ones take less on slices of two
// words, a round of them (us an insert, activity-driven, 19,000 nodes, two-word
// slices, one-word slices and columns: 1 event 37, 30, 113; 600 83, 135, 110;
// 1,500 110, 182, 110; 2,000 126, 196, 118; 4,000 154, 254, 127).
inline bool rowor_column_stream(uint32_t n, int64_t events) {
    return rowor_column_rounds(n) == 1 || 12 * events >= (int64_t)n;
}
// Whether a chunk of so many events of such a stream runs on word columns: fewer
// touch so few rows that slices in memory take less (us on two-word slices,
// one-word slices and columns: 10,000 nodes, 1 event 49, 56, 57, 100 53, 68, 54;
// 12,000 nodes, 100 events 39, 41, 53, 200 58, 69, 54; 16,000 nodes 48, 44, 66 and
// 59, 66, 66; 20,400 nodes 54, 51, 121, 300 69, 97, 120, 600 85, 138, 115).
inline bool rowor_column_chunk(uint32_t n, int64_t events) {
    return n <= 10240 || (rowor_column_rounds(n) == 1 ? 80 : 48) * events >= (int64_t)n;
}
// Whether a plan of so many ops runs on word columns where only its matrix is asked
// for: of fewer, slices in memory after an identity written by whole lines take
// less (us on slices and columns, activity-driven: 3,000 nodes, no ops 7 and 7,
// 30 ops 24 and 7; 8,000, none 7 and 14, 80 ops 20 and 15; 9,500, 19 ops 18 and 21,
// 95 ops 21 and 21; 12,000, none 8 and 25, 120 ops 26 and 26; 16,000, 160 ops 29
// and 32, 800 64 and 34; 20,000, none 10 and 48, 200 ops 31 and 50, 1,000 64 and
// 49).  Without saturation the slices forward rows from op to op and keep no
// bitmaps, so the line lies higher (5,000 nodes, 10 ops 11 and 10; 6,000, 30 ops 11
// and 12, 120 ops 13 and 13, 325 ops 22 and 13; 8,000, 80 ops 15 and 15, on slices
// of two words from 8,065 nodes on 10,000, 20 ops 12 and 20, 310 ops 19 and 21,
// 525 ops 29 and 22; 16,000, 330 ops 30 and 33, 485 ops 38 and 33; 20,000, 1,000
// uniform ops 44 and 49, 2,045 ops 64 and 58).  With the sizes, which come with the
// columns, columns are always faster or as fast (20,000 nodes, 200 ops 73 and 67).
inline bool rowor_column_plan(uint32_t n, int64_t ops, bool saturation) {
    if (n <= 4096) return true;
    if (saturation && n <= 10240) return ops > 0 && (n <= 9216 || 128 * ops >= (int64_t)n);
    if (n <= 5120) return ops > 0;
    const int64_t line = (int64_t)n * rowor_column_rounds(n);
    return (saturation || n <= 8064 ? 64 : 32) * ops >= line;
}
// The column form of s (s.column not empty, or no ops): blocks and levels set.
inline ColumnNet column_net(const HostSchedule &s) {
    ColumnNet net{};
    net.blocks = (uint32_t)(s.column.size() / 128);
    net.levels = s.Lops;
    return net;
}
// Component sizes with a launch from the identity (either nullable): out-sizes
// are added to out, which is 0 before, in-sizes written to in.
struct ColumnSizes {
    int32_t *out = nullptr;
    int32_t *in = nullptr;
};
// One network.  It loads and stores C once, keeps persist when given, and
// counts those loads and stores in traffic (nullable); with saturation a
// column stops once every real row of it is all ones.  fresh: C starts as the
// identity, written here with its row padding, and the traffic counters are
// set, not added to, and half columns will do.  scratch_rows: those in use.
// sizes: with fresh.
hipError_t launch_rowor_column(const ColumnNet &net, uint32_t n, uint32_t scratch_rows,
                               unsigned long long *traffic, bool saturation, bool fresh,
                               unsigned int *done_count, hipStream_t st,
                               const ColumnSizes &sizes = {});
// Many networks of n nodes (nets: DEVICE array), scratch rows in use up to
// max_scratch_rows in every one; blocks, levels: theirs together.  fresh: every
// matrix starts as the identity.
hipError_t launch_rowor_columns(const ColumnNet *nets, uint32_t count, uint32_t n,
                                uint32_t max_scratch_rows, int64_t blocks, int64_t levels,
                                bool saturation, bool fresh, unsigned int *done_count, hipStream_t st);

// Word columns of networks of any sizes: workgroup b runs column tiles[b].y of
// nets[tiles[b].x] (DEVICE arrays) from the identity; rows: the most that n
// real and the scratch rows in use of one of them take.
struct ColumnTileNet {
    ColumnNet net;
    uint32_t n, nwords;
};
hipError_t launch_rowor_column_tiles(const ColumnTileNet *nets, const uint2 *tiles, uint32_t count,
                                     uint32_t rows, uint32_t threads, bool saturation,
                                     hipStream_t st);

}  // namespace tn
