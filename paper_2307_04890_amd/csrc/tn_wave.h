// The row-OR stream of small networks on one wavefront per word column
// (Sec. 3.1 Algorithm 1 in reverse time, Sec. 3.4), and of many such
// networks in one launch (the hashed proxies, Sec. 4.3).
#pragma once

#include "tn_internal.h"

namespace tn {

// Small networks: the row-OR stream of one-word slices with the column in
// LDS, one wavefront per word column and no barrier (k_rowor_wave_flat), for
// n real plus scratch rows in kRoworWaveLds bytes.  It loads and stores C
// once and keeps persist (as launch_rowor_global's with one-word slices)
// when given; traffic counts those loads and stores.  With saturation a
// column stops once every real row of it is all ones.
constexpr size_t kRoworWaveLds = 64 * 1024;
bool rowor_wave_fits(uint32_t n, uint32_t scratch_rows);
// Levels average more than this many ops: a wavefront takes too many turns,
// one workgroup per column is faster (both sides at rowor_column_pays).
constexpr int64_t kRoworWaveWideOps = 80;
bool rowor_wave_wide(int64_t ops, int64_t levels);
// fits and is not wide
bool rowor_wave_pays(uint32_t n, uint32_t scratch_rows, int64_t ops, int64_t levels);
// One network of a launch on word columns (many of them: the hashed proxies):
// its op schedule, its matrix (n rows of ld words) and its per-column state
// (nullable; the layout of launch_rowor_global's with one-word slices).
struct WaveNet {
    DevOps s;
    uint64_t *C;
    int64_t ld;
    uint32_t *persist;
};

// Flat schedules of many networks (k_rowor_wave_flat): ops in level order
// as {a, b, d1, d2} LDS byte offsets of the rows in a column (n real rows,
// then the scratch rows; kFlatNone for no second target), with kFlatEnd set
// in a on the last op of each level.  The DevOps of a WaveNet then holds
// only ops and nops.
constexpr uint32_t kFlatEnd = 0x80000000u;
constexpr uint32_t kFlatOffMask = 0x7fffffffu;
constexpr uint32_t kFlatNone = 0xffffffffu;
// Writes the flat form of schedule s of a network of n nodes to out
// (4 uint32 per op, flat_ops_bytes(s) bytes).
size_t flat_ops_bytes(const HostSchedule &s);
void flat_ops_pack(const HostSchedule &s, uint32_t n, uint32_t *out);
// count networks of n nodes each, one wavefront per word column of each;
// nets: DEVICE array; scratch rows up to max_scratch_rows in every network.
// traffic (nullable) counts the row words loaded and stored.
hipError_t launch_rowor_wave_flat(const WaveNet *nets, uint32_t count, uint32_t n,
                                  uint32_t max_scratch_rows, bool saturation,
                                  unsigned int *done_count, unsigned long long *traffic,
                                  hipStream_t st);
// One network (a resident plan): flat_ops a DEVICE array of nops flat ops;
// no per-column state; traffic nullable.
hipError_t launch_rowor_wave_flat1(const uint32_t *flat_ops, uint32_t nops, uint32_t n,
                                   uint64_t *C, int64_t ld, uint32_t scratch_rows,
                                   unsigned long long *traffic, bool saturation, hipStream_t st);

// Networks whose word columns (n real and the scratch rows) fit in LDS: one
// workgroup per column, a barrier per level (tn_column.hip).
bool rowor_column_fits(uint32_t n, uint32_t scratch_rows);
// ... and whether that is the way to run one.  Where no wavefront's column
// fits, always (activity-driven events on 10^4 nodes, 54 ops a level: 519 us,
// on slices of C in memory 2809), save that without saturation those slices
// run and count every op.  Elsewhere where levels are wide: a barrier costs
// more than a wavefront's next level, more wavefronts take fewer turns (us on
// wavefronts and here; 10^3 nodes, 15 ops a level: 226, 281; 39: 16, 15; 93:
// 269, 178; 119: 39, 18; 3 * 10^3 nodes, 19: 350, 431; 281: 393, 146).
bool rowor_column_pays(uint32_t n, uint32_t scratch_rows, int64_t ops, int64_t levels,
                       bool saturation);
// It loads and stores C once and keeps persist as launch_rowor_wave_flat does.
// fresh: C starts as the identity, written here with its row padding, and the
// traffic counters are set, not added to.
hipError_t launch_rowor_column(const DevOps &s, uint32_t n, uint64_t *C, int64_t ld,
                               uint32_t scratch_rows, unsigned long long *traffic, bool saturation,
                               bool fresh, uint32_t *persist, unsigned int *done_count,
                               hipStream_t st);
// Many networks, as launch_rowor_wave_flat (their ops not in the flat form).
hipError_t launch_rowor_columns(const WaveNet *nets, uint32_t count, uint32_t n,
                                uint32_t max_scratch_rows, bool saturation, unsigned int *done_count, hipStream_t st);

}  // namespace tn
