// The level loop of kernels that hold one column of every row in LDS, a
// workgroup each (word columns, HyperLogLog registers).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace tn {

constexpr uint32_t kLevelDepth = 8;  // blocks a wavefront has requested ahead

// The ops of one block as its wavefront holds them.
struct LevelOps {
    uint32_t a, b, d1, d2;  // the lane's op: rows a and b merge into d1 and d2
    uint64_t ends;          // lanes that end a level
    uint32_t l0;            // level of the block's first op
};

// Runs `blocks` blocks of 64 ops in level order (every level has ops) on the
// first `turn` wavefronts: block j is a turn of wavefront j % turn.  The ops of
// one level within a block act together, then a barrier ends the level; a block
// names its first level, so a wavefront needs no level starts and only counts
// barriers until then.  While the rows of a block's first level are read, the
// wavefront unpacks its next block and requests another.
//
// unpack: a lane's op, as stored, to LevelOps (wavefront-uniform ends and l0).
//
// With sat, rows are at rest once full(row), and the stream ends when all n
// are: every 32 levels each of the wavefronts moves past the rows of its own
// that are (levels 32 k look, 32 k + 1 read *open, LDS and 0 at first, 32 k + 2
// clear it: other wavefronts of the workgroup end by the same rule).
//
// There is one barrier before the first level, one after each.  The whole loop
// is uniform within a wavefront, the ops of a level apart, and tests at its
// bottom (else the compiler waits for the writes before the next block's
// reads).  Measured on word columns: a divergent check cost 15 to 25 %,
// unpacking after the writes 15 %, 4 blocks ahead 25 %.
template <typename V, typename T, class Unpack, class Merge, class Full>
__device__ __forceinline__ void run_levels(T *rows, const uint2 *__restrict__ ops, uint32_t blocks,
                                           uint32_t levels, uint32_t turn, uint32_t n, bool sat,
                                           uint32_t *open, Unpack unpack, Merge merge, Full full) {
    const uint32_t lane = threadIdx.x & 63u, last = blocks - 1;
    // the load of a block is unconditional, so that the wait before its
    // use counts the blocks after it (past the last block none is used)
    auto load = [&](uint32_t j) { return ops[64 * (size_t)min(j, last) + lane]; };
    const uint32_t j0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // the wavefront
    uint32_t j = j0;
    uint2 win[kLevelDepth];
#pragma unroll
    for (uint32_t k = 0; k < kLevelDepth; ++k) win[k] = load(j + k * turn);
    __syncthreads();
    uint32_t l = 0, row = 64 * j0;
    uint64_t rest = 0;                // lanes of the block whose ops are still to act
    uint32_t look = sat ? 32u : ~0u;  // the next level with a part of the check
    // ends the level; the stream's end leaves no blocks and no lanes
    auto advance = [&] {
        __syncthreads();
        ++l;
        if (__builtin_expect(l != look, 1)) return;
        bool stop = false;
        if ((l & 31u) == 0) {
            while (row < n && __all(row + lane >= n || full((V)rows[row + lane]))) row += 64 * turn;
            if (row < n) *open = 1;
            ++look;
        } else if ((l & 31u) == 1) {
            stop = __builtin_amdgcn_readfirstlane(*open) == 0;
            ++look;
        } else {
            if (j0 == 0) *open = 0;
            look += 30;
        }
        if (stop) {
            l = levels;
            blocks = 0;
            rest = 0;
        }
    };
    LevelOps cur = unpack(win[0]);
    V ra, rb;  // the rows read
    auto act = [&] {
        // the lanes up to the next end
        const uint64_t in = (cur.ends ^ (cur.ends - 1)) & rest;
        const V r = merge(ra, rb);
        asm volatile("" : : "v"(r));
        if (__builtin_amdgcn_inverse_ballot_w64(in)) {
            rows[cur.d1] = (T)r;
            rows[cur.d2] = (T)r;
        }
        rest ^= in;
        asm volatile("" : "+s"(rest));
    };
    for (;; j += kLevelDepth * turn) {
        bool more = true;
#pragma unroll
        for (uint32_t k = 0; k < kLevelDepth; ++k) {
            if (j + k * turn >= blocks) {
                more = false;
                break;
            }
            rest = ~0ull;
            while (l < cur.l0) advance();
            ra = rows[cur.a];
            rb = rows[cur.b];
            // the next block's ops, while the rows are read
            const LevelOps next = unpack(win[(k + 1) % kLevelDepth]);
            win[k] = load(j + (k + kLevelDepth) * turn);
            asm volatile("" : : "v"(next.a), "v"(next.b), "v"(next.d1), "v"(next.d2),
                         "s"(next.ends), "s"(next.l0));
            act();
            while (rest) {
                cur.ends &= cur.ends - 1;
                advance();
                ra = rows[cur.a];
                rb = rows[cur.b];
                act();
            }
            cur = next;
        }
        if (!more) break;
    }
    while (l < levels) advance();  // the other wavefronts' levels
}

}  // namespace tn
