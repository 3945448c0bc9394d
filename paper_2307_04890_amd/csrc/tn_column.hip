// gfx950 kernels of the row-OR stream of networks whose word columns fit in
// LDS: one workgroup per word column keeps the column of every row in LDS
// and runs the levels with a barrier each (Sec. 3.1 Algorithm 1 in reverse
// time, Sec. 3.4; each word column evolves on its own).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "tn_device.h"
#include "tn_column.h"
#include "tn_levels.h"

namespace tn {

namespace {

// Stores the column as rowor_column does, adds each row's popcount to the row's
// out-size, and writes the column popcounts of its nodes (their in-sizes): a
// lane's rows enter bit-sliced counters (7 planes: at most 127 rows a lane),
// which six exchanges between lanes turn into one count a lane.  The column is
// given up.  Execution and sizes take 13.9 us at 1,000 nodes (10.3 without the
// sizes), 163 at 10,007 (153), 713 at 20,000 (679).  (A byte of popcount a row and
// word column, summed by a second kernel, took 705 at 20,000, but n^2 / 64 bytes of
// the context's, which executions on several streams and captured ones would
// share.)
template <typename T>
__device__ __forceinline__ void column_sizes(const ColumnNet &net, uint32_t w, uint32_t n,
                                             const ColumnSizes &sizes) {
    constexpr uint32_t kBits = 8 * sizeof(T);
    extern __shared__ uint64_t column[];
    const T *const rows = reinterpret_cast<const T *>(column);
    T *const C = reinterpret_cast<T *>(net.C);
    const size_t ld = (size_t)net.ld * (64 / kBits);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, W = blockDim.x;
    uint64_t c[7] = {};
    for (uint32_t r0 = tid; r0 < n; r0 += 4 * W) {
        uint64_t x[4], t[2], u;
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t r = r0 + k * W;
            x[k] = r < n ? rows[r] : 0ull;
            if (r < n) {
                C[(size_t)r * ld + w] = (T)x[k];
                if (sizes.out && x[k]) atomicAdd(sizes.out + r, (int32_t)__popcll(x[k]));
            }
        }
        full_add(c[0], x[0], x[1], c[0], t[0]);
        full_add(c[0], x[2], x[3], c[0], t[1]);
        full_add(c[1], t[0], t[1], c[1], u);
#pragma unroll
        for (int i = 2; i < 7; ++i) {
            const uint64_t v = c[i] & u;
            c[i] ^= u;
            u = v;
        }
    }
    if (!sizes.in) return;
    // halves of the bits go to halves of the lanes, planes added: bit `lane`
    // stays (bits past it are other lanes' and of no account)
    uint32_t p[13] = {};
#pragma unroll
    for (int i = 0; i < 7; ++i) p[i] = (uint32_t)(lane & 32u ? c[i] >> 32 : c[i]);
    {
        uint32_t carry = 0;
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            const uint32_t other = (uint32_t)(lane & 32u ? c[i] : c[i] >> 32);
            const uint32_t y = (uint32_t)__shfl_xor((int)other, 32, 64);
            const uint32_t s = p[i] ^ y ^ carry;
            carry = (p[i] & y) | (carry & (p[i] | y));
            p[i] = s;
        }
        p[7] = carry;
    }
#pragma unroll
    for (int step = 1; step < 6; ++step) {
        const uint32_t half = 32u >> step;
        const bool hi = lane & half;
        uint32_t carry = 0;
#pragma unroll
        for (int i = 0; i < 7 + step; ++i) {
            const uint32_t keep = hi ? p[i] >> half : p[i], send = hi ? p[i] : p[i] >> half;
            const uint32_t y = (uint32_t)__shfl_xor((int)send, (int)half, 64);
            p[i] = keep ^ y ^ carry;
            carry = (keep & y) | (carry & (keep | y));
        }
        p[7 + step] = carry;
    }
    int32_t v = 0;
#pragma unroll
    for (int i = 0; i < 13; ++i) v |= (int32_t)(p[i] & 1u) << i;
    // the wavefronts' counts add up where the first rows were
    int32_t *const count = reinterpret_cast<int32_t *>(column);
    __syncthreads();
    if (tid < 64) count[tid] = 0;
    __syncthreads();
    atomicAdd(&count[lane], v);
    __syncthreads();
    if (tid < kBits && kBits * w + tid < n) sizes.in[kBits * w + tid] = count[tid];
}

// Word column w of one network (n real rows, then the scratch rows and the
// row of padding ops, in LDS).
//
// With sat the column stops once every real row is all ones: rows only gain
// bits.
//
// FRESH: the column starts as the identity's and the row padding is written
// too, so that no launch has to write the matrix before.
//
// Bound by the latency of a level (LDS reads, writes, the barrier; 144 ns) where
// levels are narrow, by LDS bank conflicts where they are wide (700 ops: 340 ns).
// Events, nodes, ops a level: activity-driven, 500, 9: 125 us (250 on a
// wavefront with an LDS ring of 16-byte ops), 10^4, 55: 275 (3270 on slices of C
// in memory); random, 16,000, 699: 391 (6140 so); uniform, 1,000, 119: 16.  16
// hashed proxies of 4096 nodes in one launch: 218 us, 1032 on wavefronts.
//
// T: a word, or half a word, where a column of words does not fit (from the
// identity only, and no state is kept).  Twice the columns, of half the LDS
// traffic each: where both fit, words are as fast or faster (us, words and
// halves: activity-driven, 20,000 nodes, 10 events a node, 698 and 699; uniform, 20
// a node, 304 and 313; random, 10,007 nodes, 300,007 one-way events, 155 and 197),
// and past that halves save the slices in memory (activity-driven, 10
// events a node, 25,000 nodes: 2017 and 1446; uniform, 5, 31,000: 1139 and 428).
template <bool FRESH, bool SIZES = false, typename T = uint64_t>
__device__ __forceinline__ void
rowor_column(const ColumnNet &net, uint32_t w, uint32_t n, uint32_t nwords, bool sat,
             unsigned int *__restrict__ done_count, const ColumnSizes &sizes = {},
             unsigned long long *__restrict__ traffic = nullptr) {
    constexpr uint32_t kBits = 8 * sizeof(T);
    extern __shared__ uint64_t column[];
    T *const rows = reinterpret_cast<T *>(column);
    __shared__ uint32_t open, total;
    T *const C = reinterpret_cast<T *>(net.C);
    const int64_t ld = net.ld * (64 / kBits);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, W = blockDim.x;
    const uint32_t rwords = (n + 31) / 32, tail = n % kBits;
    const T fullw = (w + 1 < nwords || tail == 0) ? (T)~(T)0 : (T)(((T)1 << tail) - 1);
    uint32_t *pst = net.persist ? net.persist + (size_t)w * (2 * (size_t)rwords + 2) : nullptr;
    if (!FRESH && net.blocks == 0) return;  // C is left as it is
    if (pst && pst[0]) return;              // all ones already (uniform)
    if (traffic && tid < 2) atomicAdd(traffic + tid, (unsigned long long)n);
    if (tid == 0) open = total = 0;
    if (FRESH) {
        for (uint32_t r = tid; r < n; r += W) rows[r] = r / kBits == w ? (T)1 << (r % kBits) : (T)0;
    } else {
        for (uint32_t r0 = tid; r0 < n; r0 += 8 * W) {  // eight loads in flight
            T x[8];
#pragma unroll
            for (uint32_t k = 0; k < 8; ++k) x[k] = C[(size_t)min(r0 + k * W, n - 1) * ld + w];
#pragma unroll
            for (uint32_t k = 0; k < 8; ++k)
                if (r0 + k * W < n) rows[r0 + k * W] = x[k];
        }
    }
    if (net.blocks) {
        run_levels<T>(
            rows, net.ops, net.blocks, net.levels, W / 64, n, sat, &open,
            [](const uint2 &o) {
                return LevelOps{o.x & kColumnRow, (o.x >> 16) & kColumnRow, o.y & kColumnRow,
                                (o.y >> 16) & kColumnRow, __ballot((int32_t)o.x < 0),
                                (uint32_t)__ballot((int32_t)o.y < 0)};
            },
            [](T x, T y) { return x | y; },
            [=](T v) { return v == fullw; });
    }
    __syncthreads();
    if constexpr (SIZES) column_sizes<T>(net, w, n, sizes);
    else
        for (uint32_t r = tid; r < n; r += W) C[(size_t)r * ld + w] = rows[r];
    if (FRESH)
        for (int64_t p = (int64_t)nwords + w; p < ld; p += nwords)
            for (uint32_t r = tid; r < n; r += W) C[(size_t)r * ld + p] = (T)0;
    if (kBits != 64 || !pst) return;
    // the slice state, as the other kernels of the stream keep it
    uint32_t nfull = 0;
    for (uint32_t k = tid & ~63u; k < n; k += W) {
        const uint64_t v = k + lane < n ? rows[k + lane] : 0ull;
        const uint64_t fb = __ballot(k + lane < n && v == fullw), nz = __ballot(v != 0);
        if (lane < 2 && k / 32 + lane < rwords) {
            pst[2 + k / 32 + lane] = (uint32_t)(fb >> (32 * lane));
            pst[2 + rwords + k / 32 + lane] = (uint32_t)(nz >> (32 * lane));
        }
        if (lane == 0) nfull += __popcll(fb);
    }
    if (nfull) atomicAdd(&total, nfull);
    __syncthreads();
    if (tid == 0) {
        pst[1] = total;
        if (total == n) {
            pst[0] = 1u;
            atomicAdd(done_count, 1u);
        }
    }
}

// One network, one workgroup per word column.  traffic (nullable): the row
// words loaded and stored, written here where FRESH (each word once, as if the
// identity were read), else those of the columns not done before added.
template <bool FRESH, bool SIZES, typename T>
__global__ void __launch_bounds__(1024)
k_rowor_column(ColumnNet net, uint32_t n, uint32_t nwords, bool sat,
               unsigned int *__restrict__ done_count, unsigned long long *__restrict__ traffic,
               ColumnSizes sizes) {
    if (FRESH && traffic && blockIdx.x == 0 && threadIdx.x < 2)
        traffic[threadIdx.x] = net.blocks ? (unsigned long long)n * ((n + 63) / 64) : 0ull;
    rowor_column<FRESH, SIZES, T>(net, xcd_slice(blockIdx.x, gridDim.x), n, nwords, sat,
                                  done_count, sizes, FRESH ? nullptr : traffic);
}

// Many networks of n nodes (the hashed proxies): workgroup b runs word column
// b % nwords of network b / nwords.
template <bool FRESH>
__global__ void __launch_bounds__(1024)
k_rowor_columns(const ColumnNet *__restrict__ nets, uint32_t n, uint32_t nwords, bool sat,
                unsigned int *__restrict__ done_count) {
    const uint32_t b = xcd_slice(blockIdx.x, gridDim.x);
    rowor_column<FRESH>(nets[b / nwords], b % nwords, n, nwords, sat, done_count);
}

// Columns of networks of any sizes (a batch): workgroup b runs tiles[b].
__global__ void __launch_bounds__(1024)
k_rowor_column_tiles(const ColumnTileNet *__restrict__ nets, const uint2 *__restrict__ tiles,
                     bool sat) {
    const uint2 tile = tiles[blockIdx.x];
    const ColumnTileNet &t = nets[tile.x];
    rowor_column<true>(t.net, tile.y, t.n, t.nwords, sat, nullptr);
}

// (256 bytes at least: column_sizes' counts)
size_t column_lds(uint32_t n, uint32_t scratch_rows, size_t row_bytes = 8) {
    return std::max<size_t>(((size_t)n + scratch_rows + 1) * row_bytes, 256);
}

// Threads of a workgroup, from the ops of a level on average: enough
// wavefronts for a level's blocks, no more, as each takes part in every barrier
// (us with 256, 512 and 1024: 55 ops a level 275, 282, 296; 92: 320, 318, 334;
// 286: 146, 116, 118; 593: 308, 233, 202; 699: 609, 422, 391).
uint32_t column_threads(int64_t ops, int64_t levels) {
    return ops > 400 * levels ? 1024u : ops > 90 * levels ? 512u : 256u;
}

}  // namespace

hipError_t launch_rowor_column(const ColumnNet &net, uint32_t n, uint32_t scratch_rows,
                               unsigned long long *traffic, bool saturation, bool fresh,
                               unsigned int *done_count, hipStream_t st, const ColumnSizes &sizes) {
    if (!fresh && net.blocks == 0) return hipSuccess;
    const bool half = !rowor_column_fits(n, scratch_rows);
    if (half && (!fresh || net.persist || !rowor_half_column_fits(n, scratch_rows)))
        return hipErrorInvalidValue;
    const size_t lds = column_lds(n, scratch_rows, half ? 4 : 8);
    const uint32_t threads = column_threads(64 * (int64_t)net.blocks, net.levels);
    const bool sized = sizes.out || sizes.in;
    auto k = half        ? (sized ? k_rowor_column<true, true, uint32_t>
                                  : k_rowor_column<true, false, uint32_t>)
             : sized     ? k_rowor_column<true, true, uint64_t>
             : fresh     ? k_rowor_column<true, false, uint64_t>
                         : k_rowor_column<false, false, uint64_t>;
    hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
    const uint32_t nwords = half ? (n + 31) / 32 : (n + 63) / 64;
    hipLaunchKernelGGL(k, dim3(nwords), dim3(threads), lds, st, net, n, nwords, saturation,
                       done_count, traffic, sizes);
    return hipGetLastError();
}

hipError_t launch_rowor_columns(const ColumnNet *nets, uint32_t count, uint32_t n,
                                uint32_t max_scratch_rows, int64_t blocks, int64_t levels,
                                bool saturation, bool fresh, unsigned int *done_count, hipStream_t st) {
    if (count == 0) return hipSuccess;
    if (!rowor_column_fits(n, max_scratch_rows)) return hipErrorInvalidValue;
    const size_t lds = column_lds(n, max_scratch_rows);
    const uint32_t threads = column_threads(64 * blocks, levels);
    auto k = fresh ? k_rowor_columns<true> : k_rowor_columns<false>;
    hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
    const uint32_t nwords = (n + 63) / 64;
    hipLaunchKernelGGL(k, dim3(count * nwords), dim3(threads), lds, st, nets, n, nwords, saturation,
                       done_count);
    return hipGetLastError();
}

hipError_t launch_rowor_column_tiles(const ColumnTileNet *nets, const uint2 *tiles, uint32_t count,
                                     uint32_t rows, uint32_t threads, bool saturation,
                                     hipStream_t st) {
    if (count == 0) return hipSuccess;
    if (!rowor_column_fits(rows, 0)) return hipErrorInvalidValue;
    const size_t lds = column_lds(rows, 0);
    hipError_t e = hipFuncSetAttribute((const void *)k_rowor_column_tiles,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_rowor_column_tiles, dim3(count), dim3(threads), lds, st, nets, tiles,
                       saturation);
    return hipGetLastError();
}

}  // namespace tn
