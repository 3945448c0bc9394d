// gfx950 kernels of the row-OR stream of networks whose word columns fit in
// LDS: one workgroup per word column keeps the column of every row in LDS
// and runs the levels with a barrier each (Sec. 3.1 Algorithm 1 in reverse
// time, Sec. 3.4; each word column evolves on its own).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "tn_device.h"
#include "tn_wave.h"

namespace tn {

namespace {

// Waits for the wavefront's memory loads (vmcnt 0) here and now: a load that
// only some levels make, were its wait left to its use, would have every
// level wait there for the windows in flight.
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Word column w of one network (n real rows, then scratch rows and one idle
// row per lane, in LDS).  The ops come in windows of one per thread, each
// requested four windows before it is used; within a window the threads of a
// level's ops act, then the barrier ends the level (a level that runs past
// its window goes on in the next one without a barrier: its ops are
// independent).  A wavefront without an op of the level skips it whole.  The
// starts of 64 levels sit in the lanes of every wavefront.
//
// With sat the column stops once every real row is all ones (rows only gain
// bits): every 32 levels each thread moves past the rows of its own that are.
//
// FRESH: the column starts as the identity's and the row padding is written
// too, so that no launch has to write the matrix before.
//
// Bound by the latency of a level (two LDS reads, two writes, the barrier),
// where the kernel on slices of C in memory waits for L2 in each: random
// events on 10,007 nodes, 698 ops a level, 1366 -> 282 us; on 16,000 nodes
// 3760 -> 456; activity-driven events on 10^4 nodes, 54 ops a level, 2809 ->
// 519.  16 hashed proxies of 4096 nodes in one launch 1032 -> 392.
template <bool FRESH>
__device__ __forceinline__ void
rowor_column(const WaveNet &net, uint32_t w, uint32_t n, uint32_t nwords, uint32_t scratch_rows,
             bool sat, unsigned int *__restrict__ done_count) {
    extern __shared__ uint64_t rows[];
    __shared__ uint32_t open, total;
    const DevOps &s = net.s;
    uint64_t *const C = net.C;
    const int64_t ld = net.ld;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, W = blockDim.x;
    const uint32_t rwords = (n + 31) / 32, tail = n & 63u;
    const uint64_t fullw = (w + 1 < nwords || tail == 0) ? ~0ull : (1ull << tail) - 1ull;
    uint32_t *pst = net.persist ? net.persist + (size_t)w * (2 * (size_t)rwords + 2) : nullptr;
    if (!FRESH && (s.L == 0 || s.nops == 0)) return;  // C is left as it is
    if (pst && pst[0]) return;                        // all ones already (uniform)
    if (tid == 0) open = total = 0;
    for (uint32_t r = tid; r < n; r += W)
        rows[r] = FRESH ? ((r >> 6) == w ? 1ull << (r & 63u) : 0ull) : C[(size_t)r * ld + w];
    if (s.nops) {
        uint32_t l0 = 0, ends;
        auto bounds = [&] {
            ends = s.lvl[min(l0 + lane + 1, s.L)];
            wait_loads();
        };
        bounds();
        // the load of a window is unconditional, so that the wait before its
        // use counts the windows after it (past the last op nothing is used)
        auto load = [&](uint32_t base) {
            return reinterpret_cast<const op4 *>(s.ops)[min(base + tid, s.nops - 1)];
        };
        op4 w0 = load(0), w1 = load(W), w2 = load(2 * W), w3 = load(3 * W);
        const uint32_t first = __builtin_amdgcn_readfirstlane(tid);  // the wavefront's
        const uint32_t idle = n + scratch_rows + lane;
        auto row = [&](uint32_t id) { return (id & kScratchBit) ? n + (id & kNodeMask) : id; };
        __syncthreads();
        uint32_t l = 0, pos = 0, full = tid;
        // the levels' ops in one window; true at the stream's end
        auto window = [&](const op4 &it, uint32_t base) -> bool {
            const uint32_t a = row(it.x), b = row(it.y), d1 = row(it.z);
            const uint32_t d2 = it.w == kNoRow ? idle : row(it.w);
            for (;;) {
                // kept in scalar registers (every lane's are the same)
                l = __builtin_amdgcn_readfirstlane(l);
                l0 = __builtin_amdgcn_readfirstlane(l0);
                pos = __builtin_amdgcn_readfirstlane(pos);
                if (l >= s.L) return true;
                const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)ends, (int)(l - l0));
                const uint32_t hi = min(end, base + W);
                if (base + first < hi && base + first + 64 > pos) {
                    const bool in = base + tid - pos < hi - pos;
                    const uint64_t r = rows[in ? a : idle] | rows[in ? b : idle];
                    rows[in ? d1 : idle] = r;
                    rows[in ? d2 : idle] = r;
                }
                pos = hi;
                if (end > base + W) return false;
                __syncthreads();
                ++l;
                if (sat && l > 1 && (l & 31u) < 3u) {
                    // after levels 32 k: look; 32 k + 1: all are; 32 k + 2: reset
                    if ((l & 31u) == 0) {
                        while (full < n && rows[full] == fullw) full += W;
                        if (full < n) open = 1;
                    } else if ((l & 31u) == 1) {
                        if (__builtin_amdgcn_readfirstlane(open) == 0) l = s.L;
                    } else if (tid == 0) {
                        open = 0;
                    }
                }
                if (l - l0 >= 64 && l < s.L) {
                    l0 = l;
                    bounds();
                }
            }
        };
        for (uint32_t base = 0;; base += 4 * W) {
            if (window(w0, base)) break;
            w0 = load(base + 4 * W);
            if (window(w1, base + W)) break;
            w1 = load(base + 5 * W);
            if (window(w2, base + 2 * W)) break;
            w2 = load(base + 6 * W);
            if (window(w3, base + 3 * W)) break;
            w3 = load(base + 7 * W);
        }
    }
    __syncthreads();
    for (uint32_t r = tid; r < n; r += W) C[(size_t)r * ld + w] = rows[r];
    if (FRESH)
        for (int64_t p = (int64_t)nwords + w; p < ld; p += nwords)
            for (uint32_t r = tid; r < n; r += W) C[(size_t)r * ld + p] = 0ull;
    if (!pst) return;
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
// words loaded and stored, written here where FRESH, else added.
template <bool FRESH>
__global__ void __launch_bounds__(1024)
k_rowor_column(WaveNet net, uint32_t n, uint32_t nwords, uint32_t scratch_rows, bool sat,
               unsigned int *__restrict__ done_count, unsigned long long *__restrict__ traffic) {
    if (traffic && threadIdx.x < 2) {
        if (FRESH) {
            if (blockIdx.x == 0)
                traffic[threadIdx.x] = net.s.nops ? (unsigned long long)n * nwords : 0ull;
        } else {
            atomicAdd(traffic + threadIdx.x, (unsigned long long)n);
        }
    }
    rowor_column<FRESH>(net, xcd_slice(blockIdx.x, gridDim.x), n, nwords, scratch_rows, sat,
                        done_count);
}

// Many networks of n nodes (the hashed proxies): workgroup b runs word column
// b % nwords of network b / nwords.
__global__ void __launch_bounds__(1024)
k_rowor_columns(const WaveNet *__restrict__ nets, uint32_t n, uint32_t nwords,
                uint32_t scratch_rows, bool sat, unsigned int *__restrict__ done_count) {
    const uint32_t b = xcd_slice(blockIdx.x, gridDim.x);
    rowor_column<false>(nets[b / nwords], b % nwords, n, nwords, scratch_rows, sat, done_count);
}

constexpr size_t kColumnLds = 160 * 1024 - 64;  // LDS of a workgroup, the statics aside
size_t column_lds(uint32_t n, uint32_t scratch_rows) { return ((size_t)n + scratch_rows + 64) * 8; }

// Threads of a workgroup, from the ops of a level on average: 1024 save the
// second window of wide levels (n = 16,000, 708 ops a level: 456 us against
// 540 with 512 and 828 with 256), 512 the bookkeeping of idle wavefronts in
// narrow ones (n = 10^4, 54 ops: 519 us against 559 with 1024, 535 with 256).
uint32_t column_threads(int64_t ops, int64_t levels) { return ops > 320 * levels ? 1024u : 512u; }

}  // namespace

bool rowor_column_fits(uint32_t n, uint32_t scratch_rows) {
    return column_lds(n, scratch_rows) <= kColumnLds;
}

bool rowor_column_pays(uint32_t n, uint32_t scratch_rows, int64_t ops, int64_t levels,
                       bool saturation) {
    if (!rowor_column_fits(n, scratch_rows)) return false;
    return rowor_wave_fits(n, scratch_rows) ? rowor_wave_wide(ops, levels) : saturation;
}

hipError_t launch_rowor_column(const DevOps &s, uint32_t n, uint64_t *C, int64_t ld,
                               uint32_t scratch_rows, unsigned long long *traffic, bool saturation,
                               bool fresh, uint32_t *persist, unsigned int *done_count,
                               hipStream_t st) {
    if (!fresh && (s.L == 0 || s.nops == 0)) return hipSuccess;
    if (!rowor_column_fits(n, scratch_rows)) return hipErrorInvalidValue;
    const size_t lds = column_lds(n, scratch_rows);
    auto k = fresh ? k_rowor_column<true> : k_rowor_column<false>;
    hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
    const uint32_t threads = column_threads(s.nops, std::max<int64_t>(s.L, 1));
    const uint32_t nwords = (n + 63) / 64;
    hipLaunchKernelGGL(k, dim3(nwords), dim3(threads), lds, st, WaveNet{s, C, ld, persist}, n, nwords,
                       scratch_rows, saturation, done_count, traffic);
    return hipGetLastError();
}

hipError_t launch_rowor_columns(const WaveNet *nets, uint32_t count, uint32_t n,
                                uint32_t max_scratch_rows, bool saturation, unsigned int *done_count, hipStream_t st) {
    if (count == 0) return hipSuccess;
    if (!rowor_column_fits(n, max_scratch_rows)) return hipErrorInvalidValue;
    const size_t lds = column_lds(n, max_scratch_rows);
    hipError_t e = hipFuncSetAttribute((const void *)k_rowor_columns,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const uint32_t nwords = (n + 63) / 64;
    // 512 threads, so that a CU holds several columns (16 networks of 4096
    // nodes: 392 us, with 256 threads 423, with 1024 566)
    hipLaunchKernelGGL(k_rowor_columns, dim3(count * nwords), dim3(512), lds, st, nets, n, nwords,
                       max_scratch_rows, saturation, done_count);
    return hipGetLastError();
}

}  // namespace tn
