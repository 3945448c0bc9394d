// gfx950 kernels of the row-OR stream of small networks: one wavefront per
// word column keeps the column of every row in LDS (Sec. 3.1 Algorithm 1 in
// reverse time, Sec. 3.4; each word column evolves on its own).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "tn_device.h"
#include "tn_wave.h"

namespace tn {

namespace {

// Small networks: one wavefront per word column keeps that column of every
// row and scratch row in LDS and runs every level of the op schedule with
// no barrier.  The ops of a level touch disjoint rows, and one wavefront's
// LDS accesses complete in program order, so level l + 1 sees level l.
// The loop is software-pipelined so that a group of up to 64 ops of one
// level costs one LDS round trip.  The ops live in an LDS ring of two
// windows; the window after those is loaded from HBM into registers one
// window ahead of use.
constexpr uint32_t kWaveWin = 512;
constexpr uint32_t kWaveRing = 2 * kWaveWin;
constexpr uint32_t kWavePre = kWaveWin / 64;  // entries per lane of a prefetched window

// A ring of two windows of T in LDS fed from src[0 .. count) (the last
// entry repeated past the end), with the window after them in registers.
template <typename T>
struct WaveRing {
    T *ring;
    const T *src;
    uint32_t count, nwin, next;  // windows below next are (or were) in the ring
    T pre[kWavePre];
    __device__ void fetch(uint32_t win, uint32_t lane) {
#pragma unroll
        for (uint32_t k = 0; k < kWavePre; ++k) pre[k] = src[min(win * kWaveWin + 64 * k + lane, count - 1)];
    }
    __device__ void store(uint32_t win, uint32_t lane) {
#pragma unroll
        for (uint32_t k = 0; k < kWavePre; ++k) ring[(win * kWaveWin + 64 * k + lane) % kWaveRing] = pre[k];
    }
    __device__ void init(T *r, const T *s, uint32_t c, uint32_t lane) {
        ring = r;
        src = s;
        count = c;
        nwin = (c + kWaveWin - 1) / kWaveWin;
        next = min(nwin, 2u);
        for (uint32_t win = 0; win < next; ++win) {
            fetch(win, lane);
            store(win, lane);
        }
        if (next < nwin) fetch(next, lane);
    }
    // makes entries up to `last` readable (true when that took a new
    // window); reads advance by less than a window at a time, so the ring
    // slot refilled held a window no longer read
    __device__ bool need(uint32_t last, uint32_t lane) {
        if (last / kWaveWin >= next && next < nwin) {
            store(next, lane);
            ++next;
            if (next < nwin) fetch(next, lane);
            return true;
        }
        return false;
    }
    __device__ T at(uint32_t i) const { return ring[i % kWaveRing]; }
};

// The schedule is in the flat form: ops in level order, their rows as LDS byte
// offsets of the column (kFlatNone: no second target) and bit 31 of the
// first offset set on the last op of every level.  A group is up to 64 ops
// of one level; the next group's ops are read ahead, and one ballot of
// their level-end bits gives its size, so the loop keeps no level starts.
// With sat, the column stops once every real row is all ones: rows only
// gain bits, so nothing later in the schedule can change it.  It is checked
// whenever a new window of ops enters the ring (every kWaveWin ops, off the
// per-group path), by a scan of the column in LDS that ends at the first
// 64-row block holding a row not yet full.
// Word column w of one network (one wavefront); sink: a word per lane that
// takes the idle lanes' accesses.
__device__ __forceinline__ void
rowor_wave_flat_column(const WaveNet &net, uint32_t w, uint32_t n, uint32_t nwords, bool sat,
                       unsigned int *__restrict__ done_count,
                       unsigned long long *__restrict__ traffic) {
    extern __shared__ uint64_t rows[];
    __shared__ op4 oring[kWaveRing];
    __shared__ uint64_t sink[64];
    const uint32_t lane = threadIdx.x;
    const uint32_t rwords = (n + 31) / 32;
    const uint32_t tail = n & 63u;
    const uint64_t fullw = (w + 1 < nwords || tail == 0) ? ~0ull : (1ull << tail) - 1ull;
    uint32_t *pst = net.persist ? net.persist + (size_t)w * (2 * (size_t)rwords + 2) : nullptr;
    const uint32_t nops = net.s.nops;
    if (nops == 0) return;       // nothing to apply: C is left as it is
    if (pst && pst[0]) return;   // the column is all ones already (uniform)
    uint64_t *const C = net.C;
    const int64_t ld = net.ld;
    for (uint32_t r = lane; r < n; r += 64) rows[r] = C[(size_t)r * ld + w];
    WaveRing<op4> opr;
    opr.init(oring, reinterpret_cast<const op4 *>(net.s.ops), nops, lane);
    unsigned char *const base = reinterpret_cast<unsigned char *>(rows);
    uint64_t *const own = sink + lane;
    auto row = [&](uint32_t off) { return reinterpret_cast<uint64_t *>(base + (off & kFlatOffMask)); };
    auto group = [&](const op4 &o, uint32_t q) -> uint32_t {
        const uint64_t ends = __ballot(q + lane < nops && (o.x >> 31));
        const uint32_t g = ends ? (uint32_t)__ffsll((unsigned long long)ends) : 64u;
        return min(g, nops - q);
    };
    uint32_t q = 0;
    op4 op = opr.at(lane);
    uint32_t size = group(op, 0);
    for (;;) {
        const uint32_t nq = q + size;
        const bool more = nq < nops;
        bool stop = false;
        if (more && opr.need(min(nq + 64, nops) - 1, lane) && sat) {
            // every group before this one has been applied; this one is
            // applied all the same (it cannot change a full column)
            bool full = true;
            for (uint32_t r0 = 0; r0 < n && full; r0 += 64)
                full = __all(r0 + lane >= n || rows[r0 + lane] == fullw);
            stop = full;
        }
        const op4 nop = opr.at(nq + lane);
        {
            const bool act = lane < size;
            const uint64_t r = *(act ? row(op.x) : own) | *(act ? row(op.y) : own);
            asm volatile("" : : "v"(nop.x), "v"(nop.y), "v"(nop.z), "v"(nop.w));
            *(act && op.z != kFlatNone ? row(op.z) : own) = r;
            *(act && op.w != kFlatNone ? row(op.w) : own) = r;
        }
        if (!more || stop) break;
        size = group(nop, nq);
        op = nop;
        q = nq;
    }
    for (uint32_t r = lane; r < n; r += 64) C[(size_t)r * ld + w] = rows[r];
    if (traffic && lane == 0) {
        atomicAdd(traffic, (unsigned long long)n);
        atomicAdd(traffic + 1, (unsigned long long)n);
    }
    if (!pst) return;
    int32_t nfull = 0;
    for (uint32_t k = lane; k < rwords; k += 64) {
        uint32_t fb = 0, nz = 0;
        for (uint32_t bb = 0; bb < 32 && 32 * k + bb < n; ++bb) {
            const uint64_t v = rows[32 * k + bb];
            fb |= (uint32_t)(v == fullw) << bb;
            nz |= (uint32_t)(v != 0) << bb;
        }
        pst[2 + k] = fb;
        pst[2 + rwords + k] = nz;
        nfull += __popc(fb);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) nfull += __shfl_xor(nfull, off);
    if (lane == 0) {
        pst[1] = (uint32_t)nfull;
        if (nfull == (int32_t)n) {
            pst[0] = 1u;
            atomicAdd(done_count, 1u);
        }
    }
}

// count networks (nets: device array), one block per (network, column)
__global__ void __launch_bounds__(64)
k_rowor_wave_flat(const WaveNet *__restrict__ nets, uint32_t n, uint32_t nwords, bool sat,
                  unsigned int *__restrict__ done_count,
                  unsigned long long *__restrict__ traffic) {
    const uint32_t b = xcd_slice(blockIdx.x, gridDim.x);
    rowor_wave_flat_column(nets[b / nwords], b % nwords, n, nwords, sat, done_count, traffic);
}

// one network passed by value (a resident plan), one block per column
__global__ void __launch_bounds__(64)
k_rowor_wave_flat1(WaveNet net, uint32_t n, uint32_t nwords, bool sat,
                   unsigned long long *__restrict__ traffic) {
    rowor_wave_flat_column(net, xcd_slice(blockIdx.x, gridDim.x), n, nwords, sat, nullptr,
                           traffic);
}

}  // namespace

size_t flat_ops_bytes(const HostSchedule &s) { return std::max<size_t>(256, 4 * s.ops.size()); }

void flat_ops_pack(const HostSchedule &s, uint32_t n, uint32_t *out) {
    auto byte_off = [n](uint32_t id) -> uint32_t {
        return 8u * ((id & kScratchBit) ? n + (id & kNodeMask) : id);
    };
    for (uint32_t l = 0; l < s.Lops; ++l) {
        const uint32_t q1 = s.lvl_op[l + 1];
        for (uint32_t q = s.lvl_op[l]; q < q1; ++q) {
            const uint32_t *src = &s.ops[4 * (size_t)q];
            uint32_t *o = out + 4 * (size_t)q;
            o[0] = byte_off(src[0]) | (q + 1 == q1 ? kFlatEnd : 0u);
            o[1] = byte_off(src[1]);
            o[2] = src[2] == kNoRow ? kFlatNone : byte_off(src[2]);
            o[3] = src[3] == kNoRow ? kFlatNone : byte_off(src[3]);
        }
    }
}

hipError_t launch_rowor_wave_flat(const WaveNet *nets, uint32_t count, uint32_t n,
                                  uint32_t max_scratch_rows, bool saturation,
                                  unsigned int *done_count, unsigned long long *traffic,
                                  hipStream_t st) {
    if (count == 0) return hipSuccess;
    if (!rowor_wave_fits(n, max_scratch_rows)) return hipErrorInvalidValue;
    const uint32_t nwords = (n + 63) / 64;
    const size_t lds = ((size_t)n + max_scratch_rows + 1) * 8;
    hipError_t e = hipFuncSetAttribute((const void *)k_rowor_wave_flat,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_rowor_wave_flat, dim3(count * nwords), dim3(64), lds, st, nets, n, nwords,
                       saturation, done_count, traffic);
    return hipGetLastError();
}

hipError_t launch_rowor_wave_flat1(const uint32_t *flat_ops, uint32_t nops, uint32_t n,
                                   uint64_t *C, int64_t ld, uint32_t scratch_rows,
                                   unsigned long long *traffic, bool saturation, hipStream_t st) {
    if (nops == 0) return hipSuccess;
    if (!rowor_wave_fits(n, scratch_rows)) return hipErrorInvalidValue;
    const uint32_t nwords = (n + 63) / 64;
    const size_t lds = ((size_t)n + scratch_rows + 1) * 8;
    hipError_t e = hipFuncSetAttribute((const void *)k_rowor_wave_flat1,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    WaveNet net{};
    net.s.nops = nops;
    net.s.ops = reinterpret_cast<const uint4 *>(flat_ops);
    net.C = C;
    net.ld = ld;
    hipLaunchKernelGGL(k_rowor_wave_flat1, dim3(nwords), dim3(64), lds, st, net, n, nwords,
                       saturation, traffic);
    return hipGetLastError();
}

bool rowor_wave_fits(uint32_t n, uint32_t scratch_rows) {
    return ((size_t)n + scratch_rows + 1) * 8 <= kRoworWaveLds;
}

bool rowor_wave_pays(uint32_t n, uint32_t scratch_rows, int64_t ops, int64_t levels) {
    return rowor_wave_fits(n, scratch_rows) && !rowor_wave_wide(ops, levels);
}

bool rowor_wave_wide(int64_t ops, int64_t levels) { return ops > kRoworWaveWideOps * levels; }

}  // namespace tn
