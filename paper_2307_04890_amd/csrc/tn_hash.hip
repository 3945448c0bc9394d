// Network hashing (Sec. 4.1) and fusion of the hashed proxies (Sec. 4.2).
//
// Hash: h_j(u) = (acc_0(x0) ^ acc_1(x1) ^ acc_2(x2)) mod K, where x0 / x1 are
// the low / high 32 bits of u, x2 = x0 + x1, and acc_i folds the coefficients
// of row i of table A_j with (x * acc + a) mod (2^61 - 1).  The product is
// formed exactly in 128 bits and reduced with 2^61 = 1 (mod 2^61 - 1).
//
// Fusion: the estimated out-component of u keeps node w iff bit h_j(w) of row
// h_j(u) of every proxy P_j is set.  For a chunk q of 64 nodes w and a hash
// j, the lifted table Lt[q][j][r] packs those 64 bits for every super-node
// r; it is the transpose of the 64 proxy columns h_j(w), so it is built from
// the transposed proxies with 64 x 64 bit transposes inside a wavefront.  The
// estimate of u is then sum_q popcount(AND_j Lt[q][j][h_j(u)]), evaluated
// with the tables of a chunk staged in LDS.
#include <hip/hip_runtime.h>

#include "tn_device.h"
#include <algorithm>

#include "tn_hash.h"

namespace tn {

namespace {

constexpr uint64_t kP61 = (1ull << 61) - 1;

// (x * acc + a) mod (2^61 - 1), x < 2^34, acc < 2^61, a < 2^61 - 1.
__device__ __forceinline__ uint64_t mult_add_mod(uint64_t x, uint64_t acc, uint64_t a) {
    uint64_t lo = x * acc;
    uint64_t hi = __umul64hi(x, acc);
    const uint64_t lo2 = lo + a;
    hi += (lo2 < lo) ? 1ull : 0ull;
    lo = lo2;
    // value = hi * 2^64 + lo;  2^64 = 8 (mod p), 2^61 = 1 (mod p)
    uint64_t r = (lo & kP61) + (lo >> 61) + (hi << 3);
    r = (r & kP61) + (r >> 61);
    return r >= kP61 ? r - kP61 : r;
}

__device__ __forceinline__ uint64_t poly(const uint64_t *__restrict__ Ai, int order, uint64_t x) {
    uint64_t acc = Ai[0] % kP61;
    for (int l = 1; l < order; ++l) acc = mult_add_mod(x, acc, Ai[l]);
    return acc;
}

__global__ void __launch_bounds__(256)
k_hash_buckets(uint32_t n, uint32_t H, const uint64_t *__restrict__ coeffs, int order, uint32_t K,
               uint32_t *__restrict__ bucket) {
    const size_t total = (size_t)n * H;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (size_t)gridDim.x * blockDim.x) {
        const uint32_t j = (uint32_t)(i / n);
        const uint64_t u = i - (size_t)j * n;
        const uint64_t *A = coeffs + (size_t)j * 3 * order;
        const uint64_t x0 = u & 0xffffffffull, x1 = u >> 32, x2 = x0 + x1;
        const uint64_t h = poly(A, order, x0) ^ poly(A + order, order, x1) ^
                           poly(A + 2 * order, order, x2);
        bucket[i] = (uint32_t)(h % K);
    }
}

__global__ void __launch_bounds__(256) k_zero_i32(int32_t *__restrict__ p, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

__global__ void __launch_bounds__(256)
k_bucket_counts(uint32_t n, uint32_t H, uint32_t K, const uint32_t *__restrict__ bucket,
                int32_t *__restrict__ count) {
    const size_t total = (size_t)n * H;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (size_t)gridDim.x * blockDim.x) {
        const uint32_t j = (uint32_t)(i / n);
        atomicAdd(count + (size_t)j * K + bucket[i], 1);
    }
}

// Transposes the 64 x 64 bit block held one row per lane (bit b of lane i's
// word is entry (i, b)); afterwards lane b holds column b.
__device__ __forceinline__ uint64_t wave_transpose64(uint64_t x) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t masks[6] = {0x00000000ffffffffull, 0x0000ffff0000ffffull,
                               0x00ff00ff00ff00ffull, 0x0f0f0f0f0f0f0f0full,
                               0x3333333333333333ull, 0x5555555555555555ull};
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const uint32_t s = 32u >> k;
        const uint64_t y = (uint64_t)__shfl_xor((unsigned long long)x, (int)s, 64);
        if (lane & s) {
            const uint64_t t = ((y >> s) ^ x) & masks[k];
            x ^= t;
        } else {
            const uint64_t t = ((x >> s) ^ y) & masks[k];
            x ^= t << s;
        }
    }
    return x;
}

// PT_j = transpose of P_j (K x K bits): one wavefront per run of kLiftRun
// 64 x 64 blocks along a row block; lane i reads kLiftRun consecutive words
// of row 64 br + i (the loads after the first hit the sector the first
// brought in), then each block is transposed and written.
constexpr uint32_t kLiftRun = 8;
__global__ void __launch_bounds__(256)
k_transpose_proxies(uint32_t H, uint32_t K, int64_t ldK, const uint64_t *__restrict__ P,
                    uint64_t *__restrict__ PT) {
    const uint32_t kw = (K + 63) / 64;
    const uint32_t runs = (kw + kLiftRun - 1) / kLiftRun;
    const size_t jobs = (size_t)H * kw * runs;
    const uint32_t lane = threadIdx.x & 63u;
    for (size_t job = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; job < jobs;
         job += ((size_t)gridDim.x * blockDim.x) >> 6) {
        const uint32_t j = (uint32_t)(job / ((size_t)kw * runs));
        const uint32_t rem = (uint32_t)(job - (size_t)j * kw * runs);
        const uint32_t br = rem / runs, bc0 = rem % runs * kLiftRun;  // row block, first word block
        const uint64_t *Pj = P + (size_t)j * K * ldK;
        const uint32_t r = br * 64 + lane;
        uint64_t x[kLiftRun];
#pragma unroll
        for (uint32_t t = 0; t < kLiftRun; ++t)
            x[t] = (r < K && bc0 + t < kw) ? Pj[(size_t)r * ldK + bc0 + t] : 0ull;
#pragma unroll
        for (uint32_t t = 0; t < kLiftRun; ++t) {
            if (bc0 + t >= kw) break;  // uniform: the whole wave
            const uint64_t y = wave_transpose64(x[t]);  // lane b: bits r of column 64 (bc0 + t) + b
            const uint32_t c = (bc0 + t) * 64 + lane;
            if (c < K) PT[(size_t)j * K * ldK + (size_t)c * ldK + br] = y;
        }
    }
}

// bsum[j][wd] = sum of count[j][c] over the 64 super-nodes c of word wd
// (those below K): one wavefront per (j, wd).
__global__ void __launch_bounds__(256)
k_block_sums(uint32_t H, uint32_t K, const int32_t *__restrict__ count, int32_t *__restrict__ bsum) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t kw = (K + 63) / 64;
    const size_t blocks = (size_t)H * kw;
    for (size_t b = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; b < blocks;
         b += ((size_t)gridDim.x * blockDim.x) >> 6) {
        const uint32_t j = (uint32_t)(b / kw), c = (uint32_t)(b % kw) * 64 + lane;
        int32_t v = c < K ? count[(size_t)j * K + c] : 0;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if (lane == 0) bsum[b] = v;
    }
}

// One pass over every proxy row r of P_j, one wavefront per row, its lanes
// on consecutive words: rowsum[j][r] = {sum of count[j][c] over the super-nodes c
// set in the row, 1 iff the row has all K bits set}.
// A full word adds its block sum, an empty one nothing,
// and each other word one count load per lane (lane l: super-node 64 wd + l).
__global__ void __launch_bounds__(256)
k_row_sums(uint32_t H, uint32_t K, int64_t ldK, const uint64_t *__restrict__ P,
           const int32_t *__restrict__ count, const int32_t *__restrict__ bsum,
           int2 *__restrict__ rowsum) {
    const uint32_t lane = threadIdx.x & 63u;
    const size_t rows = (size_t)H * K;
    const uint32_t kw = (K + 63) / 64;
    const uint64_t last = (K % 64) ? ((1ull << (K % 64)) - 1ull) : ~0ull;
    for (size_t row = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; row < rows;
         row += ((size_t)gridDim.x * blockDim.x) >> 6) {
        const uint32_t j = (uint32_t)(row / K);
        const uint64_t *Pr = P + (size_t)j * K * ldK + (row - (size_t)j * K) * ldK;
        const int32_t *cj = count + (size_t)j * K;
        int32_t acc = 0;
        bool all = true;
        for (uint32_t wd0 = 0; wd0 < kw; wd0 += 64) {
            const uint32_t wd = wd0 + lane;
            const uint64_t word = wd < kw ? Pr[wd] : 0ull;
            const bool fullw = wd < kw && word == (wd + 1 == kw ? last : ~0ull);
            all &= wd >= kw || fullw;
            if (fullw) acc += bsum[(size_t)j * kw + wd];
            // the other non-empty words, one at a time over the wavefront
            uint64_t partial = __ballot(wd < kw && word != 0ull && !fullw);
            while (partial) {
                const uint32_t p = (uint32_t)__builtin_ctzll(partial);
                partial &= partial - 1ull;
                const uint64_t wp =
                    ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(word >> 32), (int)p) << 32) |
                    (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)word, (int)p);
                const uint32_t c = (wd0 + p) * 64 + lane;
                if (c < K && ((wp >> lane) & 1ull)) acc += cj[c];
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
        const bool row_full = __ballot(!all) == 0ull;
        if (lane == 0) rowsum[row] = make_int2(acc, row_full ? 1 : 0);
    }
}

// Lt[(q - q0) * H * K + j * K + r], bit i = P_j[r][h_j(64 q + i)] (0 past n):
// one wavefront per (q, j, run of kLiftRun 64-row blocks); lane i gathers
// words br of the transposed proxy row h_j(64 q + i) for the run's blocks
// (consecutive words of one row, so the loads after the first hit the
// sector it brought in), then each block is transposed and written.
__global__ void __launch_bounds__(256)
k_build_lifted(uint32_t n, uint32_t H, uint32_t K, int64_t ldK, const uint64_t *__restrict__ PT,
               const uint32_t *__restrict__ bucket, uint32_t q0, uint32_t nq,
               uint64_t *__restrict__ Lt) {
    const uint32_t kw = (K + 63) / 64;
    const uint32_t runs = (kw + kLiftRun - 1) / kLiftRun;
    const size_t jobs = (size_t)nq * H * runs;
    const uint32_t lane = threadIdx.x & 63u;
    for (size_t job = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6; job < jobs;
         job += ((size_t)gridDim.x * blockDim.x) >> 6) {
        const uint32_t br0 = (uint32_t)(job % runs) * kLiftRun;
        const uint32_t j = (uint32_t)((job / runs) % H);
        const uint32_t qq = (uint32_t)(job / ((size_t)runs * H));
        const uint64_t w = (uint64_t)(q0 + qq) * 64 + lane;
        uint64_t x[kLiftRun];
        const uint64_t *row = nullptr;
        if (w < n) row = PT + (size_t)j * K * ldK + (size_t)bucket[(size_t)j * n + w] * ldK;
#pragma unroll
        for (uint32_t t = 0; t < kLiftRun; ++t)
            x[t] = (row && br0 + t < kw) ? row[br0 + t] : 0ull;
#pragma unroll
        for (uint32_t t = 0; t < kLiftRun; ++t) {
            if (br0 + t >= kw) break;  // uniform: the whole wave
            const uint64_t y = wave_transpose64(x[t]);
            const uint32_t r = (br0 + t) * 64 + lane;
            if (r < K) Lt[((size_t)qq * H + j) * K + r] = y;
        }
    }
}

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) void glb_void;

// Tables of g hashes of one chunk (g K words at src) into LDS at dst,
// straight from memory with no registers: a wave's 64 lanes fill 64 units
// from the wave's LDS base, lane l at l units; 16-byte units where the
// tables start on 16 bytes (K even), else 4-byte ones.  Completes at the
// next barrier (which waits for the wave's own transfers).
__device__ __forceinline__ void stage_tables(const uint64_t *src, uint32_t words, uint32_t K,
                                             uint64_t *dst) {
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t waves = blockDim.x >> 6;
    if (K % 2 == 0) {
        const uint32_t units = words / 2;
        for (uint32_t c0 = wave * 64; c0 < units; c0 += waves * 64)
            if (c0 + lane < units)
                __builtin_amdgcn_global_load_lds((glb_void *)(src + 2 * (size_t)(c0 + lane)),
                                                 (lds_void *)(dst + 2 * (size_t)c0), 16, 0, 0);
    } else {
        const uint32_t units = words * 2;
        const uint32_t *s32 = (const uint32_t *)src;
        uint32_t *d32 = (uint32_t *)dst;
        for (uint32_t c0 = wave * 64; c0 < units; c0 += waves * 64)
            if (c0 + lane < units)
                __builtin_amdgcn_global_load_lds((glb_void *)(s32 + c0 + lane),
                                                 (lds_void *)(d32 + c0), 4, 0, 0);
    }
}

// est[u] += sum over the chunks q of this launch of popcount(AND_j Lt[q][j][h_j(u)]).
// A workgroup owns kUPT nodes u per thread (a node block) and one of the
// launch's ranges of `per` chunks; the counts of the ranges add up in est
// (integer atomics, so the order does not matter).  Every node block stages
// the same tables, so the workgroups of one chunk range are numbered
// consecutively and given to one XCD (xcd_slice): they run there together
// and read the tables through that XCD's L2 rather than each from HBM.  With
// LDS,
// the tables of G hashes of one chunk are staged in LDS at a time (K words
// each), else (tables too large for LDS) they are read where they are, in
// L2; the AND of a chunk is carried in registers across the hash groups.
constexpr int kUPT = 8;
constexpr int kQB = 2;
constexpr uint32_t kRecombineThreads = 1024;
constexpr size_t kRecombineLds = 160 * 1024;  // LDS of one CU
template <bool LDS>
__global__ void __launch_bounds__(kRecombineThreads)
k_recombine_est(uint32_t n, uint32_t H, uint32_t K, uint32_t G, const uint32_t *__restrict__ bucket,
                const uint64_t *__restrict__ Lt, uint32_t q_first, uint32_t q_last, uint32_t per,
                uint32_t q0, const uint32_t *__restrict__ list, uint32_t nlist, uint32_t ublocks,
                int32_t *__restrict__ est) {
    extern __shared__ uint64_t tab[];
    const uint32_t tid = threadIdx.x;
    const uint32_t L = xcd_slice(blockIdx.x, gridDim.x);
    const uint64_t ubase = (uint64_t)(L % ublocks) * blockDim.x * kUPT;
    const uint32_t q_begin = q_first + (L / ublocks) * per;
    const uint32_t q_end = min(q_last, q_begin + per);
    // uniform: the whole workgroup leaves
    if (ubase >= nlist || q_begin >= q_end) return;
    uint32_t u[kUPT];
    int32_t cnt[kUPT];
#pragma unroll
    for (int k = 0; k < kUPT; ++k) {
        const uint64_t i = ubase + tid + (uint64_t)k * blockDim.x;
        u[k] = i < nlist ? list[i] : 0xffffffffu;
        cnt[k] = 0;
    }
    for (uint32_t qb = q_begin; qb < q_end; qb += kQB) {
        const uint32_t nqb = min((uint32_t)kQB, q_end - qb);
        uint64_t acc[kQB][kUPT];
#pragma unroll
        for (int a = 0; a < kQB; ++a) {
            // nodes past n in the last chunk never count
            const uint64_t first = (uint64_t)(qb + a) * 64;
            const uint64_t valid = (a < (int)nqb && first < n)
                                       ? ((n - first >= 64) ? ~0ull : ((1ull << (n - first)) - 1ull))
                                       : 0ull;
#pragma unroll
            for (int k = 0; k < kUPT; ++k) acc[a][k] = valid;
        }
        for (uint32_t j0 = 0; j0 < H; j0 += G) {
            const uint32_t g = min(G, H - j0);
            uint32_t b[kUPT][4];
            // buckets of this hash group (G <= 4)
#pragma unroll
            for (int k = 0; k < kUPT; ++k)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj)
                    b[k][jj] = (u[k] != 0xffffffffu && jj < (int)g) ? bucket[(size_t)(j0 + jj) * n + u[k]] : 0u;
#pragma unroll
            for (int a = 0; a < kQB; ++a) {
                if (a >= (int)nqb) break;
                const uint64_t *src = Lt + ((size_t)(qb + a - q0) * H + j0) * K;
                const uint64_t *tb = src;
                if (LDS) {
                    __syncthreads();
                    stage_tables(src, g * K, K, tab);
                    __syncthreads();
                    tb = tab;
                }
#pragma unroll
                for (int k = 0; k < kUPT; ++k)
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj)
                        if (jj < (int)g) acc[a][k] &= tb[(size_t)jj * K + b[k][jj]];
            }
        }
#pragma unroll
        for (int a = 0; a < kQB; ++a)
#pragma unroll
            for (int k = 0; k < kUPT; ++k) cnt[k] += __popcll(acc[a][k]);
    }
#pragma unroll
    for (int k = 0; k < kUPT; ++k)
        if (u[k] != 0xffffffffu && cnt[k]) atomicAdd(est + u[k], cnt[k]);
}

// The same sums as k_recombine_est with LDS, for tables of GB hashes whose
// two copies fit in LDS together: while a stage (one chunk, one group of GB
// hashes) is read from one buffer, the next stage's tables stream into the
// other, and the next group's buckets are requested before them (loads
// retire in order, so they must not queue behind the tables).
template <int GB>
__global__ void __launch_bounds__(kRecombineThreads)
k_recombine_est2(uint32_t n, uint32_t H, uint32_t K, const uint32_t *__restrict__ bucket,
                 const uint64_t *__restrict__ Lt, uint32_t q_first, uint32_t q_last, uint32_t per,
                 uint32_t q0, const uint32_t *__restrict__ list, uint32_t nlist, uint32_t ublocks,
                 int32_t *__restrict__ est) {
    extern __shared__ uint64_t tab[];  // two buffers of GB K words
    const uint32_t tid = threadIdx.x;
    const uint32_t L = xcd_slice(blockIdx.x, gridDim.x);
    const uint64_t ubase = (uint64_t)(L % ublocks) * blockDim.x * kUPT;
    const uint32_t q_begin = q_first + (L / ublocks) * per;
    const uint32_t q_end = min(q_last, q_begin + per);
    // uniform: the whole workgroup leaves
    if (ubase >= nlist || q_begin >= q_end) return;
    uint32_t u[kUPT];
    int32_t cnt[kUPT];
#pragma unroll
    for (int k = 0; k < kUPT; ++k) {
        const uint64_t i = ubase + tid + (uint64_t)k * blockDim.x;
        u[k] = i < nlist ? list[i] : 0xffffffffu;
        cnt[k] = 0;
    }
    const uint32_t groups = (H + GB - 1) / GB;
    const size_t bufw = (size_t)GB * K;
    uint32_t bc[kUPT][GB], bn[kUPT][GB];
    auto load_buckets = [&](uint32_t (&b)[kUPT][GB], uint32_t grp) {
        const uint32_t g = min((uint32_t)GB, H - grp * GB);
#pragma unroll
        for (int k = 0; k < kUPT; ++k)
#pragma unroll
            for (int jj = 0; jj < GB; ++jj)
                b[k][jj] = (u[k] != 0xffffffffu && jj < (int)g)
                               ? bucket[(size_t)(grp * GB + jj) * n + u[k]]
                               : 0u;
    };
    load_buckets(bc, 0);
    stage_tables(Lt + (size_t)(q_begin - q0) * H * K, min((uint32_t)GB, H) * K, K, tab);
    uint32_t buf = 0;
    for (uint32_t qb = q_begin; qb < q_end; qb += kQB) {
        const uint32_t nqb = min((uint32_t)kQB, q_end - qb);
        uint64_t acc[kQB][kUPT];
#pragma unroll
        for (int a = 0; a < kQB; ++a) {
            // nodes past n in the last chunk never count
            const uint64_t first = (uint64_t)(qb + a) * 64;
            const uint64_t valid = (a < (int)nqb && first < n)
                                       ? ((n - first >= 64) ? ~0ull : ((1ull << (n - first)) - 1ull))
                                       : 0ull;
#pragma unroll
            for (int k = 0; k < kUPT; ++k) acc[a][k] = valid;
        }
        for (uint32_t grp = 0; grp < groups; ++grp) {
            const uint32_t g = min((uint32_t)GB, H - grp * GB);
#pragma unroll
            for (int a = 0; a < kQB; ++a) {
                if (a >= (int)nqb) break;
                // the stage after this one
                const bool last_a = a + 1 == (int)nqb;
                uint32_t qb2 = qb, grp2 = grp, a2 = a + 1;
                if (last_a) {
                    a2 = 0;
                    grp2 = grp + 1;
                    if (grp2 == groups) {
                        grp2 = 0;
                        qb2 = qb + kQB;
                    }
                }
                const bool more = qb2 < q_end;
                // this stage's tables are in, and every wave is done with
                // the other buffer
                __syncthreads();
                if (more && last_a) load_buckets(bn, grp2);
                if (more)
                    stage_tables(Lt + ((size_t)(qb2 + a2 - q0) * H + grp2 * GB) * K,
                                 min((uint32_t)GB, H - grp2 * GB) * K, K,
                                 tab + (buf ^ 1u) * bufw);
                const uint64_t *tb = tab + buf * bufw;
                if (g == GB) {
                    // a whole group: every read unconditional, so they can be
                    // in flight together
#pragma unroll
                    for (int k = 0; k < kUPT; ++k)
#pragma unroll
                        for (int jj = 0; jj < GB; ++jj)
                            acc[a][k] &= tb[(size_t)jj * K + bc[k][jj]];
                } else {
#pragma unroll
                    for (int k = 0; k < kUPT; ++k)
#pragma unroll
                        for (int jj = 0; jj < GB; ++jj)
                            if (jj < (int)g) acc[a][k] &= tb[(size_t)jj * K + bc[k][jj]];
                }
                if (more && last_a) {
                    // after this stage's reads: the next group's buckets
#pragma unroll
                    for (int k = 0; k < kUPT; ++k)
#pragma unroll
                        for (int jj = 0; jj < GB; ++jj)
                            asm volatile("" : "=v"(bc[k][jj]) : "0"(bn[k][jj]) : "memory");
                }
                buf ^= 1u;
            }
        }
#pragma unroll
        for (int a = 0; a < kQB; ++a)
#pragma unroll
            for (int k = 0; k < kUPT; ++k) cnt[k] += __popcll(acc[a][k]);
    }
#pragma unroll
    for (int k = 0; k < kUPT; ++k)
        if (u[k] != 0xffffffffu && cnt[k]) atomicAdd(est + u[k], cnt[k]);
}

// ---- fusion by lists -------------------------------------------------------
//
// The tables above cost every node n / 64 words of each hash, whatever its
// rows hold.  But a row that lifts to nearly all nodes, or to few, is a short
// list: of the nodes it leaves out, or of those it keeps; any other row that
// some node meets is a bitmap of n bits, built once for all its nodes.  A
// node is then
//  - done: every row is full, est = n, or one lifts to none, est = 0;
//  - an intersection node where some row has a list of kept nodes: est = the
//    nodes of the shortest one that every other row keeps too;
//  - else a union node: est = n - |union of the nodes its rows leave out|, a
//    small one where its lists fit a wavefront's table in LDS, else a wide
//    one.
// fuse_by_lists (tn_hash.cpp) says when this beats the tables: with 2*10^5
// nodes and 4*10^4 events (H = 16, K = 4096), rows that leave out 39 nodes of
// a hash on average, a call takes 0.65 ms against 5.80 ms.
constexpr uint32_t kListPart = 64;        // lists of left-out nodes hold at most n / 64
constexpr uint32_t kInterMax = 1u << 10;  // lists of kept nodes
constexpr uint32_t kListSplit = 16;       // node ranges of a hash in the bucket sort
constexpr uint32_t kListMinN = 24576;
constexpr uint32_t kHashSlots = 2048;     // a small node's table: 8 KB
constexpr uint32_t kSmallHashed = kHashSlots / 2, kSmallMarked = 2560;  // entries of a small node
enum : uint8_t { kNodeDone = 0, kNodeSmall = 1, kNodeInter = 2, kNodeWide = 3 };
// The lists a row can have (the two top bits of its descriptor's length).
enum : uint32_t { kRowOut = 0, kRowKept = 1, kRowBits = 2 };

// How a row that lifts to s of n nodes is held, and its list's entries (none:
// a bitmap).
__device__ __forceinline__ uint32_t row_list(uint32_t n, int32_t s, uint32_t &len) {
    const uint32_t ones = (uint32_t)s, zeros = n - ones;
    len = 0;
    if (zeros <= n / kListPart) {
        len = zeros;
        return kRowOut;
    }
    if (ones <= kInterMax) {
        len = ones;
        return kRowKept;
    }
    return kRowBits;
}

// A 64-bit weight of (hash, super-node): the sums of it over the nodes' buckets
// and over the counts agree when the counts are the buckets' own.  Two products
// of one mixed word: 64-bit ones took every node and hash 7 multiplications, 3 us
// a call of 2*10^5 nodes and 16 hashes.
__device__ __forceinline__ unsigned long long bucket_mix(uint32_t j, uint32_t r) {
    uint32_t a = (r + j * 0x9e3779b9u) * 0x7f4a7c15u;
    a ^= a >> 15;
    uint32_t hi = a * 0xbf58476du, lo = a * 0x1ce4e5b9u;
    hi ^= hi >> 16;
    lo ^= lo >> 13;
    return (unsigned long long)hi << 32 | lo;
}

// The lists' entries and the bitmaps of hash j's rows that some node meets, and
// the sum of bucket_mix over its counts, added to stats; workgroup `part` of
// kTotalParts.  tot: 3 words of LDS.
constexpr uint32_t kTotalParts = 4;
__device__ __forceinline__ void list_totals(uint32_t n, uint32_t K, uint32_t j, uint32_t part,
                                            const int32_t *__restrict__ count,
                                            const int2 *__restrict__ rowsum,
                                            unsigned long long *tot,
                                            unsigned long long *__restrict__ stats) {
    unsigned long long v[3] = {};  // entries, bitmaps, mix
    for (uint32_t r = part * blockDim.x + threadIdx.x; r < K; r += kTotalParts * blockDim.x) {
        const int32_t c = count[(size_t)j * K + r];
        v[2] += bucket_mix(j, r) * (unsigned long long)(uint32_t)c;
        uint32_t len = 0;
        if (c && row_list(n, rowsum[(size_t)j * K + r].x, len) == kRowBits) ++v[1];
        v[0] += c ? len : 0u;
    }
    __syncthreads();  // tot is clear
#pragma unroll
    for (int k = 0; k < 3; ++k) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v[k] += __shfl_xor(v[k], off, 64);
        if ((threadIdx.x & 63u) == 0) atomicAdd(&tot[k], v[k]);
    }
    __syncthreads();
    if (threadIdx.x < 2 && tot[threadIdx.x])
        atomicAdd(stats + kFuseRows + 16 * threadIdx.x + j, tot[threadIdx.x]);
    if (threadIdx.x == 2)
        atomicAdd(stats + kFuseStats + 8 * ((kTotalParts * j + part) % kFuseParts) + 4, tot[2]);
}

// Each node's kind (cls), its lifted sizes (lifted, nullable), est (n where
// every row is full, else 0), the nodes some row of which is not full (open)
// and of them the wide ones (wide, from its start) and the small ones (wide,
// from its end); totals in stats.  Without LISTS only what the tables need: the
// lifted sizes, est and the open nodes.  With LISTS the last kTotalParts workgroups
// of each hash add up its rows (list_totals) beside the others: in a launch of
// their own, with the sum of bucket_mix over the nodes, they took each call 10 us.
template <bool LISTS, uint32_t B>  // B hashes at a time
__global__ void __launch_bounds__(256)
k_classify(uint32_t n, uint32_t H, uint32_t K, const uint32_t *__restrict__ bucket,
           const int32_t *__restrict__ count, const int2 *__restrict__ rowsum,
           int32_t *__restrict__ lifted, uint8_t *__restrict__ cls, int32_t *__restrict__ est,
           uint32_t *__restrict__ open, uint32_t *__restrict__ wide,
           unsigned long long *__restrict__ stats) {
    __shared__ uint32_t part[4][3], base[3];  // open, wide and small nodes
    __shared__ unsigned long long tot[4];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    if (threadIdx.x < 4) tot[threadIdx.x] = 0;
    const uint32_t groups = gridDim.x - (LISTS ? kTotalParts * H : 0u);
    if (LISTS && blockIdx.x >= groups) {
        const uint32_t k = blockIdx.x - groups;
        list_totals(n, K, k / kTotalParts, k % kTotalParts, count, rowsum, tot, stats);
        return;
    }
    unsigned long long entries = 0, bits = 0, inter = 0, mix = 0;
    const uint32_t small = n <= kMarkBits ? kSmallMarked : kSmallHashed;
    for (uint32_t t0 = blockIdx.x * blockDim.x; t0 < n; t0 += groups * blockDim.x) {
        const uint32_t u = t0 + threadIdx.x;
        bool all = true;
        uint8_t c = kNodeDone;
        if (u < n) {
            uint64_t out = 0;
            uint32_t smin = 0xffffffffu, nbits = 0;
            for (uint32_t j0 = 0; j0 < H; j0 += B) {
                // past the last hash its loads again: none depends on a branch, so
                // that all are in flight
                uint32_t b[B];
                int2 s[B];
#pragma unroll
                for (uint32_t k = 0; k < B; ++k)
                    b[k] = bucket[(size_t)min(j0 + k, H - 1) * n + u];
#pragma unroll
                for (uint32_t k = 0; k < B; ++k) s[k] = rowsum[(size_t)min(j0 + k, H - 1) * K + b[k]];
#pragma unroll
                for (uint32_t k = 0; k < B; ++k) {
                    if (j0 + k >= H) continue;
                    if (lifted) lifted[(size_t)(j0 + k) * n + u] = s[k].x;
                    all &= s[k].y != 0;
                    if (!LISTS) continue;
                    mix += bucket_mix(j0 + k, b[k]);
                    uint32_t len;
                    const uint32_t kind = row_list(n, s[k].x, len);
                    if (kind == kRowOut) out += len;
                    if (kind == kRowKept) smin = min(smin, len);
                    if (kind == kRowBits) ++nbits;
                }
            }
            // an empty row keeps no node; rows without a left-out node make a
            // small node of no entries
            if (LISTS && !all && smin != 0) {
                if (smin != 0xffffffffu) {
                    c = kNodeInter;
                    inter += smin;
                } else {
                    c = nbits == 0 && out <= small ? kNodeSmall : kNodeWide;
                    entries += out;
                    bits += nbits;
                }
            }
            if (LISTS) cls[u] = c;
            est[u] = all ? (int32_t)n : 0;
        }
        if (!__syncthreads_or(!all)) continue;
        const uint64_t in[3] = {__ballot(!all), __ballot(c == kNodeWide), __ballot(c == kNodeSmall)};
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (lane == 0) part[wave][k] = (uint32_t)__popcll(in[k]);
        __syncthreads();
        if (lane == 0 && wave < (LISTS ? 3u : 1u)) {  // a wavefront's atomic each
            uint32_t some = 0;
            for (uint32_t w = 0; w < blockDim.x >> 6; ++w) some += part[w][wave];
            constexpr int at[3] = {kFuseOpen, kFuseWide, kFuseSmall};
            if (some) base[wave] = (uint32_t)atomicAdd(stats + at[wave], (unsigned long long)some);
        }
        __syncthreads();
        uint32_t slot[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            slot[k] = base[k] + (uint32_t)__popcll(in[k] & ((1ull << lane) - 1ull));
            for (uint32_t w = 0; w < wave; ++w) slot[k] += part[w][k];
        }
        if (!all) open[slot[0]] = u;
        if (c == kNodeWide) wide[slot[1]] = u;
        if (c == kNodeSmall) wide[n - 1 - slot[2]] = u;
    }
    if (!LISTS) return;
    __syncthreads();  // tot is clear
    auto add = [&](int k, unsigned long long v) {
        if (__ballot(v != 0) == 0) return;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if (lane == 0) atomicAdd(&tot[k], v);
    };
    add(0, entries);
    add(1, bits);
    add(2, inter);
    add(3, mix);
    __syncthreads();
    // (hundreds of workgroups' atomics on one word took as long as the rest)
    if (threadIdx.x < 4 && tot[threadIdx.x])
        atomicAdd(stats + kFuseStats + 8 * (blockIdx.x % kFuseParts) + threadIdx.x, tot[threadIdx.x]);
}

// The nodes of each hash sorted by bucket, in three kernels over (range of
// nodes, hash): counts of each range in LDS, their exclusive sums, the
// ranges' nodes at their places.
__global__ void __launch_bounds__(512)
k_bucket_hist(uint32_t n, uint32_t K, const uint32_t *__restrict__ bucket,
              uint32_t *__restrict__ hist) {
    extern __shared__ uint32_t cnt[];
    const uint32_t j = blockIdx.y, per = (n + kListSplit - 1) / kListSplit;
    const uint32_t w0 = min(n, blockIdx.x * per), w1 = min(n, w0 + per);
    for (uint32_t r = threadIdx.x; r < K; r += blockDim.x) cnt[r] = 0;
    __syncthreads();
    for (uint32_t w = w0 + threadIdx.x; w < w1; w += blockDim.x) {
        const uint32_t b = bucket[(size_t)j * n + w];
        if (b < K) atomicAdd(cnt + b, 1u);
    }
    __syncthreads();
    uint32_t *h = hist + ((size_t)j * kListSplit + blockIdx.x) * K;
    for (uint32_t r = threadIdx.x; r < K; r += blockDim.x) h[r] = cnt[r];
}

// Exclusive sum of v over the workgroup's 1024 threads, its total in `total`.
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t *part, uint32_t &total) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)x, off, 64);
        if ((int)lane >= off) x += y;
    }
    __syncthreads();
    if (lane == 63) part[wave] = x;
    __syncthreads();
    uint32_t before = 0;
    total = 0;
    for (uint32_t k = 0; k < (blockDim.x >> 6); ++k) {
        before += k < wave ? part[k] : 0u;
        total += part[k];
    }
    return before + x - v;
}

// One workgroup per hash: the bucket starts and each range's places.
__global__ void __launch_bounds__(1024)
k_bucket_starts(uint32_t K, uint32_t *__restrict__ hist, uint32_t *__restrict__ start) {
    __shared__ uint32_t part[16];
    const uint32_t j = blockIdx.x;
    uint32_t *h = hist + (size_t)j * kListSplit * K;
    uint32_t carry = 0;
    for (uint32_t r0 = 0; r0 < K; r0 += blockDim.x) {
        const uint32_t r = r0 + threadIdx.x;
        uint32_t c[kListSplit], tot = 0;
#pragma unroll
        for (uint32_t s = 0; s < kListSplit; ++s) c[s] = r < K ? h[(size_t)s * K + r] : 0u;
#pragma unroll
        for (uint32_t s = 0; s < kListSplit; ++s) tot += c[s];
        uint32_t all;
        uint32_t at = carry + block_scan(tot, part, all);
        carry += all;
        if (r < K) {
            start[(size_t)j * (K + 1) + r] = at;
#pragma unroll
            for (uint32_t s = 0; s < kListSplit; ++s) {
                h[(size_t)s * K + r] = at;
                at += c[s];
            }
        }
    }
    if (threadIdx.x == 0) start[(size_t)j * (K + 1) + K] = carry;
}

__global__ void __launch_bounds__(512)
k_bucket_nodes(uint32_t n, uint32_t K, const uint32_t *__restrict__ bucket,
               const uint32_t *__restrict__ hist, uint32_t *__restrict__ nodes) {
    extern __shared__ uint32_t cnt[];
    const uint32_t j = blockIdx.y, per = (n + kListSplit - 1) / kListSplit;
    const uint32_t w0 = min(n, blockIdx.x * per), w1 = min(n, w0 + per);
    const uint32_t *h = hist + ((size_t)j * kListSplit + blockIdx.x) * K;
    for (uint32_t r = threadIdx.x; r < K; r += blockDim.x) cnt[r] = h[r];
    __syncthreads();
    for (uint32_t w = w0 + threadIdx.x; w < w1; w += blockDim.x) {
        const uint32_t b = bucket[(size_t)j * n + w];
        if (b < K) nodes[(size_t)j * n + atomicAdd(cnt + b, 1u)] = w;
    }
}

// rows[j K + r] = {first entry of the row's list, its length} or {its bitmap,
// 0}, the length's two top bits its kind, and the row of each bitmap.  One
// workgroup per hash, its entries and bitmaps after those of the hashes
// before it.
__global__ void __launch_bounds__(1024)
k_list_starts(uint32_t n, uint32_t K, const int32_t *__restrict__ count,
              const int2 *__restrict__ rowsum, const unsigned long long *__restrict__ stats,
              uint2 *__restrict__ rows, uint32_t *__restrict__ bitmap_row) {
    __shared__ uint32_t part[16];
    const uint32_t j = blockIdx.x;
    uint32_t entries = 0, bitmaps = 0;
    for (uint32_t i = 0; i < j; ++i) {
        entries += (uint32_t)stats[kFuseRows + i];
        bitmaps += (uint32_t)stats[kFuseRows + 16 + i];
    }
    for (uint32_t r0 = 0; r0 < K; r0 += blockDim.x) {
        const uint32_t r = r0 + threadIdx.x;
        uint32_t kind = kRowOut, len = 0, all;
        if (r < K && count[(size_t)j * K + r]) kind = row_list(n, rowsum[(size_t)j * K + r].x, len);
        const uint32_t e = entries + block_scan(len, part, all);
        entries += all;
        const uint32_t m = bitmaps + block_scan(kind == kRowBits ? 1u : 0u, part, all);
        bitmaps += all;
        if (r < K) rows[(size_t)j * K + r] = make_uint2(kind == kRowBits ? m : e, len | kind << 30);
        if (kind == kRowBits) bitmap_row[m] = j * K + r;
    }
}

// The bitmaps: bit w of a row's = the row leaves node w out.  A workgroup per
// (bitmap, one of gridDim.y ranges of nodes), the row in LDS, the hash's
// buckets in order, 64 verdicts a word.
constexpr uint32_t kListMaxK = (uint32_t)(kRecombineLds / 4);  // K counters in LDS
__global__ void __launch_bounds__(256)
k_fill_bitmaps(uint32_t n, uint32_t K, int64_t ldK, const uint64_t *__restrict__ P,
               const uint32_t *__restrict__ bucket, const uint32_t *__restrict__ bitmap_row,
               uint64_t *__restrict__ bitmaps) {
    __shared__ uint32_t prow[kListMaxK / 32];
    const size_t row = bitmap_row[blockIdx.x];
    const uint32_t *Pr = (const uint32_t *)(P + row * ldK);  // row r of matrix j: j K + r rows on
    for (uint32_t i = threadIdx.x; i < (K + 63) / 64 * 2; i += blockDim.x) prow[i] = Pr[i];
    __syncthreads();
    const uint32_t *bj = bucket + row / K * n;
    uint64_t *out = bitmaps + (size_t)blockIdx.x * ((n + 63) / 64);
    for (uint32_t w0 = blockIdx.y * 4 * blockDim.x + (threadIdx.x & ~63u); w0 < n;
         w0 += gridDim.y * 4 * blockDim.x) {
        uint32_t hb[4];
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            const uint32_t w = w0 + q * blockDim.x + (threadIdx.x & 63u);
            hb[q] = w < n ? bj[w] : 0xffffffffu;
        }
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            const uint32_t w = w0 + q * blockDim.x;
            const bool left = hb[q] != 0xffffffffu && !((prow[hb[q] >> 5] >> (hb[q] & 31u)) & 1u);
            const uint64_t m = __ballot(left);
            if ((threadIdx.x & 63u) == 0 && w < n) out[w >> 6] = m;
        }
    }
}

// The rows' lists, one wavefront per row.  Of 64 words at a time (inverted
// for a list of left-out nodes) the super-nodes go to LDS, then 64 of them at
// a time to the lanes, each reading where its nodes are; with RUNS (16 nodes
// and more on average) the wavefront copies one super-node's nodes at a time,
// four in flight, else every lane copies its own.
template <bool RUNS>
__global__ void __launch_bounds__(64)
k_fill_lists(uint32_t n, uint32_t H, uint32_t K, int64_t ldK, const uint64_t *__restrict__ P,
             const uint32_t *__restrict__ start, const uint32_t *__restrict__ nodes,
             const uint2 *__restrict__ rows, uint32_t *__restrict__ lists) {
    __shared__ uint16_t ids[64 * 64];  // K <= kListMaxK < 2^16
    const uint32_t lane = threadIdx.x;
    const size_t row = blockIdx.x;
    const uint2 d = rows[row];
    const uint32_t len = d.y & 0x3fffffffu;
    if (len == 0) return;
    const bool kept = d.y >> 30 == kRowKept;
    const uint32_t j = (uint32_t)(row / K), kw = (K + 63) / 64;
    const uint64_t last = (K % 64) ? ((1ull << (K % 64)) - 1ull) : ~0ull;
    const uint64_t *Pr = P + row * ldK;  // row r of matrix j: j K + r rows on
    const uint32_t *sj = start + (size_t)j * (K + 1);
    const uint32_t *nj = nodes + (size_t)j * n;
    uint32_t *out = lists + d.x;
    uint32_t at = 0;  // entries so far
    // exclusive sum over the lanes; total from the last
    auto scan = [&](uint32_t v, uint32_t &total) {
        uint32_t x = v;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)x, off, 64);
            if ((int)lane >= off) x += y;
        }
        total = (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
        return x - v;
    };
    for (uint32_t wd0 = 0; wd0 < kw && at < len; wd0 += 64) {
        const uint32_t wd = wd0 + lane;
        uint64_t x = 0;
        if (wd < kw) {
            x = kept ? Pr[wd] : ~Pr[wd];
            if (wd + 1 == kw) x &= last;
        }
        uint32_t some;
        uint32_t o = scan((uint32_t)__popcll(x), some);
        __syncthreads();  // one wavefront: the last block's ids are read
        for (; x; x &= x - 1ull) ids[o++] = (uint16_t)(wd * 64 + (uint32_t)__builtin_ctzll(x));
        __syncthreads();
        for (uint32_t i0 = 0; i0 < some; i0 += 64) {
            uint32_t s0 = 0, k = 0;
            if (i0 + lane < some) {
                const uint32_t c = ids[i0 + lane];
                s0 = sj[c];
                k = sj[c + 1] - s0;
            }
            uint32_t total;
            uint32_t to = at + scan(k, total);
            // never past the row's own length
            k = to < len ? min(k, len - to) : 0u;
            at += total;
            if (RUNS) {
                const uint32_t m = min(64u, some - i0);
                for (uint32_t q0 = 0; q0 < m; q0 += 4) {
                    uint32_t v[4], longest = 0;
#pragma unroll
                    for (uint32_t q = 0; q < 4; ++q) {
                        const uint32_t kk = q0 + q < m ? __builtin_amdgcn_readlane(k, q0 + q) : 0u;
                        longest = max(longest, kk);
                        v[q] = lane < kk ? nj[__builtin_amdgcn_readlane(s0, q0 + q) + lane] : 0u;
                    }
#pragma unroll
                    for (uint32_t q = 0; q < 4; ++q) {
                        const uint32_t kk = q0 + q < m ? __builtin_amdgcn_readlane(k, q0 + q) : 0u;
                        if (lane < kk) out[__builtin_amdgcn_readlane(to, q0 + q) + lane] = v[q];
                    }
                    if (longest <= 64) continue;
                    for (uint32_t q = 0; q < 4 && q0 + q < m; ++q) {
                        const uint32_t kk = __builtin_amdgcn_readlane(k, q0 + q);
                        const uint32_t from = __builtin_amdgcn_readlane(s0, q0 + q);
                        const uint32_t dst = __builtin_amdgcn_readlane(to, q0 + q);
                        for (uint32_t i = 64 + lane; i < kk; i += 64) out[dst + i] = nj[from + i];
                    }
                }
            } else {
                for (uint32_t i = 0; i < k; ++i) out[to + i] = nj[s0 + i];
            }
        }
    }
}

// What a wavefront needs of a node's lists: lane j < H holds the descriptor
// of its row in hash j.  The lists of left-out nodes are read in chunks of 64
// entries; lane t gets where chunk t0 + t starts and how many it has.
constexpr uint32_t kListHashes = 16;
struct Chunks {
    uint32_t offset, len, before, count;  // the lane's list, the chunks before it; all chunks
    bool single;  // no list has more than 64 entries: chunk t is list t
    __device__ __forceinline__ explicit Chunks(uint2 d) {
        offset = d.x;
        len = d.y >> 30 == kRowOut ? d.y : 0u;
        single = __ballot(len > 64) == 0;
        before = 0;
        count = kListHashes;
        if (single) return;
        const uint32_t mine = (len + 63) / 64;
        uint32_t upto = mine;
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)upto, off, 16);
            if ((int)(threadIdx.x & 15u) >= off) upto += y;
        }
        before = upto - mine;
        count = (uint32_t)__builtin_amdgcn_readlane((int)upto, 15);
    }
    __device__ __forceinline__ void at(uint32_t t0, uint32_t &from, uint32_t &entries) const {
        const uint32_t t = t0 + (threadIdx.x & 63u);
        from = offset;
        entries = len;
        if (single) return;
        from = entries = 0;
#pragma unroll
        for (uint32_t j = 0; j < kListHashes; ++j) {
            const uint32_t c0 = (uint32_t)__builtin_amdgcn_readlane((int)before, (int)j);
            const uint32_t l = (uint32_t)__builtin_amdgcn_readlane((int)len, (int)j);
            const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)offset, (int)j);
            const uint32_t k = t - c0;  // chunk of this list
            if (t >= c0 && 64 * k < l) {
                from = o + 64 * k;
                entries = min(64u, l - 64 * k);
            }
        }
    }
};

// The estimates of intersection nodes, a wavefront (a workgroup) each: 64 nodes
// of the shortest list at a time against 4 hashes at a time, until none is left.
// Bound by the latency of a node's chain of reads, hidden by 32 wavefronts a CU.
constexpr uint32_t kBatch = 8;
__global__ void __launch_bounds__(64)
k_fuse_inter(uint32_t n, uint32_t H, uint32_t K, int64_t ldK, const uint64_t *__restrict__ P,
             const uint32_t *__restrict__ bucket, const uint8_t *__restrict__ cls,
             const uint2 *__restrict__ rows, const uint32_t *__restrict__ lists,
             int32_t *__restrict__ est) {
    const uint32_t lane = threadIdx.x;
    // 64 classes at a time
    for (uint32_t u0 = blockIdx.x * 64; u0 < n; u0 += gridDim.x * 64) {
        uint64_t some = __ballot(u0 + lane < n && cls[u0 + lane] == kNodeInter);
        for (; some; some &= some - 1) {
            const uint32_t u = u0 + __builtin_ctzll(some);
            const uint32_t bu = lane < H ? bucket[(size_t)lane * n + u] : 0u;
            uint2 d = make_uint2(0u, 0u);
            if (lane < H) d = rows[(size_t)lane * K + bu];
            uint32_t mine = 0;
        // the shortest list of kept nodes
        uint32_t key = d.y >> 30 == kRowKept ? (d.y & 0x3fffffffu) << 4 | lane : 0xffffffffu;
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) key = min(key, (uint32_t)__shfl_xor(key, off, 16));
        key = __builtin_amdgcn_readfirstlane(key);
        const uint32_t js = key & 15u, len = key >> 4;
        const uint32_t o = __builtin_amdgcn_readlane(d.x, js);
        for (uint32_t i0 = 0; i0 < len; i0 += 64) {
            const uint32_t w = i0 + lane < len ? lists[o + i0 + lane] : 0xffffffffu;
            bool alive = w < n;
            // the other hashes, from the one after js on
            for (uint32_t k0 = 1; k0 < H; k0 += 4) {
                uint32_t hb[4];
                uint64_t x[4];
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k) {
                    const uint32_t j = (js + k0 + k) % H;
                    hb[k] = alive && k0 + k < H ? bucket[(size_t)j * n + w] : 0u;
                }
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k) {
                    const uint32_t j = (js + k0 + k) % H;
                    const size_t r = (size_t)j * K + __builtin_amdgcn_readlane(bu, j);
                    x[k] = alive && k0 + k < H ? P[r * ldK + (hb[k] >> 6)] >> (hb[k] & 63u) : 1ull;
                }
                alive = alive && (x[0] & x[1] & x[2] & x[3] & 1ull);
                if (__ballot(alive) == 0) break;
            }
            mine += alive ? 1u : 0u;
        }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off, 64);
            if (lane == 0) est[u] = (int32_t)mine;
        }
    }
}

// The estimates of small union nodes, one wavefront (one workgroup) per node at
// a time, where a bitmap of n bits leaves room for a few wavefronts on a CU
// (n <= kMarkBits): an entry is marked by an atomic OR whose old word tells a
// node met before.
//
// A node passes five stages, one a turn, every load of which is unconditional
// and has a whole turn to arrive: its number; its buckets; its rows' descriptors;
// the map of its lists' chunks of 64 entries (chunk t in lane t) and the loads of
// the first kMarkSlots; the marks.  A lane past a chunk's end (entries of other
// lists, or past the last list) marks no bit.  Four nodes are in hand, and the
// number of a fifth, so the turns are written out by fours, each node staying in
// its registers.
//
// Bound by vector instructions (300 a node; 1143 with a hash table of 8 KB by
// compare-and-swap, whatever the wavefronts) and the latency that 6 wavefronts a
// CU (n = 2*10^5) leave.  185,000 nodes of 160 to 2560 entries and the 15,000 wider
// ones take 0.39 ms there; with the table (to 1024 entries) and the wide nodes'
// workgroups for the rest it was 0.75.  24 slots 0.34 where 16 take 0.32.
constexpr uint32_t kMarkSlots = 16;
struct MarkNode {
    uint32_t u, b;       // the node; the lane's bucket
    uint2 d;             // the lane's row
    uint32_t from, len;  // chunk `lane`
    uint32_t count;      // chunks
};
__global__ void __launch_bounds__(64)
k_fuse_marked(uint32_t n, uint32_t H, uint32_t K, const uint32_t *__restrict__ bucket,
              const uint32_t *__restrict__ small, uint32_t nsmall, const uint2 *__restrict__ rows,
              const uint32_t *__restrict__ lists, int32_t *__restrict__ est) {
    extern __shared__ __align__(16) uint32_t htab[];
    const uint32_t lane = threadIdx.x, G = gridDim.x, words = ((n + 127) / 128) * 4;
    auto clear = [&] {
        for (uint32_t i = 4 * lane; i < words; i += 256)
            *(uint4 *)(htab + i) = make_uint4(0u, 0u, 0u, 0u);
    };
    clear();
    const uint32_t hash = lane < H ? lane : 0u;
    const uint32_t *const mine = bucket + (size_t)hash * n;
    const uint2 *const desc = rows + (size_t)hash * K;
    // (past the list's end the last node again, of no chunk then)
    auto number = [&](uint32_t i) { return small[min(i, nsmall - 1)]; };
    auto buckets = [&](uint32_t u, MarkNode &x) {
        x.u = u;
        x.b = mine[u];
    };
    auto descriptors = [&](MarkNode &x) { x.d = desc[x.b]; };
    // chunk t of the node's lists goes to lane t
    auto chunks = [&](uint32_t i, MarkNode &x) {
        const uint32_t l = i < nsmall && lane < H && x.d.y >> 30 == kRowOut ? x.d.y : 0u;
        const uint32_t parts = (l + 63) / 64;
        uint32_t upto = parts;
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)upto, off, 16);
            if ((int)(lane & 15u) >= off) upto += y;
        }
        x.count = (uint32_t)__builtin_amdgcn_readlane((int)upto, 15);
        const uint32_t first = upto - parts;
        x.from = x.len = 0;
        for (uint32_t k = 0; __ballot(k < parts); ++k) {
            // a lane without a chunk k pushes nothing, to the last lane (there
            // are fewer chunks than lanes)
            const bool has = k < parts;
            const int to = (int)(has ? 4 * (first + k) : 4 * 63u);
            x.from += (uint32_t)__builtin_amdgcn_ds_permute(to, (int)(has ? x.d.x + 64 * k : 0u));
            x.len += (uint32_t)__builtin_amdgcn_ds_permute(to, (int)(has ? min(64u, l - 64 * k) : 0u));
        }
    };
    auto entry = [&](const MarkNode &x, uint32_t t) {
        return (lists + (uint32_t)__builtin_amdgcn_readlane((int)x.from, (int)t))[lane];
    };
    // the marks of 8 chunks from t on, and the words marked; adds the entries
    // and those met before
    auto mark = [&](const MarkNode &x, uint32_t t, const uint32_t *w, uint32_t *at, uint32_t &all,
                    uint32_t &again) {
        uint32_t bit[8], old[8];
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k) {
            const uint32_t l = (uint32_t)__builtin_amdgcn_readlane((int)x.len, (int)(t + k));
            const uint32_t v = min(w[k], n - 1);
            all += l;
            at[k] = v >> 5;
            bit[k] = lane < l ? 1u << (v & 31u) : 0u;
            old[k] = atomicOr(htab + at[k], bit[k]);
        }
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k) again += (uint32_t)__popcll(__ballot(old[k] & bit[k]));
    };
    uint32_t ahead;  // the node of the turn after `last`
    auto turn = [&](uint32_t i, MarkNode &now, MarkNode &next, MarkNode &third, MarkNode &last,
                    uint32_t *w, uint32_t *wn) {
        chunks(i + G, next);
#pragma unroll
        for (uint32_t t = 0; t < kMarkSlots; ++t) wn[t] = entry(next, t);
        descriptors(third);
        buckets(ahead, last);
        ahead = number(i + 4 * G);
        uint32_t at[kMarkSlots], all = 0, again = 0;
#pragma unroll
        for (uint32_t t = 0; t < kMarkSlots; t += 8) mark(now, t, w + t, at + t, all, again);
        if (now.count > kMarkSlots) {
            for (uint32_t t = kMarkSlots; t < now.count; t += 8) {
                uint32_t x[8], words[8];
#pragma unroll
                for (uint32_t k = 0; k < 8; ++k) x[k] = entry(now, t + k);
                mark(now, t, x, words, all, again);
            }
            clear();
        } else {
#pragma unroll
            for (uint32_t t = 0; t < kMarkSlots; ++t) htab[at[t]] = 0u;
        }
        if (lane == 0) est[now.u] = (int32_t)(n - (all - again));
    };
    MarkNode a, b, c, d;
    uint32_t w0[kMarkSlots], w1[kMarkSlots];
    uint32_t i = blockIdx.x;
    buckets(number(i), a);
    buckets(number(i + G), b);
    descriptors(a);
    buckets(number(i + 2 * G), c);
    descriptors(b);
    ahead = number(i + 3 * G);
    chunks(i, a);
#pragma unroll
    for (uint32_t t = 0; t < kMarkSlots; ++t) w0[t] = entry(a, t);
    for (;;) {
        turn(i, a, b, c, d, w0, w1);
        if ((i += G) >= nsmall) break;
        turn(i, b, c, d, a, w1, w0);
        if ((i += G) >= nsmall) break;
        turn(i, c, d, a, b, w0, w1);
        if ((i += G) >= nsmall) break;
        turn(i, d, a, b, c, w1, w0);
        if ((i += G) >= nsmall) break;
    }
}

// The same where n bits are too many: entries go into a hash table of 8 KB by
// compare-and-swap (at most half full: kSmallHashed entries), kBatch chunks in
// flight, 20 wavefronts a CU.  147,000 nodes of 600 entries took 0.53 ms here
// (n = 2*10^5; 0.21 by marks).
__global__ void __launch_bounds__(64)
k_fuse_hashed(uint32_t n, uint32_t H, uint32_t K,
             const uint32_t *__restrict__ bucket, const uint8_t *__restrict__ cls,
             const uint2 *__restrict__ rows, const uint32_t *__restrict__ lists,
             int32_t *__restrict__ est) {
    extern __shared__ __align__(16) uint32_t htab[];
    const uint32_t lane = threadIdx.x;
    const uint32_t none = 0xffffffffu, words = kHashSlots;
    auto clear = [&] {
        for (uint32_t i = 4 * lane; i < words; i += 256)
            *(uint4 *)(htab + i) = make_uint4(none, none, none, none);
    };
    clear();
    __syncthreads();  // one wavefront: orders its LDS accesses
    auto buckets = [&](uint32_t u, uint32_t &b, uint32_t &c) {
        c = u < n ? cls[u] : (uint32_t)kNodeDone;
        b = u < n && lane < H ? bucket[(size_t)lane * n + u] : 0u;
    };
    uint32_t b, c;
    buckets(blockIdx.x, b, c);
    for (uint32_t u = blockIdx.x; u < n; u += gridDim.x) {
        const uint32_t bu = b, cu = __builtin_amdgcn_readfirstlane(c);
        uint2 d = make_uint2(0u, 0u);
        if (cu == kNodeSmall && lane < H) d = rows[(size_t)lane * K + bu];
        buckets(n - u > gridDim.x ? u + gridDim.x : n, b, c);
        uint32_t mine = 0;
        if (cu == kNodeSmall) {
            const Chunks ch(d);
            for (uint32_t t0 = 0; t0 < ch.count; t0 += 64) {
                uint32_t from, entries;
                ch.at(t0, from, entries);
                const uint32_t some = min(64u, ch.count - t0);
                for (uint32_t q0 = 0; q0 < some; q0 += kBatch) {
                    uint32_t w[kBatch];
#pragma unroll
                    for (uint32_t q = 0; q < kBatch; ++q) {
                        w[q] = 0xffffffffu;
                        if (q0 + q < some) {
                            const uint32_t o = __builtin_amdgcn_readlane(from, q0 + q);
                            if (lane < (uint32_t)__builtin_amdgcn_readlane(entries, q0 + q))
                                w[q] = lists[o + lane];
                        }
                    }
#pragma unroll
                    for (uint32_t h = 0; h < kBatch; h += 4) {
                        uint32_t at[4];
                        bool open[4];
#pragma unroll
                        for (uint32_t k = 0; k < 4; ++k) {
                            at[k] = (w[h + k] * 2654435761u) >> 21;
                            open[k] = w[h + k] < n;
                        }
                        while (__ballot(open[0] | open[1] | open[2] | open[3])) {
                            uint32_t old[4];
#pragma unroll
                            for (uint32_t k = 0; k < 4; ++k)
                                if (open[k]) old[k] = atomicCAS(htab + at[k], none, w[h + k]);
#pragma unroll
                            for (uint32_t k = 0; k < 4; ++k)
                                if (open[k]) {
                                    mine += old[k] == none ? 1u : 0u;
                                    open[k] = old[k] != none && old[k] != w[h + k];
                                    at[k] = (at[k] + 1) & (kHashSlots - 1);
                                }
                        }
                    }
                }
            }
            __syncthreads();
            clear();
            __syncthreads();
        } else {
            continue;
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off, 64);
        if (lane == 0) est[u] = (int32_t)(n - mine);
    }
}

// The estimates of wide union nodes, one workgroup per node at a time: the
// bitmaps of its rows are ORed into one in LDS, 16 bytes a thread, then its
// lists marked there, the chunks dealt to the wavefronts, kBatch in flight
// each.  Bound by the bitmaps' reads (n / 8 bytes each, from L2 where nodes
// of a bucket share them) and the latency of the lists'; n bits of LDS limit
// the nodes at work on a CU, so a workgroup has as many wavefronts as fill it
// (launch_fuse_lists): 53,000 nodes of 1400 entries (n = 2*10^5) in 0.22 ms.
__global__ void __launch_bounds__(1024)
k_fuse_wide(uint32_t n, uint32_t H, uint32_t K, const uint32_t *__restrict__ bucket,
            const uint2 *__restrict__ rows, const uint32_t *__restrict__ lists,
            const uint64_t *__restrict__ bitmaps, const uint32_t *__restrict__ list, uint32_t nlist,
            int32_t *__restrict__ est) {
    extern __shared__ __align__(16) uint32_t bm[];
    __shared__ uint32_t sums[2];
    const uint32_t tid = threadIdx.x, T = blockDim.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = T >> 6;
    const uint32_t nw = (n + 63) / 64;
    uint64_t *bm64 = (uint64_t *)bm;
    if (tid < 2) sums[tid] = 0;
    uint32_t turn = 0;
    __syncthreads();
    for (uint32_t i = blockIdx.x; i < nlist; i += gridDim.x) {
        const uint32_t u = list[i];
        uint2 d = make_uint2(0u, 0u);
        if (lane < H) d = rows[(size_t)lane * K + bucket[(size_t)lane * n + u]];
        const uint32_t maps = (uint32_t)__ballot(d.y >> 30 == kRowBits);
        uint32_t mine = 0;
        for (uint32_t k0 = tid; k0 < nw; k0 += 4 * T) {
            uint64_t x[4] = {};
            for (uint32_t rest = maps; rest; rest &= rest - 1u) {
                const uint64_t *m =
                    bitmaps + (size_t)(uint32_t)__builtin_amdgcn_readlane(d.x, __builtin_ctz(rest)) * nw;
                uint64_t y[4];
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) y[q] = k0 + q * T < nw ? m[k0 + q * T] : 0ull;
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) x[q] |= y[q];
            }
#pragma unroll
            for (uint32_t q = 0; q < 4; ++q)
                if (k0 + q * T < nw) {
                    bm64[k0 + q * T] = x[q];
                    mine += (uint32_t)__popcll(x[q]);
                }
        }
        const Chunks ch(d);
        __syncthreads();
        for (uint32_t t0 = 0; t0 < ch.count; t0 += 64) {
            uint32_t from, entries;
            ch.at(t0, from, entries);
            const uint32_t some = min(64u, ch.count - t0);
            for (uint32_t q0 = wave; q0 < some; q0 += kBatch * waves) {
                uint32_t w[kBatch];
#pragma unroll
                for (uint32_t q = 0; q < kBatch; ++q) {
                    const uint32_t t = q0 + q * waves;
                    w[q] = 0xffffffffu;
                    if (t < some) {
                        const uint32_t o = __builtin_amdgcn_readlane(from, t);
                        if (lane < (uint32_t)__builtin_amdgcn_readlane(entries, t)) w[q] = lists[o + lane];
                    }
                }
#pragma unroll
                for (uint32_t q = 0; q < kBatch; ++q)
                    if (w[q] < n) {
                        const uint32_t bit = 1u << (w[q] & 31u);
                        mine += (atomicOr(bm + (w[q] >> 5), bit) & bit) ? 0u : 1u;
                    }
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off, 64);
        // two sums in turn: the other one is cleared while this one is read
        if (lane == 0) atomicAdd(&sums[turn], mine);
        __syncthreads();  // and the bitmap may be written again
        if (tid == 0) {
            est[u] = (int32_t)(n - sums[turn]);
            sums[turn ^ 1u] = 0;
        }
        turn ^= 1u;
    }
}

uint32_t grid_for(size_t items, uint32_t per_block, uint32_t cap = 65536) {
    size_t g = (items + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (uint32_t)g;
}

}  // namespace

hipError_t launch_hash_buckets(uint32_t n, uint32_t H, const uint64_t *coeffs, int order, uint32_t K,
                               uint32_t *bucket, int32_t *count, hipStream_t st) {
    const size_t total = (size_t)n * H;
    hipLaunchKernelGGL(k_hash_buckets, dim3(grid_for(total, 256)), dim3(256), 0, st, n, H, coeffs,
                       order, K, bucket);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_zero_i32, dim3(grid_for((size_t)H * K, 256)), dim3(256), 0, st, count,
                       (size_t)H * K);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bucket_counts, dim3(grid_for(total, 256)), dim3(256), 0, st, n, H, K,
                       bucket, count);
    return hipGetLastError();
}

hipError_t launch_transpose_proxies(uint32_t H, uint32_t K, int64_t ldK, const uint64_t *P,
                                    uint64_t *PT, hipStream_t st) {
    const size_t kw = (K + 63) / 64;
    const size_t runs = (kw + kLiftRun - 1) / kLiftRun;
    hipLaunchKernelGGL(k_transpose_proxies, dim3(grid_for((size_t)H * kw * runs * 64, 256)), dim3(256),
                       0, st, H, K, ldK, P, PT);
    return hipGetLastError();
}

hipError_t launch_row_sums(uint32_t H, uint32_t K, int64_t ldK, const uint64_t *P,
                           const int32_t *count, int32_t *bsum, int2 *rowsum, hipStream_t st) {
    const size_t kw = (K + 63) / 64;
    hipLaunchKernelGGL(k_block_sums, dim3(grid_for((size_t)H * kw * 64, 256)), dim3(256), 0, st, H, K,
                       count, bsum);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_row_sums, dim3(grid_for((size_t)H * K * 64, 256)), dim3(256), 0, st, H, K, ldK,
                       P, count, bsum, rowsum);
    return hipGetLastError();
}

static size_t fuse_wide_lds(uint32_t n) { return ((size_t)n + 63) / 64 * 8; }

bool fuse_lists_fit(uint32_t n, uint32_t H, uint32_t K) {
    return n >= kListMinN && H <= kListHashes && K <= kListMaxK && fuse_wide_lds(n) + 64 <= kRecombineLds;
}

size_t fuse_hist_words(uint32_t H, uint32_t K) { return (size_t)H * kListSplit * K; }

hipError_t launch_classify(uint32_t n, uint32_t H, uint32_t K, const uint32_t *bucket,
                           const int32_t *count, const int2 *rowsum,
                           int32_t *lifted, bool lists, uint8_t *cls, int32_t *est,
                           uint32_t *open, uint32_t *wide, unsigned long long *stats,
                           hipStream_t st) {
    hipLaunchKernelGGL(k_zero_i32, dim3(1), dim3(64), 0, st, (int32_t *)stats,
                       (size_t)2 * (lists ? kFuseWords : 1));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // a wavefront a workgroup spreads few nodes, more keep them in order for the
    // estimates' reads (us a call without lists, 64 and 256 threads: 4,000 nodes,
    // 16 hashes 113.4 and 115.3; 11,843 278.7 and 275.5; 20,009 308.9 and 306.9)
    const uint32_t threads = lists || n >= 8192 ? 256 : 64;
    auto k = H <= 8 ? (lists ? k_classify<true, 8> : k_classify<false, 8>)
                    : (lists ? k_classify<true, 16> : k_classify<false, 16>);
    const uint32_t groups = grid_for(n, threads, lists ? 1024 : 512) + (lists ? kTotalParts * H : 0u);
    hipLaunchKernelGGL(k, dim3(groups), dim3(threads), 0, st, n, H, K, bucket, count, rowsum,
                       lifted, cls, est, open, wide, stats);
    return hipGetLastError();
}

hipError_t launch_fuse_lists(uint32_t n, uint32_t H, uint32_t K, int64_t ldK, const uint64_t *P,
                             const uint32_t *bucket, const int32_t *count, const int2 *rowsum,
                             const uint8_t *cls, const unsigned long long *stats, FuseScratch s,
                             uint32_t nbitmaps, const uint32_t *wide,
                             const unsigned long long *stats_host, int32_t *est, hipStream_t st) {
    uint32_t *lists = (uint32_t *)(s.bitmaps + (size_t)nbitmaps * ((n + 63) / 64));
    size_t lds = (size_t)K * 4;
    for (const void *k : {(const void *)k_bucket_hist, (const void *)k_bucket_nodes}) {
        hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_bucket_hist, dim3(kListSplit, H), dim3(512), lds, st, n, K, bucket, s.hist);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bucket_starts, dim3(H), dim3(1024), 0, st, K, s.hist, s.start);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bucket_nodes, dim3(kListSplit, H), dim3(512), lds, st, n, K, bucket, s.hist,
                       s.nodes);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_list_starts, dim3(H), dim3(1024), 0, st, n, K, count, rowsum, stats, s.rows,
                       s.bitmap_row);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    auto fill = n / K >= 16 ? k_fill_lists<true> : k_fill_lists<false>;
    hipLaunchKernelGGL(fill, dim3(H * K), dim3(64), 0, st, n, H, K, ldK, P, s.start, s.nodes, s.rows,
                       lists);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (stats_host[kFuseInter]) {
        hipLaunchKernelGGL(k_fuse_inter, dim3(grid_for(n, 64, 256 * 32)), dim3(64), 0, st, n, H, K, ldK,
                           P, bucket, cls, s.rows, lists, est);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const uint32_t nsmall = (uint32_t)stats_host[kFuseSmall], nwide = (uint32_t)stats_host[kFuseWide];
    if (nsmall && n <= kMarkBits) {
        lds = ((size_t)n + 127) / 128 * 16;
        const uint32_t per_cu = (uint32_t)std::min<size_t>(kRecombineLds / lds, 20);
        hipLaunchKernelGGL(k_fuse_marked, dim3(grid_for(nsmall, 1, 256 * per_cu)), dim3(64), lds, st, n,
                           H, K, bucket, wide + n - nsmall, nsmall, s.rows, lists, est);
    } else if (nsmall) {
        lds = kHashSlots * 4;
        const uint32_t per_cu = (uint32_t)std::min<size_t>(kRecombineLds / lds, 32);
        hipLaunchKernelGGL(k_fuse_hashed, dim3(grid_for(n, 1, 256 * per_cu)), dim3(64), lds, st, n, H, K,
                           bucket, cls, s.rows, lists, est);
    }
    e = hipGetLastError();
    if (e != hipSuccess || nwide == 0) return e;
    if (nbitmaps) {
        const uint32_t splits = std::max(1u, std::min(n / 1024, 4096u / nbitmaps));
        hipLaunchKernelGGL(k_fill_bitmaps, dim3(nbitmaps, splits), dim3(256), 0, st, n, K, ldK, P,
                           bucket, s.bitmap_row, s.bitmaps);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    lds = fuse_wide_lds(n);
    e = hipFuncSetAttribute((const void *)k_fuse_wide, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds);
    if (e != hipSuccess) return e;
    // as many bitmaps as a CU's LDS holds, at most 16, and about 24 wavefronts
    // over them
    const uint32_t fit = (uint32_t)std::min<size_t>(kRecombineLds / (lds + 64), 16);
    uint32_t threads = 64;
    while (threads < 1024 && fit * threads < 24 * 64) threads *= 2;
    const uint32_t resident = std::min(fit, 2048u / threads);
    hipLaunchKernelGGL(k_fuse_wide, dim3(grid_for(nwide, 1, 256 * resident)), dim3(threads), lds, st, n,
                       H, K, bucket, s.rows, lists, s.bitmaps, wide, nwide, est);
    return hipGetLastError();
}

hipError_t launch_build_lifted(uint32_t n, uint32_t H, uint32_t K, int64_t ldK, const uint64_t *PT,
                               const uint32_t *bucket, uint32_t q0, uint32_t nq, uint64_t *Lt,
                               hipStream_t st) {
    const size_t kw = (K + 63) / 64;
    const size_t runs = (kw + kLiftRun - 1) / kLiftRun;
    hipLaunchKernelGGL(k_build_lifted, dim3(grid_for((size_t)nq * H * runs * 64, 256)), dim3(256), 0,
                       st, n, H, K, ldK, PT, bucket, q0, nq, Lt);
    return hipGetLastError();
}

// Hashes whose chunk tables fit in LDS together (at most 4); 0 when one
// table does not fit, and the tables are read from global memory.
uint32_t recombine_group(uint32_t K) {
    const size_t budget = kRecombineLds;
    size_t g = budget / ((size_t)K * 8);
    if (g > 4) g = 4;
    return (uint32_t)g;
}

hipError_t launch_recombine_est(uint32_t n, uint32_t H, uint32_t K, const uint32_t *bucket,
                                const uint64_t *Lt, uint32_t q0, uint32_t nq, const uint32_t *list,
                                uint32_t nlist, int32_t *est, hipStream_t st) {
    const uint32_t GL = recombine_group(K);
    const bool in_lds = GL > 0;
    const uint32_t G = in_lds ? GL : 4u;
    // two copies of the tables of GB hashes when they fit (the next stage
    // streams in while this one is read), else one copy of G hashes, else
    // the tables are read where they are
    const uint32_t GB = (size_t)K * 8 * 2 * 2 <= kRecombineLds ? 2u
                      : (size_t)K * 8 * 2 <= kRecombineLds  ? 1u
                                                            : 0u;
    const size_t lds = GB ? (size_t)2 * GB * K * 8 : in_lds ? (size_t)G * K * 8 : 0;
    const void *kern = GB == 2 ? (const void *)k_recombine_est2<2>
                     : GB == 1 ? (const void *)k_recombine_est2<1>
                     : in_lds  ? (const void *)k_recombine_est<true>
                               : (const void *)k_recombine_est<false>;
    hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const uint32_t threads = kRecombineThreads;
    const uint32_t utiles = (uint32_t)((nlist + (size_t)threads * kUPT - 1) / ((size_t)threads * kUPT));
    if (utiles == 0) return hipSuccess;
    // split the chunk range over the second grid dimension so that the
    // launch has enough workgroups
    uint32_t splits = 1;
    while ((size_t)utiles * splits < 1024 && splits * kQB * 2 <= nq) splits *= 2;
    const uint32_t per = ((nq + splits - 1) / splits + kQB - 1) / kQB * kQB;
    splits = (nq + per - 1) / per;
    if (GB == 2)
        hipLaunchKernelGGL(k_recombine_est2<2>, dim3(utiles * splits), dim3(threads), lds, st, n, H,
                           K, bucket, Lt, q0, q0 + nq, per, q0, list, nlist, utiles, est);
    else if (GB == 1)
        hipLaunchKernelGGL(k_recombine_est2<1>, dim3(utiles * splits), dim3(threads), lds, st, n, H,
                           K, bucket, Lt, q0, q0 + nq, per, q0, list, nlist, utiles, est);
    else if (in_lds)
        hipLaunchKernelGGL(k_recombine_est<true>, dim3(utiles * splits), dim3(threads), lds, st, n,
                           H, K, G, bucket, Lt, q0, q0 + nq, per, q0, list, nlist, utiles, est);
    else
        hipLaunchKernelGGL(k_recombine_est<false>, dim3(utiles * splits), dim3(threads), lds, st, n,
                           H, K, G, bucket, Lt, q0, q0 + nq, per, q0, list, nlist, utiles, est);
    return hipGetLastError();
}

}  // namespace tn
