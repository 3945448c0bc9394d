// Launchers of the hashing and fusion kernels (tn_hash.hip).
#pragma once

#include "tn_internal.h"

namespace tn {

// Nodes whose bitmap leaves room for four on a CU (k_fuse_marked).
constexpr uint32_t kMarkBits = 327680;

hipError_t launch_hash_buckets(uint32_t n, uint32_t H, const uint64_t *coeffs, int order, uint32_t K,
                               uint32_t *bucket, int32_t *count, hipStream_t st);
hipError_t launch_transpose_proxies(uint32_t H, uint32_t K, int64_t ldK, const uint64_t *P,
                                    uint64_t *PT, hipStream_t st);
// rowsum[j K + r] = {the nodes that row r of P_j lifts to: the sum of count[j] over
// the super-nodes set in it, 1 iff the row is full} (bsum: scratch of H
// ceil(K/64) int32).  One pair, so that a node's row takes one read.
hipError_t launch_row_sums(uint32_t H, uint32_t K, int64_t ldK, const uint64_t *P,
                           const int32_t *count, int32_t *bsum, int2 *rowsum, hipStream_t st);
hipError_t launch_build_lifted(uint32_t n, uint32_t H, uint32_t K, int64_t ldK, const uint64_t *PT,
                               const uint32_t *bucket, uint32_t q0, uint32_t nq, uint64_t *Lt,
                               hipStream_t st);
// Fusion by lists (tn_hash.hip).  Totals of a call, uint64 on the device:
enum : int {
    kFuseOpen = 0,      // nodes some row of which is not full
    kFuseWide = 1,      // ... the wide union nodes among them
    kFuseEntries = 2,   // list entries and bitmaps that the union nodes read
    kFuseBits = 3,
    kFuseInter = 4,     // entries of the intersection nodes' shortest lists
    kFuseNodeMix = 5,   // sums that agree where the counts are the buckets' own
    kFuseCountMix = 6,
    kFuseSmall = 7,     // the small union nodes
    kFuseRows = 8,      // entries of each hash's lists, up to 16 hashes, and bitmaps
    kFuseStats = 8 + 2 * 16,
    // parts of kFuseEntries .. kFuseInter, kFuseNodeMix and kFuseCountMix, which
    // the host adds up: kFuseParts of 64 bytes after the rest (hundreds of
    // workgroups' atomics on one word took as long as the kernel's work)
    kFuseParts = 32,
    kFuseWords = kFuseStats + 8 * kFuseParts
};
struct FuseScratch {
    uint32_t *hist;        // fuse_hist_words
    uint32_t *start;       // H (K + 1)
    uint32_t *nodes;       // H n
    uint2 *rows;           // H K
    uint32_t *bitmap_row;  // H K
    uint64_t *bitmaps;     // the sum of stats[kFuseRows + 16 ..], of ceil(n/64) words, then
                           // the lists' entries (uint32, the sum of stats[kFuseRows ..])
};
// whether the lists' kernels take this size (kListMinN nodes and more, up to 16
// hashes, LDS for K counters and n bits)
bool fuse_lists_fit(uint32_t n, uint32_t H, uint32_t K);
size_t fuse_hist_words(uint32_t H, uint32_t K);
// cls[u] (the node's kind), lifted[j n + u] = rowsum[j K + h_j(u)].x (nullable),
// est[u] = n where every row is full, else 0 and u in open[0 ..
// stats[kFuseOpen]); the wide nodes in wide[0 .. stats[kFuseWide]), the small
// ones in the last stats[kFuseSmall] of wide's n; with lists also the rows'
// totals.
hipError_t launch_classify(uint32_t n, uint32_t H, uint32_t K, const uint32_t *bucket,
                           const int32_t *count, const int2 *rowsum,
                           int32_t *lifted, bool lists, uint8_t *cls, int32_t *est,
                           uint32_t *open, uint32_t *wide, unsigned long long *stats,
                           hipStream_t st);
// The estimates of union and intersection nodes (stats_host: stats' values).
hipError_t launch_fuse_lists(uint32_t n, uint32_t H, uint32_t K, int64_t ldK, const uint64_t *P,
                             const uint32_t *bucket, const int32_t *count, const int2 *rowsum,
                             const uint8_t *cls, const unsigned long long *stats, FuseScratch s,
                             uint32_t nbitmaps, const uint32_t *wide,
                             const unsigned long long *stats_host, int32_t *est, hipStream_t st);
hipError_t launch_recombine_est(uint32_t n, uint32_t H, uint32_t K, const uint32_t *bucket,
                                const uint64_t *Lt, uint32_t q0, uint32_t nq, const uint32_t *list,
                                uint32_t nlist, int32_t *est, hipStream_t st);
uint32_t recombine_group(uint32_t K);

}  // namespace tn
