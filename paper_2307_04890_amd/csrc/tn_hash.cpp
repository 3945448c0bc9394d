// C ABI of network hashing (Sec. 4.1) and fusion (Sec. 4.2).
#include <algorithm>
#include <chrono>
#include <atomic>
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "tn_batch.h"
#include "tn_hash.h"
#include "tn_column.h"

namespace {
constexpr uint64_t kP61 = (1ull << 61) - 1;
constexpr size_t kLiftedBudget = (size_t)1 << 30;  // bytes of lifted tables per pass
inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Whether fusion by lists beats the tables, from the call's totals: the
// microseconds of either as fitted on calls of n = 10^4 to 3*10^5 nodes and H = 5
// to 16 hashes (lists against tables, H = 16, K = 4096 and activity-driven
// events unless said: n = 2*10^5 with m/n = 0.2 and 0.15 events per node 0.66
// against 5.80 and 4.59 against 5.73 ms; n = 6*10^4, K = 2048, 0.33 0.21 against
// 0.59, K = 4096 3.97 against 0.96; n = 10^5, 0.3 2.07 against 1.79, H = 5, 0.4
// 0.30 against 0.63; n = 10^4, H = 8, K = 512, 0.4 0.142 against 0.105).  The
// tables cost their building and staging (n H K) and n / 64 words of each hash
// per open node; the lists' side is the setup per row and entry, the union
// nodes' entries and bitmaps (more where a node takes a hash table, past
// kMarkBits nodes), and the random reads of intersections.  Below
// kListMinN nodes the lists gain little (n = 10^4, H = 16, K = 512 0.106 against
// 0.116 ms) or lose (n = 2*10^4, 0.43 against 0.33).
bool fuse_by_lists(uint32_t n, uint32_t H, uint32_t K, const unsigned long long *stats,
                   unsigned long long entries, unsigned long long nbitmaps, size_t room) {
    using namespace tn;
    // the lists take their lengths from the counts, and their room from the tables'
    if (stats[kFuseNodeMix] != stats[kFuseCountMix]) return false;
    // (64 entries more: the last list's chunk is read whole)
    if ((entries + 64) * 4 + nbitmaps * ((n + 63) / 64) * 8 > room) return false;
    const double N = n, rows = (double)H * K, open = (double)stats[kFuseOpen];
    const bool marked = n <= kMarkBits;
    const double tables = 105 + 78e-9 * N * rows + 7.3e-9 * open * N * H;
    const double lists = 100 + 8e-4 * rows + 8e-6 * (double)entries + 0.5e-6 * (double)nbitmaps * N +
                         (marked ? 1.3e-6 : 1.7e-6) * (double)stats[kFuseEntries] +
                         (marked ? 0.9e-3 : 2.5e-3) * open +
                         1.25e-8 * (double)stats[kFuseBits] * N + 1e-4 * (double)stats[kFuseInter];
    return lists < tables;
}
}  // namespace

extern "C" {

tn_status tn_hash_compress(tn_ctx *ctx, uint32_t n, int64_t m, const uint32_t *src,
                           const uint32_t *dst, const int64_t *t, uint32_t flags, uint32_t H,
                           uint32_t K, const uint64_t *coeffs, int32_t order, uint32_t *bucket,
                           int32_t *count, tn_batch **proxies) {
    using namespace tn;
    if (!ctx || !proxies) return fail(TN_E_ARG, "ctx or proxies is NULL");
    *proxies = nullptr;
    if (n == 0 || H == 0 || K == 0 || order < 1) return fail(TN_E_ARG, "n, H, K and order must be > 0");
    if (K > 65536) return fail(TN_E_UNSUPPORTED, "K must be <= 65536");
    if (!coeffs || !bucket || !count) return fail(TN_E_ARG, "null coefficient or output array");
    for (size_t i = 0; i < (size_t)H * 3 * order; ++i)
        if (coeffs[i] >= kP61) return fail(TN_E_ARG, "hash coefficients must be < 2^61 - 1");
    if (m < 0 || (m > 0 && (!src || !dst || !t))) return fail(TN_E_ARG, "bad event arrays");
    if (flags & TN_FORWARD) return fail(TN_E_ARG, "hashing takes no TN_FORWARD");
    for (int64_t e = 0; e < m; ++e) {
        if (src[e] >= n || dst[e] >= n) return fail(TN_E_RANGE, "event " + std::to_string(e) + " has a node id >= n");
        if (e > 0 && t[e] < t[e - 1]) return fail(TN_E_ORDER, "event " + std::to_string(e) + " is earlier than its predecessor");
    }
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(TN_E_HIP, "cannot select the context's device");
    const size_t cbytes = sizeof(uint64_t) * H * 3 * order;
    tn_status st = ensure_scratch(ctx, cbytes);
    if (st != TN_OK) return st;
    hipError_t e = hipMemcpyAsync(ctx->scratch, coeffs, cbytes, hipMemcpyHostToDevice, ctx->stream);
    if (e != hipSuccess) return hip_fail(e, "coefficient upload");
    {
        ProfScope ps(ctx, TN_K_HASH);
        e = launch_hash_buckets(n, H, (const uint64_t *)ctx->scratch, order, K, bucket, count,
                                ctx->stream);
    }
    if (e != hipSuccess) return hip_fail(e, "hash kernel launch");
    // the host planner needs the bucket map of every hash: into the
    // context's pinned staging (one DMA, no page faults on a fresh array)
    st = ensure_host_staging(ctx, sizeof(uint32_t) * H * n);
    if (st != TN_OK) return st;
    const uint32_t *hb = (const uint32_t *)ctx->host_staging;
    e = hipMemcpyAsync(ctx->host_staging, bucket, sizeof(uint32_t) * H * n, hipMemcpyDeviceToHost,
                       ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return hip_fail(e, "bucket download");
    std::vector<uint32_t> ns(H, K);
    std::vector<int64_t> ms(H, m);
    std::vector<const uint32_t *> ss(H, src), ds(H, dst), maps(H);
    std::vector<const int64_t *> ts(H, t);
    for (uint32_t j = 0; j < H; ++j) maps[j] = hb + (size_t)j * n;
    return batch_create(ctx, (int32_t)H, ns.data(), ms.data(), ss.data(), ds.data(), ts.data(),
                        flags, proxies, maps.data(), n);
}

}  // extern "C"

namespace tn {
namespace {
// Proxies of at most this many super-nodes run on word columns in LDS, the
// H of them in one launch, larger ones as batched tiles (streamed builds, ms, on
// tiles and on columns: 16 proxies of 8192, random events, 27.9 and 67.3; 4 of
// 10^4, uniform events, 6.8 and 8.8, their op schedules taking the host longer).
constexpr uint32_t kColumnProxyK = 4096;

// Host image of one chunk of small proxies: the H op schedules at 256-byte
// aligned offsets off[j], then room for the H ColumnNet records at off[H].
// Images are packed by the planner threads and recycled from chunk to
// chunk.  A long stream keeps them in pinned memory, so that an upload is
// one DMA; with few chunks the pinning would cost more than it saves.
struct ColumnImage {
    unsigned char *pin = nullptr;
    size_t cap = 0;
    size_t bytes = 0;
    bool pinned = false;
    std::vector<size_t> off;
    std::vector<ColumnNet> nets;
    ColumnImage() = default;
    ColumnImage(const ColumnImage &) = delete;
    ColumnImage &operator=(const ColumnImage &) = delete;
    ColumnImage(ColumnImage &&o) noexcept { swap(o); }
    ColumnImage &operator=(ColumnImage &&o) noexcept {
        swap(o);
        return *this;
    }
    ~ColumnImage() { release(); }
    void swap(ColumnImage &o) noexcept {
        std::swap(pin, o.pin);
        std::swap(cap, o.cap);
        std::swap(bytes, o.bytes);
        std::swap(pinned, o.pinned);
        off.swap(o.off);
        nets.swap(o.nets);
    }
    void release() {
        if (pin && pinned) (void)hipHostFree(pin);
        else delete[] pin;
        pin = nullptr;
        cap = 0;
    }
};

// The H schedules in the column form.
tn_status column_image_pack(const std::vector<HostSchedule> &hs, ColumnImage &w, bool pinned) {
    const uint32_t H = (uint32_t)hs.size();
    w.off.assign(H + 1, 0);
    for (uint32_t j = 0; j < H; ++j)
        w.off[j + 1] = w.off[j] + ((std::max<size_t>(4 * hs[j].column.size(), 4) + 255) & ~(size_t)255);
    w.bytes = w.off[H] + sizeof(ColumnNet) * H;
    w.nets.resize(H);
    if (w.bytes > w.cap || w.pinned != pinned) {
        const size_t cap = std::max(w.bytes, w.cap + w.cap / 2);
        w.release();
        w.pinned = pinned;
        if (pinned) {
            if (hipHostMalloc((void **)&w.pin, cap, 0) != hipSuccess) {
                w.pin = nullptr;
                return TN_E_NOMEM;
            }
        } else {
            w.pin = new (std::nothrow) unsigned char[cap];
            if (!w.pin) return TN_E_NOMEM;
        }
        w.cap = cap;
    }
    for (uint32_t j = 0; j < H; ++j) {
        w.nets[j] = column_net(hs[j]);
        if (!hs[j].column.empty())
            std::memcpy(w.pin + w.off[j], hs[j].column.data(), 4 * hs[j].column.size());
    }
    return TN_OK;
}

// One chunk of small proxies: uploads the packed image, runs the H op
// schedules on one workgroup per word column of each proxy (slice state per
// column in state, col_words per proxy; fresh: the proxies start as the
// identity), reads the done count into *done_host and waits.
tn_status run_column_chunk(tn_ctx *ctx, const std::vector<HostSchedule> &hs, ColumnImage &img,
                         uint32_t K, const std::vector<uint64_t *> &Cs, int64_t ldK,
                         uint32_t *state, size_t col_words, unsigned int *done_dev,
                         unsigned int *done_host, int64_t &levels, StreamSlot &buf, bool fresh) {
    const uint32_t H = (uint32_t)hs.size();
    uint32_t scratch = 0;
    int64_t blocks = 0, lv = 0;
    for (uint32_t j = 0; j < H; ++j) {
        scratch = std::max(scratch, hs[j].scratch_used);
        blocks += img.nets[j].blocks;
        lv += hs[j].Lops;
    }
    levels += lv;
    hipError_t e = hipSuccess;
    if (img.bytes > buf.dev_bytes) {
        // the previous chunk's copy and launch are complete (it was waited for)
        const size_t cap = std::max(img.bytes, buf.dev_bytes + buf.dev_bytes / 2);
        if (buf.dev) (void)hipFree(buf.dev);
        buf.dev = nullptr;
        buf.dev_bytes = 0;
        e = hipMalloc(&buf.dev, cap);
        if (e != hipSuccess) {
            buf.dev = nullptr;
            return fail(TN_E_NOMEM, "proxy schedule allocation failed");
        }
        buf.dev_bytes = cap;
    }
    unsigned char *dev = (unsigned char *)buf.dev;
    for (uint32_t j = 0; j < H; ++j) {
        ColumnNet &net = img.nets[j];
        net.ops = reinterpret_cast<const uint2 *>(dev + img.off[j]);
        net.C = Cs[j];
        net.ld = ldK;
        net.persist = ctx->saturation ? state + (size_t)j * col_words : nullptr;
        std::memcpy(img.pin + img.off[H] + sizeof(ColumnNet) * j, &net, sizeof(ColumnNet));
    }
    e = hipMemcpyAsync(dev, img.pin, img.bytes, hipMemcpyHostToDevice, ctx->stream);
    if (e == hipSuccess) {
        ProfScope ps(ctx, TN_K_BATCH);
        e = launch_rowor_columns((const ColumnNet *)(dev + img.off[H]), H, K, scratch, blocks, lv,
                                 ctx->saturation, fresh, done_dev, ctx->stream);
    }
    if (e == hipSuccess)
        e = hipMemcpyAsync(done_host, done_dev, sizeof(unsigned int), hipMemcpyDeviceToHost,
                           ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return hip_fail(e, "proxy chunk");
    return TN_OK;
}
}  // namespace
}  // namespace tn

extern "C" {

// Streamed build of the H proxies (Sec. 4.3: the hashed networks are
// independent and built in parallel; Sec. 3.4: each is a reverse-time
// stream).  The event list is cut into chunks of whole time steps from its
// end; for each chunk the H mapped sub-streams are planned on host threads
// and applied in one batched launch that resumes from the proxies in HBM.
// Every tile carries its saturation state from chunk to chunk, and the
// build stops once every tile of every proxy is all ones.
tn_status tn_hash_build_proxies(tn_ctx *ctx, uint32_t n, int64_t m, const uint32_t *src,
                                const uint32_t *dst, const int64_t *t, uint32_t flags,
                                uint32_t H, uint32_t K, const uint64_t *coeffs, int32_t order,
                                uint32_t *bucket, int32_t *count, uint64_t *P, int64_t ldK,
                                int64_t chunk_events, tn_stream_stats *stats) {
    using namespace tn;
    const auto t0 = std::chrono::steady_clock::now();
    if (!ctx) return fail(TN_E_ARG, "ctx is NULL");
    if (n == 0 || H == 0 || K == 0 || order < 1) return fail(TN_E_ARG, "n, H, K and order must be > 0");
    if (K > 65536) return fail(TN_E_UNSUPPORTED, "K must be <= 65536");
    if (!coeffs || !bucket || !count || !P) return fail(TN_E_ARG, "null coefficient or output array");
    if (ldK < (int64_t)((K + 63) / 64)) return fail(TN_E_ARG, "ldK must be >= ceil(K/64)");
    if (chunk_events < 0) return fail(TN_E_ARG, "chunk_events must be >= 0");
    if (flags & ~(uint32_t)(TN_DIRECTED | TN_TIES_SEQUENTIAL))
        return fail(TN_E_ARG, "unknown flag bits (hashing takes TN_DIRECTED | TN_TIES_SEQUENTIAL)");
    for (size_t i = 0; i < (size_t)H * 3 * order; ++i)
        if (coeffs[i] >= kP61) return fail(TN_E_ARG, "hash coefficients must be < 2^61 - 1");
    if (m < 0 || (m > 0 && (!src || !dst || !t))) return fail(TN_E_ARG, "bad event arrays");
    if (m >= (int64_t)0xffffffffLL) return fail(TN_E_UNSUPPORTED, "m must be < 2^32 - 1");
    {
        std::string err;
        tn_status st = validate_events(n, m, src, dst, t, err);
        if (st != TN_OK) return fail(st, err);
    }
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(TN_E_HIP, "cannot select the context's device");
    const size_t cbytes = sizeof(uint64_t) * H * 3 * order;
    tn_status st = ensure_scratch(ctx, cbytes);
    if (st != TN_OK) return st;
    hipError_t e = hipMemcpyAsync(ctx->scratch, coeffs, cbytes, hipMemcpyHostToDevice, ctx->stream);
    if (e != hipSuccess) return hip_fail(e, "coefficient upload");
    {
        ProfScope ps(ctx, TN_K_HASH);
        e = launch_hash_buckets(n, H, (const uint64_t *)ctx->scratch, order, K, bucket, count,
                                ctx->stream);
    }
    if (e != hipSuccess) return hip_fail(e, "hash kernel launch");
    // the bucket maps into the context's pinned staging (one DMA, no page
    // faults on a fresh host array)
    st = ensure_host_staging(ctx, sizeof(uint32_t) * H * n);
    if (st != TN_OK) return st;
    const uint32_t *hb = (const uint32_t *)ctx->host_staging;
    e = hipMemcpyAsync(ctx->host_staging, bucket, sizeof(uint32_t) * H * n, hipMemcpyDeviceToHost,
                       ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return hip_fail(e, "bucket download");
    int64_t first = 0;
    // proxies of K << n super-nodes saturate within few events: start small
    default_chunks(m, chunk_events, first, 16);
    std::vector<std::pair<int64_t, int64_t>> bounds;
    stream_chunks(m, t, chunk_events, first, flags & TN_TIES_SEQUENTIAL, false, bounds);
    if (bounds.empty()) bounds.emplace_back(0, 0);  // no events: identity proxies
    std::vector<uint32_t> ns(H, K);
    std::vector<const uint32_t *> maps(H);
    std::vector<uint64_t *> Cs(H);
    std::vector<int64_t> lds(H, ldK);
    for (uint32_t j = 0; j < H; ++j) {
        maps[j] = hb + (size_t)j * n;
        Cs[j] = P + (size_t)j * K * ldK;
    }
    // Small proxies (K <= kColumnProxyK) run as op schedules on word columns in
    // LDS, larger ones as batched tiles.  One stream keeps one kind, as the two
    // keep different slice states, so columns are taken only when every chunk's
    // schedule fits: the op planner never needs more than max(default, K - 1)
    // scratch rows for K nodes.
    const bool columns = K <= kColumnProxyK && rowor_column_fits(K, std::max(kOpsScratchRows, K - 1));
    const uint32_t kw = (K + 63) / 64;
    const size_t column_words = 2 * (size_t)((K + 31) / 32) + 2;  // slice state words per column
    std::vector<uint32_t> lw;
    std::vector<uint32_t *> pst(H, nullptr);
    uint32_t *state = nullptr;
    StreamBuffers *buf = nullptr;
    unsigned int *done_host = nullptr;
    unsigned int *done_dev = nullptr;
    uint64_t tiles = 0;
    int64_t launched = 0, run_events = 0, levels = 0;
    bool all_done = false;
    // the slice state's room (word columns; tiles make their own) and the
    // done counter
    st = stream_buffers_take(ctx, columns ? (size_t)H * kw * column_words + 1 : 0, &buf);
    if (st != TN_OK) return st;
    done_host = buf->ring[0].done_host;
    e = hipEventRecord(buf->init_ev, ctx->stream);
    if (e != hipSuccess) {
        stream_buffers_give(ctx, buf);
        return hip_fail(e, "stream set-up");
    }
    // Chunk 0 is planned here on every host thread: its latency comes first,
    // and proxies of few super-nodes often saturate within it.  Only if they
    // do not, later chunks are planned by background threads, one proxy of
    // one chunk per task (so that few chunks still use every thread), ahead
    // of the launches by at most `window` chunks and about 2^26 mapped
    // events, so that host planning overlaps the device.
    const size_t nch = bounds.size();
    struct Planned {
        std::vector<HostSchedule> hs;
        ColumnImage img;  // small proxies: the packed schedules
        tn_status st = TN_OK;
        std::string err;
        uint32_t left = 0;  // under mu: proxies of the chunk still being planned
        bool ready = false;
    };
    std::vector<ColumnImage> spare;  // under mu: images of launched chunks
    std::vector<Planned> plans(nch);
    for (size_t c = 1; c < nch; ++c) {
        plans[c].hs.assign(H, HostSchedule());
        plans[c].left = H;
    }
    std::mutex mu;
    std::condition_variable cv;
    std::atomic<size_t> next{H};  // background tasks: proxy j of chunk c is task c * H + j
    std::atomic<bool> stop{false};  // set under mu: no more chunks are wanted
    size_t consumed = 0;  // under mu: chunks launched
    bool pin_images = false;  // set below, before the first chunk is planned
    auto plan_chunk = [&](size_t c, unsigned threads) {
        const int64_t a = bounds[c].first, mc = bounds[c].second - bounds[c].first;
        std::vector<int64_t> ms(H, mc);
        std::vector<const uint32_t *> ss(H, src ? src + a : nullptr), ds(H, dst ? dst + a : nullptr);
        std::vector<const int64_t *> ts(H, t ? t + a : nullptr);
        std::vector<HostSchedule> hs;
        std::string err;
        const tn_status ps = plan_batch((int32_t)H, ns.data(), ms.data(), ss.data(), ds.data(),
                                        ts.data(), flags, hs, err, maps.data(), n, threads,
                                        columns ? kFormColumn : kFormGather);
        ColumnImage img;
        tn_status ws = TN_OK;
        if (columns && ps == TN_OK) {
            {
                std::lock_guard<std::mutex> lk(mu);
                if (!spare.empty()) {
                    img = std::move(spare.back());
                    spare.pop_back();
                }
            }
            // chunk 0 is uploaded once and its latency comes first: never pinned
            ws = column_image_pack(hs, img, pin_images && c > 0);
        }
        {
            std::lock_guard<std::mutex> lk(mu);
            plans[c].hs = std::move(hs);
            plans[c].img = std::move(img);
            plans[c].st = ps == TN_OK ? ws : ps;
            plans[c].err = ps == TN_OK && ws != TN_OK ? "schedule image allocation failed"
                                                      : std::move(err);
            plans[c].ready = true;
        }
        cv.notify_all();
    };
    // proxy j of chunk c >= 1, on a background thread; the last proxy of a
    // chunk to finish packs the chunk's image
    auto plan_one = [&](size_t c, uint32_t j) {
        const int64_t a = bounds[c].first, mc = bounds[c].second - bounds[c].first;
        HostSchedule h;
        std::string err;
        const tn_status ps = plan_events(K, mc, src ? src + a : nullptr, dst ? dst + a : nullptr,
                                         t ? t + a : nullptr, flags, h, err, maps[j], n,
                                         columns ? kFormColumn : kFormGather, &stop);
        bool last;
        {
            std::lock_guard<std::mutex> lk(mu);
            plans[c].hs[j] = std::move(h);
            if (ps != TN_OK && plans[c].st == TN_OK) {
                plans[c].st = ps;
                plans[c].err = "network " + std::to_string(j) + ": " + err;
            }
            last = --plans[c].left == 0;
        }
        if (!last || stop) return;
        // every other task of chunk c has finished: its schedules are ours
        ColumnImage img;
        tn_status ws = TN_OK;
        if (columns && plans[c].st == TN_OK) {
            {
                std::lock_guard<std::mutex> lk(mu);
                if (!spare.empty()) {
                    img = std::move(spare.back());
                    spare.pop_back();
                }
            }
            ws = column_image_pack(plans[c].hs, img, pin_images);
        }
        {
            std::lock_guard<std::mutex> lk(mu);
            plans[c].img = std::move(img);
            if (ws != TN_OK && plans[c].st == TN_OK) {
                plans[c].st = ws;
                plans[c].err = "schedule image allocation failed";
            }
            plans[c].ready = true;
        }
        cv.notify_all();
    };
    const unsigned hw = std::max(1u, std::thread::hardware_concurrency());
    const size_t nth = std::min<size_t>(std::min<unsigned>(hw, 16u), (nch - 1) * H);
    const size_t window = std::max<size_t>(
        1, std::min<size_t>(nth, ((size_t)1 << 26) / std::max<size_t>(1, (size_t)H * chunk_events)));
    // at most window + 1 images are live at once: pin them when each is
    // reused a few times (chunk 0's never: pinning a fresh image costs
    // more than one pageable upload, at K = 4096, H = 16 about 7 ms)
    pin_images = nch >= 4 * (window + 1);
    auto worker = [&]() {
        (void)hipSetDevice(ctx->device);  // for the pinned image allocations
        for (;;) {
            const size_t task = next.fetch_add(1);
            const size_t c = task / H;
            if (c >= nch) return;
            {
                std::unique_lock<std::mutex> lk(mu);
                cv.wait(lk, [&] { return stop || c < consumed + window; });
                if (stop) return;
            }
            plan_one(c, (uint32_t)(task % H));
        }
    };
    plan_chunk(0, 0);
    std::vector<std::thread> pool;
    for (size_t c = 0; c < nch && st == TN_OK; ++c) {
        const int64_t mc = bounds[c].second - bounds[c].first;
        {
            std::unique_lock<std::mutex> lk(mu);
            cv.wait(lk, [&] { return plans[c].ready; });
        }
        if (plans[c].st != TN_OK) {
            st = fail(plans[c].st, plans[c].err);
            break;
        }
        if (columns) {
            if (c == 0) {
                // per-column slice state of every proxy, the done counter
                const size_t words = (size_t)H * kw * column_words;
                state = buf->persist;
                done_dev = state + words;
                tiles = (uint64_t)H * kw;
                e = launch_fill_u32(state, words + 1, 0u, ctx->stream);
                if (e != hipSuccess) {
                    st = hip_fail(e, "proxy initialisation");
                    break;
                }
            }
            st = run_column_chunk(ctx, plans[c].hs, plans[c].img, K, Cs, ldK, state, column_words * kw,
                                done_dev, done_host, levels, buf->ring[0], c == 0);
            plans[c].hs.clear();
            if (st != TN_OK) break;
            ++launched;
            run_events += mc;
            {
                std::lock_guard<std::mutex> lk(mu);
                consumed = c + 1;
                spare.push_back(std::move(plans[c].img));
            }
            cv.notify_all();
            if (ctx->saturation && *done_host == tiles) {
                all_done = true;
                break;
            }
            if (c == 0)
                for (size_t k = 0; k < nth; ++k) pool.emplace_back(worker);
            continue;
        }
        BatchStream bs;
        bs.lw = c ? lw.data() : nullptr;
        bs.persist = c ? pst.data() : nullptr;
        bs.resume = c ? 1u : 0u;
        bs.done_count = done_dev;
        tn_batch *b = nullptr;
        st = batch_from_plans(ctx, (int32_t)H, ns.data(), flags, plans[c].hs, &b, &bs);
        plans[c].hs.clear();
        if (st != TN_OK) break;
        if (c == 0) {
            // slice state of every tile of every proxy, then the done counter
            batch_slice_log2(b, lw);
            std::vector<size_t> off(H + 1, 0);
            for (uint32_t j = 0; j < H; ++j) {
                off[j + 1] = off[j] + batch_persist_words(K, lw[j]);
                tiles += (((K + 63) / 64) + (1u << lw[j]) - 1) >> lw[j];
            }
            e = hipMalloc((void **)&state, sizeof(uint32_t) * (off[H] + 1));
            if (e != hipSuccess) {
                batch_destroy(b);
                st = fail(TN_E_NOMEM, "slice state allocation failed");
                break;
            }
            for (uint32_t j = 0; j < H; ++j) pst[j] = state + off[j];
            done_dev = state + off[H];
            e = launch_fill_u32(state, off[H] + 1, 0u, ctx->stream);
            if (e != hipSuccess) {
                batch_destroy(b);
                st = hip_fail(e, "slice state clear");
                break;
            }
            batch_set_persist(b, pst.data(), done_dev);
        }
        st = batch_execute(ctx, b, Cs.data(), lds.data());
        if (st == TN_OK) {
            e = hipMemcpyAsync(done_host, done_dev, sizeof(unsigned int), hipMemcpyDeviceToHost,
                               ctx->stream);
            if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
            if (e != hipSuccess) st = hip_fail(e, "chunk completion");
        }
        std::vector<tn_plan_stats> bstats(H);
        (void)tn_batch_get_stats(b, bstats.data(), nullptr, nullptr);
        for (const auto &x : bstats) levels += x.levels;
        batch_destroy(b);
        if (st != TN_OK) break;
        ++launched;
        run_events += mc;
        {
            std::lock_guard<std::mutex> lk(mu);
            consumed = c + 1;
        }
        cv.notify_all();
        if (ctx->saturation && *done_host == tiles) {
            all_done = true;
            break;
        }
        if (c == 0)
            for (size_t k = 0; k < nth; ++k) pool.emplace_back(worker);
    }
    {
        std::lock_guard<std::mutex> lk(mu);
        stop = true;
    }
    cv.notify_all();
    for (auto &th : pool) th.join();
    (void)hipStreamSynchronize(ctx->stream);
    if (state && !columns) (void)hipFree(state);
    stream_buffers_give(ctx, buf);
    if (stats) {
        stats->chunks = (int64_t)bounds.size();
        stats->chunks_run = launched;
        stats->events_run = run_events;
        stats->levels_run = levels;
        stats->saturated = all_done ? 1 : 0;
        stats->slice_words = columns ? 1 : (lw.empty() ? 0 : (int32_t)(1u << lw[0]));
        stats->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    }
    return st;
}

tn_status tn_recombine(tn_ctx *ctx, uint32_t n, uint32_t H, uint32_t K, const uint64_t *P,
                       int64_t ldK, const uint32_t *bucket, const int32_t *count, int32_t *est,
                       int32_t *lifted) {
    using namespace tn;
    if (!ctx) return fail(TN_E_ARG, "ctx is NULL");
    if (n == 0 || H == 0 || K == 0) return fail(TN_E_ARG, "n, H and K must be > 0");
    if (K > 65536) return fail(TN_E_UNSUPPORTED, "K must be <= 65536");
    if (ldK < (int64_t)((K + 63) / 64)) return fail(TN_E_ARG, "ldK must be >= ceil(K/64)");
    if (!P || !bucket || !count || !est) return fail(TN_E_ARG, "null device array");
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(TN_E_HIP, "cannot select the context's device");
    const uint32_t nq = (n + 63) / 64;
    const size_t per_q = (size_t)H * K * 8;
    uint32_t qr = (uint32_t)std::max<size_t>(4, std::min<size_t>(nq, kLiftedBudget / per_q));
    qr = (qr + 3) / 4 * 4;
    bool lists_fit = fuse_lists_fit(n, H, K);
    // the totals first (8-byte entries), then what the tables need, the lifted
    // ones last of it: bitmaps and lists take their place in a call without
    // tables; then the lists' set-up, without which the tables serve too
    size_t need = 0;
    auto part = [&](size_t bytes) {
        const size_t at = need;
        need += align256(bytes);
        return at;
    };
    const size_t rows = (size_t)H * K, lt_bytes = (size_t)qr * per_q;
    const size_t o_stats = part(kFuseWords * 8), o_pt = part(rows * ldK * 8), o_rs = part(rows * 8),
                 o_cls = part(n), o_open = part((size_t)n * 4),
                 o_wide = part((size_t)n * 4), o_bs = part((size_t)H * ((K + 63) / 64) * 4),
                 o_lt = part(lt_bytes), tables = need,
                 o_hist = part(fuse_hist_words(H, K) * 4), o_start = part((rows + H) * 4),
                 o_nodes = part((size_t)H * n * 4), o_rows = part(rows * 8), o_brow = part(rows * 4);
    tn_status st = ensure_scratch(ctx, lists_fit ? need : tables);
    if (st == TN_E_NOMEM && lists_fit) {
        lists_fit = false;
        st = ensure_scratch(ctx, tables);
    }
    if (st != TN_OK) return st;
    unsigned char *base = (unsigned char *)ctx->scratch;
    unsigned long long *stats = (unsigned long long *)(base + o_stats);
    uint64_t *PT = (uint64_t *)(base + o_pt), *Lt = (uint64_t *)(base + o_lt);
    int2 *rowsum = (int2 *)(base + o_rs);
    int32_t *bsum = (int32_t *)(base + o_bs);
    uint8_t *cls = base + o_cls;
    uint32_t *open = (uint32_t *)(base + o_open), *wide = (uint32_t *)(base + o_wide);
    hipError_t e;
    unsigned long long host[kFuseWords] = {};
    {
        ProfScope ps(ctx, TN_K_AUX);
        e = launch_row_sums(H, K, ldK, P, count, bsum, rowsum, ctx->stream);
        if (e == hipSuccess)
            e = launch_classify(n, H, K, bucket, count, rowsum, lifted, lists_fit, cls, est, open,
                                wide, stats, ctx->stream);
    }
    if (e == hipSuccess)
        e = hipMemcpyAsync(host, stats, lists_fit ? sizeof(host) : sizeof(host[0]),
                           hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return hip_fail(e, "recombine set-up kernels");
    for (int k = 0; k < kFuseParts; ++k)
        for (int t = 0; t < 5; ++t) host[kFuseEntries + t] += host[kFuseStats + 8 * k + t];
    const uint32_t nlist = (uint32_t)host[kFuseOpen];
    if (nlist == 0) return TN_OK;  // est = n everywhere
    if (lists_fit) {
        unsigned long long entries = 0, nbitmaps = 0;
        for (uint32_t j = 0; j < H; ++j) {
            entries += host[kFuseRows + j];
            nbitmaps += host[kFuseRows + 16 + j];
        }
        if (fuse_by_lists(n, H, K, host, entries, nbitmaps, lt_bytes)) {
            ProfScope ps(ctx, TN_K_RECOMBINE);
            const FuseScratch fs = {(uint32_t *)(base + o_hist), (uint32_t *)(base + o_start),
                                    (uint32_t *)(base + o_nodes), (uint2 *)(base + o_rows),
                                    (uint32_t *)(base + o_brow), Lt};
            e = launch_fuse_lists(n, H, K, ldK, P, bucket, count, rowsum, cls, stats, fs,
                                  (uint32_t)nbitmaps, wide, host, est, ctx->stream);
            return e == hipSuccess ? TN_OK : hip_fail(e, "list fusion launch");
        }
    }
    {
        ProfScope ps(ctx, TN_K_AUX);
        e = launch_transpose_proxies(H, K, ldK, P, PT, ctx->stream);
        if (e != hipSuccess) return hip_fail(e, "proxy transpose launch");
    }
    for (uint32_t q0 = 0; q0 < nq; q0 += qr) {
        const uint32_t cnt = std::min(qr, nq - q0);
        {
            ProfScope ps(ctx, TN_K_AUX);
            e = launch_build_lifted(n, H, K, ldK, PT, bucket, q0, cnt, Lt, ctx->stream);
        }
        if (e != hipSuccess) return hip_fail(e, "lifted-table kernel launch");
        {
            ProfScope ps(ctx, TN_K_RECOMBINE);
            e = launch_recombine_est(n, H, K, bucket, Lt, q0, cnt, open, nlist, est, ctx->stream);
        }
        if (e != hipSuccess) return hip_fail(e, "recombine kernel launch");
    }
    return TN_OK;
}

}  // extern "C"
