// libalphacx: host orchestration and the C ABI declared in include/alphacx.h.
//
// One call runs the whole pipeline of kernels.hpp on one HIP stream. Device
// memory comes from a per-device caching pool, so repeated calls of similar
// size allocate nothing from the runtime after the first.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <limits>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <queue>
#include <string>
#include <thread>
#include <type_traits>
#include <vector>

#include "alphacx.h"
#include "kernels.hpp"
#include "simplices.hpp"
#include "emit.hpp"
#include "measure.hpp"
#include "sweep.hpp"
#include "partition.hpp"
#include "plan.hpp"

using namespace acx;

// ---------------------------------------------------------------------------
// Errors
static thread_local std::string g_last_error;

static ac_status set_error(ac_status st, const std::string &msg) {
    g_last_error = msg;
    return st;
}

struct HipError {
    ac_status st;
    std::string msg;
};

#define HIP_TRY(expr)                                                                                         \
    do {                                                                                                      \
        hipError_t e_ = (expr);                                                                               \
        if (e_ != hipSuccess) {                                                                               \
            throw HipError{e_ == hipErrorOutOfMemory ? AC_E_NOMEM : AC_E_DEVICE,                              \
                           std::string(#expr) + ": " + hipGetErrorString(e_)};                                \
        }                                                                                                     \
    } while (0)

#define LAUNCH_CHECK() HIP_TRY(hipGetLastError())

// ---------------------------------------------------------------------------
// Caching device allocator: blocks are kept per device and size class (next
// power of two) and reused; nothing is returned to the runtime until
// ac_release_workspace().
namespace {
struct Pool {
    std::mutex mu;
    std::map<int, std::multimap<size_t, void *>> free_blocks;  // device -> size -> ptr
    std::map<void *, std::pair<int, size_t>> live;
};
Pool &pool() {
    static Pool *p = new Pool();
    return *p;
}
size_t size_class(size_t n) {
    size_t c = 256;
    while (c < n) c <<= 1;
    return c;
}
}  // namespace

// Bump allocation from a caller-provided region instead of the pool, set for
// the duration of one call on the calling thread (the no-allocation entry
// point): every device buffer of the call, results included, then comes from
// that region, and read-backs go to pageable memory, so the call makes no
// allocation of its own.
struct Arena {
    char *base = nullptr;
    size_t cap = 0, used = 0, peak = 0;
};
static thread_local Arena *t_arena = nullptr;

// Allocations of a recorded build (ac_plan), kept for the plan's lifetime:
// the first fixed run takes pool blocks and records them in order; the run
// that is captured in a graph gets the same blocks back in the same order (its
// requests are the same, since every size is fixed), so the graph's launches
// address memory the plan owns.
struct Recorder {
    std::vector<std::pair<void *, size_t>> blocks;
    size_t next = 0;
    bool replay = false;
};
static thread_local Recorder *t_rec = nullptr;

static void *dev_alloc(size_t n) {
    if (Arena *a = t_arena) {
        const size_t at = (a->used + 255) & ~(size_t)255;
        if (n > a->cap || at > a->cap - n)
            throw HipError{AC_E_CAPACITY, "the call needs more than the " + std::to_string(a->cap >> 20) +
                                              " MiB of fixed scratch (" + std::to_string((at + n) >> 20) +
                                              " MiB requested so far)"};
        a->used = at + n;
        a->peak = std::max(a->peak, a->used);
        return a->base + at;
    }
    if (Recorder *r = t_rec) {
        if (r->replay) {
            if (r->next >= r->blocks.size() || r->blocks[r->next].second < n)
                throw HipError{AC_E_DEVICE, "internal error: a recorded build asked for other buffers than recorded"};
            return r->blocks[r->next++].first;
        }
        t_rec = nullptr;  // a pool block, recorded
        void *p = nullptr;
        try {
            p = dev_alloc(n);
        } catch (...) {
            t_rec = r;
            throw;
        }
        t_rec = r;
        r->blocks.emplace_back(p, n);
        return p;
    }
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    const size_t c = size_class(n ? n : 1);
    Pool &P = pool();
    {
        std::lock_guard<std::mutex> g(P.mu);
        auto &fb = P.free_blocks[dev];
        auto it = fb.find(c);
        if (it != fb.end()) {
            void *p = it->second;
            fb.erase(it);
            P.live[p] = {dev, c};
            return p;
        }
    }
    void *p = nullptr;
    hipError_t e = hipMalloc(&p, c);
    if (e != hipSuccess) {
        // drop cached blocks of this device and retry once
        (void)hipGetLastError();
        {
            std::lock_guard<std::mutex> g(P.mu);
            for (auto &kv : P.free_blocks[dev]) (void)hipFree(kv.second);
            P.free_blocks[dev].clear();
        }
        HIP_TRY(hipMalloc(&p, c));
    }
    std::lock_guard<std::mutex> g(P.mu);
    P.live[p] = {dev, c};
    return p;
}

static void dev_free(void *p) {
    if (!p) return;
    if (const Arena *a = t_arena)
        if (static_cast<char *>(p) >= a->base && static_cast<char *>(p) < a->base + a->cap) return;
    if (t_rec) return;  // recorded blocks belong to the plan
    Pool &P = pool();
    std::lock_guard<std::mutex> g(P.mu);
    auto it = P.live.find(p);
    if (it == P.live.end()) return;
    P.free_blocks[it->second.first].emplace(it->second.second, p);
    P.live.erase(it);
}

// Pinned host memory of results (host copies of rows and Sizes) and of uploads:
// size classes like the device pool's, at most HOST_POOL_BYTES of unused blocks
// kept (a copy into pageable memory is staged, and fresh pages fault in one by
// one: 16 MB of results took 1.2 ms of a 58,674-atom host call). nullptr when
// the host has no more to pin; callers then use pageable memory.
namespace {
constexpr size_t HOST_POOL_BYTES = (size_t)256 << 20;
struct HostPool {
    std::mutex mu;
    std::multimap<size_t, void *> free_blocks;
    size_t unused = 0;
};
HostPool &host_pool() {
    static HostPool *p = new HostPool();
    return *p;
}
}  // namespace
static void *host_alloc(size_t n) {
    const size_t c = size_class(n < 4096 ? 4096 : n);
    HostPool &P = host_pool();
    {
        std::lock_guard<std::mutex> g(P.mu);
        auto it = P.free_blocks.find(c);
        if (it != P.free_blocks.end()) {
            void *p = it->second;
            P.free_blocks.erase(it);
            P.unused -= c;
            return p;
        }
    }
    void *p = nullptr;
    if (hipHostMalloc(&p, c, hipHostMallocPortable) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    return p;
}
static void host_free(void *p, size_t n) {
    if (!p) return;
    const size_t c = size_class(n < 4096 ? 4096 : n);
    HostPool &P = host_pool();
    {
        std::lock_guard<std::mutex> g(P.mu);
        if (P.unused + c <= HOST_POOL_BYTES) {
            P.free_blocks.emplace(c, p);
            P.unused += c;
            return;
        }
    }
    (void)hipHostFree(p);
}

// Allocations of one call, returned to the pool when the call ends.
struct Scope {
    std::vector<void *> held;
    template <class T>
    T *get(size_t count) {
        void *p = dev_alloc(count * sizeof(T));
        held.push_back(p);
        return static_cast<T *>(p);
    }
    ~Scope() {
        for (void *p : held) dev_free(p);
    }
};

// ---------------------------------------------------------------------------
// Result object
struct ac_complex {
    int64_t count[4] = {0, 0, 0, 0};
    int64_t cand[4] = {0, 0, 0, 0};
    int64_t fallbacks = 0;
    int64_t work[2] = {0, 0};
    int64_t n = 0;  // balls in the input
    int64_t n_mol = 1;
    int64_t alpha_q = 0;  // the alpha the complex was built at (mA^2)
    bool batch = false;   // made by ac_alpha_complex_batch
    std::vector<int64_t> mol_rows[4];  // per dimension: first row of each molecule, n_mol + 1 entries
    std::vector<int32_t> h_mol[4];     // per dimension: molecule of each row (built on first ac_molecule)
    int32_t *d_simp[4] = {nullptr, nullptr, nullptr, nullptr};
    double *d_size[4] = {nullptr, nullptr, nullptr, nullptr};
    // host copies: in one pinned block per dimension (Sizes, then rows), or in
    // the vectors (streamed builds, or no pinned memory)
    void *h_block[4] = {nullptr, nullptr, nullptr, nullptr};
    size_t h_bytes[4] = {0, 0, 0, 0};
    std::vector<int32_t> h_simp[4];
    std::vector<double> h_size[4];
    bool host_ready[4] = {false, false, false, false};
    bool device_result = false;
    int device = 0;
    double stage_ms[32];
    // vertex -> incidence slots of the simplices, built on first use by the
    // union-measure backward (slot of corner k of simplex s of dimension d:
    // sum_{e<d} count[e] (e+1) + s (d+1) + k)
    int32_t *inc_slot = nullptr;
    int32_t *inc_start = nullptr;
    // work buffers of the union-measure calls, kept with the complex so that
    // those calls need no allocation or host synchronisation after the first
    double *meas_part = nullptr;    // block partial sums of V and A, then V, A
    double4 *meas_contrib = nullptr;  // per incidence slot gradient terms
};

static void free_complex(ac_complex *c) {
    if (!c) return;
    for (int d = 0; d < 4; d++) {
        dev_free(c->d_simp[d]);
        dev_free(c->d_size[d]);
        host_free(c->h_block[d], c->h_bytes[d]);
    }
    dev_free(c->inc_slot);
    dev_free(c->inc_start);
    dev_free(c->meas_part);
    dev_free(c->meas_contrib);
    delete c;
}

// ---------------------------------------------------------------------------
static inline unsigned grid_for(long long n) {
    long long b = (n + BLOCK - 1) / BLOCK;
    return (unsigned)(b < 1 ? 1 : b);
}

template <class T>
static void fill(T *p, T v, long long n, hipStream_t s) {
    if (n <= 0) return;
    long long b = (n + BLOCK - 1) / BLOCK;
    if (b > 65536) b = 65536;
    k_fill<T><<<(unsigned)b, BLOCK, 0, s>>>(p, v, n);
    LAUNCH_CHECK();
}

// out[0..n] = exclusive scan of in[0..n), out[n] = total (also stored to
// *total_to when given). One launch up to SCAN_SMALL items, three above
// (tile scan, scan of tile sums, add).
static void scan_i32(const int *in, int *out, long long n, hipStream_t s, Scope &sc, int *total_to = nullptr) {
    if (n <= 0) {
        fill<int>(out, 0, 1, s);
        if (total_to) fill<int>(total_to, 0, 1, s);
        return;
    }
    if (n <= SCAN_SMALL) {
        k_scan_small<<<1, SCAN_SMALL_BLOCK, 0, s>>>(in, out, (int)n, total_to);
        LAUNCH_CHECK();
        return;
    }
    const long long tiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    int *sums = sc.get<int>(tiles);
    int *offs = sc.get<int>(tiles + 1);
    k_scan_tiles<<<(unsigned)tiles, SCAN_BLOCK, 0, s>>>(in, out, sums, n);
    LAUNCH_CHECK();
    scan_i32(sums, offs, tiles, s, sc);
    k_scan_add_total<<<(unsigned)tiles, SCAN_BLOCK, 0, s>>>(out, offs, n, (int)tiles, total_to);
    LAUNCH_CHECK();
}

// Pinned host block of this thread for device-to-host read-backs (a copy to
// pageable memory takes a slower staged path). Every use synchronises the
// stream before the block is read or reused, so one block per thread serves
// all calls; it is kept until the process ends.
static void *pinned_block(size_t bytes) {
    thread_local void *p = nullptr;
    thread_local size_t cap = 0;
    if (bytes > cap) {
        if (p) HIP_TRY(hipHostFree(p));
        p = nullptr;
        cap = 0;
        const size_t c = std::max<size_t>(bytes, 4096);
        HIP_TRY(hipHostMalloc(&p, c, hipHostMallocPortable));
        cap = c;
    }
    return p;
}

// Mail block of this thread (see Mail): one message at a time, numbered so that
// an earlier one is never taken for it. Every build waits for the messages it
// asks for, or for its stream when it fails, so none arrives after its build.
struct MailBox {
    Mail *host = nullptr, *dev = nullptr;
    unsigned seq = 0;
};
static MailBox &mail_box() {
    thread_local MailBox b;
    if (!b.host) {
        void *p = nullptr, *d = nullptr;
        HIP_TRY(hipHostMalloc(&p, sizeof(Mail), hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent));
        if (hipHostGetDevicePointer(&d, p, 0) != hipSuccess) {
            (void)hipHostFree(p);
            throw HipError{AC_E_DEVICE, "pinned host memory has no device address"};
        }
        std::memset(p, 0, sizeof(Mail));
        b.host = static_cast<Mail *>(p);
        b.dev = static_cast<Mail *>(d);
    }
    return b;
}

// Waits for message `seq`. The stream is asked now and then: when its work has
// ended (or failed) no message can come any more.
static const Mail &mail_wait(const MailBox &b, unsigned seq, hipStream_t s) {
    for (long long spin = 0;; spin++) {
        if (__atomic_load_n(&b.host->seq, __ATOMIC_ACQUIRE) == seq) return *b.host;
        if ((spin & 0xfff) == 0xfff) {
            const hipError_t e = hipStreamQuery(s);
            if (e == hipErrorNotReady) continue;
            HIP_TRY(e);
            if (__atomic_load_n(&b.host->seq, __ATOMIC_ACQUIRE) == seq) return *b.host;
            throw HipError{AC_E_DEVICE, "internal error: the build ended without its message"};
        }
        __builtin_ia32_pause();
    }
}

// Copies n items from the device into h through the pinned block (synchronises s).
template <class T>
static void read_back(T *h, const T *d, size_t n, hipStream_t s) {
    if (n == 0) return;
    if (t_arena) {
        // no pinned block (that would be an allocation): pageable copy
        HIP_TRY(hipMemcpyAsync(h, d, n * sizeof(T), hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
        return;
    }
    void *b = pinned_block(n * sizeof(T));
    HIP_TRY(hipMemcpyAsync(b, d, n * sizeof(T), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    std::memcpy(h, b, n * sizeof(T));
}

template <class T>
static T read_one(const T *d, hipStream_t s) {
    T h;
    read_back(&h, d, 1, s);
    return h;
}

// Exact 64-bit sum of n int32 counts, to *out on the device (the counted
// passes check their totals with it before 32-bit scans).
static void sum_i64(const int *x, long long n, long long *out, hipStream_t s, Scope &sc) {
    long long b = (n + BLOCK - 1) / BLOCK;
    b = b < 1 ? 1 : (b > 1024 ? 1024 : b);
    long long *part = sc.get<long long>(b);
    k_sum_i64<<<(unsigned)b, BLOCK, 0, s>>>(x, n, part);
    k_fold_i64<<<1, BLOCK, 0, s>>>(part, (int)b, out);
    LAUNCH_CHECK();
}

// The same, read back (synchronises the stream).
static long long total_i64(const int *x, long long n, hipStream_t s, Scope &sc) {
    if (n <= 0) return 0;
    long long *t = sc.get<long long>(1);
    sum_i64(x, n, t, s, sc);
    return read_one(t, s);
}

static void check_total(long long t, const char *what) {
    if (!has_index(t))
        throw HipError{AC_E_CAPACITY, "more than " + std::to_string(INDEX_LAST) + " " + what + " (32-bit indices)"};
}

static long long isqrt_ceil(long long v) {
    if (v <= 0) return 0;
    long long r = (long long)std::sqrt((double)v);
    while (r * r > v) r--;
    while (r * r < v) r++;
    return r;
}

// Stable LSD radix sort of (key, payload) on bits [lo, hi) of key, 8 bits per
// pass. key / pay are set to the buffers that hold the result (the inputs' or
// scratch of the scope); *spare_key / *spare_pay (if given) to two other
// buffers of n entries.
template <class P>
static void radix_sort(unsigned *&key, P *&pay, int n, int lo, int hi, hipStream_t s, Scope &sc,
                       unsigned **spare_key = nullptr, P **spare_pay = nullptr) {
    unsigned *k2 = sc.get<unsigned>(n > 0 ? n : 1);
    P *p2 = sc.get<P>(n > 0 ? n : 1);
    unsigned *kin = key, *kout = k2;
    P *pin = pay, *pout = p2;
    if (n > 1 && hi > lo) {
        const int tiles = (n + RS_TILE - 1) / RS_TILE;
        int *hist = sc.get<int>((size_t)RS_BINS * tiles);
        int *totals = sc.get<int>(RS_BINS);
        for (int shift = lo; shift < hi; shift += RS_BITS) {
            k_rs_hist<<<tiles, RS_BLOCK, 0, s>>>(kin, n, shift, hist, tiles);
            if (tiles > RS_FEW) k_rs_digit_prefix<<<RS_BINS, RS_PREFIX_BLOCK, 0, s>>>(hist, tiles, totals);
            k_rs_scatter<P><<<tiles, RS_BLOCK, 0, s>>>(kin, pin, kout, pout, n, shift, hist, totals, tiles);
            LAUNCH_CHECK();
            std::swap(kin, kout);
            std::swap(pin, pout);
        }
    }
    key = kin;
    pay = pin;
    if (spare_key) *spare_key = kout;
    if (spare_pay) *spare_pay = pout;
}

static int bits_for(long long n) {
    int b = 1;
    while ((1LL << b) < n) b++;
    return b;
}

// Merge keys of dimension K - 1 for n balls and M rows: rows are keyed by
// their least input id (< n); a bucket is 2^shift ids, at most EK_KEYS, at
// least 256 buckets where n allows (so that small inputs still spread over
// many blocks), and small enough that the expected largest bucket, 2^shift K
// M / n rows, stays within 95% of what a block orders in LDS; nb buckets hold
// every id, and keys fit in `bits` bits. The radix sort orders bits [shift, bits).
struct EmitKeys {
    int bits, shift, nb;
};
template <int K>
static EmitKeys emit_keys(int n, long long M) {
    EmitKeys k;
    k.shift = EK_SHIFT;
    while (k.shift > 0 && ((n >> k.shift) < 256 ||
                           (double)(1LL << k.shift) * K * (double)M > 0.95 * ek_rows<K>() * (double)n))
        k.shift--;
    k.nb = ((n - 1) >> k.shift) + 1;
    k.bits = bits_for(n);
    return k;
}

// start[0..nb] of the ranges of key >> shift in m sorted keys (k_key_starts).
static void key_starts(const unsigned *key, long long m, int shift, int nb, int *start, hipStream_t s) {
    const long long threads = m / KS_PT + 1;  // rows 0..m
    k_key_starts<<<(unsigned)((threads + KS_BLOCK - 1) / KS_BLOCK), KS_BLOCK, 0, s>>>(key, (int)m, shift, nb, start);
    LAUNCH_CHECK();
}

// Merge of dimension d = K - 1 from the rows' keys (least input id) and
// payloads: a radix sort over the key bits above the bucket (2^shift ids,
// emit_keys) makes each bucket contiguous, k_key_starts finds the buckets'
// starts and k_emit_block orders each bucket and writes its rows; up to
// EK_KEYS balls one block takes every row, unsorted. The row count goes to
// *m_out on the device. Sizes are copied (they are A^2 already).
template <int K>
static void emit_dim(unsigned *key, typename EmitPay<K>::type *pay, const double *size_in, int M, int n,
                     hipStream_t s, Scope &sc, ac_complex *res, int d, int *m_out) {
    typedef typename EmitPay<K>::type P;
    res->d_simp[d] = static_cast<int32_t *>(dev_alloc((size_t)(M > 0 ? M : 1) * K * sizeof(int32_t)));
    res->d_size[d] = static_cast<double *>(dev_alloc((size_t)(M > 0 ? M : 1) * sizeof(double)));
    if (M == 0) {
        fill<int>(m_out, 0, 1, s);
        return;
    }
    if (n <= EK_KEYS && M <= ek_rows<K>()) {
        // a few hundred balls: one block orders every row, no radix sort
        k_emit_block<K><<<1, EK_BLOCK, 0, s>>>(key, pay, nullptr, EK_SHIFT, 1, nullptr, nullptr, size_in,
                                              res->d_simp[d], res->d_size[d], m_out, M);
        LAUNCH_CHECK();
        return;
    }
    const EmitKeys ek = emit_keys<K>(n, M);
    unsigned *gkey = nullptr;
    P *gpay = nullptr;
    radix_sort<P>(key, pay, M, ek.shift, ek.bits, s, sc, &gkey, &gpay);
    const int nb = ek.nb;
    int *start = sc.get<int>((size_t)nb + 1);
    key_starts(key, M, ek.shift, nb, start, s);
    LAUNCH_CHECK();
    k_emit_block<K><<<(unsigned)nb, EK_BLOCK, 0, s>>>(key, pay, start, ek.shift, nb, gkey, gpay, size_in,
                                                     res->d_simp[d], res->d_size[d], m_out);
    LAUNCH_CHECK();
}

// Bytes of the minima of the alphas that a sweep takes in one launch.
constexpr size_t SWEEP_ROOM = 256u << 20;

// Bytes of output rows a build allocates for candidates that may not be kept
// (see run_pipeline).
constexpr long long OUT_ROOM = 64LL << 20;

struct Options {
    int cell_mA = 0;
    int force_exact = 0;
    int vertex_shortcut = 0;
    int profile = 0;
    int cell_order = ORDER_ROW;
};

// Stages timed by HIP events when profiling. A stage lasts from its mark to
// the next mark; "edges_ac2" and "triangles_ac2" are marked only when the AC2
// tests of edges and triangles run as kernels of their own.
enum Stage {
    ST_QUANTISE, ST_BIN, ST_NBR_COUNT, ST_NBR_SCAN, ST_NBR_FILL, ST_TRI_COUNT, ST_TRI_SCAN, ST_TRI_FILL,
    ST_TRI_GABRIEL, ST_TET_COUNT, ST_TET_FILL, ST_TETRA, ST_TRI_FINAL, ST_EDGE_FINAL, ST_VERT_FINAL, ST_EMIT,
    ST_EDGE_AC2, ST_TRI_AC2, ST_COUNT
};
static const char *kStageNames[ST_COUNT] = {
    "quantise", "binning", "neighbours_count", "neighbours_scan", "neighbours_fill", "triangles_count",
    "triangles_scan", "triangles_fill", "triangles_ac2_tetrahedra", "tetrahedra_scan", "tetrahedra_fill", "tetrahedra_ac2",
    "triangles_final", "edges_final", "vertices_final", "emit", "edges_ac2", "triangles_ac2"};
// profile value of the per-step arrangement: every stage timed, edge and
// triangle AC2 in kernels of their own
constexpr int PROFILE_SPLIT = ST_COUNT + 2;

// Events at stage boundaries. Each recorded event costs a few microseconds of
// idle device time between two kernels, so a caller may ask for one stage
// only (its two boundary events). The events come from a per-thread pool
// (creating one in the middle of a build would hold up the host's launches),
// one pool per device (an event belongs to the device it was created on).
static std::vector<hipEvent_t> &event_pool() {
    thread_local std::map<int, std::vector<hipEvent_t>> pools;
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    return pools[dev];
}
struct StageTimer {
    bool on = false;
    int only = -1;  // >= 0: record the boundaries of this stage only
    int cur = -1;   // stage running since the last mark
    hipStream_t s = nullptr;
    std::vector<hipEvent_t> ev;
    int ev_start[ST_COUNT], ev_end[ST_COUNT];
    void start(int profile, hipStream_t st) {
        on = profile != 0;
        only = (profile >= 2 && profile < PROFILE_SPLIT) ? profile - 2 : -1;
        s = st;
        for (int i = 0; i < ST_COUNT; i++) ev_start[i] = ev_end[i] = -1;
    }
    // stage i starts now (i = ST_COUNT: the last stage ends)
    void mark(int i) {
        if (!on) return;
        const bool need = only < 0 || i == only || cur == only;
        if (need) {
            hipEvent_t e;
            std::vector<hipEvent_t> &pool = event_pool();
            if (!pool.empty()) {
                e = pool.back();
                pool.pop_back();
            } else {
                // timing only: no system-scope fence (an L2 writeback and
                // invalidate at every record, which stalls the next kernels)
                HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableSystemFence));
            }
            ev.push_back(e);
            HIP_TRY(hipEventRecord(e, s));
            const int k = (int)ev.size() - 1;
            if (cur >= 0) ev_end[cur] = k;
            if (i < ST_COUNT) ev_start[i] = k;
        }
        cur = i;
    }
    void collect(double *ms) {
        for (int i = 0; i < ST_COUNT; i++) {
            ms[i] = -1.0;
            if (on && ev_start[i] >= 0 && ev_end[i] >= 0) {
                float f = 0.f;
                if (hipEventElapsedTime(&f, ev[ev_start[i]], ev[ev_end[i]]) == hipSuccess) ms[i] = f;
            }
        }
    }
    ~StageTimer() {
        // back to the pool of this thread and device, for a later build (a
        // re-record of an event still pending only moves it)
        if (ev.empty()) return;
        try {
            std::vector<hipEvent_t> &pool = event_pool();
            for (hipEvent_t e : ev) pool.push_back(e);
        } catch (...) {
            for (hipEvent_t e : ev) (void)hipEventDestroy(e);
        }
    }
};

// Molecules of one call: balls [off[m], off[m+1]) form molecule m, each with
// its own grid (cell side cell_mA[m] if given).
struct Batch {
    std::vector<int64_t> off;
    std::vector<int32_t> cell_mA;
};

// Blocks of the quantise kernel: tiles of at most QTILE balls, each inside one
// molecule; molecule m's tiles are [tile_first[m], tile_first[m+1]).
static void quantise_tiles(const Batch &bt, std::vector<int2> &tiles, std::vector<int> &tile_first) {
    const int n_mol = (int)bt.off.size() - 1;
    tiles.clear();
    tile_first.assign(n_mol + 1, 0);
    for (int m = 0; m < n_mol; m++) {
        tile_first[m] = (int)tiles.size();
        for (int64_t a = bt.off[m]; a < bt.off[m + 1]; a += QTILE)
            tiles.push_back(make_int2((int)a, (int)std::min<int64_t>(a + QTILE, bt.off[m + 1])));
    }
    tile_first[n_mol] = (int)tiles.size();
}

// Sizes of a recorded build (ac_plan). A learning run (learn = true) is an
// ordinary build that notes them; a fixed run takes them, with the plan's
// capacities, instead of reading any count back, so that it is a fixed
// sequence of launches with no host synchronisation (see plan.hpp).
struct Fixed {
    bool learn = true;
    // noted by the learning run
    std::vector<Grid> grids;       // per molecule: cell side, reach, order, balls
    std::vector<long long> cells;  // per molecule: grid cells
    PredParams pp{};
    int wmax = 0, gshift = 0;
    long long rule = 0;  // radius that chooses the kernels
    long long E = 0, P = 0, T = 0, Q = 0;  // candidate edges, pairs, candidate triangles, kept tetrahedra
    long long tet_most = 0;  // candidate tetrahedra of the fullest group where one outgrew its slab, else 0
    long long tet_limit = 0;  // most entries of a slab
    bool two_pass = false;  // a stage needed a counted pass
    // given to a fixed run (device arrays uploaded before it)
    long long ncell = 0;  // cells of all molecules' capacities
    int E_cap = 1, T_cap = 1, Q_cap = 1;
    bool counted = false;  // the triangles are counted first (room for T_cap), else there is room for P_cap pairs
    long long P_cap = 1;
    const int2 *d_tiles = nullptr;
    const int *d_tile_first = nullptr;
    const Grid *d_tmpl = nullptr;       // recorded grids with each molecule's first cell
    const long long *d_cell_cap = nullptr;
    const long long *d_bound = nullptr;  // first ball of each molecule, n_mol + 1
    // left by a fixed run (device)
    Counters *cnt = nullptr;
    long long *d_rows = nullptr;
};

// Output arrays of the caller (the build without allocation): rows go there if
// every dimension fits.
struct Ext {
    int32_t *const *simp;
    double *const *size;
    const int64_t *cap;
    bool fits;
};

// The whole pipeline from device arrays, for n_alpha >= 1 alpha values: one
// candidate search at the largest, then pruning and output per value (the
// candidates of a smaller alpha are those of the larger that pass AC3 at the
// smaller, and AC2 does not depend on alpha). Returns AC_OK and outs[k] for
// alphas[k] on success; nothing is left allocated on failure.
static ac_status run_pipeline(const double *d_xyz, const double *d_r, int64_t n64, const Batch &bt,
                              const double *alphas, int n_alpha, const Options &o, hipStream_t s, ac_complex **outs,
                              Fixed *fx = nullptr, Ext *ext = nullptr) {
    for (int k = 0; k < n_alpha; k++) outs[k] = nullptr;
    // fixed: sizes from fx, nothing read back (only with one alpha)
    const bool fixed = fx && !fx->learn;
    if (fx && n_alpha != 1) return set_error(AC_E_INVALID, "a recorded build takes one alpha");
    if (n64 < 1 || n64 >= (1 << 26)) return set_error(AC_E_INVALID, "n must be in [1, 2^26)");
    if (n_alpha < 1 || n_alpha > AC_MAX_SWEEP) return set_error(AC_E_INVALID, "number of alpha values out of range");
    std::vector<long long> aqs(n_alpha);
    for (int k = 0; k < n_alpha; k++) {
        if (!std::isfinite(alphas[k])) return set_error(AC_E_INVALID, "alpha is not finite");
        const double as = alphas[k] * 1e6;
        if (!(std::fabs(as) < 67108864.0)) return set_error(AC_E_RANGE, "|alpha| too large for the exact bit budget");
        aqs[k] = (long long)std::nearbyint(as);
    }
    const long long aq = *std::max_element(aqs.begin(), aqs.end());
    const int n = (int)n64;
    Scope sc;
    StageTimer tm;
    std::vector<ac_complex *> rs(n_alpha, nullptr);
    auto new_result = [&]() {
        ac_complex *r = new ac_complex();
        for (double &x : r->stage_ms) x = -1.0;
        HIP_TRY(hipGetDevice(&r->device));
        r->device_result = true;
        return r;
    };
    ac_complex *res = nullptr;
    try {
        for (int k = 0; k < n_alpha; k++) rs[k] = new_result();
        res = rs[0];
        tm.start(o.profile, s);
        const bool split = o.profile == PROFILE_SPLIT;  // AC2 of edges and triangles as kernels of their own
        // ---- quantise + stats (per molecule) ----
        tm.mark(ST_QUANTISE);
        const int n_mol = (int)bt.off.size() - 1;
        int4 *q = sc.get<int4>(n);
        Counters *cnt = sc.get<Counters>(1);
        // messages to the host: not from a recorded build, and not on fixed
        // scratch (the mail block would be an allocation)
        MailBox *mb = fixed || t_arena ? nullptr : &mail_box();
        Mail *const mail = mb ? mb->dev : nullptr;
        std::vector<Stats> hs(n_mol);
        const int wlarge = (int)(LARGE_SGC * LARGE_SGC - aq);
        Stats *st = sc.get<Stats>(n_mol);
        if (n_mol == 1) {
            const int n_tiles = (n + QTILE - 1) / QTILE;
            Stats *part = sc.get<Stats>(n_tiles);
            const unsigned seq = mb ? ++mb->seq : 0;
            const bool one = n_tiles == 1;
            k_quantise<<<n_tiles, BLOCK, 0, s>>>(d_xyz, d_r, nullptr, n, wlarge, q, one ? st : part, cnt, one ? mail : nullptr, seq);
            if (!one) k_stats_reduce<<<1, BLOCK, 0, s>>>(part, nullptr, n_tiles, st, mail, seq);
            LAUNCH_CHECK();
            if (mb) hs[0] = mail_wait(*mb, seq, s).st;
            else if (!fixed) read_back(hs.data(), st, 1, s);
        } else {
            std::vector<int2> tiles;
            std::vector<int> tile_first;
            quantise_tiles(bt, tiles, tile_first);
            const int2 *d_tiles = fixed ? fx->d_tiles : sc.get<int2>(tiles.size());
            const int *d_tile_first = fixed ? fx->d_tile_first : sc.get<int>(n_mol + 1);
            Stats *part = sc.get<Stats>(tiles.size());
            if (!fixed) {
                HIP_TRY(hipMemcpyAsync(const_cast<int2 *>(d_tiles), tiles.data(), tiles.size() * sizeof(int2),
                                       hipMemcpyHostToDevice, s));
                HIP_TRY(hipMemcpyAsync(const_cast<int *>(d_tile_first), tile_first.data(), (n_mol + 1) * sizeof(int),
                                       hipMemcpyHostToDevice, s));
            }
            k_quantise<<<(unsigned)tiles.size(), BLOCK, 0, s>>>(d_xyz, d_r, d_tiles, n, wlarge, q, part, cnt, nullptr, 0);
            LAUNCH_CHECK();
            k_stats_reduce<<<(unsigned)n_mol, BLOCK, 0, s>>>(part, d_tile_first, 0, st, nullptr, 0);
            LAUNCH_CHECK();
            if (!fixed) read_back(hs.data(), st, (size_t)n_mol, s);
        }
        int flags = 0, wmax = 0;
        long long large = 0;
        for (const Stats &x : hs) {
            flags |= x.flags;
            wmax = std::max(wmax, x.wmax);
            large += x.large;
        }
        if (fixed) wmax = fx->wmax;  // the device checks that no radius exceeds it
        if (flags & 1) throw HipError{AC_E_INVALID, "non-finite coordinate, or radius not positive"};
        if (flags & 2) throw HipError{AC_E_RANGE, "coordinate or radius outside the exact bit budget"};
        const long long sg2 = (long long)wmax + aq;
        if (sg2 >= (1LL << 26)) throw HipError{AC_E_RANGE, "r_max^2 + alpha too large for the exact bit budget"};
        PredParams pp;
        pp.aq = aq;
        pp.sg2 = sg2 < 0 ? 0 : sg2;
        const long long sgc = isqrt_ceil(pp.sg2);
        pp.sgc = sgc;
        pp.bmax = 2.0 * (double)sgc;
        pp.gmax = 4.0 * (double)pp.sg2 + (double)wmax;
        pp.force_exact = o.force_exact;
        pp.fast = pp.sg2 < (1LL << 25);
        if (fx && fx->learn) {
            fx->pp = pp;
            fx->wmax = wmax;
        }

        // ---- grids: one per molecule, cells numbered consecutively ----
        std::vector<Grid> grids(n_mol);
        long long ncell = 0;
        if (fx && fx->learn) fx->cells.assign(n_mol, 0);
        for (int m = 0; m < n_mol && !fixed; m++) {
            const Stats &h = hs[m];
            const long long nm = bt.off[m + 1] - bt.off[m];
            Grid &g = grids[m];
            g.ox = h.minx; g.oy = h.miny; g.oz = h.minz;
            const long long ex = (long long)h.maxx - h.minx + 1, ey = (long long)h.maxy - h.miny + 1,
                            ez = (long long)h.maxz - h.minz + 1;
            long long side = !bt.cell_mA.empty() ? bt.cell_mA[m] : (o.cell_mA > 0 ? o.cell_mA : (sgc > 0 ? sgc : 1));
            const long long cell_limit = n_mol == 1 ? std::max<long long>(8LL * nm, 1LL << 22)
                                                    : std::max<long long>(8LL * nm, 1LL << 15);
            // cells of the grid: the box, or for a Morton order the cube of
            // 2^L cells a side that holds it (2^(3L) codes)
            auto ncell_of = [&](long long sd) {
                const long long gx = (ex + sd - 1) / sd, gy = (ey + sd - 1) / sd, gz = (ez + sd - 1) / sd;
                if (o.cell_order != ORDER_MORTON) return gx * gy * gz;
                int L = 0;
                while ((1LL << L) < std::max(gx, std::max(gy, gz))) L++;
                return L > MORTON_MAX_BITS ? LLONG_MAX : 1LL << (3 * L);
            };
            while (ncell_of(side) > cell_limit) side = side + side / 4 + 1;
            g.s = (int)side;
            g.nx = (int)((ex + side - 1) / side); g.ny = (int)((ey + side - 1) / side); g.nz = (int)((ez + side - 1) / side);
            g.reach = (int)((2 * sgc + side - 1) / side);
            g.base = ncell;
            g.a0 = (int)bt.off[m];
            g.a1 = (int)bt.off[m + 1];
            g.order = o.cell_order;
            if (fx && fx->learn) fx->cells[m] = ncell_of(side);
            ncell += ncell_of(side);
        }
        if (fx && fx->learn) fx->grids = grids;
        if (fixed) ncell = fx->ncell;
        if (ncell >= (long long)INT_MAX) throw HipError{AC_E_CAPACITY, "too many grid cells"};
        // one molecule's grid is an argument of the kernels that need it
        Grid *d_grids = fixed || n_mol > 1 ? sc.get<Grid>(n_mol) : nullptr;
        const Grid g0 = fixed || n_mol > 1 ? Grid{} : grids[0];
        if (fixed) {
            // this run's boxes, the recorded sides and capacities
            k_plan_grids<<<grid_for(n_mol), BLOCK, 0, s>>>(st, n_mol, fx->d_tmpl, fx->d_cell_cap, fx->wmax, d_grids,
                                                           cnt);
            LAUNCH_CHECK();
        } else if (n_mol > 1) {
            HIP_TRY(hipMemcpyAsync(d_grids, grids.data(), n_mol * sizeof(Grid), hipMemcpyHostToDevice, s));
        }

        // ---- binning ----
        tm.mark(ST_BIN);
        int *cell_start = sc.get<int>(ncell + 1);
        int4 *atom = sc.get<int4>(n);
        int2 *sball = sc.get<int2>((size_t)n + SCAN_PAD);
        int *perm = sc.get<int>(n);
        if (n <= SMALL_BALLS && ncell <= SMALL_CELLS) {
            k_bin_small<<<1, SMALL_BLOCK, 0, s>>>(q, n, d_grids, n_mol, g0, (int)ncell, cell_start, atom, sball,
                                                 (int)aq, perm, cnt);
            LAUNCH_CHECK();
        } else {
            // bucket: at most BIN_CELLS cells, and a bucket of full cells within
            // BIN_ROWS balls; as few radix passes as that allows, and of the shifts
            // these passes reach the least that leaves a bucket 128 balls on average
            int side = 0;
            for (const Grid &g : fixed ? fx->grids : grids) side = std::max(side, g.s);
            const double full = full_cell(n, ncell, side);
            const int bits = bits_for(ncell);
            int most = 0;
            while (most < BIN_SHIFT && most < bits - 1 &&
                   (double)(2LL << most) * full <= (double)BIN_ROWS)
                most++;
            int shift = std::max(0, bits - RS_BITS * ((bits - most + RS_BITS - 1) / RS_BITS));
            while (shift < most && (double)(1LL << shift) * (double)n < 128.0 * (double)ncell) shift++;
            const int nb = (int)((ncell - 1) >> shift) + 1;
            const int tiles = (n + RS_TILE - 1) / RS_TILE;
            unsigned *kin = sc.get<unsigned>(n), *kout = sc.get<unsigned>(n);
            unsigned *pin = sc.get<unsigned>(n), *pout = sc.get<unsigned>(n);
            int *hist = sc.get<int>((size_t)RS_BINS * tiles), *totals = sc.get<int>(RS_BINS);
            int *start = sc.get<int>((size_t)nb + 1);
            for (int sh = shift; sh < bits; sh += RS_BITS) {
                const bool first = sh == shift;
                if (first)
                    k_cell_hist<<<tiles, RS_BLOCK, 0, s>>>(q, n, d_grids, n_mol, g0, kin, sh, hist, tiles);
                else
                    k_rs_hist<<<tiles, RS_BLOCK, 0, s>>>(kin, n, sh, hist, tiles);
                if (tiles > RS_FEW) k_rs_digit_prefix<<<RS_BINS, RS_PREFIX_BLOCK, 0, s>>>(hist, tiles, totals);
                if (first)
                    k_rs_scatter<unsigned, true><<<tiles, RS_BLOCK, 0, s>>>(kin, nullptr, kout, pout, n, sh, hist, totals, tiles);
                else
                    k_rs_scatter<unsigned><<<tiles, RS_BLOCK, 0, s>>>(kin, pin, kout, pout, n, sh, hist, totals, tiles);
                LAUNCH_CHECK();
                std::swap(kin, kout);
                std::swap(pin, pout);
            }
            if (n > KS_SEARCH) key_starts(kin, n, shift, nb, start, s);
            k_bin_finish<<<nb, BIN_BLOCK, 0, s>>>(kin, pin, n > KS_SEARCH ? start : nullptr, n, shift, ncell, q, pout, kout, cell_start, atom, sball,
                                                   (int)aq, perm, cnt);
            LAUNCH_CHECK();
        }

        // ---- neighbours and candidate edges: one pass into per-block slabs,
        // then compaction; count, scan and fill if a ball's rows overflow ----
        int *deg_n = sc.get<int>(n), *deg_up = sc.get<int>(n);
        int *nbr_start = sc.get<int>(n + 1), *up_start = sc.get<int>(n + 1);
        unsigned char *vgab = sc.get<unsigned char>(n);
        long long *vert_min = sc.get<long long>(n);
        const unsigned nbN = grid_for(n);
        // the radius that chooses the kernels
        long long rule = fixed ? fx->rule : kernel_radius(pp.sgc, large, n);
        if (fx && fx->learn) fx->rule = rule;
        int slot, lpb, nbs;
        unsigned nbB;  // blocks of the search
        int *nslab, *nbtot, *uoff, *poff;
        unsigned char *eng = sc.get<unsigned char>(n);
        const int *stop = fixed ? &cnt->stop : nullptr;  // kernels of a stopped recorded build return at once
        // f(SLOT, LPB) with the two as constants
        auto with_slot = [&](auto &&f) {
            using std::integral_constant;
            auto lanes = [&](auto sl) {
                if (lpb == 1) f(sl, integral_constant<int, 1>{});
                else if (lpb == 4) f(sl, integral_constant<int, 4>{});
                else f(sl, integral_constant<int, 16>{});
            };
            if (slot == NB_SLOT_SAS) f(integral_constant<int, NB_SLOT_SAS>{}, integral_constant<int, 4>{});
            else if (slot == NB_SLOT_WIDE) lanes(integral_constant<int, NB_SLOT_WIDE>{});
            else lanes(integral_constant<int, NB_SLOT>{});
        };
        Counters c0{};
        for (;;) {
            slot = neighbour_slot(rule, n, fx != nullptr);
            // lanes per ball: the search of a few balls is a chain of dependent
            // loads; from 2^18 balls on one lane each fills the GPU. Rows of the
            // widest slot are always shared by four (a lane lists at most 32).
            lpb = slot == NB_SLOT_SAS ? 4 : n >= (1 << 18) ? 1 : n >= (1 << 13) ? 4 : 16;
            nbB = (unsigned)((n + BLOCK / lpb - 1) / (BLOCK / lpb));
            nslab = sc.get<int>((size_t)nbB * (BLOCK / lpb) * slot + NBR_PAD);
            nbs = (int)(nbB + 3) & ~3;
            nbtot = sc.get<int>(3 * (size_t)nbs);
            uoff = sc.get<int>(nbB);
            poff = sc.get<int>(nbB);
            tm.mark(ST_NBR_COUNT);
            with_slot([&](auto sl, auto lp) {
                constexpr int SLOT = decltype(sl)::value, LPB = decltype(lp)::value;
                if (n_mol == 1)
                    k_neighbours<SLOT, LPB, true><<<nbB, BLOCK, 0, s>>>(atom, sball, perm, n, d_grids, n_mol, g0, cell_start, pp,
                                                                       deg_n, deg_up, nslab, nbtot, vgab, vert_min, cnt);
                else
                    k_neighbours<SLOT, LPB, false><<<nbB, BLOCK, 0, s>>>(atom, sball, perm, n, d_grids, n_mol, g0, cell_start, pp,
                                                                        deg_n, deg_up, nslab, nbtot, vgab, vert_min, cnt);
            });
            LAUNCH_CHECK();
            tm.mark(ST_NBR_SCAN);
            const unsigned nbr_seq = mb ? ++mb->seq : 0;
            k_nbr_scan<<<1, NBS_BLOCK, 0, s>>>(nbtot, (int)nbB, nbs, uoff, poff, cnt, mail, nbr_seq);
            LAUNCH_CHECK();
            if (fixed) {
                k_plan_guard<<<1, WAVE, 0, s>>>(cnt, fx->E_cap, fx->P_cap);
                LAUNCH_CHECK();
                c0.E = fx->E_cap;
            } else {
                c0 = mb ? mail_wait(*mb, nbr_seq, s).c : read_one(cnt, s);
            }
            // (fixed scratch has no room for the wide slots too: the counted search)
            if (fx || t_arena || !c0.overflow || rule == pp.sgc) break;
            rule = pp.sgc;
            fill<int>(&cnt->overflow, 0, 1, s);
        }
        if (c0.dup) throw HipError{AC_E_DUPLICATE, "two balls have equal quantised centres"};
        const bool nbr_two_pass = c0.overflow != 0;
        // (the search's edges: fewer than there are where rows outgrew their slots)
        const int gshift = fixed ? fx->gshift : group_shift(n, slot, c0.E);
        if (fx && fx->learn) fx->gshift = gshift;
        const int groups = ((n - 1) >> gshift) + 1;
        int *pair_base = sc.get<int>((size_t)groups + 1);
        int *pairs = nullptr;
        if (nbr_two_pass) {
            // exact counts and totals: neighbour entries, candidate edges, pairs
            k_nbr_rows<false><<<nbN, BLOCK, 0, s>>>(atom, sball, perm, n, d_grids, n_mol, g0, cell_start, pp, deg_n, deg_up, vgab,
                                                   nullptr, nullptr, nullptr, nullptr, nullptr, vert_min, cnt);
            pairs = sc.get<int>(groups);
            k_group_pairs<<<(groups + NWAVE - 1) / NWAVE, BLOCK, 0, s>>>(deg_up, n, gshift, groups, pairs, eng);
            LAUNCH_CHECK();
            sum_i64(deg_n, n, &cnt->Nn, s, sc);
            sum_i64(deg_up, n, &cnt->E, s, sc);
            sum_i64(pairs, groups, &cnt->P, s, sc);
            fill<int>(&cnt->overflow, 0, 1, s);
            c0 = read_one(cnt, s);
        }
        check_total(c0.Nn, "neighbour entries");
        check_total(c0.E, "candidate edges");
        // room for every pair, or (too many pairs) the counted triangles
        if (nbr_two_pass && rule < SAS_SGC && long_rows(c0.P, c0.E) &&
            !(t_arena && counts_triangles_in((long long)(t_arena->cap - t_arena->used), c0.P, n, c0.E, c0.Nn, groups,
                                             tet_slab(SAS_SGC, gshift, groups, 0))))
            rule = SAS_SGC;
        const int cut = nbr_two_pass && !t_arena && rule > APEX_SGC ? tet_split(groups) : 0, slices = groups << cut;
        const int tet_cap = tet_slab(rule, gshift, slices, fixed ? fx->tet_most : 0);
        const bool counted = fixed     ? fx->counted
                             : t_arena ? counts_triangles_in((long long)(t_arena->cap - t_arena->used), c0.P, n, c0.E, c0.Nn,
                                                             groups, tet_cap)
                                       : counts_triangles(c0.P);
        const int E = (int)c0.E;
        const long long Nn = c0.Nn;
        if (fx && fx->learn) {
            fx->E = E;
            fx->P = c0.P;
            fx->two_pass |= nbr_two_pass;
        }
        // neighbour rows: in the slabs after the one-pass search, else in CSR
        const size_t E1 = E > 0 ? E : 1;
        int *nbr = nbr_two_pass ? sc.get<int>((size_t)(Nn > 0 ? Nn : 1) + NBR_PAD) : nslab;
        int *up = sc.get<int>(E1), *up_id = sc.get<int>(E1), *edge_i = sc.get<int>(E1);
        tm.mark(ST_NBR_FILL);
        if (!nbr_two_pass) {
            with_slot([&](auto sl, auto lp) {
                constexpr int SLOT = decltype(sl)::value, LPB = decltype(lp)::value;
                // the balls of a block: as many as one lane each where the search
                // had one lane per ball, else one wave's
                constexpr int CB = LPB == 1 ? BLOCK : WAVE;
                k_nbr_compact<SLOT, LPB, CB><<<(n + CB - 1) / CB, BLOCK, 0, s>>>(deg_n, deg_up, n, nslab, uoff, poff, perm,
                                                                                nbr_start, up_start, up, up_id, edge_i,
                                                                                pair_base, gshift, eng, stop);
            });
            LAUNCH_CHECK();
        } else {
            scan_i32(deg_n, nbr_start, n, s, sc);
            scan_i32(deg_up, up_start, n, s, sc);
            if (!counted) scan_i32(pairs, pair_base, groups, s, sc);
            // the search's slabs are free again
            const bool in_slab = 2 * E1 <= (size_t)nbB * (BLOCK / lpb) * slot;
            int *up_scan = in_slab ? nslab : sc.get<int>(E1), *id_scan = in_slab ? nslab + E1 : sc.get<int>(E1);
            k_nbr_rows<true><<<nbN, BLOCK, 0, s>>>(atom, sball, perm, n, d_grids, n_mol, g0, cell_start, pp, nullptr, nullptr,
                                                  nullptr, nbr_start, up_start, nbr, up_scan, edge_i, vert_min, cnt);
            k_up_ids<<<grid_for(E), BLOCK, 0, s>>>(up_scan, E, perm, id_scan);
            k_up_rank<<<grid_for(E), BLOCK, 0, s>>>(up_scan, id_scan, E, edge_i, up_start, up, up_id);
            LAUNCH_CHECK();
        }
        unsigned char *egab = sc.get<unsigned char>(E1);
        long long *edge_min = sc.get<long long>(E1);

        // ---- candidate triangles of every group ----
        Cands cd{};
        cd.atom = atom;
        cd.perm = perm;
        cd.nbr_start = nbr_start;
        cd.nbr_cnt = deg_n;
        cd.nbr = nbr;
        cd.up_start = up_start;
        cd.up = up;
        cd.up_id = up_id;
        cd.edge_i = edge_i;
        cd.tri_base = pair_base;
        cd.tri_cnt = sc.get<int>(groups);
        cd.n = n;
        cd.gshift = gshift;
        // balls of a block of k_ac2: no more than a group, and rows that fit
        cd.sshift = gshift;
        while ((slot << cd.sshift) > AC2_ROWS) cd.sshift--;
        cd.tri_sub = sc.get<int>(((size_t)(n - 1) >> cd.sshift) + 1);
        tm.mark(ST_TRI_COUNT);
        long long room = fixed ? fx->P_cap : c0.P;
        auto triangles = [&](auto count, long long *mins) {
            if (nbr_two_pass)
                k_triangles<decltype(count)::value, true><<<groups, BLOCK, 0, s>>>(cd, pp, mins, cnt, stop);
            else
                k_triangles<decltype(count)::value, false><<<groups, BLOCK, 0, s>>>(cd, pp, mins, cnt, stop);
            LAUNCH_CHECK();
        };
        if (counted) {
            triangles(std::true_type{}, nullptr);
            if (fixed) {
                sum_i64(cd.tri_cnt, groups, &cnt->T, s, sc);
                k_plan_guard_triangles<<<1, WAVE, 0, s>>>(cnt, fx->T_cap);
                LAUNCH_CHECK();
                room = fx->T_cap;
            } else {
                room = total_i64(cd.tri_cnt, groups, s, sc);
            }
            check_total(room, "candidate triangles");
            scan_i32(cd.tri_cnt, pair_base, groups, s, sc);
        }
        const size_t T1 = room > 0 ? (size_t)room : 1;
        cd.tri_e = sc.get<int>(T1);
        cd.tri_f = sc.get<int>(T1);
        cd.tri_first = sc.get<int>(E1);
        long long *tri_min = sc.get<long long>(T1);
        unsigned char *tgab = sc.get<unsigned char>(T1);
        double *tsize = sc.get<double>(T1);
        triangles(std::false_type{}, tri_min);
        tm.mark(ST_TRI_SCAN);  // the triangles are in place: no scan, no fill
        tm.mark(ST_TRI_FILL);

        // ---- AC2 of the edges and triangles, candidate tetrahedra and Step 2.
        // Kept tetrahedra are those of the regular triangulation, about 6.8 a
        // ball at most where the radii are large, far fewer at alpha = 0 with
        // van der Waals radii; a group past its slab is counted and run again
        const bool use_apex = rule > APEX_SGC;
        int2 *apex = use_apex ? sc.get<int2>(T1) : nullptr;
        Tets tt{};
        tt.cap = tet_cap;
        tt.split = cut;
        tt.num = sc.get<int>(slices);
        tt.kept = sc.get<int>(groups);
        tt.cand = sc.get<int>(groups);
        tt.slice_cand = cut > 0 ? sc.get<int>(slices) : tt.cand;
        auto tet_room = [&](size_t rows) {
            if (rows < 1) rows = 1;
            tt.t = sc.get<int>(rows);
            tt.t2 = sc.get<int>(rows);
            tt.size = sc.get<double>(rows);
            if (n_alpha > 1) tt.face = sc.get<int4>(rows);
        };
        tet_room((size_t)slices * tt.cap);
        auto tetrahedra = [&]() {
            if (use_apex)
                k_tetrahedra<true><<<slices, BLOCK, 0, s>>>(cd, pp, apex, tt, cnt, stop);
            else
                k_tetrahedra<false><<<groups, BLOCK, 0, s>>>(cd, pp, apex, tt, cnt, stop);
            LAUNCH_CHECK();
        };
        auto tet_ac2 = [&]() {
            const bool few = rule <= 2000;  // below one candidate a ball
            auto run = [&](auto sweep) {
                constexpr bool SW = decltype(sweep)::value;
                if (nbr_two_pass) {
                    k_tet_test<<<dim3(slices, std::max(1, tests_split(groups) >> cut)), BLOCK, 0, s>>>(cd, pp, tt, cnt);
                    k_tet_ac2<SW, BLOCK, true><<<groups, BLOCK, 0, s>>>(cd, pp, tgab, tri_min, tt, cnt, stop);
                } else if (few) {
                    k_tet_ac2<SW, WAVE><<<groups, WAVE, 0, s>>>(cd, pp, tgab, tri_min, tt, cnt, stop);
                } else {
                    k_tet_ac2<SW, BLOCK><<<groups, BLOCK, 0, s>>>(cd, pp, tgab, tri_min, tt, cnt, stop);
                }
                LAUNCH_CHECK();
            };
            if (n_alpha > 1) run(std::true_type{});
            else run(std::false_type{});
        };
        // counted ranges for every group's tetrahedra, after an overflow: both
        // kernels again (k_tet_ac2 did nothing the first time)
        auto tet_counted = [&]() {
            const long long q = total_i64(tt.num, slices, s, sc);
            check_total(q, "candidate tetrahedra");
            int *base = sc.get<int>((size_t)slices + 1);
            scan_i32(tt.num, base, slices, s, sc);
            tt.tet_base = base;
            tet_room((size_t)q);
            fill<int>(&cnt->overflow, 0, 1, s);
            if (fx && fx->learn) {
                std::vector<int> num(slices);
                read_back(num.data(), tt.num, (size_t)slices, s);
                fx->tet_most = *std::max_element(num.begin(), num.end());
                fx->tet_limit = INDEX_LAST / slices;
            }
            tetrahedra();
            tet_ac2();
        };
        const Ac2Out ao{egab, edge_min, eng, tgab, tsize, apex};
        const int parts = (int)((n - 1) >> cd.sshift) + 1;
        auto ac2 = [&](auto sl, int what) {
            constexpr int SLOT = decltype(sl)::value;
            const dim3 blocks(parts, SLOT ? 1 : rows_split(parts));
            if (use_apex)
                k_ac2<SLOT, true><<<blocks, AC2_BLOCK, 0, s>>>(cd, pp, what, ao, cnt, stop);
            else
                k_ac2<SLOT, false><<<blocks, AC2_BLOCK, 0, s>>>(cd, pp, what, ao, cnt, stop);
            LAUNCH_CHECK();
        };
        auto ac2_of = [&](int what) {
            if (nbr_two_pass) ac2(std::integral_constant<int, 0>{}, what);
            else with_slot([&](auto sl, auto) { ac2(sl, what); });
        };
        if (split) {
            tm.mark(ST_EDGE_AC2);
            ac2_of(AC2_EDGES);
            tm.mark(ST_TRI_AC2);
            ac2_of(AC2_TRIANGLES);
            tm.mark(ST_TRI_GABRIEL);
            tetrahedra();
        } else if (n <= TET_AC2_BALLS && !use_apex && !nbr_two_pass) {
            tm.mark(ST_TRI_GABRIEL);
            with_slot([&](auto sl, auto) {
                k_tetrahedra_ac2<decltype(sl)::value><<<groups + parts, BLOCK, 0, s>>>(cd, pp, groups, tt, ao, cnt, stop);
                LAUNCH_CHECK();
            });
        } else {
            tm.mark(ST_TRI_GABRIEL);
            ac2_of(AC2_EDGES | AC2_TRIANGLES);
            tetrahedra();
        }
        tm.mark(ST_TET_COUNT);  // in place: no scan, no fill
        tm.mark(ST_TET_FILL);
        tm.mark(ST_TETRA);
        tet_ac2();

        // ---- pruning and output ----
        int4 *rec = sc.get<int4>((size_t)n + 1);
        const int rec_tiles = (n + REC_TILE - 1) / REC_TILE;
        int4 *tile_sum = rec_tiles > 1 ? sc.get<int4>(rec_tiles) : nullptr;
        OutCap out_cap{INT_MAX, INT_MAX, INT_MAX};
        if (fixed) out_cap = {fx->E_cap, fx->T_cap, fx->Q_cap};
        // the records scanned, and the vertices (out0 / size0; a sweep's records hold none)
        unsigned rec_seq = 0;
        auto scan_records = [&](int *out0, double *size0) {
            rec_seq = mb ? ++mb->seq : 0;
            const bool sums = rec_tiles > 1 && rec_tiles <= REC_BLOCK, scanned = rec_tiles > REC_BLOCK;
            if (rec_tiles > 1) k_rec_sums<<<rec_tiles, REC_BLOCK, 0, s>>>(rec, vert_min, n, tile_sum, stop);
            if (scanned)
                k_rec_prefix<<<1, 1024, 0, s>>>(tile_sum, rec_tiles, cd.tri_cnt, tt.cand, groups, cnt, fixed, out_cap,
                                               STOP_CAPACITY, mail, rec_seq);
            k_rec_apply<<<rec_tiles, REC_BLOCK, 0, s>>>(rec, vert_min, n, tile_sum, sums, out0, size0, cd.tri_cnt, tt.cand,
                                                       groups, cnt, fixed, out_cap, STOP_CAPACITY,
                                                       scanned ? nullptr : mail, rec_seq);
            LAUNCH_CHECK();
        };
        // the counters as the scan of the records left them
        auto rec_counters = [&]() { return mb ? mail_wait(*mb, rec_seq, s).c : read_one(cnt, s); };
        auto dev_rows = [&](ac_complex *r, int d, long long rows) {
            const size_t m = rows > 0 ? (size_t)rows : 1;
            r->d_simp[d] = static_cast<int32_t *>(dev_alloc(m * (d + 1) * sizeof(int32_t)));
            r->d_size[d] = static_cast<double *>(dev_alloc(m * sizeof(double)));
        };
        long long *d_bound = nullptr;
        if (n_mol > 1 && fixed) {
            d_bound = const_cast<long long *>(fx->d_bound);
        } else if (n_mol > 1) {
            d_bound = sc.get<long long>(n_mol + 1);
            HIP_TRY(hipMemcpyAsync(d_bound, bt.off.data(), (n_mol + 1) * sizeof(long long), hipMemcpyHostToDevice, s));
        }
        long long *d_rows = n_mol > 1 ? sc.get<long long>((size_t)n_alpha * 4 * (n_mol + 1)) : nullptr;
        Counters cf{};
        std::vector<Counters> cm(n_alpha);

        if (n_alpha == 1) {
            int2 *ball_cnt = sc.get<int2>(n);
            dev_rows(res, 0, n);
            int *tri_list = use_apex ? sc.get<int>(T1) : nullptr, *tri_kept = use_apex ? sc.get<int>(groups) : nullptr;
            auto prune = [&]() {
                if (use_apex)
                    k_tri_final<true><<<groups, BLOCK, 0, s>>>(cd, tgab, tsize, tri_min, egab, eng, edge_min, tt, ball_cnt,
                                                               tri_list, tri_kept, cnt, stop);
                else
                    k_tri_final<false><<<groups, BLOCK, 0, s>>>(cd, tgab, tsize, tri_min, egab, eng, edge_min, tt, ball_cnt,
                                                                nullptr, nullptr, cnt, stop);
                LAUNCH_CHECK();
                tm.mark(ST_EDGE_FINAL);
                k_edge_final<<<grid_for(n), BLOCK, 0, s>>>(cd, pp, o.vertex_shortcut, egab, edge_min, vgab, eng, vert_min,
                                                          ball_cnt, rec, cnt, stop);
                LAUNCH_CHECK();
                tm.mark(ST_VERT_FINAL);
                scan_records(res->d_simp[0], res->d_size[0]);
                if (n_mol > 1) {
                    k_mol_rows<<<(unsigned)((n_mol + 256) / 256), 256, 0, s>>>(rec, d_bound, n_mol, d_rows, stop);
                    LAUNCH_CHECK();
                }
            };
            auto write_rows = [&]() {
                auto rows = [&](auto list) {
                    k_rows<decltype(list)::value><<<groups, BLOCK, 0, s>>>(
                        cd, pp, rec, egab, edge_min, tgab, tsize, tri_min, tt, ball_cnt, tri_list, tri_kept, res->d_simp[1],
                        res->d_size[1], res->d_simp[2], res->d_size[2], res->d_simp[3], res->d_size[3], stop);
                };
                if (use_apex) rows(std::true_type{});
                else rows(std::false_type{});
                LAUNCH_CHECK();
            };
            tm.mark(ST_TRI_FINAL);
            prune();
            // Outputs sized for every candidate where that is little memory: the
            // rows are then written before the counts are read, one wait in
            // all. Else the counts are read first.
            const long long q_room = (long long)slices * tt.cap;
            const bool roomy = fixed || !ext && E * 16LL + room * 20LL + q_room * 24LL <= OUT_ROOM;
            if (roomy) {
                dev_rows(res, 1, fixed ? fx->E_cap : E);
                dev_rows(res, 2, fixed ? fx->T_cap : room);
                dev_rows(res, 3, fixed ? fx->Q_cap : q_room);
                tm.mark(ST_EMIT);
                write_rows();
                tm.mark(ST_COUNT);
            }
            if (fixed) {
                // nothing is read back: the plan reads the counters after a replay
                fx->cnt = cnt;
                fx->d_rows = d_rows;
                outs[0] = res;
                return AC_OK;
            }
            cf = rec_counters();
            const bool again = cf.overflow != 0;  // a group kept more tetrahedra than its slab holds
            if (again) {
                tet_counted();
                prune();
                cf = rec_counters();
            }
            if (cf.lookup) throw HipError{AC_E_DEVICE, "internal error: a facet of a kept simplex is not a candidate"};
            if (again && roomy) {
                dev_free(res->d_simp[3]);
                dev_free(res->d_size[3]);
                res->d_simp[3] = nullptr;
                res->d_size[3] = nullptr;
                dev_rows(res, 3, cf.m3);
            }
            if (ext) {
                // into the caller's arrays, if they are large enough
                const int m[4] = {cf.m0, cf.m1, cf.m2, cf.m3};
                ext->fits = true;
                for (int d = 0; d < 4; d++) ext->fits = ext->fits && m[d] <= ext->cap[d];
                if (ext->fits) {
                    for (int d = 1; d < 4; d++) {
                        res->d_simp[d] = ext->simp[d];
                        res->d_size[d] = ext->size[d];
                    }
                    if (m[0] > 0) {
                        HIP_TRY(hipMemcpyAsync(ext->simp[0], res->d_simp[0], (size_t)m[0] * sizeof(int32_t),
                                               hipMemcpyDeviceToDevice, s));
                        HIP_TRY(hipMemcpyAsync(ext->size[0], res->d_size[0], (size_t)m[0] * sizeof(double),
                                               hipMemcpyDeviceToDevice, s));
                    }
                }
            } else if (!roomy) {
                dev_rows(res, 1, cf.m1);
                dev_rows(res, 2, cf.m2);
                dev_rows(res, 3, cf.m3);
            }
            if ((again || !roomy) && !(ext && !ext->fits)) {
                tm.mark(ST_EMIT);
                write_rows();
                tm.mark(ST_COUNT);
            }
            // the scratch goes back to the pool: its last reader has to end
            HIP_TRY(hipStreamSynchronize(s));
            if (ext)
                for (int d = 1; d < 4; d++) {
                    res->d_simp[d] = nullptr;
                    res->d_size[d] = nullptr;
                }
            cm[0] = cf;
            if (fx && fx->learn) {
                fx->T = cf.T;
                fx->Q = cf.m3;
            }
        } else {
            // ---- sweep: the output order of every candidate and each
            // candidate's AC3 threshold once; then per alpha, comparisons,
            // pruning and compaction in output order ----
            auto places = [&]() {
                k_sweep_counts<<<groups, BLOCK, 0, s>>>(cd, tt, rec);
                LAUNCH_CHECK();
                scan_records(nullptr, nullptr);
                return rec_counters();
            };
            Counters cp = places();
            if (cp.overflow) {
                tet_counted();
                cp = places();
            }
            const int M[4] = {n, cp.m1, cp.m2, cp.m3};
            const int T = M[2], Q = M[3];
            const size_t T1s = T > 0 ? T : 1, Q1 = Q > 0 ? Q : 1;
            int *rows_s[4] = {}, *thr[4] = {};
            double *szp[4] = {};
            for (int d = 1; d <= 3; d++) {
                const size_t m = M[d] > 0 ? M[d] : 1;
                rows_s[d] = sc.get<int>(m * (d + 1));
                thr[d] = sc.get<int>(m);
                szp[d] = sc.get<double>(m);
            }
            int2 *vert = sc.get<int2>(n);
            int4 *face2 = sc.get<int4>(T1s);
            int4 *face3 = sc.get<int4>(Q1);
            int4 *adj = sc.get<int4>(n);
            k_sweep_adj<<<groups, BLOCK, 0, s>>>(cd, tt, rec, adj);
            if (E > 0)
                k_sweep_prep_edge<<<grid_for(E), BLOCK, 0, s>>>(cd, E, egab, adj, aq, thr[1], szp[1], rows_s[1]);
            k_sweep_prep_tri<<<groups, BLOCK, 0, s>>>(cd, tgab, tsize, adj, pp, thr[2], szp[2], rows_s[2], face2, cnt);
            k_sweep_prep_tet<<<groups, BLOCK, 0, s>>>(cd, tt, adj, pp, thr[3], szp[3], rows_s[3], face3, cnt);
            k_sweep_prep_vert<<<grid_for(n), BLOCK, 0, s>>>(cd, vgab, o.vertex_shortcut, vert);
            LAUNCH_CHECK();
            // per-alpha kept counts (m0..m3 of cs[k]); the main counters keep
            // the candidate totals, the fallback count and the lookup flag
            Counters *cs = sc.get<Counters>(n_alpha);
            HIP_TRY(hipMemsetAsync(cs, 0, n_alpha * sizeof(Counters), s));
            // alphas of a launch: as many as their minima have room for
            const size_t per = (size_t)n + E + T;
            const int chunk = (int)std::min<long long>(std::min(n_alpha, SWEEP_ALPHAS),
                                                       std::max<long long>(1, (long long)(SWEEP_ROOM / (8 * per))));
            Sweep sw{};
            sw.vert = vert;
            sw.face2 = face2;
            sw.face3 = face3;
            long long *mins = sc.get<long long>(per * chunk);
            sw.mins[0] = mins;
            sw.mins[1] = mins + (size_t)n * chunk;
            sw.mins[2] = sw.mins[1] + (size_t)E * chunk;
            for (int d = 0; d < 4; d++) {
                sw.m[d] = M[d];
                sw.nb[d] = M[d] > 0 ? (int)grid_for(M[d]) : 0;
                sw.thr[d] = thr[d];
                sw.sz[d] = szp[d];
                sw.rows[d] = rows_s[d];
                sw.tsum[d] = sc.get<int>((size_t)std::max(sw.nb[d], 1) * chunk);
            }
            tm.mark(ST_TRI_FINAL);
            tm.mark(ST_EDGE_FINAL);
            tm.mark(ST_VERT_FINAL);
            tm.mark(ST_EMIT);
            for (int k0 = 0; k0 < n_alpha; k0 += chunk) {
                const int na = std::min(chunk, n_alpha - k0);
                for (int a = 0; a < na; a++) {
                    sw.aq[a] = aqs[k0 + a];
                    sw.totals[a] = cs + k0 + a;
                    for (int d = 0; d < 4; d++) {
                        dev_rows(rs[k0 + a], d, M[d]);
                        sw.out[a][d] = rs[k0 + a]->d_simp[d];
                        sw.out_size[a][d] = rs[k0 + a]->d_size[d];
                    }
                }
                fill<long long>(mins, ORDERED_POS_INF, (long long)per * chunk, s);
                if (sw.nb[3]) k_sweep_mark<3><<<dim3(sw.nb[3], na), BLOCK, 0, s>>>(sw, cnt);
                if (sw.nb[2]) k_sweep_mark<2><<<dim3(sw.nb[2], na), BLOCK, 0, s>>>(sw, cnt);
                if (sw.nb[1]) k_sweep_mark<1><<<dim3(sw.nb[1], na), BLOCK, 0, s>>>(sw, cnt);
                k_sweep_mark<0><<<dim3(sw.nb[0], na), BLOCK, 0, s>>>(sw, cnt);
                k_sweep_scan<<<dim3(4, na), 1024, 0, s>>>(sw);
                k_sweep_write<<<dim3(sw.nb[0] + sw.nb[1] + sw.nb[2] + sw.nb[3], na), BLOCK, 0, s>>>(sw);
                LAUNCH_CHECK();
            }
            tm.mark(ST_COUNT);
            read_back(cm.data(), cs, (size_t)n_alpha, s);
            cf = read_one(cnt, s);
            if (cf.lookup) throw HipError{AC_E_DEVICE, "internal error: a facet of a kept simplex is not a candidate"};
        }

        // ---- results ----
        std::vector<int64_t> rows;
        if (n_mol > 1) {
            rows.resize((size_t)n_alpha * 4 * (n_mol + 1));
            read_back(rows.data(), (const int64_t *)d_rows, rows.size(), s);
        }
        tm.collect(res->stage_ms);
        for (int k = 0; k < n_alpha; k++) {
            ac_complex *r = rs[k];
            if (k > 0) std::copy(res->stage_ms, res->stage_ms + 32, r->stage_ms);
            r->n_mol = n_mol;
            r->alpha_q = aqs[k];
            r->cand[0] = n;
            r->cand[1] = E;
            r->cand[2] = cf.T;
            r->cand[3] = cf.Q;
            r->fallbacks = (int64_t)cf.exact_fallbacks;
            r->work[0] = ncell;
            r->work[1] = Nn;
            r->n = n;
            r->count[0] = cm[k].m0;
            r->count[1] = cm[k].m1;
            r->count[2] = cm[k].m2;
            r->count[3] = cm[k].m3;
            for (int d = 0; d < 4; d++) {
                if (n_mol > 1) {
                    const int64_t *b0 = rows.data() + ((size_t)k * 4 + d) * (n_mol + 1);
                    r->mol_rows[d].assign(b0, b0 + (n_mol + 1));
                } else {
                    r->mol_rows[d] = {0, r->count[d]};
                }
            }
        }
    } catch (const HipError &e) {
        (void)hipStreamSynchronize(s);
        if (ext && res)
            for (int d = 1; d < 4; d++) {  // the caller's
                res->d_simp[d] = nullptr;
                res->d_size[d] = nullptr;
            }
        for (ac_complex *r : rs) free_complex(r);
        return set_error(e.st, e.msg);
    }
    for (int k = 0; k < n_alpha; k++) outs[k] = rs[k];
    g_last_error.clear();
    return AC_OK;
}

static ac_status run_pipeline(const double *d_xyz, const double *d_r, int64_t n64, const Batch &bt, double alpha,
                              const Options &o, hipStream_t s, ac_complex **out) {
    return run_pipeline(d_xyz, d_r, n64, bt, &alpha, 1, o, s, out);
}

// ---------------------------------------------------------------------------
// Partitioned build (partition.hpp): slabs along x with a halo of 4 s_g plus
// 2 A, one pipeline run per slab, owned rows kept, then merged in output
// order. Peak scratch memory is that of the largest slab's build.

// Rows of dimension K - 1 that slab k owns, in emit form: flags, their scan
// and count (read back: the slab's memory is freed next), then the packed
// keys, payloads and (tetrahedra) Sizes, appended to the per-slab lists.
struct OwnedRows {
    std::vector<void *> key, pay, size;  // per slab with owned rows
    std::vector<int> count;
    long long total = 0;
    ~OwnedRows() {
        for (auto *v : {&key, &pay, &size})
            for (void *p : *v) dev_free(p);
    }
};

template <int K>
static void own_rows(const ac_complex *ck, const int *sel, const int4 *q, int x0, int w, int parts, int k,
                     hipStream_t s, Scope &sc, OwnedRows &own) {
    typedef typename EmitPay<K>::type P;
    const int d = K - 1;
    const int m = (int)ck->count[d];
    if (m == 0) return;
    int *flag = sc.get<int>(m);
    int *pos = sc.get<int>((size_t)m + 1);
    int *cnt = sc.get<int>(1);
    k_own_flags<K><<<grid_for(m), BLOCK, 0, s>>>(ck->d_simp[d], m, sel, q, x0, w, parts, k, flag);
    LAUNCH_CHECK();
    scan_i32(flag, pos, m, s, sc, cnt);
    const int c = read_one(cnt, s);
    if (c == 0) return;
    check_total(own.total + c, "simplices of one dimension");
    unsigned *key = static_cast<unsigned *>(dev_alloc((size_t)c * sizeof(unsigned)));
    own.key.push_back(key);
    P *pay = static_cast<P *>(dev_alloc((size_t)c * sizeof(P)));
    own.pay.push_back(pay);
    double *size = K == 4 ? static_cast<double *>(dev_alloc((size_t)c * sizeof(double))) : nullptr;
    if (size) own.size.push_back(size);
    k_own_emit<K><<<grid_for(m), BLOCK, 0, s>>>(ck->d_simp[d], ck->d_size[d], m, flag, pos, sel, (int)own.total, key,
                                                pay, size);
    LAUNCH_CHECK();
    own.count.push_back(c);
    own.total += c;
}

// All slabs' owned rows of dimension K - 1 in output order (into r).
template <int K>
static void merge_rows(OwnedRows &own, int n, hipStream_t s, Scope &sc, ac_complex *r, int *m_out) {
    typedef typename EmitPay<K>::type P;
    const int m = (int)own.total;
    unsigned *key = sc.get<unsigned>(m > 0 ? m : 1);
    P *pay = sc.get<P>(m > 0 ? m : 1);
    double *size = K == 4 ? sc.get<double>(m > 0 ? m : 1) : nullptr;
    long long off = 0;
    for (size_t j = 0; j < own.count.size(); j++) {
        const size_t c = (size_t)own.count[j];
        HIP_TRY(hipMemcpyAsync(key + off, own.key[j], c * sizeof(unsigned), hipMemcpyDeviceToDevice, s));
        HIP_TRY(hipMemcpyAsync(pay + off, own.pay[j], c * sizeof(P), hipMemcpyDeviceToDevice, s));
        if (size) HIP_TRY(hipMemcpyAsync(size + off, own.size[j], c * sizeof(double), hipMemcpyDeviceToDevice, s));
        off += (long long)c;
    }
    emit_dim<K>(key, pay, size, m, n, s, sc, r, K - 1, m_out);
}

static ac_status run_partitioned(const double *d_xyz, const double *d_r, int64_t n64, double alpha, int parts,
                                 const Options &o, hipStream_t s, ac_complex **out) {
    *out = nullptr;
    if (n64 < 1 || n64 >= (1 << 26)) return set_error(AC_E_INVALID, "n must be in [1, 2^26)");
    if (parts < 1 || parts > 64) return set_error(AC_E_INVALID, "parts must be in [1, 64]");
    if (!std::isfinite(alpha)) return set_error(AC_E_INVALID, "alpha is not finite");
    const double as = alpha * 1e6;
    if (!(std::fabs(as) < 67108864.0)) return set_error(AC_E_RANGE, "|alpha| too large for the exact bit budget");
    const long long aq = (long long)std::nearbyint(as);
    const int n = (int)n64;
    Scope sc;
    ac_complex *res = nullptr;
    ac_complex *ck = nullptr;
    try {
        // quantised centres, bounding box and the largest weight
        int4 *q = sc.get<int4>(n);
        const int n_tiles = (n + QTILE - 1) / QTILE;
        Stats *part = sc.get<Stats>(n_tiles);
        Stats *st = sc.get<Stats>(1);
        k_quantise<<<n_tiles, BLOCK, 0, s>>>(d_xyz, d_r, nullptr, n, INT_MAX, q, part, nullptr, nullptr, 0);
        k_stats_reduce<<<1, BLOCK, 0, s>>>(part, nullptr, n_tiles, st, nullptr, 0);
        LAUNCH_CHECK();
        const Stats h = read_one(st, s);
        if (h.flags & 1) throw HipError{AC_E_INVALID, "non-finite coordinate, or radius not positive"};
        if (h.flags & 2) throw HipError{AC_E_RANGE, "coordinate or radius outside the exact bit budget"};
        const long long sg2 = (long long)h.wmax + aq;
        if (sg2 >= (1LL << 26)) throw HipError{AC_E_RANGE, "r_max^2 + alpha too large for the exact bit budget"};
        const int halo = (int)(4 * isqrt_ceil(sg2 < 0 ? 0 : sg2) + 2000);
        const int x0 = h.minx;
        const int w = (int)(((long long)h.maxx - h.minx + parts) / parts);  // ceil((extent + 1) / parts)

        OwnedRows own[4];
        int *kept = sc.get<int>(n);
        double *vsize = sc.get<double>(n);
        fill<int>(kept, 0, n, s);
        int *flag = sc.get<int>(n);
        int *pos = sc.get<int>((size_t)n + 1);
        int *m_sub = sc.get<int>(1);
        long long fallbacks = 0;
        for (int k = 0; k < parts; k++) {
            const int lo = x0 + k * w, hi = k == parts - 1 ? INT_MAX - halo : lo + w;
            k_slab_flags<<<grid_for(n), BLOCK, 0, s>>>(q, n, lo, hi, halo, flag);
            LAUNCH_CHECK();
            scan_i32(flag, pos, n, s, sc, m_sub);
            const int ms = read_one(m_sub, s);
            if (ms == 0) continue;
            double *sub_xyz = sc.get<double>((size_t)ms * 3);
            double *sub_r = sc.get<double>(ms);
            int *sel = sc.get<int>(ms);
            k_slab_gather<<<grid_for(n), BLOCK, 0, s>>>(flag, pos, n, d_xyz, d_r, sub_xyz, sub_r, sel);
            LAUNCH_CHECK();
            Batch bt;
            bt.off = {0, ms};
            Options ok = o;
            ok.profile = 0;
            const ac_status stp = run_pipeline(sub_xyz, sub_r, ms, bt, alpha, ok, s, &ck);
            if (stp != AC_OK) throw HipError{stp, g_last_error};
            fallbacks += ck->fallbacks;
            if (ck->count[0] > 0) {
                k_own_vertices<<<grid_for(ck->count[0]), BLOCK, 0, s>>>(ck->d_simp[0], ck->d_size[0],
                                                                        (int)ck->count[0], sel, q, x0, w, parts, k,
                                                                        kept, vsize);
                LAUNCH_CHECK();
            }
            own_rows<2>(ck, sel, q, x0, w, parts, k, s, sc, own[1]);
            own_rows<3>(ck, sel, q, x0, w, parts, k, s, sc, own[2]);
            own_rows<4>(ck, sel, q, x0, w, parts, k, s, sc, own[3]);
            HIP_TRY(hipStreamSynchronize(s));  // the slab's result is consumed; free it
            free_complex(ck);
            ck = nullptr;
        }
        res = new ac_complex();
        for (double &x : res->stage_ms) x = -1.0;
        HIP_TRY(hipGetDevice(&res->device));
        res->device_result = true;
        // vertices: kept flags by input id
        int *m0 = sc.get<int>(1);
        scan_i32(kept, pos, n, s, sc, m0);
        res->d_simp[0] = static_cast<int32_t *>(dev_alloc((size_t)n * sizeof(int32_t)));
        res->d_size[0] = static_cast<double *>(dev_alloc((size_t)n * sizeof(double)));
        k_vertex_rows<<<grid_for(n), BLOCK, 0, s>>>(kept, pos, vsize, n, res->d_simp[0], res->d_size[0]);
        LAUNCH_CHECK();
        res->count[0] = read_one(m0, s);
        // higher dimensions: every slab's owned rows merged into output order
        int *mcount = sc.get<int>(4);
        merge_rows<2>(own[1], n, s, sc, res, mcount + 1);
        merge_rows<3>(own[2], n, s, sc, res, mcount + 2);
        merge_rows<4>(own[3], n, s, sc, res, mcount + 3);
        for (int d = 1; d <= 3; d++) res->count[d] = own[d].total;
        HIP_TRY(hipStreamSynchronize(s));
        res->n = n;
        res->n_mol = 1;
        for (int d = 0; d < 4; d++) {
            res->cand[d] = -1;
            res->mol_rows[d] = {0, res->count[d]};
        }
        res->fallbacks = fallbacks;
        res->alpha_q = aq;
        res->work[0] = res->work[1] = -1;
    } catch (const HipError &e) {
        (void)hipStreamSynchronize(s);
        free_complex(ck);
        free_complex(res);
        return set_error(e.st, e.msg);
    }
    *out = res;
    g_last_error.clear();
    return AC_OK;
}

// ---------------------------------------------------------------------------
// Host-streamed partitioned build: inputs and results stay in host memory.
// One slab at a time (its core and halo) is copied to the device, built, and
// the rows it owns are copied back in emit form; the slabs' lists, each
// sorted already, are merged on the host. Device memory is that of one
// slab's build.

template <int K> struct HostPay { static constexpr int words = K == 2 ? 3 : 4; };

// Owned rows of dimension K - 1 of all slabs, in host memory.
struct HostRows {
    std::vector<std::vector<uint32_t>> key, pay;  // per slab
    std::vector<std::vector<double>> size;        // per slab (K = 4)
};

template <int K>
static void own_rows_host(const ac_complex *ck, const int *sel, const int *qx, int x0, int w, int parts, int k,
                          hipStream_t s, Scope &sc, HostRows &hr) {
    typedef typename EmitPay<K>::type P;
    const int d = K - 1;
    const int m = (int)ck->count[d];
    if (m == 0) return;
    int *flag = sc.get<int>(m);
    int *pos = sc.get<int>((size_t)m + 1);
    int *cnt = sc.get<int>(1);
    k_own_flags_local<K><<<grid_for(m), BLOCK, 0, s>>>(ck->d_simp[d], m, sel, qx, x0, w, parts, k, flag);
    LAUNCH_CHECK();
    scan_i32(flag, pos, m, s, sc, cnt);
    const int c = read_one(cnt, s);
    if (c == 0) return;
    unsigned *key = sc.get<unsigned>(c);
    P *pay = sc.get<P>(c);
    double *size = K == 4 ? sc.get<double>(c) : nullptr;
    k_own_emit<K><<<grid_for(m), BLOCK, 0, s>>>(ck->d_simp[d], ck->d_size[d], m, flag, pos, sel, 0, key, pay, size);
    LAUNCH_CHECK();
    static_assert(sizeof(P) == HostPay<K>::words * sizeof(uint32_t), "payload words");
    hr.key.emplace_back((size_t)c);
    hr.pay.emplace_back((size_t)c * HostPay<K>::words);
    HIP_TRY(hipMemcpyAsync(hr.key.back().data(), key, (size_t)c * sizeof(unsigned), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipMemcpyAsync(hr.pay.back().data(), pay, (size_t)c * sizeof(P), hipMemcpyDeviceToHost, s));
    if (size) {
        hr.size.emplace_back((size_t)c);
        HIP_TRY(hipMemcpyAsync(hr.size.back().data(), size, (size_t)c * sizeof(double), hipMemcpyDeviceToHost, s));
    }
    HIP_TRY(hipStreamSynchronize(s));
}

// K-way merge of the slabs' sorted lists into output order (rows of K input
// ids, Sizes), in parallel over ranges of the least id.
template <int K>
static void merge_host(const HostRows &hr, int n, std::vector<int32_t> &rows, std::vector<double> &sizes) {
    constexpr int W = HostPay<K>::words;
    const size_t L = hr.key.size();
    size_t M = 0;
    for (const auto &k : hr.key) M += k.size();
    rows.assign(M * K + 1, 0);
    sizes.assign(M + 1, 0.0);
    if (M == 0) return;
    auto row_less = [&](size_t a, size_t ra, size_t b, size_t rb) {
        if (hr.key[a][ra] != hr.key[b][rb]) return hr.key[a][ra] < hr.key[b][rb];
        for (int u = 0; u < K - 1; u++) {
            const uint32_t x = hr.pay[a][ra * W + u], y = hr.pay[b][rb * W + u];
            if (x != y) return x < y;
        }
        return false;
    };
    const int T = (int)std::max<size_t>(1, std::min<size_t>(16, std::thread::hardware_concurrency()));
    std::vector<std::vector<size_t>> lo(T + 1, std::vector<size_t>(L));
    std::vector<size_t> start(T + 1, 0);
    for (int t = 0; t <= T; t++) {
        const uint32_t u = (uint32_t)((long long)n * t / T);
        for (size_t j = 0; j < L; j++) {
            lo[t][j] = t == T ? hr.key[j].size()
                              : (size_t)(std::lower_bound(hr.key[j].begin(), hr.key[j].end(), u) - hr.key[j].begin());
            start[t] += lo[t][j];
        }
    }
    auto work = [&](int t) {
        std::vector<size_t> at = lo[t];
        auto greater = [&](size_t a, size_t b) { return row_less(b, at[b], a, at[a]); };
        std::priority_queue<size_t, std::vector<size_t>, decltype(greater)> heap(greater);
        for (size_t j = 0; j < L; j++)
            if (at[j] < lo[t + 1][j]) heap.push(j);
        size_t out = start[t];
        while (!heap.empty()) {
            const size_t j = heap.top();
            heap.pop();
            const size_t r = at[j];
            rows[out * K] = (int32_t)hr.key[j][r];
            for (int u = 1; u < K; u++) rows[out * K + u] = (int32_t)hr.pay[j][r * W + u - 1];
            if constexpr (K == 4) {
                sizes[out] = hr.size[j][r];
            } else {
                const uint64_t b = (uint64_t)hr.pay[j][r * W + K - 1] | ((uint64_t)hr.pay[j][r * W + K] << 32);
                double z;
                std::memcpy(&z, &b, sizeof z);
                sizes[out] = z;
            }
            out++;
            if (++at[j] < lo[t + 1][j]) heap.push(j);
        }
    };
    std::vector<std::thread> th;
    for (int t = 1; t < T; t++) th.emplace_back(work, t);
    work(0);
    for (auto &x : th) x.join();
}

static ac_status run_streamed(const double *xyz, const double *r, int64_t n64, double alpha, int parts, const Options &o,
                              ac_complex **out) {
    *out = nullptr;
    if (!xyz || !r) return set_error(AC_E_INVALID, "NULL input pointer");
    if (n64 < 1 || n64 >= (1 << 26)) return set_error(AC_E_INVALID, "n must be in [1, 2^26)");
    if (parts < 1 || parts > 1024) return set_error(AC_E_INVALID, "parts must be in [1, 1024]");
    if (!std::isfinite(alpha)) return set_error(AC_E_INVALID, "alpha is not finite");
    const double as = alpha * 1e6;
    if (!(std::fabs(as) < 67108864.0)) return set_error(AC_E_RANGE, "|alpha| too large for the exact bit budget");
    const long long aq = (long long)std::nearbyint(as);
    const int n = (int)n64;
    // the slabs' bounds need the quantised x of every ball and the largest
    // weight: the same rounding (half to even) and checks as the device's
    std::vector<int> qx((size_t)n);
    long long wmax = 0;
    for (int i = 0; i < n; i++) {
        const double v = xyz[3 * (size_t)i];
        if (!std::isfinite(v)) return set_error(AC_E_INVALID, "non-finite coordinate, or radius not positive");
        const double sx = v * 1000.0;
        if (!(std::fabs(sx) < 524288.0)) return set_error(AC_E_RANGE, "coordinate or radius outside the exact bit budget");
        qx[i] = (int)std::nearbyint(sx);
        if (qx[i] >= 524288 || qx[i] <= -524288)
            return set_error(AC_E_RANGE, "coordinate or radius outside the exact bit budget");
        const double rv = r[i];
        if (!std::isfinite(rv) || !(rv > 0.0)) return set_error(AC_E_INVALID, "non-finite coordinate, or radius not positive");
        if (!(rv * 1000.0 < 8192.0)) return set_error(AC_E_RANGE, "coordinate or radius outside the exact bit budget");
        const long long R = (long long)std::nearbyint(rv * 1000.0);
        wmax = std::max(wmax, R * R);
    }
    const long long sg2 = wmax + aq;
    if (sg2 >= (1LL << 26)) return set_error(AC_E_RANGE, "r_max^2 + alpha too large for the exact bit budget");
    const int halo = (int)(4 * isqrt_ceil(sg2 < 0 ? 0 : sg2) + 2000);
    const int x0 = *std::min_element(qx.begin(), qx.end()), x1 = *std::max_element(qx.begin(), qx.end());
    const int w = (int)(((long long)x1 - x0 + parts) / parts);  // ceil((extent + 1) / parts)
    hipStream_t s = nullptr;
    ac_complex *res = nullptr, *ck = nullptr;
    void *pin = nullptr;
    try {
        // the slabs' balls (input order) and the largest slab
        std::vector<std::vector<int>> slab((size_t)parts);
        size_t big = 0;
        for (int k = 0; k < parts; k++) {
            const int lo = x0 + k * w, hi = k == parts - 1 ? INT_MAX - halo : lo + w;
            for (int i = 0; i < n; i++)
                if (qx[i] >= lo - halo && qx[i] < hi + halo) slab[k].push_back(i);
            big = std::max(big, slab[k].size());
        }
        const size_t stage = big * (4 * sizeof(double) + 2 * sizeof(int));
        HIP_TRY(hipHostMalloc(&pin, stage > 0 ? stage : 1, hipHostMallocDefault));
        double *hx = static_cast<double *>(pin), *hrad = hx + 3 * big;
        int *hsel = reinterpret_cast<int *>(hrad + big), *hqx = hsel + big;
        std::vector<double> vsize((size_t)n, std::numeric_limits<double>::quiet_NaN());
        HostRows rows[4];
        long long fallbacks = 0;
        for (int k = 0; k < parts; k++) {
            const int ms = (int)slab[k].size();
            if (ms == 0) continue;
            for (int t = 0; t < ms; t++) {
                const int i = slab[k][t];
                hx[3 * t] = xyz[3 * (size_t)i];
                hx[3 * t + 1] = xyz[3 * (size_t)i + 1];
                hx[3 * t + 2] = xyz[3 * (size_t)i + 2];
                hrad[t] = r[i];
                hsel[t] = i;
                hqx[t] = qx[i];
            }
            Scope sc;  // this slab's device memory, back to the pool after the slab
            double *dx = sc.get<double>(3 * (size_t)ms), *dr = sc.get<double>(ms);
            int *dsel = sc.get<int>(ms), *dqx = sc.get<int>(ms);
            HIP_TRY(hipMemcpyAsync(dx, hx, 3 * (size_t)ms * sizeof(double), hipMemcpyHostToDevice, s));
            HIP_TRY(hipMemcpyAsync(dr, hrad, (size_t)ms * sizeof(double), hipMemcpyHostToDevice, s));
            HIP_TRY(hipMemcpyAsync(dsel, hsel, (size_t)ms * sizeof(int), hipMemcpyHostToDevice, s));
            HIP_TRY(hipMemcpyAsync(dqx, hqx, (size_t)ms * sizeof(int), hipMemcpyHostToDevice, s));
            Batch bt;
            bt.off = {0, ms};
            Options ok = o;
            ok.profile = 0;
            const ac_status stp = run_pipeline(dx, dr, ms, bt, alpha, ok, s, &ck);
            if (stp != AC_OK) throw HipError{stp, g_last_error};
            fallbacks += ck->fallbacks;
            // vertices the slab owns: input id and Size
            const int m0 = (int)ck->count[0];
            if (m0 > 0) {
                int *flag = sc.get<int>(m0), *pos = sc.get<int>((size_t)m0 + 1), *cnt = sc.get<int>(1);
                k_own_flags_local<1><<<grid_for(m0), BLOCK, 0, s>>>(ck->d_simp[0], m0, dsel, dqx, x0, w, parts, k, flag);
                LAUNCH_CHECK();
                scan_i32(flag, pos, m0, s, sc, cnt);
                const int c = read_one(cnt, s);
                if (c > 0) {
                    int *oid = sc.get<int>(c);
                    double *osz = sc.get<double>(c);
                    k_own_vertices_local<<<grid_for(m0), BLOCK, 0, s>>>(ck->d_simp[0], ck->d_size[0], m0, flag, pos, dsel,
                                                                        oid, osz);
                    LAUNCH_CHECK();
                    std::vector<int> hid((size_t)c);
                    std::vector<double> hsz((size_t)c);
                    HIP_TRY(hipMemcpyAsync(hid.data(), oid, (size_t)c * sizeof(int), hipMemcpyDeviceToHost, s));
                    HIP_TRY(hipMemcpyAsync(hsz.data(), osz, (size_t)c * sizeof(double), hipMemcpyDeviceToHost, s));
                    HIP_TRY(hipStreamSynchronize(s));
                    for (int t = 0; t < c; t++) vsize[hid[t]] = hsz[t];
                }
            }
            own_rows_host<2>(ck, dsel, dqx, x0, w, parts, k, s, sc, rows[1]);
            own_rows_host<3>(ck, dsel, dqx, x0, w, parts, k, s, sc, rows[2]);
            own_rows_host<4>(ck, dsel, dqx, x0, w, parts, k, s, sc, rows[3]);
            HIP_TRY(hipStreamSynchronize(s));
            free_complex(ck);
            ck = nullptr;
        }
        res = new ac_complex();
        for (double &x : res->stage_ms) x = -1.0;
        HIP_TRY(hipGetDevice(&res->device));
        res->device_result = false;
        // vertices in input order
        std::vector<int32_t> &v0 = res->h_simp[0];
        std::vector<double> &z0 = res->h_size[0];
        for (int i = 0; i < n; i++)
            if (vsize[i] == vsize[i]) {
                v0.push_back(i);
                z0.push_back(vsize[i]);
            }
        res->count[0] = (int64_t)v0.size();
        v0.push_back(0);
        z0.push_back(0.0);
        merge_host<2>(rows[1], n, res->h_simp[1], res->h_size[1]);
        merge_host<3>(rows[2], n, res->h_simp[2], res->h_size[2]);
        merge_host<4>(rows[3], n, res->h_simp[3], res->h_size[3]);
        for (int d = 1; d <= 3; d++) res->count[d] = (int64_t)res->h_size[d].size() - 1;
        for (int d = 0; d < 4; d++) {
            res->host_ready[d] = true;
            res->cand[d] = -1;
            res->mol_rows[d] = {0, res->count[d]};
        }
        res->n = n;
        res->n_mol = 1;
        res->alpha_q = aq;
        res->fallbacks = fallbacks;
        res->work[0] = res->work[1] = -1;
        HIP_TRY(hipHostFree(pin));
        pin = nullptr;
    } catch (const HipError &e) {
        (void)hipStreamSynchronize(s);
        free_complex(ck);
        free_complex(res);
        if (pin) (void)hipHostFree(pin);
        return set_error(e.st, e.msg);
    } catch (const std::bad_alloc &) {
        (void)hipStreamSynchronize(s);
        free_complex(ck);
        free_complex(res);
        if (pin) (void)hipHostFree(pin);
        return set_error(AC_E_NOMEM, "host allocation failed");
    }
    *out = res;
    g_last_error.clear();
    return AC_OK;
}

// ---------------------------------------------------------------------------
// Union volume / area (measure.hpp)

static long long incidence_count(const ac_complex *c) {
    long long M = 0;
    for (int d = 0; d < 4; d++) M += c->count[d] * (d + 1);
    return M;
}

static void check_measure_args(const ac_complex *c, const double *d_xyz, const double *d_radii, int64_t n) {
    if (!c) throw HipError{AC_E_INVALID, "complex is NULL"};
    if (!d_xyz || !d_radii) throw HipError{AC_E_INVALID, "NULL input pointer"};
    if (n != c->n) throw HipError{AC_E_INVALID, "n differs from the number of balls the complex was built on"};
    if (c->alpha_q != 0)
        throw HipError{AC_E_INVALID, "the complex was built at alpha != 0; for the union of grown balls build the "
                                     "complex of radii sqrt(r^2 + alpha) at alpha = 0"};
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != c->device) throw HipError{AC_E_INVALID, "the complex lives on another device"};
    if (!has_index(incidence_count(c))) throw HipError{AC_E_CAPACITY, "too many simplex corners"};
}

static Simplices simplices_of(const ac_complex *c) {
    Simplices sx{};
    long long first = 0;
    int block0 = 0;
    for (int d = 0; d < 4; d++) {
        const long long corners = c->count[d] * (d + 1);
        sx.simp[d] = c->d_simp[d];
        sx.count[d] = c->count[d];
        sx.first[d] = first;
        sx.blocks[d] = (int)((corners + MEASURE_BLOCK - 1) / MEASURE_BLOCK);
        sx.block0[d] = block0;
        first += corners;
        block0 += sx.blocks[d];
    }
    return sx;
}
static int measure_blocks(const Simplices &sx) { return sx.block0[3] + sx.blocks[3]; }

// Sorts the corners of all simplices by ball id once per complex.
static void ensure_incidence(ac_complex *c, hipStream_t s) {
    if (c->inc_slot) return;
    const int M = (int)incidence_count(c);
    const int n = (int)c->n;
    int32_t *slot = static_cast<int32_t *>(dev_alloc((size_t)(M > 0 ? M : 1) * sizeof(int32_t)));
    int32_t *start = nullptr;
    try {
        start = static_cast<int32_t *>(dev_alloc((size_t)(n + 1) * sizeof(int32_t)));
        Scope sc;
        if (M > 0) {
            const IncBuckets ib = inc_buckets(n);
            const int passes = ib.passes, shift = ib.shift;
            const int nb = ((n - 1) >> shift) + 1;
            const int tiles = (M + RS_TILE - 1) / RS_TILE;
            unsigned *kin = sc.get<unsigned>(M), *kout = sc.get<unsigned>(M);
            unsigned *pin = sc.get<unsigned>(M), *pout = sc.get<unsigned>(M);
            int *hist = sc.get<int>((size_t)RS_BINS * tiles), *totals = sc.get<int>(RS_BINS);
            int *first = sc.get<int>((size_t)nb + 1);
            const Simplices sx = simplices_of(c);
            for (int k = 0, sh = shift; k < passes; k++, sh += RS_BITS) {
                if (k == 0)
                    k_inc_hist<<<tiles, RS_BLOCK, 0, s>>>(sx, M, kin, sh, hist, tiles);
                else
                    k_rs_hist<<<tiles, RS_BLOCK, 0, s>>>(kin, M, sh, hist, tiles);
                if (tiles > RS_FEW) k_rs_digit_prefix<<<RS_BINS, RS_PREFIX_BLOCK, 0, s>>>(hist, tiles, totals);
                if (k == 0)
                    k_rs_scatter<unsigned, true><<<tiles, RS_BLOCK, 0, s>>>(kin, nullptr, kout, pout, M, sh, hist, totals, tiles);
                else
                    k_rs_scatter<unsigned><<<tiles, RS_BLOCK, 0, s>>>(kin, pin, kout, pout, M, sh, hist, totals, tiles);
                LAUNCH_CHECK();
                std::swap(kin, kout);
                std::swap(pin, pout);
            }
            if (M > KS_SEARCH) key_starts(kin, M, shift, nb, first, s);
            k_inc_finish<<<nb, INC_BLOCK, 0, s>>>(kin, pin, M > KS_SEARCH ? first : nullptr, M, shift, n, start, slot);
            LAUNCH_CHECK();
        } else {
            fill<int>(start, 0, n + 1, s);
        }
        HIP_TRY(hipStreamSynchronize(s));  // before the scope's blocks go back to the pool
    } catch (...) {
        dev_free(slot);
        dev_free(start);
        throw;
    }
    c->inc_slot = slot;
    c->inc_start = start;
}

// Launches the measure kernels of every dimension.
template <bool VA, bool GRAD>
static void measure_launch(const Simplices &sx, const double *x, const double *r, const double *g, double4 *contrib,
                           double *part, hipStream_t s) {
    const int nb = measure_blocks(sx);
    if (nb > 0) k_measure<VA, GRAD><<<nb, MEASURE_BLOCK, 0, s>>>(sx, x, r, g, contrib, part);
    LAUNCH_CHECK();
}

// The complex's buffer of block parts, then V and A.
static double *measure_parts(ac_complex *c, int nb) {
    if (!c->meas_part) c->meas_part = static_cast<double *>(dev_alloc((size_t)(2 * (size_t)nb + 2) * sizeof(double)));
    return c->meas_part;
}

// Writes V, A to d_out (device), or to the complex's own buffer if d_out is
// NULL; returns where they are.
static double *measure_forward(ac_complex *c, const double *x, const double *r, double *d_out, hipStream_t s) {
    const Simplices sx = simplices_of(c);
    const int nb = measure_blocks(sx);
    double *part = measure_parts(c, nb);
    if (!d_out) d_out = part + 2 * (size_t)nb;
    measure_launch<true, false>(sx, x, r, nullptr, nullptr, part, s);
    k_measure_total<<<1, MEASURE_BLOCK, 0, s>>>(part, nb, d_out);
    LAUNCH_CHECK();
    return d_out;
}

// Validated molecule offsets of a batch call.
static ac_status batch_from(const int64_t *offsets, int64_t n_mol, const int32_t *cell_mA, Batch &bt) {
    if (!offsets) return set_error(AC_E_INVALID, "offsets is NULL");
    if (n_mol < 1 || n_mol > (1 << 20)) return set_error(AC_E_INVALID, "n_mol must be in [1, 2^20]");
    if (offsets[0] != 0) return set_error(AC_E_INVALID, "offsets[0] must be 0");
    bt.off.assign(offsets, offsets + n_mol + 1);
    for (int64_t m = 0; m < n_mol; m++)
        if (bt.off[m + 1] <= bt.off[m]) return set_error(AC_E_INVALID, "offsets must increase strictly (no empty molecule)");
    if (bt.off[n_mol] >= (1 << 26)) return set_error(AC_E_INVALID, "total balls must be below 2^26");
    bt.cell_mA.clear();
    if (cell_mA) {
        bt.cell_mA.assign(cell_mA, cell_mA + n_mol);
        for (int32_t c : bt.cell_mA)
            if (c < 1) return set_error(AC_E_INVALID, "cell sides must be positive");
    }
    return AC_OK;
}

// Time of one pipeline run on its stream (ms): two HIP events around the
// whole run, so that the idle time of its host synchronisations counts and
// no event between stages perturbs it.
static ac_status timed_run(const double *x, const double *r, int64_t n, const Batch &bt, double alpha, Options o,
                           hipStream_t s, double *ms) {
    o.profile = 0;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    HIP_TRY(hipEventCreate(&e0));
    if (hipEventCreate(&e1) != hipSuccess) {
        (void)hipEventDestroy(e0);
        throw HipError{AC_E_DEVICE, "hipEventCreate failed"};
    }
    ac_complex *c = nullptr;
    ac_status st = hipEventRecord(e0, s) == hipSuccess ? run_pipeline(x, r, n, bt, alpha, o, s, &c) : AC_E_DEVICE;
    float f = 0.f;
    if (st == AC_OK && (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                        hipEventElapsedTime(&f, e0, e1) != hipSuccess))
        st = set_error(AC_E_DEVICE, "timing events failed");
    free_complex(c);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    *ms = f;
    return st;
}

// Options of a call, validated: every field has a documented range and a
// value outside it is an argument error, not silently replaced.
static Options parse(const ac_options *opt) {
    Options o;
    if (!opt) return o;
    if (opt->reserved != 0) throw HipError{AC_E_INVALID, "ac_options.reserved must be 0"};
    if (opt->cell_mA < 0) throw HipError{AC_E_INVALID, "ac_options.cell_mA must be >= 0"};
    if (opt->wave_tile != 0)
        throw HipError{AC_E_INVALID, "ac_options.wave_tile must be 0 (every kernel maps one item to one lane)"};
    if (opt->capacity_hint != 0)
        throw HipError{AC_E_INVALID, "ac_options.capacity_hint must be 0 (buffers are sized from exact counts)"};
    if (opt->force_exact != 0 && opt->force_exact != 1) throw HipError{AC_E_INVALID, "ac_options.force_exact must be 0 or 1"};
    if (opt->vertex_shortcut != 0 && opt->vertex_shortcut != 1)
        throw HipError{AC_E_INVALID, "ac_options.vertex_shortcut must be 0 or 1"};
    if (opt->profile < 0 || opt->profile > PROFILE_SPLIT)
        throw HipError{AC_E_INVALID, "ac_options.profile must be 0, 1, 2 + a stage index or 2 + the stage count"};
    if (opt->cell_order != ORDER_ROW && opt->cell_order != ORDER_MORTON)
        throw HipError{AC_E_INVALID, "ac_options.cell_order must be 0 (row-major) or 1 (Morton)"};
    o.cell_mA = opt->cell_mA;
    o.force_exact = opt->force_exact;
    o.vertex_shortcut = opt->vertex_shortcut;
    o.profile = opt->profile;
    o.cell_order = opt->cell_order;
    return o;
}

// ---------------------------------------------------------------------------
// Recorded batch builds: one learning build notes the sizes, the fixed
// pipeline is run once to take its buffers and once under stream capture,
// and the captured graph is then replayed on new coordinates.
struct ac_plan {
    int device = 0;
    hipStream_t cap_stream = nullptr;  // the stream the graph was captured on
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    Fixed fx;
    Recorder rec;                 // the build's buffers, owned by the plan
    std::vector<void *> consts;   // uploaded tiles, grid templates, capacities, molecule bounds
    // what an ordinary build needs when a replay stops
    const double *d_xyz = nullptr, *d_r = nullptr;
    int64_t n = 0;
    Batch bt;
    double alpha = 0;
    Options o;
    int32_t *out_simp[4] = {};
    double *out_size[4] = {};
    int last_stop = 0;
    int64_t ordinary_builds = 0;
};

static void free_plan(ac_plan *p) {
    if (!p) return;
    if (p->exec) (void)hipGraphExecDestroy(p->exec);
    if (p->graph) (void)hipGraphDestroy(p->graph);
    if (p->cap_stream) {
        (void)hipStreamSynchronize(p->cap_stream);
        (void)hipStreamDestroy(p->cap_stream);
    }
    for (auto &b : p->rec.blocks) dev_free(b.first);
    for (void *c : p->consts) dev_free(c);
    delete p;
}

template <class T>
static T *upload(ac_plan *p, const T *h, size_t n, hipStream_t s) {
    T *d = static_cast<T *>(dev_alloc((n ? n : 1) * sizeof(T)));
    p->consts.push_back(d);
    if (n) HIP_TRY(hipMemcpyAsync(d, h, n * sizeof(T), hipMemcpyHostToDevice, s));
    return d;
}

// Sets t_rec for the duration of a scope.
struct RecordingOn {
    explicit RecordingOn(Recorder *r) { t_rec = r; }
    ~RecordingOn() { t_rec = nullptr; }
};

static ac_status plan_create(const double *d_xyz, const double *d_r, const Batch &bt, double alpha, const Options &o,
                             double headroom, hipStream_t s, ac_plan **out) {
    ac_plan *p = new ac_plan();
    try {
        HIP_TRY(hipGetDevice(&p->device));
        p->d_xyz = d_xyz;
        p->d_r = d_r;
        p->n = bt.off.back();
        p->bt = bt;
        p->alpha = alpha;
        p->o = o;
        const int n_mol = (int)bt.off.size() - 1;
        // 1. an ordinary build notes the sizes
        Fixed &fx = p->fx;
        fx.learn = true;
        ac_complex *r0 = nullptr;
        ac_status st = run_pipeline(d_xyz, d_r, p->n, bt, &alpha, 1, o, s, &r0, &fx);
        if (st != AC_OK) {
            free_plan(p);
            return st;
        }
        free_complex(r0);
        if (fx.two_pass)
            throw HipError{AC_E_CAPACITY, "a stage of this input needs the counted fill (rows longer than the "
                                          "single-pass slots); it has no recorded build"};
        // 2. capacities: the learned sizes with headroom; every molecule's
        // grid gets at least a cell per ball (a stopped molecule uses that)
        auto grow = [&](long long v) {
            const double c = std::ceil((double)v * headroom) + 256.0;
            if (c > (double)INDEX_LAST) throw HipError{AC_E_CAPACITY, "planned capacity beyond 2^31"};
            return (int)c;
        };
        fx.E_cap = grow(fx.E);
        const long long pairs = (long long)std::ceil((double)fx.P * headroom) + 256;
        fx.counted = counts_triangles(pairs);
        fx.P_cap = fx.counted ? LLONG_MAX : pairs;
        fx.T_cap = grow(fx.T);
        fx.Q_cap = grow(fx.Q);
        if (fx.tet_most > 0) fx.tet_most = grow(fx.tet_most);
        if (fx.tet_most > fx.tet_limit) throw HipError{AC_E_CAPACITY, "planned tetrahedron slabs beyond 2^31"};
        std::vector<long long> cap(n_mol);
        std::vector<Grid> tmpl = fx.grids;
        long long base = 0;
        for (int m = 0; m < n_mol; m++) {
            cap[m] = std::max<long long>((long long)std::ceil((double)fx.cells[m] * headroom), bt.off[m + 1] - bt.off[m]);
            tmpl[m].base = base;
            base += cap[m];
        }
        if (base >= (long long)INT_MAX) throw HipError{AC_E_CAPACITY, "planned grid cells beyond 2^31"};
        fx.ncell = base;
        std::vector<int2> tiles;
        std::vector<int> tile_first;
        quantise_tiles(bt, tiles, tile_first);
        std::vector<long long> bound(bt.off.begin(), bt.off.end());
        fx.d_tiles = upload(p, tiles.data(), tiles.size(), s);
        fx.d_tile_first = upload(p, tile_first.data(), tile_first.size(), s);
        fx.d_tmpl = upload(p, tmpl.data(), tmpl.size(), s);
        fx.d_cell_cap = upload(p, cap.data(), cap.size(), s);
        fx.d_bound = upload(p, bound.data(), bound.size(), s);
        HIP_TRY(hipStreamSynchronize(s));  // the host arrays above go out of scope
        fx.learn = false;
        // 3. the fixed pipeline once, taking (and recording) its buffers
        HIP_TRY(hipStreamCreateWithFlags(&p->cap_stream, hipStreamNonBlocking));
        ac_complex *r1 = nullptr;
        {
            const RecordingOn on(&p->rec);
            st = run_pipeline(d_xyz, d_r, p->n, bt, &alpha, 1, o, p->cap_stream, &r1, &fx);
            if (st != AC_OK) {
                free_plan(p);
                return st;
            }
            for (int d = 0; d < 4; d++) {
                p->out_simp[d] = r1->d_simp[d];
                p->out_size[d] = r1->d_size[d];
            }
            free_complex(r1);  // host object; its arrays are recorded blocks
        }
        Counters c{};
        read_back(&c, fx.cnt, 1, p->cap_stream);
        if (c.stop) throw HipError{AC_E_DEVICE, "internal error: the recorded build stopped on its own input"};
        // 4. the same launches captured in a graph, on the recorded buffers
        p->rec.replay = true;
        p->rec.next = 0;
        {
            const RecordingOn on(&p->rec);
            HIP_TRY(hipStreamBeginCapture(p->cap_stream, hipStreamCaptureModeThreadLocal));
            ac_complex *r2 = nullptr;
            try {
                st = run_pipeline(d_xyz, d_r, p->n, bt, &alpha, 1, o, p->cap_stream, &r2, &fx);
            } catch (...) {
                hipGraph_t g = nullptr;
                (void)hipStreamEndCapture(p->cap_stream, &g);
                if (g) (void)hipGraphDestroy(g);
                throw;
            }
            HIP_TRY(hipStreamEndCapture(p->cap_stream, &p->graph));
            if (st != AC_OK) {
                free_plan(p);
                return st;
            }
            bool same = p->rec.next == p->rec.blocks.size();
            for (int d = 0; d < 4; d++) same = same && r2->d_simp[d] == p->out_simp[d] && r2->d_size[d] == p->out_size[d];
            free_complex(r2);
            if (!same) throw HipError{AC_E_DEVICE, "internal error: the captured build used other buffers"};
        }
        HIP_TRY(hipGraphInstantiate(&p->exec, p->graph, nullptr, nullptr, 0));
        *out = p;
        g_last_error.clear();
        return AC_OK;
    } catch (const HipError &e) {
        t_rec = nullptr;
        free_plan(p);
        return set_error(e.st, e.msg);
    }
}

static ac_status plan_result(ac_plan *p, hipStream_t s, ac_complex **out) {
    const int n_mol = (int)p->bt.off.size() - 1;
    const Fixed &fx = p->fx;
    // Rows by capacity where that is little memory: their copies are enqueued
    // behind the replay, and the wait for the counts is the wait for the rows. Else
    // the counts come first. Either way the rows have left the plan's buffers and
    // are complete for every stream when this returns: host copies, the next
    // replay and ac_free order nothing.
    const bool roomy = p->n * 12LL + fx.E_cap * 16LL + fx.T_cap * 20LL + fx.Q_cap * 24LL <= OUT_ROOM;
    Counters c{};
    if (!roomy) read_back(&c, fx.cnt, 1, s);
    ac_complex *r = nullptr;
    std::vector<int64_t> rows;
    try {
        if (!c.stop) {
            r = new ac_complex();
            CopyList cl{};
            const long long cap[4] = {p->n, fx.E_cap, fx.T_cap, fx.Q_cap};
            const int m[4] = {c.m0, c.m1, c.m2, c.m3};
            long long most = 0;
            for (int d = 0; d < 4; d++) {
                const long long k = std::max<long long>(roomy ? cap[d] : m[d], 1);
                r->d_simp[d] = static_cast<int32_t *>(dev_alloc((size_t)k * (d + 1) * sizeof(int32_t)));
                r->d_size[d] = static_cast<double *>(dev_alloc((size_t)k * sizeof(double)));
                cl.src[2 * d] = p->out_simp[d];
                cl.dst[2 * d] = r->d_simp[d];
                cl.src[2 * d + 1] = reinterpret_cast<const int *>(p->out_size[d]);
                cl.dst[2 * d + 1] = reinterpret_cast<int *>(r->d_size[d]);
                most = std::max(most, k * std::max(2, d + 1));
            }
            k_copy_list<<<dim3((unsigned)std::min<long long>(most / 1024 + 1, roomy ? 256 : 2048), 8), 256, 0, s>>>(cl, fx.cnt);
            LAUNCH_CHECK();
        }
        if (roomy) read_back(&c, fx.cnt, 1, s);
        else HIP_TRY(hipStreamSynchronize(s));
        p->last_stop = c.stop;
        if (c.stop) {
            // the input did not fit the recording: an ordinary build of the same
            // arguments (it also reports invalid input)
            free_complex(r);
            r = nullptr;
            p->ordinary_builds++;
            const ac_status st = run_pipeline(p->d_xyz, p->d_r, p->n, p->bt, &p->alpha, 1, p->o, s, out);
            if (st == AC_OK) (*out)->batch = true;
            return st;
        }
        if (c.lookup) throw HipError{AC_E_DEVICE, "internal error: a facet of a kept simplex is not a candidate"};
        if (n_mol > 1) {
            rows.resize(4 * (size_t)(n_mol + 1));
            read_back(rows.data(), (const int64_t *)fx.d_rows, rows.size(), s);
        }
        for (double &x : r->stage_ms) x = -1.0;
        r->device = p->device;
        r->device_result = true;
        r->batch = true;
        r->n_mol = n_mol;
        r->n = p->n;
        r->alpha_q = (int64_t)std::nearbyint(p->alpha * 1e6);
        const int m[4] = {c.m0, c.m1, c.m2, c.m3};
        r->cand[0] = p->n;
        r->cand[1] = c.E;
        r->cand[2] = c.T;
        r->cand[3] = c.Q;
        r->fallbacks = (int64_t)c.exact_fallbacks;
        r->work[0] = fx.ncell;
        r->work[1] = c.Nn;
        for (int d = 0; d < 4; d++) {
            r->count[d] = m[d];
            if (n_mol > 1) {
                const int64_t *b0 = rows.data() + (size_t)d * (n_mol + 1);
                r->mol_rows[d].assign(b0, b0 + (n_mol + 1));
            } else {
                r->mol_rows[d] = {0, r->count[d]};
            }
        }
    } catch (...) {
        (void)hipStreamSynchronize(s);
        free_complex(r);
        throw;
    }
    *out = r;
    return AC_OK;
}

// ---------------------------------------------------------------------------
// Fixed device scratch of ac_alpha_complex_noalloc. Every device the library
// runs on holds one copy of this array until the process ends. In host code
// its name is only a stand-in: the device address of a device's copy comes
// from hipGetSymbolAddress, taken once per device with that device current,
// and only that address is handed to kernels and copies.
constexpr size_t NOALLOC_SCRATCH_BYTES = (size_t)AC_NOALLOC_SCRATCH_MIB << 20;
// a ball needs more than this much scratch whatever the input (quantised and
// sorted balls, sort keys, neighbour slots)
constexpr size_t NOALLOC_MIN_BYTES_PER_BALL = 128;
static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int NOALLOC_MAX_DEVICES = 64;
std::mutex g_scratch_mu[NOALLOC_MAX_DEVICES];  // held for a whole call: one call per device at a time
void *g_scratch_ptr[NOALLOC_MAX_DEVICES] = {};  // device address of each device's copy, once known
}  // namespace

// Device address of the scratch array on device `dev` (the current device;
// the caller holds g_scratch_mu[dev]).
static char *scratch_on(int dev) {
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) throw HipError{AC_E_DEVICE, "hipGetSymbolAddress gave no address for the scratch array"};
        g_scratch_ptr[dev] = p;
    }
    return static_cast<char *>(g_scratch_ptr[dev]);
}

// Host copies of dimensions d0..d1 of a device result: every copy enqueued,
// then one wait. False (with the error set) on a failed copy.
static bool host_copies(ac_complex *c, int d0, int d1) {
    for (int d = d0; d <= d1; d++) {
        const size_t m = (size_t)c->count[d];
        const size_t rows = m * (d + 1) * sizeof(int32_t), sizes = m * sizeof(double);
        void *rp = nullptr;
        double *zp = nullptr;
        if (!c->h_block[d]) {
            c->h_block[d] = host_alloc(rows + sizes + sizeof(double));
            c->h_bytes[d] = rows + sizes + sizeof(double);
        }
        if (c->h_block[d]) {
            zp = static_cast<double *>(c->h_block[d]);
            rp = zp + m;
        } else {
            c->h_simp[d].resize(m * (d + 1) + 1);
            c->h_size[d].resize(m + 1);
            rp = c->h_simp[d].data();
            zp = c->h_size[d].data();
        }
        if (m && (hipMemcpyAsync(rp, c->d_simp[d], rows, hipMemcpyDeviceToHost, nullptr) != hipSuccess ||
                  hipMemcpyAsync(zp, c->d_size[d], sizes, hipMemcpyDeviceToHost, nullptr) != hipSuccess)) {
            (void)hipStreamSynchronize(nullptr);
            set_error(AC_E_DEVICE, "device-to-host copy failed");
            return false;
        }
    }
    if (hipStreamSynchronize(nullptr) != hipSuccess) {
        set_error(AC_E_DEVICE, "device-to-host copy failed");
        return false;
    }
    for (int d = d0; d <= d1; d++) c->host_ready[d] = true;
    return true;
}

// ---------------------------------------------------------------------------
// C ABI
extern "C" {

ac_status ac_alpha_complex_device(const double *d_xyz, const double *d_radii, int64_t n, double alpha,
                                  const ac_options *opt, void *stream, ac_complex **out) {
    if (!out) return set_error(AC_E_INVALID, "out is NULL");
    *out = nullptr;
    try {
        const Options o = parse(opt);
        if (!d_xyz || !d_radii) return set_error(AC_E_INVALID, "NULL input pointer");
        Batch bt;
        bt.off = {0, n};
        return run_pipeline(d_xyz, d_radii, n, bt, alpha, o, static_cast<hipStream_t>(stream), out);
    } catch (const HipError &e) {
        return set_error(e.st, e.msg);
    } catch (...) {
        return set_error(AC_E_DEVICE, "unexpected host exception");
    }
}

ac_status ac_alpha_complex_noalloc(const double *d_xyz, const double *d_radii, int64_t n, double alpha,
                                   const ac_options *opt, void *stream, int32_t *const *d_simp,
                                   double *const *d_size, const int64_t *capacity, int64_t *counts) {
    if (!d_simp || !d_size || !capacity || !counts) return set_error(AC_E_INVALID, "NULL output argument");
    for (int d = 0; d < 4; d++) counts[d] = -1;
    ac_complex *c = nullptr;
    hipStream_t s = static_cast<hipStream_t>(stream);
    int dev = -1;
    try {
        const Options o = parse(opt);
        if (o.profile != 0) return set_error(AC_E_INVALID, "ac_options.profile must be 0 (profiling creates HIP events)");
        if (!d_xyz || !d_radii) return set_error(AC_E_INVALID, "NULL input pointer");
        if (n < 1 || n >= (1 << 26)) return set_error(AC_E_INVALID, "n must be in [1, 2^26)");
        for (int d = 0; d < 4; d++) {
            if (capacity[d] < 0) return set_error(AC_E_INVALID, "capacity must be >= 0");
            if (capacity[d] > 0 && (!d_simp[d] || !d_size[d]))
                return set_error(AC_E_INVALID, "NULL output buffer with a non-zero capacity");
        }
        if ((size_t)n > NOALLOC_SCRATCH_BYTES / NOALLOC_MIN_BYTES_PER_BALL)
            return set_error(AC_E_CAPACITY, "n exceeds what the " + std::to_string(AC_NOALLOC_SCRATCH_MIB) +
                                                " MiB of fixed scratch can hold");
        HIP_TRY(hipGetDevice(&dev));
        if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return set_error(AC_E_DEVICE, "device index out of range");
    } catch (const HipError &e) {
        return set_error(e.st, e.msg);
    } catch (...) {
        return set_error(AC_E_DEVICE, "unexpected host exception");
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu[dev]);
    Arena ar;
    struct ArenaOn {
        explicit ArenaOn(Arena *a) { t_arena = a; }
        ~ArenaOn() { t_arena = nullptr; }
    };
    try {
        ar.base = scratch_on(dev);
        ar.cap = NOALLOC_SCRATCH_BYTES;
        const ArenaOn on(&ar);
        Batch bt;
        bt.off = {0, n};
        const Options o = parse(opt);
        Ext ext{d_simp, d_size, capacity, false};
        const ac_status st = run_pipeline(d_xyz, d_radii, n, bt, &alpha, 1, o, s, &c, nullptr, &ext);  // synchronises s
        if (st != AC_OK) return st;
        const bool fits = ext.fits;
        for (int d = 0; d < 4; d++) counts[d] = c->count[d];
        free_complex(c);  // host object only: its arrays lie in the scratch
        c = nullptr;
        if (!fits) return set_error(AC_E_CAPACITY, "an output buffer is smaller than the result (counts holds the sizes)");
        g_last_error.clear();
        return AC_OK;
    } catch (const HipError &e) {
        (void)hipStreamSynchronize(s);
        if (c) {
            const ArenaOn on(&ar);  // its arrays are scratch, not pool blocks
            free_complex(c);
        }
        return set_error(e.st, e.msg);
    } catch (...) {
        (void)hipStreamSynchronize(s);
        return set_error(AC_E_DEVICE, "unexpected host exception");
    }
}

ac_status ac_alpha_complex_partitioned(const double *d_xyz, const double *d_radii, int64_t n, double alpha,
                                       int32_t parts, const ac_options *opt, void *stream, ac_complex **out) {
    if (!out) return set_error(AC_E_INVALID, "out is NULL");
    *out = nullptr;
    try {
        const Options o = parse(opt);
        if (!d_xyz || !d_radii) return set_error(AC_E_INVALID, "NULL input pointer");
        return run_partitioned(d_xyz, d_radii, n, alpha, parts, o, static_cast<hipStream_t>(stream), out);
    } catch (const HipError &e) {
        return set_error(e.st, e.msg);
    } catch (...) {
        return set_error(AC_E_DEVICE, "unexpected host exception");
    }
}

ac_status ac_alpha_complex_partitioned_host(const double *xyz, const double *radii, int64_t n, double alpha,
                                            int32_t parts, const ac_options *opt, ac_complex **out) {
    if (!out) return set_error(AC_E_INVALID, "out is NULL");
    *out = nullptr;
    try {
        const Options o = parse(opt);
        return run_streamed(xyz, radii, n, alpha, parts, o, out);
    } catch (const HipError &e) {
        return set_error(e.st, e.msg);
    } catch (...) {
        return set_error(AC_E_DEVICE, "unexpected host exception");
    }
}

ac_status ac_alpha_sweep_device(const double *d_xyz, const double *d_radii, int64_t n, const double *alphas,
                                int64_t n_alpha, const ac_options *opt, void *stream, ac_complex **out) {
    if (!out) return set_error(AC_E_INVALID, "out is NULL");
    if (n_alpha < 1 || n_alpha > AC_MAX_SWEEP) return set_error(AC_E_INVALID, "number of alpha values out of range");
    for (int64_t k = 0; k < n_alpha; k++) out[k] = nullptr;
    try {
        const Options o = parse(opt);
        if (!d_xyz || !d_radii || !alphas) return set_error(AC_E_INVALID, "NULL input pointer");
        Batch bt;
        bt.off = {0, n};
        return run_pipeline(d_xyz, d_radii, n, bt, alphas, (int)n_alpha, o, static_cast<hipStream_t>(stream), out);
    } catch (const HipError &e) {
        return set_error(e.st, e.msg);
    } catch (...) {
        return set_error(AC_E_DEVICE, "unexpected host exception");
    }
}

ac_status ac_alpha_complex(const double *xyz, const double *radii, int64_t n, double alpha, const ac_options *opt,
                           ac_complex **out) {
    if (!out) return set_error(AC_E_INVALID, "out is NULL");
    *out = nullptr;
    void *dx = nullptr, *dr = nullptr, *stage = nullptr;
    size_t stage_bytes = 0;
    auto release = [&]() {
        // a failed call may leave copies in flight
        if (stage) (void)hipStreamSynchronize(nullptr);
        dev_free(dx);
        dev_free(dr);
        host_free(stage, stage_bytes);
    };
    try {
        const Options o = parse(opt);
        if (!xyz || !radii) return set_error(AC_E_INVALID, "NULL input pointer");
        if (n < 1 || n >= (1 << 26)) return set_error(AC_E_INVALID, "n must be in [1, 2^26)");
        dx = dev_alloc((size_t)n * 3 * sizeof(double));
        dr = dev_alloc((size_t)n * sizeof(double));
        const size_t xb = (size_t)n * 3 * sizeof(double), rb = (size_t)n * sizeof(double);
        // through pinned memory where that is a moderate block; it stays in use
        // until the build below has ended
        if (xb + rb <= HOST_POOL_BYTES / 4) stage = host_alloc(stage_bytes = xb + rb);
        if (stage) {
            std::memcpy(stage, xyz, xb);
            std::memcpy(static_cast<char *>(stage) + xb, radii, rb);
            HIP_TRY(hipMemcpyAsync(dx, stage, xb, hipMemcpyHostToDevice, nullptr));
            HIP_TRY(hipMemcpyAsync(dr, static_cast<char *>(stage) + xb, rb, hipMemcpyHostToDevice, nullptr));
        } else {
            HIP_TRY(hipMemcpy(dx, xyz, xb, hipMemcpyHostToDevice));
            HIP_TRY(hipMemcpy(dr, radii, rb, hipMemcpyHostToDevice));
        }
        Batch bt;
        bt.off = {0, n};
        ac_status st = run_pipeline(static_cast<double *>(dx), static_cast<double *>(dr), n, bt, alpha, o, nullptr, out);
        release();
        dx = dr = stage = nullptr;
        if (st != AC_OK) return st;
        (*out)->device_result = false;
        if (!host_copies(*out, 0, 3)) {
            ac_free(*out);
            *out = nullptr;
            return AC_E_DEVICE;
        }
        return AC_OK;
    } catch (const HipError &e) {
        release();
        return set_error(e.st, e.msg);
    } catch (...) {
        release();
        return set_error(AC_E_DEVICE, "unexpected host exception");
    }
}

ac_status ac_alpha_complex_batch(const double *d_xyz, const double *d_radii, const int64_t *offsets, int64_t n_mol,
                                 double alpha, const ac_options *opt, const int32_t *cell_mA, void *stream,
                                 ac_complex **out) {
    if (!out) return set_error(AC_E_INVALID, "out is NULL");
    *out = nullptr;
    try {
        const Options o = parse(opt);
        if (!d_xyz || !d_radii) return set_error(AC_E_INVALID, "NULL input pointer");
        Batch bt;
        const ac_status st = batch_from(offsets, n_mol, cell_mA, bt);
        if (st != AC_OK) return st;
        const ac_status sp = run_pipeline(d_xyz, d_radii, bt.off[n_mol], bt, alpha, o, static_cast<hipStream_t>(stream), out);
        if (sp == AC_OK) (*out)->batch = true;
        return sp;
    } catch (const HipError &e) {
        return set_error(e.st, e.msg);
    } catch (...) {
        return set_error(AC_E_DEVICE, "unexpected host exception");
    }
}

ac_status ac_plan_create(const double *d_xyz, const double *d_radii, const int64_t *offsets, int64_t n_mol, double alpha,
                         const ac_options *opt, const int32_t *cell_mA, double headroom, void *stream, ac_plan **out) {
    if (!out) return set_error(AC_E_INVALID, "out is NULL");
    *out = nullptr;
    try {
        const Options o = parse(opt);
        if (o.profile != 0) return set_error(AC_E_INVALID, "ac_options.profile must be 0 for a recorded build");
        if (!d_xyz || !d_radii) return set_error(AC_E_INVALID, "NULL input pointer");
        if (!std::isfinite(alpha)) return set_error(AC_E_INVALID, "alpha is not finite");
        if (!(headroom >= 1.0 && headroom <= 16.0)) return set_error(AC_E_INVALID, "headroom must be in [1, 16]");
        Batch bt;
        const ac_status st = batch_from(offsets, n_mol, cell_mA, bt);
        if (st != AC_OK) return st;
        return plan_create(d_xyz, d_radii, bt, alpha, o, headroom, static_cast<hipStream_t>(stream), out);
    } catch (const HipError &e) {
        return set_error(e.st, e.msg);
    } catch (...) {
        return set_error(AC_E_DEVICE, "unexpected host exception");
    }
}

ac_status ac_plan_launch(ac_plan *p, void *stream) {
    if (!p) return set_error(AC_E_INVALID, "plan is NULL");
    try {
        int dev = -1;
        HIP_TRY(hipGetDevice(&dev));
        if (dev != p->device) return set_error(AC_E_INVALID, "the plan was made on another device");
        HIP_TRY(hipGraphLaunch(p->exec, static_cast<hipStream_t>(stream)));
        return AC_OK;
    } catch (const HipError &e) {
        return set_error(e.st, e.msg);
    }
}

ac_status ac_plan_result(ac_plan *p, void *stream, ac_complex **out) {
    if (!out) return set_error(AC_E_INVALID, "out is NULL");
    *out = nullptr;
    if (!p) return set_error(AC_E_INVALID, "plan is NULL");
    try {
        int dev = -1;
        HIP_TRY(hipGetDevice(&dev));
        if (dev != p->device) return set_error(AC_E_INVALID, "the plan was made on another device");
        const ac_status st = plan_result(p, static_cast<hipStream_t>(stream), out);
        if (st == AC_OK) g_last_error.clear();
        return st;
    } catch (const HipError &e) {
        return set_error(e.st, e.msg);
    } catch (...) {
        return set_error(AC_E_DEVICE, "unexpected host exception");
    }
}

int32_t ac_plan_stopped(const ac_plan *p) { return p ? p->last_stop : -1; }

int64_t ac_plan_ordinary_builds(const ac_plan *p) { return p ? p->ordinary_builds : -1; }

void ac_plan_free(ac_plan *p) { free_plan(p); }

int64_t ac_molecule_count(const ac_complex *c) { return c ? c->n_mol : -1; }

const int64_t *ac_molecule_rows(const ac_complex *c, int dim) {
    if (!c || dim < 0 || dim > 3 || c->mol_rows[dim].empty()) return nullptr;
    return c->mol_rows[dim].data();
}

const int32_t *ac_molecule(ac_complex *c, int dim) {
    if (!c || dim < 0 || dim > 3 || !c->batch || c->mol_rows[dim].size() != (size_t)c->n_mol + 1) return nullptr;
    std::vector<int32_t> &h = c->h_mol[dim];
    if (h.empty()) {
        const std::vector<int64_t> &r = c->mol_rows[dim];
        h.assign((size_t)c->count[dim] + 1, 0);  // one spare entry: never a zero-length array
        for (int64_t m = 0; m < c->n_mol; m++)
            std::fill(h.begin() + r[m], h.begin() + r[m + 1], (int32_t)m);
    }
    return h.data();
}

ac_status ac_tune_cells(const double *d_xyz, const double *d_radii, const int64_t *offsets, int64_t n_mol, double alpha,
                        const ac_options *opt, void *stream, int32_t *cell_mA_out, int32_t *bucket_out) {
    try {
        const Options o = parse(opt);
        if (!d_xyz || !d_radii || !cell_mA_out) return set_error(AC_E_INVALID, "NULL pointer");
        Batch all;
        ac_status st = batch_from(offsets, n_mol, nullptr, all);
        if (st != AC_OK) return st;
        hipStream_t s = static_cast<hipStream_t>(stream);
        // grown radius s_g (mA): the default cell side the candidates scale
        double rmax = 0;
        {
            std::vector<double> hr((size_t)all.off[n_mol]);
            HIP_TRY(hipMemcpyAsync(hr.data(), d_radii, hr.size() * sizeof(double), hipMemcpyDeviceToHost, s));
            HIP_TRY(hipStreamSynchronize(s));
            for (double v : hr) rmax = std::max(rmax, v);
        }
        const double sg = std::sqrt(std::max(rmax * rmax + alpha, 1e-6)) * 1000.0;
        static const double kFactor[] = {0.5, 0.7, 1.0, 1.4, 2.0};
        // size buckets: [0, 2k), [2k, 8k), [8k, 32k), [32k, inf)
        auto bucket_of = [](int64_t nm) { return nm < 2000 ? 0 : nm < 8000 ? 1 : nm < 32000 ? 2 : 3; };
        for (int b = 0; b < 4; b++) {
            std::vector<int64_t> mols;
            for (int64_t m = 0; m < n_mol; m++)
                if (bucket_of(all.off[m + 1] - all.off[m]) == b) mols.push_back(m);
            if (mols.empty()) continue;
            // the bucket's molecules, copied into one contiguous sub-batch
            Batch sub;
            sub.off.push_back(0);
            for (int64_t m : mols) sub.off.push_back(sub.off.back() + all.off[m + 1] - all.off[m]);
            const int64_t ns = sub.off.back();
            Scope sc;
            double *x = sc.get<double>(3 * ns), *r = sc.get<double>(ns);
            for (size_t k = 0; k < mols.size(); k++) {
                const int64_t m = mols[k], nm = all.off[m + 1] - all.off[m];
                HIP_TRY(hipMemcpyAsync(x + 3 * sub.off[k], d_xyz + 3 * all.off[m], 3 * nm * sizeof(double),
                                       hipMemcpyDeviceToDevice, s));
                HIP_TRY(hipMemcpyAsync(r + sub.off[k], d_radii + all.off[m], nm * sizeof(double), hipMemcpyDeviceToDevice, s));
            }
            // each side: one warm-up run (fills the pool), then the median of
            // kTuneReps timed runs; another side replaces the default s_g only
            // when it is faster by more than kTuneMargin (run-to-run noise is a
            // few per cent)
            constexpr int kTuneReps = 5;
            constexpr double kTuneMargin = 0.03;
            std::vector<double> med(std::size(kFactor));
            for (size_t fi = 0; fi < std::size(kFactor); fi++) {
                const int32_t side = std::max<int32_t>(1, (int32_t)std::lround(kFactor[fi] * sg));
                sub.cell_mA.assign(mols.size(), side);
                std::vector<double> ts;
                for (int rep = 0; rep <= kTuneReps; rep++) {
                    double tr = 0;
                    st = timed_run(x, r, ns, sub, alpha, o, s, &tr);
                    if (st != AC_OK) return st;
                    if (rep > 0) ts.push_back(tr);
                }
                std::nth_element(ts.begin(), ts.begin() + ts.size() / 2, ts.end());
                med[fi] = ts[ts.size() / 2];
            }
            size_t def = 0;
            while (kFactor[def] != 1.0) def++;
            size_t bi = def;
            for (size_t fi = 0; fi < med.size(); fi++)
                if (med[fi] < med[bi]) bi = fi;
            if (bi != def && med[bi] > (1.0 - kTuneMargin) * med[def]) bi = def;
            const int32_t best = std::max<int32_t>(1, (int32_t)std::lround(kFactor[bi] * sg));
            for (int64_t m : mols) {
                cell_mA_out[m] = best;
                if (bucket_out) bucket_out[m] = b;
            }
            HIP_TRY(hipStreamSynchronize(s));
        }
    } catch (const HipError &e) {
        return set_error(e.st, e.msg);
    } catch (...) {
        return set_error(AC_E_DEVICE, "unexpected host exception");
    }
    g_last_error.clear();
    return AC_OK;
}

int64_t ac_count(const ac_complex *c, int dim) {
    if (!c || dim < 0 || dim > 3) return -1;
    return c->count[dim];
}

const int32_t *ac_simplices(ac_complex *c, int dim) {
    if (!c || dim < 0 || dim > 3) return nullptr;
    if (!c->host_ready[dim] && !host_copies(c, dim, dim)) return nullptr;
    if (c->h_block[dim]) return reinterpret_cast<const int32_t *>(static_cast<const double *>(c->h_block[dim]) + c->count[dim]);
    return c->h_simp[dim].data();
}

const double *ac_sizes(ac_complex *c, int dim) {
    if (!ac_simplices(c, dim)) return nullptr;
    if (c->h_block[dim]) return static_cast<const double *>(c->h_block[dim]);
    return c->h_size[dim].data();
}

const int32_t *ac_simplices_device(const ac_complex *c, int dim) {
    if (!c || dim < 0 || dim > 3 || !c->device_result) return nullptr;
    return c->d_simp[dim];
}

const double *ac_sizes_device(const ac_complex *c, int dim) {
    if (!c || dim < 0 || dim > 3 || !c->device_result) return nullptr;
    return c->d_size[dim];
}

int64_t ac_candidate_count(const ac_complex *c, int dim) {
    if (!c || dim < 0 || dim > 3) return -1;
    return c->cand[dim];
}

int64_t ac_exact_fallbacks(const ac_complex *c) { return c ? c->fallbacks : -1; }

int64_t ac_work_count(const ac_complex *c, int which) {
    if (!c || which < 0 || which > 1) return -1;
    return c->work[which];
}

ac_status ac_union_measure_device(ac_complex *c, const double *d_xyz, const double *d_radii, int64_t n,
                                  double *d_out, void *stream) {
    try {
        check_measure_args(c, d_xyz, d_radii, n);
        if (!d_out) throw HipError{AC_E_INVALID, "out is NULL"};
        measure_forward(c, d_xyz, d_radii, d_out, static_cast<hipStream_t>(stream));
    } catch (const HipError &e) {
        return set_error(e.st, e.msg);
    } catch (...) {
        return set_error(AC_E_DEVICE, "unexpected host exception");
    }
    g_last_error.clear();
    return AC_OK;
}

ac_status ac_union_measure(ac_complex *c, const double *d_xyz, const double *d_radii, int64_t n, double *V,
                           double *A, void *stream) {
    if (!V || !A) return set_error(AC_E_INVALID, "V or A is NULL");
    try {
        check_measure_args(c, d_xyz, d_radii, n);
        hipStream_t s = static_cast<hipStream_t>(stream);
        const double *d_out = measure_forward(c, d_xyz, d_radii, nullptr, s);
        double h[2];
        read_back(h, d_out, 2, s);
        *V = h[0];
        *A = h[1];
    } catch (const HipError &e) {
        return set_error(e.st, e.msg);
    } catch (...) {
        return set_error(AC_E_DEVICE, "unexpected host exception");
    }
    g_last_error.clear();
    return AC_OK;
}

// Backward (and, with d_out, the forward in the same pass) on stream s.
static void measure_backward(ac_complex *c, const double *x, const double *r, int64_t n, const double *g,
                             double *dx, double *dr, double *d_out, hipStream_t s) {
    ensure_incidence(c, s);
    const long long M = incidence_count(c);
    if (!c->meas_contrib) c->meas_contrib = static_cast<double4 *>(dev_alloc((size_t)(M > 0 ? M : 1) * sizeof(double4)));
    const Simplices sx = simplices_of(c);
    const int nb = measure_blocks(sx);
    double *part = d_out ? measure_parts(c, nb) : nullptr;
    if (d_out)
        measure_launch<true, true>(sx, x, r, g, c->meas_contrib, part, s);
    else
        measure_launch<false, true>(sx, x, r, g, c->meas_contrib, nullptr, s);
    constexpr int BALLS = MEASURE_BLOCK / GATHER_LPB;
    k_measure_gather<<<(unsigned)((n + BALLS - 1) / BALLS) + (d_out ? 1 : 0), MEASURE_BLOCK, 0, s>>>(
        c->inc_start, c->inc_slot, c->meas_contrib, (int)n, dx, dr, part, nb, d_out);
    LAUNCH_CHECK();
}

ac_status ac_union_measure_fused(ac_complex *c, const double *d_xyz, const double *d_radii, int64_t n,
                                 const double *d_grad, double *d_out, double *d_dxyz, double *d_dradii, void *stream) {
    try {
        check_measure_args(c, d_xyz, d_radii, n);
        if (!d_grad || !d_out || !d_dxyz || !d_dradii) throw HipError{AC_E_INVALID, "NULL output or gradient pointer"};
        measure_backward(c, d_xyz, d_radii, n, d_grad, d_dxyz, d_dradii, d_out, static_cast<hipStream_t>(stream));
    } catch (const HipError &e) {
        return set_error(e.st, e.msg);
    } catch (...) {
        return set_error(AC_E_DEVICE, "unexpected host exception");
    }
    g_last_error.clear();
    return AC_OK;
}

ac_status ac_union_measure_backward(ac_complex *c, const double *d_xyz, const double *d_radii, int64_t n,
                                    const double *d_grad, double *d_dxyz, double *d_dradii, void *stream) {
    try {
        check_measure_args(c, d_xyz, d_radii, n);
        if (!d_grad || !d_dxyz || !d_dradii) throw HipError{AC_E_INVALID, "NULL gradient pointer"};
        measure_backward(c, d_xyz, d_radii, n, d_grad, d_dxyz, d_dradii, nullptr, static_cast<hipStream_t>(stream));
    } catch (const HipError &e) {
        return set_error(e.st, e.msg);
    } catch (...) {
        return set_error(AC_E_DEVICE, "unexpected host exception");
    }
    g_last_error.clear();
    return AC_OK;
}

void ac_free(ac_complex *c) { free_complex(c); }

int ac_stage_count(void) { return ST_COUNT; }

const char *ac_stage_name(int i) { return (i >= 0 && i < ST_COUNT) ? kStageNames[i] : ""; }

double ac_stage_ms(const ac_complex *c, int i) {
    if (!c || i < 0 || i >= ST_COUNT) return -1.0;
    return c->stage_ms[i];
}

ac_status ac_release_workspace(void) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return set_error(AC_E_DEVICE, "hipGetDevice failed");
    Pool &P = pool();
    std::lock_guard<std::mutex> g(P.mu);
    for (auto &kv : P.free_blocks[dev]) (void)hipFree(kv.second);
    P.free_blocks[dev].clear();
    HostPool &H = host_pool();
    std::lock_guard<std::mutex> gh(H.mu);
    for (auto &kv : H.free_blocks) (void)hipHostFree(kv.second);
    H.free_blocks.clear();
    H.unused = 0;
    return AC_OK;
}

const char *ac_status_str(ac_status s) {
    switch (s) {
        case AC_OK: return "ok";
        case AC_E_INVALID: return "invalid argument";
        case AC_E_DUPLICATE: return "duplicate centres";
        case AC_E_RANGE: return "input outside the exact-arithmetic range";
        case AC_E_NOMEM: return "out of memory";
        case AC_E_DEVICE: return "HIP device error";
        case AC_E_CAPACITY: return "candidate buffer capacity exceeded";
    }
    return "unknown status";
}

const char *ac_last_error(void) { return g_last_error.c_str(); }

}  // extern "C"
