// C-ABI of the library (include/spd.h): argument checks, planning on the host, scratch
// layout, and the sequence of launches of one spd_pairwise / spd_knn call.
#include <hip/hip_runtime.h>

#include <chrono>
#include <cmath>
#include <cstdlib>
#include <cstdio>
#include <cstring>
#include <atomic>
#include <condition_variable>
#include <functional>
#include <mutex>
#include <optional>
#include <string>
#include <thread>
#include <vector>

#include "../../include/spd.h"
#include "../../include/spd_testing.h"
#include "spd_direct.h"
#include "spd_kernels.h"
#include "spd_match.h"
#include "spd_plan.h"

using namespace spd;

// Scratch of the entry point that allocates nothing (spd_pairwise_static): one array per GPU, held
// from the moment the library's code is loaded on that GPU until the process ends.  In host code
// the array's name is only a stand-in for the symbol; the address a kernel can use is asked for
// once per device (spd_create, with that device current) and kept in g_static_scratch.
constexpr size_t kStaticScratchBytes = (size_t)SPD_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kStaticScratchDevices = 64;
static void *g_static_scratch[kStaticScratchDevices];
static std::mutex g_static_scratch_mutex;
// Pinned staging memory every handle holds from its creation, so that a call may not have to
// allocate any: three buffers of this size.
constexpr size_t kInitialPinnedBytes = (size_t)SPD_STATIC_STAGING_BYTES;

// A helper thread that runs one job at a time beside the caller's thread (the plan of A is
// made there while the caller plans B, uploads its plan and starts the repack).  A sleeping
// thread can take longer to wake than the job takes: when the caller comes to wait and the
// helper has not begun yet, the caller runs the job itself.
class Helper {
public:
    ~Helper() {
        if (!th_.joinable()) return;
        { std::lock_guard<std::mutex> g(m_); quit_ = true; }
        cv_.notify_all();
        th_.join();
    }
    void post(std::function<void()> job) {
        if (!th_.joinable()) th_ = std::thread([this] { loop(); });
        { std::lock_guard<std::mutex> g(m_); job_ = std::move(job); state_ = kPosted; posted_.store(true, std::memory_order_release); }
        cv_.notify_all();
    }
    void wait() {
        std::unique_lock<std::mutex> g(m_);
        if (state_ == kPosted) {                 // not begun: do it here
            state_ = kRunning;
            posted_.store(false, std::memory_order_relaxed);
            std::function<void()> job = std::move(job_);
            g.unlock();
            job();
            g.lock();
            state_ = kIdle;
            return;
        }
        cv_.wait(g, [this] { return state_ == kIdle; });
    }
private:
    enum State { kIdle, kPosted, kRunning };
    void loop() {
        std::unique_lock<std::mutex> g(m_);
        for (;;) {
            // calls tend to come back to back: look out for the next job for a little while
            // before going to sleep (waking a sleeping thread takes as long as a small plan)
            if (state_ != kPosted && !quit_) {
                g.unlock();
                const auto until = std::chrono::steady_clock::now() + std::chrono::microseconds(kSpinMicros);
                while (!posted_.load(std::memory_order_acquire) && std::chrono::steady_clock::now() < until) {
#if defined(__x86_64__)
                    __builtin_ia32_pause();
#endif
                }
                g.lock();
            }
            cv_.wait(g, [this] { return state_ == kPosted || quit_; });
            posted_.store(false, std::memory_order_relaxed);
            if (quit_) return;
            state_ = kRunning;
            std::function<void()> job = std::move(job_);
            g.unlock();
            job();
            g.lock();
            state_ = kIdle;
            cv_.notify_all();
        }
    }
    std::thread th_;
    std::mutex m_;
    std::condition_variable cv_;
    std::function<void()> job_;
    State state_ = kIdle;
    bool quit_ = false;
    std::atomic<bool> posted_{false};           // what the helper polls while it spins
    static constexpr int kSpinMicros = 300;
};

struct spd_handle {
    hipStream_t stream = nullptr;
    int device = 0;
    PlanOptions opt;
    std::string err;
    // Pinned staging memory: three buffers taken in turn, so that a call may fill one while the
    // copies of the calls before it are still waiting in the stream.  `pinned` is the one the
    // current call holds.
    struct PinnedSlot { void *ptr = nullptr; size_t bytes = 0; hipEvent_t done = nullptr; bool pending = false; };
    static constexpr int kPinnedSlots = 3;
    PinnedSlot pinned_slots[kPinnedSlots];
    int pinned_next = 0, pinned_held = -1;
    void *pinned = nullptr;
    size_t pinned_bytes = 0;
    void *ws = nullptr;          // device scratch in use
    size_t ws_bytes = 0;
    bool ws_external = false;
    void *own_ws = nullptr;      // the handle's own allocation
    size_t own_ws_bytes = 0;
    int32_t *flag = nullptr;     // device words: the first one for spd_csr_validate, the one at kRowsWord for RowsVerdict
    static constexpr int kRowsWord = 32;
    uint32_t rows_looked_at = 0; // calls that had their row pointers looked at on the device
    void *static_ws = nullptr;   // this device's copy of `scratch`
    bool no_alloc = false;       // inside spd_pairwise_static: nothing may be allocated
    bool profile = false;
    bool check_plan = false;
    bool no_byte_counters = false;   // option "byte_counters" 0: set metrics through the dot product
    int cuckoo_attempts = 3;     // option "cuckoo_attempts"
    int knn_seed = 1;            // option "knn_seed"
    int match_lists = 1;         // option "match_lists": 0 never, 1 where it pays, 2 wherever the product allows it, 3 over A's columns
    size_t lists_refused = SIZE_MAX;     // the least scratch for the column lists that the device had no memory for
    int swap_operands = 1;       // option "swap_operands": 0 never, 1 where it pays, 2 wherever the distance allows it
    int direct = 1;              // option "direct": 0 never, 1 where it pays
    int side_streams = 3;        // option "side_streams": how many internal streams the small launches may use beside the large one
    static constexpr int kSideStreams = 3;
    hipStream_t side[kSideStreams] = {nullptr, nullptr, nullptr};
    hipEvent_t fork_event = nullptr, join_event[kSideStreams] = {nullptr, nullptr, nullptr};     // full consistency check of every plan before launching
    struct Timed { spd_kernel_time rec; hipEvent_t start, stop; };
    std::vector<Timed> timed;    // launches of the last call (profile mode)
    std::vector<hipEvent_t> event_pool;
    APlan plan_of_a;             // kept between calls: the planner reuses their buffers
    BPlan plan_of_b;
    Helper helper;
    std::vector<int64_t> knn_row_off;
    std::vector<int32_t> knn_row_lists;
};

// B of a distance, planned and repacked once (spd_index_create): the plan on the host, and on
// the device the plan's arrays, the packed slabs and the row norms in one allocation.
struct spd_index {
    spd_csr matrix;              // the caller's arrays (they must stay valid and unchanged)
    int64_t chain = 0, knn_chain = 0;    // of its rows (direct_knn_chain), where a call may be one launch
    int metric = 0;
    float p = 1.0f;
    int device = 0;
    BPlan plan;
    void *dev = nullptr;
    size_t dev_bytes = 0;
    BDevice bd;
    MatchB match{};              // the column lists of the same rows, where the product has them (values == nullptr: none)
    void *match_dev = nullptr;
    int match_op = -1;
};

namespace {

const char *const kMetricNames[SPD_METRIC_COUNT] = {
    "inner_product", "cosine", "l2_expanded", "correlation", "jaccard", "dice", "hellinger", "l1",
    "chebyshev", "minkowski", "canberra", "hamming", "kl_divergence", "jensen_shannon", "russell_rao",
    "l2_unexpanded", "kl_divergence_strict", "jaccard_literal"};

spd_status fail(spd_handle *h, spd_status st, const std::string &msg) {
    if (h) h->err = msg;
    return st;
}

spd_status hip_fail(spd_handle *h, hipError_t e, const char *where) {
    return fail(h, SPD_ERR_HIP, std::string(where) + ": " + hipGetErrorString(e));
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// Sequential carving of the scratch buffer.
struct Carver {
    size_t off = 0;
    size_t take(size_t bytes) { size_t at = off; off = align256(off + bytes); return at; }
};

spd_status check_csr_args(spd_handle *h, const spd_csr *M, const char *name) {
    if (!M) return fail(h, SPD_ERR_NULL, std::string(name) + " is NULL");
    if (M->n_rows < 0 || M->n_cols < 0 || M->nnz < 0)
        return fail(h, SPD_ERR_DIM_MISMATCH, std::string(name) + " has a negative size");
    if (!M->indptr) return fail(h, SPD_ERR_NULL, std::string(name) + ".indptr is NULL");
    if (M->nnz > 0 && (!M->indices || !M->values))
        return fail(h, SPD_ERR_NULL, std::string(name) + ".indices / .values is NULL");
    if (M->n_rows >= ((int64_t)1 << 31) - 1 || M->n_cols >= ((int64_t)1 << 31) - 1)
        return fail(h, SPD_ERR_UNSUPPORTED, std::string(name) + ": more than 2^31-2 rows or columns");
    if (M->nnz >= ((int64_t)1 << 40))
        return fail(h, SPD_ERR_UNSUPPORTED, std::string(name) + ": more than 2^40 stored entries");
    return SPD_OK;
}

// The distance of Table 1 (or one of the library's variants of them) that a semiring call spells,
// or -1: such a call runs on the distance's own kernels.  The inner product is left out for k-NN
// (spd_knn returns its largest values, spd_semiring_knn the smallest), and so is Chebyshev, whose
// value between two empty rows is 0 where the semiring's is the identity of max.
int table1_metric(const spd_semiring &s, bool knn) {
    if (s.sum != SPD_SUM_PLUS) return -1;
    const int T = (int)s.transform, E = (int)s.epilogue;
    const bool U = s.over_union != 0;
    switch (s.product) {
    case SPD_PRODUCT_TIMES:          // (0 annihilates: the union adds nothing to the intersection)
        if (T == SPD_TRANSFORM_NONE) {
            if (E == SPD_EPILOGUE_NONE) return knn ? -1 : (int)SPD_INNER_PRODUCT;
            if (E == SPD_EPILOGUE_COSINE) return SPD_COSINE;
            if (E == SPD_EPILOGUE_L2) return SPD_L2_EXPANDED;
            if (E == SPD_EPILOGUE_CORRELATION) return SPD_CORRELATION;
            if (E == SPD_EPILOGUE_JACCARD) return SPD_JACCARD_LITERAL;
        } else if (T == SPD_TRANSFORM_NONZERO) {
            if (E == SPD_EPILOGUE_JACCARD) return SPD_JACCARD;
            if (E == SPD_EPILOGUE_DICE) return SPD_DICE;
            if (E == SPD_EPILOGUE_RUSSELL_RAO) return SPD_RUSSELL_RAO;
        } else if (T == SPD_TRANSFORM_SQRT) {
            if (E == SPD_EPILOGUE_HELLINGER) return SPD_HELLINGER;
        }
        return -1;
    case SPD_PRODUCT_ABS_DIFF: return (U && T == SPD_TRANSFORM_NONE && E == SPD_EPILOGUE_NONE) ? (int)SPD_L1 : -1;
    case SPD_PRODUCT_ABS_DIFF_POW: return (U && T == SPD_TRANSFORM_NONE && E == SPD_EPILOGUE_ROOT_P) ? (int)SPD_MINKOWSKI : -1;
    case SPD_PRODUCT_SQ_DIFF:
        return (U && T == SPD_TRANSFORM_NONE && E == SPD_EPILOGUE_ROOT_P && s.p == 2.0f) ? (int)SPD_L2_UNEXPANDED : -1;
    case SPD_PRODUCT_CANBERRA: return (U && T == SPD_TRANSFORM_NONE && E == SPD_EPILOGUE_NONE) ? (int)SPD_CANBERRA : -1;
    case SPD_PRODUCT_NOT_EQUAL: return (U && T == SPD_TRANSFORM_NONE && E == SPD_EPILOGUE_DIV_K) ? (int)SPD_HAMMING : -1;
    case SPD_PRODUCT_X_LOG_X_OVER_Y:
        if (U || T != SPD_TRANSFORM_NONE) return -1;
        return E == SPD_EPILOGUE_NONE ? (int)SPD_KL_DIVERGENCE : (E == SPD_EPILOGUE_STRICT ? (int)SPD_KL_STRICT : -1);
    case SPD_PRODUCT_JS_TERM: return (U && T == SPD_TRANSFORM_NONE && E == SPD_EPILOGUE_SQRT_HALF) ? (int)SPD_JENSEN_SHANNON : -1;
    default: return -1;
    }
}

spd_status check_call_args(spd_handle *h, const spd_csr *A, const spd_csr *B, spd_metric metric, float p, int knn_k,
                           bool is_knn, const void *o1, const void *o2, const spd_semiring *semiring = nullptr,
                           bool is_semiring = false) {
    if (!h) return SPD_ERR_NULL;
    h->err.clear();
    spd_status st = check_csr_args(h, A, is_knn ? "Q" : "A");
    if (st != SPD_OK) return st;
    st = check_csr_args(h, B, is_knn ? "Index" : "B");
    if (st != SPD_OK) return st;
    if (A->n_cols != B->n_cols) return fail(h, SPD_ERR_DIM_MISMATCH, "the two matrices differ in n_cols");
    if (is_semiring) {
        if (!semiring) return fail(h, SPD_ERR_NULL, "semiring is NULL");
        if ((int)semiring->product < 0 || (int)semiring->product >= SPD_PRODUCT_COUNT)
            return fail(h, SPD_ERR_BAD_METRIC, "unknown product");
        if ((int)semiring->sum < 0 || (int)semiring->sum >= SPD_SUM_COUNT) return fail(h, SPD_ERR_BAD_METRIC, "unknown sum");
        if ((int)semiring->transform < 0 || (int)semiring->transform >= SPD_TRANSFORM_COUNT)
            return fail(h, SPD_ERR_BAD_METRIC, "unknown transform");
        if ((int)semiring->epilogue < 0 || (int)semiring->epilogue >= SPD_EPILOGUE_COUNT)
            return fail(h, SPD_ERR_BAD_METRIC, "unknown epilogue");
        if (semiring->product == SPD_PRODUCT_X_LOG_X_OVER_Y && semiring->over_union)
            return fail(h, SPD_ERR_BAD_METRIC, "x log(x/y) has no value where y is absent: it is offered over the columns both rows store");
        if ((semiring->product == SPD_PRODUCT_ABS_DIFF_POW || semiring->epilogue == SPD_EPILOGUE_ROOT_P) &&
            !(semiring->p > 0.0f && std::isfinite(semiring->p)))
            return fail(h, SPD_ERR_BAD_P, "the semiring needs a finite degree p > 0");
        if (semiring->epilogue > SPD_EPILOGUE_SQRT_HALF && table1_metric(*semiring, false) < 0)
            return fail(h, SPD_ERR_BAD_METRIC, "this epilogue is an expansion over row norms: it is defined for the product, "
                                               "sum and transform of its own distance only");
    } else {
        if ((int)metric < 0 || (int)metric >= SPD_METRIC_COUNT) return fail(h, SPD_ERR_BAD_METRIC, "unknown metric");
        if (metric == SPD_MINKOWSKI && !(p > 0.0f && std::isfinite(p)))
            return fail(h, SPD_ERR_BAD_P, "Minkowski needs a finite p > 0");
    }
    if (is_knn) {
        if (knn_k < 1 || (int64_t)knn_k > B->n_rows || knn_k > SPD_KNN_MAX_K)
            return fail(h, SPD_ERR_BAD_K, "k must lie in [1, min(Index.n_rows, SPD_KNN_MAX_K)]");
        if (A->n_rows > 0 && (!o1 || !o2)) return fail(h, SPD_ERR_NULL, "out_idx / out_dist is NULL");
    } else {
        if (A->n_rows > 0 && B->n_rows > 0 && !o1) return fail(h, SPD_ERR_NULL, "out is NULL");
    }
    return SPD_OK;
}

// Holds one of the handle's pinned buffers for the length of a call: waits until the copies the
// buffer's last call enqueued have run, and on the way out marks the point in the stream after
// which it may be written again.
struct PinnedLease {
    spd_handle *h;
    explicit PinnedLease(spd_handle *hh) : h(hh) {
        const int i = h->pinned_next;
        h->pinned_next = (i + 1) % spd_handle::kPinnedSlots;
        spd_handle::PinnedSlot &s = h->pinned_slots[i];
        if (s.pending) { (void)hipEventSynchronize(s.done); s.pending = false; }
        h->pinned = s.ptr;
        h->pinned_bytes = s.bytes;
        h->pinned_held = i;
    }
    ~PinnedLease() {
        spd_handle::PinnedSlot &s = h->pinned_slots[h->pinned_held];
        s.ptr = h->pinned;
        s.bytes = h->pinned_bytes;
        if (!s.done && hipEventCreateWithFlags(&s.done, hipEventDisableTiming) != hipSuccess) s.done = nullptr;
        if (s.done && hipEventRecord(s.done, h->stream) == hipSuccess) s.pending = true;
        else (void)hipStreamSynchronize(h->stream);       // no event: fall back to waiting here
        h->pinned = nullptr;
        h->pinned_bytes = 0;
        h->pinned_held = -1;
    }
    PinnedLease(const PinnedLease &) = delete;
    PinnedLease &operator=(const PinnedLease &) = delete;
};

spd_status ensure_pinned(spd_handle *h, size_t bytes) {
    if (bytes <= h->pinned_bytes) return SPD_OK;
    if (h->no_alloc)
        return fail(h, SPD_ERR_WORKSPACE, "operands too large for the entry point that allocates nothing: the plan needs " +
                                              std::to_string(bytes) + " bytes of staging memory, a handle holds " +
                                              std::to_string(h->pinned_bytes));
    if (h->pinned) { hipError_t e = hipStreamSynchronize(h->stream); (void)e; (void)hipHostFree(h->pinned); h->pinned = nullptr; h->pinned_bytes = 0; }
    size_t want = align256(bytes + bytes / 4);
    hipError_t e = hipHostMalloc(&h->pinned, want, hipHostMallocDefault);
    if (e != hipSuccess) return hip_fail(h, e, "hipHostMalloc");
    h->pinned_bytes = want;
    return SPD_OK;
}

spd_status ensure_workspace(spd_handle *h, size_t bytes) {
    if (h->ws_external) {
        if (bytes > h->ws_bytes)
            return fail(h, SPD_ERR_WORKSPACE,
                        h->no_alloc ? "operands too large for the entry point that allocates nothing: they need " +
                                          std::to_string(bytes) + " bytes of scratch, the static array holds " +
                                          std::to_string(h->ws_bytes)
                                    : "caller workspace too small: need " + std::to_string(bytes) + " bytes");
        return SPD_OK;
    }
    if (bytes > h->own_ws_bytes) {
        if (h->own_ws) {
            hipError_t e = hipStreamSynchronize(h->stream);
            if (e != hipSuccess) return hip_fail(h, e, "hipStreamSynchronize");
            (void)hipFree(h->own_ws);
            h->own_ws = nullptr; h->own_ws_bytes = 0;
        }
        size_t want = align256(bytes + bytes / 8);
        hipError_t e = hipMalloc(&h->own_ws, want);
        if (e != hipSuccess) return fail(h, SPD_ERR_WORKSPACE, std::string("hipMalloc of scratch failed: ") + hipGetErrorString(e));
        h->own_ws_bytes = want;
    }
    h->ws = h->own_ws;
    h->ws_bytes = h->own_ws_bytes;
    return SPD_OK;
}

// Profile mode: events around one launch.
struct LaunchTimer {
    spd_handle *h;
    bool on;
    spd_handle::Timed t;
    hipStream_t stream;
    LaunchTimer(spd_handle *hh, const char *name, int R, int kind, int block, uint32_t lds, int64_t a_rows, int64_t wgs,
                hipStream_t st = nullptr)
        : h(hh), on(hh->profile), stream(st ? st : hh->stream) {
        if (!on) return;
        std::memset(&t.rec, 0, sizeof t.rec);
        std::snprintf(t.rec.name, sizeof t.rec.name, "%s", name);
        t.rec.rows_per_group = R; t.rec.staging_kind = kind; t.rec.block = block; t.rec.lds_bytes = (int32_t)lds;
        t.rec.a_rows = a_rows; t.rec.workgroups = wgs; t.rec.ms = -1.0;
        auto get = [&](hipEvent_t &e) {
            if (!h->event_pool.empty()) { e = h->event_pool.back(); h->event_pool.pop_back(); return true; }
            return hipEventCreate(&e) == hipSuccess;
        };
        if (!get(t.start) || !get(t.stop)) { on = false; return; }
        (void)hipEventRecord(t.start, stream);
    }
    void done() {
        if (!on) return;
        (void)hipEventRecord(t.stop, stream);
        h->timed.push_back(t);
    }
};

// Everything one call uploads, laid out in one pinned blob mirrored 1:1 in the scratch.
struct Upload {
    std::vector<std::pair<size_t, std::pair<const void *, size_t>>> parts;   // scratch offset, (src, bytes)
    void add(size_t off, const void *src, size_t bytes) { if (bytes) parts.push_back({off, {src, bytes}}); }
};

size_t workspace_bound(const spd_handle *h, const spd_csr *A, const spd_csr *B, int metric, int k_neighbors);

// Where B's plan, its packed slabs and its norms sit in a device buffer: the plan's arrays first,
// contiguous, so that one copy moves them.
struct BLayout {
    size_t slab_base, slab_steps, slab_split, seg_start, seg_len, seg_row, seg_glog, plan_end, packed, norms, end;
};

BLayout layout_b(const BPlan &bp, int64_t n, Carver &cv) {
    const size_t lanes = (size_t)bp.n_slabs * kWave;
    BLayout L;
    L.slab_base = cv.take(bp.slab_base.size() * 8);
    L.slab_steps = cv.take(bp.slab_steps.size() * 4);
    L.slab_split = cv.take(bp.slab_split.size());
    L.seg_start = cv.take(lanes * 8);
    L.seg_len = cv.take(lanes * 4);
    L.seg_row = cv.take(lanes * 4);
    L.seg_glog = cv.take(lanes);
    L.plan_end = cv.off;
    L.packed = cv.take((size_t)bp.slab_base[(size_t)bp.n_slabs] * 8);
    L.norms = cv.take((size_t)n * 16);
    L.end = cv.off;
    return L;
}

// Copies B's plan through the pinned buffer at `pin` into the device buffer `dev` (laid out by
// `L`) and starts the repack there.  Everything is enqueued on the handle's stream.
spd_status stage_b_into(spd_handle *h, const spd_csr *B, const BPlan &bp, const BLayout &L, unsigned char *dev,
                        unsigned char *pin, int metric, const MetricInfo &mi, const OpParams &q, uint32_t padcol,
                        BDevice &bd) {
    const size_t lanes = (size_t)bp.n_slabs * kWave;
    auto put = [&](size_t off, const void *src, size_t bytes) { if (bytes) std::memcpy(pin + off, src, bytes); };
    put(L.slab_base, bp.slab_base.data(), bp.slab_base.size() * 8);
    put(L.slab_steps, bp.slab_steps.data(), bp.slab_steps.size() * 4);
    put(L.slab_split, bp.slab_split.data(), bp.slab_split.size());
    put(L.seg_start, bp.seg_start.data(), lanes * 8);
    put(L.seg_len, bp.seg_len.data(), lanes * 4);
    put(L.seg_row, bp.seg_row.data(), lanes * 4);
    put(L.seg_glog, bp.seg_glog.data(), lanes);
    if (L.plan_end) {
        hipError_t err = hipMemcpyAsync(dev, pin, L.plan_end, hipMemcpyHostToDevice, h->stream);
        if (err != hipSuccess) return hip_fail(h, err, "upload of B's plan");
    }
    bd.packed = reinterpret_cast<const uint2 *>(dev + L.packed);
    bd.slab_base = reinterpret_cast<const int64_t *>(dev + L.slab_base);
    bd.slab_steps = reinterpret_cast<const int32_t *>(dev + L.slab_steps);
    bd.slab_split = dev + L.slab_split;
    bd.seg_start = reinterpret_cast<const int64_t *>(dev + L.seg_start);
    bd.seg_len = reinterpret_cast<const int32_t *>(dev + L.seg_len);
    bd.seg_row = reinterpret_cast<const int32_t *>(dev + L.seg_row);
    bd.seg_glog = dev + L.seg_glog;
    bd.norms = reinterpret_cast<const double *>(dev + L.norms);
    bd.n_slabs = bp.n_slabs;
    bd.n_rows = B->n_rows;
    LaunchTimer lt(h, "pack_b", 0, 0, 0, 0, 0, bp.n_slabs);
    hipError_t err = launch_pack_b(h->stream, B->indptr, B->indices, B->values, bd, reinterpret_cast<uint2 *>(dev + L.packed),
                                   reinterpret_cast<double *>(dev + L.norms), metric, mi.transform, mi.norm, q.p, q.k, padcol);
    if (err != hipSuccess) return hip_fail(h, err, "pack kernel");
    lt.done();
    return SPD_OK;
}

// The parameters of a metric's product as the kernels read them.
OpParams op_params(int metric, float p, int64_t n_cols, const spd_semiring *semiring) {
    OpParams q;
    q.p = p;
    if (metric == SPD_L2_UNEXPANDED) q.p = 2.0f;
    q.inv_p = (metric == SPD_MINKOWSKI) ? 1.0f / p : (metric == SPD_L2_UNEXPANDED ? 0.5f : 1.0f);
    q.k = (double)n_cols;
    q.metric = metric;
    if (metric != SPD_MINKOWSKI && metric != SPD_L2_UNEXPANDED) q.p = 1.0f;
    if (semiring) {
        q.product = (int)semiring->product;
        q.over_union = semiring->over_union != 0;
        q.sign = semiring->sum == SPD_SUM_MIN ? -1.0f : 1.0f;
        q.epilogue = (int)semiring->epilogue;          // (only the first four reach the kernels)
        if (semiring->product == SPD_PRODUCT_ABS_DIFF_POW || semiring->epilogue == SPD_EPILOGUE_ROOT_P) {
            q.p = semiring->p;
            q.inv_p = 1.0f / semiring->p;
        }
    }
    return q;
}

// The metric a call runs as (Minkowski of degree 1 is the Manhattan distance, whose product is
// a third of the work).
int effective_metric(int metric, float p) { return (metric == SPD_MINKOWSKI && p == 1.0f) ? (int)SPD_L1 : metric; }

// `metric` is a spd_metric, or, with `semiring` set, the internal id its sum() runs as.  With
// `index` set, B is that index's matrix and its plan, packed slabs and norms are taken from it.
// Whether a pairwise call stages B and streams A instead of the other way round.  A lane holds
// the results of one streamed row against the R staged rows; with A staged these are R different
// rows of the output and the 64 lanes of a store fall on 64 different cache lines (the streamed
// rows of a slab are the ones of similar length inside a window, not neighbours), which costs
// three times the output in write traffic.  With B staged in groups of consecutive rows a lane's
// R results are neighbours in its own output row: whole 32-byte sectors.  The roles can be
// exchanged for every distance that is symmetric in its two rows, and pay where the scan of a pair
// is short against its store (short rows of B) and A is large enough to be worth sweeping.
bool operands_may_swap(int metric, const spd_semiring *semiring) {
    if (semiring && semiring->product == SPD_PRODUCT_X_LOG_X_OVER_Y) return false;
    return metric != SPD_KL_DIVERGENCE && metric != SPD_KL_STRICT;
}
bool operands_swap_pays(const spd_csr *A, const spd_csr *B) {
    return A->nnz >= ((int64_t)1 << 18) && A->n_rows >= 1024 && B->nnz <= 96 * B->n_rows;
}
// (of a pairwise call without an index)
bool swap_wanted(const spd_handle *h, const spd_csr *A, const spd_csr *B, int metric, const spd_semiring *semiring) {
    return operands_may_swap(metric, semiring) && (h->swap_operands == 2 || (h->swap_operands == 1 && operands_swap_pays(A, B)));
}

// What the planner, or check_rows in its place, found wrong with an operand.
spd_status refuse_plan(spd_handle *h, const char *name, const std::string &why) {
    return fail(h, why.find("pointers") != std::string::npos ? SPD_ERR_BAD_CSR : SPD_ERR_UNSUPPORTED, std::string(name) + ": " + why);
}

// ------------------------------------------------------------------------------------
// Column lists (spd_match.h): the second way of computing a distance
// ------------------------------------------------------------------------------------
// The product a call's kernels run.
int product_of(const spd_handle *h, int metric, float p) {
    int op = metric_info(metric).op;
    // the set metrics count shared columns in byte lanes, or (option) as a dot product of 0/1 values
    if (op == OP_CNT && (h->no_byte_counters || h->opt.force_kind == KIND_BLOOM)) op = OP_DOT;
    // Minkowski: the small integer degrees share one set of kernels, every other degree has its own
    if (op == OP_MINK && degree_class(metric == SPD_L2_UNEXPANDED ? 2.0f : p) == 0) op = OP_MINK_ANY;
    return op;
}

struct MatchLayout { size_t values, rows, ptr, norms, least, ranks, tops, end; };
// (`spare`: bytes behind the entries' rows)
MatchLayout layout_match(const MatchShape &s, int op, int64_t n, int64_t nnz, size_t spare, Carver &cv) {
    MatchLayout L;
    L.values = cv.take((size_t)s.list_entries(nnz) * 4);
    L.rows = cv.take((size_t)s.list_entries(nnz) * 2 + spare);
    L.ptr = cv.take((size_t)s.n_tiles * (size_t)s.ptr_stride * 4);
    L.norms = cv.take((size_t)n * 16);
    L.least = cv.take((size_t)s.n_tiles * 16);
    L.ranks = L.tops = 0;
    if (op == OP_CHEB) {
        L.ranks = cv.take((size_t)nnz);
        L.tops = cv.take((size_t)n * kRanks * 4);
    }
    L.end = cv.off;
    return L;
}
MatchB match_b_at(const MatchShape &s, const MatchLayout &L, unsigned char *dev) {
    return MatchB{reinterpret_cast<float *>(dev + L.values), reinterpret_cast<uint16_t *>(dev + L.rows), reinterpret_cast<uint32_t *>(dev + L.ptr),
                  reinterpret_cast<double *>(dev + L.norms), reinterpret_cast<double *>(dev + L.least),
                  L.tops ? reinterpret_cast<uint8_t *>(dev + L.ranks) : nullptr, reinterpret_cast<float *>(dev + L.tops), s, nullptr};
}
// Grid of the column-list kernel: groups of tiles times slices of A's rows, one workgroup for each
// compute unit of the chip.  Where the lists are more than the L2 caches hold, the tiles are dealt to the
// eight XCDs, and the workgroups of an XCD go through its tiles together; smaller lists are in every L2
// anyway, and each tile is a group.  Rows of A from `shared_len` entries on are shared by the wavefronts of a workgroup.
struct MatchGrid { int slices = 1, groups = 1, by_xcd = 0, run = 1; int64_t share = 0, shared_len = 0; };         // share: of A's entries, a wavefront's
MatchGrid match_grid(const PlanOptions &opt, const MatchShape &s, int op, int64_t m, int64_t nnz_a, int64_t nnz_b, bool knn) {
    MatchGrid g;
    const int64_t cus = std::max(1, opt.n_cus), rows_slices = std::max<int64_t>(1, (m + s.waves - 1) / s.waves);
    if (s.n_tiles >= 16 && nnz_b * 8 > kMatchL2Bytes) {
        const int64_t per_xcd = std::max<int64_t>(1, cus / 8);
        g.by_xcd = 1;
        g.slices = (int)std::min(per_xcd, rows_slices);
        g.groups = (int)std::min<int64_t>(s.n_tiles, per_xcd / g.slices * 8);
    } else {
        // (k-NN: as few groups as fill the chip, since every group's lists start empty)
        g.groups = (int)std::min<int64_t>(s.n_tiles, knn ? (cus + rows_slices - 1) / rows_slices : cus);
        g.slices = (int)std::max<int64_t>(1, std::min(rows_slices, cus / g.groups));
    }
    const int64_t tiles = (s.n_tiles + g.groups - 1) / g.groups;
    // Shared rows: those of a third of a wavefront's share of A's entries.  Where the wavefronts add to one strip, such a row costs one wait:
    // it pays from half that length on, and pairwise, where they form its distances together too, short rows are as well with a
    // wavefront each.  (A third / a sixth / a twelfth of the share, us: sets, Jaccard, k-NN 8,816 / 8,489 / 8,785; from 128 / 256 /
    // 512 entries on: 10,000 x 10,000 rows of 38, L1 297 / 298 / 288.  Fp64 sums take a strip for each wavefront: inner products of 2,000 x
    // 30,000 counts, a third / a sixth, 7,766 / 8,379.)
    g.share = nnz_a * tiles / ((int64_t)g.slices * s.waves);
    const bool one_strip = match_any_order(op);
    g.shared_len = std::max<int64_t>(one_strip && !knn ? 512 : 256, g.share / (one_strip ? 6 : 3));
    // A strip for each wavefront, and the sum of the strips, is paid for where the (tile, row)s are too few for the wavefronts to end together, or by rows of twice the mean
    // length at least.  Too few are less than one or one and a quarter to the wavefront where a row's walk takes less than its strips' sum, and
    // more where it takes longer; with k-NN, whose selection is one wavefront's, fewer.  (All rows of 256 entries or a third of the share shared / where there is
    // one for every wavefront not / so, the walk in us: cosine, 64 x 60,000 counts 898 / 920 / 835, k-NN 1,150 / 942 / 946, 1,500 x 6,000 words 208 / 173 / 173; KL, 32 x
    // 60,000 counts 593 / 678 / 571, 130 x 60,000 1,519 / 1,603 / 1,442; Minkowski, 130 x 20,000 1,146 / 1,470 / 1,141.)
    if (!one_strip) {
        const double per_wave = (double)((m / g.slices) * tiles) / s.waves, list = (double)nnz_b / ((double)s.n_tiles * (double)s.ptr_stride);
        const bool light = (double)nnz_a / (double)m * std::max(1.0, list / 16.0) / 2.0 < (double)s.tile_rows;
        const double enough = light ? (knn ? 1.0 : 1.25) : (knn ? 1.5 : 2.75 * match_cell_bytes(op) / 8.0);
        if (per_wave >= enough) g.shared_len = std::max<int64_t>(g.shared_len, 2 * nnz_a / m);
    }
    // Chebyshev: a row of A that is like many of B's costs its wavefront two microseconds a pair (spd_match_impl.h).  Where a wavefront to the row
    // leaves half of the compute units idle, rows of some length are all shared: 500 x 500 rows of 50 ones over one support 880 -> 152 us
    // (staged scan 271), 1,000 x 1,000 of 100 1,258 -> 639 (1,314), of 100 normal values 205 -> 136; 237 x 5,101 rows of 223 194 -> 145.
    if (op == OP_CHEB && !g.by_xcd && 2 * (int64_t)g.slices * g.groups <= cus && nnz_a >= 16 * m) {
        g.slices = (int)std::max<int64_t>(1, std::min<int64_t>(m, cus / g.groups));
        g.shared_len = 0;
    }
    // A wavefront goes through a run of tiles with a row: as many as leave every wavefront four rows' runs, and whose lists
    // (and bounds) together lie in half of an L2.  What a row costs besides its lists is then paid once a run, and with
    // k-NN its nearest are merged into the row's list once a run.
    const double tile_bytes = 8.0 * (double)nnz_b / s.n_tiles + 4.0 * (double)s.ptr_stride;
    const int64_t rows_here = std::max<int64_t>(1, m / g.slices);
    g.run = (int)std::max<int64_t>(1, std::min<int64_t>({tiles, (int64_t)((double)(kMatchL2Bytes / 2) / tile_bytes), rows_here * tiles / (4 * s.waves)}));
    return g;
}
// (tile, row)s that the wavefronts of a workgroup share out among themselves, numbered in 32 bits.
int64_t match_items(const MatchShape &s, const MatchGrid &g, int64_t m) {
    return ((m + g.slices - 1) / g.slices) * ((s.n_tiles + g.groups - 1) / g.groups);
}
// Counters and locks that go up with A's rows, all 0 (MatchArgs::next).
size_t match_counters_bytes(const MatchGrid &g, bool knn) { return (size_t)g.groups * (knn ? 1 + kMatchRowLocks : 1) * 4; }
struct ColumnsLayout { size_t words, sums, totals, masks, before, a_indices, b_indptr, b_indices, b_values; };
struct MatchScratch { MatchLayout b; ColumnsLayout c; size_t rows, norms_a, scales_a, ranks_a, tops_a, tau, part, row_off, row_lists, end; };
// `columns`: 0, or the operands' column count where both are copied over A's columns first (spd_match_columns.hip).
MatchScratch layout_match_call(const MatchShape &s, const MatchGrid &g, int op, int64_t m, int64_t nnz_a, int64_t n, int64_t nnz_b, int knn_k,
                               bool with_b, int64_t columns) {
    MatchScratch L{};
    Carver cv;
    // (eight bytes to a stored entry in scratch, what its gaps leave of them spare, so that scratch of a given size, the static array among it, sends
    // the same calls to the staged scan as when an entry took eight)
    if (with_b) L.b = layout_match(s, op, n, nnz_b, (size_t)std::max<int64_t>(0, 2 * nnz_b - 6 * (s.room_of(nnz_b) - nnz_b)), cv);
    if (columns > 0) {
        const size_t words = ((size_t)columns + 31) / 32, masks = ((size_t)nnz_b + 63) / 64;
        L.c.words = cv.take(words * 8);
        L.c.sums = cv.take(std::max(words, masks) / 64 * 4 + 256);
        L.c.totals = cv.take(8);
        L.c.masks = cv.take(masks * 8);
        L.c.before = cv.take(masks * 4);
        L.c.a_indices = cv.take((size_t)nnz_a * 4);
        L.c.b_indptr = cv.take((size_t)(n + 1) * 8);
        L.c.b_indices = cv.take((size_t)nnz_b * 4);
        L.c.b_values = cv.take((size_t)nnz_b * 4);
    }
    L.rows = cv.take((size_t)m * sizeof(MatchRow) + match_counters_bytes(g, knn_k > 0));       // (the counters behind them)
    L.norms_a = cv.take((size_t)m * 16);
    if (match_fixed(op)) L.scales_a = cv.take((size_t)m * 2);
    if (op == OP_CHEB) {
        L.ranks_a = cv.take((size_t)nnz_a);
        L.tops_a = cv.take((size_t)m * kRanks * 4);
    }
    if (knn_k > 0) {
        L.tau = cv.take((size_t)m * 8);
        L.row_off = cv.take((size_t)m * 8);
        L.row_lists = cv.take((size_t)m * 4);
        L.part = cv.take((size_t)m * (size_t)g.groups * (size_t)knn_k * sizeof(KnnEntry));
    }
    L.end = cv.off;
    return L;
}
// Option "check_plan" for the column lists: what the kernels' indexes and LDS rest on.  Empty if consistent.
std::string match_check(const PlanOptions &opt, const MatchShape &s, const MatchGrid &g, int op, int64_t m, int64_t n, int64_t n_cols,
                        int64_t nnz_b) {
    const int64_t T = s.tile_rows, tiles = s.n_tiles, blocks = s.blocks, cell = match_cell_bytes(op);
    if (op == OP_CHEB && T > kRankedRows) return "ranked rows";
    if (T < kWave || T % kWave != 0 || tiles * T < n || (tiles - 1) * T >= n) return "tiles do not cover B";
    if (s.waves != match_waves((int)cell) || s.lds_bytes != (uint32_t)s.waves * match_strip_bytes((int)cell, (int)T) ||
        (int64_t)s.lds_bytes + match_static_lds((int)cell) > opt.lds_budget) return "strips over the LDS";
    if (s.block_shift < 2 || s.block_shift > 13 || s.stage < 64 || T > 2496 || (blocks << s.block_shift) < n_cols || ((blocks - 1) << s.block_shift) >= n_cols)
        return "column blocks";
    if (s.ptr_stride < n_cols + blocks) return "list bounds";
    if (s.dense_per < 1 || s.dense_per > (int32_t)kBuildDensePer || s.dense_shift < s.block_shift || s.dense_shift > 13 || s.dense_from < 1 ||
        s.dense_from > T + 1 || s.tile_extra != (int64_t)s.dense_before((int32_t)blocks) * s.dense_room()) return "dense columns";
    if (s.list_entries(nnz_b) >= (int64_t)1 << 29) return "list positions";
    if (s.aligned && 1.3125 * std::min((double)nnz_b, (double)T * (double)n_cols) + (double)s.tile_extra >= (double)s.position_bits())
        return "list positions and gaps";
    const int64_t build = (int64_t)s.stage * 6 + ((int64_t)4 << s.block_shift) + 4 * T;
    if ((int64_t)s.build_lds_bytes != build || s.stage % 8 != 0 || (build + 1024) * kBuildPerCu > opt.lds_budget) return "build over the LDS";
    if (g.slices < 1 || g.groups < 1 || g.run < 1 || g.run > tiles || g.groups > tiles || (g.by_xcd && g.groups < tiles && g.groups % 8 != 0)) return "grid";
    if (match_items(s, g, m) >= (int64_t)1 << 30) return "(tile, row)s of a workgroup";
    return std::string();
}
// ... and A's rows as the kernel takes them: every row once, where the row pointers say, the first ones shared.
std::string match_check_rows(const MatchRow *rows, int64_t m, int64_t shared, int64_t shared_len, const int64_t *a_ip) {
    std::vector<bool> seen((size_t)m, false);
    int64_t longer = 0;
    for (int64_t i = 0; i < m; ++i) {
        const MatchRow &r = rows[i];
        if (r.row < 0 || r.row >= m || seen[(size_t)r.row]) return "A's rows are not a permutation";
        seen[(size_t)r.row] = true;
        if (r.start != a_ip[r.row] || r.start + r.len != a_ip[r.row + 1]) return "A row range";
        longer += r.len > shared_len ? 1 : 0;
    }
    return shared == longer ? std::string() : "shared rows";
}
// The knobs that pick the staged scan's paths: a caller that turns one wants that kernel.
bool scan_knobs_untouched(const spd_handle *h) {
    const PlanOptions d;
    const PlanOptions &o = h->opt;
    return o.force_kind == d.force_kind && o.max_rows == d.max_rows && o.split_len == d.split_len && o.window == d.window &&
           o.chunks == d.chunks && o.chunk_scale == d.chunk_scale && o.waves_per_cu == d.waves_per_cu &&
           o.bloom_long_rows == d.bloom_long_rows && o.sort_slack == d.sort_slack && o.partial_groups == d.partial_groups &&
           o.lds_budget >= 64 * 1024 && !h->no_byte_counters && h->cuckoo_attempts == 3 && h->knn_seed == 1 &&
           h->swap_operands == 1;
}
// The list bounds, a word per tile and column, are kept to the size of the lists, or to 64 MiB.  Over A's columns to twice that: they are laid out for as
// many columns as A has entries, of which it stores a third, and what is laid out beyond these is never touched.  (4,096 x 500,000 sets, Jaccard, k-NN, with
// 687,000 entries of A's: the bounds are 2.1 words to an entry of B, and the call took 32.7 ms by the scan that lists serve in 6.9.)
bool match_bounds_fit(const MatchShape &s, int64_t nnz, int words = 2) {
    return (int64_t)s.n_tiles * s.ptr_stride <= std::max<int64_t>(words * nnz, 16 << 20);
}
bool match_light(int op) { return op == OP_DOT || op == OP_L1 || op == OP_HAMM; }
// Where an eighth of B's cells are stored (half, for a dear product), most visits meet something.
bool match_dense(const spd_csr *B, int op) { return (double)B->nnz > (match_light(op) ? 0.125 : 0.5) * (double)B->n_cols * (double)B->n_rows; }
// Whether B's rows have lists for a product at all, under the option's setting.
bool match_possible(const spd_handle *h, const spd_csr *B, int op, MatchShape &s) {
    if (h->match_lists == 0 || !match_serves(op)) return false;
    if (B->n_rows <= 0 || B->n_cols <= 0 || B->n_cols >= ((int64_t)1 << 31) - 8) return false;
    s = match_shape(h->opt.lds_budget, op, B->n_rows, B->n_cols, B->nnz);
    // (list positions are 32-bit byte offsets)
    return s.n_tiles > 0 && s.list_entries(B->nnz) < ((int64_t)1 << 29);
}
// Whether some call could do better by them, as far as B tells.
bool match_suits(const spd_handle *h, const spd_csr *B, int op, const MatchShape &s) {
    return scan_knobs_untouched(h) && !match_dense(B, op) && match_bounds_fit(s, B->nnz);
}
// Whether an index keeps the lists, and their layout in its memory: only lists that a call may want, and no more of
// them than the header states (a small B over many columns has more bounds than entries).
bool index_keeps_lists(const spd_handle *h, const spd_csr *B, int op, MatchShape &s, MatchLayout &L) {
    if (!match_possible(h, B, op, s) || !match_serves_knn(op)) return false;
    const int64_t most = 20 * B->nnz + 16 * B->n_rows + (1 << 20);
    auto lay_out = [&] {
        Carver cv;
        L = layout_match(s, op, B->n_rows, B->nnz, 0, cv);
    };
    lay_out();
    if ((int64_t)L.end > most && s.aligned) {      // (what fits without gaps is kept without them)
        s.aligned = 0;
        lay_out();
    }
    if (h->match_lists == 2) return true;
    if (op == OP_CNT) return false;                // (counts come out the same by the scan, which is as fast where a call has no B to prepare)
    return match_suits(h, B, op, s) && (int64_t)L.end <= most;
}
// What a call costs by lists and by the staged scan, in picoseconds of the whole chip.  A wavefront pays for every entry of
// its row of A in every tile (its list's bounds), for every entry of a list it walks and for
// every (tile, row); the last round of (tile, row)s leaves wavefronts idle, unless rows are so long that a workgroup's wavefronts share
// them.  The staged scan pays for every visit (a staged row, a streamed entry), and for a streamed entry's look-up, which the rows that are staged
// together share: how many these are and behind which kind of map, the planner says.  Both pay for what they make of B, where no index
// has it, for the pairs they finish, for their launches, and the longer rows are, for the last and longest of them; the scan also for the launches that
// staged rows of many lengths take, but for a dense strip, which has one.  Lists over A's columns are walked as those over all columns are;
// what the copy leaves of B is the share of its columns that A stores, were they uniform, and the more the less they are: its fourth root.  Columns are
// seldom uniform where they are many: lists are taken to be met up to 40 times as often as if they were, as far as the density leaves room for that
// (words, Zipf columns, rows of 230 over 102,660: some 40 times).
// The constants are fitted to the times of 11,400 calls by all three ways (of the working range: words, counts, ratings, sets, n-grams, skewed lengths; and of 8 to
// 11,000 rows against 64 to 2,000,000, of equal, log-normal and power-law lengths of 1.5 to 3,000 entries, A's as long as B's and not, uniform and Zipf columns, 64 to
// 2^22 of them; every product, k-NN with k = 1 to 64 and pairwise, with an index and without); nine of ten estimates are within 0.54 to 1.66 of the
// times, because row pointers do not show how A's columns meet B's, nor the longest row.  What 2,232 further calls took beyond the best way, on the mean: of the working range
// 1.8 %, of the others 4.5 %, correlation, pairwise, 8 %.  (The scan by steps of the column count and lists by a weight for each product, k-NN and way, in place of maps, rows' lengths
// and launches: 4.6, 6.4 and, correlation weighed by 1.65, 16 %; constants from lists that took up to a third longer 12, 11 and 13 %.)
struct OpCost { double entry, match, row, knn_row, visit, pair, knn_pair; };
constexpr OpCost op_cost(int op) {
    switch (op) {
    case OP_DOT: return {9.23, 0.536, 0, 116, 0.0859, 2.23, 1.60};
    case OP_L1: return {8.61, 0.421, 0, 0, 0.109, 1.29, 1.81};
    case OP_HAMM: return {13.3, 0.451, 825, 1180, 0.157, 2.29, 2.23};
    case OP_CNT: return {11.0, 0.450, 482, 691, 0.0710, 2.96, 1.67};
    case OP_CANB: return {7.84, 0.599, 137, 35, 0.298, 2.35, 2.13};
    case OP_KL: return {10.2, 0.894, 22, 580, 0.335, 2.24, 1.85};
    case OP_JS: return {4.88, 1.06, 174, 1070, 0.729, 4.35, 4.32};
    case OP_CHEB: return {8.10, 0.587, 687, 0, 0.433, 1.87, 75.9};
    case OP_MINK_ANY: return {10.6, 2.19, 767, 912, 0.870, 3.50, 5.02};
    default: return {10.3, 1.69, 411, 540, 0.489, 3.16, 2.79};
    }
}
// The columns that lists over A's columns alone are laid out for (how many A stores, the host does not know).
int64_t columns_of(const spd_csr *A) { return std::min(A->n_cols, std::max<int64_t>(A->nnz, 1)); }
// (`of_a`: over A's columns alone, after a copy; an index brings the lists over all columns)
double lists_cost(const spd_handle *h, const spd_csr *A, const spd_csr *B, int op, int metric, const MatchShape &s, bool knn, bool with_index, bool of_a) {
    const double m = (double)A->n_rows, n = (double)B->n_rows, nnz_a = (double)A->nnz, nnz_b = (double)B->nnz, tiles = (double)s.n_tiles, cols = (double)A->n_cols;
    const OpCost c = op_cost(op);
    const MatchGrid g = match_grid(h->opt, s, op, A->n_rows, A->nnz, B->nnz, knn);
    const double rows = std::ceil(m / g.slices), runs = std::ceil(tiles / g.groups);          // of a workgroup
    double idle = rows * runs * (double)h->opt.n_cus / (m * tiles);
    if (nnz_a <= (double)g.shared_len * m) idle *= std::ceil(rows * runs / s.waves) * s.waves / (rows * runs);
    const double density = nnz_b / n / cols, skew = density > 0.0 ? std::max(1.0, 0.0693 / density) : 1.0;
    // (sets' tiles are twice as long, and more of what they are met by are dense columns, which cost every row of the tile: 184 x 9,756 words, Jaccard, k-NN, by the scan 184 us, by
    // lists 313; 65 x 33,887 267 and 390)
    const double met = op == OP_CNT ? std::min(80.0, std::pow(skew, 1.2)) : std::min(40.0, skew);
    const double kept = of_a ? std::sqrt(std::sqrt(1.0 - std::exp(-nnz_a / cols))) : 1.0;
    const double make = with_index && !of_a ? 0.0 : (knn ? 7.64e6 : 15e6) + 15.7 * kept * nnz_b + 6.81 * tiles * (of_a ? (double)columns_of(A) : cols) + 329.0 * n;
    // (two norms a pair: 573 x 3,605 rows of 319, all of a length / log-normal, correlation, by the scan 138 / 207 us, by lists 160 / 131)
    const bool two_norms = metric == MT_CORRELATION || op == OP_MINK || op == OP_MINK_ANY;
    // (counts without an index: where both estimates are alike the scan's times spread further, so that what lists gain is more than what they lose.  Hamming, 6,533 x
    // 70,554 rows of 240 and 36, k-NN, 3,581 us by the scan and 1,408 by lists, which are estimated the higher)
    const double weight = with_index ? 1.0 : (op == OP_HAMM ? 0.88 : (op == OP_CNT ? 0.94 : 1.0));
    return weight * ((knn ? 52.4e6 : 13.5e6) + make + (of_a ? 39.1e6 + 7.21 * nnz_b : 0.0) + 5050.0 * m + (two_norms ? 1.65 : 0.985) * m * n +
                     2.18e6 * std::sqrt(nnz_a / m) + 0.802e6 * std::sqrt(nnz_b / n) +
                     idle * (nnz_a * tiles * c.entry + c.match * met * nnz_a * density * n + (c.row + (knn ? c.knn_row : 0.0)) * m * tiles));
}
double staged_cost(const spd_handle *h, const spd_csr *A, const spd_csr *B, int op, int metric, bool swapped, bool knn, bool made) {
    const double m = (double)A->n_rows, n = (double)B->n_rows, nnz_a = (double)A->nnz, nnz_b = (double)B->nnz;
    const OpCost c = op_cost(op);
    const double staged = swapped ? nnz_b / n : nnz_a / m, streamed = swapped ? nnz_a / m : nnz_b / n;           // entries of a row
    const Staging of = staging_of(A->n_cols, metric, op, knn, staged, h->opt);
    const double look_up = of.kind == KIND_STRIP ? 0.0 : (of.kind == KIND_SLOT ? 0.189 : (of.kind == KIND_BITMAP ? 0.385 : 0.859));
    const double launches = of.kind == KIND_STRIP ? 0.0 : (of.kind == KIND_SLOT ? 2.02e6 : (of.kind == KIND_BITMAP ? 2.62e6 : 3.31e6));
    // (what making B ready takes grows with its rows' lengths, some 2.3 times an entry's at 1,820: without that 204 calls of up to 200 such rows against many took 10 % more than
    // by the best way, with it 1.4 %; k-NN, Hellinger, 88 x 26,958 1,973 us, by lists 1,069, pairwise, Canberra, 31 x 19,632 1,086 / 762)
    const double make = made ? 0.0 : (knn ? 0.0 : 7.96e6) + (7.87 + 0.0055 * std::min(2000.0, nnz_b / n)) * nnz_b + 2830.0 * n;
    // (Chebyshev ranks the entries of the rows that it stages: 34 x 969 rows of 1,550 2,777 us, by lists 554; 304 x 604 rows of 23 186 / 94;
    // 2,026 x 7,507 ratings 11,152 / 703; 3,148 x 4,764 rows of 1,790 25,963 / 3,002)
    return (knn ? 61.6e6 : 30.2e6) + make + 5900.0 * m + 5.97 * nnz_a + (op == OP_CHEB ? 865000.0 * staged : 0.0) + launches * std::sqrt(staged) + 2.01e6 * std::sqrt(streamed) +
           (c.visit + look_up / std::max(1, of.rows)) * (swapped ? n * nnz_a : m * nnz_b) + (knn ? c.knn_pair : c.pair) * m * n;
}
// Whether a call is computed by lists over all columns, were an index to keep them (`staged`: the staged scan's estimate).
bool match_wanted(const spd_handle *h, const spd_csr *A, const spd_csr *B, int op, int metric, const spd_semiring *semiring, double staged, bool knn,
                  bool with_index, double *cost = nullptr) {
    MatchShape s;
    if (semiring || A->n_rows <= 0 || !match_possible(h, B, op, s)) return false;
    if ((knn || with_index) && !match_serves_knn(op)) return false;
    if (match_items(s, match_grid(h->opt, s, op, A->n_rows, A->nnz, B->nnz, knn), A->n_rows) >= (int64_t)1 << 30) return false;
    if (!match_launches_fit(s, op, A->n_rows, A->nnz, B->n_rows, false)) return false;
    if (h->match_lists == 2) return true;
    if (!match_suits(h, B, op, s)) return false;
    // Both sides measured, staged / lists in ms: 10,000 x 10,000 rows of 38, L1 0.65 / 0.26; 1,024 x 300,000 of 230, cosine
    // 11.4 / 5.2; 4,096 x 65,536 of 1,820, L1 87 / 23.6, Jensen-Shannon 349 / 35; 238 x 6,574 of 95, Canberra, with an index 0.21 / 0.026; 1,000 x
    // 10,000 of 1,360 and 20, L1 0.14 / 0.70; set metrics: 3,247 x 7,668 counts, Jaccard 4.6 / 2.1, 72 x 15,967 rows of 218, k-NN 0.22 / 0.41.
    const double lists = lists_cost(h, A, B, op, metric, s, knn, with_index, false);
    if (cost) *cost = lists;
    return lists <= staged;
}
// Whether a call is computed by lists over the columns that A stores, after a copy of both operands over these.
bool columns_wanted(const spd_handle *h, const spd_csr *A, const spd_csr *B, int op, int metric, const spd_semiring *semiring, double staged, bool knn, bool with_index, double *cost) {
    if (semiring || h->match_lists == 0 || !match_serves_knn(op) || A->n_rows <= 0 || A->nnz <= 0 || B->n_rows <= 0 || B->nnz <= 0) return false;
    if (A->n_cols > kMatchMostColumns) return false;
    const MatchShape s = match_shape(h->opt.lds_budget, op, B->n_rows, columns_of(A), B->nnz);
    if (s.n_tiles <= 0 || s.list_entries(B->nnz) >= ((int64_t)1 << 29)) return false;
    if (match_items(s, match_grid(h->opt, s, op, A->n_rows, A->nnz, B->nnz, knn), A->n_rows) >= (int64_t)1 << 30) return false;
    if (!match_launches_fit(s, op, A->n_rows, A->nnz, B->n_rows, true)) return false;
    if (h->match_lists == 3) return true;
    if (h->match_lists != 1 || !scan_knobs_untouched(h) || match_dense(B, op) || !match_bounds_fit(s, B->nnz, 4)) return false;
    // Both sides measured, staged / lists over A's columns in ms, k-NN: 4,096 x 500,000 sets over 2^20 columns, Jaccard 30.6 /
    // 6.4, 371 x 33,325 of them, Dice 0.81 / 0.33 (over all columns 0.48), 59 x 15,538 0.51 / 0.24 (0.31); 4,096 x 663,000 rows of 2.2 over 858,000, cosine 5.3 /
    // 2.0.  Few columns may have no room for their bounds beside many short rows either: 200 x 1,000,000 rows of 5 over 32,768, cosine, pairwise 3.4 / 0.75; 3,000 x
    // 900,000 of 3, Canberra 9.0 / 1.5; 4,096 x 2,000,000 of 2 over 16,384, cosine 18.1 / 4.8.
    *cost = lists_cost(h, A, B, op, metric, s, knn, with_index, true);
    return *cost <= staged;
}
// The way a call is computed: 0 the staged scan, 1 lists over all columns, 2 lists over the columns that A stores; and how.
// `room`: bytes of scratch that there may be.
struct MatchWay { int way = 0; int64_t columns = 0; MatchShape s{}; MatchGrid g; MatchScratch L{}; };
MatchWay match_way(const spd_handle *h, const spd_csr *A, const spd_csr *B, int op, int metric, const spd_semiring *semiring, bool swapped, int knn_k,
                   bool with_index, bool index_has_lists, size_t room) {
    MatchWay w;
    const bool knn = knn_k > 0;
    // (`swapped`: the staged scan would exchange the operands' roles)
    const double staged = h->match_lists == 1 && !semiring && A->n_rows > 0 && B->n_rows > 0 ? staged_cost(h, A, B, op, metric, swapped, knn, with_index) : 0.0;
    double over_all = 0.0, over_a = 0.0;
    const bool all = h->match_lists != 3 && (!with_index || index_has_lists) && match_wanted(h, A, B, op, metric, semiring, staged, knn, with_index, &over_all);
    const bool of_a = h->match_lists != 2 && columns_wanted(h, A, B, op, metric, semiring, staged, knn, with_index, &over_a);
    auto lay_out = [&](int way) {
        w.way = way;
        w.columns = way == 2 ? columns_of(A) : A->n_cols;
        w.s = match_shape(h->opt.lds_budget, op, B->n_rows, w.columns, B->nnz);
        w.g = match_grid(h->opt, w.s, op, A->n_rows, A->nnz, B->nnz, knn);
        w.L = layout_match_call(w.s, w.g, op, A->n_rows, A->nnz, B->n_rows, B->nnz, knn_k, way == 2 || !with_index, way == 2 ? A->n_cols : 0);
    };
    if (!all && !of_a) return w;
    if (all && of_a && over_a < over_all) {          // (the copy may cost less than the bounds and the entries of columns that A does not store)
        lay_out(2);
        if (w.L.end <= room) return w;                // (it may also take more scratch)
    }
    lay_out(all ? 1 : 2);
    return w;
}
// The scratch that a call's lists may take: what the caller lends, or less than the device refused.
size_t scratch_room(const spd_handle *h) { return h->ws_external ? h->ws_bytes : h->lists_refused - 1; }


// The norms of B's rows, and their lists.
spd_status stage_norms(spd_handle *h, const spd_csr *B, const MatchB &mb, int metric, const MetricInfo &mi, const OpParams &q, const RowsVerdict &seen) {
    LaunchTimer norms(h, "norms_b", 0, 0, 0, 0, 0, 0);
    hipError_t e = launch_match_norms(h->stream, B->indptr, B->values, B->n_rows, B->nnz, metric, mi.transform, mi.norm, q.p, q.k,
                                      seen, mb.norms, nullptr);
    if (e != hipSuccess) return hip_fail(h, e, "norm kernel");
    norms.done();
    return SPD_OK;
}
// (`knn`: and each tile's row of the least norm)
spd_status stage_lists(spd_handle *h, const spd_csr *B, MatchB mb, int op, const MetricInfo &mi, bool knn, const RowsVerdict &seen) {
    if (!knn) mb.least = nullptr;
    LaunchTimer lists(h, "lists_b", 0, 0, 0, 0, 0, mb.shape.n_tiles);
    hipError_t e = launch_match_build(h->stream, B->indptr, B->indices, B->values, B->n_rows, B->nnz, (uint32_t)B->n_cols, mb,
                           op, mi.transform, seen);
    if (e != hipSuccess) return hip_fail(h, e, "column-list kernels");
    lists.done();
    return SPD_OK;
}

// What of a call by lists needs no row pointers on the host: B's norms and lists, A's norms.
struct MatchStart { MatchB b; spd_csr listed; const int32_t *a_indices; };
spd_status start_match(spd_handle *h, const spd_csr *A, const spd_csr *B, int metric, int op, int knn_k, const OpParams &q,
                       const MetricInfo &mi, const MatchWay &way, const spd_index *index, const RowsVerdict &seen, MatchStart &start) {
    const int64_t m = A->n_rows, n = B->n_rows;
    const MatchShape &s = way.s;
    const MatchScratch &L = way.L;
    const bool compact = way.way == 2, index_lists = index && !compact;
    spd_status st = SPD_OK;
    if (h->check_plan) {
        std::string why = match_check(h->opt, s, way.g, op, m, n, way.columns, B->nnz);
        if (why.empty() && L.end > h->ws_bytes) why = "scratch";
        if (!why.empty()) return fail(h, SPD_ERR_UNSUPPORTED, "internal plan check failed: " + why);
    }
    unsigned char *ws = reinterpret_cast<unsigned char *>(h->ws);         // (run() has seen to its size)
    hipError_t e;
    start.b = index_lists ? index->match : match_b_at(s, L.b, ws);
    start.a_indices = A->indices;
    start.listed = *B;
    if (!index_lists) {
        if (op == OP_CHEB) {
            LaunchTimer lt(h, "norms_b", 0, 0, 0, 0, 0, 0);
            e = launch_match_ranks(h->stream, RankedRows{B->indptr, B->values, n, B->nnz, 0, start.b.ranks, start.b.tops},
                                   RankedRows{A->indptr, A->values, m, A->nnz, 1, reinterpret_cast<uint8_t *>(ws + L.ranks_a),
                                              reinterpret_cast<float *>(ws + L.tops_a)}, seen);
            if (e != hipSuccess) return hip_fail(h, e, "rank kernel");
            lt.done();
        } else {
            st = stage_norms(h, B, start.b, metric, mi, q, seen);
        }
        if (st != SPD_OK) return st;
        if (compact) {
            const MatchColumns c{reinterpret_cast<uint2 *>(ws + L.c.words), reinterpret_cast<uint32_t *>(ws + L.c.sums),
                                 reinterpret_cast<uint32_t *>(ws + L.c.totals), reinterpret_cast<uint64_t *>(ws + L.c.masks),
                                 reinterpret_cast<uint32_t *>(ws + L.c.before), reinterpret_cast<int32_t *>(ws + L.c.a_indices),
                                 reinterpret_cast<int64_t *>(ws + L.c.b_indptr), reinterpret_cast<int32_t *>(ws + L.c.b_indices),
                                 reinterpret_cast<float *>(ws + L.c.b_values)};
            LaunchTimer lt(h, "columns", 0, 0, 0, 0, 0, 0);
            e = launch_match_columns(h->stream, A->indices, A->nnz, B->indptr, B->indices, B->values, n, B->nnz, (uint32_t)A->n_cols, c);
            if (e != hipSuccess) return hip_fail(h, e, "column kernels");
            lt.done();
            start.a_indices = c.a_indices;
            start.listed.indptr = c.b_indptr;
            start.listed.indices = c.b_indices;
            start.listed.values = c.b_values;
            start.listed.n_cols = way.columns;
            start.b.cols = c.totals;
        }
        st = stage_lists(h, &start.listed, start.b, op, mi, knn_k > 0, seen);
        if (st != SPD_OK) return st;
    }
    if (op == OP_CHEB) return SPD_OK;
    LaunchTimer lt(h, "norms_a", 0, 0, 0, 0, 0, 0);
    e = launch_match_norms(h->stream, A->indptr, A->values, m, A->nnz, metric, mi.transform, mi.norm, q.p, q.k, seen,
                           reinterpret_cast<double *>(ws + L.norms_a), match_fixed(op) ? reinterpret_cast<int16_t *>(ws + L.scales_a) : nullptr);
    if (e != hipSuccess) return hip_fail(h, e, "norm kernel");
    lt.done();
    return SPD_OK;
}

// ... and the rest of it.
spd_status run_match(spd_handle *h, const spd_csr *A, const spd_csr *B, int metric, int op, int knn_k, const OpParams &q,
                     const MetricInfo &mi, const MatchWay &way, const MatchStart &start, const int64_t *a_ip, size_t ip_bytes, float *out,
                     int64_t *out_idx, float *out_dist) {
    const int64_t m = A->n_rows, n = B->n_rows;
    const MatchShape &s = way.s;
    const MatchGrid &g = way.g;
    const MatchScratch &L = way.L;
    unsigned char *ws = reinterpret_cast<unsigned char *>(h->ws);
    hipError_t e;
    spd_status st = SPD_OK;
    // A's rows, longest first (to within an eighth of their length): a counting sort into the pinned buffer
    int64_t shared = 0;
    const size_t rows_bytes = (size_t)m * sizeof(MatchRow) + match_counters_bytes(g, knn_k > 0);
    st = ensure_pinned(h, align256(ip_bytes) + rows_bytes);
    if (st != SPD_OK) return st;
    MatchRow *rows = reinterpret_cast<MatchRow *>(reinterpret_cast<unsigned char *>(h->pinned) + align256(ip_bytes));
    {
        auto bucket = [](int64_t len) -> uint32_t {
            uint32_t v = (uint32_t)len, b;
            if (v < 16) b = v;
            else { const int lg = 31 - __builtin_clz(v); b = (uint32_t)(lg - 3) * 8u + ((v >> (lg - 3)) & 7u) + 8u; }
            return 255u - std::min(b, 255u);
        };
        uint32_t at[257] = {0u};
        for (int64_t i = 0; i < m; ++i) ++at[bucket(a_ip[i + 1] - a_ip[i]) + 1];
        for (int b = 1; b <= 256; ++b) at[b] += at[b - 1];
        for (int64_t i = 0; i < m; ++i) {
            const int64_t len = a_ip[i + 1] - a_ip[i];
            shared += len > g.shared_len ? 1 : 0;
            rows[at[bucket(len)]++] = MatchRow{a_ip[i], (int32_t)len, (int32_t)i};
        }
    }
    if (h->check_plan) {
        const std::string why = match_check_rows(rows, m, shared, g.shared_len, a_ip);
        if (!why.empty()) return fail(h, SPD_ERR_UNSUPPORTED, "internal plan check failed: " + why);
    }
    std::memset(rows + m, 0, match_counters_bytes(g, knn_k > 0));
    e = hipMemcpyAsync(ws + L.rows, rows, rows_bytes, hipMemcpyHostToDevice, h->stream);
    if (e != hipSuccess) return hip_fail(h, e, "upload of A's rows");
    MatchArgs a;
    a.a_indices = start.a_indices;
    a.a_values = A->values;
    a.rows = reinterpret_cast<const MatchRow *>(ws + L.rows);
    a.m = (int32_t)m;
    a.norms_a = reinterpret_cast<const double *>(ws + L.norms_a);
    a.scales_a = reinterpret_cast<const int16_t *>(ws + L.scales_a);
    a.ranks_a = reinterpret_cast<const uint8_t *>(ws + L.ranks_a);
    a.tops_a = reinterpret_cast<const float *>(ws + L.tops_a);
    a.b_indices = start.listed.indices;
    a.b_values = start.listed.values;
    a.b_indptr = start.listed.indptr;
    a.b_nnz = B->nnz;
    a.b = start.b;
    a.norms_b = start.b.norms + (metric == MT_COSINE ? n : 0);
    a.n = n;
    a.k = (uint32_t)way.columns;
    a.transform = mi.transform;
    a.q = q;
    a.m_shared = (int32_t)shared;
    a.next = reinterpret_cast<uint32_t *>(ws + L.rows + (size_t)m * sizeof(MatchRow));
    a.slices = g.slices;
    a.groups = g.groups;
    a.by_xcd = g.by_xcd;
    a.run = g.run;
    a.out = out;
    a.knn_k = knn_k;
    a.knn_part = reinterpret_cast<KnnEntry *>(ws + L.part);
    a.knn_tau = reinterpret_cast<unsigned long long *>(ws + L.tau);
    if (knn_k > 0) {
        LaunchTimer lt(h, "knn_begin", 0, 0, 0, 0, m, 0);
        e = launch_match_knn_begin(h->stream, a.knn_tau, reinterpret_cast<int64_t *>(ws + L.row_off),
                                   reinterpret_cast<int32_t *>(ws + L.row_lists), a.knn_part, m, g.groups, knn_k);
        if (e != hipSuccess) return hip_fail(h, e, "k-NN start kernel");
        lt.done();
    }
    {
        LaunchTimer lt(h, "scan", 1, kMatchStagingKind, s.waves * kWave, s.lds_bytes, m, (int64_t)g.groups * g.slices);
        e = launch_match(h->stream, op, a, s.lds_bytes);
        if (e != hipSuccess) return hip_fail(h, e, "column-list scan kernel");
        lt.done();
    }
    if (knn_k > 0) {
        LaunchTimer lt(h, "knn_merge", 0, 0, 0, 0, m, (m + 3) / 4);
        e = launch_knn_merge(h->stream, a.knn_part, reinterpret_cast<const int64_t *>(ws + L.row_off),
                             reinterpret_cast<const int32_t *>(ws + L.row_lists), m, knn_k, metric == SPD_INNER_PRODUCT ? 1 : 0,
                             out_idx, out_dist);
        if (e != hipSuccess) return hip_fail(h, e, "k-NN merge kernel");
        lt.done();
    }
    return SPD_OK;
}

// Whether a call can be the one launch of spd_direct.hip: few columns, so that its strips fit, and few pairs and entries.
bool direct_possible(const spd_handle *h, const spd_csr *A, const spd_csr *B, int op, const spd_semiring *semiring, int knn_k) {
    if (semiring || h->direct == 0 || !direct_serves(op) || A->n_cols <= 0 || A->n_cols > kDirectColumns) return false;
    if (knn_k > 0 && B->n_rows > kDirectKnnRows) return false;
    // (scratch that the caller lends is asked for as before: a call it does not hold is refused)
    if ((h->ws_external && !h->no_alloc) || !scan_knobs_untouched(h) || h->match_lists != 1) return false;
    return B->n_rows <= kDirectMostRows && A->n_rows * B->n_rows <= ((int64_t)1 << 19) && A->nnz <= (1 << 16) && B->nnz <= (1 << 16);
}
// Entries that a lane to each row of B goes through one after the other, the chain of a call: the longest row, or with k-NN, where all
// rows pass through a workgroup, 256 at a time, the longest of a wavefront's 64 rows each time.
int64_t direct_knn_chain(const int64_t *ip, int64_t n) {
    constexpr int kWaves = kDirectRowsB / kWave;
    int64_t of[kWaves] = {0};
    for (int64_t j0 = 0; j0 < n; j0 += kWave) {
        int64_t longest = 0;
        for (int64_t j = j0; j < std::min(n, j0 + kWave); ++j) longest = std::max(longest, ip[j + 1] - ip[j]);
        of[j0 / kWave % kWaves] += longest;
    }
    return *std::max_element(of, of + kWaves);
}
// Lanes to a row of B; 0: the call's launch would take longer than the other ways do.  In microseconds: a launch, and in
// every round of workgroups that the chip holds the chain of a lane's entries, whose loads are waited for four at a time, and with
// k-NN the selection; against the launches, the uploads and the host's planning of the other ways.  The constants are fitted
// to both ways' times of 10,000 pairs of operands (1 to 2^19 rows of 0 to 2,048 entries, one long row among short ones, Zipf
// and equal lengths, 1 to 2,048 columns, every product, with an index and without).  Of 13,900 others two in 1,000 lose more
// than a twentieth by the line between them, up to 1.5 times; while a lane took every row, whatever its length, a third did, up
// to 53 times.  Both sides, other ways / one launch in us:
//   7 x 194 rows of 1 and 337 over 512 columns, L1                                  52 / 91 with one lane, 30 with four
//   16 x 1,024 rows of 17 and 53 (Zipf, the longest 1,000), Minkowski, k = 10       73 / 3,546 with one lane
//   256 x 256 rows of 10, L1                                                        27 / 8.5 with one
// Four lanes to the row from 16 entries on: at chains of 8 to 16 either takes the same (0.95 to 0.97), at 16 to 24 four
// take 0.75 times as long, at 64 to 96 0.4 to 0.5 times.
int direct_lanes(const spd_handle *h, const spd_csr *A, const spd_csr *B, int op, int knn_k, int64_t chain, bool with_index) {
    const double m = (double)A->n_rows, n = (double)B->n_rows, cus = (double)std::max(1, h->opt.n_cus);
    const bool knn = knn_k > 0;
    const int lanes = chain >= 16 ? kDirectLanes : 1;
    double entry = 0.82;
    switch (op) {
    case OP_DOT: case OP_L1: entry = 0.24; break;
    case OP_HAMM: case OP_CNT: case OP_KL: entry = 0.31; break;
    case OP_CANB: entry = 0.36; break;
    case OP_JS: entry = 0.49; break;
    case OP_MINK_ANY: entry = 0.6; break;
    default: break;
    }
    const double groups = std::ceil(m / kDirectRows) * (knn ? 1.0 : std::ceil(n / kDirectRowsB));
    const int held = std::max(1, std::min(2048 / (kDirectRowsB * lanes), (160 * 1024) / (int)(direct_lds_bytes(A->n_cols, B->n_rows, knn_k) + 64)));
    const double rounds = std::ceil(groups / (cus * held));
    const double one = 7.0 + rounds * ((double)chain * entry / lanes + (knn ? (lanes > 1 ? 0.018 : 0.012) * n : 0.0)) + 1e-6 * m * (double)B->nnz + 2e-3 * groups;
    const double others = (knn ? 39.0 : 28.0) - (with_index ? 11.0 : 0.0) + 2.5e-3 * m + (with_index ? 0.12e-3 : 0.42e-3) * (double)B->nnz +
                          0.15e-3 * (double)A->nnz + (knn ? 50e-6 : 6e-6) * m * n;
    return one <= 0.85 * others ? lanes : 0;
}
// (A and B have been looked through: check_rows)
spd_status run_direct(spd_handle *h, const spd_csr *A, const spd_csr *B, int metric, int op, int knn_k, const OpParams &q,
                      const MetricInfo &mi, int lanes, float *out, int64_t *out_idx, float *out_dist) {
    DirectArgs a;
    a.a = DirectCsr{A->indptr, A->indices, A->values, A->n_rows, A->nnz};
    a.b = DirectCsr{B->indptr, B->indices, B->values, B->n_rows, B->nnz};
    a.q = q;
    a.transform = mi.transform;
    a.norm = mi.norm;
    a.k = (uint32_t)A->n_cols;
    a.out = out;
    a.knn_k = knn_k;
    a.out_idx = out_idx;
    a.out_dist = out_dist;
    LaunchTimer lt(h, "scan", kDirectRows, kDirectStagingKind, kDirectRowsB * lanes, direct_lds_bytes(A->n_cols, B->n_rows, knn_k), A->n_rows,
                   (A->n_rows + kDirectRows - 1) / kDirectRows * (knn_k > 0 ? 1 : (B->n_rows + kDirectRowsB - 1) / kDirectRowsB));
    const hipError_t e = launch_direct(h->stream, op, a, lanes);
    if (e != hipSuccess) return hip_fail(h, e, "direct kernel");
    lt.done();
    return SPD_OK;
}

// (the staged scan's planner refuses a row that is longer than the column count in the operand it stages)
spd_status refuse_rows(spd_handle *h, const char *name, const int64_t *ip, int64_t rows, int64_t n_cols, bool staged, int64_t *longest = nullptr) {
    const std::string why = check_rows(ip, rows, staged ? n_cols : INT64_MAX, longest);
    return why.empty() ? SPD_OK : refuse_plan(h, name, why);
}

spd_status run(spd_handle *h, const spd_csr *A, const spd_csr *B, int metric, float p, const spd_semiring *semiring,
               int knn_k, float *out, int64_t *out_idx, float *out_dist, const spd_index *index = nullptr) {
    for (auto &t : h->timed) { h->event_pool.push_back(t.start); h->event_pool.push_back(t.stop); }
    h->timed.clear();
    if (A->n_rows == 0 || B->n_rows == 0) return SPD_OK;
    hipError_t e = hipSetDevice(h->device);
    if (e != hipSuccess) return hip_fail(h, e, "hipSetDevice");
    metric = effective_metric(metric, p);
    const int op = product_of(h, metric, p);
    const bool swap = knn_k == 0 && !index && swap_wanted(h, A, B, metric, semiring);
    MatchWay way;
    auto choose_way = [&] { way = match_way(h, A, B, op, metric, semiring, swap, knn_k, index != nullptr, index && index->match.values, scratch_room(h)); };

    // ---- row pointers on the host: the caller's copies, or read back (the call's only
    //      synchronisation) ----------------------------------------------------------------
    const spd_csr *const A0 = A, *const B0 = B;
    const bool same = !index && A->indptr == B->indptr && A->n_rows == B->n_rows;
    const int64_t *a_host = A->host_indptr ? A->host_indptr : (same ? B->host_indptr : nullptr);
    const int64_t *b_host = index ? nullptr : (B->host_indptr ? B->host_indptr : (same ? A->host_indptr : nullptr));
    const bool copy_a = !a_host;
    const bool copy_b = !index && !same && !b_host;
    const size_t ip_bytes = (copy_a ? (size_t)(A->n_rows + 1) * 8 : 0) + (copy_b ? (size_t)(B->n_rows + 1) * 8 : 0);
    bool swapped = false;
    std::optional<PinnedLease> lease;
    const int64_t *a_ip = nullptr, *b_ip = nullptr;
    // where the two arrays are read from: the caller's memory, or the start of the pinned buffer
    auto locate = [&]() {
        int64_t *pin = reinterpret_cast<int64_t *>(h->pinned);
        a_ip = a_host ? a_host : pin;
        b_ip = b_host ? b_host : (same ? a_ip : pin + (copy_a ? A0->n_rows + 1 : 0));
        if (swapped) std::swap(a_ip, b_ip);
    };
    // (into a buffer that holds `more` bytes behind them; `meanwhile` enqueues what does not need them before they are waited for)
    auto read_rows = [&](size_t more, auto &&meanwhile) -> spd_status {
        lease.emplace(h);
        const spd_status st = ensure_pinned(h, ip_bytes + more);
        if (st != SPD_OK) return st;
        int64_t *pin = reinterpret_cast<int64_t *>(h->pinned);
        if (copy_a) {
            e = hipMemcpyAsync(pin, A0->indptr, (size_t)(A0->n_rows + 1) * 8, hipMemcpyDeviceToHost, h->stream);
            if (e != hipSuccess) return hip_fail(h, e, "copy of A.indptr");
        }
        if (copy_b) {
            e = hipMemcpyAsync(pin + (copy_a ? A0->n_rows + 1 : 0), B0->indptr, (size_t)(B0->n_rows + 1) * 8, hipMemcpyDeviceToHost, h->stream);
            if (e != hipSuccess) return hip_fail(h, e, "copy of B.indptr");
        }
        if (copy_a || copy_b) {
            const hipEvent_t copied = h->pinned_slots[h->pinned_held].done;
            const bool marked = copied && hipEventRecord(copied, h->stream) == hipSuccess;
            const spd_status begun = marked ? meanwhile() : SPD_OK;
            e = marked ? hipEventSynchronize(copied) : hipStreamSynchronize(h->stream);
            if (e != hipSuccess) return hip_fail(h, e, "hipStreamSynchronize");
            return begun;
        }
        return SPD_OK;
    };
    auto nothing = [] { return SPD_OK; };
    spd_status st = SPD_OK;
    auto check_ends = [&]() -> spd_status {
        if (a_ip[A->n_rows] != A->nnz || (!index && b_ip[B->n_rows] != B->nnz)) return fail(h, SPD_ERR_BAD_CSR, "indptr[n_rows] != nnz");
        return SPD_OK;
    };
    // (a small call's way depends on the lengths of B's rows, where even equal ones would do; row pointers that are not at hand
    // are read back for it)
    int direct = 0;
    bool b_checked = false;
    if (direct_possible(h, A, B, op, semiring, knn_k)) {
        int64_t chain = (B->nnz + B->n_rows - 1) / B->n_rows;
        if (index) chain = knn_k > 0 ? index->knn_chain : index->chain;
        direct = direct_lanes(h, A, B, op, knn_k, chain, index != nullptr);
        if (direct && !index) {
            if (ip_bytes) st = read_rows(80 * ((size_t)std::max(A->n_rows, B->n_rows) + 4096), nothing);         // (whichever operand is staged)
            if (st != SPD_OK) return st;
            locate();
            st = check_ends();
            if (st == SPD_OK) st = refuse_rows(h, "B", b_ip, B->n_rows, A->n_cols, false, &chain);
            if (st != SPD_OK) return st;
            b_checked = true;
            if (knn_k > 0) chain = direct_knn_chain(b_ip, B->n_rows);
            direct = direct_lanes(h, A, B, op, knn_k, chain, false);
        }
    }
    if (!direct) choose_way();
    bool lists = way.way != 0;
    while (lists) {
        if (way.way == 1 && index) {
            MatchShape kept = index->match.shape;
            kept.aligned = way.s.aligned;               // (an index may hold its lists without gaps)
            if (index->match_op != op || std::memcmp(&kept, &way.s, sizeof way.s) != 0) lists = false;              // (created under other options)
        }
        // (a caller's scratch that does not hold the lists still serves the staged scan)
        if (h->ws_external && way.L.end > h->ws_bytes) lists = false;
        // (and so does a device that has no memory left for them; so much is not asked for again)
        if (!lists || h->ws_external) break;
        const spd_status room = way.L.end < h->lists_refused ? ensure_workspace(h, way.L.end) : SPD_ERR_WORKSPACE;
        if (room == SPD_OK) break;
        if (room != SPD_ERR_WORKSPACE) return room;
        h->lists_refused = std::min(h->lists_refused, way.L.end);
        h->err.clear();
        (void)hipGetLastError();
        // (the lists over all columns, where the copy was preferred to them, may still have room)
        const bool copied = way.way == 2;
        if (copied) choose_way();
        lists = copied && way.way == 1;
    }
    swapped = swap && !lists && !direct;
    if (swapped) std::swap(A, B);           // from here on A is the staged operand, B the streamed one
    const int64_t m = A->n_rows, n = B->n_rows;
    const int64_t out_stride_staged = swapped ? 1 : n, out_stride_streamed = swapped ? m : 1;
    static const bool host_times = std::getenv("SPD_HOST_TIMES") != nullptr;
    auto now = [] { return std::chrono::steady_clock::now(); };
    auto t_begin = now();
    auto lap = [&](const char *what) {
        if (!host_times) return;
        auto t = now();
        std::fprintf(stderr, "[spd host] %-12s %8.1f us\n", what, std::chrono::duration<double, std::micro>(t - t_begin).count());
        t_begin = t;
    };

    // Where the row pointers have to be read back, the kernels that read them on the device run meanwhile (and do nothing where a
    // first look at them there finds what the host will refuse), and a call that is then refused waits for them: 1,531 x 28,301
    // ratings, Canberra, 521 -> 496 us a call.
    const OpParams params = op_params(metric, p, A->n_cols, nullptr);
    MatchStart start;
    bool begun = false;
    auto begin_lists = [&](const RowsVerdict &seen) -> spd_status {
        begun = true;
        return start_match(h, A, B, metric, op, knn_k, params, metric_info(metric), way, index, seen, start);
    };
    auto begin_unseen = [&]() -> spd_status {
        if (!lists) return SPD_OK;
        uint32_t *const word = reinterpret_cast<uint32_t *>(h->flag) + spd_handle::kRowsWord;
        if (h->rows_looked_at++ == 0u) {                       // (0 is no call's number; such a call waits for a copy: it is not captured)
            e = hipMemsetAsync(word, 0, sizeof *word, h->stream);
            if (e != hipSuccess) return hip_fail(h, e, "hipMemsetAsync");
            h->rows_looked_at = 1u;
        }
        e = launch_match_look_at_rows(h->stream, A->indptr, m, A->nnz, index || same ? nullptr : B->indptr, n, B->nnz, word, h->rows_looked_at);
        if (e != hipSuccess) return hip_fail(h, e, "kernel of the row pointers");
        return begin_lists(RowsVerdict{word, h->rows_looked_at});
    };
    auto refused = [&](spd_status why) {                         // (a call that is refused leaves nothing running)
        if (begun) (void)hipStreamSynchronize(h->stream);
        return why;
    };
    // (a direct call stages nothing else; the entry point that allocates nothing refuses what its staging memory does not hold, whichever
    // way a call runs)
    if (!lease && (!direct || ip_bytes || h->no_alloc)) {
        // (sized for the two plan uploads as well, which follow the row pointers in the buffer)
        st = read_rows((index ? 0 : 32 * ((size_t)n + 4096)) + 48 * ((size_t)m + 4096), begin_unseen);
        if (st != SPD_OK) return refused(st);
    }
    locate();
    st = check_ends();
    lap("indptr d2h");
    if (st == SPD_OK && (lists || direct)) {
        const bool b_staged = knn_k == 0 && !index && swap;
        st = index || (b_checked && !b_staged) ? SPD_OK : refuse_rows(h, "B", b_ip, n, A->n_cols, b_staged);
        if (st == SPD_OK) st = refuse_rows(h, "A", a_ip, m, A->n_cols, !b_staged);
    }
    if (st != SPD_OK) return refused(st);
    if (direct) return run_direct(h, A, B, metric, op, knn_k, params, metric_info(metric), direct, out, out_idx, out_dist);
    if (lists) {
        if (!begun) st = begin_lists(RowsVerdict{nullptr, 0u});
        if (st != SPD_OK) return st;
        return run_match(h, A, B, metric, op, knn_k, params, metric_info(metric), way, start, a_ip, ip_bytes, out, out_idx, out_dist);
    }

    // ---- B first: plan it, upload its plan and start the repack, so that the device is
    //      busy while the host plans A (an index brings all of that with it) ---------------
    MetricInfo mi = metric_info(metric);
    if (semiring && mi.norm == NORM_SEMI) mi.norm = NORM_SEMI + (int)semiring->product;
    if (semiring) mi.transform = (int)semiring->transform;
    APlan &ap = h->plan_of_a;
    const BPlan &bp = index ? index->plan : h->plan_of_b;
    // A is planned on the helper thread meanwhile; every way out of this function waits for it
    std::string why_a;
    {
        const int64_t *a_rows_ptr = a_ip;
        PlanOptions opt_a = h->opt;
        opt_a.consecutive_groups = swapped ? 1 : 0;
        h->helper.post([&why_a, &ap, opt_a, a_rows_ptr, m, A, metric, op, knn_k] {
            try {
                why_a = plan_a(a_rows_ptr, m, A->n_cols, metric, op, knn_k, opt_a, ap);
            } catch (const std::exception &ex) {
                why_a = std::string("planning failed: ") + ex.what();
            }
        });
    }
    struct WaitForHelper { Helper &w; ~WaitForHelper() { w.wait(); } } wait_for_helper{h->helper};
    std::string why;
    if (!index) {
        PlanOptions opt_b = h->opt;
        opt_b.window = window_for(h->opt, knn_k > 0 || swapped ? WINDOW_NO_SCATTERED_STORES : WINDOW_SCATTERED_STORES);
        why = plan_b(b_ip, n, opt_b, h->plan_of_b);
        if (!why.empty()) return refuse_plan(h, "B", why);
        lap("plan b");
    }
    int a_kind = 0, a_max_r = 1, a_min_r = 1;
    uint64_t a_dmax = 0;
    why = plan_staging(A->n_cols, metric, op, knn_k > 0, h->opt, a_kind, a_max_r, a_min_r, a_dmax);
    if (!why.empty()) return fail(h, SPD_ERR_UNSUPPORTED, "A: " + why);
    // The column an idle lane looks up: no row stores it, so every kind of map sends it to the
    // table's zero row.
    const uint32_t padcol = (uint32_t)A->n_cols;
    const OpParams q = op_params(metric, p, A->n_cols, semiring);

    const int planes = metric_planes(metric);
    Carver cv;
    // (1) B's plan, then what the repack produces (none of it with an index)
    BLayout bl{};
    if (!index) bl = layout_b(bp, n, cv);
    const size_t b_end = cv.off;
    if (!index) {
        // room for A's part as well, from the documented bound, so that the scratch does not
        // have to move once the repack has been started (checked again below)
        size_t guess = 0;
        if (!h->ws_external) guess = workspace_bound(h, A, B, metric, knn_k);
        st = ensure_workspace(h, std::max(b_end, guess));
        if (st != SPD_OK) return st;
    }
    // pinned staging: [row pointers | B's plan | A's plan]
    const size_t pin_b = align256(ip_bytes);
    const size_t pin_a = pin_b + align256(bl.plan_end);
    if (h->pinned_bytes < pin_a + (size_t)m * (sizeof(ARow) + 16) + (64 << 10)) {
        // growing the pinned buffer moves it: let the helper finish reading, keep the row pointers
        h->helper.wait();
        std::vector<unsigned char> keep(ip_bytes);
        std::memcpy(keep.data(), h->pinned, ip_bytes);
        st = ensure_pinned(h, pin_a + (size_t)m * (sizeof(ARow) + 16) + (64 << 10));
        if (st != SPD_OK) return st;
        std::memcpy(h->pinned, keep.data(), ip_bytes);
        locate();
    }
    BDevice bd;
    auto stage_b = [&]() -> spd_status {
        return stage_b_into(h, B, bp, bl, reinterpret_cast<unsigned char *>(h->ws),
                            reinterpret_cast<unsigned char *>(h->pinned) + pin_b, metric, mi, q, padcol, bd);
    };
    if (index) {
        bd = index->bd;
    } else {
        st = stage_b();
        if (st != SPD_OK) return st;
        lap("stage b");
    }

    // ---- A, while the repack runs -------------------------------------------------------
    h->helper.wait();
    why = why_a;
    if (!why.empty()) return refuse_plan(h, "A", why);
    lap("wait for plan a");
    {
        PlanOptions opt_c = h->opt;
        opt_c.chunk_scale = chunk_scale_for(h->opt, knn_k > 0);
        for (AClass &c : ap.classes) plan_chunks(bp, c, opt_c);
    }
    lap("chunks");
    if (h->check_plan) {
        std::vector<int64_t> index_rows;
        const int64_t *b_rows_ptr = b_ip;
        if (index) {
            // the index keeps no host copy of the row pointers: rebuild them from its segments
            index_rows.assign((size_t)n + 1, 0);
            for (size_t l = 0; l < index->plan.seg_row.size(); ++l)
                if (index->plan.seg_row[l] >= 0) index_rows[(size_t)index->plan.seg_row[l] + 1] += index->plan.seg_len[l];
            for (int64_t j = 0; j < n; ++j) index_rows[(size_t)j + 1] += index_rows[(size_t)j];
            b_rows_ptr = index_rows.data();
        }
        why = plan_check(ap, bp, a_ip, b_rows_ptr, A->n_cols, metric, op, knn_k, h->opt);
        if (!why.empty()) return fail(h, SPD_ERR_UNSUPPORTED, "internal plan check failed: " + why);
    }
    for (const AClass &c : ap.classes)
        if ((int64_t)c.n_groups * c.n_chunks >= ((int64_t)1 << 31) || (int64_t)c.lds_bytes + kStaticLds > h->opt.lds_budget ||
            (c.kind != a_kind && c.kind != KIND_BLOOM))
            return fail(h, SPD_ERR_UNSUPPORTED, "internal: launch outside the device limits");
    lap("plan check");

    // (2) A's plan, contiguous again, then what the scans produce
    Upload up;
    const size_t a_plan_begin = cv.off;
    std::vector<size_t> o_rows(ap.classes.size()), o_sumlen(ap.classes.size()), o_chunks(ap.classes.size());
    for (size_t ci = 0; ci < ap.classes.size(); ++ci) {
        const AClass &c = ap.classes[ci];
        o_rows[ci] = cv.take(c.rows.size() * sizeof(ARow));
        o_sumlen[ci] = cv.take(c.sumlen.size() * 4);
        o_chunks[ci] = cv.take(c.chunk_begin.size() * 4);
        up.add(o_rows[ci], c.rows.data(), c.rows.size() * sizeof(ARow));
        up.add(o_sumlen[ci], c.sumlen.data(), c.sumlen.size() * 4);
        up.add(o_chunks[ci], c.chunk_begin.data(), c.chunk_begin.size() * 4);
    }
    const size_t o_spilled = cv.take(ap.spilled.size() * sizeof(SpilledRow));
    up.add(o_spilled, ap.spilled.data(), ap.spilled.size() * sizeof(SpilledRow));
    // k-NN: every (row, chunk of its launch) owns a list of k candidates
    std::vector<int64_t> &knn_row_off = h->knn_row_off;
    std::vector<int32_t> &knn_row_lists = h->knn_row_lists;
    size_t o_knn_off = 0, o_knn_lists = 0;
    int64_t knn_entries = 0;
    if (knn_k > 0) {
        knn_row_off.assign((size_t)m, 0);
        knn_row_lists.assign((size_t)m, 0);
        for (const AClass &c : ap.classes)
            for (const ARow &r : c.rows)
                if (r.out >= 0) {
                    knn_row_off[(size_t)r.out] = knn_entries;
                    knn_row_lists[(size_t)r.out] = c.n_chunks;
                    knn_entries += (int64_t)c.n_chunks * knn_k;
                }
        // a spilled row: one list per tile of columns its finalize kernel walks
        const int64_t tiles = (n + kFinalizeTile - 1) / kFinalizeTile;
        for (const SpilledRow &sr : ap.spilled) {
            knn_row_off[(size_t)sr.row] = knn_entries;
            knn_row_lists[(size_t)sr.row] = (int32_t)tiles;
            knn_entries += tiles * knn_k;
        }
        o_knn_off = cv.take((size_t)m * 8);
        o_knn_lists = cv.take((size_t)m * 4);
        up.add(o_knn_off, knn_row_off.data(), (size_t)m * 8);
        up.add(o_knn_lists, knn_row_lists.data(), (size_t)m * 4);
    }
    const size_t a_plan_end = cv.off;
    const size_t o_partial = cv.take((size_t)ap.n_partial_slots * planes * (size_t)n * 8);
    const size_t o_partial_norms = cv.take((size_t)ap.n_partial_slots * 16);
    const size_t o_knn_part = cv.take((size_t)knn_entries * sizeof(KnnEntry));
    if (cv.off > h->ws_bytes || pin_a + (a_plan_end - a_plan_begin) > h->pinned_bytes) {
        // the bound was too small after all (or, with an index, this is where the scratch is
        // sized): growing waits for the repack, discards it and runs it again in the new buffers
        st = ensure_workspace(h, cv.off);
        if (st != SPD_OK) return st;
        st = ensure_pinned(h, pin_a + (a_plan_end - a_plan_begin));
        if (st != SPD_OK) return st;
        if (!index) {
            if (h->profile && !h->timed.empty()) {
                h->event_pool.push_back(h->timed.back().start); h->event_pool.push_back(h->timed.back().stop);
                h->timed.pop_back();
            }
            st = stage_b();
            if (st != SPD_OK) return st;
        }
    }
    unsigned char *ws = reinterpret_cast<unsigned char *>(h->ws);
    if (a_plan_end > a_plan_begin) {
        unsigned char *pin = reinterpret_cast<unsigned char *>(h->pinned) + pin_a;
        for (auto &pt : up.parts) std::memcpy(pin + (pt.first - a_plan_begin), pt.second.first, pt.second.second);
        e = hipMemcpyAsync(ws + a_plan_begin, pin, a_plan_end - a_plan_begin, hipMemcpyHostToDevice, h->stream);
        if (e != hipSuccess) return hip_fail(h, e, "upload of A's plan");
    }
    lap("upload a");

    // The launch with the most work stays on the caller's stream; the others go round-robin
    // to side streams that fork after the repack and join before whatever follows, so that
    // launches too small to fill the chip overlap with the large one.
    size_t main_class = 0;
    std::vector<int> lane_of(ap.classes.size(), -1);        // -1: caller's stream
    int side_used = 0;
    {
        int64_t best = -1;
        for (size_t ci = 0; ci < ap.classes.size(); ++ci) {
            int64_t work = (int64_t)ap.classes[ci].n_groups * ap.classes[ci].R;
            if (work > best) { best = work; main_class = ci; }
        }
        // A launch goes beside the large one only if it is small against it: two large launches
        // side by side push each other's share of B out of the L2 caches.
        auto small = [&](size_t ci) {
            return ci != main_class && (int64_t)ap.classes[ci].n_groups * ap.classes[ci].R * 4 <= best;
        };
        // ... and only if the small launches are worth hiding.  Beside a long launch over a large B,
        // a few workgroups that sweep B in an order of their own cost more (config 3: 6 % of the
        // call, the pairwise calls of config 2: 13 %) than the time they would take in line.  They
        // are worth it when the large launch is short (by the planner's estimate: under some 2 ms),
        // so that what a launch costs beside its sweep counts, or when they hold a tenth or more of
        // the call's sweeps over B (a group's sweep weighed by its rows plus the column lookup).
        auto sweeps = [&](size_t ci) { return (double)ap.classes[ci].n_groups * (3.0 + ap.classes[ci].R); };
        int n_small = 0;
        double small_sweeps = 0.0;
        for (size_t ci = 0; ci < ap.classes.size(); ++ci)
            if (small(ci)) { ++n_small; small_sweeps += sweeps(ci); }
        const bool worth = !ap.classes.empty() &&
                           (ap.classes[main_class].cost < 8000.0 || small_sweeps * 10.0 >= sweeps(main_class));
        if (h->side_streams > 0 && n_small > 0 && worth) {
            const int want = std::min<int>(h->side_streams, n_small);
            for (int q = 0; q < want; ++q) {
                if (!h->side[q] && hipStreamCreateWithFlags(&h->side[q], hipStreamNonBlocking) != hipSuccess) { h->side[q] = nullptr; break; }
                if (!h->join_event[q] && hipEventCreateWithFlags(&h->join_event[q], hipEventDisableTiming) != hipSuccess) break;
                side_used = q + 1;
            }
            if (!h->fork_event && hipEventCreateWithFlags(&h->fork_event, hipEventDisableTiming) != hipSuccess) side_used = 0;
        }
        if (side_used > 0) {
            e = hipEventRecord(h->fork_event, h->stream);
            if (e != hipSuccess) return hip_fail(h, e, "hipEventRecord");
            for (int q = 0; q < side_used; ++q) {
                e = hipStreamWaitEvent(h->side[q], h->fork_event, 0);
                if (e != hipSuccess) return hip_fail(h, e, "hipStreamWaitEvent");
            }
            int next = 0;
            for (size_t ci = 0; ci < ap.classes.size(); ++ci)
                if (small(ci)) { lane_of[ci] = next; next = (next + 1) % side_used; }
        }
    }
    // the large launch goes first: every microsecond the host spends on the others would
    // otherwise delay it
    std::vector<size_t> launch_order;
    if (!ap.classes.empty()) launch_order.push_back(main_class);
    for (size_t ci = 0; ci < ap.classes.size(); ++ci) if (ci != main_class) launch_order.push_back(ci);
    for (size_t ci : launch_order) {
        hipStream_t st_launch = lane_of[ci] >= 0 ? h->side[lane_of[ci]] : h->stream;
        const AClass &c = ap.classes[ci];
        ScanArgs sa;
        sa.a_indices = A->indices;
        sa.a_values = A->values;
        sa.arows = reinterpret_cast<const ARow *>(ws + o_rows[ci]);
        sa.sumlen = reinterpret_cast<const int32_t *>(ws + o_sumlen[ci]);
        sa.n_groups = c.n_groups;
        sa.chunk_begin = reinterpret_cast<const int32_t *>(ws + o_chunks[ci]);
        sa.n_chunks = c.n_chunks;
        sa.b_indptr = B->indptr;
        sa.b_indices = B->indices;
        sa.b = bd;
        sa.q = q;
        sa.kind = c.kind;
        sa.hscale = c.hscale;
        sa.cuckoo_attempts = h->cuckoo_attempts;
        sa.knn_seed = h->knn_seed;
        sa.transform = mi.transform;
        sa.norm = mi.norm;
        sa.k = (uint32_t)A->n_cols;
        sa.padcol = padcol;
        sa.out = out;
        sa.out_stride_staged = out_stride_staged;
        sa.out_stride_streamed = out_stride_streamed;
        sa.partial = reinterpret_cast<double *>(ws + o_partial);
        sa.partial_norms = reinterpret_cast<double *>(ws + o_partial_norms);
        sa.planes = planes;
        sa.knn_k = knn_k;
        sa.knn_part = reinterpret_cast<KnnEntry *>(ws + o_knn_part);
        sa.knn_row_off = reinterpret_cast<const int64_t *>(ws + o_knn_off);
        int64_t live_rows = 0;
        for (const ARow &r : c.rows) live_rows += (r.out != -1);
        LaunchTimer lt(h, "scan", c.R, c.kind, c.block, c.lds_bytes, live_rows, (int64_t)c.n_groups * c.n_chunks,
                       st_launch);
        e = launch_scan(st_launch, op, c.R, c.block, c.lds_bytes, sa);
        if (e != hipSuccess) {
            // what already runs on the side streams still has to be ordered before the caller's next work
            for (int q = 0; q < side_used; ++q)
                if (hipEventRecord(h->join_event[q], h->side[q]) == hipSuccess) (void)hipStreamWaitEvent(h->stream, h->join_event[q], 0);
            return hip_fail(h, e, "scan kernel");
        }
        lt.done();
    }

    {
        hipError_t first_error = hipSuccess;
        for (int q = 0; q < side_used; ++q) {
            e = hipEventRecord(h->join_event[q], h->side[q]);
            if (e == hipSuccess) e = hipStreamWaitEvent(h->stream, h->join_event[q], 0);
            if (e != hipSuccess && first_error == hipSuccess) first_error = e;      // the other streams are still joined
        }
        if (first_error != hipSuccess) return hip_fail(h, first_error, "joining the side streams");
    }

    if (!ap.spilled.empty()) {
        FinalizeArgs fa;
        fa.spilled = reinterpret_cast<const SpilledRow *>(ws + o_spilled);
        fa.n_spilled = (int32_t)ap.spilled.size();
        fa.partial = reinterpret_cast<const double *>(ws + o_partial);
        fa.partial_norms = reinterpret_cast<const double *>(ws + o_partial_norms);
        fa.norms_b = bd.norms;
        fa.planes = planes;
        fa.n_b = n;
        fa.q = q;
        fa.out = out;
        fa.out_stride_staged = out_stride_staged;
        fa.out_stride_streamed = out_stride_streamed;
        fa.knn_k = knn_k;
        fa.knn_part = reinterpret_cast<KnnEntry *>(ws + o_knn_part);
        fa.knn_row_off = reinterpret_cast<const int64_t *>(ws + o_knn_off);
        LaunchTimer lt(h, "finalize", 0, 0, 0, 0, (int64_t)ap.spilled.size(), 0);
        e = launch_finalize(h->stream, fa);
        if (e != hipSuccess) return hip_fail(h, e, "finalize kernel");
        lt.done();
    }
    lap("launches");
    if (knn_k > 0) {
        LaunchTimer lt(h, "knn_merge", 0, 0, 0, 0, m, (m + 3) / 4);
        e = launch_knn_merge(h->stream, reinterpret_cast<const KnnEntry *>(ws + o_knn_part),
                             reinterpret_cast<const int64_t *>(ws + o_knn_off),
                             reinterpret_cast<const int32_t *>(ws + o_knn_lists), m, knn_k,
                             metric == SPD_INNER_PRODUCT ? 1 : 0, out_idx, out_dist);
        if (e != hipSuccess) return hip_fail(h, e, "k-NN merge kernel");
        lt.done();
    }
    return SPD_OK;
}

}  // namespace

extern "C" {

spd_status spd_create(spd_handle **handle, void *hip_stream) {
    if (!handle) return SPD_ERR_NULL;
    *handle = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return SPD_ERR_HIP;
    spd_handle *h = new (std::nothrow) spd_handle();
    if (!h) return SPD_ERR_WORKSPACE;
    h->device = dev;
    h->stream = reinterpret_cast<hipStream_t>(hip_stream);
    int lds = 0, cus = 0;
    if (hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess && lds > 0)
        h->opt.lds_budget = std::min<int64_t>(lds, 160 * 1024);
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0)
        h->opt.n_cus = cus;
    e = hipMalloc(reinterpret_cast<void **>(&h->flag), 256);
    if (e != hipSuccess) { delete h; return SPD_ERR_HIP; }
    // this device's copy of the static scratch array: its address is asked for once per device
    if (dev >= 0 && dev < kStaticScratchDevices) {
        std::lock_guard<std::mutex> g(g_static_scratch_mutex);
        if (!g_static_scratch[dev]) {
            void *ptr = nullptr;
            e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
            if (e != hipSuccess || !ptr) { (void)hipFree(h->flag); delete h; return SPD_ERR_HIP; }
            g_static_scratch[dev] = ptr;
        }
        h->static_ws = g_static_scratch[dev];
    }
    // staging memory and the events that guard it, so that a call of modest size allocates nothing
    for (spd_handle::PinnedSlot &ps : h->pinned_slots) {
        if (hipHostMalloc(&ps.ptr, kInitialPinnedBytes, hipHostMallocDefault) != hipSuccess) { ps.ptr = nullptr; break; }
        ps.bytes = kInitialPinnedBytes;
        if (hipEventCreateWithFlags(&ps.done, hipEventDisableTiming) != hipSuccess) ps.done = nullptr;
    }
    *handle = h;
    return SPD_OK;
}

spd_status spd_destroy(spd_handle *h) {
    if (!h) return SPD_ERR_NULL;
    hipError_t e = hipStreamSynchronize(h->stream);
    (void)e;
    for (spd_handle::PinnedSlot &ps : h->pinned_slots) {
        if (ps.ptr) (void)hipHostFree(ps.ptr);
        if (ps.done) (void)hipEventDestroy(ps.done);
    }
    if (h->own_ws) (void)hipFree(h->own_ws);
    if (h->flag) (void)hipFree(h->flag);
    for (auto &t : h->timed) { (void)hipEventDestroy(t.start); (void)hipEventDestroy(t.stop); }
    for (hipEvent_t ev : h->event_pool) (void)hipEventDestroy(ev);
    for (int q = 0; q < spd_handle::kSideStreams; ++q) {
        if (h->side[q]) { (void)hipStreamSynchronize(h->side[q]); (void)hipStreamDestroy(h->side[q]); }
        if (h->join_event[q]) (void)hipEventDestroy(h->join_event[q]);
    }
    if (h->fork_event) (void)hipEventDestroy(h->fork_event);
    delete h;
    return SPD_OK;
}

spd_status spd_workspace_bytes(const spd_handle *h, const spd_csr *A, const spd_csr *B, spd_metric metric,
                               int k_neighbors, size_t *bytes) {
    if (!h || !A || !B || !bytes) return SPD_ERR_NULL;
    if ((int)metric < 0 || (int)metric >= SPD_METRIC_COUNT) return SPD_ERR_BAD_METRIC;
    if (A->n_rows < 0 || B->n_rows < 0 || A->nnz < 0 || B->nnz < 0 || A->n_cols != B->n_cols) return SPD_ERR_DIM_MISMATCH;
    *bytes = workspace_bound(h, A, B, (int)metric, k_neighbors);
    // (a pairwise call may exchange the roles of its operands)
    if (k_neighbors == 0 && h->swap_operands != 0 && operands_may_swap((int)metric, nullptr))
        *bytes = std::max(*bytes, workspace_bound(h, B, A, (int)metric, 0));
    // (a call may take the column lists; Minkowski of degree 1 runs as L1)
    for (const int as_metric : {(int)metric, metric == SPD_MINKOWSKI ? (int)SPD_L1 : (int)metric}) {
        const int op = product_of(h, as_metric, 2.0f);
        const bool swap = k_neighbors == 0 && swap_wanted(h, A, B, as_metric, nullptr);
        // (without an index, with one that keeps no lists and with one that does)
        for (const int index : {0, 1, 2}) {
            const MatchWay w = match_way(h, A, B, op, as_metric, nullptr, swap && index == 0, k_neighbors, index > 0, index == 2, SIZE_MAX);
            if (w.way != 0) *bytes = std::max(*bytes, w.L.end);
        }
    }
    return SPD_OK;
}

}  // extern "C"

namespace {
size_t workspace_bound(const spd_handle *h, const spd_csr *A, const spd_csr *B, int metric, int k_neighbors) {
    const PlanOptions &o = h->opt;
    const size_t m = (size_t)A->n_rows, n = (size_t)B->n_rows;
    const int split_len = split_len_for(o, B->nnz);
    const size_t seg_target = (size_t)std::max(1, std::max(2, split_len) / 2);
    const size_t window = (size_t)std::max(64, window_for(o, WINDOW_SCATTERED_STORES));   // the narrowest: the largest bound
    size_t slabs = n / 64 + n / window + (n + 4 * (size_t)B->nnz / seg_target) / 64 + 4;
    size_t lanes = slabs * 64;
    // at most 15 launches (5 group sizes x 3 occupancies), each cutting B at most 4096 times and
    // never into more than 4 workgroups per slot of the chip (times the chunk scale) plus one per group
    const size_t launches = 15;
    const size_t chunk_words = launches * 4097;
    // rows of A that do not fit alone are cut into slices of at least 1/2 of the largest
    // slice the budget admits; 512 entries is a floor for any budget the planner accepts
    size_t slices = 2 * (size_t)A->nnz / 512 + 2;
    slices = std::min(slices, (size_t)A->nnz / 64 + 2);
    size_t planes = (size_t)metric_planes(metric);
    size_t total = 0;
    auto add = [&](size_t b) { total += align256(b); };
    // padded slabs: at most 64 idle entries per step of the longest row of each window, one per
    // lane of a split row, and the rounding of each group of split rows
    size_t padded = (size_t)B->nnz + (size_t)B->nnz * 64 / (size_t)std::max(2, split_len) +
                    64 * (size_t)std::max(2, split_len) * (n / window + 8) + 64 * (size_t)kScanUnroll * slabs;
    add(padded * 8); add(n * 16); add((slabs + 1) * 8); add(slabs * 4); add(slabs);
    add(lanes * 8); add(lanes * 4); add(lanes * 4); add(lanes); add(chunk_words * 4); total += launches * 256;
    // (a group may leave a quarter of its places empty: up to a third more places than rows)
    const size_t places = m + slices + (m + slices) / 3 + 32 * 6;
    add(places * sizeof(ARow)); add((m + slices + 6) * 4); total += 12 * 256;
    add(slices * sizeof(SpilledRow));
    // partial results exist only for sliced rows; a row needs slicing only above ~9,000 entries
    size_t sliced_rows_max = (size_t)A->nnz / 4096 + 1;
    size_t partial_slots = std::min(slices, 2 * sliced_rows_max + (size_t)A->nnz / 4096);
    add(partial_slots * planes * n * 8); add(partial_slots * 16);
    if (k_neighbors > 0) {
        size_t lists = o.chunks > 0 ? (m + m / 3 + 16 * launches) * (size_t)o.chunks
                                    : launches * 16 * (16 * (size_t)o.n_cus * (size_t)chunk_scale_for(o, true) + 1) + m + m / 3 + 16 * launches;
        lists += std::min(sliced_rows_max, m) * (n / (size_t)kFinalizeTile + 1);     // the tiles of spilled rows
        add(lists * (size_t)k_neighbors * sizeof(KnnEntry)); add(m * 8); add(m * 4);
    }
    return total;
}
}  // namespace

extern "C" {

spd_status spd_set_workspace(spd_handle *h, void *device_ptr, size_t bytes) {
    if (!h) return SPD_ERR_NULL;
    h->err.clear();
    if (!device_ptr || bytes == 0) {
        h->ws_external = false;
        h->ws = h->own_ws;
        h->ws_bytes = h->own_ws_bytes;
        return SPD_OK;
    }
    if ((reinterpret_cast<uintptr_t>(device_ptr) & 255u) != 0) return fail(h, SPD_ERR_WORKSPACE, "workspace must be 256-byte aligned");
    h->ws_external = true;
    h->ws = device_ptr;
    h->ws_bytes = bytes;
    return SPD_OK;
}

spd_status spd_pairwise(spd_handle *h, const spd_csr *A, const spd_csr *B, spd_metric metric, float p, float *out) {
    spd_status st = check_call_args(h, A, B, metric, p, 0, false, out, nullptr);
    if (st != SPD_OK) return st;
    return run(h, A, B, (int)metric, p, nullptr, 0, out, nullptr, nullptr);
}

spd_status spd_pairwise_static(spd_handle *h, const spd_csr *A, const spd_csr *B, spd_metric metric, float p,
                               float *out) {
    spd_status st = check_call_args(h, A, B, metric, p, 0, false, out, nullptr);
    if (st != SPD_OK) return st;
    if (!A->host_indptr || !B->host_indptr)
        return fail(h, SPD_ERR_NULL, "spd_pairwise_static needs host_indptr of both operands (it neither copies the row "
                                     "pointers back nor waits for the stream)");
    if (!h->static_ws) return fail(h, SPD_ERR_HIP, "no static scratch on this device");
    for (const spd_handle::PinnedSlot &ps : h->pinned_slots)
        if (!ps.ptr || !ps.done) return fail(h, SPD_ERR_WORKSPACE, "the handle holds no staging memory");
    // the call runs as spd_pairwise does, with the static array as its scratch, on the handle's
    // stream alone and without launch timers (internal streams and events would have to be created)
    struct Saved {
        spd_handle *h; void *ws; size_t ws_bytes; bool ws_external; int side_streams; bool profile;
        ~Saved() { h->ws = ws; h->ws_bytes = ws_bytes; h->ws_external = ws_external; h->side_streams = side_streams;
                   h->profile = profile; h->no_alloc = false; }
    } saved{h, h->ws, h->ws_bytes, h->ws_external, h->side_streams, h->profile};
    h->ws = h->static_ws;
    h->ws_bytes = kStaticScratchBytes;
    h->ws_external = true;
    h->side_streams = 0;
    h->profile = false;
    h->no_alloc = true;
    return run(h, A, B, (int)metric, p, nullptr, 0, out, nullptr, nullptr);
}

spd_status spd_knn(spd_handle *h, const spd_csr *Q, const spd_csr *Index, spd_metric metric, float p, int k,
                   int64_t *out_idx, float *out_dist) {
    spd_status st = check_call_args(h, Q, Index, metric, p, k, true, out_idx, out_dist);
    if (st != SPD_OK) return st;
    return run(h, Q, Index, (int)metric, p, nullptr, k, nullptr, out_idx, out_dist);
}

spd_status spd_semiring_pairwise(spd_handle *h, const spd_csr *A, const spd_csr *B, const spd_semiring *semiring,
                                 float *out) {
    spd_status st = check_call_args(h, A, B, SPD_INNER_PRODUCT, 0.0f, 0, false, out, nullptr, semiring, true);
    if (st != SPD_OK) return st;
    const int as_metric = table1_metric(*semiring, false);
    if (as_metric >= 0) return run(h, A, B, as_metric, semiring->p, nullptr, 0, out, nullptr, nullptr);
    return run(h, A, B, semiring->sum == SPD_SUM_PLUS ? MT_SEMI_SUM : MT_SEMI_EXT, 1.0f, semiring, 0, out, nullptr, nullptr);
}

spd_status spd_semiring_knn(spd_handle *h, const spd_csr *Q, const spd_csr *Index, const spd_semiring *semiring, int k,
                            int64_t *out_idx, float *out_dist) {
    spd_status st = check_call_args(h, Q, Index, SPD_INNER_PRODUCT, 0.0f, k, true, out_idx, out_dist, semiring, true);
    if (st != SPD_OK) return st;
    const int as_metric = table1_metric(*semiring, true);
    if (as_metric >= 0) return run(h, Q, Index, as_metric, semiring->p, nullptr, k, nullptr, out_idx, out_dist);
    return run(h, Q, Index, semiring->sum == SPD_SUM_PLUS ? MT_SEMI_SUM : MT_SEMI_EXT, 1.0f, semiring, k, nullptr, out_idx,
               out_dist);
}

spd_status spd_index_create(spd_handle *h, const spd_csr *Index, spd_metric metric, float p, spd_index **out) {
    if (!h) return SPD_ERR_NULL;
    h->err.clear();
    if (!out) return fail(h, SPD_ERR_NULL, "index is NULL");
    *out = nullptr;
    spd_status st = check_csr_args(h, Index, "Index");
    if (st != SPD_OK) return st;
    if ((int)metric < 0 || (int)metric >= SPD_METRIC_COUNT) return fail(h, SPD_ERR_BAD_METRIC, "unknown metric");
    if (metric == SPD_MINKOWSKI && !(p > 0.0f && std::isfinite(p))) return fail(h, SPD_ERR_BAD_P, "Minkowski needs a finite p > 0");
    for (auto &t : h->timed) { h->event_pool.push_back(t.start); h->event_pool.push_back(t.stop); }
    h->timed.clear();
    hipError_t e = hipSetDevice(h->device);
    if (e != hipSuccess) return hip_fail(h, e, "hipSetDevice");
    const int64_t n = Index->n_rows;
    spd_index *ix = new (std::nothrow) spd_index();
    if (!ix) return fail(h, SPD_ERR_WORKSPACE, "out of host memory");
    struct Guard { spd_index *p; ~Guard() { if (p) { if (p->dev) (void)hipFree(p->dev); if (p->match_dev) (void)hipFree(p->match_dev); delete p; } } } guard{ix};
    ix->matrix = *Index;
    ix->metric = (int)metric;
    ix->p = p;
    ix->device = h->device;
    PinnedLease lease(h);
    st = ensure_pinned(h, (size_t)(n + 1) * 8 + 32 * ((size_t)n + 4096));
    if (st != SPD_OK) return st;
    const int64_t *b_ip = Index->host_indptr;
    if (!b_ip) {
        int64_t *pin = reinterpret_cast<int64_t *>(h->pinned);
        e = hipMemcpyAsync(pin, Index->indptr, (size_t)(n + 1) * 8, hipMemcpyDeviceToHost, h->stream);
        if (e != hipSuccess) return hip_fail(h, e, "copy of Index.indptr");
        e = hipStreamSynchronize(h->stream);
        if (e != hipSuccess) return hip_fail(h, e, "hipStreamSynchronize");
        b_ip = pin;
    }
    if (b_ip[n] != Index->nnz) return fail(h, SPD_ERR_BAD_CSR, "indptr[n_rows] != nnz");
    if (n <= kDirectMostRows)
        for (int64_t j = 0; j < n; ++j) ix->chain = std::max(ix->chain, b_ip[j + 1] - b_ip[j]);
    if (n <= kDirectKnnRows) ix->knn_chain = direct_knn_chain(b_ip, n);
    std::string why;
    try {
        PlanOptions opt_b = h->opt;
        opt_b.window = window_for(h->opt, WINDOW_SCATTERED_STORES);      // an index serves pairwise calls that stage A as well
        why = plan_b(b_ip, n, opt_b, ix->plan);
    } catch (const std::exception &ex) {
        why = std::string("planning failed: ") + ex.what();
    }
    if (!why.empty()) return refuse_plan(h, "Index", why);
    Carver cv;
    const BLayout bl = layout_b(ix->plan, n, cv);
    ix->dev_bytes = std::max<size_t>(cv.off, 256);
    e = hipMalloc(&ix->dev, ix->dev_bytes);
    if (e != hipSuccess) { ix->dev = nullptr; return fail(h, SPD_ERR_WORKSPACE, std::string("hipMalloc of the index failed: ") + hipGetErrorString(e)); }
    // (the row pointers have served: the plan's arrays may overwrite them in the pinned buffer)
    st = ensure_pinned(h, bl.plan_end + 256);
    if (st != SPD_OK) return st;
    const int run_as = effective_metric((int)metric, p);
    const MetricInfo mi = metric_info(run_as);
    const OpParams q = op_params(run_as, p, Index->n_cols, nullptr);
    if (n > 0) {
        st = stage_b_into(h, Index, ix->plan, bl, reinterpret_cast<unsigned char *>(ix->dev),
                          reinterpret_cast<unsigned char *>(h->pinned), run_as, mi, q, (uint32_t)Index->n_cols, ix->bd);
        if (st != SPD_OK) return st;
    }
    const int op = product_of(h, run_as, p);
    MatchShape shape;
    MatchLayout lists;
    if (index_keeps_lists(h, Index, op, shape, lists)) {
        if (hipMalloc(&ix->match_dev, lists.end) == hipSuccess) {
            ix->match = match_b_at(shape, lists, reinterpret_cast<unsigned char *>(ix->match_dev));
            ix->match_op = op;
            st = stage_norms(h, Index, ix->match, run_as, mi, q, RowsVerdict{nullptr, 0u});
            if (st == SPD_OK) st = stage_lists(h, Index, ix->match, op, mi, true, RowsVerdict{nullptr, 0u});
            if (st != SPD_OK) return st;
        } else {                         // (no memory left for the lists: the packed copy serves every call)
            ix->match_dev = nullptr;
            (void)hipGetLastError();
        }
    }
    guard.p = nullptr;
    *out = ix;
    return SPD_OK;
}

spd_status spd_index_destroy(spd_handle *h, spd_index *index) {
    if (!h) return SPD_ERR_NULL;
    h->err.clear();
    if (!index) return SPD_OK;
    hipError_t e = hipStreamSynchronize(h->stream);      // calls that read the index may still be running
    (void)e;
    if (index->dev) (void)hipFree(index->dev);
    if (index->match_dev) (void)hipFree(index->match_dev);
    delete index;
    return SPD_OK;
}

spd_status spd_index_pairwise(spd_handle *h, const spd_csr *A, const spd_index *index, float *out) {
    if (!h) return SPD_ERR_NULL;
    if (!index) { h->err = "index is NULL"; return SPD_ERR_NULL; }
    spd_status st = check_call_args(h, A, &index->matrix, (spd_metric)index->metric, index->p, 0, false, out, nullptr);
    if (st != SPD_OK) return st;
    if (index->device != h->device) return fail(h, SPD_ERR_UNSUPPORTED, "the index lives on another device");
    return run(h, A, &index->matrix, index->metric, index->p, nullptr, 0, out, nullptr, nullptr, index);
}

spd_status spd_index_knn(spd_handle *h, const spd_csr *Q, const spd_index *index, int k, int64_t *out_idx,
                         float *out_dist) {
    if (!h) return SPD_ERR_NULL;
    if (!index) { h->err = "index is NULL"; return SPD_ERR_NULL; }
    spd_status st = check_call_args(h, Q, &index->matrix, (spd_metric)index->metric, index->p, k, true, out_idx, out_dist);
    if (st != SPD_OK) return st;
    if (index->device != h->device) return fail(h, SPD_ERR_UNSUPPORTED, "the index lives on another device");
    return run(h, Q, &index->matrix, index->metric, index->p, nullptr, k, nullptr, out_idx, out_dist, index);
}

spd_status spd_csr_validate(spd_handle *h, const spd_csr *M, int require_nonnegative) {
    if (!h) return SPD_ERR_NULL;
    h->err.clear();
    spd_status st = check_csr_args(h, M, "M");
    if (st != SPD_OK) return st;
    if (M->n_rows == 0) return M->nnz == 0 ? SPD_OK : fail(h, SPD_ERR_BAD_CSR, "no rows but nnz > 0");
    hipError_t e = hipMemsetAsync(h->flag, 0, 4, h->stream);
    if (e != hipSuccess) return hip_fail(h, e, "hipMemsetAsync");
    e = launch_validate(h->stream, M->indptr, M->indices, M->values, M->n_rows, M->n_cols, M->nnz,
                        require_nonnegative, h->flag);
    if (e != hipSuccess) return hip_fail(h, e, "validate kernel");
    int32_t flag = 0;
    e = hipMemcpyAsync(&flag, h->flag, 4, hipMemcpyDeviceToHost, h->stream);
    if (e != hipSuccess) return hip_fail(h, e, "hipMemcpyAsync");
    e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return hip_fail(h, e, "hipStreamSynchronize");
    if (flag) {
        std::string what;
        if (flag & 1) what += " row pointers;";
        if (flag & 2) what += " column order or range;";
        if (flag & 4) what += " values;";
        return fail(h, SPD_ERR_BAD_CSR, "invalid CSR:" + what);
    }
    return SPD_OK;
}

spd_status spd_set_option(spd_handle *h, const char *name, int64_t value) {
    if (!h || !name) return SPD_ERR_NULL;
    h->err.clear();
    std::string s(name);
    PlanOptions &o = h->opt;
    if (s == "lds_budget") {
        if (value < 8192 || value > 160 * 1024) return fail(h, SPD_ERR_UNSUPPORTED, "lds_budget must lie in [8192, 163840]");
        o.lds_budget = value;
    } else if (s == "force_kind") {
        if (value < 0 || value > 5) return fail(h, SPD_ERR_UNSUPPORTED, "force_kind must be 0..5");
        o.force_kind = (int)value;
    } else if (s == "max_rows") {
        if (value != 1 && value != 2 && value != 4 && value != 8 && value != 16)
            return fail(h, SPD_ERR_UNSUPPORTED, "max_rows must be 1, 2, 4, 8 or 16");
        o.max_rows = (int)value;
    } else if (s == "split_len") {
        if (value != 0 && (value < 2 || value > (1 << 20)))
            return fail(h, SPD_ERR_UNSUPPORTED, "split_len must be 0 (automatic) or lie in [2, 2^20]");
        o.split_len = (int)value;
    } else if (s == "window") {
        if (value != 0 && (value < 64 || value > (1 << 24)))
            return fail(h, SPD_ERR_UNSUPPORTED, "window must be 0 (automatic) or lie in [64, 2^24]");
        o.window = (int)value;
    } else if (s == "chunk_scale") {
        if (value < 0 || value > 8) return fail(h, SPD_ERR_UNSUPPORTED, "chunk_scale must lie in [0, 8]");
        o.chunk_scale = (int)value;
    } else if (s == "chunks") {
        if (value < 0 || value > 4096) return fail(h, SPD_ERR_UNSUPPORTED, "chunks must lie in [0, 4096]");
        o.chunks = (int)value;
    } else if (s == "byte_counters") {
        if (value != 0 && value != 1) return fail(h, SPD_ERR_UNSUPPORTED, "byte_counters must be 0 or 1");
        h->no_byte_counters = value == 0;
    } else if (s == "waves_per_cu") {
        if (value != 0 && value != 8 && value != 16 && value != 32)
            return fail(h, SPD_ERR_UNSUPPORTED, "waves_per_cu must be 0 (automatic), 8, 16 or 32");
        o.waves_per_cu = (int)value;
    } else if (s == "sort_slack") {
        if (value != 0 && value != 1) return fail(h, SPD_ERR_UNSUPPORTED, "sort_slack must be 0 or 1");
        o.sort_slack = (int)value;
    } else if (s == "partial_groups") {
        if (value < 0 || value > 2) return fail(h, SPD_ERR_UNSUPPORTED, "partial_groups must be 0, 1 or 2");
        o.partial_groups = (int)value;
    } else if (s == "bloom_long_rows") {
        if (value != 0 && value != 1) return fail(h, SPD_ERR_UNSUPPORTED, "bloom_long_rows must be 0 or 1");
        o.bloom_long_rows = (int)value;
    } else if (s == "side_streams") {
        if (value < 0 || value > spd_handle::kSideStreams) return fail(h, SPD_ERR_UNSUPPORTED, "side_streams must lie in [0, 3]");
        h->side_streams = (int)value;
    } else if (s == "knn_seed") {
        if (value < 0 || value > 1) return fail(h, SPD_ERR_UNSUPPORTED, "knn_seed must be 0 or 1");
        h->knn_seed = (int)value;
    } else if (s == "cuckoo_attempts") {
        if (value < 0 || value > 3) return fail(h, SPD_ERR_UNSUPPORTED, "cuckoo_attempts must lie in [0, 3]");
        h->cuckoo_attempts = (int)value;
    } else if (s == "direct") {
        if (value < 0 || value > 1) return fail(h, SPD_ERR_UNSUPPORTED, "direct must be 0 or 1");
        h->direct = (int)value;
    } else if (s == "match_lists") {
        if (value < 0 || value > 3) return fail(h, SPD_ERR_UNSUPPORTED, "match_lists must be 0, 1, 2 or 3");
        h->match_lists = (int)value;
        h->lists_refused = SIZE_MAX;
    } else if (s == "swap_operands") {
        if (value < 0 || value > 2) return fail(h, SPD_ERR_UNSUPPORTED, "swap_operands must be 0, 1 or 2");
        h->swap_operands = (int)value;
    } else if (s == "check_plan") {
        if (value != 0 && value != 1) return fail(h, SPD_ERR_UNSUPPORTED, "check_plan must be 0 or 1");
        h->check_plan = value != 0;
    } else if (s == "profile") {
        if (value != 0 && value != 1) return fail(h, SPD_ERR_UNSUPPORTED, "profile must be 0 or 1");
        h->profile = value != 0;
    } else {
        return fail(h, SPD_ERR_UNSUPPORTED, "unknown option " + s);
    }
    return SPD_OK;
}

int spd_profile_read(spd_handle *h, spd_kernel_time *out, int cap) {
    if (!h || (cap > 0 && !out)) return -1;
    if (h->timed.empty()) return 0;
    if (hipEventSynchronize(h->timed.back().stop) != hipSuccess) return -2;
    int n = 0;
    for (auto &t : h->timed) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, t.start, t.stop) == hipSuccess) t.rec.ms = (double)ms;
        if (n < cap) out[n] = t.rec;
        ++n;
    }
    return n;
}

const char *spd_last_error(const spd_handle *h) { return h ? h->err.c_str() : "null handle"; }

const char *spd_metric_name(spd_metric metric) {
    return ((int)metric >= 0 && (int)metric < SPD_METRIC_COUNT) ? kMetricNames[(int)metric] : "unknown";
}

const char *spd_version(void) { return "spd 0.1 (gfx950)"; }

// A test hook (include/spd_testing.h): it touches no GPU.
spd_status spd_host_list_plan(int64_t a_rows, int64_t a_nnz, int64_t b_rows, int64_t b_nnz, int64_t n_cols, spd_metric metric, float p,
                              int k_neighbors, int with_index, const char *const *option_names, const int64_t *option_values,
                              int n_options, spd_list_plan *out) {
    if (!out) return SPD_ERR_NULL;
    if ((int)metric < 0 || (int)metric >= SPD_METRIC_COUNT) return SPD_ERR_BAD_METRIC;
    spd_handle h;
    for (int i = 0; i < n_options; ++i) {
        if (std::strcmp(option_names[i], "scratch") == 0) {
            h.ws_external = true;
            h.ws_bytes = (size_t)option_values[i];
            continue;
        }
        const spd_status st = spd_set_option(&h, option_names[i], option_values[i]);
        if (st != SPD_OK) return st;
    }
    const spd_csr A{a_rows, n_cols, a_nnz, nullptr, nullptr, nullptr, nullptr}, B{b_rows, n_cols, b_nnz, nullptr, nullptr, nullptr, nullptr};
    const int run_as = effective_metric((int)metric, p), op = product_of(&h, run_as, p);
    const bool knn = k_neighbors > 0, swap = !knn && !with_index && swap_wanted(&h, &A, &B, run_as, nullptr);
    std::memset(out, 0, sizeof *out);
    out->wanted = match_wanted(&h, &A, &B, op, run_as, nullptr, a_rows > 0 && b_rows > 0 ? staged_cost(&h, &A, &B, op, run_as, swap, knn, with_index != 0) : 0.0, knn, with_index != 0);
    MatchShape kept;
    MatchLayout L;
    const bool keeps = index_keeps_lists(&h, &B, op, kept, L);
    out->index_bytes = keeps ? (int64_t)L.end : 0;
    out->index_aligned = keeps ? kept.aligned : 0;
    const Staging staging = staging_of(n_cols, run_as, op, knn, swap ? (double)b_nnz / (double)std::max<int64_t>(b_rows, 1) : (double)a_nnz / (double)std::max<int64_t>(a_rows, 1), h.opt);
    out->staged_kind = staging.kind;
    out->staged_rows = staging.rows;
    MatchWay w = match_way(&h, &A, &B, op, run_as, nullptr, swap, k_neighbors, with_index != 0, keeps, scratch_room(&h));
    if (w.way != 0 && h.ws_external && w.L.end > h.ws_bytes) w.way = 0;
    out->way = w.way;
    if (w.way == 0) {                    // (the cut that the lists over all columns would have)
        w.columns = n_cols;
        w.s = match_shape(h.opt.lds_budget, op, b_rows, n_cols, b_nnz);
        if (w.s.n_tiles <= 0) return SPD_OK;
        w.g = match_grid(h.opt, w.s, op, a_rows, a_nnz, b_nnz, knn);
        w.L = layout_match_call(w.s, w.g, op, a_rows, a_nnz, b_rows, b_nnz, k_neighbors, !with_index, 0);
    }
    out->columns = w.columns;
    out->block_columns = (int64_t)1 << w.s.block_shift;
    out->aligned = w.s.aligned;
    out->tiles = w.s.n_tiles;
    out->tile_rows = w.s.tile_rows;
    out->slices = w.g.slices;
    out->groups = w.g.groups;
    out->run = w.g.run;
    out->shared_len = w.g.shared_len;
    out->consistent = match_check(h.opt, w.s, w.g, op, a_rows, b_rows, w.columns, b_nnz).empty();
    out->scratch_bytes = (int64_t)w.L.end;
    return SPD_OK;
}

spd_status spd_host_direct_lanes(const int64_t *b_indptr, int64_t b_rows, int64_t a_rows, int64_t a_nnz, int64_t n_cols, spd_metric metric,
                                 float p, int k_neighbors, int with_index, int *lanes) {
    if (!b_indptr || !lanes) return SPD_ERR_NULL;
    if ((int)metric < 0 || (int)metric >= SPD_METRIC_COUNT) return SPD_ERR_BAD_METRIC;
    spd_handle h;
    const spd_csr A{a_rows, n_cols, a_nnz, nullptr, nullptr, nullptr, nullptr}, B{b_rows, n_cols, b_indptr[b_rows], nullptr, nullptr, nullptr, nullptr};
    const int op = product_of(&h, effective_metric((int)metric, p), p);
    int64_t chain = 0;
    if (!check_rows(b_indptr, b_rows, INT64_MAX, &chain).empty()) return SPD_ERR_BAD_CSR;
    if (k_neighbors > 0) chain = direct_knn_chain(b_indptr, b_rows);
    *lanes = direct_possible(&h, &A, &B, op, nullptr, k_neighbors) ? direct_lanes(&h, &A, &B, op, k_neighbors, chain, with_index != 0) : 0;
    return SPD_OK;
}

}  // extern "C"
