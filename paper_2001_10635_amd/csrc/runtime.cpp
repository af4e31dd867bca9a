// C-ABI runtime of the reachability library: argument validation, launch
// planning (tile shape, steps per HBM pass, ping-pong buffers), the batch
// path with its captured hipGraph, the one-launch-per-query baseline, the
// autotuner and the continuous-batching server.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <map>
#include <condition_variable>
#include <functional>
#include <memory>
#include <mutex>
#include <string>
#include <thread>
#include <unordered_map>
#include <vector>

#include "../../include/reach.h"
#include "kernels.hpp"

using namespace reach;

void reach::kernel_params(int kind, const double* prm, double out[5]) {
    for (int i = 0; i < 5; ++i) out[i] = 0.0;
    if (kind == REACH_CTM) {
        out[0] = prm[0]; out[1] = prm[1]; out[2] = prm[1] * prm[2]; out[3] = prm[3];
    } else if (kind == REACH_RD) {
        const double ih2 = 1.0 / (prm[0] * prm[0]);
        out[0] = ih2;
        out[1] = 2.0 * ih2;
    } else {
        out[0] = prm[0]; out[1] = prm[1]; out[2] = prm[2]; out[3] = prm[3];
    }
}

namespace {

constexpr int64_t kMaxN = (int64_t)1 << 40;
constexpr int64_t kBatchMaxN = 512;

struct GraphKey {
    int64_t nq;
    void* ws;
    void* staging;
    int64_t grid;
    hipStream_t stream;
    bool operator<(const GraphKey& o) const {
        return std::tie(nq, ws, staging, grid, stream) < std::tie(o.nq, o.ws, o.staging, o.grid, o.stream);
    }
};

struct TuneEntry { int E; int K; int S; };

// The last shapes estimated (fastest_shape), by what they depend on: a call of a
// few microseconds would otherwise spend one on the estimate each time.  Under a
// lock of its own: planning otherwise only reads the context.
struct ShapeMemo {
    std::mutex m;
    struct Slot { int64_t n = 0, K = 0; int kind = 0, dtype = 0, flags = 0; TuneEntry t{0, 0, 0}; };
    Slot slot[16];
    int next = 0;
};

// Device memory of the passes of a chain that one window holds and that is cut
// into several all the same (see plan_embed).  Such a call needs no workspace of
// the caller's, and calls on different streams or threads do not wait for each
// other's host side, so each stream gets a slot of its own as long as there are
// any; after that the one used longest ago is taken over.  What keeps two runs in
// one slot apart is the slot's lock (a run's passes are issued under it) and its
// event (a run waits for the one before, on whichever stream that was); the
// stream's handle only chooses the slot.
struct CutScratch {
    static constexpr int kSlots = 16;
    static constexpr size_t kSlotBytes = 32768;   // 2n values: 2048 FP64 or 4096 FP32 cells
    struct Slot {
        std::mutex m;
        hipEvent_t done = nullptr;   // the slot's last run
        bool recorded = false;       // under m
        bool taken = false;          // under CutScratch::m
        hipStream_t stream = nullptr;
        uint64_t last = 0;
    };
    std::mutex m;
    uint64_t calls = 0;
    Slot slot[kSlots];
    char* mem = nullptr;

    int pick(hipStream_t s) {
        std::lock_guard<std::mutex> lk(m);
        int k = -1;
        for (int i = 0; i < kSlots && k < 0; ++i)
            if (slot[i].taken && slot[i].stream == s) k = i;
        for (int i = 0; i < kSlots && k < 0; ++i)
            if (!slot[i].taken) k = i;
        if (k < 0) {
            k = 0;
            for (int i = 1; i < kSlots; ++i)
                if (slot[i].last < slot[k].last) k = i;
        }
        slot[k].taken = true;
        slot[k].stream = s;
        slot[k].last = ++calls;
        return k;
    }
};

// A run's hold on a slot: from the wait for the slot's previous run to the event
// of its own last pass, which is recorded however the run's issue ends.
struct CutRun {
    CutScratch::Slot* slot = nullptr;
    hipStream_t stream = nullptr;
    char* mem = nullptr;
    hipError_t begin(CutScratch& c, hipStream_t s) {
        const int k = c.pick(s);
        c.slot[k].m.lock();
        slot = &c.slot[k];
        stream = s;
        mem = c.mem + (size_t)k * CutScratch::kSlotBytes;
        if (!slot->done) return hipEventCreateWithFlags(&slot->done, hipEventDisableTiming);
        return slot->recorded ? hipStreamWaitEvent(s, slot->done, 0) : hipSuccess;
    }
    ~CutRun() {
        if (!slot) return;
        if (!slot->done) {
            slot->m.unlock();
            return;
        }
        slot->recorded |= hipEventRecord(slot->done, stream) == hipSuccess;
        slot->m.unlock();
    }
};

}  // namespace

// Host worker threads kept for the life of a context (starting threads per
// call costs more than the work they share on a batch of 10^5 queries).
// run(nth, fn) calls fn(0) on the caller and fn(1 .. nth-1) on workers and
// returns when all have finished.  A batch plan runs five such phases back to
// back, so a worker that finishes one watches the job counter for up to
// kSpinUs before it sleeps on the condition variable (a wake-up from sleep
// costs tens of microseconds per phase), and the caller likewise watches for
// the last worker before it sleeps.  A worker that sees the new job while
// watching takes it without the mutex (the job is published before the
// counter, release / acquire), so that the workers of a phase do not queue on
// one lock.
class HostPool {
  public:
    explicit HostPool(int n) : n_(n) {
        for (int i = 1; i < n; ++i) th_.emplace_back([this, i] { loop(i); });
    }
    ~HostPool() {
        {
            std::lock_guard<std::mutex> g(m_);
            stop_.store(true, std::memory_order_relaxed);
            ++gen_;
            agen_.store(gen_, std::memory_order_release);
        }
        start_.notify_all();
        for (auto& t : th_) t.join();
    }
    int size() const { return n_; }
    void run(int nth, const std::function<void(int)>& fn) {
        if (nth <= 1 || n_ <= 1) {
            fn(0);
            return;
        }
        {
            std::lock_guard<std::mutex> g(m_);
            job_.store(&fn, std::memory_order_relaxed);
            job_n_.store(std::min(nth, n_), std::memory_order_relaxed);
            pending_.store(n_ - 1, std::memory_order_relaxed);
            ++gen_;
            agen_.store(gen_, std::memory_order_release);
        }
        start_.notify_all();
        fn(0);
        spin([&] { return pending_.load(std::memory_order_acquire) == 0; });
        std::unique_lock<std::mutex> lk(m_);
        done_.wait(lk, [&] { return pending_.load(std::memory_order_acquire) == 0; });
    }

  private:
    static constexpr int kSpinUs = 200;
    template <class P>
    static void spin(P&& ready) {
        const auto until = std::chrono::steady_clock::now() + std::chrono::microseconds(kSpinUs);
        while (!ready()) {
            for (int k = 0; k < 64 && !ready(); ++k) __builtin_ia32_pause();
            if (ready() || std::chrono::steady_clock::now() > until) return;
        }
    }
    void loop(int id) {
        uint64_t seen = 0;
        for (;;) {
            spin([&] { return agen_.load(std::memory_order_acquire) != seen; });
            uint64_t g = agen_.load(std::memory_order_acquire);
            if (g == seen) {
                std::unique_lock<std::mutex> lk(m_);
                start_.wait(lk, [&] { return gen_ != seen; });
                g = gen_;
            }
            seen = g;
            if (stop_.load(std::memory_order_acquire)) return;
            const std::function<void(int)>* job = job_.load(std::memory_order_relaxed);
            const int jn = job_n_.load(std::memory_order_relaxed);
            if (id < jn) (*job)(id);
            if (pending_.fetch_sub(1, std::memory_order_acq_rel) == 1) {
                std::lock_guard<std::mutex> g(m_);
                done_.notify_one();
            }
        }
    }
    int n_;
    std::vector<std::thread> th_;
    std::mutex m_;
    std::condition_variable start_, done_;
    std::atomic<const std::function<void(int)>*> job_{nullptr};
    std::atomic<int> job_n_{0};
    std::atomic<int> pending_{0};
    uint64_t gen_ = 0;               // under m_; agen_ mirrors it for watchers
    std::atomic<uint64_t> agen_{0};
    std::atomic<bool> stop_{false};
};

struct reach_ctx {
    int device = 0;
    int cus = 256;
    std::string arch;
    unsigned int* status = nullptr;      // device status word
    std::string err;
    std::map<std::string, int64_t> opt;
    // (kind, dtype, log2 n bucket, per-cell inputs)
    std::map<std::tuple<int, int, int, int>, TuneEntry> tune;
    ShapeMemo shapes;
    CutScratch cut;                      // its memory follows the status word
    std::map<std::pair<int, int>, int> batch_tune;        // (kind, log2 n bucket) -> pack E cap
    int64_t batch_waves[2] = {0, 0};                     // autotuned resident waves of the
                                                         // narrow / wide packing kernel (0 = none)
    int batch_cap = 0;                                   // autotuned pack E cap of all buckets (0 = none)
    int last_packed = 0;                                 // kernel of the last batch (launch_batch)
    // batch staging (pinned host) and graph cache
    QDesc* staging = nullptr;            // [nq] descriptors, [nq] items, item count
    int64_t staging_cap = 0;
    hipEvent_t staging_ev = nullptr;     // the last batch's uploads from the staging are done
    hipEvent_t batch_ev = nullptr;       // the last batch's kernel is done
    hipEvent_t block_ev[2] = {nullptr, nullptr};   // the last kernel that read workspace block b
    bool batch_ev_recorded = false;
    bool block_ev_recorded[2] = {false, false};
    int next_block = 0;                  // workspace block of the next batch
    void* last_ws = nullptr;             // workspace and query count of the last batch
    int64_t last_nq = 0;
    hipStream_t copy_stream = nullptr;   // batch uploads, beside the previous batch's kernel
    std::map<GraphKey, hipGraphExec_t> graphs;
    std::vector<hipStream_t> each_streams;
    bool log = false;                    // REACH_LOG: one JSON line per call on stderr
    std::unique_ptr<HostPool> pool;      // batch preparation threads (on first large batch)
};

namespace {

reach_status fail(reach_ctx* c, reach_status st, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (c) c->err = buf;
    return st;
}

// One "reach: {...}" line on stderr when the context logs (REACH_LOG).
void log_call(const reach_ctx* c, const char* fmt, ...) {
    if (!c || !c->log) return;
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    std::fprintf(stderr, "reach: {%s}\n", buf);
}

const char* dtype_name(reach_dtype d) { return d == REACH_F64 ? "f64" : "f32"; }

reach_status hip_fail(reach_ctx* c, hipError_t e, const char* what) {
    return fail(c, REACH_E_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

#define HIPCHK(c, expr)                                          \
    do {                                                         \
        hipError_t _e = (expr);                                  \
        if (_e != hipSuccess) return hip_fail((c), _e, #expr);   \
    } while (0)

size_t dsize(reach_dtype d) { return d == REACH_F64 ? 8 : 4; }

int64_t opt_get(const reach_ctx* c, const char* k) {
    if (c->opt.empty()) return 0;   // no option was ever set: the small calls' path
    auto it = c->opt.find(k);
    return it == c->opt.end() ? 0 : it->second;
}

reach_status check_system_kind(reach_ctx* c, const reach_system* s, reach_dtype dtype,
                               bool user) {
    if (!s) return fail(c, REACH_E_INVAL, "system is NULL");
    if (s->bc != REACH_BC_DEFAULT)
        return fail(c, REACH_E_UNSUPPORTED, "bc = %d: only each kind's own boundary conditions "
                    "(REACH_BC_DEFAULT) are built", s->bc);
    if (s->kind == REACH_USER && !user)
        return fail(c, REACH_E_INVAL, "REACH_USER systems run through reach_embed_rk4_user");
    if (s->kind != REACH_CTM && s->kind != REACH_RD && s->kind != REACH_LIN3 &&
        s->kind != REACH_HEAT3D && s->kind != REACH_USER)
        return fail(c, REACH_E_INVAL, "unknown system kind %d", s->kind);
    if (user && s->kind != REACH_USER)
        return fail(c, REACH_E_INVAL, "reach_embed_rk4_user takes a REACH_USER system");
    if (dtype != REACH_F64 && dtype != REACH_F32) return fail(c, REACH_E_INVAL, "bad dtype %d", dtype);
    if (s->n < 1 || s->n >= kMaxN) return fail(c, REACH_E_INVAL, "n = %lld out of range", (long long)s->n);
    if (s->n_in != 0 && s->n_in != 1 && s->n_in != s->n)
        return fail(c, REACH_E_INVAL, "n_in must be 0, 1 or n");
    if (s->kind == REACH_CTM && s->n_in != 0)
        return fail(c, REACH_E_UNSUPPORTED, "the CTM chain takes no inputs");
    for (int i = 0; i < 8; ++i)
        if (!std::isfinite(s->prm[i])) return fail(c, REACH_E_INVAL, "parameter %d not finite", i);
    if (s->kind == REACH_RD && !(s->prm[0] > 0.0)) return fail(c, REACH_E_INVAL, "RD spacing h must be > 0");
    if (s->kind == REACH_HEAT3D) {
        if (s->n_in != 0) return fail(c, REACH_E_UNSUPPORTED, "the 3-D heat grid takes no inputs");
        int64_t prod = 1;
        for (int d = 0; d < 3; ++d) {
            const double g = s->prm[d];
            if (!(g >= 1.0 && g < 2147483648.0 && g == std::floor(g)))
                return fail(c, REACH_E_INVAL, "heat grid extent %d must be an integer in [1, 2^31)", d);
            prod *= (int64_t)g;
            if (prod > s->n) break;
        }
        if (prod != s->n) return fail(c, REACH_E_INVAL, "n must equal nx * ny * nz");
        if (!(s->prm[3] >= 0.0)) return fail(c, REACH_E_INVAL, "heat diffusivity must be >= 0");
        if (!(s->prm[4] > 0.0)) return fail(c, REACH_E_INVAL, "heat grid spacing must be > 0");
    }
    return REACH_OK;
}

reach_status check_system(reach_ctx* c, const reach_system* s, reach_dtype dtype) {
    return check_system_kind(c, s, dtype, false);
}

// Steps of every launch that only the chain kernels implement.
reach_status chains_only(reach_ctx* c, const reach_system* s, const char* what) {
    if (s->kind == REACH_HEAT3D)
        return fail(c, REACH_E_UNSUPPORTED, "%s runs the chain systems only", what);
    return REACH_OK;
}

void kernel_prm(const reach_system* s, double out[5]) { kernel_params(s->kind, s->prm, out); }

// Whether [p, p + np) and [q, q + nq) share a byte (p may be NULL).
bool overlaps(const void* p, size_t np, const void* q, size_t nq) {
    return p && (const char*)p < (const char*)q + nq && (const char*)q < (const char*)p + np;
}

int ceil_pow2_E(int64_t n) {
    int E = 1;
    while ((int64_t)64 * E < n) E *= 2;
    return E;
}

// ------------------------------------------------------------ planning --
struct EmbedPlan {
    int E = 1;
    int S = 2;           // sides per wave
    int K = 1;           // steps per pass
    int64_t W = 1;       // tiles
    int64_t OUT = 0;
    int H = 0;
    int64_t passes = 1;
    bool cut_one = false;   // several windows although one holds the chain
};

// Defaults measured on MI355X for the 2^26-cell chains (overridden by the
// autotuner or its cache).  Cooperative chains run one side per wave.
// Measured defaults per system, dtype, input mode (cell_in: per-cell inputs)
// and size.
TuneEntry default_tune(int kind, int dtype, bool cell_in, int64_t n) {
    if (kind == REACH_HEAT3D) return TuneEntry{2, 1, 1};   // rows per wave, 16 waves per block
    // LIN3, 2^24 cells, us per step: FP64 per-cell inputs 43.2 at 12 cells (over
    // 256 VGPRs there) and 32.1 at 8, scalar 29.0 at 12 and 30.8 at 8; FP32
    // scalar 22.5 at 16 and 23.4 at 12, per-cell 23.9 and 23.4
    if (kind == REACH_LIN3) {
        if (dtype == REACH_F64) return cell_in ? TuneEntry{8, 10, 2} : TuneEntry{12, 12, 2};
        return cell_in ? TuneEntry{12, 10, 2} : TuneEntry{16, 12, 2};
    }
    // FP32 instructions of different waves overlap, so three waves per SIMD at
    // 32 cells beat two at 48: CTM 2^27 153 against 175 us per step, RD 2^25 37.4
    // against 43.3 (per-cell inputs: 41.4 at 24, 42.7 at 32)
    if (dtype == REACH_F32) return cell_in ? TuneEntry{24, 12, 1} : TuneEntry{32, 12, 1};
    // RD with shared inputs fits 28 cells per lane in 256 VGPRs (the CTM
    // chain and per-cell inputs need more there).  The wider tile pays on
    // long chains (2^26: 1.5% faster); below that its fewer waves leave a
    // larger share of the last round empty (2^24: 5% slower than 24).
    if (kind == REACH_RD && !cell_in && n >= ((int64_t)1 << 26)) return TuneEntry{28, 24, 1};
    return TuneEntry{24, 20, 1};
}
int n_bucket(int64_t n) {
    int b = 0;
    while (((int64_t)1 << (b + 1)) <= n) ++b;
    return b;
}

TuneEntry tuned(const reach_ctx* c, int kind, int dtype, int64_t n, bool cell_in) {
    auto it = c->tune.find({kind, dtype, n_bucket(n), cell_in ? 1 : 0});
    if (it != c->tune.end()) return it->second;
    return default_tune(kind, dtype, cell_in, n);
}

int smallest_E(int kind, int dtype, int S, int64_t n) {
    for (int E : {1, 2, 4, 6, 8, 12, 16, 20, 24, 28, 32, 48, 64})
        if (embed_has_shape(kind, dtype, E, S) && (int64_t)64 * E >= n) return E;
    return 0;
}

// A multi-window plan's windows: steps per pass K, halo, stride, count.
void set_windows(EmbedPlan* p, int E, int S, int64_t K, int64_t n, int64_t nsteps) {
    const int64_t span = (int64_t)64 * E;
    p->E = E;
    p->S = S;
    p->K = (int)K;
    p->H = (int)(4 * K);
    p->OUT = span - 2 * p->H;
    p->W = (n <= span) ? 1 : 1 + (n - span + p->OUT - 1) / p->OUT;
    p->passes = (nsteps + K - 1) / K;
}

// Issue time of one cell and RK4 step (both sides for S = 2) of a lane of E cells.
double cell_us(int kind, int dtype, bool cell_in, int S, int E, bool* over) {
    const bool f64 = dtype == REACH_F64;
    const int wide = S == 2 ? (f64 ? (cell_in ? 8 : 12) : 16)
                            : (f64 ? (cell_in ? 24 : 28) : 48);
    *over = E > wide;
    const double c = kind == REACH_LIN3 ? 0.0765 : kind == REACH_RD ? 0.0438 : f64 ? 0.051 : 0.040;
    return *over ? c * (S == 2 ? 2.0 : 1.2) : c;   // register moves
}

// Estimated time of one RK4 step (microseconds) of a chain whose windows do not
// fill the chip several times over, at E cells per lane and K steps per pass
// (measured on MI355X, chains of 12000 to 10^6 cells):
//   - a wave with its SIMD to itself takes c E + 0.06 us per step, c the issue
//     time of one cell (both sides for S = 2); the launch waits for the SIMDs
//     that hold the most waves, so r waves cost r c E;
//   - every pass costs 2.5 us of launch, first loads and last stores, plus the
//     reading and writing of the state at 7 TB/s (the waves of so few rounds
//     load, compute and store at the same time, so this is not hidden).
// Windows of more than 256 registers run one to a SIMD; they count only where
// no SIMD gets a second one.
double step_us(int kind, int dtype, bool cell_in, int S, int E, int64_t K, int64_t n,
               int64_t simds) {
    const int64_t span = (int64_t)64 * E;
    if (8 * K >= span) return 1e300;
    const int64_t OUT = span - 8 * K;
    const int64_t W = n <= span ? 1 : 1 + (n - span + OUT - 1) / OUT;
    const int64_t r = ((S == 1 ? 2 : 1) * W + simds - 1) / simds;
    bool over = false;
    const double c = cell_us(kind, dtype, cell_in, S, E, &over);
    if (over && r > 1) return 1e300;
    const double bytes = (double)n * (dtype == REACH_F64 ? 8.0 : 4.0) * (cell_in ? 6.0 : 4.0);
    return (double)r * c * E + 0.06 + (2.5 + bytes / 7.0e6) / (double)K;
}

// Steps of a run that, not in place, never needs the workspace: one pass of the
// default windows (and of those that per-cell LIN3 inputs took at 12 cells a lane).
int64_t one_pass_steps(int kind, int dtype, bool cell_in, int64_t n) {
    return std::max(12, default_tune(kind, dtype, cell_in, n).K);
}

// The shape of the least estimated step time, at K steps per pass (K = 0: the
// best K as well, up to 64), among the embedding's shapes or (gb) the growth
// bound's.  A chain of several windows takes no smaller K than one_pass_steps, so
// that what one pass of the default windows did stays one pass, which leaves the
// workspace alone (200003 RD cells, FP64: 0.667 us a step at K = 47 for 0.638 at 15).
TuneEntry fastest_shape(reach_ctx* c, int kind, int dtype, bool cell_in, int64_t n, int64_t K,
                        bool gb = false) {
    const int64_t simds = (int64_t)4 * c->cus;
    const int flags = (cell_in ? 1 : 0) | (gb ? 2 : 0);
    {
        std::lock_guard<std::mutex> lk(c->shapes.m);
        for (const ShapeMemo::Slot& m : c->shapes.slot)
            if (m.n == n && m.K == K && m.kind == kind && m.dtype == dtype && m.flags == flags)
                return m.t;
    }
    const int S = kind == REACH_LIN3 ? 2 : 1;
    const int64_t least =
        gb || smallest_E(kind, dtype, S, n) ? 4 : one_pass_steps(kind, dtype, cell_in, n);
    TuneEntry best{0, 0, S};
    double t_best = 1e300;
    for (int E : {1, 2, 4, 6, 8, 12, 16, 20, 24, 28, 32, 48, 64}) {
        if (gb ? !gb_has_E(E) : !embed_has_shape(kind, dtype, E, S)) continue;
        const int64_t top = std::min<int64_t>(64, 8 * E - 1);
        for (int64_t k = K ? K : least; k <= (K ? K : top); ++k) {
            const double t = step_us(kind, dtype, cell_in, S, E, k, n, simds);
            if (t < t_best) { t_best = t; best.E = E; best.K = (int)k; }
        }
    }
    std::lock_guard<std::mutex> lk(c->shapes.m);
    ShapeMemo::Slot& m = c->shapes.slot[c->shapes.next];
    c->shapes.next = (c->shapes.next + 1) % 16;
    m.n = n; m.K = K; m.kind = kind; m.dtype = dtype; m.flags = flags; m.t = best;
    return best;
}

// Estimated time of a run in the one window of E cells a lane that holds the chain.
// Padding costs the LIN3 chain's selects a third (at 16 cells a lane its moves are
// fewer than cell_us says), the others a few percent (measured, us a step, FP64 RD:
// 4 cells 0.254, 8 0.454, 12 0.581, 16 0.746, 32 1.80; FP64 CTM: 4 0.276, 8 0.515; FP32
// CTM: 4 0.202, 16 0.693, 32 1.31, 64 3.62; FP64 LIN3: 4 0.500, 8 0.912, 12 1.33, 16 1.75).
double one_window_us(int kind, int dtype, bool cell_in, int S, int E, int64_t n, int64_t nsteps) {
    bool over = false;
    const double step = cell_us(kind, dtype, cell_in, S, E, &over) * E + 0.06;
    const double pad = n == (int64_t)64 * E ? 1.0 : S == 2 ? (over ? 0.7 : 1.36) : 1.05;
    return 2.5 + (double)nsteps * step * pad;
}

// Whether a chain that one window holds is cut into several, whose run is estimated
// to take many_us (hold: in CutScratch, whose event takes 3 us of a call).  A call
// alone gains wherever that is less, but one window leaves the chip to other
// streams' calls, of which four run at once, while a cut chain's passes are launches
// of about 3 us for the host: with 8 streams a call of 100 steps takes, in one
// window and cut, 30 and 18 us at 1000 RD cells (79 and 31 alone), 24 and 24 at 700
// (62 and 28), and 11 and 19 at 130 (28 and 30).  So it has to gain more than half
// as much again alone, and its passes have to keep up with four windows at a time.
bool cut_pays(double one_us, double many_us, int64_t passes, bool hold) {
    if (hold) many_us += 3.0;
    return 1.6 * many_us <= one_us &&
           (passes == 1 || one_us >= 7.0 * (double)passes + (hold ? 5.0 : 0.0));
}

// A second block of two waves on a compute unit lands on the SIMDs of the first
// while the other two stay idle: W such blocks, one window each, take up to 1.65
// times as long as blocks of one wave where they are more than the compute units
// and at most twice as many (growth bound, 8 FP64 RD cells a lane, 200 steps: 256
// windows 100 us, 284 166 in blocks of two and 102 of one, 512 167 and 122, 520 168 and
// 168; with more windows than that blocks of two are up to 15% faster).
bool pairs_share(const reach_ctx* c, int64_t W) { return W > c->cus && W <= 2 * (int64_t)c->cus; }

// Whether a last pass of W FP64 windows of E cells a lane and `steps` steps does better
// in blocks of one wave, its two sides brought together by a kernel of its own that
// moves `bytes` (FP32 instructions of two waves on a SIMD overlap: no gain there).  At two
// waves per SIMD a second round of windows ends alike (`rounds`; RD, 20 steps: 500000
// cells, 446 windows, 39 us in blocks of two and 27 with the check apart; 2 * 10^6 cells,
// 1454 windows, 92 and 78).
bool part_last_pass(const reach_ctx* c, int kind, int dtype, bool cell_in, int64_t W, int E,
                    int64_t steps, double bytes, bool rounds) {
    const int64_t round = (int64_t)4 * c->cus;
    const int64_t rest = rounds && W < 2 * round ? W % round : W;
    bool over = false;
    const double step = 0.8 * cell_us(kind, dtype, cell_in, 1, E, &over) * E;
    return dtype == REACH_F64 && !over && pairs_share(c, rest) &&
           step * (double)steps > 2.5 + bytes / 5.0e6;
}

// Blocks of the kernel that brings two sides together: as many as keep a large sweep
// busy, but behind waves that had a SIMD each no more than find a place at once.  After
// 2048 blocks or more the next kernel's waves share SIMDs again (20 steps, 24 FP64 RD cells
// a lane, one call behind another: 400 windows 50 us, 31 behind 1024 blocks).
constexpr int64_t kSweepBlocks = 8192, kPartBlocks = 1024;

// The estimate decides on chains whose default windows put at most 8 waves on a
// SIMD; longer ones keep the shapes measured at 2^26 and 2^31 cells (there the
// rounds run into each other and the last one weighs little).
bool estimated(int kind, int dtype, bool cell_in, int64_t n, int64_t simds) {
    const TuneEntry d = default_tune(kind, dtype, cell_in, n);
    const int64_t OUT = (int64_t)64 * d.E - 8 * d.K;
    return (d.S == 1 ? 2 : 1) * (n / OUT) <= 8 * simds;
}

// Runs of at most this many steps keep a chain that one window holds in one
// window (one launch): splitting it would save a few microseconds.
// A tube of many short runs does split it, and so does the LIN3 chain, whose wave
// holds both sides (n = 1000, 8 steps: 23 us in one window, 16 in several).
constexpr int64_t kSplitSteps = 8;

// Default shape of a multi-window run of many steps.
TuneEntry default_shape(reach_ctx* c, int kind, int dtype, bool cell_in, int64_t n) {
    const int64_t simds = (int64_t)4 * c->cus;
    if (kind != REACH_HEAT3D && estimated(kind, dtype, cell_in, n, simds)) {
        const TuneEntry t = fastest_shape(c, kind, dtype, cell_in, n, 0);
        if (t.E) return t;
    }
    return default_tune(kind, dtype, cell_in, n);
}

// have_ws: the caller has the workspace of a multi-pass run, so that a chain of
// several windows may be cut into more of them, and more passes, than the fewest;
// cut_one: a chain that one window holds may be cut (its passes run in CutScratch);
// one_steps: the longest run that keeps such a chain in that window.
reach_status plan_embed(reach_ctx* c, const reach_system* s, reach_dtype dtype, int64_t nsteps,
                        EmbedPlan* p, bool have_ws = true, bool cut_one = true,
                        int64_t one_steps = kSplitSteps) {
    const int64_t n = s->n;
    const bool cell_in = s->n_in > 1;
    const int64_t oE = opt_get(c, "embed.E"), oK = opt_get(c, "embed.K"), oS = opt_get(c, "embed.S");
    const int64_t simds = (int64_t)4 * c->cus;
    // (a tuned shape is for the chains of its bucket that no single window holds)
    const bool is_tuned =
        !c->tune.empty() && c->tune.count({s->kind, dtype, n_bucket(n), cell_in ? 1 : 0}) != 0;
    // (up to two cells per lane one window is always the better one)
    if ((have_ws || cut_one) && n > 128 && !oE && !oK && !oS &&
        estimated(s->kind, dtype, cell_in, n, simds)) {
        const int one = smallest_E(s->kind, dtype, s->kind == REACH_LIN3 ? 2 : 1, n);
        if (one ? cut_one && nsteps > (s->kind == REACH_LIN3 ? 1 : one_steps)
                : have_ws && !is_tuned) {
            // the best K for many steps gives the pass count; the steps are
            // spread evenly over the passes, and the shape is the best for those
            const TuneEntry t = fastest_shape(c, s->kind, dtype, cell_in, n, 0);
            const int64_t steps = std::max<int64_t>(nsteps, 1);
            const int64_t passes = (steps + t.K - 1) / t.K;
            const int64_t K = (steps + passes - 1) / passes;
            const TuneEntry u = fastest_shape(c, s->kind, dtype, cell_in, n, K);
            const double many_us =
                (double)steps * step_us(s->kind, dtype, cell_in, t.S, u.E, K, n, simds);
            // (a tube's slots share one hold on the scratch)
            if (u.E && (!one || cut_pays(one_window_us(s->kind, dtype, cell_in, t.S, one, n, steps),
                                         many_us, passes, passes > 1 && one_steps == kSplitSteps))) {
                set_windows(p, u.E, u.S, K, n, nsteps);
                p->cut_one = one != 0;
                if (p->W > 1) return REACH_OK;
            }
        }
    }
    p->cut_one = false;
    const TuneEntry te = tuned(c, s->kind, dtype, n, cell_in);
    int S = oS ? (int)oS : (oE ? (s->kind == REACH_LIN3 ? 2 : te.S) : te.S);
    if (s->kind == REACH_LIN3 && S == 1)
        return fail(c, REACH_E_INVAL, "the coupled LIN3 chain needs both sides per wave");
    int E = oE ? (int)oE : 0;
    if (E && !embed_has_shape(s->kind, dtype, E, S))
        return fail(c, REACH_E_INVAL, "tile shape E = %d, S = %d not built", E, S);
    if (!E) {
        const int small = smallest_E(s->kind, dtype, S, n);
        E = (small && !oK) ? small : te.E;
        if (!embed_has_shape(s->kind, dtype, E, S)) E = embed_max_E(dtype, S);
    }
    p->E = E;
    p->S = S;
    const int64_t span = (int64_t)64 * E;
    if (n <= span && !oK) {
        // one window covers the chain: both ends are true boundaries, no halo
        p->K = (int)std::min<int64_t>(std::max<int64_t>(nsteps, 1), INT32_MAX);
        p->W = 1; p->OUT = 0; p->H = 0;
        p->passes = nsteps > 0 ? 1 : 0;
        return REACH_OK;
    }
    int K = oK ? (int)oK : te.K;
    if (K < 1) K = 1;
    // (per-cell LIN3 inputs: runs of more steps than the default pass that need
    // no workspace)
    if (!oK && !is_tuned && nsteps > K &&
        nsteps <= one_pass_steps(s->kind, dtype, cell_in, n) && 8 * nsteps < span)
        K = (int)nsteps;
    if ((int64_t)8 * K >= span) return fail(c, REACH_E_INVAL, "K = %d too large for E = %d", K, E);
    if (!oK && nsteps > 0) {
        // the same number of passes with the steps spread evenly: a smaller
        // halo (e.g. 100 steps at K = 24 run as 5 passes of 20, not 4 x 24 + 4)
        const int64_t passes = (nsteps + K - 1) / K;
        K = (int)((nsteps + passes - 1) / passes);
    }
    set_windows(p, E, S, K, n, nsteps);
    return REACH_OK;
}

// ------------------------------------------------------------ 3-D heat --
struct HeatPlan {
    int P = 4, WV = 8;        // rows per wave, waves per block
    int OX = 0, OY = 0;       // output cells of a tile along x / y
    int64_t TX = 0, TY = 0;   // tiles per side along x / y
    int64_t ZC = 1, LZ = 0;   // z chunks per tile, output planes of a chunk (ZC = 1: all)
};

// The waves per block and the z chunks of a grid at 2 rows per wave.  A launch takes
// about rounds * iterations: rounds of `cus` blocks, and iterations in groups of 6, of
// LZ planes plus 4 for the pipeline and, when cut, 4 halo planes before the chunk
// (those behind it are read while the pipeline drains); the start costs about 9 more.
// An iteration of 12 or 8 waves takes 0.82 or 0.64 of one of 16 (measured: 0.66,
// 0.55 and 0.42 us FP32, 0.95, 0.77 and 0.60 FP64), for 16 or 8 output rows
// instead of 24: the narrower blocks pay where the grid is too small to occupy the
// chip with wide ones (at most 4 rounds: 600 x 600 x 25 FP32 takes 80 us with 8 waves in
// 7 rounds, 75 with 16 in 3).  Two FP32 blocks of 8 waves share a compute unit and
// then take 1.53 times one's time instead of twice.
//
// The uncut sweep of 16 waves stays unless the best is 10% shorter by that count: a
// launch of many rounds is bound by memory, where the halo planes cost more than
// the last round's idle units (1000^3: 5.9 rounds, uncut).  Measured per step, FP32 / FP64:
//                      uncut        16 waves, cut   12 waves        8 waves
//   40^3                              14 / 18       12 / 15          9.4 / 12
//   100^3              79 / 115       19 / 27       19 / 25         20 / 27
//   200 x 180 x 150   105 / 151       40 / 64       51 / 74         54 / 98
// (the FP64 kernel of 16 waves spills in its cut instance, 4 to 11 scratch accesses
// per six planes, which these figures hold)
void heat_z_chunks(int64_t nx, int64_t ny, int64_t nz, bool f64, int64_t cus, HeatPlan* p) {
    double best = 0.0;
    for (const int WV : {16, 12, 8}) {
        const int64_t OX = 64 - 8, OY = HEAT_CUT_ROWS * WV - 8;
        const int64_t TX = (nx + OX - 1) / OX, TY = (ny + OY - 1) / OY;
        const double it = WV == 16 ? 1.0 : WV == 12 ? 0.82 : 0.64;
        for (int64_t want = 1; want == 1 || want <= std::min<int64_t>(nz / 4, 256); ++want) {
            const int64_t LZ = want == 1 ? nz : std::max<int64_t>(4, (nz + want - 1) / want);
            const int64_t ZC = (nz + LZ - 1) / LZ;
            const int64_t planes = LZ + 4 + (ZC > 1 ? 4 : 0);
            const int64_t r = (2 * TX * TY * ZC + cus - 1) / cus;
            if (WV < 16 && r > 4) break;   // (more chunks only add rounds)
            const double rounds = !f64 && WV == 8 ? 1.0 + 0.53 * (double)(r - 1) : (double)r;
            const double t = it * rounds * (double)(6 * ((planes + 5) / 6) + 9);
            if (WV == 16 && want == 1) best = 0.9 * t;   // the plan as it stands
            else if (t < best) {
                best = t;
                p->WV = WV; p->OY = (int)OY; p->TY = TY;
                p->ZC = ZC; p->LZ = LZ;
            }
        }
    }
}

// Level j of a step: w <- y + cw[j] (s - 6 w), cw[j] = a dt / (4 - j)
// (the RK4 stability polynomial in nested form, see the heat kernel).
void heat_level_constants(HeatPass* a) {
    for (int l = 0; l < 4; ++l) {
        const double cl = a->a * a->dt / (double)(4 - l);
        a->cw[l] = cl;
        a->m6cw[l] = -6.0 * cl;
        a->cwf[l] = (float)cl;
        a->m6cwf[l] = (float)(-6.0 * cl);
    }
}

int heat_waves(int P) {
    return P == 4 ? 8 : P == 5 ? 8 : P == 2 ? 16 : P == 8 ? 4 : P == 3 ? 12 : 0;
}

reach_status plan_heat(reach_ctx* c, const reach_system* s, reach_dtype dtype, HeatPlan* p) {
    int P = (int)opt_get(c, "heat.P");
    if (!P) P = tuned(c, REACH_HEAT3D, dtype, s->n, false).E;
    const int WV = heat_waves(P);
    if (!WV || !heat_has_shape(dtype == REACH_F64 ? 0 : 1, P, WV))
        return fail(c, REACH_E_INVAL, "heat.P = %d not built for this dtype", P);
    p->P = P;
    p->WV = WV;
    p->OX = 64 - 8;
    p->OY = WV * P - 8;
    const int64_t nx = (int64_t)s->prm[0], ny = (int64_t)s->prm[1];
    p->TX = (nx + p->OX - 1) / p->OX;
    p->TY = (ny + p->OY - 1) / p->OY;
    p->LZ = (int64_t)s->prm[2];
    if (P == HEAT_CUT_ROWS) heat_z_chunks(nx, ny, p->LZ, dtype == REACH_F64, c->cus, p);
    return REACH_OK;
}

// Which buffer each of `passes` passes reads and writes: 0 = x, 1 = r,
// 2 = workspace.  The last pass writes r unless r aliases x and the pass
// count makes the ping-pong end in the workspace (then final_copy).  Computed per
// pass: a long run of a short chain has millions of them.
struct PassIo {
    int64_t passes;
    bool inplace;      // every pass reads and writes r (the first reads x)
    bool ws_first;     // the ping-pong starts in the workspace
    PassIo(int64_t n, bool inplace_ok, bool alias)
        : passes(n), inplace(inplace_ok), ws_first(!inplace_ok && alias && n % 2 == 1) {}
    int dst(int64_t p) const {
        if (inplace) return 1;
        return (ws_first ? p % 2 == 1 : (passes - 1 - p) % 2 == 0) ? 1 : 2;
    }
    int src(int64_t p) const { return p ? dst(p - 1) : 0; }
    bool final_copy() const { return passes > 0 && dst(passes - 1) == 2; }
};

reach_status embed_heat3d(reach_ctx* c, const reach_system* s, reach_dtype dtype,
                          const void* x_lo, const void* x_hi, double dt, int64_t nsteps,
                          void* r_lo, void* r_hi, void* ws, size_t ws_bytes, hipStream_t hs) {
    HeatPlan hp;
    reach_status st = plan_heat(c, s, dtype, &hp);
    if (st != REACH_OK) return st;
    log_call(c, "\"call\": \"embed\", \"kind\": %d, \"dtype\": \"%s\", \"n\": %lld, "
                "\"nsteps\": %lld, \"rows_per_wave\": %d, \"tiles\": %lld, \"passes\": %lld",
             s->kind, dtype_name(dtype), (long long)s->n, (long long)nsteps, hp.P,
             (long long)(2 * hp.TX * hp.TY * hp.ZC), (long long)nsteps);
    const size_t bytes = (size_t)s->n * dsize(dtype);
    const bool alias = (r_lo == x_lo) || (r_hi == x_hi) || (r_lo == x_hi) || (r_hi == x_lo);
    const int64_t passes = nsteps;   // one RK4 step per pass
    const bool need_ws = passes >= 2 || alias;
    void *w_lo = nullptr, *w_hi = nullptr;
    if (need_ws) {
        if (!ws || ws_bytes < 2 * bytes)
            return fail(c, REACH_E_INVAL, "workspace of %zu bytes needed", 2 * bytes);
        w_lo = ws;
        w_hi = (char*)ws + bytes;
    }
    const PassIo io(passes, false, alias);
    const void* lo_of[3] = {x_lo, r_lo, w_lo};
    const void* hi_of[3] = {x_hi, r_hi, w_hi};
    HeatPass a{};
    a.nx = (int64_t)s->prm[0]; a.ny = (int64_t)s->prm[1]; a.nz = (int64_t)s->prm[2];
    a.TX = (int32_t)hp.TX; a.TY = (int32_t)hp.TY; a.OX = hp.OX; a.OY = hp.OY;
    a.sides = 2;
    a.ZC = hp.ZC; a.LZ = hp.LZ;
    const int64_t tiles = 2 * hp.TX * hp.TY * hp.ZC;
    a.per_xcd = (int32_t)((tiles + 7) / 8);
    a.a = s->prm[3] / (s->prm[4] * s->prm[4]);
    a.h2 = dt / 2.0; a.dt = dt; a.dt6 = dt / 6.0;
    heat_level_constants(&a);
    a.status = c->status;
    const int64_t grid = 8 * (int64_t)a.per_xcd;
    const int dt_id = dtype == REACH_F64 ? 0 : 1;
    for (int64_t p = 0; p < passes; ++p) {
        a.src[0] = lo_of[io.src(p)];
        a.src[1] = hi_of[io.src(p)];
        a.dst[0] = (void*)lo_of[io.dst(p)];
        a.dst[1] = (void*)hi_of[io.dst(p)];
        hipError_t e = launch_heat3d(dt_id, hp.P, hp.WV, a, grid, hs);
        if (e != hipSuccess) return hip_fail(c, e, "3-D heat kernel launch");
    }
    hipError_t e = launch_order_check(dt_id, lo_of[io.dst(passes - 1)], hi_of[io.dst(passes - 1)],
                                      s->n, c->status, kSweepBlocks, hs);
    if (e != hipSuccess) return hip_fail(c, e, "order check launch");
    if (io.final_copy()) {
        HIPCHK(c, hipMemcpyAsync(r_lo, w_lo, bytes, hipMemcpyDeviceToDevice, hs));
        HIPCHK(c, hipMemcpyAsync(r_hi, w_hi, bytes, hipMemcpyDeviceToDevice, hs));
    }
    return REACH_OK;
}

// Growth bound of the heat grid: the system is linear with non-negative
// couplings, so its own matrix is a contraction matrix and the half-width
// follows the heat equation too; both runs share each launch.
reach_status gb_heat3d(reach_ctx* c, const reach_system* s, reach_dtype dtype, const void* x_lo,
                       const void* x_hi, double dt, int64_t nsteps, void* r_lo, void* r_hi,
                       void* ws, hipStream_t hs) {
    HeatPlan hp;
    reach_status st = plan_heat(c, s, dtype, &hp);
    if (st != REACH_OK) return st;
    log_call(c, "\"call\": \"growth_bound\", \"kind\": %d, \"dtype\": \"%s\", \"n\": %lld, "
                "\"nsteps\": %lld, \"rows_per_wave\": %d, \"tiles\": %lld, \"passes\": %lld",
             s->kind, dtype_name(dtype), (long long)s->n, (long long)nsteps, hp.P,
             (long long)(2 * hp.TX * hp.TY * hp.ZC), (long long)nsteps);
    const size_t bytes = (size_t)s->n * dsize(dtype);
    const int dt_id = dtype == REACH_F64 ? 0 : 1;
    char* A = (char*)ws;
    char* B = (char*)ws + 2 * bytes;
    hipError_t e = launch_center_radius(dt_id, x_lo, x_hi, s->n, B, B + bytes, hs);
    if (e != hipSuccess) return hip_fail(c, e, "center / radius launch");
    HeatPass a{};
    a.nx = (int64_t)s->prm[0]; a.ny = (int64_t)s->prm[1]; a.nz = (int64_t)s->prm[2];
    a.TX = (int32_t)hp.TX; a.TY = (int32_t)hp.TY; a.OX = hp.OX; a.OY = hp.OY;
    a.sides = 2;
    a.ZC = hp.ZC; a.LZ = hp.LZ;
    const int64_t tiles = 2 * hp.TX * hp.TY * hp.ZC;
    a.per_xcd = (int32_t)((tiles + 7) / 8);
    a.a = s->prm[3] / (s->prm[4] * s->prm[4]);
    a.h2 = dt / 2.0; a.dt = dt; a.dt6 = dt / 6.0;
    heat_level_constants(&a);
    a.status = c->status;
    const int64_t grid = 8 * (int64_t)a.per_xcd;
    char* cur = B;
    for (int64_t p = 0; p < nsteps; ++p) {
        char* dst = (cur == A) ? B : A;
        a.src[0] = cur; a.src[1] = cur + bytes;
        a.dst[0] = dst; a.dst[1] = dst + bytes;
        e = launch_heat3d(dt_id, hp.P, hp.WV, a, grid, hs);
        if (e != hipSuccess) return hip_fail(c, e, "3-D heat kernel launch");
        cur = dst;
    }
    e = launch_gb_combine(dt_id, cur, cur + bytes, s->n, r_lo, r_hi, c->status, kSweepBlocks, hs);
    if (e != hipSuccess) return hip_fail(c, e, "growth-bound combine launch");
    return REACH_OK;
}

void save_tune_entry(const reach_ctx* c, int kind, int dtype, int bucket, int cell_in, TuneEntry t,
                     double ps);

// Times every built (rows, waves) shape of the heat kernel, keeps the fastest.
reach_status autotune_heat3d(reach_ctx* c, const reach_system* s, reach_dtype dtype,
                             const void* x_lo, const void* x_hi, double dt, int64_t trial_steps,
                             void* r_lo, void* r_hi, void* ws, size_t ws_bytes, hipStream_t hs,
                             int64_t* best) {
    const int64_t saveP = opt_get(c, "heat.P");
    hipEvent_t e0, e1;
    HIPCHK(c, hipEventCreate(&e0));
    HIPCHK(c, hipEventCreate(&e1));
    double best_ps = 1e300;
    int bestP = 0;
    reach_status st = REACH_OK;
    for (int P : {2, 3, 4, 5, 8}) {
        if (!heat_has_shape(dtype == REACH_F64 ? 0 : 1, P, heat_waves(P))) continue;
        c->opt["heat.P"] = P;
        st = embed_heat3d(c, s, dtype, x_lo, x_hi, dt, trial_steps, r_lo, r_hi, ws, ws_bytes, hs);
        if (st != REACH_OK) break;
        if (hipEventRecord(e0, hs) != hipSuccess) { st = REACH_E_DEVICE; break; }
        for (int rep = 0; rep < 2 && st == REACH_OK; ++rep)
            st = embed_heat3d(c, s, dtype, x_lo, x_hi, dt, trial_steps, r_lo, r_hi, ws, ws_bytes,
                              hs);
        if (st != REACH_OK) break;
        if (hipEventRecord(e1, hs) != hipSuccess || hipEventSynchronize(e1) != hipSuccess) {
            st = REACH_E_DEVICE;
            break;
        }
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, e0, e1) != hipSuccess) { st = REACH_E_DEVICE; break; }
        const double ps = (double)ms * 1e9 / (2.0 * 2.0 * (double)s->n * (double)trial_steps);
        if (ps < best_ps) { best_ps = ps; bestP = P; }
    }
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    c->opt["heat.P"] = saveP;
    if (st != REACH_OK) return st;
    const int bucket = n_bucket(s->n);
    const TuneEntry bt{bestP, 1, 1};
    c->tune[{s->kind, dtype, bucket, 0}] = bt;
    save_tune_entry(c, s->kind, dtype, bucket, 0, bt, best_ps);
    best[0] = bestP;
    best[1] = 1;
    best[2] = (int64_t)std::llround(best_ps * 1000.0);
    best[3] = 1;
    return REACH_OK;
}

size_t embed_ws_bytes(reach_ctx* c, const reach_system* s, reach_dtype dtype) {
    if (s->kind == REACH_HEAT3D) return (size_t)2 * (size_t)s->n * dsize(dtype);
    EmbedPlan p;
    if (plan_embed(c, s, dtype, (int64_t)1 << 20, &p, true, false) != REACH_OK) return (size_t)-1;
    if (p.W == 1) return 0;
    return (size_t)2 * (size_t)s->n * dsize(dtype);
}

// ------------------------------------------------------------- Monte Carlo
int mc_E(int dtype, int64_t n) {
    const int E = ceil_pow2_E(n);
    return E <= mc_max_E(dtype) ? E : -1;
}

int64_t mc_waves(const reach_ctx* c, int64_t m) {
    int64_t w = opt_get(c, "mc.waves");
    if (w <= 0) w = (int64_t)c->cus * 8;
    return std::max<int64_t>(1, std::min<int64_t>(std::min(w, kMcMaxWaves), m));
}

// Room for one partial of 64 E values per wave; the kernel writes one of n values
// per workgroup of kMcWavesPerGroup waves, so every plan of mc_plan fits.
size_t mc_ws_bytes(const reach_ctx* c, const reach_system* s, reach_dtype dtype, int64_t m) {
    const int E = mc_E(dtype, s->n);
    if (E < 0) return (size_t)-1;
    return (size_t)2 * (size_t)mc_waves(c, m) * (size_t)(64 * E) * dsize(dtype);
}

struct McPlan {
    int E = 1;
    int L = 0;          // lanes of a sample (segment layout), 0: plain layout
    int spw = 1;        // samples per wave
    int64_t nw = 1;     // resident waves
};

// Cells per lane and samples per wave by the least estimated time, in issued
// instructions per SIMD: a stage costs c E and a fixed part (lane shifts, and
// in the segment layout the boundary selects), a sample's draws one Philox
// block (about 440 instructions' time) per four cells.  A sample spread thin (one
// cell per lane) has the shortest chain of stages, which decides while each SIMD
// has at most one wave; with more samples the fixed part counts, and wide lanes
// with several samples to a wave are cheaper (CTM FP64 n = 64, 13000 samples:
// 8 cells per lane and 8 samples per wave).
McPlan mc_plan(const reach_ctx* c, int kind, int dtype, bool cell_in, int64_t n, int64_t m,
               int64_t nsteps) {
    const double simds = 4.0 * c->cus;
    const bool f64 = dtype == 0;
    const double cc = kind == REACH_CTM && f64 ? 6.75 : 5.75;
    const double word = f64 ? 2.0 : 1.0;   // registers a lane shift or a select moves
    McPlan best;
    double t_best = 1e300;
    for (int E = 1; E <= mc_max_E(dtype); ++E) {
        const int64_t L = (n + E - 1) / E;
        if (L > 64) continue;
        const bool plain = n == 64 * E && mc_has_plain(dtype, E);
        if (!plain && !(mc_has_segments(dtype, E) && n >= (int64_t)(E - 1) * L)) continue;
        const int64_t spw = plain ? 1 : 64 / L;
        const double waves = (double)((m + spw - 1) / spw);
        const double stage = cc * E + (plain ? 2.0 : 6.0) * word;
        const double blocks = (plain && E % 4 == 0 ? E / 4 : E == 1 ? 1 : E / 4 + 1) +
                              (cell_in ? E / 4 + 1 : 0);
        const double one = 4.0 * (double)nsteps * stage + 440.0 * blocks;
        // a lone wave waits for its own results at every stage
        const double alone = one + 4.0 * (double)nsteps * 15.0;
        // a launch ends with the SIMD that holds the most waves; lanes of more
        // than 208 registers of state leave room for one wave only
        const int regs = (cell_in ? 4 : 3) * E * (f64 ? 2 : 1);
        const double t = std::max(alone, std::ceil(waves / simds) * one) * (regs > 208 ? 1.4 : 1.0);
        if (t < t_best) {
            t_best = t;
            best.E = E;
            best.L = plain ? 0 : (int)L;
            best.spw = (int)spw;
        }
    }
    if (t_best >= 1e300) {   // FP32, n just past 3840: the widest lanes, select per cell
        best.E = mc_E(dtype, n);
        best.L = 0;
        best.spw = 1;
    }
    // four waves per SIMD: as many as pay where the registers leave room for them
    // (short lanes spend their time waiting, and FP32 instructions of different
    // waves overlap), and where they do not, shorter waves to even out the end
    // of the launch (CTM FP32 n = 4096, 16384 samples: 4.08 ms at two, 3.91 at four)
    int64_t w = opt_get(c, "mc.waves");
    if (w <= 0) w = (int64_t)c->cus * 16;
    best.nw = std::max<int64_t>(
        1, std::min<int64_t>(std::min(w, kMcMaxWaves), (m + best.spw - 1) / best.spw));
    return best;
}


// Autotune cache: one line per entry, each tagged with the format "reach2":
//   reach2 embed <arch> <kind> <dtype> <log2 n bucket> <per-cell inputs 0/1> <E> <K> <S> <ps per state-step>
//     (E = 0: the default shape, which takes back an earlier line of the bucket)
//   reach2 batch <arch> <kind> <log2 n bucket> <pack E cap> <ns per batch>
// Lines of any other form (an older format without the input mode among
// them) are ignored.
void load_tune_cache(reach_ctx* c) {
    const char* path = std::getenv("REACH_AUTOTUNE_CACHE");
    if (!path || !*path) return;
    FILE* f = std::fopen(path, "r");
    if (!f) return;
    char line[512];
    while (std::fgets(line, sizeof line, f)) {
        char arch[64];
        int kind, dtype, bucket, cell, E, K, S, cap;
        double ps;
        if (std::sscanf(line, "reach2 embed %63s %d %d %d %d %d %d %d %lf", arch, &kind, &dtype,
                        &bucket, &cell, &E, &K, &S, &ps) == 9) {
            const bool heat_ok = kind == REACH_HEAT3D && heat_waves(E) &&
                                 heat_has_shape(dtype == REACH_F64 ? 0 : 1, E, heat_waves(E));
            if (c->arch == arch && E == 0)
                c->tune.erase({kind, dtype, bucket, cell});
            else if (c->arch == arch && (cell == 0 || cell == 1) &&
                (heat_ok || (embed_has_shape(kind, dtype, E, S) && K >= 1 && 8 * K < 64 * E)))
                c->tune[{kind, dtype, bucket, cell}] = TuneEntry{E, K, S};
        } else if (std::sscanf(line, "reach2 batch %63s %d %d %d %lf", arch, &kind, &bucket, &cap,
                               &ps) == 5) {
            const bool cap_ok = cap == 2 || cap == 4 || cap == 8 || cap == 16;
            if (c->arch == arch && cap_ok && kind == -1 && bucket == -1)
                c->batch_cap = cap;   // the whole batch's width
            else if (c->arch == arch && cap_ok)
                c->batch_tune[{kind, bucket}] = cap;
        }
    }
    std::fclose(f);
}

void save_tune_entry(const reach_ctx* c, int kind, int dtype, int bucket, int cell_in, TuneEntry t,
                     double ps) {
    const char* path = std::getenv("REACH_AUTOTUNE_CACHE");
    if (!path || !*path) return;
    FILE* f = std::fopen(path, "a");
    if (!f) return;
    std::fprintf(f, "reach2 embed %s %d %d %d %d %d %d %d %.3f\n",
                 c->arch.empty() ? "unknown" : c->arch.c_str(), kind, dtype, bucket, cell_in, t.E,
                 t.K, t.S, ps);
    std::fclose(f);
}

void save_batch_tune_entry(const reach_ctx* c, int kind, int bucket, int cap, double ns) {
    const char* path = std::getenv("REACH_AUTOTUNE_CACHE");
    if (!path || !*path) return;
    FILE* f = std::fopen(path, "a");
    if (!f) return;
    std::fprintf(f, "reach2 batch %s %d %d %d %.0f\n", c->arch.empty() ? "unknown" : c->arch.c_str(),
                 kind, bucket, cap, ns);
    std::fclose(f);
}
}  // namespace

// =================================================================== ABI ==

extern "C" {

reach_status reach_ctx_create(int device, reach_ctx** out) {
    if (!out) return REACH_E_INVAL;
    *out = nullptr;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) return REACH_E_DEVICE;
    if (hipSetDevice(device) != hipSuccess) return REACH_E_DEVICE;
    reach_ctx* c = new reach_ctx();
    c->device = device;
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess && cus > 0)
        c->cus = cus;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) == hipSuccess) {
        c->arch = prop.gcnArchName;
        const size_t colon = c->arch.find(':');
        if (colon != std::string::npos) c->arch.resize(colon);
    }
    load_tune_cache(c);
    // the no-allocation Monte Carlo's scratch address on this device (its
    // failure is reported by that entry point, not here)
    (void)noalloc_setup(device);
    if (const char* e = std::getenv("REACH_LOG")) c->log = e[0] && std::strcmp(e, "0") != 0;
    if (hipMalloc((void**)&c->status, 256 + CutScratch::kSlots * CutScratch::kSlotBytes) != hipSuccess) {
        delete c;
        return REACH_E_DEVICE;
    }
    c->cut.mem = (char*)c->status + 256;
    if (hipMemset(c->status, 0, 256) != hipSuccess) { hipFree(c->status); delete c; return REACH_E_DEVICE; }
    if (hipEventCreateWithFlags(&c->staging_ev, hipEventDisableTiming) != hipSuccess) {
        hipFree(c->status); delete c; return REACH_E_DEVICE;
    }
    bool ok = hipEventCreateWithFlags(&c->batch_ev, hipEventDisableTiming) == hipSuccess;
    for (int k = 0; k < 2 && ok; ++k)
        ok = hipEventCreateWithFlags(&c->block_ev[k], hipEventDisableTiming) == hipSuccess;
    ok = ok && hipStreamCreateWithFlags(&c->copy_stream, hipStreamNonBlocking) == hipSuccess;
    if (!ok) {
        for (hipEvent_t e : {c->staging_ev, c->batch_ev, c->block_ev[0], c->block_ev[1]})
            if (e) hipEventDestroy(e);
        hipFree(c->status);
        delete c;
        return REACH_E_DEVICE;
    }
    *out = c;
    return REACH_OK;
}

__attribute__((visibility("hidden"))) void reach_server_destroy_internal(reach_ctx* c);

void reach_ctx_destroy(reach_ctx* c) {
    if (!c) return;
    hipSetDevice(c->device);
    reach_server_destroy_internal(c);
    hipDeviceSynchronize();
    for (auto& kv : c->graphs) hipGraphExecDestroy(kv.second);
    for (auto s : c->each_streams) hipStreamDestroy(s);
    if (c->staging) hipHostFree(c->staging);
    if (c->staging_ev) hipEventDestroy(c->staging_ev);
    if (c->batch_ev) hipEventDestroy(c->batch_ev);
    for (hipEvent_t e : c->block_ev)
        if (e) hipEventDestroy(e);
    for (CutScratch::Slot& k : c->cut.slot)
        if (k.done) hipEventDestroy(k.done);
    if (c->copy_stream) hipStreamDestroy(c->copy_stream);
    if (c->status) hipFree(c->status);
    c->pool.reset();
    delete c;
}

const char* reach_last_error(const reach_ctx* c) { return c ? c->err.c_str() : "no context"; }

reach_status reach_set_option(reach_ctx* c, const char* key, int64_t value) {
    if (!c || !key) return REACH_E_INVAL;
    static const char* keys[] = {"embed.K", "embed.E", "embed.S", "mc.waves", "batch.waves",
                                 "batch.split", "batch.pack", "batch.E",
                                 "serve.mode", "serve.waves", "gb.E", "gb.K", "heat.P",
                                 "user.E", "user.K"};
    bool known = false;
    for (const char* k : keys) known |= (std::strcmp(k, key) == 0);
    if (!known) return fail(c, REACH_E_INVAL, "unknown option %s", key);
    if (value < 0) return fail(c, REACH_E_INVAL, "option %s must be >= 0", key);
    if (!std::strcmp(key, "embed.E") && value && !embed_has_shape(REACH_CTM, REACH_F32, (int)value, 2) &&
        !embed_has_shape(REACH_CTM, REACH_F32, (int)value, 1) &&
        !embed_has_shape(REACH_CTM, REACH_F64, (int)value, 1))
        return fail(c, REACH_E_INVAL, "embed.E = %lld not built", (long long)value);
    if (!std::strcmp(key, "embed.S") && value != 0 && value != 1 && value != 2)
        return fail(c, REACH_E_INVAL, "embed.S must be 0, 1 or 2");
    if (!std::strcmp(key, "batch.pack") && value > 2)
        return fail(c, REACH_E_INVAL, "batch.pack must be 0 (auto), 1 (always) or 2 (never)");
    if (!std::strcmp(key, "batch.E") && value && value != 2 && value != 4 && value != 8 &&
        value != 16)
        return fail(c, REACH_E_INVAL, "batch.E must be 0, 2, 4, 8 or 16");
    if (!std::strcmp(key, "heat.P") && value && !heat_waves((int)value))
        return fail(c, REACH_E_INVAL, "heat.P must be 0, 2, 3, 4, 5 or 8");
    c->opt[key] = value;
    return REACH_OK;
}

int64_t reach_get_option(const reach_ctx* c, const char* key) {
    return (c && key) ? opt_get(c, key) : 0;
}

reach_status reach_plan_embed(reach_ctx* c, const reach_system* s, reach_dtype dtype,
                              int64_t nsteps, int64_t* out) {
    if (!c || !out) return REACH_E_INVAL;
    reach_status st = check_system(c, s, dtype);
    if (st != REACH_OK) return st;
    if (nsteps < 0) return fail(c, REACH_E_INVAL, "nsteps < 0");
    if (s->kind == REACH_HEAT3D) {
        HeatPlan hp;
        st = plan_heat(c, s, dtype, &hp);
        if (st != REACH_OK) return st;
        out[0] = hp.P; out[1] = 1; out[2] = hp.TX * hp.TY; out[3] = hp.OX; out[4] = 4;
        out[5] = nsteps; out[6] = 1;
        return REACH_OK;
    }
    EmbedPlan p;
    st = plan_embed(c, s, dtype, nsteps, &p);
    if (st != REACH_OK) return st;
    out[0] = p.E; out[1] = p.K; out[2] = p.W; out[3] = p.OUT; out[4] = p.H; out[5] = p.passes;
    out[6] = p.S;
    return REACH_OK;
}

size_t reach_workspace_bytes(reach_ctx* c, const reach_system* s, reach_dtype dtype, int64_t m) {
    if (!c || check_system(c, s, dtype) != REACH_OK || m < 0) return (size_t)-1;
    return m > 0 ? mc_ws_bytes(c, s, dtype, m) : embed_ws_bytes(c, s, dtype);
}

reach_status reach_sync(reach_ctx* c, void* stream) {
    if (!c) return REACH_E_INVAL;
    HIPCHK(c, hipSetDevice(c->device));
    HIPCHK(c, hipStreamSynchronize((hipStream_t)stream));
    unsigned int st = 0;
    HIPCHK(c, hipMemcpy(&st, c->status, sizeof st, hipMemcpyDeviceToHost));
    HIPCHK(c, hipMemset(c->status, 0, sizeof st));
    if (st & STATUS_NONFINITE) return fail(c, REACH_E_NONFINITE, "a result was not finite");
    if (st & STATUS_ORDER) return fail(c, REACH_E_ORDER, "a lower bound exceeded its upper bound");
    return REACH_OK;
}

// Whether work issued to this stream now goes into a graph (as far as can be told).
static bool capturing(hipStream_t s) {
    if (!s) return false;   // the default stream cannot be captured
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

static reach_status embed_run(reach_ctx* c, const reach_system* s, reach_dtype dtype,
                              const void* x_lo, const void* x_hi, const void* p_lo,
                              const void* p_hi, double t0, double dt, int64_t nsteps, void* r_lo,
                              void* r_hi, void* ws, size_t ws_bytes, void* stream,
                              int64_t one_steps, CutRun* cut) {
    if (!c) return REACH_E_INVAL;
    reach_status st = check_system(c, s, dtype);
    if (st != REACH_OK) return st;
    if (!x_lo || !x_hi || !r_lo || !r_hi) return fail(c, REACH_E_INVAL, "NULL state pointer");
    if (s->n_in > 0 && (!p_lo || !p_hi)) return fail(c, REACH_E_INVAL, "NULL input pointer");
    if (!(std::isfinite(dt) && dt > 0.0)) return fail(c, REACH_E_INVAL, "dt must be finite and > 0");
    if (!std::isfinite(t0)) return fail(c, REACH_E_INVAL, "t0 must be finite");
    if (nsteps < 0) return fail(c, REACH_E_INVAL, "nsteps < 0");
    HIPCHK(c, hipSetDevice(c->device));
    hipStream_t hs = (hipStream_t)stream;
    const size_t bytes = (size_t)s->n * dsize(dtype);
    if (nsteps == 0) {
        if (r_lo != x_lo) HIPCHK(c, hipMemcpyAsync(r_lo, x_lo, bytes, hipMemcpyDeviceToDevice, hs));
        if (r_hi != x_hi) HIPCHK(c, hipMemcpyAsync(r_hi, x_hi, bytes, hipMemcpyDeviceToDevice, hs));
        return REACH_OK;
    }
    if (s->kind == REACH_HEAT3D)
        return embed_heat3d(c, s, dtype, x_lo, x_hi, dt, nsteps, r_lo, r_hi, ws, ws_bytes, hs);
    EmbedPlan pl;
    const bool have_ws = ws && ws_bytes >= 2 * bytes;
    const bool alias = (r_lo == x_lo) || (r_hi == x_hi) || (r_lo == x_hi) || (r_hi == x_lo);
    // one window has read all its inputs before it writes a result; several read
    // the per-cell inputs again in every pass and the box beside each other's
    // results, so result arrays over either (the box's own aside) keep to the one
    bool cut_one = true;
    const size_t in_bytes = (size_t)s->n_in * dsize(dtype);
    for (const void* r : {(const void*)r_lo, (const void*)r_hi}) {
        cut_one &= !overlaps(p_lo, in_bytes, r, bytes) && !overlaps(p_hi, in_bytes, r, bytes);
        for (const void* x : {x_lo, x_hi}) cut_one &= r == x || !overlaps(x, bytes, r, bytes);
    }
    st = plan_embed(c, s, dtype, nsteps, &pl, have_ws, cut_one, one_steps);
    if (st != REACH_OK) return st;
    // a cut chain that one window holds runs its passes in the context's scratch,
    // which a captured call (replayed at any time, beside anything) does not use
    if (pl.cut_one && (pl.passes >= 2 || alias)) {
        if (2 * bytes > CutScratch::kSlotBytes || capturing(hs)) {
            st = plan_embed(c, s, dtype, nsteps, &pl, have_ws, false, one_steps);
            if (st != REACH_OK) return st;
        } else {
            if (!cut->slot) HIPCHK(c, cut->begin(c->cut, hs));
            ws = cut->mem;
            ws_bytes = CutScratch::kSlotBytes;
        }
    }
    log_call(c, "\"call\": \"embed\", \"kind\": %d, \"dtype\": \"%s\", \"n\": %lld, "
                "\"nsteps\": %lld, \"E\": %d, \"K\": %d, \"S\": %d, \"tiles\": %lld, "
                "\"passes\": %lld",
             s->kind, dtype_name(dtype), (long long)s->n, (long long)nsteps, pl.E, pl.K, pl.S,
             (long long)(pl.S == 1 ? 2 * pl.W : pl.W), (long long)pl.passes);

    // buffers: the last pass writes r; multi-tile passes never run in place
    const bool inplace_ok = (pl.W == 1);
    const bool need_ws = !inplace_ok && (pl.passes >= 2 || alias);
    void *w_lo = nullptr, *w_hi = nullptr;
    if (need_ws) {
        if (!ws || ws_bytes < 2 * bytes)
            return fail(c, REACH_E_INVAL, "workspace of %zu bytes needed", 2 * bytes);
        w_lo = ws;
        w_hi = (char*)ws + bytes;
    }
    const PassIo io(pl.passes, inplace_ok, alias);
    const void* lo_of[3] = {x_lo, r_lo, w_lo};
    const void* hi_of[3] = {x_hi, r_hi, w_hi};

    EmbedPass a{};
    a.p_lo = p_lo; a.p_hi = p_hi;
    a.n = s->n; a.W = pl.W; a.OUT = pl.OUT; a.H = pl.H;
    kernel_prm(s, a.prm);
    a.h2 = dt / 2.0; a.dt = dt; a.dt6 = dt / 6.0;
    a.status = c->status;
    const int mode = s->n_in > 1 ? 1 : 0;   // per-cell inputs
    if (s->n_in == 0) { a.p_lo = nullptr; a.p_hi = nullptr; }
    bool part = false;
    int64_t done = 0;
    for (int64_t p = 0; p < pl.passes; ++p) {
        a.src_lo = lo_of[io.src(p)];
        a.src_hi = hi_of[io.src(p)];
        a.dst_lo = (void*)lo_of[io.dst(p)];
        a.dst_hi = (void*)hi_of[io.dst(p)];
        a.ksteps = std::min<int64_t>(pl.K, nsteps - done);
        a.check = (p == pl.passes - 1) ? 1 : 0;
        // a one-step pass is a pure stream: its reads and writes bypass the
        // caches' retention (non-temporal), 1.8% faster at 2^26 cells
        a.nt = a.ksteps == 1 ? 1 : 0;
        // one side per wave: the last pass has both sides of a window in one
        // block, which checks the order (unless such blocks would share SIMDs), and
        // so has every pass of a single window, whose sides may write over each
        // other's inputs
        part = pl.S == 1 && a.check &&
               part_last_pass(c, s->kind, dtype, mode == 1, pl.W, pl.E, a.ksteps,
                              2.0 * (double)bytes, true);
        const bool pair = pl.S == 1 && (a.check || pl.W == 1) && !part;
        const int64_t tiles = pl.S == 1 && !pair ? 2 * pl.W : pl.W;
        a.per_xcd = (int32_t)((tiles + 7) / 8);
        const int64_t grid = 8 * (int64_t)a.per_xcd;
        hipError_t e = launch_embed(s->kind, mode, dtype == REACH_F64 ? 0 : 1, pl.E, pl.S, pair,
                                    a, grid, hs);
        if (e != hipSuccess) return hip_fail(c, e, "embedding kernel launch");
        done += a.ksteps;
    }
    if (part) {
        hipError_t e = launch_order_check(dtype == REACH_F64 ? 0 : 1, a.dst_lo, a.dst_hi, s->n,
                                          c->status, kPartBlocks, hs);
        if (e != hipSuccess) return hip_fail(c, e, "order check launch");
    }
    if (io.final_copy()) {
        HIPCHK(c, hipMemcpyAsync(r_lo, w_lo, bytes, hipMemcpyDeviceToDevice, hs));
        HIPCHK(c, hipMemcpyAsync(r_hi, w_hi, bytes, hipMemcpyDeviceToDevice, hs));
    }
    return REACH_OK;
}

reach_status reach_embed_rk4(reach_ctx* c, const reach_system* s, reach_dtype dtype,
                             const void* x_lo, const void* x_hi, const void* p_lo,
                             const void* p_hi, double t0, double dt, int64_t nsteps, void* r_lo,
                             void* r_hi, void* ws, size_t ws_bytes, void* stream) {
    CutRun cut;
    return embed_run(c, s, dtype, x_lo, x_hi, p_lo, p_hi, t0, dt, nsteps, r_lo, r_hi, ws, ws_bytes,
                     stream, kSplitSteps, &cut);
}

reach_status reach_embed_rk4_tube(reach_ctx* c, const reach_system* s, reach_dtype dtype,
                                  const void* x_lo, const void* x_hi, const void* p_lo,
                                  const void* p_hi, double t0, double dt, int64_t nsteps,
                                  int64_t every, void* tube_lo, void* tube_hi, void* ws,
                                  size_t ws_bytes, void* stream) {
    if (!c) return REACH_E_INVAL;
    reach_status st = check_system(c, s, dtype);
    if (st != REACH_OK) return st;
    if (every < 1 || nsteps < 1 || nsteps % every != 0)
        return fail(c, REACH_E_INVAL, "nsteps must be a positive multiple of every");
    if (!tube_lo || !tube_hi) return fail(c, REACH_E_INVAL, "NULL tube pointer");
    const size_t bytes = (size_t)s->n * dsize(dtype);
    const int64_t slots = nsteps / every;
    const void* src_lo = x_lo;
    const void* src_hi = x_hi;
    CutRun cut;
    for (int64_t k = 0; k < slots; ++k) {
        void* dlo = (char*)tube_lo + (size_t)k * bytes;
        void* dhi = (char*)tube_hi + (size_t)k * bytes;
        // each slot continues from the previous one: resumed runs are bitwise
        // the same as one run
        st = embed_run(c, s, dtype, src_lo, src_hi, p_lo, p_hi, t0 + (double)(k * every) * dt, dt,
                       every, dlo, dhi, ws, ws_bytes, stream, slots > 1 ? 1 : kSplitSteps, &cut);
        if (st != REACH_OK) return st;
        src_lo = dlo;
        src_hi = dhi;
    }
    return REACH_OK;
}

reach_status reach_autotune_embed(reach_ctx* c, const reach_system* s, reach_dtype dtype,
                                  const void* x_lo, const void* x_hi, const void* p_lo,
                                  const void* p_hi, double dt, int64_t trial_steps, void* r_lo,
                                  void* r_hi, void* ws, size_t ws_bytes, void* stream,
                                  int64_t* best) {
    if (!c || !best) return REACH_E_INVAL;
    reach_status st = check_system(c, s, dtype);
    if (st != REACH_OK) return st;
    if (trial_steps < 1) return fail(c, REACH_E_INVAL, "trial_steps must be >= 1");
    HIPCHK(c, hipSetDevice(c->device));
    hipStream_t hs = (hipStream_t)stream;
    if (s->kind == REACH_HEAT3D)
        return autotune_heat3d(c, s, dtype, x_lo, x_hi, dt, trial_steps, r_lo, r_hi, ws, ws_bytes,
                               hs, best);
    const int64_t saveE = opt_get(c, "embed.E"), saveK = opt_get(c, "embed.K");
    static const int Es[] = {4, 8, 12, 16, 24, 28, 32, 48, 64};
    static const int Ks[] = {2, 4, 6, 8, 10, 12, 16, 20, 24};
    const int64_t saveS = opt_get(c, "embed.S");
    hipEvent_t e0, e1;
    HIPCHK(c, hipEventCreate(&e0));
    HIPCHK(c, hipEventCreate(&e1));
    // picoseconds per state-step of one shape: `reps` timed calls of `steps`
    // steps after one untimed call, the fastest call counted (the least
    // disturbed by anything else on the device)
    auto time_shape = [&](const TuneEntry& t, int64_t steps, int reps, double* ps) -> reach_status {
        c->opt["embed.E"] = t.E;
        c->opt["embed.K"] = t.K;
        c->opt["embed.S"] = t.S;
        reach_status r = reach_embed_rk4(c, s, dtype, x_lo, x_hi, p_lo, p_hi, 0.0, dt, steps,
                                         r_lo, r_hi, ws, ws_bytes, stream);
        double best_ms = 1e300;
        for (int rep = 0; rep < reps && r == REACH_OK; ++rep) {
            if (hipEventRecord(e0, hs) != hipSuccess) return REACH_E_DEVICE;
            r = reach_embed_rk4(c, s, dtype, x_lo, x_hi, p_lo, p_hi, 0.0, dt, steps, r_lo, r_hi,
                                ws, ws_bytes, stream);
            if (hipEventRecord(e1, hs) != hipSuccess || hipEventSynchronize(e1) != hipSuccess)
                return REACH_E_DEVICE;
            float ms = 0.f;
            if (hipEventElapsedTime(&ms, e0, e1) != hipSuccess) return REACH_E_DEVICE;
            best_ms = std::min(best_ms, (double)ms);
        }
        *ps = best_ms * 1e9 / (2.0 * (double)s->n * (double)steps);
        return r;
    };
    // coarse scan of every built shape, then the four fastest and the default
    // shape again with ten times the steps
    std::vector<std::pair<double, TuneEntry>> scan;
    st = REACH_OK;
    for (int S : {2, 1})
    for (int E : Es) {
        if (st != REACH_OK) break;
        if (!embed_has_shape(s->kind, dtype, E, S) || (int64_t)64 * E >= 4 * s->n) continue;
        for (int K : Ks) {
            if (8 * K >= 64 * E) continue;
            double ps = 0;
            st = time_shape(TuneEntry{E, K, S}, trial_steps, 2, &ps);
            if (st != REACH_OK) break;
            scan.push_back({ps, TuneEntry{E, K, S}});
        }
    }
    double best_ps = 1e300;
    TuneEntry bt{0, 0, 0};
    bool default_won = false;
    if (st == REACH_OK && !scan.empty()) {
        std::stable_sort(scan.begin(), scan.end(),
                         [](const auto& a, const auto& b) { return a.first < b.first; });
        std::vector<TuneEntry> finals;
        for (size_t q = 0; q < scan.size() && q < 4; ++q) finals.push_back(scan[q].second);
        const TuneEntry d = default_shape(c, s->kind, dtype, s->n_in > 1, s->n);
        bool have_d = false;
        for (const auto& f : finals) have_d |= (f.E == d.E && f.K == d.K && f.S == d.S);
        // (a default of a width or a K that the scan leaves out is timed with the finals)
        if (!have_d && embed_has_shape(s->kind, dtype, d.E, d.S) && 8 * d.K < 64 * d.E)
            finals.push_back(d);
        // the finals in three rounds, each shape once per round (a warm-up and
        // two timed calls), so that a drift of the clock over the trials
        // favours none of them; the measured default stays unless a shape
        // beats it by more than 2%: shapes within run-to-run noise of each
        // other (at 2^26 FP64 RD, K = 16, 20 and 24) would otherwise take
        // turns from run to run
        constexpr double kKeepDefault = 0.02;
        std::vector<double> fps(finals.size(), 1e300);
        for (int round = 0; round < 3 && st == REACH_OK; ++round)
            for (size_t k = 0; k < finals.size() && st == REACH_OK; ++k) {
                double ps = 0;
                st = time_shape(finals[k], 10 * trial_steps, 2, &ps);
                fps[k] = std::min(fps[k], ps);
            }
        double d_ps = 1e300;
        for (size_t k = 0; k < finals.size() && st == REACH_OK; ++k) {
            if (fps[k] < best_ps) { best_ps = fps[k]; bt = finals[k]; }
            if (finals[k].E == d.E && finals[k].K == d.K && finals[k].S == d.S) d_ps = fps[k];
        }
        if (st == REACH_OK && d_ps <= best_ps * (1.0 + kKeepDefault)) {
            best_ps = d_ps;
            bt = d;
            default_won = true;
        }
    }
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    c->opt["embed.E"] = saveE;
    c->opt["embed.K"] = saveK;
    c->opt["embed.S"] = saveS;
    if (st != REACH_OK) return st;
    if (bt.E == 0) return fail(c, REACH_E_UNSUPPORTED, "n too small to tile: nothing to tune");
    const int bucket = n_bucket(s->n);
    const int cell_in = s->n_in > 1 ? 1 : 0;
    // (where the default wins nothing is recorded for the rest of the bucket, whose
    // default may be another; the line written takes back an earlier one)
    if (default_won) c->tune.erase({s->kind, dtype, bucket, cell_in});
    else c->tune[{s->kind, dtype, bucket, cell_in}] = bt;
    save_tune_entry(c, s->kind, dtype, bucket, cell_in, default_won ? TuneEntry{0, 0, 0} : bt,
                    best_ps);
    best[0] = bt.E;
    best[1] = bt.K;
    best[2] = (int64_t)std::llround(best_ps * 1000.0);
    best[3] = bt.S;
    return REACH_OK;
}

reach_status reach_montecarlo_range(reach_ctx* c, const reach_system* s, reach_dtype dtype,
                                    const void* x_lo, const void* x_hi, const void* p_lo,
                                    const void* p_hi, double t0, double dt, int64_t nsteps,
                                    int64_t s0, int64_t m, uint64_t seed, void* r_min,
                                    void* r_max, void* ws, size_t ws_bytes, void* stream) {
    if (!c) return REACH_E_INVAL;
    reach_status st = check_system(c, s, dtype);
    if (st != REACH_OK) return st;
    st = chains_only(c, s, "Monte Carlo");
    if (st != REACH_OK) return st;
    if (!x_lo || !x_hi || !r_min || !r_max) return fail(c, REACH_E_INVAL, "NULL pointer");
    if (s->n_in > 0 && (!p_lo || !p_hi)) return fail(c, REACH_E_INVAL, "NULL input pointer");
    if (!(std::isfinite(dt) && dt > 0.0)) return fail(c, REACH_E_INVAL, "dt must be finite and > 0");
    if (!std::isfinite(t0)) return fail(c, REACH_E_INVAL, "t0 must be finite");
    if (nsteps < 0) return fail(c, REACH_E_INVAL, "nsteps < 0");
    if (m < 1) return fail(c, REACH_E_INVAL, "m must be >= 1");
    if (s0 < 0) return fail(c, REACH_E_INVAL, "s0 must be >= 0");
    if (mc_E(dtype, s->n) < 0)
        return fail(c, REACH_E_UNSUPPORTED, "Monte Carlo holds a sample in one wave: n <= %d",
                    64 * mc_max_E(dtype));
    const size_t need = mc_ws_bytes(c, s, dtype, m);
    if (!ws || ws_bytes < need) return fail(c, REACH_E_INVAL, "workspace of %zu bytes needed", need);
    HIPCHK(c, hipSetDevice(c->device));
    McArgs a{};
    a.x_lo = x_lo; a.x_hi = x_hi; a.p_lo = p_lo; a.p_hi = p_hi;
    const int mode = s->n_in > 1 ? 1 : 0;
    const int dt_id = dtype == REACH_F64 ? 0 : 1;
    const McPlan pl = mc_plan(c, s->kind, dt_id, mode == 1, s->n, m, nsteps);
    a.nw = pl.nw;
    a.L = pl.L;
    a.spw = pl.spw;
    a.part_min = ws;
    a.part_max = (char*)ws + need / 2;
    a.n = s->n; a.n_in = s->n_in; a.nsteps = nsteps; a.s0 = s0; a.m = m; a.seed = seed;
    kernel_prm(s, a.prm);
    a.h2 = dt / 2.0; a.dt = dt; a.dt6 = dt / 6.0;
    hipStream_t hs = (hipStream_t)stream;
    log_call(c, "\"call\": \"montecarlo\", \"kind\": %d, \"dtype\": \"%s\", \"n\": %lld, "
                "\"nsteps\": %lld, \"s0\": %lld, \"m\": %lld, \"E\": %d, \"samples_per_wave\": %d, "
                "\"waves\": %lld",
             s->kind, dtype_name(dtype), (long long)s->n, (long long)nsteps, (long long)s0,
             (long long)m, pl.E, pl.spw, (long long)a.nw);
    hipError_t e = launch_mc(s->kind, mode, dt_id, pl.E, a, hs);
    if (e != hipSuccess) return hip_fail(c, e, "Monte Carlo kernel launch");
    e = launch_mc_reduce(dt_id, 0, a.part_min, a.part_max,
                         (a.nw + kMcWavesPerGroup - 1) / kMcWavesPerGroup, s->n, r_min, r_max,
                         c->status, hs);
    if (e != hipSuccess) return hip_fail(c, e, "Monte Carlo reduction launch");
    return REACH_OK;
}

reach_status reach_montecarlo(reach_ctx* c, const reach_system* s, reach_dtype dtype,
                              const void* x_lo, const void* x_hi, const void* p_lo,
                              const void* p_hi, double t0, double dt, int64_t nsteps, int64_t m,
                              uint64_t seed, void* r_min, void* r_max, void* ws, size_t ws_bytes,
                              void* stream) {
    return reach_montecarlo_range(c, s, dtype, x_lo, x_hi, p_lo, p_hi, t0, dt, nsteps, 0, m, seed,
                                  r_min, r_max, ws, ws_bytes, stream);
}

int64_t reach_mc_samples(int64_t n, double eps, double delta) {
    if (n < 1 || !(eps > 0.0 && eps < 1.0) || !(delta > 0.0 && delta < 1.0)) return -1;
    const double nn = 2.0 * (double)n;
    const double m = std::ceil((nn / eps) * std::log(nn / delta));
    if (!(m < 9.0e18)) return -1;
    return (int64_t)m;
}

}  // extern "C"


// ---------------------------------------------------------- growth bound --
namespace {

void contraction_params(const reach_system* s, double out[5]) {
    for (int i = 0; i < 5; ++i) out[i] = 0.0;
    if (s->kind == REACH_CTM) {
        out[0] = s->prm[0]; out[1] = 0.0; out[2] = s->prm[1]; out[3] = 0.0;
    } else if (s->kind == REACH_RD) {
        const double h2 = s->prm[0] * s->prm[0];
        out[0] = 1.0 / h2; out[1] = -2.0 / h2; out[2] = 1.0 / h2; out[3] = 1.0;
    } else {
        out[0] = std::fabs(s->prm[0]); out[1] = s->prm[1]; out[2] = std::fabs(s->prm[2]);
        out[3] = std::fabs(s->prm[3]);
    }
}

}  // namespace

extern "C" {

size_t reach_growth_bound_workspace_bytes(reach_ctx* c, const reach_system* s, reach_dtype dtype) {
    if (!c || check_system(c, s, dtype) != REACH_OK) return (size_t)-1;
    return (size_t)4 * (size_t)s->n * dsize(dtype);
}

reach_status reach_growth_bound(reach_ctx* c, const reach_system* s, reach_dtype dtype,
                                const void* x_lo, const void* x_hi, const void* p_lo,
                                const void* p_hi, double t0, double dt, int64_t nsteps,
                                void* r_lo, void* r_hi, void* ws, size_t ws_bytes, void* stream) {
    if (!c) return REACH_E_INVAL;
    reach_status st = check_system(c, s, dtype);
    if (st != REACH_OK) return st;
    if (!x_lo || !x_hi || !r_lo || !r_hi) return fail(c, REACH_E_INVAL, "NULL state pointer");
    if (s->n_in > 0 && (!p_lo || !p_hi)) return fail(c, REACH_E_INVAL, "NULL input pointer");
    if (!(std::isfinite(dt) && dt > 0.0)) return fail(c, REACH_E_INVAL, "dt must be finite and > 0");
    if (!std::isfinite(t0)) return fail(c, REACH_E_INVAL, "t0 must be finite");
    if (nsteps < 0) return fail(c, REACH_E_INVAL, "nsteps < 0");
    const size_t bytes = (size_t)s->n * dsize(dtype);
    if (!ws || ws_bytes < 4 * bytes) return fail(c, REACH_E_INVAL, "workspace of %zu bytes needed", 4 * bytes);
    HIPCHK(c, hipSetDevice(c->device));
    hipStream_t hs = (hipStream_t)stream;
    if (s->kind == REACH_HEAT3D)
        return gb_heat3d(c, s, dtype, x_lo, x_hi, dt, nsteps, r_lo, r_hi, ws, hs);
    // plan: the windows of the one-side embedding tiles (both runs cost a cell
    // what an RD cell costs; K_LIN3's own embedding runs both sides per wave, so
    // its shapes are not asked for)
    int E = (int)opt_get(c, "gb.E");
    int K = (int)opt_get(c, "gb.K");
    if (E && !gb_has_E(E)) return fail(c, REACH_E_INVAL, "gb.E = %d not built", E);
    const int64_t n = s->n;
    const bool cell_in = s->n_in > 1;
    const int like = s->kind == REACH_CTM ? REACH_CTM : REACH_RD;
    bool single = false;
    if (!E) {
        // (a K of the caller's has to fit the window's halo, which the narrower of
        // the widths, 2, 12 and 20 cells, would refuse at sizes that 4, 16 and 24 take)
        int one = 0;
        for (int e : {1, 2, 4, 8, 12, 16, 20, 24, 28, 32})
            if ((int64_t)64 * e >= n && !(K && (e == 2 || e == 12 || e == 20))) { one = e; break; }
        const int64_t simds = (int64_t)4 * c->cus;
        TuneEntry t{0, 0, 1};
        if (!K && nsteps > 0 && estimated(like, dtype, cell_in, n, simds)) {
            t = fastest_shape(c, like, dtype, cell_in, n, 0, true);
            const int64_t passes = (nsteps + t.K - 1) / t.K;
            t.K = (int)((nsteps + passes - 1) / passes);
            t = fastest_shape(c, like, dtype, cell_in, n, t.K, true);
            // one window: no passes at all
            if (one && (nsteps <= kSplitSteps || (int64_t)64 * t.E >= n ||
                        !cut_pays(one_window_us(like, dtype, cell_in, 1, one, n, nsteps),
                                  (double)nsteps * step_us(like, dtype, cell_in, 1, t.E, t.K, n, simds),
                                  passes, false)))
                t.E = 0;
        }
        if (t.E) {
            E = t.E;
            K = t.K;
        } else if (one) {
            E = one;
            single = !K;
        } else {
            // FP64 with shared inputs fits 28 cells per lane in 256 VGPRs (two
            // waves per SIMD; per-cell inputs need more there), which pays on
            // long chains only (see default_tune)
            E = dtype == REACH_F64 ? (cell_in || n < ((int64_t)1 << 26) ? 24 : 28) : 32;
        }
    } else if ((int64_t)64 * E >= n && !K) {
        single = true;
    }
    const int64_t span = (int64_t)64 * E;
    GbPass a{};
    a.x_lo = x_lo; a.x_hi = x_hi;
    a.p_lo = s->n_in ? p_lo : nullptr;
    a.p_hi = s->n_in ? p_hi : nullptr;
    a.n = n;
    kernel_prm(s, a.prm);
    contraction_params(s, a.prm_r);
    a.h2 = dt / 2.0; a.dt = dt; a.dt6 = dt / 6.0;
    int64_t passes;
    if (single) {
        K = (int)std::min<int64_t>(std::max<int64_t>(nsteps, 1), INT32_MAX);
        a.W = 1; a.OUT = 0; a.H = 0;
        passes = 1;
    } else {
        // steps per pass, measured on the 2^26 RD chain (FP64, 1000 steps): at
        // E = 24, K = 20 (104.1 ms; K = 12 is 5% slower, K = 24 ties); at E = 28,
        // K = 24 (101.1 ms against 102.3 at K = 20 and 104.1 at K = 16)
        if (!K) K = E == 28 ? 24 : 20;
        if ((int64_t)8 * K >= span) return fail(c, REACH_E_INVAL, "gb.K = %d too large for E = %d", K, E);
        a.H = 4 * K;
        a.OUT = span - 2 * a.H;
        a.W = (n <= span) ? 1 : 1 + (n - span + a.OUT - 1) / a.OUT;
        passes = std::max<int64_t>(1, (nsteps + K - 1) / K);
    }
    // The last pass writes the box itself unless the result arrays overlap what
    // other windows still read then (per-cell inputs; in a run of one pass the
    // box): such a call combines in a kernel of its own.
    const size_t in_bytes = (size_t)s->n_in * dsize(dtype);
    bool fused = true;
    if (a.W > 1)
        for (const void* q : {(const void*)r_lo, (const void*)r_hi}) {
            fused &= !overlaps(a.p_lo, in_bytes, q, bytes) && !overlaps(a.p_hi, in_bytes, q, bytes);
            if (passes == 1)
                fused &= !overlaps(x_lo, bytes, q, bytes) && !overlaps(x_hi, bytes, q, bytes);
        }
    const bool part = part_last_pass(c, like, dtype, cell_in, a.W, E, nsteps - (passes - 1) * K,
                                     4.0 * (double)bytes, false);
    fused &= !part;
    a.r_lo = r_lo; a.r_hi = r_hi;
    a.status = c->status;
    log_call(c, "\"call\": \"growth_bound\", \"kind\": %d, \"dtype\": \"%s\", \"n\": %lld, "
                "\"nsteps\": %lld, \"E\": %d, \"K\": %d, \"tiles\": %lld, \"passes\": %lld",
             s->kind, dtype_name(dtype), (long long)n, (long long)nsteps, E, K,
             (long long)(2 * a.W), (long long)passes);
    // (c, r) ping-pong in the workspace; the last pass writes buffer A
    char* A = (char*)ws;
    char* B = (char*)ws + 2 * bytes;
    const int mode = s->n_in > 1 ? 1 : 0;
    const int dt_id = dtype == REACH_F64 ? 0 : 1;
    int64_t done = 0;
    for (int64_t p = 0; p < passes; ++p) {
        char* dst = ((passes - 1 - p) % 2 == 0) ? A : B;
        char* src = ((passes - 1 - p) % 2 == 0) ? B : A;
        a.first = (p == 0) ? 1 : 0;
        a.last = fused && p == passes - 1 ? 1 : 0;
        a.pair = a.last || !pairs_share(c, a.W) ? 1 : 0;
        a.src_c = src; a.src_r = src + bytes;
        a.dst_c = dst; a.dst_r = dst + bytes;
        a.ksteps = std::min<int64_t>(K, nsteps - done);
        hipError_t e = launch_gb(s->kind, mode, dt_id, E, a, hs);
        if (e != hipSuccess) return hip_fail(c, e, "growth-bound kernel launch");
        done += a.ksteps;
    }
    if (fused) return REACH_OK;
    hipError_t e = launch_gb_combine(dt_id, A, A + bytes, n, r_lo, r_hi, c->status,
                                     part ? kPartBlocks : kSweepBlocks, hs);
    if (e != hipSuccess) return hip_fail(c, e, "growth-bound combine launch");
    return REACH_OK;
}

}  // extern "C"

// ================================================================ batch ==

namespace {

reach_status make_desc(reach_ctx* c, const reach_query& q, int64_t tag, QDesc* d) {
    reach_status st = check_system(c, &q.sys, q.dtype);
    if (st != REACH_OK) return st;
    st = chains_only(c, &q.sys, "the batch path");
    if (st != REACH_OK) return st;
    if (q.dtype != REACH_F64) return fail(c, REACH_E_UNSUPPORTED, "batched queries are FP64");
    if (q.sys.n > kBatchMaxN) return fail(c, REACH_E_UNSUPPORTED, "batched queries need n <= 512");
    if (q.sys.n_in > 1) return fail(c, REACH_E_UNSUPPORTED, "batched queries take n_in 0 or 1");
    if (!(std::isfinite(q.dt) && q.dt > 0.0)) return fail(c, REACH_E_INVAL, "dt must be finite and > 0");
    if (!std::isfinite(q.t0)) return fail(c, REACH_E_INVAL, "t0 must be finite");
    if (q.nsteps < 0) return fail(c, REACH_E_INVAL, "nsteps < 0");
    if (!q.x_lo || !q.x_hi || !q.r_lo || !q.r_hi) return fail(c, REACH_E_INVAL, "NULL state pointer");
    if (q.sys.n_in == 1 && (!q.p_lo || !q.p_hi)) return fail(c, REACH_E_INVAL, "NULL input pointer");
    std::memset(d, 0, sizeof *d);
    d->kind = q.sys.kind;
    d->E = batch_cells_per_lane(q.sys.n);
    d->n = q.sys.n;
    d->nsteps = q.nsteps;
    kernel_prm(&q.sys, d->prm);
    d->h2 = q.dt / 2.0; d->dt = q.dt; d->dt6 = q.dt / 6.0;
    d->x_lo = (const double*)q.x_lo; d->x_hi = (const double*)q.x_hi;
    d->r_lo = (double*)q.r_lo; d->r_hi = (double*)q.r_hi;
    d->tag = tag;
    if (q.sys.n_in == 1) {
        d->p_lo = (const double*)q.p_lo;
        d->p_hi = (const double*)q.p_hi;
    }
    return REACH_OK;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Host threads for preparing a batch of nq queries (1 below 16384 queries,
// at most kMaxHostThreads).
constexpr int64_t kMaxHostThreads = 16;
int batch_host_threads(int64_t nq) {
    if (nq < 16384) return 1;
    const unsigned hw = std::thread::hardware_concurrency();
    const int64_t by_size = nq / 4096;
    return (int)std::max<int64_t>(
        1, std::min<int64_t>({by_size, kMaxHostThreads, hw ? (int64_t)hw : 1}));
}

// fn(t) for t in [0, nth): t = 0 on the calling thread, the rest on the pool's
// workers (nth <= the pool's size; without a pool nth must be 1).
template <class F>
void run_threads(HostPool* pool, int nth, F&& fn) {
    if (nth <= 1 || !pool) {
        for (int t = 0; t < nth; ++t) fn(t);
        return;
    }
    pool->run(nth, std::function<void(int)>(fn));
}

// fn(u) for every u in [0, nu) on nth threads, each thread taking the next
// unclaimed u: a thread the system holds back delays only the unit it holds,
// and the outputs, kept per unit, do not depend on which thread ran which.
template <class F>
void run_units(HostPool* pool, int nth, int nu, F&& fn) {
    std::atomic<int> next{0};
    run_threads(pool, std::min(nth, nu), [&](int) {
        for (int u = next.fetch_add(1); u < nu; u = next.fetch_add(1)) fn(u);
    });
}

// The context's pool, started on first use with batch_host_threads' maximum.
HostPool* host_pool(reach_ctx* c) {
    if (!c) return nullptr;
    if (!c->pool) {
        const unsigned hw = std::thread::hardware_concurrency();
        c->pool.reset(new HostPool(
            (int)std::max<int64_t>(1, std::min<int64_t>(kMaxHostThreads, hw ? hw : 1))));
    }
    return c->pool.get();
}

// Descriptors (the caller's order), work items, the item count and the items'
// query indices, uploaded as one block.
size_t batch_block_bytes(int64_t nq) {
    return (sizeof(QDesc) + sizeof(BatchItem) + sizeof(uint32_t)) * (size_t)nq + sizeof(uint64_t);
}
struct BatchBlock {
    QDesc* desc;
    BatchItem* items;
    uint64_t* count;
    uint32_t* members;
};
BatchBlock batch_block(void* base, int64_t nq) {
    BatchBlock b;
    b.desc = (QDesc*)base;
    b.items = (BatchItem*)(b.desc + nq);
    b.count = (uint64_t*)(b.items + nq);
    b.members = (uint32_t*)(b.count + 1);
    return b;
}

// 1/16-octave class of a wave time, larger for shorter work (the launch
// order takes classes in increasing order: longest first).
int wave_time_bucket(uint64_t cost) {
    constexpr int kBuckets = 64 * 16;
    const uint64_t c1 = cost + 1u;      // never 0
    const int msb = 63 - __builtin_clzll(c1);
    const int frac = msb >= 4 ? (int)((c1 >> (msb - 4)) & 15u) : (int)((c1 << (4 - msb)) & 15u);
    return kBuckets - 1 - (msb * 16 + frac);
}

// Segment packing of a batch.  A query of n cells in a pack at E cells per
// lane takes L = ceil(n / E) lanes and needs the balanced layout
// n >= (E - 1) L; its estimated issue cost per cell is (kCellOps + kSegLaneOps
// / E) L E / n (arithmetic per cell and stage, plus the lane shifts and
// boundary selects per lane and stage, over the cells the lanes hold).
// seg_E picks the cheapest E of kSegE up to cap (ties to the wider), or the
// narrowest valid E above cap when none up to it is valid.
constexpr double kCellOps = 6.0, kSegLaneOps = 12.0;
// Default cap on E before the batch autotuner has run.
constexpr int kSegECap = 16;

int seg_E(int64_t n, int cap) {
    double best = 1e300;
    int bestE = 0, above = 0;
    for (int E : kSegE) {
        const int64_t L = (n + E - 1) / E;
        if (L > 64 || n < (int64_t)(E - 1) * L) continue;
        if (E > cap) {
            if (!above) above = E;
            continue;
        }
        const double cost = (kCellOps + kSegLaneOps / E) * (double)(L * E) / (double)n;
        if (cost <= best) { best = cost; bestE = E; }
    }
    return bestE ? bestE : above;
}

// Cells per lane of a packed query by size: cap[c], the cheapest up to 2 << c cells,
// and down[k], the widest narrower than kSegE[k] that its lanes still fit (0: none).
struct PackWidths {
    int8_t cap[4][513], down[4][513];
};
const PackWidths& pack_widths() {
    static const PackWidths t = [] {
        PackWidths w{};
        for (int64_t n = 1; n <= 512; ++n)
            for (int k = 0; k < 4; ++k) {
                w.cap[k][n] = (int8_t)seg_E(n, 2 << k);
                for (int j = 0; j < k; ++j) {
                    const int e = kSegE[j];
                    const int64_t L = (n + e - 1) / e;
                    if (L <= 64 && n >= (int64_t)(e - 1) * L) w.down[k][n] = (int8_t)e;
                }
            }
        return w;
    }();
    return t;
}

// Whether one side's result lies over what the other side reads.  A wave that
// holds both sides reads both before it writes; waves of one side each do not
// wait for each other.  (A LIN3 query always runs whole.)
bool crossed(const reach_query& q) {
    if (q.sys.kind == REACH_LIN3) return false;
    const size_t box = sizeof(double) * (size_t)q.sys.n, in = sizeof(double) * (size_t)q.sys.n_in;
    return overlaps(q.x_hi, box, q.r_lo, box) || overlaps(q.p_hi, in, q.r_lo, box) ||
           overlaps(q.x_lo, box, q.r_hi, box) || overlaps(q.p_lo, in, q.r_hi, box);
}

// Least E * steps of a pack or query that may run one side per wave: the two waves
// exchange the end of their item through memory, which writes back caches (700
// queries of 20 steps: 88 us by sides, 52 whole; 4500 of 20 steps in packs: 428 and 294).
constexpr uint64_t kMinSidePack = 1600, kMinSideQuery = 200;

// Whether a batch packs: option batch.pack 1 always, 2 never, 0 (default)
// when it has more queries than 16 per compute unit, or than twice option
// batch.waves (below that every query side gets a wave of its own and packing
// would only lengthen the longest).
bool batch_packs(const reach_ctx* c, int64_t nq) {
    const int64_t mode = c ? opt_get(c, "batch.pack") : 0;
    if (mode == 1) return true;
    if (mode == 2) return false;
    int64_t waves = c ? opt_get(c, "batch.waves") : 0;
    if (waves <= 0) waves = (int64_t)(c ? c->cus : 256) * 8;
    return nq > 2 * waves;
}

// Largest cells per lane of a pack for (kind, size bucket): option batch.E,
// else the bucket's autotuned cap, else the autotuned cap of the whole batch
// (reach_autotune_batch), else kSegECap.
int batch_ecap(const reach_ctx* c, int kind, int bucket) {
    if (c) {
        const int64_t e = opt_get(c, "batch.E");
        if (e > 0) return (int)e;
        auto it = c->batch_tune.find({kind, bucket});
        if (it != c->batch_tune.end()) return it->second;
        if (c->batch_cap) return c->batch_cap;
    }
    return kSegECap;
}

// The schedule of a batch: the descriptors descs[nq] in the caller's order
// and the work items in launch order (items[k] covers members[start .. start
// + count), indices into q, contiguous in launch order).
//
// Two parallel passes over nu work units (up to two per thread, claimed
// dynamically; every output is kept per unit, so the plan does not depend on
// which thread ran which unit).  First each unit reads a contiguous chunk of
// the caller's array once: it validates every query (without touching the
// context; the first bad query, lowest index, is re-checked with the context
// afterwards to set the error message).  When the batch does not pack
// (batch_packs), every query is an item of its own, run alone over a whole
// wave.  When it packs, every item is a segment pack, and each query gets,
// once the batch's load is known, a pack key: its constants class (bitwise equal kind, dt and parameters),
// cells per lane E (seg_E under the bucket's cap) and 1/16-octave step
// bucket.  Then unit u owns the keys of the (E, bucket) pairs r with r mod
// nu = u and scans the queries of its keys in caller order, placing each in
// the first of up to kOpen open packs of its key with room (at most 64 lanes
// and kPackMax queries; when none has room the fullest is closed); the packs
// still open at the end are packed again per key, widest query first into
// the first pack with room.  Items are then ordered longest first by the wave
// time (E * steps of the longest member; ceil(n / 64) * steps alone) at 1/16
// octave, ties in unit order.  Packs of a batch too small for its longest query
// are narrowed, and the longest items run one side per wave (see there).
//
// cross (may be NULL): set when some query is `crossed`, the plan then unfinished;
// whole: the plan for such a batch, packed whatever its size and the options,
// every pack's sides in one wave.
struct PlanTimes {
    double pass1_ms = 0, pass_ms = 0, order_ms = 0, members_ms = 0;
};

reach_status plan_batch(reach_ctx* c, HostPool* pool, const reach_query* q, int64_t nq,
                        int split, int nth, QDesc* descs, std::vector<uint32_t>* members_out,
                        std::vector<BatchItem>* items_out, int* packed, int64_t* sides_out,
                        PlanTimes* times = nullptr,
                        const std::function<void()>& descs_done = nullptr, bool whole = false,
                        bool* cross = nullptr) {
    using clk = std::chrono::steady_clock;
    auto since = [](clk::time_point t0) {
        return std::chrono::duration<double, std::milli>(clk::now() - t0).count();
    };
    auto t0 = clk::now();
    int nu = 1;   // work units (set below)
    auto chunk = [&](int t, int64_t total, int64_t* lo, int64_t* hi) {
        *lo = total * t / nu;
        *hi = total * (t + 1) / nu;
    };
    constexpr int kBuckets = 64 * 16;
    constexpr int kLanes = 64;
    constexpr int kOpen = 8;             // open packs per key
    constexpr int kNE = (int)(sizeof(kSegE) / sizeof(kSegE[0]));
    constexpr int kNB = 10;              // size buckets floor(log2 n), n <= 512
    constexpr int kMaxClasses = 16;      // per thread (4 bits of a key); further classes run alone
    struct Item {
        uint32_t first;    // into the thread's member list
        uint16_t count;
        uint16_t E;
        int16_t bucket;
    };
    struct Consts {
        int32_t kind;
        double dt;
        double prm[8];
        bool operator==(const Consts& o) const {
            return kind == o.kind && std::memcmp(&dt, &o.dt, sizeof dt) == 0 &&
                   std::memcmp(prm, o.prm, sizeof prm) == 0;
        }
    };
    struct Open {
        int lanes = 0;
        int count = 0;
        int E = 0;
        int64_t max_steps = 0;
        uint32_t mem[kPackMax];
    };
    const bool packs = whole || (!split && batch_packs(c, nq));
    *packed = packs ? 1 : 0;
    int ecap[4][kNB];
    for (int k = 0; k < 4; ++k)
        for (int b = 0; b < kNB; ++b) ecap[k][b] = batch_ecap(c, k, b);
    auto push_alone = [&](std::vector<Item>& items, std::vector<uint32_t>& members, uint32_t i) {
        const QDesc& d = descs[i];
        const uint64_t cost = (uint64_t)d.E * (uint64_t)std::min<int64_t>(d.nsteps, (int64_t)1 << 40);
        items.push_back(Item{(uint32_t)members.size(), 1, 0, (int16_t)wave_time_bucket(cost)});
        members.push_back(i);
        return cost;
    };
    auto push_pack = [&](std::vector<Item>& items, std::vector<uint32_t>& members, Open& o) {
        if (o.count >= 1) {
            const uint64_t cost = (uint64_t)o.E * (uint64_t)std::min<int64_t>(o.max_steps, (int64_t)1 << 40);
            items.push_back(Item{(uint32_t)members.size(), (uint16_t)o.count, (uint16_t)o.E,
                                 (int16_t)wave_time_bucket(cost)});
            for (int m = 0; m < o.count; ++m) members.push_back(o.mem[m]);
        }
        o.count = 0;
        o.lanes = 0;
        o.max_steps = 0;
    };
    // work units: contiguous chunks of the queries in pass 1, (E, step bucket)
    // partitions in pass 2, item ranges after; several per thread, claimed
    // dynamically (run_units)
    nu = nth > 1 ? (int)std::min<int64_t>(2 * (int64_t)nth, std::max<int64_t>(nth, nq / 2048)) : 1;
    std::vector<std::vector<Item>> titems((size_t)nu);
    std::vector<std::vector<uint32_t>> tmembers((size_t)nu);
    std::vector<int64_t> bad((size_t)nu, nq);
    std::vector<uint8_t> crosses((size_t)nu, 0);
    const auto& etab = pack_widths().cap;
    // pass 1: descriptors, validation, pack keys (class ids local to the
    // chunk); a chunk's packed queries are listed by the partition owning
    // their (E, step bucket) pair, r mod nu
    // what pass 2 needs of a query, carried in the lists so that it never
    // reads the descriptors other chunks wrote
    struct QRef {
        uint32_t i;
        int32_t key;       // (E index, step bucket) << 4 | chunk-local class
        int64_t nsteps;
        int32_t L;         // lanes at the key's E
        uint16_t n;
        uint8_t E;
        int8_t cls;        // -1: a class beyond the unit's table
    };
    std::vector<std::vector<Consts>> tclasses((size_t)nu);
    std::vector<std::vector<QRef>> lists((size_t)nu);          // by partition, caller order within
    std::vector<std::vector<uint32_t>> list_at((size_t)nu);    // partition p: [at[p], at[p + 1])
    std::vector<std::vector<QRef>> refs((size_t)nu);           // a chunk's packed queries
    std::vector<std::pair<uint64_t, uint64_t>> loads((size_t)nu);   // sum and longest
    // the keys of a chunk's queries, and the lists by partition
    const auto key_refs = [&](int t, bool narrow, uint64_t load) {
        std::vector<QRef>& mine = refs[(size_t)t];
        titems[(size_t)t].clear();
        tmembers[(size_t)t].clear();
        std::vector<uint32_t>& at = list_at[(size_t)t];
        at.assign((size_t)nu + 1, 0);
        for (QRef& r : mine) {
            const uint64_t steps = (uint64_t)std::min<int64_t>(r.nsteps, (int64_t)1 << 32);
            while (narrow && r.E * steps > load + load / 4) {
                const int e = pack_widths().down[r.E == 16 ? 3 : r.E == 8 ? 2 : r.E == 4 ? 1 : 0][r.n];
                if (!e) break;
                r.E = (uint8_t)e;
            }
            r.L = (int32_t)(((unsigned)r.n + r.E - 1) / r.E);
            if (r.cls < 0) {
                // a class beyond the unit's table: a pack of its own
                Open o;
                o.E = r.E;
                o.mem[o.count++] = r.i;
                o.lanes = r.L;
                o.max_steps = r.nsteps;
                push_pack(titems[(size_t)t], tmembers[(size_t)t], o);
                continue;
            }
            int ei = 0;
            while (kSegE[ei] != r.E) ++ei;
            const int b = wave_time_bucket((uint64_t)std::min<int64_t>(r.nsteps, (int64_t)1 << 40));
            r.key = ((ei * kBuckets + b) << 4) | r.cls;
            ++at[(size_t)((r.key >> 4) % nu) + 1];
        }
        // by partition (counting sort, caller order kept within a partition)
        for (int u = 0; u < nu; ++u) at[(size_t)u + 1] += at[(size_t)u];
        std::vector<QRef>& out = lists[(size_t)t];
        out.resize(at[(size_t)nu]);
        std::vector<uint32_t> put(at.begin(), at.end() - 1);
        for (const QRef& r : mine)
            if (r.cls >= 0) out[put[(size_t)((r.key >> 4) % nu)]++] = r;
    };
    // (on several threads the keys at the first width are formed at once, which
    // saves a batch without a tail a hand-over between them)
    const bool keyed = nth > 1;
    run_units(pool, nth, nu, [&](int t) {
        int64_t lo, hi;
        chunk(t, nq, &lo, &hi);
        std::vector<Item> items;
        std::vector<uint32_t> members;
        int64_t my_bad = nq;
        bool my_cross = false;
        uint64_t my_cost = 0, longest = 0;
        std::vector<Consts> classes;
        std::vector<QRef> mine;
        if (packs) mine.reserve((size_t)(hi - lo));
        for (int64_t i = lo; i < hi; ++i) {
            QDesc& d = descs[i];
            if (make_desc(nullptr, q[i], i, &d) != REACH_OK) {
                my_bad = std::min(my_bad, i);
                continue;
            }
            if (cross) my_cross |= crossed(q[i]);
            if (!packs) {
                my_cost += push_alone(items, members, (uint32_t)i);
                continue;
            }
            const int cap = ecap[d.kind & 3][std::min(n_bucket(d.n), kNB - 1)];
            const int E = etab[cap >= 16 ? 3 : cap >= 8 ? 2 : cap >= 4 ? 1 : 0][d.n];
            const uint64_t steps = (uint64_t)std::min<int64_t>(d.nsteps, (int64_t)1 << 32);
            my_cost += ((unsigned)d.n + (unsigned)E - 1) / (unsigned)E * (unsigned)E * steps;
            longest = std::max(longest, (uint64_t)E * steps);
            int cls = -1;
            Consts cs;
            std::memset(&cs, 0, sizeof cs);
            cs.kind = q[i].sys.kind;
            cs.dt = q[i].dt;
            std::memcpy(cs.prm, q[i].sys.prm, sizeof cs.prm);
            for (size_t u = 0; u < classes.size(); ++u)
                if (classes[u] == cs) { cls = (int)u; break; }
            if (cls < 0 && (int)classes.size() < kMaxClasses) {
                classes.push_back(cs);
                cls = (int)classes.size() - 1;
            }
            mine.push_back(QRef{(uint32_t)i, 0, d.nsteps, 0, (uint16_t)d.n, (uint8_t)E, (int8_t)cls});
        }
        titems[(size_t)t] = std::move(items);
        tmembers[(size_t)t] = std::move(members);
        tclasses[(size_t)t] = std::move(classes);
        bad[(size_t)t] = my_bad;
        refs[(size_t)t] = std::move(mine);
        if (packs && keyed) key_refs(t, false, 0);
        crosses[(size_t)t] = my_cross ? 1 : 0;
        loads[(size_t)t] = {my_cost, longest};
    });
    const int64_t first_bad = *std::min_element(bad.begin(), bad.end());
    if (first_bad < nq) {
        QDesc tmp;
        return make_desc(c, q[first_bad], first_bad, &tmp);
    }
    if (cross) {
        *cross = std::find(crosses.begin(), crosses.end(), 1) != crosses.end();
        if (*cross) return REACH_OK;
    }
    // every descriptor is written: the caller may start moving them while
    // the items are formed
    if (descs_done) descs_done();
    // The batch's load: the wave time E * steps of its items over the SIMDs (of packs,
    // by the lanes their queries take).  An item longer than that holds up the end of
    // the launch: it runs one side per wave (*sides_out).  Packs fill about four fifths
    // of their lanes and narrower ones spend a ninth more on shifts and selects, so
    // the packs of a batch are left as they are unless the longest takes 1.45 loads
    // (7000 queries of 100 steps: 966 packs of 16 cells 204 us, 1574 of 8 cells 215);
    // else queries whose packs would take more than 1.25 loads go to narrower ones (as
    // far as their lanes fit a wave), and the items still longer than one load to two
    // waves.  A 10^4-query mix (4-512 cells, 10-1000 steps) has a load of about 4200: 16
    // cells for 1000 steps would take 16000, 8 cells and one side the time of 4000.
    uint64_t load = 0, longest = 0;
    for (const auto& v : loads) {
        load += v.first;
        longest = std::max(longest, v.second);
    }
    load /= (uint64_t)(packs ? kLanes : 1) * 4 * (uint64_t)(c ? c->cus : 256);
    const bool tail = (double)longest > 1.45 * (double)load;
    // (a caller who asks for packs or for a width gets the widths as they are)
    const bool narrow = tail && !(c && (opt_get(c, "batch.pack") || opt_get(c, "batch.E")));
    if (packs && (narrow || !keyed)) run_units(pool, nth, nu, [&](int t) { key_refs(t, narrow, load); });
    if (times) times->pass1_ms = since(t0);
    if (packs) {
        // global class ids (the chunks' tables merged in chunk order)
        std::vector<Consts> global;
        std::vector<std::vector<int32_t>> remap((size_t)nu);
        for (int t = 0; t < nu; ++t)
            for (const Consts& cs : tclasses[(size_t)t]) {
                int g = -1;
                for (size_t u = 0; u < global.size(); ++u)
                    if (global[u] == cs) { g = (int)u; break; }
                if (g < 0) {
                    global.push_back(cs);
                    g = (int)global.size() - 1;
                }
                remap[(size_t)t].push_back(g);
            }
        const size_t G = global.size();
        // key = (E index, step bucket) * G + global class; partition t owns
        // the (E index, step bucket) pairs r with r mod nu == t
        std::vector<uint32_t> local((size_t)kNE * kBuckets);
        std::vector<uint32_t> owned((size_t)nu, 0);
        for (size_t r = 0; r < local.size(); ++r) local[r] = owned[r % (size_t)nu]++;
        // pass 2: partition t packs the keys it owns, scanning the queries in
        // caller order.  The scan only assigns each query a pack (fill levels
        // in a small table, a key's kOpen current packs side by side); the
        // packs' member lists are then formed by a counting sort on the pack.
        run_units(pool, nth, nu, [&](int t) {
            std::vector<Item>& items = titems[(size_t)t];
            std::vector<uint32_t>& members = tmembers[(size_t)t];
            struct Pack {
                int32_t lanes, count, E, key;
                int64_t max_steps;
            };
            std::vector<Pack> packs;
            std::vector<int32_t> slot((size_t)owned[(size_t)t] * G * kOpen, -1);
            std::vector<const QRef*> refs;
            std::vector<int32_t> assign;
            for (int u = 0; u < nu; ++u) {
                const std::vector<int32_t>& rm = remap[(size_t)u];
                const std::vector<uint32_t>& at = list_at[(size_t)u];
                for (uint32_t k = at[(size_t)t]; k < at[(size_t)t + 1]; ++k) {
                    const QRef& qr = lists[(size_t)u][k];
                    const size_t r = (size_t)(qr.key >> 4);
                    const int E = kSegE[r / kBuckets];
                    const int L = qr.L;
                    const size_t key = (size_t)local[r] * G + (size_t)rm[(size_t)(qr.key & 15)];
                    int32_t* sl = &slot[key * kOpen];
                    if (sl[0] < 0)
                        for (int j = 0; j < kOpen; ++j) {
                            sl[j] = (int32_t)packs.size();
                            packs.push_back(Pack{0, 0, E, (int32_t)key, 0});
                        }
                    int j = 0;
                    while (j < kOpen && packs[(size_t)sl[j]].lanes + L > kLanes) ++j;
                    if (j == kOpen) {
                        // every open pack is too full for this query: close the
                        // fullest and open a new one in its place
                        j = 0;
                        for (int k = 1; k < kOpen; ++k)
                            if (packs[(size_t)sl[k]].lanes > packs[(size_t)sl[j]].lanes) j = k;
                        sl[j] = (int32_t)packs.size();
                        packs.push_back(Pack{0, 0, E, (int32_t)key, 0});
                    }
                    Pack& pk = packs[(size_t)sl[j]];
                    pk.lanes += L;
                    pk.max_steps = std::max(pk.max_steps, qr.nsteps);
                    refs.push_back(&qr);
                    assign.push_back(sl[j]);
                    if (++pk.count == kPackMax || pk.lanes == kLanes) {
                        sl[j] = (int32_t)packs.size();
                        packs.push_back(Pack{0, 0, E, (int32_t)key, 0});
                    }
                }
            }
            // members by pack (counting sort, scan order kept within a pack)
            std::vector<int32_t> start(packs.size() + 1, 0);
            for (const int32_t p : assign) ++start[(size_t)p + 1];
            for (size_t p = 0; p < packs.size(); ++p) start[p + 1] += start[p];
            std::vector<const QRef*> by_pack(refs.size());
            {
                std::vector<int32_t> at(start.begin(), start.end() - 1);
                for (size_t k = 0; k < refs.size(); ++k) by_pack[(size_t)at[(size_t)assign[k]]++] = refs[k];
            }
            // packs still open at the end (those the slots point to) are packed
            // again per key below; every other pack is final
            std::vector<uint8_t> open_now(packs.size(), 0);
            for (const int32_t p : slot)
                if (p >= 0) open_now[(size_t)p] = 1;
            for (size_t p = 0; p < packs.size(); ++p) {
                const Pack& pk = packs[p];
                if (open_now[p] || pk.count == 0) continue;
                const uint64_t cost = (uint64_t)pk.E * (uint64_t)std::min<int64_t>(pk.max_steps, (int64_t)1 << 40);
                items.push_back(Item{(uint32_t)members.size(), (uint16_t)pk.count, (uint16_t)pk.E,
                                     (int16_t)wave_time_bucket(cost)});
                for (int32_t k = start[p]; k < start[p + 1]; ++k) members.push_back(by_pack[(size_t)k]->i);
            }
            // each key's open packs: their queries again, widest first into
            // the first pack with room (first fit decreasing)
            std::vector<const QRef*> rest;
            std::vector<Open> merged;
            for (size_t k = 0; k < slot.size(); k += kOpen) {
                if (slot[k] < 0) continue;
                rest.clear();
                int E = 0;
                for (int j = 0; j < kOpen; ++j) {
                    const size_t p = (size_t)slot[k + (size_t)j];
                    E = packs[p].E;
                    for (int32_t m = start[p]; m < start[p + 1]; ++m) rest.push_back(by_pack[(size_t)m]);
                }
                if (rest.empty()) continue;
                std::sort(rest.begin(), rest.end(), [](const QRef* x, const QRef* y) {
                    return x->L != y->L ? x->L > y->L : x->i < y->i;
                });
                merged.clear();
                for (const QRef* rr : rest) {
                    Open* o = nullptr;
                    for (Open& oj : merged)
                        if (oj.lanes + rr->L <= kLanes && oj.count < kPackMax) { o = &oj; break; }
                    if (!o) {
                        merged.emplace_back();
                        o = &merged.back();
                        o->E = E;
                    }
                    o->mem[o->count++] = rr->i;
                    o->lanes += rr->L;
                    o->max_steps = std::max(o->max_steps, rr->nsteps);
                }
                for (Open& o : merged) push_pack(items, members, o);
            }
        });
    }
    if (times) times->pass_ms = since(t0);
    t0 = clk::now();
    // launch order: bucket-major, then unit, then the unit's item order.  A
    // count of items and of their members per (unit, bucket), one prefix over
    // (bucket, unit), then every unit places its own items and members.
    // (the counts live in buffers kept by the calling thread: fresh ones of this
    // size would cost page faults on every call)
    thread_local std::vector<int64_t> hist_buf, mhist_buf;
    if (hist_buf.size() < (size_t)nu * kBuckets) {
        hist_buf.resize((size_t)nu * kBuckets);
        mhist_buf.resize((size_t)nu * kBuckets);
    }
    int64_t* hist = hist_buf.data();
    int64_t* mhist = mhist_buf.data();
    std::vector<int> blo((size_t)nu, kBuckets), bhi((size_t)nu, -1);   // buckets in use
    run_units(pool, nth, nu, [&](int t) {
        int64_t* h = &hist[(size_t)t * kBuckets];
        int64_t* mh = &mhist[(size_t)t * kBuckets];
        std::fill(h, h + kBuckets, 0);
        std::fill(mh, mh + kBuckets, 0);
        for (const Item& it : titems[(size_t)t]) {
            ++h[it.bucket];
            mh[it.bucket] += it.count;
            blo[(size_t)t] = std::min<int>(blo[(size_t)t], it.bucket);
            bhi[(size_t)t] = std::max<int>(bhi[(size_t)t], it.bucket);
        }
    });
    const int b0 = *std::min_element(blo.begin(), blo.end());
    const int b1 = *std::max_element(bhi.begin(), bhi.end());
    int64_t ni = 0, nm = 0;
    for (int b = b0; b <= b1; ++b)
        for (int t = 0; t < nu; ++t) {
            const size_t x = (size_t)t * kBuckets + b;
            const int64_t v = hist[x], mv = mhist[x];
            hist[x] = ni;
            mhist[x] = nm;
            ni += v;
            nm += mv;
        }
    // items longer than the load come first: those of the buckets before its own
    *sides_out = 0;
    if (split && !whole) *sides_out = ni;
    else if (packs ? tail && !whole : true) {
        const int lb = wave_time_bucket(std::max(load, packs ? kMinSidePack : kMinSideQuery));
        // (the counts are item indices now: that of unit 0 in the load's bucket is
        // the number of items in the buckets before)
        *sides_out = lb <= b0 ? 0 : lb > b1 ? ni : hist[lb];
    }
    if (times) times->order_ms = since(t0);
    t0 = clk::now();
    std::vector<BatchItem>& io = *items_out;
    std::vector<uint32_t>& mo = *members_out;
    io.resize((size_t)ni);
    mo.resize((size_t)nq);
    std::vector<uint8_t> wide((size_t)nu, 0);
    run_units(pool, nth, nu, [&](int t) {
        int64_t* h = &hist[(size_t)t * kBuckets];
        int64_t* mh = &mhist[(size_t)t * kBuckets];
        for (const Item& it : titems[(size_t)t]) {
            const int64_t k = h[it.bucket]++;
            const int64_t m = mh[it.bucket];
            mh[it.bucket] += it.count;
            io[(size_t)k] = BatchItem{(uint32_t)m, it.count, it.E};
            std::memcpy(&mo[(size_t)m], &tmembers[(size_t)t][it.first], sizeof(uint32_t) * it.count);
            if (it.E > 8) wide[(size_t)t] = 1;
        }
    });
    if (std::find(wide.begin(), wide.end(), 1) != wide.end()) *packed = 2;
    if (times) times->members_ms = since(t0);
    return REACH_OK;
}

}  // namespace

extern "C" {

// batch workspace: [work counter][per-query flags][per-query side counters]
// and two blocks of [descriptors, items, item count, members], used by turns
size_t reach_batch_workspace_bytes(int64_t nq) {
    if (nq < 0) return (size_t)-1;
    return align256(8) + 2 * align256(4 * (size_t)nq) + 2 * align256(batch_block_bytes(nq));
}

reach_status reach_plan_batch(reach_ctx* c, const reach_query* q, int64_t nq,
                              int64_t* item_start, int32_t* item_count, int32_t* item_E,
                              int64_t* member, int64_t* n_items) {
    if (nq < 0 || !n_items || (nq > 0 && (!q || !item_start || !item_count || !item_E || !member)))
        return c ? fail(c, REACH_E_INVAL, "bad arguments") : REACH_E_INVAL;
    *n_items = 0;
    if (nq == 0) return REACH_OK;
    const int split = (c && opt_get(c, "batch.split")) ? 1 : 0;
    std::vector<QDesc> descs((size_t)nq);
    std::vector<uint32_t> members;
    std::vector<BatchItem> items;
    // without a context a large plan gets a pool of its own for this call,
    // so the schedule is computed the same way as for the batch
    std::unique_ptr<HostPool> local;
    HostPool* pool = host_pool(c);
    if (!pool && batch_host_threads(nq) > 1) {
        local.reset(new HostPool(batch_host_threads(nq)));
        pool = local.get();
    }
    const int nth = pool ? std::min(batch_host_threads(nq), pool->size()) : 1;
    int packed = 0;
    int64_t sides = 0;
    const reach_status st = plan_batch(c, pool, q, nq, split, nth, descs.data(), &members, &items,
                                       &packed, &sides);
    if (st != REACH_OK) return st;
    for (size_t k = 0; k < items.size(); ++k) {
        item_start[k] = items[k].start;
        item_count[k] = (int32_t)items[k].count;
        item_E[k] = (int32_t)items[k].E;
    }
    for (int64_t p = 0; p < nq; ++p) member[p] = members[(size_t)p];
    *n_items = (int64_t)items.size();
    return REACH_OK;
}

reach_status reach_embed_rk4_batch(reach_ctx* c, const reach_query* q, int64_t nq, void* ws,
                                   size_t ws_bytes, void* stream) {
    if (!c) return REACH_E_INVAL;
    if (nq < 0 || (nq > 0 && !q)) return fail(c, REACH_E_INVAL, "bad query array");
    if (nq == 0) return REACH_OK;
    const size_t need = reach_batch_workspace_bytes(nq);
    if (!ws || ws_bytes < need) return fail(c, REACH_E_NOMEM, "workspace of %zu bytes needed", need);
    HIPCHK(c, hipSetDevice(c->device));
    hipStream_t hs = (hipStream_t)stream;
    // batch.split = 1 turns packing off and runs each side of a cooperative query in a
    // wave of its own
    const int split = opt_get(c, "batch.split") ? 1 : 0;
    HostPool* pool = batch_host_threads(nq) > 1 ? host_pool(c) : nullptr;
    const int nth = pool ? std::min(batch_host_threads(nq), pool->size()) : 1;
    // pinned staging (reused; wait for the previous upload from it, which
    // ends before that batch's kernel starts).  Growing it drops the cached
    // graphs, after every launched one has finished.
    if (c->staging_cap < nq) {
        HIPCHK(c, hipDeviceSynchronize());
        if (c->staging) HIPCHK(c, hipHostFree(c->staging));
        c->staging = nullptr;
        for (auto& kv : c->graphs) hipGraphExecDestroy(kv.second);
        c->graphs.clear();
        int64_t cap = std::max<int64_t>(nq, 1024);
        HIPCHK(c, hipHostMalloc((void**)&c->staging, batch_block_bytes(cap), hipHostMallocDefault));
        c->staging_cap = cap;
    } else {
        HIPCHK(c, hipEventSynchronize(c->staging_ev));
    }
    const BatchBlock hb = batch_block(c->staging, nq);
    char* base = (char*)ws;
    auto* counter = (unsigned long long*)base;
    auto* qflags = (unsigned int*)(base + align256(8));
    auto* pair = (unsigned int*)(base + align256(8) + align256(4 * (size_t)nq));
    // two blocks of descriptors and work items, used by turns: this batch's
    // upload (on the context's copy stream) waits only for the kernel that
    // read its block two batches ago, so it runs beside the previous batch's
    // kernel; the counter reset and the kernel wait for that kernel, on any
    // stream, and for the upload
    const int blk = c->next_block;
    const BatchBlock db = batch_block(base + align256(8) + 2 * align256(4 * (size_t)nq) +
                                      (size_t)blk * align256(batch_block_bytes(nq)), nq);
    hipStream_t cs = c->copy_stream;
    if (c->block_ev_recorded[blk]) HIPCHK(c, hipStreamWaitEvent(cs, c->block_ev[blk], 0));
    // another workspace or query count moves the blocks, which may then
    // overlap what the previous batch's kernel still uses: wait for it too
    if (c->batch_ev_recorded && (ws != c->last_ws || nq != c->last_nq))
        HIPCHK(c, hipStreamWaitEvent(cs, c->batch_ev, 0));
    const auto t_start = std::chrono::steady_clock::now();
    std::vector<uint32_t> members;
    std::vector<BatchItem> items;
    PlanTimes pt;
    int packed = 0;
    int64_t sides = 0;   // leading items of a packed batch that run one side per wave
    // the descriptors go up as soon as they are written, while the host forms
    // the work items
    hipError_t desc_err = hipSuccess;
    const size_t desc_bytes = sizeof(QDesc) * (size_t)nq;
    const auto upload = [&] {
        desc_err = hipMemcpyAsync(db.desc, hb.desc, desc_bytes, hipMemcpyHostToDevice, cs);
    };
    bool cross = false;
    reach_status pst = plan_batch(c, pool, q, nq, split, nth, hb.desc, &members, &items, &packed,
                                  &sides, &pt, upload, false, &cross);
    if (pst == REACH_OK && cross)
        pst = plan_batch(c, pool, q, nq, split, nth, hb.desc, &members, &items, &packed, &sides,
                         &pt, upload, true);
    if (pst != REACH_OK) return pst;
    if (desc_err != hipSuccess) return hip_fail(c, desc_err, "descriptor upload");
    const int64_t ni = (int64_t)items.size();
    std::memcpy(hb.items, items.data(), sizeof(BatchItem) * (size_t)ni);
    std::memcpy(hb.members, members.data(), sizeof(uint32_t) * (size_t)nq);
    *hb.count = (uint64_t)ni | ((uint64_t)sides << 32);
    const auto t_plan = std::chrono::steady_clock::now();

    int64_t grid = opt_get(c, "batch.waves");
    if (grid <= 0) {
        if (packed) grid = c->batch_waves[packed - 1];
        if (grid <= 0)
            grid = (int64_t)c->cus * (packed == 2 ? kWideWavesPerCU
                                      : packed == 1 ? kPackWavesPerCU : kBatchWavesPerCU);
        // the wide packing kernel holds at most two waves per SIMD
        if (packed == 2) grid = std::min<int64_t>(grid, (int64_t)c->cus * 8);
    }
    c->last_packed = packed;
    // (a coupled item of the leading ones runs whole, its second half is empty: waves
    // for those would leave SIMDs with two items beside SIMDs with none)
    int64_t units = ni + sides;
    if (ni < grid)
        for (int64_t k = 0; k < sides; ++k)
            units -= hb.desc[hb.members[hb.items[k].start]].kind == REACH_LIN3 ? 1 : 0;
    grid = std::min<int64_t>(grid, units);

    if (c->log) {
        using ms = std::chrono::duration<double, std::milli>;
        log_call(c, "\"call\": \"batch\", \"queries\": %lld, \"items\": %lld, \"packed\": %lld, "
                    "\"waves\": %lld, \"split\": %d, \"host_threads\": %d, \"plan_ms\": %.3f, "
                    "\"plan_pass1_ms\": %.3f, \"plan_pass_ms\": %.3f, \"plan_order_ms\": %.3f, "
                    "\"plan_members_ms\": %.3f",
                 (long long)nq, (long long)ni, (long long)(nq - (int64_t)std::count_if(
                     items.begin(), items.end(), [](const BatchItem& x) { return x.count == 1; })),
                 (long long)grid, sides > 0 ? 1 : 0, nth, ms(t_plan - t_start).count(), pt.pass1_ms,
                 pt.pass_ms, pt.order_ms, pt.members_ms);
    }
    // the rest of the block (items, their count, the members) follows; the
    // staging is free for the next call once both copies are done, so the
    // next call plans while this batch's kernel runs
    HIPCHK(c, hipMemcpyAsync(db.items, hb.items, batch_block_bytes(nq) - desc_bytes,
                             hipMemcpyHostToDevice, cs));
    HIPCHK(c, hipEventRecord(c->staging_ev, cs));
    HIPCHK(c, hipStreamWaitEvent(hs, c->staging_ev, 0));
    if (c->batch_ev_recorded) HIPCHK(c, hipStreamWaitEvent(hs, c->batch_ev, 0));
    auto enqueue = [&](hipStream_t s) -> hipError_t {
        hipError_t e = launch_zero(base, (int64_t)(align256(8) + 2 * align256(4 * (size_t)nq)) / 4, s);
        if (e != hipSuccess) return e;
        return launch_batch(db.desc, db.items, db.members, db.count, counter, qflags, pair,
                            c->status, sides > 0, packed, grid, s);
    };

    if (hs == nullptr) {
        hipError_t e = enqueue(hs);
        if (e != hipSuccess) return hip_fail(c, e, "batch launch");
    } else {
        GraphKey key{nq, ws, c->staging, (((grid * 2 + (sides > 0)) * 3 + packed) * 2 + blk), hs};
        auto it = c->graphs.find(key);
        if (it == c->graphs.end()) {
            hipGraph_t g = nullptr;
            HIPCHK(c, hipStreamBeginCapture(hs, hipStreamCaptureModeRelaxed));
            hipError_t e = enqueue(hs);
            hipError_t e2 = hipStreamEndCapture(hs, &g);
            if (e != hipSuccess) { if (g) hipGraphDestroy(g); return hip_fail(c, e, "batch capture"); }
            if (e2 != hipSuccess) return hip_fail(c, e2, "hipStreamEndCapture");
            hipGraphExec_t ge = nullptr;
            e = hipGraphInstantiate(&ge, g, nullptr, nullptr, 0);
            hipGraphDestroy(g);
            if (e != hipSuccess) return hip_fail(c, e, "hipGraphInstantiate");
            it = c->graphs.emplace(key, ge).first;
        }
        HIPCHK(c, hipGraphLaunch(it->second, hs));
    }
    HIPCHK(c, hipEventRecord(c->batch_ev, hs));
    HIPCHK(c, hipEventRecord(c->block_ev[blk], hs));
    c->batch_ev_recorded = true;
    c->block_ev_recorded[blk] = true;
    c->next_block = 1 - blk;
    c->last_ws = ws;
    c->last_nq = nq;
    (void)counter;
    return REACH_OK;
}

// Batch autotuner, on the caller's whole batch (a bucket's queries alone
// would be too few to fill the device, and their timing would favour short
// items over dense ones).  After kTuneWarm untimed calls, every comparison
// times the batch (one warm-up and four timed calls, fastest kept) with the
// candidate setting and then again with the current one, and takes the
// candidate only when it is faster by more than kTuneGain.  In order: the
// width of the whole batch (every bucket's cap 16, the wide kernel, against
// 8, the narrow one); then, bucket by bucket, most queries first, for every
// (kind, size bucket) with at least kTuneMinQueries queries, the narrower
// caps 8, 4 and 2; then 4, 8 and (narrow kernel only) 12 resident waves per
// compute unit.  Results are those of the batch at any setting (bitwise).
reach_status reach_autotune_batch(reach_ctx* c, const reach_query* q, int64_t nq, void* ws,
                                  size_t ws_bytes, void* stream, int64_t* best) {
    if (!c) return REACH_E_INVAL;
    if (!best || nq < 1 || !q) return fail(c, REACH_E_INVAL, "bad arguments");
    constexpr int64_t kTuneMinQueries = 256;
    constexpr double kTuneGain = 0.01;
    constexpr int kTuneWarm = 8;
    constexpr int kNB = 10;
    hipStream_t hs = (hipStream_t)stream;
    HIPCHK(c, hipSetDevice(c->device));
    hipEvent_t e0 = nullptr, e1 = nullptr;
    HIPCHK(c, hipEventCreate(&e0));
    if (hipEventCreate(&e1) != hipSuccess) {
        hipEventDestroy(e0);
        return fail(c, REACH_E_DEVICE, "hipEventCreate failed");
    }
    // fastest of four timed calls after a warm-up, in nanoseconds (host
    // planning and the descriptor upload included)
    auto time_batch = [&](double* ns) -> reach_status {
        double bestms = 1e300;
        for (int r = 0; r < 5; ++r) {
            if (hipEventRecord(e0, hs) != hipSuccess) return fail(c, REACH_E_DEVICE, "event");
            const reach_status st = reach_embed_rk4_batch(c, q, nq, ws, ws_bytes, stream);
            if (st != REACH_OK) return st;
            if (hipEventRecord(e1, hs) != hipSuccess || hipEventSynchronize(e1) != hipSuccess)
                return fail(c, REACH_E_DEVICE, "event");
            float ms = 0.f;
            if (hipEventElapsedTime(&ms, e0, e1) != hipSuccess) return fail(c, REACH_E_DEVICE, "event");
            if (r > 0) bestms = std::min(bestms, (double)ms);
        }
        *ns = bestms * 1e6;
        return REACH_OK;
    };
    const int64_t save_E = opt_get(c, "batch.E"), save_waves = opt_get(c, "batch.waves");
    c->opt["batch.E"] = 0;
    // widths are timed at each packing kernel's default wave count
    c->batch_waves[0] = c->batch_waves[1] = 0;
    // a few untimed calls first, so that the device clock has left its idle
    // level before anything is compared
    reach_status st = REACH_OK;
    for (int w = 0; w < kTuneWarm && st == REACH_OK; ++w)
        st = reach_embed_rk4_batch(c, q, nq, ws, ws_bytes, stream);
    if (st == REACH_OK && hipStreamSynchronize(hs) != hipSuccess)
        st = fail(c, REACH_E_DEVICE, "batch warm-up");
    double cur = 0;
    if (st == REACH_OK) st = time_batch(&cur);
    // a setting replaces the current one only when the batch timed with it is
    // faster by kTuneGain than the batch timed again with the current one
    // right after (drift of the device clock hits both alike)
    auto trial = [&](const std::function<void()>& cand, const std::function<void()>& keep,
                     bool* won) -> reach_status {
        double tc = 0, tk = 0;
        cand();
        reach_status r = time_batch(&tc);
        keep();
        if (r == REACH_OK) r = time_batch(&tk);
        if (r != REACH_OK) return r;
        *won = tc < tk * (1.0 - kTuneGain);
        if (*won) {
            cand();
            cur = tc;
        } else {
            cur = tk;
        }
        return REACH_OK;
    };
    const bool packs = !opt_get(c, "batch.split") && batch_packs(c, nq);
    if (st == REACH_OK && packs) {
        // (kind, bucket) groups, most queries first
        std::map<std::pair<int, int>, int64_t> count;
        for (int64_t i = 0; i < nq; ++i) {
            const reach_system& sy = q[i].sys;
            ++count[{sy.kind, std::min(n_bucket(sy.n), kNB - 1)}];
        }
        std::vector<std::pair<int64_t, std::pair<int, int>>> order;
        for (const auto& kv : count)
            if (kv.second >= kTuneMinQueries) order.push_back({-kv.second, kv.first});
        std::sort(order.begin(), order.end());
        // the whole batch's width first: every bucket at 8 cells per lane (the
        // narrow kernel, two waves per SIMD) against 16 (the wide kernel, one)
        for (const auto& kv : count) c->batch_tune.erase(kv.first);
        const int first = c->batch_cap ? c->batch_cap : kSegECap;
        const int other = first == 16 ? 8 : 16;
        bool won = false;
        st = trial([&] { c->batch_cap = other; }, [&] { c->batch_cap = first; }, &won);
        if (st == REACH_OK) save_batch_tune_entry(c, -1, -1, c->batch_cap, cur);
        // then narrower caps bucket by bucket
        for (size_t k = 0; k < order.size() && st == REACH_OK; ++k) {
            const auto key = order[k].second;
            const int keep = batch_ecap(c, key.first, key.second);
            for (int cap : {8, 4, 2}) {
                if (cap >= batch_ecap(c, key.first, key.second)) continue;
                const int now = batch_ecap(c, key.first, key.second);
                st = trial([&] { c->batch_tune[key] = cap; }, [&] { c->batch_tune[key] = now; },
                           &won);
                if (st != REACH_OK) break;
            }
            if (st == REACH_OK && batch_ecap(c, key.first, key.second) != keep)
                save_batch_tune_entry(c, key.first, key.second,
                                      batch_ecap(c, key.first, key.second), cur);
        }
    }
    int64_t best_waves = save_waves;
    if (st == REACH_OK && packs && save_waves == 0) {
        // from the kernel's default (one wave per SIMD for the wide kernel,
        // two for the narrow one), which the last timed call used
        const bool wide = c->last_packed == 2;
        int64_t& tuned = c->batch_waves[wide ? 1 : 0];
        int64_t now = (int64_t)c->cus * (wide ? kWideWavesPerCU : kPackWavesPerCU);
        for (int64_t per_cu : {4, 8, 12}) {
            const int64_t w = per_cu * c->cus;
            // the wide packing kernel holds at most two waves per SIMD
            if (w == now || (wide && per_cu > 8)) continue;
            bool won = false;
            const int64_t was = now;
            st = trial([&] { tuned = w; }, [&] { tuned = was; }, &won);
            if (st != REACH_OK) break;
            if (won) now = w;
        }
        best_waves = now;
    }
    c->opt["batch.E"] = save_E;
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    if (st != REACH_OK) return st;
    best[0] = best_waves;
    best[1] = (int64_t)std::llround(cur);
    return REACH_OK;
}

reach_status reach_embed_rk4_each(reach_ctx* c, const reach_query* q, int64_t nq, int32_t nstreams) {
    if (!c) return REACH_E_INVAL;
    if (nq < 0 || (nq > 0 && !q)) return fail(c, REACH_E_INVAL, "bad query array");
    if (nstreams < 1 || nstreams > 16) return fail(c, REACH_E_INVAL, "nstreams must be 1..16");
    HIPCHK(c, hipSetDevice(c->device));
    while ((int32_t)c->each_streams.size() < nstreams) {
        hipStream_t s;
        HIPCHK(c, hipStreamCreateWithFlags(&s, hipStreamNonBlocking));
        c->each_streams.push_back(s);
    }
    std::vector<QDesc> d(nq);
    for (int64_t i = 0; i < nq; ++i) {
        reach_status st = make_desc(c, q[i], i, &d[i]);
        if (st != REACH_OK) return st;
    }
    for (int64_t i = 0; i < nq; ++i) {
        hipError_t e = launch_single(d[i], c->status, nullptr, c->each_streams[i % nstreams]);
        if (e != hipSuccess) return hip_fail(c, e, "single-query launch");
    }
    for (int32_t k = 0; k < nstreams; ++k) HIPCHK(c, hipStreamSynchronize(c->each_streams[k]));
    return REACH_OK;
}

}  // extern "C"


// ------------------------------------------------ services for user.cpp --
namespace reach {
namespace rt {

int ctx_device(const reach_ctx* c) { return c->device; }
int ctx_cus(const reach_ctx* c) { return c->cus; }
unsigned int* ctx_status(reach_ctx* c) { return c->status; }
int64_t option(const reach_ctx* c, const char* key) { return opt_get(c, key); }
reach_status set_error(reach_ctx* c, reach_status st, const std::string& msg) {
    return fail(c, st, "%s", msg.c_str());
}
reach_status validate_user(reach_ctx* c, const reach_system* s, reach_dtype dtype) {
    return check_system_kind(c, s, dtype, true);
}
void pass_buffers(int64_t passes, bool inplace_ok, bool alias,
                  std::vector<std::pair<int, int>>* io, bool* final_copy) {
    const PassIo b(passes, inplace_ok, alias);
    io->clear();
    for (int64_t p = 0; p < passes; ++p) io->push_back({b.src(p), b.dst(p)});
    *final_copy = b.final_copy();
}

}  // namespace rt
}  // namespace reach
