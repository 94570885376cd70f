// libbsse C ABI: argument checking, payoff packing, device bookkeeping and the chunked sweep
// driver.  Everything numeric happens in the kernels; nothing here evaluates a payoff.
#include "../../include/bsse.h"
#include "bsse_internal.h"

#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <algorithm>
#include <mutex>
#include <vector>

using namespace bsse;

// ------------------------------------------------------------------------------ errors
static thread_local char g_err[320] = "";

static bsse_status fail(bsse_status s, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return s;
}

extern "C" const char *bsse_last_error(void) { return g_err; }

extern "C" const char *bsse_status_name(bsse_status s)
{
    // (a C caller can hand over any integer: read it as one)
    int code;
    memcpy(&code, &s, sizeof(code));
    static_assert(sizeof(code) == sizeof(s), "status codes are ints");
    switch (code) {
    case BSSE_OK: return "BSSE_OK";
    case BSSE_EINVAL: return "BSSE_EINVAL";
    case BSSE_ENOTFINITE: return "BSSE_ENOTFINITE";
    case BSSE_EOVERFLOW: return "BSSE_EOVERFLOW";
    case BSSE_ENOMEM: return "BSSE_ENOMEM";
    case BSSE_EDEVICE: return "BSSE_EDEVICE";
    case BSSE_ESTATE: return "BSSE_ESTATE";
    }
    return "BSSE_?";
}

#define HIP_TRY(call)                                                                         \
    do {                                                                                      \
        hipError_t e_ = (call);                                                               \
        if (e_ != hipSuccess)                                                                 \
            return fail(e_ == hipErrorOutOfMemory ? BSSE_ENOMEM : BSSE_EDEVICE, "%s: %s",     \
                        #call, hipGetErrorString(e_));                                        \
    } while (0)

// ------------------------------------------------------------------------------ handle
constexpr int MAX_FLAGS = 1024;

struct HostOut {            // pinned, device-visible: kernels write results here directly
    RunningBest run;        // the running best itself: read and rewritten by every merge, on the device or (one-call sweeps) here
    float fin_v;            // the winner's value as its re-evaluation gave it
    unsigned epoch;         // small-game kernel: of the current sweep, once a chunk has been recorded into a graph
};

// Device scratch of the prior batch: kept by the handle and grown on demand, so that repeated
// calls do not allocate.
struct PriorScratch {
    float *L = nullptr, *priors = nullptr, *blk_v = nullptr, *rows = nullptr;
    bsse::PriorBest *run = nullptr;
    size_t cap_L = 0, cap_priors = 0, cap_blk_v = 0, cap_rows = 0, cap_run = 0;
    unsigned char *host = nullptr;   // pinned staging: priors on the way in, results on the way out
    size_t cap_host = 0;
    void release()
    {
        if (host) (void)hipHostFree(host);
        (void)hipFree(L); (void)hipFree(priors); (void)hipFree(blk_v); (void)hipFree(rows); (void)hipFree(run);
    }
};

// Device scratch of the top-k entry point: kept by the handle and grown on demand.
struct TopkScratch {
    float *V = nullptr, *rows = nullptr;
    unsigned long long *heads = nullptr;
    size_t cap_V = 0, cap_rows = 0, cap_heads = 0;
    unsigned char *host = nullptr;   // pinned: the records
    size_t cap_host = 0;
    void release()
    {
        if (host) (void)hipHostFree(host);
        (void)hipFree(V); (void)hipFree(rows); (void)hipFree(heads);
    }
};

// Device scratch of bsse_solve_realised, and the payoffs as given to create.
struct RealisedScratch {
    float *V = nullptr, *payoffs = nullptr;
    int32_t *br = nullptr;
    unsigned char *table = nullptr;
    unsigned long long *list = nullptr, *sel = nullptr;
    double *v = nullptr, *x = nullptr;
    int *rc = nullptr;
    size_t cap_V = 0, cap_br = 0, cap_table = 0, cap_list = 0, cap_sel = 0, cap_v = 0, cap_x = 0, cap_rc = 0;
    unsigned char *host = nullptr;   // pinned: the best program
    size_t cap_host = 0;
    void release()
    {
        if (host) (void)hipHostFree(host);
        (void)hipFree(V); (void)hipFree(payoffs); (void)hipFree(br); (void)hipFree(table); (void)hipFree(list);
        (void)hipFree(sel); (void)hipFree(v); (void)hipFree(x); (void)hipFree(rc);
    }
};

// Scratch of the streamed sweep: one record per workgroup of a chunk, the running best, the winning row,
// the tie counter and (small-game kernel) the workgroups' running-best slots.  Owned by the handle and
// grown on demand, or (`fixed`) a carving of the library's static scratch array that cannot grow.  The
// handle's own running best and winning row are the pinned ones (HostOut::run, h_x) and have no second
// copy: a graph of recorded chunks may merge into them at any time, unseen by the host.
struct Work {
    float *blk_v = nullptr;
    long long *blk_i = nullptr;
    long long blk_cap = 0;
    SmallSlot *slots = nullptr;      // slot_sets sets of small_num_slots() slots
    int slot_sets = 0;
    RunningBest *run = nullptr;
    float *best_x = nullptr;
    unsigned long long *tie_counter = nullptr;
    bool fixed = false;
};

struct bsse_game {
    int m = 0, n = 0, K = 0, storage = 0, device = 0;
    PathKind path = PATH_VALU;
    hipStream_t stream = nullptr;
    GameView view{};
    // device allocations
    float *dB = nullptr, *dAT = nullptr, *dprior = nullptr;
    void *dBpack = nullptr, *dATpack = nullptr;
    float *gen = nullptr;
    long long gen_count = -1;
    size_t gen_cap = 0;
    unsigned long long *lat_table = nullptr;
    size_t lat_table_cap = 0;
    int lat_table_N = -1;        // resolution the table on the device was built for (-1: none)
    Work w;                      // the scratch in use
    // small-game kernel: per-workgroup running bests of the current sweep, folded on demand
    unsigned epoch = 0;          // of the current sweep (slots of other epochs are stale)
    // A chunk has been recorded into a graph, whose replays the host does not see: from then on the
    // epoch lives in h_out->epoch, where kernels of the stream advance and read it.
    bool recorded = false;
    // Memory of the handle that recorded calls name (`kept`), and what of it has been replaced since: freed
    // with the handle, for a graph may be replayed as long as that lives.
    std::vector<void *> kept, retired;
    bool fold_pending = false;   // chunks swept since the last fold
    bool fold_first = true;      // the next fold is the first of its sweep
    bool ties_dirty = false;     // the device tie counter may be non-zero
    // Chunks of generated rows need no input from the caller's stream, so after the first chunk of
    // a sweep they alternate between two streams of the handle's own (slot sets 0 and 1; chunks on
    // the caller's stream use set 2): the end of one launch then overlaps the start of the next.
    // Events order them behind the caller's stream (fork) and the fold behind them (join).
    hipStream_t aux[2] = { nullptr, nullptr };
    hipEvent_t aux_fork = nullptr, aux_join[2] = { nullptr, nullptr };
    bool aux_used[2] = { false, false };           // work enqueued since the last join
    unsigned chunk_seq = 0;                        // chunks of the current sweep
    int set_used[3] = { 0, 0, 0 };                 // slots of each set that its chunks may have written
    PriorScratch pri;
    TopkScratch topk;
    RealisedScratch real;
    // host copies of the game as given to create (fp32, unrounded): the profile LP of bsse_polish
    std::vector<float> hA, hB, hprior;
    float *stage = nullptr;                        // generated rows on their way into a sweep
    size_t stage_cap = 0;
    float *centre_dev = nullptr;                   // [.][m] centres of local candidate sets
    size_t cap_centre = 0;
    float *h_centre = nullptr;                     // pinned: the same on the way
    size_t cap_h_centre = 0;
    unsigned char *h_pol = nullptr;                // pinned: rows, values and best responses of bsse_polish
    size_t cap_pol = 0;
    // pinned host memory, one block: what the kernels report
    HostOut *h_out = nullptr;
    unsigned *h_flag = nullptr;             // completion flags [MAX_FLAGS]
    unsigned seq = 0;                       // of the call that last set out to wait for flags
    int32_t *h_br = nullptr;                // the winner's best responses [K]
    float *h_x = nullptr;                   // its row [m]
    float *h_l = nullptr;                   // its per-type leader payoffs [K] (general and any-shape kernel)
    std::vector<float> won_x;               // row and best responses of the result last reported
    std::vector<int32_t> won_br;
    float *row_l = nullptr;                 // per-type outputs of sliced launches, type-major
    int32_t *row_br = nullptr;
    size_t cap_row_l = 0, cap_row_br = 0;
    unsigned char *h_rec = nullptr;         // pinned: records of launch_finish_rows
    size_t cap_rec = 0;
    long long n_evals = 0;
    bool fresh = true;       // the next chunk starts a new sweep
    bool result_valid = false;   // bsse_sweep_result has reported the sweep in the handle's own scratch
    // kernel timing
    bool timing = false;
    std::vector<hipEvent_t> ev;      // start/stop pairs of recorded launches
    std::vector<hipEvent_t> ev_pool; // recycled events
    double timed_ms = 0.0;
    long long timed_launches = 0;
};

namespace {

struct DeviceGuard {
    int prev = -1;
    bool ok = false;
    explicit DeviceGuard(int dev)
    {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        ok = (prev == dev) || hipSetDevice(dev) == hipSuccess;
        if (prev == dev) prev = -1;
    }
    ~DeviceGuard() { if (prev >= 0) (void)hipSetDevice(prev); }
};

float host_round_bf16(float v)
{
    uint32_t b;
    memcpy(&b, &v, 4);
    b += 0x7FFFu + ((b >> 16) & 1u);
    b &= 0xFFFF0000u;
    memcpy(&v, &b, 4);
    return v;
}

// C(N+m-1, m-1) with overflow detection; returns false when it exceeds `cap`.
bool lattice_count_checked(int m, int N, unsigned long long cap, unsigned long long *out)
{
    unsigned long long k = (unsigned long long)(m - 1), a = (unsigned long long)N + k;
    if (k > (unsigned long long)N) k = (unsigned long long)N;       // C(a,k) = C(a,a-k)
    unsigned __int128 c = 1;
    for (unsigned long long i = 1; i <= k; ++i) {
        c = c * (a - k + i) / i;             // exact: a product of i consecutive integers / i!
        if (c > (unsigned __int128)cap) return false;
    }
    *out = (unsigned long long)c;
    return true;
}

constexpr unsigned long long LATTICE_MAX = 1ull << 40;
constexpr long long CHUNK_MAX = 1ll << 31;

void free_game(bsse_game *g)
{
    if (!g) return;
    DeviceGuard dg(g->device);
    (void)hipFree(g->dB); (void)hipFree(g->dAT); (void)hipFree(g->dprior);
    (void)hipFree(g->dBpack); (void)hipFree(g->dATpack);
    (void)hipFree(g->gen); (void)hipFree(g->lat_table);
    (void)hipFree(g->w.blk_v); (void)hipFree(g->w.blk_i); (void)hipFree(g->w.slots);
    (void)hipFree(g->w.tie_counter);
    g->pri.release();
    g->topk.release();
    g->real.release();
    if (g->h_pol) (void)hipHostFree(g->h_pol);
    for (int q = 0; q < 2; ++q) {
        if (g->aux[q]) { (void)hipStreamSynchronize(g->aux[q]); (void)hipStreamDestroy(g->aux[q]); }
        if (g->aux_join[q]) (void)hipEventDestroy(g->aux_join[q]);
    }
    if (g->aux_fork) (void)hipEventDestroy(g->aux_fork);
    (void)hipFree(g->centre_dev); (void)hipFree(g->stage);
    if (g->h_out) (void)hipHostFree(g->h_out);
    if (g->h_rec) (void)hipHostFree(g->h_rec);
    if (g->h_centre) (void)hipHostFree(g->h_centre);
    (void)hipFree(g->row_l); (void)hipFree(g->row_br);
    for (void *q : g->retired) (void)hipFree(q);
    for (hipEvent_t e : g->ev) (void)hipEventDestroy(e);
    for (hipEvent_t e : g->ev_pool) (void)hipEventDestroy(e);
    delete g;
}

// Whether the handle's stream is being captured.  Asynchronous calls then go without the per-type scratch
// (uncut): it cannot be allocated there.
bool recording(const bsse_game *g)
{
    hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(g->stream, &c) != hipSuccess || c != hipStreamCaptureStatusNone;
}

// A call that names `ptr` is being recorded: it stays.
bsse_status keep(bsse_game *g, void *ptr)
{
    if (!ptr || std::find(g->kept.begin(), g->kept.end(), ptr) != g->kept.end()) return BSSE_OK;
    try { g->kept.push_back(ptr); } catch (...) { return fail(BSSE_ENOMEM, "host allocation failed"); }
    return BSSE_OK;
}
bool is_kept(const bsse_game *g, void *ptr) { return std::find(g->kept.begin(), g->kept.end(), ptr) != g->kept.end(); }
// Device memory that the handle has no more use for but that enqueued work or a graph may still use.  (No
// room to note it: it is never freed.)
void retire(bsse_game *g, void *ptr) noexcept
{
    g->kept.erase(std::remove(g->kept.begin(), g->kept.end(), ptr), g->kept.end());
    try { if (ptr) g->retired.push_back(ptr); } catch (...) { }
}
// The same where nothing enqueued still uses it.
void drop(bsse_game *g, void *ptr)
{
    if (is_kept(g, ptr)) retire(g, ptr); else (void)hipFree(ptr);
}
// A larger block for an asynchronous call, which must not wait: at least twice the old one, so that what is
// retired stays below what is used.
bsse_status grow_async(bsse_game *g, void **ptr, size_t *cap, size_t bytes)
{
    if (bytes <= *cap) return BSSE_OK;
    bytes = std::max(bytes, 2 * *cap);
    void *p = nullptr;
    HIP_TRY(hipMalloc(&p, bytes));
    retire(g, *ptr);
    *ptr = p; *cap = bytes;
    return BSSE_OK;
}
// The same for a buffer of candidates that may lie in the handle's generated set.
bsse_status keep_rows(bsse_game *g, const float *X)
{
    const auto *p = reinterpret_cast<const unsigned char *>(X), *gen = reinterpret_cast<const unsigned char *>(g->gen);
    return g->gen && p >= gen && p < gen + g->gen_cap ? keep(g, g->gen) : BSSE_OK;
}

bsse_status ensure_blocks(bsse_game *g, long long nblocks)
{
    if (nblocks <= g->w.blk_cap) return BSSE_OK;
    if (g->w.fixed)
        return fail(BSSE_EOVERFLOW, "%lld workgroup records exceed the %lld the static scratch holds",
                    nblocks, g->w.blk_cap);
    if (recording(g))
        return fail(BSSE_ESTATE, "%lld workgroup records are needed and nothing can be allocated while the stream is captured: "
                    "sweep a chunk of this size before", nblocks);
    size_t cap_v = (size_t)g->w.blk_cap * sizeof(float), cap_i = (size_t)g->w.blk_cap * sizeof(long long);
    g->w.blk_cap = 0;
    bsse_status st = grow_async(g, (void **)&g->w.blk_v, &cap_v, (size_t)nblocks * sizeof(float));
    if (st == BSSE_OK) st = grow_async(g, (void **)&g->w.blk_i, &cap_i, (size_t)nblocks * sizeof(long long));
    if (st == BSSE_OK) g->w.blk_cap = (long long)std::min(cap_v / sizeof(float), cap_i / sizeof(long long));
    return st;
}

bsse_status ensure_gen(bsse_game *g, unsigned long long rows)
{
    const unsigned long long bytes = rows * (unsigned long long)g->m * sizeof(float);
    if (bytes <= g->gen_cap) return BSSE_OK;
    HIP_TRY(hipStreamSynchronize(g->stream));
    drop(g, g->gen);
    g->gen = nullptr; g->gen_cap = 0; g->gen_count = -1;
    size_t free_b = 0, total_b = 0;
    HIP_TRY(hipMemGetInfo(&free_b, &total_b));
    if (bytes > free_b)
        return fail(BSSE_EOVERFLOW, "candidate buffer of %llu bytes exceeds free device memory (%zu)",
                    bytes, free_b);
    HIP_TRY(hipMalloc((void **)&g->gen, (size_t)bytes));
    g->gen_cap = (size_t)bytes;
    return BSSE_OK;
}

bool on_tiny(const bsse_game *g) { return g->path == PATH_VALU && g->view.variant == kTinyVariant; }
bool on_any(const bsse_game *g) { return g->path != PATH_VALU && g->view.variant == kAnyVariant; }

hipError_t launch_sweep_on(bsse_game *g, const SweepArgs &a, bool eval, hipStream_t stream)
{
    if (on_tiny(g)) return launch_sweep_tiny(g->view, a, eval, 1, TinyRecs{}, stream);
    if (g->path == PATH_VALU) return launch_sweep_valu(g->view, a, eval, stream);
    if (on_any(g)) return launch_sweep_any(g->view, a, 1, stream);
    (void)eval;
    return launch_sweep_mfma(g->view, a, stream);
}

hipError_t launch_sweep(bsse_game *g, const SweepArgs &a, bool eval)
{
    return launch_sweep_on(g, a, eval, g->stream);
}

long long sweep_blocks(const bsse_game *g, long long count)
{
    if (on_any(g)) return any_num_blocks(g->view, count);
    if (on_tiny(g)) return tiny_num_blocks(count);
    return g->path == PATH_VALU ? valu_num_blocks(count) : mfma_num_blocks(g->view.variant, count);
}

// Records that `count` candidates or fewer may need uncut (a recorded chunk finds room after a greater one).
long long sweep_records(const bsse_game *g, long long count)
{
    return on_any(g) ? any_max_blocks(g->view, count) : sweep_blocks(g, count);
}

// A block of handle-owned memory of at least `bytes`; nothing enqueued may still use the old one.
bsse_status grow_device(bsse_game *g, void **ptr, size_t *cap, size_t bytes)
{
    if (bytes <= *cap) return BSSE_OK;
    HIP_TRY(hipStreamSynchronize(g->stream));
    drop(g, *ptr);
    *ptr = nullptr; *cap = 0;
    HIP_TRY(hipMalloc(ptr, bytes));
    *cap = bytes;
    return BSSE_OK;
}

bsse_status grow_pinned(bsse_game *g, void **ptr, size_t *cap, size_t bytes)
{
    if (bytes <= *cap) return BSSE_OK;
    HIP_TRY(hipStreamSynchronize(g->stream));
    if (*ptr) (void)hipHostFree(*ptr);
    *ptr = nullptr; *cap = 0;
    if (hipHostMalloc(ptr, bytes, hipHostMallocDefault) != hipSuccess)
        return fail(BSSE_ENOMEM, "hipHostMalloc of %zu bytes failed", bytes);
    memset(*ptr, 0, bytes);                      // (no completion flag is set)
    *cap = bytes;
    return BSSE_OK;
}

// Per-type outputs of a sliced launch: at most this many (64 MiB of leader payoffs).
constexpr long long ROW_SCRATCH_MAX = 1LL << 24;

// Paths whose launches can be cut over the types, and whether `count` rows are few enough for it.
bool cuts_types(const bsse_game *g)
{
    return on_any(g) || on_tiny(g) || (g->path != PATH_VALU && !mfma_is_small(g->view.variant));
}
bool few_rows(const bsse_game *g, long long count)
{
    if (!cuts_types(g) || count * g->K > ROW_SCRATCH_MAX) return false;
    return on_any(g) ? any_shares(g->view, count) > 1
           : on_tiny(g) ? tiny_slices(g->view, count) > 1 : mfma_few_rows(g->view, count);
}

// A launch cut over the types where that pays: a.l_out (and a.br_out) only.
hipError_t launch_rows(bsse_game *g, const SweepArgs &a, hipStream_t stream)
{
    if (on_any(g)) return launch_sweep_any(g->view, a, any_shares(g->view, a.count), stream);
    if (on_tiny(g)) return launch_sweep_tiny(g->view, a, true, tiny_slices(g->view, a.count), TinyRecs{}, stream);
    return launch_sweep_mfma(g->view, a, stream);
}
// Workgroups of such a launch, each with a completion flag.
long long row_blocks(const bsse_game *g, long long count)
{
    return on_any(g) ? any_row_blocks(g->view, count) : on_tiny(g) ? tiny_row_blocks(g->view, count) : mfma_row_blocks(g->view, count);
}

// Per-candidate outputs (a.V_out, a.br_out [count][K], a.l_out with the caller's strides; each nullable).
bsse_status launch_eval(bsse_game *g, SweepArgs a)
{
    a.br_sc = g->K; a.br_st = 1;
    const bool record = recording(g);
    bsse_status st;
    if (record && (st = keep_rows(g, a.X)) != BSSE_OK) return st;
    if (!cuts_types(g)) { HIP_TRY(launch_sweep(g, a, true)); return BSSE_OK; }
    if (!a.V_out && (a.l_out || on_any(g) || on_tiny(g))) { HIP_TRY(launch_rows(g, a, g->stream)); return BSSE_OK; }
    if (a.l_out || !few_rows(g, a.count) || record) {
        HIP_TRY(launch_sweep(g, a, true));
        return BSSE_OK;
    }
    if ((st = grow_async(g, (void **)&g->row_l, &g->cap_row_l, (size_t)a.count * g->K * sizeof(float))) != BSSE_OK) return st;
    FinishRowsArgs f{};
    f.l = g->row_l; f.prior = g->dprior; f.count = a.count; f.K = g->K; f.m = g->m; f.V_out = a.V_out;
    a.V_out = nullptr; a.l_out = g->row_l; a.l_sc = 1; a.l_st = a.count;
    HIP_TRY(launch_rows(g, a, g->stream));
    if (f.V_out) HIP_TRY(launch_finish_rows(f, g->stream));
    return BSSE_OK;
}

// The completion flags of the call's last launch: a sequence number no flag holds yet.
Done new_done(bsse_game *g)
{
    g->seq += 1;
    if (g->seq == 0) g->seq = 1;                 // 0 is the state of a flag never set
    return Done{ g->h_flag, g->seq };
}

// Waits until `n` words, `stride` bytes apart, hold the handle's sequence number.  Polling ends by
// itself: after SPIN_US the stream is synchronised instead, which also reports a failed launch.
constexpr long long SPIN_US = 50000;
bsse_status wait_words(bsse_game *g, const unsigned *word, int n, size_t stride)
{
    const auto *p = reinterpret_cast<const unsigned char *>(word);
    std::chrono::steady_clock::time_point t0{};
    bool started = false, synced = false;
    for (int i = 0; i < n; ++i) {
        const unsigned *w = reinterpret_cast<const unsigned *>(p + (size_t)i * stride);
        for (unsigned k = 1; __atomic_load_n(w, __ATOMIC_ACQUIRE) != g->seq; ++k) {
            if (synced) return fail(BSSE_EDEVICE, "internal: completion flag %d was not set", i);
            __builtin_ia32_pause();
            if (k % 1024 != 0) continue;
            const auto now = std::chrono::steady_clock::now();
            if (!started) { t0 = now; started = true; }
            if (std::chrono::duration_cast<std::chrono::microseconds>(now - t0).count() < SPIN_US) continue;
            HIP_TRY(hipStreamSynchronize(g->stream));
            synced = true;
        }
    }
    return BSSE_OK;
}
bsse_status wait_flags(bsse_game *g, int n) { return wait_words(g, g->h_flag, n, sizeof(unsigned)); }

// Best responses [rows][K] of a few rows into pinned memory, as the last launch of a call (`last`: it
// sets completion flags, *flags of them; 0 when there would be too many).  Values too, if asked for: l
// receives the leader payoffs [rows][K] on paths that are cut over the types (the host sums, value_of),
// V the values on the others.
bsse_status launch_winners(bsse_game *g, const float *X, long long rows, int32_t *br, bool last, int *flags,
                           float *V = nullptr, float *l = nullptr)
{
    SweepArgs a{};
    a.X = X; a.count = rows;
    a.br_out = br; a.br_sc = g->K; a.br_st = 1;
    const long long blocks = cuts_types(g) ? row_blocks(g, rows) : sweep_blocks(g, rows);
    *flags = last && blocks <= MAX_FLAGS ? (int)blocks : 0;
    if (*flags) a.done = new_done(g);
    if (!cuts_types(g)) { a.V_out = V; HIP_TRY(launch_sweep(g, a, true)); return BSSE_OK; }
    a.l_out = l; a.l_sc = g->K; a.l_st = 1;
    if (!on_any(g) && !on_tiny(g) && !l) {       // (the general kernel is cut only when asked for leader payoffs)
        bsse_status st = grow_device(g, (void **)&g->row_l, &g->cap_row_l, (size_t)rows * g->K * sizeof(float));
        if (st != BSSE_OK) return st;
        a.l_out = g->row_l;
    }
    HIP_TRY(launch_rows(g, a, g->stream));
    return BSSE_OK;
}
bsse_status wait_winners(bsse_game *g, int flags)
{
    if (flags) return wait_flags(g, flags);
    HIP_TRY(hipStreamSynchronize(g->stream));
    return BSSE_OK;
}

bsse_status take_event(bsse_game *g, hipEvent_t *e)
{
    if (!g->ev_pool.empty()) { *e = g->ev_pool.back(); g->ev_pool.pop_back(); return BSSE_OK; }
    HIP_TRY(hipEventCreate(e));
    return BSSE_OK;
}

// Wait for everything the handle has enqueued, on the caller's stream and on its own.
bsse_status sync_all(bsse_game *g)
{
    for (int q = 0; q < 2; ++q)
        if (g->aux[q]) { HIP_TRY(hipStreamSynchronize(g->aux[q])); g->aux_used[q] = false; }
    HIP_TRY(hipStreamSynchronize(g->stream));
    return BSSE_OK;
}

bsse_status drain_timing(bsse_game *g)
{
    for (size_t i = 0; i + 1 < g->ev.size(); i += 2) {
        float ms = 0.0f;
        HIP_TRY(hipEventElapsedTime(&ms, g->ev[i], g->ev[i + 1]));
        g->timed_ms += ms;
        g->timed_launches += 1;
    }
    for (hipEvent_t e : g->ev) g->ev_pool.push_back(e);
    g->ev.clear();
    return BSSE_OK;
}

}  // namespace

// ---------------------------------------------------------------------- static scratch
// Scratch of bsse_sweep_static: a file-scope device array, so that the entry point allocates
// nothing.  Every GPU the library runs on holds its own copy (3.2 MiB) until the process ends; the
// array's name is only a host-side stand-in, the device address is looked up once per device with
// hipGetSymbolAddress and that pointer is what kernels and fills are given.
namespace {

constexpr long long STATIC_MAX_BLOCKS = 65536;    // workgroup records of one chunk, as the limit counts them
constexpr long long STATIC_HELD_BLOCKS = 4 * STATIC_MAX_BLOCKS;      // (see mfma_limit_blocks)
constexpr int STATIC_MAX_M = 4096, STATIC_MAX_SLOTS = 2048;
constexpr size_t ST_OFF_RUN = 0, ST_OFF_TIES = 256, ST_OFF_BESTX = 512,
                 ST_OFF_BLKV = ST_OFF_BESTX + (size_t)STATIC_MAX_M * sizeof(float),
                 ST_OFF_BLKI = ST_OFF_BLKV + (size_t)STATIC_HELD_BLOCKS * sizeof(float),
                 ST_OFF_SLOTS = ST_OFF_BLKI + (size_t)STATIC_HELD_BLOCKS * sizeof(long long),
                 STATIC_BYTES = ST_OFF_SLOTS + (size_t)STATIC_MAX_SLOTS * sizeof(SmallSlot);
static_assert(sizeof(RunningBest) <= 256 && sizeof(SmallSlot) == 64, "scratch layout");
static_assert(ST_OFF_BLKV % 256 == 0 && ST_OFF_BLKI % 256 == 0 &&
              ST_OFF_SLOTS % 256 == 0, "scratch parts stay 256-byte aligned");

}  // namespace

static __device__ __align__(256) unsigned char scratch[STATIC_BYTES];

namespace {

constexpr int MAX_DEVICES = 64;
unsigned char *g_scratch_ptr[MAX_DEVICES];      // per device: the address of its copy of `scratch`
std::mutex g_scratch_mutex;

// With device `dev` current: the device address of that device's scratch array (looked up on the
// first call per device).
bsse_status static_scratch(int dev, unsigned char **out)
{
    if (dev < 0 || dev >= MAX_DEVICES) return fail(BSSE_EDEVICE, "device ordinal %d is beyond %d", dev, MAX_DEVICES - 1);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(BSSE_EDEVICE, "hipGetSymbolAddress returned a null address");
        g_scratch_ptr[dev] = static_cast<unsigned char *>(p);
    }
    *out = g_scratch_ptr[dev];
    return BSSE_OK;
}

}  // namespace

// ------------------------------------------------------------------------------ create
extern "C" bsse_status bsse_create(int m, int n, int K, const float *A, const float *B,
                                   const float *prior, bsse_game **out)
{
    bsse_options opt = { BSSE_STORAGE_F32, BSSE_PATH_AUTO, -1 };
    return bsse_create_ex(m, n, K, A, B, prior, &opt, out);
}

extern "C" bsse_status bsse_create_ex(int m, int n, int K, const float *A, const float *B,
                                      const float *prior, const bsse_options *opt,
                                      bsse_game **out)
{
    g_err[0] = 0;
    if (!out) return fail(BSSE_EINVAL, "out is NULL");
    if (!A || !B || !prior) return fail(BSSE_EINVAL, "A, B and prior must not be NULL");
    if (!opt) return fail(BSSE_EINVAL, "opt is NULL");
    if (m < 1 || n < 1 || K < 1) return fail(BSSE_EINVAL, "m, n, K must be >= 1 (got %d, %d, %d)", m, n, K);
    if (m > 4096 || n > 65535 || K > 65535)
        return fail(BSSE_EINVAL, "limits: m <= 4096, n <= 65535, K <= 65535 (got %d, %d, %d)", m, n, K);
    const unsigned long long elems = (unsigned long long)m * n * K;
    if (elems > (1ull << 28)) return fail(BSSE_EINVAL, "K*m*n = %llu exceeds 2^28", elems);
    if (opt->storage != BSSE_STORAGE_F32 && opt->storage != BSSE_STORAGE_BF16)
        return fail(BSSE_EINVAL, "unknown storage option %d", opt->storage);
    if (opt->path != BSSE_PATH_AUTO && opt->path != BSSE_PATH_VALU && opt->path != BSSE_PATH_MFMA &&
        opt->path != BSSE_PATH_MFMA_SPLIT)
        return fail(BSSE_EINVAL, "unknown path option %d", opt->path);
    if (opt->device < -1) return fail(BSSE_EINVAL, "bad device ordinal %d", opt->device);
    for (unsigned long long e = 0; e < elems; ++e)
        if (!std::isfinite(A[e]) || !std::isfinite(B[e]))
            return fail(BSSE_ENOTFINITE, "payoff entry %llu is not finite", e);
    double psum = 0.0;
    for (int t = 0; t < K; ++t) {
        if (!std::isfinite(prior[t])) return fail(BSSE_ENOTFINITE, "prior[%d] is not finite", t);
        if (prior[t] < 0.0f) return fail(BSSE_EINVAL, "prior[%d] is negative", t);
        psum += (double)prior[t];
    }
    if (std::fabs(psum - 1.0) > 1e-6) return fail(BSSE_EINVAL, "prior sums to %.9g, not 1", psum);
    // which kernel family: the small-game kernel, the split path, plain MFMA, else VALU
    const bool bf = opt->storage == BSSE_STORAGE_BF16;
    bool exact = true;                       // every payoff is a bf16 number
    for (unsigned long long e = 0; e < elems && exact; ++e)
        exact = host_round_bf16(A[e]) == A[e] && host_round_bf16(B[e]) == B[e];
    // The three bf16 parts of a number are exact while the smallest of them is not subnormal and the
    // greatest does not round up to infinity.
    const auto in_parts = [](float v) { v = std::fabs(v); return v == 0.0f || (v >= 0x1p-100f && v <= 0x1p120f); };
    int variant = -1;
    PathKind path = PATH_VALU;
    if (opt->path == BSSE_PATH_MFMA_SPLIT) {
        if (bf) return fail(BSSE_EINVAL, "the split path takes fp32 storage");
        variant = mfma_select(m, n, K, 2, exact);
        if (variant < 0) return fail(BSSE_EINVAL, "shape m=%d n=%d K=%d has no split MFMA path", m, n, K);
        path = PATH_MFMA_SPLIT;
    } else if (opt->path == BSSE_PATH_MFMA) {
        variant = mfma_select(m, n, K, bf ? 1 : 0, exact);
        if (variant < 0) return fail(BSSE_EINVAL, "shape m=%d n=%d K=%d has no MFMA path", m, n, K);
        path = bf ? PATH_MFMA_BF16 : PATH_MFMA_F32;
    } else if (opt->path == BSSE_PATH_AUTO) {
        if (bf) {
            variant = mfma_select(m, n, K, 1, exact);
            if (variant >= 0) path = PATH_MFMA_BF16;
        } else {
            if (small_supported(m, n, K, 0)) {
                variant = mfma_select(m, n, K, 0, exact);
                path = PATH_MFMA_F32;
            } else if ((variant = mfma_select(m, n, K, 2, exact)) >= 0) {
                path = PATH_MFMA_SPLIT;
            } else if ((variant = mfma_select(m, n, K, 0, exact)) >= 0) {
                path = PATH_MFMA_F32;
            }
        }
        // every other shape the matrix cores pay for, tiles padded as needed; payoffs near the ends of
        // the fp32 range stay on the vector unit
        bool ordinary = path == PATH_VALU && any_supported(m, n);
        for (unsigned long long e = 0; e < elems && ordinary; ++e) ordinary = in_parts(A[e]) && in_parts(B[e]);
        if (ordinary) {
            variant = kAnyVariant;
            path = bf ? PATH_MFMA_BF16 : PATH_MFMA_SPLIT;
        }
    }
    const bool use_mfma = path != PATH_VALU;

    // ---- device
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1)
        return fail(BSSE_EDEVICE, "no HIP device is visible");
    int dev = opt->device;
    if (dev < 0 && hipGetDevice(&dev) != hipSuccess) return fail(BSSE_EDEVICE, "hipGetDevice failed");
    if (dev >= ndev) return fail(BSSE_EINVAL, "device %d of %d does not exist", dev, ndev);
    hipDeviceProp_t prop;
    HIP_TRY(hipGetDeviceProperties(&prop, dev));
    if (strncmp(prop.gcnArchName, "gfx950", 6) != 0)
        return fail(BSSE_EDEVICE, "device %d is %s; this library holds gfx950 code only", dev,
                    prop.gcnArchName);

    bsse_game *g = new (std::nothrow) bsse_game;
    if (!g) return fail(BSSE_ENOMEM, "host allocation failed");
    g->m = m; g->n = n; g->K = K; g->storage = opt->storage; g->device = dev;
    g->path = path;
    bool half = false;
    try {
        g->hA.assign(A, A + elems); g->hB.assign(B, B + elems); g->hprior.assign(prior, prior + K);
        g->hprior.resize((size_t)2 * K, 0.0f);          // (the filter's margins behind it)
        if (use_mfma) variant = mfma_filter(variant, m, n, K, A, B, g->hprior.data() + K);
        half = variant == kAnyVariant && !bf && !exact && any_half_suits(m, n, K, B);
        g->won_x.resize((size_t)m); g->won_br.resize((size_t)K);
    } catch (...) { delete g; return fail(BSSE_ENOMEM, "host allocation failed"); }
    g->view.variant = variant;
    if (mfma_is_six_bit(variant)) g->view.any.row_end = row_end_of(elems, B);

    DeviceGuard dg(dev);
    if (!dg.ok) { free_game(g); return fail(BSSE_EDEVICE, "hipSetDevice(%d) failed", dev); }

    // ---- vector path: pack on the host: optional bf16 rounding, B as given, A transposed per type
    // (short rows: both transposed, padded with zeros)
    std::vector<float> hB, hAT;
    const int tiny = use_mfma ? 0 : tiny_pad(m);
    if (tiny) {
        g->view.variant = kTinyVariant;
        hB.assign((size_t)K * n * tiny, 0.0f); hAT.assign((size_t)K * n * tiny, 0.0f);
        for (int t = 0; t < K; ++t)
            for (int i = 0; i < m; ++i)
                for (int j = 0; j < n; ++j) {
                    const size_t from = ((size_t)t * m + i) * n + j, to = ((size_t)t * n + j) * tiny + i;
                    hB[to] = bf ? host_round_bf16(B[from]) : B[from];
                    hAT[to] = bf ? host_round_bf16(A[from]) : A[from];
                }
    } else if (!use_mfma) {
        hB.resize(elems); hAT.resize(elems);
        for (unsigned long long e = 0; e < elems; ++e) hB[e] = bf ? host_round_bf16(B[e]) : B[e];
        for (int t = 0; t < K; ++t)
            for (int i = 0; i < m; ++i)
                for (int j = 0; j < n; ++j) {
                    const float a = A[((size_t)t * m + i) * n + j];
                    hAT[((size_t)t * n + j) * m + i] = bf ? host_round_bf16(a) : a;
                }
    }

    bsse_status st = BSSE_OK;
    auto up = [&](void **dst, const void *src, size_t bytes) -> bsse_status {
        HIP_TRY(hipMalloc(dst, bytes));
        HIP_TRY(hipMemcpy(*dst, src, bytes, hipMemcpyHostToDevice));
        return BSSE_OK;
    };
    auto zeroed = [&](void **dst, size_t bytes) -> bsse_status {
        HIP_TRY(hipMalloc(dst, bytes));
        HIP_TRY(hipMemset(*dst, 0, bytes));
        return BSSE_OK;
    };
    do {
        if (!use_mfma && (st = up((void **)&g->dB, hB.data(), hB.size() * 4)) != BSSE_OK) break;
        if (!use_mfma && (st = up((void **)&g->dAT, hAT.data(), hAT.size() * 4)) != BSSE_OK) break;
        if ((st = up((void **)&g->dprior, g->hprior.data(), g->hprior.size() * 4)) != BSSE_OK) break;
        g->view.m = m; g->view.n = n; g->view.K = K;
        g->view.m_pad = tiny ? tiny : m; g->view.n_pad = n;
        if (use_mfma && variant == kAnyVariant) {
            // packed on the device from the payoffs as given
            g->view.any = any_geometry(m, n, K, bf ? 1 : exact ? 3 : half ? 2 : 6);
            if (half) g->view.any.row_end = row_end_of(elems, B);
            size_t bb = 0, ab = 0;
            any_pack_sizes(g->view, &bb, &ab);
            float *rawA = nullptr, *rawB = nullptr, *scale = nullptr;
            st = up((void **)&rawA, A, elems * 4);
            if (st == BSSE_OK) st = up((void **)&rawB, B, elems * 4);
            hipError_t pe = hipSuccess;
            if (st == BSSE_OK && half) pe = hipMalloc((void **)&scale, (size_t)K * 4);
            if (st == BSSE_OK && pe == hipSuccess && (pe = hipMalloc(&g->dBpack, bb)) == hipSuccess && (pe = hipMalloc(&g->dATpack, ab)) == hipSuccess &&
                (pe = launch_any_pack(g->view, rawA, rawB, g->dBpack, g->dATpack, g->dprior + K, scale, nullptr)) == hipSuccess &&
                (pe = hipStreamSynchronize(nullptr)) == hipSuccess)
                pe = any_prepare(g->view);
            (void)hipFree(rawA); (void)hipFree(rawB); (void)hipFree(scale);
            if (st == BSSE_OK && pe != hipSuccess)
                st = fail(pe == hipErrorOutOfMemory ? BSSE_ENOMEM : BSSE_EDEVICE, "packing: %s", hipGetErrorString(pe));
            if (st != BSSE_OK) break;
        } else if (use_mfma) {
            void *pb = nullptr, *pa = nullptr;
            size_t bb = 0, ab = 0;
            mfma_pack(variant, m, n, K, A, B, &pb, &bb, &pa, &ab, &g->view.m_pad, &g->view.n_pad);
            if (!pb || !pa) { free(pb); free(pa); st = fail(BSSE_ENOMEM, "host allocation failed"); break; }
            st = up(&g->dBpack, pb, bb);
            if (st == BSSE_OK) st = up(&g->dATpack, pa, ab);
            free(pb); free(pa);
            if (st != BSSE_OK) break;
            hipError_t pe = mfma_prepare(variant);
            if (pe != hipSuccess) { st = fail(BSSE_EDEVICE, "mfma_prepare: %s", hipGetErrorString(pe)); break; }
        }
        if ((st = zeroed((void **)&g->w.tie_counter, 8)) != BSSE_OK) break;
        if (use_mfma && mfma_is_small(variant) &&       // epoch 0 marks a slot never written
            (st = zeroed((void **)&g->w.slots, (size_t)3 * small_num_slots() * sizeof(SmallSlot))) != BSSE_OK) break;
        g->w.slot_sets = g->w.slots ? 3 : 0;
        const size_t off_flag = 256, off_br = off_flag + MAX_FLAGS * sizeof(unsigned), off_l = off_br + (size_t)K * 4,
                     off_x = (off_l + (size_t)K * 4 + 63) / 64 * 64, host_bytes = off_x + (size_t)m * 4;     // (an aligned row)
        static_assert(sizeof(HostOut) <= 256, "the flags start behind it");
        hipError_t e = hipHostMalloc((void **)&g->h_out, host_bytes, hipHostMallocDefault);
        if (e != hipSuccess) { st = fail(BSSE_ENOMEM, "hipHostMalloc: %s", hipGetErrorString(e)); break; }
        unsigned char *hb = reinterpret_cast<unsigned char *>(g->h_out);
        memset(hb, 0, host_bytes);
        g->h_flag = reinterpret_cast<unsigned *>(hb + off_flag);
        g->h_br = reinterpret_cast<int32_t *>(hb + off_br);
        g->h_l = reinterpret_cast<float *>(hb + off_l);
        g->h_x = reinterpret_cast<float *>(hb + off_x);
        g->w.run = &g->h_out->run; g->w.best_x = g->h_x;
    } while (0);
    if (st != BSSE_OK) { free_game(g); return st; }

    {   // set-up of the static scratch for this device (bsse_sweep_static reports a failure itself)
        unsigned char *unused = nullptr;
        (void)static_scratch(dev, &unused);
        g_err[0] = 0;
    }
    g->view.m = m; g->view.n = n; g->view.K = K;
    g->view.x_bf16 = bf ? 1 : 0;
    g->view.B = g->dB; g->view.AT = g->dAT; g->view.prior = g->dprior;
    g->view.Bpack = g->dBpack; g->view.ATpack = g->dATpack;
    *out = g;
    return BSSE_OK;
}

extern "C" void bsse_destroy(bsse_game *g)
{
    if (!g) return;
    {
        DeviceGuard dg(g->device);
        (void)sync_all(g);
    }
    free_game(g);
}

extern "C" bsse_status bsse_set_stream(bsse_game *g, void *hip_stream)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    DeviceGuard dg(g->device);
    bsse_status st = sync_all(g);                 // earlier work keeps its order
    if (st != BSSE_OK) return st;
    g->stream = (hipStream_t)hip_stream;
    return BSSE_OK;
}

extern "C" const char *bsse_path_name(const bsse_game *g)
{
    if (!g) return "";
    switch (g->path) {
    case PATH_VALU: return g->storage == BSSE_STORAGE_BF16 ? "valu_bf16" : "valu";
    case PATH_MFMA_F32:
    case PATH_MFMA_BF16:
    case PATH_MFMA_SPLIT: return on_any(g) ? any_name(g->view.any) : mfma_variant_name(g->view.variant);
    }
    return "";
}

// --------------------------------------------------------------------------- generation
extern "C" bsse_status bsse_lattice_count(int m, int N, int64_t *count_out)
{
    g_err[0] = 0;
    if (!count_out) return fail(BSSE_EINVAL, "count_out is NULL");
    if (m < 1 || m > 4096) return fail(BSSE_EINVAL, "m must be in 1..4096 (got %d)", m);
    if (N < 1 || N > (1 << 24)) return fail(BSSE_EINVAL, "N must be in 1..2^24 (got %d)", N);
    unsigned long long c = 0;
    if (!lattice_count_checked(m, N, LATTICE_MAX, &c))
        return fail(BSSE_EOVERFLOW, "lattice of resolution %d in %d parts has more than 2^40 points", N, m);
    *count_out = (int64_t)c;
    return BSSE_OK;
}

namespace {

// centre (host [m]) and radius of a local set: validated, the centre uploaded to the handle
bsse_status check_around(const bsse_game *g, const float *centre, float radius)
{
    if (!centre) return fail(BSSE_EINVAL, "centre is NULL");
    if (!(radius >= 0.0f && radius <= 1.0f)) return fail(BSSE_EINVAL, "radius %g outside 0..1", (double)radius);
    for (int i = 0; i < g->m; ++i)
        if (!std::isfinite(centre[i])) return fail(BSSE_ENOTFINITE, "centre[%d] is not finite", i);
    return BSSE_OK;
}

bsse_status upload_centre(bsse_game *g, const float *centre)
{
    bsse_status st = grow_device(g, (void **)&g->centre_dev, &g->cap_centre, (size_t)g->m * sizeof(float));
    if (st != BSSE_OK) return st;
    HIP_TRY(hipMemcpyAsync(g->centre_dev, centre, (size_t)g->m * sizeof(float), hipMemcpyHostToDevice, g->stream));
    HIP_TRY(hipStreamSynchronize(g->stream));          // the host array is the caller's again
    return BSSE_OK;
}

bsse_status lattice_impl(bsse_game *g, int N, const float *centre, float radius, int64_t *count_out);

}  // namespace

extern "C" bsse_status bsse_lattice(bsse_game *g, int N, int64_t *count_out)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    if (!count_out) return fail(BSSE_EINVAL, "count_out is NULL");
    return lattice_impl(g, N, nullptr, 1.0f, count_out);
}

extern "C" bsse_status bsse_lattice_around(bsse_game *g, int N, const float *centre, float radius,
                                           int64_t *count_out)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    if (!count_out) return fail(BSSE_EINVAL, "count_out is NULL");
    bsse_status st = check_around(g, centre, radius);
    if (st != BSSE_OK) return st;
    return lattice_impl(g, N, centre, radius, count_out);
}

namespace {

// The table of resolution N on the device (which is current).
bsse_status ensure_lattice_table(bsse_game *g, int N)
{
    const int m = g->m;
    const size_t tab_elems = (size_t)(m + 1) * (N + 1);
    if (tab_elems > (1ull << 27)) return fail(BSSE_EOVERFLOW, "lattice table of %zu entries is too large", tab_elems);
    if (g->lat_table_N != N) {                    // (the table of the last resolution stays on the device)
        // W(R,q) = C(R+q-1, q-1) for q = 0..m, R = 0..N by Pascal's rule; every entry <= cnt
        std::vector<unsigned long long> tab(tab_elems, 0ull);
        for (int q = 1; q <= m; ++q)
            for (int R = 0; R <= N; ++R) {
                unsigned long long v;
                if (q == 1 || R == 0) v = 1;
                else v = tab[(size_t)q * (N + 1) + R - 1] + tab[(size_t)(q - 1) * (N + 1) + R];
                tab[(size_t)q * (N + 1) + R] = v;
            }
        g->lat_table_N = -1;
        if (tab_elems * 8 > g->lat_table_cap || is_kept(g, g->lat_table)) {
            HIP_TRY(hipStreamSynchronize(g->stream));
            drop(g, g->lat_table);
            g->lat_table = nullptr; g->lat_table_cap = 0;
            HIP_TRY(hipMalloc((void **)&g->lat_table, tab_elems * 8));
            g->lat_table_cap = tab_elems * 8;
        }
        HIP_TRY(hipMemcpyAsync(g->lat_table, tab.data(), tab_elems * 8, hipMemcpyHostToDevice, g->stream));
        HIP_TRY(hipStreamSynchronize(g->stream));     // `tab` is pageable and dies with this block
        g->lat_table_N = N;
    }
    return BSSE_OK;
}

bsse_status lattice_impl(bsse_game *g, int N, const float *centre, float radius, int64_t *count_out)
{
    int64_t cnt = 0;
    bsse_status st = bsse_lattice_count(g->m, N, &cnt);
    if (st != BSSE_OK) return st;
    const int m = g->m;
    DeviceGuard dg(g->device);
    if (!dg.ok) return fail(BSSE_EDEVICE, "hipSetDevice failed");
    if ((st = ensure_gen(g, (unsigned long long)cnt)) != BSSE_OK) return st;
    if ((st = ensure_lattice_table(g, N)) != BSSE_OK) return st;
    if (centre && (st = upload_centre(g, centre)) != BSSE_OK) return st;
    if (recording(g) && ((st = keep(g, g->gen)) != BSSE_OK || (st = keep(g, g->lat_table)) != BSSE_OK)) return st;
    HIP_TRY(launch_lattice(g->lat_table, m, N, cnt, centre ? g->centre_dev : nullptr, radius, 1, g->gen, g->stream));
    g->gen_count = cnt;
    *count_out = cnt;
    return BSSE_OK;
}

bsse_status dirichlet_impl(bsse_game *g, uint64_t seed, int64_t first, int64_t count, const float *centre,
                           float radius, float *out_dev);

}  // namespace

extern "C" bsse_status bsse_dirichlet(bsse_game *g, uint64_t seed, int64_t first, int64_t count,
                                      float *out_dev)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    return dirichlet_impl(g, seed, first, count, nullptr, 1.0f, out_dev);
}

extern "C" bsse_status bsse_dirichlet_around(bsse_game *g, uint64_t seed, int64_t first, int64_t count,
                                             const float *centre, float radius, float *out_dev)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    bsse_status st = check_around(g, centre, radius);
    if (st != BSSE_OK) return st;
    return dirichlet_impl(g, seed, first, count, centre, radius, out_dev);
}

namespace {

bsse_status dirichlet_impl(bsse_game *g, uint64_t seed, int64_t first, int64_t count, const float *centre,
                           float radius, float *out_dev)
{
    if (first < 0 || count < 0) return fail(BSSE_EINVAL, "first and count must be >= 0");
    if (count > CHUNK_MAX) return fail(BSSE_EOVERFLOW, "count exceeds 2^31 rows per call");
    if (first > INT64_MAX - count) return fail(BSSE_EOVERFLOW, "first + count overflows");
    DeviceGuard dg(g->device);
    if (!dg.ok) return fail(BSSE_EDEVICE, "hipSetDevice failed");
    float *dst = out_dev;
    if (!dst) {
        bsse_status st = ensure_gen(g, (unsigned long long)count);
        if (st != BSSE_OK) return st;
        dst = g->gen;
        if (recording(g) && (st = keep(g, dst)) != BSSE_OK) return st;
    }
    if (centre) {
        bsse_status st = upload_centre(g, centre);
        if (st != BSSE_OK) return st;
    }
    HIP_TRY(launch_dirichlet(seed, first, count, g->m, centre ? g->centre_dev : nullptr, radius, 1, dst, g->stream));
    if (!out_dev) g->gen_count = count;
    return BSSE_OK;
}

}  // namespace

extern "C" bsse_status bsse_candidates(bsse_game *g, const float **dev_out, int64_t *count_out)
{
    g_err[0] = 0;
    if (!g || !dev_out || !count_out) return fail(BSSE_EINVAL, "NULL argument");
    if (g->gen_count < 0) return fail(BSSE_ESTATE, "no candidate set has been generated on this handle");
    *dev_out = g->gen;
    *count_out = g->gen_count;
    return BSSE_OK;
}

// -------------------------------------------------------------------------------- sweep
extern "C" bsse_status bsse_sweep_reset(bsse_game *g)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    DeviceGuard dg(g->device);
    if (!dg.ok) return fail(BSSE_EDEVICE, "hipSetDevice failed");
    g->fresh = true;          // consumed by the merge kernel of the next chunk: no launch here
    g->result_valid = false;
    g->n_evals = 0;
    return BSSE_OK;
}

static bsse_status resolve_candidates(bsse_game *g, const float **X, int64_t *count)
{
    if (*count < 0) return fail(BSSE_EINVAL, "count must be >= 0");
    if (!*X) {
        if (g->gen_count < 0)
            return fail(BSSE_ESTATE, "candidates is NULL but no set has been generated on this handle");
        if (*count != 0 && *count != g->gen_count)
            return fail(BSSE_EINVAL, "count %lld does not match the generated set (%lld)",
                        (long long)*count, g->gen_count);
        *X = g->gen;
        *count = g->gen_count;
    }
    if (*count > CHUNK_MAX) return fail(BSSE_EOVERFLOW, "count exceeds 2^31 rows per call");
    const uintptr_t need = (g->m % 4 == 0) ? 15 : 3;      // whole rows of 16 bytes keep 16-byte alignment
    if (((uintptr_t)*X & need) != 0)
        return fail(BSSE_EINVAL, "candidates must be %d-byte aligned", (int)need + 1);
    return BSSE_OK;
}

namespace {

// One chunk through the sweep kernel and the merge into the running best.  a.X / a.gen*, a.count
// and a.index_base are set by the caller; the device is current.
bool on_small_kernel(const bsse_game *g)
{
    return g->path != PATH_VALU && mfma_is_small(g->view.variant);
}

// The value of a re-evaluated winner on the any-shape path, from its per-type leader payoffs: the
// kernel's own sum, term by term.
float value_of(const bsse_game *g, const float *l)
{
    float v = 0.0f;
    for (int t = 0; t < g->K; ++t) v = std::fmaf(g->hprior[t], l[t], v);
    return v == v ? v : -INFINITY;               // (as the kernels report it)
}

// The caller's stream waits for whatever the handle's own streams still have in flight.
bsse_status join_aux(bsse_game *g)
{
    for (int q = 0; q < 2; ++q) {
        if (!g->aux_used[q]) continue;
        HIP_TRY(hipEventRecord(g->aux_join[q], g->aux[q]));
        HIP_TRY(hipStreamWaitEvent(g->stream, g->aux_join[q], 0));
        g->aux_used[q] = false;
    }
    return BSSE_OK;
}

bsse_status ensure_aux(bsse_game *g)
{
    if (g->aux[0]) return BSSE_OK;
    HIP_TRY(hipEventCreateWithFlags(&g->aux_fork, hipEventDisableTiming));
    for (int q = 0; q < 2; ++q) {
        HIP_TRY(hipStreamCreateWithFlags(&g->aux[q], hipStreamNonBlocking));     // default priority
        HIP_TRY(hipEventCreateWithFlags(&g->aux_join[q], hipEventDisableTiming));
    }
    return BSSE_OK;
}

bsse_status sweep_chunk_impl(bsse_game *g, SweepArgs a)
{
    bsse_status st;
    const long long count = a.count;
    const bool small = on_small_kernel(g);
    long long nblocks = 0;
    hipStream_t stream = g->stream;
    const bool record = recording(g);
    const bool rows = !small && !g->w.fixed && few_rows(g, count) && !record;     // (the static scratch holds records only)
    if (record && a.X && (st = a.X == g->stage ? keep(g, g->stage) : keep_rows(g, a.X)) != BSSE_OK) return st;
    FinishRowsArgs f{};
    if (small) {
        // every workgroup keeps its own running best over the chunks: nothing but the sweep
        // kernel runs per chunk; bsse_sweep_result folds
        if (record && !g->recorded) { g->h_out->epoch = g->epoch; g->recorded = true; }
        if (g->fresh) {
            if ((st = join_aux(g)) != BSSE_OK) return st;        // an abandoned sweep may still be running
            g->epoch += 1;
            if (g->epoch == 0) g->epoch = 1;         // 0 is the mark of a slot never written
            g->fold_first = !g->recorded;
            g->chunk_seq = 0;
            if (g->recorded) {                       // (and a replay may still write any slot that a recorded chunk writes)
                HIP_TRY(launch_new_epoch(&g->h_out->epoch, g->w.tie_counter, g->w.run, g->stream));
            } else {
                g->set_used[0] = g->set_used[1] = g->set_used[2] = 0;
                if (g->ties_dirty) HIP_TRY(launch_clear_u64(g->w.tie_counter, g->stream));   // an abandoned sweep's
            }
        }
        int set = g->w.slot_sets - 1;                // the caller's stream (the last set)
        if (a.gen && g->chunk_seq > 0 && g->w.slot_sets == 3 && !record) {
            // (the first chunk stays on the caller's stream, so a one-chunk sweep pays for no events)
            if ((st = ensure_aux(g)) != BSSE_OK) return st;
            set = (int)(g->chunk_seq & 1u);
            if (!g->aux_used[set]) {
                HIP_TRY(hipEventRecord(g->aux_fork, g->stream));
                HIP_TRY(hipStreamWaitEvent(g->aux[set], g->aux_fork, 0));
                g->aux_used[set] = true;
            }
            stream = g->aux[set];
        }
        g->chunk_seq += 1;
        g->set_used[set] = std::max(g->set_used[set], (int)sweep_blocks(g, count));
        a.small.slots = g->w.slots + (size_t)set * small_num_slots(); a.small.epoch = g->epoch;
        a.small.epoch_now = g->recorded ? &g->h_out->epoch : nullptr;
        a.tie_counter = g->w.tie_counter;
    } else {
        nblocks = rows ? (count + FINISH_ROWS - 1) / FINISH_ROWS : sweep_blocks(g, count);
        // (enough for the same chunk uncut, as it is recorded)
        if ((st = ensure_blocks(g, std::max(nblocks, sweep_records(g, count)))) != BSSE_OK) return st;
        if (record && ((st = keep(g, g->w.blk_v)) != BSSE_OK || (st = keep(g, g->w.blk_i)) != BSSE_OK)) return st;
        a.tie_counter = g->w.tie_counter;
        if (rows) {
            if ((st = grow_async(g, (void **)&g->row_l, &g->cap_row_l, (size_t)count * g->K * sizeof(float))) != BSSE_OK) return st;
            a.l_out = g->row_l; a.l_sc = 1; a.l_st = count;
            f.l = g->row_l; f.prior = g->dprior; f.count = count; f.index_base = a.index_base; f.K = g->K; f.m = g->m;
            f.blk_v = g->w.blk_v; f.blk_i = g->w.blk_i;
        } else {
            a.blk_v = g->w.blk_v; a.blk_i = g->w.blk_i;
        }
    }
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (g->timing) {
        if ((st = take_event(g, &e0)) != BSSE_OK) return st;
        if ((st = take_event(g, &e1)) != BSSE_OK) { g->ev_pool.push_back(e0); return st; }
        HIP_TRY(hipEventRecord(e0, stream));
    }
    hipError_t le = rows ? launch_rows(g, a, stream) : launch_sweep_on(g, a, false, stream);
    if (g->timing) {
        (void)hipEventRecord(e1, stream);
        g->ev.push_back(e0); g->ev.push_back(e1);
    }
    HIP_TRY(le);
    if (small) {
        g->fold_pending = true; g->ties_dirty = true;
    } else {
        if (rows) HIP_TRY(launch_finish_rows(f, g->stream));
        HIP_TRY(launch_reduce_merge(g->w.blk_v, g->w.blk_i, nblocks, a.X, a.index_base, g->m,
                                    g->fresh ? 1 : 0, g->w.tie_counter, g->w.run, &g->h_out->run, g->w.best_x,
                                    g->h_x, g->stream));
    }
    g->fresh = false;
    g->result_valid = false;  // until bsse_sweep_result has brought the new state to the host
    g->n_evals += count * g->K;
    return BSSE_OK;
}

// Waits for the handle's stream by a one-thread kernel whose flag is polled.
bsse_status wait_stream(bsse_game *g)
{
    HIP_TRY(launch_signal(new_done(g), g->stream));
    return wait_flags(g, 1);
}

// Small-game kernel: fold the workgroups' running bests into the handle's result (value, index,
// row, best responses, tie count) and wait for it; for the stream alone when nothing can have been swept
// since the last fold.
bsse_status fold_small(bsse_game *g)
{
    if (!g->fold_pending && !g->recorded) return wait_stream(g);
    bsse_status st = join_aux(g);
    if (st != BSSE_OK) return st;
    FinishArgs f{};
    f.slots = g->w.slots; f.epoch = g->epoch; f.epoch_now = g->recorded ? &g->h_out->epoch : nullptr;
    for (int q = 0; q < 3; ++q) f.used[q] = g->set_used[q];
    f.first = g->fold_first ? 1 : 0;
    f.tie_counter = g->w.tie_counter;
    f.run = g->w.run; f.run_host = &g->h_out->run; f.x_host = g->h_x;
    f.win_v = &g->h_out->fin_v; f.win_br = g->h_br;
    f.done = new_done(g);
    HIP_TRY(launch_finish_small(g->view, f, g->stream));
    g->fold_pending = false; g->fold_first = false; g->ties_dirty = false;
    return wait_flags(g, 1);
}

bool fuses_generation(const bsse_game *g) { return on_small_kernel(g); }

// Rows of the staging buffer generated candidates pass through (at most 2^26 floats).
long long stage_rows(const bsse_game *g) { return (1LL << 26) / g->m; }

bsse_status check_rows(int64_t first, int64_t count)
{
    if (first < 0 || count < 0) return fail(BSSE_EINVAL, "first and count must be >= 0");
    if (count > CHUNK_MAX) return fail(BSSE_EOVERFLOW, "count exceeds 2^31 rows per call");
    if (first > INT64_MAX - count) return fail(BSSE_EOVERFLOW, "first + count overflows");
    return BSSE_OK;
}

}  // namespace

extern "C" bsse_status bsse_sweep_chunk(bsse_game *g, const float *candidates_dev, int64_t count,
                                        int64_t index_base)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    if (index_base < 0) return fail(BSSE_EINVAL, "index_base must be >= 0");
    bsse_status st = resolve_candidates(g, &candidates_dev, &count);
    if (st != BSSE_OK) return st;
    if (index_base > INT64_MAX - count) return fail(BSSE_EOVERFLOW, "index_base + count overflows");
    if (count == 0) return BSSE_OK;
    DeviceGuard dg(g->device);
    if (!dg.ok) return fail(BSSE_EDEVICE, "hipSetDevice failed");
    SweepArgs a{};
    a.X = candidates_dev; a.count = count; a.index_base = index_base;
    return sweep_chunk_impl(g, a);
}

extern "C" bsse_status bsse_sweep_dirichlet_chunk(bsse_game *g, uint64_t seed, int64_t first,
                                                  int64_t count, int64_t index_base)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    if (index_base < 0) return fail(BSSE_EINVAL, "index_base must be >= 0");
    bsse_status st = check_rows(first, count);
    if (st != BSSE_OK) return st;
    if (index_base > INT64_MAX - count) return fail(BSSE_EOVERFLOW, "index_base + count overflows");
    if (count == 0) return BSSE_OK;
    DeviceGuard dg(g->device);
    if (!dg.ok) return fail(BSSE_EDEVICE, "hipSetDevice failed");
    if (fuses_generation(g)) {
        SweepArgs a{};
        a.count = count; a.index_base = index_base;
        a.gen = 1; a.gen_k0 = (unsigned)(seed & 0xFFFFFFFFull); a.gen_k1 = (unsigned)(seed >> 32);
        a.gen_first = first;
        return sweep_chunk_impl(g, a);
    }
    // other shapes: the rows pass through a staging buffer of the handle (at most 2^26 floats),
    // piece by piece on the handle's stream
    const long long piece = count < stage_rows(g) ? count : stage_rows(g);
    if ((st = grow_device(g, (void **)&g->stage, &g->stage_cap, (size_t)piece * g->m * sizeof(float))) != BSSE_OK) return st;
    for (long long base = 0; base < count; base += piece) {
        const long long rows = count - base < piece ? count - base : piece;
        HIP_TRY(launch_dirichlet(seed, first + base, rows, g->m, nullptr, 1.0f, 1, g->stage, g->stream));
        SweepArgs a{};
        a.X = g->stage; a.count = rows; a.index_base = index_base + base;
        if ((st = sweep_chunk_impl(g, a)) != BSSE_OK) return st;
    }
    return BSSE_OK;
}

namespace {
bool sweeps_at_once(const bsse_game *g, long long count);
bsse_status sweep_once(bsse_game *g, const float *X, long long count, bsse_result *res, int32_t *best_response_out);
}

extern "C" bsse_status bsse_sweep_dirichlet(bsse_game *g, uint64_t seed, int64_t first, int64_t count,
                                            bsse_result *res, int32_t *best_response_out)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    if (!res) return fail(BSSE_EINVAL, "res is NULL");
    bsse_status st = check_rows(first, count);
    if (st != BSSE_OK) return st;
    if ((st = bsse_sweep_reset(g)) != BSSE_OK) return st;
    if (sweeps_at_once(g, count) && count <= stage_rows(g)) {
        DeviceGuard dg(g->device);
        if (!dg.ok) return fail(BSSE_EDEVICE, "hipSetDevice failed");
        if ((st = grow_device(g, (void **)&g->stage, &g->stage_cap, (size_t)count * g->m * sizeof(float))) != BSSE_OK) return st;
        HIP_TRY(launch_dirichlet(seed, first, count, g->m, nullptr, 1.0f, 1, g->stage, g->stream));
        return sweep_once(g, g->stage, count, res, best_response_out);
    }
    if ((st = bsse_sweep_dirichlet_chunk(g, seed, first, count, 0)) != BSSE_OK) return st;
    return bsse_sweep_result(g, res, best_response_out);
}

namespace {
bsse_status report_result(bsse_game *g, bsse_result *res, int32_t *best_response_out);
}

extern "C" bsse_status bsse_sweep_result(bsse_game *g, bsse_result *res, int32_t *best_response_out)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    if (!res) return fail(BSSE_EINVAL, "res is NULL");
    DeviceGuard dg(g->device);
    if (!dg.ok) return fail(BSSE_EDEVICE, "hipSetDevice failed");
    if (g->fresh) {                        // nothing swept since the last reset
        HIP_TRY(hipStreamSynchronize(g->stream));
        res->best_value = 0.0; res->best_index = -1; res->n_evals = 0; res->n_tie_evals = 0;
        return BSSE_OK;
    }
    // best responses of the winner: the same kernel, one row, per-candidate outputs written
    // straight into pinned host memory (the small-game kernel carries them with its records)
    bsse_status st = BSSE_OK;
    if (on_small_kernel(g)) {
        st = fold_small(g);
    } else {
        SweepArgs a{};
        a.X = g->w.best_x; a.count = 1;
        a.br_out = g->h_br; a.br_sc = g->K; a.br_st = 1;
        a.done = new_done(g);
        if (cuts_types(g)) {
            // one row against every type: the types are spread over the chip, and the host sums
            a.l_out = g->h_l; a.l_sc = g->K; a.l_st = 1;
            HIP_TRY(launch_rows(g, a, g->stream));
            if ((st = wait_flags(g, (int)row_blocks(g, 1))) == BSSE_OK && g->h_out->run.has) g->h_out->fin_v = value_of(g, g->h_l);
        } else {
            a.V_out = &g->h_out->fin_v;
            HIP_TRY(launch_sweep(g, a, true));
            st = wait_flags(g, 1);
        }
    }
    if (st != BSSE_OK) return st;
    return report_result(g, res, best_response_out);
}

namespace {

// The result in the handle's host memory (everything that writes it has run).
bsse_status report_result(bsse_game *g, bsse_result *res, int32_t *best_response_out)
{
    const bool has = g->h_out->run.has != 0;
    if (has && !(g->h_out->fin_v == g->h_out->run.value))
        return fail(BSSE_EDEVICE, "internal: re-evaluated winner value %.9g differs from swept value %.9g",
                    (double)g->h_out->fin_v, (double)g->h_out->run.value);
    res->best_value = has ? (double)g->h_out->run.value : 0.0;
    res->best_index = has ? (int64_t)g->h_out->run.index : -1;
    res->n_evals = g->n_evals;
    res->n_tie_evals = (int64_t)g->h_out->run.ties;
    if (has && best_response_out) memcpy(best_response_out, g->h_br, (size_t)g->K * 4);
    g->result_valid = has && !g->w.fixed;
    if (g->result_valid) {
        memcpy(g->won_x.data(), g->h_x, (size_t)g->m * sizeof(float));
        memcpy(g->won_br.data(), g->h_br, (size_t)g->K * sizeof(int32_t));
    }
    return BSSE_OK;
}

// Whether the records of a sweep of few rows, each with a row and its best responses, are few enough
// to go to the host (256 KiB: a few microseconds over the bus).
constexpr int MAX_HOST_RECS = 2048;
bool host_folds(const bsse_game *g, long long count)
{
    const long long nrec = (count + FINISH_ROWS - 1) / FINISH_ROWS;
    return few_rows(g, count) && nrec <= MAX_HOST_RECS && nrec * (g->m + g->K) <= (1LL << 16);
}
// The same for the one launch of the short-row kernel.
bool one_launch(const bsse_game *g, long long count)
{
    const long long nrec = tiny_num_blocks(count);
    return on_tiny(g) && !few_rows(g, count) && nrec <= MAX_HOST_RECS && nrec * (g->m + g->K) <= (1LL << 16);
}

// Whether sweep_once takes a sweep.
bool sweeps_at_once(const bsse_game *g, long long count)
{
    return count > 0 && (host_folds(g, count) || one_launch(g, count) || (on_any(g) && !few_rows(g, count)));
}

// One whole sweep (already reset) of rows that stay put until it is done, on the any-shape path, or on
// the general one when the rows are few: two launches and one wait, whatever the size; on the short-row
// kernel one launch.  Few rows: a type-sliced launch, and one that sums the
// values and leaves a record per 256 rows, with that record's row and best responses, in pinned memory;
// the host folds the records.  Many rows: the sweep, and one launch whose workgroups each fold its
// records and evaluate their slice of the types at the winner.
bsse_status sweep_once(bsse_game *g, const float *X, long long count, bsse_result *res, int32_t *best_response_out)
{
    const int m = g->m, K = g->K;
    bsse_status st;
    const bool rows = host_folds(g, count), single = !rows && one_launch(g, count), recs = rows || single;
    const long long nrec = single ? tiny_num_blocks(count) : (count + FINISH_ROWS - 1) / FINISH_ROWS;
    const long long used = recs ? nrec : 0;
    SweepArgs a{};
    a.X = X; a.count = count; a.tie_counter = g->w.tie_counter;
    // (the records have a place of their own: nothing else is ever written where a flag is looked for)
    const size_t off_x = (size_t)MAX_HOST_RECS * sizeof(FinishRec), off_br = off_x + (size_t)used * m * sizeof(float);
    if (recs && (st = grow_pinned(g, (void **)&g->h_rec, &g->cap_rec, off_br + (size_t)nrec * K * sizeof(int32_t))) != BSSE_OK) return st;
    auto *rec = reinterpret_cast<FinishRec *>(g->h_rec);
    auto *rec_x = reinterpret_cast<float *>(g->h_rec + off_x);
    auto *rec_br = reinterpret_cast<int32_t *>(g->h_rec + off_br);
    if (single) {
        a.tie_counter = nullptr;                     // (in the records)
    } else if (rows) {
        if ((st = grow_device(g, (void **)&g->row_l, &g->cap_row_l, (size_t)count * K * sizeof(float))) != BSSE_OK) return st;
        if ((st = grow_device(g, (void **)&g->row_br, &g->cap_row_br, (size_t)count * K * sizeof(int32_t))) != BSSE_OK) return st;
        a.l_out = g->row_l; a.l_sc = 1; a.l_st = count;
        a.br_out = g->row_br; a.br_sc = 1; a.br_st = count;
    } else {
        if ((st = ensure_blocks(g, any_max_blocks(g->view, count))) != BSSE_OK) return st;
        a.blk_v = g->w.blk_v; a.blk_i = g->w.blk_i;
    }
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (g->timing) {
        if ((st = take_event(g, &e0)) != BSSE_OK) return st;
        if ((st = take_event(g, &e1)) != BSSE_OK) { g->ev_pool.push_back(e0); return st; }
        HIP_TRY(hipEventRecord(e0, g->stream));
    }
    const TinyRecs tr{ rec, rec_x, rec_br, single ? new_done(g).seq : 0u };
    const hipError_t le = rows ? launch_rows(g, a, g->stream)
                          : single ? launch_sweep_tiny(g->view, a, false, 1, tr, g->stream) : launch_sweep_any(g->view, a, 1, g->stream);
    if (g->timing) {
        (void)hipEventRecord(e1, g->stream);
        g->ev.push_back(e0); g->ev.push_back(e1);
    }
    HIP_TRY(le);
    if (rows) {
        FinishRowsArgs f{};
        f.l = g->row_l; f.br = g->row_br; f.prior = g->dprior; f.X = X; f.count = count; f.K = K; f.m = m;
        f.rec = rec; f.rec_x = rec_x; f.rec_br = rec_br;
        f.ties = g->w.tie_counter;
        f.seq = new_done(g).seq;
        HIP_TRY(launch_finish_rows(f, g->stream));
    } else if (!single) {
        SweepArgs e{};
        e.X = X; e.count = 1; e.index_base = 0;
        e.fold_v = g->w.blk_v; e.fold_i = g->w.blk_i; e.fold_n = (int)any_num_blocks(g->view, count);
        e.fold_ties = g->w.tie_counter; e.fold_run = &g->h_out->run;
        e.row_host = g->h_x;
        e.br_out = g->h_br; e.br_sc = K; e.br_st = 1;
        e.l_out = g->h_l; e.l_sc = K; e.l_st = 1;
        e.done = new_done(g);
        HIP_TRY(launch_rows(g, e, g->stream));
    }
    g->fresh = false;
    g->n_evals += count * K;
    st = recs ? wait_words(g, &rec->seq, (int)nrec, sizeof(FinishRec))
              : wait_flags(g, (int)row_blocks(g, 1));
    if (st != BSSE_OK) return st;
    if (recs) {
        long long b = 0;
        unsigned long long ties = rec[0].ties;
        for (long long r = 1; r < nrec; ++r) {
            if (rec[r].value > rec[b].value || (rec[r].value == rec[b].value && rec[r].index < rec[b].index)) b = r;
            if (single) ties += rec[r].ties;
        }
        RunningBest &run = g->h_out->run;
        run.value = rec[b].value; run.index = rec[b].index; run.has = 1; run.ties = ties;
        memcpy(g->h_x, rec_x + (size_t)b * m, (size_t)m * sizeof(float));
        memcpy(g->h_br, rec_br + (size_t)b * K, (size_t)K * sizeof(int32_t));
        g->h_out->fin_v = run.value;
    } else if (g->h_out->run.has) {
        g->h_out->fin_v = value_of(g, g->h_l);
    }
    return report_result(g, res, best_response_out);
}

}  // namespace

extern "C" bsse_status bsse_sweep_best_row(bsse_game *g, float *x_out)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    if (!x_out) return fail(BSSE_EINVAL, "x_out is NULL");
    DeviceGuard dg(g->device);
    if (!dg.ok) return fail(BSSE_EDEVICE, "hipSetDevice failed");
    // (a graph of recorded chunks, or other work of the caller, may still be on the stream)
    bsse_status st = !g->fresh && on_small_kernel(g) ? fold_small(g) : wait_stream(g);
    if (st != BSSE_OK) return st;
    if (g->fresh || !g->h_out->run.has) return fail(BSSE_ESTATE, "no candidate has been swept since the last reset");
    memcpy(x_out, g->h_x, (size_t)g->m * sizeof(float));
    return BSSE_OK;
}

extern "C" bsse_status bsse_sweep(bsse_game *g, const float *candidates_dev, int64_t count,
                                  bsse_result *res, int32_t *best_response_out)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    if (!res) return fail(BSSE_EINVAL, "res is NULL");
    {   // argument errors first, before anything is enqueued
        const float *x = candidates_dev;
        int64_t c = count;
        bsse_status st = resolve_candidates(g, &x, &c);
        if (st != BSSE_OK) return st;
    }
    bsse_status st = bsse_sweep_reset(g);
    if (st != BSSE_OK) return st;
    {
        const float *x = candidates_dev;
        int64_t c = count;
        if ((st = resolve_candidates(g, &x, &c)) != BSSE_OK) return st;
        if (sweeps_at_once(g, c)) {
            DeviceGuard dg(g->device);
            if (!dg.ok) return fail(BSSE_EDEVICE, "hipSetDevice failed");
            return sweep_once(g, x, c, res, best_response_out);
        }
    }
    if ((st = bsse_sweep_chunk(g, candidates_dev, count, 0)) != BSSE_OK) return st;
    return bsse_sweep_result(g, res, best_response_out);
}

// bsse_sweep with every piece of device scratch taken from the static array: no allocation of any
// kind happens in this call (device, pinned host or stream/event objects).
extern "C" bsse_status bsse_sweep_static(bsse_game *g, const float *candidates_dev, int64_t count,
                                         bsse_result *res, int32_t *best_response_out)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    if (!res) return fail(BSSE_EINVAL, "res is NULL");
    if (!candidates_dev) return fail(BSSE_EINVAL, "candidates is NULL (the static sweep takes an explicit buffer)");
    {
        const float *x = candidates_dev;
        int64_t c = count;
        bsse_status st = resolve_candidates(g, &x, &c);
        if (st != BSSE_OK) return st;
    }
    const bool small = on_small_kernel(g);
    // (every vector-path game has the documented limit, also where the short-row kernel needs fewer records)
    const long long records = g->path == PATH_VALU ? valu_num_blocks(count)
                              : small || on_any(g) || on_tiny(g) ? sweep_records(g, count) : mfma_limit_blocks(g->view.variant, count);
    if (!small && records > STATIC_MAX_BLOCKS)
        return fail(BSSE_EOVERFLOW, "%lld candidates need %lld workgroup records; the static scratch holds %lld "
                    "(sweep in pieces, or use bsse_sweep)", (long long)count, records, STATIC_MAX_BLOCKS);
    if (small && small_num_slots() > STATIC_MAX_SLOTS)
        return fail(BSSE_EOVERFLOW, "the static scratch holds %d running-best slots, %d needed", STATIC_MAX_SLOTS,
                    small_num_slots());
    if (g->m > STATIC_MAX_M) return fail(BSSE_EOVERFLOW, "the static scratch holds rows of %d", STATIC_MAX_M);
    DeviceGuard dg(g->device);
    if (!dg.ok) return fail(BSSE_EDEVICE, "hipSetDevice failed");
    unsigned char *ptr = nullptr;
    bsse_status st = static_scratch(g->device, &ptr);
    if (st != BSSE_OK) return st;

    // the handle works on the static scratch for the length of this call; its own sweep state
    // is what bsse_sweep leaves behind as well: reset
    struct Swap {
        bsse_game *g; Work own; bool timing, ties_dirty; int used[3];
        ~Swap()
        {
            g->w = own; g->timing = timing; g->ties_dirty = ties_dirty;
            for (int q = 0; q < 3; ++q) g->set_used[q] = used[q];
            g->fresh = true; g->fold_pending = false; g->result_valid = false; g->n_evals = 0;
        }
    } swap{ g, g->w, g->timing, g->ties_dirty, { g->set_used[0], g->set_used[1], g->set_used[2] } };
    for (int &u : g->set_used) u = 0;          // (the array holds one set of slots)
    Work w;
    w.run = reinterpret_cast<RunningBest *>(ptr + ST_OFF_RUN);
    w.tie_counter = reinterpret_cast<unsigned long long *>(ptr + ST_OFF_TIES);
    w.best_x = reinterpret_cast<float *>(ptr + ST_OFF_BESTX);
    w.blk_v = reinterpret_cast<float *>(ptr + ST_OFF_BLKV);
    w.blk_i = reinterpret_cast<long long *>(ptr + ST_OFF_BLKI);
    w.blk_cap = STATIC_HELD_BLOCKS;
    w.slots = small ? reinterpret_cast<SmallSlot *>(ptr + ST_OFF_SLOTS) : nullptr;
    w.slot_sets = small ? 1 : 0;
    w.fixed = true;
    g->w = w;
    g->timing = false;              // (event pairs would be created on demand)
    g->ties_dirty = false;
    // the array keeps the last call's contents, possibly another handle's: the running best, the
    // tie counter and (small-game kernel) the slots' epochs start from zero.  A fill kernel, not a
    // memset node, so that the call stays safe to capture.
    HIP_TRY(launch_fill_zero(ptr, ST_OFF_BESTX, g->stream));
    if (small) HIP_TRY(launch_fill_zero(ptr + ST_OFF_SLOTS, (size_t)small_num_slots() * sizeof(SmallSlot), g->stream));
    if ((st = bsse_sweep_reset(g)) != BSSE_OK) return st;
    if ((st = bsse_sweep_chunk(g, candidates_dev, count, 0)) != BSSE_OK) return st;
    return bsse_sweep_result(g, res, best_response_out);
}

extern "C" bsse_status bsse_eval(bsse_game *g, const float *candidates_dev, int64_t count,
                                 float *values_dev_out, int32_t *br_dev_out)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    bsse_status st = resolve_candidates(g, &candidates_dev, &count);
    if (st != BSSE_OK) return st;
    if (count == 0 || (!values_dev_out && !br_dev_out)) return BSSE_OK;
    DeviceGuard dg(g->device);
    if (!dg.ok) return fail(BSSE_EDEVICE, "hipSetDevice failed");
    SweepArgs a{};
    a.X = candidates_dev; a.count = count; a.index_base = 0;
    a.V_out = values_dev_out; a.br_out = br_dev_out;
    return launch_eval(g, a);
}

// ------------------------------------------------------------------------ prior batch
extern "C" bsse_status bsse_sweep_priors(bsse_game *g, const float *candidates_dev, int64_t count,
                                         const float *priors, int P, bsse_result *res,
                                         int32_t *best_response_out)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    if (!priors) return fail(BSSE_EINVAL, "priors is NULL");
    if (!res) return fail(BSSE_EINVAL, "res is NULL");
    if (P < 1 || P > 65536) return fail(BSSE_EINVAL, "P = %d outside 1..65536", P);
    const int K = g->K, m = g->m;
    for (int p = 0; p < P; ++p) {
        double psum = 0.0;
        for (int t = 0; t < K; ++t) {
            const float v = priors[(size_t)p * K + t];
            if (!std::isfinite(v)) return fail(BSSE_ENOTFINITE, "priors[%d][%d] is not finite", p, t);
            if (v < 0.0f) return fail(BSSE_EINVAL, "priors[%d][%d] is negative", p, t);
            psum += (double)v;
        }
        if (std::fabs(psum - 1.0) > 1e-6)
            return fail(BSSE_EINVAL, "priors[%d] sums to %.9g, not 1", p, psum);
    }
    bsse_status st = resolve_candidates(g, &candidates_dev, &count);
    if (st != BSSE_OK) return st;
    if (count == 0) {
        for (int p = 0; p < P; ++p) { res[p].best_value = 0.0; res[p].best_index = -1; res[p].n_evals = 0; res[p].n_tie_evals = 0; }
        return BSSE_OK;
    }
    DeviceGuard dg(g->device);
    if (!dg.ok) return fail(BSSE_EDEVICE, "hipSetDevice failed");

    // the leader-payoff matrix is built chunk by chunk: at most 2^28 entries (1 GiB) at a time
    long long chunk = (1LL << 28) / K;
    if (chunk < 4096) chunk = 4096;
    if (chunk > count) chunk = count;
    const long long ld = (chunk + 3) & ~3LL;
    const int ldp = prior_batch_ld(P);
    PriorScratch &w = g->pri;
    // transposed priors, then the tie counter (zero), in one block each in pinned and in device memory
    const size_t in_words = ((size_t)K * ldp + 1) / 2 * 2, in_bytes = in_words * 4 + sizeof(unsigned long long);
    if ((st = grow_device(g, (void **)&w.L, &w.cap_L, (size_t)ld * K * sizeof(float))) != BSSE_OK) return st;
    if ((st = grow_device(g, (void **)&w.priors, &w.cap_priors, in_bytes)) != BSSE_OK) return st;
    // (a last, shorter chunk is cut finer where it has few steps: whichever has more records)
    const long long last = count - (count - 1) / chunk * chunk;
    const size_t records = (size_t)std::max(prior_batch_blocks(chunk, P), prior_batch_blocks(last, P)) * P;
    if ((st = grow_device(g, (void **)&w.blk_v, &w.cap_blk_v, records * sizeof(float))) != BSSE_OK) return st;
    if ((st = grow_device(g, (void **)&w.run, &w.cap_run, (size_t)P * sizeof(PriorBest))) != BSSE_OK) return st;
    if ((st = grow_device(g, (void **)&w.rows, &w.cap_rows, (size_t)P * m * sizeof(float))) != BSSE_OK) return st;
    const size_t off_run = (in_bytes + 15) / 16 * 16, off_ties = off_run + (size_t)P * sizeof(PriorBest), off_br = off_ties + 16;
    if ((st = grow_pinned(g, (void **)&w.host, &w.cap_host, off_br + (size_t)P * K * sizeof(int32_t))) != BSSE_OK) return st;
    float *priT = reinterpret_cast<float *>(w.host);
    for (int t = 0; t < K; ++t) {
        for (int p = 0; p < P; ++p) priT[(size_t)t * ldp + p] = priors[(size_t)p * K + t];
        for (int p = P; p < ldp; ++p) priT[(size_t)t * ldp + p] = 0.0f;
    }
    memset(w.host + in_words * 4, 0, sizeof(unsigned long long));
    HIP_TRY(launch_copy_words(w.host, w.priors, in_bytes / 4, g->stream));
    auto *ties_dev = reinterpret_cast<unsigned long long *>(w.priors + in_words);
    auto *run = reinterpret_cast<PriorBest *>(w.host + off_run);
    auto *ties = reinterpret_cast<unsigned long long *>(w.host + off_ties);
    auto *br = reinterpret_cast<int32_t *>(w.host + off_br);
    for (long long base = 0; base < count; base += chunk) {
        const long long rows = count - base < chunk ? count - base : chunk;
        SweepArgs a{};
        a.X = candidates_dev + base * m; a.count = rows; a.index_base = base;
        a.l_out = w.L; a.l_sc = 1; a.l_st = ld; a.tie_counter = ties_dev;
        if ((st = launch_eval(g, a)) != BSSE_OK) return st;
        PriorFoldArgs f{};
        f.L = w.L; f.count = (unsigned)rows; f.ld = (unsigned)ld; f.K = K; f.priT = w.priors; f.index_base = base;
        f.first = base == 0 ? 1 : 0; f.run = w.run; f.m = m;
        if (base + rows == count) {
            f.rows = w.rows; f.X = candidates_dev; f.run_host = run; f.ties = ties_dev; f.ties_host = ties;
        }
        HIP_TRY(launch_prior_batch(f, P, w.blk_v, g->stream));
    }
    // best responses of the P winners: their rows, evaluated once more with per-candidate outputs
    int flags = 0;
    if ((st = launch_winners(g, w.rows, P, br, true, &flags)) != BSSE_OK) return st;
    if ((st = wait_winners(g, flags)) != BSSE_OK) return st;
    for (int p = 0; p < P; ++p) {
        res[p].best_value = run[p].has ? (double)run[p].value : 0.0;
        res[p].best_index = run[p].has ? (int64_t)run[p].index : -1;
        res[p].n_evals = (int64_t)count * K;
        res[p].n_tie_evals = (int64_t)*ties;
    }
    if (best_response_out) memcpy(best_response_out, br, (size_t)P * K * sizeof(int32_t));
    return BSSE_OK;
}

// --------------------------------------------------------------------------------- top-k
namespace {

// Evaluation of `sets` sets of `count` rows each (one behind the other at X) and the k best of every
// set: values, indices, best responses and (rows_host) rows into pinned memory.  `flags` as in
// launch_winners.
bsse_status enqueue_topk(bsse_game *g, const float *X, long long count, int sets, int k, long long index_base,
                         float *val, long long *idx, int32_t *br, float *rows_host, bool last, int *flags)
{
    TopkScratch &w = g->topk;
    const int m = g->m;
    const long long total = count * sets;
    bsse_status st;
    if ((st = grow_device(g, (void **)&w.V, &w.cap_V, (size_t)total * sizeof(float))) != BSSE_OK) return st;
    if ((st = grow_device(g, (void **)&w.heads, &w.cap_heads, topk_heads_bytes(count, sets))) != BSSE_OK) return st;
    if ((st = grow_device(g, (void **)&w.rows, &w.cap_rows, (size_t)sets * k * m * sizeof(float))) != BSSE_OK) return st;
    SweepArgs a{};
    a.X = X; a.count = total; a.V_out = w.V;
    if ((st = launch_eval(g, a)) != BSSE_OK) return st;
    TopkArgs t{};
    t.V = w.V; t.heads = w.heads; t.X = X; t.count = (unsigned)count; t.k = k; t.m = m; t.index_base = index_base;
    t.val = val; t.idx = idx; t.rows = w.rows; t.rows_host = rows_host;
    HIP_TRY(launch_topk(t, sets, g->stream));
    return launch_winners(g, w.rows, (long long)sets * k, br, last, flags);
}

}  // namespace

extern "C" bsse_status bsse_sweep_topk(bsse_game *g, const float *candidates_dev, int64_t count, int k,
                                       double *values_out, int64_t *indices_out,
                                       int32_t *best_response_out, int *found_out)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    if (!values_out || !indices_out || !found_out) return fail(BSSE_EINVAL, "NULL argument");
    if (k < 1 || k > 256) return fail(BSSE_EINVAL, "k = %d outside 1..256", k);
    bsse_status st = resolve_candidates(g, &candidates_dev, &count);
    if (st != BSSE_OK) return st;
    if (count == 0) { *found_out = 0; return BSSE_OK; }
    DeviceGuard dg(g->device);
    if (!dg.ok) return fail(BSSE_EDEVICE, "hipSetDevice failed");
    const int K = g->K;

    // chunks of at most 2^26 candidates, each with its own k best; the host merges them
    const long long chunk = count < (1LL << 26) ? count : (1LL << 26);
    const long long nchunks = (count + chunk - 1) / chunk;
    const size_t recs = (size_t)nchunks * k;
    const size_t off_idx = 0, off_val = recs * sizeof(long long), off_br = off_val + recs * sizeof(float);
    if ((st = grow_pinned(g, (void **)&g->topk.host, &g->topk.cap_host, off_br + recs * K * sizeof(int32_t))) != BSSE_OK) return st;
    long long *hi = reinterpret_cast<long long *>(g->topk.host + off_idx);
    float *hv = reinterpret_cast<float *>(g->topk.host + off_val);
    int32_t *hb = reinterpret_cast<int32_t *>(g->topk.host + off_br);
    int flags = 0;
    struct Part { long long at, end; };                  // what is left of a chunk's records
    std::vector<Part> part;
    try { part.resize((size_t)nchunks); } catch (...) { return fail(BSSE_ENOMEM, "host allocation failed"); }
    for (long long c = 0; c < nchunks; ++c) {
        const long long base = c * chunk, n = count - base < chunk ? count - base : chunk;
        const int kk = n < k ? (int)n : k;
        part[(size_t)c] = { c * k, c * k + kk };
        if ((st = enqueue_topk(g, candidates_dev + base * g->m, n, 1, kk, base, hv + c * k, hi + c * k, hb + c * k * K,
                               nullptr, c + 1 == nchunks, &flags)) != BSSE_OK) return st;
    }
    if ((st = wait_winners(g, flags)) != BSSE_OK) return st;
    const int found = count < k ? (int)count : k;
    for (int r = 0; r < found; ++r) {
        Part *best = nullptr;                            // (an earlier chunk's index is the lower one)
        for (Part &p : part)
            if (p.at < p.end && (!best || hv[p.at] > hv[best->at])) best = &p;
        const long long e = best->at++;
        values_out[r] = (double)hv[e]; indices_out[r] = (int64_t)hi[e];
        if (best_response_out) memcpy(best_response_out + (size_t)r * K, hb + e * K, (size_t)K * sizeof(int32_t));
    }
    *found_out = found;
    return BSSE_OK;
}

// ------------------------------------------------------------------------------- refinement
extern "C" bsse_status bsse_refine(bsse_game *g, int k, int rounds, int lattice_N, int64_t cloud_count,
                                   uint64_t seed, float radius, float shrink, float *x_out,
                                   bsse_result *res, int32_t *best_response_out)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    if (!x_out || !res) return fail(BSSE_EINVAL, "NULL argument");
    if (k < 1 || k > 256) return fail(BSSE_EINVAL, "k = %d outside 1..256", k);
    if (rounds < 1 || rounds > 64) return fail(BSSE_EINVAL, "rounds = %d outside 1..64", rounds);
    if ((lattice_N > 0) == (cloud_count > 0))
        return fail(BSSE_EINVAL, "give either lattice_N > 0 or cloud_count > 0");
    if (!(radius > 0.0f && radius <= 1.0f) || !(shrink > 0.0f && shrink <= 1.0f))
        return fail(BSSE_EINVAL, "radius and shrink must lie in (0, 1]");
    if (g->gen_count <= 0) return fail(BSSE_ESTATE, "no candidate set has been generated on this handle");
    const int m = g->m, K = g->K;
    DeviceGuard dg(g->device);
    if (!dg.ok) return fail(BSSE_EDEVICE, "hipSetDevice failed");

    // survivors: value, row, best responses; kept sorted by (value desc, order of discovery)
    struct Survivor { double v; std::vector<float> x; std::vector<int32_t> br; };
    std::vector<Survivor> pool;
    // what a round finds, in the order of discovery; x and br stay where the records are
    struct Found { double v; const float *x; const int32_t *br; };
    std::vector<Found> found;
    long long evals = 0;
    bsse_status st;
    // the k best distinct points of `found` become the pool
    auto keep_best = [&]() {
        std::stable_sort(found.begin(), found.end(), [](const Found &a, const Found &b) { return a.v > b.v; });
        std::vector<Survivor> out;
        for (const Found &f : found) {
            // the same point may be found from two centres: keep one
            bool dupl = false;
            for (const Survivor &o : out) if (std::equal(o.x.begin(), o.x.end(), f.x)) { dupl = true; break; }
            if (!dupl) out.push_back({ f.v, std::vector<float>(f.x, f.x + m), std::vector<int32_t>(f.br, f.br + K) });
            if ((int)out.size() == k) break;
        }
        pool.swap(out);
    };
    // Room for the records of `sets` sets in pinned memory, and those of `nsets` sets of `kk` appended to
    // `found`.
    std::vector<double> vals;
    std::vector<int64_t> idx;
    long long *hi = nullptr;
    float *hv = nullptr, *hx = nullptr;
    int32_t *hb = nullptr;
    auto records = [&](size_t recs) -> bsse_status {
        const size_t off_v = recs * sizeof(long long), off_b = off_v + recs * sizeof(float), off_x = off_b + recs * K * sizeof(int32_t);
        bsse_status s = grow_pinned(g, (void **)&g->topk.host, &g->topk.cap_host, off_x + recs * m * sizeof(float));
        hi = reinterpret_cast<long long *>(g->topk.host);
        hv = reinterpret_cast<float *>(g->topk.host + off_v);
        hb = reinterpret_cast<int32_t *>(g->topk.host + off_b);
        hx = reinterpret_cast<float *>(g->topk.host + off_x);
        return s;
    };
    auto append = [&](size_t recs) {
        for (size_t r = 0; r < recs; ++r) found.push_back({ (double)hv[r], hx + r * m, hb + r * K });
    };
    // A set too large for one selection (2^26 rows): bsse_sweep_topk, which cuts it, and copies of the
    // rows.  The records are copied here, for the next set overwrites the pinned ones.
    std::vector<std::vector<float>> big_x;
    std::vector<std::vector<int32_t>> big_br;
    auto harvest_big = [&]() -> bsse_status {
        vals.resize((size_t)k); idx.resize((size_t)k);
        std::vector<int32_t> brs((size_t)k * K);
        int n = 0;
        bsse_status s = bsse_sweep_topk(g, nullptr, 0, k, vals.data(), idx.data(), brs.data(), &n);
        if (s != BSSE_OK) return s;
        std::vector<float> xs((size_t)n * m);
        for (int r = 0; r < n; ++r)
            HIP_TRY(hipMemcpyAsync(&xs[(size_t)r * m], g->gen + (size_t)idx[r] * m, (size_t)m * sizeof(float), hipMemcpyDeviceToHost, g->stream));
        HIP_TRY(hipStreamSynchronize(g->stream));
        big_x.push_back(std::move(xs)); big_br.push_back(std::move(brs));
        for (int r = 0; r < n; ++r) found.push_back({ vals[r], big_x.back().data() + (size_t)r * m, big_br.back().data() + (size_t)r * K });
        return BSSE_OK;
    };
    constexpr long long SET_MAX = 1LL << 26;             // rows one selection takes
    try {
        int flags = 0;
        evals += (long long)g->gen_count * K;
        if (g->gen_count > SET_MAX) {
            if ((st = harvest_big()) != BSSE_OK) return st;
        } else {
            const int kk = (int)std::min<long long>(k, g->gen_count);
            if ((st = records((size_t)kk)) != BSSE_OK) return st;
            if ((st = enqueue_topk(g, g->gen, g->gen_count, 1, kk, 0, hv, hi, hb, hx, true, &flags)) != BSSE_OK) return st;
            if ((st = wait_winners(g, flags)) != BSSE_OK) return st;
            append((size_t)kk);
        }
        keep_best();
        int64_t cnt = cloud_count;
        if (lattice_N > 0) {
            if ((st = bsse_lattice_count(m, lattice_N, &cnt)) != BSSE_OK) return st;
            if (cnt <= SET_MAX && (st = ensure_lattice_table(g, lattice_N)) != BSSE_OK) return st;
        }
        // The local sets of a round do not depend on each other: as many as fit 2^26 floats (but one at
        // least) are generated, evaluated and selected together, five launches and one wait for all of them.
        const bool big = cnt > SET_MAX;                      // (any number the caller gave)
        const int kk = (int)std::min<long long>(k, cnt);
        const long long together = big ? 1 : std::max<long long>(1, std::min<long long>(k, (1LL << 26) / (cnt * m)));
        // A set that goes alone is generated in the handle-owned buffer: no second one of its size.
        const bool staged = together > 1;
        float rad = radius;
        for (int round = 0; round < rounds; ++round) {
            found.clear(); big_x.clear(); big_br.clear();
            for (const Survivor &s : pool) found.push_back({ s.v, s.x.data(), s.br.data() });   // a centre survives unless it is beaten
            const uint64_t rseed = seed + (uint64_t)round * 1000003ull;
            const size_t nc = pool.size();
            // (the handle-owned set ends as the last local set, as if each had been generated there)
            if (!big && (!staged || round + 1 == rounds) && (st = ensure_gen(g, (unsigned long long)cnt)) != BSSE_OK) return st;
            if (!big) {
                evals += (long long)nc * cnt * K;
                const size_t bytes = nc * m * sizeof(float);
                if ((st = grow_device(g, (void **)&g->centre_dev, &g->cap_centre, bytes)) != BSSE_OK) return st;
                if ((st = grow_pinned(g, (void **)&g->h_centre, &g->cap_h_centre, bytes)) != BSSE_OK) return st;
                for (size_t c = 0; c < nc; ++c) memcpy(g->h_centre + c * m, pool[c].x.data(), (size_t)m * sizeof(float));
                HIP_TRY(launch_copy_words(g->h_centre, g->centre_dev, nc * m, g->stream));
                if (staged && (st = grow_device(g, (void **)&g->stage, &g->stage_cap, (size_t)together * cnt * m * sizeof(float))) != BSSE_OK) return st;
                if ((st = records((size_t)nc * kk)) != BSSE_OK) return st;
            }
            auto generate = [&](size_t c0, int sets, float *out) -> bsse_status {
                if (lattice_N > 0) HIP_TRY(launch_lattice(g->lat_table, m, lattice_N, cnt, g->centre_dev + c0 * m, rad, sets, out, g->stream));
                else HIP_TRY(launch_dirichlet(rseed + c0, 0, cnt, m, g->centre_dev + c0 * m, rad, sets, out, g->stream));
                return BSSE_OK;
            };
            for (size_t c0 = 0; c0 < nc; c0 += (size_t)(big ? 1 : together)) {
                if (big) {
                    int64_t n = 0;
                    st = lattice_N > 0 ? bsse_lattice_around(g, lattice_N, pool[c0].x.data(), rad, &n)
                                       : bsse_dirichlet_around(g, rseed + c0, 0, cnt, pool[c0].x.data(), rad, nullptr);
                    if (st == BSSE_OK) st = harvest_big();
                    if (st != BSSE_OK) return st;
                    evals += (long long)cnt * K;
                    continue;
                }
                const int sets = (int)std::min<size_t>((size_t)together, nc - c0);
                const bool last = c0 + sets == nc;
                if ((st = generate(c0, sets, staged ? g->stage : g->gen)) != BSSE_OK) return st;
                if (staged && last && round + 1 == rounds && (st = generate(nc - 1, 1, g->gen)) != BSSE_OK) return st;
                if (!staged || (last && round + 1 == rounds)) g->gen_count = cnt;
                const size_t at = c0 * kk;
                if ((st = enqueue_topk(g, staged ? g->stage : g->gen, cnt, sets, kk, 0, hv + at, hi + at, hb + at * K, hx + at * m, last, &flags)) != BSSE_OK) return st;
            }
            if (!big) {
                if ((st = wait_winners(g, flags)) != BSSE_OK) return st;
                append(nc * kk);
            }
            keep_best();
            rad *= shrink;
        }
    } catch (...) { return fail(BSSE_ENOMEM, "host allocation failed"); }
    if (pool.empty()) return fail(BSSE_ESTATE, "the candidate set is empty");
    memcpy(x_out, pool[0].x.data(), (size_t)m * sizeof(float));
    res->best_value = pool[0].v;
    res->best_index = -1;                                  // the point is not a member of one indexed set
    res->n_evals = evals;
    res->n_tie_evals = 0;
    if (best_response_out) memcpy(best_response_out, pool[0].br.data(), (size_t)K * sizeof(int32_t));
    return BSSE_OK;
}

// ----------------------------------------------------------------------------- LP polish
namespace {

bsse_status check_profile(int n, int K, const int32_t *profile)
{
    for (int t = 0; t < K; ++t)
        if (profile[t] < 0 || profile[t] >= n)
            return fail(BSSE_EINVAL, "profile[%d] = %d outside 0..%d", t, (int)profile[t], n - 1);
    return BSSE_OK;
}

constexpr int kPolishRows = 8;       // segment points evaluated by bsse_polish

}  // namespace

extern "C" bsse_status bsse_profile_lp(int m, int n, int K, const float *A, const float *B,
                                       const float *prior, const int32_t *profile, double *x_out,
                                       double *value_out, int *feasible_out)
{
    g_err[0] = 0;
    if (m < 1 || n < 1 || K < 1 || m > 4096 || n > 65535 || K > 65535)
        return fail(BSSE_EINVAL, "bad dimensions m=%d n=%d K=%d", m, n, K);
    if (!A || !B || !prior || !profile || !x_out || !value_out || !feasible_out)
        return fail(BSSE_EINVAL, "NULL argument");
    // the dual tableau holds m rows of 2 + K(n-1) + m columns
    const double cells = (double)m * (2.0 + (double)K * (n - 1) + m);
    if (cells > (double)(1u << 28)) return fail(BSSE_EOVERFLOW, "the program's tableau (%.3g cells) is too large", cells);
    bsse_status st = check_profile(n, K, profile);
    if (st != BSSE_OK) return st;
    const size_t elems = (size_t)K * m * n;
    for (size_t e = 0; e < elems; ++e)
        if (!std::isfinite(A[e]) || !std::isfinite(B[e]))
            return fail(BSSE_ENOTFINITE, "payoff entry %zu is not finite", e);
    for (int t = 0; t < K; ++t)
        if (!std::isfinite(prior[t]) || prior[t] < 0.0f)
            return fail(std::isfinite(prior[t]) ? BSSE_EINVAL : BSSE_ENOTFINITE, "bad prior[%d]", t);
    std::vector<double> x;
    try { x.resize((size_t)m); } catch (...) { return fail(BSSE_ENOMEM, "host allocation failed"); }
    double v = 0.0;
    int rc;
    try { rc = solve_profile_lp(m, n, K, A, B, prior, profile, x.data(), &v); }
    catch (...) { return fail(BSSE_ENOMEM, "host allocation failed"); }
    if (rc == 2) return fail(BSSE_ESTATE, "the simplex method did not converge");
    if (rc == 0) { memcpy(x_out, x.data(), (size_t)m * sizeof(double)); *value_out = v; }
    *feasible_out = rc == 0 ? 1 : 0;
    return BSSE_OK;
}

extern "C" bsse_status bsse_polish(bsse_game *g, const int32_t *profile, float *x_out,
                                   bsse_result *res, int32_t *best_response_out,
                                   double *lp_value_out)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    if (!x_out || !res) return fail(BSSE_EINVAL, "NULL argument");
    if (!g->result_valid)
        return fail(BSSE_ESTATE, "no sweep result to polish: call bsse_sweep (or _chunk and then _result) first");
    const int m = g->m, n = g->n, K = g->K;
    if (profile) {
        bsse_status st = check_profile(n, K, profile);
        if (st != BSSE_OK) return st;
    }
    const double cells = (double)m * (2.0 + (double)K * (n - 1) + m);
    if (cells > (double)(1u << 28)) return fail(BSSE_EOVERFLOW, "the program's tableau (%.3g cells) is too large", cells);
    DeviceGuard dg(g->device);
    if (!dg.ok) return fail(BSSE_EDEVICE, "hipSetDevice failed");
    std::vector<int32_t> prof((size_t)K);
    std::vector<float> start((size_t)m), rows((size_t)kPolishRows * m), vals((size_t)kPolishRows);
    std::vector<int32_t> brs((size_t)kPolishRows * K);
    std::vector<double> x((size_t)m);
    memcpy(prof.data(), profile ? profile : g->won_br.data(), (size_t)K * sizeof(int32_t));
    memcpy(start.data(), g->won_x.data(), (size_t)m * sizeof(float));
    double v_lp = 0.0;
    const int rc = solve_profile_lp(m, n, K, g->hA.data(), g->hB.data(), g->hprior.data(), prof.data(),
                                    x.data(), &v_lp);
    if (rc == 2) return fail(BSSE_ESTATE, "the simplex method did not converge");
    if (rc == 1) return fail(BSSE_EINVAL, "the profile is a best response nowhere on the simplex");
    // the segment from the program's vertex to the sweep's winner: the vertex sits on the boundary
    // of the profile's region, where fp32 rounding of x can tip a follower over to another action;
    // V is linear along the segment inside the region, so the best evaluated point is kept
    static const double eps[kPolishRows] = { 0.0, 0x1p-22, 0x1p-19, 0x1p-16, 0x1p-13, 0x1p-10, 0x1p-6, 1.0 };
    for (int e = 0; e < kPolishRows; ++e)
        for (int i = 0; i < m; ++i)
            rows[(size_t)e * m + i] = (float)((1.0 - eps[e]) * x[i] + eps[e] * (double)start[i]);
    // the kernel reads the rows from pinned memory and leaves its results there: one launch, one wait
    const size_t off_v = rows.size() * sizeof(float), off_br = off_v + vals.size() * sizeof(float);
    bsse_status st = grow_pinned(g, (void **)&g->h_pol, &g->cap_pol, off_br + brs.size() * sizeof(int32_t) + (size_t)kPolishRows * K * sizeof(float));
    if (st != BSSE_OK) return st;
    float *pol_v = reinterpret_cast<float *>(g->h_pol + off_v);
    int32_t *pol_br = reinterpret_cast<int32_t *>(g->h_pol + off_br);
    float *pol_l = reinterpret_cast<float *>(pol_br + brs.size());
    memcpy(g->h_pol, rows.data(), rows.size() * sizeof(float));
    int flags = 0;
    if ((st = launch_winners(g, reinterpret_cast<const float *>(g->h_pol), kPolishRows, pol_br, true, &flags, pol_v, pol_l)) != BSSE_OK) return st;
    if ((st = wait_winners(g, flags)) != BSSE_OK) return st;
    memcpy(brs.data(), pol_br, brs.size() * sizeof(int32_t));
    for (int e = 0; e < kPolishRows; ++e) {
        vals[e] = cuts_types(g) ? value_of(g, pol_l + (size_t)e * K) : pol_v[e];
    }
    int best = kPolishRows - 1;                          // the sweep's own winner, unless a point beats it
    for (int e = kPolishRows - 2; e >= 0; --e)
        if (vals[e] >= vals[best]) best = e;             // equal values: the point nearest the vertex
    memcpy(x_out, &rows[(size_t)best * m], (size_t)m * sizeof(float));
    res->best_value = (double)vals[best];
    res->best_index = best;
    res->n_evals = (int64_t)kPolishRows * K;
    res->n_tie_evals = 0;
    if (best_response_out) memcpy(best_response_out, &brs[(size_t)best * K], (size_t)K * sizeof(int32_t));
    if (lp_value_out) *lp_value_out = v_lp;
    return BSSE_OK;
}

extern "C" bsse_status bsse_solve_realised(bsse_game *g, const float *candidates_dev, int64_t count,
                                           int max_profiles, float *x_out, double *value_out,
                                           int32_t *profile_out, int *n_profiles_out, int *n_solved_out)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    if (!x_out || !value_out || !n_profiles_out || !n_solved_out) return fail(BSSE_EINVAL, "NULL argument");
    if (max_profiles < 1) return fail(BSSE_EINVAL, "max_profiles must be >= 1");
    bsse_status st = resolve_candidates(g, &candidates_dev, &count);
    if (st != BSSE_OK) return st;
    const int m = g->m, n = g->n, K = g->K;
    if (count == 0) return fail(BSSE_EINVAL, "no candidates");
    if ((double)count * K > (double)(1u << 27)) return fail(BSSE_EOVERFLOW, "count * K exceeds 2^27 best responses");
    const double cells = (double)m * (2.0 + (double)K * (n - 1) + m);
    if (cells > (double)(1u << 28)) return fail(BSSE_EOVERFLOW, "the program's tableau (%.3g cells) is too large", cells);
    DeviceGuard dg(g->device);
    if (!dg.ok) return fail(BSSE_EDEVICE, "hipSetDevice failed");
    RealisedScratch &w = g->real;
    // (no more profiles than rows, nor than n to the K)
    int64_t most64 = std::min<int64_t>(max_profiles, count), profiles = 1;
    for (int t = 0; t < K && profiles < most64; ++t) profiles *= n;          // (both factors below 2^28: no overflow)
    most64 = std::min(most64, n == 1 ? (int64_t)1 : profiles);
    const unsigned nslots = profile_table_slots(count), most = (unsigned)most64;
    // One workgroup and one vertex of doubles in memory per program: beyond four million the host keeps
    // one of each.
    const bool on_device = lp_on_device(m, n, K) && most <= (1u << 22);
    const size_t table_bytes = (size_t)nslots * 12 + 16;             // keys, slots, counter
    struct Release {                     // scratch of a large set is not kept
        RealisedScratch &w;
        ~Release() { if (w.cap_br + w.cap_table + w.cap_x > (size_t)1 << 30) { w.release(); w = RealisedScratch(); } }
    } release{ w };
    if ((st = grow_device(g, (void **)&w.V, &w.cap_V, (size_t)count * sizeof(float))) != BSSE_OK) return st;
    if ((st = grow_device(g, (void **)&w.br, &w.cap_br, (size_t)count * K * sizeof(int32_t))) != BSSE_OK) return st;
    if ((st = grow_device(g, (void **)&w.table, &w.cap_table, table_bytes)) != BSSE_OK) return st;
    if ((st = grow_device(g, (void **)&w.list, &w.cap_list, (size_t)count * sizeof(unsigned long long))) != BSSE_OK) return st;
    if ((st = grow_device(g, (void **)&w.sel, &w.cap_sel, (size_t)most * sizeof(unsigned long long))) != BSSE_OK) return st;
    auto *best = reinterpret_cast<unsigned long long *>(w.table);
    auto *slots = reinterpret_cast<unsigned *>(best + nslots), *n_dev = slots + nslots;
    HIP_TRY(launch_fill_zero(w.table, table_bytes, g->stream));
    SweepArgs a{};
    a.X = candidates_dev; a.count = count; a.index_base = 0;
    a.V_out = w.V; a.br_out = w.br;
    if ((st = launch_eval(g, a)) != BSSE_OK) return st;
    // distinct profiles, each with the best value a candidate reached under it; the most promising of
    // them by that value
    HIP_TRY(launch_profiles(w.V, w.br, count, K, slots, best, n_dev, w.list, most, w.sel, g->stream));
    if (on_device) {
        const size_t elems = (size_t)K * m * n * sizeof(float);
        if (!w.payoffs) {                // as given to create, once per game
            float *p = nullptr;
            HIP_TRY(hipMalloc((void **)&p, 2 * elems));
            hipError_t e = hipMemcpyAsync(p, g->hA.data(), elems, hipMemcpyHostToDevice, g->stream);
            if (e == hipSuccess) e = hipMemcpyAsync(p + elems / sizeof(float), g->hB.data(), elems, hipMemcpyHostToDevice, g->stream);
            if (e != hipSuccess) {
                (void)hipStreamSynchronize(g->stream);
                (void)hipFree(p);
                return fail(BSSE_EDEVICE, "payoffs: %s", hipGetErrorString(e));
            }
            w.payoffs = p;               // (only once it is on its way)
        }
        if ((st = grow_device(g, (void **)&w.v, &w.cap_v, (size_t)most * sizeof(double))) != BSSE_OK) return st;
        if ((st = grow_device(g, (void **)&w.x, &w.cap_x, (size_t)most * m * sizeof(double))) != BSSE_OK) return st;
        if ((st = grow_device(g, (void **)&w.rc, &w.cap_rc, (size_t)most * sizeof(int))) != BSSE_OK) return st;
        const size_t off_x = 64, off_prof = off_x + (size_t)m * sizeof(double);
        if ((st = grow_pinned(g, (void **)&w.host, &w.cap_host, off_prof + (size_t)K * sizeof(int32_t))) != BSSE_OK) return st;
        static_assert(sizeof(LpBest) <= 64, "the vertex starts behind it");
        LpArgs p{};
        p.A = w.payoffs; p.B = w.payoffs + elems / sizeof(float); p.prior = g->dprior;
        p.m = m; p.n_act = n; p.K = K; p.br = w.br; p.sel = w.sel; p.n = n_dev; p.most = most;
        p.v = w.v; p.x = w.x; p.rc = w.rc;
        auto *out = reinterpret_cast<LpBest *>(w.host);
        auto *hx = reinterpret_cast<double *>(w.host + off_x);
        auto *hp = reinterpret_cast<int32_t *>(w.host + off_prof);
        HIP_TRY(launch_profile_lps(p, out, hx, hp, new_done(g), g->stream));
        if ((st = wait_flags(g, 1)) != BSSE_OK) return st;
        *n_profiles_out = (int)out->profiles;
        if (out->failed) return fail(BSSE_ESTATE, "the simplex method did not converge");
        *n_solved_out = (int)out->solved;
        if (!out->found) return fail(BSSE_ESTATE, "no realised profile has a feasible program");
        for (int i = 0; i < m; ++i) x_out[i] = (float)hx[i];
        *value_out = out->value;
        if (profile_out) memcpy(profile_out, hp, (size_t)K * sizeof(int32_t));
        return BSSE_OK;
    }
    // programs too large for one workgroup's LDS: one after the other on the host
    unsigned n_prof = 0;
    std::vector<unsigned long long> sel;
    std::vector<int32_t> hb;
    HIP_TRY(hipMemcpyAsync(&n_prof, n_dev, sizeof(n_prof), hipMemcpyDeviceToHost, g->stream));
    HIP_TRY(hipStreamSynchronize(g->stream));
    const size_t todo = std::min(n_prof, most);
    try { sel.resize(todo); hb.resize((size_t)count * K); } catch (...) { return fail(BSSE_ENOMEM, "host allocation failed"); }
    HIP_TRY(hipMemcpyAsync(sel.data(), w.sel, todo * sizeof(sel[0]), hipMemcpyDeviceToHost, g->stream));
    HIP_TRY(hipMemcpyAsync(hb.data(), w.br, hb.size() * sizeof(int32_t), hipMemcpyDeviceToHost, g->stream));
    HIP_TRY(hipStreamSynchronize(g->stream));
    std::sort(sel.begin(), sel.end(), [](unsigned long long x, unsigned long long y) { return x > y; });
    *n_profiles_out = (int)n_prof;
    std::vector<double> x((size_t)m), xbest((size_t)m);
    double vbest = 0.0;
    int64_t cbest = -1;
    for (size_t i = 0; i < todo; ++i) {
        double v = 0.0;
        const int64_t c = 0xFFFFFFFFu - (unsigned)sel[i];            // the candidate in the key
        const int rc = solve_profile_lp(m, n, K, g->hA.data(), g->hB.data(), g->hprior.data(),
                                        &hb[(size_t)c * K], x.data(), &v);
        if (rc == 2) return fail(BSSE_ESTATE, "the simplex method did not converge");
        if (rc == 1) continue;        // realised under rounded operands only (bf16 storage)
        if (cbest < 0 || v > vbest) { vbest = v; cbest = c; xbest = x; }
    }
    *n_solved_out = (int)todo;
    if (cbest < 0) return fail(BSSE_ESTATE, "no realised profile has a feasible program");
    for (int i = 0; i < m; ++i) x_out[i] = (float)xbest[(size_t)i];
    *value_out = vbest;
    if (profile_out) memcpy(profile_out, &hb[(size_t)cbest * K], (size_t)K * sizeof(int32_t));
    return BSSE_OK;
}

// ------------------------------------------------------------------------------- timing
extern "C" bsse_status bsse_set_timing(bsse_game *g, int enabled)
{
    g_err[0] = 0;
    if (!g) return fail(BSSE_EINVAL, "game is NULL");
    DeviceGuard dg(g->device);
    bsse_status st0 = sync_all(g);
    if (st0 != BSSE_OK) return st0;
    for (hipEvent_t e : g->ev) g->ev_pool.push_back(e);
    g->ev.clear();
    g->timed_ms = 0.0; g->timed_launches = 0;
    g->timing = enabled != 0;
    return BSSE_OK;
}

extern "C" bsse_status bsse_get_timing(bsse_game *g, double *kernel_ms_out, int64_t *launches_out)
{
    g_err[0] = 0;
    if (!g || !kernel_ms_out || !launches_out) return fail(BSSE_EINVAL, "NULL argument");
    DeviceGuard dg(g->device);
    bsse_status st = sync_all(g);
    if (st != BSSE_OK) return st;
    st = drain_timing(g);
    if (st != BSSE_OK) return st;
    *kernel_ms_out = g->timed_ms;
    *launches_out = g->timed_launches;
    return BSSE_OK;
}
