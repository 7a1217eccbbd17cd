// C ABI of the SpeCache decode-step library (see include/specache.h): argument
// checks, buffer ownership, the append bookkeeping of the residual policy and the
// stream/event protocol between the main stream and the prefetch side stream.
// All arithmetic of the method lives in the kernels.
#include "../../include/specache.h"

#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "kernels.h"
#include "layout.h"
#include "rows_args.h"
#include <cstdlib>

#include <link.h>
#include <unistd.h>

using namespace specache;

namespace specache {
LaunchEvents& pending_launch_events() {
    static thread_local LaunchEvents le;
    return le;
}
int& merger_polls() {
    static int polls = kMergerPolls;
    return polls;
}
int& kernel_choice() {
    static int choice = 0;
    return choice;
}
}  // namespace specache

namespace {

struct Layer {
    LayerView view{};
    int N = 0, Nq = 0;
    void* host_alloc = nullptr;
    uint16_t* slot[2] = {nullptr, nullptr};
    int32_t* slot_idx[2] = {nullptr, nullptr};
    bool slot_filled[2] = {false, false};
    hipEvent_t gathered[2] = {nullptr, nullptr};
    hipStream_t gather_stream[2] = {nullptr, nullptr};
    // Ordering of a slot's reader (attend) before its next writer (gather).  An event record costs
    // the stream about as much as a small kernel, so attend records `attended` only when the later
    // gather could not be ordered otherwise: an attend enqueued on the stream of the layer's last
    // score_topk precedes, in that stream, the next score_topk's `idx_ready` record, which every
    // gather waits for.  The sequence numbers tell whether that record came after the attend.
    hipEvent_t attended[2] = {nullptr, nullptr};
    bool attended_recorded[2] = {false, false};
    hipStream_t attend_stream[2] = {nullptr, nullptr};
    uint64_t attend_seq[2] = {0, 0};     // 0: no attend has read the slot
    hipEvent_t idx_ready = nullptr;
    bool idx_ready_recorded = false;
    hipStream_t idx_ready_stream = nullptr;       // where idx_ready was recorded
    hipStream_t select_origin_stream = nullptr;   // the stream score_topk was called on (the same, unless ArgTopK runs aside)
    uint64_t idx_ready_seq = 0;
    const int32_t* last_gather_idx = nullptr;
    int last_gather_slot = -1;
    // ArgTopK on the gather's stream (specache_score + specache_select_gather): the layer has a key
    // array of its own, which the selection reads on the side stream while the caller's stream goes
    // on to other layers.  The next scoring pass of the layer waits for the gather that followed
    // that selection; the attend after it then needs no wait of its own for the same slot.
    uint32_t* keys = nullptr;            // [rows][logit_stride]
    bool keys_valid = false;
    int keys_Nq = 0;
    int keys_reader_slot = -1;           // slot of the select_gather that read `keys` last
    bool gathered_waited_set[2] = {false, false};
    hipStream_t gathered_waited[2] = {nullptr, nullptr};   // stream that has already waited for gathered[s]
    // Where scoring and attention are one call the merge of its partial results stores `scored_value` to the word `scored_word`, and the
    // selection's stream waits for that value: an event, pending as it always is when the selection is enqueued, costs
    // the issuing thread 10 us more (launch, event, wait, launch on the other stream: 19.7 us; with the word: 8.6).
    uint32_t* arrived = nullptr;         // [rows + 1][kFinishStride] counters of the merge inside a launch (finish_row.h), zero between launches
    uint64_t* scored_word = nullptr;     // signal memory, one word per layer (layers may be stepped on different streams)
    uint64_t scored_value = 0;
    bool scored_by_word = false;         // the layer's last scoring announced itself through the word, not idx_ready
    hipEvent_t selected = nullptr;       // a selection without a gather behind it (select_gather with slot -1)
    bool selected_pending = false;
    hipStream_t selected_stream = nullptr;
};

thread_local std::string g_create_error;
int g_fail_alloc_at = 0;   // specache_debug_fail_alloc

}  // namespace

struct specache_ctx {
    specache_config cfg{};
    int device = 0;
    float sm_scale = 0.f;
    std::vector<Layer> layers;
    void* device_memory = nullptr;   // every buffer on the device is part of this one
    float* logits = nullptr;     // [rows*G*2][logit_stride]
    uint32_t* keys = nullptr;    // [rows][logit_stride]
    float* lse = nullptr;        // (max, sum) per slice of every head's speculative row (log-probability selection)
    size_t logit_stride = 0;
    AttendScratch scratch{};
    TopkScratch topk_scratch{};
    int scored_layer = -1, scored_rows = 0, scored_N = 0, scored_Nq = 0;
    bool logits_kept = false;    // the last scoring pass left its logits in `logits` (the one-pass score + attend need not)
    bool q_kept = false;         // it left a copy of its queries in `lse` instead (that buffer serves the other selection form)
    uint64_t seq = 0;            // counts the calls that order streams (see Layer)
    hipStream_t last_gather_stream = nullptr;   // stream of the previous specache_gather, of any layer
    bool last_gather_stream_set = false;
    // ArgTopK on a stream of the library's own (async_select): the scoring pass stays on the caller's
    // stream, which goes on to the attention kernels while the selection runs beside them
    bool async_select = false;
    hipStream_t select_stream = nullptr;
    hipEvent_t scored = nullptr;            // scoring pass done (recorded on the caller's stream)
    hipEvent_t last_select = nullptr;       // idx_ready of the most recent selection: it has read ctx->keys
    // selections on the gather's stream: those of two side streams may overlap, so the candidate
    // arrays of the two-launch ArgTopK exist twice, each remembering its last user
    bool select_on_gather = false;
    // Whether a word may order the selection (see Layer::scored_word, words_may_order).  No: the device cannot wait for one,
    // the caller wants events, or kernels of different queues may run one at a time.
    bool scores_by_word = false, events_wanted = false, one_at_a_time = false;
    unsigned long long objects_seen = 0;   // how many objects had been loaded into the process when they were looked at last
    struct SelectScratch { TopkScratch s{}; bool used = false; hipStream_t stream = nullptr; hipEvent_t done = nullptr; };
    SelectScratch select_scratch[2];
    int select_scratch_next = 0;
    std::string err;
    // optional per-kernel timing: (start, stop) event pairs recorded around each launch
    bool timing = false;
    std::vector<hipEvent_t> ev_pool;
    struct Span { int kind; hipEvent_t a, b; };
    std::vector<Span> spans;
};

namespace {

int fail(specache_ctx* ctx, int code, const std::string& msg) {
    if (ctx) ctx->err = msg; else g_create_error = msg;
    return code;
}

int fail_hip(specache_ctx* ctx, hipError_t e, const char* what) {
    (void)hipGetLastError();
    return fail(ctx, e == hipErrorOutOfMemory ? SPECACHE_ENOMEM : SPECACHE_EHIP,
                std::string(what) + ": " + hipGetErrorString(e));
}

#define SPC_HIP(ctx, call)                                     \
    do {                                                       \
        hipError_t e_ = (call);                                \
        if (e_ != hipSuccess) return fail_hip(ctx, e_, #call); \
    } while (0)

// Brackets one launcher call with a pair of timing events when timing is on.  on_kernel: the
// events are handed to the launcher's first SPC_LAUNCH instead, which times that kernel alone.
struct TimedLaunch {
    specache_ctx* ctx;
    hipStream_t st;
    int kind;
    bool on_kernel;
    hipEvent_t a = nullptr, b = nullptr;
    static hipEvent_t take(specache_ctx* c) {
        if (!c->ev_pool.empty()) { hipEvent_t e = c->ev_pool.back(); c->ev_pool.pop_back(); return e; }
        hipEvent_t e = nullptr;
        return hipEventCreate(&e) == hipSuccess ? e : nullptr;
    }
    TimedLaunch(specache_ctx* c, hipStream_t s, int k, bool kernel_events = false)
        : ctx(c), st(s), kind(k), on_kernel(kernel_events) {
        if (!c->timing) return;
        a = take(c);
        b = take(c);
        if (!a || !b) return;
        if (on_kernel) pending_launch_events() = LaunchEvents{a, b};
        else (void)hipEventRecord(a, st);
    }
    ~TimedLaunch() {
        if (!a || !b) return;
        if (on_kernel) {
            LaunchEvents& le = pending_launch_events();
            if (le.stop) {   // no kernel took them (nothing was launched): no span
                le = LaunchEvents{};
                ctx->ev_pool.push_back(a);
                ctx->ev_pool.push_back(b);
                return;
            }
        } else {
            (void)hipEventRecord(b, st);
        }
        ctx->spans.push_back({kind, a, b});
    }
};

bool being_captured(hipStream_t st) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(st, &status) != hipSuccess || status != hipStreamCaptureStatusNone;
}

// An ordering event completed by a kernel's own dispatch packet instead of a record behind it: one call
// into the runtime less per event, and the issuing thread's calls are what bounds a step with little to
// fetch.  Between arm() and landed() exactly one launcher runs; landed() is false when that launcher
// launched nothing, when the launch carries timing events, or when st is being captured: there a record is an edge of the
// graph, and an event that a launch carries is none (the caller then records the event itself).
struct CarriedEvent {
    bool armed = false;
    CarriedEvent(specache_ctx* c, hipStream_t st, hipEvent_t ev) {
        if (c->timing || !ev || being_captured(st)) return;
        pending_launch_events() = LaunchEvents{nullptr, ev};
        armed = true;
    }
    bool landed() {
        if (!armed) return false;
        armed = false;
        LaunchEvents& le = pending_launch_events();
        const bool taken = le.stop == nullptr;
        le = LaunchEvents{};
        return taken;
    }
    ~CarriedEvent() { if (armed) pending_launch_events() = LaunchEvents{}; }
};

// The wait for a word is a kernel without a bound, which ends only if the merging launch on another queue runs beside it or before
// it.  Submission order sees to that (the merge is enqueued first) unless something between the streams and the queues holds
// kernels back: a tool that collects counters or traces threads runs the kernels of all queues one at a time, and without direct
// dispatch a thread per stream submits them in an order of its own.  No call reports such a tool, so every sign of one
// counts: its variables in the environment, and its libraries among the process's objects, however late they are loaded.
bool environment_names_a_tool() {
    for (char** e = environ; e && *e; ++e)
        for (const char* name : {"ROCPROF", "ROCP_", "HSA_TOOLS_LIB="})
            if (std::strncmp(*e, name, std::strlen(name)) == 0) return true;
    const char* direct = std::getenv("AMD_DIRECT_DISPATCH");
    return direct && std::strcmp(direct, "0") == 0;
}

int look_at_object(dl_phdr_info* info, size_t, void* data) {
    specache_ctx* ctx = (specache_ctx*)data;
    const char* slash = info->dlpi_name ? std::strrchr(info->dlpi_name, '/') : nullptr;
    const char* name = slash ? slash + 1 : info->dlpi_name ? info->dlpi_name : "";
    // (every HIP process has the library that tools register with, and markers alone hold nothing back)
    if (std::strncmp(name, "librocprofiler", 14) == 0 && !std::strstr(name, "-register") && !std::strstr(name, "roctx"))
        ctx->one_at_a_time = true;
    ctx->objects_seen = info->dlpi_adds;
    return 0;
}

int objects_loaded(dl_phdr_info* info, size_t, void* data) {
    *(unsigned long long*)data = info->dlpi_adds;
    return 1;   // the count comes with every object: one is enough
}

bool words_may_order(specache_ctx* ctx) {
    if (!ctx->scores_by_word || ctx->events_wanted || ctx->one_at_a_time) return false;
    unsigned long long loaded = 0;
    dl_iterate_phdr(objects_loaded, &loaded);
    if (loaded != ctx->objects_seen) dl_iterate_phdr(look_at_object, ctx);
    return !ctx->one_at_a_time;
}

int check_ctx_layer(specache_ctx* ctx, int32_t layer) {
    if (!ctx) return SPECACHE_EINVAL;
    if (layer < 0 || layer >= ctx->cfg.n_layers) return fail(ctx, SPECACHE_EINVAL, "layer out of range");
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != ctx->device)
        return fail(ctx, SPECACHE_EINVAL, "the context's device is not the current HIP device");
    return SPECACHE_OK;
}

void free_all(specache_ctx* ctx) {
    for (Layer& L : ctx->layers) {
        if (L.host_alloc) (void)hipHostFree(L.host_alloc);
        for (int s = 0; s < 2; ++s) {
            if (L.gathered[s]) (void)hipEventDestroy(L.gathered[s]);
            if (L.attended[s]) (void)hipEventDestroy(L.attended[s]);
        }
        if (L.idx_ready) (void)hipEventDestroy(L.idx_ready);
        if (L.selected) (void)hipEventDestroy(L.selected);
        (void)hipFree(L.scored_word);
    }
    for (auto& sp : ctx->spans) { (void)hipEventDestroy(sp.a); (void)hipEventDestroy(sp.b); }
    for (hipEvent_t e : ctx->ev_pool) (void)hipEventDestroy(e);
    (void)hipFree(ctx->device_memory);
    if (ctx->select_stream) (void)hipStreamDestroy(ctx->select_stream);
    if (ctx->scored) (void)hipEventDestroy(ctx->scored);
}

// The scoring pass of one layer on stream st: low-bit logits of every query row, selection keys of
// the last row, and the optional rewrites of those keys (mixed-cache selection, log-probability form).
// done / done_carried: an event to complete when the keys are final; *done_carried tells whether the scoring
// launch's own dispatch packet does that (only where no rewrite of the keys follows it).
int score_phase(specache_ctx* ctx, Layer& L, const void* q, int n_rows, uint32_t* keys, hipStream_t st,
                const LayerView* fused_view = nullptr, hipEvent_t done = nullptr, bool* done_carried = nullptr) {
    if (L.Nq > 0) {
        TimedLaunch t(ctx, st, SPECACHE_K_SCORE, /*kernel_events=*/true);
        const bool rewrites = (ctx->cfg.select_cache == SPECACHE_SELECT_MIXED && L.last_gather_slot >= 0) ||
                              (ctx->cfg.select_form == SPECACHE_SELECT_MAX_LOGPROB && L.view.G > 1);
        CarriedEvent carried(ctx, st, rewrites ? nullptr : done);
        SPC_HIP(ctx, launch_score(fused_view ? *fused_view : L.view, q, n_rows, L.Nq, ctx->sm_scale, ctx->logits, ctx->logit_stride, keys,
                                  ctx->logit_stride, st));
        if (done_carried) *done_carried = carried.landed();
        // selection on the mixed cache: the positions staged by the layer's last gather are scored with
        // their 16-bit keys (that slot is the one the coming attend reads; the next gather into it
        // waits for this stream's next selection event, so it cannot overtake the patch)
        if (ctx->cfg.select_cache == SPECACHE_SELECT_MIXED && L.last_gather_slot >= 0) {
            const int sl = L.last_gather_slot;
            if (L.gather_stream[sl] != st) SPC_HIP(ctx, hipStreamWaitEvent(st, L.gathered[sl], 0));
            SPC_HIP(ctx, launch_patch_staged(L.view, q, n_rows, L.Nq, ctx->sm_scale, L.slot[sl], L.slot_idx[sl], ctx->logits,
                                             ctx->logit_stride, keys, ctx->logit_stride, st));
        }
        // several query heads per KV head and the log-probability form: the keys are rewritten from
        // the logits shifted by every head's log-sum-exp (one head: same order, nothing to do)
        if (ctx->cfg.select_form == SPECACHE_SELECT_MAX_LOGPROB && L.view.G > 1)
            SPC_HIP(ctx, launch_select_logprob(L.view, n_rows, L.Nq, ctx->logits, ctx->logit_stride, ctx->lse, keys,
                                               ctx->logit_stride, st));
    }
    return SPECACHE_OK;
}

// Orders a gather into `slot` on stream st after the attend that read the slot last.
int order_gather_after_attend(specache_ctx* ctx, Layer& L, int slot, hipStream_t st) {
    if (L.attend_seq[slot] != 0 && L.attend_stream[slot] != st) {
        const bool behind_idx_ready = L.idx_ready_recorded && L.attend_stream[slot] == L.select_origin_stream &&
                                      L.attend_seq[slot] < L.idx_ready_seq;
        if (!L.attended_recorded[slot] && !behind_idx_ready) {
            // a second gather into the slot without a new score_topk in between: record now, on the
            // attend's stream, which orders this gather after everything enqueued there so far
            SPC_HIP(ctx, hipEventRecord(L.attended[slot], L.attend_stream[slot]));
            L.attended_recorded[slot] = true;
        }
        if (L.attended_recorded[slot]) SPC_HIP(ctx, hipStreamWaitEvent(st, L.attended[slot], 0));
    }
    return SPECACHE_OK;
}

// Launches the gather of `idx` into `slot` on st and records its completion.  select_out: the gather's launch also ranks
// the layer's keys, and idx (= select_out) receives the positions it fetches.
int gather_phase(specache_ctx* ctx, Layer& L, int Nq, const int32_t* idx, int slot, hipStream_t st, int32_t* select_out = nullptr) {
    // the slot's previous gather, if it ran on another stream that this one has not waited for
    if (L.slot_filled[slot] && L.gather_stream[slot] != st && !(L.gathered_waited_set[slot] && L.gathered_waited[slot] == st))
        SPC_HIP(ctx, hipStreamWaitEvent(st, L.gathered[slot], 0));
    bool gathered_carried = false;
    {
        TimedLaunch t(ctx, st, SPECACHE_K_GATHER);
        CarriedEvent gathered(ctx, st, L.gathered[slot]);
        // a caller that alternates side streams has two gathers on the link at a time
        const bool link_shared = ctx->last_gather_stream_set && ctx->last_gather_stream != st;
        if (select_out)
            SPC_HIP(ctx, launch_select_gather(L.view, Nq, L.keys, ctx->logit_stride, select_out, L.slot[slot], L.slot_idx[slot],
                                              link_shared, st));
        else
            SPC_HIP(ctx, launch_gather(L.view, Nq, idx, L.slot[slot], L.slot_idx[slot], link_shared,
                                       L.idx_ready_recorded && L.idx_ready_stream == st, st));
        gathered_carried = gathered.landed();
        ctx->last_gather_stream = st;
        ctx->last_gather_stream_set = true;
    }
    if (!gathered_carried) SPC_HIP(ctx, hipEventRecord(L.gathered[slot], st));
    L.gather_stream[slot] = st;
    L.gathered_waited_set[slot] = false;
    L.slot_filled[slot] = true;
    L.last_gather_idx = idx;
    L.last_gather_slot = slot;
    return SPECACHE_OK;
}

// ---- scratch memory for callers that cannot allocate (specache_attend_static) ----------------------
// A file-scope device array holds the attention partials of such a call.  Every GPU the library
// runs on carries its own copy at its own address; in host code the array's name is only a handle
// for hipGetSymbolAddress, never an address to hand to a kernel.  The address is looked up once
// per device, with that device current, and kept.
constexpr size_t kStaticScratchBytes = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
float* g_static_scratch[kMaxDevices] = {};

int static_scratch_of_current_device(specache_ctx* ctx, float** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail_hip(ctx, e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail(ctx, SPECACHE_EINVAL, "device ordinal beyond the static scratch table");
    if (!g_static_scratch[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) return fail_hip(ctx, e != hipSuccess ? e : hipErrorInvalidSymbol, "hipGetSymbolAddress(scratch)");
        g_static_scratch[dev] = (float*)ptr;
    }
    *out = g_static_scratch[dev];
    return SPECACHE_OK;
}

}  // namespace

extern "C" {

int specache_plan_append(int32_t residual, int32_t group, int32_t n_tokens, int32_t n_quantized, int32_t n_new,
                         int32_t* n_flush_groups) {
    if (group <= 0 || residual < group || residual % group || n_tokens < n_quantized || n_quantized < 0 ||
        n_tokens - n_quantized >= residual || n_new < 0 || !n_flush_groups)
        return SPECACHE_EINVAL;
    const long total = (long)(n_tokens - n_quantized) + n_new;
    *n_flush_groups = total >= residual ? (int32_t)((total - residual) / group + 1) : 0;
    return SPECACHE_OK;
}

int specache_create(const specache_config* cfg, specache_ctx** out) {
    if (out) *out = nullptr;
    if (!cfg || !out) return fail(nullptr, SPECACHE_EINVAL, "null config or output pointer");
    const specache_config& c = *cfg;
    if (c.n_layers < 1 || c.batch < 1 || c.n_kv_heads < 1 || c.n_q_heads < 1)
        return fail(nullptr, SPECACHE_EINVAL, "n_layers, batch and head counts must be positive");
    if (c.n_q_heads % c.n_kv_heads) return fail(nullptr, SPECACHE_EINVAL, "n_q_heads must be a multiple of n_kv_heads");
    const int G = c.n_q_heads / c.n_kv_heads;
    if (G != 1 && G != 2 && G != 4 && G != 8) return fail(nullptr, SPECACHE_EINVAL, "n_q_heads / n_kv_heads must be 1, 2, 4 or 8");
    if (c.head_dim != kD) return fail(nullptr, SPECACHE_EINVAL, "head_dim must be 128");
    if (c.bits != 1 && c.bits != 2 && c.bits != 4) return fail(nullptr, SPECACHE_EINVAL, "bits must be 1, 2 or 4");
    if (c.one_bit_form != SPECACHE_1BIT_IMPROVED && c.one_bit_form != SPECACHE_1BIT_KIVI)
        return fail(nullptr, SPECACHE_EINVAL, "one_bit_form must be SPECACHE_1BIT_IMPROVED or SPECACHE_1BIT_KIVI");
    if (c.async_select < 0 || c.async_select > 2) return fail(nullptr, SPECACHE_EINVAL, "async_select must be 0, 1 or 2");
    if (c.select_cache != SPECACHE_SELECT_LOWBIT && c.select_cache != SPECACHE_SELECT_MIXED)
        return fail(nullptr, SPECACHE_EINVAL, "select_cache must be SPECACHE_SELECT_LOWBIT or SPECACHE_SELECT_MIXED");
    if (c.select_form != SPECACHE_SELECT_MAX_LOGIT && c.select_form != SPECACHE_SELECT_MAX_LOGPROB)
        return fail(nullptr, SPECACHE_EINVAL, "select_form must be SPECACHE_SELECT_MAX_LOGIT or SPECACHE_SELECT_MAX_LOGPROB");
    if (c.group != 32 && c.group != 64 && c.group != 128)
        return fail(nullptr, SPECACHE_EINVAL, "group must be 32, 64 or 128");
    if (c.residual < c.group || c.residual % c.group || c.residual > 256)
        return fail(nullptr, SPECACHE_EINVAL, "residual must be a multiple of group in [group, 256]");
    if (c.max_seq < 64 || c.max_seq % 64) return fail(nullptr, SPECACHE_EINVAL, "max_seq must be a positive multiple of 64");
    if (c.topk < 1 || c.topk > 4096) return fail(nullptr, SPECACHE_EINVAL, "topk must be in [1, 4096]");
    if (c.dtype != SPECACHE_FP16 && c.dtype != SPECACHE_BF16) return fail(nullptr, SPECACHE_EINVAL, "dtype must be fp16 or bf16");
    {
        // attend splits a row into chunks whose partial results one workgroup merges
        int most = 0;
        for (int n = 1; n <= 2; ++n) {
            const int ch = attend_main_chunk_tokens(G * n), ec = attend_extra_chunk_tokens();
            const int chunks = (c.max_seq + ch - 1) / ch + (c.topk + c.residual + 1 + ec - 1) / ec;
            most = chunks > most ? chunks : most;
        }
        if (most > attend_max_chunks())
            return fail(nullptr, SPECACHE_EINVAL, "max_seq is beyond what attend splits into chunks (about 650000 tokens, "
                                                  "320000 with 8 query heads per KV head)");
    }

    specache_ctx* ctx = new (std::nothrow) specache_ctx();
    if (!ctx) return fail(nullptr, SPECACHE_ENOMEM, "host allocation failed");
    ctx->cfg = c;
    ctx->sm_scale = c.sm_scale > 0.f ? c.sm_scale : 1.0f / std::sqrt((float)kD);
    hipError_t e = hipGetDevice(&ctx->device);
    if (e != hipSuccess) { delete ctx; return fail_hip(nullptr, e, "hipGetDevice"); }

    const int rows = c.batch * c.n_kv_heads;
    const size_t cap = (size_t)c.max_seq;
    ctx->layers.resize(c.n_layers);
    auto bail = [&](hipError_t err, const char* what) {
        const int rc = fail_hip(nullptr, err, what);
        free_all(ctx);
        delete ctx;
        return rc;
    };
    // specache_debug_fail_alloc: the n-th allocating call of this create reports hipErrorOutOfMemory instead of running
    int fail_at = g_fail_alloc_at;
    g_fail_alloc_at = 0;
    int alloc_no = 0;
#define SPC_ALLOC(call)                                                             \
    do {                                                                            \
        hipError_t e_ = ++alloc_no == fail_at ? hipErrorOutOfMemory : (call);       \
        if (e_ != hipSuccess) return bail(e_, #call);                               \
    } while (0)

    // The events only order streams of this device among themselves and the host never waits on
    // them, so they need no system-scope fence (measured: 2.3 us per layer-step less).
    const unsigned kOrderEventFlags = hipEventDisableTiming | hipEventDisableSystemFence;
    for (Layer& L : ctx->layers) {
        LayerView& v = L.view;
        v.rows = rows; v.G = G; v.bits = c.bits; v.group = c.group; v.R = c.residual;
        v.one_bit_plain = c.bits == 1 && c.one_bit_form == SPECACHE_1BIT_KIVI;
        v.max_seq = c.max_seq; v.topk = c.topk; v.bf16 = c.dtype == SPECACHE_BF16;
        v.kc_stride = (cap + kTileTokens - 1) / kTileTokens * k_tile_bytes(c.bits);
        v.vc_stride = cap / kBlockTokens * code_block_bytes(c.bits);
        v.km_stride = cap / c.group * kD;
        v.vm_stride = cap * (kD / c.group);
        SPC_ALLOC(hipHostMalloc(&L.host_alloc, (size_t)rows * cap * kRowBytes, hipHostMallocDefault));
        void* dev_view = nullptr;
        SPC_ALLOC(hipHostGetDevicePointer(&dev_view, L.host_alloc, 0));
        v.host = (uint16_t*)dev_view;
        for (int s = 0; s < 2; ++s) {
            SPC_ALLOC(hipEventCreateWithFlags(&L.gathered[s], kOrderEventFlags));
            SPC_ALLOC(hipEventCreateWithFlags(&L.attended[s], kOrderEventFlags));
        }
        SPC_ALLOC(hipEventCreateWithFlags(&L.idx_ready, kOrderEventFlags));
    }
    ctx->async_select = c.async_select == SPECACHE_SELECT_STREAM_OWN;
    ctx->select_on_gather = c.async_select == SPECACHE_SELECT_STREAM_GATHER;
    if (ctx->select_on_gather) {
        int waits = 0;
        (void)hipDeviceGetAttribute(&waits, hipDeviceAttributeCanUseStreamWaitValue, ctx->device);
        ctx->scores_by_word = waits != 0;
        ctx->one_at_a_time = environment_names_a_tool();
        dl_iterate_phdr(look_at_object, ctx);
        for (Layer& L : ctx->layers) {
            SPC_ALLOC(hipEventCreateWithFlags(&L.selected, kOrderEventFlags));
            if (ctx->scores_by_word) {
                SPC_ALLOC(hipExtMallocWithFlags((void**)&L.scored_word, 8, hipMallocSignalMemory));
                *L.scored_word = 0;
            }
        }
    }
    if (ctx->async_select) {
        SPC_ALLOC(hipStreamCreateWithFlags(&ctx->select_stream, hipStreamNonBlocking));
        SPC_ALLOC(hipEventCreateWithFlags(&ctx->scored, kOrderEventFlags));
    }
    // One allocation for the device's buffers: a context of two layers has 27 (33 where a row may take two launches to select), whose
    // hipMalloc and hipFree took 75 of the 135 us of its creation and as many of closing it.  The pass without a base adds the sizes up.
    ctx->logit_stride = cap;
    int max_main = 0;
    for (int n = 1; n <= 2; ++n) {
        const int ch = attend_main_chunk_tokens(G * n);
        const int m = (int)((cap + ch - 1) / ch);
        max_main = m > max_main ? m : max_main;
    }
    if (rows_max_main_chunks(rows, (int)cap) > max_main) max_main = rows_max_main_chunks(rows, (int)cap);
    const int ec = attend_extra_chunk_tokens();
    ctx->scratch.max_chunks = max_main + (c.topk + c.residual + 1 + ec - 1) / ec;
    // no more than the merge kernel takes: with that many candidates rows_kernel splits a row less finely
    if (ctx->scratch.max_chunks > attend_max_chunks()) ctx->scratch.max_chunks = attend_max_chunks();
    const int parts = topk_parts((int)cap, c.topk);
    ctx->topk_scratch.max_parts = parts;
    for (auto& ss : ctx->select_scratch) ss.s.max_parts = ctx->select_on_gather ? parts : 0;
    size_t used = 0, idx_end = 0, cleared_end = 0;
    bool refused = false;   // by specache_debug_fail_alloc, to which a buffer's place is an allocation like any other
    for (int pass = 0; pass < 2; ++pass) {
        uint8_t* base = (uint8_t*)ctx->device_memory;
        used = 0;
        auto place = [&](auto*& ptr, size_t bytes) {
            const size_t align = bytes >= 65536 ? 4096 : 256;
            used = (used + align - 1) / align * align;
            if (base && ++alloc_no == fail_at) refused = true;
            ptr = base ? reinterpret_cast<std::remove_reference_t<decltype(ptr)>>(base + used) : nullptr;
            used += bytes;
        };
        // what starts at a value of its own first: index lists (-1), then counters (0)
        for (Layer& L : ctx->layers)
            for (int s = 0; s < 2; ++s) place(L.slot_idx[s], (size_t)rows * c.topk * 4);
        idx_end = used;
        for (Layer& L : ctx->layers) place(L.arrived, ((size_t)rows + 1) * kFinishStride * 4);
        cleared_end = used;
        for (Layer& L : ctx->layers) {
            LayerView& v = L.view;
            place(v.kc, rows * v.kc_stride);
            place(v.vc, rows * v.vc_stride);
            place(v.km, rows * v.km_stride * 4);
            place(v.vm, rows * v.vm_stride * 4);
            place(v.ring, (size_t)rows * c.residual * kRowBytes);
            for (int s = 0; s < 2; ++s) place(L.slot[s], (size_t)rows * c.topk * kRowBytes);
            if (ctx->select_on_gather) place(L.keys, (size_t)rows * cap * 4);
        }
        place(ctx->logits, (size_t)rows * G * 2 * cap * 4);
        place(ctx->keys, (size_t)rows * cap * 4);
        const size_t floats = select_logprob_scratch_floats(rows, G, cap), queries = (size_t)rows * G * 2 * kD / 2;
        place(ctx->lse, (floats > queries ? floats : queries) * 4);
        place(ctx->scratch.part_o, (size_t)rows * ctx->scratch.max_chunks * G * 2 * kD * 4);
        place(ctx->scratch.part_ml, (size_t)rows * ctx->scratch.max_chunks * G * 2 * 2 * 4);
        for (TopkScratch* s : {&ctx->topk_scratch, &ctx->select_scratch[0].s, &ctx->select_scratch[1].s})
            if (s->max_parts > 1) {
                place(s->cand_keys, (size_t)rows * parts * c.topk * 4);
                place(s->cand_idx, (size_t)rows * parts * c.topk * 4);
            }
        if (pass == 0) SPC_ALLOC(hipMalloc(&ctx->device_memory, used));
    }
    if (refused) return bail(hipErrorOutOfMemory, "a buffer's place");
    SPC_ALLOC(hipMemset(ctx->device_memory, 0xFF, idx_end));
    SPC_ALLOC(hipMemset((uint8_t*)ctx->device_memory + idx_end, 0, cleared_end - idx_end));
    SPC_ALLOC(hipDeviceSynchronize());
#undef SPC_ALLOC
    {
        // the static scratch array's address on this device, for specache_attend_static (a failure
        // here only surfaces when that entry point is called, with its own message)
        float* unused = nullptr;
        (void)static_scratch_of_current_device(nullptr, &unused);
    }
    *out = ctx;
    return SPECACHE_OK;
}

int specache_destroy(specache_ctx* ctx) {
    if (!ctx) return SPECACHE_OK;
    (void)hipDeviceSynchronize();
    free_all(ctx);
    delete ctx;
    return SPECACHE_OK;
}

const char* specache_last_error(const specache_ctx* ctx) { return ctx ? ctx->err.c_str() : g_create_error.c_str(); }

int specache_counts(const specache_ctx* ctx, int32_t layer, int32_t* n_tokens, int32_t* n_quantized) {
    if (!ctx || layer < 0 || layer >= ctx->cfg.n_layers) return SPECACHE_EINVAL;
    if (n_tokens) *n_tokens = ctx->layers[layer].N;
    if (n_quantized) *n_quantized = ctx->layers[layer].Nq;
    return SPECACHE_OK;
}

int specache_quantize_append(specache_ctx* ctx, int32_t layer, const void* k_new, const void* v_new, int32_t n_new,
                             void* stream) {
    if (int rc = check_ctx_layer(ctx, layer)) return rc;
    if (n_new < 0 || (n_new > 0 && (!k_new || !v_new))) return fail(ctx, SPECACHE_EINVAL, "null k_new/v_new or negative n_new");
    if (n_new == 0) return SPECACHE_OK;
    Layer& L = ctx->layers[layer];
    if ((long)L.N + n_new > ctx->cfg.max_seq) return fail(ctx, SPECACHE_ECAPACITY, "append exceeds max_seq");
    int32_t n_flush = 0;
    if (specache_plan_append(ctx->cfg.residual, ctx->cfg.group, L.N, L.Nq, n_new, &n_flush) != SPECACHE_OK)
        return fail(ctx, SPECACHE_ESTATE, "inconsistent token counts");
    const int Nq1 = L.Nq + n_flush * ctx->cfg.group, N1 = L.N + n_new;
    hipStream_t st = (hipStream_t)stream;
    const int ring_from = Nq1 > L.N ? Nq1 : L.N;
    // The flush reads residual tokens from the ring, so it precedes the ring update, unless that leaves their places alone: nothing in
    // the ring, or not more than it holds (tokens a ring's length apart share a place).  Timed, the two are launches of their own.
    const bool together = n_flush > 0 && !ctx->timing && (L.N == L.Nq || N1 - L.Nq <= ctx->cfg.residual);
    if (n_flush > 0) {
        TimedLaunch t(ctx, st, SPECACHE_K_FLUSH);
        SPC_HIP(ctx, launch_flush(L.view, k_new, v_new, n_new, L.N, L.Nq, n_flush, together ? ring_from : -1, st));
    }
    if (!together) {
        TimedLaunch t(ctx, st, SPECACHE_K_APPEND_COPY);
        SPC_HIP(ctx, launch_append_copy(L.view, k_new, v_new, n_new, L.N, ring_from, st));
    }
    L.N = N1;
    L.Nq = Nq1;
    return SPECACHE_OK;
}

int specache_score_topk(specache_ctx* ctx, int32_t layer, const void* q, int32_t n_rows, int32_t* topk_idx_out,
                        void* stream) {
    if (int rc = check_ctx_layer(ctx, layer)) return rc;
    if (!q || !topk_idx_out) return fail(ctx, SPECACHE_EINVAL, "null q or topk_idx_out");
    if (n_rows != 1 && n_rows != 2) return fail(ctx, SPECACHE_EINVAL, "n_rows must be 1 or 2");
    if ((uintptr_t)q & 15) return fail(ctx, SPECACHE_EINVAL, "q must be 16-byte aligned");
    Layer& L = ctx->layers[layer];
    hipStream_t st = (hipStream_t)stream;
    hipStream_t tk = ctx->async_select ? ctx->select_stream : st;   // where ArgTopK runs
    // a gather still reading this index buffer must finish before it is overwritten
    if (L.last_gather_idx == topk_idx_out && L.last_gather_slot >= 0)
        SPC_HIP(ctx, hipStreamWaitEvent(tk, L.gathered[L.last_gather_slot], 0));
    // the key array is shared by all layers: the previous selection, running aside, must have read it
    if (ctx->async_select && ctx->last_select) SPC_HIP(ctx, hipStreamWaitEvent(st, ctx->last_select, 0));
    if (int rc = score_phase(ctx, L, q, n_rows, ctx->keys, st)) return rc;
    if (ctx->async_select) {
        SPC_HIP(ctx, hipEventRecord(ctx->scored, st));
        SPC_HIP(ctx, hipStreamWaitEvent(tk, ctx->scored, 0));
    }
    bool ready_carried = false;
    {
        TimedLaunch t(ctx, tk, SPECACHE_K_TOPK, /*kernel_events=*/true);
        CarriedEvent ready(ctx, tk, L.idx_ready);
        SPC_HIP(ctx, launch_topk(L.view.rows, L.Nq, ctx->cfg.topk, ctx->keys, ctx->logit_stride, topk_idx_out,
                                 ctx->topk_scratch, tk));
        ready_carried = ready.landed();
    }
    if (!ready_carried) SPC_HIP(ctx, hipEventRecord(L.idx_ready, tk));
    ctx->last_select = L.idx_ready;
    L.idx_ready_recorded = true;
    L.idx_ready_stream = tk;
    L.select_origin_stream = st;
    L.idx_ready_seq = ++ctx->seq;
    ctx->scored_layer = layer;
    ctx->scored_rows = n_rows;
    ctx->scored_N = L.N;
    ctx->scored_Nq = L.Nq;
    ctx->logits_kept = true;
    return SPECACHE_OK;
}

// The layer's key array is about to be rewritten on st: the selections that read it come first.
static int wait_for_keys_readers(specache_ctx* ctx, Layer& L, hipStream_t st) {
    // the layer's previous selection read L.keys on the stream of the gather that followed it
    if (L.keys_reader_slot >= 0) {
        const int sl = L.keys_reader_slot;
        if (L.gather_stream[sl] != st && !(L.gathered_waited_set[sl] && L.gathered_waited[sl] == st)) {
            SPC_HIP(ctx, hipStreamWaitEvent(st, L.gathered[sl], 0));
            L.gathered_waited[sl] = st;
            L.gathered_waited_set[sl] = true;
        }
        L.keys_reader_slot = -1;
    }
    if (L.selected_pending) {
        if (L.selected_stream != st) SPC_HIP(ctx, hipStreamWaitEvent(st, L.selected, 0));
        L.selected_pending = false;
    }
    return SPECACHE_OK;
}

// st waits for the layer's last scoring
static int wait_for_scored(specache_ctx* ctx, Layer& L, hipStream_t st) {
    if (st == L.idx_ready_stream) return SPECACHE_OK;
    if (!L.scored_by_word) {
        SPC_HIP(ctx, hipStreamWaitEvent(st, L.idx_ready, 0));
        return SPECACHE_OK;
    }
    // recorded into a graph the wait would be for a value long passed (waiting for an event from outside is an error there, too)
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    SPC_HIP(ctx, hipStreamIsCapturing(st, &capture));
    if (capture != hipStreamCaptureStatusNone)
        return fail(ctx, SPECACHE_ESTATE, "the side stream is being captured and the layer was scored outside the capture");
    SPC_HIP(ctx, hipStreamWaitValue64(st, L.scored_word, L.scored_value, hipStreamWaitValueGte));
    return SPECACHE_OK;
}

// "scored": what the selection waits for, and what orders a gather after the attends enqueued so far
static int record_scored(specache_ctx* ctx, Layer& L, int32_t layer, int32_t n_rows, hipStream_t st, bool carried = false,
                         bool by_word = false) {
    if (!carried && !by_word) SPC_HIP(ctx, hipEventRecord(L.idx_ready, st));
    L.scored_by_word = by_word;
    L.idx_ready_recorded = true;
    L.idx_ready_stream = st;
    L.select_origin_stream = st;
    L.idx_ready_seq = ++ctx->seq;
    L.keys_valid = true;
    L.keys_Nq = L.Nq;
    ctx->scored_layer = layer;
    ctx->scored_rows = n_rows;
    ctx->scored_N = L.N;
    ctx->scored_Nq = L.Nq;
    return SPECACHE_OK;
}

// specache_score, optionally with the copy of one new token carried by the scoring launch
static int score_impl(specache_ctx* ctx, int32_t layer, const void* q, int32_t n_rows, void* stream, const void* k_new,
                      const void* v_new) {
    if (int rc = check_ctx_layer(ctx, layer)) return rc;
    if (!ctx->select_on_gather) return fail(ctx, SPECACHE_ESTATE, "specache_score needs async_select = SPECACHE_SELECT_STREAM_GATHER");
    if (!q) return fail(ctx, SPECACHE_EINVAL, "null q");
    if (n_rows != 1 && n_rows != 2) return fail(ctx, SPECACHE_EINVAL, "n_rows must be 1 or 2");
    if ((uintptr_t)q & 15) return fail(ctx, SPECACHE_EINVAL, "q must be 16-byte aligned");
    Layer& L = ctx->layers[layer];
    hipStream_t st = (hipStream_t)stream;
    if (int rc = wait_for_keys_readers(ctx, L, st)) return rc;
    bool carried = false;
    if (k_new) {
        // the scoring launch appends token N: one more workgroup per row copies the pair
        LayerView fused = L.view;
        fused.tail_k = (const uint16_t*)k_new;
        fused.tail_v = (const uint16_t*)v_new;
        fused.tail_N0 = L.N;
        if (int rc = score_phase(ctx, L, q, n_rows, L.keys, st, &fused, L.idx_ready, &carried)) return rc;
        L.N += 1;   // only once the launch that copies the token is enqueued
    } else if (int rc = score_phase(ctx, L, q, n_rows, L.keys, st, nullptr, L.idx_ready, &carried)) {
        return rc;
    }
    ctx->logits_kept = true;
    return record_scored(ctx, L, layer, n_rows, st, carried);
}

int specache_score(specache_ctx* ctx, int32_t layer, const void* q, int32_t n_rows, void* stream) {
    return score_impl(ctx, layer, q, n_rows, stream, nullptr, nullptr);
}

int specache_append_score(specache_ctx* ctx, int32_t layer, const void* k_new, const void* v_new, const void* q,
                          int32_t n_rows, void* stream) {
    if (int rc = check_ctx_layer(ctx, layer)) return rc;
    if (!ctx->select_on_gather)
        return fail(ctx, SPECACHE_ESTATE, "specache_append_score needs async_select = SPECACHE_SELECT_STREAM_GATHER");
    if (!k_new || !v_new) return fail(ctx, SPECACHE_EINVAL, "null k_new or v_new");
    Layer& L = ctx->layers[layer];
    if ((long)L.N + 1 > ctx->cfg.max_seq) return fail(ctx, SPECACHE_ECAPACITY, "append exceeds max_seq");
    int32_t n_flush = 0;
    if (specache_plan_append(ctx->cfg.residual, ctx->cfg.group, L.N, L.Nq, 1, &n_flush) != SPECACHE_OK)
        return fail(ctx, SPECACHE_ESTATE, "inconsistent token counts");
    // a group leaves the residual with this token, or nothing is quantised yet (no scoring launch): two steps
    if (n_flush > 0 || L.Nq == 0) {
        if (int rc = specache_quantize_append(ctx, layer, k_new, v_new, 1, stream)) return rc;
        return score_impl(ctx, layer, q, n_rows, stream, nullptr, nullptr);
    }
    return score_impl(ctx, layer, q, n_rows, stream, k_new, v_new);
}

int specache_select_gather(specache_ctx* ctx, int32_t layer, int32_t* topk_idx_out, int32_t slot, void* side_stream) {
    if (int rc = check_ctx_layer(ctx, layer)) return rc;
    if (!ctx->select_on_gather)
        return fail(ctx, SPECACHE_ESTATE, "specache_select_gather needs async_select = SPECACHE_SELECT_STREAM_GATHER");
    if (!topk_idx_out) return fail(ctx, SPECACHE_EINVAL, "null topk_idx_out");
    if (slot < -1 || slot > 1) return fail(ctx, SPECACHE_EINVAL, "slot must be -1, 0 or 1");
    Layer& L = ctx->layers[layer];
    if (!L.keys_valid) return fail(ctx, SPECACHE_ESTATE, "specache_select_gather must follow specache_score of the layer");
    hipStream_t st = (hipStream_t)side_stream;
    if (int rc = wait_for_scored(ctx, L, st)) return rc;
    // a gather on another stream that still reads this index buffer must finish before it is overwritten
    if (L.last_gather_idx == topk_idx_out && L.last_gather_slot >= 0 && L.gather_stream[L.last_gather_slot] != st)
        SPC_HIP(ctx, hipStreamWaitEvent(st, L.gathered[L.last_gather_slot], 0));
    if (slot >= 0)
        if (int rc = order_gather_after_attend(ctx, L, slot, st)) return rc;
    // an earlier selection of the same keys on another stream: the next scoring pass waits for the
    // latest selection only, so this one goes behind it
    if (L.keys_reader_slot >= 0 && L.gather_stream[L.keys_reader_slot] != st)
        SPC_HIP(ctx, hipStreamWaitEvent(st, L.gathered[L.keys_reader_slot], 0));
    if (L.selected_pending && L.selected_stream != st) SPC_HIP(ctx, hipStreamWaitEvent(st, L.selected, 0));
    specache_ctx::SelectScratch* ss = nullptr;
    if (topk_parts(L.keys_Nq, ctx->cfg.topk) > 1) {   // (a row of one launch needs none, and waits for nobody's)
        // the candidate arrays last used on this stream, else the set whose turn it is (after its last user)
        for (auto& c : ctx->select_scratch)
            if (c.used && c.stream == st) ss = &c;
        if (!ss) {
            ss = &ctx->select_scratch[ctx->select_scratch_next];
            ctx->select_scratch_next ^= 1;
            if (ss->used) SPC_HIP(ctx, hipStreamWaitEvent(st, ss->done, 0));
        }
    }
    const TopkScratch& scratch = ss ? ss->s : ctx->select_scratch[0].s;
    const bool together = slot >= 0 && selects_and_gathers(L.view.rows, L.keys_Nq, ctx->cfg.topk);
    if (!together) {
        TimedLaunch t(ctx, st, SPECACHE_K_TOPK, /*kernel_events=*/true);
        SPC_HIP(ctx, launch_topk(L.view.rows, L.keys_Nq, ctx->cfg.topk, L.keys, ctx->logit_stride, topk_idx_out, scratch, st));
    }
    if (slot >= 0) {
        if (int rc = gather_phase(ctx, L, L.keys_Nq, topk_idx_out, slot, st, together ? topk_idx_out : nullptr)) return rc;
        L.keys_reader_slot = slot;
    } else {
        // selection only: an event of its own tells the layer's next scoring pass that the keys were read
        SPC_HIP(ctx, hipEventRecord(L.selected, st));
        L.selected_pending = true;
        L.selected_stream = st;
    }
    if (ss) {
        ss->used = true;
        ss->stream = st;
        ss->done = slot >= 0 ? L.gathered[slot] : L.selected;   // recorded behind the selection on this stream
    }
    return SPECACHE_OK;
}

int specache_gather(specache_ctx* ctx, int32_t layer, const int32_t* idx, int32_t slot, void* side_stream) {
    if (int rc = check_ctx_layer(ctx, layer)) return rc;
    if (!idx) return fail(ctx, SPECACHE_EINVAL, "null idx");
    if (slot != 0 && slot != 1) return fail(ctx, SPECACHE_EINVAL, "slot must be 0 or 1");
    Layer& L = ctx->layers[layer];
    hipStream_t st = (hipStream_t)side_stream;
    if (L.idx_ready_recorded)
        if (int rc = wait_for_scored(ctx, L, st)) return rc;
    if (int rc = order_gather_after_attend(ctx, L, slot, st)) return rc;
    if (int rc = gather_phase(ctx, L, L.Nq, idx, slot, st)) return rc;
    return SPECACHE_OK;
}

// the attention kernels that read `slot` are enqueued on st: remember it for the slot's next gather
static int record_attended(specache_ctx* ctx, Layer& L, int slot, hipStream_t st) {
    if (slot >= 0) {
        L.attend_stream[slot] = st;
        L.attend_seq[slot] = ++ctx->seq;
        L.attended_recorded[slot] = false;
        if (!(L.idx_ready_recorded && st == L.select_origin_stream)) {
            SPC_HIP(ctx, hipEventRecord(L.attended[slot], st));
            L.attended_recorded[slot] = true;
        }
    }
    return SPECACHE_OK;
}

// The logits of the last scoring pass from the copy of its queries that it left.
static int score_again(specache_ctx* ctx, Layer& L, hipStream_t st) {
    // (into ctx->keys: a selection on another stream may be reading the layer's own)
    SPC_HIP(ctx, launch_score(L.view, ctx->lse, ctx->scored_rows, ctx->scored_Nq, ctx->sm_scale, ctx->logits, ctx->logit_stride, ctx->keys,
                              ctx->logit_stride, st));
    ctx->logits_kept = true;
    return SPECACHE_OK;
}

// specache_attend with the partial results in `scratch`: the context's own, or the static array
static int attend_impl(specache_ctx* ctx, int32_t layer, const void* q, int32_t n_rows, const void* k_spec,
                       const void* v_spec, int32_t slot, float* out, void* stream, const AttendScratch* static_scratch) {
    if (int rc = check_ctx_layer(ctx, layer)) return rc;
    if (!q || !out) return fail(ctx, SPECACHE_EINVAL, "null q or out");
    if (n_rows != 1 && n_rows != 2) return fail(ctx, SPECACHE_EINVAL, "n_rows must be 1 or 2");
    if ((k_spec == nullptr) != (v_spec == nullptr)) return fail(ctx, SPECACHE_EINVAL, "k_spec and v_spec must both be given or both be null");
    if (slot < -1 || slot > 1) return fail(ctx, SPECACHE_EINVAL, "slot must be -1, 0 or 1");
    Layer& L = ctx->layers[layer];
    if (ctx->scored_layer != layer || ctx->scored_rows != n_rows || ctx->scored_N != L.N || ctx->scored_Nq != L.Nq)
        return fail(ctx, SPECACHE_ESTATE, "attend must follow score_topk of the same layer, n_rows and cache state");
    // several query heads per KV head: the one-launch scoring and attention keeps its queries, and an attend behind it scores again
    const bool rescore = !ctx->logits_kept && ctx->q_kept;
    if (!ctx->logits_kept && !rescore)
        return fail(ctx, SPECACHE_ESTATE, "the last scoring pass of this layer was specache_score_attend, which keeps no logits");
    if (slot >= 0 && !L.slot_filled[slot]) return fail(ctx, SPECACHE_ESTATE, "slot was never gathered");
    if (L.N == 0 && !k_spec) return fail(ctx, SPECACHE_ESTATE, "no attention candidate");
    AttendScratch scratch = ctx->scratch;
    if (static_scratch) {
        // partial outputs [rows][chunks][NR][128] floats, then the (max, sum) pairs [rows][chunks][NR][2]
        const int NR = L.view.G * n_rows;
        const int n_16bit = (slot >= 0 ? ctx->cfg.topk : 0) + (L.N - L.Nq) + (k_spec ? 1 : 0);
        int chunks = attend_chunks(NR, L.Nq, n_16bit);
        const size_t chunk_floats = (size_t)L.view.rows * NR * (kD + 2);
        if (chunks * chunk_floats * sizeof(float) > kStaticScratchBytes)
            return fail(ctx, SPECACHE_ECAPACITY, "specache_attend_static: the partial results of this call (rows x chunks x query rows "
                                                 "x 130 floats) exceed the 16 MiB static scratch array; use specache_attend");
        if (rows_uses_matrix_cores(L.view, n_rows)) {
            // that kernel splits a row as finely as the array and the merge kernel have room for
            const int room = (int)(kStaticScratchBytes / (chunk_floats * sizeof(float)));
            chunks = rows_chunks(L.view, n_rows, L.Nq, n_16bit, room < attend_max_chunks() ? room : attend_max_chunks());
        }
        const size_t o_floats = (size_t)L.view.rows * chunks * NR * kD;
        scratch.part_o = static_scratch->part_o;
        scratch.part_ml = static_scratch->part_o + o_floats;
        scratch.max_chunks = chunks;
    }
    hipStream_t st = (hipStream_t)stream;
    if (slot >= 0 && L.gather_stream[slot] != st && !(L.gathered_waited_set[slot] && L.gathered_waited[slot] == st))
        SPC_HIP(ctx, hipStreamWaitEvent(st, L.gathered[slot], 0));
    if (rescore)
        if (int rc = score_again(ctx, L, st)) return rc;
    // The layer's counters go with the context's scratch, which calls of one context share in any case.  A call with scratch memory of
    // its own may overlap one of those on another stream, and both would count their workgroups together: it merges in a launch of its own.
    uint32_t* const arrived = static_scratch ? nullptr : L.arrived;
    for (int phase : {kAttendPartial, kAttendCombine}) {
        TimedLaunch t(ctx, st, phase == kAttendPartial ? SPECACHE_K_ATTEND : SPECACHE_K_ATTEND_COMBINE, /*kernel_events=*/true);
        SPC_HIP(ctx, launch_attend(L.view, q, n_rows, L.N, L.Nq, ctx->sm_scale, ctx->logits, ctx->logit_stride,
                                   slot >= 0 ? L.slot[slot] : nullptr, slot >= 0 ? L.slot_idx[slot] : nullptr, k_spec,
                                   v_spec, scratch, out, phase, arrived, st));
    }
    return record_attended(ctx, L, slot, st);
}

int specache_attend(specache_ctx* ctx, int32_t layer, const void* q, int32_t n_rows, const void* k_spec,
                    const void* v_spec, int32_t slot, float* out, void* stream) {
    return attend_impl(ctx, layer, q, n_rows, k_spec, v_spec, slot, out, stream, nullptr);
}

// specache_score_attend, optionally with the append of one new token in front (carried by the same launch when
// that launch exists and no group leaves the residual with the token)
static int score_attend_impl(specache_ctx* ctx, int32_t layer, const void* k_new, const void* v_new, const void* q,
                             int32_t n_rows, const void* k_spec, const void* v_spec, int32_t slot, float* out, void* stream) {
    if (int rc = check_ctx_layer(ctx, layer)) return rc;
    if (!ctx->select_on_gather)
        return fail(ctx, SPECACHE_ESTATE, "specache_score_attend needs async_select = SPECACHE_SELECT_STREAM_GATHER");
    if ((k_new == nullptr) != (v_new == nullptr)) return fail(ctx, SPECACHE_EINVAL, "k_new and v_new must both be given or both be null");
    Layer& L = ctx->layers[layer];
    int32_t n_flush = 0;
    if (k_new) {
        if ((long)L.N + 1 > ctx->cfg.max_seq) return fail(ctx, SPECACHE_ECAPACITY, "append exceeds max_seq");
        if (specache_plan_append(ctx->cfg.residual, ctx->cfg.group, L.N, L.Nq, 1, &n_flush) != SPECACHE_OK)
            return fail(ctx, SPECACHE_ESTATE, "inconsistent token counts");
    }
    const bool rows_pass = (n_rows == 1 || n_rows == 2) && rows_in_one_launch(L.view, n_rows) &&
                           ctx->cfg.select_form == SPECACHE_SELECT_MAX_LOGIT;
    const bool one_pass = (rows_pass || (L.view.G == 1 && n_rows == 2 && attend_uses_int8_matrix_cores(L.view, n_rows) &&
                                         !(kernel_choice() & (kChoiceScoreValu | kChoiceAttendValu)))) &&
                          L.Nq > 0 && ctx->cfg.select_cache == SPECACHE_SELECT_LOWBIT && q && out && !((uintptr_t)q & 15);
    const bool carry = k_new && one_pass && n_flush == 0;
    if (k_new && !carry)
        if (int rc = specache_quantize_append(ctx, layer, k_new, v_new, 1, stream)) return rc;
    if (!one_pass) {
        // other shapes and options: the two passes one after the other, same results
        if (int rc = score_impl(ctx, layer, q, n_rows, stream, nullptr, nullptr)) return rc;
        return attend_impl(ctx, layer, q, n_rows, k_spec, v_spec, slot, out, stream, nullptr);
    }
    if ((k_spec == nullptr) != (v_spec == nullptr)) return fail(ctx, SPECACHE_EINVAL, "k_spec and v_spec must both be given or both be null");
    if (slot < -1 || slot > 1) return fail(ctx, SPECACHE_EINVAL, "slot must be -1, 0 or 1");
    if (slot >= 0 && !L.slot_filled[slot]) return fail(ctx, SPECACHE_ESTATE, "slot was never gathered");
    hipStream_t st = (hipStream_t)stream;
    if (int rc = wait_for_keys_readers(ctx, L, st)) return rc;
    if (slot >= 0 && L.gather_stream[slot] != st && !(L.gathered_waited_set[slot] && L.gathered_waited[slot] == st))
        SPC_HIP(ctx, hipStreamWaitEvent(st, L.gathered[slot], 0));
    const bool keep = (kernel_choice() & kChoiceKeepLogits) != 0;
    LayerView view = L.view;
    if (carry) {
        view.tail_k = (const uint16_t*)k_new;
        view.tail_v = (const uint16_t*)v_new;
        view.tail_N0 = L.N;
    }
    const int N1 = L.N + (carry ? 1 : 0);
    // Under capture the word is no order: a replayed merge stores the value of its capture again, and the selection's
    // stream, if it is not part of the capture, would wait at once for a value that only a replay stores.  An event it is.
    const bool by_word = !being_captured(st) && words_may_order(ctx);
    bool scored_carried = false, merged = false;
    Finish finish;
    finish.arrived = L.arrived;
    finish.out = out;
    finish.word = by_word ? L.scored_word : nullptr;
    finish.value = L.scored_value + 1;
    finish.rows = L.view.rows;
    {
        TimedLaunch t(ctx, st, SPECACHE_K_SCORE_ATTEND, /*kernel_events=*/true);
        CarriedEvent scored(ctx, st, by_word ? nullptr : L.idx_ready);
        if (rows_pass) {
            RowsArgs R{};
            R.at.q = (const uint16_t*)q;
            R.at.logits_out = keep ? ctx->logits : nullptr;
            R.at.q_out = keep ? nullptr : (uint16_t*)ctx->lse;
            R.at.logit_stride = ctx->logit_stride;
            R.at.slot = slot >= 0 ? L.slot[slot] : nullptr;
            R.at.slot_idx = slot >= 0 ? L.slot_idx[slot] : nullptr;
            R.at.k_spec = (const uint16_t*)k_spec;
            R.at.v_spec = (const uint16_t*)v_spec;
            R.at.part_o = ctx->scratch.part_o;
            R.at.part_ml = ctx->scratch.part_ml;
            R.at.max_chunks = ctx->scratch.max_chunks;
            R.at.N = N1;
            R.at.Nq = L.Nq;
            R.at.sm_scale = ctx->sm_scale;
            R.keys = L.keys;
            R.key_stride = ctx->logit_stride;
            R.n_rows = n_rows;
            R.at.fin = finish;
            SPC_HIP(ctx, launch_rows(view, R, kRowsBoth, &merged, st));
        } else {
            SPC_HIP(ctx, launch_attend_i8_partial(view, q, N1, L.Nq, ctx->sm_scale, nullptr, ctx->logit_stride,
                                                  slot >= 0 ? L.slot[slot] : nullptr, slot >= 0 ? L.slot_idx[slot] : nullptr, k_spec,
                                                  v_spec, ctx->scratch, L.keys, ctx->logit_stride, keep ? ctx->logits : nullptr, finish, &merged, st));
        }
        scored_carried = scored.landed();
    }
    L.N = N1;   // only once the launch that copies the token is enqueued
    ctx->logits_kept = keep;
    ctx->q_kept = rows_pass && !keep;
    // the keys are complete here, in front of a merge kernel: the event says so, or else that kernel as it starts (a launch that
    // merged says so itself), and the selection on the side stream runs beside it
    if (!by_word)
        if (int rc = record_scored(ctx, L, layer, n_rows, st, scored_carried)) return rc;
    if (!merged) {
        TimedLaunch t(ctx, st, SPECACHE_K_ATTEND_COMBINE, /*kernel_events=*/true);
        SPC_HIP(ctx, launch_attend(L.view, q, n_rows, L.N, L.Nq, ctx->sm_scale, ctx->logits, ctx->logit_stride,
                                   slot >= 0 ? L.slot[slot] : nullptr, slot >= 0 ? L.slot_idx[slot] : nullptr, k_spec, v_spec,
                                   ctx->scratch, out, kAttendCombine, nullptr, st, by_word ? Announce{L.scored_word, L.scored_value + 1} : Announce{}));
    }
    if (by_word) {
        ++L.scored_value;
        if (int rc = record_scored(ctx, L, layer, n_rows, st, false, true)) return rc;
    }
    return record_attended(ctx, L, slot, st);
}

int specache_score_attend(specache_ctx* ctx, int32_t layer, const void* q, int32_t n_rows, const void* k_spec,
                          const void* v_spec, int32_t slot, float* out, void* stream) {
    return score_attend_impl(ctx, layer, nullptr, nullptr, q, n_rows, k_spec, v_spec, slot, out, stream);
}

int specache_append_score_attend(specache_ctx* ctx, int32_t layer, const void* k_new, const void* v_new, const void* q,
                                 int32_t n_rows, const void* k_spec, const void* v_spec, int32_t slot, float* out,
                                 void* stream) {
    if (ctx && (!k_new || !v_new)) return fail(ctx, SPECACHE_EINVAL, "null k_new or v_new");
    return score_attend_impl(ctx, layer, k_new, v_new, q, n_rows, k_spec, v_spec, slot, out, stream);
}

int specache_decode_step(specache_ctx* ctx, int32_t layer, const void* k_new, const void* v_new, const void* q,
                         const void* k_spec, const void* v_spec, int32_t read_slot, float* out, void* stream,
                         int32_t* topk_idx_out, int32_t fill_slot, void* side_stream) {
    if (int rc = specache_append_score_attend(ctx, layer, k_new, v_new, q, 2, k_spec, v_spec, read_slot, out, stream)) return rc;
    return specache_select_gather(ctx, layer, topk_idx_out, fill_slot, side_stream);
}

int specache_attend_static(specache_ctx* ctx, int32_t layer, const void* q, int32_t n_rows, const void* k_spec,
                           const void* v_spec, int32_t slot, float* out, void* stream) {
    if (!ctx) return SPECACHE_EINVAL;
    float* base = nullptr;
    if (int rc = static_scratch_of_current_device(ctx, &base)) return rc;
    const AttendScratch st{base, nullptr, 0};
    return attend_impl(ctx, layer, q, n_rows, k_spec, v_spec, slot, out, stream, &st);
}

int specache_order_by_events(specache_ctx* ctx, int32_t enable) {
    if (!ctx) return SPECACHE_EINVAL;
    ctx->events_wanted = enable != 0;
    return SPECACHE_OK;
}

int specache_debug_scored_by_word(specache_ctx* ctx, int32_t layer, int32_t* by_word) {
    if (int rc = check_ctx_layer(ctx, layer)) return rc;
    if (!by_word) return fail(ctx, SPECACHE_EINVAL, "null by_word");
    *by_word = ctx->layers[layer].scored_by_word;
    return SPECACHE_OK;
}

int specache_debug_fail_alloc(int32_t nth) {
    if (nth < 0) return SPECACHE_EINVAL;
    g_fail_alloc_at = nth;
    return SPECACHE_OK;
}

int specache_debug_merger_polls(int32_t polls) {
    if (polls < -1) return SPECACHE_EINVAL;
    merger_polls() = polls < 0 ? kMergerPolls : polls;
    return SPECACHE_OK;
}

int specache_debug_kernel_choice(int32_t flags) {
    if (flags < 0 || flags > (SPECACHE_SCORE_ON_VECTOR_ALU | SPECACHE_ATTEND_ON_VECTOR_ALU | SPECACHE_KEEP_ONE_PASS_LOGITS))
        return SPECACHE_EINVAL;
    kernel_choice() = (flags & SPECACHE_SCORE_ON_VECTOR_ALU ? kChoiceScoreValu : 0) |
                      (flags & SPECACHE_ATTEND_ON_VECTOR_ALU ? kChoiceAttendValu : 0) |
                      (flags & SPECACHE_KEEP_ONE_PASS_LOGITS ? kChoiceKeepLogits : 0);
    return SPECACHE_OK;
}

int specache_debug_poison_slot(specache_ctx* ctx, int32_t layer, int32_t slot, void* stream) {
    if (int rc = check_ctx_layer(ctx, layer)) return rc;
    if (slot != 0 && slot != 1) return fail(ctx, SPECACHE_EINVAL, "slot must be 0 or 1");
    Layer& L = ctx->layers[layer];
    // every 16-bit word becomes 0xFFFF, a NaN in binary16 and in bfloat16
    SPC_HIP(ctx, hipMemsetAsync(L.slot[slot], 0xFF, (size_t)L.view.rows * ctx->cfg.topk * kRowBytes, (hipStream_t)stream));
    return SPECACHE_OK;
}

int specache_export_quantized(specache_ctx* ctx, int32_t layer, uint8_t* k_codes, uint16_t* k_minmax,
                              float* k_scale_zero, uint8_t* v_codes, uint16_t* v_minmax, float* v_scale_zero) {
    if (int rc = check_ctx_layer(ctx, layer)) return rc;
    Layer& L = ctx->layers[layer];
    SPC_HIP(ctx, hipDeviceSynchronize());
    const size_t rows = L.view.rows, Nq = L.Nq, g = ctx->cfg.group;
    if (Nq == 0) return SPECACHE_OK;
    const size_t n_codes = rows * Nq * kD, n_kg = rows * (Nq / g) * kD, n_vg = rows * Nq * (kD / g);
    struct Buf { void* host; size_t bytes; void* dev; };
    Buf bufs[6] = {{k_codes, n_codes, nullptr},        {k_minmax, n_kg * 4, nullptr}, {k_scale_zero, n_kg * 8, nullptr},
                   {v_codes, n_codes, nullptr},        {v_minmax, n_vg * 4, nullptr}, {v_scale_zero, n_vg * 8, nullptr}};
    int rc = SPECACHE_OK;
    for (Buf& b : bufs)
        if (b.host && rc == SPECACHE_OK) {
            hipError_t e = hipMalloc(&b.dev, b.bytes);
            if (e != hipSuccess) rc = fail_hip(ctx, e, "hipMalloc(export)");
        }
    if (rc == SPECACHE_OK) {
        hipError_t e = launch_export(L.view, L.Nq, (uint8_t*)bufs[0].dev, (uint16_t*)bufs[1].dev, (float*)bufs[2].dev,
                                     (uint8_t*)bufs[3].dev, (uint16_t*)bufs[4].dev, (float*)bufs[5].dev, nullptr);
        if (e == hipSuccess) e = hipDeviceSynchronize();
        for (Buf& b : bufs)
            if (b.dev && e == hipSuccess) e = hipMemcpy(b.host, b.dev, b.bytes, hipMemcpyDeviceToHost);
        if (e != hipSuccess) rc = fail_hip(ctx, e, "export");
    }
    for (Buf& b : bufs) (void)hipFree(b.dev);
    return rc;
}

int specache_export_rows(specache_ctx* ctx, int32_t layer, int32_t first, int32_t count, uint16_t* out) {
    if (int rc = check_ctx_layer(ctx, layer)) return rc;
    Layer& L = ctx->layers[layer];
    if (!out || first < 0 || count < 0 || first + count > L.N) return fail(ctx, SPECACHE_EINVAL, "bad row range or null output");
    SPC_HIP(ctx, hipDeviceSynchronize());
    const uint8_t* src = (const uint8_t*)L.host_alloc;
    for (int r = 0; r < L.view.rows; ++r)
        std::memcpy((uint8_t*)out + (size_t)r * count * kRowBytes,
                    src + ((size_t)r * ctx->cfg.max_seq + first) * kRowBytes, (size_t)count * kRowBytes);
    return SPECACHE_OK;
}

int specache_timing(specache_ctx* ctx, int32_t enable, double* total_us, int64_t* launches) {
    if (!ctx) return SPECACHE_EINVAL;
    SPC_HIP(ctx, hipDeviceSynchronize());
    if (total_us) for (int k = 0; k < SPECACHE_K_COUNT; ++k) total_us[k] = 0.0;
    if (launches) for (int k = 0; k < SPECACHE_K_COUNT; ++k) launches[k] = 0;
    for (auto& sp : ctx->spans) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, sp.a, sp.b) == hipSuccess) {
            if (total_us) total_us[sp.kind] += 1e3 * (double)ms;
            if (launches) launches[sp.kind] += 1;
        }
        ctx->ev_pool.push_back(sp.a);
        ctx->ev_pool.push_back(sp.b);
    }
    ctx->spans.clear();
    ctx->timing = enable != 0;
    return SPECACHE_OK;
}

int specache_debug_logits(specache_ctx* ctx, float* out) {
    if (!ctx || !out) return SPECACHE_EINVAL;
    if (ctx->scored_layer < 0) return fail(ctx, SPECACHE_ESTATE, "nothing scored yet");
    if (!ctx->logits_kept && !ctx->q_kept)
        return fail(ctx, SPECACHE_ESTATE, "specache_score_attend kept no logits (see specache_debug_kernel_choice)");
    SPC_HIP(ctx, hipDeviceSynchronize());
    if (!ctx->logits_kept) {
        if (int rc = score_again(ctx, ctx->layers[ctx->scored_layer], nullptr)) return rc;
        SPC_HIP(ctx, hipDeviceSynchronize());
    }
    const size_t n = (size_t)ctx->layers[ctx->scored_layer].view.rows * ctx->layers[ctx->scored_layer].view.G * ctx->scored_rows;
    const size_t Nq = ctx->scored_Nq;
    if (Nq == 0) return SPECACHE_OK;
    SPC_HIP(ctx, hipMemcpy2D(out, Nq * 4, ctx->logits, ctx->logit_stride * 4, Nq * 4, n, hipMemcpyDeviceToHost));
    return SPECACHE_OK;
}

}  // extern "C"
