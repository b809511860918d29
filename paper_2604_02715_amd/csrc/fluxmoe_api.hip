// Host side of libfluxmoe.so: context, offline encode driver, tier binding, the
// materialize / expert-FFN enqueue paths and the event protocol between them.
//
// Event protocol = PagedTensor synchronization (paper Alg. 1), generalised from the two
// reusable layer blocks to individual staging slots: a materialize waits for the inference
// event of every layer whose FFN last read one of its target slots (write-after-read); an
// FFN call waits for its layer's load event (read-after-write) and records the layer's
// inference event.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <atomic>
#include <cstdlib>
#include <cmath>
#include <cstring>
#include <new>

#include "crew.h"
#include "decode_plan.h"
#include "encode_core.h"
#include "fluxmoe_internal.h"

namespace fluxmoe {

static thread_local char g_err[512] = "";

int set_error(int status, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return status;
}

}  // namespace fluxmoe

using namespace fluxmoe;

#define HIPCHECK(call)                                                                  \
    do {                                                                                \
        hipError_t e_ = (call);                                                         \
        if (e_ != hipSuccess)                                                           \
            return set_error(FLUXMOE_EHIP, "%s failed: %s", #call, hipGetErrorString(e_)); \
    } while (0)

namespace {
constexpr int kRing = 4;
// Events between kernels of this device: no fence towards the host and other devices, which holds the stream for another
// 1.5 us (one token's FFN call 29.5 -> 27.8 us).  Loads keep it (a layer's load can end with copies), as do host-tier copies
// and the fork to a second stream (a command upload, staged blocks or the caller's own copies can lie in front of it).
constexpr unsigned kOrderOnly = hipEventDisableTiming | hipEventDisableSystemFence;
constexpr uint32_t kLutBytes = kLutEntries * 4;

// What one half of the host-tier staging buffer currently holds.
struct StageHalf {
    int64_t layer = -1;            // layer whose host-tier blocks are staged, -1 = nothing
    std::vector<int64_t> off[2];   // per expert: byte offset of the tensor's host part, -1 = absent
};

}  // namespace

// FFN scratch of fluxmoe_expert_ffn_static: one array per GPU, part of the loaded code object, held until
// the process ends.  In host code the array's name is only a handle for hipGetSymbolAddress; the device
// address of each GPU's copy is resolved once per device (resolve_static_scratch, called by
// fluxmoe_bind_arenas with that device current) and kept in g_static_scratch.
constexpr uint64_t kStaticScratchBytes = FLUXMOE_STATIC_SCRATCH_BYTES;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) uint8_t scratch[kStaticScratchBytes];
static uint8_t* g_static_scratch[kMaxDevices] = {};

struct fluxmoe_ctx {
    fluxmoe_desc d;
    int device = -1;                      // HIP device the arenas were bound on
    uint64_t elems13 = 0, elems2 = 0;
    std::vector<LayerMeta> layers;
    // arenas
    uint8_t* slots13 = nullptr;
    uint8_t* slots2 = nullptr;
    uint8_t* ws = nullptr;
    size_t ws_bytes = 0;
    bool arenas_bound = false;
    int n_cus = 256;
    // pool workspace layout
    uint64_t lut_off = 0, cmd_off = 0, err_off = 0, pool_ws_bytes = 0;
    uint32_t max_jobs = 0, max_upd = 0, cmd_bytes = 0;
    // command ring (pinned host mirror of the device command buffers)
    uint8_t* pinned_cmd = nullptr;
    hipEvent_t ring_ev[kRing] = {};
    bool ring_used[kRing] = {};
    int ring_next = 0;
    // page-table mirror and slot ownership
    std::vector<int32_t> pt;
    std::vector<int64_t> slot_owner;      // layer * E + expert, or -1
    // Alg. 1 state
    std::vector<hipEvent_t> ev_load, ev_rel;   // per layer: last materialize / release
    // Per layer: the last two FFN calls (call g records event g & 1), so that a materialize into slots the one before the
    // last read does not wait for the last; ev_routed: the last wave-mode call has read the page table.
    std::vector<std::array<hipEvent_t, 2>> ev_infer;
    std::vector<hipEvent_t> ev_routed;
    std::vector<uint64_t> infer_gen;           // FFN calls of the layer so far; 0 = none
    std::vector<uint64_t> routed_gen;          // the call behind ev_routed, 0 = none
    std::vector<uint8_t> load_valid, rel_valid;
    // Order in which the calls behind those events were made (0 = under stream capture or never).  A later call of a layer
    // has waited for the earlier event, so its own event covers both and one wait is enough: a wait for another stream
    // holds the queue for about 10 us even when the event completed long ago.
    std::vector<uint64_t> load_seq, rel_seq;
    std::vector<std::array<uint64_t, 2>> infer_seq;
    std::vector<std::array<uint64_t, 2>> infer_capture;    // the stream capture the call behind ev_infer was made in, 0 = none
    uint64_t seq = 0;
    std::vector<int32_t> slot_last_reader; // layer whose FFN last read the slot, or -1
    std::vector<uint64_t> slot_reader_gen; // which of that layer's FFN calls it was
    bool events_ready = false;
    // host-tier staging
    uint8_t* staging = nullptr;
    size_t staging_bytes = 0;
    StageHalf half[2];                      // layer l stages into half l & 1
    hipEvent_t ev_copied[2] = {};           // copies into the half have completed
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;   // fluxmoe_materialize_two_streams
    // The load event of the materialize that read the half last (nullptr: none) and the stream capture it was made in.  A
    // later load of that layer covers it, except across a capture's border: that one records the spare event instead.
    hipEvent_t half_read[2] = {}, half_spare[2] = {};
    uint64_t half_capture[2] = {0, 0};
    bool copied_valid[2] = {false, false};  // ev_copied[h] has been recorded
    // launch shape of the decode kernel (FLUXMOE_DECODE_WAVES / FLUXMOE_DECODE_BLOCKS_PER_WAVE override)
    int tune_waves = 8;
    int tune_blocks_per_wave = 0;         // 0 = by the number of blocks, where the launch is made
    int tune_tiled_waves = 2;             // FLUXMOE_FFN_TILED_WAVES: 2 = LDS-direct loads (default), 8 = register-staged,
                                          // 4 = register-staged with four wavefronts of 128 x 128
    int tune_tiled_persist = 1;           // FLUXMOE_FFN_TILED_PERSIST: 0 = one workgroup per tile, n = n x 256 workgroups walking the tiles
    int tune_tiled_group = 0;             // FLUXMOE_FFN_TILED_GROUP: 1..8 super-rows per group of the tiled gate/up kernel, 0 = from the shape
    // optional kernel timing (fluxmoe_profile_*)
    bool profiling = false;
    uint32_t profile_mask = 0x1F;         // kinds that are bracketed while profiling
    bool span_open = false;               // the span begun last is being recorded
    struct Span { hipEvent_t a, b; int kind; };
    std::vector<Span> spans;
};

namespace {

void compute_layout(fluxmoe_ctx* c) {
    const uint64_t E = c->d.n_experts;
    c->max_jobs = uint32_t(2 * E + 2);
    c->max_upd = uint32_t(2 * E + 2);
    c->cmd_bytes = uint32_t(align_up(sizeof(DecodeCmd) + 2ull * c->max_jobs * sizeof(DecodeJob) +
                                     c->max_upd * 8ull, 256));
    c->lut_off = 0;
    c->cmd_off = align_up(uint64_t(c->d.n_layers) * 2 * kLutBytes, 256);
    c->err_off = c->cmd_off + uint64_t(kRing) * c->cmd_bytes;
    c->pool_ws_bytes = align_up(c->err_off + 256, 4096);
}

FfnShape ffn_shape(const fluxmoe_ctx* c, uint32_t n_experts) {
    return FfnShape{n_experts, c->d.hidden, c->d.ffn, c->n_cus, c->tune_tiled_waves, true};
}

// Pair table of the decode kernel, indexed by the next 12 stream bits (first stream bit in bit 0).
// Entry: bits 0..5 bits to advance, 7..14 first exponent, 15..18 length of the first code, 23..30
// second exponent, bit 31 set when the second code does not end inside the 12 bits (the entry then
// covers the first symbol only).  Bit patterns no code matches (only possible with a single used
// symbol) decode as the first used symbol with length 1: valid streams never reach them.
void build_lut(const uint8_t lens[256], uint32_t* lut) {
    uint16_t codes[256];
    canonical_codes(lens, codes);
    int fallback = -1;
    for (int s = 0; s < 256; ++s)
        if (lens[s]) { fallback = s; break; }
    // single-symbol table: 12 stream bits -> (symbol, length)
    std::vector<uint16_t> one(kLutEntries, uint16_t(fallback < 0 ? 1 : ((fallback << 4) | 1)));
    for (int s = 0; s < 256; ++s) {
        const uint32_t L = lens[s];
        if (!L || L > kLutBits) continue;
        uint32_t rev = 0;   // first code bit in bit 0: that is how the stream is peeked
        for (uint32_t b = 0; b < L; ++b) rev |= ((codes[s] >> (L - 1 - b)) & 1u) << b;
        for (uint32_t hi = 0; hi < (1u << (kLutBits - L)); ++hi)
            one[rev | (hi << L)] = uint16_t((s << 4) | L);
    }
    for (uint32_t i = 0; i < kLutEntries; ++i) {
        const uint32_t s0 = one[i] >> 4, l0 = one[i] & 15u;
        uint32_t entry = 0x80000000u | (l0 << 15) | (s0 << 7) | l0;
        if (l0 < kLutBits) {
            // the second code must end inside the remaining 12 - l0 bits; the bits above them are zero
            // in this index, so a match longer than what remains is not a match
            const uint32_t rest = i >> l0;
            const uint32_t s1 = one[rest] >> 4, l1 = one[rest] & 15u;
            bool real = false;                      // is `rest` really the code of s1, not the fallback?
            if (lens[s1] == l1) {
                uint32_t rev = 0;
                for (uint32_t b = 0; b < l1; ++b) rev |= ((codes[s1] >> (l1 - 1 - b)) & 1u) << b;
                real = (rest & ((1u << l1) - 1u)) == rev;
            }
            if (real && l0 + l1 <= kLutBits) entry = (s1 << 23) | (l0 << 15) | (s0 << 7) | (l0 + l1);
        }
        lut[i] = entry;
    }
}

int check_layer(const fluxmoe_ctx* c, uint32_t layer, bool need_encoded) {
    if (!c) return set_error(FLUXMOE_EINVAL, "ctx is NULL");
    if (layer >= c->d.n_layers)
        return set_error(FLUXMOE_ERANGE, "layer %u out of range (n_layers %u)", layer, c->d.n_layers);
    if (need_encoded && !c->layers[layer].encoded)
        return set_error(FLUXMOE_ESTATE, "layer %u has not been encoded", layer);
    return FLUXMOE_OK;
}

int ensure_events(fluxmoe_ctx* c) {
    if (c->events_ready) return FLUXMOE_OK;
    const uint32_t N = c->d.n_layers;
    c->ev_load.assign(N, nullptr);
    c->ev_infer.assign(N, {nullptr, nullptr});
    c->ev_routed.assign(N, nullptr);
    c->ev_rel.assign(N, nullptr);
    for (uint32_t i = 0; i < N; ++i) {
        HIPCHECK(hipEventCreateWithFlags(&c->ev_load[i], hipEventDisableTiming));
        for (hipEvent_t& e : c->ev_infer[i]) HIPCHECK(hipEventCreateWithFlags(&e, kOrderOnly));
        HIPCHECK(hipEventCreateWithFlags(&c->ev_routed[i], kOrderOnly));
        HIPCHECK(hipEventCreateWithFlags(&c->ev_rel[i], kOrderOnly));
    }
    for (int i = 0; i < kRing; ++i)
        HIPCHECK(hipEventCreateWithFlags(&c->ring_ev[i], hipEventDisableTiming));
    HIPCHECK(hipEventCreateWithFlags(&c->ev_fork, hipEventDisableTiming));
    HIPCHECK(hipEventCreateWithFlags(&c->ev_join, kOrderOnly));
    for (int i = 0; i < 2; ++i) {
        HIPCHECK(hipEventCreateWithFlags(&c->ev_copied[i], hipEventDisableTiming));
        HIPCHECK(hipEventCreateWithFlags(&c->half_spare[i], hipEventDisableTiming));
    }
    HIPCHECK(hipHostMalloc(reinterpret_cast<void**>(&c->pinned_cmd), size_t(kRing) * c->cmd_bytes,
                           hipHostMallocDefault));
    c->events_ready = true;
    return FLUXMOE_OK;
}

int resolve_static_scratch(int dev) {
    if (dev < 0 || dev >= kMaxDevices) return set_error(FLUXMOE_EHIP, "device index %d out of range", dev);
    if (g_static_scratch[dev]) return FLUXMOE_OK;
    void* ptr = nullptr;
    HIPCHECK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return set_error(FLUXMOE_EHIP, "hipGetSymbolAddress returned a NULL address");
    g_static_scratch[dev] = static_cast<uint8_t*>(ptr);
    return FLUXMOE_OK;
}

// The capture a stream is part of (0: none).  kNoCaptureId where that cannot be told.
constexpr uint64_t kNoCaptureId = ~0ull;
uint64_t capture_of(hipStream_t s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    unsigned long long id = 0;
    if (hipStreamGetCaptureInfo(s, &st, &id) != hipSuccess) {
        (void)hipGetLastError();
        return kNoCaptureId;
    }
    return st == hipStreamCaptureStatusNone ? 0 : (st == hipStreamCaptureStatusActive && id ? id : kNoCaptureId);
}

// The event for a launch that is to complete with it, or nullptr where it has to be recorded after the launch instead:
// under stream capture a recorded event becomes part of the graph's dependencies, an attached one does not.
hipEvent_t attachable(hipEvent_t ev, hipStream_t s) { return capture_of(s) == 0 ? ev : nullptr; }

hipError_t span_begin(fluxmoe_ctx* c, int kind, hipStream_t s) {
    c->span_open = c->profiling && ((c->profile_mask >> kind) & 1u);
    if (!c->span_open) return hipSuccess;
    fluxmoe_ctx::Span sp{nullptr, nullptr, kind};
    hipError_t e = hipEventCreate(&sp.a);
    if (e != hipSuccess) return e;
    e = hipEventCreate(&sp.b);
    if (e != hipSuccess) return e;
    c->spans.push_back(sp);
    return hipEventRecord(sp.a, s);
}

hipError_t span_end(fluxmoe_ctx* c, hipStream_t s) {
    if (!c->span_open) return hipSuccess;
    c->span_open = false;
    return hipEventRecord(c->spans.back().b, s);
}

void ffn_span_hook(void* user, int kind, int begin, hipStream_t s) {
    fluxmoe_ctx* c = static_cast<fluxmoe_ctx*>(user);
    if (begin) (void)span_begin(c, kind, s); else (void)span_end(c, s);
}

}  // namespace

extern "C" {

const char* fluxmoe_last_error(void) { return g_err; }

int fluxmoe_create(const fluxmoe_desc* desc, fluxmoe_ctx** out_ctx) {
    if (!desc || !out_ctx) return set_error(FLUXMOE_EINVAL, "desc/out_ctx is NULL");
    fluxmoe_desc d = *desc;
    if (d.max_code_len == 0) d.max_code_len = 12;
    if (d.n_layers == 0 || d.n_experts == 0 || d.hidden == 0 || d.ffn == 0 || d.n_slots == 0)
        return set_error(FLUXMOE_EINVAL, "n_layers, n_experts, hidden, ffn, n_slots must be > 0");
    if (d.hidden % 8 || d.ffn % 8)
        return set_error(FLUXMOE_EINVAL, "hidden (%u) and ffn (%u) must be multiples of 8", d.hidden, d.ffn);
    if (d.block_bytes != 4096)
        return set_error(FLUXMOE_EINVAL, "block_bytes must be 4096 (got %u)", d.block_bytes);
    if (d.max_code_len < 8 || d.max_code_len > kLutBits)
        return set_error(FLUXMOE_EINVAL, "max_code_len must be in 8..12 (got %u)", d.max_code_len);
    if (d.flags != 0) return set_error(FLUXMOE_EINVAL, "flags must be 0");
    if (uint64_t(d.hidden) * d.ffn * 2 >= (1ull << 31))
        return set_error(FLUXMOE_EINVAL, "hidden * ffn * 2 bytes (one expert matrix) must stay under 2 GiB: "
                                         "the FFN kernels address a matrix with 32-bit byte offsets");
    if (d.n_experts > 4096) return set_error(FLUXMOE_EINVAL, "n_experts must be <= 4096");
    fluxmoe_ctx* c = new (std::nothrow) fluxmoe_ctx();
    if (!c) return set_error(FLUXMOE_ENOMEM, "out of host memory");
    c->d = d;
    c->elems2 = uint64_t(d.hidden) * d.ffn;
    c->elems13 = 2 * c->elems2;
    c->layers.resize(d.n_layers);
    c->pt.assign(size_t(d.n_layers) * d.n_experts, -1);
    c->slot_owner.assign(d.n_slots, -1);
    c->slot_last_reader.assign(d.n_slots, -1);
    c->slot_reader_gen.assign(d.n_slots, 0);
    c->load_valid.assign(d.n_layers, 0);
    c->infer_gen.assign(d.n_layers, 0);
    c->routed_gen.assign(d.n_layers, 0);
    c->rel_valid.assign(d.n_layers, 0);
    c->load_seq.assign(d.n_layers, 0);
    c->infer_seq.assign(d.n_layers, {0, 0});
    c->infer_capture.assign(d.n_layers, {0, 0});
    c->rel_seq.assign(d.n_layers, 0);
    compute_layout(c);
    if (const char* v = std::getenv("FLUXMOE_DECODE_WAVES")) {
        const int w = std::atoi(v);
        if (w == 4 || w == 8 || w == 16) c->tune_waves = w;
    }
    if (const char* v = std::getenv("FLUXMOE_DECODE_BLOCKS_PER_WAVE")) {
        const int w = std::atoi(v);
        if (w >= 1 && w <= 1024) c->tune_blocks_per_wave = w;
    }
    if (const char* v = std::getenv("FLUXMOE_FFN_TILED_WAVES")) {
        const int w = std::atoi(v);
        if (w == 1 || w == 2 || w == 4 || w == 8) c->tune_tiled_waves = w;
    }
    if (const char* v = std::getenv("FLUXMOE_FFN_TILED_PERSIST")) {
        const int w = std::atoi(v);
        if (w >= 0 && w <= 16) c->tune_tiled_persist = w;
    }
    if (const char* v = std::getenv("FLUXMOE_FFN_TILED_GROUP")) {
        const int w = std::atoi(v);
        if (w >= 1 && w <= 8) c->tune_tiled_group = w;
    }
    *out_ctx = c;
    g_err[0] = 0;
    return FLUXMOE_OK;
}

int fluxmoe_destroy(fluxmoe_ctx* c) {
    if (!c) return FLUXMOE_OK;
    if (c->events_ready) {
        for (auto e : c->ev_load) if (e) (void)hipEventDestroy(e);
        for (auto& pair : c->ev_infer) for (auto e : pair) if (e) (void)hipEventDestroy(e);
        for (auto e : c->ev_routed) if (e) (void)hipEventDestroy(e);
        for (auto e : c->ev_rel) if (e) (void)hipEventDestroy(e);
        for (int i = 0; i < kRing; ++i) if (c->ring_ev[i]) (void)hipEventDestroy(c->ring_ev[i]);
        for (int i = 0; i < 2; ++i) if (c->ev_copied[i]) (void)hipEventDestroy(c->ev_copied[i]);
        for (int i = 0; i < 2; ++i) if (c->half_spare[i]) (void)hipEventDestroy(c->half_spare[i]);
        if (c->ev_fork) (void)hipEventDestroy(c->ev_fork);
        if (c->ev_join) (void)hipEventDestroy(c->ev_join);
        if (c->pinned_cmd) (void)hipHostFree(c->pinned_cmd);
    }
    delete c;
    return FLUXMOE_OK;
}

int fluxmoe_query_sizes(const fluxmoe_ctx* c, fluxmoe_sizes* out) {
    if (!c || !out) return set_error(FLUXMOE_EINVAL, "ctx/out is NULL");
    out->sigma1 = c->elems13 * 2;
    out->sigma2 = c->elems2 * 2;
    out->slots13_bytes = out->sigma1 * c->d.n_slots;
    out->slots2_bytes = out->sigma2 * c->d.n_slots;
    out->page_table_bytes = uint64_t(c->d.n_layers) * c->d.n_experts * 4;
    // worst case: every element costs 1 raw byte + max_code_len bits, plus headers and one
    // partly filled block per tensor
    const uint64_t per_block = c->d.block_bytes - kHeaderBytes;
    auto bound = [&](uint64_t elems) {
        const uint64_t bytes = elems + (elems * c->d.max_code_len + 7) / 8;
        return (bytes / (per_block - 8 * kGroup) + 2) * c->d.block_bytes;
    };
    out->layer_blob_bound = uint64_t(c->d.n_experts) * (bound(c->elems13) + bound(c->elems2));
    out->pool_workspace_bytes = c->pool_ws_bytes;
    return FLUXMOE_OK;
}

uint64_t fluxmoe_ffn_workspace_bytes(const fluxmoe_ctx* c, uint32_t T, uint32_t K, int shared_expert) {
    if (!c) return 0;
    const uint64_t need = ffn_bytes(ffn_shape(c, c->d.n_experts), T, K);
    return shared_expert ? std::max(need, shared_bytes(ffn_shape(c, 1), T)) : need;          // same shapes, a single expert
}

int fluxmoe_ffn_plan(const fluxmoe_ctx* c, uint32_t T, uint32_t K, uint32_t* rows_per_tile, uint32_t* k_splits) {
    if (!c || !rows_per_tile || !k_splits) return set_error(FLUXMOE_EINVAL, "NULL argument");
    if (K == 0 || K > c->d.n_experts) return set_error(FLUXMOE_EINVAL, "K must be in 1..n_experts");
    FfnShape shape = ffn_shape(c, c->d.n_experts);
    shape.ragged = false;                        // as documented: the strips' plan, whose place tiles may take
    const FfnPlan p = plan_ffn(shape, T, K);
    *rows_per_tile = p.m_tile;
    *k_splits = p.ksplit;
    return FLUXMOE_OK;
}

int fluxmoe_encode_pool(fluxmoe_ctx* c, uint32_t layer, const uint16_t* w13, const uint16_t* w2,
                        void* dst, size_t dst_cap, size_t* dst_used, int n_threads) {
    if (int rc = check_layer(c, layer, false)) return rc;
    if (!w13 || !w2 || !dst || !dst_used) return set_error(FLUXMOE_EINVAL, "NULL argument");
    const uint32_t E = c->d.n_experts, B = c->d.block_bytes;
    n_threads = std::max(1, std::min(n_threads, 256));
    LayerMeta& L = c->layers[layer];
    L.encoded = false;
    L.bound = false;
    const uint64_t elems[2] = {c->elems13, c->elems2};
    const uint16_t* base[2] = {w13, w2};
    const bool vector = encode_vector_available();
    auto tensor = [&](uint32_t i) { return base[i / E] + size_t(i % E) * elems[i / E]; };      // i: type index * E + expert

    // One set of threads goes through the three passes over the weights; between them the last to arrive does what has to be
    // done once.  Units are pieces of tensors, so that the threads end together whatever the number of tensors is.
    constexpr uint64_t kCountElems = 1u << 17, kBlocksPerUnit = 16;
    try {
    Crew crew(n_threads);
    std::vector<std::array<uint64_t, 512>> hist(crew.size(), std::array<uint64_t, 512>{});
    Coder coder[2];
    std::vector<uint64_t> unit_end(2 * size_t(E));           // encode units up to and with each tensor's
    const uint64_t count_units[2] = {(elems[0] + kCountElems - 1) / kCountElems, (elems[1] + kCountElems - 1) / kCountElems};
    uint8_t* const out = static_cast<uint8_t*>(dst);
    bool fits = false;
    crew.run([&](uint32_t me) {
        // 1. exponent histograms, one per tensor type over all experts
        for (uint64_t u; (u = crew.take()) < E * (count_units[0] + count_units[1]);) {
            const int ti = u < E * count_units[0] ? 0 : 1;
            const uint64_t v = ti ? u - E * count_units[0] : u, at = v % count_units[ti] * kCountElems;
            count_exponents(base[ti] + size_t(v / count_units[ti]) * elems[ti] + at, std::min(kCountElems, elems[ti] - at), hist[me].data() + 256 * ti);
        }
        crew.wait([&]() {
            for (int ti = 0; ti < 2; ++ti) {
                uint64_t total[256] = {};
                for (const auto& h : hist)
                    for (int s = 0; s < 256; ++s) total[s] += h[256 * ti + s];
                uint16_t codes[256];
                limited_code_lengths(total, c->d.max_code_len, L.lens[ti]);
                canonical_codes(L.lens[ti], codes);
                coder[ti] = Coder(L.lens[ti], codes);
                L.payload_bits[ti] = 0;
                for (int s = 0; s < 256; ++s) L.payload_bits[ti] += total[s] * L.lens[ti][s];
                L.tensors[ti].assign(E, TensorMeta());
            }
        });
        // 2. block plan of every tensor
        for (uint64_t i; (i = crew.take()) < 2 * uint64_t(E);)
            plan_tensor(tensor(uint32_t(i)), elems[i / E], coder[i / E], B, L.tensors[i / E][i % E].first_elem, vector);
        crew.wait([&]() {
            // blob order: down tensors (type 2) first, then fused gate/up tensors
            uint64_t nb = 0, units = 0;
            for (int ti : {1, 0})
                for (uint32_t e = 0; e < E; ++e) {
                    L.tensors[ti][e].first_block = nb;
                    nb += L.tensors[ti][e].n_blocks();
                }
            for (uint32_t i = 0; i < 2 * E; ++i) unit_end[i] = units += (L.tensors[i / E][i % E].n_blocks() + kBlocksPerUnit - 1) / kBlocksPerUnit;
            L.n_blocks = nb;
            fits = size_t(nb) * B <= dst_cap;
        });
        // 3. encode
        if (!fits) return;
        for (uint64_t u; (u = crew.take()) < unit_end.back();) {
            const uint32_t i = uint32_t(std::upper_bound(unit_end.begin(), unit_end.end(), u) - unit_end.begin());
            const TensorMeta& tm = L.tensors[i / E][i % E];
            const uint64_t k0 = (u - (i ? unit_end[i - 1] : 0)) * kBlocksPerUnit;
            encode_blocks(tensor(i), tm.first_elem, k0, std::min(k0 + kBlocksPerUnit, tm.n_blocks()), coder[i / E], B, out + size_t(tm.first_block) * B, vector);
        }
    });
    *dst_used = size_t(L.n_blocks) * B;
    if (!fits)
        return set_error(FLUXMOE_ENOMEM, "layer blob needs %zu bytes, dst_cap is %zu", size_t(L.n_blocks) * B, dst_cap);
    L.encoded = true;
    return FLUXMOE_OK;
    } catch (const std::bad_alloc&) {
        return set_error(FLUXMOE_ENOMEM, "out of host memory");
    }
}

int fluxmoe_layer_info_get(const fluxmoe_ctx* c, uint32_t layer, fluxmoe_layer_info* out) {
    if (int rc = check_layer(c, layer, true)) return rc;
    if (!out) return set_error(FLUXMOE_EINVAL, "out is NULL");
    const LayerMeta& L = c->layers[layer];
    out->n_blocks = L.n_blocks;
    out->payload_bits[0] = L.payload_bits[0];
    out->payload_bits[1] = L.payload_bits[1];
    out->elements[0] = c->elems13 * c->d.n_experts;
    out->elements[1] = c->elems2 * c->d.n_experts;
    return FLUXMOE_OK;
}

static int type_index(int type) { return type == 1 ? 0 : (type == 2 ? 1 : -1); }

int fluxmoe_code_lengths(const fluxmoe_ctx* c, uint32_t layer, int type, uint8_t out_lens[256]) {
    if (int rc = check_layer(c, layer, true)) return rc;
    const int ti = type_index(type);
    if (ti < 0 || !out_lens) return set_error(FLUXMOE_EINVAL, "type must be 1 or 2, out non-NULL");
    std::memcpy(out_lens, c->layers[layer].lens[ti], 256);
    return FLUXMOE_OK;
}

int fluxmoe_tensor_blocks(const fluxmoe_ctx* c, uint32_t layer, int type, uint32_t expert,
                          uint64_t* first_block, uint64_t* n_blocks) {
    if (int rc = check_layer(c, layer, true)) return rc;
    const int ti = type_index(type);
    if (ti < 0 || !first_block || !n_blocks) return set_error(FLUXMOE_EINVAL, "bad type or NULL out");
    if (expert >= c->d.n_experts) return set_error(FLUXMOE_ERANGE, "expert %u out of range", expert);
    const TensorMeta& tm = c->layers[layer].tensors[ti][expert];
    *first_block = tm.first_block;
    *n_blocks = tm.n_blocks();
    return FLUXMOE_OK;
}

int fluxmoe_tensor_first_elems(const fluxmoe_ctx* c, uint32_t layer, int type, uint32_t expert,
                               uint32_t* out, size_t out_cap) {
    if (int rc = check_layer(c, layer, true)) return rc;
    const int ti = type_index(type);
    if (ti < 0 || !out) return set_error(FLUXMOE_EINVAL, "bad type or NULL out");
    if (expert >= c->d.n_experts) return set_error(FLUXMOE_ERANGE, "expert %u out of range", expert);
    const TensorMeta& tm = c->layers[layer].tensors[ti][expert];
    if (out_cap < tm.first_elem.size())
        return set_error(FLUXMOE_ENOMEM, "out_cap %zu < %zu", out_cap, tm.first_elem.size());
    std::memcpy(out, tm.first_elem.data(), tm.first_elem.size() * 4);
    return FLUXMOE_OK;
}

int fluxmoe_bind_arenas(fluxmoe_ctx* c, void* slots13, void* slots2, void* workspace,
                        size_t workspace_bytes) {
    if (!c) return set_error(FLUXMOE_EINVAL, "ctx is NULL");
    if (!slots13 || !slots2 || !workspace) return set_error(FLUXMOE_EINVAL, "NULL arena");
    if ((uintptr_t(slots13) | uintptr_t(slots2) | uintptr_t(workspace)) & 255)
        return set_error(FLUXMOE_EINVAL, "arenas must be 256-byte aligned");
    if (workspace_bytes < c->pool_ws_bytes)
        return set_error(FLUXMOE_ENOMEM, "workspace needs at least %llu bytes",
                         (unsigned long long)c->pool_ws_bytes);
    int dev = 0;
    HIPCHECK(hipGetDevice(&dev));
    hipDeviceProp_t prop;
    HIPCHECK(hipGetDeviceProperties(&prop, dev));
    if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
        return set_error(FLUXMOE_EHIP, "device is %s; this library is built for gfx950 only", prop.gcnArchName);
    c->n_cus = prop.multiProcessorCount;
    if (int rc = resolve_static_scratch(dev)) return rc;
    c->device = dev;
    if (int rc = ensure_events(c)) return rc;
    c->slots13 = static_cast<uint8_t*>(slots13);
    c->slots2 = static_cast<uint8_t*>(slots2);
    c->ws = static_cast<uint8_t*>(workspace);
    c->ws_bytes = workspace_bytes;
    HIPCHECK(hipMemset(c->ws + c->err_off, 0, 256));
    c->arenas_bound = true;
    for (auto& L : c->layers) L.bound = false;
    return FLUXMOE_OK;
}

int fluxmoe_bind_layer(fluxmoe_ctx* c, uint32_t layer, const void* hbm_blocks, uint64_t n_host_blocks,
                       const void* host_blocks, const void* check_host_copy) {
    if (int rc = check_layer(c, layer, true)) return rc;
    if (!c->arenas_bound) return set_error(FLUXMOE_ESTATE, "fluxmoe_bind_arenas has not been called");
    LayerMeta& L = c->layers[layer];
    if (n_host_blocks > L.n_blocks)
        return set_error(FLUXMOE_ERANGE, "n_host_blocks %llu > n_blocks %llu",
                         (unsigned long long)n_host_blocks, (unsigned long long)L.n_blocks);
    if (n_host_blocks > 0 && !host_blocks) return set_error(FLUXMOE_EINVAL, "host_blocks is NULL");
    if (n_host_blocks < L.n_blocks && !hbm_blocks) return set_error(FLUXMOE_EINVAL, "hbm_blocks is NULL");
    if ((uintptr_t(hbm_blocks) | uintptr_t(host_blocks)) & 15)
        return set_error(FLUXMOE_EINVAL, "block arenas must be 16-byte aligned");
    if (check_host_copy) {
        const uint8_t* blob = static_cast<const uint8_t*>(check_host_copy);
        const uint32_t B = c->d.block_bytes;
        for (int ti = 0; ti < 2; ++ti)
            for (uint32_t e = 0; e < c->d.n_experts; ++e) {
                const TensorMeta& tm = L.tensors[ti][e];
                for (uint64_t k = 0; k < tm.n_blocks(); ++k) {
                    uint32_t hdr[2];
                    std::memcpy(hdr, blob + (tm.first_block + k) * B, 8);
                    if (hdr[0] != tm.first_elem[k + 1] - tm.first_elem[k] || hdr[1] != tm.first_elem[k])
                        return set_error(FLUXMOE_ECORRUPT,
                                         "layer %u type %d expert %u block %llu: header (n=%u, e0=%u) "
                                         "does not match the encoder's metadata",
                                         layer, ti + 1, e, (unsigned long long)k, hdr[0], hdr[1]);
                }
            }
    }
    std::vector<uint32_t> lut(2 * kLutEntries);
    build_lut(L.lens[0], lut.data());
    build_lut(L.lens[1], lut.data() + kLutEntries);
    HIPCHECK(hipMemcpy(c->ws + c->lut_off + uint64_t(layer) * 2 * kLutBytes, lut.data(), 2 * kLutBytes,
                       hipMemcpyHostToDevice));
    L.hbm = static_cast<const uint8_t*>(hbm_blocks);
    L.host = static_cast<const uint8_t*>(host_blocks);
    L.n_host_blocks = n_host_blocks;
    L.host_tensors = 0;
    for (int ti = 0; ti < 2; ++ti)
        for (TensorMeta& tm : L.tensors[ti]) {
            const uint64_t a = tm.first_block, b = a + tm.n_blocks();
            const uint64_t hb = std::min(b, std::max(a, n_host_blocks));
            tm.n_host = hb - a;
            tm.raw_src = nullptr;
            tm.host_src = tm.n_host ? L.host + a * c->d.block_bytes : nullptr;
            tm.hbm_src = hb < b ? L.hbm + (hb - n_host_blocks) * c->d.block_bytes : nullptr;
            L.host_tensors += tm.on_host() ? 1 : 0;
        }
    L.bound = true;
    if (c->half[layer & 1].layer == int64_t(layer)) c->half[layer & 1].layer = -1;
    return FLUXMOE_OK;
}

int fluxmoe_bind_staging(fluxmoe_ctx* c, void* staging, size_t staging_bytes) {
    if (!c) return set_error(FLUXMOE_EINVAL, "ctx is NULL");
    if (!staging || (uintptr_t(staging) & 255)) return set_error(FLUXMOE_EINVAL, "staging must be non-NULL, 256-byte aligned");
    if (staging_bytes < 2ull * c->d.block_bytes) return set_error(FLUXMOE_ENOMEM, "staging too small");
    c->staging = static_cast<uint8_t*>(staging);
    c->staging_bytes = staging_bytes;
    c->half[0].layer = c->half[1].layer = -1;
    return FLUXMOE_OK;
}

int fluxmoe_set_tensor_backing(fluxmoe_ctx* c, uint32_t layer, int type, uint32_t expert, int tier,
                               const void* blocks) {
    if (int rc = check_layer(c, layer, true)) return rc;
    LayerMeta& L = c->layers[layer];
    if (!L.bound) return set_error(FLUXMOE_ESTATE, "layer %u is not bound", layer);
    if (type != 1 && type != 2) return set_error(FLUXMOE_EINVAL, "type must be 1 or 2");
    if (expert >= c->d.n_experts) return set_error(FLUXMOE_ERANGE, "expert %u out of range", expert);
    if (tier != FLUXMOE_TIER_HBM && tier != FLUXMOE_TIER_HOST && tier != FLUXMOE_TIER_HOST_RAW)
        return set_error(FLUXMOE_EINVAL, "tier must be 0 (HBM), 1 (pinned host, compressed) or 2 (pinned host, dense)");
    if (!blocks || (uintptr_t(blocks) & 15)) return set_error(FLUXMOE_EINVAL, "blocks must be non-NULL, 16-byte aligned");
    TensorMeta& tm = L.tensors[type - 1][expert];
    L.host_tensors -= tm.on_host() ? 1 : 0;
    tm.n_host = 0;
    tm.host_src = tm.hbm_src = tm.raw_src = nullptr;
    if (tier == FLUXMOE_TIER_HOST) {
        tm.n_host = tm.n_blocks();
        tm.host_src = static_cast<const uint8_t*>(blocks);
    } else if (tier == FLUXMOE_TIER_HOST_RAW) {
        tm.raw_src = static_cast<const uint8_t*>(blocks);
    } else {
        tm.hbm_src = static_cast<const uint8_t*>(blocks);
    }
    L.host_tensors += tm.on_host() ? 1 : 0;
    if (c->half[layer & 1].layer == int64_t(layer)) c->half[layer & 1].layer = -1;   // staged copies are stale
    return FLUXMOE_OK;
}

int fluxmoe_reset_page_table(fluxmoe_ctx* c, int32_t* page_table, void* stream) {
    if (!c || !page_table) return set_error(FLUXMOE_EINVAL, "NULL argument");
    HIPCHECK(launch_fill_i32(page_table, -1, uint64_t(c->d.n_layers) * c->d.n_experts,
                             static_cast<hipStream_t>(stream)));
    std::fill(c->pt.begin(), c->pt.end(), -1);
    std::fill(c->slot_owner.begin(), c->slot_owner.end(), -1);
    return FLUXMOE_OK;
}

static int validate_ids(const fluxmoe_ctx* c, const int32_t* ids, uint32_t n) {
    if (n > c->d.n_experts) return set_error(FLUXMOE_EINVAL, "n %u > n_experts %u", n, c->d.n_experts);
    if (n && !ids) return set_error(FLUXMOE_EINVAL, "expert_ids is NULL");
    std::vector<uint8_t> seen(c->d.n_experts, 0);
    for (uint32_t i = 0; i < n; ++i) {
        if (ids[i] < 0 || uint32_t(ids[i]) >= c->d.n_experts)
            return set_error(FLUXMOE_ERANGE, "expert id %d out of range [0, %u)", ids[i], c->d.n_experts);
        if (seen[ids[i]]++) return set_error(FLUXMOE_EINVAL, "expert id %d listed twice", ids[i]);
    }
    return FLUXMOE_OK;
}

// Copies of the listed experts' host-tier blocks into the layer's staging half (layer & 1).
// The half keeps them until the next staging into it; the copies wait (on the device) for the
// last decode that read the half.
static int stage_host_blocks(fluxmoe_ctx* c, uint32_t layer, const int32_t* ids, uint32_t n,
                             hipStream_t s) {
    LayerMeta& L = c->layers[layer];
    const int h = layer & 1;
    StageHalf& st = c->half[h];
    st.layer = -1;
    st.off[0].assign(c->d.n_experts, -1);
    st.off[1].assign(c->d.n_experts, -1);
    if (L.host_tensors == 0) { st.layer = layer; return FLUXMOE_OK; }
    if (!c->staging) return set_error(FLUXMOE_ESTATE, "layer %u has host-tier blocks but no staging buffer is bound", layer);
    const uint32_t B = c->d.block_bytes;
    const uint64_t half_bytes = (c->staging_bytes / 2) / B * B;
    uint8_t* base = c->staging + h * half_bytes;
    std::vector<int32_t> sorted(ids, ids + n);
    std::sort(sorted.begin(), sorted.end());
    struct Range { const uint8_t* src; uint64_t bytes, dst; };
    std::vector<Range> ranges;               // adjacent source ranges are merged into one copy
    uint64_t cursor = 0;
    for (int ti : {1, 0})
        for (int32_t e : sorted) {
            const TensorMeta& tm = L.tensors[ti][e];
            if (!tm.on_host()) continue;
            st.off[ti][e] = int64_t(cursor);
            // dense tensors are staged whole (a multiple of 16 bytes); the cursor stays block aligned
            const uint8_t* src = tm.raw_src ? tm.raw_src : tm.host_src;
            const uint64_t bytes = tm.raw_src ? (ti == 0 ? c->elems13 : c->elems2) * 2 : tm.n_host * B;
            if (!ranges.empty() && ranges.back().src + ranges.back().bytes == src &&
                ranges.back().dst + ranges.back().bytes == cursor) ranges.back().bytes += bytes;
            else ranges.push_back({src, bytes, cursor});
            cursor += align_up(bytes, B);
        }
    if (cursor > half_bytes)
        return set_error(FLUXMOE_ENOMEM, "staging half holds %llu bytes, layer %u needs %llu",
                         (unsigned long long)half_bytes, layer, (unsigned long long)cursor);
    if (c->half_read[h]) HIPCHECK(hipStreamWaitEvent(s, c->half_read[h], 0));
    // an earlier staging into this half may have been issued on another stream (a prefetch on the copy
    // stream, then a materialize of other experts that restages on its own stream): its copies must
    // have landed before these overwrite the half with a different layout
    if (c->copied_valid[h]) HIPCHECK(hipStreamWaitEvent(s, c->ev_copied[h], 0));
    for (const Range& r : ranges)
        HIPCHECK(hipMemcpyAsync(base + r.dst, r.src, r.bytes, hipMemcpyHostToDevice, s));
    HIPCHECK(hipEventRecord(c->ev_copied[h], s));
    c->copied_valid[h] = true;
    st.layer = layer;
    return FLUXMOE_OK;
}

int fluxmoe_prefetch_host(fluxmoe_ctx* c, uint32_t layer, const int32_t* expert_ids, uint32_t n,
                          void* copy_stream) {
    if (int rc = check_layer(c, layer, true)) return rc;
    if (!c->layers[layer].bound) return set_error(FLUXMOE_ESTATE, "layer %u is not bound", layer);
    if (int rc = validate_ids(c, expert_ids, n)) return rc;
    return stage_host_blocks(c, layer, expert_ids, n, static_cast<hipStream_t>(copy_stream));
}

// Body of fluxmoe_materialize and fluxmoe_materialize_two_streams.  two_streams: the down tensors (type 2) are
// decoded on stream2_v while the fused gate/up tensors (type 1) are decoded on stream_v; stream_v waits for
// both before it records the layer's load event.
static int materialize_enqueue(fluxmoe_ctx* c, uint32_t layer, const int32_t* expert_ids, uint32_t n,
                               int32_t* page_table, const int32_t* dst_slots, void* stream_v, bool two_streams,
                               void* stream2_v) {
    if (int rc = check_layer(c, layer, true)) return rc;
    LayerMeta& L = c->layers[layer];
    if (!c->arenas_bound || !L.bound) return set_error(FLUXMOE_ESTATE, "arenas or layer %u not bound", layer);
    if (!page_table) return set_error(FLUXMOE_EINVAL, "page_table is NULL");
    if (int rc = validate_ids(c, expert_ids, n)) return rc;
    if (n && !dst_slots) return set_error(FLUXMOE_EINVAL, "dst_slots is NULL");
    {
        std::vector<uint8_t> seen(c->d.n_slots, 0);
        for (uint32_t i = 0; i < n; ++i) {
            if (dst_slots[i] < 0 || uint32_t(dst_slots[i]) >= c->d.n_slots)
                return set_error(FLUXMOE_ERANGE, "slot %d out of range [0, %u)", dst_slots[i], c->d.n_slots);
            if (seen[dst_slots[i]]++) return set_error(FLUXMOE_EINVAL, "slot %d listed twice", dst_slots[i]);
        }
    }
    if (n == 0) return FLUXMOE_OK;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    const uint32_t E = c->d.n_experts, B = c->d.block_bytes;

    // host-tier parts must be staged for exactly these experts
    bool need_host = false;
    for (uint32_t i = 0; i < n && !need_host; ++i)
        for (int ti = 0; ti < 2; ++ti)
            if (L.tensors[ti][expert_ids[i]].on_host()) need_host = true;
    bool wait_copy = false;
    if (need_host) {
        StageHalf& st = c->half[layer & 1];
        bool staged = st.layer == int64_t(layer);
        for (uint32_t i = 0; i < n && staged; ++i)
            for (int ti = 0; ti < 2; ++ti)
                if (L.tensors[ti][expert_ids[i]].on_host() && st.off[ti][expert_ids[i]] < 0)
                    staged = false;
        if (!staged) {
            if (int rc = stage_host_blocks(c, layer, expert_ids, n, stream)) return rc;
        } else {
            wait_copy = true;
        }
    }

    // ring slot for the command buffer
    const int slot = c->ring_next;
    if (c->ring_used[slot]) HIPCHECK(hipEventSynchronize(c->ring_ev[slot]));
    uint8_t* hcmd = c->pinned_cmd + size_t(slot) * c->cmd_bytes;
    uint8_t* dcmd = c->ws + c->cmd_off + size_t(slot) * c->cmd_bytes;
    DecodeCmd* cmd = reinterpret_cast<DecodeCmd*>(hcmd);
    const uint32_t jobs_off[2] = {uint32_t(sizeof(DecodeCmd)),
                                  uint32_t(sizeof(DecodeCmd) + c->max_jobs * sizeof(DecodeJob))};
    const uint32_t upd_off = uint32_t(sizeof(DecodeCmd) + 2ull * c->max_jobs * sizeof(DecodeJob));
    std::memset(cmd, 0, sizeof(DecodeCmd));

    const int half = layer & 1;
    const uint64_t half_bytes = c->staging ? (c->staging_bytes / 2) / B * B : 0;
    struct DenseCopy { const uint8_t* src; uint8_t* dst; uint64_t bytes; };
    std::vector<DenseCopy> dense_copies;     // staged uncompressed tensors: staging -> slot, no decode
    for (int ti = 0; ti < 2; ++ti) {
        DecodeJob* jobs = reinterpret_cast<DecodeJob*>(hcmd + jobs_off[ti]);
        uint32_t nj = 0, blocks = 0;
        const uint64_t sigma = (ti == 0 ? c->elems13 : c->elems2) * 2;
        uint8_t* arena = ti == 0 ? c->slots13 : c->slots2;
        for (uint32_t i = 0; i < n; ++i) {
            const TensorMeta& tm = L.tensors[ti][expert_ids[i]];
            const uint64_t nb = tm.n_blocks(), nh = tm.n_host;     // host part is the first nh blocks
            const uint64_t dst = uint64_t(uintptr_t(arena)) + uint64_t(dst_slots[i]) * sigma;
            if (tm.raw_src) {
                dense_copies.push_back({c->staging + half * half_bytes + c->half[half].off[ti][expert_ids[i]],
                                        reinterpret_cast<uint8_t*>(uintptr_t(dst)), sigma});
                continue;
            }
            if (nh) {
                const uint8_t* src = c->staging + half * half_bytes + c->half[half].off[ti][expert_ids[i]];
                jobs[nj++] = DecodeJob{uint64_t(uintptr_t(src)), dst, blocks, uint32_t(nh),
                                       uint32_t(ti == 0 ? c->elems13 : c->elems2), 0};
                blocks += uint32_t(nh);
            }
            if (nb > nh) {
                jobs[nj++] = DecodeJob{uint64_t(uintptr_t(tm.hbm_src)), dst, blocks, uint32_t(nb - nh),
                                       uint32_t(ti == 0 ? c->elems13 : c->elems2), 0};
                blocks += uint32_t(nb - nh);
            }
        }
        cmd->n_jobs[ti] = nj;
        cmd->total_blocks[ti] = blocks;
    }

    // page-table transitions on the host mirror; the touched entries go to the device
    std::vector<int64_t> touched;
    std::vector<std::pair<int32_t, uint64_t>> wait_reads;      // (layer, FFN call) that read a target slot last
    for (uint32_t i = 0; i < n; ++i) {
        const int64_t key = int64_t(layer) * E + expert_ids[i];
        const int32_t s = dst_slots[i];
        const int32_t old_slot = c->pt[key];
        if (old_slot >= 0 && old_slot != s) c->slot_owner[old_slot] = -1;
        const int64_t prev = c->slot_owner[s];
        if (prev >= 0 && prev != key) {
            c->pt[prev] = -1;
            touched.push_back(prev);
        }
        c->pt[key] = s;
        c->slot_owner[s] = key;
        touched.push_back(key);
        const int32_t lr = c->slot_last_reader[s];
        if (lr >= 0) {
            // a layer's FFN calls run in order: one older than the last two is covered by the older of those, and with a
            // capture's border between the two by the last
            const uint64_t last = c->infer_gen[lr];
            const bool older = c->slot_reader_gen[s] < last && c->infer_capture[lr][0] == c->infer_capture[lr][1];
            const std::pair<int32_t, uint64_t> read{lr, older ? last - 1 : last};
            if (std::find(wait_reads.begin(), wait_reads.end(), read) == wait_reads.end()) wait_reads.push_back(read);
        }
        c->slot_last_reader[s] = -1;
    }
    std::sort(touched.begin(), touched.end());
    touched.erase(std::unique(touched.begin(), touched.end()), touched.end());
    int32_t* upd = reinterpret_cast<int32_t*>(hcmd + upd_off);
    for (size_t i = 0; i < touched.size(); ++i) {
        upd[2 * i] = int32_t(touched[i]);
        upd[2 * i + 1] = c->pt[touched[i]];
    }
    cmd->n_pt_updates = uint32_t(touched.size());

    // enqueue: WAR waits, host-tier copies, command upload, decode, events
    // (a release of this layer, which writes the same page-table row, may have been issued on another stream; one made
    // after the layer's FFN waited for it)
    auto rel_covers = [&](uint64_t g) {
        const uint64_t at = c->infer_seq[layer][g & 1];
        return c->rel_valid[layer] && at && c->rel_seq[layer] > at;
    };
    for (const auto& [lr, g] : wait_reads)
        if (!(uint32_t(lr) == layer && rel_covers(g))) HIPCHECK(hipStreamWaitEvent(stream, c->ev_infer[lr][g & 1], 0));
    if (c->rel_valid[layer]) HIPCHECK(hipStreamWaitEvent(stream, c->ev_rel[layer], 0));
    if (wait_copy) HIPCHECK(hipStreamWaitEvent(stream, c->ev_copied[half], 0));
    // a wave of this layer still to be released: its FFN must have read the page table before this call's entries appear
    // there.  Both outside capture, or both in one capture: a wait across a capture's border orders nothing (or is refused),
    // and ordering a graph against other work is its launcher's part.
    const uint64_t capture = capture_of(stream);       // after the waits above: one of them may have taken the stream into a capture
    const uint64_t last_ffn = c->infer_gen[layer];
    if (last_ffn && c->routed_gen[layer] == last_ffn && !rel_covers(last_ffn) && c->infer_capture[layer][last_ffn & 1] == capture)
        HIPCHECK(hipStreamWaitEvent(stream, c->ev_routed[layer], 0));

    DecodeArgs args{};
    args.lut[0] = reinterpret_cast<const uint32_t*>(c->ws + c->lut_off + (uint64_t(layer) * 2 + 0) * kLutBytes);
    args.lut[1] = reinterpret_cast<const uint32_t*>(c->ws + c->lut_off + (uint64_t(layer) * 2 + 1) * kLutBytes);
    args.page_table = page_table;
    args.error_word = reinterpret_cast<uint32_t*>(c->ws + c->err_off);
    // A command that is small enough travels inside the kernel arguments, packed without the gaps of the
    // ring slot's fixed layout; a larger one is uploaded into the ring slot in front of the kernel.
    const uint64_t decode_blocks = uint64_t(cmd->total_blocks[0]) + cmd->total_blocks[1];
    const size_t jobs_bytes[2] = {cmd->n_jobs[0] * sizeof(DecodeJob), cmd->n_jobs[1] * sizeof(DecodeJob)};
    const size_t packed = sizeof(DecodeCmd) + jobs_bytes[0] + jobs_bytes[1] + touched.size() * 8;
    const bool uploaded = !(decode_blocks > 0 && packed <= kInlineCmdBytes);
    if (!need_host && c->half_read[half] == c->ev_load[layer] && c->half_capture[half] != capture)
        std::swap(c->ev_load[layer], c->half_spare[half]);
    hipEvent_t load_done = capture == 0 ? c->ev_load[layer] : nullptr; // nullptr: recorded at the end
    if (c->profiling && (c->profile_mask & 1u)) load_done = nullptr;   // the kernel's span is to hold the kernel alone
    if (!uploaded) {
        uint8_t* w = reinterpret_cast<uint8_t*>(args.inline_words);
        std::memcpy(w, cmd, sizeof(DecodeCmd));
        args.jobs_offset[0] = uint32_t(sizeof(DecodeCmd));
        args.jobs_offset[1] = uint32_t(args.jobs_offset[0] + jobs_bytes[0]);
        args.upd_offset = uint32_t(args.jobs_offset[1] + jobs_bytes[1]);
        std::memcpy(w + args.jobs_offset[0], hcmd + jobs_off[0], jobs_bytes[0]);
        std::memcpy(w + args.jobs_offset[1], hcmd + jobs_off[1], jobs_bytes[1]);
        std::memcpy(w + args.upd_offset, hcmd + upd_off, touched.size() * 8);
        args.inline_cmd = 1;
        args.cmd = nullptr;
    } else {
        const size_t used = upd_off + touched.size() * 8;
        HIPCHECK(hipMemcpyAsync(dcmd, hcmd, used, hipMemcpyHostToDevice, stream));
        args.cmd = reinterpret_cast<const DecodeCmd*>(dcmd);
        args.jobs_offset[0] = jobs_off[0];
        args.jobs_offset[1] = jobs_off[1];
        args.upd_offset = upd_off;
        args.inline_cmd = 0;
    }
    for (const DenseCopy& dc : dense_copies)
        HIPCHECK(hipMemcpyAsync(dc.dst, dc.src, dc.bytes, hipMemcpyDeviceToDevice, stream));
    const uint64_t total = uint64_t(cmd->total_blocks[0]) + cmd->total_blocks[1];
    const int waves_per_wg = c->tune_waves;
    if (total == 0) {
        // every listed tensor is an uncompressed host tensor: nothing to decode, only the page table changes
        load_done = nullptr;
        if (!touched.empty())
            HIPCHECK(launch_apply_updates(page_table, dcmd + upd_off, uint32_t(touched.size()), stream, nullptr));
    } else {
    const uint64_t per_wg = decode_per_workgroup(total, uint64_t(std::max(c->n_cus, 1)), uint64_t(waves_per_wg), uint64_t(c->tune_blocks_per_wave));
    auto wgs_for = [&](uint64_t blocks) { return uint32_t(std::min<uint64_t>((blocks + per_wg - 1) / per_wg, 1u << 20)); };
    if (two_streams && cmd->total_blocks[0] && cmd->total_blocks[1]) {
        // one launch per tensor type: the type-2 list on the second stream (after everything this call has
        // enqueued on the first one so far), the type-1 list and the page-table updates on the first
        hipStream_t stream2 = static_cast<hipStream_t>(stream2_v);
        HIPCHECK(hipEventRecord(c->ev_fork, stream));
        HIPCHECK(hipStreamWaitEvent(stream2, c->ev_fork, 0));
        DecodeArgs a2 = args;
        const uint32_t n2 = wgs_for(cmd->total_blocks[1]);
        a2.wg_split = n2;                       // every workgroup serves the type-2 list
        a2.apply_updates = 0;
        hipEvent_t join = attachable(c->ev_join, stream2);
        HIPCHECK(launch_decode(a2, n2, waves_per_wg, stream2, join));
        if (!join) HIPCHECK(hipEventRecord(c->ev_join, stream2));
        args.wg_split = 0;                      // every workgroup serves the type-1 list
        args.apply_updates = 1;
        HIPCHECK(span_begin(c, 0, stream));
        load_done = nullptr;                    // the load is done when both launches are
        HIPCHECK(launch_decode(args, wgs_for(cmd->total_blocks[0]), waves_per_wg, stream, nullptr));
        HIPCHECK(span_end(c, stream));
        HIPCHECK(hipStreamWaitEvent(stream, c->ev_join, 0));
    } else {
        uint32_t n_wg = std::max(wgs_for(total), 2u);
        uint32_t split = uint32_t((uint64_t(n_wg) * cmd->total_blocks[1] + total / 2) / total);
        split = std::min(std::max(split, 1u), n_wg - 1);
        args.wg_split = split;
        args.apply_updates = 1;
        HIPCHECK(span_begin(c, 0, stream));
        HIPCHECK(launch_decode(args, n_wg, waves_per_wg, stream, load_done));
        HIPCHECK(span_end(c, stream));
    }
    }
    if (uploaded) {                             // only then does the device read the ring slot
        HIPCHECK(hipEventRecord(c->ring_ev[slot], stream));
        c->ring_used[slot] = true;
        c->ring_next = (slot + 1) % kRing;
    }
    if (!load_done) HIPCHECK(hipEventRecord(c->ev_load[layer], stream));
    c->load_valid[layer] = 1;
    c->load_seq[layer] = capture ? 0 : ++c->seq;
    if (need_host) {
        c->half_read[half] = c->ev_load[layer];
        c->half_capture[half] = capture;
    }
    return FLUXMOE_OK;
}

int fluxmoe_materialize(fluxmoe_ctx* c, uint32_t layer, const int32_t* expert_ids, uint32_t n,
                        int32_t* page_table, const int32_t* dst_slots, void* stream) {
    return materialize_enqueue(c, layer, expert_ids, n, page_table, dst_slots, stream, false, nullptr);
}

int fluxmoe_materialize_two_streams(fluxmoe_ctx* c, uint32_t layer, const int32_t* expert_ids, uint32_t n,
                                    int32_t* page_table, const int32_t* dst_slots, void* stream,
                                    void* stream_type2) {
    return materialize_enqueue(c, layer, expert_ids, n, page_table, dst_slots, stream, stream_type2 != stream, stream_type2);
}

int fluxmoe_release(fluxmoe_ctx* c, uint32_t layer, const int32_t* expert_ids, uint32_t n,
                    int32_t* page_table, void* stream_v) {
    if (int rc = check_layer(c, layer, false)) return rc;
    if (!c->arenas_bound) return set_error(FLUXMOE_ESTATE, "fluxmoe_bind_arenas has not been called");
    if (!page_table) return set_error(FLUXMOE_EINVAL, "page_table is NULL");
    if (expert_ids) {
        if (int rc = validate_ids(c, expert_ids, n)) return rc;
    } else if (n != 0) {
        return set_error(FLUXMOE_EINVAL, "expert_ids is NULL but n is %u", n);
    }
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    const uint32_t E = c->d.n_experts;
    const int slot = c->ring_next;
    if (c->ring_used[slot]) HIPCHECK(hipEventSynchronize(c->ring_ev[slot]));
    uint8_t* hcmd = c->pinned_cmd + size_t(slot) * c->cmd_bytes;
    uint8_t* dcmd = c->ws + c->cmd_off + size_t(slot) * c->cmd_bytes;
    int32_t* upd = reinterpret_cast<int32_t*>(hcmd);
    uint32_t m = 0;
    const uint32_t count = expert_ids ? n : E;
    for (uint32_t i = 0; i < count; ++i) {
        const int64_t key = int64_t(layer) * E + (expert_ids ? expert_ids[i] : int32_t(i));
        const int32_t s = c->pt[key];
        if (s < 0) continue;
        c->pt[key] = -1;
        c->slot_owner[s] = -1;       // the slot keeps its last-reader layer: reuse still waits
        upd[2 * m] = int32_t(key);
        upd[2 * m + 1] = -1;
        ++m;
    }
    if (m == 0) return FLUXMOE_OK;
    // the entries are read by the layer's FFN and written by its materialize, possibly on other streams
    const uint64_t last_ffn = c->infer_gen[layer];
    if (last_ffn) HIPCHECK(hipStreamWaitEvent(stream, c->ev_infer[layer][last_ffn & 1], 0));
    const bool infer_covers_load = last_ffn && c->load_seq[layer] && c->infer_seq[layer][last_ffn & 1] > c->load_seq[layer];
    if (c->load_valid[layer] && !infer_covers_load) HIPCHECK(hipStreamWaitEvent(stream, c->ev_load[layer], 0));
    const hipEvent_t done = attachable(c->ev_rel[layer], stream);
    if (m <= kInlineUpdates) {
        HIPCHECK(launch_apply_updates_inline(page_table, upd, m, stream, done));     // the pairs travel in the kernel arguments
    } else {
        HIPCHECK(hipMemcpyAsync(dcmd, hcmd, size_t(m) * 8, hipMemcpyHostToDevice, stream));
        HIPCHECK(launch_apply_updates(page_table, dcmd, m, stream, done));
        HIPCHECK(hipEventRecord(c->ring_ev[slot], stream));
        c->ring_used[slot] = true;
        c->ring_next = (slot + 1) % kRing;
    }
    if (!done) HIPCHECK(hipEventRecord(c->ev_rel[layer], stream));
    c->rel_valid[layer] = 1;
    c->rel_seq[layer] = done ? ++c->seq : 0;
    return FLUXMOE_OK;
}

// Shared body of fluxmoe_expert_ffn and fluxmoe_expert_ffn_static: `w` is the FFN scratch (pair order, tile
// list, h, split-K partials) of `w_bytes` bytes, `w_name` says where it comes from in error texts.
static int expert_ffn_enqueue(fluxmoe_ctx* c, uint32_t layer, const uint16_t* tokens, uint32_t T,
                              const int32_t* topk_ids, const float* topk_w, uint32_t K,
                              const int32_t* page_table, float* out, uint32_t flags, void* stream_v,
                              uint8_t* w, uint64_t w_bytes, const char* w_name) {
    if (!tokens || !topk_ids || !topk_w || !page_table || !out) return set_error(FLUXMOE_EINVAL, "NULL argument");
    if (K == 0 || K > c->d.n_experts) return set_error(FLUXMOE_EINVAL, "K must be in 1..n_experts");
    if (flags & ~3u) return set_error(FLUXMOE_EINVAL, "unknown flags 0x%x", flags);
    if (uint64_t(T) * K >= (1ull << 31) || T > 65535) return set_error(FLUXMOE_EINVAL, "T too large");
    if (uint64_t(T) * c->d.hidden * 2 >= (1ull << 32))
        return set_error(FLUXMOE_EINVAL, "tokens (T * hidden * 2 bytes) must stay under 4 GiB");
    if ((uintptr_t(tokens) | uintptr_t(out)) & 15) return set_error(FLUXMOE_EINVAL, "tokens/out must be 16-byte aligned");
    uint32_t mapped = 0;
    for (uint32_t e = 0; e < c->d.n_experts; ++e) mapped += c->pt[size_t(layer) * c->d.n_experts + e] >= 0 ? 1u : 0u;
    const FfnPlan p = plan_ffn(ffn_shape(c, c->d.n_experts), T, K, w_bytes, mapped);
    if (p.bytes > w_bytes)
        return set_error(FLUXMOE_ENOMEM, "%s holds %llu bytes, T=%u K=%u needs %llu", w_name,
                         (unsigned long long)w_bytes, T, K, (unsigned long long)p.bytes);
    if (p.tiles_cap > kMaxRowTiles) return set_error(FLUXMOE_EINVAL, "too many row tiles (%u)", p.tiles_cap);
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    FfnCall a{};
    a.tokens = tokens;
    a.topk_ids = topk_ids;
    a.topk_w = topk_w;
    a.page_table = page_table + size_t(layer) * c->d.n_experts;
    a.slots13 = reinterpret_cast<const uint16_t*>(c->slots13);
    a.slots2 = reinterpret_cast<const uint16_t*>(c->slots2);
    a.out = out;
    a.T = T; a.K = K; a.H = c->d.hidden; a.F = c->d.ffn; a.E = c->d.n_experts;
    a.flags = flags;
    a.expert_count = reinterpret_cast<int32_t*>(w + p.off_count);
    a.expert_offset = reinterpret_cast<int32_t*>(w + p.off_offset);
    a.sorted_pair = reinterpret_cast<int32_t*>(w + p.off_sorted);
    a.pair_pos = reinterpret_cast<int32_t*>(w + p.off_pos);
    a.tile_rec = reinterpret_cast<int4*>(w + p.off_tile);
    a.n_tiles = reinterpret_cast<int32_t*>(w + p.off_ntiles);
    a.chunk_count = reinterpret_cast<int32_t*>(w + p.off_h);
    a.n_chunks = p.n_chunks;
    a.hbuf = reinterpret_cast<uint16_t*>(w + p.off_h);
    a.ybuf = reinterpret_cast<float*>(w + p.off_y);
    a.error_word = reinterpret_cast<uint32_t*>(c->ws + c->err_off);
    a.pairs_cap = p.pairs_cap; a.tiles_cap = p.tiles_cap; a.m_tile = p.m_tile; a.tiled = p.tiled; a.halves = p.halves; a.g1_xcd = p.g1_xcd; a.ksplit = p.ksplit; a.ksplit1 = p.ksplit1; a.split_tiles = p.split_tiles;
    a.mapped = mapped;
    a.part = reinterpret_cast<float*>(w + p.off_part);
    a.tail = p.tail ? reinterpret_cast<float*>(w + p.off_tail) : nullptr;
    a.few = p.few;
    a.few_fused = p.few_fused;
    a.few2 = p.few_splits != 0;
    a.n_cus = uint32_t(std::max(c->n_cus, 1));
    a.tiled_waves = c->tune_tiled_waves;
    a.tiled_group = uint32_t(c->tune_tiled_group);
    a.tiled_persist = uint32_t(c->tune_tiled_persist);

    const bool load_covers_rel = c->load_seq[layer] > c->rel_seq[layer] && c->rel_seq[layer];
    const bool rel_covers_load = c->rel_seq[layer] > c->load_seq[layer] && c->load_seq[layer];
    if (c->load_valid[layer] && !rel_covers_load) HIPCHECK(hipStreamWaitEvent(stream, c->ev_load[layer], 0));
    if (c->rel_valid[layer] && !load_covers_rel) HIPCHECK(hipStreamWaitEvent(stream, c->ev_rel[layer], 0));
    const uint64_t gen = c->infer_gen[layer] + 1;
    const uint64_t capture = capture_of(stream);
    const hipEvent_t ev = c->ev_infer[layer][gen & 1], free_ev = capture == 0 ? ev : nullptr;
    const bool timed = c->profiling && (c->profile_mask & 0x1Eu);       // the kernels' spans are to hold the kernels alone
    const hipEvent_t done = timed ? nullptr : free_ev;
    // a call that skips unmapped experts is a wave: the next wave's materialize, into other slots, may follow before the release
    const hipEvent_t routed = flags & FLUXMOE_FFN_SKIP_UNMAPPED ? c->ev_routed[layer] : nullptr;
    HIPCHECK(launch_ffn(a, c->n_cus, stream, done, routed, capture == 0, c->profiling ? ffn_span_hook : nullptr, c));
    if (!done) HIPCHECK(hipEventRecord(ev, stream));
    c->infer_gen[layer] = gen;
    c->infer_seq[layer][gen & 1] = free_ev ? ++c->seq : 0;
    c->infer_capture[layer][gen & 1] = capture;
    if (routed) c->routed_gen[layer] = gen;
    const int64_t lo = int64_t(layer) * c->d.n_experts, hi = lo + c->d.n_experts;
    for (uint32_t s = 0; s < c->d.n_slots; ++s)
        if (c->slot_owner[s] >= lo && c->slot_owner[s] < hi) { c->slot_last_reader[s] = int32_t(layer); c->slot_reader_gen[s] = gen; }
    return FLUXMOE_OK;
}

int fluxmoe_expert_ffn(fluxmoe_ctx* c, uint32_t layer, const uint16_t* tokens, uint32_t T,
                       const int32_t* topk_ids, const float* topk_w, uint32_t K,
                       const int32_t* page_table, float* out, uint32_t flags, void* stream_v) {
    if (int rc = check_layer(c, layer, false)) return rc;
    if (!c->arenas_bound) return set_error(FLUXMOE_ESTATE, "fluxmoe_bind_arenas has not been called");
    if (T == 0) return FLUXMOE_OK;
    return expert_ffn_enqueue(c, layer, tokens, T, topk_ids, topk_w, K, page_table, out, flags, stream_v,
                              c->ws + c->pool_ws_bytes, c->ws_bytes - c->pool_ws_bytes, "the bound workspace past the pool part");
}

int fluxmoe_expert_ffn_static(fluxmoe_ctx* c, uint32_t layer, const uint16_t* tokens, uint32_t T,
                              const int32_t* topk_ids, const float* topk_w, uint32_t K,
                              const int32_t* page_table, float* out, uint32_t flags, void* stream_v) {
    if (int rc = check_layer(c, layer, false)) return rc;
    if (!c->arenas_bound) return set_error(FLUXMOE_ESTATE, "fluxmoe_bind_arenas has not been called");
    if (T == 0) return FLUXMOE_OK;
    uint8_t* w = (c->device >= 0 && c->device < kMaxDevices) ? g_static_scratch[c->device] : nullptr;
    if (!w) return set_error(FLUXMOE_ESTATE, "the static scratch of device %d was not resolved at bind time", c->device);
    int dev = -1;
    HIPCHECK(hipGetDevice(&dev));
    if (dev != c->device)
        return set_error(FLUXMOE_ESTATE, "current device is %d, the context was bound on device %d", dev, c->device);
    return expert_ffn_enqueue(c, layer, tokens, T, topk_ids, topk_w, K, page_table, out, flags, stream_v,
                              w, kStaticScratchBytes, "the static FFN scratch");
}

int fluxmoe_shared_expert_ffn(fluxmoe_ctx* c, const uint16_t* w13, const uint16_t* w2,
                              const uint16_t* tokens, uint32_t T, float* out, uint32_t flags,
                              void* stream_v) {
    if (!c) return set_error(FLUXMOE_EINVAL, "ctx is NULL");
    if (!c->arenas_bound) return set_error(FLUXMOE_ESTATE, "fluxmoe_bind_arenas has not been called");
    if (T == 0) return FLUXMOE_OK;
    if (!w13 || !w2 || !tokens || !out) return set_error(FLUXMOE_EINVAL, "NULL argument");
    if (flags & ~1u) return set_error(FLUXMOE_EINVAL, "only FLUXMOE_FFN_ACCUMULATE is accepted");
    if (T > 65535) return set_error(FLUXMOE_EINVAL, "T too large");
    if (uint64_t(T) * c->d.hidden * 2 >= (1ull << 32))
        return set_error(FLUXMOE_EINVAL, "tokens (T * hidden * 2 bytes) must stay under 4 GiB");
    if ((uintptr_t(w13) | uintptr_t(w2) | uintptr_t(tokens) | uintptr_t(out)) & 15)
        return set_error(FLUXMOE_EINVAL, "pointers must be 16-byte aligned");
    // this model's shapes, a single always-mapped expert
    const FfnPlan p = plan_shared(ffn_shape(c, 1), T, c->ws_bytes - c->pool_ws_bytes);
    if (c->pool_ws_bytes + p.bytes > c->ws_bytes)
        return set_error(FLUXMOE_ENOMEM, "workspace has %zu bytes, the shared expert with T=%u needs %llu",
                         c->ws_bytes, T, (unsigned long long)(c->pool_ws_bytes + p.bytes));
    if (p.tiles_cap > kMaxRowTiles) return set_error(FLUXMOE_EINVAL, "too many row tiles (%u)", p.tiles_cap);
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    uint8_t* w = c->ws + c->pool_ws_bytes;
    FfnCall a{};
    a.tokens = tokens;
    a.identity = 1;
    a.slots13 = w13;
    a.slots2 = w2;
    a.out = out;
    a.T = T; a.K = 1; a.H = c->d.hidden; a.F = c->d.ffn; a.E = 1;
    a.flags = flags;
    a.expert_count = reinterpret_cast<int32_t*>(w + p.off_count);
    a.expert_offset = reinterpret_cast<int32_t*>(w + p.off_offset);
    a.sorted_pair = reinterpret_cast<int32_t*>(w + p.off_sorted);
    a.pair_pos = reinterpret_cast<int32_t*>(w + p.off_pos);
    a.tile_rec = reinterpret_cast<int4*>(w + p.off_tile);
    a.n_tiles = reinterpret_cast<int32_t*>(w + p.off_ntiles);
    a.chunk_count = reinterpret_cast<int32_t*>(w + p.off_h);
    a.n_chunks = p.n_chunks;
    a.hbuf = reinterpret_cast<uint16_t*>(w + p.off_h);
    a.ybuf = reinterpret_cast<float*>(w + p.off_y);
    a.error_word = reinterpret_cast<uint32_t*>(c->ws + c->err_off);
    a.pairs_cap = p.pairs_cap; a.tiles_cap = p.tiles_cap; a.m_tile = p.m_tile; a.tiled = p.tiled; a.halves = p.halves; a.g1_xcd = p.g1_xcd; a.ksplit = p.ksplit; a.ksplit1 = p.ksplit1;
    a.ring1 = p.ring1; a.ring2 = p.ring2;
    a.part = a.ybuf;
    a.split_tiles = ~0u;                        // the plan knew the rows
    a.n_cus = uint32_t(std::max(c->n_cus, 1));
    a.tiled_waves = c->tune_tiled_waves;
    a.tiled_group = uint32_t(c->tune_tiled_group);
    a.tiled_persist = uint32_t(c->tune_tiled_persist);
    HIPCHECK(launch_ffn(a, c->n_cus, stream, nullptr, nullptr, false, c->profiling ? ffn_span_hook : nullptr, c));
    return FLUXMOE_OK;
}

int fluxmoe_stream_copy(void* dst, const void* src, uint64_t bytes, uint32_t n_workgroups, void* stream) {
    if (!dst || !src) return set_error(FLUXMOE_EINVAL, "NULL argument");
    if ((uintptr_t(dst) | uintptr_t(src) | bytes) & 15) return set_error(FLUXMOE_EINVAL, "16-byte alignment required");
    if (n_workgroups == 0 || n_workgroups > (1u << 20)) return set_error(FLUXMOE_EINVAL, "bad n_workgroups");
    HIPCHECK(launch_stream_copy(dst, src, bytes, n_workgroups, static_cast<hipStream_t>(stream)));
    return FLUXMOE_OK;
}

int fluxmoe_stream_mix(void* dst, uint64_t dst_bytes, const void* src, uint64_t src_bytes, uint32_t out_bytes_small,
                       uint32_t waves_per_workgroup, uint32_t blocks_per_wave, uint32_t order, uint64_t* bytes_written,
                       void* stream) {
    if (!dst || !src) return set_error(FLUXMOE_EINVAL, "NULL argument");
    if ((uintptr_t(dst) | uintptr_t(src)) & 127) return set_error(FLUXMOE_EINVAL, "128-byte alignment required");
    if (out_bytes_small < 128 || out_bytes_small > 16384 || out_bytes_small % 128)
        return set_error(FLUXMOE_EINVAL, "out_bytes_small must be a multiple of 128 in [128, 16384]");
    if (waves_per_workgroup != 4 && waves_per_workgroup != 8 && waves_per_workgroup != 16)
        return set_error(FLUXMOE_EINVAL, "waves_per_workgroup must be 4, 8 or 16");
    if (blocks_per_wave == 0 || blocks_per_wave > 1024) return set_error(FLUXMOE_EINVAL, "bad blocks_per_wave");
    if (order > 2) return set_error(FLUXMOE_EINVAL, "order must be 0, 1 or 2");
    const uint64_t n_blocks = src_bytes / 4096;
    if (n_blocks == 0 || n_blocks > (1ull << 30)) return set_error(FLUXMOE_EINVAL, "src must hold 1 to 2^30 blocks of 4096 bytes");
    const uint64_t need = stream_mix_out_bytes(n_blocks, out_bytes_small);
    if (dst_bytes < need)
        return set_error(FLUXMOE_EINVAL, "dst holds %llu bytes, %llu blocks write %llu", (unsigned long long)dst_bytes,
                         (unsigned long long)n_blocks, (unsigned long long)need);
    const uint64_t per_wg = uint64_t(waves_per_workgroup) * blocks_per_wave;
    const uint64_t n_wg = (n_blocks + per_wg - 1) / per_wg;
    if (n_wg > (1u << 24)) return set_error(FLUXMOE_EINVAL, "too many workgroups (%llu)", (unsigned long long)n_wg);
    HIPCHECK(launch_stream_mix(dst, src, uint32_t(n_blocks), out_bytes_small, int(waves_per_workgroup), blocks_per_wave,
                               order, uint32_t(n_wg), static_cast<hipStream_t>(stream)));
    if (bytes_written) *bytes_written = need;
    return FLUXMOE_OK;
}

int fluxmoe_mfma_probe(const void* operands, float* out, uint32_t n_workgroups, uint32_t iters, void* stream) {
    if (!operands || !out) return set_error(FLUXMOE_EINVAL, "NULL argument");
    if ((uintptr_t(operands) & 15) || (uintptr_t(out) & 3)) return set_error(FLUXMOE_EINVAL, "operands must be 16-byte aligned");
    if (n_workgroups == 0 || n_workgroups > (1u << 16) || iters == 0) return set_error(FLUXMOE_EINVAL, "bad n_workgroups or iters");
    HIPCHECK(launch_mfma_probe(operands, out, n_workgroups, iters, static_cast<hipStream_t>(stream)));
    return FLUXMOE_OK;
}

int fluxmoe_profile_enable(fluxmoe_ctx* c, int on) {
    if (!c) return set_error(FLUXMOE_EINVAL, "ctx is NULL");
    c->profiling = on != 0;
    c->profile_mask = (on & 0x100) ? uint32_t(on & 0x1F) : 0x1Fu;
    return FLUXMOE_OK;
}

int fluxmoe_profile_collect(fluxmoe_ctx* c, double out_ms[FLUXMOE_PROFILE_KINDS],
                            uint32_t out_count[FLUXMOE_PROFILE_KINDS]) {
    if (!c || !out_ms || !out_count) return set_error(FLUXMOE_EINVAL, "NULL argument");
    for (int k = 0; k < FLUXMOE_PROFILE_KINDS; ++k) { out_ms[k] = 0; out_count[k] = 0; }
    for (auto& sp : c->spans) {
        HIPCHECK(hipEventSynchronize(sp.b));
        float ms = 0;
        HIPCHECK(hipEventElapsedTime(&ms, sp.a, sp.b));
        out_ms[sp.kind] += ms;
        out_count[sp.kind] += 1;
        (void)hipEventDestroy(sp.a);
        (void)hipEventDestroy(sp.b);
    }
    c->spans.clear();
    return FLUXMOE_OK;
}

int fluxmoe_device_errors(fluxmoe_ctx* c, uint32_t* out_flags) {
    if (!c || !out_flags) return set_error(FLUXMOE_EINVAL, "NULL argument");
    if (!c->arenas_bound) return set_error(FLUXMOE_ESTATE, "fluxmoe_bind_arenas has not been called");
    HIPCHECK(hipDeviceSynchronize());
    HIPCHECK(hipMemcpy(out_flags, c->ws + c->err_off, 4, hipMemcpyDeviceToHost));
    HIPCHECK(hipMemset(c->ws + c->err_off, 0, 4));
    return FLUXMOE_OK;
}

}  // extern "C"
