// Host side of libpgcm: the C ABI of include/pgcm.h — argument checks, which way a batch goes and how it
// is cut, descriptors and kernel launches.  No cipher arithmetic happens on the host.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <type_traits>

#include <chrono>
#include <mutex>
#include <new>
#include <vector>

#include "../../include/pgcm.h"
#include "pgcm_contexts.h"
#include "pgcm_host_ivs.h"
#include "pgcm_kernels.h"
#include "pgcm_one_launch.h"
#include "pgcm_routes.h"
#include "pgcm_spans.h"

using namespace pgcm;

namespace {

thread_local int g_last_hip_error = 0;

inline bool hip_failed(hipError_t e) {
    if (e == hipSuccess) return false;
    g_last_hip_error = (int)e;
    return true;
}

#define PGCM_HIP(call)                             \
    do {                                           \
        if (hip_failed(call)) return PGCM_ERR_HIP; \
    } while (0)

// descriptor staging buffers a context uses in turn; a buffer is free again once the batch that
// used it has ended on its stream, so this is how many batches the host may run ahead of the GPU
constexpr int kStages = 4;
constexpr uint32_t kTimingRing = 256;
// limits of the entry point that allocates nothing (pgcm_encrypt_batch_static)
constexpr size_t kScratchBytes = PGCM_STATIC_WORKSPACE_BYTES;
constexpr size_t kFixedMaxChunks = PGCM_STATIC_MAX_CHUNKS;
constexpr int kMaxDevices = 64;
// a fold level with at most this many items (one workgroup each fits the chip at once) is folded
// by the tree kernel
constexpr uint32_t kFoldTreeMaxItems = 256;

// Per-chunk schedule: units are counted back from the chunk's end, so that every unit but the
// first is full and all row boundaries line up with the end of the chunk.
struct UnitPlan {
    uint32_t nunits, first_blocks;
};

inline UnitPlan plan_chunk(uint64_t len, uint32_t unit_power) {
    uint64_t nblk = (len + 15) / 16;
    UnitPlan p{0, 0};
    if (nblk == 0) return p;
    uint64_t nunits = (nblk + ((uint64_t)1 << unit_power) - 1) >> unit_power;
    p.nunits = (uint32_t)nunits;
    p.first_blocks = (uint32_t)(nblk - ((nunits - 1) << unit_power));
    return p;
}

// Partial sets of a chunk are folded kFan at a time until at most kFan remain for the final
// step.  Returns the number of fold levels and, per level, the number of sets it produces.
// More than kMaxLevels levels (only possible when a small unit is forced on a huge chunk) is
// reported as kMaxLevels + 1 with nothing written past the array.
inline uint32_t fold_levels(uint32_t nunits, uint32_t out_counts[kMaxLevels]) {
    uint32_t levels = 0, c = nunits;
    while (c > kFan) {
        if (levels == kMaxLevels) return kMaxLevels + 1;
        c = (c + kFan - 1) / kFan;
        out_counts[levels++] = c;
    }
    return levels;
}

// Unit size of a batch: the smallest, from one row up, with which the batch has at most
// wave_slots units (the wavefronts the device holds at once: sixteen per compute unit), so that
// every unit gets a wavefront of its own at once; kUnitPower and the dynamic schedule when even
// that leaves more.  (Larger units that would again give every
// wavefront exactly one unit, e.g. a whole 320 KiB block each for 4096 of them, can be forced but
// are never chosen: wavefronts do not all run at the same speed, and a launch that cannot hand
// the slow ones less work ends when its slowest wavefront does.)  `order` as for run_batch.
inline uint32_t choose_unit_power(size_t n, const uint32_t* order, const uint64_t* len,
                                  uint32_t wave_slots) {
    constexpr uint32_t kChoices = kUnitPower - kMinUnitPower + 1;
    uint64_t units[kChoices] = {};
    for (size_t k = 0; k < n; ++k) {
        const uint64_t l = len[order ? order[k] : k];
        if (l > PGCM_MAX_CHUNK_BYTES) return kUnitPower;  // rejected later
        const uint64_t nblk = (l + 15) / 16;
        for (uint32_t c = 0; c < kChoices; ++c) {
            const uint32_t u = kMinUnitPower + c;
            units[c] += (nblk + ((uint64_t)1 << u) - 1) >> u;
        }
        if (units[kChoices - 1] > wave_slots) return kUnitPower;
    }
    for (uint32_t c = 0; c < kChoices; ++c)
        if (units[c] <= wave_slots) return kMinUnitPower + c;
    return kUnitPower;
}

}  // namespace

namespace {

struct KeptBuffer {
    uint8_t* p;
    size_t bytes;
    bool host;  // pinned host memory; otherwise device memory
};

// What one batch in flight needs besides the key's tables: pinned staging buffers for the
// descriptors the host writes, and the device workspace the kernels of the batch share.  Batches
// that use one context are ordered by the stream the context is bound to, which is what makes
// reusing its buffers from batch to batch safe; batches on different streams (or from different
// host threads) take different contexts.
struct Context : Binding {
    bool growable = true;   // false: the buffers are fixed and a batch that needs more is refused
    uint8_t* stage[kStages] = {};
    size_t stage_cap[kStages] = {};
    hipEvent_t stage_done[kStages] = {};  // end of the batch that last used the buffer
    bool stage_used[kStages] = {};
    unsigned long long stage_capture[kStages] = {};  // fixed buffers: the capture that last took it
    int next_stage = 0;
    // device workspace: descriptors, unit maps, fold lists, unit counter, per-chunk E_K(J0),
    // partial sets; or arrival slots, then descriptors
    uint8_t* work = nullptr;
    size_t work_cap = 0;
    uint32_t* counter_at = nullptr;  // where the unit counter was last known to be zero
    bool counter_dirty = true;
    size_t clean_slots = 0;  // so many ArriveSlots at the start of `work` are zero
    // A batch of its was captured into a graph, whose replays may come between any two other batches:
    // nothing is taken for clean from one batch to the next any more, the context keeps its stream,
    // and what a replay reads or writes is kept until the key is freed.
    bool captured = false;
    std::vector<KeptBuffer> graph_buffers;
    SpanScratch scratch;     // of the call that is using the context
    uint64_t allocations = 0;  // times a batch or pgcm_reserve had to get any of these more room
    // stage whose event marks the end of its most recent batch, unless nothing does
    int last_stage = -1;
    bool left_no_mark = false;
};

}  // namespace

struct pgcm_key {
    int device = -1;
    int num_cu = 0;
    uint32_t wave_slots = kWaveSlots;  // wavefronts the device holds at once: 16 per CU
    int rounds = 0;  // 10, 12 or 14
    uint32_t forced_unit_power = 0;  // 0: chosen per batch
    bool one_launch = true;          // batches of few chunks that do not fill the chip: one kernel
    bool matrix_hash = false;        // unit kernel: GHASH row multiplication on the matrix cores
    KeyTables* tables = nullptr;  // device
    std::mutex mu;                 // guards `contexts` and the binding fields of each context
    std::vector<Context*> contexts;
    uint64_t use_tick = 0;
    ShortStreams short_streams;  // by `mu` as well
    ArriveSlot (*short_slots)[kSwapChunkGroups] = nullptr;  // device: their areas, behind the tables
    // the context of the entry point that allocates nothing: fixed staging buffers, and the
    // device's static scratch array as workspace
    Context fixed;
    bool fixed_used = false;
    // optional timing of the kernel that touches the payload (pgcm_set_timing):
    // a ring of event pairs, one pair per timed launch, so that a run of batches can be timed
    // without a host wait in between
    bool timing = false;
    uint64_t timed = 0;  // launches timed since timing was switched on
    hipEvent_t bulk_start[kTimingRing] = {}, bulk_stop[kTimingRing] = {};
};

// Device workspace of the entry point that allocates nothing: one array per GPU, held from the
// moment the library is loaded until the process ends, shared by every such call on that GPU.
// Host code must never pass this name to a kernel: the address the device sees comes from
// hipGetSymbolAddress (scratch_of_device) and is what the kernels get.
static __device__ __align__(256) uint8_t scratch[kScratchBytes];

namespace {

std::mutex g_scratch_mu;
uint8_t* g_scratch_ptr[kMaxDevices] = {};

// Address of `scratch` on `device`, which must be the current device; looked up once per device.
int scratch_of_device(int device, uint8_t** out) {
    if (device < 0 || device >= kMaxDevices) return PGCM_ERR_ARG;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[device] == nullptr) {
        void* p = nullptr;
        PGCM_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (p == nullptr) return PGCM_ERR_HIP;
        g_scratch_ptr[device] = static_cast<uint8_t*>(p);
    }
    *out = g_scratch_ptr[device];
    return PGCM_OK;
}

int create_stage_events(Context* c) {
    for (int s = 0; s < kStages; ++s)
        PGCM_HIP(hipEventCreateWithFlags(&c->stage_done[s], hipEventDisableTiming));
    return PGCM_OK;
}

void destroy_context(Context* c, bool wipe_work) {
    for (const KeptBuffer& b : c->graph_buffers) {
        if (b.host) {
            memset(b.p, 0, b.bytes);
            (void)hipHostFree(b.p);
        } else {
            if (wipe_work) (void)hipMemset(b.p, 0, b.bytes);
            (void)hipFree(b.p);
        }
    }
    if (c->work && c->growable) {
        // the workspace holds key-dependent values (tag masks, partial hashes)
        if (wipe_work) (void)hipMemset(c->work, 0, c->work_cap);
        (void)hipFree(c->work);
    }
    for (int s = 0; s < kStages; ++s) {
        if (c->stage[s]) {
            memset(c->stage[s], 0, c->stage_cap[s]);
            (void)hipHostFree(c->stage[s]);
        }
        if (c->stage_done[s]) (void)hipEventDestroy(c->stage_done[s]);
    }
}

// Makes stage s of the context free (waits for the batch that last used it) and at least `bytes`
// large.  capture: the one under way, or 0; it cannot have the same buffer twice.
int ensure_stage(Context* c, int s, size_t bytes, unsigned long long capture = 0) {
    if (capture != 0 && c->stage_capture[s] == capture) return PGCM_ERR_CAPACITY;
    if (c->stage_used[s]) {
        PGCM_HIP(hipEventSynchronize(c->stage_done[s]));
        c->stage_used[s] = false;
    }
    if (c->stage_cap[s] >= bytes) return PGCM_OK;
    if (!c->growable) return PGCM_ERR_CAPACITY;
    if (c->stage[s]) {
        PGCM_HIP(hipHostFree(c->stage[s]));
        c->stage[s] = nullptr;
        c->stage_cap[s] = 0;
    }
    size_t cap = bytes + bytes / 2 + 4096;
    void* p = nullptr;
    if (hip_failed(hipHostMalloc(&p, cap, hipHostMallocDefault))) return PGCM_ERR_NOMEM;
    c->stage[s] = (uint8_t*)p;
    c->stage_cap[s] = cap;
    ++c->allocations;
    return PGCM_OK;
}

int ensure_work(Context* c, size_t bytes, hipStream_t stream) {
    if (c->work_cap >= bytes) return PGCM_OK;
    if (!c->growable) return PGCM_ERR_CAPACITY;
    if (c->work) {
        if (c->captured) {
            try {
                c->graph_buffers.push_back(KeptBuffer{c->work, c->work_cap, false});
            } catch (const std::bad_alloc&) {
                return PGCM_ERR_NOMEM;
            }
        } else {
            // earlier batches on this stream may still read the old workspace
            PGCM_HIP(hipStreamSynchronize(stream));
            PGCM_HIP(hipFree(c->work));
        }
        c->work = nullptr;
        c->work_cap = 0;
    }
    c->counter_at = nullptr;  // new memory holds anything, even if it lands at the old address
    c->clean_slots = 0;
    size_t cap = bytes + bytes / 2 + 65536;
    void* p = nullptr;
    if (hip_failed(hipMalloc(&p, cap))) return PGCM_ERR_NOMEM;
    c->work = (uint8_t*)p;
    c->work_cap = cap;
    ++c->allocations;
    return PGCM_OK;
}

void release_context(pgcm_key* key, Context* c) {
    if (c == &key->fixed) return;
    std::lock_guard<std::mutex> lock(key->mu);
    leave_call(c, c->captured, c->left_no_mark);
}

// The context a batch on `stream` runs with (pick_context).
int acquire_context(pgcm_key* key, hipStream_t stream, Context** out) {
    std::unique_lock<std::mutex> lock(key->mu);
    bool must_wait = false;
    // (A context that pgcm_reserve has bound and no batch has used yet is left for its stream.)
    auto ended = [](const Context* c) {
        if (c->last_stage < 0) return false;
        if (hipEventQuery(c->stage_done[c->last_stage]) == hipSuccess) return true;
        (void)hipGetLastError();  // "not ready" is not an error of this call
        return false;
    };
    Context* pick = pick_context(key->contexts, stream, ended, &must_wait);
    must_wait = must_wait && pick->last_stage >= 0;
    if (pick == nullptr) {
        Context* c = new (std::nothrow) Context();
        if (c == nullptr) return PGCM_ERR_NOMEM;
        int rc = create_stage_events(c);
        if (rc == PGCM_OK) {
            try {
                key->contexts.push_back(c);
            } catch (const std::bad_alloc&) {
                rc = PGCM_ERR_NOMEM;
            }
        }
        if (rc != PGCM_OK) {
            destroy_context(c, false);
            delete c;
            return rc;
        }
        pick = c;
    }
    enter_call(key->contexts, pick, stream, ++key->use_tick);
    lock.unlock();
    if (pick->bound && pick->stream != stream) {
        // re-binding: everything it enqueued on its old stream must have ended
        if (must_wait && hip_failed(hipEventSynchronize(pick->stage_done[pick->last_stage]))) {
            release_context(key, pick);
            return PGCM_ERR_HIP;
        }
        for (int s = 0; s < kStages; ++s) pick->stage_used[s] = false;
    }
    pick->stream = stream;
    *out = pick;
    return PGCM_OK;
}

// The event that marks the end of a batch is attached to the batch's last kernel: the kernel's own
// completion signal serves, where a recorded event is a packet of its own that the next kernel
// waits behind (2.8 us per call between back-to-back kernels of 5 us; 0.1 us this way).  A stream
// that is being captured into a graph takes no such launch; nothing waits for a captured batch
// (end_of_batch).
template <class... P, class... A>
void launch_last(void (*kernel)(P...), dim3 grid, dim3 block, hipStream_t stream, bool capturing,
                 hipEvent_t done, A... args) {
    if (capturing)
        hipLaunchKernelGGL(kernel, grid, block, 0, stream, P(args)...);
    else
        hipExtLaunchKernelGGL(kernel, grid, block, 0, stream, nullptr, done, 0, P(args)...);
}

// The end of a batch whose last kernel was enqueued with stage s's event.  staged: it reads the staging
// buffer as well.  A captured batch has not run, and its replays read the buffer whenever they come:
// the buffer goes to the graph.  (The fixed context has no other; its buffers are used in turn again.)
// marked: it had that event.
int end_of_batch(Context* c, int s, unsigned long long capture, bool staged, bool marked = true) {
    c->bound = true;
    if (staged) c->next_stage = (s + 1) % kStages;
    if (capture == 0) {
        if (staged) c->stage_used[s] = true;
        if (marked) c->last_stage = s;
        c->left_no_mark = !marked;
        return PGCM_OK;
    }
    c->captured = true;
    c->clean_slots = 0;
    c->counter_at = nullptr;
    if (staged && !c->growable) c->stage_capture[s] = capture;
    if (staged && c->growable) {
        try {
            c->graph_buffers.push_back(KeptBuffer{c->stage[s], c->stage_cap[s], true});
        } catch (const std::bad_alloc&) {
            return PGCM_ERR_NOMEM;
        }
        c->stage[s] = nullptr;
        c->stage_cap[s] = 0;
        c->stage_used[s] = false;
    }
    return PGCM_OK;
}

constexpr size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// the kernels that run the cipher are compiled once per round count
template <bool kDecrypt, bool kMatrixHash, class... Args>
void launch_bulk_rounds(int rounds, dim3 grid, hipStream_t stream, Args... args) {
    if (rounds == 10)
        hipLaunchKernelGGL((bulk_kernel<kDecrypt, 10, kMatrixHash>), grid, dim3(kGroupThreads), 0,
                           stream, args...);
    else if (rounds == 12)
        hipLaunchKernelGGL((bulk_kernel<kDecrypt, 12, kMatrixHash>), grid, dim3(kGroupThreads), 0,
                           stream, args...);
    else
        hipLaunchKernelGGL((bulk_kernel<kDecrypt, 14, kMatrixHash>), grid, dim3(kGroupThreads), 0,
                           stream, args...);
}

// ... and once per engine of the row hash (matrix cores or LDS tables)
template <bool kDecrypt, class... Args>
void launch_bulk(int rounds, bool matrix_hash, dim3 grid, hipStream_t stream, Args... args) {
    if (matrix_hash)
        launch_bulk_rounds<kDecrypt, true>(rounds, grid, stream, args...);
    else
        launch_bulk_rounds<kDecrypt, false>(rounds, grid, stream, args...);
}

// many chunks of one row: a wavefront per chunk
template <bool kDecrypt, class... Args>
void launch_small(int rounds, uint32_t nchunks, hipStream_t stream, bool capturing, hipEvent_t done,
                  Args... args) {
    auto* kernel = rounds == 10   ? small_kernel<kDecrypt, 10>
                   : rounds == 12 ? small_kernel<kDecrypt, 12>
                                  : small_kernel<kDecrypt, 14>;
    launch_last(kernel, dim3((nchunks + kSmallChunksPerGroup - 1) / kSmallChunksPerGroup),
                dim3(kSmallChunksPerGroup * 64), stream, capturing, done, args...);
}

// The caller's arrays of one batch call.  `order` (may be null) picks the batch's chunks out of
// them: chunk k of the batch is the caller's chunk order[k]; null means 0, 1, .., n - 1.
struct BatchArgs {
    bool decrypt;
    size_t n;
    const uint32_t* order;
    const uint8_t* ivs;
    uint32_t iv_len;
    const void* const* aad;
    const uint32_t* aad_len;
    const void* const* src;
    const uint64_t* len;
    void* const* dst;
    uint8_t* tags;
    uint8_t* ok;
    hipStream_t stream;
    bool capturing = false;  // the stream is being captured into a graph
    unsigned long long capture = 0;  // ... which capture that is
    bool fixed = false;  // run in the key's fixed context: allocate nothing, refuse what does not fit
    bool host_ivs = false;  // `ivs`, 96 bits each, is pinned memory whose contents stay as they are

    size_t at(size_t k) const { return order ? order[k] : k; }
};

// what must hold for the arrays of a batch as a whole
int check_batch(const BatchArgs& a) {
    if (a.iv_len == 0) return PGCM_ERR_ARG;  // GCM takes no empty IV
    if (a.n == 0) return PGCM_OK;
    if (a.ivs == nullptr || a.src == nullptr || a.len == nullptr || a.dst == nullptr ||
        a.tags == nullptr)
        return PGCM_ERR_ARG;
    if ((a.aad == nullptr) != (a.aad_len == nullptr)) return PGCM_ERR_ARG;
    if (a.decrypt && a.ok == nullptr) return PGCM_ERR_ARG;
    if (a.n > 0x7FFFFFFFull) return PGCM_ERR_ARG;
    return PGCM_OK;
}

// ... and for the caller's chunk i
inline int check_chunk(const BatchArgs& a, size_t i) {
    if (a.len[i] > PGCM_MAX_CHUNK_BYTES) return PGCM_ERR_LEN;
    if (a.len[i] != 0) {
        if (a.src[i] == nullptr || a.dst[i] == nullptr) return PGCM_ERR_ARG;
        if (((uintptr_t)a.src[i] | (uintptr_t)a.dst[i]) & 15) return PGCM_ERR_ALIGN;
    }
    if (a.aad_len != nullptr && a.aad_len[i] != 0 && a.aad[i] == nullptr) return PGCM_ERR_ARG;
    return PGCM_OK;
}

inline void describe_chunk(const BatchArgs& a, size_t i, ChunkDesc& d) {
    memset(&d, 0, sizeof(d));
    d.src = (const uint8_t*)a.src[i];
    d.dst = (uint8_t*)a.dst[i];
    d.len = a.len[i];
    d.aad_len = a.aad_len ? a.aad_len[i] : 0;
    d.aad = d.aad_len ? (const uint8_t*)a.aad[i] : nullptr;
    d.index = (uint32_t)i;
}

inline uint64_t span_rows(const BatchArgs& a, size_t i) {
    return pgcm::span_rows(a.len[i], a.aad_len ? a.aad_len[i] : 0);
}

// What decides which way a batch goes, found while every chunk is validated.
int survey_batch(const BatchArgs& a, BatchSurvey* out) {
    BatchSurvey v;
    for (size_t k = 0; k < a.n; ++k) {
        const size_t i = a.at(k);
        const int rc = check_chunk(a, i);
        if (rc != PGCM_OK) return rc;
        v.add(a.len[i], a.aad_len ? a.aad_len[i] : 0);
    }
    *out = v;
    return PGCM_OK;
}

// Sizes of a batch's schedule of units; filled by plan_batch.
struct BatchPlan {
    uint32_t unit_power;  // log2 of the blocks per unit
    uint32_t nunits;
    uint32_t nslots;      // partial sets: one per unit and one per fold output
    uint32_t fold_count[kMaxLevels], fold_first[kMaxLevels], nfold;
    uint32_t ncoarse;
};

// forced_unit_power: 0 = chosen for the batch; wave_slots: see choose_unit_power
int plan_batch(uint32_t forced_unit_power, uint32_t wave_slots, const BatchArgs& a,
               BatchPlan* plan) {
    plan->unit_power = forced_unit_power ? forced_unit_power
                                         : choose_unit_power(a.n, a.order, a.len, wave_slots);
    uint64_t nunits = 0, nslots = 0;
    uint64_t fold_items[kMaxLevels] = {0, 0, 0, 0};
    for (size_t k = 0; k < a.n; ++k) {
        const size_t i = a.at(k);
        const uint32_t nu = plan_chunk(a.len[i], plan->unit_power).nunits;
        uint32_t outs[kMaxLevels];
        const uint32_t levels = fold_levels(nu, outs);
        // a forced unit the chunk cannot be cut into: too many fold levels, or sets of the last
        // step further apart than the largest power of H with a table
        if (levels > kMaxLevels || plan->unit_power + kFanPower * levels >= kNumPowers)
            return PGCM_ERR_LEN;
        nunits += nu;
        nslots += nu;
        for (uint32_t l = 0; l < levels; ++l) {
            fold_items[l] += outs[l];
            nslots += outs[l];
        }
    }
    if (nslots > 0xFFFFFFF0ull / 64) return PGCM_ERR_ARG;  // set indices are 32-bit
    plan->nunits = (uint32_t)nunits;
    plan->nslots = (uint32_t)nslots;
    plan->nfold = 0;
    for (uint32_t l = 0; l < kMaxLevels; ++l) {
        plan->fold_count[l] = (uint32_t)fold_items[l];
        plan->fold_first[l] = plan->nfold;
        plan->nfold += plan->fold_count[l];
    }
    plan->ncoarse = (plan->nunits >> kCoarseShift) + 1;
    return PGCM_OK;
}

// Byte offsets of the regions of the device workspace.  The regions up to upload_bytes are
// written by the host into a staging buffer of the same layout and uploaded.
struct WorkLayout {
    size_t desc, ubase, coarse, fold, upload_bytes, counter, ekj0, j0, sets, bytes;
};

WorkLayout lay_out(const BatchArgs& a, const BatchPlan& p) {
    WorkLayout w;
    w.desc = 0;
    w.ubase = round_up(w.desc + sizeof(ChunkDesc) * a.n, 256);
    w.coarse = round_up(w.ubase + sizeof(uint32_t) * (a.n + 1), 256);
    w.fold = round_up(w.coarse + sizeof(uint32_t) * (size_t)p.ncoarse, 256);
    w.upload_bytes = round_up(w.fold + sizeof(FoldItem) * (size_t)p.nfold, 256);
    w.counter = w.upload_bytes;
    w.ekj0 = w.counter + 256;
    w.j0 = w.ekj0 + sizeof(Block) * a.n;  // pre-counter blocks: only for IVs not 96 bits long
    w.sets = round_up(w.j0 + (a.iv_len == 12 ? 0 : sizeof(Block) * a.n), 1024);
    w.bytes = w.sets + sizeof(Block) * 64 * (size_t)p.nslots;
    return w;
}

// Upper bounds of a batch's staging and workspace bytes, for any batch of at most n chunks with
// at most `bytes` bytes of payload in all.  False when the numbers are out of range.
bool worst_case_sizes(uint32_t forced_unit_power, uint32_t wave_slots, size_t n, uint64_t bytes,
                      size_t* stage_bytes, size_t* work_bytes) {
    // units: with the unit chosen per batch a batch either has at most wave_slots units or is cut
    // into full-size units, each chunk adding at most one short unit
    const uint32_t up = forced_unit_power ? forced_unit_power : kUnitPower;
    uint64_t units = (bytes >> (up + 4)) + n;
    if (!forced_unit_power && units < wave_slots) units = wave_slots;
    // every fold level leaves at most units / 32 + n sets; four levels
    const uint64_t folds = units / (kFan - 1) + kMaxLevels * (uint64_t)n + 1;
    const uint64_t slots = units + folds;
    if (slots > 0xFFFFFFF0ull / 64 || n > 0x7FFFFFFFull) return false;
    BatchArgs a{};
    a.n = n;
    a.iv_len = 16;  // any length but 12: room for the pre-counter blocks as well
    BatchPlan p{};
    p.nunits = (uint32_t)units;
    p.nslots = (uint32_t)slots;
    p.nfold = (uint32_t)folds;
    p.ncoarse = (p.nunits >> kCoarseShift) + 1;
    const WorkLayout w = lay_out(a, p);
    // the other paths stage descriptors only, of chunks or of workgroups
    const size_t small = sizeof(ChunkDesc) * n > sizeof(GroupDesc) * kSwapMaxGroups
                             ? sizeof(ChunkDesc) * n : sizeof(GroupDesc) * kSwapMaxGroups;
    *stage_bytes = w.upload_bytes > small ? w.upload_bytes : small;
    *work_bytes = w.bytes;
    return true;
}

// Staging bytes any batch can need that passes the fixed context's other limits: at most
// kFixedMaxChunks descriptors and unit-map entries, and a coarse map and fold list for at most
// kScratchBytes / 1024 partial sets.
constexpr size_t kFixedStageBytes = round_up(
    (sizeof(ChunkDesc) * kFixedMaxChunks + 256) + (4 * (kFixedMaxChunks + 1) + 256) +
        (4 * (kScratchBytes / 1024 / 16 + 1) + 256) +
        (sizeof(FoldItem) * (kScratchBytes / 1024) + 256),
    4096);  // the staging buffers are slices of one block: each must start aligned

// Descriptors, unit maps and fold lists of the batch, written into the staging buffer.
void fill_schedule(const BatchArgs& a, const BatchPlan& p, const WorkLayout& w, uint8_t* stage) {
    ChunkDesc* h_desc = reinterpret_cast<ChunkDesc*>(stage + w.desc);
    uint32_t* h_ubase = reinterpret_cast<uint32_t*>(stage + w.ubase);
    uint32_t* h_coarse = reinterpret_cast<uint32_t*>(stage + w.coarse);
    FoldItem* h_fold = reinterpret_cast<FoldItem*>(stage + w.fold);
    uint32_t unit = 0, slot = p.nunits, coarse_next = 0;
    uint32_t fold_fill[kMaxLevels] = {0, 0, 0, 0};
    for (size_t k = 0; k < a.n; ++k) {
        const size_t i = a.at(k);
        const UnitPlan up = plan_chunk(a.len[i], p.unit_power);
        ChunkDesc& d = h_desc[k];
        describe_chunk(a, i, d);
        d.unit_base = unit;
        d.nunits = up.nunits;
        d.first_blocks = up.first_blocks;
        h_ubase[k] = unit;
        // coarse map: for every 2^kCoarseShift-th unit, the chunk that holds it
        while (coarse_next < p.ncoarse &&
               ((uint64_t)coarse_next << kCoarseShift) < (uint64_t)unit + up.nunits)
            h_coarse[coarse_next++] = (uint32_t)k;
        // fold levels: groups of kFan sets counted back from the end, the first one short
        uint32_t base = unit, count = up.nunits, power = p.unit_power, level = 0;
        while (count > kFan) {
            const uint32_t groups = (count + kFan - 1) / kFan;
            const uint32_t first = count - (groups - 1) * kFan;
            FoldItem* items = h_fold + p.fold_first[level] + fold_fill[level];
            for (uint32_t g = 0; g < groups; ++g) {
                items[g].in_base = base + (g == 0 ? 0 : first + (g - 1) * kFan);
                items[g].in_count = g == 0 ? first : kFan;
                items[g].out_slot = slot + g;
                items[g].pad_ = 0;
            }
            fold_fill[level] += groups;
            base = slot;
            slot += groups;
            count = groups;
            power += kFanPower;
            ++level;
        }
        d.final_base = base;
        d.final_count = count;
        d.final_power = power;
        unit += up.nunits;
    }
    h_ubase[a.n] = unit;
    while (coarse_next < p.ncoarse) h_coarse[coarse_next++] = (uint32_t)a.n - 1;
}

int record_timing_start(pgcm_key* key, hipStream_t stream) {
    if (key->timing) PGCM_HIP(hipEventRecord(key->bulk_start[key->timed % kTimingRing], stream));
    return PGCM_OK;
}

int record_timing_stop(pgcm_key* key, hipStream_t stream) {
    if (key->timing) {
        PGCM_HIP(hipEventRecord(key->bulk_stop[key->timed % kTimingRing], stream));
        ++key->timed;
    }
    return PGCM_OK;
}

// Many chunks of one row: one kernel, descriptors read straight from the pinned staging buffer, no
// device workspace.
int run_small_batch(pgcm_key* key, Context* ctx, const BatchArgs& a) {
    const uint32_t nchunks = (uint32_t)a.n;
    const int s = ctx->next_stage;
    int rc = ensure_stage(ctx, s, sizeof(ChunkDesc) * a.n, a.capture);
    if (rc != PGCM_OK) return rc;
    ChunkDesc* h_desc = reinterpret_cast<ChunkDesc*>(ctx->stage[s]);
    for (size_t k = 0; k < a.n; ++k) describe_chunk(a, a.at(k), h_desc[k]);
    const KeyTables* kt = key->tables;
    rc = record_timing_start(key, a.stream);
    if (rc != PGCM_OK) return rc;
    if (a.decrypt)
        launch_small<true>(key->rounds, nchunks, a.stream, a.capturing, ctx->stage_done[s], kt, (const ChunkDesc*)h_desc,
                           nchunks, a.ivs, a.iv_len, a.tags, a.ok);
    else
        launch_small<false>(key->rounds, nchunks, a.stream, a.capturing, ctx->stage_done[s], kt, (const ChunkDesc*)h_desc,
                            nchunks, a.ivs, a.iv_len, a.tags, (uint8_t*)nullptr);
    // from here on the stream will read the staging buffer: mark its end even if a later call
    // fails, so that the buffer is not rewritten under a running kernel
    const int rc_end = end_of_batch(ctx, s, a.capture, true);
    rc = record_timing_stop(key, a.stream);
    if (rc != PGCM_OK) return rc;
    PGCM_HIP(hipGetLastError());
    return rc_end;
}

// A key's device memory.
struct KeyMemory {
    KeyTables tables;
    ArriveSlot short_slots[kShortStreams][kSwapChunkGroups];
};

// The slots for short chunks in so many workgroups on this stream, or null.  (hipStreamPerThread names a
// stream of every thread.)
ArriveSlot* short_slots(pgcm_key* key, hipStream_t stream, uint32_t groups) {
    if (stream == hipStreamPerThread || groups > kSwapChunkGroups) return nullptr;
    std::lock_guard<std::mutex> lock(key->mu);
    const size_t area = key->short_streams.area_of(stream);
    return area < kShortStreams ? key->short_slots[area] : nullptr;
}

// Workspace of the one-launch path: a slot per workgroup.
constexpr size_t kSwapWorkBytes = sizeof(ArriveSlot) * kSwapMaxGroups;

// Makes the first n slots of the workspace zero.  Every batch leaves them zero; they
// need clearing when the workspace is new, was used by a batch with units, or is shared between
// keys, and in a graph, before whose replays any of that may happen, as well as wherever a replay may
// have come in between.
void use_slots(Context* ctx, size_t n, hipStream_t stream, bool capturing) {
    const bool trusted = ctx->growable && !capturing && !ctx->captured;
    if (ctx->clean_slots < n || !trusted) {
        const uint32_t n_clear = (uint32_t)(n * (sizeof(ArriveSlot) / 16));
        const uint32_t groups = (n_clear + 255) / 256;
        hipLaunchKernelGGL(upload_kernel, dim3(groups < 1024 ? groups : 1024), dim3(256), 0, stream,
                           (uint4*)nullptr, (const uint4*)nullptr, 0u,
                           reinterpret_cast<uint4*>(ctx->work), n_clear);
        if (trusted && ctx->clean_slots < n) ctx->clean_slots = n;
    }
    ctx->counter_at = nullptr;  // the unit counter of other batches may lie under them
}

// A batch in one launch, its chunks described by `args` or, in swap_kernel and if that is not null, by `staged`.
template <class Args>
void launch_burst(const pgcm_key* key, const BatchArgs& a, const SwapShape& shape, hipEvent_t done, uint32_t nchunks,
                  const Args& args, ArriveSlot* slots) {
    const BurstKind kind = burst_kind(shape, (uint32_t)key->num_cu, a.decrypt);
    const bool more = kind == BurstKind::kWords;
    const dim3 grid(shape.groups), block(64u * ((1u << shape.wave_power) + more));
    const bool in_place = a.host_ivs && std::is_same_v<Args, ArgOne>;
    const SwapMeta meta = swap_meta(nchunks, shape.unit_power, shape.wave_power, shape.alone, a.order == nullptr,
                                    shape.groups, (uint32_t)key->rounds, in_place);
    auto burst = [&](auto of) {
        constexpr BurstKind kKind = decltype(of)::value;
        const bool long_iv = a.iv_len > kShortIvBytes;
        auto* kernel = long_iv ? burst_kernel<true, true, kKind, Args> : burst_kernel<true, false, kKind, Args>;
        if constexpr (kKind != BurstKind::kFoldApart)
            if (!a.decrypt)
                kernel = long_iv ? burst_kernel<false, true, kKind, Args> : burst_kernel<false, false, kKind, Args>;
        return kernel;
    };
    decltype(burst(std::integral_constant<BurstKind, BurstKind::kWords>{})) kernel = nullptr;
    switch (kind) {
        case BurstKind::kWords: kernel = burst(std::integral_constant<BurstKind, BurstKind::kWords>{}); break;
        case BurstKind::kFold: kernel = burst(std::integral_constant<BurstKind, BurstKind::kFold>{}); break;
        case BurstKind::kFoldApart: kernel = burst(std::integral_constant<BurstKind, BurstKind::kFoldApart>{}); break;
        case BurstKind::kSweep: kernel = burst(std::integral_constant<BurstKind, BurstKind::kSweep>{}); break;
        case BurstKind::kFoldShared:
        case BurstKind::kWordsShared:
            if constexpr (!std::is_same_v<Args, ArgOne>)
                kernel = kind == BurstKind::kFoldShared
                             ? burst(std::integral_constant<BurstKind, BurstKind::kFoldShared>{})
                             : burst(std::integral_constant<BurstKind, BurstKind::kWordsShared>{});
            break;
    }
    // one chunk: its place in the caller's arrays is in the pointers
    const size_t first = std::is_same_v<Args, ArgOne> ? a.at(0) : 0;
    const uint8_t* ivs = a.ivs + first * a.iv_len;
    uint32_t iv_len = a.iv_len;
    if (in_place) {
        uint64_t words;
        memcpy(&iv_len, ivs + 8, 4);
        memcpy(&words, ivs, 8);
        ivs = reinterpret_cast<const uint8_t*>(words);
    }
    launch_last(kernel, grid, block, a.stream, a.capturing, done, (const KeyTables*)key->tables, ivs, iv_len, meta,
                slots, a.tags + 16 * first, a.ok != nullptr ? a.ok + first : nullptr, args);
}
void launch_swap(const pgcm_key* key, const BatchArgs& a, const SwapShape& shape, hipEvent_t done,
                 const ArgBatch& batch, const GroupDesc* staged, ArriveSlot* slots) {
    const uint32_t more = shape.wave_power < 4;  // a wavefront beyond those with units
    const dim3 grid(shape.groups), block(64u * ((1u << shape.wave_power) + more));
    const KeyTables* kt = key->tables;
    const SwapMeta meta = swap_meta(staged ? 0 : (uint32_t)a.n, shape.unit_power, shape.wave_power,
                                    shape.alone, a.order == nullptr, shape.groups,
                                    (uint32_t)key->rounds);
    auto* const swap = key->rounds == 10   ? (a.decrypt ? swap_kernel<true, 10> : swap_kernel<false, 10>)
                       : key->rounds == 12 ? (a.decrypt ? swap_kernel<true, 12> : swap_kernel<false, 12>)
                                           : (a.decrypt ? swap_kernel<true, 14> : swap_kernel<false, 14>);
    launch_last(swap, grid, block, a.stream, a.capturing, done, kt, a.ivs, a.iv_len, meta, slots, a.tags, a.ok,
                staged, batch);
}

// A batch of few chunks that does not fill the chip: one kernel.  Up to kArgChunks chunks travel as
// its arguments, nothing staged; when moreover every chunk has one workgroup, which needs no
// slots, or `slots` are given, the call needs no context at all (ctx is null).
int run_one_launch(pgcm_key* key, Context* ctx, const BatchArgs& a, const SwapShape& shape, ArriveSlot* slots) {
    const bool one = shape.burst && a.n == 1, in_args = a.n <= kArgChunks;
    ArgOne only;
    ArgBatch batch;
    GroupDesc* h_groups = nullptr;
    int s = 0;
    if (ctx != nullptr) s = ctx->next_stage;
    if (!in_args) {
        const int rc = ensure_stage(ctx, s, sizeof(GroupDesc) * shape.groups, a.capture);
        if (rc != PGCM_OK) return rc;
        h_groups = reinterpret_cast<GroupDesc*>(ctx->stage[s]);
    }
    auto describe = [&](size_t i) {
        ArgChunk c;
        c.src = (const uint8_t*)a.src[i];
        c.dst = (uint8_t*)a.dst[i];
        c.len = a.len[i];
        c.aad_len = a.aad_len ? a.aad_len[i] : 0;
        c.aad = c.aad_len ? (const uint8_t*)a.aad[i] : nullptr;
        c.index = (uint32_t)i;
        return c;
    };
    if (one) {
        only.c = describe(a.at(0));
    } else {
        if (in_args || !shape.burst) batch = ArgBatch{};  // (it goes out whole)
        const ShapeBatch lens{a.n, a.order, a.aad_len, a.len};
        uint32_t groups = 0;
        for (size_t k = 0; k < a.n; ++k) {
            const size_t i = a.at(k);
            const ArgChunk c = describe(i);
            const uint32_t of_chunk =
                !shape.burst  ? swap_groups(lens, i, shape.unit_power, shape.wave_power)
                : shape.alone ? 1
                              : (uint32_t)burst_groups(burst_passes(burst_blocks(lens, i), shape.wave_power),
                                                       shape.unit_power, shape.spare);
            if (in_args) {
                batch.c[k] = c;
                batch.group_base[k] = groups;
            } else {
                for (uint32_t g = 0; g < of_chunk; ++g)
                    h_groups[groups + g] = GroupDesc{c, groups, of_chunk};
            }
            groups += of_chunk;
        }
        if (in_args) batch.group_base[a.n] = groups;
    }
    if (!shape.alone && slots == nullptr) {
        const int rc = ensure_work(ctx, kSwapWorkBytes, a.stream);
        if (rc != PGCM_OK) return rc;
        use_slots(ctx, shape.groups, a.stream, a.capturing);
        slots = reinterpret_cast<ArriveSlot*>(ctx->work);
    }
    int rc_timing = record_timing_start(key, a.stream);
    // Where no staging buffer is used but the workspace is, the batch's end is marked on the event
    // of the stage whose turn it is, without taking the turn, or not at all.  (If that event still
    // guards an earlier batch's staging buffer, that batch ends before this one on the same stream, so
    // using it again only moves the guard later.)
    const bool marked = ctx != nullptr && !(in_args && ctx->quiet);
    const hipEvent_t done = marked ? ctx->stage_done[s] : nullptr;
    if (!shape.burst)
        launch_swap(key, a, shape, done, batch, h_groups, slots);
    else if (one)
        launch_burst(key, a, shape, done, 1, only, slots);
    else if (in_args)
        launch_burst(key, a, shape, done, (uint32_t)a.n, batch, slots);
    else
        launch_burst(key, a, shape, done, 0, ArgStaged{h_groups}, slots);
    if (rc_timing == PGCM_OK) rc_timing = record_timing_stop(key, a.stream);
    int rc_end = PGCM_OK;
    if (!in_args) {
        rc_end = end_of_batch(ctx, s, a.capture, true);
    } else if (ctx != nullptr) {
        rc_end = end_of_batch(ctx, s, a.capture, false, marked);
    }
    if (rc_timing != PGCM_OK) return rc_timing;
    if (hip_failed(hipGetLastError())) {
        if (ctx != nullptr) ctx->clean_slots = 0;
        return PGCM_ERR_HIP;
    }
    return rc_end;
}

// The kernels of one batch that goes through the unit schedule, enqueued with context `ctx`.
int run_unit_batch(pgcm_key* key, Context* ctx, const BatchArgs& a, const BatchPlan& p) {
    const uint32_t nchunks = (uint32_t)a.n;
    const WorkLayout w = lay_out(a, p);
    if (!ctx->growable && (a.n > kFixedMaxChunks || w.bytes > ctx->work_cap))
        return PGCM_ERR_CAPACITY;
    const int s = ctx->next_stage;
    int rc = ensure_stage(ctx, s, w.upload_bytes, a.capture);
    if (rc != PGCM_OK) return rc;
    rc = ensure_work(ctx, w.bytes, a.stream);
    if (rc != PGCM_OK) return rc;
    fill_schedule(a, p, w, ctx->stage[s]);
    ctx->clean_slots = 0;  // the descriptors land there
    uint32_t* d_counter = reinterpret_cast<uint32_t*>(ctx->work + w.counter);
    {
        // the unit counter is left at zero by the last kernel of every batch; it only needs
        // clearing when the workspace is new, the counter's place in it has moved, an earlier
        // batch was cut short, or the workspace is shared with other keys (the fixed context) or with
        // replays of a graph
        const bool clear = ctx->counter_at != d_counter || ctx->counter_dirty || !ctx->growable ||
                           ctx->captured || a.capturing;
        ctx->counter_at = d_counter;
        ctx->counter_dirty = true;
        const uint32_t n16 = (uint32_t)(w.upload_bytes / 16);
        uint32_t groups = (n16 + 255) / 256;
        if (groups > 1024) groups = 1024;
        hipLaunchKernelGGL(upload_kernel, dim3(groups), dim3(256), 0, a.stream,
                           reinterpret_cast<uint4*>(ctx->work),
                           reinterpret_cast<const uint4*>(ctx->stage[s]), n16,
                           reinterpret_cast<uint4*>(d_counter), clear ? 1u : 0u);
    }

    const KeyTables* kt = key->tables;
    const ChunkDesc* d_desc = reinterpret_cast<const ChunkDesc*>(ctx->work + w.desc);
    const uint32_t* d_ubase = reinterpret_cast<const uint32_t*>(ctx->work + w.ubase);
    const uint32_t* d_coarse = reinterpret_cast<const uint32_t*>(ctx->work + w.coarse);
    const FoldItem* d_fold = reinterpret_cast<const FoldItem*>(ctx->work + w.fold);
    Block* d_ekj0 = reinterpret_cast<Block*>(ctx->work + w.ekj0);
    Block* d_sets = reinterpret_cast<Block*>(ctx->work + w.sets);
    Block* d_j0 = a.iv_len == 12 ? nullptr : reinterpret_cast<Block*>(ctx->work + w.j0);
    if (d_j0 != nullptr)
        hipLaunchKernelGGL(j0_kernel, dim3((nchunks + 63) / 64), dim3(64), 0, a.stream, kt, d_desc,
                           a.ivs, a.iv_len, nchunks, d_j0);

    int rc_timing = PGCM_OK;
    if (p.nunits > 0) {
        uint32_t groups = (p.nunits + kWavesPerGroup - 1) / kWavesPerGroup;
        if (groups > (uint32_t)key->num_cu) groups = (uint32_t)key->num_cu;
        rc_timing = record_timing_start(key, a.stream);
        if (a.decrypt)
            launch_bulk<true>(key->rounds, key->matrix_hash, dim3(groups), a.stream, kt, d_desc,
                              d_ubase, d_coarse, p.nunits, p.unit_power, d_counter, a.ivs,
                              (const Block*)d_j0, d_ekj0, d_sets);
        else
            launch_bulk<false>(key->rounds, key->matrix_hash, dim3(groups), a.stream, kt, d_desc,
                               d_ubase, d_coarse, p.nunits, p.unit_power, d_counter, a.ivs,
                               (const Block*)d_j0, d_ekj0, d_sets);
        if (rc_timing == PGCM_OK) rc_timing = record_timing_stop(key, a.stream);
    }
    for (uint32_t l = 0; l < kMaxLevels; ++l) {
        if (p.fold_count[l] == 0) continue;
        const uint32_t power = p.unit_power + kFanPower * l;
        // few items: a workgroup each, folding as a tree; many: a wavefront each, as a chain
        if (p.fold_count[l] <= kFoldTreeMaxItems)
            hipLaunchKernelGGL(fold_tree_kernel, dim3(p.fold_count[l]), dim3(kFoldTreeWaves * 64),
                               0, a.stream, kt, d_fold + p.fold_first[l], power, d_sets);
        else
            hipLaunchKernelGGL(fold_kernel, dim3(p.fold_count[l]), dim3(64), 0, a.stream, kt,
                               d_fold + p.fold_first[l], power, d_sets);
    }
    // one wavefront per chunk; few chunks are spread over the compute units rather than packed
    // sixteen to a workgroup
    uint32_t per_group = (nchunks + (uint32_t)key->num_cu - 1) / (uint32_t)key->num_cu;
    if (per_group > kFinalWaves) per_group = kFinalWaves;
    const dim3 final_grid((nchunks + per_group - 1) / per_group);
    launch_last(a.decrypt ? final_kernel<true> : final_kernel<false>, final_grid,
                dim3(kFinalWaves * 64), a.stream, a.capturing, ctx->stage_done[s], kt, d_desc,
                nchunks, a.ivs, d_j0, d_ekj0, d_sets, a.tags, a.ok, p.unit_power, d_counter,
                per_group);
    // the stream now reads the staging buffer and the workspace: their end is marked whatever
    // else fails below
    const int rc_end = end_of_batch(ctx, s, a.capture, true);
    if (rc_timing != PGCM_OK) return rc_timing;
    PGCM_HIP(hipGetLastError());
    if (rc_end != PGCM_OK) return rc_end;
    ctx->counter_dirty = false;
    return PGCM_OK;
}

// ---- Spans (span_kernel) ----

// One batch in spans, of one key or of several: the context is that of the first.
int run_span_batch(Context* ctx, const BatchArgs& a, KeyPart* keys, size_t nkeys) {
    const uint32_t ngroups = deal_groups(keys, nkeys, (uint32_t)keys[0].key->num_cu);
    const size_t parts_at = span_parts_at(ngroups), most = span_image_bytes(a.n + ngroups, ngroups);
    const int s = ctx->next_stage;
    int rc = ensure_stage(ctx, s, most > kSpanHostBytes ? most : kSpanHostBytes);
    if (rc != PGCM_OK) return rc;
    // Each workgroup's list right behind its descriptor, to be read from host memory, if they are few and
    // none is longer than what is held of it (map_spans); otherwise uploaded, one list after the other.
    uint8_t* const stage = ctx->stage[s];
    uint8_t* image = stage;
    SpanPlan plan;
    SpanGroup* groups;
    SpanPart* all_parts;
    const size_t held = ctx->scratch.capacity();
    try {
        if (most <= kSpanHostBytes) {
            ctx->scratch.image.resize(kSpanHostBytes);
            image = ctx->scratch.image.data();
        }
        groups = reinterpret_cast<SpanGroup*>(image);
        all_parts = reinterpret_cast<SpanPart*>(image + parts_at);
        const SpanBatch b{a.n, a.order, a.aad, a.aad_len, a.src, a.len, a.dst};
        plan = plan_spans(b, keys, nkeys, ctx->scratch, groups, all_parts);
    } catch (const std::bad_alloc&) {
        return PGCM_ERR_NOMEM;
    }
    if (ctx->scratch.capacity() != held) ++ctx->allocations;
    SpanMap map;
    size_t packed = 0;
    uint32_t mapped = map_spans(keys, nkeys, groups, plan, &map, &packed);
    if (image == stage) mapped &= ~kSpanPlaced;
    const bool in_host = mapped & kSpanPlaced;
    const size_t bytes = in_host ? 0 : span_image_bytes(plan.nparts, ngroups);
    // the descriptors go behind every slot that is kept clean
    const size_t nslots = plan.nparts;
    const size_t behind =
        round_up(sizeof(ArriveSlot) * (nslots > ctx->clean_slots ? nslots : ctx->clean_slots), 256);
    rc = ensure_work(ctx, behind + bytes, a.stream);
    if (rc != PGCM_OK) return rc;
    use_slots(ctx, nslots, a.stream, a.capturing);
    const uint8_t* packets = stage;
    const SpanPart* parts = nullptr;
    if (in_host) {
        uint8_t* to = stage;
        for (uint32_t g = 0; g < ngroups; ++g) {
            const SpanGroup& d = groups[g];
            memcpy(to, &d, sizeof(d));
            memcpy(to + sizeof(d), all_parts + d.part, sizeof(SpanPart) * d.nparts);
            to += packet_bytes(d.nparts);
        }
    } else {
        if (image != stage) memcpy(stage, image, bytes);
        const uint32_t n16 = (uint32_t)(bytes / 16);
        hipLaunchKernelGGL(upload_kernel, dim3((n16 + 255) / 256 < 1024 ? (n16 + 255) / 256 : 1024),
                           dim3(256), 0, a.stream, reinterpret_cast<uint4*>(ctx->work + behind),
                           reinterpret_cast<const uint4*>(stage), n16, (uint4*)nullptr, 0u);
        packets = ctx->work + behind;
        parts = reinterpret_cast<const SpanPart*>(packets + parts_at);
    }
    // one pair of events per key object, which may be listed more than once
    auto timed_already = [&](size_t q) {
        if (keys[q].key->timing)
            for (size_t p = 0; p < q; ++p)
                if (keys[p].key == keys[q].key) return true;
        return false;
    };
    int rc_timing = PGCM_OK;
    for (size_t q = 0; q < nkeys && rc_timing == PGCM_OK; ++q)
        if (!timed_already(q)) rc_timing = record_timing_start(keys[q].key, a.stream);
    const bool long_iv = a.iv_len > kShortIvBytes;
    auto* const kernel = a.decrypt ? (long_iv ? span_kernel<true, true> : span_kernel<true, false>)
                                   : (long_iv ? span_kernel<false, true> : span_kernel<false, false>);
    launch_last(kernel, dim3(ngroups), dim3(kGroupThreads), a.stream, a.capturing, ctx->stage_done[s],
                (const KeyTables*)(nkeys == 1 ? keys[0].key->tables : nullptr), packets, parts,
                a.iv_len, mapped, a.ivs, reinterpret_cast<ArriveSlot*>(ctx->work), a.tags, a.ok, map);
    for (size_t q = 0; q < nkeys && rc_timing == PGCM_OK; ++q)
        if (!timed_already(q)) rc_timing = record_timing_stop(keys[q].key, a.stream);
    const int rc_end = end_of_batch(ctx, s, a.capture, true);
    if (hip_failed(hipGetLastError())) {
        ctx->clean_slots = 0;
        return PGCM_ERR_HIP;
    }
    return rc_timing != PGCM_OK ? rc_timing : rc_end;
}

int note_capture(BatchArgs& a) {
    if (a.stream != nullptr) {
        hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
        PGCM_HIP(hipStreamIsCapturing(a.stream, &status));
        a.capturing = status == hipStreamCaptureStatusActive;
        if (a.capturing) PGCM_HIP(hipStreamGetCaptureInfo(a.stream, &status, &a.capture));
    }
    return PGCM_OK;
}

RouteOptions route_options(const pgcm_key* key, bool fixed) {
    return RouteOptions{(uint32_t)key->num_cu, key->one_launch, key->matrix_hash, key->forced_unit_power, fixed,
                        false, false};
}

// One batch under one key: validate everything, choose the way it goes, pick a context unless it
// needs none, then enqueue its kernels on the stream.
int run_batch(pgcm_key* key, BatchArgs a) {
    if (key == nullptr || key->tables == nullptr) return PGCM_ERR_ARG;
    int rc = check_batch(a);
    if (rc != PGCM_OK || a.n == 0) return rc;
    BatchSurvey v;
    rc = survey_batch(a, &v);
    if (rc != PGCM_OK) return rc;
    // the units, unless they are not wanted anyway; nothing touched so far
    BatchPlan p{};
    RouteOptions options = route_options(key, a.fixed);
    if (!may_go_in_spans(options, v))
        rc = plan_batch(key->forced_unit_power, key->wave_slots, a, &p);
    if (rc != PGCM_OK) return rc;
    int cur_device = -1;
    PGCM_HIP(hipGetDevice(&cur_device));
    if (cur_device != key->device) return PGCM_ERR_ARG;  // the key lives on another GPU
    rc = note_capture(a);
    if (rc != PGCM_OK) return rc;
    const ShapeBatch lens{a.n, a.order, a.aad_len, a.len};
    SwapShape shape{};
    const bool short_args = v.all_small() && a.n <= kArgChunks;
    options.spread = short_args && !a.fixed && !a.capturing;
    if (v.all_small() && !short_args && !a.capturing) {
        std::lock_guard<std::mutex> lock(key->mu);
        options.clears_slots = a.fixed || clears_slots(key->contexts, a.stream);
    }
    Route route = route_batch(lens, options, v, &shape);
    ArriveSlot* slots = nullptr;
    if (short_args && route == Route::kOneLaunch && !shape.alone) {
        slots = short_slots(key, a.stream, shape.groups);
        options.spread = slots != nullptr;
        if (slots == nullptr) route = route_batch(lens, options, v, &shape);
    }
    if (a.fixed && a.n > kFixedMaxChunks) return PGCM_ERR_CAPACITY;
    const bool one_launch = route == Route::kOneLaunch;
    if (one_launch && (shape.alone || slots != nullptr) && a.n <= kArgChunks)
        return run_one_launch(key, nullptr, a, shape, slots);
    Context* ctx = nullptr;
    if (a.fixed) {
        ctx = &key->fixed;
        key->fixed_used = true;
    } else {
        rc = acquire_context(key, a.stream, &ctx);
        if (rc != PGCM_OK) return rc;
    }
    if (one_launch) {
        rc = run_one_launch(key, ctx, a, shape, nullptr);
    } else if (route == Route::kOneRow) {
        rc = run_small_batch(key, ctx, a);
    } else if (route == Route::kSpans) {
        KeyPart part{key, key->tables, (uint32_t)key->rounds, 0, a.n, v.rows, v.longest, 0};
        rc = run_span_batch(ctx, a, &part, 1);
    } else {
        rc = run_unit_batch(key, ctx, a, p);
    }
    release_context(key, ctx);
    return rc;
}

// The parts of several keys as one batch in spans, in a context of the first part's key.  (Nothing that
// is derived from the other keys outlives the batch in there: the kernel leaves its slots zero.)
int run_span_parts(BatchArgs a, KeyPart* parts, size_t nparts) {
    int rc = note_capture(a);
    if (rc != PGCM_OK) return rc;
    pgcm_key* const key = parts[0].key;
    Context* ctx = nullptr;
    rc = acquire_context(key, a.stream, &ctx);
    if (rc != PGCM_OK) return rc;
    rc = run_span_batch(ctx, a, parts, nparts);
    release_context(key, ctx);
    return rc;
}

// A batch whose chunks name their key: the chunks are grouped by key (keeping their order), and the
// keys' parts go in as few launches as share_launch allows, a part that does not go with others as
// a batch of its key, one after the other on the stream.
int run_batch_keys(pgcm_key* const* keys, size_t nkeys, const uint32_t* key_index,
                   const BatchArgs& all) {
    if (keys == nullptr || nkeys == 0 || nkeys > 0x7FFFFFFFull) return PGCM_ERR_ARG;
    int cur_device = -1;
    PGCM_HIP(hipGetDevice(&cur_device));
    for (size_t k = 0; k < nkeys; ++k)
        if (keys[k] == nullptr || keys[k]->tables == nullptr || keys[k]->device != cur_device)
            return PGCM_ERR_ARG;
    int rc = check_batch(all);
    if (rc != PGCM_OK || all.n == 0) return rc;
    if (key_index == nullptr) return PGCM_ERR_ARG;
    // every chunk is checked before anything is enqueued
    std::vector<KeyPart> parts;  // of each key; then of those with chunks, in the order they go in
    std::vector<size_t> keys_in_turn, alone, launches;  // launches: the first part of each, the end
    std::vector<uint32_t> fill, order;
    try {
        parts.resize(nkeys);
        for (size_t i = 0; i < all.n; ++i) {
            if (key_index[i] >= nkeys) return PGCM_ERR_ARG;
            rc = check_chunk(all, i);
            if (rc != PGCM_OK) return rc;
            KeyPart& part = parts[key_index[i]];
            ++part.n;
            part.rows += span_rows(all, i);
            if (all.len[i] > part.longest) part.longest = all.len[i];
        }
        const size_t num_cu = (size_t)keys[0]->num_cu;
        size_t n = 0;
        uint64_t rows = 0;
        for (size_t k = 0; k < nkeys; ++k) {
            const KeyPart& part = parts[k];
            if (part.n == 0) continue;
            if (!takes_spans(route_options(keys[k], false), part.rows, part.longest) ||
                !share_launch(1, part.n, part.rows, num_cu)) {
                alone.push_back(k);
                continue;
            }
            const size_t at = keys_in_turn.size();
            if (launches.empty() ||
                !share_launch(at - launches.back() + 1, n + part.n, rows + part.rows, num_cu)) {
                launches.push_back(at);
                n = 0, rows = 0;
            }
            n += part.n, rows += part.rows;
            keys_in_turn.push_back(k);
        }
        for (size_t k : alone) {
            launches.push_back(keys_in_turn.size());
            keys_in_turn.push_back(k);
        }
        launches.push_back(keys_in_turn.size());
        fill.resize(nkeys);
        std::vector<KeyPart> sorted;
        sorted.reserve(keys_in_turn.size());
        size_t first = 0;
        for (size_t k : keys_in_turn) {
            KeyPart part = parts[k];
            part.key = keys[k];
            part.tables = keys[k]->tables;
            part.rounds = (uint32_t)keys[k]->rounds;
            part.first = first;
            fill[k] = (uint32_t)first;
            first += part.n;
            sorted.push_back(part);
        }
        parts.swap(sorted);
        order.resize(all.n);
    } catch (const std::bad_alloc&) {
        return PGCM_ERR_NOMEM;
    }
    for (size_t i = 0; i < all.n; ++i) order[fill[key_index[i]]++] = (uint32_t)i;
    for (size_t l = 0; l + 1 < launches.size(); ++l) {
        KeyPart *const begin = parts.data() + launches[l], *const end = parts.data() + launches[l + 1];
        BatchArgs a = all;
        a.order = order.data() + begin->first;
        a.n = end[-1].first + end[-1].n - begin->first;
        if (end - begin == 1) {
            rc = run_batch(begin->key, a);
        } else {
            const size_t first = begin->first;
            for (KeyPart* part = begin; part < end; ++part) part->first -= first;
            rc = run_span_parts(a, begin, (size_t)(end - begin));
        }
        if (rc != PGCM_OK) return rc;
    }
    return PGCM_OK;
}

}  // namespace

namespace pgcm {

int encrypt_with_host_ivs(pgcm_key_t* key, size_t n, const uint8_t* ivs, const void* const* src, const uint64_t* len,
                          void* const* dst, uint8_t* tags, hipStream_t stream) {
    BatchArgs a{false, n, nullptr, ivs, 12, nullptr, nullptr, src, len, dst, tags, nullptr, stream};
    a.host_ivs = true;
    return run_batch(key, a);
}

int decrypt_with_host_ivs(pgcm_key_t* key, size_t n, const uint8_t* ivs, const void* const* src, const uint64_t* len,
                          void* const* dst, const uint8_t* tags, uint8_t* ok, hipStream_t stream) {
    BatchArgs a{true, n, nullptr, ivs, 12, nullptr, nullptr, src, len, dst, const_cast<uint8_t*>(tags), ok, stream};
    a.host_ivs = true;
    return run_batch(key, a);
}

}  // namespace pgcm

extern "C" {
#pragma GCC visibility push(default)

int pgcm_expand_key(const uint8_t key[32], void* hip_stream, pgcm_key_t** out) {
    return pgcm_expand_key_bytes(key, 32, hip_stream, out);
}

int pgcm_expand_key_bytes(const uint8_t* key, uint32_t key_bytes, void* hip_stream,
                          pgcm_key_t** out) {
    if (key == nullptr || out == nullptr) return PGCM_ERR_ARG;
    *out = nullptr;
    if (key_bytes != 16 && key_bytes != 24 && key_bytes != 32) return PGCM_ERR_ARG;
    pgcm_key* k = new (std::nothrow) pgcm_key();
    if (k == nullptr) return PGCM_ERR_NOMEM;
    hipStream_t stream = (hipStream_t)hip_stream;
    int rc = PGCM_OK;
    uint32_t* d_key = nullptr;
    do {
        if (hip_failed(hipGetDevice(&k->device))) { rc = PGCM_ERR_HIP; break; }
        if (hip_failed(hipDeviceGetAttribute(&k->num_cu, hipDeviceAttributeMultiprocessorCount,
                                             k->device))) { rc = PGCM_ERR_HIP; break; }
        if (k->num_cu < 1) k->num_cu = 1;
        KeyMemory* memory = nullptr;
        if (hip_failed(hipMalloc((void**)&memory, sizeof(KeyMemory)))) { rc = PGCM_ERR_NOMEM; break; }
        k->tables = &memory->tables;
        k->short_slots = memory->short_slots;
        if (hip_failed(hipMalloc((void**)&d_key, 32))) { rc = PGCM_ERR_NOMEM; break; }
        k->wave_slots = (uint32_t)k->num_cu * kWavesPerGroup;
        // the fixed context: one pinned block cut into the staging buffers, the device's static
        // scratch array as workspace; nothing of it ever grows
        k->fixed.growable = false;
        if ((rc = create_stage_events(&k->fixed)) != PGCM_OK) break;
        {
            void* p = nullptr;
            if (hip_failed(hipHostMalloc(&p, kStages * kFixedStageBytes, hipHostMallocDefault))) {
                rc = PGCM_ERR_NOMEM;
                break;
            }
            for (int s = 0; s < kStages; ++s) {
                k->fixed.stage[s] = static_cast<uint8_t*>(p) + (size_t)s * kFixedStageBytes;
                k->fixed.stage_cap[s] = kFixedStageBytes;
            }
        }
        if ((rc = scratch_of_device(k->device, &k->fixed.work)) != PGCM_OK) break;
        k->fixed.work_cap = kScratchBytes;
        // a pageable copy of at most 32 bytes: staged by the runtime, complete on return for this size
        if (hip_failed(hipMemcpyAsync(d_key, key, key_bytes, hipMemcpyHostToDevice, stream))) { rc = PGCM_ERR_HIP; break; }
        k->rounds = (int)(key_bytes / 4 + 6);
        hipLaunchKernelGGL(expand_key_kernel, dim3(1), dim3(1024), 0, stream, k->tables, d_key,
                           key_bytes / 4, reinterpret_cast<uint4*>(k->short_slots),
                           (uint32_t)(sizeof(KeyMemory::short_slots) / 16));
        if (hip_failed(hipGetLastError())) { rc = PGCM_ERR_HIP; break; }
        if (hip_failed(hipMemsetAsync(d_key, 0, 32, stream))) { rc = PGCM_ERR_HIP; break; }
        if (hip_failed(hipStreamSynchronize(stream))) { rc = PGCM_ERR_HIP; break; }
    } while (0);
    if (d_key) (void)hipFree(d_key);
    if (rc != PGCM_OK) {
        pgcm_free_key(k);
        return rc;
    }
    *out = k;
    return PGCM_OK;
}

void pgcm_free_key(pgcm_key_t* k) {
    if (k == nullptr) return;
    if (k->tables) {
        (void)hipMemset(k->tables, 0, sizeof(KeyMemory));
        (void)hipFree(k->tables);
    }
    for (Context* c : k->contexts) {
        destroy_context(c, true);
        delete c;
    }
    // the fixed context: its staging buffers are slices of one allocation, and its workspace is
    // the device's static array, which is wiped (it holds tag masks and partial hashes) but stays
    if (k->fixed.work && k->fixed_used) (void)hipMemset(k->fixed.work, 0, kScratchBytes);
    if (k->fixed.stage[0]) {
        memset(k->fixed.stage[0], 0, kStages * kFixedStageBytes);
        (void)hipHostFree(k->fixed.stage[0]);
    }
    for (int s = 0; s < kStages; ++s)
        if (k->fixed.stage_done[s]) (void)hipEventDestroy(k->fixed.stage_done[s]);
    for (uint32_t i = 0; i < kTimingRing; ++i) {
        if (k->bulk_start[i]) (void)hipEventDestroy(k->bulk_start[i]);
        if (k->bulk_stop[i]) (void)hipEventDestroy(k->bulk_stop[i]);
    }
    delete k;
}

int pgcm_encrypt_batch(pgcm_key_t* key, size_t n, const uint8_t* ivs, const void* const* aad,
                       const uint32_t* aad_len, const void* const* src, const uint64_t* len,
                       void* const* dst, uint8_t* tags, void* hip_stream) {
    return run_batch(key, BatchArgs{false, n, nullptr, ivs, 12, aad, aad_len, src, len, dst, tags,
                                    nullptr, (hipStream_t)hip_stream});
}

int pgcm_encrypt_batch_iv(pgcm_key_t* key, size_t n, const uint8_t* ivs, uint32_t iv_bytes,
                          const void* const* aad, const uint32_t* aad_len, const void* const* src,
                          const uint64_t* len, void* const* dst, uint8_t* tags, void* hip_stream) {
    return run_batch(key, BatchArgs{false, n, nullptr, ivs, iv_bytes, aad, aad_len, src, len, dst,
                                    tags, nullptr, (hipStream_t)hip_stream});
}

int pgcm_encrypt_batch_static(pgcm_key_t* key, size_t n, const uint8_t* ivs,
                              const void* const* aad, const uint32_t* aad_len,
                              const void* const* src, const uint64_t* len, void* const* dst,
                              uint8_t* tags, void* hip_stream) {
    BatchArgs a{false, n, nullptr, ivs, 12, aad, aad_len, src, len, dst, tags, nullptr,
                (hipStream_t)hip_stream};
    a.fixed = true;
    return run_batch(key, a);
}

int pgcm_reserve(pgcm_key_t* key, void* hip_stream, size_t n_max, uint64_t payload_bytes_max) {
    if (key == nullptr || key->tables == nullptr || n_max > 0x7FFFFFFFull) return PGCM_ERR_ARG;
    int cur_device = -1;
    PGCM_HIP(hipGetDevice(&cur_device));
    if (cur_device != key->device) return PGCM_ERR_ARG;
    size_t stage_bytes = 0, work_bytes = 0;
    if (!worst_case_sizes(key->forced_unit_power, key->wave_slots, n_max, payload_bytes_max,
                          &stage_bytes, &work_bytes))
        return PGCM_ERR_ARG;
    const hipStream_t stream = (hipStream_t)hip_stream;
    Context* ctx = nullptr;
    int rc = acquire_context(key, stream, &ctx);
    if (rc != PGCM_OK) return rc;
    // for whichever path such a batch takes: units (above), one launch, spans
    const size_t num_cu = (size_t)key->num_cu;
    const size_t clean = ctx->clean_slots > kSwapMaxGroups ? ctx->clean_slots : kSwapMaxGroups;
    const size_t span_stage = span_stage_bytes(n_max, num_cu);
    const size_t span_work = span_work_bytes(n_max, num_cu, clean);
    if (stage_bytes < span_stage) stage_bytes = span_stage;
    if (work_bytes < kSwapWorkBytes) work_bytes = kSwapWorkBytes;
    if (work_bytes < span_work) work_bytes = span_work;
    for (int s = 0; s < kStages && rc == PGCM_OK; ++s) rc = ensure_stage(ctx, s, stage_bytes);
    if (rc == PGCM_OK) rc = ensure_work(ctx, work_bytes, stream);
    if (rc == PGCM_OK) {
        try {
            ctx->scratch.reserve(n_max, num_cu);
        } catch (const std::bad_alloc&) {
            rc = PGCM_ERR_NOMEM;
        }
    }
    if (rc == PGCM_OK) {
        // the context now belongs to this stream, so that the stream's batches find it
        std::lock_guard<std::mutex> lock(key->mu);
        ctx->bound = true;
    }
    release_context(key, ctx);
    return rc;
}

int pgcm_decrypt_verify_batch(pgcm_key_t* key, size_t n, const uint8_t* ivs,
                              const void* const* aad, const uint32_t* aad_len,
                              const void* const* src, const uint64_t* len, void* const* dst,
                              const uint8_t* tags, uint8_t* ok, void* hip_stream) {
    return run_batch(key, BatchArgs{true, n, nullptr, ivs, 12, aad, aad_len, src, len, dst,
                                    const_cast<uint8_t*>(tags), ok, (hipStream_t)hip_stream});
}

int pgcm_decrypt_verify_batch_iv(pgcm_key_t* key, size_t n, const uint8_t* ivs, uint32_t iv_bytes,
                                 const void* const* aad, const uint32_t* aad_len,
                                 const void* const* src, const uint64_t* len, void* const* dst,
                                 const uint8_t* tags, uint8_t* ok, void* hip_stream) {
    return run_batch(key, BatchArgs{true, n, nullptr, ivs, iv_bytes, aad, aad_len, src, len, dst,
                                    const_cast<uint8_t*>(tags), ok, (hipStream_t)hip_stream});
}

int pgcm_encrypt_batch_keys(pgcm_key_t* const* keys, size_t nkeys, const uint32_t* key_index,
                            size_t n, const uint8_t* ivs, uint32_t iv_bytes,
                            const void* const* aad, const uint32_t* aad_len,
                            const void* const* src, const uint64_t* len, void* const* dst,
                            uint8_t* tags, void* hip_stream) {
    return run_batch_keys(keys, nkeys, key_index,
                          BatchArgs{false, n, nullptr, ivs, iv_bytes, aad, aad_len, src, len, dst,
                                    tags, nullptr, (hipStream_t)hip_stream});
}

int pgcm_decrypt_verify_batch_keys(pgcm_key_t* const* keys, size_t nkeys,
                                   const uint32_t* key_index, size_t n, const uint8_t* ivs,
                                   uint32_t iv_bytes, const void* const* aad,
                                   const uint32_t* aad_len, const void* const* src,
                                   const uint64_t* len, void* const* dst, const uint8_t* tags,
                                   uint8_t* ok, void* hip_stream) {
    return run_batch_keys(keys, nkeys, key_index,
                          BatchArgs{true, n, nullptr, ivs, iv_bytes, aad, aad_len, src, len, dst,
                                    const_cast<uint8_t*>(tags), ok, (hipStream_t)hip_stream});
}

const char* pgcm_strerror(int status) {
    switch (status) {
        case PGCM_OK: return "success";
        case PGCM_ERR_ARG: return "invalid argument";
        case PGCM_ERR_ALIGN: return "src or dst pointer not 16-byte aligned";
        case PGCM_ERR_LEN: return "chunk longer than the GCM limit of 2^36 - 32 bytes, or too long for a forced unit size";
        case PGCM_ERR_NOMEM: return "out of host or device memory";
        case PGCM_ERR_HIP: return "a HIP runtime call failed";
        case PGCM_ERR_BUSY: return "every buffer of the pool is held";
        case PGCM_ERR_CAPACITY: return "the batch needs more than the fixed buffers of an entry point that does not allocate";
        default: return "unknown status";
    }
}

int pgcm_last_hip_error(void) { return g_last_hip_error; }

int64_t pgcm_plan_units(size_t n, const uint64_t* len, uint32_t* nunits, uint32_t* first_blocks,
                        uint32_t* unit_base, uint32_t* final_count, uint32_t* final_power) {
    if (n != 0 && len == nullptr) return PGCM_ERR_ARG;
    uint64_t total = 0;
    const uint32_t unit_power = choose_unit_power(n, nullptr, len, kWaveSlots);
    for (size_t i = 0; i < n; ++i) {
        if (len[i] > PGCM_MAX_CHUNK_BYTES) return PGCM_ERR_LEN;
        UnitPlan p = plan_chunk(len[i], unit_power);
        uint32_t outs[kMaxLevels];
        const uint32_t levels = fold_levels(p.nunits, outs);
        if (levels > kMaxLevels) return PGCM_ERR_LEN;  // cannot happen with the chosen unit
        if (nunits) nunits[i] = p.nunits;
        if (first_blocks) first_blocks[i] = p.first_blocks;
        if (unit_base) unit_base[i] = (uint32_t)total;
        if (final_count) final_count[i] = levels ? outs[levels - 1] : p.nunits;
        if (final_power) final_power[i] = unit_power + kFanPower * levels;
        total += p.nunits;
        if (total > 0xFFFFFFF0ull / 64) return PGCM_ERR_ARG;
    }
    return (int64_t)total;
}

uint32_t pgcm_unit_bytes(void) { return kUnitBytes; }

uint32_t pgcm_batch_unit_bytes(size_t n, const uint64_t* len) {
    if (n != 0 && len == nullptr) return 0;
    return 16u << choose_unit_power(n, nullptr, len, kWaveSlots);
}

int pgcm_describe_schedule(size_t n, const uint64_t* len, uint32_t unit_bytes, uint32_t wave_slots,
                           pgcm_schedule_info* info, void* image, size_t image_capacity) {
    if (info == nullptr || (n != 0 && len == nullptr) || n > 0x7FFFFFFFull) return PGCM_ERR_ARG;
    uint32_t forced = 0;
    if (unit_bytes != 0) {
        for (uint32_t u = kMinUnitPower; u <= kMaxUnitPower; ++u)
            if (unit_bytes == (16u << u)) forced = u;
        if (forced == 0) return PGCM_ERR_ARG;
    }
    memset(info, 0, sizeof(*info));
    // stand-ins for the device pointers a real batch carries (16-byte aligned, never followed)
    std::vector<const void*> ptrs;
    try {
        ptrs.assign(n, reinterpret_cast<const void*>((uintptr_t)4096));
    } catch (const std::bad_alloc&) {
        return PGCM_ERR_NOMEM;
    }
    BatchArgs a{false, n, nullptr, reinterpret_cast<const uint8_t*>((uintptr_t)4096), 12, nullptr,
                nullptr, ptrs.data(), len, const_cast<void* const*>(ptrs.data()),
                reinterpret_cast<uint8_t*>((uintptr_t)4096), nullptr, nullptr};
    BatchSurvey v;
    int rc = survey_batch(a, &v);
    if (rc != PGCM_OK) return rc;
    BatchPlan p{};
    rc = plan_batch(forced, wave_slots ? wave_slots : kWaveSlots, a, &p);
    if (rc != PGCM_OK) return rc;
    const WorkLayout w = lay_out(a, p);
    info->desc_offset = w.desc;
    info->unit_base_offset = w.ubase;
    info->coarse_map_offset = w.coarse;
    info->fold_items_offset = w.fold;
    info->image_bytes = w.upload_bytes;
    info->workspace_bytes = w.bytes;
    info->unit_power = p.unit_power;
    info->nunits = p.nunits;
    info->nslots = p.nslots;
    info->ncoarse = p.ncoarse;
    info->nfold = p.nfold;
    for (uint32_t l = 0; l < kMaxLevels; ++l) {
        info->fold_count[l] = p.fold_count[l];
        info->fold_first[l] = p.fold_first[l];
    }
    info->path = n == 0 ? 0 : v.all_one_row() ? 1 : (v.all_small() && n <= kSmallMaxChunks) ? 2 : 0;
    if (image != nullptr) {
        if (image_capacity < w.upload_bytes) return PGCM_ERR_CAPACITY;
        memset(image, 0, w.upload_bytes);
        if (n != 0) fill_schedule(a, p, w, static_cast<uint8_t*>(image));
    }
    return PGCM_OK;
}

int pgcm_describe_context(pgcm_key_t* key, void* hip_stream, pgcm_context_info* info,
                          void* workspace, size_t bytes) {
    if (key == nullptr || info == nullptr || (workspace == nullptr && bytes != 0))
        return PGCM_ERR_ARG;
    std::lock_guard<std::mutex> lock(key->mu);
    for (const Context* c : key->contexts) {
        if (c->in_call || !c->bound || c->stream != (hipStream_t)hip_stream) continue;
        info->allocations = c->allocations;
        info->workspace_bytes = c->work_cap;
        info->stage_bytes = c->stage_cap[0];
        for (int s = 1; s < kStages; ++s)
            if (c->stage_cap[s] < info->stage_bytes) info->stage_bytes = c->stage_cap[s];
        if (bytes > c->work_cap) return PGCM_ERR_CAPACITY;
        if (bytes != 0) {
            PGCM_HIP(hipDeviceSynchronize());
            PGCM_HIP(hipMemcpy(workspace, c->work, bytes, hipMemcpyDeviceToHost));
        }
        return PGCM_OK;
    }
    return PGCM_ERR_ARG;
}

size_t pgcm_key_tables_bytes(void) { return kPublicTablesBytes; }

int pgcm_copy_key_tables(pgcm_key_t* key, void* out, size_t bytes) {
    if (key == nullptr || key->tables == nullptr || (out == nullptr && bytes != 0))
        return PGCM_ERR_ARG;
    if (bytes > kPublicTablesBytes) bytes = kPublicTablesBytes;
    PGCM_HIP(hipDeviceSynchronize());
    if (bytes != 0) PGCM_HIP(hipMemcpy(out, key->tables, bytes, hipMemcpyDeviceToHost));
    return PGCM_OK;
}

int pgcm_set_unit_bytes(pgcm_key_t* key, uint32_t unit_bytes) {
    if (key == nullptr) return PGCM_ERR_ARG;
    if (unit_bytes == 0) {
        key->forced_unit_power = 0;
        return PGCM_OK;
    }
    for (uint32_t u = kMinUnitPower; u <= kMaxUnitPower; ++u)
        if (unit_bytes == (16u << u)) {
            key->forced_unit_power = u;
            return PGCM_OK;
        }
    return PGCM_ERR_ARG;
}

int pgcm_bitsliced_keystream(pgcm_key_t* key, const uint8_t iv[12], uint32_t ctr_base,
                             uint64_t nblocks, void* out, void* hip_stream) {
    constexpr uint64_t kPerGroup = pgcm_bitsliced::kLaneBlocks * pgcm_bitsliced::kGroupLanes;
    if (key == nullptr || key->tables == nullptr || iv == nullptr || out == nullptr)
        return PGCM_ERR_ARG;
    if (ctr_base % pgcm_bitsliced::kLaneBlocks != 0 || nblocks % kPerGroup != 0 ||
        nblocks > ((uint64_t)1 << 31) || ((uintptr_t)out & 15))
        return PGCM_ERR_ARG;
    if (nblocks == 0) return PGCM_OK;
    int cur_device = -1;
    PGCM_HIP(hipGetDevice(&cur_device));
    if (cur_device != key->device) return PGCM_ERR_ARG;
    uint32_t w[3];
    memcpy(w, iv, 12);  // little-endian loads of the IV bytes, like the round-key words
    const dim3 grid((uint32_t)(nblocks / kPerGroup)), block(pgcm_bitsliced::kGroupLanes);
    const hipStream_t stream = (hipStream_t)hip_stream;
    const KeyTables* kt = key->tables;
    uint32_t* o = static_cast<uint32_t*>(out);
    if (key->rounds == 10)
        hipLaunchKernelGGL(pgcm_bitsliced::keystream_kernel<10>, grid, block, 0, stream, kt, w[0],
                           w[1], w[2], ctr_base, o);
    else if (key->rounds == 12)
        hipLaunchKernelGGL(pgcm_bitsliced::keystream_kernel<12>, grid, block, 0, stream, kt, w[0],
                           w[1], w[2], ctr_base, o);
    else
        hipLaunchKernelGGL(pgcm_bitsliced::keystream_kernel<14>, grid, block, 0, stream, kt, w[0],
                           w[1], w[2], ctr_base, o);
    PGCM_HIP(hipGetLastError());
    return PGCM_OK;
}

int pgcm_set_matrix_hash(pgcm_key_t* key, int enable) {
    if (key == nullptr) return PGCM_ERR_ARG;
    key->matrix_hash = enable != 0;
    return PGCM_OK;
}

int pgcm_set_one_launch(pgcm_key_t* key, int enable) {
    if (key == nullptr) return PGCM_ERR_ARG;
    key->one_launch = enable != 0;
    return PGCM_OK;
}

int pgcm_set_timing(pgcm_key_t* key, int enable) {
    if (key == nullptr) return PGCM_ERR_ARG;
    if (enable && key->bulk_start[0] == nullptr) {
        for (uint32_t i = 0; i < kTimingRing; ++i) {
            PGCM_HIP(hipEventCreate(&key->bulk_start[i]));
            PGCM_HIP(hipEventCreate(&key->bulk_stop[i]));
        }
    }
    key->timing = enable != 0;
    key->timed = 0;
    return PGCM_OK;
}

int pgcm_measure_passes(pgcm_key_t* key, size_t n, const uint8_t* ivs, uint32_t iv_bytes,
                        const void* const* aad,
                        const uint32_t* aad_len, const void* const* src, const uint64_t* len,
                        void* const* cipher, void* const* back, uint8_t* tags, uint8_t* ok,
                        void* hip_stream, uint32_t steps, int direction, double* host_ms) {
    if (host_ms == nullptr || direction < 0 || direction > 2) return PGCM_ERR_ARG;
    const hipStream_t stream = (hipStream_t)hip_stream;
    PGCM_HIP(hipStreamSynchronize(stream));
    const auto t0 = std::chrono::steady_clock::now();
    for (uint32_t k = 0; k < steps; ++k) {
        int rc = PGCM_OK;
        if (direction != 2)
            rc = pgcm_encrypt_batch_iv(key, n, ivs, iv_bytes, aad, aad_len, src, len, cipher, tags,
                                       hip_stream);
        if (rc == PGCM_OK && direction != 1)
            rc = pgcm_decrypt_verify_batch_iv(key, n, ivs, iv_bytes, aad, aad_len,
                                              reinterpret_cast<const void* const*>(cipher), len,
                                              back, tags, ok, hip_stream);
        if (rc != PGCM_OK) return rc;
    }
    PGCM_HIP(hipStreamSynchronize(stream));
    *host_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0)
                   .count();
    return PGCM_OK;
}

int pgcm_last_bulk_kernel_ms(pgcm_key_t* key, float* ms) {
    if (key == nullptr || ms == nullptr || key->timed == 0) return PGCM_ERR_ARG;
    const uint32_t slot = (uint32_t)((key->timed - 1) % kTimingRing);
    PGCM_HIP(hipEventSynchronize(key->bulk_stop[slot]));
    PGCM_HIP(hipEventElapsedTime(ms, key->bulk_start[slot], key->bulk_stop[slot]));
    return PGCM_OK;
}

int64_t pgcm_bulk_kernel_ms_history(pgcm_key_t* key, float* ms, size_t max) {
    if (key == nullptr || (ms == nullptr && max != 0)) return PGCM_ERR_ARG;
    uint64_t count = key->timed < kTimingRing ? key->timed : kTimingRing;
    if (count > max) count = max;
    for (uint64_t i = 0; i < count; ++i) {
        const uint32_t slot = (uint32_t)((key->timed - count + i) % kTimingRing);
        PGCM_HIP(hipEventSynchronize(key->bulk_stop[slot]));
        PGCM_HIP(hipEventElapsedTime(&ms[i], key->bulk_start[slot], key->bulk_stop[slot]));
    }
    return (int64_t)count;
}

#pragma GCC visibility pop
}  // extern "C"
