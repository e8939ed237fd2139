// Which way a batch of one key goes, and which of burst_kernel's kinds it takes.  Host only, plain C++.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include "pgcm_one_launch.h"
#include "pgcm_spans.h"
#include "pgcm_types.h"

namespace pgcm {

// What decides besides the chunks: the device, what the key is set to, and the entry point.
struct RouteOptions {
    uint32_t num_cu;
    bool one_launch, matrix_hash;
    uint32_t forced_unit_power;  // 0: chosen for the batch
    bool fixed;                  // the entry point that allocates nothing
    bool spread;                 // short chunks, at most kArgChunks of them, may have several workgroups
    bool clears_slots;           // the slots that chunks of several workgroups need take a launch that clears them
};

// What decides of the chunks.
struct BatchSurvey {
    uint64_t rows = 0;     // in spans
    uint64_t longest = 0;  // in bytes

    void add(uint64_t len, uint32_t aad_len) {
        if (len > longest) longest = len;
        rows += span_rows(len, aad_len);
    }
    bool all_small() const { return longest <= kSmallChunkBytes; }   // every chunk is a short transfer
    bool all_one_row() const { return longest <= kSmallRowBytes; }   // ... and one of one row
};

// May a batch of chunks of at most this length, and this many rows in all, go in spans?  (The bounds
// are those of the powers of H a key has and of 32-bit row numbers.)
inline bool takes_spans(const RouteOptions& o, uint64_t rows, uint64_t longest) {
    return o.one_launch && !o.matrix_hash && !o.forced_unit_power && rows <= kSpanMaxRows &&
           longest / (16 * kRowBlocks) + 2 < (uint64_t)kRowHopEntries * kFarHopEntries;
}

inline bool may_go_in_spans(const RouteOptions& o, const BatchSurvey& v) {
    return !o.fixed && !v.all_one_row() && takes_spans(o, v.rows, v.longest);
}

enum class Route {
    kOneLaunch,  // burst_kernel or swap_kernel, as `shape` says
    kOneRow,     // small_kernel
    kSpans,      // span_kernel
    kUnits,      // bulk_kernel and what follows it
};

// `shape` is filled in for kOneLaunch.
inline Route route_batch(const ShapeBatch& a, const RouteOptions& o, const BatchSurvey& v, SwapShape* shape) {
    const bool spans = may_go_in_spans(o, v);
    // What short chunks in several workgroups need, and those with a workgroup each do not, is slots.
    const bool spread = a.n <= kArgChunks ? o.one_launch && o.spread : !o.clears_slots;
    if (swap_shape(a, o.num_cu, o.one_launch, o.forced_unit_power, v.all_small(), spread, shape) &&
        (!spans || shape->burst ||
         units_before_spans(*shape, v.rows, (uint64_t)o.num_cu * kWavesPerGroup)))
        return Route::kOneLaunch;
    return v.all_one_row() ? Route::kOneRow : spans ? Route::kSpans : Route::kUnits;
}

// Up to eight wavefronts with blocks have one more that has none, where no two workgroups share a compute unit; what
// decrypts in two passes of sixteen hashes them beside the cipher (see burst_kernel).  One chunk, whose workgroups have
// a compute unit each, never takes a shared kind.
inline BurstKind burst_kind(const SwapShape& s, uint32_t num_cu, bool decrypt) {
    const bool shared = s.groups > num_cu;
    if (s.wave_power < 4) return shared ? BurstKind::kWordsShared : BurstKind::kWords;
    if (shared) return BurstKind::kFoldShared;
    if (s.unit_power + s.spare > kFoldPasses) return BurstKind::kSweep;
    return decrypt && s.unit_power == 2 ? BurstKind::kFoldApart : BurstKind::kFold;
}

}  // namespace pgcm
