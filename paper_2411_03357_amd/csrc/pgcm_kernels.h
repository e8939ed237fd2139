// Kernel declarations shared by the kernel file and the host side of the library.
#pragma once
#include <hip/hip_runtime.h>

#include "pgcm_types.h"

namespace pgcm {

// clear: n_clear elements that are made zero besides
__global__ void expand_key_kernel(KeyTables* kt, const uint32_t* key_words, uint32_t nk, uint4* clear,
                                  uint32_t n_clear);

__global__ void j0_kernel(const KeyTables* kt, const ChunkDesc* chunks, const uint8_t* ivs,
                          uint32_t iv_len, uint32_t nchunks, Block* j0);

// kRounds: 10, 12 or 14; kMatrixHash: the GHASH multiplication of every row runs on the matrix
// cores (from KeyTables::row_matrix) instead of table lookups in LDS
template <bool kDecrypt, int kRounds, bool kMatrixHash>
__global__ void bulk_kernel(const KeyTables* kt, const ChunkDesc* chunks,
                            const uint32_t* unit_base, const uint32_t* coarse_map,
                            uint32_t nunits_total, uint32_t unit_power, uint32_t* counter,
                            const uint8_t* ivs, const Block* j0, Block* ekj0, Block* sets);

// The whole invocation of a few chunks in one launch, 2^wave_power wavefronts of units a workgroup (at
// least four) and, below sixteen, one more.  The chunks come as arguments, or, when `staged` is not
// null, with a descriptor per workgroup there (batch is not looked at then).
// slots: one per workgroup; not touched if no chunk has more than one workgroup.  Units
// of two to sixteen rows, of eight or sixteen unless their size is forced.
// The arguments before `batch` come in registers (compiled for that, they are the first fourteen
// words), so that the tables are fetched while the rest of the arguments is.
template <bool kDecrypt, int kRounds>
__global__ void swap_kernel(const KeyTables* kt, const uint8_t* ivs, uint32_t iv_len, SwapMeta meta,
                            ArriveSlot* slots, uint8_t* tags, uint8_t* ok, const GroupDesc* staged,
                            ArgBatch batch);

// The same for batches whose time is that of one chain of steps: 2^wave_power wavefronts of sixteen blocks
// a workgroup, which makes meta.unit_power() passes, or, if it is a chunk's first, as many as are left,
// or, if it has a chunk to itself, as many as that takes.  It serves any key.  kLongIv: iv_len exceeds
// kShortIvBytes.  kWords: at most eight wavefronts, one pass, and a wavefront more (which it counts on: a workgroup
// has 2^wave_power + 1); kWordsShared: none more, and two workgroups fit a compute unit.  kFold: sixteen, and at most
// kFoldPasses; kFoldApart: the same, decrypting two, but for chunks' first workgroups of fewer or of one more; kSweep:
// kSweptPasses; kFoldShared: kFoldPasses - 1, and two workgroups fit a compute unit.  Args: ArgOne (not of the shared
// kinds), ArgBatch or ArgStaged.
template <bool kDecrypt, bool kLongIv, BurstKind kKind, class Args>
__global__ void burst_kernel(const KeyTables* kt, const uint8_t* ivs, uint32_t iv_len, SwapMeta meta,
                             ArriveSlot* slots, uint8_t* tags, uint8_t* ok, Args args);

// Spans of rows, one per wavefront, of chunks of one key (`key`) or of several (null).  mapped: what of `map`
// is filled in.  With kSpanKeysMapped the workgroups' keys, which are in their SpanGroup otherwise; with
// kSpanPlaced where in `packets`, which may be host memory then, a workgroup's SpanGroup and its parts lie, at
// most kSpanLdsParts; otherwise `packets` is the SpanGroup of all, and their parts are in `parts`.  slots: one per
// part.  kLongIv: iv_len exceeds kShortIvBytes.
template <bool kDecrypt, bool kLongIv>
__global__ void span_kernel(const KeyTables* key, const uint8_t* packets, const SpanPart* parts,
                            uint32_t iv_len, uint32_t mapped, const uint8_t* ivs, ArriveSlot* slots,
                            uint8_t* tags, uint8_t* ok, SpanMap map);

__global__ void fold_kernel(const KeyTables* kt, const FoldItem* items, uint32_t power,
                            Block* sets);

constexpr uint32_t kFoldTreeWaves = 16;
__global__ void fold_tree_kernel(const KeyTables* kt, const FoldItem* items, uint32_t power,
                                 Block* sets);

template <bool kDecrypt>
__global__ void final_kernel(const KeyTables* kt, const ChunkDesc* chunks, uint32_t nchunks,
                             const uint8_t* ivs, const Block* j0, const Block* ekj0,
                             const Block* sets, uint8_t* tags, uint8_t* ok, uint32_t unit_power,
                             uint32_t* counter, uint32_t chunks_per_group);
constexpr uint32_t kFinalWaves = 16;  // wavefronts of a final_kernel workgroup

constexpr uint32_t kSmallChunksPerGroup = 4;

// chunks of at most kSmallRowBytes each
template <bool kDecrypt, int kRounds>
__global__ void small_kernel(const KeyTables* kt, const ChunkDesc* chunks_host, uint32_t nchunks,
                             const uint8_t* ivs, uint32_t iv_len, uint8_t* tags, uint8_t* ok);

// copies, and sets the n_clear pieces of sixteen bytes from `clear` on to zero
__global__ void upload_kernel(uint4* dst, const uint4* src_host, uint32_t n16, uint4* clear,
                              uint32_t n_clear);

}  // namespace pgcm

namespace pgcm_bitsliced {
// pgcm_bitsliced.hip: keystream of counter blocks by a bitsliced round function (measurement)
constexpr uint32_t kLaneBlocks = 32;   // counter blocks per lane: one per bit of a register
constexpr uint32_t kGroupLanes = 64;
template <int kRounds>
__global__ void keystream_kernel(const pgcm::KeyTables* kt, uint32_t iv0, uint32_t iv1,
                                 uint32_t iv2, uint32_t ctr_base, uint32_t* out);
}  // namespace pgcm_bitsliced
