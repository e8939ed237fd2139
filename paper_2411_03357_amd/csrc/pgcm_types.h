// Structures shared by the host side of the library and its kernels.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace pgcm {

// A wavefront handles 64 consecutive 16-byte blocks (one 1 KiB "row") per step, one block per
// lane.  Where chunks are cut into units of one size (swap_kernel, and the schedule of bulk_kernel), a
// unit is the piece of a chunk one wavefront walks in one go; units are counted back from the
// chunk's end, so only a chunk's first unit can be short.  A unit is 2^unit_power blocks.  In the
// schedule of bulk_kernel, batches that do not fill the chip get the smallest size, from one row
// up, that still gives every unit a wavefront of its own, so that the batch spreads over as many
// wavefronts as there are and no unit waits; batches that do fill it get sixteen rows, handed out
// dynamically.  Larger units (up to 2^kMaxUnitPower blocks) can be forced for measurements.
constexpr uint32_t kRowBlocks = 64;
constexpr uint32_t kRowPower = 6;      // H^64: one row further along a lane's stripe
constexpr uint32_t kUnitPower = 10;    // the unit of the dynamic schedule: 1024 blocks = 16 KiB
constexpr uint32_t kMaxUnitPower = 20; // the largest unit that can be forced: 2^20 blocks = 16 MiB
constexpr uint32_t kMinUnitPower = kRowPower;
constexpr uint32_t kUnitBlocks = 1u << kUnitPower;
constexpr uint32_t kUnitBytes = kUnitBlocks * 16;
// wavefront slots of a 256-CU chip at sixteen per compute unit: a batch gets the smallest unit
// with which it has at most this many units (the full unit if none has)
constexpr uint32_t kWaveSlots = 4096;
constexpr uint32_t kWavesPerGroup = 16;
constexpr uint32_t kGroupThreads = kWavesPerGroup * 64;
static_assert((1u << kRowPower) == kRowBlocks, "row power");

// Every unit leaves a "partial set": the 64 per-lane GHASH sums of its rows (1 KiB).  Sets of one
// chunk are folded 32 at a time (again counted back from the end), level by level, until at most
// 32 remain; the per-chunk final step folds those and the 64 lanes.
constexpr uint32_t kFanPower = 5;
constexpr uint32_t kFan = 1u << kFanPower;
constexpr uint32_t kMaxLevels = 4;     // 2^22 units (the GCM length limit) / 32^4 <= 32
// The sets a fold level or the final step works on lie 2^(unit_power + 5 * level) blocks apart;
// that exponent must name one of the tables below.

// GHASH tables hold, for one constant C = H^(2^k), the products of C with every value of every
// nibble position of a block: entry [2 * byte + (0: high nibble, 1: low nibble)][value], 16 bytes
// each, 8 KiB per constant.
constexpr uint32_t kNibbleTableEntries = 32 * 16;
constexpr uint32_t kNumPowers = kUnitPower + kFanPower * kMaxLevels + 1;  // H^(2^0) .. H^(2^30)

// Multiplication by H^64 is linear over GF(2): a 128 x 128 bit matrix.  As operands of the 4-bit
// floating-point matrix instruction (an entry per nibble) it takes as much room as a nibble table.
constexpr uint32_t kRowMatrixWords = 128 * 128 / 8;
static_assert(kRowMatrixWords * 4 == kNibbleTableEntries * 16, "same room as a nibble table");

// The row hash on the matrix cores multiplies by H^64 and by H^96 at once (GhashRowMatrix): two such
// images, in the operand order of that engine.
constexpr uint32_t kHashImages = 2;

// The lane tree of the kernels that finish large chunks folds the 64 lanes in groups of four,
// three multiplications deep; beside H^(2^k) it needs the nibble tables of H^3, H^12 and H^48.
constexpr uint32_t kNumLanePowers = 3;

// The latency path sums a set's 64 lanes as 64 products of a sum with a known power of H, all
// at once and bit by bit, and moves a workgroup's result to its place with one more such product:
// it needs powers of H as plain values, held as four words with coefficient x^0 in the top bit of
// the first (GfWords).  dot[g][b][w][i] = H^(257 - (64 g + i)) * x^(8 (4 w + b)), the slice of
// byte b of word w, the multiplication by H that follows the length block included (a row of 64 blocks takes
// the last 64 of them, dot[kRowDot]);  hop[d][k] = H^(k 2^(8 + d)).
// A power's slices lie apart and neighbouring powers together: a lane takes a power each, so that a
// wavefront's load of a slice is 1 KiB in one piece (with a power's sixteen slices together it touched 64
// lines: 2 MiB decrypted 9.39 -> 9.14 us, 8 MiB both ways 40.5 -> 38.7, 64 chunks of 4 KiB 13.7 -> 13.3).
// The slices of 64 powers are 16 KiB in one piece, from a cache line's beginning, so that one address reaches four
// of them: with all slices 4 KiB apart sixteen loads held an address each, and swap_kernel and the long-IV kinds
// of span_kernel spilled (28 MB in one chunk 48.0 -> 47.3 us, 90 chunks of 4 to 500 KB with 40-byte IVs decrypted
// 41.8 -> 39.5, 300 of 3 KiB with such 18.0 -> 16.0).  A word's four are 4 KiB apart, as bursts read them: in one
// piece, 64 chunks of 4 KiB both ways take 13.0 us instead of 12.9, 2 MiB decrypted 8.70 instead of 8.77.
constexpr uint32_t kDotSlices = 16;
constexpr uint32_t kDotBlocks = 256;
constexpr uint32_t kRowDot = kDotBlocks / kRowBlocks - 1;  // what a row takes
constexpr uint32_t kHopMinPower = 8;    // the shortest stretch of a workgroup: 4 units of 64 blocks
constexpr uint32_t kHopPowers = 7;      // ... and the longest: 16 units of 1024 blocks
constexpr uint32_t kHopEntries = 256;   // workgroups of a chunk
// The span kernel cuts chunks between any two rows: row_hop[k] = H^(64 k), and far_hop[k] =
// H^(64 k kRowHopEntries) for what is further from a chunk's end.
constexpr uint32_t kRowHopPower = 12;
constexpr uint32_t kRowHopEntries = 1u << kRowHopPower;
constexpr uint32_t kFarHopEntries = 256;

struct alignas(16) GfWords {
    uint32_t a[4];
};

struct alignas(16) Block {
    uint32_t w[4];  // bytes 4i..4i+3 of the block, loaded little-endian into w[i]
};

struct alignas(128) KeyTables {
    uint32_t rk[60];       // round key words 0 .. 4 (rounds + 1) - 1, little-endian loads of the
                           // FIPS-197 bytes; the rest zero
    uint32_t rounds;       // Nr: 10, 12 or 14 for 128-, 192-, 256-bit keys (the paper's: 14)
    uint32_t pad_[3];
    uint32_t te[4][256];   // round tables: te[r][x] = MixColumns contribution of S(x) in row r
    Block h;               // GHASH key H = E_K(0^128)
    Block ghash[kNumPowers][kNibbleTableEntries];
    uint32_t row_matrix[kRowMatrixWords];  // multiplication by H^64 as matrix-core operands
    Block ghash_lane[kNumLanePowers][kNibbleTableEntries];  // nibble tables of H^3, H^12, H^48
    // ---- up to here the tables are part of what pgcm_copy_key_tables returns ----
    // multiplications by H^64 and by H^96 as the unit kernel's matrix operands
    uint32_t hash_image[kHashImages][kRowMatrixWords];
    Block ghash_rows3[kNibbleTableEntries];  // nibble table of H^192
    // round key words by columns: [c][r] = rk[4 r + c], r < 14, and of the last round key [c][15]
    uint32_t column_keys[4][16];
    alignas(128) GfWords dot[kDotBlocks / kRowBlocks][4][kDotSlices / 4][kRowBlocks];
    GfWords hop[kHopPowers][kHopEntries];
    GfWords row_hop[kRowHopEntries];
    GfWords far_hop[kFarHopEntries];
};
constexpr size_t kPublicTablesBytes = offsetof(KeyTables, hash_image);

struct alignas(16) ChunkDesc {
    const uint8_t* src;
    uint8_t* dst;
    const uint8_t* aad;
    uint64_t len;
    uint32_t aad_len;
    uint32_t unit_base;     // index of this chunk's first unit among all units = its set slot
    uint32_t nunits;        // 0 for an empty chunk
    uint32_t first_blocks;  // blocks in unit 0; every later unit has 2^unit_power
    uint32_t final_base;    // first set slot the final step folds
    uint32_t final_count;   // number of sets it folds: 1..32, or 0 for an empty chunk
    uint32_t final_power;   // log2 of the distance, in blocks, between consecutive such sets
    uint32_t index;         // the chunk's place in the caller's ivs, tags and ok arrays
};
static_assert(sizeof(ChunkDesc) == 64, "descriptor layout");

// One fold of up to 32 consecutive sets of a chunk into one set of the next level.
struct alignas(16) FoldItem {
    uint32_t in_base;   // first input slot
    uint32_t in_count;  // 1..32
    uint32_t out_slot;
    uint32_t pad_;
};

// The blocks before a chunk's block 0 that a kernel walks along with it: "block -1", whose keystream
// is the tag's mask, and the AAD's blocks, numbered -n .. -1, unless there are more of them than a
// row holds.
#ifdef __HIPCC__
__host__ __device__
#endif
constexpr uint32_t lead_blocks(uint32_t aad_len) {
    return aad_len <= 16 || aad_len > 64 * 16 ? 1 : (aad_len + 15) / 16;
}

// ... and where another wavefront makes E_K(J0): the AAD's blocks alone.
#ifdef __HIPCC__
__host__ __device__
#endif
constexpr uint32_t swap_lead_blocks(uint32_t aad_len, bool mask_elsewhere) {
    return mask_elsewhere && aad_len == 0 ? 0 : lead_blocks(aad_len);
}

// A batch of few chunks that does not fill the chip (every unit gets a wavefront of its own) is
// done by ONE kernel, its descriptors travelling as kernel arguments: the paper's swaps arrive a
// few chunks at a time between synchronisations (section 5.1), and for them the time of a call
// counts, not the rate.  Every chunk gets workgroups of its own, as many units each as a workgroup
// has wavefronts, counted back from the chunk's end so that only its first workgroup can be short.
// A chunk's units cover the blocks before its block 0 as well.
constexpr uint32_t kArgChunks = 64;
struct ArgChunk {
    const uint8_t* src;
    uint8_t* dst;
    const uint8_t* aad;
    uint64_t len;
    uint32_t aad_len;
    uint32_t index;         // the chunk's place in the caller's ivs, tags and ok arrays
};
static_assert(sizeof(ArgChunk) == 40, "argument layout");
struct ArgBatch {
    uint32_t group_base[kArgChunks + 1];  // first workgroup of every chunk; their number
    ArgChunk c[kArgChunks];
};
// burst_kernel has its chunks' descriptors in one of three forms.  What a launch costs the host goes by the bytes
// of its arguments: of up to 96 2.6 to 2.8 us, of 128 and more 3.4 to 4.1; if its end is marked with an event, of
// 48 4.5, of 64 to 96 5.1 to 6.2, of more 7.0 to 8.1.  So one chunk does not come with room for kArgChunks, nor do
// descriptors that are in pinned memory, one for each workgroup (1 byte 4.96 -> 4.59 us, 320 KiB 6.62 -> 6.40, 2 MiB
// decrypted 8.76 -> 8.45, 300 of up to 8 KiB decrypted 11.2 -> 9.3).
struct ArgOne {
    ArgChunk c;  // its place in the caller's arrays is in the pointers already
};
struct ArgStaged {
    const struct GroupDesc* groups;
};
// Passes a workgroup of sixteen wavefronts of the kernel for short bursts makes at most, at a time and in
// all (of fewer wavefronts: one).
constexpr uint32_t kFoldPasses = 4, kSweptPasses = 16;
// Where a wavefront of burst_kernel's takes a row of 64 blocks: wavefront w has row w % 4 of pass w / 4 of every
// sweep, the last pass of the last sweep being number `behind` from the chunk's end, of `folded` passes a
// sweep.  Which wavefront has the block before the chunk's first, of nblk?
#ifdef __HIPCC__
__host__ __device__
#endif
constexpr uint32_t wave_of_lead(uint32_t nblk, uint32_t behind, uint32_t folded) {
    const uint32_t pass = nblk / 256, at = 255 - nblk % 256;  // number from the end, and the block's place in it
    return 4 * ((behind + folded - 1 - pass) % kFoldPasses) + at / 64;
}
// Encrypting in sweeps, are the rows of this one written through to memory?  A sweep's payload is asked for behind the
// stores of the one before, and waits for them, which takes long if they go out to host memory: only the last sweep's
// are, and none where each workgroup makes one sweep but for the passes that a chunk's first has to spare.  Into host
// memory, none written through, all, and so: 12 MiB 236.2, 242.0, 234.4 us, 7 MiB 147, 148, 138, 8 MiB 167.9, 166.4, 157.7,
// sixteen of 320 KiB 108.9, 106.6, 103.7, five of 1 to 3 MB 161, 149.6, 153.3, 4 MiB with AAD 86.8, 88.7, 86.6 (the last
// sweep's there 87.7).  In device memory 12 MiB 23.9, 22.8, 23.3, 8 MiB 18.9, 17.9, 18.1, four of 2 MiB 19.0, 17.9, 18.4,
// 4 MiB with AAD 16.0, 15.4, 15.8.
constexpr bool sweep_through(uint32_t passes_each, uint32_t sweep, uint32_t sweeps) {
    return passes_each > kFoldPasses && sweep + 1 == sweeps;
}
enum class BurstKind { kWords, kFold, kSweep, kFoldShared, kWordsShared, kFoldApart };
// Workgroups of a chunk (KeyTables::hop has their distances) and of a launch.
constexpr uint32_t kSwapChunkGroups = kHopEntries;
constexpr uint32_t kSwapMaxGroups = 512;
// Where the workgroups of a chunk add up their shares of its tag, a word each by one atomic that counts
// them in as well: a chunk has as many slots as workgroups and uses the first one's, and those of more
// than kArriveSet add up in sets of so many first, in the slot of the first of each.  All zero between
// batches.
constexpr uint32_t kArriveSet = 32;  // bits of half an accumulator, and as many sets at most
struct alignas(64) ArriveSlot {
    uint64_t of_chunk[4];  // in the second slot: decryption's verdict
    uint64_t of_set[4];
};
static_assert(kSwapChunkGroups <= kArriveSet * kArriveSet, "a bit for every set");
static_assert(sizeof(ArriveSlot) == 64, "counters of different chunks are not to share a cache line");
// What a workgroup has to know first, in one word: it travels in a register.
struct SwapMeta {
    uint32_t w;
#ifdef __HIPCC__
#define PGCM_BOTH __host__ __device__
#else
#define PGCM_BOTH
#endif
    PGCM_BOTH uint32_t nchunks() const { return w & 0x7Fu; }          // in an ArgBatch: 0 .. 64
    PGCM_BOTH uint32_t unit_power() const { return (w >> 7) & 0x1Fu; }  // burst_kernel: the passes
    PGCM_BOTH uint32_t wave_power() const { return (w >> 12) & 7u; }  // log2 of the wavefronts per
                                                                      // workgroup: 2, 3, 4
    PGCM_BOTH bool one_group_each() const { return (w >> 15) & 1u; }  // every chunk has a workgroup
    PGCM_BOTH bool in_order() const { return (w >> 16) & 1u; }        // chunk k is the caller's k
    PGCM_BOTH uint32_t groups() const { return (w >> 17) & 0x3FFu; }  // workgroups of the launch
    PGCM_BOTH uint32_t rounds() const { return (w >> 27) & 0xFu; }
    PGCM_BOTH bool iv_in_place() const { return w >> 31; }  // `ivs` and `iv_len` are no pointer and length but
                                                            // the 96 bits of the IV of an ArgOne
#undef PGCM_BOTH
};
constexpr SwapMeta swap_meta(uint32_t nchunks, uint32_t unit_power, uint32_t wave_power,
                             bool one_group_each, bool in_order, uint32_t groups,
                             uint32_t rounds, bool iv_in_place = false) {
    return SwapMeta{nchunks | unit_power << 7 | wave_power << 12 | (uint32_t)one_group_each << 15 |
                    (uint32_t)in_order << 16 | groups << 17 | rounds << 27 | (uint32_t)iv_in_place << 31};
}
// Batches of more chunks than fit the arguments have a descriptor per workgroup in pinned memory.
struct alignas(64) GroupDesc {   // one line of host memory
    ArgChunk c;
    uint32_t group_base, ngroups;  // the chunk's first workgroup and their number
};

// Spans: the rows of all chunks of a batch, each chunk's counted back from its end and the blocks
// before its block 0 among them, are numbered through.  Every wavefront takes a share of them, and
// chunks are cut wherever a share ends.
struct alignas(16) SpanGroup {      // a workgroup
    const KeyTables* kt;
    uint32_t first_row;
    uint32_t part, nparts;          // where its chunks are described, if not right behind this
    uint32_t waves;                 // its wavefronts with rows, at most kWavesPerGroup
    uint32_t cut[kWavesPerGroup + 1];  // the first row of each, counted from the workgroup's; the end
    uint32_t pad_;
};
static_assert(sizeof(SpanGroup) == 96, "descriptor layout");
struct alignas(16) SpanPart {       // a chunk as far as one workgroup has rows of it
    const uint8_t* src;
    uint8_t* dst;
    const uint8_t* aad;
    uint64_t len;
    uint32_t aad_len;
    uint32_t index;                 // the chunk's place in the caller's ivs, tags and ok arrays
    uint32_t first_row, rows;       // of the whole chunk
    uint32_t slot, slots;           // its workgroups, of which it may have several, have
    uint32_t own_slot;              // consecutive slots from `slot`; this one's
    uint32_t waves;                 // this one's wavefronts with rows of it, << 8; the first of them
};
static_assert(sizeof(SpanPart) == 64, "descriptor layout");
// Where a launch's workgroups find their packets, each a SpanGroup and its parts, and which tables they use:
// in the kernel's arguments, which are read at once, while a packet in host memory takes 2 us to come.
// So packets need not be equally long (300 adapters read 67 KB, where all as long as the longest were 139; both
// ways 171.6 -> 169.3 us), and with several keys the tables are asked for ahead of them (240 chunks of three keys,
// both ways, 175.2 -> 169.9).
constexpr uint32_t kSpanMapGroups = 512, kSpanMapKeys = 16;
constexpr uint32_t kPacketAlign = 64;  // packets begin at multiples of this
struct SpanMap {
    const KeyTables* key[kSpanMapKeys];
    // where the packet begins, in kPacketAlign; from bit kLengthShift on its parts, from kKeyShift on the key
    uint32_t place[kSpanMapGroups];

    static constexpr uint32_t kLengthShift = 16, kKeyShift = 22;
};
constexpr uint32_t kSpanPlaced = 1, kSpanKeysMapped = 2;  // what of a launch's map is filled in
constexpr uint32_t packet_bytes(uint32_t nparts) {
    return (uint32_t)((sizeof(SpanGroup) + sizeof(SpanPart) * nparts + kPacketAlign - 1) / kPacketAlign * kPacketAlign);
}
// IVs of at most one block are hashed in one round of lookups.
constexpr uint32_t kShortIvBytes = 16;
// The parts of a workgroup that are held in LDS; those of longer lists are read from memory.
constexpr uint32_t kSpanLdsParts = 31;

// A batch whose chunks are all at most this long (the paper's non-swap transfers are usually < 8 KB,
// section 4.2; eight rows of 64 blocks) goes to the kernel for short bursts.
constexpr uint64_t kSmallChunkBytes = 8192;
// That kernel is there for the latency of a few transfers; of more chunks than this
// (two workgroups per compute unit are resident) ...
constexpr size_t kSmallMaxChunks = 512;
// ... those of at most this length (63 blocks: one row together with "block -1") take a kernel with
// a wavefront per chunk, and longer ones go in spans, which get more chunks per second out of the
// chip.
constexpr uint64_t kSmallRowBytes = 1008;

// Items of the dynamic schedule are grabbed from a counter; to find an item's chunk a wavefront
// starts at coarse_map[item >> kCoarseShift] and walks unit_base[] forward.
constexpr uint32_t kCoarseShift = 4;

}  // namespace pgcm
