// How a batch is cut into spans of rows (span_kernel): which workgroups and wavefronts take which rows
// of which chunks, and the descriptors they read.  Host only, plain C++.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <vector>

#include "pgcm_types.h"

struct pgcm_key;

namespace pgcm {

// The caller's arrays as far as the cutter looks at them.
struct SpanBatch {
    size_t n;
    const uint32_t* order;  // chunk k of the batch is the caller's chunk order[k]; null: chunk k
    const void* const* aad;
    const uint32_t* aad_len;
    const void* const* src;
    const uint64_t* len;
    void* const* dst;

    size_t at(size_t k) const { return order ? order[k] : k; }
};

inline uint64_t span_rows(uint64_t len, uint32_t aad_len) {
    const uint64_t blocks = (len + 15) / 16 + lead_blocks(aad_len);
    return (blocks + kRowBlocks - 1) / kRowBlocks;
}

// Bytes of descriptors up to which the workgroups read theirs from host memory themselves.
constexpr size_t kSpanHostBytes = 256 << 10;

// Descriptors of a batch: the workgroups', then, at a multiple of 256, the parts'.
constexpr size_t span_parts_at(size_t ngroups) { return (sizeof(SpanGroup) * ngroups + 255) / 256 * 256; }
constexpr size_t span_image_bytes(size_t nparts, size_t ngroups) {
    return span_parts_at(ngroups) + (sizeof(SpanPart) * nparts + 255) / 256 * 256;
}

// (the bound of 32-bit row numbers, with room for sums of them)
constexpr uint64_t kSpanMaxRows = 1u << 27;

// Several keys' chunks share a launch, and with it a context of one of the keys, if their descriptors
// fit what every context that was reserved for spans has room for, however little it was reserved
// for: kSpanHostBytes of staging, a slot for each of so many descriptors, and such an image behind.
constexpr bool share_launch(size_t nkeys, size_t n, uint64_t rows, size_t num_cu) {
    return nkeys <= num_cu && rows <= kSpanMaxRows &&
           span_image_bytes(n + num_cu + nkeys, num_cu + nkeys) <= kSpanHostBytes;
}
constexpr size_t kSharedParts = kSpanHostBytes / sizeof(SpanPart);

// What a batch of one key and at most n chunks, or one of several keys that share a launch, takes at
// most on a device of num_cu compute units.  Workgroups: every key's share of the compute units may
// be rounded up to one (deal_groups).
constexpr size_t span_most_groups(size_t num_cu) { return 2 * num_cu; }
constexpr size_t span_most_parts(size_t n, size_t num_cu) {
    const size_t parts = n + span_most_groups(num_cu);
    return parts > kSharedParts ? parts : kSharedParts;
}
constexpr size_t span_stage_bytes(size_t n, size_t num_cu) {
    const size_t groups = span_most_groups(num_cu), bytes = span_image_bytes(n + groups, groups);
    return bytes > kSpanHostBytes ? bytes : kSpanHostBytes;
}
// clean_slots: those a workspace keeps clean already; descriptors go behind them
constexpr size_t span_work_bytes(size_t n, size_t num_cu, size_t clean_slots) {
    const size_t parts = span_most_parts(n, num_cu);
    return (sizeof(ArriveSlot) * (parts > clean_slots ? parts : clean_slots) + 255) / 256 * 256 +
           span_stage_bytes(n, num_cu);
}

// What is kept from call to call for cutting batches.
struct SpanScratch {
    std::vector<uint8_t> image;                // descriptors
    std::vector<uint32_t> rows, cuts, waves;

    void reserve(size_t n, size_t num_cu) {
        const size_t groups = span_most_groups(num_cu);
        image.resize(kSpanHostBytes);
        rows.reserve(span_most_parts(n, num_cu));
        cuts.reserve(groups * kWavesPerGroup + 1);
        waves.reserve(groups + 1);
    }
    size_t capacity() const {
        return image.capacity() + rows.capacity() + cuts.capacity() + waves.capacity();
    }
};

// What one more piece costs a workgroup of sixteen wavefronts, in rows (300 adapters both ways with 8, 6, 5:
// 159.9, 158.0, 157.9 us; 150 of 0.1 to 1 MB 139.3, 136.2, 136.0; 60 of 1 to 4 MB 294, 290, 287; 240 chunks of 4 KB to
// 2 MB, 400 of 320 KiB, 500 of 50 to 300 KB, 700 of 16 to 256 and 1000 of 50 to 250 within 1 %); and a wavefront among them, in half
// rows, which are 2.2 us (300 adapters with 3, 4, 6: 160.1, 160.1, 159.5; 600 of 16 to 128 KB 101.1, 103.2,
// 101.5; 100 of 0.1 to 1 MB 108.7, 108.8, 106.7).
constexpr uint32_t kPieceRows = 6;
constexpr uint32_t kPieceHalfRows = 6;
// Shares of up to so many rows are cut with regard to the pieces they make all over the batch (17 long
// chunks of two keys both ways 57 -> 35 us, 284 chunks of 44 to 97 KB 87 -> 79).  Longer ones are dealt
// out to the workgroups by weight: with the line at 9, 100 of 0.1 to 1 MB take 104.0 instead of 106.9 us, 120
// of 320 KiB 106.5 instead of 105.0, 400 of 64 to 128 KB and 50 of 0.2 to 2 MB the same.
constexpr uint32_t kFineRows = 12;
// Of these, up to so many rows and five chunks for four workgroups, a workgroup's wavefronts get shares with regard
// to its own pieces: cut equal, the wavefront with a chunk's end and the next one's beginning is the last by
// 6 half rows (300 adapters both ways, 17 rows a share, 162.0 -> 159.5 us; 240 chunks of three keys 161.9 ->
// 158.6; with up to 256 rows the same).  With more chunks the workgroup has as many such wavefronts as others, and
// finding the shares takes the host longer.  On 256 compute units, both ways back to back and encrypted and waited
// for: 256 of 16 KB to 1 MB 162.0 -> 156.7 and 104.5 -> 103.1 us, 300 of 80 to 400 KB 150.1 -> 145.6 and 98.3 -> 96.0, of
// 256 KiB 178.6 -> 179.3 and 112.5 -> 114.8; but 350 of 80 to 400 KB 164.1 -> 164.6 and 106.3 -> 108.0, 400 of 16 KB to
// 1 MB 222.7 -> 220.8 and 133.3 -> 135.5, 512 of 80 to 400 KB 229.8 -> 228.5 and 137.8 -> 140.6, 800 of 160 KiB 278.3 ->
// 278.6 and 160.9 -> 166.1, 1024 of 128 KiB 284.4 -> 285.1 and 162.4 -> 169.0.
constexpr uint32_t kEvenRows = 64;
constexpr uint32_t kEvenChunks = 5, kEvenGroups = 4;

// One key's chunks of a batch: n of them from the batch's chunk `first` on.
struct KeyPart {
    pgcm_key* key;
    const KeyTables* tables;  // of the key
    uint32_t rounds;
    size_t first, n;
    uint64_t rows, longest;   // the longest in bytes
    uint32_t groups;          // workgroups

    uint64_t weight() const { return rows + kPieceRows * n; }
};

// Deals the compute units out to the parts, a workgroup each, so that the one with the most work per
// workgroup has as little as can be: a row costs a table lookup per round and byte and the hash as
// much as three rounds.  A workgroup gets four rows at least, if there are that many: with no more
// wavefronts than that a row takes 2.6 us instead of 4.3.  Returns the number of workgroups.
inline uint32_t deal_groups(KeyPart* parts, size_t nparts, uint32_t num_cu) {
    uint64_t work = 0;
    auto cost = [](const KeyPart& p) { return p.weight() * (uint64_t)(p.rounds + 3); };
    auto most = [](const KeyPart& p) { return p.rows < 4 ? 1 : p.rows / 4; };
    for (size_t q = 0; q < nparts; ++q) work += cost(parts[q]);
    uint32_t total = 0;
    for (size_t q = 0; q < nparts; ++q) {
        uint64_t g = cost(parts[q]) * num_cu / work;
        if (g > most(parts[q])) g = most(parts[q]);
        parts[q].groups = g == 0 ? 1 : (uint32_t)g;
        total += parts[q].groups;
    }
    while (total < num_cu) {
        KeyPart* worst = nullptr;
        for (size_t q = 0; q < nparts; ++q) {
            KeyPart& p = parts[q];
            if (p.groups < most(p) &&
                (worst == nullptr || cost(p) * worst->groups > cost(*worst) * p.groups))
                worst = &p;
        }
        if (worst == nullptr) break;
        ++worst->groups, ++total;
    }
    return total;
}

// The rows of neighbouring pieces in shares of wavefronts: a share holds `limit` half rows, the pieces'
// beginnings and ends (kPieceHalfRows each) among them.  A piece that follows in a share with no room for a
// row more goes to the next.
struct ShareFill {
    uint32_t limit, left, used;

    explicit ShareFill(uint32_t half_rows) : limit(half_rows), left(half_rows), used(1) {}
    uint32_t whole() const { return (limit - kPieceHalfRows) / 2; }  // rows of a share with one piece
    // a piece of r rows from row `at` on; cut(row) where a share begins
    template <class Cut>
    void add(uint32_t at, uint32_t r, Cut&& cut) {
        if (left >= kPieceHalfRows + 2) {
            const uint32_t room = (left - kPieceHalfRows) / 2;
            if (r <= room) {
                left -= kPieceHalfRows + 2 * r;
                return;
            }
            r -= room, at += room;
        }
        const uint32_t n = (r - 1) / whole() + 1;
        for (uint32_t i = 0; i < n; ++i) cut(at + i * whole());
        used += n;
        left = limit - kPieceHalfRows - 2 * (r - (n - 1) * whole());
    }
};

// Cuts a key's rows, which begin at `row`, into shares of at most 16 * key.groups wavefronts and deals
// these out to its workgroups: the first rows of all wavefronts are appended to `cuts`, and
// waves[g] is the number of the first wavefront of workgroup g.  rows: of each chunk.
inline void cut_key(const KeyPart& key, uint32_t row, const uint32_t* rows, std::vector<uint32_t>& cuts,
             uint32_t* waves) {
    const uint32_t most = key.groups * kWavesPerGroup, base = (uint32_t)cuts.size();
    auto counted = [](uint32_t) {};
    auto kept = [&](uint32_t at) { cuts.push_back(at); };
    if (key.rows <= (uint64_t)most * kFineRows && key.n <= 2 * (size_t)most) {
        // Where shares are short, what a wavefront spends on beginning and finishing pieces decides: as
        // many half rows a share as it takes for the wavefronts to do.
        uint32_t limit = (uint32_t)((2 * key.rows + kPieceHalfRows * (key.n + most) + most - 1) / most);
        if (limit < kPieceHalfRows + 2) limit = kPieceHalfRows + 2;
        for (;; limit += 1 + limit / 32) {
            ShareFill fill(limit);
            for (size_t k = 0; k < key.n; ++k) fill.add(0, rows[k], counted);
            if (fill.used <= most) break;
        }
        ShareFill fill(limit);
        cuts.push_back(row);
        for (size_t k = 0; k < key.n; ++k) {
            fill.add(row, rows[k], kept);
            row += rows[k];
        }
        const uint32_t used = (uint32_t)cuts.size() - base;
        for (uint32_t g = 0; g < key.groups; ++g)
            waves[g] = base + (uint32_t)((uint64_t)used * g / key.groups);
        return;
    }
    // A workgroup begins where the weight so far reaches its share; a chunk's own weight comes before
    // its rows'.  Its rows go to its wavefronts in equal parts, or, where these are not long, with regard
    // to its pieces.
    uint64_t weight = 0, next = 0;
    uint32_t group = 0, begin = row;
    const bool even =
        key.rows <= (uint64_t)most * kEvenRows && kEvenGroups * key.n <= kEvenChunks * (size_t)key.groups;
    size_t first = 0;          // the chunk with row `begin`
    uint32_t first_end = row + rows[0];  // ... and its end
    auto deal = [&](uint32_t end) {
        if (group > 0) {
            const uint32_t n = end - begin, w = n < kWavesPerGroup ? n : kWavesPerGroup;
            while (first_end <= begin) first_end += rows[++first];
            if (even && first_end < end) {
                auto pieces = [&](ShareFill& fill, auto&& cut) {
                    size_t k = first;
                    for (uint32_t at = begin, till = first_end; at < end;) {
                        const uint32_t stop = till < end ? till : end;
                        fill.add(at, stop - at, cut);
                        at = stop;
                        if (at < end) till += rows[++k];
                    }
                };
                uint32_t count = 1;
                for (uint32_t till = first_end, k = (uint32_t)first; till < end; till += rows[++k]) ++count;
                if (count < w) count = w;
                uint32_t limit = (2 * n + kPieceHalfRows * count) / w;
                if (limit < kPieceHalfRows + 2) limit = kPieceHalfRows + 2;
                for (;; limit += 1 + limit / 64) {
                    ShareFill fill(limit);
                    pieces(fill, counted);
                    if (fill.used <= w) break;
                }
                ShareFill fill(limit);
                cuts.push_back(begin);
                pieces(fill, kept);
            } else {
                for (uint32_t i = 0; i < w; ++i) cuts.push_back(begin + (uint32_t)((uint64_t)n * i / w));
            }
        }
        begin = end;
    };
    for (size_t k = 0; k < key.n; ++k) {
        const uint64_t weight_end = weight + rows[k] + kPieceRows;
        while (group < key.groups && next < weight_end) {
            deal(next > weight + kPieceRows ? row + (uint32_t)(next - weight - kPieceRows) : row);
            waves[group++] = (uint32_t)cuts.size();
            next = key.weight() * group / key.groups;
        }
        row += rows[k];
        weight = weight_end;
    }
    deal(row);
}

// Cuts the keys' chunks.  parts: room for n and the number of workgroups.
struct SpanPlan {
    uint32_t nparts;
    uint32_t longest;  // list of parts of a workgroup
};
inline SpanPlan plan_spans(const SpanBatch& a, const KeyPart* keys, size_t nkeys, SpanScratch& scratch,
                    SpanGroup* groups, SpanPart* parts) {
    std::vector<uint32_t>&rows = scratch.rows, &cuts = scratch.cuts, &waves = scratch.waves;
    rows.resize(a.n);
    for (size_t k = 0; k < a.n; ++k) {
        const size_t i = a.at(k);
        rows[k] = (uint32_t)span_rows(a.len[i], a.aad_len ? a.aad_len[i] : 0);
    }
    cuts.clear();
    uint32_t row = 0, group = 0;
    for (size_t q = 0; q < nkeys; ++q) {
        waves.resize(group + keys[q].groups + 1);
        cut_key(keys[q], row, rows.data() + keys[q].first, cuts, waves.data() + group);
        row += (uint32_t)keys[q].rows;
        group += keys[q].groups;
    }
    waves[group] = (uint32_t)cuts.size();
    cuts.push_back(row);

    SpanPlan plan{0, 0};
    uint32_t g = 0, np = 0;
    row = 0;
    for (size_t q = 0; q < nkeys; ++q) {
        bool begun = false;  // workgroup g has a part already
        uint32_t wave = 0;   // of the workgroup, the one with `row`
        for (size_t k = keys[q].first; k < keys[q].first + keys[q].n; ++k) {
            const size_t i = a.at(k);
            SpanPart c;
            c.src = (const uint8_t*)a.src[i];
            c.dst = (uint8_t*)a.dst[i];
            c.len = a.len[i];
            c.aad_len = a.aad_len ? a.aad_len[i] : 0;
            c.aad = c.aad_len ? (const uint8_t*)a.aad[i] : nullptr;
            c.index = (uint32_t)i;
            c.first_row = row;
            c.rows = rows[k];
            c.slot = np;
            const uint32_t chunk_end = row + rows[k];
            while (row < chunk_end) {
                SpanGroup& d = groups[g];
                const uint32_t *cut = cuts.data() + waves[g], n = waves[g + 1] - waves[g];
                if (!begun) {
                    begun = true;
                    wave = 0;
                    d.kt = keys[q].tables;
                    d.first_row = row;
                    d.part = np;
                    d.waves = n;
                    for (uint32_t w = 0; w <= n; ++w) d.cut[w] = cut[w] - row;
                    d.pad_ = 0;
                }
                const uint32_t end = cut[n] < chunk_end ? cut[n] : chunk_end;
                while (cut[wave + 1] <= row) ++wave;
                const uint32_t first = wave;
                while (cut[wave + 1] < end) ++wave;
                c.waves = (wave - first + 1) << 8 | first;
                c.own_slot = np;
                parts[np++] = c;
                row = end;
                if (end == cut[n]) {
                    d.nparts = np - d.part;
                    if (d.nparts > plan.longest) plan.longest = d.nparts;
                    begun = false;
                    ++g;
                }
            }
            for (uint32_t p = c.slot; p < np; ++p) parts[p].slots = np - c.slot;
        }
    }
    plan.nparts = np;
    return plan;
}

// Fills in a launch's map as far as it goes: the keys, if there are several and they have a place each, and
// the workgroups' packets one behind the other, if no list is longer than what is held of one and all of them
// together are read from host memory.  What is not is zero: a map goes out whole, as a kernel argument.  Returns
// what is filled in; *bytes: the packets'.
inline uint32_t map_spans(const KeyPart* keys, size_t nkeys, const SpanGroup* groups, const SpanPlan& plan,
                          SpanMap* map, size_t* bytes) {
    uint32_t filled = nkeys > 1 && nkeys <= kSpanMapKeys ? kSpanKeysMapped : 0, g = 0;
    size_t at = 0;
    *map = SpanMap{};
    for (size_t q = 0; q < nkeys; ++q) {
        if (g + keys[q].groups > kSpanMapGroups) return 0;
        if (filled) map->key[q] = keys[q].tables;
        for (uint32_t end = g + keys[q].groups; g < end; ++g) {
            map->place[g] = (filled ? (uint32_t)q << SpanMap::kKeyShift : 0) |
                            (groups[g].nparts & 63) << SpanMap::kLengthShift | ((uint32_t)(at / kPacketAlign) & 0xFFFF);
            at += packet_bytes(groups[g].nparts);
        }
    }
    if (plan.longest <= kSpanLdsParts && at <= kSpanHostBytes) filled |= kSpanPlaced;
    *bytes = at;
    return filled;
}
static_assert(kSpanHostBytes / kPacketAlign <= 1u << SpanMap::kLengthShift, "places of packets");
static_assert(kSpanLdsParts < 1u << (SpanMap::kKeyShift - SpanMap::kLengthShift), "lengths of lists");

}  // namespace pgcm
