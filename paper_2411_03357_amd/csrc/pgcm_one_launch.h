// How a batch of few chunks is cut for the kernels that do it in one launch (burst_kernel, swap_kernel).
// Host only, plain C++.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include "pgcm_types.h"

namespace pgcm {

// The caller's arrays as far as the shape depends on them.
struct ShapeBatch {
    size_t n;
    const uint32_t* order;  // chunk k of the batch is the caller's chunk order[k]; null: chunk k
    const uint32_t* aad_len;
    const uint64_t* len;

    size_t at(size_t k) const { return order ? order[k] : k; }
    uint32_t aad(size_t i) const { return aad_len ? aad_len[i] : 0; }
};

// How a batch is cut for the one-launch path, if it takes it.
struct SwapShape {
    bool burst;                               // burst_kernel
    bool alone;                               // every chunk has one workgroup
    // burst: a workgroup's passes for unit_power, and what a chunk's first workgroup may have beyond them
    uint32_t unit_power, wave_power, groups, spare;
};

inline uint32_t swap_groups(const ShapeBatch& a, size_t i, uint32_t unit_power, uint32_t wave_power) {
    const uint32_t lead = swap_lead_blocks(a.aad(i), wave_power < 4);
    const uint64_t blocks = (a.len[i] + 15) / 16 + lead;
    const uint64_t units = (blocks + ((uint64_t)1 << unit_power) - 1) >> unit_power;
    const uint64_t groups = (units + ((uint64_t)1 << wave_power) - 1) >> wave_power;
    return groups == 0 ? 1 : (uint32_t)groups;
}

// burst_kernel: the passes that a chunk takes, and its workgroups if they make so many each, the first of
// them up to `spare` more
inline uint64_t burst_blocks(const ShapeBatch& a, size_t i) {
    return (a.len[i] + 15) / 16 + swap_lead_blocks(a.aad(i), true);
}
inline uint64_t burst_passes(uint64_t blocks, uint32_t wave_power) {
    const uint32_t shift = 4 + wave_power;
    return (blocks + ((uint64_t)1 << shift) - 1) >> shift;
}
inline uint64_t burst_groups(uint64_t of_chunk, uint32_t passes, uint32_t spare) {
    return of_chunk <= passes + spare ? 1 : (of_chunk - spare + passes - 1) / passes;
}

// What workgroups of sixteen wavefronts may make, in the order in which it is looked for: one pass, one and
// a spare one for a chunk's first workgroup, two, and so on to kSweptPasses with none to spare.  A later
// choice never takes more workgroups than an earlier one.
struct BurstChoice {
    uint32_t passes, spare;
};
constexpr uint32_t kBurstChoices = 2 * kSweptPasses - 1;
constexpr BurstChoice burst_choice(uint32_t i) { return BurstChoice{i / 2 + 1, i % 2}; }

// Workgroups of chunks of so many passes each, fewer than 2^28: multiplied by the passes' inverse, rounded
// up, which is exact for these and goes several chunks at a time.
inline uint64_t burst_groups_of_all(const uint32_t* of_chunk, size_t n, BurstChoice c) {
    const uint64_t inverse = (((uint64_t)1 << 32) + c.passes - 1) / c.passes;
    uint64_t sum = 0;
    for (size_t k = 0; k < n; ++k) {
        const uint64_t g = ((of_chunk[k] - c.spare + c.passes - 1) * inverse) >> 32;
        sum += of_chunk[k] <= c.passes + c.spare ? 1 : g;
    }
    return sum;
}

// The first choice with which n chunks, of `passes` passes in all, have at most `most` workgroups, n <= most;
// groups(choice): how many they have.  False: none.  A chunk has at least (its passes - spare) / passes
// workgroups, which bounds the choice from below, and mostly hits it; the rest is bisection, so that the
// chunks are gone over seven times at most.  With all choices in turn a call's host time was up to 30 us
// longer: 256 chunks that fit none 30 us, now 0.1; 256 of 64 KiB 29, now 0.25; 200 of 30 to 60 KB, where
// it takes the bisection, 15, now 1.8.
template <class Groups>
inline bool first_burst_choice(uint64_t passes, size_t n, uint64_t most, Groups groups, BurstChoice* choice,
                               uint64_t* total) {
    if (passes > kSweptPasses * most) return false;
    const uint64_t least = passes > n ? (passes - n + most - 1) / most : 0;
    uint32_t low = least > 1 ? 2 * (uint32_t)(least - 1) : 0;  // everything before it has too many
    if (passes > burst_choice(low).passes * most) ++low;
    uint32_t fits = low;
    *total = groups(burst_choice(low));
    if (*total > most) {
        fits = kBurstChoices - 1;
        if (low == fits || (*total = groups(burst_choice(fits))) > most) return false;
        while (fits - low > 1) {
            const uint32_t mid = (low + fits) / 2;
            const uint64_t t = groups(burst_choice(mid));
            if (t > most) low = mid;
            else fits = mid, *total = t;
        }
    }
    *choice = burst_choice(fits);
    return true;
}

// Passes of 64 blocks, or of 128, if no workgroup has to make more than one.  Their workgroups multiply every
// word by its own power and have no rows to fold, and four or eight wavefronts bring the tables in and make
// their blocks sooner than sixteen do.  Of 64 where there are compute units for them, unless only of 128 a
// chunk's shares are added up in one set (kArriveSet; 40 KiB in 20 workgroups 5.52 us, in 40 5.66).  Per call,
// passes of 256, 128 and 64 blocks: 16 KiB 6.4, 5.5, 5.1; 96 KiB 6.6, 5.9, 5.6; 250 KiB 7.0, 5.9, 5.6; 16 of
// 12 KiB 7.4, 6.9, 6.2; 320 KiB 7.1, 6.0; 20 of 20 KiB 7.4, 6.9; three of 100 KiB, which 256 blocks have in one
// set each, 7.2, 7.1.  Two workgroups on a compute unit are longer (10 of 90 KiB 8.8 instead of 7.2, three of 256 KiB 8.8
// instead of 7.8, two of 450 KiB 8.6 instead of 7.5), and were so, as a first workgroup with a pass more and two passes of
// 128 blocks (320 KiB 8.4, 700 KiB 8.8 instead of 7.6), when up to eight wavefronts had two round tables to bring in.
inline bool one_pass_each(const ShapeBatch& a, uint32_t most, SwapShape* shape) {
    uint64_t total[2] = {0, 0}, longest[2] = {0, 0};
    for (size_t k = 0; k < a.n; ++k) {
        const uint64_t blocks = burst_blocks(a, a.at(k));
        for (uint32_t w = 0; w < 2; ++w) {
            const uint64_t groups = burst_groups(burst_passes(blocks, 2 + w), 1, 0);
            total[w] += groups;
            if (groups > longest[w]) longest[w] = groups;
        }
    }
    const bool four = total[0] <= most && (longest[0] <= kArriveSet || longest[1] > kArriveSet);
    if (!four && total[1] > most) return false;
    const uint64_t groups = total[four ? 0 : 1];
    *shape = SwapShape{true, groups == a.n, 1, four ? 2u : 3u, (uint32_t)groups, 0};
    return true;
}

// Batches of short chunks, and others of at most sixteen passes for every compute unit, go to burst_kernel.
// As long as there is a compute unit for every short chunk, a workgroup takes a whole one, with no
// more wavefronts than it has blocks for.  Up to kArgChunks of them, one longer than a pass of 256 blocks, go in
// workgroups of one pass instead (one_pass_each), if `spread` lets them, which it does where the stream has slots for
// them at hand (ShortStreams): back to back and waited for, one of 8 KiB 7.0 -> 5.1 and 17.5 -> 15.5 us, with AAD
// 8.8 -> 5.0 and 19.2 -> 15.5, 32 of 8 KiB 7.6 -> 6.1 and 18.5 -> 16.7, 64 of 4 KiB with AAD 7.5 -> 6.5 and 18.6 -> 17.7,
// on any stream that has them.  More of them are no better off (120 of up to 8 KiB 9.1 -> 9.2, decrypted 8.7 -> 9.1).  Chunks
// of 129 to 256 blocks alone have a workgroup each, which dates from when up to eight wavefronts had two round tables to bring
// in (16 of 4 KiB 6.6 -> 6.3 and 18.5 -> 18.8, 64 of them decrypted 6.7 -> 7.0); passes of 64 blocks would be better now (one
// of 4 KiB 5.7 -> 4.7 and 15.9 -> 15.1, 16 of them 6.0 -> 5.8 and 17.0 -> 16.7, 64 of them 6.0 -> 5.9 and 17.3 -> 17.2,
// decrypted 6.1 -> 6.0 and 17.3 either way), of 128 not (5.5, 6.8, 6.7 and 6.7).
// Of more chunks than compute units, two workgroups share one: if `spread`, of at most
// eight wavefronts and one pass, of which the longer chunks take several, if 512 of them do; otherwise of
// sixteen and one pass, if 512 of these do (346 chunks of 1.6 to 8.1 KB 10.9 us, a workgroup each 13.6; 450 of up
// to 8 KB 10.6, 13.2); otherwise of sixteen and a whole chunk, as also where a launch has to clear the slots (300 of up
// to 8 KB on a stream with a captured batch, when each call passed 2.8 KB of arguments, 17.4 us with several workgroups a
// chunk, 13.9 with one each; in a graph, where that launch costs less, 15.4 and 15.6: there they have several).  Longer
// chunks are spread over workgroups of four or eight that make one pass (one_pass_each), or over as many of sixteen as there
// are compute units, with the fewest passes that go: first with none spare, then with one for the first workgroup of each
// chunk, which is what a few blocks too many take (back to back and waited for, 2 MiB with AAD, 257 workgroups of two passes if none had one to spare,
// 9.9 and 20.2, in three passes 9.9 and 20.5; 8 of 256 KiB with AAD 9.9 and 20.2, in three 9.9 and 20.8), then with one more
// (2.3 to 3 MB in three 10.0, 4 MiB in four 11.7).
// What is left has more than four rows for each wavefront of the device, and takes units of eight rows or
// sixteen, a wavefront each, with a workgroup of sixteen a compute unit.  Units of sixteen rows, and those of a
// forced size, take the fewest wavefronts a workgroup, four at least, with which they still fit: chunks
// of whole 128 KiB without AAD, which eight wavefronts with units of sixteen rows cover, are a block
// ("block -1") too long for sixteen with units of eight, as these have no further wavefront for it.
constexpr uint32_t kLongUnitPower = kRowPower + 3;
// forced: log2 of the blocks of a unit, or 0; all_small: no chunk is longer than kSmallChunkBytes; spread: of
// these a chunk may have several workgroups, for which the batch needs slots.
inline bool swap_shape(const ShapeBatch& a, uint32_t num_cu, bool one_launch, uint32_t forced, bool all_small,
                       bool spread, SwapShape* shape) {
    if (a.n > kSmallMaxChunks || (!all_small && !one_launch)) return false;
    uint64_t total = 0;
    const uint32_t most = num_cu < kSwapChunkGroups ? num_cu : kSwapChunkGroups;
    if (all_small) {
        uint64_t most_blocks = 0, of_eight = 0, of_sixteen = 0;
        for (size_t k = 0; k < a.n; ++k) {
            const uint64_t blocks = burst_blocks(a, a.at(k));
            if (blocks > most_blocks) most_blocks = blocks;
            of_eight += burst_groups(burst_passes(blocks, 3), 1, 0);
            of_sixteen += burst_groups(burst_passes(blocks, 4), 1, 0);
        }
        uint32_t wp = 2, passes = kFoldPasses;
        while (wp < 4 && most_blocks > (uint64_t)16 << wp) ++wp;
        if (spread && a.n <= kArgChunks && a.n <= most && most_blocks > (uint64_t)16 << wp &&
            one_pass_each(a, most, shape))
            return true;
        total = a.n;
        const bool apart = spread && a.n > num_cu;
        if (apart && wp > 2 && of_eight <= kSwapMaxGroups) wp = 3, passes = 1, total = of_eight;
        else if (apart && wp == 4 && of_sixteen <= kSwapMaxGroups) passes = 1, total = of_sixteen;
        *shape = SwapShape{true, total == a.n, passes, wp, (uint32_t)total, 0};
        return true;
    }
    if (a.n > most) return false;
    uint64_t bytes = 0;
    for (size_t k = 0; k < a.n; ++k) bytes += a.len[a.at(k)];
    if (bytes > (uint64_t)most * kWavesPerGroup * kUnitBytes) return false;
    if (forced <= kMinUnitPower) {
        uint32_t of_chunk[kSwapChunkGroups];
        uint64_t passes = 0;
        for (size_t k = 0; k < a.n; ++k) {
            of_chunk[k] = (uint32_t)burst_passes(burst_blocks(a, a.at(k)), 4);
            passes += of_chunk[k];
        }
        BurstChoice c;
        if (passes <= most && one_pass_each(a, most, shape)) return true;
        if (first_burst_choice(
                passes, a.n, most, [&](BurstChoice b) { return burst_groups_of_all(of_chunk, a.n, b); },
                &c, &total)) {
            *shape = SwapShape{true, total == a.n, c.passes, 4, (uint32_t)total, c.spare};
            return true;
        }
    }
    auto groups = [&](uint32_t unit_power, uint32_t wave_power, uint32_t* most_of_one) {
        uint64_t sum = 0;
        *most_of_one = 0;
        for (size_t k = 0; k < a.n; ++k) {
            const uint32_t g = swap_groups(a, a.at(k), unit_power, wave_power);
            if (g > *most_of_one) *most_of_one = g;
            sum += g;
        }
        return sum;
    };
    uint32_t up = forced ? forced : kLongUnitPower, wp = 4, longest = 0;
    if (up > kUnitPower) return false;
    while ((total = groups(up, wp, &longest)) > most) {
        if (forced || up == kUnitPower) return false;
        ++up;
    }
    while ((forced || up == kUnitPower) && wp > 2) {
        uint32_t l = 0;
        const uint64_t t = groups(up, wp - 1, &l);
        if (t > most) break;
        --wp, total = t, longest = l;
    }
    *shape = SwapShape{false, longest <= 1, up, wp, (uint32_t)total, 0};
    return true;
}

// Where units of swap_kernel and spans could both take a batch of so many rows: are units no longer?  Spans
// have fewer rows for a wavefront, as units are a power of two, but their descriptors are planned on the
// host.  Units of eight rows take 46 us, whatever part of them is filled; spans, at the clock of the machine that both
// were timed on, 18 and 3.75 a row of a wavefront, and 5 to 8 more on the host, which shows where a call is waited for
// (back to back / waited for, units and spans: 12 of 2 MiB 46.3 / 57.0, 42.3 / 58.9; one of 28 MB
// 46.6 / 57.1, 45.9 / 62.4; 14 of 2 MiB decrypted 46.1 / 57.1, 42.7 / 61.6; one of 31 MB decrypted
// 46.2 / 56.9, 45.3 / 63.8).  Units of sixteen rows take 49 with eight wavefronts a workgroup (one of 32 MiB
// 49.2 / 59.6, 51.2 / 67.8, decrypted 48.6 / 59.3, 48.0 / 66.6; 256 of 128 KiB 49.3 / 64.0, 49.7 / 68.7, decrypted
// 48.7 / 63.7, 46.3 / 67.8; 228 of them, 7.1 rows a wavefront, 49.0 / 64.0, 47.3 / 67.7) and 81 with sixteen, and spans no
// longer than that.
inline bool units_before_spans(const SwapShape& s, uint64_t rows, uint64_t wave_slots) {
    if (s.unit_power == kLongUnitPower) return 2 * rows >= 13 * wave_slots;
    return s.wave_power == 3 && 2 * rows >= 15 * wave_slots;
}

}  // namespace pgcm
