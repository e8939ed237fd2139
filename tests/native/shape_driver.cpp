// Cuts thousands of random batches for the one-launch kernels and compares the shape with the one found by
// trying every choice in turn with plain divisions, as the choice is defined; run under sanitizers.
// Prints how many batches went which way, and the most often that chunks were gone over for one batch.
// Test infrastructure.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "pgcm_one_launch.h"

using namespace pgcm;

static uint64_t state = 88172645463325252ull;
static uint64_t rnd() {
    state ^= state << 13;
    state ^= state >> 7;
    state ^= state << 17;
    return state;
}
static uint64_t below(uint64_t n) { return (rnd() >> 11) % n; }
static uint64_t log_between(double lo, double hi) {
    return (uint64_t)(lo * std::pow(hi / lo, (double)(rnd() >> 11) / 9007199254740992.0));
}

static unsigned long long g_batch, g_spread, g_words, g_bursts, g_swept, g_units, g_none, g_most;
#define CHECK(cond)                                                      \
    do {                                                                 \
        if (!(cond)) {                                                   \
            printf("batch %llu, line %d: %s\n", g_batch, __LINE__, #cond); \
            exit(1);                                                     \
        }                                                                \
    } while (0)

// workgroups if each makes so many passes over 64 << wave_power / 4 blocks, a chunk's first up to `spare` more
static uint64_t groups_of(const ShapeBatch& a, uint64_t pass_blocks, uint64_t passes, uint64_t spare) {
    uint64_t sum = 0;
    for (size_t k = 0; k < a.n; ++k) {
        const size_t i = a.at(k);
        const uint64_t aad = a.aad(i), lead = aad == 0 ? 0 : aad <= 16 || aad > 1024 ? 1 : (aad + 15) / 16;
        const uint64_t blocks = (a.len[i] + 15) / 16 + lead;
        uint64_t left = (blocks + pass_blocks - 1) / pass_blocks, g = 1;
        for (left = left > passes + spare ? left - (passes + spare) : 0; left > 0;
             left = left > passes ? left - passes : 0)
            ++g;
        sum += g;
    }
    return sum;
}

static uint64_t most_groups(const ShapeBatch& a, uint64_t pass_blocks) {
    uint64_t most = 0;
    for (size_t k = 0; k < a.n; ++k) {
        const uint64_t i = a.at(k), g = groups_of(ShapeBatch{1, nullptr, a.aad_len ? a.aad_len + i : nullptr, a.len + i},
                                                  pass_blocks, 1, 0);
        if (g > most) most = g;
    }
    return most;
}

// the passes of a chunk's first workgroup, which makes the most
static uint64_t most_passes(const ShapeBatch& a, const SwapShape& s) {
    uint64_t most = 0;
    for (size_t k = 0; k < a.n; ++k) {
        const uint64_t of_chunk = burst_passes(burst_blocks(a, a.at(k)), s.wave_power);
        const uint64_t g = s.alone ? 1 : burst_groups(of_chunk, s.unit_power, s.spare);
        CHECK(of_chunk >= (g - 1) * s.unit_power);
        const uint64_t first = of_chunk - (g - 1) * s.unit_power;
        if (first > most) most = first;
    }
    return most;
}

static void check(const ShapeBatch& a, uint32_t num_cu, uint32_t forced) {
    uint64_t bytes = 0, longest = 0;
    for (size_t k = 0; k < a.n; ++k) {
        bytes += a.len[a.at(k)];
        if (a.len[a.at(k)] > longest) longest = a.len[a.at(k)];
    }
    const bool all_small = longest <= kSmallChunkBytes;
    SwapShape s{};
    const bool spread = g_batch % 2 != 0;
    const bool goes = swap_shape(a, num_cu, true, forced, all_small, spread, &s);
    ++g_batch;
    if (all_small) {
        CHECK(goes == (a.n <= kSmallMaxChunks));
        if (!goes) return;
        CHECK(s.burst && s.spare == 0 && s.groups >= a.n && s.groups <= kSwapMaxGroups);
        CHECK(s.alone == (s.groups == a.n));
        // a pass of 64 or 128 blocks for every workgroup of few chunks, one of them longer than 256
        const uint32_t most = num_cu < kSwapChunkGroups ? num_cu : kSwapChunkGroups;
        if (spread && a.n <= kArgChunks && a.n <= most && most_groups(a, 256) > 1 && groups_of(a, 128, 1, 0) <= most) {
            const uint64_t of_four = groups_of(a, 64, 1, 0);
            CHECK(!s.alone && s.unit_power == 1 && s.wave_power == (of_four <= most ? 2u : 3u));
            CHECK(s.groups == (of_four <= most ? of_four : groups_of(a, 128, 1, 0)) && most_passes(a, s) == 1);
            ++g_spread;
            return;
        }
        if (s.alone) CHECK(groups_of(a, (uint64_t)16 << s.wave_power, s.unit_power, 0) == a.n || a.n > num_cu);
        if (spread && a.n > num_cu && s.wave_power > 2) {
            const uint64_t of_eight = groups_of(a, 128, 1, 0), of_sixteen = groups_of(a, 256, 1, 0);
            CHECK(s.groups == (of_eight <= kSwapMaxGroups     ? of_eight
                               : of_sixteen <= kSwapMaxGroups ? of_sixteen
                                                              : a.n));
            CHECK(s.wave_power == (of_eight <= kSwapMaxGroups ? 3u : 4u) && (s.alone || s.unit_power == 1));
        } else {
            CHECK(s.alone);
        }
        // what the kinds of burst_kernel are compiled for
        CHECK(most_passes(a, s) <= (s.wave_power < 4 ? 1 : s.groups > num_cu ? kFoldPasses - 1 : kFoldPasses));
        ++g_bursts;
        return;
    }
    const uint32_t most = num_cu < kSwapChunkGroups ? num_cu : kSwapChunkGroups;
    const bool considered = a.n <= most && bytes <= (uint64_t)most * kWavesPerGroup * kUnitBytes;
    bool found = false;
    // a pass of 64 or 128 blocks for every workgroup
    for (uint32_t wp = 2; considered && forced <= kMinUnitPower && wp <= 3 && !found; ++wp) {
        const uint64_t total = groups_of(a, 16u << wp, 1, 0);
        if (total > most || (wp == 2 && most_groups(a, 64) > kArriveSet && most_groups(a, 128) <= kArriveSet)) continue;
        CHECK(goes && s.burst && s.wave_power == wp && s.unit_power == 1 && s.spare == 0 && s.groups == total);
        CHECK(s.alone == (total == a.n) && most_passes(a, s) == 1);
        ++g_words;
        return;
    }
    for (uint32_t passes = 1; considered && forced <= kMinUnitPower && passes <= kSweptPasses && !found; ++passes)
        for (uint32_t spare = 0; spare <= (passes < kSweptPasses ? 1u : 0u) && !found; ++spare) {
            const uint64_t total = groups_of(a, 256, passes, spare);
            if (total > most) continue;
            found = true;
            CHECK(goes && s.burst && s.wave_power == 4);
            CHECK(s.unit_power == passes && s.spare == spare && s.groups == total);
            CHECK(s.alone == (total == a.n));
            CHECK(s.groups <= num_cu);
            CHECK(most_passes(a, s) <= (passes + spare <= kFoldPasses ? kFoldPasses : kSweptPasses));
            // as the descriptors are filled in
            uint64_t sum = 0;
            for (size_t k = 0; k < a.n; ++k)
                sum += burst_groups(burst_passes(burst_blocks(a, a.at(k)), 4), passes, spare);
            CHECK(sum == total);
            ++(passes > kFoldPasses ? g_swept : g_bursts);
        }
    // how often the chunks are gone over
    if (considered) {
        std::vector<uint32_t> of_chunk(a.n);
        uint64_t passes = 0, total = 0;
        for (size_t k = 0; k < a.n; ++k)
            passes += of_chunk[k] = (uint32_t)burst_passes(burst_blocks(a, a.at(k)), 4);
        unsigned long long times = 0;
        BurstChoice c;
        const bool fits = first_burst_choice(
            passes, a.n, most,
            [&](BurstChoice b) {
                ++times;
                const uint64_t sum = burst_groups_of_all(of_chunk.data(), a.n, b);
                CHECK(sum == groups_of(a, 256, b.passes, b.spare));
                return sum;
            },
            &c, &total);
        CHECK(fits == found || forced > kMinUnitPower);
        if (times > g_most) g_most = times;
    }
    if (found) return;
    if (!goes) {
        ++g_none;
        return;
    }
    ++g_units;
    CHECK(considered && !s.burst && s.groups <= most && s.unit_power <= kUnitPower && s.wave_power >= 2);
    // the smallest size that would go with sixteen wavefronts, and then the fewest wavefronts
    auto units_fit = [&](uint32_t up, uint32_t wp) {
        uint64_t sum = 0;
        for (size_t k = 0; k < a.n; ++k) sum += swap_groups(a, a.at(k), up, wp);
        return sum <= most;
    };
    uint32_t up = forced ? forced : kMinUnitPower + 1, wp = 4;
    while (!forced && up < kUnitPower && !units_fit(up, wp)) ++up;
    while (wp > 2 && units_fit(up, wp - 1)) --wp;
    CHECK(s.unit_power == up && s.wave_power == wp);
    uint64_t sum = 0;
    bool alone = true;
    for (size_t k = 0; k < a.n; ++k) {
        const uint32_t g = swap_groups(a, a.at(k), s.unit_power, s.wave_power);
        sum += g;
        alone &= g == 1;
    }
    CHECK(sum == s.groups && alone == s.alone);
}

// A chunk's first workgroup, in rows: one wavefront has the block before the chunk's first, in one of its sweeps,
// and wave_of_lead names it.
static void check_lead(uint64_t nblk, uint32_t lead, uint32_t passes, uint32_t spare) {
    const uint64_t in_chunk = (nblk + lead + 255) / 256;
    const uint32_t ngroups = (uint32_t)burst_groups(in_chunk, passes, spare);
    const uint32_t of_each = ngroups == 1 ? (uint32_t)in_chunk : passes;
    const uint32_t behind = (ngroups - 1) * of_each, have = (uint32_t)in_chunk - behind;
    CHECK(have >= 1 && have <= kSweptPasses);
    if (nblk <= ((uint64_t)behind << 8) + 256) return;  // not in rows
    const uint32_t sweeps = (have + kFoldPasses - 1) / kFoldPasses, folded = sweeps > 1 ? kFoldPasses : have;
    uint32_t found = 0;
    for (uint32_t wave = 0; wave < 16; ++wave)
        for (uint32_t sweep = 0; sweep < sweeps; ++sweep) {
            // as the kernel has it
            if (!(wave < 4 * folded && (sweep > 0 || wave / 4 >= sweeps * folded - have))) continue;
            const uint32_t m1 = behind + folded - wave / 4 + kFoldPasses * (sweeps - 1 - sweep);
            const int64_t first = (int64_t)nblk - ((int64_t)m1 << 8) + (wave & 3) * 64;
            if (first > -1 || first + 64 <= -1) continue;
            ++found;
            CHECK(wave == wave_of_lead((uint32_t)nblk, behind, folded));
        }
    CHECK(found == 1);
}

int main() {
    for (int trial = 0; trial < 20000; ++trial) {
        const uint32_t passes = 1 + (uint32_t)below(kSweptPasses), spare = passes < kSweptPasses ? (uint32_t)below(2) : 0;
        check_lead(257 + log_between(1, 256 * 256 * 8) - below(257), 1 + (uint32_t)below(64), passes, spare);
    }
    const uint32_t cus[] = {256, 256, 256, 1, 2, 32, 304};
    for (int trial = 0; trial < 20000; ++trial) {
        const uint32_t num_cu = cus[below(7)];
        const size_t n = log_between(1, trial % 4 ? 290 : 600);
        const int kind = trial % 5;
        const double lo = log_between(1, 3e6), hi = lo * log_between(1, 1000);
        const bool whole = kind == 4 && below(2);  // whole 128 KiB, which sixteen rows of eight wavefronts cover
        std::vector<uint64_t> len(n);
        std::vector<uint32_t> aad_len(!whole && below(3) ? n : 0), order(n);
        for (size_t i = 0; i < n; ++i) {
            order[i] = (uint32_t)(n - 1 - i);
            len[i] = kind == 0   ? log_between(lo, hi)
                     : kind == 1 ? below(kSmallChunkBytes + 1)
                     : kind == 2 ? 4096 * (1 + below(64)) - below(2) * 16
                     : kind == 3 ? (below(5) ? below(2000) : log_between(1000, 3e7))
                                 : whole ? (1 + below(16)) << 17
                                         : (uint64_t)lo;
            // within what is considered, mostly
            if (!whole && below(8)) len[i] = 1 + len[i] % ((size_t)64 * 1024 * num_cu / n + 9000);
            if (!aad_len.empty()) aad_len[i] = below(4) ? below(80) : below(1200);
        }
        const ShapeBatch a{n, below(2) ? order.data() : nullptr, aad_len.empty() ? nullptr : aad_len.data(),
                           len.data()};
        check(a, num_cu, below(6) ? 0 : kMinUnitPower + below(kUnitPower - kMinUnitPower + 1));
    }
    printf("batches %llu: in passes of 64 and 128 %llu, short ones %llu, other bursts %llu, in sweeps %llu, in units %llu, neither %llu; chunks gone over %llu times at most\n",
           g_batch, g_words, g_spread, g_bursts, g_swept, g_units, g_none, g_most);
    return 0;
}
