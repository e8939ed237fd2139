// Cuts thousands of random batches into spans and checks what span_kernel assumes when it reads the
// result; run under sanitizers, with arrays of exactly the sizes the host allots.  Prints how many
// batches, workgroups and parts it looked at.  Test infrastructure.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "pgcm_spans.h"

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

#define CHECK(cond)                                                                       \
    do {                                                                                  \
        if (!(cond)) {                                                                    \
            printf("batch %llu, line %d: %s\n", (unsigned long long)g_batch, __LINE__, #cond); \
            exit(1);                                                                      \
        }                                                                                 \
    } while (0)
static uint64_t g_batch, g_groups, g_parts, g_shared, g_even;

static void check(const std::vector<uint64_t>& len, const std::vector<uint32_t>& aad_len,
                  const std::vector<uint32_t>& order, std::vector<KeyPart>& keys, uint32_t num_cu) {
    const size_t n = order.size();
    const std::vector<const void*> ptrs(len.size(), nullptr);
    std::vector<void*> dst(len.size(), nullptr);
    const SpanBatch b{n, order.data(), ptrs.data(), aad_len.empty() ? nullptr : aad_len.data(),
                      ptrs.data(), len.data(), dst.data()};
    auto rows_of = [&](size_t k) {
        return span_rows(len[order[k]], aad_len.empty() ? 0 : aad_len[order[k]]);
    };
    uint64_t total = 0;
    for (KeyPart& key : keys) {
        key.rows = 0;
        for (size_t k = key.first; k < key.first + key.n; ++k) key.rows += rows_of(k);
        total += key.rows;
    }
    const uint32_t ngroups = deal_groups(keys.data(), keys.size(), num_cu);
    uint32_t dealt = 0;
    for (const KeyPart& key : keys) {
        CHECK(key.groups >= 1 && key.groups <= key.rows);
        dealt += key.groups;
    }
    CHECK(dealt == ngroups && ngroups <= num_cu + keys.size() - 1);

    // as a context keeps it: what is in it is what the last batch left; once reserved it does not grow,
    // for keys that share a launch even if it was reserved for one chunk
    static SpanScratch kept;
    SpanScratch fresh;
    const bool shared = share_launch(keys.size(), n, total, num_cu);
    SpanScratch& scratch = shared ? fresh : kept;
    const size_t reserved = shared ? 1 : n;
    scratch.reserve(reserved, num_cu);
    const size_t held = scratch.capacity();
    std::vector<SpanGroup> groups(ngroups);
    std::vector<SpanPart> parts(n + ngroups);
    const SpanPlan plan = plan_spans(b, keys.data(), keys.size(), scratch, groups.data(), parts.data());
    CHECK(plan.nparts >= n && plan.nparts <= n + ngroups);
    CHECK(scratch.capacity() == held && ngroups <= span_most_groups(num_cu));
    CHECK(span_image_bytes(n + ngroups, ngroups) <= span_stage_bytes(reserved, num_cu));
    CHECK((sizeof(ArriveSlot) * plan.nparts + 255) / 256 * 256 + span_image_bytes(plan.nparts, ngroups) <=
          span_work_bytes(reserved, num_cu, 0));
    g_shared += shared && keys.size() > 1;

    // the workgroups tile the rows and the parts, and their wavefronts tile each of them
    uint64_t row = 0;
    uint32_t part = 0, longest = 0, g = 0;
    for (const KeyPart& key : keys) {
        for (uint32_t k = 0; k < key.groups; ++k, ++g) {
            const SpanGroup& d = groups[g];
            CHECK(d.kt == key.tables && d.first_row == row && d.part == part);
            CHECK(d.waves >= 1 && d.waves <= kWavesPerGroup && d.cut[0] == 0);
            for (uint32_t w = 0; w < d.waves; ++w) CHECK(d.cut[w] < d.cut[w + 1]);
            CHECK(d.nparts >= 1 && part + d.nparts <= plan.nparts);
            // Shares cut with regard to the workgroup's pieces.  A share but the last is full up to the half
            // rows of a piece of a row, less one, so that with limit >= mean + kPieceHalfRows + 2 no more
            // are begun than there are wavefronts; the limit is the first tried that will do.
            const uint64_t most = (uint64_t)key.groups * kWavesPerGroup;
            if ((key.rows > most * kFineRows || key.n > 2 * most) && key.rows <= most * kEvenRows &&
                kEvenGroups * key.n <= (uint64_t)kEvenChunks * key.groups && d.nparts > 1) {
                const uint32_t rows = d.cut[d.waves], w = rows < kWavesPerGroup ? rows : kWavesPerGroup;
                uint32_t enough = (2 * rows + kPieceHalfRows * (d.nparts + w)) / w + kPieceHalfRows + 3;
                enough += 1 + enough / 64;
                for (uint32_t i = 0; i < d.waves; ++i) {
                    uint32_t cost = 2 * (d.cut[i + 1] - d.cut[i]);
                    for (uint32_t q = 0; q < d.nparts; ++q) {
                        const SpanPart& c = parts[part + q];
                        cost += i >= (c.waves & 0xFF) && i < (c.waves & 0xFF) + (c.waves >> 8) ? kPieceHalfRows : 0;
                    }
                    CHECK(cost <= enough);
                }
                ++g_even;
            }
            row += d.cut[d.waves];
            part += d.nparts;
            if (d.nparts > longest) longest = d.nparts;
        }
    }
    CHECK(row == total && part == plan.nparts && longest == plan.longest);

    // every chunk: its parts are consecutive and cover its rows, in workgroups of its key
    row = 0, part = 0, g = 0;
    uint32_t in_group = 0;  // parts of g seen
    for (const KeyPart& key : keys) {
        uint64_t key_end = row + key.rows;
        for (size_t k = key.first; k < key.first + key.n; ++k) {
            const uint32_t first = part;
            const uint64_t chunk_end = row + rows_of(k), chunk_row = row;
            while (row < chunk_end) {
                const SpanPart& c = parts[part];
                const SpanGroup& d = groups[g];
                const uint64_t group_end = (uint64_t)d.first_row + d.cut[d.waves];
                const uint64_t end = group_end < chunk_end ? group_end : chunk_end;
                CHECK(d.kt == key.tables && d.part + in_group == part);
                CHECK(c.index == order[k] && c.len == len[order[k]]);
                CHECK(c.first_row == chunk_row && c.rows == rows_of(k));
                CHECK(c.slot == first && c.own_slot == part);
                // its wavefronts are those with rows of it
                const uint32_t w0 = c.waves & 0xFF, nw = c.waves >> 8;
                CHECK(nw >= 1 && w0 + nw <= d.waves);
                for (uint32_t w = 0; w < d.waves; ++w) {
                    const uint64_t from = (uint64_t)d.first_row + d.cut[w],
                                   to = (uint64_t)d.first_row + d.cut[w + 1];
                    CHECK((from < end && to > row) == (w >= w0 && w < w0 + nw));
                    // a wavefront starts with the last part that does not begin behind its first row
                    if (from >= row && from < end)
                        CHECK(in_group + 1 == d.nparts || parts[part + 1].first_row > from);
                }
                CHECK((chunk_end - end) / kRowHopEntries < kFarHopEntries);
                row = end;
                ++part, ++in_group;
                if (end == group_end) {
                    CHECK(in_group == d.nparts);
                    in_group = 0, ++g;
                }
            }
            for (uint32_t p = first; p < part; ++p) CHECK(parts[p].slots == part - first);
        }
        CHECK(row == key_end);
    }
    CHECK(g == ngroups);
    ++g_batch, g_groups += ngroups, g_parts += plan.nparts;
}

int main() {
    // keys are only told apart by it
    const KeyTables* const tables = reinterpret_cast<const KeyTables*>((uintptr_t)1 << 32);
    const uint32_t cus[] = {256, 256, 256, 1, 2, 32, 304};
    for (int trial = 0; trial < 6000; ++trial) {
        const uint32_t num_cu = cus[below(7)];
        const size_t n = trial % 50 == 0 ? log_between(2000, 20000) : log_between(1, 700);
        const int kind = trial % 6;
        const double lo = log_between(1, 300000), hi = lo * log_between(1, 1000);
        std::vector<uint64_t> len(n);
        std::vector<uint32_t> aad_len(below(3) ? n : 0), key_of(n), order;
        // as many keys as compute units at most
        const size_t nkeys = below(2) ? 1 : 1 + below(below(4) && num_cu > 6 ? 6 : num_cu);
        for (size_t i = 0; i < n; ++i) {
            len[i] = kind == 0   ? log_between(lo, hi)
                     : kind == 1 ? 1024 * below(20) + below(3) * 16 + below(3)
                     : kind == 2 ? 64 * 1024 * (1 + below(4))
                     : kind == 3 ? (below(5) ? below(2000) : log_between(1000, 3e7))
                     : kind == 4 ? (uint64_t)lo
                                 : 1024 * (1 + below(40)) - 16 - 16 * below(3);
            if (n > 700 && len[i] > 300000) len[i] %= 300000;
            if (!aad_len.empty()) aad_len[i] = below(4) ? below(80) : below(1200);
            key_of[i] = (uint32_t)(below(3) ? below(nkeys) : 0);
        }
        std::vector<KeyPart> keys;
        for (size_t q = 0; q < nkeys; ++q) {
            KeyPart key{nullptr, reinterpret_cast<const KeyTables*>((uintptr_t)tables + 16 * q), (uint32_t)(10 + 2 * below(3)), order.size(), 0, 0, 0, 0};
            for (size_t i = 0; i < n; ++i)
                if (key_of[i] == q) order.push_back((uint32_t)i);
            key.n = order.size() - key.first;
            if (key.n) keys.push_back(key);
        }
        check(len, aad_len, order, keys, num_cu);
    }
    // about a chunk a workgroup, of mixed lengths: shares cut with regard to the workgroup's pieces
    for (int trial = 0; trial < 120; ++trial) {
        const uint32_t num_cu = trial % 2 ? 256 : cus[below(7)];
        const size_t n = 1 + below(3 * num_cu / 2);
        const double rows = (double)num_cu * kWavesPerGroup * (double)(kFineRows + below(kEvenRows)) / n;
        std::vector<uint64_t> len(n);
        std::vector<uint32_t> order(n);
        for (size_t i = 0; i < n; ++i) {
            len[i] = trial % 3 ? log_between(rows * 256, rows * 4096) : (uint64_t)(rows * 1024);
            order[i] = (uint32_t)i;
        }
        std::vector<KeyPart> keys{KeyPart{nullptr, tables, 14, 0, n, 0, 0, 0}};
        check(len, {}, order, keys, num_cu);
    }
    // the longest chunk that goes in spans: as many rows as there are powers of H for
    {
        const uint64_t rows = (uint64_t)kRowHopEntries * kFarHopEntries - 3;
        std::vector<KeyPart> keys{KeyPart{nullptr, tables, 14, 0, 2, 0, 0, 0}};
        check({rows * 16 * kRowBlocks, 5}, {1024, 1025}, {1, 0}, keys, 256);
    }
    CHECK(g_even > 10000);
    printf("batches %llu, %llu of them of keys that share a launch, workgroups %llu, parts %llu\n",
           (unsigned long long)g_batch, (unsigned long long)g_shared, (unsigned long long)g_groups,
           (unsigned long long)g_parts);
    return 0;
}
