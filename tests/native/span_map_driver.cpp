// Fills in the maps of span_kernel's launches (map_spans) for batches of several sizes and numbers of keys,
// and checks what the kernel takes from one: that every workgroup finds its packet, apart from the others'
// and inside the staging buffer, its length and its key.  With an argument: reads batches, a line each of the
// number of keys and, for every chunk, its length, its AAD's and the number of its key, and prints of the launch
// that they share the longest list and what is filled in of the map.  Test infrastructure.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <iostream>
#include <sstream>
#include <string>
#include <vector>

#include "pgcm_spans.h"

using namespace pgcm;

#define CHECK(cond)                                                                              \
    do {                                                                                         \
        if (!(cond)) printf("n %zu, keys %zu, line %d: %s\n", n, nkeys, __LINE__, #cond), exit(1); \
    } while (0)

static const KeyTables* const tables = reinterpret_cast<const KeyTables*>((uintptr_t)1 << 32);
static const uint32_t num_cu = 256;

static void describe(const std::string& line) {
    std::istringstream in(line);
    size_t nkeys = 0;
    in >> nkeys;
    std::vector<uint64_t> len;
    std::vector<uint32_t> aad_len, of_key, order;
    for (uint64_t l, a, k; in >> l >> a >> k;) len.push_back(l), aad_len.push_back((uint32_t)a), of_key.push_back((uint32_t)k);
    const size_t n = len.size();
    std::vector<const void*> src(n, nullptr);
    std::vector<void*> dst(n, nullptr);
    std::vector<KeyPart> keys;
    uint64_t rows = 0;
    for (size_t q = 0; q < nkeys; ++q) {
        KeyPart key{nullptr, reinterpret_cast<const KeyTables*>((uintptr_t)tables + 16 * q), 14, order.size(), 0, 0, 0, 0};
        for (size_t i = 0; i < n; ++i)
            if (of_key[i] == q) order.push_back((uint32_t)i), ++key.n, key.rows += span_rows(len[i], aad_len[i]);
        rows += key.rows;
        keys.push_back(key);
    }
    CHECK(order.size() == n && (nkeys == 1 || share_launch(nkeys, n, rows, num_cu)));
    const SpanBatch b{n, order.data(), src.data(), aad_len.data(), src.data(), len.data(), dst.data()};
    const uint32_t ngroups = deal_groups(keys.data(), nkeys, num_cu);
    std::vector<SpanGroup> groups(ngroups);
    std::vector<SpanPart> parts(n + ngroups);
    SpanScratch scratch;
    const SpanPlan plan = plan_spans(b, keys.data(), nkeys, scratch, groups.data(), parts.data());
    SpanMap map;
    size_t bytes = 0;
    const uint32_t filled = map_spans(keys.data(), nkeys, groups.data(), plan, &map, &bytes);
    printf("%u%s%s\n", plan.longest, filled & kSpanPlaced ? " placed" : "", filled & kSpanKeysMapped ? " keys" : "");
}

int main(int argc, char**) {
    if (argc > 1) {
        for (std::string line; std::getline(std::cin, line);) describe(line);
        return 0;
    }
    unsigned placed = 0, mapped = 0, all = 0;
    for (size_t nkeys : {1, 2, 16, 17, 255, 256})
        for (size_t n : {256, 300, 600, 1700, 3000, 4096, 9000})
            for (uint64_t lo : {1, 40000, 2000000}) {
                std::vector<uint64_t> len(n);
                for (size_t i = 0; i < n; ++i) len[i] = i % 7 < 4 ? lo : lo * (i % 7 + 1) + 5000;
                if (lo == 40000) for (size_t i = 0; i < n / 8; ++i) len[i] = 100;  // long lists
                std::vector<const void*> src(n, nullptr);
                std::vector<void*> dst(n, nullptr);
                const SpanBatch b{n, nullptr, src.data(), nullptr, src.data(), len.data(), dst.data()};
                std::vector<KeyPart> keys;
                for (size_t q = 0; q < nkeys; ++q) {
                    const size_t first = n * q / nkeys, end = n * (q + 1) / nkeys;
                    KeyPart key{nullptr, reinterpret_cast<const KeyTables*>((uintptr_t)tables + 16 * q), 14, first, end - first, 0, 0, 0};
                    for (size_t i = first; i < end; ++i) key.rows += span_rows(len[i], 0);
                    keys.push_back(key);
                }
                const uint32_t ngroups = deal_groups(keys.data(), nkeys, num_cu);
                std::vector<SpanGroup> groups(ngroups);
                std::vector<SpanPart> parts(n + ngroups);
                SpanScratch scratch;
                const SpanPlan plan = plan_spans(b, keys.data(), nkeys, scratch, groups.data(), parts.data());
                SpanMap map;
                memset(&map, 0xA5, sizeof(map));
                size_t bytes = 0;
                const uint32_t filled = map_spans(keys.data(), nkeys, groups.data(), plan, &map, &bytes);
                CHECK(ngroups <= kSpanMapGroups);
                CHECK(((filled & kSpanKeysMapped) != 0) == (nkeys > 1 && nkeys <= kSpanMapKeys));
                CHECK(((filled & kSpanPlaced) != 0) == (plan.longest <= kSpanLdsParts && bytes <= kSpanHostBytes));
                size_t at = 0;
                for (uint32_t g = 0; g < ngroups; ++g) {
                    const uint32_t place = map.place[g];
                    if (filled & kSpanPlaced) {
                        CHECK((size_t)(place % (1u << SpanMap::kLengthShift)) * kPacketAlign == at);
                        CHECK((place >> SpanMap::kLengthShift) % 64 == groups[g].nparts);
                        at += (sizeof(SpanGroup) + sizeof(SpanPart) * groups[g].nparts + 63) / 64 * 64;
                    }
                    if (filled & kSpanKeysMapped) CHECK(map.key[place >> SpanMap::kKeyShift] == groups[g].kt);
                }
                if (filled & kSpanPlaced) CHECK(at == bytes && at <= kSpanHostBytes);
                for (uint32_t g = ngroups; g < kSpanMapGroups; ++g) CHECK(map.place[g] == 0);
                for (size_t q = filled & kSpanKeysMapped ? nkeys : 0; q < kSpanMapKeys; ++q) CHECK(map.key[q] == nullptr);
                ++all, placed += (filled & kSpanPlaced) != 0, mapped += (filled & kSpanKeysMapped) != 0;
            }
    printf("maps %u, with packets %u, with keys %u\n", all, placed, mapped);
    return 0;
}
