// Reads batches, a line each: compute units, one launch (0, 1), matrix hash, forced unit bytes, 1 for
// fixed buffers, 2 if captured or 3 where the stream's context was and the stream has no slots for short chunks, then
// for every chunk its length and its AAD's.  Prints which kernel takes each; called with "enc" or "dec", of those that
// burst_kernel takes the instance that this direction has, and the wavefronts of its workgroups that have blocks.
// Test infrastructure.
#include <cstdint>
#include <iostream>
#include <sstream>
#include <string>
#include <vector>

#include "pgcm_routes.h"

using namespace pgcm;

const char* instance(BurstKind k) {
    switch (k) {
        case BurstKind::kWords: return "words";
        case BurstKind::kWordsShared: return "words_shared";
        case BurstKind::kFold: return "fold";
        case BurstKind::kFoldApart: return "fold_apart";
        case BurstKind::kFoldShared: return "fold_shared";
        case BurstKind::kSweep: return "sweep";
    }
    return "none";
}

int main(int argc, char** argv) {
    const std::string direction = argc > 1 ? argv[1] : "";
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        uint32_t num_cu = 0, unit_bytes = 0;
        int one_launch = 0, matrix_hash = 0, fixed = 0;
        in >> num_cu >> one_launch >> matrix_hash >> unit_bytes >> fixed;
        uint32_t forced = 0;
        while (unit_bytes >= 16u << (forced + 1)) ++forced;
        std::vector<uint64_t> len;
        std::vector<uint32_t> aad_len;
        for (uint64_t l, a; in >> l >> a;) len.push_back(l), aad_len.push_back((uint32_t)a);
        BatchSurvey v;
        for (size_t i = 0; i < len.size(); ++i) v.add(len[i], aad_len[i]);
        const RouteOptions o{num_cu, one_launch != 0, matrix_hash != 0, forced, fixed == 1, fixed == 0, fixed == 1 || fixed == 3};
        SwapShape s{};
        switch (route_batch(ShapeBatch{len.size(), nullptr, aad_len.data(), len.data()}, o, v, &s)) {
            case Route::kOneRow: std::cout << "small\n"; break;
            case Route::kSpans: std::cout << "span\n"; break;
            case Route::kUnits: std::cout << "bulk\n"; break;
            case Route::kOneLaunch:
                if (!s.burst) {
                    std::cout << "swap " << (16u << s.unit_power) << "\n";
                    break;
                }
                if (!direction.empty()) {
                    std::cout << instance(burst_kind(s, num_cu, direction == "dec")) << " " << (1u << s.wave_power) << "\n";
                    break;
                }
                switch (burst_kind(s, num_cu, false)) {
                    case BurstKind::kWords:
                    case BurstKind::kWordsShared: std::cout << "words\n"; break;
                    case BurstKind::kFoldApart:
                    case BurstKind::kFold: std::cout << "fold " << s.unit_power + s.spare << "\n"; break;
                    case BurstKind::kSweep: std::cout << "sweep " << s.unit_power + s.spare << "\n"; break;
                    case BurstKind::kFoldShared: std::cout << (s.alone ? "shared\n" : "shared apart\n"); break;
                }
        }
    }
    return 0;
}
