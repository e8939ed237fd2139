// The end of a chunk that several workgroups make: every lane's steps (pgcm_arrive.h) one at a time, in every
// order there is for two and three workgroups and in random ones for more, so that the words of a tag are
// completed by one workgroup or by different ones; run under sanitizers.  Encrypting, every word is written
// once and right; decrypting, there is one verdict, and it is right; and the slots are zero again, which the
// next chunk relies on: they are not cleared in between.  Prints how many ends of each kind there were.
// Test infrastructure.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "pgcm_arrive.h"

using namespace pgcm;

static unsigned long long g_ends, g_one, g_split[5];
#define CHECK(cond)                                                     \
    do {                                                                \
        if (!(cond)) {                                                  \
            printf("end %llu, line %d: %s\n", g_ends, __LINE__, #cond);  \
            exit(1);                                                    \
        }                                                               \
    } while (0)

static uint64_t state = 88172645463325252ull;
static uint64_t below(uint64_t n) {
    state ^= state << 13;
    state ^= state >> 7;
    state ^= state << 17;
    return (state >> 11) % n;
}

struct Plain {
    static uint64_t fetch_xor(uint64_t* at, uint64_t v) { const uint64_t was = *at; *at ^= v; return was; }
    static uint32_t fetch_add(uint32_t* at, uint32_t v) { const uint32_t was = *at; *at += v; return was; }
    template <class T>
    static void clear(T* at) { *at = 0; }
};

// A wavefront at the end of its workgroup's part, as last_of_chunk has it: an atomic of four lanes, whose
// results it waits for before the next.
struct Wave {
    uint32_t g, word[4];
    int step;             // 0: in sets, 1: for the chunk, 2: a verdict to count, 3: done
    uint32_t to_do;       // lanes whose atomic of this step is still to come
    uint32_t whole;       // lanes that completed theirs
};

struct Chunk {
    uint32_t n;
    bool decrypt;
    ArriveSlot* slots;
    std::vector<Wave> waves;
    uint32_t tag[4], received[4];
    // what came out
    uint32_t written[4];
    int times_written[4], verdicts, accepted, completed_by;

    void begin(uint32_t wrong) {
        waves.resize(n);
        for (int w = 0; w < 4; ++w) tag[w] = 0, times_written[w] = 0;
        verdicts = accepted = completed_by = 0;
        for (uint32_t g = 0; g < n; ++g) {
            waves[g] = Wave{g, {}, n > kArriveSet ? 0 : 1, 0xF, 0};
            for (int w = 0; w < 4; ++w) tag[w] ^= waves[g].word[w] = (uint32_t)below(1ull << 32);
        }
        for (int w = 0; w < 4; ++w) received[w] = tag[w] ^ ((wrong >> w & 1) ? 1u << below(32) : 0);
    }
    bool can(const Wave& v, int lane) const { return v.step < 2 ? v.to_do >> lane & 1 : v.step == 2 && lane == 0; }
    void go(Wave& v, uint32_t lane) {
        if (v.step == 2) {
            uint32_t words = 0;
            bool differs = false;
            for (int w = 0; w < 4; ++w)
                if (v.whole >> w & 1) ++words, differs |= v.word[w] != received[w];
            const uint32_t count = count_verdict<Plain>(slots, words, differs);
            if (verdict_whole(count)) {
                ++verdicts;
                accepted = !verdict_differs(count);
                clear_verdict<Plain>(slots);
            }
            v.step = 3;
            return;
        }
        const ChunkMember m = n > kArriveSet ? set_of_chunk(v.g, n) : ChunkMember{v.g, n};
        const bool whole = v.step == 0 ? add_in_set<Plain>(slots, v.g, n, lane, v.word[lane])
                                       : add_in_chunk<Plain>(slots, m, lane, v.word[lane]);
        v.whole |= (uint32_t)whole << lane;
        v.to_do &= ~(1u << lane);
        if (v.to_do != 0) return;
        if (v.step == 0 && v.whole != 0) {
            v.step = 1, v.to_do = v.whole, v.whole = 0;
            return;
        }
        v.step = 3;
        if (v.whole == 0) return;
        ++completed_by;
        if (v.whole == 0xF && decrypt) {
            ++verdicts;
            accepted = 1;
            for (int w = 0; w < 4; ++w) accepted &= v.word[w] == received[w];
        } else if (decrypt) {
            v.step = 2;
        } else {
            for (int w = 0; w < 4; ++w)
                if (v.whole >> w & 1) written[w] = v.word[w], ++times_written[w];
        }
    }
    void check_end() {
        for (const Wave& v : waves) CHECK(v.step == 3);
        if (decrypt) {
            bool same = true;
            for (int w = 0; w < 4; ++w) same &= tag[w] == received[w];
            CHECK(verdicts == 1 && accepted == (int)same);
        } else {
            for (int w = 0; w < 4; ++w) CHECK(times_written[w] == 1 && written[w] == tag[w]);
        }
        for (uint32_t g = 0; g < n; ++g)
            for (int w = 0; w < 4; ++w) CHECK(slots[g].of_chunk[w] == 0 && slots[g].of_set[w] == 0);
        CHECK(completed_by >= 1 && completed_by <= 4);
        ++g_ends;
        ++(completed_by == 1 ? g_one : g_split[completed_by]);
    }
    // every order from here on
    void all_orders() {
        bool any = false;
        for (uint32_t g = 0; g < n; ++g)
            for (uint32_t lane = 0; lane < 4; ++lane)
                if (can(waves[g], lane)) {
                    any = true;
                    const Chunk saved = *this;
                    std::vector<ArriveSlot> at(slots, slots + n);
                    go(waves[g], lane);
                    all_orders();
                    *this = saved;
                    for (uint32_t k = 0; k < n; ++k) slots[k] = at[k];
                }
        if (!any) check_end();
    }
    // one order: of every word, the workgroups as `of_word` says, and the verdicts as `last` says
    void in_order(const std::vector<std::vector<uint32_t>>& of_word, const std::vector<uint32_t>& last) {
        for (uint32_t w = 0; w < 4; ++w)
            for (uint32_t g : of_word[w]) go(waves[g], w);
        for (uint32_t g : last)
            if (can(waves[g], 0)) go(waves[g], 0);
        check_end();
    }
    // a random one; `apart`: lanes by themselves, otherwise mostly a wavefront's together
    void random_order(bool apart) {
        std::vector<uint32_t> open(n);
        for (uint32_t g = 0; g < n; ++g) open[g] = g;
        while (!open.empty()) {
            const size_t i = below(open.size());
            Wave& v = waves[open[i]];
            const uint32_t first = (uint32_t)below(4), lanes = apart || below(8) == 0 ? 1 : 4;
            const int step = v.step;
            for (uint32_t k = 0, made = 0; k < 4 && made < lanes && v.step == step; ++k)
                if (can(v, (first + k) % 4)) go(v, (first + k) % 4), ++made;
            if (v.step == 3) open[i] = open.back(), open.pop_back();
        }
        check_end();
    }
};

int main() {
    // slots of chunks before and behind, as in a launch of several chunks
    std::vector<ArriveSlot> slots(1 + kSwapChunkGroups + 1);
    for (ArriveSlot& s : slots) s = ArriveSlot{};
    const ArriveSlot other{{7, 7, 7, 7}, {7, 7, 7, 7}};
    Chunk c{};
    c.slots = slots.data() + 1;
    auto start = [&](uint32_t n, bool decrypt, uint32_t wrong) {
        c.n = n, c.decrypt = decrypt;
        slots[0] = slots[1 + n] = other;
        c.begin(wrong);
    };
    auto neighbours = [&] {
        for (ArriveSlot* s : {&slots[0], &slots[1 + c.n]}) {
            for (int w = 0; w < 4; ++w) CHECK(s->of_chunk[w] == 7 && s->of_set[w] == 7);
            *s = ArriveSlot{};
        }
    };
    // two workgroups, every order of all eight atomics and the verdicts
    for (uint32_t wrong : {0u, 1u, 4u, 0xAu}) {
        for (bool decrypt : {false, true}) {
            start(2, decrypt, wrong);
            c.all_orders();
            neighbours();
        }
    }
    // three: the words do not touch each other, so every order of each word's, and of the verdicts
    const std::vector<std::vector<uint32_t>> p = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};
    for (int code = 0; code < 6 * 6 * 6 * 6; ++code)
        for (const auto& last : p)
            for (uint32_t wrong = 0; wrong <= 16; ++wrong) {
                start(3, wrong < 16, wrong % 16);
                c.in_order({p[code % 6], p[code / 6 % 6], p[code / 36 % 6], p[code / 216]}, last);
                neighbours();
            }
    for (uint32_t n : {2u, 3u, 31u, 32u, 33u, 34u, 63u, 64u, 65u, 96u, 97u, 255u, 256u})
        for (int trial = 0; trial < 400; ++trial) {
            start(n, trial & 1, trial % 3 ? 0 : (uint32_t)below(16));
            c.random_order(trial & 2);
            neighbours();
        }
    printf("ends %llu: words from one workgroup %llu, from two %llu, three %llu, four %llu\n", g_ends, g_one, g_split[2],
           g_split[3], g_split[4]);
    return 0;
}
