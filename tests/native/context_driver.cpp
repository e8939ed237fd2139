// Threads that make batches with the contexts of one key, on streams of their own and on shared ones, as the
// library's host code does: the choice under a mutex, the call outside it.  Run under ThreadSanitizer: what a
// call writes without the mutex nobody else may read.  Then the streams that get areas of slots for short chunks.
// Prints how many contexts there were at the end.
// Test infrastructure.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <mutex>
#include <thread>
#include <vector>

#include "pgcm_contexts.h"

using namespace pgcm;

// as in the host code: what a call in progress has to itself
struct Context : Binding {
    bool captured = false, left_no_mark = false;
    int batches = 0;
};

static std::mutex mu;
static std::vector<Context*> contexts;
static uint64_t tick;

#define CHECK(cond)                                    \
    do {                                               \
        if (!(cond)) {                                 \
            printf("line %d: %s\n", __LINE__, #cond);  \
            exit(1);                                   \
        }                                              \
    } while (0)

static void batch(void* stream, uint64_t random) {
    Context* c;
    {
        std::lock_guard<std::mutex> lock(mu);
        bool must_wait;
        const bool own = clears_slots(contexts, stream);
        auto ended = [&](const Context* o) { return !o->in_call && (random & 4); };
        c = pick_context(contexts, stream, ended, &must_wait);
        // a new one while there are few, or where the others cannot be re-bound
        size_t free = 0, kept = 0;
        for (const Context* o : contexts)
            if (!o->replayed && !o->unmarked) ++kept, free += !o->in_call;
        CHECK(c != nullptr || free == 0 || kept < kMaxContexts);
        if (c == nullptr) contexts.push_back(c = new Context());
        CHECK(!c->in_call && (!c->bound || c->stream == stream || !(c->replayed || c->unmarked)));
        // of another stream: its last batch has ended, or is waited for where no more are made, the oldest
        CHECK(!c->bound || c->stream == stream || must_wait || ended(c));
        CHECK(!must_wait || kept >= kMaxContexts);
        if (must_wait)
            for (const Context* o : contexts)
                CHECK(o->replayed || o->unmarked || o->in_call || o->last_use >= c->last_use);
        CHECK(own == (c->replayed && c->stream == stream));
        enter_call(contexts, c, stream, ++tick);
    }
    c->stream = stream;
    c->bound = true;
    ++c->batches;
    c->left_no_mark = c->quiet;
    if (random % 512 == 0) c->captured = true;
    std::lock_guard<std::mutex> lock(mu);
    leave_call(c, c->captured, c->left_no_mark);
    size_t unmarked = 0, others = 0;
    for (const Context* o : contexts) (o->unmarked ? unmarked : others) += !o->replayed;
    CHECK(unmarked <= kMaxQuietContexts && others <= kMaxContexts + 8);  // a new one a thread at a time
}

// A key that has had many contexts at a time: streams that settle afterwards still leave their ends
// unmarked, kMaxQuietContexts of them.
static void settle_late() {
    std::vector<Context*> own;
    static char streams[24];
    Context all[24];
    for (int i = 0; i < 24; ++i) {
        own.push_back(&all[i]);
        all[i].stream = &streams[i], all[i].bound = true;
    }
    uint64_t t = 0;
    size_t quiet = 0;
    for (int i = 0; i < 24; ++i) {
        for (uint32_t k = 0; k <= kQuietStreak; ++k) {
            bool must_wait;
            Context* c = pick_context(own, &streams[i], [](const Context*) { return false; }, &must_wait);
            CHECK(c == &all[i] && !must_wait);
            enter_call(own, c, c->stream, ++t);
            CHECK(!c->quiet || k + 1 >= kQuietStreak);
            leave_call(c, false, c->quiet);
        }
        quiet += all[i].unmarked;
    }
    CHECK(quiet == kMaxQuietContexts);
    // one that gives its place back
    enter_call(own, &all[0], all[0].stream, ++t);
    leave_call(&all[0], false, false);
    enter_call(own, &all[20], all[20].stream, ++t);
    CHECK(all[20].quiet);
    enter_call(own, &all[0], all[0].stream, ++t);
    CHECK(!all[0].quiet);
}

// Areas of slots: the same one for a stream whenever it asks, of no other stream's, kShortStreams of them
static void short_streams() {
    static char streams[2 * kShortStreams];
    ShortStreams s;
    for (int turn = 0; turn < 3; ++turn) {
        CHECK(s.area_of(nullptr) == 0);  // the null stream is one of them
        for (size_t i = 0; i < 2 * kShortStreams; ++i)
            CHECK(s.area_of(&streams[i]) == (i + 1 < kShortStreams ? i + 1 : kShortStreams));
    }
}

int main() {
    settle_late();
    short_streams();
    static char streams[64];
    std::vector<std::thread> threads;
    for (int t = 0; t < 6; ++t)
        threads.emplace_back([t] {
            uint64_t state = 88172645463325252ull + t;
            for (int i = 0; i < 6000; ++i) {
                state ^= state << 13, state ^= state >> 7, state ^= state << 17;
                // half of them on a stream of the thread's own
                batch(&streams[state & 8 ? t : 6 + (state >> 20) % 24], state >> 32);
            }
        });
    for (std::thread& t : threads) t.join();
    printf("contexts %zu\n", contexts.size());
    for (Context* c : contexts) delete c;
    return 0;
}
