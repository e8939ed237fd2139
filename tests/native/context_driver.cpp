// Threads that make batches with the contexts of one key, on streams of their own and on shared ones, as the
// library's host code does: the choice under a mutex, the call outside it.  Run under ThreadSanitizer: what a
// call writes without the mutex nobody else may read.  Prints how many contexts there were at the end.
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
        c = pick_context(contexts, stream, [&](const Context* o) { return !o->in_call && (random & 4); }, &must_wait);
        if (c == nullptr) contexts.push_back(c = new Context());
        CHECK(!c->in_call && (!c->bound || c->stream == stream || !(c->replayed || c->unmarked)));
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

int main() {
    settle_late();
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
