// Which of a key's contexts a batch on a stream runs with.  Host only, plain C++.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <vector>

namespace pgcm {

// contexts that could go to another stream a key keeps before it starts re-binding the least recently
// used one of them to a new stream
constexpr size_t kMaxContexts = 16;
// contexts that could not, at most
constexpr size_t kMaxQuietContexts = 8;
// batches in a row on one stream after which a context may leave their end unmarked
constexpr uint32_t kQuietStreak = 32;

// The part of a context that other threads look at, under the key's mutex.  While a call is using the context
// `stream` and `bound` are that call's alone, and others look at the rest only.
struct Binding {
    void* stream = nullptr;
    bool bound = false;     // has run a batch on `stream`
    bool in_call = false;   // a host thread is inside a batch call with it
    bool replayed = false;  // a graph replays a batch of its
    bool unmarked = false;  // nothing marks the end of its most recent batch (see `quiet`)
    uint64_t last_use = 0;
    // The stream has used the context long enough, and there are few enough of them, that batches
    // which use no staging buffer end unmarked: an event a batch costs the host up to 3.3 us, 2.3 us a
    // call where calls follow each other (one 320 KiB block 11.9 -> 9.2 us, a 2 MiB piece 13.4 -> 11.8;
    // on machines that take its interrupts quickly nothing).  Without that mark the context is never
    // given to another stream, so only while there are few of them; streams that come and go have
    // kMaxContexts beside those.
    uint32_t streak = 0;  // batches in a row on `stream`
    bool quiet = false;
};

// In order of preference: a context already bound to the stream; one whose last batch has ended (it is
// re-bound); a new one (null); and, once the key has kMaxContexts that can be re-bound, the least recently
// used one, after waiting for its last batch (*must_wait).  Never taken are contexts that another host
// thread is using at this moment.  Never re-bound are those whose batches a graph replays, and those whose
// last batch left no mark to wait for, at most kMaxQuietContexts; they stay with their streams and leave the
// others their number.  ended(c): has the last batch of c, which is bound and in no call, ended?
template <class C, class Ended>
C* pick_context(const std::vector<C*>& contexts, const void* stream, Ended ended, bool* must_wait) {
    *must_wait = false;
    for (C* c : contexts)
        if (!c->in_call && c->bound && c->stream == stream) return c;
    C* lru = nullptr;
    size_t kept = 0;  // that can be re-bound
    for (C* c : contexts) {
        if (c->replayed || c->unmarked) continue;
        ++kept;
        if (c->in_call) continue;
        if (!c->bound || ended(c)) return c;
        if (lru == nullptr || c->last_use < lru->last_use) lru = c;
    }
    *must_wait = lru != nullptr && kept >= kMaxContexts;
    return *must_wait ? lru : nullptr;
}

// The contexts besides c whose last batch left no mark, or may be leaving none now.  (All contexts counted
// would do as well for the bound, but contexts stay until the key is freed: a key that once had more of
// them would leave no end unmarked again.)
template <class C>
size_t quiet_contexts(const std::vector<C*>& contexts, const C* c) {
    size_t n = 0;
    for (const C* o : contexts) n += o != c && (o->unmarked || (o->in_call && o->quiet));
    return n;
}

// A call on `stream` begins with c, which is one of `contexts` by now.
template <class C>
void enter_call(const std::vector<C*>& contexts, C* c, const void* stream, uint64_t tick) {
    c->in_call = true;
    c->last_use = tick;
    if (!c->bound || c->stream != stream) c->streak = 0;
    else if (c->streak < kQuietStreak) ++c->streak;
    c->quiet = c->streak >= kQuietStreak && !c->replayed &&
               quiet_contexts(contexts, c) < kMaxQuietContexts;
}

// ... and ends.
inline void leave_call(Binding* c, bool replayed, bool unmarked) {
    c->replayed = replayed;
    c->unmarked = unmarked;
    c->in_call = false;
}

// Which of a key's areas of slots the short chunks of a stream that have several workgroups add up in.  An area
// goes to one of the first streams that ask and stays with it: its batches are ordered by the stream, so that such a
// call needs no context, gets no memory, waits for nobody and marks no end.  (Streams beyond those have a workgroup
// a chunk, 8 KiB in 8.1 us instead of 5.7.  With a context each such calls paid for what a workgroup a chunk does
// without: an event a call, where a context is not quiet, 64 chunks of 4 KiB with AAD waited for 19.8 -> 20.6 us; a launch
// that clears the slots, where it was captured, 8.1 -> 11.4; and memory and waits as for any other batch.)
constexpr size_t kShortStreams = 8;
struct ShortStreams {
    size_t n = 0;
    const void* stream[kShortStreams];

    // the stream's area; kShortStreams if there is none left
    size_t area_of(const void* of) {
        for (size_t i = 0; i < n; ++i)
            if (stream[i] == of) return i;
        if (n == kShortStreams) return n;
        stream[n] = of;
        return n++;
    }
};

// Does a graph replay batches of the context that a batch on `stream` would be given now?  Such a context
// has its slots cleared by every batch.
template <class C>
bool clears_slots(const std::vector<C*>& contexts, const void* stream) {
    for (const C* c : contexts)
        if (!c->in_call && c->bound && c->stream == stream) return c->replayed;
    return false;
}

}  // namespace pgcm
