// The descriptor ring's bookkeeping: which slot a call's descriptors go to, which slot has them already, and what has to be waited for before a slot is written
// again.  Host code that reaches streams and events through Runtime alone, so that a program without a GPU can walk it:
//   Stream, Event, Status (0 = success)
//   Status record(Event, Stream), wait(Event), wait_all();  bool done(Event)
//   StreamState state(Stream, uint64_t* capture)   capture: number of the one that the stream is under, 0 if none
//   uint64_t thread(Stream)   0 if the handle names one queue, else (a queue of every thread's own) the calling thread's number, never given out again
#pragma once
#include <cstddef>
#include <cstdint>

namespace symb {

enum class StreamState { Known, Unsure, Gone };         // Unsure: the default stream beside a capture; Gone: destroyed

template <class Runtime>
struct DescRing {
    using Stream = typename Runtime::Stream;
    using Event = typename Runtime::Event;
    using Status = typename Runtime::Status;
    static constexpr int kSlots = 32;                   // (a training step of 7 projections makes 21 different blobs)
    static constexpr int kStreams = 2, kSealCalls = 8;  // streams whose calls share events, calls per event while there is one such stream (seal)
    static constexpr int kIdleCalls = 64;               // calls of others after which a stream is taken to have stopped

    struct Queue {                        // what work is in order on
        Stream stream{};
        uint64_t thread = 0;
        bool operator==(const Queue& o) const { return stream == o.stream && thread == o.thread; }
        bool operator!=(const Queue& o) const { return !(*this == o); }
    };
    struct Slot {
        Event done{};                     // recorded behind the slot's copy and, if sealed, behind its last call
        bool used = false, sealed = false;
        uint64_t last = 0;                // the last call that read it
        size_t size = 0;                  // what its device copy holds: a call whose blob is already there (same bytes, copied on
        uint64_t hash = 0;                // the same queue) reads that copy instead of sending the bytes again
        Queue queue;
        uint64_t graph = 0;               // the copy belongs to that capture: only calls under it find it done
    } slot[kSlots];
    struct StreamUse {
        Queue queue;
        Event ev{};                       // recorded behind call number `covered` or a later one of the stream
        uint64_t covered = 0, last = 0;   // (last: its last call)
        int since = 0;                    // calls since
        bool used = false, active = false;              // active: its calls share events; else an event is behind all that did
    } uses[kStreams];
    uint64_t seq = 0;                     // calls so far
    int next = 0;                         // the slot the next new blob goes to (round robin)
    int cur = 0;                          // the slot this call's kernels read
    // this call's queue, capture, and whether it may do without an event of its own
    Queue queue;
    uint64_t graph = 0;
    bool shares = false;

    void begin(Runtime& rt, Stream st) {
        queue = Queue{st, rt.thread(st)};
        graph = 0;
        shares = rt.state(st, &graph) == StreamState::Known && !queue.thread;
    }
    StreamUse* use_of(const Queue& q) {
        for (StreamUse& u : uses)
            if (u.used && u.queue == q) return &u;
        return nullptr;
    }
    // The slot that holds a blob already, -1 if none does.  same(i): slot i's pinned copy is that blob.  A call under capture leaves the slot as it is: its launches run
    // when the graph does, and what guards the ordinary calls before it stays behind them.
    template <class Same>
    int find(size_t n, uint64_t hash, Same&& same) {
        for (int j = 0; j < kSlots; ++j) {
            Slot& s = slot[j];
            if (!s.used || s.size != n || s.hash != hash || s.queue != queue || (s.graph && s.graph != graph) || !same(j)) continue;
            cur = j;
            if (graph) return j;
            s.last = ++seq;
            s.sealed = false;
            return j;
        }
        return -1;
    }
    // A slot for a new blob, both of whose copies may be written from here on (the device copy in stream order): `cur`.
    // The next slot in turn that no other stream may still read without an event behind that call.  The device copy of a slot of this stream is
    // overwritten in stream order; its pinned copy, and any other slot, is waited for.  A slot that hangs on another stream's event goes first only if that has come, as it may lie behind
    // calls that are far from done; one used in the last eight calls only if there is no other, so that a stream that comes to the ring gets a share of it.  A
    // copy under capture runs with the graph, on whatever stream: no slot is in its order.
    Status take(Runtime& rt) {
        int at = -1;
        for (int i = 0; i < 2 * kSlots && at < 0; ++i) {
            const int j = (next + i) % kSlots;
            const Slot& s = slot[j];
            const StreamUse* u = nullptr;
            if (s.used) {
                if (!s.sealed && (graph || s.queue != queue)) {
                    u = use_of(s.queue);
                    if (!u || s.last > u->covered) continue;
                }
                if (i < kSlots && (s.last + 8 > seq || (u && !rt.done(u->ev)))) continue;
                if (u) {
                    const Status e = rt.wait(u->ev);
                    if (e != Status{}) return e;
                }
            }
            at = j;
        }
        if (at < 0) {                      // (calls that failed behind their descriptors have no event: they may hold every slot in the end)
            const Status e = rt.wait_all();
            if (e != Status{}) return e;
            for (Slot& s : slot) s.sealed = true;
            at = next;
        }
        next = (at + 1) % kSlots;
        cur = at;
        if (slot[at].used) {
            const Status e = rt.wait(slot[at].done);
            if (e != Status{}) return e;
        }
        slot[at].used = false;             // until the copy is enqueued, the slot holds nothing a later call may reuse
        return Status{};
    }
    // The copy of a new blob to `cur` is enqueued.
    Status sent(Runtime& rt, size_t n, uint64_t hash) {
        Slot& s = slot[cur];
        s.size = n;
        s.hash = hash;
        s.queue = queue;
        s.graph = graph;
        s.used = true;
        s.sealed = graph != 0;            // (no ordinary call reads it)
        s.last = ++seq;
        return rt.record(s.done, queue.stream);      // a call that fails before its kernels still leaves the slot guarded
    }
    // Ends a call: its slot is busy until everything enqueued so far on `st` has run (kernels read it).  An event costs 2.8 us on the stream, a quarter of a small call (one user's decode
    // step on 4096 x 4096 14.1 -> 11.3 us without, a training step of 16 rows 42.1 -> 33.8), and what it guards against, the slot's next batch, is in stream order for this
    // stream.  So only every kSealCalls-th call of a stream records one, which covers all before it; with two streams every fourth.  A slot
    // that another stream still reads without an event behind it is passed over (take): at most 7 + 3 of them for the kStreams streams that
    // share events.  Calls of further streams, and of streams that every thread has its own of, record the slot's own event, as all calls did.  A stream that has made no call for the last
    // kIdleCalls gets an event behind its last one, which frees its slots and, once it has come, its place.
    Status seal(Runtime& rt) {
        if (graph) return Status{};
        StreamUse* u = use_of(queue);
        int active = 0;
        for (StreamUse& w : uses) {
            if (w.active && &w != u && seq - w.last > kIdleCalls) retire(rt, w);
            active += w.active;
        }
        if (shares && !u)
            for (StreamUse& w : uses)
                if (!u && !w.active && (!w.used || rt.done(w.ev))) {
                    for (Slot& s : slot)
                        if (w.used && s.queue == w.queue && s.last <= w.covered) s.sealed = true;      // (over)
                    u = &w;
                    u->queue = queue;
                    u->used = true;
                    u->covered = 0;
                }
        if (!u || !shares) {
            slot[cur].sealed = true;
            return rt.record(slot[cur].done, queue.stream);
        }
        if (!u->active) {
            u->active = true;
            u->since = 0;
            ++active;
        }
        u->last = seq;
        if (++u->since >= kSealCalls / active) {
            u->covered = seq;
            u->since = 0;
            return rt.record(u->ev, queue.stream);
        }
        return Status{};
    }
    void retire(Runtime& rt, StreamUse& u) {
        uint64_t number = 0;
        const StreamState is = rt.state(u.queue.stream, &number);
        if (is == StreamState::Unsure || number) return;               // (an event now would be the capture's, or disturb one)
        if (is == StreamState::Known && rt.record(u.ev, u.queue.stream) != Status{}) return;
        u.covered = seq;                                               // (of a stream that is gone all calls are over)
        u.active = false;
    }
};

}  // namespace symb
