// Walks the descriptor ring's bookkeeping (csrc/symb_ring.hpp) with made-up streams: queues on which nothing runs before somebody waits for it, a handle value that names another
// queue in every thread, handles that are destroyed and given out again, calls under capture.  What it checks, call by call: a slot's device copy is written only behind all
// launches that read it (on their own queue, or after they have ended), its pinned copy only after the copy from it, and a call that takes a slot in place reads its own blob.
//   ring_walk SCENARIO   prints "SCENARIO fails=N"; exit status 0 = none
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "../../paper_2507_03220_amd/csrc/symb_ring.hpp"

struct At {
    int queue = -1;                 // -1: nothing
    uint64_t pos = 0;
};
struct World {
    struct Queue { uint64_t enqueued = 0, done = 0; };
    std::vector<Queue> queues;
    std::map<std::pair<long, int>, int> live;           // (handle value, thread or -1) -> queue
    std::map<long, int> graph;                          // handle values under capture -> number of the capture
    std::vector<At> events;
    int thread = 0, records = 0, waits = 0, full_waits = 0;
    static constexpr long PER_THREAD = 2;

    int queue(long st) {
        const std::pair<long, int> k{st, st == PER_THREAD ? thread : -1};
        auto it = live.find(k);
        if (it != live.end()) return it->second;
        if (st != PER_THREAD && st != 0) return -1;     // destroyed
        queues.push_back({});
        return live[k] = (int)queues.size() - 1;
    }
    void create(long st) { queues.push_back({}); live[{st, -1}] = (int)queues.size() - 1; }
    void destroy(long st) {                             // (drained before, as the contract asks)
        Queue& q = queues[live[{st, -1}]];
        q.done = q.enqueued;
        live.erase({st, -1});
    }
    At enqueue(long st) {
        const int q = queue(st);
        return {q, ++queues[q].enqueued};
    }
    bool over(At a) const { return a.queue < 0 || queues[a.queue].done >= a.pos; }
    void finish(At a) { if (a.queue >= 0 && queues[a.queue].done < a.pos) queues[a.queue].done = a.pos; }
};
struct SimRuntime {
    using Stream = long;
    using Event = int;
    using Status = int;
    World* w;
    Status record(Event ev, Stream st) {
        if (w->graph.count(st)) return 0;               // belongs to the capture: nothing is behind it
        const int q = w->queue(st);
        if (q < 0) return 1;
        ++w->records;
        w->events[ev] = {q, w->queues[q].enqueued};
        return 0;
    }
    Status wait(Event ev) { ++w->waits; w->finish(w->events[ev]); return 0; }
    Status wait_all() { ++w->full_waits; for (auto& q : w->queues) q.done = q.enqueued; return 0; }
    bool done(Event ev) { return w->over(w->events[ev]); }
    symb::StreamState state(Stream st, uint64_t* capture) {
        const auto g = w->graph.find(st);
        *capture = g == w->graph.end() ? 0 : (uint64_t)g->second;
        return w->queue(st) < 0 ? symb::StreamState::Gone : symb::StreamState::Known;
    }
    uint64_t thread(Stream st) { return st == World::PER_THREAD ? 1 + (uint64_t)w->thread : 0; }
};
using Ring = symb::DescRing<SimRuntime>;

struct Walk {
    World w;
    SimRuntime rt{&w};
    Ring ring;
    struct Copy {
        int pinned = -1, device = -1;                   // batch numbers; device -1: unknown
        int graph = 0;                                  // capture that holds the copy
        At copied;                                      // the copy's place
        std::vector<At> readers;
    } copy[Ring::kSlots];
    int fails = 0, sent = 0, calls = 0;

    Walk() {
        w.create(0);
        int n = 0;
        for (auto& s : ring.slot) s.done = n++;
        for (auto& u : ring.uses) u.ev = n++;
        w.events.resize(n);
    }
    void expect(bool ok, const char* what) {
        if (ok) return;
        if (fails++ < 5) std::fprintf(stderr, "call %d: %s\n", calls, what);
    }
    // one call of batch number `batch`; ended: false = it fails after its descriptors have gone out
    void call(long st, int batch, bool ended = true) {
        ++calls;
        const auto g = w.graph.find(st);
        const int graph = g == w.graph.end() ? 0 : g->second;
        const int q = w.queue(st);
        ring.begin(rt, st);
        int at = ring.find(100, (uint64_t)batch, [&](int j) { return copy[j].pinned == batch; });
        if (at >= 0) {
            Copy& c = copy[at];
            expect(c.graph ? c.graph == graph : c.device == batch && (c.copied.queue == q || w.over(c.copied)), "in place, but the blob is not there");
        } else {
            ++sent;
            expect(ring.take(rt) == 0, "no slot");
            at = ring.cur;
            Copy& c = copy[at];
            expect(w.over(c.copied), "pinned copy written under the copy from it");
            for (const At& r : c.readers) expect(w.over(r) || (r.queue == q && !graph), "device copy written under a launch that reads it");
            c.readers.clear();
            c.pinned = batch;
            c.graph = graph;
            c.device = graph ? -1 : batch;
            c.copied = graph ? At{} : w.enqueue(st);
            expect(ring.sent(rt, 100, (uint64_t)batch) == 0, "event");
        }
        if (!graph) copy[at].readers.push_back(w.enqueue(st));       // its launches
        if (ended) expect(ring.seal(rt) == 0, "event");
        else ring.slot[at].size = (size_t)-1;
    }
};

static unsigned lcg = 4711u;
static int rnd(int n) {
    lcg = lcg * 1664525u + 1013904223u;
    return (int)((lcg >> 8) % (unsigned)n);
}

static int run(const std::string& name) {
    Walk k;
    const auto streams = [&](int n) { for (int i = 1; i <= n; ++i) k.w.create(100 + i); };
    if (name == "one_stream") {                          // events: every eighth call of repeated batches; no wait but for copies
        for (int i = 0; i < 800; ++i) k.call(0, i % 21);
        k.expect(k.sent == 21, "batches that fit the ring are sent once");
        k.expect(k.w.records == 21 + 100 && k.w.waits == 0, "events of repeated calls");
        for (int i = 0; i < 400; ++i) k.call(0, 1000 + i);
        k.expect(k.w.full_waits == 0, "waits");
    } else if (name == "streams") {                      // two to seven at a time, batches of all reuse distances, the GPU at work now and then
        streams(7);
        for (int i = 0; i < 60000; ++i) {
            const int n = 1 + i / 10000, st = 101 + rnd(n + 1);
            k.call(st, st * 1000 + rnd(1 + rnd(60)));
            if (rnd(20) == 0) {
                World::Queue& q = k.w.queues[rnd((int)k.w.queues.size())];
                q.done += (q.enqueued - q.done) * (uint64_t)rnd(5) / 4;
            }
        }
        k.expect(k.w.full_waits == 0, "waits for the whole device");
    } else if (name == "per_thread") {                   // one handle value, a queue in every thread: other batches, the same ones, other streams beside them
        streams(2);
        for (int i = 0; i < 200; ++i) {
            k.w.thread = 0;
            k.call(World::PER_THREAD, 7);                // (a long one, say: nothing has run yet)
            k.w.thread = 1;
            for (int j = 0; j < Ring::kSlots; ++j) k.call(World::PER_THREAD, 100 + 50 * i + j);
            k.call(World::PER_THREAD, 7);
        }
        for (int i = 0; i < 20000; ++i) {
            k.w.thread = rnd(4);
            const int st = rnd(4);
            k.call(st < 2 ? World::PER_THREAD : 99 + st, rnd(i < 10000 ? 20 : 200));
        }
    } else if (name == "recycled") {                     // streams that come and go, their handle values given out again
        for (int i = 0; i < 3000; ++i) {
            const int st = 101 + rnd(3);
            if (k.w.live.count({st, -1})) k.w.destroy(st);
            k.w.create(st);
            for (int j = rnd(60); j > 0; --j) k.call(rnd(3) ? st : 0, rnd(40));
        }
    } else if (name == "capture") {                      // captured calls between ordinary ones, in place and with blobs of their own, two captures after one another
        streams(4);
        for (int i = 0; i < 400; ++i) {
            const int st = 101 + i % 2, other = 103 + i % 2;
            for (int j = rnd(20); j >= 0; --j) k.call(st, 1);
            k.w.graph[st] = i + 1;
            k.call(st, 1);
            for (int j = 0; j < 3; ++j) k.call(st, 500 + 3 * i + j % 2);
            k.w.graph.erase(st);
            k.call(st, 500 + 3 * i);                     // (its copy is in the graph)
            k.w.graph[st] = 1000 + i;
            k.call(st, 501 + 3 * i);
            k.w.graph.erase(st);
            for (int j = 0; j < Ring::kSlots; ++j) k.call(i % 4 < 2 ? other : 0, 100000 + 100 * i + j);
        }
        for (int i = 0; i < 30000; ++i) {
            const int st = 101 + rnd(4);
            if (rnd(10) == 0 && !k.w.graph.erase(st)) k.w.graph[st] = 10000 + i;
            k.call(st, rnd(60));
        }
        k.expect(k.w.full_waits == 0, "waits for the whole device");
    } else if (name == "idle" || name == "gone") {       // two streams that share events stop, or are destroyed; then others, one after the other, get their events and all of their slots
        streams(9);
        for (int st = 101; st <= 102; ++st)
            for (int i = 0; i < 300; ++i) k.call(st, 100 * st + (i < 293 ? 0 : i));
        if (name == "gone") k.w.destroy(101), k.w.destroy(102);
        for (int st = 103; st <= 109; ++st) {
            int sent = 0, records = 0;
            for (int i = 0; i < 4000; ++i) {
                if (i == 2000) sent = k.sent, records = k.w.records;
                k.call(st, 100 * st + i % 30);
                if (i % 100 == 0)
                    for (auto& q : k.w.queues) q.done = q.enqueued;
            }
            k.expect(k.sent == sent && k.w.records == records + 2000 / 8, "one stream alone");
        }
        k.w.graph[109] = 1;                              // (stops under capture: no event behind its calls)
        for (int i = 0; i < 4000; ++i) k.call(108, 77000 + i % 40);
        k.w.graph.erase(109);
        if (name == "idle")
            for (int i = 0; i < 20000; ++i) k.call(101 + i / 100 % 9, rnd(50));
        k.expect(k.w.full_waits == 0, "waits for the whole device");
    } else if (name == "failing_calls") {                // their slots stay guarded, and the ring does not run out of others
        streams(3);
        for (int i = 0; i < 20000; ++i) k.call(101 + rnd(3), rnd(100), rnd(4) != 0);
        k.expect(k.w.full_waits == 0, "waits for the whole device");
        for (int i = 0; i < 100; ++i) k.call(103, 5000 + i, false);      // (of the one that shares no events)
        for (int i = 0; i < 1000; ++i) k.call(101, i);
        k.expect(k.w.full_waits <= 1, "waits for the whole device");
    } else {
        std::fprintf(stderr, "no scenario %s\n", name.c_str());
        return 1;
    }
    std::printf("%s fails=%d sent=%d records=%d waits=%d full=%d\n", name.c_str(), k.fails, k.sent, k.w.records, k.w.waits, k.w.full_waits);
    return k.fails ? 1 : 0;
}

int main(int argc, char** argv) {
    int bad = argc < 2;
    for (int i = 1; i < argc; ++i) bad |= run(argv[i]);
    return bad;
}
