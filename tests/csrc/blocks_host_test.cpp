// Host test of the workspaces that plans keep (paper_2307_09226_amd/csrc/
// rs_blocks.h) on a device of the test's own: streams complete when the test
// says so, memory is finite, and every use of a block is checked against the
// work that may still be using it.  Prints "ALL OK" and exits 0 on success.
#include "rs_blocks.h"

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <memory>
#include <thread>
#include <vector>

#define CHECK(cond)                                                                       \
    do {                                                                                  \
        if (!(cond)) {                                                                    \
            std::fprintf(stderr, "%s:%d: CHECK failed: %s\n", __FILE__, __LINE__, #cond); \
            std::exit(1);                                                                 \
        }                                                                                 \
    } while (0)

// Streams are numbers.  Work on a stream is a running count; an event records a
// stream's count; a stream that waited for an event knows that count of the other.
struct fake {
    typedef int stream;
    typedef int event;   // index + 1

    static std::recursive_mutex m;
    static size_t limit, used;
    static std::map<void *, size_t> live;
    static std::map<int, long> issued, finished;              // per stream
    static std::map<std::pair<int, int>, long> waited;        // (stream, of stream) -> count
    static std::vector<std::pair<int, long>> events;          // (stream, count)
    static std::map<void *, std::pair<int, long>> last;       // block -> its last work
    static int fail_record, queries;

    static void reset(size_t bytes)
    {
        CHECK(live.empty());
        limit = bytes;
        used = 0;
        issued.clear();
        finished.clear();
        waited.clear();
        events.clear();
        last.clear();
        fail_record = queries = 0;
    }
    static bool ordered(int st, std::pair<int, long> w)
    {
        return w.first == st || finished[w.first] >= w.second || waited[{st, w.first}] >= w.second;
    }

    static bool create(event *e)
    {
        std::lock_guard<std::recursive_mutex> g(m);
        events.push_back({-1, 0});
        *e = (int)events.size();
        return true;
    }
    static void destroy(event) {}
    static bool done(event e)
    {
        std::lock_guard<std::recursive_mutex> g(m);
        ++queries;
        const auto w = events[e - 1];
        return w.first < 0 || finished[w.first] >= w.second;
    }
    static bool wait(stream st, event e)
    {
        std::lock_guard<std::recursive_mutex> g(m);
        const auto w = events[e - 1];
        if (w.first >= 0 && w.first != st) waited[{st, w.first}] = std::max(waited[{st, w.first}], w.second);
        return true;
    }
    static bool record(event e, stream st)
    {
        std::lock_guard<std::recursive_mutex> g(m);
        if (fail_record) return false;
        events[e - 1] = {st, issued[st]};
        return true;
    }
    static bool alloc(void **p, size_t bytes, stream)
    {
        std::lock_guard<std::recursive_mutex> g(m);
        if (used + bytes > limit) return false;
        used += bytes;
        *p = std::malloc(1);
        live[*p] = bytes;
        last.erase(*p);
        return true;
    }
    static bool free(void *p, stream st)
    {
        std::lock_guard<std::recursive_mutex> g(m);
        CHECK(live.count(p));
        // freed in the order of st: what used the block is behind it
        if (st && last.count(p)) CHECK(ordered(st, last[p]));
        used -= live[p];
        live.erase(p);
        std::free(p);
        return true;
    }
    static void finish(stream st)
    {
        std::lock_guard<std::recursive_mutex> g(m);
        finished[st] = issued[st];
    }

    // a call's work on a block
    static void use(void *p, stream st, size_t bytes)
    {
        std::lock_guard<std::recursive_mutex> g(m);
        CHECK(live.count(p) && live[p] >= bytes);
        if (last.count(p)) CHECK(ordered(st, last[p]));
        last[p] = {st, ++issued[st]};
    }
};
std::recursive_mutex fake::m;
size_t fake::limit, fake::used;
std::map<void *, size_t> fake::live;
std::map<int, long> fake::issued, fake::finished;
std::map<std::pair<int, int>, long> fake::waited;
std::vector<std::pair<int, long>> fake::events;
std::map<void *, std::pair<int, long>> fake::last;
int fake::fail_record, fake::queries;

typedef rs_block_pool<fake> pool;
constexpr size_t MiB = (size_t)1 << 20;

// One call: true if it ran on a kept block.
static bool call(pool &k, size_t bytes, int st)
{
    pool::block *x = k.take(bytes, st);
    if (!x) return false;
    fake::use(x->p, st, bytes);
    return k.give(x, st);
}

// The same stream finds its block again; a larger call replaces it.
static void same_stream()
{
    fake::reset(1000 * MiB);
    pool k(0);
    CHECK(call(k, 5 * MiB, 1));
    const size_t one = fake::used;
    CHECK(one >= 5 * MiB && one <= 5 * MiB * 9 / 8);
    for (int i = 0; i < 20; ++i) CHECK(call(k, 1 + (size_t)i * 1000, 1));
    CHECK(fake::used == one && fake::queries == 0);
    CHECK(call(k, 9 * MiB, 1) && fake::live.size() == 1 && fake::used >= 9 * MiB);
    CHECK(!call(k, 257 * MiB, 1) && fake::live.size() == 1);
}

// A stream per request, never used again: places and memory come back once the
// streams' work has completed, and are not touched before.
static void stream_per_request()
{
    fake::reset(100000 * MiB);
    pool k(0);
    for (int st = 1; st <= 8; ++st) CHECK(call(k, 30 * MiB, st));
    CHECK(!call(k, 30 * MiB, 9));                       // all of it still running
    for (int st = 1; st <= 8; ++st) CHECK(fake::finished[st] == 0 && (fake::waited[{9, st}] == 0));
    int kept = 0;
    for (int st = 10; st < 200; ++st) {
        for (int old = 1; old < st - 2; ++old) fake::finish(old);
        kept += call(k, (st % 3 ? 20 : 31) * MiB, st);
        CHECK(fake::used <= kKeepBytes && fake::live.size() <= kBlocks);
    }
    CHECK(kept == 190);
}

// The plan's bound with blocks of few streams.
static void bounds_of_a_plan()
{
    fake::reset(100000 * MiB);
    pool k(0);
    CHECK(call(k, 120 * MiB, 1) && call(k, 120 * MiB, 2));
    CHECK(!call(k, 100 * MiB, 3));                      // both are in use
    fake::finish(1);
    CHECK(call(k, 100 * MiB, 3) && fake::used <= kKeepBytes && fake::live.size() == 2);
    CHECK(call(k, 120 * MiB, 2));                       // stream 2's is still there
}

// Many plans: the device's bound, the least recently used ones give way.
static void bounds_of_a_device()
{
    fake::reset(100000 * MiB);
    std::vector<std::unique_ptr<pool>> k;
    for (int i = 0; i < 40; ++i) {
        k.emplace_back(new pool(0));
        CHECK(call(*k.back(), 200 * MiB, 1));
        fake::finish(1);
        CHECK(fake::used <= kKeepAll && pool::kept(0) == fake::used);
    }
    pool other(1);
    CHECK(call(other, 200 * MiB, 2) && pool::kept(1) > 0);   // another device has its own bound
    for (int i = 0; i < 40; ++i) {
        CHECK(call(*k[i], 200 * MiB, 1));
        fake::finish(1);
    }
    // work in flight everywhere: nothing gives way, nothing waits
    for (int i = 36; i < 40; ++i) CHECK(call(*k[i], 200 * MiB, 1));
    CHECK(!call(*k[0], 200 * MiB, 3));
    k.clear();
    CHECK(pool::kept(0) == 0);
}

// An allocation that fails: the idle blocks of all plans come back, those whose
// work still runs behind it.
static void short_memory()
{
    fake::reset(600 * MiB);
    pool a(0), b(0), c(1);
    CHECK(call(a, 200 * MiB, 1) && call(b, 200 * MiB, 2) && call(c, 100 * MiB, 3));
    fake::finish(1);
    void *p = nullptr;
    CHECK(!fake::alloc(&p, 450 * MiB, 4));
    pool::block *own = b.take(10, 2);                   // a call owns one of them
    CHECK(own);
    CHECK(pool::release_idle(0, 4) && pool::kept(0) > 0);
    CHECK(!fake::alloc(&p, 450 * MiB, 4));
    fake::use(own->p, 2, 10);
    CHECK(b.give(own, 2));
    CHECK(pool::release_idle(0, 4) && pool::kept(0) == 0 && pool::kept(1) > 0);
    CHECK(fake::alloc(&p, 450 * MiB, 4) && fake::free(p, 4));
    CHECK(!pool::release_idle(0, 4));
    // a block that could not be allocated leaves its place usable
    fake::limit = 0;
    CHECK(!call(a, 10 * MiB, 1));
    fake::limit = 600 * MiB;
    CHECK(call(a, 10 * MiB, 1));
}

static void record_failure()
{
    fake::reset(100 * MiB);
    pool k(0);
    fake::fail_record = 1;
    CHECK(!call(k, MiB, 1) && fake::finished[1] == fake::issued[1]);
    fake::fail_record = 0;
    CHECK(call(k, MiB, 1));
}

// Threads with a stream each on shared plans, one releasing now and then.
static void threads()
{
    fake::reset(500 * MiB);
    std::vector<std::unique_ptr<pool>> k;
    for (int i = 0; i < 3; ++i) k.emplace_back(new pool(0));
    std::atomic<int> kept{0};
    std::vector<std::thread> t;
    for (int i = 0; i < 6; ++i)
        t.emplace_back([&, i] {
            unsigned r = 7u * i + 1;
            for (int n = 0; n < 3000; ++n) {
                r = r * 1664525u + 1013904223u;
                const int st = i % 4 + 1;   // some streams are shared by two threads
                kept += call(*k[(r >> 8) % 3], (size_t)(r >> 10) % (70 * MiB) + 1, st);
                if ((r >> 20) % 97 == 0) fake::finish(st);
                if (i == 0 && n % 50 == 0) pool::release_idle(0, 9);
                if (i == 5 && n % 400 == 399) {
                    pool extra(0);
                    call(extra, MiB, 6);
                }
            }
        });
    for (auto &x : t) x.join();
    CHECK(kept > 1000);
    k.clear();
    CHECK(fake::live.empty());
}

int main()
{
    same_stream();
    stream_per_request();
    bounds_of_a_plan();
    bounds_of_a_device();
    short_memory();
    record_failure();
    threads();
    CHECK(fake::live.empty());
    std::puts("ALL OK");
    return 0;
}
