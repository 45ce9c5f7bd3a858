// Workspaces that the allocating calls keep with their plan (rs_workspace):
// plain C++ over a device interface Dev, so that the host tests can drive it.
//
// A plan keeps a block per stream that uses it, found again by the next call on
// that stream.  Taking one from the device's pool and handing it back cost a
// NUFFT request of 5,204 pixels 20 us of host time a call (45 -> 25 us; a pool of
// its own for each plan is worse: 76 us when three plans take turns), and a call
// that is waited for 60-90 us more, as the device's pool unmaps at every
// synchronisation (4,057-pixel request, waited for: 99 -> 37 us; the 65,536-pixel
// NUFFT frame 197 -> 119 us).
//
// Ownership: a call owns its block from take to give, so calls of several
// threads have a block each.  The event recorded at give is waited for at the
// next take, which costs nothing on the same stream and keeps a stream that got
// the handle of a destroyed one behind its work.  A stream is never ordered
// behind another: it takes over or frees another stream's block only if that
// block's event has completed.
//
// Bounds: kBlocks blocks and kKeepBytes a plan, kKeepAll on a device over all
// plans; the least recently used idle block makes room, whatever finds none uses
// the device's pool.  Blocks go with their plan, and all idle ones when an
// allocation fails (release_idle).  A larger call on a stream replaces its
// block.  Sizes are rounded up by an eighth at most: the runtime maps 2 MiB and
// more on its own (a first call that needs 1.8 MB: 155 us with a block of 2 MiB,
// 72 us with 1.9).
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <mutex>

constexpr int kBlocks = 8;
constexpr size_t kKeepBytes = (size_t)256 << 20;
constexpr size_t kKeepAll = (size_t)1 << 30;
constexpr size_t kMinBlock = (size_t)16 << 10;

// Dev: types stream and event; bool create(event *), destroy(event), done(event),
// wait(stream, event), record(event, stream), alloc(void **, size_t, stream),
// free(void *, stream) -- false on failure, with no error left behind -- and
// finish(stream).
template <class Dev>
class rs_block_pool {
public:
    typedef typename Dev::stream stream;
    typedef typename Dev::event event;

    struct block {
        void *p = nullptr;
        size_t bytes = 0;      // allocated, or about to be
        stream st{};           // the stream of its last call
        event used{};          // behind that call
        bool has_event = false;
        bool taken = false;    // owned by a call (or being replaced for one)
        uint64_t tick = 0;     // when it was last handed back
    };

    explicit rs_block_pool(int dev) : device(dev)
    {
        std::lock_guard<std::mutex> g(all().m);
        next = all().head;
        if (next) next->prev = this;
        all().head = this;
    }

    // None of the plan's calls is in flight.  The blocks go back to the
    // device's pool, which releases them at the next synchronisation.
    ~rs_block_pool()
    {
        {
            std::lock_guard<std::mutex> g(all().m);
            (prev ? prev->next : all().head) = next;
            if (next) next->prev = prev;
        }
        for (block &x : b) {
            if (x.p) (void)Dev::free(x.p, stream{});
            if (x.has_event) Dev::destroy(x.used);
        }
    }

    rs_block_pool(const rs_block_pool &) = delete;
    rs_block_pool &operator=(const rs_block_pool &) = delete;

    // A block of at least `bytes` for a call on st, or NULL: use the device's pool.
    block *take(size_t bytes, stream st)
    {
        if (bytes > kKeepBytes) return nullptr;
        size_t step = kMinBlock;   // an eighth of the power of two below
        while (16 * step <= bytes) step <<= 1;
        const size_t size = (bytes + step - 1) / step * step;
        block *x = own(st);
        if (x) {
            if (!Dev::wait(st, x->used)) return back(x);
            if (x->bytes >= bytes) return x;
            if (!grow(x, size, st)) return back(x);
            if (!Dev::free(x->p, st)) {
                std::lock_guard<std::mutex> g(all().m);
                x->bytes = 0;   // not known to be free or held: drop it
            }
            x->p = nullptr;
        } else {
            x = place(size, st);
            if (!x || x->p) return x;
        }
        if ((x->has_event || (x->has_event = Dev::create(&x->used))) && x->bytes >= bytes &&
            Dev::alloc(&x->p, x->bytes, st))
            return x;
        x->p = nullptr;
        std::lock_guard<std::mutex> g(all().m);
        x->bytes = 0;
        x->taken = false;
        return nullptr;
    }

    // Hands a call's block back behind its work on st; false if the device
    // reported an error (the work is then waited for).
    bool give(block *x, stream st)
    {
        const bool ok = Dev::record(x->used, st);
        if (!ok) Dev::finish(st);
        std::lock_guard<std::mutex> g(all().m);
        x->tick = ++all().tick;
        x->taken = false;
        return ok;
    }

    // Frees every idle block on the device in the order of st (behind their
    // last calls) and waits for st, so that the memory is the device's again;
    // false if there was none.
    static bool release_idle(int dev, stream st)
    {
        bool any = false;
        {
            std::lock_guard<std::mutex> g(all().m);
            for (rs_block_pool *k = all().head; k; k = k->next)
                for (block &x : k->b)
                    if (k->device == dev && !x.taken && x.p && (Dev::done(x.used) || Dev::wait(st, x.used)))
                        any |= drop(x, st);
        }
        if (any) Dev::finish(st);
        return any;
    }

    // Bytes of blocks on the device, over all plans.
    static size_t kept(int dev)
    {
        std::lock_guard<std::mutex> g(all().m);
        return held(dev);
    }

private:
    struct registry {
        std::mutex m;   // guards every pool's table; device calls on a block that a call owns are made without it
        rs_block_pool *head = nullptr;
        uint64_t tick = 0;
    };
    static registry &all()
    {
        static registry r;
        return r;
    }

    // The stream's largest idle block, now owned.
    block *own(stream st)
    {
        std::lock_guard<std::mutex> g(all().m);
        block *x = nullptr;
        for (block &c : b)
            if (!c.taken && c.p && c.st == st && (!x || c.bytes > x->bytes)) x = &c;
        if (x) x->taken = true;
        return x;
    }

    block *back(block *x)
    {
        std::lock_guard<std::mutex> g(all().m);
        x->taken = false;
        return nullptr;
    }

    // Room for an owned block to become `size` bytes.
    bool grow(block *x, size_t size, stream st)
    {
        std::lock_guard<std::mutex> g(all().m);
        const size_t old = x->bytes;
        x->bytes = 0;
        const bool ok = room(size, st);
        x->bytes = ok ? size : old;
        return ok;
    }

    // A place for a new block of `size` bytes (p is NULL), or another stream's
    // finished block that is large enough.
    block *place(size_t size, stream st)
    {
        std::lock_guard<std::mutex> g(all().m);
        block *x = nullptr;
        for (block &c : b)
            if (!c.taken && !c.p) x = &c;
        if (!x) {
            x = oldest(this, this->next);
            if (!x) return nullptr;
            if (x->bytes < size || x->bytes / 2 > size) {
                if (!drop(*x, st)) return nullptr;
            }
        }
        if (!x->p) {
            if (!room(size, st)) return nullptr;
            x->bytes = size;
        }
        x->st = st;
        x->taken = true;
        return x;
    }

    // Whether `size` more bytes fit, idle blocks making room (this plan's for the
    // plan's bound, then any plan's for the device's).
    bool room(size_t size, stream st)
    {
        while (mine() + size > kKeepBytes) {
            block *x = oldest(this, this->next);
            if (!x || !drop(*x, st)) return false;
        }
        while (held(device) + size > kKeepAll) {
            block *x = oldest(all().head, nullptr);
            if (!x || !drop(*x, st)) return false;
        }
        return true;
    }

    size_t mine() const
    {
        size_t s = 0;
        for (const block &c : b) s += c.bytes;
        return s;
    }
    static size_t held(int dev)
    {
        size_t s = 0;
        for (rs_block_pool *k = all().head; k; k = k->next)
            if (k->device == dev) s += k->mine();
        return s;
    }

    // The least recently used idle block of the pools from .. to (excluded) on
    // this device whose work has completed.
    block *oldest(rs_block_pool *from, rs_block_pool *to)
    {
        block *x = nullptr;
        for (rs_block_pool *k = from; k != to; k = k->next)
            for (block &c : k->b)
                if (k->device == device && !c.taken && c.p && (!x || c.tick < x->tick) && Dev::done(c.used)) x = &c;
        return x;
    }

    // Frees an idle block whose work has completed or that st waits for.
    static bool drop(block &x, stream st)
    {
        if (!Dev::free(x.p, st)) return false;
        x.p = nullptr;
        x.bytes = 0;
        return true;
    }

    const int device;
    block b[kBlocks];
    rs_block_pool *prev = nullptr, *next = nullptr;
};
