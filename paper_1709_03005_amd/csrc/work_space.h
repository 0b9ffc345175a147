// Work space of a context's calls (solver bases, mat-vec partials, staging of
// host arrays), kept between calls: a hipFree waits for the whole device and
// unmaps, and with several large contexts resident a product of 1 ms spent 11
// ms on it (D = 24011; a solve at D = 8000 2.5 of its 14.5 ms).
//
// take() reuses an idle block of at most twice the size, else allocates. The
// blocks belong to one context, whose calls run one at a time and queue their
// kernels on one stream, so a reused block's earlier work is ordered before its
// next. give() makes a block idle. What is idle is never in the way of another
// allocation: all work spaces of a device together keep at most `keep` idle
// bytes (the largest blocks go first, whichever context's), and an allocation
// that fails, in any context, frees every idle block of the device and is tried
// again. One lock over all work spaces of the process covers this; it is taken a
// few times a call.
//
// Dev: an error type Err (Err(0): success), static Err alloc(int device, void **,
// size_t), on that device whichever is current, and static void release(void *).
#pragma once
#include <algorithm>
#include <cstddef>
#include <mutex>
#include <vector>

namespace cch {

template <class Dev>
class WorkSpace {
public:
    using Err = typename Dev::Err;

    WorkSpace() = default;
    WorkSpace(const WorkSpace &) = delete;
    WorkSpace &operator=(const WorkSpace &) = delete;
    ~WorkSpace() { close(); }

    // a work space on `device` that keeps idle blocks while the device's hold at
    // most `keep` bytes (0: none of its own)
    void open(int device, size_t keep)
    {
        const std::lock_guard<std::mutex> lock(all().m);
        if (!open_) all().spaces.push_back(this);
        open_ = true;
        device_ = device;
        keep_ = keep;
        trim();
    }

    // frees every block
    void close()
    {
        const std::lock_guard<std::mutex> lock(all().m);
        for (auto &b : blocks_) Dev::release(b.p);
        blocks_.clear();
        idle_ = 0;
        auto &s = all().spaces;
        s.erase(std::remove(s.begin(), s.end(), this), s.end());
        open_ = false;
    }

    Err take(void **p, size_t bytes)
    {
        bytes = (std::max<size_t>(bytes, 1) + 255) / 256 * 256;
        const std::lock_guard<std::mutex> lock(all().m);
        Block *best = nullptr;
        for (auto &b : blocks_)
            if (!b.used && b.bytes >= bytes && b.bytes / 2 <= bytes && (!best || b.bytes < best->bytes)) best = &b;
        if (best) {
            best->used = true;
            idle_ -= best->bytes;
            *p = best->p;
            return Err(0);
        }
        const Err e = alloc_locked(device_, p, bytes);
        if (e == Err(0)) blocks_.push_back({*p, bytes, true});
        return e;
    }

    void give(void *p)
    {
        if (!p) return;
        const std::lock_guard<std::mutex> lock(all().m);
        for (auto &b : blocks_)
            if (b.p == p && b.used) {
                b.used = false;
                idle_ += b.bytes;
            }
        trim();
    }

    // memory that is no work space (a plan's buffers, a call's lists): Dev::alloc,
    // and once more with every idle block of the device freed if that fails
    static Err alloc(int device, void **p, size_t bytes)
    {
        const std::lock_guard<std::mutex> lock(all().m);
        return alloc_locked(device, p, bytes);
    }

private:
    struct Block {
        void *p;
        size_t bytes;
        bool used;
    };
    struct All {
        std::mutex m;
        std::vector<WorkSpace *> spaces;
    };
    static All &all()
    {
        static All *a = new All;   // (never destroyed: contexts may outlive static objects)
        return *a;
    }

    Block *largest()
    {
        Block *at = nullptr;
        for (auto &b : blocks_)
            if (!b.used && (!at || b.bytes > at->bytes)) at = &b;
        return at;
    }
    void drop(Block *b)
    {
        Dev::release(b->p);
        idle_ -= b->bytes;
        blocks_.erase(blocks_.begin() + (b - blocks_.data()));
    }

    static Err alloc_locked(int device, void **p, size_t bytes)
    {
        const Err e = Dev::alloc(device, p, bytes);
        if (e == Err(0)) return e;
        bool freed = false;
        for (WorkSpace *w : all().spaces)
            if (w->device_ == device)
                while (Block *b = w->largest()) {
                    w->drop(b);
                    freed = true;
                }
        return freed ? Dev::alloc(device, p, bytes) : e;
    }

    // frees idle blocks until what is kept is within the bounds
    void trim()
    {
        if (keep_ == 0) {
            while (Block *b = largest()) drop(b);
            return;
        }
        for (;;) {
            size_t total = 0;
            for (WorkSpace *w : all().spaces) total += w->device_ == device_ ? w->idle_ : 0;
            if (total <= keep_) return;
            WorkSpace *from = nullptr;
            for (WorkSpace *w : all().spaces)
                if (w->device_ == device_ && w->idle_ > 0 &&
                    (!from || w->largest()->bytes > from->largest()->bytes))
                    from = w;
            from->drop(from->largest());
        }
    }

    std::vector<Block> blocks_;
    int device_ = 0;
    size_t keep_ = 0, idle_ = 0;   // idle_: bytes of the blocks not in use
    bool open_ = false;
};

}  // namespace cch
