// Device blocks kept for reuse: the library's allocator behind every buffer of
// a build and a handle.  Host code without HIP types: the driver's calls come
// from the template argument, so the policy runs without a device as well.
//
// Builds allocate and release the same large pools again and again (capacity
// scratch, factor and near-field pools); returning them to the driver and
// mapping them anew each time costs seconds on a busy device, so released
// blocks are kept per device and reused best-fit (a block serves requests of
// 3/4 of its size or more).
//
// Kept blocks must not take the last of the device's memory: the runtime (a
// kernel's private segments, signals, code objects) and the process's other
// allocators ask the driver directly and cannot have them given back.  A
// process that had held three FP64 handles of 40-50 GB kept all but some MB of
// the card in idle blocks, and its next kernel with a private segment aborted
// the queue (out of resources).  So while large blocks are kept, kReserve bytes of
// the device are free as long as blocks can go that the last kRecent allocations
// passed over, and kFloor bytes whatever goes: a miss gives idle blocks back until
// the request fits beside them, and so does a large block that comes back.
// The blocks passed over go first, the oldest before others (a program that has
// moved on to other sizes loses the blocks of the earlier ones and keeps its
// own), then the smallest that covers what is missing, else the largest.  Either
// rule alone has the program map its own blocks anew in every pass: the best fit
// unmaps the pass's scratch while the blocks of earlier handles stay (a build of
// N = 2^20 points 3.8 s instead of 63 ms), the oldest first more than is missing,
// and what the next step needs, once all blocks are of the running pass.
//
// Blocks enter the cache only after the work using them has completed (the
// build synchronises its stream before releasing scratch, destroy
// synchronises the device).
#pragma once
#include <cstddef>
#include <cstdint>
#include <iterator>
#include <map>
#include <mutex>
#include <unordered_set>

namespace hmx {

// Driver: int device(); bool alloc(void**, size_t, bool* oom); bool free(void*);
// void sync(); bool free_bytes(size_t*) (of the current device, 0 on failure)
template <typename Driver>
class BlockCache {
   public:
    // room for a kernel's private segments (8192 waves of 64 lanes: 1 GB at 2 KB a
    // lane), the runtime's own buffers and small tensors
    static constexpr size_t kReserve = (size_t)2 << 30;
    // what stays free where every block is of the running passes (the library's own
    // kernels have no private memory).  A learned BF16 build of N = 2^22 points takes
    // 303 GB of the card's 309 at its peak, beside 4.3 of torch: its second pass takes
    // 0.45 s with its own blocks, 2.7 to 4.9 s where the reserve unmaps some
    static constexpr size_t kFloor = (size_t)256 << 20;
    // a block of at least this size looks at the free memory when it comes
    // back (smaller ones do not move the reserve)
    static constexpr size_t kLarge = (size_t)64 << 20;

    // a build makes about 100 allocations: blocks of the last three passes or so
    static constexpr uint64_t kRecent = 300;

    explicit BlockCache(Driver d = Driver()) : drv_(d) {}

    static size_t round(size_t bytes) {
        const size_t g = bytes >= kLarge ? ((size_t)2 << 20) : 256;
        return (bytes + g - 1) / g * g;
    }

    // *bytes: requested size in, size of the block handed out on return (up to
    // 4/3 of the request); false: the driver has no such block (*oom: for lack
    // of memory)
    bool alloc(void** p, size_t* bytes, bool* oom) {
        const int dev = drv_.device();
        *oom = false;
        {
            std::lock_guard<std::mutex> lk(mu_);
            ++clock_;
            for (auto it = idle_.lower_bound(*bytes); it != idle_.end(); ++it) {
                if (it->first / 4 * 3 > *bytes) break;
                if (it->second.dev != dev) continue;
                *p = it->second.p;
                *bytes = it->first;
                cached_ -= it->first;
                idle_.erase(it);
                return true;
            }
            make_room(dev, *bytes);
        }
        bool ok = drv_.alloc(p, *bytes, oom);
        if (!ok && *oom) {
            std::lock_guard<std::mutex> lk(mu_);
            drv_.sync();
            give_back_all(dev);
            ++flushes_;
            ok = drv_.alloc(p, *bytes, oom);
        }
        if (ok) {
            std::lock_guard<std::mutex> lk(mu_);
            owned_.insert(*p);
            fresh_ += (int64_t)*bytes;
        }
        return ok;
    }

    // a block back into the cache; a pointer that did not come from alloc is
    // never cached (so the cache never frees memory another allocator owns)
    void free(void* p, size_t bytes) {
        const int dev = drv_.device();
        std::lock_guard<std::mutex> lk(mu_);
        if (owned_.count(p) == 0) return;
        idle_.insert({bytes, Block{dev, p, clock_}});
        cached_ += bytes;
        if (bytes >= kLarge) make_room(dev, 0);
    }

    // every idle block of every device back to the driver; their bytes
    int64_t trim() {
        std::lock_guard<std::mutex> lk(mu_);
        drv_.sync();
        return give_back_all(-1);
    }

    size_t cached() {
        std::lock_guard<std::mutex> lk(mu_);
        return cached_;
    }
    // bytes obtained from the driver, and times that idle blocks went back to
    // it for lack of memory, over the process
    int64_t fresh_bytes() {
        std::lock_guard<std::mutex> lk(mu_);
        return fresh_;
    }
    int64_t flushes() {
        std::lock_guard<std::mutex> lk(mu_);
        return flushes_;
    }

   private:
    struct Block {
        int dev;
        void* p;
        uint64_t since;  // allocations made until it came back
    };
    using Idle = std::multimap<size_t, Block>;  // by size

    // large idle blocks of dev back to the driver until `bytes` and what has to stay
    // free beside them are, or none is left that may go
    void make_room(int dev, size_t bytes) {
        if (idle_.empty()) return;
        size_t fr = 0;
        if (!drv_.free_bytes(&fr) || fr >= bytes + kReserve) return;
        bool any = false;
        while (fr < bytes + kReserve) {
            const size_t missing = fr < bytes + kFloor ? bytes + kFloor - fr : 0;
            auto pick = idle_.end();
            bool old = false, covers = false;
            for (auto it = idle_.lower_bound(kLarge); it != idle_.end(); ++it) {  // by size
                if (it->second.dev != dev) continue;
                if (clock_ - it->second.since > kRecent) {
                    if (!old || it->second.since < pick->second.since) pick = it;
                    old = true;
                } else if (missing > 0 && !old && !covers) {
                    pick = it;
                    covers = it->first >= missing;
                }
            }
            if (pick == idle_.end()) break;
            if (!any) drv_.sync();
            any = true;
            const size_t b = pick->first;
            if (!give_back(pick)) break;
            fr += b;
        }
        if (any) ++flushes_;
    }

    bool give_back(typename Idle::iterator it) {
        if (!drv_.free(it->second.p)) return false;
        owned_.erase(it->second.p);
        cached_ -= it->first;
        idle_.erase(it);
        return true;
    }

    // (dev < 0: of every device)
    int64_t give_back_all(int dev) {
        int64_t tot = 0;
        for (auto it = idle_.begin(); it != idle_.end();) {
            const auto next = std::next(it);
            const int64_t b = (int64_t)it->first;
            if ((dev < 0 || it->second.dev == dev) && give_back(it)) tot += b;
            it = next;
        }
        return tot;
    }

    Driver drv_;
    std::mutex mu_;
    Idle idle_;
    uint64_t clock_ = 0;
    size_t cached_ = 0;
    // every block obtained from the driver and not given back: only these
    // may enter the cache and be freed by it
    std::unordered_set<void*> owned_;
    int64_t fresh_ = 0, flushes_ = 0;
};

// b grown to at least `bytes` (the block handed out may be larger than asked, so
// each buffer is held to its own size): grow(b, bytes) replaces it
template <typename Buf, typename Grow>
void fit(Buf& b, size_t bytes, Grow&& grow) {
    if (!b.p || b.bytes < bytes) grow(b, bytes);
}

// keys and work space of a sort that is repeated with other counts
template <typename Buf>
struct SortSpace {
    Buf keys, scratch;
    template <typename Grow>
    void reserve(size_t keys_bytes, size_t scratch_bytes, Grow&& grow) {
        fit(keys, keys_bytes, grow);
        fit(scratch, scratch_bytes, grow);
    }
};

}  // namespace hmx
