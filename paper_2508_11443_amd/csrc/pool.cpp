// The library's own device memory: what a build takes when the caller gives no allocator.
//
// Building a map takes and returns a handful of blocks of up to gigabytes.  Through
// hipMallocAsync / hipFreeAsync the same build and release in a loop cost far more than its
// kernels: a release 0.3-0.6 ms of host time, and a build now and then 10 ms to 1.4 s when the
// runtime mapped new memory instead of reusing what had just been returned (build + 10^7
// lookups + release: 0.75 ms at best, 9-18 ms on average).  Here blocks are cut from segments
// of hipMalloc'd memory, best fit, and merged with their neighbours when they come back.
//
// Order.  A block that comes back "settled" (the host has waited for its last use) may be
// handed out again at once.  One that comes back on the null stream may still be in use by work
// queued before that; it is handed to the null stream as it is, and to another stream after
// that stream has been made to wait for the null stream.  One that comes back on any other
// stream carries an event recorded there and stays aside until the event is done, or until a
// stream that needs a block of its size is made to wait for the event.  No kept stream handle
// is used: a stream may be destroyed after the call.
//
// Segments.  A block that lives on (a map's) has a segment to itself, so that its memory can go back
// to the driver when it comes back; a free segment is taken for it only if it is at most an eighth
// larger.  Scratch, which comes back when its call is over, is cut from any free memory.  Blocks of
// up to kSmall bytes of either kind share segments of kSmallSegment (the driver's own allocations are
// multiples of 2 MiB: 4000 maps of 20000 keys, 2.7 GB, held 8.4 GB with a segment for each table).  A
// build that cannot know its table's size yet takes room for a larger one (take_room) and gives back the
// end; such ends, which only scratch and small blocks can use while the table lives, hold at most
// a 64th of the device's memory, and beyond that no room is to be had.  (When every table had room and later tables' blocks were cut from the ends
// of earlier ones, 44 maps of 2^25 keys held 43 GB more than their tables, and none of it could go back.)
//
// Bounds.  Of free memory, at most an eighth of the device's is kept: whole free segments go back to
// the driver, largest first, when a build or a release call leaves more than 7/64 of the device's memory
// in them (hipFree waits for the device, so nothing queued still uses them), and all of them before an
// allocation fails.  Lookups (kTry) neither wait for anything nor give anything to the driver.
// One mutex per device; streams under capture take hipMallocAsync, which a graph can record.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <set>
#include <vector>

#include "fks_internal.hpp"

namespace fks {
namespace {

constexpr size_t kAlign = 512;
constexpr size_t kSmall = 4 << 20;           // largest block of a small segment
constexpr size_t kSmallSegment = 32 << 20;
constexpr size_t kPage = 2 << 20;            // large segments are whole pages
constexpr int kMaxDevices = 64;

// While another thread captures a graph in the default (global) mode, hipMalloc, hipFree and calls on
// events (hipEventQuery, which every call here may make) are refused, and spoil the capture; none
// of them touches its streams.  Held wherever a pool makes such calls.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

class Pool {
  public:
    Pool() {
        RelaxedCapture relaxed;
        size_t free_now = 0, total = 0;
        if (hipMemGetInfo(&free_now, &total) == hipSuccess) eighth_ = total / 8;
    }

    void* take(size_t bytes, hipStream_t s, PoolUse use) {
        bytes = round_up(bytes, kAlign);
        std::unique_lock<std::mutex> lk(mu_);
        collect(false);
        if (void* p = find(bytes, s, use)) return p;
        if (grow(bytes)) return fit(bytes, s, use);
        if (use == kTry) return nullptr;
        // the driver has no more: wait for what is on its way back, then return every free segment
        collect(true);
        if (void* p = fit(bytes, s, use)) return p;
        const std::vector<char*> freed = shrink(0);
        lk.unlock();
        to_driver(freed);
        lk.lock();
        return grow(bytes) ? fit(bytes, s, use) : nullptr;
    }

    // a block that lives on, of `most` bytes, of which about `least` will be used and the rest trimmed
    void* take_room(size_t most, size_t least, hipStream_t s) {
        most = round_up(most, kAlign);
        const size_t spare = most - std::min(most, least);
        std::lock_guard<std::mutex> lk(mu_);
        if (ends_ + spare > eighth_ / 8) return nullptr;
        collect(false);
        void* p = find(most, s, kKept);
        if (!p && grow(most)) p = fit(most, s, kKept);
        if (p) {
            chunks_.find((char*)p)->second.end = spare;
            ends_ += spare;
        }
        return p;
    }

    // false: the pointer is not one of this pool's
    bool give(void* p, hipStream_t s, bool settled, PoolUse use) {
        std::unique_lock<std::mutex> lk(mu_);
        auto it = chunks_.find((char*)p);
        if (it == chunks_.end() || it->second.state != kUsed) return false;
        ends_ -= it->second.end;
        it->second.end = 0;
        if (settled) {
            release(it, kIdle);
        } else if (s == nullptr) {
            ++null_gives_;
            release(it, kNull);
        } else {
            RelaxedCapture relaxed;
            hipEvent_t ev = nullptr;
            if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) ev = nullptr;
            if (ev && hipEventRecord(ev, s) != hipSuccess) {
                (void)hipEventDestroy(ev);
                ev = nullptr;
            }
            if (ev) {
                it->second.state = kPending;
                pending_.push_back({it->first, ev, s});
                pending_bytes_ += it->second.size;
            } else {
                (void)hipGetLastError();
                (void)hipStreamSynchronize(s);
                release(it, kIdle);
            }
        }
        if (use != kTry && whole_bytes_ > eighth_ - eighth_ / 8) {
            const std::vector<char*> freed = shrink(eighth_ - eighth_ / 8);
            lk.unlock();
            to_driver(freed);
        }
        return true;
    }

    // the end of a block, from `bytes` on, is not needed and nothing uses it
    bool trim(void* p, size_t bytes) {
        bytes = round_up(bytes, kAlign);
        std::lock_guard<std::mutex> lk(mu_);
        auto it = chunks_.find((char*)p);
        if (it == chunks_.end() || it->second.state != kUsed) return false;
        const size_t end = it->second.size < bytes + kAlign ? 0 : it->second.size - bytes;
        ends_ += end - it->second.end;
        it->second.end = end;
        if (!end) return true;
        it->second.size = bytes;
        Chunk rest{end, 0, kUsed, false, it->second.small};
        release(chunks_.emplace_hint(std::next(it), it->first + bytes, rest), kIdle);
        return true;
    }

  private:
    enum State { kUsed, kIdle, kNull, kPending };
    enum Kind { kInSmall, kPart, kWhole };   // of free memory: of a small segment, part of a segment, all of it
    struct Chunk {
        size_t size;
        size_t end;          // used blocks: what was or will be trimmed of it, in ends_
        State state;
        bool first, small;   // first: a segment starts here
    };
    using Chunks = std::map<char*, Chunk>;
    using Index = std::set<std::pair<size_t, char*>>;
    using Found = std::pair<Index*, Index::iterator>;

    static size_t round_up(size_t n, size_t to) { return (n + to - 1) & ~(to - 1); }

    // all of a segment
    bool whole(Chunks::iterator it) const {
        auto next = std::next(it);
        return it->second.first && (next == chunks_.end() || next->second.first);
    }
    Index& index(Chunks::iterator it) {
        return free_[it->second.state == kNull][it->second.small ? kInSmall : whole(it) ? kWhole : kPart];
    }
    void list(Chunks::iterator it, State st) {
        it->second.state = st;
        index(it).insert({it->second.size, it->first});
        if (whole(it)) whole_bytes_ += it->second.size;
    }
    void unlist(Chunks::iterator it) {
        index(it).erase({it->second.size, it->first});
        if (whole(it)) whole_bytes_ -= it->second.size;
    }
    static bool is_free(const Chunk& c) { return c.state == kIdle || c.state == kNull; }

    // a block comes back: merged with its free neighbours of the same segment
    void release(Chunks::iterator it, State st) {
        auto next = std::next(it);
        if (next != chunks_.end() && !next->second.first && is_free(next->second)) {
            unlist(next);
            if (next->second.state == kNull) st = kNull;
            it->second.size += next->second.size;
            chunks_.erase(next);
        }
        if (!it->second.first) {
            auto prev = std::prev(it);
            if (is_free(prev->second)) {
                unlist(prev);
                if (prev->second.state == kNull) st = kNull;
                prev->second.size += it->second.size;
                chunks_.erase(it);
                it = prev;
            }
        }
        list(it, st);
    }

    // The smallest free memory for a block, of one order.  (Scratch from the ends of tables before whole
    // segments: 10^7 keys' build, lookup and release 504 us instead of 497, as the lookup's then was not
    // what the build had just used.)
    Found best(size_t bytes, bool null_ordered, PoolUse use) {
        Index* const kinds = free_[null_ordered];
        auto in = [&](Kind k, size_t most) -> Found {
            auto it = kinds[k].lower_bound({bytes, nullptr});
            return it != kinds[k].end() && it->first <= most ? Found{&kinds[k], it} : Found{nullptr, {}};
        };
        if (bytes <= kSmall) return in(kInSmall, ~(size_t)0);
        if (use == kKept) return in(kWhole, std::max(bytes + bytes / 8, segment(bytes)));
        const Found a = in(kPart, ~(size_t)0), b = in(kWhole, ~(size_t)0);
        return !a.first || (b.first && b.second->first < a.second->first) ? b : a;
    }

    void* fit(size_t bytes, hipStream_t s, PoolUse use) {
        const Found a = best(bytes, false, use), b = best(bytes, true, use);
        if (!a.first && !b.first) return nullptr;
        // a block that another stream has to wait for only when there is no other
        const bool from_b = !a.first || (b.first && s == nullptr && b.second->first < a.second->first);
        if (from_b && s != nullptr && !after_null(s)) return nullptr;
        auto it = chunks_.find(from_b ? b.second->second : a.second->second);
        const State st = it->second.state;
        unlist(it);
        it->second.state = kUsed;
        if (it->second.size - bytes >= kAlign && (it->second.small || use != kKept)) {
            Chunk rest{it->second.size - bytes, 0, kUsed, false, it->second.small};
            it->second.size = bytes;
            list(chunks_.emplace_hint(std::next(it), it->first + bytes, rest), st);
        }
        return it->first;
    }

    void* find(size_t bytes, hipStream_t s, PoolUse use) {
        if (void* p = fit(bytes, s, use)) return p;
        return bytes <= kSmall ? nullptr : adopt(bytes, s, use);
    }

    // Stream s waits for everything that was queued on the null stream when its last block came back.  One
    // event serves all blocks that came back until then (2^16 keys' build, lookup and release on a stream
    // of the caller's 82 us, 126 with an event created and waited for by each block).
    bool after_null(hipStream_t s) {
        RelaxedCapture relaxed;
        if (!fence_ && hipEventCreateWithFlags(&fence_, hipEventDisableTiming) != hipSuccess) fence_ = nullptr;
        bool ok = fence_ != nullptr;
        if (ok && fenced_ != null_gives_) {
            ok = hipEventRecord(fence_, nullptr) == hipSuccess;
            if (ok) fenced_ = null_gives_;
        }
        if (ok && hipEventQuery(fence_) != hipSuccess) {
            (void)hipGetLastError();   // not done
            ok = hipStreamWaitEvent(s, fence_, 0) == hipSuccess;
        }
        if (!ok) (void)hipGetLastError();
        return ok;
    }

    // blocks whose events are done become free
    void collect(bool wait) {
        if (pending_.empty()) return;
        RelaxedCapture relaxed;
        for (size_t i = 0; i < pending_.size();) {
            const hipError_t e = wait ? hipEventSynchronize(pending_[i].done) : hipEventQuery(pending_[i].done);
            if (e != hipSuccess) {
                (void)hipGetLastError();
                ++i;
                continue;
            }
            auto it = chunks_.find(pending_[i].block);
            forget(i);
            release(it, kIdle);
        }
    }
    void forget(size_t i) {
        pending_bytes_ -= chunks_.find(pending_[i].block)->second.size;
        (void)hipEventDestroy(pending_[i].done);
        pending_[i] = pending_.back();
        pending_.pop_back();
    }

    // A large block that another call's work may still use, for stream s to use after it: one that
    // came back on a stream of the same handle (nothing is waited for unless the stream is a
    // new one), or any, once more waits on its way back than the pool keeps free.  So calls queued
    // one behind the other share a block, and calls on many streams cannot pile up memory.
    void* adopt(size_t bytes, hipStream_t s, PoolUse use) {
        if (pending_.empty()) return nullptr;
        RelaxedCapture relaxed;
        for (size_t i = 0; i < pending_.size(); ++i) {
            auto it = chunks_.find(pending_[i].block);
            if (it->second.small || it->second.size < bytes) continue;
            if (use == kKept ? !whole(it) || it->second.size > bytes + bytes / 8 : it->second.size / 2 > bytes) continue;
            if (pending_[i].stream != s && pending_bytes_ <= eighth_) continue;
            if (hipStreamWaitEvent(s, pending_[i].done, 0) != hipSuccess) {
                (void)hipGetLastError();
                continue;
            }
            forget(i);
            it->second.state = kUsed;
            return it->first;
        }
        return nullptr;
    }

    // bytes of a segment for such a block
    static size_t segment(size_t bytes) {
        return bytes <= kSmall ? kSmallSegment : round_up(bytes, kPage);
    }
    bool grow(size_t bytes) {
        RelaxedCapture relaxed;
        void* p = nullptr;
        if (hipMalloc(&p, segment(bytes)) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        list(chunks_.emplace((char*)p, Chunk{segment(bytes), 0, kUsed, true, bytes <= kSmall}).first, kIdle);
        return true;
    }

    // whole free segments, the largest first, until at most `keep` bytes of them are left; they are the
    // caller's, to be given to the driver without the lock (hipFree waits)
    std::vector<char*> shrink(size_t keep) {
        std::vector<char*> out;
        while (whole_bytes_ > keep) {
            auto largest = chunks_.end();
            for (Index(&kinds)[3] : free_)
                for (int k : {kWhole, kInSmall}) {   // a free small segment is the largest of its kind
                    if (kinds[k].empty()) continue;
                    auto it = chunks_.find(kinds[k].rbegin()->second);
                    if (whole(it) && (largest == chunks_.end() || it->second.size > largest->second.size)) largest = it;
                }
            if (largest == chunks_.end()) break;
            out.push_back(largest->first);
            unlist(largest);
            chunks_.erase(largest);
        }
        return out;
    }
    static void to_driver(const std::vector<char*>& segments) {
        RelaxedCapture relaxed;
        for (char* p : segments)
            if (hipFree(p) != hipSuccess) (void)hipGetLastError();
    }

    std::mutex mu_;
    size_t eighth_ = 4ull << 30;   // of the device's memory
    size_t whole_bytes_ = 0;       // of free segments
    size_t ends_ = 0;              // trimmed, or to be trimmed, of blocks in use
    Chunks chunks_;                // every block, by address
    Index free_[2][3];             // free memory by size: [settled, null-ordered][Kind]
    struct Pending {
        char* block;
        hipEvent_t done;
        hipStream_t stream;   // compared, never used: it may have been destroyed
    };
    hipEvent_t fence_ = nullptr;             // on the null stream, behind the first fenced_ blocks returned on it
    uint64_t null_gives_ = 0, fenced_ = 0;
    std::vector<Pending> pending_;
    size_t pending_bytes_ = 0;
};

std::mutex g_mu;
Pool* g_pool[kMaxDevices];   // never destroyed: objects may outlive static destructors

Pool* pool_of(int dev, bool create) {
    if (dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g_pool[dev] && create) g_pool[dev] = new Pool;
    return g_pool[dev];
}

// The lists above take host memory, and callers are C entry points: what they throw ends here, and
// counts as no memory (a block that could not be listed stays unused).
template <typename Call, typename Result>
Result guarded(Call call, Result otherwise) {
    try {
        return call();
    } catch (...) {
        return otherwise;
    }
}

// the current device's pool, for work on stream s; null while s is captured
Pool* pool_for(hipStream_t s) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (s != nullptr && hipStreamIsCapturing(s, &cap) != hipSuccess) (void)hipGetLastError();
    return cap == hipStreamCaptureStatusNone ? pool_of(dev, true) : nullptr;
}

}  // namespace

void* pool_take(size_t bytes, hipStream_t s, PoolUse use) {
    void* p = guarded([&]() -> void* {
        Pool* pool = pool_for(s);
        return pool ? pool->take(bytes, s, use) : nullptr;
    }, (void*)nullptr);
    if (p || use == kTry) return p;
    const hipError_t e = hipMallocAsync(&p, bytes, s);
    if (e != hipSuccess) {
        set_hip_error(e);
        (void)hipGetLastError();
        return nullptr;
    }
    return p;
}

void* pool_take_room(size_t most, size_t least, hipStream_t s) {
    return guarded([&]() -> void* {
        Pool* pool = pool_for(s);
        return pool ? pool->take_room(most, least, s) : nullptr;
    }, (void*)nullptr);
}

void pool_give(void* p, hipStream_t s, bool settled, PoolUse use) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    const bool ours = guarded([&] {
        Pool* pool = pool_of(dev, false);
        return pool && pool->give(p, s, settled, use);
    }, true);
    if (!ours) (void)hipFreeAsync(p, s);
}

bool pool_trim(void* p, size_t bytes) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    return guarded([&] {
        Pool* pool = pool_of(dev, false);
        return pool && bytes && pool->trim(p, bytes);
    }, false);
}

}  // namespace fks
