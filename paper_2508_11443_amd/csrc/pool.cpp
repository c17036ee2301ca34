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
// Bounds.  Free memory above an eighth of the device's is given back to the driver, whole
// segments at a time (hipFree waits for the device, so nothing queued still uses them); when the
// driver has none left every free segment is given back before an allocation fails.  Small
// blocks have segments of their own, so that a small map does not pin a large segment.
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
constexpr size_t kSmall = 1 << 20;           // largest block of a small segment
constexpr size_t kSmallSegment = 32 << 20;
constexpr size_t kPage = 2 << 20;            // large segments are whole pages of this size
constexpr int kMaxDevices = 64;

// hipMalloc and hipFree are refused, and spoil the capture, while another thread captures a
// graph in the default (global) mode; they do not touch its streams
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

class Pool {
  public:
    explicit Pool(int dev) : dev_(dev) {
        size_t free_now = 0, total = 0;
        if (hipMemGetInfo(&free_now, &total) == hipSuccess) keep_ = total / 8;
    }

    void* take(size_t bytes, hipStream_t s) {
        bytes = (bytes + kAlign - 1) & ~(kAlign - 1);
        std::lock_guard<std::mutex> lk(mu_);
        collect(false);
        const bool small = bytes <= kSmall;
        if (void* p = fit(bytes, small, s)) return p;
        if (void* p = small ? nullptr : adopt(bytes, s)) return p;
        const size_t seg = small ? kSmallSegment : (bytes + kPage - 1) & ~(kPage - 1);
        if (!grow(seg, small)) {
            // the driver has no more: wait for what is on its way back, then return every free segment
            collect(true);
            if (void* p = fit(bytes, small, s)) return p;
            shrink(0);
            if (!grow(seg, small)) return nullptr;
        }
        return fit(bytes, small, s);
    }

    // false: the pointer is not one of this pool's
    bool give(void* p, hipStream_t s, bool settled) {
        std::lock_guard<std::mutex> lk(mu_);
        auto it = chunks_.find((char*)p);
        if (it == chunks_.end() || it->second.state != kUsed) return false;
        if (settled) {
            release(it, kIdle);
        } else if (s == nullptr) {
            release(it, kNull);
        } else {
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
        if (free_bytes_ > keep_) shrink(keep_);
        return true;
    }

    // the end of a block, from `bytes` on, is not needed and nothing uses it
    bool trim(void* p, size_t bytes) {
        bytes = (bytes + kAlign - 1) & ~(kAlign - 1);
        std::lock_guard<std::mutex> lk(mu_);
        auto it = chunks_.find((char*)p);
        if (it == chunks_.end() || it->second.state != kUsed) return false;
        if (it->second.size < bytes + kAlign) return true;
        Chunk rest{it->second.size - bytes, kUsed, false, it->second.small};
        it->second.size = bytes;
        release(chunks_.emplace_hint(std::next(it), it->first + bytes, rest), kIdle);
        return true;
    }

  private:
    enum State { kUsed, kIdle, kNull, kPending };
    struct Chunk {
        size_t size;
        State state;
        bool first, small;   // first: a segment starts here
    };
    using Chunks = std::map<char*, Chunk>;
    using Index = std::set<std::pair<size_t, char*>>;

    Index& index(State st, bool small) { return free_[st == kNull ? 1 : 0][small ? 1 : 0]; }

    void list(Chunks::iterator it, State st) {
        it->second.state = st;
        index(st, it->second.small).insert({it->second.size, it->first});
        free_bytes_ += it->second.size;
    }
    void unlist(Chunks::iterator it) {
        index(it->second.state, it->second.small).erase({it->second.size, it->first});
        free_bytes_ -= it->second.size;
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

    void* fit(size_t bytes, bool small, hipStream_t s) {
        auto a = index(kIdle, small).lower_bound({bytes, nullptr});
        auto b = index(kNull, small).lower_bound({bytes, nullptr});
        const bool has_a = a != index(kIdle, small).end(), has_b = b != index(kNull, small).end();
        if (!has_a && !has_b) return nullptr;
        // a block that another stream has to wait for only when there is no other
        const bool from_b = !has_a || (has_b && s == nullptr && b->first < a->first);
        if (from_b && s != nullptr && !after_null(s)) return nullptr;
        auto it = chunks_.find(from_b ? b->second : a->second);
        unlist(it);
        if (it->second.size - bytes >= kAlign) {
            Chunk rest{it->second.size - bytes, it->second.state, false, small};
            it->second.size = bytes;
            auto r = chunks_.emplace_hint(std::next(it), it->first + bytes, rest);
            list(r, rest.state);
        }
        it->second.state = kUsed;
        return it->first;
    }

    // stream s waits for everything queued on the null stream so far
    static bool after_null(hipStream_t s) {
        hipEvent_t ev = nullptr;
        if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) return false;
        const bool ok = hipEventRecord(ev, nullptr) == hipSuccess && hipStreamWaitEvent(s, ev, 0) == hipSuccess;
        (void)hipEventDestroy(ev);   // released once it is done
        if (!ok) (void)hipGetLastError();
        return ok;
    }

    // blocks whose events are done become free
    void collect(bool wait) {
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
    void* adopt(size_t bytes, hipStream_t s) {
        for (size_t i = 0; i < pending_.size(); ++i) {
            auto it = chunks_.find(pending_[i].block);
            if (it->second.small || it->second.size < bytes || it->second.size / 2 > bytes) continue;
            if (pending_[i].stream != s && pending_bytes_ <= keep_) continue;
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

    bool grow(size_t seg, bool small) {
        RelaxedCapture relaxed;
        void* p = nullptr;
        const hipError_t e = hipMalloc(&p, seg);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        list(chunks_.emplace((char*)p, Chunk{seg, kIdle, true, small}).first, kIdle);
        return true;
    }

    // gives back whole free segments, the largest first, until at most `keep` free bytes are left
    void shrink(size_t keep) {
        RelaxedCapture relaxed;
        for (bool more = true; more && free_bytes_ > keep;) {
            more = false;
            auto best = chunks_.end();
            for (auto it = chunks_.begin(); it != chunks_.end(); ++it) {
                auto next = std::next(it);
                const bool whole = it->second.first && (next == chunks_.end() || next->second.first);
                if (whole && is_free(it->second) && (best == chunks_.end() || it->second.size > best->second.size))
                    best = it;
            }
            if (best != chunks_.end() && hipFree(best->first) == hipSuccess) {
                unlist(best);
                chunks_.erase(best);
                more = true;
            }
        }
    }

    const int dev_;
    std::mutex mu_;
    size_t keep_ = 4ull << 30, free_bytes_ = 0;
    Chunks chunks_;                 // every block, by address
    Index free_[2][2];              // free blocks by size: [settled, null-ordered][large, small]
    struct Pending {
        char* block;
        hipEvent_t done;
        hipStream_t stream;   // compared, never used: it may have been destroyed
    };
    std::vector<Pending> pending_;
    size_t pending_bytes_ = 0;
};

std::mutex g_mu;
Pool* g_pool[kMaxDevices];   // never destroyed: objects may outlive static destructors

Pool* pool_of(int dev, bool create) {
    if (dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g_pool[dev] && create) g_pool[dev] = new Pool(dev);
    return g_pool[dev];
}

}  // namespace

void* pool_take(size_t bytes, hipStream_t s) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (s != nullptr && hipStreamIsCapturing(s, &cap) != hipSuccess) (void)hipGetLastError();
    Pool* pool = cap == hipStreamCaptureStatusNone ? pool_of(dev, true) : nullptr;
    void* p = pool ? pool->take(bytes, s) : nullptr;
    if (p) return p;
    const hipError_t e = hipMallocAsync(&p, bytes, s);
    if (e != hipSuccess) {
        set_hip_error(e);
        (void)hipGetLastError();
        return nullptr;
    }
    return p;
}

void pool_give(void* p, hipStream_t s, bool settled) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    Pool* pool = pool_of(dev, false);
    if (pool && pool->give(p, s, settled)) return;
    (void)hipFreeAsync(p, s);
}

bool pool_trim(void* p, size_t bytes) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    Pool* pool = pool_of(dev, false);
    return pool && bytes && pool->trim(p, bytes);
}

}  // namespace fks
