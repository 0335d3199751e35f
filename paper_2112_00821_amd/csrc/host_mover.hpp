// Copies between device memory and a caller's host memory.
//
// The runtime's own copy to pageable memory moves one staged chunk at a time
// and empties it with one thread: 17 GB/s here, where the link does about 50
// and one thread's memcpy is what it waits for.  A HostMover keeps two
// pinned slots: while one is emptied by the calling thread and a few helpers,
// the next chunk crosses the link into the other.  41 MB of maps (1920x1080):
// 2.4 ms before, 1.05 ms so.  Page-locked destinations need none of it: the
// runtime copies straight into them (41 MB: 0.76 ms, 1.09 ms by the slots).
//
// A mover belongs to one handle (or server) and is used under its lock; slots
// and helper threads are made on first use and given back with it.  Helpers
// sleep between transfers.  Without free CPUs, memory for the slots, or
// threads, the runtime copies.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

namespace fmvs {

// `rows` rows of `bytes` bytes.
struct HostPiece {
    uint8_t *dst;
    const uint8_t *src;
    size_t bytes, rows, dst_pitch, src_pitch;
    void copy() const {
        for (size_t r = 0; r < rows; ++r) std::memcpy(dst + r * dst_pitch, src + r * src_pitch, bytes);
    }
};

struct DeviceRange {
    void *dst;
    const void *src;
    size_t bytes;
};

// A frame's maps, or one transfer (in place: copies need no host memory).
struct DeviceRanges {
    DeviceRange r[3];
    size_t n = 0;
    void add(void *dst, const void *src, size_t bytes) {
        if (dst && bytes) r[n++] = DeviceRange{dst, src, bytes};
    }
};

// A thread of the process inside a call that copies, or waits to.
struct HostCaller {
    HostCaller() { now().fetch_add(1); }
    ~HostCaller() { now().fetch_sub(1); }
    HostCaller(const HostCaller &) = delete;
    static std::atomic<int> &now() {
        static std::atomic<int> n{0};
        return n;
    }
};

class HostMover {
public:
    HostMover() = default;
    HostMover(const HostMover &) = delete;
    HostMover &operator=(const HostMover &) = delete;
    ~HostMover() {
        {
            std::lock_guard<std::mutex> lk(m_);
            stop_ = true;
        }
        cv_.notify_all();
        for (auto &t : threads_) t.join();
        for (auto &e : events_)
            if (e) hipEventDestroy(e);
        if (pin_) hipHostFree(pin_);
    }

    // Copy pieces between host buffers with helpers, where that is worth
    // waking them and CPUs are free; false: nothing is copied.
    bool copy(const std::vector<HostPiece> &pieces) {
        size_t total = 0;
        for (auto &p : pieces) total += p.bytes * p.rows;
        if (total < kShare) return false;
        Session s(*this);
        if (s.taken == 0) return false;
        s.wake();
        share(pieces.data(), pieces.size());
        return true;
    }

    // Device ranges to host memory, after the work already on the stream;
    // returns when the bytes are there, on an error when no copy still runs.
    // Ranges whose destination the runtime knows go straight there in one
    // copy.
    hipError_t to_host(const DeviceRanges &ranges, hipStream_t stream) {
        if (ranges.n == 0) return hipSuccess;
        DeviceRanges staged, direct;
        if (!split(ranges, staged, direct)) return whole(ranges, stream);
        Session s(*this);
        if (s.taken == 0 || !slots()) return whole(ranges, stream);
        hipError_t e = whole(direct, stream);
        if (e == hipSuccess) e = through_slots(staged, stream, s);
        if (e != hipSuccess) (void)hipStreamSynchronize(stream);
        return e;
    }

    // What the first to_host of these ranges (of so many bytes) would make,
    // slots and helpers, ahead of it: while a frame runs.
    void prepare(const DeviceRanges &ranges) {
        DeviceRanges staged, direct;
        if (!pin_ && split(ranges, staged, direct)) prepare(kShare);
    }
    void prepare(size_t bytes) {
        if (!pin_ && bytes >= kShare && free_cpus() >= kLeast && slots()) helpers();
    }

    static constexpr size_t kPiece = 128 << 10;

private:
    // 2 MB slots (1 MB: 31 GB/s, 2 MB: 39, 4 MB: 44; a third and fourth slot
    // change nothing); below 1 MB a transfer is not worth waking helpers
    static constexpr size_t kSlot = 2 << 20, kSlots = 2, kShare = 1 << 20;
    static constexpr int kHelpers = 5;   // 3: 37 GB/s, 5: 39, 7: the same
    // Helpers wait actively for their pieces, so they are for CPUs that are
    // free: kCallerCpus are left to each thread that polls, copies or submits
    // now (its own, the runtime's and the program's work), and fewer than
    // kLeast helpers are not worth the slots: without them the runtime copies.
    // 640x480 frames a second of 1, 2, 4, 8 and 14 threads with a handle each,
    // 16 CPUs: always with helpers 1410, 2100, 2560, 1490 and 1770, never 1190,
    // 1900, 3310, 3950 and 4210, by this rule 1465, 2350, 3110, 3775 and 4160.
    static constexpr int kLeast = 2, kCallerCpus = 5;
    int free_cpus() const { return cpus_ - kCallerCpus * std::max(1, HostCaller::now().load()); }
    // Helpers of running sessions, over all movers.
    static std::atomic<int> &in_use() {
        static std::atomic<int> n{0};
        return n;
    }

    uint8_t *slot(size_t k) { return pin_ + k * kSlot; }

    // Whether p is ordinary host memory: neither page-locked nor device
    // memory, which one copy by the runtime reaches at link rate.
    static bool pageable(const void *p) {
        hipPointerAttribute_t a;
        if (hipPointerGetAttributes(&a, p) == hipSuccess) return a.type == hipMemoryTypeUnregistered;
        (void)hipGetLastError();
        return true;
    }

    // The ranges into ordinary memory and the others; whether the first are
    // worth the slots.
    static bool split(const DeviceRanges &ranges, DeviceRanges &staged, DeviceRanges &direct) {
        size_t total = 0;
        for (size_t i = 0; i < ranges.n; ++i) total += ranges.r[i].bytes;
        if (total < kShare) return false;
        total = 0;
        for (size_t i = 0; i < ranges.n; ++i) {
            const DeviceRange &r = ranges.r[i];
            const bool own = pageable(r.dst);
            (own ? staged : direct).add(r.dst, r.src, r.bytes);
            total += own ? r.bytes : 0;
        }
        return total >= kShare;
    }

    // One copy each, by the runtime.
    static hipError_t whole(const DeviceRanges &ranges, hipStream_t stream) {
        if (ranges.n == 0) return hipSuccess;
        hipError_t e = hipSuccess;
        for (size_t i = 0; i < ranges.n && e == hipSuccess; ++i)
            e = hipMemcpyAsync(ranges.r[i].dst, ranges.r[i].src, ranges.r[i].bytes, hipMemcpyDeviceToHost, stream);
        const hipError_t es = hipStreamSynchronize(stream);
        return e == hipSuccess ? es : e;
    }

    struct Session;

    // With the helpers of a session; after an error copies into the slots may
    // still run.
    hipError_t through_slots(const DeviceRanges &ranges, hipStream_t stream, Session &s) {
        DeviceRange in[kSlots];   // what each slot receives
        size_t at = 0, off = 0, sent = 0;
        auto send = [&] {   // the next chunk
            const DeviceRange &r = ranges.r[at];
            const size_t k = sent++ % kSlots, bytes = std::min(kSlot, r.bytes - off);
            in[k] = DeviceRange{(uint8_t *)r.dst + off, (const uint8_t *)r.src + off, bytes};
            off += bytes;
            if (off == r.bytes) {
                ++at;
                off = 0;
            }
            const hipError_t e = hipMemcpyAsync(slot(k), in[k].src, bytes, hipMemcpyDeviceToHost, stream);
            return e == hipSuccess ? hipEventRecord(events_[k], stream) : e;
        };
        hipError_t e = hipSuccess;
        while (e == hipSuccess && sent < kSlots && at < ranges.n) e = send();
        s.wake();   // (while the first chunk is on its way)
        for (size_t i = 0; i < sent && e == hipSuccess; ++i) {
            const size_t k = i % kSlots;
            if ((e = hipEventSynchronize(events_[k])) != hipSuccess) break;
            HostPiece pieces[kSlot / kPiece];
            size_t n = 0;
            for (size_t o = 0; o < in[k].bytes; o += kPiece)
                pieces[n++] = HostPiece{(uint8_t *)in[k].dst + o, slot(k) + o, std::min(kPiece, in[k].bytes - o), 1, 0, 0};
            share(pieces, n);
            if (at < ranges.n) e = send();
        }
        return e;
    }

    bool slots() {
        if (pin_) return true;
        void *p = nullptr;
        if (hipHostMalloc(&p, kSlot * kSlots) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        for (auto &e : events_)
            if (!e && hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
                (void)hipGetLastError();
                e = nullptr;
                hipHostFree(p);
                return false;
            }
        pin_ = (uint8_t *)p;
        return true;
    }

    void helpers() {
        try {
            while ((int)threads_.size() < kHelpers) threads_.emplace_back([this, i = (int)threads_.size()] { help(i); });
        } catch (...) {   // no thread, or no memory for one: with fewer
        }
    }

    // Helpers are a session's from its start and take part from wake() on.
    struct Session {
        HostMover &m;
        int taken = 0;
        explicit Session(HostMover &mm) : m(mm) {
            int n = in_use().load();
            do {
                taken = std::min(kHelpers, m.free_cpus() - n);
                if (taken < kLeast) {
                    taken = 0;
                    return;
                }
            } while (!in_use().compare_exchange_weak(n, n + taken));
            m.helpers();
            const int made = (int)m.threads_.size() < kLeast ? 0 : std::min(taken, (int)m.threads_.size());
            in_use().fetch_sub(taken - made);
            taken = made;
        }
        void wake() {
            {
                std::lock_guard<std::mutex> lk(m.m_);
                m.active_.store(taken);
            }
            m.cv_.notify_all();
        }
        Session(const Session &) = delete;
        ~Session() {
            m.active_.store(0);
            in_use().fetch_sub(taken);
        }
    };

    // One batch: every piece copied when this returns.  state_ holds the
    // batch's number and the next piece to take.  A taker reads it before
    // count_, and count_ before pieces_; here they are set in that order and
    // count_ is 0 between batches, so what it reads belongs to one batch or
    // its exchange fails.
    void share(const HostPiece *pieces, size_t n) {
        if (n == 0) return;
        state_.store(((state_.load() >> 32) + 1) << 32);
        done_.store(0);
        pieces_.store(pieces);
        count_.store((uint32_t)n);
        work();
        while (done_.load() < n) pause();
        count_.store(0);
    }

    void work() {
        for (;;) {
            uint64_t s = state_.load();
            if ((uint32_t)s >= count_.load()) return;
            const HostPiece *p = pieces_.load();
            if (!state_.compare_exchange_weak(s, s + 1)) continue;
            p[(uint32_t)s].copy();
            done_.fetch_add(1);
        }
    }

    void help(int i) {   // of the session's taken helpers, if i is one
        std::unique_lock<std::mutex> lk(m_);
        for (;;) {
            cv_.wait(lk, [this, i] { return stop_ || i < active_.load(); });
            if (stop_) return;
            lk.unlock();
            while (i < active_.load()) {
                work();
                pause();
            }
            lk.lock();
        }
    }

    static void pause() { __builtin_ia32_pause(); }

    const int cpus_ = (int)std::thread::hardware_concurrency();   // (a call of some microseconds)
    uint8_t *pin_ = nullptr;
    hipEvent_t events_[kSlots] = {};
    std::vector<std::thread> threads_;
    std::mutex m_;
    std::condition_variable cv_;
    bool stop_ = false;
    std::atomic<int> active_{0};   // helpers of the running session
    std::atomic<uint64_t> state_{0};
    std::atomic<const HostPiece *> pieces_{nullptr};
    std::atomic<uint32_t> count_{0};
    std::atomic<size_t> done_{0};
};

}  // namespace fmvs
