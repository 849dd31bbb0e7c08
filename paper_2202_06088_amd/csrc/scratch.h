// Blocks of scratch that are kept between calls, without the device headers:
// the runtime's calls come from a class of the includer, so that the host can
// check the bookkeeping (render.hip gives HIP's).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <mutex>

namespace neuvv {

// Kept blocks of one device. A stream-ordered allocation and its release cost
// the host 36 us together, more than the three launches of a small render
// (11 us). A block belongs to one call at a time, and afterwards to the stream
// of that call: the next call on the stream takes it behind the event recorded
// at its release, so that stream order protects it as it would a stream-ordered
// allocation (the event also covers a new stream that the runtime gives the
// handle of a destroyed one). Calls on other streams, and further calls of other
// threads on the same stream, have blocks of their own. Once kBlocks blocks or
// kBytes are kept, a call without a block takes over an idle one of another
// stream, or its room, if that one's event has passed (a program may have
// dropped the stream), and has the pool serve it alone otherwise. A stream that
// needs a larger block gives up its smaller idle ones.
//
// Rt has the types Status, Stream and Event, the status `ok`, and
//   Status alloc(void**, size_t, Stream)   from the pool, in stream order
//   static bool no_memory(Status)          whether alloc failed for want of memory
//   Status free(void*, Stream)             to the pool, in stream order
//   Status create(Event*)  void destroy(Event)
//   Status record(Event, Stream)  Status wait(Stream, Event)
//   bool passed(Event)  Status sync(Event)
//   Status finish(Stream)                  waits for the stream
//   Status trim()                          the pool's free memory goes back to the device
template <class Rt>
class KeptScratch {
  public:
    using Status = typename Rt::Status;
    using Stream = typename Rt::Stream;
    using Event = typename Rt::Event;
    static constexpr size_t kSmallest = (size_t)64 << 10;
    // Calls that need more run for some 300 us on the device and hide the host's 36 us; the event's packets between
    // their kernels cost them more (640 x 360 per-point adjoint, 118 MiB: 297 us from the pool, 311 us kept).
    static constexpr size_t kLargest = (size_t)64 << 20;
    static constexpr size_t kBytes = (size_t)320 << 20;   // the smallest adjoints of eight streams, 34 MiB each
    static constexpr int kBlocks = 32;

    // The size of the block that serves a request: powers of two up to 1 MiB, then steps of 2 MiB (the smallest
    // adjoint asks for a little over 32 MiB of records and lists).
    static size_t block_bytes(size_t bytes) {
        const size_t step = (size_t)2 << 20;
        if (bytes > step / 2) return (bytes + step - 1) / step * step;
        size_t want = kSmallest;
        while (want < bytes) want *= 2;
        return want;
    }

    // A block of at least `bytes` for a call on `stream`, or *p = nullptr: the pool serves the call. A failed
    // allocation of a new block is reported (the caller may release() and try again).
    Status acquire(Rt& rt, void** p, size_t bytes, Stream stream) {
        *p = nullptr;
        if (bytes > kLargest) return Rt::ok;
        std::lock_guard<std::mutex> lk(mu_);
        Block* best = nullptr;
        for (int i = 0; i < n_; ++i) {
            Block& b = b_[i];
            if (!b.used && b.stream == stream && b.bytes >= bytes && (!best || b.bytes < best->bytes)) best = &b;
        }
        if (best) {
            if (rt.wait(stream, best->done) != Rt::ok) return Rt::ok;
            return take(*best, p);
        }
        // the stream's idle blocks are all too small for it now: back to the pool, in its order
        for (int i = n_ - 1; i >= 0; --i)
            if (!b_[i].used && b_[i].stream == stream && rt.wait(stream, b_[i].done) == Rt::ok) drop(rt, i, stream);
        const size_t want = block_bytes(bytes);
        while (n_ == kBlocks || bytes_ + want > kBytes) {
            // the idle block of another stream that fits best, else the one longest unused
            int at = -1;
            for (int i = 0; i < n_; ++i)
                if (!b_[i].used && better(b_[i], at < 0 ? nullptr : &b_[at], bytes) && rt.passed(b_[i].done)) at = i;
            if (at < 0) return Rt::ok;
            if (b_[at].bytes >= bytes) {
                b_[at].stream = stream;
                return take(b_[at], p);
            }
            drop(rt, at, stream);
        }
        Block b{nullptr, want, stream, Event(), true, 0};
        if (rt.create(&b.done) != Rt::ok) return Rt::ok;
        const Status e = rt.alloc(&b.p, want, stream);
        if (e != Rt::ok) {
            rt.destroy(b.done);
            return e;
        }
        bytes_ += want;
        b_[n_++] = b;
        *p = b.p;
        return Rt::ok;
    }

    // Scratch of a call: a kept block where `keep`, else from the pool. Where the device has no memory left, what is
    // held here and not in use goes back first (waiting for it, so not where `graph`: the stream is captured).
    Status serve(Rt& rt, void** p, size_t bytes, Stream stream, bool keep, bool graph) {
        for (bool again = false;; again = true) {
            *p = nullptr;
            if (keep) (void)acquire(rt, p, bytes, stream);
            if (*p) return Rt::ok;
            const Status e = rt.alloc(p, bytes, stream);
            if (!rt.no_memory(e) || again || graph || give_back(rt, stream) != Rt::ok) return e;
        }
    }

    // Ends a call's use of p. False: not a kept block (the caller frees it).
    bool put_back(Rt& rt, void* p, Stream stream, Status* status) {
        std::lock_guard<std::mutex> lk(mu_);
        for (int i = 0; i < n_; ++i) {
            if (b_[i].p != p || !b_[i].used) continue;
            *status = rt.record(b_[i].done, stream);
            if (*status == Rt::ok) {
                b_[i].used = false;
                b_[i].last = ++tick_;
            } else {
                drop(rt, i, stream);   // cannot be handed on behind the event
            }
            return true;
        }
        return false;
    }

    // Returns the idle blocks to the pool, on `stream`, after the calls that used them (which it waits for with the
    // table unlocked: other threads' calls go on).
    Status release(Rt& rt, Stream stream) {
        Block out[kBlocks];
        int m = 0;
        {
            std::lock_guard<std::mutex> lk(mu_);
            for (int i = n_ - 1; i >= 0; --i) {
                if (b_[i].used) continue;
                out[m++] = b_[i];
                bytes_ -= b_[i].bytes;
                b_[i] = b_[--n_];
            }
        }
        Status e = Rt::ok;
        for (int i = 0; i < m; ++i) {
            const Status s = rt.sync(out[i].done);
            const Status f = rt.free(out[i].p, stream);
            rt.destroy(out[i].done);
            if (e == Rt::ok) e = s != Rt::ok ? s : f;
        }
        return e;
    }

    // Gives what is held and not in use back to the device: the idle blocks and the pool's free memory. (The pool
    // keeps what is freed to it, so the blocks alone would stay the process's until it ends.)
    Status give_back(Rt& rt, Stream stream) {
        Status e = release(rt, stream);
        const Status f = rt.finish(stream);
        if (e == Rt::ok) e = f;
        return e == Rt::ok ? rt.trim() : e;
    }

    int blocks() {
        std::lock_guard<std::mutex> lk(mu_);
        return n_;
    }
    size_t bytes() {
        std::lock_guard<std::mutex> lk(mu_);
        return bytes_;
    }

  private:
    struct Block {
        void* p;
        size_t bytes;
        Stream stream;
        Event done;
        bool used;
        uint64_t last;   // when it was put back
    };
    // whether a is to be taken before b (nullptr: none yet) for `bytes`
    static bool better(const Block& a, const Block* b, size_t bytes) {
        if (!b) return true;
        const bool fa = a.bytes >= bytes, fb = b->bytes >= bytes;
        if (fa != fb) return fa;
        return fa ? a.bytes < b->bytes : a.last < b->last;
    }
    Status take(Block& b, void** p) {
        b.used = true;
        *p = b.p;
        return Rt::ok;
    }
    // (the block's work is behind the caller's stream, or has passed)
    void drop(Rt& rt, int i, Stream stream) {
        rt.destroy(b_[i].done);
        bytes_ -= b_[i].bytes;
        (void)rt.free(b_[i].p, stream);
        b_[i] = b_[--n_];
    }

    std::mutex mu_;
    Block b_[kBlocks];
    int n_ = 0;
    size_t bytes_ = 0;
    uint64_t tick_ = 0;
};

}  // namespace neuvv
