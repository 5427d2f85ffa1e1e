// Blocks of destroyed weights, kept for weights to come (host code, one object per device).  A program that replaces weights while it
// runs pays more for hipMalloc and hipFree of their blocks, and for the wait for the whole device that goes with them, than for encoding and packing them.
#pragma once
#include <hip/hip_runtime_api.h>

#include <cstddef>
#include <cstdint>
#include <mutex>

namespace abft {

// A freed block may still be read by work that was enqueued before.  It is used again only after a wait for the whole device, once for all
// blocks freed until then.  When that wait comes is decided by counts alone: a block that fits and has been waited for is taken at once; else, if
// kMostWaiting blocks that fit have not been, if there is no room to keep another one, or if the caller says that the device seems to be idle, the
// device is waited for; else another block is allocated.  So a weight replaced again and again settles at kMostWaiting blocks and a wait for as many
// replacements, at whatever rate, and one replaced while the device idles at a single block.  A weight that is destroyed while the device seems to be idle
// is waited for there and then if no other block would serve the next one like it: that one often comes behind the kernels that make it, on a busy stream.
// Measured, us a replacement with its first batch (64 rows of 4096x4096, 32 of 700x900), hipMalloc and hipFree / this: back to back 69 and 36 / 26 and 24, 100 us of
// other host work between them 81 and 39 / 25 and 24, 1 ms 87 and 40 / 24 and 25 (a wait by the time since the last replacement, with a limit of 50 us, took 29 and
// 23, 43 and 38, 43 and 38).  A weight of 16 MiB made anew in a program that has given up another: 95 us with its 16 MiB of random numbers, 240 without
// the wait as that one was destroyed.  The wait takes 10 us on an idle device, 60 to 90 on a busy one and, when it is the first in some milliseconds, 150 to
// 250 (the runtime catches up with all that has ended), for one block or for eight; a block that the device has not had yet takes 60 to 250.
//
// Memory: allocate(void**, size_t) as hipMalloc; wait() and release(void*): true once everything that was enqueued on the device before the call has
// ended, and the block given back.
template <class Memory>
class KeptBlocks {
public:
    static constexpr int kMost = 16, kMostWaiting = 8, kStale = 2 * kMost;
    static constexpr size_t kMostBytes = 256u << 20;

    explicit KeptBlocks(Memory memory = Memory()) : memory_(memory) {}

    // a block of at least `need` bytes, up to a sixteenth more; *size: its real size, *mark: with what it was put back, 0: a new
    // one.  idle(): whether the device seems to be (a wrong answer costs time, no more)
    template <class Idle>
    hipError_t get(size_t need, void** out, size_t* size, uint64_t* mark, Idle idle) {
        *out = nullptr;
        *mark = 0;
        if (take(need, out, size, mark)) return hipSuccess;
        if (const int waiting = count_waiting(need)) {
            if ((waiting >= kMostWaiting || !has_room(need) || idle()) && wait() && take(need, out, size, mark)) return hipSuccess;
        }
        hipError_t e = memory_.allocate(out, *size = need);
        if (e == hipErrorOutOfMemory && give_back()) e = memory_.allocate(out, need);
        if (e == hipSuccess) {
            std::lock_guard<std::mutex> lock(mutex_);
            ++live_;
        }
        return e;
    }
    // the block of a weight that is destroyed; here: with its device current; idle() as above.  Where there is no room for it, blocks that have lain unused while
    // kStale others came make room; not younger ones, of which a program that replaces several weights in turn will need the oldest next
    template <class Idle>
    void put(void* block, size_t size, uint64_t mark, bool here, Idle idle) {
        Block out[kMost + 1];
        int n_out = 0;
        bool last, ready = true;   // (ready: a block of that size need not be waited for)
        unsigned long long until;
        {
            std::lock_guard<std::mutex> lock(mutex_);
            last = --live_ == 0;
            ++released_;
            if (!last && size <= kMostBytes)
                for (int i = oldest(); !room(size) && stale(i); i = oldest()) {
                    out[n_out++] = blocks_[i];
                    drop(i);
                }
            if (!last && room(size)) {
                ready = false;
                for (int i = 0; i < n_; ++i) ready |= blocks_[i].idle && fits(blocks_[i], size);
                add({block, size, mark, released_, false});
            } else {
                out[n_out++] = {block, size, mark, released_, false};
            }
            until = released_;
        }
        if (last) (void)give_back();
        if (n_out > 0 && release(out, n_out) && here) waited(until);   // (to give a block back is a wait for the device, where it is not refused)
        else if (!ready && here && idle()) (void)wait();
    }

    // all that are kept, back to the device; false: refused for some
    bool trim() {
        (void)give_back();
        std::lock_guard<std::mutex> lock(mutex_);
        return n_ == 0;
    }

private:
    struct Block {
        void* at;
        size_t size;
        uint64_t mark;
        unsigned long long number;   // of its release
        bool idle;                   // a wait for the device lies behind that
    };
    Memory memory_;
    std::mutex mutex_;
    Block blocks_[kMost];
    int n_ = 0;
    size_t bytes_ = 0;
    unsigned long long released_ = 0;
    long long live_ = 0;   // blocks in use

    bool room(size_t size) const { return n_ < kMost && size <= kMostBytes - bytes_; }
    int oldest() const {
        int o = 0;
        for (int i = 1; i < n_; ++i)
            if (blocks_[i].number < blocks_[o].number) o = i;
        return o;
    }
    bool stale(int i) const { return i < n_ && released_ - blocks_[i].number >= kStale; }
    void add(const Block& b) {
        blocks_[n_++] = b;
        bytes_ += b.size;
    }
    void drop(int i) {
        bytes_ -= blocks_[i].size;
        blocks_[i] = blocks_[--n_];
    }
    static bool fits(const Block& b, size_t need) { return b.size >= need && b.size - need <= need / 16; }
    bool take(size_t need, void** out, size_t* size, uint64_t* mark) {
        std::lock_guard<std::mutex> lock(mutex_);
        for (int i = 0; i < n_; ++i)
            if (blocks_[i].idle && fits(blocks_[i], need)) {
                *out = blocks_[i].at;
                *size = blocks_[i].size;
                *mark = blocks_[i].mark;
                drop(i);
                ++live_;
                return true;
            }
        return false;
    }
    int count_waiting(size_t need) {
        std::lock_guard<std::mutex> lock(mutex_);
        int n = 0;
        for (int i = 0; i < n_; ++i) n += !blocks_[i].idle && fits(blocks_[i], need);
        return n;
    }
    bool has_room(size_t need) {   // (now, or once a stale block is gone)
        std::lock_guard<std::mutex> lock(mutex_);
        return room(need) || (need <= kMostBytes && stale(oldest()));
    }
    bool wait() {
        unsigned long long until;   // (blocks that other threads release during the wait are not covered)
        {
            std::lock_guard<std::mutex> lock(mutex_);
            until = released_;
        }
        if (!memory_.wait()) return false;
        waited(until);
        return true;
    }
    void waited(unsigned long long until) {
        std::lock_guard<std::mutex> lock(mutex_);
        for (int i = 0; i < n_; ++i) blocks_[i].idle |= blocks_[i].number <= until;
    }
    bool give_back() {
        Block blocks[kMost];
        int n;
        {
            std::lock_guard<std::mutex> lock(mutex_);
            n = n_;
            for (int i = 0; i < n; ++i) blocks[i] = blocks_[i];
            n_ = 0;
            bytes_ = 0;
        }
        return n > 0 && release(blocks, n);
    }
    // (refused, as hipFree is while another thread captures a graph in a mode that forbids it: kept after all, as far as there is room)
    bool release(const Block* blocks, int n) {
        bool all = true;
        for (int i = 0; i < n; ++i)
            if (!memory_.release(blocks[i].at)) {
                std::lock_guard<std::mutex> lock(mutex_);
                if (room(blocks[i].size)) add(blocks[i]);
                all = false;
            }
        return all;
    }
};

}  // namespace abft
