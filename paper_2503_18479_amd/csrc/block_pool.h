// Device blocks of destroyed plans' operators, kept for the next plan: a new
// allocation of some hundred MB has to be mapped and, once the memory that
// the GPU driver holds cleared is used up, cleared at about 36 GB/s (15 ms for the
// 539 MB of 256 loops at 65,536 points, where assembly takes 0.4 ms).
//   At most kBlocks blocks and kBytes in all, the oldest given back first; a
// block larger than kBytes is never kept.  Every allocation of the library goes
// through alloc(), which gives the device's idle blocks back and tries again
// when memory runs out, and drain_all() gives everything back.
//   Dev: alloc(void **, bytes) and free(void *) on the current device, wait()
// for all work of the device, no_memory (alloc's result when memory ran out).
// Host code without HIP, so that it can be tested without a GPU.
#pragma once
#include <cstddef>
#include <mutex>
#include <vector>

namespace cosim {

template <class Dev>
class BlockPool {
public:
    static constexpr size_t kBlocks = 8, kBytes = (size_t)1 << 30;

    BlockPool() { idle_.reserve(kBlocks + 1); }  // give() then never allocates

    // An idle block of at least `bytes` (at most a quarter more), or a new
    // allocation; *got: its size.  0 or Dev::alloc's error.
    int take(int device, size_t bytes, void **out, size_t *got) {
        bytes = (bytes + 65535) / 65536 * 65536;
        Block b{device, nullptr, 0};
        {
            std::lock_guard<std::mutex> lock(mu_);
            size_t best = idle_.size();
            for (size_t i = 0; i < idle_.size(); ++i)
                if (idle_[i].device == device && idle_[i].bytes >= bytes &&
                    idle_[i].bytes <= bytes + bytes / 4 &&
                    (best == idle_.size() || idle_[i].bytes < idle_[best].bytes))
                    best = i;
            if (best < idle_.size()) b = remove(best);
        }
        if (b.p) {
            // whatever still ran on the block when its plan was destroyed, on
            // any stream, has to end first
            if (Dev::wait() == 0) {
                *out = b.p;
                *got = b.bytes;
                return 0;
            }
            give(device, b.p, b.bytes);  // cannot wait here: a block of its own
        }
        *got = bytes;
        return alloc(device, out, bytes);
    }

    void give(int device, void *p, size_t bytes) {
        if (!p) return;
        Block back[kBlocks + 1];
        size_t n = 0;
        if (bytes > kBytes) {
            back[n++] = Block{device, p, bytes};
        } else {
            std::lock_guard<std::mutex> lock(mu_);
            idle_.push_back(Block{device, p, bytes});
            total_ += bytes;
            while (idle_.size() > kBlocks || total_ > kBytes) back[n++] = remove(0);
        }
        for (size_t i = 0; i < n; ++i) Dev::free(back[i].p);
    }

    // Dev::alloc; when memory ran out, once more without the device's idle blocks.
    int alloc(int device, void **out, size_t bytes) {
        int e = Dev::alloc(out, bytes);
        if (e == Dev::no_memory && drain(device) > 0) e = Dev::alloc(out, bytes);
        if (e != 0) *out = nullptr;
        return e;
    }

    // Gives the idle blocks of a device (-1: of all) back; how many there were.
    size_t drain(int device) {
        Block back[kBlocks + 1];
        size_t n = 0;
        {
            std::lock_guard<std::mutex> lock(mu_);
            for (size_t i = idle_.size(); i-- > 0;)
                if (device < 0 || idle_[i].device == device) back[n++] = remove(i);
        }
        for (size_t i = 0; i < n; ++i) Dev::free(back[i].p);
        return n;
    }

private:
    struct Block {
        int device = -1;
        void *p = nullptr;
        size_t bytes = 0;
        Block() = default;
        Block(int d, void *q, size_t b) : device(d), p(q), bytes(b) {}
    };
    std::mutex mu_;
    std::vector<Block> idle_;  // oldest first
    size_t total_ = 0;

    Block remove(size_t i) {
        const Block b = idle_[i];
        idle_.erase(idle_.begin() + (std::ptrdiff_t)i);
        total_ -= b.bytes;
        return b;
    }
};

}  // namespace cosim
