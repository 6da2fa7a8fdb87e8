// Device blocks kept for later use instead of freed: hipMalloc and hipFree
// cost tens of microseconds to milliseconds each, and hipFree waits for the
// device.  A block goes to any later request on its own device that it fits
// (best fit, at most twice the request).  Its last use has ended when it is
// put back (the owner waits on the block's device), so the next owner may use
// it on any stream.
//
// A block carries the device it was allocated on: its owner may be destroyed,
// from a finaliser for instance, while another device is current.
//
// Kept blocks never stand in the way of an allocation: allocate_or_empty frees
// them and tries again before it reports that the memory is out.
//
// Api: the device calls (static; an Error that is zero on success), so that the
// cache can be tested without a device:
//   Error device(int* dev)               the current device
//   Error alloc(void** p, size_t bytes)  on the current device
//   void  free(void* p)                  whatever device is current
#pragma once

#include <cstddef>
#include <mutex>
#include <vector>

namespace sipf {

struct Block {
    void* p = nullptr;
    size_t bytes = 0;
    int dev = -1;
};

template <class Api> class BlockCache {
  public:
    using Error = typename Api::Error;
    // most: bytes kept per device at most
    explicit BlockCache(size_t most) : limit_(most) {}

    // A block of at least n bytes (n > 0) on the current device; its whole size in out->bytes.
    Error get(size_t n, Block* out) {
        *out = Block{};
        int dev = 0;
        Error e = Api::device(&dev);
        if (e != Error(0)) return e;
        {
            std::lock_guard<std::mutex> lock(mu_);
            int best = -1;
            for (int i = 0; i < (int)kept_.size(); ++i) {
                const Block& b = kept_[i];
                if (b.dev == dev && b.bytes >= n && b.bytes - n <= n && (best < 0 || b.bytes < kept_[best].bytes))
                    best = i;
            }
            if (best >= 0) {
                *out = kept_[best];
                kept_.erase(kept_.begin() + best);
                return Error(0);
            }
        }
        void* p = nullptr;
        e = Api::alloc(&p, n);
        if (e == Error(0)) *out = Block{p, n, dev};
        return e;
    }

    // Take b back; nothing may be pending on it.
    void put(const Block& b) {
        if (b.p == nullptr) return;
        {
            std::lock_guard<std::mutex> lock(mu_);
            size_t held = 0;
            for (const Block& k : kept_) held += k.dev == b.dev ? k.bytes : 0;
            if (b.bytes <= limit_ && held <= limit_ - b.bytes) {
                kept_.push_back(b);
                return;
            }
        }
        Api::free(b.p);
    }

    // Free every kept block.
    void release() {
        std::vector<Block> out;
        {
            std::lock_guard<std::mutex> lock(mu_);
            out.swap(kept_);
        }
        for (const Block& b : out) Api::free(b.p);
    }

  private:
    const size_t limit_;
    std::mutex mu_;
    std::vector<Block> kept_;
};

// allocate() -> Error; when that says `full`, once more with every cache emptied.
template <class Error, class Alloc, class... Caches>
Error allocate_or_empty(Error full, Alloc allocate, Caches&... caches) {
    const Error e = allocate();
    if (e != full) return e;
    (caches.release(), ...);
    return allocate();
}

}  // namespace sipf
