// Host check of the cache of device blocks (block_cache.h) on a device that
// keeps a book of its allocations.  Prints the failed checks; exit status 0
// when there are none.
#include <cstdio>
#include <map>

#include "block_cache.h"

namespace {

struct FakeDevice {
    using Error = int;
    static int current;
    static std::map<void*, std::pair<int, size_t>> live;  // pointer -> device, bytes
    static int freed;
    static size_t room;  // bytes per device
    static char mem[1 << 16];
    static size_t used;
    static Error device(int* dev) {
        *dev = current;
        return 0;
    }
    static Error alloc(void** p, size_t n) {
        size_t held = 0;
        for (const auto& l : live) held += l.second.first == current ? l.second.second : 0;
        if (held + n > room) return 2;
        *p = mem + used;  // addresses only: nothing is stored
        used += 16;
        live[*p] = {current, n};
        return 0;
    }
    static void free(void* p) {
        if (live.erase(p) == 1) ++freed;
        else freed += 1000;  // freed twice, or never allocated
    }
};
int FakeDevice::current = 0;
std::map<void*, std::pair<int, size_t>> FakeDevice::live;
int FakeDevice::freed = 0;
size_t FakeDevice::room = 1 << 20;
char FakeDevice::mem[1 << 16];
size_t FakeDevice::used = 0;

int failures = 0;
void check(bool ok, const char* what) {
    if (ok) return;
    ++failures;
    std::printf("failed: %s\n", what);
}

}  // namespace

int main() {
    using sipf::Block;
    sipf::BlockCache<FakeDevice> cache(1000);
    Block a, b, c;

    // a block taken on device 0 and given back while device 1 is current stays device 0's
    FakeDevice::current = 0;
    check(cache.get(100, &a) == 0 && a.dev == 0 && a.bytes == 100, "a new block is the current device's");
    FakeDevice::current = 1;
    cache.put(a);
    check(cache.get(100, &b) == 0, "a block on device 1");
    check(b.p != a.p && FakeDevice::live[b.p].first == 1 && b.dev == 1, "device 1 gets memory of its own");
    FakeDevice::current = 0;
    check(cache.get(100, &c) == 0 && c.p == a.p && c.dev == 0, "device 0 gets its block again");
    cache.put(b);
    cache.put(c);
    cache.release();
    check(FakeDevice::live.empty() && FakeDevice::freed == 2, "release frees each block once");

    // smaller requests: the smallest block that fits, of at most twice the request
    check(cache.get(100, &a) == 0 && cache.get(150, &b) == 0, "two blocks");
    cache.put(b);
    cache.put(a);
    check(cache.get(49, &c) == 0 && c.p != a.p && c.p != b.p && c.bytes == 49, "a block of more than twice the request stays");
    Block d, e;
    check(cache.get(75, &d) == 0 && d.p == a.p && d.bytes == 100, "the smallest block that fits, its size with it");
    check(cache.get(101, &e) == 0 && e.p == b.p && e.bytes == 150, "the next one");
    cache.put(c);
    cache.put(d);
    cache.put(e);
    cache.release();
    check(FakeDevice::live.empty(), "no block is lost");

    // at most 1000 bytes per device stay
    Block k[4];
    for (int i = 0; i < 3; ++i) check(cache.get(400, &k[i]) == 0, "blocks of 400");
    FakeDevice::current = 1;
    check(cache.get(900, &k[3]) == 0, "a block on the other device");
    for (const Block& q : k) cache.put(q);
    check(FakeDevice::live.size() == 3 && FakeDevice::live.count(k[2].p) == 0, "the third block of 400 is freed, the other device's kept");
    check(cache.get(1100, &a) == 0, "a block above the limit");
    cache.put(a);
    check(FakeDevice::live.size() == 3, "a block above the limit is freed");
    cache.release();
    check(FakeDevice::live.empty() && FakeDevice::freed < 1000, "every block is freed once");

    // a full device: the kept blocks of every cache go back, the blocks in use stay
    FakeDevice::current = 0;
    FakeDevice::room = 1000;
    sipf::BlockCache<FakeDevice> other(1000);
    auto allocate = [&](size_t n, void** p) {
        return sipf::allocate_or_empty(2, [&] { return FakeDevice::alloc(p, n); }, cache, other);
    };
    check(cache.get(300, &a) == 0 && other.get(300, &b) == 0 && cache.get(200, &c) == 0, "three blocks");
    cache.put(a);
    other.put(b);
    void *p = nullptr, *q = nullptr;
    check(allocate(150, &p) == 0 && FakeDevice::live.size() == 4, "room for 150 beside the kept blocks");
    check(allocate(600, &q) == 0 && FakeDevice::live.size() == 3, "600 once both caches are empty");
    void* none = nullptr;
    check(allocate(100, &none) == 2 && FakeDevice::live.count(c.p) == 1, "out of memory with nothing kept");
    return failures ? 1 : 0;
}
