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
    static char mem[1 << 16];
    static size_t used;
    static Error device(int* dev) {
        *dev = current;
        return 0;
    }
    static Error alloc(void** p, size_t n) {
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
    return failures ? 1 : 0;
}
