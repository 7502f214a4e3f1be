// The kept device blocks (csrc/pool.cpp) over a device of 64 GiB that the runtime calls below
// stand for.  Prints one line per failed check; exits with their number.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <map>
#include <vector>

#include "pool.hpp"

using namespace srw;

namespace {

constexpr size_t GIB = (size_t)1 << 30, TOTAL = 64 * GIB;
std::map<void*, size_t> blocks;
size_t used = 0;
uintptr_t next_address = 1 << 20;
int allocs = 0, async_calls = 0, current = 0, failed = 0;
hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
bool mode_wrong = false;

hipError_t take(void** p, size_t bytes)
{
    if (used + bytes > TOTAL) return hipErrorOutOfMemory;
    *p = (void*)next_address;
    next_address += bytes + 4096;
    blocks[*p] = bytes;
    used += bytes;
    return hipSuccess;
}

#define CHECK(x)                                    \
    do {                                            \
        if (!(x)) {                                 \
            std::printf("line %d: %s\n", __LINE__, #x); \
            ++failed;                               \
        }                                           \
    } while (0)

void* get(size_t bytes)
{
    void* p = nullptr;
    CHECK(dev_alloc(&p, bytes) == hipSuccess);
    return p;
}

}  // namespace

extern "C" {
hipError_t hipGetDevice(int* d) { return *d = current, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMemGetInfo(size_t* f, size_t* t) { return *f = TOTAL - used, *t = TOTAL, hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m)
{
    const hipStreamCaptureMode was = mode;
    mode = *m;
    *m = was;
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t bytes)
{
    mode_wrong = mode_wrong || mode != hipStreamCaptureModeRelaxed;
    ++allocs;
    return take(p, bytes);
}
hipError_t hipMallocAsync(void** p, size_t bytes, hipStream_t)
{
    ++async_calls;
    return take(p, bytes);
}
hipError_t hipFree(void* p)
{
    mode_wrong = mode_wrong || mode != hipStreamCaptureModeRelaxed;
    const auto it = blocks.find(p);
    if (it == blocks.end()) {
        std::printf("free of an unknown block\n");
        ++failed;
        return hipErrorInvalidValue;
    }
    used -= it->second;
    blocks.erase(it);
    return hipSuccess;
}
}

int main()
{
    // a block comes back for the same and for slightly other sizes, not for much smaller ones
    void* a = get(10 << 20);
    dev_release(a);
    CHECK(get(10 << 20) == a);
    dev_release(a);
    void* b = get((10 << 20) - (1 << 20));
    CHECK(b == a);
    void* c = get(10 << 20);  // a is taken
    CHECK(c != a);
    dev_release(b);
    dev_release(c);
    void* s = get(1 << 20);
    CHECK(s != a && s != c);
    dev_release(s);
    dev_release(s);  // not live any more: nothing
    dev_release(nullptr);
    CHECK(used < 23 << 20);
    dev_trim(0);
    CHECK(used == 0 && blocks.empty());

    // what is kept is at most an eighth of the device's memory, the newest of it
    std::vector<void*> v;
    for (int i = 0; i < 20; ++i) v.push_back(get(GIB));
    for (void* p : v) dev_release(p);
    CHECK(used <= TOTAL / 8 && used >= TOTAL / 8 - 2 * GIB);
    CHECK(blocks.count(v.back()) && !blocks.count(v.front()));
    dev_release(get(20 * GIB));  // larger than all that may be kept
    CHECK(used <= TOTAL / 8);
    dev_trim(0);

    // a block that nobody takes while 2,048 others are released goes back
    void* old = get(3 << 20);
    dev_release(old);
    for (int i = 0; i < 2040; ++i) dev_release(get(64 << 10));
    CHECK(blocks.count(old));
    for (int i = 0; i < 20; ++i) dev_release(get(64 << 10));
    CHECK(!blocks.count(old) && blocks.size() == 1);
    dev_trim(0);

    // repeated builds of slightly different sizes do not grow
    size_t after = 0;
    for (int i = 0; i < 200; ++i) {
        v.clear();
        for (int k = 0; k < 25; ++k) v.push_back(get((size_t)((4 << 20) + (k << 18) + (i * 7919) % 50000)));
        for (void* p : v) dev_release(p);
        if (i == 5) after = used;
    }
    CHECK(used <= after + after / 8);
    dev_trim(0);
    CHECK(used == 0);

    // where memory is short the kept blocks make room, for either kind of allocation
    std::vector<void*> all;
    for (int i = 0; i < 7; ++i) all.push_back(get(GIB));
    for (void* p : all) dev_release(p);
    CHECK(used == 7 * GIB);
    void* big = get(60 * GIB);
    CHECK(big && used == 60 * GIB);
    dev_release(big);
    CHECK(used == 0);  // past the bound
    for (int i = 0; i < 7; ++i) all[i] = get(GIB);
    for (void* p : all) dev_release(p);
    void* stream_block = nullptr;
    async_calls = 0;
    CHECK(stream_alloc(&stream_block, 60 * GIB, nullptr) == hipSuccess && async_calls == 2);
    CHECK(used == 60 * GIB);
    void* none = &none;
    CHECK(dev_alloc(&none, 10 * GIB) == hipErrorOutOfMemory && none == nullptr);
    CHECK(stream_alloc(&none, 10 * GIB, nullptr) == hipErrorOutOfMemory);

    // blocks of another device are not handed out
    void* d0 = get(1 << 20);
    dev_release(d0);
    current = 1;
    void* d1 = get(1 << 20);
    CHECK(d1 != d0);
    dev_release(d1);
    CHECK(get(1 << 20) == d1);
    current = 64;
    CHECK(dev_alloc(&none, 1) == hipErrorInvalidDevice);
    CHECK(!mode_wrong && mode == hipStreamCaptureModeGlobal);
    return failed;
}
