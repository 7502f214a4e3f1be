// Device memory kept between calls.
//
// A build makes about 25 device allocations and a solve one.  The runtime's stream-ordered
// allocator takes 35 us for each and 200 us to free it (2 ms and more for large blocks, up
// to 160 ms when the sizes of successive builds differ and its pool has to map new memory);
// a Laplacian 50^3 built and solved spent 5.2 of 17 ms in them, the 256-grid batch 100 ms a
// build once three matrices took turns.  Blocks released here are kept for later calls.
//
// A released block has no work pending on it (the caller has synchronised the stream it
// was used on), so any stream and thread may take it next.  What is kept is bounded by an
// eighth of the device's memory; blocks that go unused while 2,048 others are released
// (some eighty builds), everything past the bound, and everything when an allocation
// fails, goes back to the device.
#include <mutex>
#include <unordered_map>
#include <vector>

#include "pool.hpp"

namespace srw {

namespace {

constexpr int MAX_DEVICES = 64;
constexpr uint64_t IDLE_RELEASES = 2048;

struct Block {
    void* p;
    size_t size;
    uint64_t stamp;  // the device's release count when the block came in
};

struct DevicePool {
    std::vector<Block> kept;  // oldest first
    size_t bytes = 0, bound = 0;
    uint64_t releases = 0;
};

struct Owner {
    int dev;
    size_t size;
};

struct Pool {
    std::mutex mu;
    DevicePool dev[MAX_DEVICES];
    std::unordered_map<void*, Owner> live;
};

// never destroyed: the runtime may be gone by the time static objects are
Pool& pool()
{
    static Pool* p = new Pool();
    return *p;
}

// Sizes in steps of an eighth, so that blocks fit the next build's slightly other sizes.
size_t size_class(size_t bytes)
{
    size_t step = 4096;
    while (step * 16 <= bytes) step *= 2;
    return (bytes + step - 1) / step * step;
}

// Allocates and frees although some stream of the process, another thread's or this one's,
// may be under capture: nothing of it enters the graph.
struct OutsideCaptures {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    OutsideCaptures() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~OutsideCaptures() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

hipError_t raw_alloc(void** p, size_t bytes)
{
    const OutsideCaptures o;
    return hipMalloc(p, bytes);
}

void raw_free(void* p)
{
    const OutsideCaptures o;
    (void)hipFree(p);
}

}  // namespace

hipError_t dev_alloc(void** out, size_t bytes)
{
    *out = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    const size_t need = size_class(bytes ? bytes : 1);
    Pool& P = pool();
    DevicePool& D = P.dev[dev];
    try {
        {
            std::lock_guard<std::mutex> lk(P.mu);
            // the smallest block that holds it, at most a quarter larger
            size_t best = D.kept.size();
            for (size_t i = 0; i < D.kept.size(); ++i)
                if (D.kept[i].size >= need && D.kept[i].size <= need + need / 4 &&
                    (best == D.kept.size() || D.kept[i].size < D.kept[best].size))
                    best = i;
            if (best < D.kept.size()) {
                const Block b = D.kept[best];
                P.live.emplace(b.p, Owner{dev, b.size});
                D.kept.erase(D.kept.begin() + (std::ptrdiff_t)best);
                D.bytes -= b.size;
                *out = b.p;
                return hipSuccess;
            }
        }
        void* p = nullptr;
        e = raw_alloc(&p, need);
        if (e == hipErrorOutOfMemory) {
            (void)hipGetLastError();
            dev_trim(dev);
            e = raw_alloc(&p, need);
        }
        if (e != hipSuccess) return e;
        try {
            std::lock_guard<std::mutex> lk(P.mu);
            P.live.emplace(p, Owner{dev, need});
        } catch (...) {
            raw_free(p);
            throw;
        }
        *out = p;
        return hipSuccess;
    } catch (...) {
        return hipErrorOutOfMemory;
    }
}

void dev_release(void* p)
{
    if (!p) return;
    Pool& P = pool();
    std::vector<void*> back;
    bool lost = false;
    try {
        std::lock_guard<std::mutex> lk(P.mu);
        const auto it = P.live.find(p);
        if (it == P.live.end()) return;
        const Owner o = it->second;
        DevicePool& D = P.dev[o.dev];
        if (D.bound == 0) {
            int cur = 0;
            size_t free_b = 0, total = 0;
            D.bound = (size_t)16 << 30;
            if (hipGetDevice(&cur) == hipSuccess && cur == o.dev && hipMemGetInfo(&free_b, &total) == hipSuccess)
                D.bound = total / 8;
        }
        P.live.erase(it);
        lost = true;  // until a list holds it
        ++D.releases;
        back.reserve(D.kept.size() + 1);
        D.kept.push_back(Block{p, o.size, D.releases});
        lost = false;
        D.bytes += o.size;
        size_t n = 0;
        while (n < D.kept.size() &&
               (D.bytes > D.bound || D.kept[n].stamp + IDLE_RELEASES < D.releases)) {
            D.bytes -= D.kept[n].size;
            back.push_back(D.kept[n].p);
            ++n;
        }
        D.kept.erase(D.kept.begin(), D.kept.begin() + (std::ptrdiff_t)n);
    } catch (...) {
    }
    if (lost) raw_free(p);
    for (void* q : back) raw_free(q);
}

void dev_trim(int dev)
{
    Pool& P = pool();
    std::vector<Block> back;
    {
        std::lock_guard<std::mutex> lk(P.mu);
        DevicePool& D = P.dev[dev];
        back.swap(D.kept);
        D.bytes = 0;
    }
    for (const Block& b : back) raw_free(b.p);
}

hipError_t stream_alloc(void** out, size_t bytes, hipStream_t s)
{
    hipError_t e = hipMallocAsync(out, bytes, s);
    int dev = 0;
    if (e == hipErrorOutOfMemory && hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < MAX_DEVICES) {
        (void)hipGetLastError();
        dev_trim(dev);
        e = hipMallocAsync(out, bytes, s);
    }
    return e;
}

}  // namespace srw
