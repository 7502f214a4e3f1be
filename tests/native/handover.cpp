// The hand-over queue of the walk kernel (csrc/handover.hpp) on host threads: one thread for
// every wave that the chip holds at once, waves started in a given order as others end.
// Arguments: bulk waves, single-walk waves, waves held at once, walks, slots, wait limit (ns,
// 0: none), start order (0: as launched, 1: shuffled), seed, 1 to let bulk waves wait without
// asking whether all have started.  Prints the walks lost, the walks run twice and "stalled"
// if every running wave has waited in vain for two seconds; on stderr, how far the tail is past
// the last slot.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <thread>
#include <vector>

#include "handover.hpp"

using namespace srw;

namespace {

using Clock = std::chrono::steady_clock;

std::atomic<bool> stalled{false};
std::atomic<uint64_t> progress{0};
struct Stalled {};

int64_t ns() { return std::chrono::duration_cast<std::chrono::nanoseconds>(Clock::now().time_since_epoch()).count(); }

struct Mem {
    std::minstd_rand* rng;
    void shake() const
    {
        if ((*rng)() % 4 == 0) std::this_thread::yield();
    }
    uint64_t load(const unsigned long long* p) const
    {
        shake();
        return __atomic_load_n(p, __ATOMIC_RELAXED);
    }
    void store(unsigned long long* p, unsigned long long v) const
    {
        shake();
        __atomic_store_n(p, v, __ATOMIC_RELAXED);
    }
    uint64_t add(unsigned long long* p, unsigned long long v) const
    {
        shake();
        return __atomic_fetch_add(p, v, __ATOMIC_RELAXED);
    }
    uint64_t cas(unsigned long long* p, unsigned long long from, unsigned long long to) const
    {
        shake();
        __atomic_compare_exchange_n(p, &from, to, false, __ATOMIC_RELAXED, __ATOMIC_RELAXED);
        return from;
    }
    uint64_t cas_uniform(unsigned long long* p, unsigned long long from, unsigned long long to) const
    {
        return cas(p, from, to);
    }
    void pause() const
    {
        std::this_thread::yield();
        if (stalled.load()) throw Stalled{};
    }
    int64_t now() const { return ns(); }
    uint32_t lane() const { return 0; }
    uint32_t lanes() const { return 1; }
};

struct Run {
    HandQueue q{};
    int walks = 0;
    bool unasked = false;
    std::atomic<int> next{0};
    std::vector<std::atomic<int>> ran;
    explicit Run(int n) : walks(n), ran(n) {}
};

void done(Run& r, int w)
{
    r.ran[w].fetch_add(1);
    progress.fetch_add(1);
}

// up to four walks at a time; a walk ends, or is handed over, at random
void bulk(Run& r, const Mem& m)
{
    std::vector<int> mine;
    bool full = r.q.cap == 0;
    for (bool more = true;;) {
        while (more && mine.size() < 4) {
            const int w = r.next.fetch_add(1);
            if (w >= r.walks) more = false;
            else mine.push_back(w);
        }
        if (mine.empty()) break;
        const size_t k = (*m.rng)() % mine.size();
        if (!full && (*m.rng)() % 2 == 0) {
            const uint32_t at = hand_reserve(m, r.q, 1, full);
            if (!hand_put(m, r.q, at, {(uint64_t)mine[k], (uint64_t)mine[k] + 7, (uint64_t)mine[k] + 9})) continue;
        } else {
            done(r, mine[k]);
        }
        mine.erase(mine.begin() + (std::ptrdiff_t)k);
    }
}

void wave(Run& r, uint32_t i, std::minstd_rand& rng)
{
    const Mem m{&rng};
    bool here;
    if (i < r.q.n_bulk) {
        m.add(r.q.hand + HAND_ARRIVED, 1);
        bulk(r, m);
        here = hand_finish(m, r.q) || r.unasked;
    } else {
        here = hand_all_started(m, r.q);
    }
    HandedWalk w;
    while (here && hand_take(m, r.q, w)) {
        if (w.w1 != w.w0 + 7 || w.w2 != w.w0 + 9) std::abort();
        done(r, (int)w.w0);
    }
    progress.fetch_add(1);
}

}  // namespace

int main(int argc, char** argv)
{
    if (argc != 10) return 2;
    auto arg = [&](int i) { return std::strtoll(argv[i], nullptr, 10); };
    Run r((int)arg(4));
    r.q.n_bulk = r.q.n_groups = (uint32_t)arg(1);
    r.q.cap = (uint32_t)arg(5);
    r.q.wait_limit = arg(6) ? arg(6) : INT64_MAX;
    r.unasked = arg(9) != 0;
    std::vector<unsigned long long> slots((size_t)r.q.cap * SLOT_WORDS, SLOT_EMPTY), hand(HAND_WORDS, 0);
    r.q.slots = slots.data();
    r.q.hand = hand.data();
    std::vector<uint32_t> order((size_t)(arg(1) + arg(2)));
    for (uint32_t i = 0; i < order.size(); ++i) order[i] = i;
    std::minstd_rand rng((unsigned)arg(8) + 1);
    if (arg(7)) std::shuffle(order.begin(), order.end(), rng);
    std::atomic<size_t> started{0};
    std::atomic<int> running{(int)arg(3)};
    std::vector<std::thread> held;
    for (int t = 0; t < arg(3); ++t)
        held.emplace_back([&, seed = (unsigned)rng()] {
            std::minstd_rand mine(seed % 1000003 + 1);
            try {
                for (size_t k; (k = started.fetch_add(1)) < order.size();) wave(r, order[k], mine);
            } catch (const Stalled&) {
            }
            running.fetch_sub(1);
        });
    uint64_t seen = 0;
    int64_t since = ns();
    while (running.load() > 0) {
        std::this_thread::sleep_for(std::chrono::milliseconds(1));
        if (progress.load() != seen) seen = progress.load(), since = ns();
        else if (ns() - since > 2000000000) stalled.store(true);
    }
    for (auto& t : held) t.join();
    int lost = 0, twice = 0;
    for (auto& n : r.ran) lost += n.load() == 0, twice += n.load() > 1;
    const uint32_t tail = (uint32_t)hand[HAND_QUEUE];
    std::printf("%d %d%s\n", lost, twice, stalled.load() ? " stalled" : "");
    std::fprintf(stderr, "%u\n", tail > r.q.cap ? tail - r.q.cap : 0u);
    return 0;
}
