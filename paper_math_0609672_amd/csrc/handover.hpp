// The queue of walks handed over from bulk waves to single-walk waves (walk.hpp).
//
// Slots are handed out in order (tail) and taken in order (head, the tickets).  A ticket
// past the tail is a wave waiting for work: it polls its own slot only (thousands of waves
// polling one address hold up every atomic on that channel by tens of microseconds).  The
// last bulk wave to finish marks the slots of the tickets past the tail as closed.
//
// The launch is an ordinary one: workgroups may start in any order, and other kernels may
// keep part of them from starting for as long as those that run stay.  So a wave waits (for
// a slot, or for the long segment to be taken) only once every bulk workgroup has started:
// bulk waves with work wait for no one, so all of them finish, and the last of them closes
// every slot that a wave may still wait for.  A wave that finds them not all started ends,
// or starts its own work, at once.  Whatever is left in the slots is taken by the last bulk
// wave, which knows that all have started.  Every wait also ends by itself: past its limit a
// wave closes its own slot and leaves, and a walk that finds its slot closed stays where it
// is, so no walk is lost and no build fails for it.
//
// The memory operations come from M: load, store, add (the wave's, uniform) and cas at
// device scope, relaxed; pause and now (ticks) for waits; lane and lanes.
#pragma once

#include <cstddef>
#include <cstdint>

namespace srw {

constexpr int SLOT_WORDS = 4;  // {chunk | walk << 32, step << 32 | line word, visits, -}
constexpr unsigned long long SLOT_EMPTY = ~0ull, SLOT_CLOSED = ~1ull;
enum : int {
    HAND_QUEUE = 0,     // tail | head << 32
    HAND_ARRIVED = 32,  // bulk workgroups that have started
    HAND_DONE = 64,     // bulk waves that have finished
    HAND_WORDS = 96
};

struct HandQueue {
    unsigned long long* slots;  // cap of SLOT_WORDS words each, SLOT_EMPTY at first
    unsigned long long* hand;   // HAND_WORDS control words, zero at first
    uint32_t cap;               // 0: no walk is handed over
    uint32_t n_bulk;            // waves that take walks from the chunk queues
    uint32_t n_groups;          // their workgroups
    int64_t wait_limit;         // ticks a wave waits at most
};

struct HandedWalk {
    uint64_t w0, w1, w2;
};

template <class M>
__device__ __forceinline__ bool hand_all_started(const M& m, const HandQueue& q)
{
    return m.load(q.hand + HAND_ARRIVED) >= q.n_groups;
}

// The first of n slots for the wave's walks; full once the slots are used up.  A wave that
// has seen that asks for no more, so the tail never passes cap by more than each wave's last
// n: carried into the head, it would hand out slots again.
template <class M>
__device__ __forceinline__ uint32_t hand_reserve(const M& m, const HandQueue& q, uint32_t n, bool& full)
{
    const uint32_t at = (uint32_t)m.add(q.hand + HAND_QUEUE, n);
    full = at >= q.cap;
    return at;
}

// A lane's walk into slot `at`; false (the lane keeps it) past the last slot, or if the
// slot's ticket holder has left.
template <class M>
__device__ __forceinline__ bool hand_put(const M& m, const HandQueue& q, uint32_t at, const HandedWalk& w)
{
    if (at >= q.cap) return false;
    unsigned long long* slot = q.slots + (size_t)at * SLOT_WORDS;
    m.store(slot + 1, w.w1);
    m.store(slot + 2, w.w2);
    return m.cas(slot, SLOT_EMPTY, w.w0) == SLOT_EMPTY;
}

// The next handed-over walk; false once none can come, or none has for wait_limit.  Only
// for waves that know every bulk workgroup to have started.
template <class M>
__device__ __forceinline__ bool hand_take(const M& m, const HandQueue& q, HandedWalk& w)
{
    const uint32_t ticket = (uint32_t)(m.add(q.hand + HAND_QUEUE, 1ull << 32) >> 32);
    if (ticket >= q.cap) return false;
    unsigned long long* slot = q.slots + (size_t)ticket * SLOT_WORDS;
    w.w0 = m.load(slot);
    if (w.w0 == SLOT_EMPTY && m.load(q.hand + HAND_DONE) >= q.n_bulk &&
        ticket >= (uint32_t)m.load(q.hand + HAND_QUEUE))
        return false;  // the tail is final and this ticket, taken after it was, is past it
    if (w.w0 == SLOT_EMPTY) {
        const int64_t t0 = m.now();
        do {
            m.pause();
            w.w0 = m.load(slot);
            if (w.w0 == SLOT_EMPTY && m.now() - t0 > q.wait_limit) {
                w.w0 = m.cas_uniform(slot, SLOT_EMPTY, SLOT_CLOSED);
                if (w.w0 == SLOT_EMPTY) return false;
            }
        } while (w.w0 == SLOT_EMPTY);
    }
    if (w.w0 == SLOT_CLOSED) return false;
    do {  // the other words are there or on their way
        w.w1 = m.load(slot + 1);
        w.w2 = m.load(slot + 2);
    } while (w.w1 == SLOT_EMPTY || w.w2 == SLOT_EMPTY);
    return true;
}

// The end of a bulk wave's own work.  True if it may take handed-over walks.
template <class M>
__device__ __forceinline__ bool hand_finish(const M& m, const HandQueue& q)
{
    if (m.add(q.hand + HAND_DONE, 1ull) != q.n_bulk - 1u) return hand_all_started(m, q);
    // the last one: the tickets past the tail, and their slots
    const uint64_t qs = m.add(q.hand + HAND_QUEUE, 0ull);
    const uint32_t taken = (uint32_t)(qs >> 32), head = taken < q.cap ? taken : q.cap;
    for (uint32_t i = (uint32_t)qs + m.lane(); i < head; i += m.lanes())
        m.store(q.slots + (size_t)i * SLOT_WORDS, SLOT_CLOSED);
    return true;
}

}  // namespace srw
