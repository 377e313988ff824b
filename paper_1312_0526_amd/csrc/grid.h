// A group of workgroups that stay on the device for a whole launch and meet at barriers.
//
// Who takes part is settled by the workgroups themselves: each takes a ticket when it starts, and
// the first one begins when the whole grid has arrived or after `wait` ticks (20 us), whichever comes
// first.  On a busy device these may be few, so the group grows: a workgroup that starts later waits,
// and the barriers marked kGrow take in all that wait (the run's place is handed to them through
// `run`).  A group that is not whole yet goes through long lists in spans of kGridSpan items per
// thread with such a barrier behind each, so the device is taken up again soon after it becomes
// free.  With the size that it began with, the group of a build of 9x10^6 keys which found 2 of 256
// compute units free, the others for 1.3 ms not, took 22 to 56 ms instead of 2.6; 3.9 so.  Every member has
// taken its ticket and is therefore running, so a barrier always ends, whatever else occupies the device (other
// streams' launches, other groups), with no cooperative launch and no assumption about how many
// workgroups fit.  A whole group pays nothing for this.
//
// Data that one member writes and another reads inside the launch goes through agent-scope atomic
// loads, stores and read-modify-writes (ag_load, ag_store): they are performed at the point all
// compute dies share, and grid_barrier waits for the wave's outstanding memory operations before
// the workgroup arrives, so what was written before a barrier is seen after it.  No cache is
// written back or invalidated: with agent fences a barrier of 64 workgroups measured 3.3 us
// instead of 1.3, and of 256 workgroups 13.8 instead of 3.9 (1.9 in two levels).  Data written
// by earlier launches needs none of this.
#pragma once

#include "common.h"

namespace mphx {

constexpr uint32_t kGridMax = 256;          // members at most
constexpr uint32_t kGridSub = 8;            // subgroups of a large group's barrier
constexpr uint32_t kGridFlat = 64;          // up to here all members count on one word
constexpr uint32_t kGridArrive = 10;        // low bits of a barrier word: arrivals
constexpr uint32_t kGridSpan = 16;          // items per thread between two chances to grow
constexpr uint32_t kGridRun = 9;            // words of a run's place
constexpr uint64_t kGridDone = 1ull << 63;

struct GridLine {  // one 128-byte line per contended word
    unsigned long long w;
    uint64_t pad[15];
};
struct GridSync {
    GridLine ticket;      // tickets taken
    GridLine admit;       // group size (0 before it begins), << 32 the phase the newest begin with, kGridDone at the end
    GridLine ring[4][1 + kGridSub];  // barrier words: ring[phase % 4] = root, then the subgroups
    GridLine grown[4];    // grown[phase % 4]: the size after a phase that says so
    GridLine cursor[3];   // append cursors of the launch
    unsigned long long run[16];      // a run's place when the newest were taken in
    unsigned long long sums[kGridMax];  // one word per member
};
static_assert(kGridRun <= 16, "run holds a place");

struct Grid {
    GridSync* s;
    uint32_t rank, members, phase;
    bool grew;         // the last barrier took workgroups in, or this one was
    uint32_t first;    // size at the start, phase of the newest (rank 0's)
    uint32_t newest;
    __device__ bool whole() const { return members == gridDim.x; }
};

template <typename T>
__device__ __forceinline__ T ag_load(const T* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T, typename U>
__device__ __forceinline__ void ag_store(T* p, U x)
{
    __hip_atomic_store(p, (T)x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T, typename U>
__device__ __forceinline__ T ag_add(T* p, U x)
{
    return __hip_atomic_fetch_add(p, (T)x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The same value in every lane, and known to be.
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ uint64_t uniform64(uint64_t x)
{
    return uniform((uint32_t)x) | (uint64_t)uniform((uint32_t)(x >> 32)) << 32;
}

// Waits until the wave's loads, stores and atomics are complete (stores and atomics without a
// return value count too).
__device__ __forceinline__ void drain_memory() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Takes part in the group, or returns false: the workgroup must then leave.  g.phase is 0 for those that
// begin the run; others take its place from g.s->run.  Without kGrow all leave unless the whole grid is
// there in time.  `lds` is three words.
template <bool kGrow>
__device__ __forceinline__ bool grid_join(GridSync* s, Grid& g, uint32_t* lds, uint32_t wait)
{
    if (threadIdx.x == 0) {
        uint32_t* ticket = reinterpret_cast<uint32_t*>(&s->ticket.w);
        const uint32_t t = ag_add(ticket, 1u);
        unsigned long long x;
        if (t == 0) {
            const uint64_t t0 = wall_clock64();
            while (ag_load(ticket) < gridDim.x && wall_clock64() - t0 < wait)
                __builtin_amdgcn_s_sleep(1);
            const uint32_t m = wait ? ag_load(ticket) : 1u;  // no wait at all: alone
            x = kGrow || m == gridDim.x ? m : kGridDone;
            ag_store(&s->admit.w, x);
        } else {
            // the first ticket's holder is running, and takes this workgroup in or ends the run
            while ((uint32_t)(x = ag_load(&s->admit.w)) <= t && !(x & kGridDone))
                __builtin_amdgcn_s_sleep(1);
        }
        lds[0] = t;
        lds[1] = (uint32_t)x > t ? (uint32_t)x : 0u;
        lds[2] = (uint32_t)((x & ~kGridDone) >> 32);
    }
    __syncthreads();
    const uint32_t members = lds[1], phase = lds[2];
    g = Grid{s, lds[0], members, phase, phase != 0, members, phase};
    return members != 0;
}

// Thread 0 of rank 0 after a barrier that grew: the newest go on from this place.
template <typename... T>
__device__ __forceinline__ void grid_admit(Grid& g, T... place)
{
    static_assert(sizeof...(T) <= kGridRun, "run holds a place");
    const unsigned long long w[] = {(unsigned long long)place...};
    for (uint32_t q = 0; q < sizeof...(T); q++)
        ag_store(&g.s->run[q], w[q]);
    drain_memory();
    g.newest = g.phase;
    ag_store(&g.s->admit.w, (unsigned long long)g.members | (unsigned long long)g.phase << 32);
}

// Thread 0 of rank 0, behind the last barrier that may grow: who still waits must leave.
__device__ __forceinline__ void grid_done(const Grid& g)
{
    ag_store(&g.s->admit.w, kGridDone | (unsigned long long)g.newest << 32 | g.members);
}

// All members arrive; each gives a payload (below 2^53 in total), which thread 0 computes once
// the workgroup's threads have met, and every thread gets the sum.  Between arriving and waiting
// every thread runs overlap(): loads of what no member changes, stores that no member reads in
// this launch.  leave() is thread 0's, before the workgroup goes on.  `lds` is one word of the
// workgroup's own.  With kGrow the group may be larger afterwards (g.grew): grid_admit must follow.
template <bool kGrow, class Payload, class Overlap, class Leave>
__device__ __forceinline__ uint64_t grid_barrier(Grid& g, uint64_t* lds, Payload payload, Overlap overlap, Leave leave)
{
    constexpr uint64_t kCount = (1ull << kGridArrive) - 1, kGrew = 1ull << 63;
    constexpr uint32_t kTotalBits = 54;  // of *lds; the new size above
    uint32_t seen = 0;  // tickets taken, where these are more than the members
    if constexpr (kGrow) {
        if (!g.whole() && g.rank == 0 && threadIdx.x == 0) {
            seen = (uint32_t)ag_load(&g.s->ticket.w);
            // every member has left phase - 4, whose word this was
            if (seen > g.members)
                ag_store(&g.s->grown[g.phase & 3].w, seen);
            else
                seen = 0;
        }
    }
    drain_memory();
    __syncthreads();
    GridLine* const w = g.s->ring[g.phase & 3];
    uint32_t need = g.members;
    uint64_t total = 0;
    if (threadIdx.x == 0) {
        total = payload();
        if (g.members > 1) {
            unsigned long long add = ((total << kGridArrive) + 1) | (seen ? kGrew : 0ull);
            bool up = true;
            if (g.members > kGridFlat) {
                // the last arriver of each subgroup carries its sum to the root
                const uint32_t q = g.rank % kGridSub;
                const uint32_t size = (g.members - q + kGridSub - 1) / kGridSub;
                const unsigned long long old = ag_add(&w[1 + q].w, add);
                up = (uint32_t)(old & kCount) == size - 1;
                add += old & ~kCount;
                need = kGridSub;
            }
            if (up)
                (void)ag_add(&w[0].w, add);
        }
    }
    overlap();
    if (threadIdx.x == 0) {
        uint64_t size = seen;
        if (g.members > 1) {
            unsigned long long x;
            while ((uint32_t)((x = ag_load(&w[0].w)) & kCount) != need)
                __builtin_amdgcn_s_sleep(1);
            total = (x & ~kGrew) >> kGridArrive;
            if (kGrow && (x & kGrew))
                size = ag_load(&g.s->grown[g.phase & 3].w);
            if (g.rank == 0) {
                // every member has left the previous phase: its words are free, and are zero
                // again before this member arrives at the next phase
                GridLine* z = g.s->ring[(g.phase + 3) & 3];
                for (uint32_t q = 0; q < 1 + kGridSub; q++)
                    ag_store(&z[q].w, 0ull);
            }
        }
        *lds = total | size << kTotalBits;
        leave();
    }
    g.phase++;
    __syncthreads();
    const uint64_t x = *lds;
    if constexpr (kGrow) {
        const uint32_t size = uniform((uint32_t)(x >> kTotalBits));
        g.grew = size != 0;
        if (size)
            g.members = size;
        return x & ((1ull << kTotalBits) - 1);
    }
    return x;
}
template <bool kGrow, class Payload, class Overlap>
__device__ __forceinline__ uint64_t grid_barrier(Grid& g, uint64_t* lds, Payload payload, Overlap overlap)
{
    return grid_barrier<kGrow>(g, lds, payload, overlap, [] {});
}
template <bool kGrow>
__device__ __forceinline__ void grid_barrier(Grid& g, uint64_t* lds)
{
    (void)grid_barrier<kGrow>(g, lds, []() -> uint64_t { return 0; }, [] {});
}

}  // namespace mphx
