// A group of workgroups that stay on the device for a whole launch and meet at barriers.
//
// Who takes part is settled by the workgroups themselves: each takes a ticket when it starts, and
// the first one closes the group when the whole grid has arrived or after 20 us, whichever comes
// first.  Workgroups that start later leave at once.  Every member is therefore already running,
// so a barrier always ends, whatever else occupies the device (other streams' launches, other
// groups), with no cooperative launch and no assumption about how many workgroups fit.
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
constexpr uint64_t kGridCloseTicks = 2000;  // 20 us of the 100 MHz wall clock
constexpr uint32_t kGridClosed = 1u << 31;

struct GridLine {  // one 128-byte line per contended word
    unsigned long long w;
    uint64_t pad[15];
};
struct GridSync {
    GridLine ticket;      // tickets taken; bit 31 once the group is closed
    GridLine members;     // group size, 0 until closed
    GridLine ring[4][1 + kGridSub];  // barrier words: ring[phase % 4] = root, then the subgroups
    GridLine cursor[3];   // append cursors of the launch
    unsigned long long sums[kGridMax];  // one word per member
};

struct Grid {
    GridSync* s;
    uint32_t rank, members, phase;
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

// Waits until the wave's loads, stores and atomics are complete (stores and atomics without a
// return value count too).
__device__ __forceinline__ void drain_memory() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Takes part in the group, or returns false: the workgroup must then leave.  `lds` is two words.
__device__ __forceinline__ bool grid_join(GridSync* s, Grid& g, uint32_t* lds)
{
    if (threadIdx.x == 0) {
        uint32_t* ticket = reinterpret_cast<uint32_t*>(&s->ticket.w);
        uint32_t* members = reinterpret_cast<uint32_t*>(&s->members.w);
        const uint32_t t = ag_add(ticket, 1u);
        uint32_t m = 0;
        if (t == 0) {
            const uint64_t t0 = wall_clock64();
            while (ag_load(ticket) < gridDim.x && wall_clock64() - t0 < kGridCloseTicks)
                __builtin_amdgcn_s_sleep(1);
            m = __hip_atomic_fetch_or(ticket, kGridClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ag_store(members, m);
        } else if (!(t & kGridClosed)) {
            while ((m = ag_load(members)) == 0)  // the first ticket's holder is running
                __builtin_amdgcn_s_sleep(1);
        }
        lds[0] = t;
        lds[1] = m;
    }
    __syncthreads();
    g = Grid{s, lds[0], lds[1], 0};
    return g.members != 0;
}

// All members arrive; each gives a payload (below 2^54 in total), which thread 0 computes once
// the workgroup's threads have met, and every thread gets the sum.  Between arriving and waiting
// every thread runs overlap(): loads of what no member changes, stores that no member reads in
// this launch.  leave() is thread 0's, before the workgroup goes on.  `lds` is one word of the
// workgroup's own.
template <class Payload, class Overlap, class Leave>
__device__ __forceinline__ uint64_t grid_barrier(Grid& g, uint64_t* lds, Payload payload, Overlap overlap, Leave leave)
{
    constexpr uint64_t kCount = (1ull << kGridArrive) - 1;
    drain_memory();
    __syncthreads();
    GridLine* const w = g.s->ring[g.phase & 3];
    uint32_t need = g.members;
    uint64_t total = 0;
    if (threadIdx.x == 0) {
        total = payload();
        if (g.members > 1) {
            unsigned long long add = (total << kGridArrive) + 1;
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
        if (g.members > 1) {
            unsigned long long x;
            while ((uint32_t)((x = ag_load(&w[0].w)) & kCount) != need)
                __builtin_amdgcn_s_sleep(1);
            total = x >> kGridArrive;
            if (g.rank == 0) {
                // every member has left the previous phase: its words are free, and are zero
                // again before this member arrives at the next phase
                GridLine* z = g.s->ring[(g.phase + 3) & 3];
                for (uint32_t q = 0; q < 1 + kGridSub; q++)
                    ag_store(&z[q].w, 0ull);
            }
        }
        *lds = total;
        leave();
    }
    g.phase++;
    __syncthreads();
    return *lds;
}
template <class Payload, class Overlap>
__device__ __forceinline__ uint64_t grid_barrier(Grid& g, uint64_t* lds, Payload payload, Overlap overlap)
{
    return grid_barrier(g, lds, payload, overlap, [] {});
}
__device__ __forceinline__ void grid_barrier(Grid& g, uint64_t* lds)
{
    (void)grid_barrier(g, lds, []() -> uint64_t { return 0; }, [] {});
}

}  // namespace mphx
