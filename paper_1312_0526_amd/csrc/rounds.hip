// Peeling rounds and the layered assignment of a run, each in ONE launch.
//
// A peel at gamma 1.23 takes about 60 synchronous rounds and as many assignment layers, and below
// some 10^7 keys a round's work is far smaller than what a launch costs: at 10^6 keys k_apply took
// 10.3 us a round and k_assign_round 4.4, of which the memory operations of a plateau round
// (about 5,000 edges) need under 1.  Here a group of workgroups (grid.h) stays on the device and
// goes through the rounds with a barrier between them.
//
// What bounds a round is then its chain of dependent accesses: edge and state, the deletes, the
// claim, the barrier.  So the next layer never leaves the compute unit that found it: each
// workgroup keeps the edges it claimed first in a list of its own in LDS and deletes them itself
// in the next round.  Claims beyond the list's size, and round 0's layer, go through a list in
// device memory that all members share.  A plateau round of 4,000 edges at 10^6 keys takes 4.1 us with
// 122 members, 1.65 of them the barrier; layers above some 50,000 edges are bound by the device's atomics
// (20 G/s).  The order of a layer's slots is free (Section 4.2), and
// the layers come out back to back as the other paths write them.
#include "common.h"
#include "grid.h"
#include "launch.h"

#include <algorithm>

namespace mphx {

constexpr uint32_t kRoundsBlock = 512;
constexpr uint32_t kPrivate = 4096;          // edges of a workgroup's own list
constexpr uint32_t kPrivateBits = 21;        // a barrier's payload: edges of private lists, then of the shared one
static_assert(kPrivate * kGridMax < 1u << kPrivateBits && kPrivateBits + 32 <= 53, "both counts fit");
// Every so many rounds all edges of the next layer go through the shared list, which deals them out
// evenly: the private lists grow by descent, and without it one of 122 workgroups held 4 times its
// share of a layer after 50 rounds at 10^6 keys.  The rounds took 397, 386, 385 and 412 us with a deal
// every 4, 8, 16 and 32 rounds there, 427 without.
constexpr uint32_t kDealRounds = 16;
constexpr uint32_t kRoundsPerLaunch = 1024;  // a longer peel goes on in another launch

__global__ __launch_bounds__(256) void k_run_init(Ctrl* ctrl, uint64_t* lstart, unsigned long long* lcount,
                                                  GridSync* sync, uint32_t nsync, uint64_t zero_words)
{
    unsigned long long* w = reinterpret_cast<unsigned long long*>(sync);
    for (uint32_t i = threadIdx.x; i < nsync * (sizeof(GridSync) / 8); i += 256)
        w[i] = 0;
    if (threadIdx.x < sizeof(Ctrl) / 8)
        reinterpret_cast<uint64_t*>(ctrl)[threadIdx.x] = 0;
    for (uint64_t i = threadIdx.x; i < zero_words; i += 256)
        lcount[i] = 0;
    __syncthreads();
    if (threadIdx.x == 0) {
        ctrl->nrounds = 0xFFFFFFFFu;
        lstart[0] = 0;
    }
}

// Lane of the active ones appends one entry: one LDS atomic per wave.
__device__ __forceinline__ uint32_t lds_append(uint32_t* counter)
{
    const uint64_t mask = __ballot(1);
    const int leader = __ffsll((long long)mask) - 1;
    uint32_t base = 0;
    if ((int)__lane_id() == leader)
        base = atomicAdd(counter, (uint32_t)__popcll(mask));
    return (uint32_t)__builtin_amdgcn_readlane((int)base, leader) + lanes_below(mask);
}

// A range shared by the members is dealt out wave by wave, so that a range shorter than the group
// still occupies as many compute units as it has waves: a layer of 3,300 edges dealt out by
// workgroups of 1024 kept four compute units busy for 4.6 us.
__device__ __forceinline__ uint64_t member_first(const Grid& g)
{
    const uint32_t wave = threadIdx.x / kWave;
    return ((uint64_t)wave * g.members + g.rank) * kWave + (threadIdx.x & (kWave - 1));
}
__device__ __forceinline__ uint64_t member_stride(const Grid& g) { return (uint64_t)g.members * kRoundsBlock; }

struct RoundsArgs {
    uint64_t* rec;
    const uint32_t* edges;
    uint32_t* state;
    uint3* slots;
    uint64_t* lstart;
    unsigned long long* lcount;
    Ctrl* ctrl;
    GridSync* sync;
    uint64_t n, P, rcap;
    uint64_t limit;  // a layer beyond it ends the launch
    uint64_t first;  // a layer 0 beyond it: nothing is done
    uint32_t wait;   // grid_join's
    const uint32_t* vin;  // static functions: see PeelState
    uint32_t* vout;
};

// Edges of kR vertices; an edge state is unclaimed or (round << kShift) | hinge position; with
// kTri the vertex of position q lies in part q and the layer slots are rewritten hinge first.
// The edge of layer r is deleted at its vertices other than the hinge; the delete that takes a
// vertex from degree 2 to 1 claims the vertex's last edge for round r + 1 (lowest position wins)
// and its first claimer appends the edge, as in k_apply.
//
// kGrow: the group may begin without the whole grid.  What it takes to grow costs rounds 5 to 14% in registers
// alone (453 against 490 us a build at 4x10^4 keys), so a group that is whole at once has a kernel of its own.
struct RoundsShared {
    uint32_t list[2][kPrivate];
    uint32_t next[2], join[3];
    uint64_t total, off;
    unsigned long long push, claims;
};

template <int kR, bool kTri, int kShift, bool kGrow>
__device__ __forceinline__ void peel_rounds(const RoundsArgs& a, Grid& g, RoundsShared& sh)
{
    static_assert(!kTri || kR == 3, "parts hold one vertex each");
    auto& s_list = sh.list;
    auto& s_next = sh.next;
    uint64_t &s_total = sh.total, &s_off = sh.off;
    unsigned long long &s_push = sh.push, &s_claims = sh.claims;
    Ctrl* const c = a.ctrl;
    const uint32_t tid = threadIdx.x;
    const bool lead = g.rank == 0 && tid == 0;
    uint64_t lo = c->run_lo, glist = c->run_list, pos = 0;  // pos: the shared list's edges that are done
    uint32_t r = c->run_r, done = 0;
    // Edges of private lists, a cursor for even and one for odd rounds: a member moves it after it has
    // arrived, so others may be one round ahead of it, but not two.
    GridLine* const pcur = a.sync->cursor;
    unsigned long long* const gcur = &a.sync->cursor[2].w;  // edges of shared lists, all rounds
    uint64_t psum = 0, pother = 0, gsum = 0;  // what the cursors passed before this round
    uint64_t ptot = 0;            // this layer's private edges
    uint32_t pc = 0, cur = 0;
    if (!kGrow || g.phase == 0) {
        if (r == 0) {
            glist = a.lcount[0];
            if (lead) {
                c->f0 = c->ftail;  // before any member adds to it
                c->layer0 = glist;
            }
        }
    } else {  // the place that admit() below gives
        auto place = [&](uint32_t q) { return uniform64(ag_load(&g.s->run[q])); };
        r = (uint32_t)place(0);
        done = (uint32_t)place(1);
        lo = place(2);
        glist = place(3);
        pos = place(4);
        ptot = place(5);
        psum = place(6);
        pother = place(7);
        gsum = place(8);
    }
    auto admit = [&](uint32_t round, uint32_t rounds) {
        if (kGrow && g.grew && lead)
            grid_admit(g, round, rounds, lo, glist, pos, ptot, psum, pother, gsum);
    };
    bool fresh = kGrow && g.grew;  // members without private edges: the next layer is dealt out
    uint64_t pbase = 0;
    unsigned long long mypush = 0, myclaims = 0;
    // this thread's first private edge and its vertices, loaded while the group waited
    uint32_t e0 = 0, v0[kR] = {};
    if (tid == 0) {
        s_next[0] = s_next[1] = 0;
        s_push = s_claims = 0;
    }
    __syncthreads();
    bool more = false;
    for (;; r++, done++) {
        if (lead && r < a.rcap + 2)
            a.lstart[r] = lo;
        if (r >= a.rcap) {
            if (lead)
                atomicOr(&c->err, kErrRounds);
            break;
        }
        // layer r: slots [lo, lo + glist) hold the shared list's edges, the private lists follow
        const uint64_t hi = lo + glist + ptot;
        if (lo == hi)
            break;
        if (done == kRoundsPerLaunch) {
            more = true;
            break;
        }
        if (hi - lo > a.limit && done) {
            // the private lists join the shared one; the hinges stay in the states
            for (uint32_t i = tid; i < pc; i += kRoundsBlock)
                a.slots[pbase + i].x = s_list[cur][i];
            glist = hi - lo;
            more = true;
            break;
        }
        // the last round of a launch leaves the next layer in the shared list
        uint32_t cap = done + 1 == kRoundsPerLaunch ? 0u : kPrivate;
        const uint32_t rr = (r + 1) << kShift;
        uint32_t* const next = s_list[cur ^ 1];
        uint32_t* const count = &s_next[cur ^ 1];
        auto append = [&](uint32_t e) {
            const uint32_t pos = lds_append(count);
            if (pos < cap) {
                next[pos] = e;
            } else {
                const uint64_t idx = wave_append(gcur, true, false) - gsum;
                ag_store(&a.slots[hi + idx].x, e);
            }
        };
        // old[q]: record of vertex v[q] before e's delete (0 where e was not deleted).  All claims
        // are in flight before the first is looked at.
        auto claim = [&](uint32_t e, const uint32_t (&v)[kR], const uint64_t (&old)[kR]) {
            uint32_t x[kR], o[kR];
#pragma unroll
            for (uint32_t q = 0; q < kR; q++) {
                if (Rec::deg(old[q]) == 2) {
                    x[q] = (uint32_t)(Rec::edge(old[q]) - e);
                    uint32_t p = q;
                    if constexpr (!kTri) {
                        const uint32_t* t = a.edges + (uint64_t)kR * x[q];
                        p = 0;
#pragma unroll
                        for (uint32_t k = 1; k < kR; k++)
                            if (t[k] == v[q])
                                p = k;
                    }
                    o[q] = __hip_atomic_fetch_min(&a.state[x[q]], rr | p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
#pragma unroll
            for (uint32_t q = 0; q < kR; q++) {
                if (Rec::deg(old[q]) == 2) {
                    const bool first = o[q] == kUnclaimed;
                    mypush++;
                    myclaims += (first || (o[q] >> kShift) == r + 1) ? 1u : 0u;
                    if (first)
                        append(x[q]);
                }
            }
        };
        auto hinge_first = [&](uint32_t h, const uint32_t (&v)[kR]) {
            return make_uint3(h == 0 ? v[0] : (h == 1 ? v[1] : v[kR - 1]), h == 0 ? v[1] : (h == 1 ? v[kR - 1] : v[0]),
                              h == 0 ? v[kR - 1] : (h == 1 ? v[0] : v[1]));
        };
        // an edge of a long list: the hinge is read first and saves its delete
        auto peel = [&](uint32_t e, uint64_t pos) {
            const uint32_t h = ag_load(&a.state[e]) & ((1u << kShift) - 1);
            const uint32_t* t = a.edges + (uint64_t)kR * e;
            uint32_t v[kR];
            uint64_t old[kR];
#pragma unroll
            for (uint32_t q = 0; q < kR; q++)
                v[q] = t[q];
#pragma unroll
            for (uint32_t q = 0; q < kR; q++)
                old[q] = q != h ? ag_add(a.rec + v[q], 0ull - (Rec::kOne + e)) : 0ull;
            if constexpr (kTri) {
                a.slots[pos] = hinge_first(h, v);
                if (a.vin)
                    a.vout[pos] = a.vin[e];
            }
            claim(e, v, old);
        };
        // a thread's first private edge: the deletes do not wait for the state -- the hinge's
        // record, of degree 1, drops to 0 -- and the slot is written after the group is told
        uint3 slot = make_uint3(0u, 0u, 0u);
        const bool mine = tid < pc;
        const uint32_t e1 = e0;
        if (mine) {
            uint64_t old[kR];
#pragma unroll
            for (uint32_t q = 0; q < kR; q++)
                old[q] = ag_add(a.rec + v0[q], 0ull - (Rec::kOne + e1));
            if constexpr (kTri)
                slot = hinge_first(ag_load(&a.state[e1]) & ((1u << kShift) - 1), v0);
            claim(e1, v0, old);
        }
        for (uint32_t i = tid + kRoundsBlock; i < pc; i += kRoundsBlock)
            peel(s_list[cur][i], pbase + i);
        for (;;) {
            const uint64_t to = !kGrow || g.whole() ? glist : min(glist, pos + member_stride(g) * kGridSpan);
            for (uint64_t j = pos + member_first(g); j < to; j += member_stride(g))
                peel(ag_load(&a.slots[lo + j].x), lo + j);
            if (!kGrow || to == glist)
                break;
            pos = to;
            grid_barrier<kGrow>(g, &s_total);
            fresh |= g.grew;
            admit(r, done);
        }
        if (g.members > 1 && (fresh || done % kDealRounds == kDealRounds - 1)) {
            __syncthreads();
            const uint32_t p = min(*count, cap);
            if (tid == 0)
                s_off = p ? ag_add(gcur, p) : 0ull;
            __syncthreads();
            for (uint32_t i = tid; i < p; i += kRoundsBlock)
                ag_store(&a.slots[hi + (s_off - gsum) + i].x, next[i]);
            cap = 0;
            fresh = false;
        }
        uint32_t pnext = 0;
        uint64_t off = 0;
        const uint64_t total = grid_barrier<kGrow>(
            g, &s_total,
            [&]() -> uint64_t {
                const uint32_t k = *count, p = min(k, cap);
                s_next[cur] = 0;
                return (uint64_t)p | (uint64_t)(k - p) << kPrivateBits;
            },
            [&] {
                if constexpr (kTri) {
                    if (mine) {
                        a.slots[pbase + tid] = slot;
                        if (a.vin)
                            a.vout[pbase + tid] = a.vin[e1];
                    }
                }
                pnext = min(*count, cap);
                // where this workgroup's private edges of the next layer go; nobody waits for it
                // before the group has met
                if (tid == 0 && pnext)
                    off = ag_add(&pcur[done & 1].w, pnext);
                if (tid < pnext) {
                    e0 = next[tid];
#pragma unroll
                    for (uint32_t q = 0; q < kR; q++)
                        v0[q] = a.edges[(uint64_t)kR * e0 + q];
                }
            },
            [&] { s_off = off; });
        lo = hi;
        ptot = total & ((1ull << kPrivateBits) - 1);
        glist = total >> kPrivateBits;
        pc = pnext;
        pbase = lo + glist + (s_off - psum);
        const uint64_t passed = psum + ptot;
        psum = pother;
        pother = passed;
        gsum += glist;
        cur ^= 1;
        if constexpr (kGrow) {
            pos = 0;
            fresh |= g.grew;
            admit(r + 1, done + 1);
        }
    }
    if (lead) {
        if constexpr (kGrow) {
            grid_done(g);
            c->joined += g.members - g.first;
        }
        if (more) {
            a.lcount[r] = glist;
            c->run_lo = lo;
            c->run_list = glist;
            c->run_r = r;
        } else if (r < a.rcap) {
            c->nrounds = min(c->nrounds, r);  // a claim-list round may have been the first empty one
            c->peeled = lo;
        }
    }
    if (mypush) atomicAdd(&s_push, mypush);
    if (myclaims) atomicAdd(&s_claims, myclaims);
    __syncthreads();
    if (tid == 0) {
        if (s_push) atomicAdd(&c->ftail, s_push);
        if (s_claims) atomicAdd(&c->claims, s_claims);
    }
}

// Without kGrow a group that does not find room for its whole grid leaves everything as it is, and the caller
// launches the other kind.
template <int kR, bool kTri, int kShift, bool kGrow>
__global__ __launch_bounds__(kRoundsBlock) void k_rounds(RoundsArgs a)
{
    __shared__ RoundsShared sh;
    // a degree above 255 (see k_round0) or a bad edge: nothing may be read off the records, and every
    // workgroup leaves.  (A launch that goes on from a later round has passed this.)
    if (a.ctrl->run_r == 0 && ((a.ctrl->err & (kErrDegree | kErrBadEdge)) || a.ctrl->degsum != (uint64_t)kR * a.n ||
                               a.lcount[0] > a.first))
        return;
    Grid g;
    if (!grid_join<kGrow>(a.sync, g, sh.join, a.wait))
        return;
    peel_rounds<kR, kTri, kShift, kGrow>(a, g, sh);
}

// The layers of a complete peel, last first, with a barrier after each: load(i) reads slot i, which
// nobody changes, and solve(item) solves it; a thread's first slot of the next layer is read while
// the group waits.  The layers at the end of a peel hold few edges: member 0 alone goes through
// those at the top that one pass of its threads covers, with barriers of its own; with kHop through any
// two such layers in a row, which the plateau of a small peel consists of.  Builds of u64 keys took 530 us
// without and 478 with at 3x10^4, 467 and 437 at 4.5x10^4, 462 and 448 at 6x10^4, 492 and 490 at 10^5; at 10^6, where
// no layer but the top ones is that small, the test itself costs 10 us.
constexpr uint32_t kLayerChunk = 1024;
constexpr uint64_t kHopMax = 100'000;  // keys
template <bool kHop, bool kGrow, class Item, class Load, class Solve>
__device__ __forceinline__ void solve_layers_as(Grid& g, const uint64_t* __restrict__ lstart, uint32_t nrounds,
                                                Ctrl* ctrl, uint64_t* s_ls, uint64_t* s_total, Load load,
                                                Solve solve)
{
    const uint32_t tid = threadIdx.x;
    const bool lead = g.rank == 0 && tid == 0;
    uint64_t first = member_first(g), stride = member_stride(g);
    bool solo = !(kGrow && g.grew), have = false;
    // a workgroup that is taken in goes on with layer left - 1, from slot `resume` on
    uint32_t left = nrounds;
    uint64_t resume = 0;
    if (kGrow && g.grew) {
        left = uniform((uint32_t)ag_load(&g.s->run[0]));
        resume = uniform64(ag_load(&g.s->run[1]));
    }
    Item ahead{};
    uint32_t top = nrounds;  // layers [base, top) have their bounds in s_ls
    while (top > 0) {
        const uint32_t base = top > kLayerChunk ? top - kLayerChunk : 0;
        if (kGrow && base >= left) {
            top = base;
            continue;
        }
        __syncthreads();
        for (uint32_t k = tid; k <= top - base; k += kRoundsBlock)
            s_ls[k] = lstart[base + k];
        __syncthreads();
        for (uint32_t k = (kGrow ? min(top, left) : top) - base; k-- > 0;) {
            const uint64_t lo = s_ls[k], hi = s_ls[k + 1];
            const uint64_t below = k ? s_ls[k - 1] : lo;  // the next layer is [below, lo)
            if (hi - lo <= kRoundsBlock && (solo || (kHop && k && lo - below <= kRoundsBlock))) {
                if (kHop && !solo) {
                    solo = true;
                    have = false;  // what was read ahead was the group's share
                }
                if (g.rank == 0) {
                    if (lo + tid < hi)
                        solve(have ? ahead : load(lo + tid));
                    have = k && lo - below <= kRoundsBlock;
                    if (have && below + tid < lo)
                        ahead = load(below + tid);
                    drain_memory();
                    __syncthreads();
                }
                continue;
            }
            if (solo) {
                solo = have = false;
                grid_barrier<false>(g, s_total);
            }
            uint64_t from = kGrow ? max(lo, resume) : lo, to;
            resume = 0;
            do {
                to = !kGrow || g.whole() ? hi : min(hi, from + stride * kGridSpan);
                uint64_t i = from + first;
                if (i < to) {
                    solve(have ? ahead : load(i));
                    for (i += stride; i < to; i += stride)
                        solve(load(i));
                }
                have = k != 0 && to == hi;
                grid_barrier<kGrow>(
                    g, s_total, []() -> uint64_t { return 0; },
                    [&] {
                        if (have && below + first < lo)
                            ahead = load(below + first);
                    });
                if (kGrow && g.grew) {
                    first = member_first(g);
                    stride = member_stride(g);
                    have = false;
                    if (lead)
                        grid_admit(g, base + k + (to == hi ? 0u : 1u), to == hi ? 0ull : to);
                }
                from = to;
            } while (to != hi);
        }
        top = base;
    }
    if (solo)
        grid_barrier<false>(g, s_total);
    if (kGrow && lead) {
        grid_done(g);
        ctrl->joined += g.members - g.first;
    }
}
template <bool kHop, class Item, class Load, class Solve>
__device__ __forceinline__ void solve_layers(Grid& g, const uint64_t* __restrict__ lstart, uint32_t nrounds,
                                             Ctrl* ctrl, uint64_t* s_ls, uint64_t* s_total, Load load, Solve solve)
{
    if (!g.grew && g.whole())  // since the beginning
        solve_layers_as<kHop, false, Item>(g, lstart, nrounds, ctrl, s_ls, s_total, load, solve);
    else
        solve_layers_as<kHop, true, Item>(g, lstart, nrounds, ctrl, s_ls, s_total, load, solve);
}

// By the group that begins the run: a barrier follows.
__device__ __forceinline__ void zero_shared(Grid& g, uint64_t* p, uint64_t words)
{
    for (uint64_t i = member_first(g); i < words; i += member_stride(g))
        ag_store(p + i, (uint64_t)0);
}

// The whole rest of an MPHF build whose peel is complete: the codes (one byte per vertex, over
// the records), layer by layer; the packed codes and rank samples, each member's share of the
// vertices after a prefix over the members.  Does nothing after an incomplete peel.  With nrounds
// given only the layers, over codes that are zero: clearing and packing up to 2^30 of them would be
// kept from growing with the group.
template <bool kHop>
__global__ __launch_bounds__(kRoundsBlock) void k_mphf_finish(const uint3* __restrict__ slots,
                                                              const uint64_t* __restrict__ lstart, Ctrl* ctrl,
                                                              GridSync* sync, uint32_t nrounds, uint64_t n, uint64_t m,
                                                              uint64_t P, uint64_t* code_words, uint64_t* __restrict__ codes,
                                                              uint64_t* __restrict__ rank, uint32_t* bcount, uint32_t wait)
{
    __shared__ uint32_t s_join[3];
    __shared__ uint64_t s_total, s_ls[kLayerChunk + 1], s_wave[kRoundsBlock / kWave], s_carry;
    const bool rest = nrounds == 0;  // enqueued behind launch_rounds
    if (rest) {
        nrounds = ctrl->nrounds;
        if (nrounds == 0xFFFFFFFFu || ctrl->peeled != n)
            return;
    }
    Grid g;
    if (!grid_join<true>(sync, g, s_join, wait))
        return;
    uint8_t* const code8 = reinterpret_cast<uint8_t*>(code_words);
    if (rest && g.phase == 0) {
        zero_shared(g, code_words, (m + 7) / 8);  // 8m bytes of records hold it
        grid_barrier<false>(g, &s_total);
    }
    solve_layers<kHop, uint3>(g, lstart, nrounds, ctrl, s_ls, &s_total, [&](uint64_t i) { return slots[i]; }, [&](uint3 t) {
        const uint32_t k = part_of(t.x, P);
        const uint32_t ca = ag_load(code8 + t.y), cb = ag_load(code8 + t.z);
        const uint32_t x = (k + 6 - (ca == 3 ? 0u : ca) - (cb == 3 ? 0u : cb)) % 3;
        ag_store(code8 + t.x, (uint8_t)(x ? x : 3));
    });
    if (!rest)
        return;
    // this member's rank blocks [b0, b1) of 512 vertices, one thread per code word of 32
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const uint64_t nwords = (m + 31) / 32, nb = (m + 511) / 512, per = (nb + g.members - 1) / g.members;
    const uint64_t b0 = min(nb, g.rank * per), b1 = min(nb, b0 + per);
    uint64_t mine = 0;
    for (uint64_t base = 16 * b0; base < 16 * b1; base += kRoundsBlock) {
        const uint64_t w = base + tid;
        uint64_t x = 0;
        if (w < 16 * b1 && w < nwords) {
            if (32 * w + 32 <= m) {
#pragma unroll
                for (uint32_t q = 0; q < 4; q++) {
                    const uint64_t d = ag_load(code_words + 4 * w + q);
#pragma unroll
                    for (uint32_t t = 0; t < 8; t++)
                        x |= (d >> (8 * t) & 3u) << (2 * (8 * q + t));
                }
            } else {
                for (uint64_t t = 0; 32 * w + t < m; t++)
                    x |= (uint64_t)(ag_load(code8 + 32 * w + t) & 3u) << (2 * t);
            }
            codes[w] = x;
        }
        uint32_t k = nz_pairs(x);
        k += __shfl_xor(k, 1, 16);
        k += __shfl_xor(k, 2, 16);
        k += __shfl_xor(k, 4, 16);
        k += __shfl_xor(k, 8, 16);
        if (w < 16 * b1 && (w & 15) == 0) {
            bcount[w >> 4] = k;  // read by this workgroup only
            mine += k;
        }
    }
    for (uint32_t d = kWave / 2; d > 0; d >>= 1)
        mine += __shfl_xor(mine, d, kWave);
    if (lane == 0)
        s_wave[wv] = mine;
    __syncthreads();
    if (tid == 0) {
        uint64_t t = 0;
        for (uint32_t q = 0; q < kRoundsBlock / kWave; q++)
            t += s_wave[q];
        ag_store(&sync->sums[g.rank], (unsigned long long)t);
        s_carry = 0;
    }
    grid_barrier<false>(g, &s_total);
    if (wv == 0) {  // hinges below this member's first vertex
        uint64_t t = 0;
        for (uint32_t q = lane; q < g.rank; q += kWave)
            t += ag_load(&sync->sums[q]);
        for (uint32_t d = kWave / 2; d > 0; d >>= 1)
            t += __shfl_xor(t, d, kWave);
        if (lane == 0)
            s_carry = t;
    }
    __syncthreads();
    for (uint64_t base = b0; base < b1; base += kRoundsBlock) {
        const uint64_t b = base + tid;
        const uint64_t x = b < b1 ? bcount[b] : 0u;
        uint64_t incl = x;
        for (uint32_t d = 1; d < kWave; d <<= 1) {
            const uint64_t y = __shfl_up(incl, d, kWave);
            if (lane >= d)
                incl += y;
        }
        if (lane == kWave - 1)
            s_wave[wv] = incl;
        __syncthreads();
        uint64_t pre = s_carry;
        for (uint32_t q = 0; q < wv; q++)
            pre += s_wave[q];
        if (b < b1)
            rank[b] = pre + incl - x;
        __syncthreads();
        if (tid == kRoundsBlock - 1)
            s_carry = pre + incl;
        __syncthreads();
    }
}

// The values u of a static function whose peel is complete (zero off the hinges), as
// k_sf_assign_round solves them.  Does nothing after an incomplete peel.  With nrounds given they
// are zero already.
template <typename T, bool kHop>
__global__ __launch_bounds__(kRoundsBlock) void k_sf_solve(const uint3* __restrict__ slots,
                                                           const uint32_t* __restrict__ vals,
                                                           const uint64_t* __restrict__ lstart, Ctrl* ctrl,
                                                           GridSync* sync, uint32_t nrounds, uint64_t n, uint64_t m,
                                                           uint64_t sigma, uint64_t* u_words, uint32_t wait)
{
    __shared__ uint32_t s_join[3];
    __shared__ uint64_t s_total, s_ls[kLayerChunk + 1];
    const bool rest = nrounds == 0;  // enqueued behind launch_rounds
    if (rest) {
        nrounds = ctrl->nrounds;
        if (nrounds == 0xFFFFFFFFu || ctrl->peeled != n)
            return;
    }
    Grid g;
    if (!grid_join<true>(sync, g, s_join, wait))
        return;
    T* const u = reinterpret_cast<T*>(u_words);
    if (rest && g.phase == 0) {
        zero_shared(g, u_words, (m * sizeof(T) + 7) / 8);
        grid_barrier<false>(g, &s_total);
    }
    auto load = [&](uint64_t i) { return make_uint4(slots[i].x, slots[i].y, slots[i].z, vals[i]); };
    solve_layers<kHop, uint4>(g, lstart, nrounds, ctrl, s_ls, &s_total, load, [&](uint4 t) {
        uint64_t x = (uint64_t)t.w + 2 * sigma - ag_load(u + t.y) - ag_load(u + t.z);
        x = x >= sigma ? x - sigma : x;
        x = x >= sigma ? x - sigma : x;
        ag_store(u + t.x, (T)x);
    });
}

// ------------------------------------------------------------------------------------------
size_t run_sync_bytes() { return 3 * sizeof(GridSync); }

// Members of a group for n edges.  Few make the barrier cheap (0.8 us at 8 members, 1.3 at 64), many
// hide the latency of the large first rounds; whole builds of u64 keys took, in us:
//   members            8     16     32     64    128    192    256
//   10^5 keys        556    487    472    490    543    564    576
//   3x10^5           934    705    607    606    654    700    714
//   10^6            2175   1279    870    734    714    735    750
//   3x10^6          5891   3139   1907   1346   1174   1174   1180
//   9x10^6         18971   9761   5891   4012   2927   2655   2582
static unsigned run_grid(const PeelState& st)
{
    const uint64_t n = st.n;
    uint64_t g = std::max({std::min<uint64_t>(n / 4096, 32), std::min<uint64_t>(n / 8192, 128), n / 40960});
    if (st.grid_cap) g = st.grid_cap;
    return (unsigned)std::min<uint64_t>(std::max<uint64_t>(g, 1), kGridMax);
}

hipError_t launch_run_init(const PeelState& st, uint64_t zero_words, hipStream_t s)
{
    k_run_init<<<1, 256, 0, s>>>(st.ctrl, st.lstart, st.lcount, st.sync, 3, zero_words);
    return hipGetLastError();
}

hipError_t launch_sync_zero(const PeelState& st, hipStream_t s) { return launch_zero(st.sync, run_sync_bytes(), s); }

// The edge states and the run's place, for rounds that go on from layer r of a claim-list run (its
// slots hold edge and hinge).
__global__ __launch_bounds__(256) void k_rounds_resume(const uint3* __restrict__ slots,
                                                       const uint64_t* __restrict__ lstart,
                                                       const unsigned long long* __restrict__ lcount,
                                                       uint32_t* __restrict__ state, Ctrl* ctrl, uint32_t r)
{
    const uint64_t lo = lstart[r], count = lcount[r], stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) {
        const uint3 t = slots[lo + i];
        state[t.x] = r << 2 | (t.y & 3u);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ctrl->run_lo = lo;
        ctrl->run_list = count;
        ctrl->run_r = r;
    }
}

hipError_t launch_rounds_resume(const PeelState& st, uint32_t r, hipStream_t s)
{
    hipError_t e = launch_sync_zero(st, s);
    if (e != hipSuccess) return e;
    k_rounds_resume<<<1024, 256, 0, s>>>(st.slots, st.lstart, st.lcount, st.state, st.ctrl, r);
    return hipGetLastError();
}

// The run's place, for rounds that go on from layer r of launches with atomic claims.
__global__ void k_rounds_from(const uint64_t* __restrict__ lstart, const unsigned long long* __restrict__ lcount,
                              Ctrl* ctrl, uint32_t r, uint64_t f0)
{
    ctrl->run_lo = lstart[r];
    ctrl->run_list = lcount[r];
    ctrl->run_r = r;
    ctrl->f0 = f0;
    ctrl->layer0 = lcount[0];
}

hipError_t launch_rounds_from(const PeelState& st, uint32_t r, uint64_t f0, hipStream_t s)
{
    k_rounds_from<<<1, 1, 0, s>>>(st.lstart, st.lcount, st.ctrl, r, f0);
    return hipGetLastError();
}

template <bool kGrow>
static hipError_t launch_rounds_as(const PeelState& st, uint32_t r, bool generic_shift, uint64_t limit, uint64_t first,
                                   hipStream_t s)
{
    const RoundsArgs a{st.rec, st.edges, st.state, st.slots, st.lstart, st.lcount, st.ctrl, st.sync,
                       st.n,   st.P,     st.rcap,  limit,    first,      st.wait,   st.vin,    st.vout};
    const unsigned g = run_grid(st);
    if (st.tripartite) {
        if (r != 3 || generic_shift) return hipErrorInvalidValue;
        k_rounds<3, true, 2, kGrow><<<g, kRoundsBlock, 0, s>>>(a);
        return hipGetLastError();
    }
    if (!generic_shift) {
        if (r != 3) return hipErrorInvalidValue;
        k_rounds<3, false, 2, kGrow><<<g, kRoundsBlock, 0, s>>>(a);
        return hipGetLastError();
    }
    switch (r) {
    case 2: k_rounds<2, false, 3, kGrow><<<g, kRoundsBlock, 0, s>>>(a); break;
    case 3: k_rounds<3, false, 3, kGrow><<<g, kRoundsBlock, 0, s>>>(a); break;
    case 4: k_rounds<4, false, 3, kGrow><<<g, kRoundsBlock, 0, s>>>(a); break;
    case 5: k_rounds<5, false, 3, kGrow><<<g, kRoundsBlock, 0, s>>>(a); break;
    case 6: k_rounds<6, false, 3, kGrow><<<g, kRoundsBlock, 0, s>>>(a); break;
    case 7: k_rounds<7, false, 3, kGrow><<<g, kRoundsBlock, 0, s>>>(a); break;
    case 8: k_rounds<8, false, 3, kGrow><<<g, kRoundsBlock, 0, s>>>(a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_rounds(const PeelState& st, uint32_t r, bool generic_shift, uint64_t limit, uint64_t first, bool grow,
                         hipStream_t s)
{
    return grow ? launch_rounds_as<true>(st, r, generic_shift, limit, first, s)
                : launch_rounds_as<false>(st, r, generic_shift, limit, first, s);
}

__global__ void k_copy_ctrl(const uint64_t* __restrict__ ctrl, const unsigned long long* __restrict__ layer,
                            uint64_t* __restrict__ out)
{
    constexpr uint32_t kWords = sizeof(Ctrl) / 8;
    static_assert(offsetof(Ctrl, layer) == 8 * (kWords - 1), "the last word");
    if (threadIdx.x < kWords)
        out[threadIdx.x] = threadIdx.x == kWords - 1 && layer ? *layer : ctrl[threadIdx.x];
}

hipError_t launch_copy_ctrl(const Ctrl* ctrl, const unsigned long long* layer, Ctrl* out, hipStream_t s)
{
    k_copy_ctrl<<<1, 64, 0, s>>>(reinterpret_cast<const uint64_t*>(ctrl), layer, reinterpret_cast<uint64_t*>(out));
    return hipGetLastError();
}

hipError_t launch_mphf_finish(const PeelState& st, uint32_t nrounds, uint64_t* codes, uint64_t* rank, uint32_t* bcount,
                              hipStream_t s)
{
    auto* const finish = st.n <= kHopMax ? k_mphf_finish<true> : k_mphf_finish<false>;
    finish<<<run_grid(st), kRoundsBlock, 0, s>>>(st.slots, st.lstart, st.ctrl, st.sync + 1, nrounds, st.n, st.m, st.P,
                                                 st.rec, codes, rank, bcount, st.wait);
    return hipGetLastError();
}

hipError_t launch_sf_solve(const PeelState& st, uint32_t nrounds, uint64_t sigma, uint32_t b, hipStream_t s)
{
    const unsigned g = run_grid(st);
#define MPHX_SOLVE(T)                                                                                               \
    (st.n <= kHopMax ? k_sf_solve<T, true> : k_sf_solve<T, false>)<<<g, kRoundsBlock, 0, s>>>(                      \
        st.slots, st.vout, st.lstart, st.ctrl, st.sync + 1, nrounds, st.n, st.m, sigma, st.rec, st.wait)
    switch (sf_elem_bytes(b)) {
    case 1: MPHX_SOLVE(uint8_t); break;
    case 2: MPHX_SOLVE(uint16_t); break;
    default: MPHX_SOLVE(uint32_t);
    }
#undef MPHX_SOLVE
    return hipGetLastError();
}

}  // namespace mphx
