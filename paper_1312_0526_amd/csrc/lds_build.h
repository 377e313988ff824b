// A whole MWHC build in one workgroup with the hypergraph in LDS (key sets of up to about 26,000
// keys), retries included.
//
// What bounds such a build is latency: some 60 rounds and as many assignment layers, each a chain
// of a few accesses between two workgroup barriers.  So everything that a round or a layer touches
// is in LDS, and nothing else is kept: a vertex has a state byte (its degree in 6 bits) and the XOR
// of the other two part-local ids of its incident edges (two 16-bit halves; Section 4.1's packed
// list without edge ids), and a vertex of degree 1 reads its edge off that.  No edge array, edge
// states or layer slots exist: a hinge is never deleted from, so its word still names its edge
// when the assignment comes back to it, and the queue of vertices that reached degree 1, in order,
// is the layers.
//
// A round has one barrier.  A queued vertex of degree 1 is its edge's hinge unless a vertex of a
// lower part of the edge had degree 1 when the round began too; a hinge deletes its edge from the
// other two vertices, and a vertex taken from degree 2 to 1 joins the queue of the next round.
// Degrees change while others are still being looked at, so the two upper bits of a state byte say
// in which round (mod 3) the vertex is to leave: "degree 1, leaving in round r" is what a vertex
// looks for.  That is right although bytes change meanwhile: the hinge itself is never deleted
// from, so every other claimant of its edge sees it; a vertex that drops to degree 1 in this very
// round carries no mark yet, or the next round's; one that fell 2 -> 1 -> 0 has degree 0.
// Same rounds and hinges as the other paths, hence the same codes.
//
// Measured: 0.95 us a round and 0.35 a layer whatever the block size (256 to 1024 threads): some 170
// instructions and 7 LDS accesses of one wave in a row.  A bucket of 16,384 keys takes 137 us; as 32-bit
// records and edge states with the slots in device memory it took 200.
//
// A degree above 63 (mean 2.4) leaves the build to the caller's general path.
#pragma once

#include "common.h"

namespace mphx {

constexpr uint32_t kLdsRounds = 512;     // round starts kept in LDS; later ones in device memory
constexpr uint32_t kLdsMaxVertices = 32768;  // 16-bit ids, and rank blocks of one wave's scan
constexpr uint32_t kQueueNone = 0xFFFFu;

struct __align__(16) LdsBuildState {
    uint32_t tail, err;
    uint32_t peeled[2];  // hinges of try t: peeled[t % 2]
    uint32_t sum[3];  // of the last try: claims, hinges of layer 0, hinges of the last round
    uint32_t more[3];  // vertices queued in round r: more[r % 3]
    uint32_t bcount[kLdsMaxVertices / 512];
    uint32_t start[kLdsRounds];
};

// LDS bytes of m vertices: edge words, degrees, and the queue unless it is in device memory.
__host__ __device__ constexpr uint32_t lds_build_bytes(uint32_t m, bool queue)
{
    return (uint32_t)sizeof(LdsBuildState) + (4 * m + 15) / 16 * 16 + (m + 15) / 16 * 16 +
           (queue ? (2 * m + 15) / 16 * 16 : 0);
}

constexpr int32_t kLdsTooDense = 2;  // a degree above 63 (or rounds that nothing holds): the try is not made
constexpr int32_t kLdsHash = 3;      // the next try's strings are for a launch of their own to hash
struct LdsOutcome {
    uint64_t seed;
    uint32_t tries;
    int32_t status;  // 0; 1: a 2-core remained on every try; kLdsTooDense; kLdsHash
    uint32_t rounds, peeled, frontier0, frontier, claims, layer0;  // of the last try
};

// Room for each active lane's entries, want1 and want2 of them, with one LDS atomic per wave: where the
// lane's first goes.
__device__ __forceinline__ uint32_t queue_reserve(uint32_t* tail, bool want1, bool want2)
{
    const uint64_t b1 = __ballot(want1), b2 = __ballot(want2);
    const uint32_t total = (uint32_t)(__popcll(b1) + __popcll(b2));
    uint32_t base = 0;
    if (total) {
        const int leader = __ffsll((long long)__ballot(1)) - 1;
        if ((int)__lane_id() == leader)
            base = atomicAdd(tail, total);
        base = (uint32_t)__builtin_amdgcn_readlane((int)base, leader);
    }
    return base + lanes_below(b1) + lanes_below(b2);
}

// Builds the MPHF of n keys with parts of P vertices (m = 3P at most kLdsMaxVertices) by all kBlock
// threads of the workgroup.  fetch(i, sd) reads what key i's vertices under seed sd come from and
// locals(key, sd) gives its three part-local vertices; kAhead reads are in flight at once, unless
// slow(sd), where digest(i, sd) takes fetch's place: kAhead copies of a string's hashing cost more
// in instruction fetches than they hide (a served request of 3,638 strings took 269 us with four,
// 208 with one).  slow(sd) is 0, 1 or kLdsHash, which ends the build before that try.
// lds: lds_build_bytes(m, kQueueLds) bytes, 16-byte aligned; gqueue: m entries in device memory,
// used unless kQueueLds; gstart: n + 2 words in device memory, or null: then a peel of kLdsRounds
// rounds or more is left to the general path too.
template <int kBlock, bool kQueueLds, int kAhead, class Slow, class Fetch, class Digest, class Locals>
__device__ LdsOutcome lds_build(uint32_t n, uint32_t P, uint64_t seed, uint32_t max_tries, Slow slow, Fetch fetch,
                                Digest digest, Locals locals,
                                uint8_t* lds, uint16_t* gqueue, uint32_t* gstart, uint64_t* codes, uint64_t* rank)
{
    LdsBuildState& st = *reinterpret_cast<LdsBuildState*>(lds);
    lds += sizeof(LdsBuildState);
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1);
    const uint32_t m = 3 * P;
    uint32_t* const word = reinterpret_cast<uint32_t*>(lds);                          // m
    uint32_t* const deg4 = reinterpret_cast<uint32_t*>(lds + (4 * m + 15) / 16 * 16);  // m bytes
    uint8_t* const deg = reinterpret_cast<uint8_t*>(deg4);
    uint16_t* const queue =
        kQueueLds ? reinterpret_cast<uint16_t*>(reinterpret_cast<uint8_t*>(deg4) + (m + 15) / 16 * 16) : gqueue;
    const uint32_t dwords = (m + 3) / 4;
    constexpr uint32_t kMark = 64, kMaxLdsDegree = kMark - 1;
    // the vertices of part k's word x: parts k + 1 and k + 2
    auto part = [P](uint32_t v) { return v >= 2 * P ? 2u : (v >= P ? 1u : 0u); };
    auto vertex_a = [P](uint32_t k, uint32_t x) { return (k == 2 ? 0u : (k + 1) * P) + (x & 0xFFFFu); };
    auto vertex_b = [P](uint32_t k, uint32_t x) { return (k == 0 ? 2 * P : (k - 1) * P) + (x >> 16); };
    auto start_at = [&](uint32_t r) { return r < kLdsRounds ? st.start[r] : gstart[r]; };

    LdsOutcome out{seed, 0, 1, 0, 0, 0, 0, 0, 0};
    for (uint32_t t = 0; t < max_tries; t++) {
        const uint64_t sd = seed + t;
        const int32_t how = slow(sd);
        if (how == kLdsHash) {
            out.status = kLdsHash;
            return out;
        }
        out.seed = sd;
        out.tries = t + 1;
        for (uint32_t v = tid; v < m; v += kBlock)
            word[v] = 0;
        for (uint32_t v = tid; v < dwords; v += kBlock)
            deg4[v] = 0;
        if (tid == 0) {
            st.tail = st.err = 0;
            st.peeled[t & 1] = 0;  // the try before may still be read
            st.sum[0] = st.sum[1] = st.sum[2] = 0;
            st.more[0] = 0;
        }
        __syncthreads();
        auto insert = [&](uint3 u) {
            const uint32_t v1 = P + u.y, v2 = 2 * P + u.z;
            const uint32_t s0 = 8 * (u.x & 3), s1 = 8 * (v1 & 3), s2 = 8 * (v2 & 3);
            const uint32_t d0 = atomicAdd(&deg4[u.x >> 2], 1u << s0);
            const uint32_t d1 = atomicAdd(&deg4[v1 >> 2], 1u << s1);
            const uint32_t d2 = atomicAdd(&deg4[v2 >> 2], 1u << s2);
            atomicXor(&word[u.x], u.y | u.z << 16);
            atomicXor(&word[v1], u.z | u.x << 16);
            atomicXor(&word[v2], u.x | u.y << 16);
            if (max(d0 >> s0 & 255u, max(d1 >> s1 & 255u, d2 >> s2 & 255u)) >= kMaxLdsDegree)
                st.err = 1;
        };
        if (how) {
#pragma unroll 1
            for (uint32_t i = tid; i < n; i += kBlock)
                insert(locals(digest(i, sd), sd));
        } else {
            for (uint32_t i0 = tid; i0 < n; i0 += kAhead * kBlock) {
                decltype(fetch(0u, sd)) key[kAhead];
#pragma unroll
                for (uint32_t q = 0; q < kAhead; q++)
                    if (i0 + q * kBlock < n)
                        key[q] = fetch(i0 + q * kBlock, sd);
#pragma unroll
                for (uint32_t q = 0; q < kAhead; q++)
                    if (i0 + q * kBlock < n)
                        insert(locals(key[q], sd));
            }
        }
        __syncthreads();
        if (st.err) {
            out.status = kLdsTooDense;
            return out;
        }
        uint32_t mark = kMark;  // of the vertices that leave in this round
        for (uint32_t base = 0; base < dwords; base += kBlock) {  // degree 1 before round 0
            const uint32_t w = base + tid;
            const uint32_t x = w < dwords ? deg4[w] : 0u;
            bool one[4];
            uint32_t add = 0;
#pragma unroll
            for (uint32_t q = 0; q < 4; q++) {
                one[q] = (x >> (8 * q) & 255u) == 1;
                add |= one[q] ? mark << (8 * q) : 0u;
            }
            if (add)
                deg4[w] = x | add;
#pragma unroll
            for (uint32_t q = 0; q < 4; q += 2) {
                uint32_t at = queue_reserve(&st.tail, one[q], one[q + 1]);
                if (one[q])
                    queue[at++] = (uint16_t)(4 * w + q);
                if (one[q + 1])
                    queue[at] = (uint16_t)(4 * w + q + 1);
            }
        }
        if (tid == 0)
            st.start[0] = 0;
        __syncthreads();
        uint32_t r = 0, turn = 0, q0 = 0, q1 = st.tail, hinges = 0, claims = 0;  // turn: r % 3
        out.frontier0 = q1;
        while (q0 != q1) {  // again until a round queues nothing
            const uint32_t turn1 = turn == 2 ? 0 : turn + 1;
            const uint32_t leaves = mark | 1u, next = mark == 3 * kMark ? kMark : mark + kMark;
            for (uint32_t i = q0 + tid; i < q1; i += kBlock) {
                const uint32_t v = queue[i];
                // the word before the state: a delete changes them the other way round (one wave's
                // LDS accesses are performed in order), so the word of a vertex that is still
                // seen to leave is its edge
                const uint32_t x = word[v];
                asm volatile("" ::: "memory");
                const uint32_t d = deg[v], k = part(v);
                const uint32_t va = vertex_a(k, x), vb = vertex_b(k, x);
                // part 1 looks at part 0 (its b), part 2 at parts 0 (a) and 1 (b)
                bool hinge = d == leaves;
                if (hinge) {
                    const uint32_t da = deg[va], db = deg[vb];
                    hinge = (k == 0 || db != leaves) && (k != 2 || da != leaves);
                }
                if (!hinge) {
                    queue[i] = (uint16_t)kQueueNone;
                    continue;
                }
                const uint32_t lv = v - k * P, a = x & 0xFFFFu, b = x >> 16;
                const uint32_t sa = 8 * (va & 3), sb = 8 * (vb & 3);
                const uint32_t da = atomicSub(&deg4[va >> 2], 1u << sa) >> sa & 255u;
                const uint32_t db = atomicSub(&deg4[vb >> 2], 1u << sb) >> sb & 255u;
                asm volatile("" ::: "memory");
                atomicXor(&word[va], b | lv << 16);
                atomicXor(&word[vb], lv | a << 16);
                hinges++;
                claims += 1 + (da == leaves) + (db == leaves);  // the edge's degree-1 vertices
                if (da == 2) {
                    atomicAdd(&deg4[va >> 2], next << sa);
                    queue[q1 + atomicAdd(&st.more[turn], 1u)] = (uint16_t)va;
                }
                if (db == 2) {
                    atomicAdd(&deg4[vb >> 2], next << sb);
                    queue[q1 + atomicAdd(&st.more[turn], 1u)] = (uint16_t)vb;
                }
            }
            if (tid == 0) {
                if (r + 1 < kLdsRounds)
                    st.start[r + 1] = q1;
                else if (gstart)
                    gstart[r + 1] = q1;
                st.more[turn1] = 0;  // last read before the barrier of the round before
            }
            __syncthreads();
            const uint32_t more = st.more[turn];
            r++;
            if (more == 0)
                break;
            q0 = q1;
            q1 += more;
            mark = next;
            turn = turn1;
        }
        if (hinges)
            atomicAdd(&st.peeled[t & 1], hinges);
        __syncthreads();
        out.peeled = st.peeled[t & 1];
        if (out.peeled != n && t + 1 < max_tries)
            continue;  // of such a try only its failure counts (256 buckets of 100 keys: 278 us, 318 with the sums)
        // the last round's queue, [q0, q1), may hold no hinge: then it is no layer
        for (uint32_t i = q0 + tid; i < q1; i += kBlock)
            if (queue[i] != kQueueNone)
                st.sum[2] = 1;
        if (r) {
            uint32_t layer0 = 0;
            for (uint32_t i = tid; i < start_at(1); i += kBlock)
                layer0 += queue[i] != kQueueNone;
            if (layer0)
                atomicAdd(&st.sum[1], layer0);
        }
        if (claims)
            atomicAdd(&st.sum[0], claims);
        __syncthreads();
        out.rounds = r && !st.sum[2] ? r - 1 : r;
        out.frontier = q1;
        out.claims = st.sum[0];
        out.layer0 = st.sum[1];
        __syncthreads();
        if (out.peeled == n) {
            out.status = gstart || r < kLdsRounds ? 0 : kLdsTooDense;
            break;
        }
    }
    if (out.status)
        return out;
    // the layers, last first; the code bytes take the degrees' place.  A thread's first vertex of a
    // layer and its word are read before the barrier in front of the layer.
    for (uint32_t v = tid; v < dwords; v += kBlock)
        deg4[v] = 0;
    uint8_t* const code8 = deg;
    auto solve = [&](uint32_t v, uint32_t x) {
        const uint32_t k = part(v);
        const uint32_t ca = code8[vertex_a(k, x)], cb = code8[vertex_b(k, x)];
        const uint32_t g = (k + 6 - (ca == 3 ? 0u : ca) - (cb == 3 ? 0u : cb)) % 3;
        code8[v] = (uint8_t)(g ? g : 3);
    };
    uint32_t hi = start_at(out.rounds), lo = out.rounds ? start_at(out.rounds - 1) : hi;
    uint32_t v0 = kQueueNone, x0 = 0;
    auto ahead = [&](uint32_t from, uint32_t to) {
        v0 = from + tid < to ? queue[from + tid] : kQueueNone;
        x0 = v0 != kQueueNone ? word[v0] : 0u;
    };
    ahead(lo, hi);
    __syncthreads();
    for (uint32_t r = out.rounds; r-- > 0;) {
        const uint32_t below = r ? start_at(r - 1) : lo;
        if (v0 != kQueueNone)
            solve(v0, x0);
        for (uint32_t i = lo + tid + kBlock; i < hi; i += kBlock) {
            const uint32_t v = queue[i];
            if (v != kQueueNone)
                solve(v, word[v]);
        }
        hi = lo;
        lo = below;
        ahead(lo, hi);
        __syncthreads();
    }
    // 32 codes per word, counted per 512 vertices
    const uint32_t nwords = (m + 31) / 32, nb = (m + 511) / 512;
    for (uint32_t base = 0; base < nwords; base += kBlock) {
        const uint32_t w = base + tid;
        uint64_t x = 0;
        if (w < nwords) {
#pragma unroll
            for (uint32_t q = 0; q < 8; q++) {
                // bytes past m within the last word are the codes of no vertex: zero
                const uint32_t d = 8 * w + q < dwords ? deg4[8 * w + q] : 0u;
                const uint32_t c = (d & 3u) | (d >> 6 & 0xCu) | (d >> 12 & 0x30u) | (d >> 18 & 0xC0u);
                x |= (uint64_t)c << (8 * q);
            }
            codes[w] = x;
        }
        uint32_t c = nz_pairs(x);
        c += __shfl_xor(c, 1, 16);
        c += __shfl_xor(c, 2, 16);
        c += __shfl_xor(c, 4, 16);
        c += __shfl_xor(c, 8, 16);
        if (w < nwords && (w & 15) == 0)
            st.bcount[w >> 4] = c;
    }
    __syncthreads();
    if (tid < kWave) {  // nb <= 64
        const uint32_t c = lane < nb ? st.bcount[lane] : 0u;
        uint32_t incl = c;
        for (uint32_t d = 1; d < kWave; d <<= 1) {
            const uint32_t y = __shfl_up(incl, d, kWave);
            if (lane >= d)
                incl += y;
        }
        if (lane < nb)
            rank[lane] = incl - c;
    }
    __syncthreads();
    return out;
}

}  // namespace mphx
