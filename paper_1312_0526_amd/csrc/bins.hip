// Vertex records of mid-sized key sets and edge lists, and round 0, without device atomics on the
// records.
//
// Up to about 10^7 edges the records lie in or near the caches, and building them was bound by the
// device's rate of atomics, 24 G/s whatever their footprint: three per edge, and then one per vertex
// of degree 1 for round 0's claims.  Here each tile of edges is ordered by vertex bucket in LDS and
// its incidences go out as runs, one device atomic per tile and bucket; a bucket's incidences are
// then summed in LDS.  Neither a histogram nor a second pass is needed, as the vertices are uniform:
// a bucket of 2^s vertices receives 2.44 x 2^s incidences at gamma 1.23 and has room for 2.63 x 2^s,
// the memory of its own records and its share of the layer slots and edge states, all of them
// written later.  When a bucket overflows all the same (skewed edge lists, equal keys), k_bins_again
// builds the records with device atomics after all.
//
// The degree-1 vertices leave the buckets as one bit each too, small enough for an L2 slice (m / 8
// bytes), so round 0 needs no claims: such a vertex is its edge's hinge unless the bit of a lower
// vertex of the edge is set.  Layer 0 comes out in vertex order, and the assignment writes it in
// that order: going over the edges instead made the assignment 10% slower.
//
// Hash, records and round 0 of u64 keys, before and now: 178 and 62 us at 10^6 (atomics), 364 and 111 at
// 3x10^6, 718 and 320 at 9x10^6 (the two-pass partition of part.hip, whose dozen launches and 80 bytes
// per key go by).  What is left: k_bins writes 24 bytes of incidences per edge (1.6 TB/s), round 0 its
// states at random (22 G/s).
#include "common.h"
#include "grid.h"
#include "launch.h"

#include <algorithm>
#include <cmath>

namespace mphx {

// Below, three launches more than the atomics' two cost what they save: hash, records and round 0
// took 42 us with atomics and 52 binned at 10^5 keys, 72 and 47 at 3x10^5.
constexpr uint64_t kBinMinEdges = 3u << 16;
// Tiles of 2048 edges below, of 4096 above.  Large tiles reserve fewer runs, small ones fill the chip
// sooner: k_bins took 19.5, 23.2 and 29.4 us with tiles of 2048, 4096 and 8192 at 3x10^5 keys, 37, 33 and
// 31 at 10^6, 206, 137 and 142 at 9x10^6.
constexpr uint64_t kBinSmallTiles = 1u << 19;
// A bucket is summed in LDS (2^14 records: 128 KB) and listed in LDS by every tile (12 bytes each).
constexpr uint32_t kBinMinShift = 10, kBinMaxShift = 14, kBinMaxBuckets = 2048;
constexpr uint32_t kBinAccBlock = 512;
constexpr uint32_t kBinRound0Block = 512, kBinRound0Per = 8;
constexpr uint32_t kNoVertex = 0xFFFFFFFFu;

struct BinArgs {
    uint64_t n, m, P;
    uint64_t* rec;
    uint32_t* cursor;                // per bucket: incidences so far
    unsigned long long* full;        // not 0: a bucket has overflowed
    uint2* more;                     // per bucket: room for `extra` incidences beyond its records'
    uint32_t extra, shift, nb;
    __device__ uint32_t length(uint32_t b) const  // vertices of bucket b
    {
        return (uint32_t)min<uint64_t>(1ull << shift, m - ((uint64_t)b << shift));
    }
};

__device__ __forceinline__ bool bad_edge(uint32_t x, uint32_t y, uint32_t z, uint64_t m)
{
    return x >= m || y >= m || z >= m || x == y || x == z || y == z;
}

// Edge sources: fetch(i) loads, vertices(i, x, v) yields the edge's vertices (kNoVertex: none).
struct BinKeys {
    const uint64_t* keys;
    uint64_t seed, P;
    uint32_t* edges;
    using Raw = uint64_t;
    static constexpr bool kTri = true;
    __device__ Raw fetch(uint64_t i) const { return keys[i]; }
    __device__ void vertices(uint64_t i, Raw x, uint32_t (&v)[3]) const
    {
        edge_of_digest(x ^ seed, x ^ seed, P, v[0], v[1], v[2]);
        edges[3 * i] = v[0];
        edges[3 * i + 1] = v[1];
        edges[3 * i + 2] = v[2];
    }
};
template <bool kTripartite>
struct BinEdges {
    const uint32_t* edges;
    uint64_t m;
    Ctrl* ctrl;
    using Raw = uint3;
    static constexpr bool kTri = kTripartite;
    __device__ Raw fetch(uint64_t i) const { return make_uint3(edges[3 * i], edges[3 * i + 1], edges[3 * i + 2]); }
    __device__ void vertices(uint64_t, Raw t, uint32_t (&v)[3]) const
    {
        v[0] = t.x;
        v[1] = t.y;
        v[2] = t.z;
        if (!kTri && bad_edge(t.x, t.y, t.z, m)) {
            atomicOr(&ctrl->err, kErrBadEdge);
            v[0] = v[1] = v[2] = kNoVertex;
        }
    }
};

// Bound by its passes over LDS at 10^6 keys, by memory at 10^7.
// One tile of kBlock * kPer edges, position by position (with kTri position k's vertices lie in
// part k, which is a third of the buckets): counted per bucket, a run reserved in each bucket,
// ordered in LDS, written out.
template <uint32_t kBlock, uint32_t kPer, class Src>
__global__ __launch_bounds__(kBlock) void k_bins(Src src, BinArgs a, uint32_t width)
{
    constexpr uint32_t kTile = kBlock * kPer;
    extern __shared__ uint2 s_bins[];
    uint2* const buf = s_bins;
    uint32_t* const lst = reinterpret_cast<uint32_t*>(buf + kTile);  // width + 1: counts, then their prefix
    uint32_t* const delta = lst + width + 1;                         // run's place in its bucket - place in buf
    __shared__ uint32_t wtot[kBlock / kWave];
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const uint64_t t0 = (uint64_t)blockIdx.x * kTile;
    uint32_t v[kPer][3];
    {
        typename Src::Raw x[kPer];
#pragma unroll
        for (uint32_t q = 0; q < kPer; q++)
            x[q] = src.fetch(min<uint64_t>(t0 + q * kBlock + tid, a.n - 1));
#pragma unroll
        for (uint32_t q = 0; q < kPer; q++) {
            const uint64_t i = t0 + q * kBlock + tid;
            v[q][0] = v[q][1] = v[q][2] = kNoVertex;
            if (i < a.n)
                src.vertices(i, x[q], v[q]);
        }
    }
#pragma unroll
    for (uint32_t k = 0; k < 3; k++) {
        const uint32_t b0 = Src::kTri ? (uint32_t)((k * a.P) >> a.shift) : 0u;
        for (uint32_t j = tid; j <= width; j += kBlock)
            lst[j] = 0;
        __syncthreads();
        uint32_t rk[kPer];
#pragma unroll
        for (uint32_t q = 0; q < kPer; q++)
            if (v[q][k] != kNoVertex)
                rk[q] = atomicAdd(&lst[(v[q][k] >> a.shift) - b0], 1u);
        __syncthreads();
        // exclusive prefix in place, a row of consecutive buckets per thread
        const uint32_t row = (width + kBlock) / kBlock;
        const uint32_t j0 = min(tid * row, width + 1), j1 = min(j0 + row, width + 1);
        uint32_t sum = 0;
        for (uint32_t j = j0; j < j1; j++)
            sum += lst[j];
        uint32_t incl = sum;
        for (uint32_t d = 1; d < kWave; d <<= 1) {
            const uint32_t y = __shfl_up(incl, d, kWave);
            if (lane >= d)
                incl += y;
        }
        if (lane == kWave - 1)
            wtot[wv] = incl;
        __syncthreads();
        uint32_t run = incl - sum;
        for (uint32_t q = 0; q < wv; q++)
            run += wtot[q];
        for (uint32_t j = j0; j < j1; j++) {
            const uint32_t c = lst[j];
            lst[j] = run;
            run += c;
        }
        __syncthreads();
#pragma unroll 4
        for (uint32_t j = tid; j < width; j += kBlock) {
            const uint32_t c = lst[j + 1] - lst[j];
            if (c) {
                const uint32_t at = atomicAdd(&a.cursor[b0 + j], c);
                delta[j] = at - lst[j];
                if (at + c > a.length(b0 + j) + a.extra)
                    *a.full = 1;
            }
        }
#pragma unroll
        for (uint32_t q = 0; q < kPer; q++)
            if (v[q][k] != kNoVertex)
                buf[lst[(v[q][k] >> a.shift) - b0] + rk[q]] = make_uint2(v[q][k], (uint32_t)(t0 + q * kBlock + tid));
        __syncthreads();
        const uint32_t total = lst[width];
        for (uint32_t s = tid; s < total; s += kBlock) {
            const uint2 x = buf[s];
            const uint32_t b = x.x >> a.shift, j = s + delta[b - b0];
            const uint32_t len = a.length(b);
            if (j < len)
                reinterpret_cast<uint2*>(a.rec)[((uint64_t)b << a.shift) + j] = x;
            else if (j - len < a.extra)
                a.more[(uint64_t)b * a.extra + (j - len)] = x;
        }
        __syncthreads();
    }
}

// The records of bucket b are final in rec: writes its bit per degree-1 vertex and its counts
// (degrees in total, vertices of degree 1).  record(v) yields a vertex's record.
template <class Record>
__device__ __forceinline__ void bucket_summary(const BinArgs& a, uint32_t b, uint64_t* __restrict__ ones,
                                               uint2* __restrict__ sums, Ctrl* ctrl, Record record, uint32_t* s_sum)
{
    const uint64_t lo = (uint64_t)b << a.shift;
    const uint32_t len = a.length(b), size = 1u << a.shift;
    if (threadIdx.x < 2)
        s_sum[threadIdx.x] = 0;
    __syncthreads();
    uint32_t deg = 0, one = 0;
    for (uint32_t j = threadIdx.x; j < size; j += kBinAccBlock) {  // size >= 64: whole waves
        const uint64_t x = j < len ? record(j) : 0ull;
        const uint32_t d = Rec::deg(x);
        if (d > kMaxDegree)
            atomicOr(&ctrl->err, kErrDegree);
        deg += d;
        const bool is = d == 1 && Rec::edge(x) < a.n;
        const uint64_t mask = __ballot(is);
        one += is;
        if ((threadIdx.x & (kWave - 1)) == 0 && j < len)
            ones[(lo + j) / 64] = mask;
    }
    for (uint32_t d = kWave / 2; d > 0; d >>= 1) {
        deg += __shfl_xor(deg, d, kWave);
        one += __shfl_xor(one, d, kWave);
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        atomicAdd(&s_sum[0], deg);
        atomicAdd(&s_sum[1], one);
    }
    __syncthreads();
    if (threadIdx.x == 0)
        sums[b] = make_uint2(s_sum[0], s_sum[1]);
}

// One bucket's records from its bin, which they replace.
__global__ __launch_bounds__(kBinAccBlock) void k_bins_accum(BinArgs a, uint64_t* __restrict__ ones,
                                                             uint2* __restrict__ sums, Ctrl* ctrl)
{
    extern __shared__ unsigned long long s_rec[];
    __shared__ uint32_t s_sum[2];
    constexpr uint32_t kAhead = 8;
    if (*a.full)
        return;
    const uint32_t b = blockIdx.x, size = 1u << a.shift, mask = size - 1;
    const uint64_t lo = (uint64_t)b << a.shift;
    const uint32_t len = a.length(b), c = a.cursor[b];
    const uint2* const in = reinterpret_cast<const uint2*>(a.rec) + lo;
    const uint2* const more = a.more + (uint64_t)b * a.extra;
    for (uint32_t j = threadIdx.x; j < size; j += kBinAccBlock)
        s_rec[j] = 0;
    __syncthreads();
    for (uint32_t i0 = threadIdx.x; i0 < c; i0 += kAhead * kBinAccBlock) {
        uint2 x[kAhead];
#pragma unroll
        for (uint32_t q = 0; q < kAhead; q++) {
            const uint32_t i = min(i0 + q * kBinAccBlock, c - 1);
            x[q] = i < len ? in[i] : more[i - len];
        }
#pragma unroll
        for (uint32_t q = 0; q < kAhead; q++)
            if (i0 + q * kBinAccBlock < c)
                atomicAdd(&s_rec[x[q].x & mask], (unsigned long long)(Rec::kOne + x[q].y));
    }
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < len; j += kBinAccBlock)
        a.rec[lo + j] = s_rec[j];
    bucket_summary(a, b, ones, sums, ctrl, [&](uint32_t j) { return s_rec[j]; }, s_sum);
}

// The edge states, whose memory held incidences until now.  After an overflow also the records from
// the edges, with device atomics, and the buckets' summaries.
__global__ __launch_bounds__(kBinAccBlock) void k_bins_again(BinArgs a, const uint32_t* __restrict__ edges,
                                                             uint64_t* __restrict__ ones, uint2* __restrict__ sums,
                                                             uint32_t* __restrict__ state, Ctrl* ctrl,
                                                             GridSync* sync, uint32_t wait)
{
    __shared__ uint32_t s_join[3], s_sum[2];
    __shared__ uint64_t s_total;
    for (uint64_t i = (uint64_t)blockIdx.x * kBinAccBlock + threadIdx.x; i < a.n; i += (uint64_t)gridDim.x * kBinAccBlock)
        state[i] = kUnclaimed;
    if (*a.full == 0)
        return;
    Grid g;
    if (!grid_join<true>(sync, g, s_join, wait))
        return;
    // the records cleared, the edges added, the buckets summed up; a group that is not whole goes
    // through each in spans, with a chance to grow behind each
    uint32_t stage = 0;
    uint64_t pos = 0;
    if (g.phase) {
        stage = (uint32_t)ag_load(&g.s->run[0]);
        pos = ag_load(&g.s->run[1]);
    }
    while (stage < 3) {
        const uint64_t total = stage == 0 ? a.m : (stage == 1 ? a.n : a.nb);
        const uint64_t stride = (uint64_t)g.members * (stage < 2 ? kBinAccBlock : 1u);
        const uint64_t first = stage < 2 ? (uint64_t)g.rank * kBinAccBlock + threadIdx.x : g.rank;
        const uint64_t to = g.whole() ? total : min(total, pos + stride * (stage < 2 ? kGridSpan : 1u));
        if (stage == 0) {
            for (uint64_t v = pos + first; v < to; v += stride)
                ag_store(a.rec + v, (uint64_t)0);
        } else if (stage == 1) {
            for (uint64_t e = pos + first; e < to; e += stride) {
                const uint32_t x = edges[3 * e], y = edges[3 * e + 1], z = edges[3 * e + 2];
                if (bad_edge(x, y, z, a.m))
                    continue;  // reported by k_bins
                Rec::add(a.rec, x, (uint32_t)e);
                Rec::add(a.rec, y, (uint32_t)e);
                Rec::add(a.rec, z, (uint32_t)e);
            }
        } else {
            for (uint64_t b = pos + first; b < to; b += stride) {
                const uint64_t* const rec = a.rec + (b << a.shift);
                bucket_summary(a, (uint32_t)b, ones, sums, ctrl, [&](uint32_t j) { return ag_load(rec + j); }, s_sum);
                __syncthreads();
            }
        }
        pos = to;
        if (to == total) {
            stage++;
            pos = 0;
        }
        grid_barrier<true>(g, &s_total);
        if (g.grew && g.rank == 0 && threadIdx.x == 0)
            grid_admit(g, stage, pos);
    }
    if (g.rank == 0 && threadIdx.x == 0)
        grid_done(g);
}

// Round 0: the hinges of layer 0 write their edges' states and append the edges.  Block 0 also adds
// up the summaries.
template <bool kTri>
__global__ __launch_bounds__(kBinRound0Block) void k_bins_round0(BinArgs a, const uint32_t* __restrict__ edges,
                                                     const uint64_t* __restrict__ ones, const uint2* __restrict__ sums,
                                                     uint32_t* __restrict__ state, uint3* __restrict__ slots,
                                                     unsigned long long* __restrict__ layer, Ctrl* ctrl)
{
    constexpr uint32_t kWaves = kBinRound0Block / kWave, kPer = kBinRound0Per;
    static_assert(kPer * kWaves == kWave, "one count per lane of a wave");
    __shared__ uint32_t s_count[kPer * kWaves];
    __shared__ unsigned long long s_base, s_deg, s_one;
    const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const uint32_t* const bits = reinterpret_cast<const uint32_t*>(ones);
    auto alone = [&](uint32_t v) { return v < a.m && (bits[v / 32] >> (v & 31) & 1u); };
    if (tid == 0)
        s_deg = s_one = 0;
    const uint64_t v0 = (uint64_t)blockIdx.x * (kBinRound0Block * kPer) + tid;
    uint64_t x[kPer];
#pragma unroll
    for (uint32_t q = 0; q < kPer; q++)
        x[q] = a.rec[min<uint64_t>(v0 + q * kBinRound0Block, a.m - 1)];
    uint32_t e[kPer], t[kPer][3];
    bool hinge[kPer];
#pragma unroll
    for (uint32_t q = 0; q < kPer; q++) {
        const uint64_t v = v0 + q * kBinRound0Block;
        e[q] = Rec::edge(x[q]);
        hinge[q] = v < a.m && Rec::deg(x[q]) == 1 && e[q] < a.n;
        // part 0's vertices need no look at the others
        const uint32_t* const p = edges + (hinge[q] && !(kTri && v < a.P) ? 3 * (uint64_t)e[q] : 0ull);
        t[q][0] = p[0];
        t[q][1] = p[1];
        if constexpr (!kTri)
            t[q][2] = p[2];
    }
    uint64_t mask[kPer];
#pragma unroll
    for (uint32_t q = 0; q < kPer; q++) {
        const uint32_t v = (uint32_t)(v0 + q * kBinRound0Block);
        uint32_t k;
        if constexpr (kTri)
            k = part_of(v, a.P);
        else
            k = t[q][0] == v ? 0u : t[q][1] == v ? 1u : 2u;
        if (hinge[q] && k > 0)
            hinge[q] = !alone(t[q][0]) && !(k == 2 && alone(t[q][1]));
        if (hinge[q])
            state[e[q]] = k;
        mask[q] = __ballot(hinge[q]);
        if (lane == 0)
            s_count[q * kWaves + wv] = (uint32_t)__popcll(mask[q]);
    }
    __syncthreads();
    if (tid < kWave) {
        const uint32_t c = s_count[tid];
        uint32_t incl = c;
        for (uint32_t d = 1; d < kWave; d <<= 1) {
            const uint32_t y = __shfl_up(incl, d, kWave);
            if (lane >= d)
                incl += y;
        }
        s_count[tid] = incl - c;
        if (tid == kWave - 1)
            s_base = incl ? atomicAdd(layer, (unsigned long long)incl) : 0ull;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q < kPer; q++)
        if (hinge[q])
            slots[s_base + s_count[q * kWaves + wv] + lanes_below(mask[q])].x = e[q];
    if (blockIdx.x == 0) {
        unsigned long long deg = 0, one = 0;
        for (uint32_t b = tid; b < a.nb; b += kBinRound0Block) {
            deg += sums[b].x;
            one += sums[b].y;
        }
        atomicAdd(&s_deg, deg);
        atomicAdd(&s_one, one);
        __syncthreads();
        if (tid == 0) {
            ctrl->degsum = s_deg;
            ctrl->ftail = ctrl->claims = s_one;
        }
    }
}

// ------------------------------------------------------------------------------------------
// The bins' working memory lies in the layer sizes, of which such a run uses only the first:
// the overflow flag, the buckets' cursors and sums, the bits.
static uint64_t bins_words(uint64_t m, uint32_t nb) { return 2 + (nb + 1) / 2 + nb + (m + 63) / 64; }

uint32_t bins_shift(uint64_t n, uint64_t m, uint64_t rcap)
{
    if (n < kBinMinEdges || n > kRunMaxEdges) return 0;
    for (uint32_t s = kBinMinShift; s <= kBinMaxShift; s++) {
        const uint64_t nb = (m + (1ull << s) - 1) >> s;
        if (nb > kBinMaxBuckets || bins_words(m, (uint32_t)nb) > rcap + 2) continue;
        // a bucket's incidences are 3n 2^s / m in the mean, with a standard deviation of its root
        const double mean = 3.0 * (double)n * (double)(1ull << s) / (double)m;
        if (mean + 6.0 * std::sqrt(mean) <= (double)((1ull << s) + 2 * n / nb)) return s;
    }
    return 0;
}

template <uint32_t kBlock, uint32_t kPer, class Src>
static hipError_t bins_launch(const Src& src, const BinArgs& a, uint32_t width, hipStream_t s)
{
    constexpr uint64_t kTile = (uint64_t)kBlock * kPer;
    k_bins<kBlock, kPer><<<(unsigned)((a.n + kTile - 1) / kTile), kBlock, kTile * 8 + (2 * width + 1) * 4, s>>>(src, a,
                                                                                                             width);
    return hipGetLastError();
}

template <class Src>
static hipError_t bins_scatter(const Src& src, const BinArgs& a, hipStream_t s)
{
    // buckets that one position's vertices touch
    const uint32_t width = Src::kTri ? std::min<uint32_t>(a.nb, (uint32_t)(a.P >> a.shift) + 2) : a.nb;
    if (a.n < kBinSmallTiles) return bins_launch<512, 4>(src, a, width, s);
    return bins_launch<512, 8>(src, a, width, s);
}

static BinArgs bin_args(const PeelState& st, uint32_t shift, uint2*& sums, uint64_t*& ones)
{
    BinArgs a{st.n, st.m, st.P, st.rec, nullptr, st.lcount + 1, reinterpret_cast<uint2*>(st.slots), 0, shift,
              (uint32_t)((st.m + (1ull << shift) - 1) >> shift)};
    a.extra = (uint32_t)(2 * st.n / a.nb);  // 16n bytes of slots and states
    a.cursor = reinterpret_cast<uint32_t*>(st.lcount + 2);
    sums = reinterpret_cast<uint2*>(st.lcount + 2 + (a.nb + 1) / 2);
    ones = reinterpret_cast<uint64_t*>(sums + a.nb);
    return a;
}

uint64_t bins_zero_words(uint64_t m, uint32_t shift)
{
    return 2 + (((m + (1ull << shift) - 1) >> shift) + 1) / 2;
}

hipError_t launch_bins_scatter(const PeelState& st, uint32_t shift, const uint64_t* keys, uint64_t seed, hipStream_t s)
{
    uint2* sums;
    uint64_t* ones;
    const BinArgs a = bin_args(st, shift, sums, ones);
    if (keys) return bins_scatter(BinKeys{keys, seed, st.P, const_cast<uint32_t*>(st.edges)}, a, s);
    if (st.tripartite) return bins_scatter(BinEdges<true>{st.edges, st.m, st.ctrl}, a, s);
    return bins_scatter(BinEdges<false>{st.edges, st.m, st.ctrl}, a, s);
}

hipError_t launch_bins_accum(const PeelState& st, uint32_t shift, hipStream_t s)
{
    uint2* sums;
    uint64_t* ones;
    const BinArgs a = bin_args(st, shift, sums, ones);
    k_bins_accum<<<a.nb, kBinAccBlock, 8ull << shift, s>>>(a, ones, sums, st.ctrl);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_bins_again<<<kGridMax, kBinAccBlock, 0, s>>>(a, st.edges, ones, sums, st.state, st.ctrl, st.sync + 2, st.wait);
    return hipGetLastError();
}

hipError_t launch_bins_round0(const PeelState& st, uint32_t shift, hipStream_t s)
{
    uint2* sums;
    uint64_t* ones;
    const BinArgs a = bin_args(st, shift, sums, ones);
    constexpr uint64_t kTile = kBinRound0Block * kBinRound0Per;
    const unsigned g = (unsigned)((st.m + kTile - 1) / kTile);
    if (st.tripartite)
        k_bins_round0<true><<<g, kBinRound0Block, 0, s>>>(a, st.edges, ones, sums, st.state, st.slots, st.lcount, st.ctrl);
    else
        k_bins_round0<false><<<g, kBinRound0Block, 0, s>>>(a, st.edges, ones, sums, st.state, st.slots, st.lcount, st.ctrl);
    return hipGetLastError();
}

}  // namespace mphx
