// One small MPHF build in one workgroup and one launch, retries included (lds_build.h).  Bound by
// the latency of its rounds.  u64 keys, a launch per round before and now: 10^3 keys (three seeds, one to six
// tries) 1696 and 131 us, 13,363 keys 1530 and 170; 20,011 strings 1007 and 128.
#include "launch.h"
#include "lds_build.h"

namespace mphx {

// A thread hashes a string alone, 32 bytes a step, and there is one compute unit: strings that are longer or
// more bytes than this leave the launch, and the caller has them hashed by one of their own (20 us
// of launches and host).  A build of 2048 strings of 16,000 bytes took 3350 us hashed here, 1666 with a launch per
// round; 246 so.
constexpr uint32_t kHereKey = 512, kHereBytes = 256 * 1024;

template <int kBlock, uint32_t kBytes, bool kQueueLds>
__global__ __launch_bounds__(kBlock) void k_small_build(SmallArgs a)
{
    __shared__ __align__(16) uint8_t s_lds[kBytes];
    const uint64_t total = a.keys ? 0 : a.offs[a.n];
    const uint64_t P = a.P;
    bool here = false;  // strings may be hashed here
    // u64 keys as they are; strings as their hashed edge, or as their digest
    auto slow = [&](uint64_t sd) -> int32_t {
        if (a.keys || (a.edges && sd == a.seed))
            return 0;
        if (!here) {
            bool far = total - a.offs[0] > kHereBytes;
            for (uint32_t i = threadIdx.x; i < a.n && !far; i += kBlock)
                far = a.offs[i + 1] - a.offs[i] > kHereKey;
            here = !__syncthreads_or(far);
        }
        return here ? 1 : kLdsHash;
    };
    auto fetch = [&](uint32_t i, uint64_t) -> ulonglong2 {
        if (a.keys)
            return make_ulonglong2(a.keys[i], 0);
        const uint32_t* t = a.edges + 3 * (uint64_t)i;
        return make_ulonglong2(t[0] | (uint64_t)t[1] << 32, t[2]);
    };
    auto digest = [&](uint32_t i, uint64_t sd) -> ulonglong2 {
        const uint64_t o0 = a.offs[i], o1 = a.offs[i + 1];
        uint64_t x, y;
        digest_str(a.bytes, o0, o1 - o0, total, fin(sd + kGamma), fin(sd + 2 * kGamma), x, y);
        return make_ulonglong2(x, y);
    };
    auto locals = [&](ulonglong2 key, uint64_t sd) -> uint3 {
        uint64_t x = key.x, y = key.y;
        if (a.keys)
            x = y = key.x ^ sd;
        else if (a.edges && sd == a.seed)
            return make_uint3((uint32_t)x, (uint32_t)(x >> 32) - a.P, (uint32_t)y - 2 * a.P);
        return make_uint3((uint32_t)range_reduce(fin(x + kGamma), P), (uint32_t)range_reduce(fin(x + 2 * kGamma), P),
                          (uint32_t)range_reduce(fin(y + 3 * kGamma), P));
    };
    const LdsOutcome out = lds_build<kBlock, kQueueLds, 4>(a.n, a.P, a.seed, a.max_tries, slow, fetch, digest, locals,
                                                           s_lds, a.queue, a.start, a.codes, a.rank);
    if (threadIdx.x == 0)
        *a.out = out;
}

// Up to 7 bytes of LDS per vertex with the queue in LDS, 5 without.  256 threads while a
// round's queue (a quarter of the vertices at most, in practice) is a few waves: their barriers cost
// less than those of 1024.
constexpr uint32_t kSmallBytes = 24 * 1024, kLargeBytes = 158 * 1024;

bool small_build_fits(uint64_t n, uint64_t m)
{
    return n < 0xFFFFFFFFull && m <= kLdsMaxVertices && lds_build_bytes((uint32_t)m, false) <= kLargeBytes;
}

hipError_t launch_small_build(const SmallArgs& a, hipStream_t s)
{
    const uint32_t m = 3 * a.P;
    if (!small_build_fits(a.n, m)) return hipErrorInvalidValue;
    if (lds_build_bytes(m, true) <= kSmallBytes)
        k_small_build<256, kSmallBytes, true><<<1, 256, 0, s>>>(a);
    else if (lds_build_bytes(m, true) <= kLargeBytes)
        k_small_build<1024, kLargeBytes, true><<<1, 1024, 0, s>>>(a);
    else
        k_small_build<1024, kLargeBytes, false><<<1, 1024, 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace mphx
