// Shard transfers that ride in a GEMM's launch: workgroups behind the tiles of the grid move them.
//
// A narrow shard's step is a GEMM of 10-40 us and transfers of 5-10 us.  As launches of their own on a second stream
// the transfers cost the host a launch and two or three cross-stream waits (9 us each), and the queue about 10 us a
// wait; riding, they cost neither, and the compute units the GEMM's few tiles leave idle carry them.
#pragma once
#include "rtp_kernels.h"

namespace rtp {

typedef __attribute__((ext_vector_type(4))) unsigned int ride_u32x4;

struct RideList {
    int count;
    unsigned blocks;   // workgroups of the whole list
    int per_block;     // 16-byte units a workgroup moves
    struct {
        ride_u32x4 *out, *buf;
        const ride_u32x4 *in;
        int64_t n16;
        unsigned first; // workgroup the segment starts at
    } seg[RIDE_MAX_SEGS];
};

// the list of a launch that has about `idle` compute units to spare for it
hipError_t ride_list(const Riders &r, int idle, RideList *out);

// Bound: memory latency (a few megabytes a launch), hence eight 16-byte reads in flight per thread and direction.
// A thread reads its units of `buf` and `in` before it writes any, so a segment may send what `buf` holds and
// receive into it in one go; no two segments touch the same bytes.
template <int NTHR>
__device__ __forceinline__ void ride(const RideList &g, const unsigned block)
{
    constexpr int DEPTH = 8;
    int i = 0;
    while (i + 1 < g.count && block >= g.seg[i + 1].first) ++i;
    ride_u32x4 *const out = g.seg[i].out, *const buf = g.seg[i].buf;
    const ride_u32x4 *const in = g.seg[i].in;
    const int64_t begin = (int64_t)(block - g.seg[i].first) * g.per_block;
    const int64_t end = min(begin + g.per_block, g.seg[i].n16);
    for (int64_t e0 = begin + threadIdx.x; e0 < end; e0 += NTHR * DEPTH) {
        ride_u32x4 held[DEPTH], next[DEPTH];
#pragma unroll
        for (int j = 0; j < DEPTH; ++j) {
            const int64_t e = e0 + j * NTHR;
            if (e < end && out) held[j] = __builtin_nontemporal_load(buf + e);
            if (e < end && in) next[j] = __builtin_nontemporal_load(in + e);
        }
#pragma unroll
        for (int j = 0; j < DEPTH; ++j) {
            const int64_t e = e0 + j * NTHR;
            if (e < end && out) __builtin_nontemporal_store(held[j], out + e);
            if (e < end && in) __builtin_nontemporal_store(next[j], buf + e);
        }
    }
}

} // namespace rtp
