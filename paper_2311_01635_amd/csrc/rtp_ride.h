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
    int sums;
    unsigned sum_blocks;
    struct {
        const void *Y;
        int64_t ld;
        int rows, cols;
        const float *in;
        float *out;
        unsigned first;
    } sum[RIDE_MAX_SUMS];
};

// ---- bias gradient: column sums --------------------------------------------------------------
// out[c] = in[c] + sum over rows of Y[r, c].  Bound: memory latency (the matrix is [tokens, shard width], a few
// megabytes, and a shard is only some hundred columns wide).  A workgroup owns 32 columns: VEC
// columns per thread (16 bytes of a 16-bit matrix where the rows allow it), 32 / VEC threads across, the rest down the
// rows with four loads in flight for each of 1024 / (32 / VEC) row groups (a workgroup of fewer threads takes several); the row groups' sums meet in LDS in a fixed order, so the result does not
// depend on timing.  1024 tokens x 384 columns, fp16: 53 us with one 2-byte load in flight per thread and 256 threads
// on 64 columns; the training step of the unit they belong to went from 1.96 to 1.15 ms.
// Only the last trip tests its rows (a test on every read made 4096 x 100 bf16 16.4 us instead of 6.8, 8192 x 384 fp32 29.4
// instead of 22.6).
constexpr int COLSUM_COLS = 32, COLSUM_THREADS = 1024;
constexpr int COLSUM_LDS_FLOATS = 256 * COLSUM_COLS + 32 * COLSUM_COLS;

inline bool colsum_wide(const void *Y, int64_t ld, int cols) { return (ld & 7) == 0 && (cols & 7) == 0 && ((uintptr_t)Y & 15) == 0; }

template <typename T, int VEC, int NTHR>
__device__ __forceinline__ void colsum_block(const T *Y, int64_t ld, int rows, int cols, const float *in, float *out, const unsigned block, float *lds)
{
    constexpr int TX = COLSUM_COLS / VEC, GROUPS = COLSUM_THREADS / TX, UNROLL = 4, PER = COLSUM_THREADS / NTHR;
    typedef __attribute__((ext_vector_type(VEC))) T vec;
    float *part = lds;                                                                // [group][column]
    float(*part2)[COLSUM_COLS] = (float(*)[COLSUM_COLS])(lds + 256 * COLSUM_COLS);
    const int tid = threadIdx.x, x = tid % TX, g = tid / TX;
    const int c = block * COLSUM_COLS + x * VEC;
    float s[PER][VEC] = {};
    if (c < cols) { // (VEC > 1: cols is a multiple of VEC)
        const T *p = Y + c;
        int r0 = g;
        for (; r0 + (UNROLL - 1) * GROUPS + (PER - 1) * (GROUPS / PER) < rows; r0 += UNROLL * GROUPS) {
            vec v[PER][UNROLL];
#pragma unroll
            for (int h = 0; h < PER; ++h)
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) v[h][u] = *(const vec *)(p + (int64_t)(r0 + h * (GROUPS / PER) + u * GROUPS) * ld);
#pragma unroll
            for (int h = 0; h < PER; ++h)
#pragma unroll
                for (int u = 0; u < UNROLL; ++u)
#pragma unroll
                    for (int i = 0; i < VEC; ++i) s[h][i] += (float)v[h][u][i];
        }
        if (r0 < rows) { // a trip that reaches past the end reads the last row there, and does not add it
            vec v[PER][UNROLL];
#pragma unroll
            for (int h = 0; h < PER; ++h)
#pragma unroll
                for (int u = 0; u < UNROLL; ++u)
                    v[h][u] = *(const vec *)(p + (int64_t)min(r0 + h * (GROUPS / PER) + u * GROUPS, rows - 1) * ld);
#pragma unroll
            for (int h = 0; h < PER; ++h)
#pragma unroll
                for (int u = 0; u < UNROLL; ++u)
                    if (r0 + h * (GROUPS / PER) + u * GROUPS < rows)
#pragma unroll
                        for (int i = 0; i < VEC; ++i) s[h][i] += (float)v[h][u][i];
        }
    }
#pragma unroll
    for (int h = 0; h < PER; ++h)
#pragma unroll
        for (int i = 0; i < VEC; ++i) part[(g + h * (GROUPS / PER)) * COLSUM_COLS + x * VEC + i] = s[h][i];
    __syncthreads();
    // 32 sums per column, then one
    const int col = tid & 31;
#pragma unroll
    for (int h = 0; h < PER; ++h) {
        const int q = (tid >> 5) + h * (NTHR / 32);
        float t = 0.0f;
        for (int i = q; i < GROUPS; i += 32) t += part[i * COLSUM_COLS + col];
        part2[q][col] = t;
    }
    __syncthreads();
    if (tid < 32 && block * COLSUM_COLS + col < cols) {
        float sum = 0.0f;
#pragma unroll
        for (int i = 0; i < 32; ++i) sum += part2[i][col];
        const int cc = block * COLSUM_COLS + col;
        out[cc] = in[cc] + sum;
    }
}

// (wide sums only: a riding layer's widths are multiples of 8 and its operands start on 16 bytes)
template <typename E, int NTHR>
__device__ __forceinline__ void ride_sum(const RideList &g, const unsigned block, float *lds)
{
    const int i = g.sums > 1 && block >= g.sum[1].first ? 1 : 0;
    colsum_block<E, 8, NTHR>((const E *)g.sum[i].Y, g.sum[i].ld, g.sum[i].rows, g.sum[i].cols, g.sum[i].in, g.sum[i].out,
                             block - g.sum[i].first, lds);
}

// the list of a launch that has about `idle` compute units to spare for it
hipError_t ride_list(const Riders &r, int idle, RideList *out);

// Bound: memory latency (a few megabytes a launch), hence all of a thread's 16-byte reads in flight, up to eight a
// direction: eight in a workgroup of 512 threads with a piece of 64 KB, two with the smallest of 16 KB.
// The units go in runs of 8, 4 and 2 a thread without a bounds test: behind a test per unit the compiler waited for each
// read before it issued the next (512-token pass of the Llama-shaped unit 450 -> 437).
// A thread reads its units of `buf` and `in` before it writes them, so a segment may send what `buf` holds and
// receive into it in one go; no two segments touch the same bytes.  What the next launch reads is stored the plain way,
// what nobody reads soon past the caches: a 512-token pass of the Llama-shaped unit 505 -> 461 us, the query/key/value
// training step 1041 -> 1029.
// DEPTH units of a thread, NTHR apart, from `e` on: all reads, then all writes.  TAIL: units from `end` on do not exist (their
// reads go to the last one that does).
template <int NTHR, int DEPTH, bool OUT, bool IN, bool TAIL>
__device__ __forceinline__ void ride_units(ride_u32x4 *out, ride_u32x4 *buf, const ride_u32x4 *in, const int64_t e, const int64_t end)
{
    ride_u32x4 held[DEPTH], next[DEPTH];
#pragma unroll
    for (int j = 0; j < DEPTH; ++j) {
        const int64_t q = TAIL ? min(e + j * NTHR, end - 1) : e + j * NTHR;
        if (OUT) held[j] = __builtin_nontemporal_load(buf + q);
        if (IN) next[j] = __builtin_nontemporal_load(in + q);
    }
#pragma unroll
    for (int j = 0; j < DEPTH; ++j) {
        const int64_t q = e + j * NTHR;
        if (TAIL && q >= end) continue;
        if (OUT) __builtin_nontemporal_store(held[j], out + q);
        if (IN) buf[q] = next[j]; // the next launch reads it
    }
}

template <int NTHR, bool OUT, bool IN>
__device__ __forceinline__ void ride_run(ride_u32x4 *out, ride_u32x4 *buf, const ride_u32x4 *in, int64_t begin, const int64_t end)
{
    const int t = threadIdx.x;
    for (; begin + 8 * NTHR <= end; begin += 8 * NTHR) ride_units<NTHR, 8, OUT, IN, false>(out, buf, in, begin + t, end);
    if (begin + 4 * NTHR <= end) {
        ride_units<NTHR, 4, OUT, IN, false>(out, buf, in, begin + t, end);
        begin += 4 * NTHR;
    }
    if (begin + 2 * NTHR <= end) {
        ride_units<NTHR, 2, OUT, IN, false>(out, buf, in, begin + t, end);
        begin += 2 * NTHR;
    }
    if (begin < end) ride_units<NTHR, 2, OUT, IN, true>(out, buf, in, begin + t, end);
}

template <int NTHR>
__device__ __forceinline__ void ride(const RideList &g, const unsigned block)
{
    int i = 0;
    while (i + 1 < g.count && block >= g.seg[i + 1].first) ++i;
    ride_u32x4 *const out = g.seg[i].out, *const buf = g.seg[i].buf;
    const ride_u32x4 *const in = g.seg[i].in;
    const int64_t begin = (int64_t)(block - g.seg[i].first) * g.per_block;
    const int64_t end = min(begin + g.per_block, g.seg[i].n16);
    if (out && in)
        ride_run<NTHR, true, true>(out, buf, in, begin, end);
    else if (out)
        ride_run<NTHR, true, false>(out, buf, in, begin, end);
    else if (in)
        ride_run<NTHR, false, true>(out, buf, in, begin, end);
}

} // namespace rtp
