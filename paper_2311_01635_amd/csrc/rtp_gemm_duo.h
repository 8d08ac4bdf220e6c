// The partition GEMM for launches of few or short tiles (a prompt, narrow shards, short contractions): workgroups of four
// waves with half of a compute unit's LDS, so that two share one, on tiles of 128 x 128, 64 x 128 or 64 x 64 of C.
//
// Bound: the load path from L2 into LDS, about 27 cycles a load instruction of whole 128-byte lines and a compute unit, and
// the fixed cost of a tile.  Hence
//  * small tiles, so that a shard's GEMM reaches more compute units: the time of a launch that does not fill the machine is
//    that of the bytes one unit fetches.  us a launch, tall or 64 x 128 tile of gemm_pp_kernel -> here: 512 x 2048 x 1024 `+=`
//    12.9 -> 8.8 (64 x 64); 5696 x 512 over 1344 tokens 23.0 -> 19.4 (64 x 128); 1833 x 3904 x 768 `+=` 24.4 -> 22.8 and
//    4869 x 1152 x 4096 60.5 -> 56.1 (128 x 128);
//  * two workgroups a unit: one's prologue and epilogue run under the other's products.  Launches that keep every unit
//    multiplying for long are the tall tiles' (4096^3 109 us, here 126);
//  * sub-tiles of 64 K, whose K-contiguous rows are whole lines (of 32: 149 us for that product).  Weight gradients in
//    128 x 128 tiles have rows of two lines either way and take 32, five in flight instead of two (4096 x 688 over 1990 tokens
//    31.9 -> 25.4 us).
// All four waves fetch and multiply: an element is summed by one wave in the order of K with the MFMA of the tall tiles, and
// has their bits.  LDS layouts and fragment reads are those of rtp_gemm_small.h (32-deep ones in M- or N-contiguous form only).
// One barrier a sub-tile: behind it the next sub-tile has landed for everybody and the stage of the current one, whose
// fragments are in registers, is free for the loads of a later one.
// Lanes past K get an offset beyond the operand's descriptor and read as zeros without touching memory.
// Riding transfers go behind the tiles: ahead of them, or dealt among them, the ragged Llama-shaped step took 3368 instead of
// 3172 us.
#pragma once
#include "rtp_gemm_pp.h"

namespace rtp {

namespace ppd {
constexpr int NTHR = 256, WM = 2, WN = 2;
constexpr int SMEM_BYTES = 80 * 1024; // half of a compute unit's LDS
// depth of a sub-tile: see above
constexpr int sub_tile(int lay, int bm) { return lay == LAY_TN && bm == 128 ? 32 : 64; }
} // namespace ppd

template <int LAY, int FM, int FN, typename E>
__device__ __forceinline__ void duo_tile(const GemmArgs &p, const int tiles_m, const int tiles_n, const int pid,
                                         const int kt_begin, const int kt_count, char *smem)
{
    using namespace ppd;
    typedef __attribute__((address_space(3))) void *lds_vp;
    typedef typename ElemVec<E>::v8 frag8;
    constexpr bool A_KC = (LAY != LAY_TN), B_KC = (LAY == LAY_NT);
    constexpr int BM = FM * WM * 32, BN = FN * WN * 32, BK = sub_tile(LAY, BM), KS = BK / 16;
    constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE = A_BYTES + B_BYTES;
    constexpr int STAGES = SMEM_BYTES / STAGE < 8 ? SMEM_BYTES / STAGE : 8;
    constexpr int A_LOADS = A_BYTES / 4096, B_LOADS = B_BYTES / 4096, LOADS = A_LOADS + B_LOADS; // per wave and sub-tile
    static_assert((STAGES - 1) * LOADS < 64, "vmcnt is a 6-bit counter");
    static_assert(4 * (EPI_LDS_BYTES_PER_WAVE + EPI_LAND_BYTES_PER_WAVE) <= SMEM_BYTES, "the epilogue fits");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    constexpr int GROUP_M = 8;
    const int group_sz = GROUP_M * tiles_n;
    const int first_m = pid / group_sz * GROUP_M;
    const int gm = min(tiles_m - first_m, GROUP_M);
    const int tm = first_m + (pid % group_sz) % gm, tn = (pid % group_sz) / gm;
    const bool paired = FN == 2 && p.epi == EPI_SWIGLU_FWD;
    const int m0 = tm * BM, n0 = paired ? tn * (BN / 2) : tn * BN;
    const int M = p.M, N = p.N, K = p.K, half = p.half;

    // ---- direct loads: this lane's byte offsets in sub-tile 0 and its K indices there
    // K-contiguous: a 1 KB piece is 8 rows of 128 bytes; else 512 / width K-rows
    unsigned oa[A_LOADS], ob[B_LOADS];
    constexpr int A_KPP = 512 / BM, B_KPP = 512 / BN; // K-rows of a piece
    int ka[A_LOADS], kb[B_LOADS];
#pragma unroll
    for (int i = 0; i < A_LOADS; ++i) {
        const int j = A_LOADS * wave + i;
        if (A_KC) {
            const int row = 8 * j + (lane >> 3);
            ka[i] = ((lane & 7) ^ ((row >> 1) & 7)) * 8;
            oa[i] = (unsigned)(((int64_t)min(m0 + row, M - 1) * p.lda + ka[i]) * 2);
        } else {
            const int kr = A_KPP * j + lane / (BM / 8), pc = lane % (BM / 8);
            const int c = BM == 128 ? pc ^ (4 * (kr & 3)) : pc ^ (4 * ((kr >> 1) & 1));
            ka[i] = kr;
            oa[i] = (unsigned)(((int64_t)kr * p.lda + min(m0 + c * 8, M - 8)) * 2);
        }
    }
#pragma unroll
    for (int i = 0; i < B_LOADS; ++i) {
        const int j = B_LOADS * wave + i;
        if (B_KC) {
            const int r = 8 * j + (lane >> 3);
            const int row = paired ? (r < BN / 2 ? min(n0 + r, half - 1) : half + min(n0 + r - BN / 2, half - 1)) : min(n0 + r, N - 1);
            kb[i] = ((lane & 7) ^ ((r >> 1) & 7)) * 8;
            ob[i] = (unsigned)(((int64_t)row * p.ldb + kb[i]) * 2);
        } else {
            const int kr = B_KPP * j + lane / (BN / 8), pc = lane % (BN / 8);
            const int c = BN == 128 ? pc ^ (4 * (kr & 3)) : pc ^ (4 * ((kr >> 1) & 1));
            kb[i] = kr;
            ob[i] = (unsigned)(((int64_t)kr * p.ldb + min(n0 + c * 8, N - 8)) * 2);
        }
    }
    // (byte ranges below 2^31: the launcher has checked)
    const unsigned a_bytes = __builtin_amdgcn_readfirstlane(((unsigned)((A_KC ? M : K) - 1) * (unsigned)p.lda + (unsigned)(A_KC ? K : M)) * 2u);
    const unsigned b_bytes = __builtin_amdgcn_readfirstlane(((unsigned)((B_KC ? N : K) - 1) * (unsigned)p.ldb + (unsigned)(B_KC ? K : N)) * 2u);
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc((void *)p.A, 0, a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void *)p.B, 0, b_bytes, 0x00020000);
    const int stepA = A_KC ? BK * 2 : (int)(BK * p.lda * 2);
    const int stepB = B_KC ? BK * 2 : (int)(BK * p.ldb * 2);
    const int k_end = min(K, (kt_begin + kt_count) * BK);
    const int whole = __builtin_amdgcn_readfirstlane((k_end - kt_begin * BK) / BK); // sub-tiles not cut short by K
    constexpr unsigned PAST = 0x80000000u; // beyond every operand's byte range: reads as zero without touching memory

    auto issue = [&](const int kt, const int stage) {
        const int kk = kt_begin + kt;
        char *st = smem + stage * STAGE;
        if (kt < whole) {
#pragma unroll
            for (int i = 0; i < A_LOADS; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_vp)(st + (A_LOADS * wave + i) * 1024), 16, oa[i], kk * stepA, 0, 0);
#pragma unroll
            for (int i = 0; i < B_LOADS; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_vp)(st + A_BYTES + (B_LOADS * wave + i) * 1024), 16, ob[i], kk * stepB, 0, 0);
        } else {
#pragma unroll
            for (int i = 0; i < A_LOADS; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_vp)(st + (A_LOADS * wave + i) * 1024), 16,
                                                         kk * BK + ka[i] < k_end ? oa[i] + (unsigned)(kk * stepA) : PAST, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < B_LOADS; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_vp)(st + A_BYTES + (B_LOADS * wave + i) * 1024), 16,
                                                         kk * BK + kb[i] < k_end ? ob[i] + (unsigned)(kk * stepB) : PAST, 0, 0, 0);
        }
    };

    // ---- fragment addresses (LDS byte offsets in stage 0)
    const unsigned smem_lds = (unsigned)(uintptr_t)(__attribute__((address_space(3))) const char *)smem;
    const int q = lane >> 4, i16 = lane & 15;
    unsigned fa[FM], fb[FN];
    auto mc_off = [&](const int rb, const int width) {
        const int col = rb + (q & 1) * 16 + (i16 & 3) * 4, kr = (q >> 1) * 8 + (i16 >> 2);
        return (unsigned)(kr * width * 2 + (((col >> 3) ^ (width == 128 ? 4 * (kr & 3) : 4 * ((kr >> 1) & 1))) << 4) + (col & 7) * 2);
    };
    auto kc_off = [&](const int rb) {
        const int row = rb + (lane & 31);
        return (unsigned)(row * 128 + (((lane >> 5) ^ ((row >> 1) & 7)) << 4));
    };
#pragma unroll
    for (int f = 0; f < FM; ++f) fa[f] = A_KC ? kc_off(wm * FM * 32 + f * 32) : mc_off(wm * FM * 32 + f * 32, BM);
#pragma unroll
    for (int f = 0; f < FN; ++f) fb[f] = B_KC ? kc_off(f * WN * 32 + wn * 32) : mc_off(f * WN * 32 + wn * 32, BN);
    struct Frags {
        frag8 a[KS][FM], b[KS][FN];
    };
    auto read = [&](const int stage, Frags &f) {
        const unsigned so = stage * STAGE;
        auto one = [&](auto ks_) {
            constexpr int ks = decltype(ks_)::value;
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                if (A_KC)
                    f.a[ks][i] = *(const frag8 *)(smem + so + (fa[i] ^ (ks << 5)));
                else
                    f.a[ks][i] = frag_mc_read<frag8, ks, BM * 2>(smem_lds + so + fa[i]);
            }
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                if (B_KC)
                    f.b[ks][j] = *(const frag8 *)(smem + so + A_BYTES + (fb[j] ^ (ks << 5)));
                else
                    f.b[ks][j] = frag_mc_read<frag8, ks, BN * 2>(smem_lds + so + A_BYTES + fb[j]);
            }
        };
        one(std::integral_constant<int, 0>{});
        one(std::integral_constant<int, 1>{});
        if constexpr (KS == 4) {
            one(std::integral_constant<int, 2>{});
            one(std::integral_constant<int, 3>{});
        }
    };
    f32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    auto multiply = [&](const Frags &f) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] = mfma_32x32x16(f.a[ks][i], f.b[ks][j], acc[i][j]);
    };
    auto in_registers = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    int st = 0; // stage of sub-tile kt
    int kt = 0;
    Frags f0, f1;
    // sub-tile kt is in registers; behind the barrier its stage is free and sub-tile kt + 1 may be read
    auto next = [&](Frags &cur, Frags &nxt) {
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((STAGES - 2) * LOADS) : "memory");
        __builtin_amdgcn_sched_barrier(0);
        const int freed = st;
        st = st + 1 == STAGES ? 0 : st + 1;
        read(st, nxt);
        issue(kt + STAGES, freed);
        __builtin_amdgcn_sched_barrier(0);
        ++kt;
        multiply(cur);
        in_registers();
    };
#pragma unroll
    for (int i = 0; i < STAGES; ++i) issue(i, i);
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((STAGES - 1) * LOADS) : "memory");
    read(0, f0);
    in_registers();
    const int steps = kt_count & ~1;
    while (kt < steps) {
        next(f0, f1);
        next(f1, f0);
    }
    if (kt_count & 1) multiply(f0);
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory"); // what was issued past the end has landed; LDS is free
    gemm_epilogue_staged<E, FM, FN, WN * 32>(p, acc, (float *)(smem + wave * EPI_LDS_BYTES_PER_WAVE), m0 + wm * FM * 32, n0, wn * 32, lane,
                                             smem + 4 * EPI_LDS_BYTES_PER_WAVE + wave * EPI_LAND_BYTES_PER_WAVE);
}

template <int LAY, typename E>
__device__ __forceinline__ void duo_any_tile(const PpProblem &P, const int pid, const int kt_begin, const int kt_count, char *smem)
{
    if (P.bm == 128)
        duo_tile<LAY, 2, 2, E>(P.a, P.tiles_m, P.tiles_n, pid, kt_begin, kt_count, smem);
    else if (P.bn == 128)
        duo_tile<LAY, 1, 2, E>(P.a, P.tiles_m, P.tiles_n, pid, kt_begin, kt_count, smem);
    else
        duo_tile<LAY, 1, 1, E>(P.a, P.tiles_m, P.tiles_n, pid, kt_begin, kt_count, smem);
}

template <int LAY, typename E>
__global__ __launch_bounds__(ppd::NTHR, 2) void gemm_duo_kernel(const PpGroup g)
{
    __shared__ __attribute__((aligned(1024))) char smem[ppd::SMEM_BYTES];
    unsigned b = blockIdx.x;
    if constexpr (takes_sums(LAY)) {
        if (b < g.sum_blocks) {
            if (b < g.ride.sum_blocks) ride_sum<E, ppd::NTHR>(g.ride, b, (float *)smem);
            return;
        }
        b -= g.sum_blocks;
    }
    if (b >= g.tile_blocks) {
        ride<ppd::NTHR>(g.ride, b - g.tile_blocks);
        return;
    }
    int q, pid, kt_begin, kt_count;
    if (!pp_find_tile(g, b, [](const PpProblem &P) { return ppd::sub_tile(P.lay, P.bm); }, q, pid, kt_begin, kt_count)) return;
    const PpProblem &P = g.p[q];
    if constexpr (LAY != LAY_NN_TN)
        duo_any_tile<LAY, E>(P, pid, kt_begin, kt_count, smem);
    else if (P.lay == LAY_NN)
        duo_any_tile<LAY_NN, E>(P, pid, kt_begin, kt_count, smem);
    else
        duo_any_tile<LAY_TN, E>(P, pid, kt_begin, kt_count, smem);
}

template <int LAY, typename E>
static hipError_t launch_gemm_duo_layout(const PpGroup &g, hipStream_t s)
{
    const unsigned blocks = g.sum_blocks + g.tile_blocks + g.ride.blocks;
    hipLaunchKernelGGL((gemm_duo_kernel<LAY, E>), dim3(blocks), dim3(ppd::NTHR), 0, s, g);
    return hipGetLastError();
}

} // namespace rtp
