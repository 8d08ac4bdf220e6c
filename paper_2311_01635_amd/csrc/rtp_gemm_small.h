// The small tiles of the partition GEMM: 64 x 128 or 128 x 128 of C per workgroup of 8 waves, for problems too short of rows
// or columns to give every compute unit a 128 x 256 tile (a prompt of some hundred tokens, a shard a few hundred units wide).
// They run inside gemm_pp_kernel, so a launch may mix them with the tall tiles.
//
// Bound: the latency of the operand fetch (a tile contracts over all of K alone: K / 64 dependent steps), then the
// L2 -> LDS path (24 KB per step for 256 cycles of MFMA).  Hence
//  * sub-tiles of 64 K, five LDS stages (120 or 160 KB), four of them in flight: twice the bytes in flight per flop of the
//    tall tile's ring;
//  * waves 4-7 fetch, waves 0-3, one per SIMD, multiply: a 2 x 2 grid of 32 x 64 (64 x 64) wave tiles with the tall tile's
//    fragment shape (three LDS reads feed two MFMAs), to which the epilogues apply unchanged.  An element is summed
//    by one wave in the order of K, so its bits are those of the tall tiles, whichever the planner picks;
//  * fragments of sub-tile t + 1 are read while the MFMAs of sub-tile t run; one barrier per sub-tile.
// us per launch, as a layer's step runs them: all eight waves fetching and multiplying, each one half of a sub-tile's K
// (two sums per element, joined at the end), 200 x 768 x 2048 13.3, 512 x 2752 x 4096 23.5, 1024 x 384 x 768 8.1,
// 2048 x 1792 x 8192 84.5; eight waves of one 32 x 32 fragment each 14.2, 24.9, 8.3, 91.9; this split 11.1, 21.0,
// 7.2, 75.2.
// The 128 x 128 tile fetches a third more bytes a step than the 64 x 128 one for twice the products, and the load path is
// paid by the line: its lines are whole where those of the 128 x 256 tile (32 K) are halves.  Kernel us, best of the others -> this
// one: 1990 x 1376 x 4096 38.5 -> 27.7, 4096 x 688 over 1990 tokens 22.4 -> 18.4, where it is one round of the machine; past
// that it loses (8192 x 768 x 2048 29.2 -> 34, 4096^3 103 -> 137).  Its fragments are read half a sub-tile ahead, which keeps them
// in registers beside twice the accumulators.
// LDS layout: K-contiguous operands as 128-byte rows with the 16-byte chunk index xor-ed with (row/2)%8, M- or
// N-contiguous ones as K-rows of 128 (A) or 256 bytes (B) with the chunk index xor-ed with 4*((k/2)%2) or 4*(k%4):
// every fragment read then touches each of the 64 banks once per half-wave.
// Lanes past K (a partial last sub-tile, or a sub-tile past the end) get an offset beyond the operand's descriptor
// and read as zeros without touching memory.
#pragma once
#include "rtp_gemm_epilogue.h"
#include <type_traits>

namespace rtp {

namespace pps {
constexpr int BN = 128, BK = 64;
constexpr int WM = 2, WN = 2, FN = 2;
constexpr int STAGES = 5;
constexpr int ring_bytes(int fm) { return STAGES * (fm * WM * 32 + BN) * BK * 2; }
constexpr int RING_BYTES = ring_bytes(2);
constexpr int EPI_BYTES = 4 * (EPI_LDS_BYTES_PER_WAVE + EPI_LAND_BYTES_PER_WAVE); // after the ring: four waves' staged epilogue
} // namespace pps

// FM: 32-row fragments of a wave, 1 (64 x 128) or 2 (128 x 128)
template <int LAY, int FM, typename E, bool WIDE_ONLY>
__device__ __forceinline__ void pp_small_tile(const GemmArgs &p, const int tiles_m, const int tiles_n, const int vec_epilogue,
                                              const int pid, const int kt_begin, const int kt_count, char *smem)
{
    using namespace pps;
    typedef __attribute__((address_space(3))) void *lds_vp;
    typedef typename ElemVec<E>::v8 frag8;
    constexpr bool A_KC = (LAY != LAY_TN), B_KC = (LAY == LAY_NT);
    constexpr int BM = FM * WM * 32, A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE = A_BYTES + B_BYTES;
    constexpr int A_LOADS = 2 * FM, LOADS = A_LOADS + 4; // direct loads per fetching wave and sub-tile: 2 or 4 KB of A, 4 KB of B
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave >> 1) & 1, wn = wave & 1; // place of a multiplying wave in the 2 x 2 grid

    constexpr int GROUP_M = 4; // 4-tall column strips, as the tall tiles
    const int group_sz = GROUP_M * tiles_n;
    const int first_m = pid / group_sz * GROUP_M;
    const int gm = min(tiles_m - first_m, GROUP_M);
    const int tm = first_m + (pid % group_sz) % gm, tn = (pid % group_sz) / gm;
    const bool paired = (p.epi == EPI_SWIGLU_FWD);
    const int m0 = tm * BM, n0 = paired ? tn * (BN / 2) : tn * BN;
    const int M = p.M, N = p.N, K = p.K, half = p.half;

    // ---- direct loads (waves 4-7): this lane's byte offsets in sub-tile 0 and its K indices there ----------------
    unsigned oa[A_LOADS], ob[4];
    int ka[A_LOADS], kb[4];
    const int lw = wave & 3;
#pragma unroll
    for (int i = 0; i < A_LOADS; ++i) {
        const int j = A_LOADS * lw + i;
        if (A_KC) {
            const int row = 8 * j + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
            ka[i] = c * 8;
            oa[i] = (unsigned)(((int64_t)min(m0 + row, M - 1) * p.lda + c * 8) * 2);
        } else {
            // K-rows of 128 or 256 bytes
            const int kr = FM == 1 ? 8 * j + (lane >> 3) : 4 * j + (lane >> 4);
            const int c = FM == 1 ? (lane & 7) ^ (4 * ((kr >> 1) & 1)) : (lane & 15) ^ (4 * (kr & 3));
            ka[i] = kr;
            oa[i] = (unsigned)(((int64_t)kr * p.lda + min(m0 + c * 8, M - 8)) * 2);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int j = 4 * lw + i;
        if (B_KC) {
            const int r = 8 * j + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
            const int row = paired ? (r < BN / 2 ? min(n0 + r, half - 1) : half + min(n0 + r - BN / 2, half - 1)) : min(n0 + r, N - 1);
            kb[i] = c * 8;
            ob[i] = (unsigned)(((int64_t)row * p.ldb + c * 8) * 2);
        } else {
            const int kr = 4 * j + (lane >> 4), c = (lane & 15) ^ (4 * (kr & 3));
            kb[i] = kr;
            ob[i] = (unsigned)(((int64_t)kr * p.ldb + min(n0 + c * 8, N - 8)) * 2);
        }
    }
    // (byte ranges below 2^31: the launcher has checked)
    const unsigned a_bytes = __builtin_amdgcn_readfirstlane(((unsigned)((A_KC ? M : K) - 1) * (unsigned)p.lda + (unsigned)(A_KC ? K : M)) * 2u);
    const unsigned b_bytes = __builtin_amdgcn_readfirstlane(((unsigned)((B_KC ? N : K) - 1) * (unsigned)p.ldb + (unsigned)(B_KC ? K : N)) * 2u);
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc((void *)p.A, 0, a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void *)p.B, 0, b_bytes, 0x00020000);
    const unsigned stepA = A_KC ? BK * 2u : (unsigned)(BK * p.lda * 2);
    const unsigned stepB = B_KC ? BK * 2u : (unsigned)(BK * p.ldb * 2);
    const int k_end = min(K, (kt_begin + kt_count) * BK);
    constexpr unsigned PAST = 0x80000000u; // beyond every operand's byte range

    auto issue = [&](int kt, int stage) {
        const int kk = kt_begin + kt, k0 = kk * BK;
        char *st = smem + stage * STAGE;
#pragma unroll
        for (int i = 0; i < A_LOADS; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_vp)(st + (A_LOADS * lw + i) * 1024), 16,
                                                     k0 + ka[i] < k_end ? oa[i] + kk * stepA : PAST, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_vp)(st + A_BYTES + (4 * lw + i) * 1024), 16,
                                                     k0 + kb[i] < k_end ? ob[i] + kk * stepB : PAST, 0, 0, 0);
    };

    // ---- fragment addresses (LDS byte addresses of stage 0) ----------------
    const unsigned smem_lds = (unsigned)(uintptr_t)(__attribute__((address_space(3))) const char *)smem;
    const int q = lane >> 4, i16 = lane & 15;
    unsigned fa[FM], fb[FN];
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        const int rbase = (wm * FM + i) * 32;
        if (A_KC) {
            const int row = rbase + (lane & 31);
            fa[i] = row * 128 + (((lane >> 5) ^ ((row >> 1) & 7)) << 4);
        } else {
            const int col = rbase + (q & 1) * 16 + (i16 & 3) * 4, kr = (q >> 1) * 8 + (i16 >> 2);
            fa[i] = kr * BM * 2 + (((col >> 3) ^ (FM == 1 ? 4 * ((kr >> 1) & 1) : 4 * (kr & 3))) << 4) + (col & 7) * 2;
        }
    }
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        const int rbase = j * (WN * 32) + wn * 32;
        if (B_KC) {
            const int row = rbase + (lane & 31);
            fb[j] = row * 128 + (((lane >> 5) ^ ((row >> 1) & 7)) << 4);
        } else {
            const int col = rbase + (q & 1) * 16 + (i16 & 3) * 4, kr = (q >> 1) * 8 + (i16 >> 2);
            fb[j] = kr * 256 + (((col >> 3) ^ (4 * (kr & 3))) << 4) + (col & 7) * 2;
        }
    }
    // fragments are read a sub-tile (FM == 1) or half of one ahead of the MFMAs that take them
    constexpr int KS = BK / 16, PARTS = FM, PS = KS / PARTS; // MFMA steps of a sub-tile, and of a part
    struct Frags {
        frag8 a[PS][FM], b[PS][FN];
    };
    auto read = [&](int stage, auto part, Frags &f) {
        const unsigned so = stage * STAGE;
        auto one = [&](auto ks_) {
            constexpr int ks = decltype(part)::value * PS + decltype(ks_)::value, at = decltype(ks_)::value;
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                if (A_KC)
                    f.a[at][i] = *(const frag8 *)(smem + so + (fa[i] ^ (ks << 5)));
                else
                    f.a[at][i] = frag_mc_read<frag8, ks, BM * 2>(smem_lds + so + fa[i]);
            }
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                if (B_KC)
                    f.b[at][j] = *(const frag8 *)(smem + so + A_BYTES + (fb[j] ^ (ks << 5)));
                else
                    f.b[at][j] = frag_mc_read<frag8, ks, 256>(smem_lds + so + A_BYTES + fb[j]);
            }
        };
        one(std::integral_constant<int, 0>{});
        one(std::integral_constant<int, 1>{});
        if constexpr (PS == 4) {
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
        for (int ks = 0; ks < PS; ++ks)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] = mfma_32x32x16(f.a[ks][i], f.b[ks][j], acc[i][j]);
    };

    // One barrier per step kt: before it the fetching waves have seen sub-tile kt + 1 land and the multiplying waves
    // hold (what is left of) sub-tile kt in registers; behind it kt + 1 may be read and the stage of kt be overwritten.
    static_assert((STAGES - 1) * LOADS < 64, "vmcnt is a 6-bit counter");
    const int steps = kt_count & ~1; // taken in pairs; an odd last sub-tile needs no barrier of its own
    int st = 0;                      // stage of sub-tile kt
    if (wave >= 4) {
#pragma unroll
        for (int i = 0; i < STAGES; ++i) issue(i, i);
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((STAGES - 1) * LOADS) : "memory"); // sub-tile 0 has landed
        for (int kt = 0; kt < steps; ++kt) {
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((STAGES - 2) * LOADS) : "memory");
            issue(kt + STAGES, st);
            st = st + 1 == STAGES ? 0 : st + 1;
        }
        // what was issued past the end lands before the epilogue takes the ring's LDS
        asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
        return;
    }
    Frags f0, f1;
    typedef std::integral_constant<int, 0> First;
    typedef std::integral_constant<int, PARTS - 1> Last;
    auto read_next = [&](Frags &nxt) {
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        read(st, First{}, nxt);
        if (PARTS == 1) st = st + 1 == STAGES ? 0 : st + 1;
    };
    auto read_rest = [&](Frags &nxt) { // the second half of the sub-tile that read_next has begun
        read(st, Last{}, nxt);
        st = st + 1 == STAGES ? 0 : st + 1;
    };
    auto in_registers = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    read_next(f0);
    in_registers();
    if constexpr (PARTS == 1) {
        for (int kt = 0; kt < steps; kt += 2) {
            read_next(f1);
            multiply(f0);
            in_registers();
            read_next(f0);
            multiply(f1);
            in_registers();
        }
        if (kt_count & 1) multiply(f0);
    } else {
        for (int kt = 0; kt < steps; ++kt) {
            read_rest(f1);
            multiply(f0);
            in_registers();
            read_next(f0);
            multiply(f1);
            in_registers();
        }
        if (kt_count & 1) {
            read_rest(f1);
            multiply(f0);
            in_registers();
            multiply(f1);
        }
    }
    asm volatile("s_barrier" ::: "memory");

    if (WIDE_ONLY || vec_epilogue)
        gemm_epilogue_staged<E, FM, FN, WN * 32>(p, acc, (float *)(smem + wave * EPI_LDS_BYTES_PER_WAVE), m0 + wm * FM * 32, n0, wn * 32, lane,
                                                smem + 4 * EPI_LDS_BYTES_PER_WAVE + wave * EPI_LAND_BYTES_PER_WAVE);
    else if constexpr (!WIDE_ONLY)
        gemm_epilogue<E, FM, FN, WN * 32>(p, acc, m0 + wm * FM * 32 + 4 * (lane >> 5), n0, wn * 32 + (lane & 31));
}

} // namespace rtp
