// The small tile of the partition GEMM: 64 x 128 of C per workgroup of 8 waves, for problems too short of rows or
// columns to give every compute unit a 128 x 256 tile (a prompt of some hundred tokens, a shard a few hundred units
// wide).  It runs inside gemm_pp_kernel, so a launch may mix it with the tall tiles.
//
// Bound: the latency of the operand fetch (a tile contracts over all of K alone: K / 64 dependent steps), then the
// L2 -> LDS path (24 KB per step for 256 cycles of MFMA).  Hence
//  * sub-tiles of 64 K, five LDS stages (120 KB), four of them in flight: twice the bytes in flight per flop of the
//    tall tile's ring;
//  * the eight waves are a 2 x 2 grid of 32 x 64 wave tiles times TWO halves of every sub-tile's K: a wave keeps the
//    tall tile's fragment shape (one LDS read feeds two MFMAs) and the epilogues apply unchanged; the halves' sums
//    meet once, in LDS, in a fixed order;
//  * fragments of sub-tile t + 1 are read while the MFMAs of sub-tile t run; one barrier per sub-tile.
// LDS layout: K-contiguous operands as 128-byte rows with the 16-byte chunk index xor-ed with (row/2)%8, M- or
// N-contiguous ones as K-rows of 128 (A) or 256 bytes (B) with the chunk index xor-ed with 4*((k/2)%2) or 4*(k%4):
// every fragment read then touches each of the 64 banks once per half-wave.
// Lanes past K (a partial last sub-tile, or a sub-tile past the end) get an offset beyond the operand's descriptor
// and read as zeros without touching memory.
#pragma once
#include "rtp_gemm_epilogue.h"

namespace rtp {

namespace pps {
constexpr int BM = 64, BN = 128, BK = 64;
constexpr int WM = 2, WN = 2, FN = 2;
constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE = A_BYTES + B_BYTES;
constexpr int STAGES = 5;
constexpr int RING_BYTES = STAGES * STAGE;
constexpr int LOADS = 3; // direct loads per wave and sub-tile: 1 KB of A, 2 KB of B
// after the ring: four waves' staged epilogue, then the other four waves' sums
constexpr int EPI_BYTES = 4 * (EPI_LDS_BYTES_PER_WAVE + EPI_LAND_BYTES_PER_WAVE);
constexpr int SUM_BYTES_PER_WAVE = 64 * 32 * 4;
} // namespace pps

template <int LAY, typename E>
__device__ __forceinline__ void pp_small_tile(const GemmArgs &p, const int tiles_m, const int tiles_n, const int vec_epilogue,
                                              const int pid, const int kt_begin, const int kt_count, char *smem)
{
    using namespace pps;
    typedef __attribute__((address_space(3))) void *lds_vp;
    typedef typename ElemVec<E>::v8 frag8;
    constexpr bool A_KC = (LAY != LAY_TN), B_KC = (LAY == LAY_NT);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kh = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1; // K half, place in the 2 x 2 grid

    constexpr int GROUP_M = 4; // 4-tall column strips, as the tall tiles
    const int group_sz = GROUP_M * tiles_n;
    const int first_m = pid / group_sz * GROUP_M;
    const int gm = min(tiles_m - first_m, GROUP_M);
    const int tm = first_m + (pid % group_sz) % gm, tn = (pid % group_sz) / gm;
    const bool paired = (p.epi == EPI_SWIGLU_FWD);
    const int m0 = tm * BM, n0 = paired ? tn * (BN / 2) : tn * BN;
    const int M = p.M, N = p.N, K = p.K, half = p.half;

    // ---- direct loads: this lane's byte offset in sub-tile 0 and its K index there ----------------
    unsigned oa, ob[2];
    int ka, kb[2];
    if (A_KC) {
        const int row = 8 * wave + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
        ka = c * 8;
        oa = (unsigned)(((int64_t)min(m0 + row, M - 1) * p.lda + c * 8) * 2);
    } else {
        const int kr = 8 * wave + (lane >> 3), c = (lane & 7) ^ (4 * ((kr >> 1) & 1));
        ka = kr;
        oa = (unsigned)(((int64_t)kr * p.lda + min(m0 + c * 8, M - 8)) * 2);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int j = 2 * wave + i;
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
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_vp)(st + wave * 1024), 16, k0 + ka < k_end ? oa + kk * stepA : PAST, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 2; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_vp)(st + A_BYTES + (2 * wave + i) * 1024), 16,
                                                     k0 + kb[i] < k_end ? ob[i] + kk * stepB : PAST, 0, 0, 0);
    };

    // ---- fragment addresses (LDS byte addresses of stage 0; the wave's K half is folded in) ----------------
    const unsigned smem_lds = (unsigned)(uintptr_t)(__attribute__((address_space(3))) const char *)smem;
    const int q = lane >> 4, i16 = lane & 15;
    unsigned fa, fb[FN];
    if (A_KC) {
        const int row = wm * 32 + (lane & 31);
        fa = row * 128 + (((lane >> 5) ^ ((row >> 1) & 7)) << 4);
        fa ^= kh << 6;
    } else {
        const int col = wm * 32 + (q & 1) * 16 + (i16 & 3) * 4, kr = (q >> 1) * 8 + (i16 >> 2);
        fa = kr * 128 + (((col >> 3) ^ (4 * ((kr >> 1) & 1))) << 4) + (col & 7) * 2 + kh * 32 * 128;
    }
#pragma unroll
    for (int f = 0; f < FN; ++f) {
        const int rbase = f * (WN * 32) + wn * 32;
        if (B_KC) {
            const int row = rbase + (lane & 31);
            fb[f] = row * 128 + (((lane >> 5) ^ ((row >> 1) & 7)) << 4);
            fb[f] ^= kh << 6;
        } else {
            const int col = rbase + (q & 1) * 16 + (i16 & 3) * 4, kr = (q >> 1) * 8 + (i16 >> 2);
            fb[f] = kr * 256 + (((col >> 3) ^ (4 * (kr & 3))) << 4) + (col & 7) * 2 + kh * 32 * 256;
        }
    }
    struct Frags {
        frag8 a[2], b[2][FN];
    };
    auto read = [&](int stage, Frags &f) {
        const unsigned so = stage * STAGE;
        if (A_KC) {
            f.a[0] = *(const frag8 *)(smem + so + fa);
            f.a[1] = *(const frag8 *)(smem + so + (fa ^ 32));
        } else {
            f.a[0] = frag_mc_read<frag8, 0, 128>(smem_lds + so + fa);
            f.a[1] = frag_mc_read<frag8, 1, 128>(smem_lds + so + fa);
        }
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            if (B_KC) {
                f.b[0][j] = *(const frag8 *)(smem + so + A_BYTES + fb[j]);
                f.b[1][j] = *(const frag8 *)(smem + so + A_BYTES + (fb[j] ^ 32));
            } else {
                f.b[0][j] = frag_mc_read<frag8, 0, 256>(smem_lds + so + A_BYTES + fb[j]);
                f.b[1][j] = frag_mc_read<frag8, 1, 256>(smem_lds + so + A_BYTES + fb[j]);
            }
        }
    };

    f32x16 acc[1][FN];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[0][j][v] = 0.0f;
    auto multiply = [&](const Frags &f) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[0][j] = mfma_32x32x16(f.a[ks], f.b[ks][j], acc[0][j]);
    };

    // A step ends with this wave's reads in registers, so that behind the barrier the stage they came from may be
    // overwritten; the barrier itself follows the landing of the sub-tile that is read next (LEFT newer ones may
    // still be on their way).
    static_assert((STAGES - 2) * LOADS < 64, "vmcnt is a 6-bit counter");
    int st = 0; // stage of sub-tile kt
    auto step = [&](int kt, const Frags &cur, Frags &nxt) {
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((STAGES - 2) * LOADS) : "memory"); // sub-tile kt + 1 has landed
        __builtin_amdgcn_sched_barrier(0);
        issue(kt + STAGES, st); // sub-tile kt was in registers before the barrier
        st = st + 1 == STAGES ? 0 : st + 1;
        read(st, nxt);
        multiply(cur);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

#pragma unroll
    for (int i = 0; i < STAGES; ++i) issue(i, i);
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((STAGES - 1) * LOADS) : "memory");
    __builtin_amdgcn_sched_barrier(0);
    Frags f0, f1;
    read(0, f0);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    int kt = 0;
    for (; kt + 1 < kt_count; kt += 2) {
        step(kt, f0, f1);
        step(kt + 1, f1, f0);
    }
    if (kt < kt_count) multiply(f0);
    // what was issued past the end lands before the ring is reused
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    // ---- the two K halves' sums meet: the second half's waves park theirs, the first half's add them ----------------
    f32x4 *sums = (f32x4 *)(smem + EPI_BYTES + (wave & 3) * SUM_BYTES_PER_WAVE);
    if (kh == 1)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                f32x4 t;
                t.x = acc[0][j][4 * v]; t.y = acc[0][j][4 * v + 1]; t.z = acc[0][j][4 * v + 2]; t.w = acc[0][j][4 * v + 3];
                sums[(j * 4 + v) * 64 + lane] = t;
            }
    __syncthreads();
    if (kh == 1) return;
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const f32x4 t = sums[(j * 4 + v) * 64 + lane];
            acc[0][j][4 * v] += t.x; acc[0][j][4 * v + 1] += t.y; acc[0][j][4 * v + 2] += t.z; acc[0][j][4 * v + 3] += t.w;
        }
    if (vec_epilogue)
        gemm_epilogue_staged<E, 1, FN, WN * 32>(p, acc, (float *)(smem + wave * EPI_LDS_BYTES_PER_WAVE), m0 + wm * 32, n0, wn * 32, lane,
                                                smem + 4 * EPI_LDS_BYTES_PER_WAVE + wave * EPI_LAND_BYTES_PER_WAVE);
    else
        gemm_epilogue<E, 1, FN, WN * 32>(p, acc, m0 + wm * 32 + 4 * (lane >> 5), n0, wn * 32 + (lane & 31));
}

} // namespace rtp
