// fp32 path of the partition GEMM (the small fp32 configuration), the
// elementwise activation kernels that path uses, and the shard-staging copy.
#include "rtp_ride.h"
#include <hip/hip_ext.h>
#include <cstring>
#include <algorithm>

namespace rtp {

typedef __attribute__((ext_vector_type(4))) float f32x4;

// ---- fp32 GEMM: 64x64 tile, 256 threads, 4x4 outputs per thread -------------------
// LDS holds A as [BK][64] and B as [BK][64] whatever the HBM layout, so the
// inner product reads both with unit stride.
constexpr int FT = 64, FK = 16;

struct F32Group {
    int count;
    unsigned tile_blocks;
    struct {
        GemmArgs a;
        int lay;
        unsigned tiles_n, first; // first workgroup
    } p[F32_MAX_GROUP];
    RideList ride;
};

template <int LAY>
__device__ __forceinline__ void gemm_f32_tile(const GemmArgs &p, const int m0, const int n0, float (*sA)[FT + 4], float (*sB)[FT + 4])
{
    const float *A = (const float *)p.A, *B = (const float *)p.B;
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    float acc[4][4] = {};
    for (int k0 = 0; k0 < p.K; k0 += FK) {
        // 64*16 = 1024 elements per operand, 4 per thread
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = tid + 256 * i;
            int k, r;
            if (LAY == LAY_TN) { r = e & 63; k = e >> 6; } else { k = e & 15; r = e >> 4; }
            const int gm = m0 + r, gk = k0 + k;
            float v = 0.0f;
            if (gm < p.M && gk < p.K)
                v = (LAY == LAY_TN) ? A[(int64_t)gk * p.lda + gm] : A[(int64_t)gm * p.lda + gk];
            sA[k][r] = v;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = tid + 256 * i;
            int k, r;
            if (LAY == LAY_NT) { k = e & 15; r = e >> 4; } else { r = e & 63; k = e >> 6; }
            const int gn = n0 + r, gk = k0 + k;
            float v = 0.0f;
            if (gn < p.N && gk < p.K)
                v = (LAY == LAY_NT) ? B[(int64_t)gn * p.ldb + gk] : B[(int64_t)gk * p.ldb + gn];
            sB[k][r] = v;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < FK; ++k) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = sA[k][ty * 4 + i];
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = sB[k][tx * 4 + j];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
        }
        __syncthreads();
    }
    float *C = (float *)p.C;
    const float *bias = (const float *)p.bias;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = m0 + ty * 4 + i;
        if (row >= p.M) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int col = n0 + tx * 4 + j;
            if (col >= p.N) continue;
            if (p.epi == EPI_ACC_ADD)
                C[(int64_t)row * p.ldc + col] += acc[i][j];
            else
                C[(int64_t)row * p.ldc + col] = acc[i][j] + (bias ? bias[col] : 0.0f);
        }
    }
}

// ---- the same for outputs of few tiles: 16x32, 128 threads, 2x2 outputs per thread -----------------
// Bound: latency (a 64 x 128 output over K = 256 is 4 MFLOP).  64x64 tiles put it on two compute units, each waiting for
// its operands once per 16 K: 27.6 us, here 8.1 (128 x 256 over K = 64 11.9 -> 5.3).  Here it is 16 workgroups; the chunk of 64 K behind the one being multiplied is
// already on its way in registers, 16 bytes a load where rows and pointers allow, and the sums an `+=` adds onto are
// fetched ahead of the loop.  LDS holds both operands along K, read four K at a time: rows of 68 floats put the 16
// columns a wave reads on all 64 banks.  An element is the same chain of fused multiply-adds in the order of K, with
// the same bits.  A 32x32 tile of 256 threads would be bound by its LDS reads (four waves to one LDS) at twice the time.
constexpr int SM = 16, SN = 32, SK = 64, SPITCH = SK + 4, STHR = 128;

// ROWS x SK of an operand into registers: thread t's share, ROWS * SK / STHR floats in groups of four
template <bool KC, int ROWS>
__device__ __forceinline__ void f32_fetch(f32x4 (&v)[ROWS * SK / STHR / 4], const float *p, const int64_t ld, const int r0, const int rows,
                                          const int k0, const int K, const bool wide)
{
    constexpr int G = ROWS * SK / STHR / 4, PER = KC ? SK / 4 : ROWS / 4; // groups along the contiguous dimension
#pragma unroll
    for (int i = 0; i < G; ++i) {
        const int t = threadIdx.x + i * STHR;
        const int k = k0 + (KC ? t % PER * 4 : t / PER), r = r0 + (KC ? t / PER : t % PER * 4);
        const int left = KC ? K - k : rows - r; // elements of the group that exist
        const bool on = KC ? r < rows : k < K;
        const float *q = p + (KC ? (int64_t)r * ld + k : (int64_t)k * ld + r);
        f32x4 x = {0.0f, 0.0f, 0.0f, 0.0f};
        if (on && left >= 4 && wide) {
            x = *(const f32x4 *)q;
        } else if (on) {
            if (left > 0) x.x = q[0];
            if (left > 1) x.y = q[1];
            if (left > 2) x.z = q[2];
            if (left > 3) x.w = q[3];
        }
        v[i] = x;
    }
}
template <bool KC, int ROWS>
__device__ __forceinline__ void f32_park(float (*lds)[SPITCH], const f32x4 (&v)[ROWS * SK / STHR / 4])
{
    constexpr int G = ROWS * SK / STHR / 4, PER = KC ? SK / 4 : ROWS / 4;
#pragma unroll
    for (int i = 0; i < G; ++i) {
        const int t = threadIdx.x + i * STHR;
        if (KC) {
            *(f32x4 *)&lds[t / PER][t % PER * 4] = v[i];
        } else {
            const int k = t / PER, r = t % PER * 4;
            lds[r][k] = v[i].x; lds[r + 1][k] = v[i].y; lds[r + 2][k] = v[i].z; lds[r + 3][k] = v[i].w;
        }
    }
}

template <int LAY>
__device__ __forceinline__ void gemm_f32_small_tile(const GemmArgs &p, const int m0, const int n0, float (*sA)[SPITCH], float (*sB)[SPITCH])
{
    constexpr bool A_KC = LAY != LAY_TN, B_KC = LAY == LAY_NT;
    const float *A = (const float *)p.A, *B = (const float *)p.B;
    const bool wa = (p.lda & 3) == 0 && ((uintptr_t)A & 15) == 0, wb = (p.ldb & 3) == 0 && ((uintptr_t)B & 15) == 0;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    float *C = (float *)p.C;
    float acc[2][2] = {}, old[2][2] = {};
    f32x4 va[SM * SK / STHR / 4], vb[SN * SK / STHR / 4];
    f32_fetch<A_KC, SM>(va, A, p.lda, m0, p.M, 0, p.K, wa);
    f32_fetch<B_KC, SN>(vb, B, p.ldb, n0, p.N, 0, p.K, wb);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int row = m0 + ty + 8 * i, col = n0 + tx + 16 * j;
            if (p.epi == EPI_ACC_ADD && row < p.M && col < p.N) old[i][j] = C[(int64_t)row * p.ldc + col];
        }
    for (int k0 = 0; k0 < p.K; k0 += SK) {
        f32_park<A_KC, SM>(sA, va);
        f32_park<B_KC, SN>(sB, vb);
        __syncthreads();
        if (k0 + SK < p.K) {
            f32_fetch<A_KC, SM>(va, A, p.lda, m0, p.M, k0 + SK, p.K, wa);
            f32_fetch<B_KC, SN>(vb, B, p.ldb, n0, p.N, k0 + SK, p.K, wb);
        }
#pragma unroll
        for (int k = 0; k < SK; k += 4) { // (K indices past the end hold zeros)
            f32x4 a[2], b[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) a[i] = *(const f32x4 *)&sA[ty + 8 * i][k];
#pragma unroll
            for (int j = 0; j < 2; ++j) b[j] = *(const f32x4 *)&sB[tx + 16 * j][k];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[i][j] = fmaf(a[i][u], b[j][u], acc[i][j]);
        }
        __syncthreads();
    }
    const float *bias = (const float *)p.bias;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int row = m0 + ty + 8 * i, col = n0 + tx + 16 * j;
            if (row >= p.M || col >= p.N) continue;
            C[(int64_t)row * p.ldc + col] = p.epi == EPI_ACC_ADD ? old[i][j] + acc[i][j] : acc[i][j] + (bias ? bias[col] : 0.0f);
        }
}

__global__ __launch_bounds__(STHR) void gemm_f32_kernel(const F32Group g)
{
    __shared__ __attribute__((aligned(16))) float lds[(SM + SN) * SPITCH];
    if (blockIdx.x >= g.tile_blocks) {
        ride<STHR>(g.ride, blockIdx.x - g.tile_blocks);
        return;
    }
    const int q = g.count > 1 && blockIdx.x >= g.p[1].first ? 1 : 0;
    const unsigned b = blockIdx.x - g.p[q].first;
    const int m = (int)(b / g.p[q].tiles_n), n = (int)(b % g.p[q].tiles_n);
    float(*sA)[SPITCH] = (float(*)[SPITCH])lds, (*sB)[SPITCH] = sA + SM;
    switch (g.p[q].lay) {
    case LAY_NT: gemm_f32_small_tile<LAY_NT>(g.p[q].a, m * SM, n * SN, sA, sB); break;
    case LAY_NN: gemm_f32_small_tile<LAY_NN>(g.p[q].a, m * SM, n * SN, sA, sB); break;
    default: gemm_f32_small_tile<LAY_TN>(g.p[q].a, m * SM, n * SN, sA, sB); break;
    }
}

// 64x64 tiles, one layout and no transfers a kernel: in one with them and all three layouts, whose registers the greediest
// sets, 4096 x 4096 over K = 512 took 289 / 288 / 321 us (NT / NN / TN) instead of 245 / 257 / 252.
template <int LAY>
__global__ __launch_bounds__(256) void gemm_f32_large_kernel(const GemmArgs p, const unsigned tiles_n)
{
    __shared__ float sA[FK][FT + 4];
    __shared__ float sB[FK][FT + 4];
    gemm_f32_tile<LAY>(p, (int)(blockIdx.x / tiles_n) * FT, (int)(blockIdx.x % tiles_n) * FT, sA, sB);
}

// Up to this many small tiles the small tile is the faster one.  us, K = 1024, 64x64 -> 16x32: 256 tiles (512 x 256) 93.9 -> 24.2,
// 1024 93.7 -> 32.8, 4096 (2048 x 1024) 143 -> 103, 8192 170 -> 182, 16384 307 -> 338, 32768 506 -> 677.
constexpr int64_t F32_SMALL_MAX = 4096;

hipError_t launch_gemm_f32_riding(const int *layouts, const GemmArgs *a, int count, const Riders &r, hipStream_t s)
{
    if (count < 0 || count > F32_MAX_GROUP || r.sums != 0) return hipErrorInvalidValue;
    F32Group g;
    memset(&g, 0, sizeof g);
    int64_t small_tiles = 0;
    for (int i = 0; i < count; ++i)
        if (a[i].M > 0 && a[i].N > 0) small_tiles += (int64_t)((a[i].N + SN - 1) / SN) * ((a[i].M + SM - 1) / SM);
    const bool small = small_tiles <= F32_SMALL_MAX;
    const int tm = small ? SM : FT, tn = small ? SN : FT;
    int64_t blocks = 0;
    for (int i = 0; i < count; ++i) {
        if (a[i].M <= 0 || a[i].N <= 0) continue;
        if (a[i].K <= 0 || (a[i].epi != EPI_STORE && a[i].epi != EPI_ACC_ADD)) return hipErrorInvalidValue;
        if (layouts[i] < LAY_NT || layouts[i] > LAY_TN) return hipErrorInvalidValue;
        auto &p = g.p[g.count++];
        p.a = a[i];
        p.lay = layouts[i];
        p.tiles_n = (unsigned)((a[i].N + tn - 1) / tn);
        p.first = (unsigned)blocks;
        blocks += (int64_t)p.tiles_n * ((a[i].M + tm - 1) / tm);
    }
    if (g.count == 0) return launch_riders(r, s);
    if (blocks >= (int64_t)1 << 30) return hipErrorInvalidValue;
    if (!small) { // the transfers are nothing beside such a product
        const hipError_t e = launch_riders(r, s);
        if (e != hipSuccess) return e;
        for (int i = 0; i < g.count; ++i) {
            const auto &p = g.p[i];
            const dim3 grid((unsigned)((i + 1 < g.count ? g.p[i + 1].first : blocks) - p.first)), block(256);
            switch (p.lay) {
            case LAY_NT: hipLaunchKernelGGL(gemm_f32_large_kernel<LAY_NT>, grid, block, 0, s, p.a, p.tiles_n); break;
            case LAY_NN: hipLaunchKernelGGL(gemm_f32_large_kernel<LAY_NN>, grid, block, 0, s, p.a, p.tiles_n); break;
            default: hipLaunchKernelGGL(gemm_f32_large_kernel<LAY_TN>, grid, block, 0, s, p.a, p.tiles_n); break;
            }
        }
        return hipGetLastError();
    }
    g.tile_blocks = (unsigned)blocks;
    const hipError_t e = ride_list(r, 256, &g.ride);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(gemm_f32_kernel, dim3(g.tile_blocks + g.ride.blocks), dim3(STHR), 0, s, g);
    return hipGetLastError();
}

hipError_t launch_gemm_f32(int layout, const GemmArgs &a, hipStream_t s) { return launch_gemm_f32_riding(&layout, &a, 1, Riders(), s); }

// ---- elementwise activations for the fp32 path --------------------------------------
__device__ __forceinline__ float act_gelu_erf(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float act_gelu_erf_grad(float x)
{
    return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) + x * 0.3989422804014327f * expf(-0.5f * x * x);
}
__device__ __forceinline__ float act_gelu_tanh(float x)
{
    return 0.5f * x * (1.0f + tanhf(0.7978845608028654f * (x + 0.044715f * x * x * x)));
}
__device__ __forceinline__ float act_gelu_tanh_grad(float x)
{
    const float th = tanhf(0.7978845608028654f * (x + 0.044715f * x * x * x));
    const float du = 0.7978845608028654f * (1.0f + 3.0f * 0.044715f * x * x);
    return 0.5f * (1.0f + th) + 0.5f * x * (1.0f - th * th) * du;
}
__device__ __forceinline__ float act_sigmoid(float x) { return 1.0f / (1.0f + expf(-x)); }

// forward kinds: out[r, c] = act(pre[r, c])            (SWIGLU: silu(pre[r,c]) * pre[r, half+c])
// backward kinds: out[r, c] = in[r, c] * act'(pre[r, c])
//   SWIGLU_BWD: out[r, c] = in*b*silu'(a), out[r, half+c] = in*silu(a)
__global__ void act_f32_kernel(int kind, const float *pre, int64_t ldpre, const float *in, int64_t ldin, float *out,
                               int64_t ldout, int rows, int cols, int half)
{
    const int64_t n = (int64_t)rows * cols;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int r = (int)(e / cols), c = (int)(e % cols);
        const float z = pre[r * ldpre + c];
        switch (kind) {
        case EPI_GELU_ERF_FWD: out[r * ldout + c] = act_gelu_erf(z); break;
        case EPI_GELU_TANH_FWD: out[r * ldout + c] = act_gelu_tanh(z); break;
        case EPI_SWIGLU_FWD: out[r * ldout + c] = z * act_sigmoid(z) * pre[r * ldpre + half + c]; break;
        case EPI_GELU_ERF_BWD: out[r * ldout + c] = in[r * ldin + c] * act_gelu_erf_grad(z); break;
        case EPI_GELU_TANH_BWD: out[r * ldout + c] = in[r * ldin + c] * act_gelu_tanh_grad(z); break;
        case EPI_SWIGLU_BWD: {
            const float sg = act_sigmoid(z), b = pre[r * ldpre + half + c], g = in[r * ldin + c];
            out[r * ldout + c] = g * b * sg * (1.0f + z * (1.0f - sg));
            out[r * ldout + half + c] = g * z * sg;
            break;
        }
        default: break;
        }
    }
}

hipError_t launch_act_f32(int kind, const float *pre, int64_t ldpre, const float *in, int64_t ldin, float *out,
                          int64_t ldout, int rows, int cols, int half, hipStream_t s)
{
    if (rows <= 0 || cols <= 0) return hipSuccess;
    const int64_t n = (int64_t)rows * cols;
    const int blocks = (int)((n + 255) / 256 > 2048 ? 2048 : (n + 255) / 256);
    hipLaunchKernelGGL(act_f32_kernel, dim3(blocks), dim3(256), 0, s, kind, pre, ldpre, in, ldin, out, ldout, rows,
                       cols, half);
    return hipGetLastError();
}

// ---- staging copy ---------------------------------------------------------------------
// Each workgroup moves one piece of 32 or 64 KB with 16-byte accesses and exits, so the
// copy slips into whatever wave slots the GEMM running beside it leaves free
// instead of holding compute units for the whole transfer.  A whole piece is moved without a bounds test per unit:
// behind one, the compiler waits ahead of every store for all stores before it (Llama-shaped unit's training step
// against one reference on one box: 1.004 -> 1.027 x as fast).
// Pieces of 32 KB go faster, those of 64 KB disturb the GEMMs less: short ones where the transfers bound the step, long ones
// where many tokens do (copy_async has the line and what it measured).  Alone, 541 MB with pieces of 64, 32 and 16 KB 225, 183
// and 189 us.
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
constexpr int COPY_THREADS = 256;
constexpr int COPY_PER_THREAD = 8, COPY_LONG_PER_THREAD = 16; // x 16 bytes

// the units of a thread from `base` on
template <int PER>
__device__ __forceinline__ void copy_units(u32x4 *__restrict__ dst, const u32x4 *__restrict__ src, const int64_t base, const int64_t n16)
{
    u32x4 v[PER];
    if (base - threadIdx.x + COPY_THREADS * PER <= n16) {
#pragma unroll
        for (int i = 0; i < PER; ++i) v[i] = __builtin_nontemporal_load(src + base + i * COPY_THREADS);
#pragma unroll
        for (int i = 0; i < PER; ++i) __builtin_nontemporal_store(v[i], dst + base + i * COPY_THREADS);
        return;
    }
#pragma unroll
    for (int i = 0; i < PER; ++i)
        if (base + i * COPY_THREADS < n16) v[i] = __builtin_nontemporal_load(src + base + i * COPY_THREADS);
#pragma unroll
    for (int i = 0; i < PER; ++i)
        if (base + i * COPY_THREADS < n16) __builtin_nontemporal_store(v[i], dst + base + i * COPY_THREADS);
}

template <int PER>
__device__ __forceinline__ void copy_piece(u32x4 *__restrict__ dst, const u32x4 *__restrict__ src, int64_t n16)
{
    copy_units<PER>(dst, src, (int64_t)blockIdx.x * (COPY_THREADS * PER) + threadIdx.x, n16);
}
__global__ __launch_bounds__(COPY_THREADS) void copy_kernel(u32x4 *__restrict__ dst, const u32x4 *__restrict__ src, int64_t n16)
{
    copy_piece<COPY_PER_THREAD>(dst, src, n16);
}
__global__ __launch_bounds__(COPY_THREADS) void copy_long_kernel(u32x4 *__restrict__ dst, const u32x4 *__restrict__ src, int64_t n16)
{
    copy_piece<COPY_LONG_PER_THREAD>(dst, src, n16);
}

// The same for a copy that nothing runs beside: pieces of 16 KB, so that some workgroups read while others write.  us alone,
// past the caches, with pieces of 64 KB -> 16 KB: 33 MB 14.6 -> 13.1, 67 MB 26.4 -> 24.0, 352 MB 136 -> 115 (64 KB with a
// bounds test per unit 13.9, 25.7, 138).
constexpr int COPY_ALONE_PER_THREAD = 4;
__global__ __launch_bounds__(COPY_THREADS) void copy_alone_kernel(u32x4 *__restrict__ dst, const u32x4 *__restrict__ src, int64_t n16)
{
    copy_piece<COPY_ALONE_PER_THREAD>(dst, src, n16);
}

// done: an event that completes with the copy (the kernel's completion signal is the event's: no record packet of
// its own in the queue, and one host call less), or null.  Recorded the plain way when there is nothing to copy.
static hipError_t launch_copy_pieces(void (*kernel)(u32x4 *, const u32x4 *, int64_t), int per_thread, void *dst, const void *src,
                                     size_t bytes, hipStream_t s, hipEvent_t done)
{
    if (bytes == 0) return done ? hipEventRecord(done, s) : hipSuccess;
    if ((bytes & 15) || ((uintptr_t)dst & 15) || ((uintptr_t)src & 15)) return hipErrorInvalidValue;
    const int64_t n16 = (int64_t)(bytes >> 4);
    const int64_t per = COPY_THREADS * per_thread;
    const unsigned blocks = (unsigned)((n16 + per - 1) / per);
    if (done)
        hipExtLaunchKernelGGL(kernel, dim3(blocks), dim3(COPY_THREADS), 0, s, nullptr, done, 0, (u32x4 *)dst,
                              (const u32x4 *)src, n16);
    else
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(COPY_THREADS), 0, s, (u32x4 *)dst, (const u32x4 *)src, n16);
    return hipGetLastError();
}

hipError_t launch_copy(void *dst, const void *src, size_t bytes, hipStream_t s, hipEvent_t done)
{
    return launch_copy_pieces(copy_kernel, COPY_PER_THREAD, dst, src, bytes, s, done);
}

hipError_t launch_copy_long(void *dst, const void *src, size_t bytes, hipStream_t s, hipEvent_t done)
{
    return launch_copy_pieces(copy_long_kernel, COPY_LONG_PER_THREAD, dst, src, bytes, s, done);
}

hipError_t launch_copy_alone(void *dst, const void *src, size_t bytes, hipStream_t s, hipEvent_t done)
{
    return launch_copy_pieces(copy_alone_kernel, COPY_ALONE_PER_THREAD, dst, src, bytes, s, done);
}

// Up to COPY_MAX_SEGS independent copies as one launch: workgroups [first[i], first[i + 1]) move segment i, 32 KB
// each as above, so the segments go through the machine one after the other as separate launches would, for one
// launch's worth of host time.  The segments must not overlap one another (no order among them).
struct CopySegs {
    u32x4 *dst[COPY_MAX_SEGS];
    const u32x4 *src[COPY_MAX_SEGS];
    int64_t n16[COPY_MAX_SEGS];
    unsigned first[COPY_MAX_SEGS + 1];
    int count;
};

__global__ __launch_bounds__(COPY_THREADS) void copy_multi_kernel(const CopySegs g)
{
    int i = 0;
    while (i + 1 < g.count && blockIdx.x >= g.first[i + 1]) ++i;
    const u32x4 *__restrict__ src = g.src[i];
    u32x4 *__restrict__ dst = g.dst[i];
    const int64_t n16 = g.n16[i];
    const int64_t base = (int64_t)(blockIdx.x - g.first[i]) * (COPY_THREADS * COPY_PER_THREAD) + threadIdx.x;
    copy_units<COPY_PER_THREAD>(dst, src, base, n16);
}

hipError_t launch_copy_multi(void *const *dst, const void *const *src, const size_t *bytes, int count, hipStream_t s,
                             hipEvent_t done)
{
    if (count < 0 || count > COPY_MAX_SEGS) return hipErrorInvalidValue;
    CopySegs g;
    memset(&g, 0, sizeof g);
    const int64_t per = COPY_THREADS * COPY_PER_THREAD;
    unsigned blocks = 0;
    for (int i = 0; i < count; ++i) {
        if (bytes[i] == 0) continue;
        if ((bytes[i] & 15) || ((uintptr_t)dst[i] & 15) || ((uintptr_t)src[i] & 15)) return hipErrorInvalidValue;
        const int64_t n16 = (int64_t)(bytes[i] >> 4);
        g.dst[g.count] = (u32x4 *)dst[i];
        g.src[g.count] = (const u32x4 *)src[i];
        g.n16[g.count] = n16;
        g.first[g.count] = blocks;
        blocks += (unsigned)((n16 + per - 1) / per);
        g.count++;
    }
    if (g.count == 0) return done ? hipEventRecord(done, s) : hipSuccess;
    g.first[g.count] = blocks;
    if (g.count == 1) return launch_copy(g.dst[0], g.src[0], (size_t)g.n16[0] << 4, s, done);
    if (done)
        hipExtLaunchKernelGGL(copy_multi_kernel, dim3(blocks), dim3(COPY_THREADS), 0, s, nullptr, done, 0, g);
    else
        hipLaunchKernelGGL(copy_multi_kernel, dim3(blocks), dim3(COPY_THREADS), 0, s, g);
    return hipGetLastError();
}

// ---- transfers that ride in a launch, or go out as one of their own -------------------------
hipError_t ride_list(const Riders &r, int idle, RideList *out)
{
    memset(out, 0, sizeof *out);
    int64_t total = 0;
    for (int i = 0; i < r.count; ++i) {
        const RideSeg &q = r.seg[i];
        if (((uintptr_t)q.out | (uintptr_t)q.buf | (uintptr_t)q.in | q.bytes) & 15) return hipErrorInvalidValue;
        total += (int64_t)(q.bytes >> 4);
    }
    // pieces that fill the idle compute units once, of at least 16 KB (one round of reads in flight) and at most 64 KB
    const int64_t per = std::min<int64_t>(4096, std::max<int64_t>(1024, (total / std::max(1, idle) + 1023) / 1024 * 1024));
    out->per_block = (int)per;
    for (int i = 0; i < r.count; ++i) {
        const int64_t n16 = (int64_t)(r.seg[i].bytes >> 4);
        if (n16 == 0 || (!r.seg[i].out && !r.seg[i].in)) continue;
        auto &q = out->seg[out->count++];
        q.out = (ride_u32x4 *)r.seg[i].out;
        q.buf = (ride_u32x4 *)r.seg[i].buf;
        q.in = (const ride_u32x4 *)r.seg[i].in;
        q.n16 = n16;
        q.first = out->blocks;
        out->blocks += (unsigned)((n16 + per - 1) / per);
    }
    for (int i = 0; i < r.sums; ++i) {
        const RideSum &q = r.sum[i];
        if (q.rows < 0 || !q.in || !q.out || (q.rows > 0 && !q.Y)) return hipErrorInvalidValue;
        if (q.cols <= 0) continue;
        if (!colsum_wide(q.Y, q.ld, q.cols)) return hipErrorInvalidValue;
        auto &d = out->sum[out->sums++];
        d.Y = q.Y; d.ld = q.ld; d.rows = q.rows; d.cols = q.cols; d.in = q.in; d.out = q.out;
        d.first = out->sum_blocks;
        out->sum_blocks += (unsigned)((q.cols + COLSUM_COLS - 1) / COLSUM_COLS);
    }
    return hipSuccess;
}

__global__ __launch_bounds__(COPY_THREADS) void ride_kernel(const RideList g) { ride<COPY_THREADS>(g, blockIdx.x); }

hipError_t launch_riders(const Riders &r, hipStream_t s)
{
    for (int i = 0; i < r.sums; ++i) {
        const RideSum &q = r.sum[i];
        const hipError_t e = launch_colsum(q.elem, q.Y, q.ld, q.rows, q.cols, q.in, q.out, s);
        if (e != hipSuccess) return e;
    }
    Riders moves = r;
    moves.sums = 0;
    RideList g;
    const hipError_t e = ride_list(moves, 512, &g);
    if (e != hipSuccess || g.blocks == 0) return e;
    hipLaunchKernelGGL(ride_kernel, dim3(g.blocks), dim3(COPY_THREADS), 0, s, g);
    return hipGetLastError();
}

// Bound: HBM writes.  A thread stores one unit, past the caches, and its workgroup of 4 KB is done.  us, 4096 workgroups that
// walk the buffer -> so: 16 MB 5.3 -> 4.5, 90 MB 15.1 -> 14.5, 541 MB 122 -> 86, 1.9 GB 488 -> 296, 5.64 GB 1331 -> 879 (6.4
// TB/s); 16 KB a workgroup 984, 64 KB 1040.
__global__ __launch_bounds__(256) void fill_zero_kernel(u32x4 *dst, int64_t n16)
{
    const u32x4 z = {0u, 0u, 0u, 0u};
    const int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x;
    if (e < n16) __builtin_nontemporal_store(z, dst + e);
}

hipError_t launch_fill_zero(void *dst, size_t bytes, hipStream_t s)
{
    if (bytes == 0) return hipSuccess;
    if ((bytes & 15) || ((uintptr_t)dst & 15)) return hipErrorInvalidValue;
    constexpr int64_t MOST = (int64_t)1 << 30; // units a launch (a grid holds 2^32 threads)
    for (int64_t at = 0, n16 = (int64_t)(bytes >> 4); at < n16; at += MOST) {
        const int64_t n = std::min(MOST, n16 - at);
        hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (u32x4 *)dst + at, n);
    }
    return hipGetLastError();
}

// ---- shard layout: a full matrix into (out of) the N slots of the ring store --------------------
// Shard k of W[O, I] is a row block [w, I] (rows k w .. of W; output partition) or a column block
// stored contiguously as [O, w] (columns k w .. of W; input partition) at `off` bytes into slot k.
// Elements of the shard that lie past the matrix (a padded partition) are written as zero when
// packing and skipped when unpacking.
// Bound: HBM (every element read once and written once).  The kernel moves units of type T: 16 bytes
// where rows, shard width, slot and pointers are whole numbers of 16-byte units, else single elements.
// A workgroup takes LAYOUT_PER_THREAD x 256 consecutive units of one shard, all reads of a thread in
// flight before its first store.  That needs reads without a bounds test: behind one per
// unit the compiler kept all eight in one block of 240 registers and waited for each read before it issued the
// next.  Where a workgroup is not wholly inside the matrix (a shard's end, the last column block of a padded
// partition) a unit outside is read from one that exists and dropped.  A row block is one contiguous run of W and needs no
// row arithmetic; a column block divides by the shard width once per thread and counts from there.  Weights and
// gradients of three [11008, 4096] matrices out and weights in, whole exchange: 958 us with an element per
// thread, 707 with tests and divisions per unit, 396 so.
// Single elements of column blocks go into the matrix through the caches: its rows start inside a line that the neighbouring
// shard's workgroup fills up.  Past the caches [11008, 4096] fp32 in three shards came out in 84 us, so in 50.
typedef __attribute__((ext_vector_type(4))) unsigned int layout_u32x4;
constexpr int LAYOUT_PER_THREAD = 8;

template <typename T, bool COLS, bool UNPACK>
__global__ __launch_bounds__(256) void shard_layout_kernel(char *home, size_t slot_bytes, size_t off, T *W, int64_t O,
                                                           int64_t I, int64_t w, unsigned blocks_per_shard,
                                                           int64_t step_rows, int64_t step_cols)
{
    const int64_t k = blockIdx.x / blocks_per_shard;
    T *slot = (T *)(home + (size_t)k * slot_bytes + off);
    const int64_t per = COLS ? O * w : w * I; // units of one shard
    // a row block's units inside the matrix, a column block's columns inside it
    const int64_t rows_in = min(w, max((int64_t)0, O - k * w)), cols_in = min(w, max((int64_t)0, I - k * w));
    T *Wk = W + (COLS ? k * w : k * w * I);
    const int64_t first = (int64_t)(blockIdx.x % blocks_per_shard) * (256 * LAYOUT_PER_THREAD), base = first + threadIdx.x;
    int64_t row = 0, col = 0; // of the thread's next unit in a column block
    if (COLS) {
        row = per >> 32 == 0 ? (int64_t)((unsigned)base / (unsigned)w) : base / w; // (32-bit division where it reaches)
        col = base - row * w;
    }
    auto step = [&]() {
        row += step_rows;
        col += step_cols;
        if (col >= w) {
            col -= w;
            ++row;
        }
    };
    auto put = [](T x, T *to) {
        if (sizeof(T) == 16)
            __builtin_nontemporal_store(x, to);
        else
            *to = x;
    };
    const int64_t end = first + 256 * LAYOUT_PER_THREAD;
    if (COLS ? end <= per && cols_in == w : end <= rows_in * I) { // the workgroup's units all lie inside the matrix
        T v[LAYOUT_PER_THREAD];
        T *at[LAYOUT_PER_THREAD];
#pragma unroll
        for (int u = 0; u < LAYOUT_PER_THREAD; ++u) {
            at[u] = Wk + (COLS ? row * I + col : base + u * 256);
            if (COLS) step();
            v[u] = UNPACK ? __builtin_nontemporal_load(slot + base + u * 256) : __builtin_nontemporal_load(at[u]);
        }
#pragma unroll
        for (int u = 0; u < LAYOUT_PER_THREAD; ++u) {
            if (UNPACK)
                put(v[u], at[u]);
            else
                __builtin_nontemporal_store(v[u], slot + base + u * 256);
        }
        return;
    }
    T v[LAYOUT_PER_THREAD];
    T *at[LAYOUT_PER_THREAD];
    bool in[LAYOUT_PER_THREAD];
#pragma unroll
    for (int u = 0; u < LAYOUT_PER_THREAD; ++u) {
        const int64_t e = base + u * 256;
        in[u] = e < per && (COLS ? col < cols_in : e < rows_in * I);
        at[u] = in[u] ? Wk + (COLS ? row * I + col : e) : W;
        if (COLS) step();
        v[u] = UNPACK ? __builtin_nontemporal_load(slot + min(e, per - 1)) : __builtin_nontemporal_load(at[u]);
    }
#pragma unroll
    for (int u = 0; u < LAYOUT_PER_THREAD; ++u) {
        const int64_t e = base + u * 256;
        if (UNPACK) {
            if (in[u]) put(v[u], at[u]);
        } else if (end <= per || e < per) {
            __builtin_nontemporal_store(in[u] ? v[u] : T{}, slot + e);
        }
    }
}

template <typename T>
static hipError_t launch_shard_layout_units(void *home, size_t slot_bytes, size_t off, int n, int cols, void *W, int64_t O,
                                            int64_t I, int64_t w, int unpack, hipStream_t s)
{
    const int64_t per = cols ? O * w : w * I;
    const int64_t blocks = (per + 256 * LAYOUT_PER_THREAD - 1) / (256 * LAYOUT_PER_THREAD);
    if (blocks * n >= (int64_t)1 << 31) return hipErrorInvalidValue;
#define RTP_SHARD_LAYOUT(C, U)                                                                                          \
    hipLaunchKernelGGL((shard_layout_kernel<T, C, U>), dim3((unsigned)(blocks * n)), dim3(256), 0, s, (char *)home, slot_bytes, \
                       off, (T *)W, O, I, w, (unsigned)blocks, 256 / w, 256 % w)
    if (cols) { if (unpack) RTP_SHARD_LAYOUT(true, true); else RTP_SHARD_LAYOUT(true, false); }
    else { if (unpack) RTP_SHARD_LAYOUT(false, true); else RTP_SHARD_LAYOUT(false, false); }
#undef RTP_SHARD_LAYOUT
    return hipGetLastError();
}

hipError_t launch_shard_layout(void *home, size_t slot_bytes, size_t off, int n, int cols, void *W, int64_t O, int64_t I,
                               int64_t w, int elem_bytes, int unpack, hipStream_t s)
{
    if ((cols ? O * w : w * I) * n <= 0) return hipSuccess;
    if (elem_bytes != 2 && elem_bytes != 4) return hipErrorInvalidValue;
    const int64_t unit = 16 / elem_bytes;
    const bool wide = I % unit == 0 && (!cols || w % unit == 0) &&
                      ((slot_bytes | off | (size_t)(uintptr_t)home | (size_t)(uintptr_t)W) & 15) == 0;
    if (wide)
        return launch_shard_layout_units<layout_u32x4>(home, slot_bytes, off, n, cols, W, O, I / unit, cols ? w / unit : w, unpack, s);
    return elem_bytes == 2 ? launch_shard_layout_units<uint16_t>(home, slot_bytes, off, n, cols, W, O, I, w, unpack, s)
                           : launch_shard_layout_units<uint32_t>(home, slot_bytes, off, n, cols, W, O, I, w, unpack, s);
}

// ---- bias piece of an input-partitioned fp32 layer, added onto a slice of its output (16-bit layers: in the GEMM) ----
__global__ __launch_bounds__(256) void bias_add_kernel(float *dst, int64_t ld, int rows, int cols, const float *bias)
{
    const int c = blockIdx.x * 64 + (threadIdx.x & 63);
    if (c >= cols) return;
    const float b = bias[c];
    for (int r = blockIdx.y * 4 + (threadIdx.x >> 6); r < rows; r += gridDim.y * 4) dst[(int64_t)r * ld + c] += b;
}

hipError_t launch_bias_add(float *dst, int64_t ld, int rows, int cols, const float *bias, hipStream_t s)
{
    if (rows <= 0 || cols <= 0) return hipSuccess;
    const dim3 grid((unsigned)((cols + 63) / 64), (unsigned)std::min(1024, (rows + 3) / 4)), block(256);
    hipLaunchKernelGGL(bias_add_kernel, grid, block, 0, s, dst, ld, rows, cols, bias);
    return hipGetLastError();
}

// ---- expert partition: grouping tokens by expert, row gather and scatter ------------------------
// One workgroup: thread i owns the i-th contiguous chunk of tokens.  Per-(expert, chunk) counts
// in LDS, an exclusive scan over the chunks of each expert, the group starts from the counts,
// then every thread places its tokens in order: the result is the stable grouping whatever the
// number of threads.
constexpr int DISPATCH_THREADS = 128;

__global__ __launch_bounds__(DISPATCH_THREADS) void moe_dispatch_kernel(const int *__restrict__ route, int T, int n, int align,
                                                                        int cap, int *__restrict__ counts, int *__restrict__ perm)
{
    extern __shared__ int dispatch_lds[];
    int *hist = dispatch_lds;                     // [n][DISPATCH_THREADS]
    int *seg = dispatch_lds + n * DISPATCH_THREADS; // [n + 1] group starts
    __shared__ int bad;
    const int tid = threadIdx.x;
    const int chunk = (T + DISPATCH_THREADS - 1) / DISPATCH_THREADS;
    const int lo = min(T, tid * chunk), hi = min(T, lo + chunk);
    for (int e = 0; e < n; ++e) hist[e * DISPATCH_THREADS + tid] = 0;
    if (tid == 0) bad = 0;
    __syncthreads();
    int my_bad = 0;
    for (int t = lo; t < hi; ++t) {
        const int e = route[t];
        if ((unsigned)e < (unsigned)n) hist[e * DISPATCH_THREADS + tid]++;
        else my_bad++;
    }
    if (my_bad) atomicAdd(&bad, my_bad);
    __syncthreads();
    for (int e = tid; e < n; e += DISPATCH_THREADS) {
        int run = 0;
        for (int i = 0; i < DISPATCH_THREADS; ++i) {
            const int c = hist[e * DISPATCH_THREADS + i];
            hist[e * DISPATCH_THREADS + i] = run;
            run += c;
        }
        counts[e] = run;
        seg[e + 1] = run;
    }
    __syncthreads();
    if (tid == 0) {
        seg[0] = 0;
        for (int e = 0; e < n; ++e) seg[e + 1] = seg[e] + (seg[e + 1] + align - 1) / align * align;
        counts[n] = bad;
    }
    for (int p = tid; p < cap; p += DISPATCH_THREADS) perm[p] = -1;
    __syncthreads();
    for (int t = lo; t < hi; ++t) {
        const int e = route[t];
        if ((unsigned)e < (unsigned)n) {
            const int p = seg[e] + hist[e * DISPATCH_THREADS + tid]++;
            if (p < cap) perm[p] = t;
        }
    }
}

hipError_t launch_moe_dispatch(const int *route, int T, int n, int align, int cap, int *counts, int *perm, hipStream_t s)
{
    if (n < 1 || n > MOE_MAX_EXPERTS || T < 0 || align < 1 || cap < 0) return hipErrorInvalidValue;
    if ((int64_t)cap < (int64_t)align * (T / align + n)) return hipErrorInvalidValue;
    const size_t lds = (size_t)(n * DISPATCH_THREADS + n + 1) * sizeof(int);
    hipLaunchKernelGGL(moe_dispatch_kernel, dim3(1), dim3(DISPATCH_THREADS), lds, s, route, T, n, align, cap, counts, perm);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void gather_rows_kernel(u32x4 *__restrict__ out, const u32x4 *__restrict__ in,
                                                          const int *__restrict__ perm, int rows, int chunks)
{
    const u32x4 z = {0u, 0u, 0u, 0u};
    for (int r = blockIdx.x; r < rows; r += gridDim.x) {
        const int src = perm[r];
        for (int c = threadIdx.x; c < chunks; c += 256)
            out[(int64_t)r * chunks + c] = src >= 0 ? in[(int64_t)src * chunks + c] : z;
    }
}

__global__ __launch_bounds__(256) void scatter_rows_kernel(u32x4 *__restrict__ out, const u32x4 *__restrict__ in,
                                                           const int *__restrict__ perm, int rows, int chunks)
{
    for (int r = blockIdx.x; r < rows; r += gridDim.x) {
        const int dst = perm[r];
        if (dst < 0) continue;
        for (int c = threadIdx.x; c < chunks; c += 256) out[(int64_t)dst * chunks + c] = in[(int64_t)r * chunks + c];
    }
}

static hipError_t launch_rows(bool gather, void *out, const void *in, const int *perm, int rows, size_t row_bytes, hipStream_t s)
{
    if (rows <= 0 || row_bytes == 0) return hipSuccess;
    if ((row_bytes & 15) || ((uintptr_t)out & 15) || ((uintptr_t)in & 15) || (row_bytes >> 4) > 0x7fffffff)
        return hipErrorInvalidValue;
    const int chunks = (int)(row_bytes >> 4);
    const int blocks = rows < 8192 ? rows : 8192;
    if (gather)
        hipLaunchKernelGGL(gather_rows_kernel, dim3(blocks), dim3(256), 0, s, (u32x4 *)out, (const u32x4 *)in, perm, rows, chunks);
    else
        hipLaunchKernelGGL(scatter_rows_kernel, dim3(blocks), dim3(256), 0, s, (u32x4 *)out, (const u32x4 *)in, perm, rows, chunks);
    return hipGetLastError();
}

hipError_t launch_gather_rows(void *out, const void *in, const int *perm, int rows, size_t row_bytes, hipStream_t s)
{
    return launch_rows(true, out, in, perm, rows, row_bytes, s);
}

hipError_t launch_scatter_rows(void *out, const void *in, const int *perm, int rows, size_t row_bytes, hipStream_t s)
{
    return launch_rows(false, out, in, perm, rows, row_bytes, s);
}

// ---- bias gradient: column sums --------------------------------------------------------------
// colsum_block (rtp_ride.h) as a launch of its own
template <typename T, int VEC>
__global__ __launch_bounds__(COLSUM_THREADS) void colsum_kernel(const T *Y, int64_t ld, int rows, int cols, const float *in, float *out)
{
    __shared__ float lds[COLSUM_LDS_FLOATS];
    colsum_block<T, VEC, COLSUM_THREADS>(Y, ld, rows, cols, in, out, blockIdx.x, lds);
}

hipError_t launch_colsum(int elem, const void *Y, int64_t ld, int rows, int cols, const float *in, float *out, hipStream_t s)
{
    if (cols <= 0) return hipSuccess;
    if (rows < 0 || !in || !out || (rows > 0 && !Y)) return hipErrorInvalidValue;
    const dim3 grid((cols + COLSUM_COLS - 1) / COLSUM_COLS), block(COLSUM_THREADS);
    const bool wide = colsum_wide(Y, ld, cols);
    if (elem == ELEM_BF16 && wide)
        hipLaunchKernelGGL((colsum_kernel<__bf16, 8>), grid, block, 0, s, (const __bf16 *)Y, ld, rows, cols, in, out);
    else if (elem == ELEM_BF16)
        hipLaunchKernelGGL((colsum_kernel<__bf16, 1>), grid, block, 0, s, (const __bf16 *)Y, ld, rows, cols, in, out);
    else if (elem == ELEM_F16 && wide)
        hipLaunchKernelGGL((colsum_kernel<_Float16, 8>), grid, block, 0, s, (const _Float16 *)Y, ld, rows, cols, in, out);
    else if (elem == ELEM_F16)
        hipLaunchKernelGGL((colsum_kernel<_Float16, 1>), grid, block, 0, s, (const _Float16 *)Y, ld, rows, cols, in, out);
    else
        hipLaunchKernelGGL((colsum_kernel<float, 1>), grid, block, 0, s, (const float *)Y, ld, rows, cols, in, out);
    return hipGetLastError();
}

// ---- shader-clock probe -------------------------------------------------------------------
// Spins on the constant-rate wall clock for a bounded time and reports how many shader cycles
// went by.  One wave, a handful of registers: it fits beside any kernel.
__global__ void clock_probe_kernel(long long *out, long long wall_ticks)
{
    const long long w0 = wall_clock64(), c0 = clock64();
    long long w1 = w0;
    while (w1 - w0 < wall_ticks) w1 = wall_clock64();
    const long long c1 = clock64();
    if (threadIdx.x == 0) {
        out[0] = w1 - w0;
        out[1] = c1 - c0;
    }
}

hipError_t launch_clock_probe(long long *out, long long wall_ticks, hipStream_t s)
{
    hipLaunchKernelGGL(clock_probe_kernel, dim3(1), dim3(64), 0, s, out, wall_ticks);
    return hipGetLastError();
}

} // namespace rtp
