// float32 contraction: C_g[M,N_g] = epi(A_g[M,K] * W_g[N_g,K]^T) for a group of problems, the float32 validation mode's
// every linear layer.  Products and sums are float32 throughout (v_mfma_f32_32x32x2_f32; plain FMAs in the any-shape kernel).
//
// Three kernels, chosen by shape in launch_gemm_f32:
//   gemm_f32_mfma_kernel  operands through an LDS ring, 32x32 outputs per wavefront.  A K slice is 32 floats = 128 bytes per row, so
//                         the ring has the geometry of the bf16 kernel's 64-wide slices: global_load_lds of 16-byte chunks, chunk c of
//                         row r in slot c ^ (r & 7).  A lane reads 4 consecutive k of its row at once; since the order of k is
//                         free as long as both operands agree, MFMA i of a step takes k = i from the lower and k = 4 + i from
//                         the upper half wavefront.
//   gemm_f32_rows_kernel  few rows: bound by streaming the weights, which go straight from global memory to registers, each of
//                         the 4 wavefronts a quarter of K.
//   gemm_f32_any_kernel   any M, N, K and strides.
// The matrix cores' float32 rate is 256 FLOP per clock and compute unit, i.e. a 32x32x2 instruction takes 64 clocks while its
// operands are 512 bytes: the tile kernel is bound by the matrix cores and by how evenly the tiles divide over the compute
// units, so the smaller tile with K split over two wavefronts is taken until there are two rounds of the larger one.
// Measured at 576 rows against the any-shape kernel, which did everything before: 768 x 3072 and 768 x 768 columns x K 223 -> 25 us
// on average, 3072 x 768 136 -> 38 us, 8 problems of 768 x 3072 / 768 x 768 501 -> 163 us on average (83 TFLOP/s), 8 rows x 8
// problems 148 -> 18 us.
#include <algorithm>

#include "kernels.h"
#include "device_util.h"

namespace mt {

namespace {

typedef __attribute__((address_space(1))) const void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// acc of a 32x32 block (weight fragment first): row m = lane & 31, columns 8 q + 4 (lane >> 5) + {0..3} for q = 0..3
__device__ __forceinline__ void store_block_f32(const f32x16& acc, int m, int n_base, int M, int N, const float* bias, const float* res,
                                                int64_t ldr, float* C, int64_t ldc, int act)
{
    if (m >= M) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int n = n_base + q * 8;
        if (n >= N) continue;                              // N % 4 == 0: the four columns are all in or all out
        float4 v = make_float4(acc[q * 4 + 0], acc[q * 4 + 1], acc[q * 4 + 2], acc[q * 4 + 3]);
        if (bias) {
            const float4 b = *reinterpret_cast<const float4*>(bias + n);
            v.x += b.x; v.y += b.y; v.z += b.z; v.w += b.w;
        }
        if (act != ACT_NONE) {
            v.x = apply_act(v.x, act);
            v.y = apply_act(v.y, act);
            v.z = apply_act(v.z, act);
            v.w = apply_act(v.w, act);
        }
        if (res) {
            const float4 r = *reinterpret_cast<const float4*>(res + (size_t)m * ldr + n);
            v.x += r.x; v.y += r.y; v.z += r.z; v.w += r.w;
        }
        *reinterpret_cast<float4*>(C + (size_t)m * ldc + n) = v;
    }
}

// WM x WN wavefronts of 32x32 outputs, each with WK wavefronts that share its K range.
template <int WM, int WN, int WK, int STAGES>
__global__ __launch_bounds__(256, 2) void gemm_f32_mfma_kernel(GemmGroup g, GemmShape s)
{
    constexpr int BM = 32 * WM, BN = 32 * WN, SUB = BM + BN, ROWS = SUB * WK;          // rows of 128 bytes per stage
    constexpr int STAGE = ROWS * 128, LPS = ROWS / 8 / 4;                               // load instructions per wavefront and slice
    static_assert(WM * WN * WK == 4 && ROWS % 32 == 0, "four wavefronts");
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int grp = blockIdx.z;
    const int N = g.N[grp];
    const int M = s.d_M ? min(s.M, *s.d_M) : s.M;      // rows actually present; the grid covers the bound s.M
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    if (n0 >= N || m0 >= M) return;
    const unsigned char* A = static_cast<const unsigned char*>(g.A[grp]);
    const unsigned char* W = static_cast<const unsigned char*>(g.W[grp]);
    const uint32_t lda_b = (uint32_t)s.lda * 4, ldw_b = (uint32_t)(s.ldw ? s.ldw : s.K) * 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int wk = wave % WK, wn = (wave / WK) % WN, wm = wave / WK / WN;

    // load i of a wavefront fills stage rows (wave + 4 i) * 8 .. + 7: sub-slice row / SUB, in it BM rows of A, then BN of W
    const unsigned char* src[LPS];
#pragma unroll
    for (int i = 0; i < LPS; ++i) {
        const int row = (wave + i * 4) * 8 + (lane >> 3);
        const int sub = row / SUB, r = row - sub * SUB;
        const int off = sub * 128 + (((lane & 7) ^ (row & 7)) << 4);
        src[i] = r < BM ? A + (size_t)min(m0 + r, M - 1) * lda_b + off : W + (size_t)min(n0 + r - BM, N - 1) * ldw_b + off;
    }
    const int KT = s.K / (32 * WK);
    auto issue = [&](int kt) {
        unsigned char* base = lds + (kt % STAGES) * STAGE;
#pragma unroll
        for (int i = 0; i < LPS; ++i)
            __builtin_amdgcn_global_load_lds((gptr_t)(src[i] + (size_t)kt * (128 * WK)), (lptr_t)(base + (wave + i * 4) * 1024), 16, 0, 0);
    };
    const int a_row = wk * SUB + wm * 32 + l32, w_row = wk * SUB + BM + wn * 32 + l32;
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
    for (int p = 0; p < STAGES - 1; ++p)
        if (p < KT) issue(p);
    for (int kt = 0; kt < KT; ++kt) {
        // slice kt has landed when at most the slices after it are outstanding; the fragments of slice kt - 1 are in registers
        if (kt + STAGES - 2 < KT) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(LPS * (STAGES - 2)) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();                   // ... for every wavefront
        asm volatile("" ::: "memory");
        if (kt + STAGES - 1 < KT) issue(kt + STAGES - 1);
        const unsigned char* sb = lds + (kt % STAGES) * STAGE;
        f32x4 af[4], wf[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            af[c] = *reinterpret_cast<const f32x4*>(sb + a_row * 128 + (((c * 2 + half) ^ (a_row & 7)) << 4));
            wf[c] = *reinterpret_cast<const f32x4*>(sb + w_row * 128 + (((c * 2 + half) ^ (w_row & 7)) << 4));
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[c][i], af[c][i], acc, 0, 0, 0);
    }
    if constexpr (WK > 1) {                             // partial sums of the other K shares, added in a fixed order
        __syncthreads();
        float* part = reinterpret_cast<float*>(lds);
        if (wk > 0) {
#pragma unroll
            for (int e = 0; e < 16; ++e) part[(((wm * WN + wn) * (WK - 1) + wk - 1) * 16 + e) * 64 + lane] = acc[e];
        }
        __syncthreads();
        if (wk > 0) return;
#pragma unroll
        for (int w = 0; w < WK - 1; ++w)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[e] += part[(((wm * WN + wn) * (WK - 1) + w) * 16 + e) * 64 + lane];
    }
    store_block_f32(acc, m0 + wm * 32 + l32, n0 + wn * 32 + half * 4, M, N, g.bias[grp], g.residual[grp], s.ldr,
                    static_cast<float*>(g.C[grp]), s.ldc, s.act);
}

// 32 rows x 32 columns per workgroup, a quarter of K per wavefront, operands straight into registers.
__global__ __launch_bounds__(256) void gemm_f32_rows_kernel(GemmGroup g, GemmShape s)
{
    __shared__ __attribute__((aligned(16))) float part[3 * 16 * 64];
    constexpr int U = 12;                               // steps of 8 k in flight
    const int grp = blockIdx.z;
    const int N = g.N[grp];
    const int M = s.d_M ? min(s.M, *s.d_M) : s.M;
    const int m0 = blockIdx.y * 32, n0 = blockIdx.x * 32;
    if (n0 >= N || m0 >= M) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, half = lane >> 5;
    const int k_len = s.K / 4;
    const float* __restrict__ a = static_cast<const float*>(g.A[grp]) + (size_t)min(m0 + l32, M - 1) * s.lda + wave * k_len + half * 4;
    const float* __restrict__ w = static_cast<const float*>(g.W[grp]) + (size_t)min(n0 + l32, N - 1) * (s.ldw ? s.ldw : s.K) + wave * k_len + half * 4;
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    const int steps = k_len / 8;
    for (int st = 0; st < steps; st += U) {
        f32x4 af[U], wf[U];
        const int nb = steps - st;                      // uniform over the workgroup
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (u < nb) {
                af[u] = *reinterpret_cast<const f32x4*>(a + (st + u) * 8);
                wf[u] = *reinterpret_cast<const f32x4*>(w + (st + u) * 8);
            }
        __builtin_amdgcn_sched_barrier(0);              // all loads of the batch are in flight before the first product
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (u < nb) {
#pragma unroll
                for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[u][i], af[u][i], acc, 0, 0, 0);
            }
    }
    if (wave > 0) {
#pragma unroll
        for (int e = 0; e < 16; ++e) part[((wave - 1) * 16 + e) * 64 + lane] = acc[e];
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int v = 0; v < 3; ++v)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] += part[(v * 16 + e) * 64 + lane];
    store_block_f32(acc, m0 + l32, n0 + half * 4, M, N, g.bias[grp], g.residual[grp], s.ldr, static_cast<float*>(g.C[grp]), s.ldc, s.act);
}

// Any M, N, K, strides: 64x64 outputs per workgroup, 4x4 per thread, K staged through LDS in slices of 16, loads outside the
// problem zero-filled, stores bounds-checked.
constexpr int TM = 64, TN = 64, TK = 16;
__global__ __launch_bounds__(256) void gemm_f32_any_kernel(GemmGroup g, GemmShape s)
{
    __shared__ float As[TK][TM + 4];
    __shared__ float Ws[TK][TN + 4];
    const int grp = blockIdx.z;
    const int N = g.N[grp];
    const int M = s.d_M ? min(s.M, *s.d_M) : s.M;
    const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TN;
    if (n0 >= N || m0 >= M) return;
    const float* A = static_cast<const float*>(g.A[grp]);
    const float* W = static_cast<const float*>(g.W[grp]);
    const size_t ldw = s.ldw ? s.ldw : s.K;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int lr = threadIdx.x >> 2;          // 0..63: tile row loaded by this thread
    const int lk = (threadIdx.x & 3) * 4;     // 0,4,8,12: first of 4 k's
    float acc[4][4] = {};
    for (int k0 = 0; k0 < s.K; k0 += TK) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = k0 + lk + j;
            const int am = m0 + lr, wn = n0 + lr;
            As[lk + j][lr] = (am < M && k < s.K) ? A[(size_t)am * s.lda + k] : 0.f;
            Ws[lk + j][lr] = (wn < N && k < s.K) ? W[(size_t)wn * ldw + k] : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < TK; ++k) {
            float a[4], w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { a[i] = As[k][ty * 4 + i]; w[i] = Ws[k][tx * 4 + i]; }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], w[j], acc[i][j]);
        }
        __syncthreads();
    }
    float* C = static_cast<float*>(g.C[grp]);
    const float* bias = g.bias[grp];
    const float* res = g.residual[grp];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = m0 + ty * 4 + i;
        if (m >= M) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int n = n0 + tx * 4 + j;
            if (n >= N) continue;
            float v = acc[i][j] + (bias ? bias[n] : 0.f);
            v = apply_act(v, s.act);
            if (res) v += res[(size_t)m * s.ldr + n];
            C[(size_t)m * s.ldc + n] = v;
        }
    }
}

template <int WM, int WN, int WK, int STAGES>
hipError_t launch_mfma(const GemmGroup& g, const GemmShape& s, hipStream_t stream)
{
    constexpr int bytes = STAGES * 32 * (WM + WN) * WK * 128;
    static std::atomic<uint64_t> lds_raised{0};
    if (bytes > 64 * 1024) {
        hipError_t e = ensure_dynamic_lds((const void*)gemm_f32_mfma_kernel<WM, WN, WK, STAGES>, bytes, lds_raised);
        if (e != hipSuccess) return e;
    }
    dim3 grid((s.N + 32 * WN - 1) / (32 * WN), (s.M + 32 * WM - 1) / (32 * WM), s.G), block(256);
    hipLaunchKernelGGL((gemm_f32_mfma_kernel<WM, WN, WK, STAGES>), grid, block, bytes, stream, g, s);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_f32(const GemmGroup& g, const GemmShape& s, hipStream_t stream)
{
    if (s.G <= 0 || s.M <= 0 || s.N <= 0) return hipSuccess;
    // the matrix-core kernels move 16-byte chunks of whole 128-byte (64 for two K shares: 256-byte) slices
    bool chunks = s.K % 64 == 0 && s.N % 4 == 0 && s.lda % 4 == 0 && s.ldw % 4 == 0 && s.ldc % 4 == 0 && s.ldr % 4 == 0 &&
                  (uint64_t)s.lda * 4 < (1ull << 32) && (uint64_t)s.ldw * 4 < (1ull << 32);
    for (int i = 0; chunks && i < s.G; ++i)
        chunks = g.N[i] % 4 == 0 && (((uintptr_t)g.A[i] | (uintptr_t)g.W[i] | (uintptr_t)g.C[i] | (uintptr_t)g.bias[i] | (uintptr_t)g.residual[i]) & 15) == 0;
    if (!chunks) {
        dim3 grid((s.N + TN - 1) / TN, (s.M + TM - 1) / TM, s.G), block(256);
        hipLaunchKernelGGL(gemm_f32_any_kernel, grid, block, 0, stream, g, s);
        return hipGetLastError();
    }
    if (s.M <= 32) {
        dim3 grid((s.N + 31) / 32, (s.M + 31) / 32, s.G), block(256);
        hipLaunchKernelGGL(gemm_f32_rows_kernel, grid, block, 0, stream, g, s);
        return hipGetLastError();
    }
    // Blocks of 32 x 32, one per workgroup, its wavefronts a quarter of K each; otherwise two blocks and half of K.  While every block has a compute unit
    // that is 1.3 to 1.8 times as fast (240 blocks of one problem, K = 768: 8.8 and 12.1 us, 3072: 20.5 and 35.8; 256 blocks of 8 problems 8.7 and
    // 12.2, 24.1 and 35.8; K = 256 level).  Up to one and a half times as many it is a little ahead for one problem (264 to 384 blocks, K = 768: 11.7
    // to 12.0 and 12.1 to 12.2, 3072: 33.9 to 34.5 and 35.8), while several problems at K = 768 lose (320 and 384 blocks of 8: 12.6 and 12.2, 12.9 and 12.3).
    // By the problems with all tasks enabled: a task's logits are the same bits whichever others are.
    const long plan = std::max(s.plan, s.G), blocks = plan * ((s.M + 31) / 32) * ((s.N + 31) / 32), n_cu = device_cu_count();
    if (blocks <= (plan == 1 ? n_cu * 3 / 2 : n_cu) && s.K % 128 == 0) return launch_mfma<1, 1, 4, 2>(g, s, stream);
    const long tiles64 = (long)s.G * ((s.M + 63) / 64) * ((s.N + 63) / 64);
    if (tiles64 >= 1024) return launch_mfma<2, 2, 1, 4>(g, s, stream);
    return launch_mfma<1, 2, 2, 3>(g, s, stream);
}

}  // namespace mt
