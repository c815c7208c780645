// float32 contraction: C_g[M,N_g] = epi(A_g[M,K] * W_g[N_g,K]^T) for a group of problems, the float32 validation mode's
// every linear layer.  Products and sums are float32 throughout (v_mfma_f32_32x32x2_f32; plain FMAs in the any-shape kernel).
//
// Three kernels, chosen by shape in launch_gemm_f32:
//   gemm_f32_tile_kernel  32x32 blocks, a quarter of K per wavefront, operands through an LDS ring of each wavefront's own.  A K slice is
//                         32 floats = 128 bytes per row: buffer loads to LDS of 16-byte chunks, chunk c of row r in slot c ^ (r & 7).  A
//                         lane reads 4 consecutive k of its row at once; since the order of k is free as long as both operands agree, MFMA i
//                         of a step takes k = i from the lower and k = 4 + i from the upper half wavefront.
//   gemm_f32_short_kernel short K (of 2, 4 or 6 slices, too few for four rings; of 8 and 10 in large launches): all or most slices of a workgroup's operands in LDS at once.  Operands
//                         straight from global memory to registers instead, 32 bytes of a row at a time: 2048 rows x 4 K columns, 8 problems,
//                         K = 64 / 128 / 192 21, 51, 99 us, here 12, 31, 55.
//   gemm_f32_any_kernel   any M, N, K and strides.
// The matrix cores' float32 rate is 256 FLOP per clock and compute unit: a 32x32x2 instruction takes 64 clocks.  What the tile kernel has to do is to
// keep them coming.
//   - One block per workgroup is the finest split that needs no second pass: 753 rows x 768 columns are 576 blocks, 2.25 for each compute unit, so the
//     busiest has 3, where pairs of blocks (264 to 288 workgroups) or 64x64 tiles leave the time of 4 (768 x 3072: 43 us, 63 us before).
//   - A wavefront issues in order, and a load whose issue is held up holds up its matrix instructions: loads and LDS reads go one by one between
//     them (all of a slice's loads at its start: 53 us), and nothing in the loop branches, divides or waits for another wavefront (no barrier: a
//     wavefront reads what it has loaded itself).  1190 clocks a slice with one wavefront per SIMD, 1024 being the matrix instructions; two
//     workgroups per compute unit fill the rest.
//   - Workgroups walk a list of blocks; the first slices of the next block are under way during the last ones of a block, whose sums are put together
//     and stored behind the next one's matrix instructions.
// 753 rows x 2304 / 768 / 3072 (GELU) x 768, x 768 x 3072: 32, 14, 42, 43 us (82 TFLOP/s); the ring shared by a workgroup, fragments read behind its
// barrier and multiplied at once, 40, 20, 56, 63.  8 problems: 213, 72, 307, 263 us (101 TFLOP/s at a clock of 1.95 GHz), before 212, 92, 303, 330.
// 8 problems of 75 rows 29, 15, 39, 44; 38, 20, 60, 62.
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

__device__ __forceinline__ __amdgpu_buffer_rsrc_t f_rsrc(const void* base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}

constexpr int kRing = 2, kStage = 64 * 128, kExchange = 16 * 1024;      // stages, bytes of one (32 rows of A, 32 of W), exchanged partial sums
constexpr int kTileLds = 4 * kRing * kStage + kExchange;

// One 32x32 block at a time, a quarter of K per wavefront, two workgroups per compute unit.
__device__ __forceinline__ void gemm_f32_tile_body(const GemmGroup& g, const GemmShape& s, unsigned char* lds)
{
    const int M = s.d_M ? min(s.M, *s.d_M) : s.M;      // rows actually present; the grid covers the bound s.M
    const int tiles_n = (s.N + 31) >> 5, per_problem = ((M + 31) >> 5) * tiles_n, total = per_problem * s.G;
    if ((int)blockIdx.x >= total) return;
    const uint32_t lda_b = (uint32_t)s.lda * 4, ldw_b = (uint32_t)(s.ldw ? s.ldw : s.K) * 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    // this wavefront's slices of 32 k: a quarter of them, the first quarters one more where four do not divide them.  Of the two workgroups of a compute unit one
    // has the longer quarters on its first two SIMDs and the other on its last two (8 problems of 1200 rows x 1728 x 576 198 -> 189 us).
    const int share = (wave + (blockIdx.x >= gridDim.x / 2 ? 2 : 0)) & 3;
    const int slices = s.K >> 5, KT = (slices >> 2) + (share < (slices & 3) ? 1 : 0);
    const int k0 = ((slices >> 2) * share + min(share, slices & 3)) * 128;

    struct Ref {
        __amdgpu_buffer_rsrc_t A, W;                   // from the block's first row on; rows beyond the last one read as zero
        int grp, m0, n0;
    };
    auto locate = [&](int tile) {
        Ref t;
        t.grp = tile / per_problem;
        const int tt = tile - t.grp * per_problem, tm = tt / tiles_n;
        t.m0 = tm * 32;
        t.n0 = (tt - tm * tiles_n) * 32;
        const int rows_w = g.N[t.grp] - t.n0;          // none: a problem of fewer columns than the widest
        t.A = f_rsrc(static_cast<const unsigned char*>(g.A[t.grp]) + (size_t)t.m0 * lda_b, (min(32, M - t.m0) - 1) * lda_b + s.K * 4);
        t.W = f_rsrc(static_cast<const unsigned char*>(g.W[t.grp]) + (size_t)t.n0 * ldw_b, rows_w > 0 ? (min(32, rows_w) - 1) * ldw_b + s.K * 4 : 0);
        return t;
    };
    // load i of a slice fills 8 rows of 128 bytes, chunk c of row r in slot c ^ (r & 7)
    int va[4], vw[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = i * 8 + (lane >> 3), off = ((lane & 7) ^ (r & 7)) << 4;
        va[i] = r * lda_b + off;
        vw[i] = r * ldw_b + off;
    }
    unsigned char* mine = lds + wave * (kRing * kStage);
    auto issue = [&](const Ref& t, int kt, int st, int i) {
        unsigned char* to = mine + st * kStage + i * 1024;
        if (i < 4) __builtin_amdgcn_raw_ptr_buffer_load_lds(t.A, (lptr_t)to, 16, va[i & 3], k0 + kt * 128, 0, 0);
        else __builtin_amdgcn_raw_ptr_buffer_load_lds(t.W, (lptr_t)to, 16, vw[i & 3], k0 + kt * 128, 0, 0);
    };
    f32x4 af[4], wf[4];
    int ro[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) ro[c] = l32 * 128 + (((c * 2 + half) ^ (l32 & 7)) << 4);
    auto read = [&](int st, int c) {
        const unsigned char* p = mine + st * kStage + ro[c];
        af[c] = *reinterpret_cast<const f32x4*>(p);
        wf[c] = *reinterpret_cast<const f32x4*>(p + 4096);
    };
    f32x16 acc;
    auto mul = [&](int c, int i) {
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[c][i], af[c][i], acc, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };

    // A finished block's partial sums wait in LDS until the second slice of the next block, whose matrix instructions cover the sum, the activation and the store.
    float* const part = reinterpret_cast<float*>(lds + 4 * kRing * kStage);
    struct Out {
        int grp, m, n;
        bool ok;
        f32x4 bias;
    };
    f32x4 v;
    auto exchange = [&]() {                                              // this wavefront's share
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();                                    // everyone has read the block before
        asm volatile("" ::: "memory");
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<f32x4*>(part + ((share * 4 + q) * 64 + lane) * 4) = f32x4{acc[q * 4], acc[q * 4 + 1], acc[q * 4 + 2], acc[q * 4 + 3]};
    };
    auto gather = [&]() {                                                // columns 8 wave .. + 7 of the block, added in a fixed order
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        f32x4 p[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) p[w] = *reinterpret_cast<const f32x4*>(part + ((w * 4 + wave) * 64 + lane) * 4);
        v = p[0] + p[1] + p[2] + p[3];
    };
    auto store = [&](const Out& o) {
        if (!o.ok) return;
        if (g.residual[o.grp]) v += *reinterpret_cast<const f32x4*>(g.residual[o.grp] + (size_t)o.m * s.ldr + o.n);
        *reinterpret_cast<f32x4*>(static_cast<float*>(g.C[o.grp]) + (size_t)o.m * s.ldc + o.n) = v;
    };
    int st = 0;
    // A slice: the loads two slices ahead (left = 2) and the fragments of the next one (left > 0) between its products, and extra(i) behind product i.
    auto slice = [&](const Ref& t, int kn, auto left, auto extra) {
        constexpr int L = decltype(left)::value;
        auto next = [&](int c) {
            if constexpr (L > 0) read(st, c);
            __builtin_amdgcn_sched_barrier(0);
        };
        __builtin_amdgcn_sched_barrier(0);
        mul(0, 0);
        extra(0);
        mul(0, 1);
        extra(1);
        mul(0, 2);
        extra(2);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");               // this slice is in registers, its stage is free
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if constexpr (L == kRing) issue(t, kn, st, i);
            __builtin_amdgcn_sched_barrier(0);
            mul((3 + i) >> 2, (3 + i) & 3);
            extra(3 + i);
        }
        st ^= 1;
        if constexpr (L > 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(8 * (L - 1)) : "memory");      // the next slice has landed
        next(0);
        mul(2, 3);
        extra(11);
        next(1);
        mul(3, 0);
        extra(12);
        next(2);
        mul(3, 1);
        extra(13);
        mul(3, 2);
        mul(3, 3);
        next(3);
    };
    auto nothing = [](int) {};

    Ref cur = locate(blockIdx.x);
#pragma unroll
    for (int p = 0; p < kRing; ++p)
#pragma unroll
        for (int i = 0; i < 8; ++i) issue(cur, p, p, i);
    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
#pragma unroll
    for (int c = 0; c < 4; ++c) read(0, c);
    Out prev;
    prev.ok = false;
    for (int tile = blockIdx.x; tile < total; tile += gridDim.x) {
        // The last slices of a block fetch the next one's first.  Without a next one they fetch nothing, or (of so few slices that these are also the first
        // ones) this block's again, never read.
        const bool more = tile + (int)gridDim.x < total;
        const Ref nxt = more ? locate(tile + gridDim.x) : cur;
        Out out;
        out.grp = cur.grp;
        out.m = cur.m0 + l32;
        out.n = cur.n0 + wave * 8 + half * 4;
        out.ok = out.m < M && out.n < g.N[cur.grp];
        out.bias = f32x4{0.f, 0.f, 0.f, 0.f};
        if (g.bias[cur.grp] && out.ok) out.bias = *reinterpret_cast<const f32x4*>(g.bias[cur.grp] + out.n);
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = 0.f;
        auto ahead = [&](int kt, auto extra) {
            const bool here = kt + kRing < KT;
            const Ref t = here ? cur : nxt;
            slice(t, here ? kt + kRing : kt + kRing - KT, std::integral_constant<int, kRing>{}, extra);
        };
        ahead(0, [&](int i) {
            if (i == 11) asm volatile("" : "+v"(out.bias));               // here its load is awaited anyway; later the wait would be for the ring's too
        });
        if (tile != (int)blockIdx.x) {
            gather();
            ahead(1, [&](int i) {
                if (i == 0) v += prev.bias;
                if (s.act != ACT_NONE && i >= 1 && i <= 10 && i % 3 == 1) v[i / 3] = apply_act(v[i / 3], s.act);
                if (i == 12) store(prev);
            });
        } else {
            ahead(1, nothing);
        }
        const bool drain = !more && KT >= 2 * kRing;
        for (int kt = 2; kt < (drain ? KT - kRing : KT); ++kt) ahead(kt, nothing);
        if (drain) {
            slice(cur, 0, std::integral_constant<int, 1>{}, nothing);
            slice(cur, 0, std::integral_constant<int, 0>{}, nothing);
        }
        exchange();
        prev = out;
        cur = nxt;
    }
    gather();
    v += prev.bias;
    if (s.act != ACT_NONE)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = apply_act(v[e], s.act);
    store(prev);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // loads must land before the LDS is released
}

__global__ __launch_bounds__(256, 2) void gemm_f32_tile_kernel(GemmGroup g, GemmShape s)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    gemm_f32_tile_body(g, s, lds);
}

// The quarter of K = 32 Q that a step of 8 k belongs to: Q steps each, from 8 slices on whole slices, the first ones one more where four do not divide them (the
// shares of gemm_f32_tile_kernel).
template <int Q>
constexpr int quarter_of(int step)
{
    if (Q < 8) return step / Q;
    const int slice = step >> 2, longer = (Q / 4 + 1) * (Q % 4);
    return slice < longer ? slice / (Q / 4 + 1) : Q % 4 + (slice - longer) / (Q / 4);
}

// K = 32 Q, Q = 2, 4, .. 10: WM x WN wavefronts of 32 x 32 outputs, each with WK that share its K, slices of 32 k through a shared LDS ring.  Quarters of K are
// summed apart and added up in their order however many wavefronts they belong to: the same bits in every form.
template <int Q, int WM, int WN, int WK>
__global__ __launch_bounds__(256, 2) void gemm_f32_short_kernel(GemmGroup g, GemmShape s)
{
    constexpr int BM = 32 * WM, BN = 32 * WN, SUB = BM + BN, STAGE = SUB * WK * 128;     // 128-byte rows: BM of A, BN of W, of every share
    constexpr int KT = Q / WK, STAGES = KT * STAGE <= 65536 ? KT : 65536 / STAGE;
    constexpr int LPS = SUB * WK / 32, QUARTERS = 4 / WK, PART = QUARTERS * 16 * 64;     // loads of a wavefront and slice; floats of its partial sums
    static_assert(WM * WN * WK == 4 && Q % WK == 0 && WM * WN * (WK - 1) * PART * 4 <= STAGES * STAGE, "four wavefronts, whole slices");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[STAGES * STAGE];
    const int grp = blockIdx.z;
    const int N = g.N[grp];
    const int M = s.d_M ? min(s.M, *s.d_M) : s.M;
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    if (n0 >= N || m0 >= M) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5, wk = wave % WK, wn = wave / WK % WN, wm = wave / WK / WN;
    const size_t lda = s.lda, ldw = s.ldw ? s.ldw : s.K;
    // load i of a slice: 32 rows, 8 per wavefront, chunk c of row r in slot c ^ (r & 7); rows beyond the last one repeat it
    const int r8 = wave * 8 + (lane >> 3), off = ((lane & 7) ^ (lane >> 3)) * 4;
    const float* src[LPS];
#pragma unroll
    for (int i = 0; i < LPS; ++i) {
        const int share = i * 32 / SUB, r = i * 32 % SUB, k0 = share * (KT * 32) + off;
        src[i] = r < BM ? static_cast<const float*>(g.A[grp]) + min(m0 + r + r8, M - 1) * lda + k0 : static_cast<const float*>(g.W[grp]) + min(n0 + r - BM + r8, N - 1) * ldw + k0;
    }
    auto issue = [&](int kt) {
#pragma unroll
        for (int i = 0; i < LPS; ++i)
            __builtin_amdgcn_global_load_lds((gptr_t)(src[i] + kt * 32), (lptr_t)(lds + (kt % STAGES) * STAGE + (i * 4 + wave) * 1024), 16, 0, 0);
    };
#pragma unroll
    for (int kt = 0; kt < STAGES; ++kt) issue(kt);
    const int a_row = wk * SUB + wm * 32 + l32, w_row = wk * SUB + BM + wn * 32 + l32;
    f32x16 acc[QUARTERS];
    auto slice = [&](auto ktc) {
        constexpr int kt = decltype(ktc)::value;
        if constexpr (kt < KT) {
            // it has landed when at most the slices issued after it are outstanding; the fragments of the slice before are in registers
            constexpr int issued = kt < 2 || STAGES == KT ? STAGES : (KT < STAGES + kt - 1 ? KT : STAGES + kt - 1);
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(LPS * (issued - kt - 1)) : "memory");
            __builtin_amdgcn_s_barrier();                   // ... for every wavefront
            asm volatile("" ::: "memory");
            if constexpr (kt > 0 && kt - 1 + STAGES < KT) issue(kt - 1 + STAGES);
            const unsigned char* sb = lds + (kt % STAGES) * STAGE;
            f32x4 af[4], wf[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                af[c] = *reinterpret_cast<const f32x4*>(sb + a_row * 128 + (((c * 2 + half) ^ (a_row & 7)) << 4));
                wf[c] = *reinterpret_cast<const f32x4*>(sb + w_row * 128 + (((c * 2 + half) ^ (w_row & 7)) << 4));
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                f32x16& q = acc[quarter_of<Q>(kt * 4 + c)];
                if (kt + c == 0 || quarter_of<Q>(kt * 4 + c) != quarter_of<Q>(kt * 4 + c - 1)) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) q[e] = 0.f;
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) q = __builtin_amdgcn_mfma_f32_32x32x2f32(wf[c][i], af[c][i], q, 0, 0, 0);
            }
        }
    };
    slice(std::integral_constant<int, 0>{});
    slice(std::integral_constant<int, 1>{});
    slice(std::integral_constant<int, 2>{});
    slice(std::integral_constant<int, 3>{});
    slice(std::integral_constant<int, 4>{});
    slice(std::integral_constant<int, 5>{});
    slice(std::integral_constant<int, 6>{});
    slice(std::integral_constant<int, 7>{});
    slice(std::integral_constant<int, 8>{});
    slice(std::integral_constant<int, 9>{});
    static_assert(KT <= 10, "slices");
    if constexpr (WK > 1) {
        float* part = reinterpret_cast<float*>(lds) + (wm * WN + wn) * (WK - 1) * PART + lane;
        __syncthreads();
        if (wk > 0) {
#pragma unroll
            for (int q = 0; q < QUARTERS; ++q)
#pragma unroll
                for (int e = 0; e < 16; ++e) part[(wk - 1) * PART + (q * 16 + e) * 64] = acc[q][e];
        }
        __syncthreads();
        if (wk > 0) return;
#pragma unroll
        for (int q = 1; q < QUARTERS; ++q) acc[0] += acc[q];
#pragma unroll
        for (int q = 0; q < (WK - 1) * QUARTERS; ++q)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[0][e] += part[(q * 16 + e) * 64];
    } else {
#pragma unroll
        for (int q = 1; q < QUARTERS; ++q) acc[0] += acc[q];
    }
    store_block_f32(acc[0], m0 + wm * 32 + l32, n0 + wn * 32 + half * 4, M, N, g.bias[grp], g.residual[grp], s.ldr, static_cast<float*>(g.C[grp]), s.ldc, s.act);
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

}  // namespace

hipError_t launch_gemm_f32(const GemmGroup& g, const GemmShape& s, hipStream_t stream)
{
    if (s.G <= 0 || s.M <= 0 || s.N <= 0) return hipSuccess;
    // the matrix-core kernels move 16-byte chunks of whole slices; offsets inside a block's 32 rows are 31-bit
    bool chunks = s.K % 64 == 0 && s.N % 4 == 0 && s.lda % 4 == 0 && s.ldw % 4 == 0 && s.ldc % 4 == 0 && s.ldr % 4 == 0 &&
                  (uint64_t)s.lda * 128 < (1ull << 31) && (uint64_t)(s.ldw ? s.ldw : s.K) * 128 < (1ull << 31);
    for (int i = 0; chunks && i < s.G; ++i)
        chunks = g.N[i] % 4 == 0 && (((uintptr_t)g.A[i] | (uintptr_t)g.W[i] | (uintptr_t)g.C[i] | (uintptr_t)g.bias[i] | (uintptr_t)g.residual[i]) & 15) == 0;
    if (!chunks) {
        dim3 grid((s.N + TN - 1) / TN, (s.M + TM - 1) / TM, s.G), block(256);
        hipLaunchKernelGGL(gemm_f32_any_kernel, grid, block, 0, stream, g, s);
        return hipGetLastError();
    }
    // Each wavefront's quarter has as many slices as the ring of the tile kernel; fewer: the short-K forms.  Up to 512 blocks (two for each compute unit; K = 192:
    // 1536) a launch is a chain of latencies, which K dealt out to wavefronts shortens (3 problems of 128 rows x 4 K columns, K = 128 / 192 4.8, 5.5 us, 64 x
    // 64 outputs 5.8, 7.0; 8 problems of 200 rows x 576 x 192 9.6 and 10.9).  Beyond, 64 x 64 outputs read the operands half as often (8 problems of 2048
    // rows, K = 64 / 128 / 192 12, 31, 55 us, with K dealt out 14, 40, 62).  So they do in large launches of the shortest K of the tile kernel, whose blocks are
    // mostly fill, exchange and uneven quarters there (8 problems of 2300 rows x 1024 x 256 / 1280 x 320 94, 141 us, the tile kernel 104, 161; of 750 rows x 768 x
    // 256, 4608 blocks, 30 both).
    const long blocks = (long)s.G * ((s.M + 31) / 32) * ((s.N + 31) / 32);
    if (s.K < 4 * 32 * kRing || (s.K <= 320 && blocks > 4700 && (s.M + 63) / 64 <= 65535)) {
        const bool few = blocks <= (s.K == 192 ? 1536 : 512);
        auto launch = [&](auto kernel, int bm, int bn) {
            hipLaunchKernelGGL(kernel, dim3((s.N + bn - 1) / bn, (s.M + bm - 1) / bm, s.G), dim3(256), 0, stream, g, s);
            return hipGetLastError();
        };
        switch (s.K) {
            case 64: return few ? launch(gemm_f32_short_kernel<2, 1, 2, 2>, 32, 64) : launch(gemm_f32_short_kernel<2, 2, 2, 1>, 64, 64);
            case 128: return few ? launch(gemm_f32_short_kernel<4, 1, 1, 4>, 32, 32) : launch(gemm_f32_short_kernel<4, 2, 2, 1>, 64, 64);
            case 192: return few ? launch(gemm_f32_short_kernel<6, 1, 2, 2>, 32, 64) : launch(gemm_f32_short_kernel<6, 2, 2, 1>, 64, 64);
            case 256: return launch(gemm_f32_short_kernel<8, 2, 2, 1>, 64, 64);
            default: return launch(gemm_f32_short_kernel<10, 2, 2, 1>, 64, 64);
        }
    }
    static std::atomic<uint64_t> lds_raised{0};
    hipError_t e = ensure_dynamic_lds((const void*)gemm_f32_tile_kernel, kTileLds, lds_raised);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(gemm_f32_tile_kernel, dim3((unsigned)std::min(blocks, 2l * device_cu_count())), dim3(256), kTileLds, stream, g, s);
    return hipGetLastError();
}

}  // namespace mt
