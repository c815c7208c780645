// First-token attention of a branch's last layer on the panel layout, keys and values not projected (bfloat16 path): with
// q~[b][a] = Wk_a^T (Wq_a x_b + bq_a) the score of key j is q~ . x_j up to a constant that the softmax drops, and the head's context
// is Wv_a (sum_j p_j x_j) + bv_a.  Two launches per group of tasks (the contexts are one more, gemm_tiled_rows_kernel):
//   first_query_kernel   one workgroup per (task, 32 sequences, head): query of the sequences' first rows (gathered before: in place, 16
//                        bytes of a line at a time, every head's workgroup paid for them, 19.5 us for 8 tasks x 32 sequences), then q~, the 64 columns between them staying in LDS.  Bound by the two weight slices (98 KB each), all of whose
//                        fragments are in flight at once.
//   first_attend_kernel  one workgroup per (task, sequence): scores, softmax and weighted row sums in one pass over the sequence's rows, 32
//                        keys at a time with a running maximum; a key block is loaded while the one before is worked on.  The sums are
//                        float32 on the vector units: 2 H FMAs per key and head are what bounds it.
// Scores and sums were two kernels that read the rows once each (85 + 107 us for 8 tasks x 256 sequences).
#include "kernels.h"
#include "device_util.h"

namespace mt {

namespace {

constexpr int kHeadsPad = 16;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256, 1) void first_query_kernel(FirstTokenGroup g, int B, int H)
{
    constexpr int U = 12, MAXP = 8;
    __shared__ __attribute__((aligned(16))) float part[4][2][4][64][4];
    __shared__ __attribute__((aligned(16))) __bf16 qs[8 * 256];              // 64 columns of 32 rows, panel layout
    const int a = blockIdx.x, grp = blockIdx.z, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int b0 = blockIdx.y * 32, panels = H >> 5;
    const size_t pw = (size_t)H * 64;                                        // bytes per panel
    const int steps = H / 64;                                                // K steps of 16 of a wavefront
    const unsigned char* wq = static_cast<const unsigned char*>(g.Wq[grp]) + (size_t)a * 2 * pw + (size_t)wave * steps * 1024 + lane * 16;
    const unsigned char* wk = static_cast<const unsigned char*>(g.WkT[grp]) + (size_t)a * 4096 + lane * 16;
    // the key matrix's fragments for this wavefront's panels of q~ (wave, wave + 4, ..): needed last, in flight first
    bf16x8 kf[MAXP][4];
#pragma unroll
    for (int i = 0; i < MAXP; ++i)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) kf[i][kk] = *reinterpret_cast<const bf16x8*>(wk + (size_t)min(wave + 4 * i, panels - 1) * pw + kk * 1024);
    float4 bv[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) bv[j] = *reinterpret_cast<const float4*>(g.bq[grp] + a * 64 + j * 32 + wave * 8 + half * 4);
    const unsigned char* x = static_cast<const unsigned char*>(g.first[grp]) + (size_t)blockIdx.y * pw + (size_t)wave * steps * 1024 + lane * 16;
    f32x16 acc[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;
    auto batch = [&](int s0, int nb, auto full) {
        bf16x8 af[U], wf[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (full || u < nb) {
                wf[u][0] = *reinterpret_cast<const bf16x8*>(wq + (size_t)(s0 + u) * 1024);
                wf[u][1] = *reinterpret_cast<const bf16x8*>(wq + pw + (size_t)(s0 + u) * 1024);
                af[u] = *reinterpret_cast<const bf16x8*>(x + (size_t)(s0 + u) * 1024);
            }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (full || u < nb) {
                acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[u][0], af[u], acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[u][1], af[u], acc[1], 0, 0, 0);
            }
    };
    int s0 = 0;
    for (; s0 + U <= steps; s0 += U) batch(s0, U, std::true_type{});
    if (s0 < steps) batch(s0, steps - s0, std::false_type{});
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<f32x4*>(part[wave][j][q][lane]) = f32x4{acc[j][q * 4], acc[j][q * 4 + 1], acc[j][q * 4 + 2], acc[j][q * 4 + 3]};
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j) {                                            // this wavefront finishes chunk `wave` of both blocks
        f32x4 v = *reinterpret_cast<const f32x4*>(part[0][j][wave][lane]);
#pragma unroll
        for (int p = 1; p < 4; ++p) v += *reinterpret_cast<const f32x4*>(part[p][j][wave][lane]);
        const bf16x4 o = {(__bf16)(v[0] + bv[j].x), (__bf16)(v[1] + bv[j].y), (__bf16)(v[2] + bv[j].z), (__bf16)(v[3] + bv[j].w)};
        *reinterpret_cast<bf16x4*>(qs + (j * 4 + wave) * 256 + l32 * 8 + half * 4) = o;
    }
    __syncthreads();
    bf16x8 qf[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qs + kk * 512 + lane * 8);
    // q~ of a sequence: [H / 8 chunks][16 heads][8], the operand order of the scores
    __bf16* qt = static_cast<__bf16*>(g.qt[grp]) + (size_t)(b0 + l32) * H * kHeadsPad + a * 8 + half * 4;
#pragma unroll
    for (int i = 0; i < MAXP; ++i) {
        const int p = wave + 4 * i;
        if (p >= panels) break;
        f32x16 c;
#pragma unroll
        for (int e = 0; e < 16; ++e) c[e] = 0.f;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i][kk], qf[kk], c, 0, 0, 0);
        if (b0 + l32 < B) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bf16x4 o = {(__bf16)c[q * 4], (__bf16)c[q * 4 + 1], (__bf16)c[q * 4 + 2], (__bf16)c[q * 4 + 3]};
                *reinterpret_cast<bf16x4*>(qt + (size_t)(p * 4 + q) * 128) = o;
            }
        }
    }
}

constexpr int kChunkStride = 528;       // bytes of a chunk of 32 keys in LDS: 16 more, so that the columns of a key spread over the banks

template <int NA4>                      // heads / 4, rounded up
__global__ __launch_bounds__(512) void first_attend_kernel(FirstTokenGroup g, const int32_t* __restrict__ seq_start,
                                                           const int32_t* __restrict__ seq_len, int Smax, int H, int A, int64_t xbar_stride,
                                                           float scale_log2e)
{
    constexpr int NH = NA4 * 4, XU = 8, SU = 8;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int grp = blockIdx.y, b = blockIdx.x;
    const int row0 = seq_start[b], n = min(seq_len[b], Smax);
    if (n <= 0) return;
    const int nt = blockDim.x, nw = nt >> 6, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5, n_chunks = H >> 3;
    unsigned char* xs = lds;                                                 // [chunk][32 keys][16 B]
    float* part = reinterpret_cast<float*>(lds + n_chunks * kChunkStride);   // [wavefront][32 keys][16 heads]
    float* ps = part + nw * 512;                                             // [32 keys][16 heads]
    float* ms = ps + 512;                                                    // running maximum, sum and the block's rescale per head
    float* ls = ms + 16;
    float* al = ls + 16;
    if (tid < 16) {
        ms[tid] = -INFINITY;
        ls[tid] = 0.f;
    }
    const __bf16* __restrict__ x = static_cast<const __bf16*>(g.x[grp]);
    // this wavefront's share of the K steps and its q~ fragments (columns beyond the heads repeat others and are not used)
    const int per = (H / 16 + nw - 1) / nw, st0 = wave * per, st1 = min(st0 + per, H / 16);
    const __bf16* qt = static_cast<const __bf16*>(g.qt[grp]) + (size_t)b * H * kHeadsPad + (l32 & 15) * 8;
    bf16x8 qf[SU];
#pragma unroll
    for (int u = 0; u < SU; ++u) qf[u] = *reinterpret_cast<const bf16x8*>(qt + (size_t)(min(st0 + u, H / 16 - 1) * 2 + half) * 128);
    u32x4 xv[XU];
    auto fetch = [&](int kb) {
#pragma unroll
        for (int u = 0; u < XU; ++u) {
            const int i = tid + u * nt, key = i & 31, chunk = min(i >> 5, n_chunks - 1);
            xv[u] = *reinterpret_cast<const u32x4*>(x + tiled_offset(row0 + min(kb + key, n - 1), chunk * 8, H));
        }
    };
    float acc[NH][2];
#pragma unroll
    for (int h = 0; h < NH; ++h) acc[h][0] = acc[h][1] = 0.f;
    fetch(0);
    for (int kb = 0; kb < n; kb += 32) {
        __syncthreads();                                                     // the block before has been summed
#pragma unroll
        for (int u = 0; u < XU; ++u) {
            const int i = tid + u * nt;
            if ((i >> 5) < n_chunks) *reinterpret_cast<u32x4*>(xs + (i >> 5) * kChunkStride + (i & 31) * 16) = xv[u];
        }
        __syncthreads();
        fetch(kb + 32);                                                      // (beyond the last block: its last key again)
        f32x16 sc;
#pragma unroll
        for (int e = 0; e < 16; ++e) sc[e] = 0.f;
#pragma unroll
        for (int u = 0; u < SU; ++u)
            if (st0 + u < st1) {
                const bf16x8 kf = *reinterpret_cast<const bf16x8*>(xs + ((st0 + u) * 2 + half) * kChunkStride + l32 * 16);
                sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[u], sc, 0, 0, 0);     // row: key, column: head
            }
        if (l32 < 16) {
#pragma unroll
            for (int e = 0; e < 16; ++e) part[wave * 512 + ((e >> 2) * 8 + half * 4 + (e & 3)) * 16 + l32] = sc[e];
        }
        __syncthreads();
        // softmax step: 16 lanes per head, two keys each
        for (int h = tid >> 4; h < A; h += nt >> 4) {
            const int k = tid & 15;
            float s0 = 0.f, s1 = 0.f;
            for (int w = 0; w < nw; ++w) {
                s0 += part[w * 512 + k * 16 + h];
                s1 += part[w * 512 + (k + 16) * 16 + h];
            }
            s0 = kb + k < n ? s0 * scale_log2e : -INFINITY;
            s1 = kb + k + 16 < n ? s1 * scale_log2e : -INFINITY;
            float mx = fmaxf(s0, s1);
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
            const float m_old = ms[h], m_new = fmaxf(m_old, mx), alpha = __builtin_amdgcn_exp2f(m_old - m_new);
            const float p0 = __builtin_amdgcn_exp2f(s0 - m_new), p1 = __builtin_amdgcn_exp2f(s1 - m_new);
            float sum = p0 + p1;
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) sum += __shfl_xor(sum, o, 64);
            ps[k * 16 + h] = p0;
            ps[(k + 16) * 16 + h] = p1;
            if (k == 0) {
                const float l_old = ls[h];
                ms[h] = m_new;
                ls[h] = l_old * alpha + sum;
                al[h] = alpha;
            }
        }
        __syncthreads();
        if (tid * 2 < H) {                                                   // two columns per thread
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                const float r = al[h];
                acc[h][0] *= r;
                acc[h][1] *= r;
            }
            const unsigned char* xc = xs + (tid >> 2) * kChunkStride + (tid & 3) * 4;
            const int kn = min(32, n - kb);
#pragma unroll 4
            for (int key = 0; key < kn; ++key) {
                const uint32_t w = *reinterpret_cast<const uint32_t*>(xc + key * 16);
                const float x0 = __uint_as_float(w << 16), x1 = __uint_as_float(w & 0xFFFF0000u);
#pragma unroll
                for (int h4 = 0; h4 < NA4; ++h4) {
                    const float4 p = *reinterpret_cast<const float4*>(ps + key * 16 + h4 * 4);
                    acc[h4 * 4 + 0][0] = fmaf(p.x, x0, acc[h4 * 4 + 0][0]);
                    acc[h4 * 4 + 0][1] = fmaf(p.x, x1, acc[h4 * 4 + 0][1]);
                    acc[h4 * 4 + 1][0] = fmaf(p.y, x0, acc[h4 * 4 + 1][0]);
                    acc[h4 * 4 + 1][1] = fmaf(p.y, x1, acc[h4 * 4 + 1][1]);
                    acc[h4 * 4 + 2][0] = fmaf(p.z, x0, acc[h4 * 4 + 2][0]);
                    acc[h4 * 4 + 2][1] = fmaf(p.z, x1, acc[h4 * 4 + 2][1]);
                    acc[h4 * 4 + 3][0] = fmaf(p.w, x0, acc[h4 * 4 + 3][0]);
                    acc[h4 * 4 + 3][1] = fmaf(p.w, x1, acc[h4 * 4 + 3][1]);
                }
            }
        }
    }
    if (tid * 2 >= H) return;
    __bf16* out = static_cast<__bf16*>(g.xbar[grp]) + tiled_offset(b, tid * 2, H);
#pragma unroll
    for (int h = 0; h < NH; ++h)
        if (h < A) {
            const float inv = 1.0f / ls[h];
            const bf16x2 o = {(__bf16)(acc[h][0] * inv), (__bf16)(acc[h][1] * inv)};
            *reinterpret_cast<bf16x2*>(out + h * xbar_stride) = o;
        }
}

}  // namespace

hipError_t launch_first_query(const FirstTokenGroup& g, int G, int B, int H, int A, hipStream_t stream)
{
    if (G <= 0 || B <= 0) return hipSuccess;
    if (G > kMaxGroup || H != A * 64 || A > kHeadsPad) return hipErrorInvalidValue;
    hipLaunchKernelGGL(first_query_kernel, dim3(A, (B + 31) / 32, G), dim3(256), 0, stream, g, B, H);
    return hipGetLastError();
}

hipError_t launch_first_attend(const FirstTokenGroup& g, int G, const int32_t* seq_start, const int32_t* seq_len, int B, int S, int H, int A,
                               int64_t xbar_stride, hipStream_t stream)
{
    if (G <= 0 || B <= 0 || S <= 0) return hipSuccess;
    if (!seq_start || !seq_len || G > kMaxGroup || H != A * 64 || A > kHeadsPad) return hipErrorInvalidValue;
    const int nt = (H / 2 + 63) / 64 * 64;                                  // <= 512
    const size_t bytes = (size_t)(H / 8) * kChunkStride + (size_t)(nt / 64) * 2048 + 2048 + 3 * 64;
    const float scale = 0.125f * 1.4426950408889634f;
#define MT_ATTEND(N)                                                                                                                      \
    do {                                                                                                                                  \
        static std::atomic<uint64_t> raised{0};                                                                                           \
        if (bytes > 64 * 1024) {                                                                                                          \
            hipError_t e = ensure_dynamic_lds((const void*)first_attend_kernel<N>, 96 * 1024, raised);                                    \
            if (e != hipSuccess) return e;                                                                                                \
        }                                                                                                                                 \
        hipLaunchKernelGGL(first_attend_kernel<N>, dim3(B, G), dim3(nt), bytes, stream, g, seq_start, seq_len, S, H, A, xbar_stride, scale); \
    } while (0)
    switch ((A + 3) / 4) {
        case 1: MT_ATTEND(1); break;
        case 2: MT_ATTEND(2); break;
        case 3: MT_ATTEND(3); break;
        default: MT_ATTEND(4); break;
    }
#undef MT_ATTEND
    return hipGetLastError();
}

}  // namespace mt
