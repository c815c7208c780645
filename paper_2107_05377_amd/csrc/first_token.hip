// First-token attention of a branch's last layer on the panel layout, keys and values not projected (bfloat16 path): with
// q~[b][a] = Wk_a^T (Wq_a x_b + bq_a) the score of key j is q~ . x_j up to a constant that the softmax drops, and the head's context
// is Wv_a (sum_j p_j x_j) + bv_a.  Two launches per group of tasks (the contexts are one more, gemm_tiled_rows_kernel):
//   first_query_kernel   per (task, head) one workgroup, or as many as there are compute units for, that keep the two weight slices (98 KB each) in
//                        registers and walk over panels of 32 sequences: query of the sequences' first rows (gathered before: in place, 16
//                        bytes of a line at a time, every head's workgroup paid for them, 19.5 us for 8 tasks x 32 sequences; of up to kInPlace
//                        sequences that costs less than the launch), then q~, the 64 columns between them staying in LDS.  A chain of latencies: 10 us
//                        for the first panel, 3 for each further one (a workgroup per panel, each with weights to load: 10 and 11 tasks x 272
//                        sequences 43 + 52 us, now 23 + 32, 8 tasks x 256 35, 21).
//   first_attend_kernel  one workgroup per (task, sequence): scores, softmax and weighted row sums in one pass over the sequence's rows, a panel
//                        of 32 keys at a time, both products on the matrix cores (with the sums as 2 H FMAs per key and head on the vector
//                        units 8 tasks took 190 us for 256 sequences of up to 128 tokens and 72 for 7 of up to 509); bound by reading the rows.
//                        Four wavefronts (narrow models in large launches: one): six of 128 columns, placed 2, 2, 1, 1 on the SIMDs, left no room for a second workgroup of theirs at 168
//                        registers (200 workgroups in flight, now 450), and a compute unit stood still while its one waited for rows or stored.
//                        21 tasks x 272 short sequences 62 + 77 -> 41 + 52 us, 8 tasks x 256 112 -> 73, x 7 of up to 509 tokens 33 -> 26.
// Scores and sums were two kernels that read the rows once each (85 + 107 us for 8 tasks x 256 sequences).
#include <algorithm>

#include "kernels.h"
#include "device_util.h"

namespace mt {

namespace {

constexpr int kHeadsPad = 16;
// The softmax weights are float32 quantities and enter the product as TERMS bfloat16 terms (the value, its remainder, ..).  Three are the whole
// float32 weight: MT_FP8_LAYER, whose row-major kernels hold float32 weights.  Two, 16 bits of it, are what MT_BF16 takes: the row sums' error
// against float64 is then that of float32 weights unless the sum cancels to less than about 2^-8 of its terms (one term exceeds it 3 to 20 times
// where the sum cancels at all).  Cost of the second term: 21 tasks x 272 short sequences 2810 -> 2822 us a pass, 8 tasks x 256 sequences nothing;
// of the third 1 % of the former; MT_FP8_LAYER with it 8 tasks x 4 sequences 504 -> 508 us, x 256 sequences 4.25 -> 4.28 ms.
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// NS = H / 64: K steps of 16 of a wavefront.  A workgroup has its (task, head)'s two weight slices in registers and walks over panels of 32
// sequences, gy workgroups dealing them out.
template <int NS>
__global__ __launch_bounds__(256, 1) void first_query_kernel(int B, int A, int nb, int gy, int pairs, const int32_t* seq_start, int max_rows, FirstTokenGroup g)
{
    constexpr int H = NS * 64, PANELS = 2 * NS, P = (PANELS + 3) / 4;        // panels of the hidden columns; of a wavefront (wave, wave + 4, ..)
    __shared__ __attribute__((aligned(16))) float part[4][2][4][64][4];
    __shared__ __attribute__((aligned(16))) __bf16 qs[8 * 256];              // 64 columns of 32 rows, panel layout
    // the gy workgroups of a (task, head), which share its weight slices, follow one another on one XCD
    const int i8 = blockIdx.x >> 3, pi = gy == 1 ? i8 : i8 / gy, pair = pi * 8 + (blockIdx.x & 7);
    int yb = i8 - pi * gy;
    if (pair >= pairs) return;
    const int grp = pair / A, a = pair - grp * A, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    constexpr size_t pw = (size_t)H * 64;                                    // bytes per panel
    const unsigned char* wq = static_cast<const unsigned char*>(g.Wq[grp]) + (size_t)a * 2 * pw + (size_t)wave * NS * 1024 + lane * 16;
    const unsigned char* wk = static_cast<const unsigned char*>(g.WkT[grp]) + (size_t)a * 4096 + lane * 16;
    auto rows = [&](int y) {
        const unsigned char* x;
        if (seq_start) {                     // in place: this lane's row of all rows
            const int row = min(seq_start[min(y * 32 + l32, B - 1)], max_rows - 1);
            x = static_cast<const unsigned char*>(g.x[grp]) + (size_t)(row >> 5) * pw + half * 512 + (row & 31) * 16;
        } else {
            x = static_cast<const unsigned char*>(g.first[grp]) + (size_t)y * pw + lane * 16;
        }
        return x + (size_t)wave * NS * 1024;
    };
    bf16x8 wf[NS][2], kf[P][4], xf[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        wf[u][0] = *reinterpret_cast<const bf16x8*>(wq + (size_t)u * 1024);
        wf[u][1] = *reinterpret_cast<const bf16x8*>(wq + pw + (size_t)u * 1024);
    }
    auto fetch = [&](int y) {
        const unsigned char* x = rows(y);
#pragma unroll
        for (int u = 0; u < NS; ++u) xf[u] = *reinterpret_cast<const bf16x8*>(x + (size_t)u * 1024);
    };
    fetch(yb);
    // the key matrix's fragments for this wavefront's panels of q~
#pragma unroll
    for (int i = 0; i < P; ++i)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) kf[i][kk] = *reinterpret_cast<const bf16x8*>(wk + (size_t)min(wave + 4 * i, PANELS - 1) * pw + kk * 1024);
    float4 bv[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) bv[j] = *reinterpret_cast<const float4*>(g.bq[grp] + a * 64 + j * 32 + wave * 8 + half * 4);
    __builtin_amdgcn_sched_barrier(0);
    auto panel = [&](auto more) {
        f32x16 acc[2];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[u][0], xf[u], acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[u][1], xf[u], acc[1], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (more) fetch(yb + gy);
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<f32x4*>(part[wave][j][q][lane]) = f32x4{acc[j][q * 4], acc[j][q * 4 + 1], acc[j][q * 4 + 2], acc[j][q * 4 + 3]};
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 2; ++j) {                                        // this wavefront finishes chunk `wave` of both blocks
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
        // q~: [sequence][16 heads][H], so that a workgroup writes whole lines; the half wavefronts exchange for 8 columns per lane
        const int b = yb * 32 + l32;
        __bf16* qt = static_cast<__bf16*>(g.qt[grp]) + ((size_t)b * kHeadsPad + a) * H + half * 8;
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const int p = wave + 4 * i;
            if (PANELS % 4 != 0 && p >= PANELS) break;
            f32x16 c;
#pragma unroll
            for (int e = 0; e < 16; ++e) c[e] = 0.f;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i][kk], qf[kk], c, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; q += 2) {
                bf16x4 lo, hi;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    lo[e] = (__bf16)c[q * 4 + e];
                    hi[e] = (__bf16)c[q * 4 + 4 + e];
                }
                const u32x2 lu = __builtin_bit_cast(u32x2, lo), hu = __builtin_bit_cast(u32x2, hi);
                const auto s0 = __builtin_amdgcn_permlane32_swap(lu[0], hu[0], false, false), s1 = __builtin_amdgcn_permlane32_swap(lu[1], hu[1], false, false);
                if (b < B) *reinterpret_cast<u32x4*>(qt + (p * 4 + q) * 8) = u32x4{s0[0], s1[0], s0[1], s1[1]};
            }
        }
    };
    for (; yb + gy < nb; yb += gy) panel(std::true_type{});
    panel(std::false_type{});
}

// NW wavefronts, each STEPS x 32 of the H columns (the last ones perhaps fewer, or none).  Per key panel: a wavefront loads its columns of the 32 rows as matrix
// operands (16 x 32, straight from global memory), forms its share of the scores with q~ and leaves it in LDS; after the only barrier all
// wavefronts add the shares, each for itself, and have the weights of all heads in the operand order of the next product.  For that the
// rows are needed transposed: a product with the unit matrix, exact, moves the columns to the lanes.
template <int NW, int STEPS, int TERMS>
__global__ __launch_bounds__(NW * 64, 2) void first_attend_kernel(const int32_t* __restrict__ seq_start,
                                                                                    const int32_t* __restrict__ seq_len, int B, int Smax, int H,
                                                                                    int A, int64_t xbar_stride, FirstTokenGroup g)
{
    constexpr float kScale = 0.125f * 1.4426950408889634f;
    __shared__ __attribute__((aligned(16))) float part[2][NW][2][64][4];
    // an XCD takes neighbouring sequences: 16 bytes of each make up the lines of the result, which its second-level cache completes
    const int per = (B + 7) >> 3, b = (blockIdx.x & 7) * per + (blockIdx.x >> 3), grp = blockIdx.y;
    if (b >= B) return;
    const int row0 = seq_start[b], n = min(seq_len[b], Smax), end = row0 + n;
    if (n <= 0) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, l4 = lane >> 4;
    const int p0 = row0 >> 5, p1 = (end + 31) >> 5;                          // panels of the sequence
    const int c0 = wave * STEPS, steps = min(STEPS, (H >> 5) - c0), c_max = (H >> 5) - 1;          // columns in units of 32
    const size_t pitch = (size_t)H * 64;                                     // bytes of a panel
    const unsigned char* x = static_cast<const unsigned char*>(g.x[grp]) + l4 * 512 + l16 * 16;
    const __bf16* qt = static_cast<const __bf16*>(g.qt[grp]) + ((size_t)b * kHeadsPad + min(l16, A - 1)) * H + l4 * 8;
    bf16x8 qf[STEPS];
    f32x4 acc[2 * STEPS];                                                            // 16 columns x 16 heads each; lane: head l16, columns 4 l4 + 0..3
#pragma unroll
    for (int k = 0; k < STEPS; ++k) {
        qf[k] = *reinterpret_cast<const bf16x8*>(qt + min(c0 + k, c_max) * 32);
        if (k >= steps) qf[k] = __builtin_bit_cast(bf16x8, u32x4{0, 0, 0, 0});          // columns beyond H repeat others, to no effect
    }
#pragma unroll
    for (int c = 0; c < 2 * STEPS; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 unit[2];                                                          // [16 columns][32]: the first and the second 16 of a step
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int d = l16 + c * 16 - l4 * 8;
        u32x4 u;
#pragma unroll
        for (int e = 0; e < 4; ++e) u[e] = d == 2 * e ? 0x3F80u : (d == 2 * e + 1 ? 0x3F800000u : 0u);
        unit[c] = __builtin_bit_cast(bf16x8, u);
    }
    float m_run = -INFINITY, l_run = 0.f;
    bf16x8 xa[2][STEPS], xb[2][STEPS];                                               // [upper or lower 16 keys][step]
    auto fetch = [&](bf16x8 (&v)[2][STEPS], int kb) {
#pragma unroll
        for (int k = 0; k < STEPS; ++k)
#pragma unroll
            for (int h = 0; h < 2; ++h) v[h][k] = *reinterpret_cast<const bf16x8*>(x + (size_t)kb * pitch + min(c0 + k, c_max) * 2048 + h * 256);
    };
    auto block = [&](const bf16x8 (&v)[2][STEPS], int kb, int buf) {
        f32x4 sc[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            sc[h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < STEPS; ++k) {                                // row: key, column: head
                if constexpr (NW == 1) {                                     // the shares of four wavefronts of a step each, added in their order: the same bits
                    const f32x4 share = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v[h][k], qf[k], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                    sc[h] = k ? sc[h] + share : share;
                } else {
                    sc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v[h][k], qf[k], sc[h], 0, 0, 0);
                }
            }
            if constexpr (NW > 1) *reinterpret_cast<f32x4*>(part[buf][wave][h][lane]) = sc[h];
        }
        if constexpr (NW > 1) {
            __syncthreads();
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                sc[h] = *reinterpret_cast<const f32x4*>(part[buf][0][h][lane]);
#pragma unroll
                for (int w = 1; w < NW; ++w) sc[h] += *reinterpret_cast<const f32x4*>(part[buf][w][h][lane]);
                if constexpr (NW > 4) __builtin_amdgcn_sched_barrier(0);     // (fewer of the shares in registers at a time)
            }
        }
        // keys 16 h + 4 l4 + e of this panel; what belongs to a neighbouring sequence counts as nothing, whatever it is
        const bool edge = kb * 32 < row0 || kb * 32 + 32 > end;
        u32x4 keep = {~0u, ~0u, ~0u, ~0u};
        if (edge) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if ((unsigned)(kb * 32 + h * 16 + l4 * 4 + e - row0) >= (unsigned)n) {
                        sc[h][e] = -INFINITY;
                        keep[h * 2 + (e >> 1)] &= (e & 1) ? 0x0000FFFFu : 0xFFFF0000u;
                    }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) mx = fmaxf(mx, sc[h][e]);
        mx = lane_pair_max<16>(mx);
        mx = lane_pair_max<32>(mx) * kScale;
        if (__any(l16 < A && mx > m_run + 8.f)) {                            // the maximum follows only when a score exceeds it by 2^8
            const float m_new = fmaxf(m_run, mx), alpha = __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
            l_run *= alpha;
#pragma unroll
            for (int c = 0; c < 2 * STEPS; ++c) acc[c] *= alpha;
        }
        bf16x8 pf[TERMS];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float p = __builtin_amdgcn_exp2f(fmaf(sc[h][e], kScale, -m_run));
                l_run += p;
#pragma unroll
                for (int t = 0; t < TERMS; ++t) {
                    pf[t][h * 4 + e] = (__bf16)p;
                    p -= (float)pf[t][h * 4 + e];
                }
            }
#pragma unroll
        for (int c = 0; c < 2 * STEPS; ++c) {
            bf16x8 xt;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x4 t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v[h][c >> 1], unit[c & 1], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
                for (int e = 0; e < 4; ++e) xt[h * 4 + e] = (__bf16)t[e];
            }
            xt = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, xt) & keep);
#pragma unroll
            for (int t = TERMS - 1; t >= 0; --t) acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xt, pf[t], acc[c], 0, 0, 0);     // row: column, column: head
            if (c & 1) __builtin_amdgcn_sched_barrier(0);                    // (two at a time, for the registers)
        }
    };
    // A panel is on its way while the one before it is worked on.  Written so that each wait has one possible number of loads behind it: after a
    // conditional fetch the compiler waits for everything, the next panel included.
    fetch(xa, p0);
    int kb = p0;
    for (; kb + 2 < p1; kb += 2) {
        fetch(xb, kb + 1);
        block(xa, kb, 0);
        fetch(xa, kb + 2);
        block(xb, kb + 1, 1);
    }
    if (kb + 1 < p1) {
        fetch(xb, kb + 1);
        block(xa, kb, 0);
        block(xb, kb + 1, 1);
    } else {
        block(xa, kb, 0);
    }
    l_run = lane_pair_sum<16>(l_run);
    l_run = lane_pair_sum<32>(l_run);
    const float inv = 1.0f / l_run;
    // 4 columns of each of two blocks per lane; lanes 16 apart exchange, so that each has a chunk's 8 columns of one
    __bf16* out = static_cast<__bf16*>(g.xbar[grp]) + l16 * xbar_stride + tiled_offset(b, c0 * 32 + (l4 & 1) * 16 + (l4 >> 1) * 8, H);
#pragma unroll
    for (int k = 0; k < STEPS; ++k) {
        uint32_t d[2][2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const f32x4& a = acc[2 * k + j];
            const bf16x4 o = {(__bf16)(a[0] * inv), (__bf16)(a[1] * inv), (__bf16)(a[2] * inv), (__bf16)(a[3] * inv)};
            const u32x2 u = __builtin_bit_cast(u32x2, o);
            d[j][0] = u[0];
            d[j][1] = u[1];
        }
        const auto lo = __builtin_amdgcn_permlane16_swap(d[0][0], d[1][0], false, false), hi = __builtin_amdgcn_permlane16_swap(d[0][1], d[1][1], false, false);
        if (k < steps && l16 < A) *reinterpret_cast<u32x4*>(out + k * 1024) = u32x4{lo[0], hi[0], lo[1], hi[1]};
    }
}

}  // namespace

hipError_t launch_first_query(const FirstTokenGroup& g, int G, int B, int H, int A, hipStream_t stream, const int32_t* seq_start, int max_rows)
{
    if (G <= 0 || B <= 0) return hipSuccess;
    if (G > kMaxGroup || H != A * 64 || A > kHeadsPad) return hipErrorInvalidValue;
    // One workgroup fills a compute unit's registers: as many per (task, head) as there are compute units for.  1 to 5 of them, launches inside passes: 8 tasks x
    // 256 sequences, 96 pairs, 31, 21, 29, 26, 26 us; 10 and 11 tasks x 272, 120 pairs 32, 23, 31, 30, 33, 132 pairs 32, 40, 31, 42, 36 (one leaves 124 compute
    // units idle, three are two uneven rounds: the pass is level); x 104, 4 panels, 19, 15, 20, 18 and 19, 25, 21, 26.
    const int nb = (B + 31) / 32, pairs = A * G, gy = std::max(1, std::min(nb, device_cu_count() / pairs));
    const dim3 grid((pairs + 7) / 8 * 8 * gy);
#define MT_QUERY(NS)                                                                                                                          \
    case NS: hipLaunchKernelGGL(first_query_kernel<NS>, grid, dim3(256), 0, stream, B, A, nb, gy, pairs, seq_start, max_rows, g); break
    switch (A) {                             // H = A * 64
        MT_QUERY(1);
        MT_QUERY(2);
        MT_QUERY(3);
        MT_QUERY(4);
        MT_QUERY(5);
        MT_QUERY(6);
        MT_QUERY(7);
        MT_QUERY(8);
        MT_QUERY(9);
        MT_QUERY(10);
        MT_QUERY(11);
        MT_QUERY(12);
        MT_QUERY(13);
        MT_QUERY(14);
        MT_QUERY(15);
        MT_QUERY(16);
    }
#undef MT_QUERY
    return hipGetLastError();
}

hipError_t launch_first_attend(const FirstTokenGroup& g, int G, const int32_t* seq_start, const int32_t* seq_len, int B, int S, int H, int A,
                               int64_t xbar_stride, hipStream_t stream, bool whole_weights)
{
    if (G <= 0 || B <= 0 || S <= 0) return hipSuccess;
    if (!seq_start || !seq_len || G > kMaxGroup || H != A * 64 || A > kHeadsPad) return hipErrorInvalidValue;
#define MT_ATTEND(N, STEPS)                                                                                                                   \
    {                                                                                                                                         \
        auto kfn = whole_weights ? first_attend_kernel<N, STEPS, 3> : first_attend_kernel<N, STEPS, 2>;                                       \
        hipLaunchKernelGGL(kfn, dim3((B + 7) / 8 * 8, G), dim3(N * 64), 0, stream, seq_start, seq_len, B, S, H, A, xbar_stride, g);           \
    }                                                                                                                                         \
    break
    switch ((H + 127) / 128) {
        // One block of columns: four wavefronts shorten a panel's chain of latencies, one leaves room for the other sequences where there are more than
        // two workgroups for each compute unit.  1 and 2 heads, up to 60 tokens, 272 / 512 / 600 / 900 / 2200 sequences: four 4.5, 4.9, 5.5, 6.3, 10.1 us, one
        // 4.7, 4.8, 4.9, 4.9, 7.9.  (3 heads, 96 columns of 2 wavefronts: level at 900 to 4000.)
        case 1:
            if ((long)B * G > 2l * device_cu_count()) { MT_ATTEND(1, 4); }
            MT_ATTEND(4, 1);
        case 2: MT_ATTEND(4, 2);
        case 3: MT_ATTEND(4, 3);
        case 4: MT_ATTEND(4, 4);
        case 5: MT_ATTEND(4, 5);
        case 6: MT_ATTEND(4, 6);
        default: MT_ATTEND(8, 4);
    }
#undef MT_ATTEND
    return hipGetLastError();
}

}  // namespace mt
