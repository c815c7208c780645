// Attention of the bfloat16 path on the panel layout of tiled_offset() (kernels.h): softmax(q k^T / 8) v per sequence and head of
// width 64.
//
// A 32-row panel of the projections holds, per head, the queries and keys as matrix operands (1 KB of contiguous memory per 32 x 16
// fragment) and the values transposed, as the contraction that made them stored them (TiledShape::vt_panel).  So nothing has to be
// rearranged: a wavefront owns the 32 queries of a panel and walks over the key panels of its sequence, all fragments straight from
// global memory to registers, with no LDS and no barrier.  Key and query blocks are the panels themselves; what of a first or
// last panel belongs to a neighbouring sequence is masked (its values are cleared: they may be anything).  The scores are computed
// transposed (keys x queries), which leaves a lane with the weights of its query in the operand order of the product with the
// values.
//
// A weight is rounded to bfloat16 for the product.  The running maximum follows every key panel, so that the largest weight is 1 and not
// rounded, and the normaliser adds up the rounded weights, so that a rounding moves the context along (value - context) only.  With a maximum
// that followed when a score exceeded it by 2^8, and unrounded weights in the normaliser, the error against float64 was 1 to 25 % larger
// (12 heads, 8 x 128 and 2 x 509 tokens, scores of standard deviation 0.3 to 3; passes 0.2 % shorter, 7 x 509 tokens 0.5 %).
//
// Bound by memory when the batch is large: 18.6 k rows of 12 heads are 114 MB in 29 us (staging keys and values in LDS 32, on 7
// sequences of up to 509 tokens 23.5 instead of 10.1, on 128 of up to 256 with 16 heads 79 instead of 43), by the chain of its loads
// when it is small (one sequence: 4.1 us, 6.3).  Loads run one block ahead: a block's keys are fetched after the scores of the one before, its values after the product, and
// in large launches (DEEP) no wait is for what the next block needs (instead of for all of it at every product; 32 x 128 tokens 9.4 -> 8.8 us a layer).  The four
// wavefronts of a workgroup take neighbouring query panels of a head, so that keys and values come from the first-level cache for
// three of them; where that gives too few wavefronts (long sequences of a small batch), KS of them share a query panel and take
// every KS-th key panel each, merged through LDS.
#include "kernels.h"
#include "device_util.h"

namespace mt {

namespace {

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// two neighbouring chunks (8 columns each) of a context block: 4 of a chunk's columns per lane -> 8, the lower half wavefront the
// first chunk, the upper the second
__device__ __forceinline__ u32x4 pack_chunks(const float (&v)[8])
{
    bf16x4 x, y;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        x[e] = (__bf16)v[e];
        y[e] = (__bf16)v[4 + e];
    }
    const u32x2 xu = __builtin_bit_cast(u32x2, x), yu = __builtin_bit_cast(u32x2, y);
    const auto s0 = __builtin_amdgcn_permlane32_swap(xu[0], yu[0], false, false);
    const auto s1 = __builtin_amdgcn_permlane32_swap(xu[1], yu[1], false, false);
    return u32x4{s0[0], s1[0], s0[1], s1[1]};
}

// nq: workgroups per (sequence, head).  pairs == 0: one each, grid (heads, sequences, problems).  Otherwise a flat grid in which an XCD
// owns a contiguous range of (problem, head, sequence, workgroup), so that its second-level cache holds a sequence's keys and values,
// and the panels that sequences share, once.
template <int KS, bool DEEP, class Ahead>
__global__ __launch_bounds__(KS == 1 ? 512 : 256, KS == 1 ? 4 : 3) void attention_tiled_kernel(const unsigned char* base_qkv, unsigned char* base_ctx,
                                                              const int32_t* __restrict__ seq_start, const int32_t* __restrict__ seq_len, int B, int S,
                                                              int A, int nq_nw, int pairs, int G, AttnTiledGroup g, Ahead ahead)
{
    if constexpr (Ahead::kAny) {
        if ((int)blockIdx.z >= G) {
            read_ahead(ahead, ((blockIdx.z - G) * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x);
            return;
        }
    }
    const int nq = nq_nw & 0xFFFF, QW = KS == 1 ? nq_nw >> 16 : 4 / KS;      // query panels of a workgroup at a time
    constexpr float kScale = 0.125f * 1.4426950408889634f;                   // exponents of two
    __shared__ __attribute__((aligned(16))) float s_o[KS > 1 ? 4 : 1][8][KS > 1 ? 64 : 1][4];
    __shared__ float s_m[KS > 1 ? 4 : 1][64], s_l[KS > 1 ? 4 : 1][64];
    int a = blockIdx.x, b = blockIdx.y, grp = blockIdx.z, qg = 0;
    if (pairs) {
        const int total = pairs * nq, xcd = blockIdx.x & 7, i = blockIdx.x >> 3, per = (total + 7) >> 3, at = xcd * per + i;
        if (i >= per || at >= total) return;
        const int pair = nq == 1 ? at : at / nq, ga = pair / B;
        qg = at - pair * nq;
        b = pair - ga * B;
        grp = ga / A;
        a = ga - grp * A;
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, half = lane >> 5, ks = wave % KS, qi = wave / KS;
    const int row0 = seq_start[b], n = min(seq_len[b], S), end = row0 + n;
    if (n <= 0) return;
    const int p0 = row0 >> 5, p1 = (end + 31) >> 5;                          // panels of the sequence
    const int H = A * 64;
    const size_t pitch = (size_t)H * 192;                                    // bytes of a panel of projections
    const unsigned char* qkv = base_qkv + (size_t)g.qkv[grp] * 256 + a * 4096 + (DEEP ? 0 : lane * 16);

    for (int pb = p0 + qg * QW; pb < p1; pb += nq * QW) {
        const int qp = pb + qi;
        const bool active = qp < p1;
        float m_run = -INFINITY, l_run = 0.f;
        f32x16 o[2];
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
        const bool q_real = (unsigned)(qp * 32 + l32 - row0) < (unsigned)n;
        if (active && p0 + ks < p1) {
            bf16x8 qf[4], kf[4], vf[2][2];
            // After a conditional fetch the compiler waits for everything under way before a block's values are used, the next block's keys included.  DEEP: behind
            // the last block (not real) the loads are issued too, but read nothing, and no wait is for what only the next block needs.
            auto load = [&](bf16x8& to, const unsigned char* from, int at, bool real) {
                if constexpr (DEEP)
                    to = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                                                        __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(from), 0, real ? 4096 : 0, 0x00020000), lane * 16 + at, 0, 0));
                else to = *reinterpret_cast<const bf16x8*>(from + at);
            };
            auto load_k = [&](int kb, bool real) {
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) load(kf[kk], qkv + (size_t)kb * pitch + (size_t)H * 64, kk * 1024, real);
            };
            auto load_v = [&](int kb, bool real) {
#pragma unroll
                for (int mf = 0; mf < 2; ++mf)
#pragma unroll
                    for (int dt = 0; dt < 2; ++dt) load(vf[mf][dt], qkv + (size_t)kb * pitch + (size_t)H * 128, dt * 2048 + mf * 1024, real);
            };
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qkv + (size_t)qp * pitch + (DEEP ? lane * 16 : 0) + kk * 1024);
            int kb = p0 + ks;
            load_k(kb, true);
            load_v(kb, true);
            for (;;) {
                f32x16 sc;
#pragma unroll
                for (int e = 0; e < 16; ++e) sc[e] = 0.f;
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], qf[kk], sc, 0, 0, 0);
                const int kn = kb + KS;
                const bool more = kn < p1;
                if constexpr (DEEP) {
                    __builtin_amdgcn_sched_barrier(0);                       // (into the registers that the scores have used)
                    load_k(kn, more);
                    __builtin_amdgcn_sched_barrier(0);
                } else if (more) {
                    load_k(kn, true);
                }
                if (kb * 32 < row0 || kb * 32 + 32 > end) {                  // a panel shared with a neighbour
                    const int r0 = kb * 32 + half * 4 - row0;
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        if ((unsigned)(r0 + (e >> 2) * 8 + (e & 3)) >= (unsigned)n) sc[e] = -INFINITY;
#pragma unroll
                    for (int mf = 0; mf < 2; ++mf) {
                        u32x4 keep;
#pragma unroll
                        for (int d = 0; d < 4; ++d) {
                            const int r = r0 + mf * 16 + (d >> 1) * 8 + (d & 1) * 2;
                            keep[d] = ((unsigned)r < (unsigned)n ? 0xFFFFu : 0u) | ((unsigned)(r + 1) < (unsigned)n ? 0xFFFF0000u : 0u);
                        }
#pragma unroll
                        for (int dt = 0; dt < 2; ++dt) vf[mf][dt] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, vf[mf][dt]) & keep);
                    }
                }
                float mx = sc[0];
#pragma unroll
                for (int e = 1; e < 16; ++e) mx = fmaxf(mx, sc[e]);
                mx = lane_pair_max<32>(mx);
                if (__any(q_real && mx * kScale > m_run)) {
                    const float m_new = fmaxf(m_run, mx * kScale), alpha = __builtin_amdgcn_exp2f(m_run - m_new);
                    m_run = m_new;
                    l_run *= alpha;
#pragma unroll
                    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                        for (int e = 0; e < 16; ++e) o[dt][e] *= alpha;
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) sc[e] = __builtin_amdgcn_exp2f(fmaf(sc[e], kScale, -m_run));        // bare v_exp_f32: tiny weights flush to 0
#pragma unroll
                for (int mf = 0; mf < 2; ++mf) {
                    bf16x8 pf;
#pragma unroll
                    for (int e = 0; e < 8; ++e) pf[e] = (__bf16)sc[mf * 8 + e];
                    const u32x4 pu = __builtin_bit_cast(u32x4, pf);
#pragma unroll
                    for (int e = 0; e < 4; ++e)                              // the weights as the product takes them
                        l_run = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, (uint32_t)pu[e]), __builtin_bit_cast(bf16x2, 0x3F803F80u), l_run, false);
#pragma unroll
                    for (int dt = 0; dt < 2; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[mf][dt], pf, o[dt], 0, 0, 0);
                }
                if constexpr (DEEP) {
                    __builtin_amdgcn_sched_barrier(0);
                    load_v(kn, more);
                }
                if (!more) break;
                kb = kn;
                if constexpr (!DEEP) load_v(kb, true);
            }
            l_run = lane_pair_sum<32>(l_run);
        }
        unsigned char* ctx = base_ctx + (size_t)g.ctx[grp] * 256 + (size_t)qp * H * 64 + a * 4096 + lane * 16;
        if constexpr (KS == 1) {
            if (active) {
                const float inv = 1.0f / l_run;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    float v[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] = o[c >> 1][(c & 1) * 8 + e] * inv;
                    const u32x4 w = pack_chunks(v);
                    if (q_real) *reinterpret_cast<u32x4*>(ctx + c * 1024) = w;
                }
            }
        } else {
            __syncthreads();                                                 // the panel before has been read
#pragma unroll
            for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<f32x4*>(s_o[wave][dt * 4 + q][lane]) = f32x4{o[dt][q * 4], o[dt][q * 4 + 1], o[dt][q * 4 + 2], o[dt][q * 4 + 3]};
            s_m[wave][lane] = m_run;
            s_l[wave][lane] = l_run;
            __syncthreads();
            if (active) {
                float w[KS], m = -INFINITY, l = 0.f;
#pragma unroll
                for (int k = 0; k < KS; ++k) m = fmaxf(m, s_m[qi * KS + k][lane]);
#pragma unroll
                for (int k = 0; k < KS; ++k) {                               // a share without keys has weight 0
                    w[k] = __builtin_amdgcn_exp2f(s_m[qi * KS + k][lane] - m);
                    l += w[k] * s_l[qi * KS + k][lane];
                }
                const float inv = 1.0f / l;
#pragma unroll
                for (int cc = 0; cc < 4 / KS; ++cc) {                        // this wavefront's chunks of the context
                    const int c = ks * (4 / KS) + cc;
                    float v[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] = 0.f;
#pragma unroll
                    for (int k = 0; k < KS; ++k)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const f32x4 u = *reinterpret_cast<const f32x4*>(s_o[qi * KS + k][c * 2 + h][lane]);
#pragma unroll
                            for (int e = 0; e < 4; ++e) v[h * 4 + e] += w[k] * u[e];
                        }
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] *= inv;
                    const u32x4 r = pack_chunks(v);
                    if (q_real) *reinterpret_cast<u32x4*>(ctx + c * 1024) = r;
                }
            }
        }
    }
}

}  // namespace

hipError_t launch_attention_tiled(const AttnTiledGroup& g, int G, const int32_t* seq_start, const int32_t* seq_len, int B, int S, int H, int A,
                                  hipStream_t stream, AheadQueue* queue)
{
    if (G <= 0 || B <= 0 || S <= 0) return hipSuccess;
    if (!seq_start || !seq_len || H != A * 64 || G > kMaxGroup || (long)A * B * G > (1 << 24)) return hipErrorInvalidValue;
    // Two wavefronts per query panel where one each would leave SIMDs idle over a long loop (7 sequences of up to 509 tokens, 12 heads:
    // 10.1 us, 12.0 with one, 10.6 with four).  Else a wavefront per panel that a sequence can touch, 3 or 4 to a workgroup (an idle
    // wavefront holds registers: 9 panels by 2 x 5 took 62 us, by 3 x 3 43); the fifth panel of a sequence of up to 128 tokens has
    // one of its own up to 2048 (sequence, head) pairs, where launches of 16 to 128 tokens cross: 384 pairs 8.9 us, 10.6 without; 1536 17.6
    // and 18.6; 2052 21.1 and 21.2; 3072 36.6 and 33.8.  (100 to 128 tokens cross at 1500: 1152 19.0 and 19.9, 1536 28.3 and 27.1.)
    const int panels = (S + 31) / 32 + 1, groups = A * B * G;
    const int ks = panels > 8 && (long)groups * panels <= 2048 ? 2 : 1;
    int nq = panels <= 5 ? 1 : (panels + 3) / 4, nw = (panels + nq - 1) / nq;
    if (panels == 5 && groups >= 2048) nw = 4;
    if (ks == 2) {
        nw = 4;
        nq = panels / 2;
    }
    // a small launch saves the divisions of the flat order
    const bool flat = nq > 1 || groups >= 1024;
    ReadAhead ahead;
    if (!flat && queue) ahead = queue->take();
    const dim3 grid = flat ? dim3((groups * nq + 7) / 8 * 8) : dim3(A, B, G + (ahead.blocks() + A * B - 1) / (A * B)), block(nw * 64);
    const int pairs = flat ? groups : 0, nq_nw = nq | nw << 16;
    const unsigned char* q = static_cast<const unsigned char*>(g.base_qkv);
    unsigned char* c = static_cast<unsigned char*>(g.base_ctx);
    // DEEP costs a block of loads that read nothing, and gains where wavefronts are many and loop: 32 / 64 / 256 x 128 tokens of 12 heads 8.2, 11.8, 29.3 us with 2 to 3 %
    // less, 64 and 128 x 256, 16 x 512 3 to 7 %; 1 x 20 to 512, 4 x 100, 3 x 300, 32 x 40, 272 x 20, 512 x 32 1 to 4 % more, 7 x 509 level (16 heads 8.4 and
    // 9.9).
    const bool deep = S > 50 && (long)B * S >= 4096;
    auto launch = [&](auto kfn, auto a) { hipLaunchKernelGGL(kfn, grid, block, 0, stream, q, c, seq_start, seq_len, B, S, A, nq_nw, pairs, G, g, a); };
    if (ahead.blocks()) ks == 2 ? launch(attention_tiled_kernel<2, false, ReadAhead>, ahead) : launch(attention_tiled_kernel<1, false, ReadAhead>, ahead);
    else if (deep) ks == 2 ? launch(attention_tiled_kernel<2, true, NoAhead>, NoAhead{}) : launch(attention_tiled_kernel<1, true, NoAhead>, NoAhead{});
    else ks == 2 ? launch(attention_tiled_kernel<2, false, NoAhead>, NoAhead{}) : launch(attention_tiled_kernel<1, false, NoAhead>, NoAhead{});
    return hipGetLastError();
}

}  // namespace mt
