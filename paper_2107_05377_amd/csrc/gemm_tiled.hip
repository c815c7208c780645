// bfloat16 contraction of the serving path:  C_g[M,N] = epi(A_g[M,K] * W_g[N,K]^T),  g = 0..G-1 in one launch, with both
// operands and the result in the panel layout of tiled_offset() (kernels.h): 32 rows form a panel, 8 consecutive columns of a
// panel's 32 rows are stored behind one another.  In that layout
//   - a 32 x 16 MFMA operand fragment is 1 KB of contiguous memory in lane order, so global -> LDS loads are copies of whole
//     128-byte lines (64-byte row pieces, as a 32-wide K slice of a row-major matrix has, halve the rate: 28 instead of 50 bytes
//     per clock and compute unit measured with all of them loading), fragment reads from LDS need no swizzle, and a fragment may as
//     well go straight from global memory to registers (48 KB by 4 wavefronts: 0.7 us, row-major 1.7 us);
//   - the accumulator of a 32x32 block (a lane holds 4 consecutive columns of one row) is stored directly in runs of 1 KB: no
//     trip through LDS in the epilogue.
//
// gemm_tiled_kernel.  A workgroup of 4 wavefronts owns TMI panels of rows x 256 columns (KW = 1: each wavefront 64 columns and all
// rows) or x 128 columns (KW = 2: two wavefronts share 64 columns and take half of K each).  The activation slice (64 of K)
// goes through a ring of LDS stages, shared by the wavefronts; a weight fragment is used by one wavefront only and is loaded into
// its registers NB slices ahead.  Per slice and wavefront: 8 TMI matrix instructions, 4 TMI fragment reads, 8 weight and TMI KW
// activation loads, one barrier.  That leaves LDS (32 KB of reads and 8 KB of writes per 512 matrix clocks at TMI = 8) and the
// load path (32 bytes per clock at TMI = 8, 48 at TMI = 4) below their limits; with the weights in LDS as well, LDS was the limit.
// A workgroup walks a list of tiles without draining: the loads of the next tile start during the last slices of a tile.
//
// FP8 operands (F8).  An E4M3 panel has 16 columns of its 32 rows in 512 bytes, as a bf16 panel has 8, so all of the above holds with a pair
// of E4M3 values in the place of a bf16 value (K, lda and ldw count pairs): the same copies and the same fragments, of which two, 64 K
// elements, make one v_mfma_scale_f32_32x32x64_f8f6f4 of twice the clocks.  The instruction also undoes the power of two that the weights were
// stored with.  The sum starts from zero, the bias comes last, as in gemm_fp8.hip: E4M3 roundings of the results amplify any other order.
//
// The number of rows is on the device, so the tile height is chosen there (pick_height): the height with the smallest
// (tiles per compute unit, rounded up) x (height + fixed cost).  18.6 k rows x 2304 columns are 5.1 tiles of 128 rows per compute
// unit, i.e. 6 rounds, but 6.8 of 96 rows.
#include "kernels.h"
#include "device_util.h"

namespace mt {

namespace {

constexpr int kXcds = 8;
constexpr int kBand = 8;                // row-tiles per raster band

typedef __attribute__((address_space(3))) void* lptr_t;
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

template <int ACT>
__device__ __forceinline__ float t_act(float v)
{
    if constexpr (ACT == ACT_GELU_ERF) return gelu_erf_fast(v);
    else if constexpr (ACT == ACT_GELU_TANH) return gelu_tanh(v);
    else if constexpr (ACT == ACT_TANH) return tanhf(v);
    else return v;
}

// A fragment: 32 rows x 16 bf16 columns (1 KB), or 32 rows x 64 E4M3 columns (two runs of 1 KB).
template <bool F8> struct TFrag { typedef bf16x8 type; };
template <> struct TFrag<true> { typedef i32x8 type; };
// acc += first * second^T.  scale: of the first operand, an E8M0 exponent in every byte; the second one's is 1.
template <bool F8>
__device__ __forceinline__ f32x16 t_mfma(const typename TFrag<F8>::type& a, const typename TFrag<F8>::type& b, const f32x16& c, int scale)
{
    if constexpr (F8) return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, scale, 0, 0x7F7F7F7F);
    else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ i32x8 t_join(const i32x4& lo, const i32x4& hi) { return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7); }
// 32 E4M3 columns of a row, 16 each in the lanes of its two halves, from 4 of every 8 per lane (the accumulator's order)
template <int ACT>
__device__ __forceinline__ u32x4 t_pack_e4m3(const f32x16& v)
{
    uint32_t d[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        d[q] = pack_e4m3(t_act<ACT>(v[q * 4]), t_act<ACT>(v[q * 4 + 1]), t_act<ACT>(v[q * 4 + 2]), t_act<ACT>(v[q * 4 + 3]));
        __builtin_amdgcn_sched_barrier(0);           // (four at a time, for the registers)
    }
    const auto a = __builtin_amdgcn_permlane32_swap(d[0], d[2], false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(d[1], d[3], false, false);
    return u32x4{a[0], a[1], b[0], b[1]};
}
// ... and where they are stored (tiled_offset_e4m3)
__device__ __forceinline__ unsigned char* t_e4m3_at(unsigned char* c, int ldc, int pm, int pn, int lane)
{
    return c + (size_t)pm * 32 * ldc + (pn >> 1) * 2048 + (lane >> 5) * 1024 + (pn & 1) * 512 + (lane & 31) * 16;
}
// The exponent stands in front of an E4M3 matrix (kScaleSlot).  Read through the scalar cache.
__device__ __forceinline__ int t_scale(const unsigned char* w)
{
    typedef const __attribute__((address_space(4))) int* cptr_t;
    return *(cptr_t)(reinterpret_cast<uintptr_t>(w) - kScaleSlot);
}

// Scheduling of one K step: NM matrix instructions, PER fragment reads behind each of the first ones (the rest of the step covers
// their latency), the step's NV weight loads last.
template <int NM, int NF, int PER, int NV>
__device__ __forceinline__ void t_interleave()
{
    if constexpr (NM > 0) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if constexpr (NF > 0) __builtin_amdgcn_sched_group_barrier(0x100, NF < PER ? NF : PER, 0);
        t_interleave<NM - 1, (NF > PER ? NF - PER : 0), PER, NV>();
    } else {
        __builtin_amdgcn_sched_group_barrier(0x020, NV, 0);
    }
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t t_rsrc(const void* base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}

// Ring depth and weight prefetch distance by tile height: as deep as two (KW = 1, TMI <= 4: 80 KB of LDS and 256 registers each)
// or one workgroup per compute unit allow, and within the 63 loads that a wait can count.
template <int TMI, int KW, bool F8, bool SPREAD_ = (TMI >= 7)>
struct TCfg {
    static constexpr int WN = 4 / KW;                                   // wavefronts along N
    static constexpr int AL = KW * TMI;                                 // activation loads per wavefront and slice
    static constexpr int STAGE = AL * 4096;
    static constexpr int NB = TMI >= 4 ? 2 : (TMI == 3 ? 3 : 4);        // weight slices in registers
    static constexpr int S = TMI >= 7 ? 4 : (TMI >= 5 ? 5 : (KW == 2 ? (TMI == 4 ? 3 : (TMI == 3 ? 4 : 5)) : (TMI == 4 ? 5 : 6)));
    static constexpr int XCHG = KW == 2 ? TMI * 4096 * 4 : 0;           // partial sums of the K halves
    static constexpr int LDS = S * STAGE + XCHG;
    // loads younger than the activation slice that must have landed at a slice's barrier, on every path (see below)
    static constexpr int STEPS = F8 ? 2 : 4;                            // matrix steps of a slice
    static constexpr bool SPREAD = SPREAD_;                             // loads one by one between the matrix instructions (slice_spread)
    static_assert(!SPREAD || (!F8 && KW == 1), "slice_spread loads bfloat16 weights in four steps");
    static constexpr int WAIT = (S - 2) * AL + 8 - 8 / STEPS + 8 * (NB < S - 2 ? NB : S - 2) - (SPREAD && NB >= S - 2 ? 8 - 8 / STEPS : 0);
    // activation fragments of two steps, or (where the registers of two workgroups do not hold two) each reloaded behind its last use
    static constexpr bool IN_PLACE = F8 && KW == 1 && TMI == 4;
    static_assert(WAIT <= 63 && LDS <= 160 * 1024, "ring");
};

template <int TMI, int KW, int OUT, int ACT, bool F8, bool SPREAD = (TMI >= 7)>
__device__ __forceinline__ void gemm_tiled_body(const TiledGroup& g, const TiledShape& s, unsigned char* lds, int panels_m)
{
    using Cfg = TCfg<TMI, KW, F8, SPREAD>;
    static_assert(!F8 || KW == 1, "");
    constexpr int S = Cfg::S, NB = Cfg::NB, WN = Cfg::WN, AL = Cfg::AL, STAGE = Cfg::STAGE, STEPS = Cfg::STEPS, STEP_BYTES = 4096 / STEPS;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wn = wave % WN, wk = wave / WN;
    const int panels_n = s.N >> 5;
    const int tiles_m = (panels_m + TMI - 1) / TMI, tiles_n = (panels_n + 2 * WN - 1) / (2 * WN);
    const int per_problem = tiles_m * tiles_n, total = s.G * s.splits * per_problem;
    // this workgroup's tiles: XCD x owns a contiguous range of the tile order, its workgroups stride through it
    const int xcd = blockIdx.x % kXcds, wi = blockIdx.x / kXcds, wg_x = ((int)gridDim.x - xcd + kXcds - 1) / kXcds;
    const int q8 = total / kXcds, r8 = total % kXcds, lo = xcd * q8 + min(xcd, r8), cnt = q8 + (xcd < r8 ? 1 : 0);
    if (wi >= cnt) return;                                                   // uniform over the workgroup
    const int n_mine = (cnt - wi + wg_x - 1) / wg_x;
    const int KT = s.K / (64 * KW) / s.splits;                               // slices of a wavefront's K range
    const uint32_t pa = (uint32_t)s.lda * 64, pw = (uint32_t)s.ldw * 64;     // bytes per panel
    const int voff = lane * 16;

    struct Ref {
        // A starts at the tile's first panel (the whole operand may exceed the 31 bits of an offset); a panel beyond the last one lies
        // beyond the buffer's end: reads as zero
        __amdgpu_buffer_rsrc_t A, W;
        int ao, wo, grp, split, pm0, pn0, scale;
    };
    [[maybe_unused]] float bias_v = 0.f;       // F8: the bias of the wavefront's 64 columns, one per lane
    auto locate = [&](int j, Ref& t) {
        const int tile = lo + wi + j * wg_x;
        const int gs = tile / per_problem, tt = tile - gs * per_problem;
        t.grp = gs / s.splits;
        t.split = gs - t.grp * s.splits;
        const int band_sz = kBand * tiles_n, band = tt / band_sz, rows_in_band = min(kBand, tiles_m - band * kBand), tb = tt - band * band_sz;
        const int tn = tb / rows_in_band, tm = band * kBand + tb % rows_in_band;
        t.pm0 = tm * TMI;
        t.pn0 = (tn * WN + wn) * 2;
        const int k0 = t.split * KW * KT * 4096;                             // byte offset of the K range inside a panel
        t.A = t_rsrc(static_cast<const unsigned char*>(g.A) + (size_t)g.a[t.grp] * 256 + (size_t)t.pm0 * pa, min(panels_m - t.pm0, TMI) * pa);
        t.W = t_rsrc(static_cast<const unsigned char*>(g.W) + (size_t)g.w[t.grp] * 256, panels_n * pw);
        t.scale = F8 ? t_scale(static_cast<const unsigned char*>(g.W) + (size_t)g.w[t.grp] * 256) : 0;
        t.ao = k0 + wave * 1024;
        t.wo = t.pn0 * (int)pw + k0 + wk * KT * 4096;
    };
    Ref cur, nxt;
    locate(0, cur);
    if (n_mine > 1) locate(1, nxt);
    else nxt = cur;                        // no next tile: its loads are repeats of this one, never read

    auto issueA1 = [&](const Ref& t, int kt, int stage, int i) {          // wavefront w fetches K step w of every panel
        __builtin_amdgcn_raw_ptr_buffer_load_lds(t.A, (lptr_t)(lds + stage * STAGE + (i * 4 + wave) * 1024), 16, voff,
                                                 t.ao + (i % TMI) * (int)pa + ((i / TMI) * KT + kt) * 4096, 0, 0);
    };
    auto issueA = [&](const Ref& t, int kt, int stage) {
#pragma unroll
        for (int i = 0; i < AL; ++i) issueA1(t, kt, stage, i);
    };
    typename TFrag<F8>::type wf[NB][STEPS][2], af[Cfg::IN_PLACE ? 1 : 2][TMI];
    f32x16 acc[TMI][2];
    [[maybe_unused]] auto loadW1 = [&](const Ref& t, int kt, int buf, int step, int jn) {
        if constexpr (!F8)
            wf[buf][step][jn] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(t.W, voff + step * STEP_BYTES, t.wo + jn * (int)pw + kt * 4096, 0));
    };
    auto loadW = [&](const Ref& t, int kt, int buf, int step) {
#pragma unroll
        for (int jn = 0; jn < 2; ++jn) {
            const auto lo = __builtin_amdgcn_raw_buffer_load_b128(t.W, voff + step * STEP_BYTES, t.wo + jn * (int)pw + kt * 4096, 0);
            if constexpr (F8) {
                const auto hi = __builtin_amdgcn_raw_buffer_load_b128(t.W, voff + step * STEP_BYTES + 1024, t.wo + jn * (int)pw + kt * 4096, 0);
                wf[buf][step][jn] = t_join(__builtin_bit_cast(i32x4, lo), __builtin_bit_cast(i32x4, hi));
            } else {
                wf[buf][step][jn] = __builtin_bit_cast(bf16x8, lo);
            }
        }
    };
    auto read1 = [&](int buf, int stage, int step, int i) {
        const unsigned char* p = lds + stage * STAGE + (wk * TMI + i) * 4096 + step * STEP_BYTES + voff;
        if constexpr (F8) af[buf][i] = t_join(*reinterpret_cast<const i32x4*>(p), *reinterpret_cast<const i32x4*>(p + 1024));
        else af[buf][i] = *reinterpret_cast<const bf16x8*>(p);
    };
    auto readA = [&](int buf, int stage, int step) {
#pragma unroll
        for (int i = 0; i < TMI; ++i) read1(buf, stage, step, i);
    };
    // accumulators start from the bias (the first K share's do), with E4M3 operands from zero
    auto init_acc = [&](const Ref& t) {
        const uint32_t bo = t.split == 0 ? g.b[t.grp] : kNoBias;
        if constexpr (F8) {
            bias_v = bo == kNoBias ? 0.f : g.bias[(size_t)bo * 64 + min(t.pn0 * 32 + lane, s.N - 1)];
#pragma unroll
            for (int i = 0; i < TMI; ++i)
#pragma unroll
                for (int jn = 0; jn < 2; ++jn)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[i][jn][e] = 0.f;
            return;
        }
#pragma unroll
        for (int jn = 0; jn < 2; ++jn) {
            f32x16 b0;
#pragma unroll
            for (int e = 0; e < 16; ++e) b0[e] = 0.f;
            if (bo != kNoBias && (KW == 1 || wk == 0)) {
                const float* bp = g.bias + (size_t)bo * 64 + min(t.pn0 + jn, panels_n - 1) * 32 + (lane >> 5) * 4;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 v = *reinterpret_cast<const float4*>(bp + q * 8);
                    b0[q * 4] = v.x; b0[q * 4 + 1] = v.y; b0[q * 4 + 2] = v.z; b0[q * 4 + 3] = v.w;
                }
            }
#pragma unroll
            for (int i = 0; i < TMI; ++i) acc[i][jn] = b0;
        }
    };
    // How results are stored, TiledShape::stream (launch_tiles has the rule): past the second-level caches, or written through them.  Either way a kernel does
    // not end by writing back what is dirty (its readers run on other dies).
    auto store16 = [&](const u32x4& v, __amdgpu_buffer_rsrc_t C, int at) {
        if (s.stream) __builtin_amdgcn_raw_buffer_store_b128(v, C, at, 0, 2);
        else __builtin_amdgcn_raw_buffer_store_b128(v, C, at, 0, 16);
    };
    auto store_block = [&](const Ref& t, const f32x16& a, int pm, int pn) {
        if (pm >= panels_m || pn >= panels_n) return;                        // uniform
        unsigned char* Cb = static_cast<unsigned char*>(g.C) + (size_t)g.c[t.grp] * 256;
        if constexpr (OUT == TILED_E4M3) {
            const auto C = t_rsrc(t_e4m3_at(Cb, s.ldc, pm, pn, 0), 2048);
            store16(t_pack_e4m3<ACT>(a), C, (lane >> 5) * 1024 + (lane & 31) * 16);
        } else if constexpr (OUT == TILED_F32) {
            const auto C = t_rsrc(reinterpret_cast<float*>(Cb) + (size_t)t.split * s.split_stride + (size_t)pm * 32 * s.ldc + pn * 1024, 4096);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                store16(__builtin_bit_cast(u32x4, f32x4{a[q * 4], a[q * 4 + 1], a[q * 4 + 2], a[q * 4 + 3]}), C, (lane & 31) * 32 + (lane >> 5) * 16 + q * 1024);
        } else {
            const auto C = t_rsrc(reinterpret_cast<__bf16*>(Cb) + (size_t)pm * 32 * s.ldc + pn * 1024, 2048);
            [[maybe_unused]] f32x16 tr;
#pragma unroll
            for (int qp = 0; qp < 2; ++qp) {
                bf16x4 x, y;                                                 // 4 of the 8 columns of two neighbouring chunks
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[e] = (__bf16)t_act<ACT>(a[qp * 8 + e]);
                    y[e] = (__bf16)t_act<ACT>(a[qp * 8 + 4 + e]);
                }
                // the half wavefronts exchange so that the lower one holds all of the first chunk, the upper one all of the second
                const u32x2 xu = __builtin_bit_cast(u32x2, x), yu = __builtin_bit_cast(u32x2, y);
                const auto s0 = __builtin_amdgcn_permlane32_swap(xu[0], yu[0], false, false);
                const auto s1 = __builtin_amdgcn_permlane32_swap(xu[1], yu[1], false, false);
                const u32x4 r = u32x4{s0[0], s1[0], s0[1], s1[1]};
                if constexpr (ACT == ACT_NONE && !F8) {
                    if (s.vt_panel && pn >= s.vt_panel) {
                        // transposed: the half block just formed is a matrix operand (32 rows x 16 columns); its product with the
                        // unit matrix moves the columns to the lanes, exactly (exchanging the operands of the whole tile instead
                        // needs a second copy of the main loop, which did not fit the registers)
                        const int d = (lane & 31) - qp * 16 - (lane >> 5) * 8;
                        u32x4 unit;
#pragma unroll
                        for (int e = 0; e < 4; ++e) unit[e] = d == 2 * e ? 0x3F80u : (d == 2 * e + 1 ? 0x3F800000u : 0u);
                        if (qp == 0) {
#pragma unroll
                            for (int e = 0; e < 16; ++e) tr[e] = 0.f;
                        }
                        tr = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, r), __builtin_bit_cast(bf16x8, unit), tr, 0, 0, 0);
                        if (qp == 1) {
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                bf16x8 v;
#pragma unroll
                                for (int e = 0; e < 8; ++e) v[e] = (__bf16)tr[h * 8 + e];
                                store16(__builtin_bit_cast(u32x4, v), C, lane * 16 + h * 1024);
                            }
                        }
                        continue;
                    }
                }
                store16(r, C, lane * 16 + qp * 1024);
            }
        }
    };

    // ---- fill, in the order of the steady state (iteration i: activation slice i + S - 1, then weight slice i + NB)
#pragma unroll
    for (int i = -(S - 1); i < 0; ++i) {
        if (i + S - 1 < KT) issueA(cur, i + S - 1, i + S - 1);
        else issueA(nxt, i + S - 1 - KT, i + S - 1);
        if (i + NB >= 0) {
#pragma unroll
            for (int st = 0; st < STEPS; ++st) loadW(i + NB < KT ? cur : nxt, i + NB < KT ? i + NB : i + NB - KT, (i + NB) % NB, st);
        }
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 2) * AL + 8 * (NB < S - 1 ? NB : S - 1) < 63 ? (S - 2) * AL + 8 * (NB < S - 1 ? NB : S - 1) : 63) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    readA(0, 0, 0);

    // ---- slices of all tiles in one sequence; the weight buffer of a slice is its number in the sequence modulo NB
    int st = 0, kt = 0, j = 0;                 // ring stage, slice of the tile, tile
    auto slice = [&](auto bufc) {
        constexpr int buf = decltype(bufc)::value;
        const int ka = kt + S - 1, kw = kt + NB;
        const Ref ta = ka < KT ? cur : nxt, tw = kw < KT ? cur : nxt;
        const int ps = st == 0 ? S - 1 : st - 1, ns = st + 1 == S ? 0 : st + 1;
        issueA(ta, ka < KT ? ka : ka - KT, ps);            // into the stage of the slice before, which everyone has read
#pragma unroll
        for (int step = 0; step < STEPS; ++step) {
            const bool last = step + 1 == STEPS;
            if (last) {
                // this slice is in registers and the next one must have landed, for every wavefront.  Loads return in order; those
                // younger than the next slice's are S - 2 activation slices and at least min(NB, S - 2) weight slices and all steps but one.
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(Cfg::WAIT) : "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            if constexpr (!Cfg::IN_PLACE) readA((step + 1) & 1, last ? ns : st, last ? 0 : step + 1);
#pragma unroll
            for (int i = 0; i < TMI; ++i) {
#pragma unroll
                for (int jn = 0; jn < 2; ++jn) acc[i][jn] = t_mfma<F8>(wf[buf][step][jn], af[Cfg::IN_PLACE ? 0 : step & 1][i], acc[i][jn], cur.scale);
                if constexpr (Cfg::IN_PLACE) read1(0, last ? ns : st, last ? 0 : step + 1, i);
            }
            loadW(tw, kw < KT ? kw : kw - KT, buf, step);
            if constexpr (!Cfg::IN_PLACE) t_interleave<TMI * 2, F8 ? 2 * TMI : TMI, F8 ? 4 : 2, 8 / STEPS>();
            __builtin_amdgcn_sched_barrier(0);
        }
        st = ns;
        ++kt;
    };
    // The same with the loads spread: a wavefront whose load waits for the load path issues no matrix instruction either, and a tall tile's compute unit
    // has no other.  18.6 k rows x 768 x 3072 78.5 -> 75.8 us (7 panels), 20.5 k x 1024 x 4096 159 -> 154 (5), 8 problems of 20 k 1130 -> 1070 (7).  (Where
    // two workgroups share a compute unit, and with K halved between wavefronts, it was level to 14 % slower.)  A step has its share of the activation slice
    // (the last one none) and the weight registers that the step before has used.
    [[maybe_unused]] auto slice_spread = [&](auto bufc) {
        constexpr int buf = decltype(bufc)::value;
        const int ka = kt + S - 1, kw = kt + NB, kp = kw - 1;
        const Ref ta = ka < KT ? cur : nxt, tw = kw < KT ? cur : nxt, tp = kp < KT ? cur : nxt;
        const int ps = st == 0 ? S - 1 : st - 1, ns = st + 1 == S ? 0 : st + 1;
        auto one_step = [&](auto stepc) {
            constexpr int step = decltype(stepc)::value, NM = 2 * TMI;
            constexpr bool last = step + 1 == STEPS;
            if constexpr (last) {
                // as above; of the slice that issued the awaited one, only the last step's weight loads are certainly younger (in the fill: all 8)
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(Cfg::WAIT) : "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            constexpr int a0 = last ? AL : AL * step / (STEPS - 1), a1 = last ? AL : AL * (step + 1) / (STEPS - 1), NL = a1 - a0 + 2, M0 = (TMI + 1) / 2;
            int l = 0, f = 0;
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const int i = m >> 1, jn = m & 1;
                acc[i][jn] = t_mfma<F8>(wf[buf][step][jn], af[step & 1][i], acc[i][jn], cur.scale);
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    if (f < TMI) read1((step + 1) & 1, last ? ns : st, last ? 0 : step + 1, f++);
                const int due = m == NM - 1 ? NL : (m < M0 ? 0 : NL * (m - M0 + 1) / (NM - M0));
#pragma unroll
                for (int k = 0; k < NL; ++k)
                    if (l < due) {
                        const int w = l - (a1 - a0);
                        if (w < 0) issueA1(ta, ka < KT ? ka : ka - KT, ps, a0 + l);
                        else if (step == 0) loadW1(tp, kp < KT ? kp : kp - KT, (buf + NB - 1) % NB, STEPS - 1, w);
                        else loadW1(tw, kw < KT ? kw : kw - KT, buf, step - 1, w);
                        ++l;
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        one_step(std::integral_constant<int, 0>{});
        one_step(std::integral_constant<int, 1>{});
        one_step(std::integral_constant<int, 2>{});
        one_step(std::integral_constant<int, 3>{});
        st = ns;
        ++kt;
    };
    auto epilogue = [&]() {
        if constexpr (F8) {
#pragma unroll
            for (int jn = 0; jn < 2; ++jn) {
                float b[16];
#pragma unroll
                for (int e = 0; e < 16; ++e) b[e] = __shfl(bias_v, jn * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3), 64);
#pragma unroll
                for (int i = 0; i < TMI; ++i) {
                    f32x16 a;
#pragma unroll
                    for (int e = 0; e < 16; ++e) a[e] = acc[i][jn][e] + b[e];
                    store_block(cur, a, cur.pm0 + i, cur.pn0 + jn);
                }
            }
        } else if constexpr (KW == 1) {
#pragma unroll
            for (int i = 0; i < TMI; ++i)
#pragma unroll
                for (int jn = 0; jn < 2; ++jn) store_block(cur, acc[i][jn], cur.pm0 + i, cur.pn0 + jn);
        } else {
            // the wavefronts of a pair exchange a column block: each finishes one
            float* x = reinterpret_cast<float*>(lds + S * STAGE);
            float* mine = x + (wk * WN + wn) * TMI * 1024;
            const float* other = x + ((1 - wk) * WN + wn) * TMI * 1024;
#pragma unroll
            for (int i = 0; i < TMI; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) mine[(i * 16 + e) * 64 + lane] = wk == 0 ? acc[i][1][e] : acc[i][0][e];
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
#pragma unroll
            for (int i = 0; i < TMI; ++i) {
                f32x16 a;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float o = other[(i * 16 + e) * 64 + lane];
                    a[e] = wk == 0 ? acc[i][0][e] + o : o + acc[i][1][e];
                }
                store_block(cur, a, cur.pm0 + i, cur.pn0 + wk);
            }
        }
        cur = nxt;
        kt = 0;
        ++j;
        if (j + 1 < n_mine) locate(j + 1, nxt);
    };
    // true when the last tile is done
    auto finish_tile = [&]() {
        if (kt < KT) return false;
        epilogue();
        if (j == n_mine) return true;
        init_acc(cur);
        return false;
    };
    if constexpr (NB == 2) {                               // an even number of slices: one copy of the epilogue
        while (j < n_mine) {
            init_acc(cur);
            while (kt < KT) {
                if constexpr (Cfg::SPREAD) {
                    slice_spread(std::integral_constant<int, 0>{});
                    slice_spread(std::integral_constant<int, 1>{});
                } else {
                    slice(std::integral_constant<int, 0>{});
                    slice(std::integral_constant<int, 1>{});
                }
            }
            epilogue();
        }
    } else {
        init_acc(cur);
        for (;;) {
            slice(std::integral_constant<int, 0>{});
            if (finish_tile()) break;
            slice(std::integral_constant<int, 1>{});
            if (finish_tile()) break;
            slice(std::integral_constant<int, 2>{});
            if (finish_tile()) break;
            if constexpr (NB > 3) {
                slice(std::integral_constant<int, 3>{});
                if (finish_tile()) break;
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the repeat loads must land before the LDS is released
}

// Tile height in panels, MINT .. MAXT: fewest rounds x cost of a tile.  Two workgroups on a compute unit share it, so rounds count
// tiles per compute unit; the fixed cost of a tile (fill, epilogue) is about that of 0.7 panels at K = 768.
// E4M3 operands: half the slices for the same epilogue, so the fixed cost counts for more (it stands still in slices), and the
// three-panel form, which has three copies of the epilogue, loses everywhere (18.6 k rows x 2304 x 768: 1 to 4 panels 64, 65, 71, 45 us; x 3072 83, 63, 61, 51;
// 2.3 k rows x 2304 13.0, 16.1, 17.9, 12.6).
template <int MINT, int MAXT, bool F8>
__device__ __forceinline__ int pick_height(int panels_m, int tiles_per_row, int n_cu, int slices)
{
    int best = MINT;
    float best_cost = 3.4e38f;
#pragma unroll
    for (int t = MAXT; t >= MINT; --t) {
        if (t >= 4 && (slices & 1)) continue;              // two weight buffers go with an even number of slices
        if (F8 && t == 3) continue;
        const int tiles = (panels_m + t - 1) / t * tiles_per_row;
        const float cost = (float)((tiles + n_cu - 1) / n_cu) * ((float)t + (F8 ? 8.4f / (float)slices : 0.7f));
        if (cost < best_cost) {
            best_cost = cost;
            best = t;
        }
    }
    return best;
}

template <int KW, int MAXT, int OUT, int ACT, bool F8>
__global__ __launch_bounds__(256, (MAXT <= 4 && KW == 1) ? 2 : 1) void gemm_tiled_kernel(TiledGroup g, TiledShape s, int n_cu, int force)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int M = s.d_M ? min(s.M, *s.d_M) : s.M;
    const int panels_m = (M + 31) >> 5;
    const int slices = s.K / (64 * KW) / s.splits;
    const int per_row = ((s.N >> 5) + 8 / KW - 1) / (8 / KW) * s.G * s.splits;
    if constexpr (MAXT == 8) {
        // Tall tiles spread their loads.  With 5 and 6 panels there are fewer matrix instructions to hide them behind: one and two problems 0.97 to 1.00 of the
        // time (4.9 and 5.7 k rows x 1024 x 4096, 2 problems, 74.9, 84.1 -> 72.8, 82.2 us), four 0.99 to 1.06 (140.8 -> 145.4; 5.7 k x 768 x 3072 106.7 ->
        // 113.5), eight 0.97 to 1.02.
        const bool spread = s.G <= 2;
        switch (force ? force : pick_height<5, 8, F8>(panels_m, per_row, n_cu, slices)) {
            case 8: gemm_tiled_body<8, KW, OUT, ACT, F8>(g, s, lds, panels_m); break;
            case 7: gemm_tiled_body<7, KW, OUT, ACT, F8>(g, s, lds, panels_m); break;
            case 6:
                if (spread) gemm_tiled_body<6, KW, OUT, ACT, F8, true>(g, s, lds, panels_m);
                else gemm_tiled_body<6, KW, OUT, ACT, F8>(g, s, lds, panels_m);
                break;
            default:
                if (spread) gemm_tiled_body<5, KW, OUT, ACT, F8, true>(g, s, lds, panels_m);
                else gemm_tiled_body<5, KW, OUT, ACT, F8>(g, s, lds, panels_m);
                break;
        }
    } else {
        switch (force ? force : pick_height<1, MAXT, F8>(panels_m, per_row, n_cu, slices)) {
            case 4: gemm_tiled_body<4, KW, OUT, ACT, F8>(g, s, lds, panels_m); break;
            case 3:
                if constexpr (!F8) gemm_tiled_body<3, KW, OUT, ACT, F8>(g, s, lds, panels_m);
                break;
            case 2: gemm_tiled_body<2, KW, OUT, ACT, F8>(g, s, lds, panels_m); break;
            default: gemm_tiled_body<1, KW, OUT, ACT, F8>(g, s, lds, panels_m); break;
        }
    }
}

// gemm_tiled_rows_kernel.  Few rows: TM x TN panels of output per workgroup, each of its 4 wavefronts a quarter of K, both operands
// straight from global memory to registers with all loads of a quarter of K = 768 in flight at once, one exchange of partial sums
// through LDS.  Such a launch is a chain of latencies (of 5.3 us at 36 rows x 2304 x 768: 1.3 from the launch before, 1.1 until the
// row count was known, 2.2 loads, 0.4 the rest), so the chain is kept short: what the first addresses need are the leading, scalar
// arguments, which the command processor preloads into registers, and the loads go out before the row count has arrived (panels
// beyond it are memory of the operand all the same).
// Packed: lda_ldw = widths in 16 columns, lda | ldw << 16; steps_pn = K steps of 16 per wavefront | column panels << 16; ldc_pm = width
// of C in 8 columns | first row panel / 65536 << 16 (more row panels than a grid can have take several launches, see launch_rows).
constexpr int kLaunchPanels = 65536;
template <int TM, int TN, int OUT, int ACT>
__device__ __forceinline__ void gemm_tiled_rows_body(const unsigned char* A, const unsigned char* W, unsigned char* C, const float* bias,
                                                     const int32_t* d_M, uint32_t lda_ldw, uint32_t steps_pn, uint32_t ldc_pm, int M, int split,
                                                     int64_t split_stride, int vt_panel)
{
    constexpr int U = 12, NBLK = TM * TN;
    __shared__ __attribute__((aligned(16))) float part[4][NBLK][4][64][4];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rows_here = *(d_M ? d_M : reinterpret_cast<const int32_t*>(A));     // in flight until the stores
    const int steps = steps_pn & 0xFFFF, panels_n = steps_pn >> 16, bound_m = (M + 31) >> 5;
    const int pn0 = blockIdx.x * TN, pm0 = (int)blockIdx.y * TM + (int)(ldc_pm & ~0xFFFFu);
    const size_t pa = (size_t)(lda_ldw & 0xFFFF) * 1024, pw = (size_t)(lda_ldw >> 16) * 1024;      // bytes per panel
    const size_t k0 = (size_t)(split * 4 + wave) * steps * 1024 + lane * 16;
    const unsigned char* a[TM];
    const unsigned char* w[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) a[i] = A + min(pm0 + i, bound_m - 1) * pa + k0;
#pragma unroll
    for (int j = 0; j < TN; ++j) w[j] = W + min(pn0 + j, panels_n - 1) * pw + k0;
    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    // blocks to store transposed are computed transposed (vt_panel is even: both column panels of a workgroup are, or none)
    const bool vt = OUT == TILED_BF16 && ACT == ACT_NONE && vt_panel && pn0 >= vt_panel;
    float4 bv[TN];
    int panels_m = 0;
    // one batch of steps: all its loads are issued before its first product (a full batch without conditions: guarded loads are
    // branches, and the loads then go out one by one)
    auto batch = [&](int s0, int nb, auto full, auto first) {
        bf16x8 af[U][TM], wf[U][TN];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (full || u < nb) {
#pragma unroll
                for (int j = 0; j < TN; ++j) wf[u][j] = *reinterpret_cast<const bf16x8*>(w[j] + (size_t)(s0 + u) * 1024);
#pragma unroll
                for (int i = 0; i < TM; ++i) af[u][i] = *reinterpret_cast<const bf16x8*>(a[i] + (size_t)(s0 + u) * 1024);
            }
        if constexpr (first) {
            // this wavefront finishes chunk `wave` of every block
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                bv[j] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (bias && split == 0) {
                    const float* bp = bias + min(pn0 + j, panels_n - 1) * 32;
                    if (vt) bv[j].x = bv[j].y = bv[j].z = bv[j].w = bp[lane & 31];
                    else bv[j] = *reinterpret_cast<const float4*>(bp + wave * 8 + (lane >> 5) * 4);
                }
            }
            asm volatile("" ::: "memory");                                   // the loads stay in front of the exit
            panels_m = ((d_M ? min(M, rows_here) : M) + 31) >> 5;
            if (pm0 >= panels_m) return false;
        }
        __builtin_amdgcn_sched_barrier(0);
        auto products = [&](auto swap) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (full || u < nb) {
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j) {
                            if constexpr (swap) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[u][i], wf[u][j], acc[i][j], 0, 0, 0);
                            else acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[u][j], af[u][i], acc[i][j], 0, 0, 0);
                        }
                }
        };
        if constexpr (OUT == TILED_BF16 && ACT == ACT_NONE) {
            if (vt) {
                products(std::true_type{});
                return true;
            }
        }
        products(std::false_type{});
        return true;
    };
    int s0 = 0;
    if (steps >= U) {
        if (!batch(0, U, std::true_type{}, std::true_type{})) return;
        for (s0 = U; s0 + U <= steps; s0 += U) batch(s0, U, std::true_type{}, std::false_type{});
        if (s0 < steps) batch(s0, steps - s0, std::false_type{}, std::false_type{});
    } else if (!batch(0, steps, std::false_type{}, std::true_type{})) {
        return;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<f32x4*>(part[wave][i * TN + j][q][lane]) = f32x4{acc[i][j][q * 4], acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2], acc[i][j][q * 4 + 3]};
    __syncthreads();
    const size_t pc = (size_t)(ldc_pm & 0xFFFF) * 256;                       // elements per panel of C
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int pm = pm0 + i, pn = pn0 + j;
            if (pm >= panels_m || pn >= panels_n) continue;
            f32x4 v = *reinterpret_cast<const f32x4*>(part[0][i * TN + j][wave][lane]);
#pragma unroll
            for (int p = 1; p < 4; ++p) v += *reinterpret_cast<const f32x4*>(part[p][i * TN + j][wave][lane]);
            v[0] = t_act<ACT>(v[0] + bv[j].x);
            v[1] = t_act<ACT>(v[1] + bv[j].y);
            v[2] = t_act<ACT>(v[2] + bv[j].z);
            v[3] = t_act<ACT>(v[3] + bv[j].w);
            const size_t at = pm * pc + pn * 1024 + (vt ? (wave >> 1) * 512 + lane * 8 + (wave & 1) * 4 : wave * 256 + (lane & 31) * 8 + (lane >> 5) * 4);
            if constexpr (OUT == TILED_F32) {
                *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(C) + (size_t)split * split_stride + at) = v;
            } else {
                const bf16x4 o = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
                *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(C) + at) = o;
            }
        }
}

template <int TM, int TN, int OUT, int ACT>
__global__ __launch_bounds__(256, TM * TN > 1 ? 1 : 2) void gemm_tiled_rows_kernel(const unsigned char* A, const unsigned char* W, unsigned char* C,
                                                                                   const float* bias, const int32_t* d_M, uint32_t lda_ldw,
                                                                                   uint32_t steps_pn, uint32_t ldc_pm, int M, int vt_panel, int64_t split_stride)
{
    gemm_tiled_rows_body<TM, TN, OUT, ACT>(A, W, C, bias, d_M, lda_ldw, steps_pn, ldc_pm, M, blockIdx.z, split_stride, vt_panel);
}

// several problems, and problems of n_sub equal ones
template <int TM, int TN, int OUT, int ACT>
__global__ __launch_bounds__(256, TM * TN > 1 ? 1 : 2) void gemm_tiled_rows_group_kernel(const int32_t* d_M, uint32_t lda_ldw, uint32_t steps_pn,
                                                                                         uint32_t ldc_pm, int M, TiledGroup g, TiledShape s)
{
    const int n_sub = s.n_sub > 1 ? s.n_sub : 1;
    const int sub = blockIdx.z % n_sub, gz = blockIdx.z / n_sub;
    const int grp = gz / s.splits, split = gz - grp * s.splits;
    const float* bias = g.b[grp] == kNoBias ? nullptr : g.bias + (size_t)(g.b[grp] + sub * s.sub_b) * 64;
    gemm_tiled_rows_body<TM, TN, OUT, ACT>(static_cast<const unsigned char*>(g.A) + (size_t)(g.a[grp] + sub * s.sub_a) * 256,
                                                     static_cast<const unsigned char*>(g.W) + (size_t)(g.w[grp] + sub * s.sub_w) * 256,
                                                     static_cast<unsigned char*>(g.C) + (size_t)(g.c[grp] + sub * s.sub_c) * 256, bias, d_M, lda_ldw,
                                                     steps_pn, ldc_pm, M, split, s.split_stride, s.vt_panel);
}

// Few rows of E4M3 operands: a wavefront has a block of 32 rows x 32 columns and all of K, which it adds up in the order of the tile forms (a result
// is the same bits in either), operands straight from global memory to registers, the next batch of steps in flight while one is
// multiplied.  290 rows x 2304 / 768 / 3072 x 768, x 768 x 3072: 5.4, 4.2, 5.8, 9.2 us, tiles 7.5, 7.4, 8.2, 13.3.
template <int OUT, int ACT>
__global__ __launch_bounds__(256, 2) void gemm_tiled_rows_fp8_kernel(const int32_t* d_M, int pm0, TiledGroup g, TiledShape s)
{
    constexpr int U = 6;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), grp = blockIdx.z;
    const int rows_here = *(d_M ? d_M : reinterpret_cast<const int32_t*>(g.A));      // in flight with the first operands
    const int panels_n = s.N >> 5, pn = blockIdx.x * 4 + wave, pm = pm0 + blockIdx.y, steps = s.K >> 5;
    if (pn >= panels_n) return;
    const unsigned char* w = static_cast<const unsigned char*>(g.W) + (size_t)g.w[grp] * 256;
    const int scale = t_scale(w);
    const unsigned char* a = static_cast<const unsigned char*>(g.A) + (size_t)g.a[grp] * 256 + (size_t)pm * s.lda * 64 + lane * 16;
    w += (size_t)pn * s.ldw * 64 + lane * 16;
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    i32x8 af[2][U], wf[2][U];
    auto get = [](const unsigned char* p) { return t_join(*reinterpret_cast<const i32x4*>(p), *reinterpret_cast<const i32x4*>(p + 1024)); };
    auto fetch = [&](int buf, int s0) {                  // steps beyond the last one repeat it
#pragma unroll
        for (int u = 0; u < U; ++u) {
            wf[buf][u] = get(w + (size_t)min(s0 + u, steps - 1) * 2048);
            af[buf][u] = get(a + (size_t)min(s0 + u, steps - 1) * 2048);
        }
    };
    auto multiply = [&](int buf, int s0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (s0 + u < steps) acc = t_mfma<true>(wf[buf][u], af[buf][u], acc, scale);
    };
    fetch(0, 0);
    const uint32_t bo = g.b[grp];
    float4 b[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
        b[q] = bo == kNoBias ? make_float4(0.f, 0.f, 0.f, 0.f) : *reinterpret_cast<const float4*>(g.bias + (size_t)bo * 64 + pn * 32 + q * 8 + (lane >> 5) * 4);
    if (steps > U) fetch(1, U);
    asm volatile("" ::: "memory");
    if (pm * 32 >= (d_M ? min(s.M, rows_here) : s.M)) return;
    for (int s0 = 0;; s0 += 2 * U) {
        __builtin_amdgcn_sched_barrier(0);
        multiply(0, s0);
        if (s0 + U >= steps) break;
        if (s0 + 2 * U < steps) fetch(0, s0 + 2 * U);
        __builtin_amdgcn_sched_barrier(0);
        multiply(1, s0 + U);
        if (s0 + 2 * U >= steps) break;
        if (s0 + 3 * U < steps) fetch(1, s0 + 3 * U);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        acc[q * 4] += b[q].x;
        acc[q * 4 + 1] += b[q].y;
        acc[q * 4 + 2] += b[q].z;
        acc[q * 4 + 3] += b[q].w;
    }
    unsigned char* c = static_cast<unsigned char*>(g.C) + (size_t)g.c[grp] * 256;
    if constexpr (OUT == TILED_E4M3) {
        *reinterpret_cast<u32x4*>(t_e4m3_at(c, s.ldc, pm, pn, lane)) = t_pack_e4m3<ACT>(acc);
    } else if constexpr (OUT == TILED_F32) {
        float* f = reinterpret_cast<float*>(c) + (size_t)pm * 32 * s.ldc + pn * 1024 + (lane & 31) * 8 + (lane >> 5) * 4;
#pragma unroll
        for (int q = 0; q < 4; ++q) *reinterpret_cast<f32x4*>(f + q * 256) = f32x4{acc[q * 4], acc[q * 4 + 1], acc[q * 4 + 2], acc[q * 4 + 3]};
    } else {
        __bf16* h = reinterpret_cast<__bf16*>(c) + (size_t)pm * 32 * s.ldc + pn * 1024 + (lane & 31) * 8 + (lane >> 5) * 4;
#pragma unroll
        for (int q = 0; q < 4; ++q) *reinterpret_cast<bf16x4*>(h + q * 256) = bf16x4{(__bf16)acc[q * 4], (__bf16)acc[q * 4 + 1], (__bf16)acc[q * 4 + 2], (__bf16)acc[q * 4 + 3]};
    }
}

template <int KW, int MAXT, int OUT, int ACT, bool F8>
hipError_t launch_tiles(const TiledGroup& g, const TiledShape& s, int n_cu, int force, hipStream_t stream)
{
    constexpr int b0 = TCfg<MAXT, KW, F8>::LDS, b1 = TCfg<MAXT - 1, KW, F8>::LDS, b2 = TCfg<MAXT - 2, KW, F8>::LDS, b3 = TCfg<MAXT - 3, KW, F8>::LDS;
    constexpr int m0 = b0 > b1 ? b0 : b1, m1 = b2 > b3 ? b2 : b3, bytes = m0 > m1 ? m0 : m1;
    auto kfn = gemm_tiled_kernel<KW, MAXT, OUT, ACT, F8>;
    static std::atomic<uint64_t> lds_raised{0};
    if (bytes > 64 * 1024) {
        hipError_t e = ensure_dynamic_lds((const void*)kfn, bytes, lds_raised);
        if (e != hipSuccess) return e;
    }
    // one (two where two fit) workgroup per compute unit, fewer if the lowest tiles of the row bound are fewer
    const int low = MAXT == 8 ? 5 : 1;
    const long tiles = (long)(((s.M + 31) / 32 + low - 1) / low) * ((s.N / 32 + 8 / KW - 1) / (8 / KW)) * s.G * s.splits;
    const long slots = (long)n_cu * ((MAXT <= 4 && KW == 1) ? 2 : 1);
    const int n_wg = (int)(tiles < slots ? (tiles < kXcds ? kXcds : tiles) : slots);
    // Large results go past the second-level caches, whose 4 MB hold the operands that a compute unit's neighbours share; small ones are written through:
    // their readers follow at once and find them in the last-level cache.  Passes with ordinary stores, all past, all written through, this rule: base
    // 8 x 32 x 128 5777, 5724, 5779, 5721 us; 4 x 32 x 128 3304, 3301, 3275, 3223; 32 x 128 1287, 1261, 1249, 1247; 7 x 509 1211, 1209, 1187, 1191;
    // eight different forks, 64 x 128 2542, 2615, 2510, 2537; routed 32 x 128 1522, 1567, 1537, 1537.  The line, by the row bound: 32 x 128 rows of one
    // problem have 13 to 25 MB, 8 problems of them or 256 x 128 rows 100 MB and more.
    TiledShape t = s;
    t.stream = (long)s.M * s.N * s.G * s.splits * (OUT == TILED_F32 ? 4 : OUT == TILED_BF16 ? 2 : 1) > (64l << 20);
    hipLaunchKernelGGL(kfn, dim3(n_wg), dim3(256), bytes, stream, g, t, n_cu, force);
    return hipGetLastError();
}

template <int TM, int TN, int OUT, int ACT>
hipError_t launch_rows(const TiledGroup& g, const TiledShape& s, hipStream_t stream)
{
    const int n_sub = s.n_sub > 1 ? s.n_sub : 1, panels = (s.M + 31) / 32;
    if (TM == 1 && panels > 65535) return hipErrorInvalidValue;      // (choose_form takes it for up to 1152 blocks)
    const uint32_t lda_ldw = (uint32_t)(s.lda / 16) | (uint32_t)(s.ldw / 16) << 16, steps_pn = (uint32_t)(s.K / s.splits / 64) | (uint32_t)(s.N / 32) << 16;
    for (int pm0 = 0; pm0 < panels; pm0 += kLaunchPanels) {
        dim3 grid((s.N / 32 + TN - 1) / TN, (std::min(panels - pm0, kLaunchPanels) + TM - 1) / TM, s.G * s.splits * n_sub), block(256);
        const uint32_t ldc_pm = (uint32_t)(s.ldc / 8) | (uint32_t)pm0;
        if (s.G == 1 && n_sub == 1)
            hipLaunchKernelGGL((gemm_tiled_rows_kernel<TM, TN, OUT, ACT>), grid, block, 0, stream,
                               static_cast<const unsigned char*>(g.A) + (size_t)g.a[0] * 256, static_cast<const unsigned char*>(g.W) + (size_t)g.w[0] * 256,
                               static_cast<unsigned char*>(g.C) + (size_t)g.c[0] * 256, g.b[0] == kNoBias ? nullptr : g.bias + (size_t)g.b[0] * 64, s.d_M,
                               lda_ldw, steps_pn, ldc_pm, s.M, s.vt_panel, s.split_stride);
        else
            hipLaunchKernelGGL((gemm_tiled_rows_group_kernel<TM, TN, OUT, ACT>), grid, block, 0, stream, s.d_M, lda_ldw, steps_pn, ldc_pm, s.M, g, s);
    }
    return hipGetLastError();
}

template <int OUT, int ACT>
hipError_t launch_form(const TiledGroup& g, const TiledShape& s, int form, int force, hipStream_t stream)
{
    const int n_cu = device_cu_count();
    switch (form) {
        case TILED_ROWS_1X1: return launch_rows<1, 1, OUT, ACT>(g, s, stream);
        case TILED_ROWS_2X1: return launch_rows<2, 1, OUT, ACT>(g, s, stream);
        case TILED_ROWS_2X2: return launch_rows<2, 2, OUT, ACT>(g, s, stream);
    }
    if constexpr (ACT != ACT_TANH) {
        switch (form) {
            case TILED_K2: return launch_tiles<2, 4, OUT, ACT, false>(g, s, n_cu, force, stream);
            case TILED_PAIR: return launch_tiles<1, 4, OUT, ACT, false>(g, s, n_cu, force, stream);
            case TILED_TALL:
                if constexpr (ACT == ACT_NONE) return launch_tiles<1, 8, OUT, ACT, false>(g, s, n_cu, force, stream);
        }
    }
    return hipErrorInvalidValue;
}

// E4M3 operands: one few-row form, and PAIR
template <int OUT, int ACT>
hipError_t launch_form_fp8(const TiledGroup& g, const TiledShape& s, int form, int force, hipStream_t stream)
{
    if (form == TILED_PAIR) return launch_tiles<1, 4, OUT, ACT, true>(g, s, device_cu_count(), force, stream);
    if (form != TILED_ROWS_1X1) return hipErrorInvalidValue;
    const int panels = (s.M + 31) / 32;
    constexpr int kPanels = kLaunchPanels / 2;                       // of a launch (a grid takes 65535)
    for (int pm0 = 0; pm0 < panels; pm0 += kPanels)
        hipLaunchKernelGGL((gemm_tiled_rows_fp8_kernel<OUT, ACT>), dim3((s.N / 32 + 3) / 4, std::min(panels - pm0, kPanels), s.G), dim3(256), 0, stream, s.d_M,
                           pm0, g, s);
    return hipGetLastError();
}

// The kernel form.  `blocks` counts the 32x32 outputs of the launch by its row bound (the rows present, known on the device, are
// about half of that in a padded batch).  Measured at BERT-base widths, 36 to 18.6 k rows, 1 and 8 problems:
//   up to 1152 blocks (72 x 2 for 36 rows x 2304 columns): one block per workgroup; a launch is a chain of latencies there and
//     more, smaller workgroups shorten it (36 rows: QKV 4.3 us, 2x1 4.4, 2x2 5.9, tiles 7.5);
//   up to 3072: two row panels per workgroup (600 rows x 2304: 8.1 us, 1x1 8.5, K2 9.1).  For up to 1024 columns K2 takes over sooner: from 2048
//     blocks on (8 problems of 288 rows x 768 x 768, 3072 blocks: K2 10.8 us, 2x1 14.3; 1920 blocks 10.3 both; with all rows of the bound
//     present 13.1 and 15.2, 11.0 and 10.9), and where K is long at once for several problems (8 x 192 rows x 768 x 3072: 19.0 us, 24.2;
//     3 x 288 rows 15.9 and 17.1; 8 x 288 rows 21.6 and 41.7) or 64 row panels of one (passes over 13 x 128 tokens, 52 panels, with K2 890 us,
//     without 851; BERT-large 6 x 200, 38 panels, 1930 and 1839);
//   beyond: tiles.  Narrow outputs of fewer tiles than fill the chip twice take K2, which halves a workgroup's serial K loop (2318
//     rows x 768 x 3072: 21.5 us, PAIR 31); long K with many tiles takes TALL (18.6 k rows x 768 x 3072: 75.5 us, PAIR 78), everything
//     else PAIR, whose two workgroups per compute unit hide each other's epilogues (GELU: 84 us, TALL 100).
// The few-row forms add K up in four quarters, K2 in two halves, PAIR and TALL in one run, and a task's result must not depend on which
// others are enabled: which of the three it is goes by the number of problems with all tasks enabled (TiledShape::plan), and only
// the choice among forms of one order by those that are there.
int choose_form(const TiledShape& s)
{
    const int pm = (s.M + 31) / 32, pn = s.N / 32;
    const long sub = s.n_sub > 1 ? s.n_sub : 1, plan = s.plan > s.G ? s.plan : s.G;
    const long blocks = (long)pm * pn * s.G * s.splits * sub, plan_blocks = (long)pm * pn * plan * s.splits * sub;
    const int slices = s.K / 64 / s.splits;
    if (s.f8) {
        // Both forms add K up in one order, so the times alone decide (few-row form, tiles).  One problem: 580 rows x 2304 / 3072 x 768, 2304 and 3072
        // blocks, 7.4, 7.7 us and 7.6, 8.5; 900 rows 9.4, 9.1; x 768 x 3072 1200 rows, 1584 blocks, 11.4, 13.9, 2318 rows, 3072 blocks, 18.0, 14.6.  8
        // problems: 90 rows x 768 x 768, 960 blocks, 6.4, 7.5, x 2304, 2880 blocks, 12.0, 8.2.  (A tile of more than four panels: 44 and 46 us for 18.6 k
        // rows x 768 x 3072.)
        return slices < 5 || blocks <= (s.G > 1 ? 1536 : s.K < 1024 ? 3072 : 2304) ? TILED_ROWS_1X1 : TILED_PAIR;
    }
    // Contexts (parts of 64 columns): one block per workgroup reads its rows twice.  Two by two pays where K is long and there are workgroups enough.  12 heads x
    // 768, 8 problems of 64 / 96 / 128 / 256 rows, 384 to 1536 blocks: 1x1 5.9, 10.7, 13.1, 17.9 us, 2x1 4.6, 9.3, 10.8, 18.6, 2x2 5.1, 6.1, 6.6, 15.5; but 1 of
    // 512 rows, 384 blocks, 4.4, 4.4, 5.1 and 2 of 200, 336, 4.3, 4.8, 5.1.  8 heads x 512, 4 of 256 rows, 512 blocks, 3.8, 3.8, 4.4, 11 of 512, 2816, 18.5,
    // 18.9, 20.4.
    if (s.n_sub > 1 && s.K >= 768 && blocks > 400) return TILED_ROWS_2X2;
    // Poolers: the few-row forms at any size.  PAIR would be faster from 3072 blocks on (21 problems of 272 rows x 768 x 1536 32 us, 2x1 44) but adds K up in
    // one run instead of four quarters: error against float64 2.2e-7 instead of 1.1e-7 there, 2.4e-7 and 1.2e-7 for 24 of 128 rows x 1024 x 2048.
    if (s.n_sub > 1 || s.act == ACT_TANH) return blocks <= 1152 ? TILED_ROWS_1X1 : TILED_ROWS_2X1;
    const bool k2_ok = s.K % (128 * s.splits) == 0 && slices / 2 >= 5, tile_ok = slices >= 5;
    if (!tile_ok) return blocks <= 1152 ? TILED_ROWS_1X1 : TILED_ROWS_2X2;
    const long most_rows = !k2_ok || pn > 32 ? 3072 : s.K < 2048 ? 2047 : plan > 1 || pm >= 64 ? 1152 : 3072;
    if (plan_blocks <= most_rows) return blocks <= 1152 ? TILED_ROWS_1X1 : TILED_ROWS_2X1;
    const long tiles4 = (long)((pm + 3) / 4) * ((pn + 7) / 8) * s.splits;           // 128 x 256, of a problem
    if (k2_ok && tiles4 * plan <= 256) return TILED_K2;
    if (s.K >= 2048 && s.act == ACT_NONE && slices % 2 == 0 && tiles4 * s.G >= 512) return TILED_TALL;
    return TILED_PAIR;
}

}  // namespace

int tiled_splits(int M, int N, int K, int most)
{
    if (K < 2048) return 1;
    const long pm = (M + 31) / 32, blocks = pm * (N / 32);
    int sp = 1;
    while (sp < most && blocks * sp < 192 && K % (128 * sp) == 0) sp *= 2;
    // One round of K2 tiles leaves a serial K loop on compute units that are not all busy: two ranges of K, where the launch takes that form
    // with two, too, and fewer than 7/8 of the compute units had a tile.  Passes without and with: BERT-base widths 20 x 128 tokens 1147 and
    // 1132 us, 32 x 128 1303 and 1294, 36 x 128 1360 and 1351, 9 x 509 1366 and 1353; BERT-large's 11 x 200 2462 and 2355, 15 x 200 2683 and
    // 2615, 16 x 200 level (-1 to +1 %).  Of fewer rows the LayerNorm's second operand costs more than it saves (13 x 128: 861 and 882; 8 x 128:
    // 734 and 748; BERT-large 6 x 200: 1842 and 1858).
    if (sp == 1 && most >= 4 && K % 128 == 0) {
        const long tiles = (pm + 3) / 4 * ((N + 127) / 128);
        TiledShape two{1, M, N, K, K, K, N, ACT_NONE, 1, nullptr, 2, 0};
        if (8 * tiles < 7 * device_cu_count() && choose_form(two) == TILED_K2) sp = 2;
    }
    return sp;
}

hipError_t launch_gemm_tiled(const TiledGroup& g, const TiledShape& s, hipStream_t stream, int form, int force)
{
    if (s.G <= 0 || s.M <= 0 || s.N <= 0) return hipSuccess;
    if (s.G > kMaxGroup || s.splits < 1 || s.N % 32 != 0 || s.K % (64 * s.splits) != 0 || s.lda % 16 != 0 || s.ldw % 16 != 0 || s.ldc % 8 != 0 ||
        s.lda < s.K || s.ldw < s.K || (s.f8 && (s.splits != 1 || s.n_sub > 1)) || (!s.f8 && s.out_f32 == TILED_E4M3) || (s.out_f32 == TILED_E4M3 && s.ldc % 64 != 0) || (s.vt_panel && (s.out_f32 || s.f8 || s.act != ACT_NONE || s.vt_panel % 2 != 0)) || (s.splits > 1 && (s.out_f32 != TILED_F32 || s.act != ACT_NONE)))
        return hipErrorInvalidValue;
    // byte offsets inside the weights, and inside the 8 row panels of a tile, are 31-bit
    if ((uint64_t)s.lda * 64 * 8 >= (1ull << 31) || (uint64_t)s.N / 32 * s.ldw * 64 >= (1ull << 31)) return hipErrorInvalidValue;
    if (form == TILED_AUTO) form = choose_form(s);
    // the tile forms: a tile's loads reach at most into the next tile, so it has at least as many slices as the ring holds ahead
    const int kw = form == TILED_K2 ? 2 : 1, slices = s.K / (64 * kw) / s.splits;
    if (form >= TILED_K2 && (s.n_sub > 1 || s.K % (64 * kw * s.splits) != 0 || slices < 5 || (form == TILED_TALL && slices % 2 != 0)))
        return hipErrorInvalidValue;
    // a given height: one of the form's, and those with two weight buffers take an even number of slices
    if (force && (form < TILED_K2 || force < (form == TILED_TALL ? 5 : 1) || force > (form == TILED_TALL ? 8 : 4) || (force >= 4 && slices % 2 != 0) || (s.f8 && force == 3)))
        return hipErrorInvalidValue;
    if (!s.f8 && form < TILED_K2 && ((long)s.G * s.splits * (s.n_sub > 1 ? s.n_sub : 1) > 65535 || s.lda / 16 > 65535 || s.ldw / 16 > 65535 || s.ldc / 8 > 65535 ||
                            s.N / 32 > 65535))
        return hipErrorInvalidValue;
    if (s.f8) {
        if (s.out_f32 == TILED_F32) return s.act == ACT_NONE ? launch_form_fp8<TILED_F32, ACT_NONE>(g, s, form, force, stream) : hipErrorInvalidValue;
        if (s.out_f32 == TILED_BF16) return s.act == ACT_NONE ? launch_form_fp8<TILED_BF16, ACT_NONE>(g, s, form, force, stream) : hipErrorInvalidValue;
        switch (s.act) {
            case ACT_GELU_ERF: return launch_form_fp8<TILED_E4M3, ACT_GELU_ERF>(g, s, form, force, stream);
            case ACT_GELU_TANH: return launch_form_fp8<TILED_E4M3, ACT_GELU_TANH>(g, s, form, force, stream);
            default: return hipErrorInvalidValue;
        }
    }
    if (s.out_f32) {
        if (s.act == ACT_TANH) return launch_form<TILED_F32, ACT_TANH>(g, s, form, force, stream);
        if (s.act != ACT_NONE) return hipErrorInvalidValue;
        return launch_form<TILED_F32, ACT_NONE>(g, s, form, force, stream);
    }
    switch (s.act) {
        case ACT_NONE: return launch_form<TILED_BF16, ACT_NONE>(g, s, form, force, stream);
        case ACT_GELU_ERF: return launch_form<TILED_BF16, ACT_GELU_ERF>(g, s, form, force, stream);
        case ACT_GELU_TANH: return launch_form<TILED_BF16, ACT_GELU_TANH>(g, s, form, force, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace mt
