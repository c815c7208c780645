// Row kernels of the bfloat16 path, on the panel layout of tiled_offset() (kernels.h).  LayerNorm and embedding: a wavefront takes 4
// rows of a panel, lane = (chunk in 8, row in 4, half of the chunk), so that a load instruction covers 8 neighbouring chunks of 128
// contiguous bytes of float32 (whole lines); the wavefronts of a workgroup complete the 128-byte lines of the bf16 copy.
// A launch of many rows is bound by HBM (or the last-level cache): a row is read and written once, a wavefront has all columns of its
// rows, and no barrier is needed.  A launch of few rows is a chain of latencies, one of some thousand has too few workgroups: there the columns are dealt out to as many wavefronts as
// they have shares, each of which waits for a quarter of the loads (36 rows of 768, one and four partial results: 4.5 and 5.3 us a launch,
// 3.4 and 3.6 so; 18.6 k rows the other way, 38 and 40 us).  Both form mean and variance from those of the shares: the same bits.
#include "kernels.h"
#include "device_util.h"

namespace mt {

namespace {

// Sum of a row's partial values over the 16 lanes that hold it.
__device__ __forceinline__ float row_sum(float v)
{
    v = lane_pair_sum<1>(v);
    v = lane_pair_sum<8>(v);
    v = lane_pair_sum<16>(v);
    v = lane_pair_sum<32>(v);
    return v;
}

// Shares of a row of NI x 64 columns that have moments of their own.
constexpr int row_shares(int NI) { return NI % 4 == 0 ? 4 : (NI % 2 == 0 ? 2 : 1); }
constexpr int kRowWaves = 4;                                                  // of a workgroup
// rows of a workgroup whose wavefronts take one share each (SPLIT) or all of them
template <int NI, bool SPLIT>
constexpr int rows_of_group = kRowWaves / (SPLIT ? row_shares(NI) : 1) * 4;

// Where a row goes: the float32 state, and operand copies (each may be null): bf16, or (split) [hi | lo] bf16 halves of a matrix twice as
// wide, and E4M3 (of the bf16 copy's values, or of the float32 ones: q_exact).
struct RowOut {
    float* f;
    __bf16* b;
    unsigned char* q;
    int split;
    bool q_exact;
};

// How the sums of a row are ordered.  SHARES: above.  WHOLE: one wavefront has the row, and the sums are those of the row-major kernels
// (layernorm_fast: 64 partial sums of every 64th group of 4 columns, added up pairwise) to the bit, which the E4M3 roundings behind them amplify.
enum RowSums : int { ROW_SHARES, ROW_WHOLE };

// sum over the row of part[k], k = 0 .. 3: the partial sums 16 k + 2 c8 + half of 64
__device__ __forceinline__ float row_sum_whole(const float (&part)[4])
{
    float v = (part[0] + part[2]) + (part[1] + part[3]);
    v = lane_pair_sum<32>(v);
    v = lane_pair_sum<16>(v);
    v = lane_pair_sum<8>(v);
    v = lane_pair_sum<1>(v);
    return v;
}

// Mean of a row, and the sum of the squares about it.  SHARES: a share's sum, and its squares about its own mean, are what the wavefronts exchange (once); the
// row's are put together from them in double.  In float, the mean one of four rounded means, 9 k rows of 768 values about 5 came out 2.2e-7 off
// float64 (rms, of results of order 1); 1.6e-7 so, 1.8e-7 with one float sum over the whole row.  Time: passes of 40 to 32 k tokens within 0.4 %.
// Nothing here may be contracted: a share's mean is kept in a register in one form and formed from LDS in the other.
template <int NI, bool SPLIT, RowSums SUMS>
__device__ __forceinline__ void row_moments(const float4 (&v)[NI / (SPLIT ? row_shares(NI) : 1)], int wave, float& mean, float& q)
{
#pragma clang fp contract(off)
    constexpr int H = NI * 64;
    if constexpr (SUMS == ROW_WHOLE) {
        static_assert(!SPLIT && NI % 4 == 0, "");
        float part[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            part[k] = 0.f;
#pragma unroll
            for (int i = k; i < NI; i += 4) part[k] += (v[i].x + v[i].y) + (v[i].z + v[i].w);
        }
        mean = row_sum_whole(part) / (float)H;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            part[k] = 0.f;
#pragma unroll
            for (int i = k; i < NI; i += 4) part[k] += ln_squares(v[i], mean);
        }
        q = row_sum_whole(part);
    } else {
        constexpr int SH = row_shares(NI), W = SPLIT ? SH : 1, NS = NI / SH, N = NS * 64;
        float s[SH], d2[SH];                 // of the shares: sum, squares about its mean
        auto mean_of = [](float sum) {
#pragma clang fp contract(off)
            return SH == 1 ? (float)((double)sum * (1.0 / H)) : sum * (1.0f / N);
        };
#pragma unroll
        for (int h = 0; h < SH / W; ++h) {
            float t = 0.f;
#pragma unroll
            for (int i = h * NS; i < (h + 1) * NS; ++i) t += (v[i].x + v[i].y) + (v[i].z + v[i].w);
            s[h] = row_sum(t);
        }
#pragma unroll
        for (int h = 0; h < SH / W; ++h) {
            const float m = mean_of(s[h]);
            float t = 0.f;
#pragma unroll
            for (int i = h * NS; i < (h + 1) * NS; ++i) t += ln_squares(v[i], m);
            d2[h] = row_sum(t);
        }
        if constexpr (W > 1) {
            __shared__ float2 share[kRowWaves / W][W][4];
            const int lane = threadIdx.x & 63, quad = wave / W, wc = wave % W, r = (lane >> 1) & 3;
            if ((lane & 57) == 0) share[quad][wc][r] = make_float2(s[0], d2[0]);
            __syncthreads();
#pragma unroll
            for (int h = 0; h < SH; ++h) {
                const float2 t = share[quad][h][r];
                s[h] = t.x;
                d2[h] = t.y;
            }
        }
        if constexpr (SH == 1) {
            mean = mean_of(s[0]);
            q = d2[0];
        } else {
            // the squares of a share about the row's mean, from those about its own mean c, d = c - mean: + N d^2 + 2 d (sum - N c).  The last term is there because
            // c is rounded: without it rows of 896 values, 4e6 of their deviations from zero, came out twice as far off as with one sum (1.03 times with it).
            double sum = s[0], squares = d2[0], u = 0.0;
#pragma unroll
            for (int h = 1; h < SH; ++h) {
                sum += s[h];
                squares += d2[h];
            }
            mean = (float)(sum * (1.0 / H));
#pragma unroll
            for (int h = 0; h < SH; ++h) {
                const double c = mean_of(s[h]), d = c - mean;
                u = fma(d, fma((double)N, d, 2.0 * fma(-(double)N, c, (double)s[h])), u);
            }
            q = (float)(squares + u);
        }
    }
}

// Normalise the NW x 4 values that a lane holds of its row, columns (wc NW + i) 64 .., and store.  STREAM: the float32 state is stored past the second-level
// cache, since it is read again three launches later only (18.6 k rows 38.7 -> 38.2 us, 8 problems of them 278 -> 268).
template <int NI, bool SPLIT, bool STREAM, RowSums SUMS>
__device__ __forceinline__ void finish_row(float4 (&v)[NI / (SPLIT ? row_shares(NI) : 1)], const float* __restrict__ gamma, const float* __restrict__ beta,
                                           int row, int wave, bool live, float eps, const RowOut& out)
{
    constexpr int H = NI * 64, W = SPLIT ? row_shares(NI) : 1, NW = NI / W;
    const int lane = threadIdx.x & 63, half = lane & 1, c8 = lane >> 3, wc = wave % W;
    float4 g[NW], b[NW];                     // in flight during the reductions
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        g[i] = *reinterpret_cast<const float4*>(gamma + ((wc * NW + i) * 8 + c8) * 8 + half * 4);
        b[i] = *reinterpret_cast<const float4*>(beta + ((wc * NW + i) * 8 + c8) * 8 + half * 4);
    }
    __builtin_amdgcn_sched_barrier(0);
    float mean, q;
    row_moments<NI, SPLIT, SUMS>(v, wave, mean, q);
    const float inv = 1.0f / sqrtf(q / (float)H + eps);
    if (!live) return;
    const size_t panel = (size_t)(row >> 5) * 32;
    const int in_chunk = (row & 31) * 8 + half * 4;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int chunk = (wc * NW + i) * 8 + c8;
        const float4 n = ln_normalise(v[i], mean, inv, g[i], b[i]);
        const f32x4 o = {n.x, n.y, n.z, n.w};
        f32x4* f = reinterpret_cast<f32x4*>(out.f + panel * H + chunk * 256 + in_chunk);
        if constexpr (STREAM) __builtin_nontemporal_store(o, f);
        else *f = o;
        const bf16x4 hi = {(__bf16)o[0], (__bf16)o[1], (__bf16)o[2], (__bf16)o[3]};
        if (out.q)
            *reinterpret_cast<uint32_t*>(out.q + tiled_offset_e4m3(row, chunk * 8 + half * 4, H)) =
                out.q_exact ? pack_e4m3(o[0], o[1], o[2], o[3]) : pack_e4m3((float)hi[0], (float)hi[1], (float)hi[2], (float)hi[3]);
        if (!out.b) continue;
        __bf16* p = out.b + panel * (out.split ? 2 * H : H) + in_chunk;
        *reinterpret_cast<bf16x4*>(p + chunk * 256) = hi;
        if (out.split) {
            const bf16x4 lo = {(__bf16)(o[0] - (float)hi[0]), (__bf16)(o[1] - (float)hi[1]), (__bf16)(o[2] - (float)hi[2]), (__bf16)(o[3] - (float)hi[3])};
            *reinterpret_cast<bf16x4*>(p + (NI * 8 + chunk) * 256) = lo;
        }
    }
}

// out = LayerNorm(sum of NP partial products + residual) (the bias is already in the first product).  All loads of a lane are issued
// before the first use, in a launch of few rows (EARLY) even before the row count has arrived: rows beyond it are memory of the
// operands all the same, but of a large padded batch reading them would be real traffic.  The pointers are leading scalar arguments,
// which the command processor preloads.
template <int NI, int NP, bool SPLIT, bool EARLY, RowSums SUMS>
__device__ __forceinline__ void layernorm_tiled_body(const float* x, const float* res, const float* gamma, const float* beta, const RowOut& out,
                                                     const int32_t* d_M, int M, int64_t part_stride, const int32_t* res_row, int res_rows, float eps)
{
    constexpr int H = NI * 64, W = SPLIT ? row_shares(NI) : 1, NW = NI / W;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rows_here = *(d_M ? d_M : reinterpret_cast<const int32_t*>(x));
    const int last = (M + 31) / 32 * 32 - 1;                                  // rows of the last panel exist
    if (!EARLY && d_M) M = min(M, rows_here);
    const int row0 = blockIdx.x * rows_of_group<NI, SPLIT>, row = row0 + wave / W * 4 + ((lane >> 1) & 3);
    const int at = (lane & 1) * 4 + (wave % W * NW * 8 + (lane >> 3)) * 256;
    if (!EARLY && row0 >= M) return;                                            // (the whole workgroup, here and below)
    x += (size_t)(min(row, last) >> 5) * 32 * H + (row & 31) * 8 + at;
    // the residual row is the same row, or (first-token layers) the row that a sequence starts at
    const int rr = res_row ? (int)min((uint32_t)res_row[min(row, M - 1)], (uint32_t)(res_rows - 1)) : min(row, last);
    res += (size_t)(rr >> 5) * 32 * H + (rr & 31) * 8 + at;
    constexpr int FIRST = (NP + 1) * NW <= 60 ? NP : 2;                       // what fits the registers
    float4 v[FIRST][NW], r[NW];
#pragma unroll
    for (int p = 0; p < FIRST; ++p)
#pragma unroll
        for (int i = 0; i < NW; ++i) v[p][i] = *reinterpret_cast<const float4*>(x + (size_t)p * part_stride + i * 2048);
#pragma unroll
    for (int i = 0; i < NW; ++i) r[i] = *reinterpret_cast<const float4*>(res + i * 2048);
    if constexpr (EARLY) {
        asm volatile("" ::: "memory");                                        // the loads stay in front of the exit
        if (d_M) M = min(M, rows_here);
        if (row0 >= M) return;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NW; ++i) {                                            // fixed order: deterministic
#pragma unroll
        for (int p = 1; p < NP; ++p) {
            const float4 u = p < FIRST ? v[p < FIRST ? p : 0][i] : *reinterpret_cast<const float4*>(x + (size_t)p * part_stride + i * 2048);
            v[0][i].x += u.x;
            v[0][i].y += u.y;
            v[0][i].z += u.z;
            v[0][i].w += u.w;
        }
        v[0][i].x += r[i].x;
        v[0][i].y += r[i].y;
        v[0][i].z += r[i].z;
        v[0][i].w += r[i].w;
    }
    finish_row<NI, SPLIT, !SPLIT, SUMS>(v[0], gamma, beta, row, wave, row < M, eps, out);
}

template <int NI, int NP, class Ahead>
__global__ __launch_bounds__(kRowWaves * 64) void layernorm_tiled_kernel(const float* x, const float* res, const int32_t* d_M, const float* gamma,
                                                              const float* beta, float* of, __bf16* ob, int M, int64_t part_stride, float eps, int groups, Ahead ahead)
{
    if constexpr (Ahead::kAny) {
        if ((int)blockIdx.x >= groups) {
            read_ahead(ahead, blockIdx.x - groups);
            return;
        }
    }
    layernorm_tiled_body<NI, NP, true, true, ROW_SHARES>(x, res, gamma, beta, RowOut{of, ob, nullptr, 0, false}, d_M, M, part_stride, nullptr, 0, eps);
}

template <int NI, int NP, bool SPLIT, bool EARLY, RowSums SUMS>
__global__ __launch_bounds__(kRowWaves * 64) void layernorm_tiled_group_kernel(TiledLnGroup g, TiledLnShape s)
{
    const int grp = blockIdx.y;
    const unsigned char* wt = static_cast<const unsigned char*>(g.wt);
    unsigned char* ws = static_cast<unsigned char*>(const_cast<void*>(g.ws));
    unsigned char* ob = ws + (size_t)g.out_b[grp] * 256;
    const RowOut out{reinterpret_cast<float*>(ws + (size_t)g.out_f[grp] * 256), s.want_b >> grp & 1 ? reinterpret_cast<__bf16*>(ob) : nullptr,
                     s.want_q >> grp & 1 ? ob + s.q_offset : nullptr, s.split, s.q_offset == 0};
    layernorm_tiled_body<NI, NP, SPLIT, EARLY, SUMS>(reinterpret_cast<const float*>(ws + (size_t)g.x[grp] * 256), reinterpret_cast<const float*>(ws + (size_t)g.res[grp] * 256),
                                      reinterpret_cast<const float*>(wt + (size_t)g.gamma[grp] * 256), reinterpret_cast<const float*>(wt + (size_t)g.beta[grp] * 256),
                                      out, s.d_M, s.M, s.part_stride, s.res_row, s.res_rows, s.eps);
}

// Embedding sum + LayerNorm of the kept rows.
template <int NI, bool SPLIT, RowSums SUMS>
__global__ __launch_bounds__(kRowWaves * 64) void embed_ln_tiled_kernel(const int32_t* __restrict__ ids, const int32_t* __restrict__ type_ids, int type_vocab,
                                                             const int32_t* __restrict__ src, const int32_t* __restrict__ d_M, int M, int S,
                                                             int vocab, const __bf16* __restrict__ word, const __bf16* __restrict__ pos,
                                                             const __bf16* __restrict__ type, const float* __restrict__ gamma,
                                                             const float* __restrict__ beta, float eps, float* of, __bf16* ob, unsigned char* oq)
{
    constexpr int H = NI * 64, W = SPLIT ? row_shares(NI) : 1, NW = NI / W;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row0 = blockIdx.x * rows_of_group<NI, SPLIT>, row = row0 + wave / W * 4 + ((lane >> 1) & 3);
    M = min(M, *d_M);
    if (row0 >= M) return;                                                    // (the whole workgroup)
    const int p = src[min(row, M - 1)];
    int id = ids[p];
    id = id < 0 ? 0 : (id >= vocab ? vocab - 1 : id);
    int seg = type_ids ? type_ids[p] : 0;
    seg = seg < 0 ? 0 : (seg >= type_vocab ? type_vocab - 1 : seg);
    const int col = (wave % W * NW * 8 + (lane >> 3)) * 8 + (lane & 1) * 4;
    const __bf16* w = word + (size_t)id * H + col;
    const __bf16* q = pos + (size_t)(p % S) * H + col;
    const __bf16* t = type + (size_t)seg * H + col;
    bf16x4 a[NW], b[NW], c[NW];
    float4 v[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        a[i] = *reinterpret_cast<const bf16x4*>(w + i * 64);
        b[i] = *reinterpret_cast<const bf16x4*>(q + i * 64);
        c[i] = *reinterpret_cast<const bf16x4*>(t + i * 64);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        v[i].x = ((float)a[i][0] + (float)b[i][0]) + (float)c[i][0];
        v[i].y = ((float)a[i][1] + (float)b[i][1]) + (float)c[i][1];
        v[i].z = ((float)a[i][2] + (float)b[i][2]) + (float)c[i][2];
        v[i].w = ((float)a[i][3] + (float)b[i][3]) + (float)c[i][3];
    }
    finish_row<NI, SPLIT, false, SUMS>(v, gamma, beta, row, wave, row < M, eps, RowOut{of, ob, oq, 0, false});
}

// Pooler operand of tasks without own layers: the tap's first-token row of every sequence as [hi | lo] bf16 halves.
__global__ __launch_bounds__(128) void split_first_rows_tiled_kernel(SplitGroup g, int H, const int32_t* __restrict__ seq_start, int max_rows)
{
    const int grp = blockIdx.y, b = blockIdx.x, row = min(seq_start[b], max_rows - 1);
    __bf16* out = reinterpret_cast<__bf16*>(g.out[grp]);
    for (int chunk = threadIdx.x; chunk < H / 8; chunk += 128) {
        const float* x = g.x[grp] + tiled_offset(row, chunk * 8, H);
        bf16x8 hi, lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            hi[e] = (__bf16)x[e];
            lo[e] = (__bf16)(x[e] - (float)hi[e]);
        }
        *reinterpret_cast<bf16x8*>(out + tiled_offset(b, chunk * 8, 2 * H)) = hi;
        *reinterpret_cast<bf16x8*>(out + tiled_offset(b, H + chunk * 8, 2 * H)) = lo;
    }
}

// Rows of a matrix copied to rows of another: dst row i = src row index[i], i < *n (or n_max), float32 and / or bf16 copies.
__global__ __launch_bounds__(256) void copy_rows_tiled_kernel(RowCopyGroup g, const int32_t* __restrict__ index, const int32_t* __restrict__ n,
                                                              int n_max, int max_rows, int H)
{
    // lane = row in 8 x chunk in 8: 8 rows of a chunk are contiguous on the writing side
    const int grp = blockIdx.y, r = blockIdx.x * 8 + (threadIdx.x & 7);
    if (n) n_max = min(n_max, *n);
    if (r >= n_max) return;
    const int from = min(index[r], max_rows - 1);
    for (int chunk = threadIdx.x >> 3; chunk < H / 8; chunk += 32) {
        const size_t a = tiled_offset(from, chunk * 8, H), b = tiled_offset(r, chunk * 8, H);
        if (g.in_f[grp]) {
            const float4 lo = *reinterpret_cast<const float4*>(g.in_f[grp] + a), hi = *reinterpret_cast<const float4*>(g.in_f[grp] + a + 4);
            *reinterpret_cast<float4*>(g.out_f[grp] + b) = lo;
            *reinterpret_cast<float4*>(g.out_f[grp] + b + 4) = hi;
        }
        if (g.in_q[grp])
            *reinterpret_cast<uint2*>(static_cast<unsigned char*>(g.out_q[grp]) + tiled_offset_e4m3(r, chunk * 8, H)) =
                *reinterpret_cast<const uint2*>(static_cast<const unsigned char*>(g.in_q[grp]) + tiled_offset_e4m3(from, chunk * 8, H));
        if (g.in_b[grp])
            *reinterpret_cast<uint4*>(reinterpret_cast<__bf16*>(g.out_b[grp]) + b) = *reinterpret_cast<const uint4*>(reinterpret_cast<const __bf16*>(g.in_b[grp]) + a);
    }
}

// logits[b][c] = Wc[c] . pooled[b] + bc[c]: one wavefront per class, pooled float32 in the panel layout, a chunk per lane.
__global__ __launch_bounds__(256) void classifier_tiled_kernel(ClsGroup g, int H, int64_t ldo, const int32_t* __restrict__ out_row)
{
    const int grp = blockIdx.y, b = blockIdx.x, lane = threadIdx.x & 63;
    const int c = blockIdx.z * 4 + (threadIdx.x >> 6);
    if (c >= g.C[grp]) return;
    const float* p = g.pooled[grp] + (size_t)(b >> 5) * 32 * H + (b & 31) * 8;
    const __bf16* w = static_cast<const __bf16*>(g.Wc[grp]) + (size_t)c * H;
    const float bias = g.bc[grp][c];
    const int ob = out_row ? out_row[b] : b;
    float acc = 0.f;
    for (int chunk = lane; chunk < H / 8; chunk += 64) {
        const float4 x0 = *reinterpret_cast<const float4*>(p + chunk * 256), x1 = *reinterpret_cast<const float4*>(p + chunk * 256 + 4);
        const bf16x8 wv = *reinterpret_cast<const bf16x8*>(w + chunk * 8);
        acc = fmaf(x0.x, (float)wv[0], acc);
        acc = fmaf(x0.y, (float)wv[1], acc);
        acc = fmaf(x0.z, (float)wv[2], acc);
        acc = fmaf(x0.w, (float)wv[3], acc);
        acc = fmaf(x1.x, (float)wv[4], acc);
        acc = fmaf(x1.y, (float)wv[5], acc);
        acc = fmaf(x1.z, (float)wv[6], acc);
        acc = fmaf(x1.w, (float)wv[7], acc);
    }
    acc = wave_sum(acc);
    if (lane == 0) g.out[grp][(size_t)ob * ldo + c] = acc + bias;
}

// The same (to the bit) for many sequences and tasks of unequal numbers of classes: a wavefront per kClsCols classes (of the list of all tasks' groups of
// so many) and kClsRows sequences, whose rows it reads once.
constexpr int kClsRows = 4, kClsCols = 4, kClsChunks = 2;                     // widths of up to 64 kClsChunks chunks
struct ClsFirst {
    int32_t at[kMaxGroup];                                                    // first group of classes of a task
};
__global__ __launch_bounds__(256) void classifier_list_kernel(ClsGroup g, ClsFirst first, int G, int total, int B, int H, int64_t ldo,
                                                               const int32_t* __restrict__ out_row)
{
    const int lane = threadIdx.x & 63, k = blockIdx.y * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), b0 = blockIdx.x * kClsRows;
    if (k >= total) return;
    const int grp = __popcll(__ballot(lane < G && first.at[min(lane, kMaxGroup - 1)] <= k)) - 1, c0 = (k - first.at[grp]) * kClsCols, C = g.C[grp];
    bf16x8 wv[kClsCols][kClsChunks];
    float4 x0[kClsRows][kClsChunks], x1[kClsRows][kClsChunks];
    float bias[kClsCols];
#pragma unroll
    for (int u = 0; u < kClsCols; ++u) {
        const __bf16* w = static_cast<const __bf16*>(g.Wc[grp]) + (size_t)min(c0 + u, C - 1) * H;
#pragma unroll
        for (int i = 0; i < kClsChunks; ++i) wv[u][i] = *reinterpret_cast<const bf16x8*>(w + min(lane + i * 64, H / 8 - 1) * 8);
        bias[u] = g.bc[grp][min(c0 + u, C - 1)];
    }
#pragma unroll
    for (int r = 0; r < kClsRows; ++r) {
        const int b = min(b0 + r, B - 1);
        const float* p = g.pooled[grp] + (size_t)(b >> 5) * 32 * H + (b & 31) * 8;
#pragma unroll
        for (int i = 0; i < kClsChunks; ++i) {
            const float* q = p + min(lane + i * 64, H / 8 - 1) * 256;
            x0[r][i] = *reinterpret_cast<const float4*>(q);
            x1[r][i] = *reinterpret_cast<const float4*>(q + 4);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < kClsRows; ++r) {
        float acc[kClsCols];
#pragma unroll
        for (int u = 0; u < kClsCols; ++u) {
            float a = 0.f;
#pragma unroll
            for (int i = 0; i < kClsChunks; ++i)
                if (lane + i * 64 < H / 8) {
                    a = fmaf(x0[r][i].x, (float)wv[u][i][0], a);
                    a = fmaf(x0[r][i].y, (float)wv[u][i][1], a);
                    a = fmaf(x0[r][i].z, (float)wv[u][i][2], a);
                    a = fmaf(x0[r][i].w, (float)wv[u][i][3], a);
                    a = fmaf(x1[r][i].x, (float)wv[u][i][4], a);
                    a = fmaf(x1[r][i].y, (float)wv[u][i][5], a);
                    a = fmaf(x1[r][i].z, (float)wv[u][i][6], a);
                    a = fmaf(x1[r][i].w, (float)wv[u][i][7], a);
                }
            acc[u] = wave_sum(a);
        }
        if (b0 + r < B) {
            float* out = g.out[grp] + (size_t)(out_row ? out_row[b0 + r] : b0 + r) * ldo + c0;
#pragma unroll
            for (int u = 0; u < kClsCols; ++u)
                if (lane == u && c0 + u < C) out[u] = acc[u] + bias[u];
        }
    }
}

}  // namespace

namespace {

template <int NI, int NP>
void ln_launch(const TiledLnGroup& g, const TiledLnShape& s, hipStream_t stream, AheadQueue* queue)
{
    unsigned char* ws = static_cast<unsigned char*>(const_cast<void*>(g.ws));
    const unsigned char* wt = static_cast<const unsigned char*>(g.wt);
    // with a row count on the device: less than a cached megabyte or two of padding.  Without, there is none.
    const bool few = !s.whole_sums && (long)s.G * s.M <= (s.d_M ? 2048 : 8192);
    // 2.3 k rows are 144 workgroups of 16 rows, too few for 256 compute units: with the columns dealt out, but the row count read first, passes of 32 x
    // 128 tokens 1294 -> 1267 us, 7 x 509 1394 -> 1379, routed 32 x 128 1597 -> 1552; a line at 8192 or 32768 rows was slower (1269, 1277; 8 x 32 x 128
    // 5934 us, 5950, 6022).
    const bool split = few || (!s.whole_sums && (long)s.G * s.M <= 16384);
    const int rows = split ? rows_of_group<NI, true> : rows_of_group<NI, false>;
    const dim3 grid((s.M + rows - 1) / rows, s.G), block(kRowWaves * 64);
    if constexpr (NI % 4 == 0 && NP == 1) {
        if (s.whole_sums) {
            hipLaunchKernelGGL((layernorm_tiled_group_kernel<NI, NP, false, false, ROW_WHOLE>), grid, block, 0, stream, g, s);
            return;
        }
    }
    if (s.G == 1 && !s.res_row && !s.split && few && (s.want_b & 1) && !(s.want_q & 1)) {
        const ReadAhead ahead = queue ? queue->take() : ReadAhead{};
        auto launch = [&](auto kfn, auto a) {
            hipLaunchKernelGGL(kfn, dim3(grid.x + ahead.blocks()), block, 0, stream, (const float*)(ws + (size_t)g.x[0] * 256),
                               (const float*)(ws + (size_t)g.res[0] * 256), s.d_M, (const float*)(wt + (size_t)g.gamma[0] * 256),
                               (const float*)(wt + (size_t)g.beta[0] * 256), (float*)(ws + (size_t)g.out_f[0] * 256), (__bf16*)(ws + (size_t)g.out_b[0] * 256),
                               s.M, s.part_stride, s.eps, (int)grid.x, a);
        };
        if (ahead.blocks()) launch(layernorm_tiled_kernel<NI, NP, ReadAhead>, ahead);
        else launch(layernorm_tiled_kernel<NI, NP, NoAhead>, NoAhead{});
    } else if (few)
        hipLaunchKernelGGL((layernorm_tiled_group_kernel<NI, NP, true, true, ROW_SHARES>), grid, block, 0, stream, g, s);
    else if (split)
        hipLaunchKernelGGL((layernorm_tiled_group_kernel<NI, NP, true, false, ROW_SHARES>), grid, block, 0, stream, g, s);
    else
        hipLaunchKernelGGL((layernorm_tiled_group_kernel<NI, NP, false, false, ROW_SHARES>), grid, block, 0, stream, g, s);
}

}  // namespace

#define MT_FOR_WIDTH(X) \
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)

hipError_t launch_layernorm_tiled(const TiledLnGroup& g, const TiledLnShape& s, hipStream_t stream, AheadQueue* ahead)
{
    if (s.G <= 0 || s.M <= 0) return hipSuccess;
    if (s.G > kMaxGroup || s.H % 64 != 0 || s.n_parts < 1 || (s.whole_sums && (s.H % 256 != 0 || s.n_parts != 1))) return hipErrorInvalidValue;
    switch (s.H / 64) {
#define X(NI)                                                    \
    case NI:                                                     \
        switch (s.n_parts) {                                     \
            case 1: ln_launch<NI, 1>(g, s, stream, ahead); break; \
            case 2: ln_launch<NI, 2>(g, s, stream, ahead); break; \
            case 4: ln_launch<NI, 4>(g, s, stream, ahead); break; \
            default: return hipErrorInvalidValue;                \
        }                                                        \
        break;
        MT_FOR_WIDTH(X)
#undef X
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_embed_ln_tiled(const int32_t* ids, const int32_t* type_ids, int type_vocab, const int32_t* src, const int32_t* d_M, int B, int S,
                                 int H, int vocab, const void* word, const void* pos, const void* type, const float* gamma, const float* beta,
                                 float eps, float* out_f32, void* out_bf16, void* out_e4m3, hipStream_t stream)
{
    const int M = B * S;
    if (M <= 0) return hipSuccess;
    if (H % 64 != 0 || !src || !d_M) return hipErrorInvalidValue;
    const bool whole = out_e4m3 != nullptr;  // (a model whose operands are E4M3)
    const bool split = !whole && M <= 4096;  // 4096 x 768, 56 % of them kept: 7.6 -> 6.5 us; 8704: level; 32768: 33 us, 38 with the rows split
    if (whole && H % 256 != 0) return hipErrorInvalidValue;
    switch (H / 64) {
#define X(NI)                                                                                                                                \
    case NI: {                                                                                                                               \
        constexpr RowSums kWhole = NI % 4 == 0 ? ROW_WHOLE : ROW_SHARES;                                                                     \
        auto kfn = whole ? embed_ln_tiled_kernel<NI, false, kWhole>                                                                          \
                         : split ? embed_ln_tiled_kernel<NI, true, ROW_SHARES> : embed_ln_tiled_kernel<NI, false, ROW_SHARES>;               \
        const int rows = split ? rows_of_group<NI, true> : rows_of_group<NI, false>;                                                         \
        hipLaunchKernelGGL(kfn, dim3((M + rows - 1) / rows), dim3(kRowWaves * 64), 0, stream, ids, type_ids, type_vocab, src, d_M, M, S,     \
                           vocab, (const __bf16*)word, (const __bf16*)pos, (const __bf16*)type, gamma, beta, eps, out_f32,                   \
                           (__bf16*)out_bf16, (unsigned char*)out_e4m3);                                                                     \
    } break;
        MT_FOR_WIDTH(X)
#undef X
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_split_first_rows_tiled(const SplitGroup& g, int G, int B, int H, const int32_t* seq_start, int max_rows, hipStream_t stream)
{
    if (G <= 0 || B <= 0) return hipSuccess;
    if (!seq_start || G > kMaxGroup || H % 8 != 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(split_first_rows_tiled_kernel, dim3(B, G), dim3(128), 0, stream, g, H, seq_start, max_rows);
    return hipGetLastError();
}

hipError_t launch_copy_rows_tiled(const RowCopyGroup& g, int G, const int32_t* index, const int32_t* n, int n_max, int max_rows, int H, hipStream_t stream)
{
    if (G <= 0 || n_max <= 0) return hipSuccess;
    if (!index || G > kMaxGroup || H % 8 != 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(copy_rows_tiled_kernel, dim3((n_max + 7) / 8, G), dim3(256), 0, stream, g, index, n, n_max, max_rows, H);
    return hipGetLastError();
}

hipError_t launch_classifier_tiled(const ClsGroup& g, int G, int B, int H, int maxC, int64_t ldo, const int32_t* out_row, hipStream_t stream)
{
    if (G <= 0 || B <= 0 || maxC <= 0) return hipSuccess;
    if (G > kMaxGroup || H % 8 != 0) return hipErrorInvalidValue;
    // Workgroups of the plain grid, of which those beyond a task's classes do nothing: 21 tasks of 2 to 50 classes, 16 sequences 4368 of them, 4.4 us
    // (the list 5.0); 272 sequences 74 thousand, 38 us (20).
    // (a grid has room for 4 x 65535 groups of classes in the list.)
    const dim3 plain(B, G, (maxC + 3) / 4);
    ClsFirst first;
    long total = 0;
    for (int i = 0; i < kMaxGroup; ++i) {
        first.at[i] = i < G ? (int32_t)total : 0;
        if (i < G) total += (g.C[i] + kClsCols - 1) / kClsCols;
    }
    if ((long)plain.x * plain.y * plain.z <= 8192 || H > 512 * kClsChunks || total > 4 * 65535) {
        hipLaunchKernelGGL(classifier_tiled_kernel, plain, dim3(256), 0, stream, g, H, ldo, out_row);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(classifier_list_kernel, dim3((B + kClsRows - 1) / kClsRows, (unsigned)((total + 3) / 4)), dim3(256), 0, stream, g, first, G, (int)total, B,
                       H, ldo, out_row);
    return hipGetLastError();
}

}  // namespace mt
