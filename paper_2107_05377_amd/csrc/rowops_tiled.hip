// Row kernels of the bfloat16 path, on the panel layout of tiled_offset() (kernels.h).  A workgroup of 8 wavefronts owns 8 rows of
// one panel: of a chunk (8 columns) they are 256 contiguous bytes of float32 or 128 of bf16, i.e. whole lines that no other
// workgroup writes.  A wavefront's load instruction covers 4 neighbouring chunks: lane = (chunk in 4, row in 8, half of the
// chunk); a row is spread over 8 lanes of every wavefront, so its sums are three lane exchanges and one through LDS.
// Both kernels are bound by HBM (or the last-level cache): a row is read and written once.
#include "kernels.h"
#include "device_util.h"

namespace mt {

namespace {

constexpr int kRowsPerGroup = 8;

// Sum over a row of this lane's partial value, for the lane's row; `red` is one [8 wavefronts][8 rows] exchange.
__device__ __forceinline__ float row_sum(float v, float (*red)[8], int wave, int lane, int r)
{
    v += __shfl_xor(v, 1, 64);
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    if ((lane & 49) == 0) red[wave][r] = v;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) t += red[w][r];
    return t;
}

// Normalise the NV x 4 values that a lane holds of its row and store: float32 state, bf16 operand copy, or (split) the row as
// [hi | lo] bf16 halves of a matrix twice as wide.  Lanes beyond the row's chunks hold zeros and store nothing.
template <int NV>
__device__ __forceinline__ void finish_row(float4 (&v)[NV], const float4 (&g)[NV], const float4 (&b)[NV], int chunk0, int n_chunks, int row,
                                           int half, int wave, int lane, bool live, int H, float eps, float* of, __bf16* ob, int split)
{
    __shared__ float red[2][8][8];
    const int r = row & 7;
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
    const float mean = row_sum(s, red[0], wave, lane, r) / (float)H;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i)
        if (chunk0 + i * 32 < n_chunks) {
            const float a = v[i].x - mean, c = v[i].y - mean, d = v[i].z - mean, e = v[i].w - mean;
            q += (a * a + c * c) + (d * d + e * e);
        }
    const float inv = 1.0f / sqrtf(row_sum(q, red[1], wave, lane, r) / (float)H + eps);
    if (!live) return;
    const size_t panel = (size_t)(row >> 5) * 32;
    const int in_chunk = (row & 31) * 8 + half * 4;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int chunk = chunk0 + i * 32;
        if (chunk >= n_chunks) continue;
        float4 o;
        o.x = g[i].x * ((v[i].x - mean) * inv) + b[i].x;
        o.y = g[i].y * ((v[i].y - mean) * inv) + b[i].y;
        o.z = g[i].z * ((v[i].z - mean) * inv) + b[i].z;
        o.w = g[i].w * ((v[i].w - mean) * inv) + b[i].w;
        if (of) *reinterpret_cast<float4*>(of + panel * H + chunk * 256 + in_chunk) = o;
        if (!ob) continue;
        const bf16x4 hi = {(__bf16)o.x, (__bf16)o.y, (__bf16)o.z, (__bf16)o.w};
        __bf16* p = ob + panel * (split ? 2 * H : H) + in_chunk;
        *reinterpret_cast<bf16x4*>(p + chunk * 256) = hi;
        if (split) {
            const bf16x4 lo = {(__bf16)(o.x - (float)hi[0]), (__bf16)(o.y - (float)hi[1]), (__bf16)(o.z - (float)hi[2]), (__bf16)(o.w - (float)hi[3])};
            *reinterpret_cast<bf16x4*>(p + (n_chunks + chunk) * 256) = lo;
        }
    }
}

// out = LayerNorm(sum of the partial products + bias + residual).  All loads of a lane are issued before the first use.
template <int NV>
__global__ __launch_bounds__(512) void layernorm_tiled_kernel(TiledLnGroup g, TiledLnShape s)
{
    const int grp = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = blockIdx.x * kRowsPerGroup + ((lane >> 1) & 7), half = lane & 1;
    const int M = s.d_M ? min(s.M, *s.d_M) : s.M;
    if (blockIdx.x * kRowsPerGroup >= M) return;
    const int H = s.H, n_chunks = H >> 3, chunk0 = wave * 4 + (lane >> 4);
    const size_t at = (size_t)(row >> 5) * 32 * H + (row & 31) * 8 + half * 4;
    const float* x = reinterpret_cast<const float*>(static_cast<const unsigned char*>(g.ws) + (size_t)g.x[grp] * 256) + at;
    // the residual row is the same row, or (first-token layers) the row that a sequence starts at
    const int rr = s.res_row ? min(s.res_row[min(row, M - 1)], s.res_rows - 1) : row;
    const float* res = reinterpret_cast<const float*>(static_cast<const unsigned char*>(g.ws) + (size_t)g.res[grp] * 256) +
                       (size_t)(rr >> 5) * 32 * H + (rr & 31) * 8 + half * 4;
    const unsigned char* wt = static_cast<const unsigned char*>(g.wt);
    const float* bias = reinterpret_cast<const float*>(wt + (size_t)g.bias[grp] * 256) + half * 4;
    const float* gamma = reinterpret_cast<const float*>(wt + (size_t)g.gamma[grp] * 256) + half * 4;
    const float* beta = reinterpret_cast<const float*>(wt + (size_t)g.beta[grp] * 256) + half * 4;
    float4 v[NV], rv[NV], bv[NV], gm[NV], bt[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int chunk = min(chunk0 + i * 32, n_chunks - 1);                 // lanes beyond the row load its last chunk
        v[i] = *reinterpret_cast<const float4*>(x + chunk * 256);
        rv[i] = *reinterpret_cast<const float4*>(res + chunk * 256);
        bv[i] = *reinterpret_cast<const float4*>(bias + chunk * 8);
        gm[i] = *reinterpret_cast<const float4*>(gamma + chunk * 8);
        bt[i] = *reinterpret_cast<const float4*>(beta + chunk * 8);
    }
    __builtin_amdgcn_sched_barrier(0);
    for (int p = 1; p < s.n_parts; ++p) {                                     // fixed order: deterministic
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const float4 t = *reinterpret_cast<const float4*>(x + (size_t)p * s.part_stride + min(chunk0 + i * 32, n_chunks - 1) * 256);
            v[i].x += t.x; v[i].y += t.y; v[i].z += t.z; v[i].w += t.w;
        }
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const bool in = chunk0 + i * 32 < n_chunks;
        v[i].x = in ? (v[i].x + bv[i].x) + rv[i].x : 0.f;
        v[i].y = in ? (v[i].y + bv[i].y) + rv[i].y : 0.f;
        v[i].z = in ? (v[i].z + bv[i].z) + rv[i].z : 0.f;
        v[i].w = in ? (v[i].w + bv[i].w) + rv[i].w : 0.f;
    }
    unsigned char* ws = static_cast<unsigned char*>(const_cast<void*>(g.ws));
    finish_row<NV>(v, gm, bt, chunk0, n_chunks, row, half, wave, lane, row < M, H, s.eps,
                   g.out_f[grp] == kNoBias ? nullptr : reinterpret_cast<float*>(ws + (size_t)g.out_f[grp] * 256),
                   g.out_b[grp] == kNoBias ? nullptr : reinterpret_cast<__bf16*>(ws + (size_t)g.out_b[grp] * 256), s.split);
}

// Embedding sum + LayerNorm of the kept rows.
template <int NV>
__global__ __launch_bounds__(512) void embed_ln_tiled_kernel(const int32_t* __restrict__ ids, const int32_t* __restrict__ type_ids, int type_vocab,
                                                             const int32_t* __restrict__ src, const int32_t* __restrict__ d_M, int M, int S, int H,
                                                             int vocab, const __bf16* __restrict__ word, const __bf16* __restrict__ pos,
                                                             const __bf16* __restrict__ type, const float* __restrict__ gamma,
                                                             const float* __restrict__ beta, float eps, float* of, __bf16* ob)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = blockIdx.x * kRowsPerGroup + ((lane >> 1) & 7), half = lane & 1;
    M = min(M, *d_M);
    if (blockIdx.x * kRowsPerGroup >= M) return;
    const int n_chunks = H >> 3, chunk0 = wave * 4 + (lane >> 4);
    const int p = src[min(row, M - 1)];
    int id = ids[p];
    id = id < 0 ? 0 : (id >= vocab ? vocab - 1 : id);
    int seg = type_ids ? type_ids[p] : 0;
    seg = seg < 0 ? 0 : (seg >= type_vocab ? type_vocab - 1 : seg);
    const __bf16* w = word + (size_t)id * H + half * 4;
    const __bf16* q = pos + (size_t)(p % S) * H + half * 4;
    const __bf16* t = type + (size_t)seg * H + half * 4;
    bf16x4 a[NV], b[NV], c[NV];
    float4 v[NV], gm[NV], bt[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int chunk = min(chunk0 + i * 32, n_chunks - 1);
        a[i] = *reinterpret_cast<const bf16x4*>(w + chunk * 8);
        b[i] = *reinterpret_cast<const bf16x4*>(q + chunk * 8);
        c[i] = *reinterpret_cast<const bf16x4*>(t + chunk * 8);
        gm[i] = *reinterpret_cast<const float4*>(gamma + half * 4 + chunk * 8);
        bt[i] = *reinterpret_cast<const float4*>(beta + half * 4 + chunk * 8);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const bool in = chunk0 + i * 32 < n_chunks;
        v[i].x = in ? ((float)a[i][0] + (float)b[i][0]) + (float)c[i][0] : 0.f;
        v[i].y = in ? ((float)a[i][1] + (float)b[i][1]) + (float)c[i][1] : 0.f;
        v[i].z = in ? ((float)a[i][2] + (float)b[i][2]) + (float)c[i][2] : 0.f;
        v[i].w = in ? ((float)a[i][3] + (float)b[i][3]) + (float)c[i][3] : 0.f;
    }
    finish_row<NV>(v, gm, bt, chunk0, n_chunks, row, half, wave, lane, row < M, H, eps, of, ob, 0);
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

}  // namespace

hipError_t launch_layernorm_tiled(const TiledLnGroup& g, const TiledLnShape& s, hipStream_t stream)
{
    if (s.G <= 0 || s.M <= 0) return hipSuccess;
    if (s.G > kMaxGroup || s.H % 8 != 0 || s.H > 2048 || s.n_parts < 1) return hipErrorInvalidValue;
    dim3 grid((s.M + kRowsPerGroup - 1) / kRowsPerGroup, s.G), block(512);
    if (s.H <= 256) hipLaunchKernelGGL((layernorm_tiled_kernel<1>), grid, block, 0, stream, g, s);
    else if (s.H <= 512) hipLaunchKernelGGL((layernorm_tiled_kernel<2>), grid, block, 0, stream, g, s);
    else if (s.H <= 768) hipLaunchKernelGGL((layernorm_tiled_kernel<3>), grid, block, 0, stream, g, s);
    else if (s.H <= 1024) hipLaunchKernelGGL((layernorm_tiled_kernel<4>), grid, block, 0, stream, g, s);
    else hipLaunchKernelGGL((layernorm_tiled_kernel<8>), grid, block, 0, stream, g, s);
    return hipGetLastError();
}

hipError_t launch_embed_ln_tiled(const int32_t* ids, const int32_t* type_ids, int type_vocab, const int32_t* src, const int32_t* d_M, int B, int S,
                                 int H, int vocab, const void* word, const void* pos, const void* type, const float* gamma, const float* beta,
                                 float eps, float* out_f32, void* out_bf16, hipStream_t stream)
{
    const int M = B * S;
    if (M <= 0) return hipSuccess;
    if (H % 8 != 0 || H > 2048 || !src || !d_M) return hipErrorInvalidValue;
    dim3 grid((M + kRowsPerGroup - 1) / kRowsPerGroup), block(512);
#define MT_EMBED(NV)                                                                                                                    \
    hipLaunchKernelGGL((embed_ln_tiled_kernel<NV>), grid, block, 0, stream, ids, type_ids, type_vocab, src, d_M, M, S, H, vocab,        \
                       (const __bf16*)word, (const __bf16*)pos, (const __bf16*)type, gamma, beta, eps, out_f32, (__bf16*)out_bf16)
    if (H <= 256) MT_EMBED(1);
    else if (H <= 512) MT_EMBED(2);
    else if (H <= 768) MT_EMBED(3);
    else if (H <= 1024) MT_EMBED(4);
    else MT_EMBED(8);
#undef MT_EMBED
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
    hipLaunchKernelGGL(classifier_tiled_kernel, dim3(B, G, (maxC + 3) / 4), dim3(256), 0, stream, g, H, ldo, out_row);
    return hipGetLastError();
}

}  // namespace mt
