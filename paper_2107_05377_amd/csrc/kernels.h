// Internal launch interface between the host scheduler and the gfx950 kernels.
// Every launcher only enqueues on `stream`; none allocates or synchronises.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

namespace mt {

typedef uint16_t bf16_t;   // raw bfloat16 bits in host-visible interfaces

constexpr int kMaxGroup = 32;   // problems per grouped launch (one per active task)

// Epilogue applied to the fp32 accumulator: v = acc + bias[n]; v = act(v); v += residual[m][n].
enum ActKind : int { ACT_NONE = 0, ACT_GELU_ERF = 1, ACT_GELU_TANH = 2, ACT_TANH = 3 };

// A group of G same-shaped problems C_g[M,N] = epi(A_g[M,K] * W_g[N,K]^T), passed by value as a
// kernel argument so that a change of the active task set needs no device-side table.
struct GemmGroup {
    const void* A[kMaxGroup];
    const void* W[kMaxGroup];
    void* C[kMaxGroup];
    const float* bias[kMaxGroup];       // may be null
    const float* residual[kMaxGroup];   // fp32 [M][ldr], may be null
    int32_t N[kMaxGroup];               // per-problem N (fp32 path only; the MFMA path needs uniform N)
    float scale[kMaxGroup];             // FP8 path only: the accumulator is multiplied by this before the bias is added
};

struct GemmShape {
    int32_t G, M, N, K;     // N = max over the group; M = row bound (grid size), see d_M
    int64_t lda, ldc, ldr;  // row strides in elements
    int32_t act;            // ActKind
    int32_t out_f32;        // 1: C is float32, 0: C has the activation element type (bf16); FP8 path also 2: C is E4M3 bytes
    const int32_t* d_M;     // optional device scalar: rows actually present (<= M); tiles beyond it exit at once
    int32_t splits;         // bf16 path, >= 1: K is cut into `splits` equal ranges, range p of problem g writing its
                            // partial product (float32, no epilogue) to C_g + p * split_stride elements
    int64_t split_stride;
    int64_t ldw;            // row stride of W in elements; 0 = dense (K)
    // Few-row kernel only (launch_gemm_bf16 routes there when n_sub > 1): every problem g consists of n_sub
    // sub-problems of the same shape, sub-problem u using A_g + u*sub_a, W_g + u*sub_w, C_g + u*sub_c and
    // bias_g + u*sub_bias (element offsets); no residual.  With d_sub_row0 / d_sub_rows (device arrays [n_sub])
    // sub-problem u additionally starts at row d_sub_row0[u] of A and C and has d_sub_rows[u] (<= M) rows:
    // a ragged batch, e.g. one sub-problem per sequence of the padding-free row order.
    int32_t n_sub;
    int64_t sub_a, sub_w, sub_c, sub_bias;
    const int32_t* d_sub_row0;
    const int32_t* d_sub_rows;
    float out_scale;        // FP8 path, out_f32 == 2: the value is multiplied by this before it is rounded to E4M3
};

// bf16 x bf16 -> fp32 accumulate on the matrix cores.  Needs K % 64 == 0, lda % 8 == 0, 16-byte aligned A/W rows.
hipError_t launch_gemm_bf16(const GemmGroup& g, const GemmShape& s, hipStream_t stream);
// FP8 (OCP E4M3) x FP8 -> float32 accumulate, both operands one byte per element, K contiguous (lda / ldw in elements =
// bytes, multiples of 16); needs K % 64 == 0 and K >= 192.  C_g = epi(g.scale[g] * A_g W_g^T + bias): out_f32 0 / 1 / 2
// = bf16 / float32 (+ residual) / E4M3 (times out_scale).  Activations: none, GELU(erf), GELU(tanh).
hipError_t launch_gemm_fp8(const GemmGroup& g, const GemmShape& s, hipStream_t stream);
// Persistent variant for launches of many 256x256 tiles (one workgroup per compute unit walks a tile list with
// its load ring never draining); launch_gemm_bf16 routes to it by itself.  gemm_bf16_persist_takes: shape supported.
bool gemm_bf16_persist_takes(const GemmShape& s);
bool gemm_bf16_persist_wants(const GemmShape& s);      // ... and measured faster than the tiled kernel
hipError_t launch_gemm_bf16_persist(const GemmGroup& g, const GemmShape& s, hipStream_t stream);
// Few-row variant (M <= 256), memory-parallel instead of tiled; launch_gemm_bf16 routes to it by itself.
hipError_t launch_gemm_skinny_bf16(const GemmGroup& g, const GemmShape& s, hipStream_t stream);
// Register-only matrix-core rate measurement: n_cu workgroups of 8 wavefronts, `iters` x 8 MFMAs each; d_out needs
// mfma_rate_out_floats(n_cu) floats.  Synchronises on the stream.
hipError_t run_mfma_rate(int iters, int n_cu, float* d_out, hipStream_t stream, float* tflops);
int mfma_rate_out_floats(int n_cu);
// ---- panel layout of the bfloat16 path: 32 rows form a panel; inside a panel the columns come in chunks of 8, a chunk holding its
// 8 columns of row 0, of row 1, ... (512 bytes of bf16, 1 KB of float32).  Weights (rows = output columns), operands and the float32
// states have it alike.  Element offset of (row, col) in a matrix of `width` columns (a multiple of 8), rows padded to a multiple of 32:
__host__ __device__ inline size_t tiled_offset(size_t row, size_t col, size_t width)
{
    return (row >> 5) * 32 * width + (col >> 3) * 256 + (row & 31) * 8 + (col & 7);
}
// Weights that later launches of a small call will need, read ahead by additional workgroups of its launches that leave most of the chip and all of the
// memory's bandwidth unused (LayerNorm and attention of the trunk): a contraction of few rows waits for its weights, which then come from the last-level
// cache (36 rows x 2304 / 3072 x 768, x 768 x 3072: 3.8 us each from memory, 3.0 from that cache).  Blocks of kAheadBlock bytes, one per workgroup, of up to
// four pieces (offsets from base in 256 bytes).
constexpr uint32_t kAheadBlock = 32768;
struct ReadAhead {
    static constexpr bool kAny = true;
    const void* base = nullptr;
    uint32_t at[4] = {}, bytes[4] = {};
    int blocks() const
    {
        int n = 0;
        for (int i = 0; i < 4; ++i) n += (int)((bytes[i] + kAheadBlock - 1) / kAheadBlock);
        return n;
    }
};
// Launches that read nothing ahead have kernels without it: its registers and arguments cost them (32 x 37 tokens of 8 tasks 705 -> 695 us a pass, 22 x 58 711 ->
// 702, 13 x 58 602 -> 597).
struct NoAhead {
    static constexpr bool kAny = false;
};
// ... in the order of their use.  A launch takes kAheadBytes: two MB more or less are level, 8 MB and what contractions of few rows could carry lengthen
// the launches by as much as the later ones gain (one request, 0 / 4 / 8 MB by each: 312, 305, 308 us; with 4 MB by each contraction as well 320).
constexpr uint32_t kAheadBytes = 4u << 20;
struct AheadQueue {
    struct Piece {
        uint32_t at, bytes;
    };
    const void* base = nullptr;
    std::vector<Piece> piece;
    size_t next = 0, used = 0;      // the next piece to read, pieces whose launches have been made
    uint32_t done = 0;              // bytes of the next piece that have been read
    ReadAhead take()
    {
        ReadAhead r;
        uint32_t budget = kAheadBytes;
        if (next < used) {
            next = used;
            done = 0;
        }
        r.base = base;
        for (int i = 0; i < 4 && budget >= kAheadBlock && next < piece.size(); ++i) {
            const uint32_t n = std::min(piece[next].bytes - done, budget / kAheadBlock * kAheadBlock);
            r.at[i] = piece[next].at + done / 256;
            r.bytes[i] = n;
            budget -= n;
            done += n;
            if (done == piece[next].bytes) {
                ++next;
                done = 0;
            }
        }
        return r;
    }
};
// Grouped problems as byte offsets from common bases, in units of 256 bytes (all buffers of the arenas are so aligned): a third of the
// kernel arguments that pointers would be, which the host writes on every launch (4.1 -> 2.9 us of host time a launch).
constexpr uint32_t kNoBias = 0xFFFFFFFFu;
struct TiledGroup {
    const void* A;          // bf16 [M][lda]
    const void* W;          // bf16 [N][ldw]
    void* C;                // bf16 or float32 [M][ldc]
    const float* bias;      // added before the activation (to the first of the partial results)
    uint32_t a[kMaxGroup], w[kMaxGroup], c[kMaxGroup], b[kMaxGroup];   // b: kNoBias = none
};
struct TiledShape {
    int32_t G, M, N, K;         // M: row bound; N % 32 == 0, K % (64 splits) == 0
    int32_t lda, ldw, ldc;      // widths of the matrices that the operands' columns are part of
    int32_t act, out_f32;       // out_f32: TILED_BF16, TILED_F32, or TILED_E4M3 (f8 only)
    const int32_t* d_M;         // optional device scalar: rows present
    int32_t splits;             // K ranges, each with a float32 partial result, split_stride elements apart
    int64_t split_stride;
    // few-row forms only: every problem is n_sub equal ones (heads) whose operands lie so far apart, in units of 256 bytes
    int32_t n_sub, sub_a, sub_w, sub_c, sub_b;
    // bf16 results without activation: from this column panel on (0 = none) a 32x32 block is stored transposed, as the operand of a
    // product over its rows: [16 rows][half][32 columns][8 rows], rows of a (16, half) run: 4 half + 0..3, 8 + 4 half + 0..3
    int32_t vt_panel;
    // problems that the launch has when every task is enabled (0 = G): decides the order in which K is added up, see choose_form
    int32_t plan;
    // both operands are E4M3 in panels of their own (tiled_offset_e4m3); K, lda and ldw count pairs of elements, splits is 1, and
    // kScaleSlot bytes in front of a weight matrix stands what its values are multiplied by, as an E8M0 exponent in each byte of an int32.
    // E4M3 results at unit scale, saturating.
    int32_t f8;
    int32_t stream;             // set by the launch: results are stored past the second-level caches
};
enum TiledOut : int { TILED_BF16 = 0, TILED_F32 = 1, TILED_E4M3 = 2 };
constexpr size_t kScaleSlot = 256;
// Byte offset of (row, col) in an E4M3 panel matrix (a multiple of 64 columns): as tiled_offset with chunks of 16 columns, of every four of
// which the middle two change places: the two 16-byte loads of a lane then bring 32 consecutive columns, in which order the products of a
// matrix instruction are added up as in the row-major kernel's (gemm_fp8.hip).
__host__ __device__ inline size_t tiled_offset_e4m3(size_t row, size_t col, size_t width)
{
    const size_t c = col >> 4, place = (c & ~(size_t)3) | (c & 1) << 1 | (c >> 1 & 1);
    return (row >> 5) * 32 * width + place * 512 + (row & 31) * 16 + (col & 15);
}
// The kernel forms (gemm_tiled.hip); TILED_AUTO chooses by shape.
enum TiledForm : int { TILED_AUTO = 0, TILED_ROWS_1X1, TILED_ROWS_2X1, TILED_ROWS_2X2, TILED_K2, TILED_PAIR, TILED_TALL };
// K ranges (1, 2 or 4, at most `most`) of one contraction with a float32 result: a long K over few output blocks (a row bound of up to 128 at 768
// columns) leaves most of the chip idle otherwise; 36 rows x 768 x 3072: 10 us whole, 4.4 us in 4 ranges that the LayerNorm adds up.  The number
// of problems that are there does not enter: a task's result must not depend on which others are enabled.
int tiled_splits(int M, int N, int K, int most);
hipError_t launch_gemm_tiled(const TiledGroup& g, const TiledShape& s, hipStream_t stream, int form = TILED_AUTO, int force_height = 0);
// compute units of the current device (cached per device)
int device_cu_count();

// LayerNorm on the panel layout: out = LN(sum_p x[p] + residual), H a multiple of 64 up to 1024, offsets as above from the
// workspace and the weights.
struct TiledLnGroup {
    const void* ws;
    const void* wt;
    uint32_t x[kMaxGroup], res[kMaxGroup], out_f[kMaxGroup], out_b[kMaxGroup];
    uint32_t gamma[kMaxGroup], beta[kMaxGroup];
};
struct TiledLnShape {
    int32_t G, M, H;
    const int32_t* d_M;
    float eps;
    int32_t n_parts;
    int64_t part_stride;        // elements
    const int32_t* res_row;     // optional: residual row of row i is res_row[i] (below res_rows)
    int32_t res_rows;
    int32_t split;              // out_b: 0 the row as bf16, 1 as [hi | lo] bf16 halves of a matrix of 2H columns
    // operand copies of problem i: bit i of want_b the one at out_b, of want_q one in E4M3 (unit scale, saturating) q_offset bytes behind out_b: of
    // the bf16 values, or (q_offset 0: in its place) of the float32 ones
    uint32_t want_b = ~0u, want_q = 0;
    int64_t q_offset = 0;
    // the order of the row-major kernel's sums, to the bit (H a multiple of 256, one part): layers whose operands are E4M3
    int32_t whole_sums = 0;
};
hipError_t launch_layernorm_tiled(const TiledLnGroup& g, const TiledLnShape& s, hipStream_t stream, AheadQueue* ahead = nullptr);
// As launch_embed_ln (bf16 tables), states in the panel layout.  out_bf16, out_e4m3: operand copies, either may be null.
hipError_t launch_embed_ln_tiled(const int32_t* ids, const int32_t* type_ids, int type_vocab, const int32_t* src, const int32_t* d_M, int B, int S,
                                 int H, int vocab, const void* word, const void* pos, const void* type, const float* gamma, const float* beta,
                                 float eps, float* out_f32, void* out_bf16, void* out_e4m3, hipStream_t stream);
struct RowCopyGroup {
    const float* in_f[kMaxGroup];
    const void* in_b[kMaxGroup];
    float* out_f[kMaxGroup];
    void* out_b[kMaxGroup];
    const void* in_q[kMaxGroup];
    void* out_q[kMaxGroup];
};
// out row i = in row index[i] for i < *n (n_max if n is null), float32, bf16 and / or E4M3 matrices of H columns (a null input: not that kind)
hipError_t launch_copy_rows_tiled(const RowCopyGroup& g, int G, const int32_t* index, const int32_t* n, int n_max, int max_rows, int H, hipStream_t stream);

// First-token attention without projected keys and values (first_token.hip).
struct FirstTokenGroup {
    const void* x[kMaxGroup];       // bf16 layer input, all rows
    const void* first[kMaxGroup];   // its first-token rows, one per sequence
    const void* Wq[kMaxGroup];      // panels of the query matrix
    const float* bq[kMaxGroup];
    const void* WkT[kMaxGroup];     // panels of the transposed key matrix
    void* qt[kMaxGroup];            // bf16 [B][16][H], rows from the number of heads on unused
    void* xbar[kMaxGroup];          // per head a bf16 [B][H] panel matrix, xbar_stride elements apart
};
// up to so many sequences' first rows are read in place (seq_start given: `first` is not used, x has max_rows rows)
constexpr int kInPlace = 8;
hipError_t launch_first_query(const FirstTokenGroup& g, int G, int B, int H, int A, hipStream_t stream, const int32_t* seq_start = nullptr, int max_rows = 0);
// whole_weights: the softmax weights enter with all their float32 bits instead of 16
hipError_t launch_first_attend(const FirstTokenGroup& g, int G, const int32_t* seq_start, const int32_t* seq_len, int B, int S, int H, int A,
                               int64_t xbar_stride, hipStream_t stream, bool whole_weights = false);

// float32 operands, products and sums; any shape.
hipError_t launch_gemm_f32(const GemmGroup& g, const GemmShape& s, hipStream_t stream);

// Token rows of a batch in padding-free order: only positions with mask == 1 are kept, sequence after
// sequence, so every row-wise kernel and every contraction runs on sum_b len_b rows instead of B*S.
struct RowMap {
    int32_t* n_rows;      // [1]  number of kept rows
    int32_t* src;         // [B*S] kept row -> b*S+s
    int32_t* row_of;      // [B*S] b*S+s -> kept row, or -1
    int32_t* seq_start;   // [B]  first kept row of sequence b
    int32_t* seq_len;     // [B]  kept rows of sequence b
};
hipError_t launch_build_row_map(const int32_t* mask, int B, int S, const RowMap& map, hipStream_t stream);
// *count = number of sequences whose position 0 is masked off (mask[b][0] == 0; an all-padding sequence is one of them)
hipError_t launch_count_bad_first_tokens(const int32_t* mask, int B, int S, int32_t* count, hipStream_t stream);
// bfloat16 [M][H] -> E4M3 [M][H] (unit scale, saturating) for up to kMaxGroup arrays in one launch; rows past *d_M are left alone
struct CastGroup {
    const void* src[kMaxGroup];
    void* dst[kMaxGroup];
};
hipError_t launch_cast_bf16_to_e4m3(const CastGroup& g, int G, int M, const int32_t* d_M, int H, hipStream_t stream);
// out[b*S+s][:] = x[row_of[b*S+s]][:] or 0 (float32, H columns)
hipError_t launch_unpack_rows(const float* x, const int32_t* row_of, int n_pos, int H, float* out, hipStream_t stream, int tiled = 0);

// Longest sequence the bf16 attention kernel takes: the keys and values of one (sequence, head) are staged in
// LDS as a whole, 260 bytes per key (rounded up to 32 keys) within the CU's 160 KB.
constexpr int kAttnBf16MaxSeq = 608;
struct AttnGroup {
    const void* qkv[kMaxGroup];   // [rows][3H]: Q | K | V
    void* ctx[kMaxGroup];         // [rows][H]
};
// Sequence b owns rows seq_start[b] .. +seq_len[b]-1 (all real tokens) when the two arrays are given;
// otherwise rows b*S .. b*S+S-1 with `mask` ([B][S], 1 = real) marking the keys.  S bounds the length.
// ctx_fmt 0: the context is written as bfloat16; 1: as E4M3 at unit scale (one byte per element, same row order).  panels: both matrices in the
// panel layout (values not transposed); packed sequences and E4M3 only.
hipError_t launch_attention_bf16(const AttnGroup& g, int G, const int32_t* mask, const int32_t* seq_start,
                                 const int32_t* seq_len, int B, int S, int H, int A, hipStream_t stream, int ctx_fmt = 0, bool panels = false);
// Panel layout, packed sequences: projections with the values transposed (TiledShape::vt_panel), context as an operand; offsets in 256 bytes.
struct AttnTiledGroup {
    const void* base_qkv;
    void* base_ctx;
    uint32_t qkv[kMaxGroup], ctx[kMaxGroup];
};
hipError_t launch_attention_tiled(const AttnTiledGroup& g, int G, const int32_t* seq_start, const int32_t* seq_len, int B, int S, int H, int A,
                                  hipStream_t stream, AheadQueue* ahead = nullptr);
hipError_t launch_attention_f32(const AttnGroup& g, int G, const int32_t* mask, const int32_t* seq_start,
                                const int32_t* seq_len, int B, int S, int H, int A, hipStream_t stream);

struct LnGroup {
    const float* x[kMaxGroup];      // [n_parts][M][H] fp32: the row to normalise is sum_p x[p] (+ bias) (+ residual)
    const float* bias[kMaxGroup];      // [H], may be null
    const float* residual[kMaxGroup];  // [M][H] fp32, may be null
    const float* gamma[kMaxGroup];
    const float* beta[kMaxGroup];
    float* out_f32[kMaxGroup];      // may be null
    bf16_t* out_bf16[kMaxGroup];    // may be null
};
// d_M (optional device scalar) = rows actually present (<= M); n_parts partial sums part_stride elements apart
// low_fmt: element type written through out_bf16: 0 bfloat16, 1 OCP FP8 E4M3 (one byte per element, saturating)
hipError_t launch_layernorm(const LnGroup& g, int G, int M, const int32_t* d_M, int H, float eps, int n_parts, int64_t part_stride,
                            hipStream_t stream, int low_fmt = 0);

// X0[r] = LN(word[ids[p]] + pos[p % S] + type[0]) with p = src[r] for the kept rows r < *d_M (p = r and all
// B*S rows when src is null); tables are bf16 (emb_bf16 != 0) or fp32.
hipError_t launch_embed_ln(const int32_t* ids, const int32_t* type_ids /* [B*S] segment ids or NULL */, int type_vocab, const int32_t* src, const int32_t* d_M, int B, int S, int H, int vocab, const void* word, const void* pos,
                           const void* type, int emb_bf16, const float* gamma, const float* beta, float eps,
                           float* out_f32, bf16_t* out_bf16, hipStream_t stream);

// Pooler input for the matrix-core path: row b of problem g is the first token of sequence b of x[g]
// (float32 rows of H; row seq_start[b], or b*rows_per_seq when seq_start is null); it is written as [hi | lo] bfloat16 halves, hi = bf16(v), lo = bf16(v - hi), into
// out[g] ([B][2H]), so that a bf16 contraction against [W | W] reproduces the float32 input to ~2^-17.
struct SplitGroup {
    const float* x[kMaxGroup];
    bf16_t* out[kMaxGroup];
    int32_t compact[kMaxGroup];   // 1: x[g] already holds one row per sequence (row b), ignore seq_start
};
// float32 validation mode: the same first-token rows copied unchanged, out[g] reinterpreted as float [B][H]
hipError_t launch_gather_rows(const SplitGroup& g, int G, int B, int H, const int32_t* seq_start, int rows_per_seq, int max_rows,
                              hipStream_t stream);
hipError_t launch_cls_split(const SplitGroup& g, int G, int B, int H, const int32_t* seq_start, int rows_per_seq, int max_rows,
                            hipStream_t stream);
// panel layout, x[g] all rows (seq_start given, none compact)
hipError_t launch_split_first_rows_tiled(const SplitGroup& g, int G, int B, int H, const int32_t* seq_start, int max_rows, hipStream_t stream);

// First-token rows of every sequence, gathered into compact [B][H] arrays: float32 and/or element-type copies.
struct FirstRowsGroup {
    const float* xf[kMaxGroup];     // [rows][H] fp32 source, may be null
    const void* xa[kMaxGroup];      // [rows][H] activation-type source (bf16 or fp32), may be null
    float* out_f[kMaxGroup];        // [B][H]
    void* out_a[kMaxGroup];         // [B][H]
};
hipError_t launch_gather_first_rows(const FirstRowsGroup& g, int G, int B, int H, int act_bytes, const int32_t* seq_start,
                                    int max_rows, hipStream_t stream);
// out[b][s][:] = (s == 0) ? x[b][:] : 0 for a [B][S][H] float32 output
hipError_t launch_place_first_rows(const float* x, int B, int S, int H, float* out, hipStream_t stream, int tiled = 0);

// Attention for the first-token query of every sequence only (the last layer of a branch needs nothing else):
// q[g] is [B][H] (one query row per sequence), keys and values come from kv[g] = [rows][3H] (columns H.. and 2H..),
// sequence b owning rows seq_start[b] .. +seq_len[b]-1; ctx[g] is [B][H].  Any head width <= 256.
struct AttnClsGroup {
    const void* q[kMaxGroup];
    const void* kv[kMaxGroup];
    void* ctx[kMaxGroup];
};
hipError_t launch_attention_cls(const AttnClsGroup& g, int G, int is_bf16, const int32_t* seq_start, const int32_t* seq_len,
                                int B, int S, int H, int A, hipStream_t stream);

// First-token attention WITHOUT projected keys and values (bf16 path).  With q~[b][a] = Wk_a^T q[b][a] the
// score of key j is q~[b][a] . x_j (+ a constant per row, which the softmax drops), and the head's context is
// Wv_a (sum_j p_j x_j) + bv_a.  This kernel takes the raw scores[g] = [rows][A_pad] (float32, x_j . q~),
// scales them, takes the softmax over each sequence's rows and writes the probability-weighted sum of the
// layer input rows x[g] = [rows][H] (bf16) per head: xbar[g] = [B][A_pad][H] (bf16).
struct PoolGroup {
    const float* scores[kMaxGroup];
    const void* x[kMaxGroup];
    void* xbar[kMaxGroup];
};
hipError_t launch_first_token_pool(const PoolGroup& g, int G, const int32_t* seq_start, const int32_t* seq_len, int B, int S, int H,
                                   int A, int A_pad, hipStream_t stream);

// logits[g][b][c] = Wc_g[c][:] . pooled_g[b][:] + bc_g[c]; one wavefront per (g, b, c).  Wc bf16 or fp32.
struct ClsGroup {
    const float* pooled[kMaxGroup];   // [B][H]
    const void* Wc[kMaxGroup];        // [C][H]
    const float* bc[kMaxGroup];
    float* out[kMaxGroup];            // first logit column of the task, row stride ldo
    int32_t C[kMaxGroup];
};
// out_row: optional device array [B], logits row of compact row b (per-sequence routing); NULL = row b.
hipError_t launch_classifier(const ClsGroup& g, int G, int B, int H, int maxC, int w_bf16, int64_t ldo, const int32_t* out_row,
                             hipStream_t stream);
// bf16 Wc, pooled in the panel layout
hipError_t launch_classifier_tiled(const ClsGroup& g, int G, int B, int H, int maxC, int64_t ldo, const int32_t* out_row, hipStream_t stream);

// Token-level heads: out[g][p*ldo + c] = Wc[g][c] . x[g][row_of[p]] + bc[g][c] for every position p = b*S+s that is a
// kept row (row_of[p] in [0, *n_rows)), zeros for the positions that are not; positions with row_of[p] == -2 are
// left untouched.  x is float32 in the padding-free order.
struct TokGroup {
    const float* x[kMaxGroup];        // [rows][H]
    const void* Wc[kMaxGroup];        // [C][H]
    const float* bc[kMaxGroup];
    float* out[kMaxGroup];            // first logit column of the task at position 0, position stride ldo
    int32_t C[kMaxGroup];
};
// tiled: x in the panel layout.
hipError_t launch_token_classifier(const TokGroup& g, int G, int n_pos, int H, int w_bf16, int64_t ldo, const int32_t* row_of,
                                   const int32_t* n_rows, hipStream_t stream, int tiled = 0);

// Several request batches served by one forward pass: request r's ids and mask ([batch][seq] each) are copied behind
// one another into contiguous staging arrays, and afterwards the logits rows of the combined batch go back to each
// request's own [batch][ldo] array, only the columns whose bit is set in col_on (bit c of word c/32).
constexpr int kMaxRequests = 64;
constexpr int kMaxLogitCols = 1024;
struct RequestPtrs {
    const int32_t* ids[kMaxRequests];
    const int32_t* mask[kMaxRequests];
    float* out[kMaxRequests];
    int32_t first[kMaxRequests + 1];     // request r owns sequences first[r] .. first[r+1]-1 of the combined batch
    uint32_t col_on[kMaxLogitCols / 32];
};
// max_batch: the largest request's sequence count (sizes the grids)
hipError_t launch_gather_requests(const RequestPtrs& rq, int n_req, int max_batch, int seq, int32_t* ids_all, int32_t* mask_all, hipStream_t stream);
hipError_t launch_scatter_logits(const RequestPtrs& rq, int n_req, int max_batch, int n_cols, const float* logits_all, hipStream_t stream);

// Per-sequence task routing: a sub-batch of the sequences, as a padding-free row order of its own.
// idx lists the chosen sequences (ascending batch indices), passed by value with the launch.
constexpr int kMaxRouted = 1024;
struct RouteIdx {
    uint16_t seq[kMaxRouted];
};
// From the batch's row map (g_start, g_len) builds the sub-batch's: c_start/c_len [n_sel], *c_n rows in all,
// c_src[r] = row of the batch order that compact row r copies, c_seq[i] = idx.seq[i] (as int32, for the logits rows).
hipError_t launch_route_map(const RouteIdx& idx, int n_sel, const int32_t* g_start, const int32_t* g_len, int32_t* c_start,
                            int32_t* c_len, int32_t* c_src, int32_t* c_seq, int32_t* c_n, hipStream_t stream);
// c_rowof[b*S+s] for all B*S positions of the batch: the sub-batch's compact row of a real token of a chosen sequence,
// -1 for its padded positions, -2 for positions of sequences outside the sub-batch (launch_token_classifier leaves
// those untouched).  row_of / g_start: the batch's row map; c_start: the sub-batch's sequence starts.
hipError_t launch_route_rowof(const RouteIdx& idx, int n_sel, int B, int S, const int32_t* row_of, const int32_t* g_start,
                              const int32_t* c_start, int32_t* c_rowof, hipStream_t stream);
// out_f[r] = in_f[c_src[r]] (float32 rows) and out_a[r] = in_a[c_src[r]] (act_bytes per element; both optional), r < *c_n <= max_rows.
hipError_t launch_route_gather(const float* in_f, const void* in_a, float* out_f, void* out_a, const int32_t* c_src, const int32_t* c_n,
                               int max_rows, int H, int act_bytes, hipStream_t stream);

}  // namespace mt
