// Host-side launchers of every HIP kernel of the layer-stack library.
// Each launcher checks nothing: shapes are validated by the callers (stack.hip, ops_api.hip).
#pragma once

#include "common.h"
#include "prof.h"

namespace lga {

// ---- one-time set-up ----------------------------------------------------------------------
// Kernels that use more dynamic LDS than a launch may ask for by default (the attention kernels, the large-tile
// GEMM) have their limit raised here, once per process, before anything is launched: lga_init_stack calls it, and
// so does every launcher of such a kernel (a flag test after the first call), so the op-level entry points need no
// stack.  It must not run for the first time on a stream that is being captured into a graph - which is why the
// stack-level entry points call it at init and refuse capturing streams.
hipError_t prepare_kernels();
hipError_t attn_prepare_kernels();      // attention_bf16.hip's part
hipError_t gemm_prepare_kernels();      // gemm_bf16.hip's part
hipError_t gemm_f32_prepare_kernels();  // gemm_f32.hip's part
hipError_t gemm_small_prepare_kernels();  // gemm_small.hip's part
hipError_t attn_wide_prepare_kernels();   // attention_wide.hip's part

// ---- element-wise / row kernels (rowops.hip) ---------------------------------------------
// fp32 -> 16-bit copy of a parameter vector ("restore": parameters converted to 16 bits before use); E = bf16 or f16.
template <class E> void launch_cast_f32_to_16(const float *src, E *dst, size_t n, hipStream_t s);
// Counter-based N(0, std^2) fill: element i gets a value that depends only on (seed, i).
void launch_fill_normal(float *dst, size_t n, float std, uint64_t seed, hipStream_t s);
void launch_fill_const(float *dst, size_t n, float value, hipStream_t s);

// LayerNorm forward over rows of length d.  Writes y = xhat * g + b and the row statistics; keep != NULL: also a copy of x there.
template <class T>
void launch_layernorm_fwd(const T *x, const float *g, const float *b, T *y, float *mean, float *rstd,
                          int rows, int d, float eps, hipStream_t s, T *keep = nullptr);
// LayerNorm backward w.r.t. the input, fused with the residual add:
//   dx = resid + rstd * (g dy - mean_row(g dy) - xhat * mean_row(g dy xhat))
// dbeta != NULL: also the gradients of the LayerNorm bias and gain,
//   dbeta[c] = beta * dbeta[c] + sum_r dy[r, c],   dgamma[c] = beta * dgamma[c] + sum_r dy[r, c] xhat[r, c],
// added up inside the same kernel where the width allows, by the column-sum kernels otherwise; partial then holds
// layernorm_bwd_partial_floats(rows, d) floats.
// batch != NULL: the second pass of those sums is left to the caller's launch_colsum_batch; partial must then stay untouched until it.
struct ColsumJob {
    const float *partial;      // [chunks][2][cols]
    float *out0, *out1;        // out1 may be NULL
    int chunks, cols;
    float beta;
};
constexpr int kColsumBatch = 6;                            // four biases and two LayerNorms of a layer
struct ColsumBatch {
    ColsumJob job[kColsumBatch];
    int n = 0;
};
void launch_colsum_batch(const ColsumBatch &batch, hipStream_t s, bool timed = true);
// biases != NULL (with dbeta): also of_resid[c] = beta * of_resid[c] + sum_r resid[r, c] and the same of dx; partial holds
// layernorm_bwd_partial_floats(rows, d) floats.
struct BiasSums {
    float *of_resid, *of_dx, *partial;
};
size_t layernorm_bwd_partial_floats(int rows, int d);
template <class T>
void launch_layernorm_bwd_dx(const T *dy, const T *x, const float *mean, const float *rstd, const float *g,
                             const T *resid, T *dx, int rows, int d, hipStream_t s, float beta = 0.f,
                             float *dbeta = nullptr, float *dgamma = nullptr, float *partial = nullptr,
                             ColsumBatch *batch = nullptr, const BiasSums *biases = nullptr);
// Whether biases come at no pass of their own over rows of d elements (of esz bytes, 16-byte aligned).
bool layernorm_bwd_adds_biases(int d, int esz);

// Column sums over rows, in two deterministic passes through `partial`:
//   out0[c] = beta * out0[c] + sum_r a[r, c]
//   out1[c] = beta * out1[c] + sum_r a[r, c] * (x[r, c] - mean[r]) * rstd[r]     (only if out1 != NULL)
// a and x have leading dimension ld.  partial must hold colsum_partial_floats(rows, cols) floats.
// timed = false keeps the launch out of the per-launch profile (no events are created for it).
size_t colsum_partial_floats(int rows, int cols);
template <class T>
void launch_colsum(const T *a, const T *x, const float *mean, const float *rstd, int rows, int cols, int ld,
                   float beta, float *out0, float *out1, float *partial, hipStream_t s, bool timed = true, ColsumBatch *batch = nullptr);
// Up to four matrices in one launch per pass, each with partial sums of its own.
template <class T> struct ColsumMatrix {
    const T *a, *x;
    const float *mean, *rstd;
    float *out0, *out1, *partial;
    int rows, cols, ld;
};
template <class T>
void launch_colsums(const ColsumMatrix<T> *m, int n, float beta, hipStream_t s, bool timed = true, ColsumBatch *batch = nullptr);

// out[c][r] = in[r][c] for matrices of 16-bit elements of any format; R, C, ldi, ldo multiples of 8, 16-byte
// aligned bases.
void launch_transpose16(const void *in, void *out, int R, int C, long ldi, long ldo, hipStream_t s);
// The same for format E, and out0[c] = beta * out0[c] + sum_r in[r, c] from the tiles as they pass through the
// transposing kernel (partial: colsum_partial_floats(R, C) floats).
template <class E>
void launch_transpose16_colsum(const E *in, E *out, int R, int C, long ldi, long ldo, float beta, float *out0,
                               float *partial, hipStream_t s);

// Up to kTransposeBatch matrices in one launch; those with partial != NULL (colsum_partial_floats(R, C) floats) also leave the first pass of their
// column sums (values of format E) there, whose second pass add_colsum adds to a batch.
struct TransposeMatrix {
    const void *in;
    void *out;
    float *partial;
    long ldi, ldo;
    int R, C;
};
constexpr int kTransposeBatch = 8;                         // the operands of a layer's four weight gradients
template <class E> void launch_transposes(const TransposeMatrix *m, int n, hipStream_t s);
// The second pass of first passes in chunks of 128 rows, left by a kernel that had the matrix in hand
void add_colsum(ColsumBatch &batch, const float *partial, int rows, int cols, float beta, float *out0);
constexpr int kGemmSumRows = 128;

// 1 into *flag if any of the n values is infinite or not a number (*flag is not cleared here).
void launch_nonfinite_flag(const float *g, size_t n, int *flag, hipStream_t s);

// Adam update of n parameters in place; optionally (w16 != NULL) also writes the 16-bit copy of the new weights in
// format E (bf16 or f16).  The gradient is multiplied by grad_mul before use (1 / loss scale).  skip != NULL: the
// whole update is left out when *skip != 0 (gradient found non-finite).
template <class E>
void launch_adam(float *w, float *m, float *v, const float *g, E *w16, size_t n, float lr, float beta1, float beta2,
                 float eps, int step, float grad_mul, const int *skip, hipStream_t s);

// The same for a layer's n parameters, with its 16-bit copies w16 and w16t (each matrix transposed, at its place); matrices in the order of their
// places, their sizes, what lies between them and every address whole 16-byte pieces of 16-bit elements.  adam_writes_copies: whether it is the
// faster way to both copies for one of `layers` layers of these widths and n parameters each.
bool adam_writes_copies(int d, int f, size_t n, int layers);
struct AdamMatrix {
    size_t at;
    int rows, cols;
};
template <class E>
void launch_adam_copies(float *w, float *m, float *v, const float *g, E *w16, E *w16t, const AdamMatrix (&matrices)[4], size_t n, float lr, float beta1,
                        float beta2, float eps, int step, float grad_mul, const int *skip, hipStream_t s);

// ---- GEMMs -------------------------------------------------------------------------------
// C[M,N] = sum_k A(m,k) B(k,n), then the epilogue.
//   a_kmajor: A is stored [M][lda] (k contiguous); otherwise [K][lda] (m contiguous).
//   b_kmajor: B is stored [N][ldb] (k contiguous); otherwise [K][ldb] (n contiguous).
// fp32 kernel (fp32 matrix instruction), any shape and alignment:
void launch_gemm_f32(const GemmParams<float> &p, bool a_kmajor, bool b_kmajor, Epilogue epi, hipStream_t s);
// Several weight gradients in one launch: EPI_ACCUM_F32, operands [K][M] and [K][N], the same K, ldc = N.  p[0].partial / partial_floats is
// scratch for all, gemm_f32_group_floats() for as many slices as gemm_f32_group_slices(); with less the k range stays whole.
int gemm_f32_group_slices(const int *M, const int *N, int n, int K);
size_t gemm_f32_group_floats(const int *M, const int *N, int n, int slices);
void launch_gemm_f32_group(const GemmParams<float> *p, int n, hipStream_t s);
// Whether an EPI_MUL_DGELU product of this size (lda = ldb = K) leaves the first pass of its column sums at p.colsum, in chunks of
// kGemmSumRows rows.
bool gemm_dgelu_adds_columns(int M, int N, int K);
// 16-bit MFMA kernel (E = bf16 or f16), fp32 accumulate.  Needs lda, ldb, ldc, N multiples of 8 and 16-byte aligned
// bases.
// Returns false, launching nothing, for a layout / epilogue pair that is not built (gemm_mfma_supports) or a leading
// dimension beyond kGemmMaxLd.
constexpr int kGemmMaxLd = ((1 << 30) - 256) / (2 * 256);      // 2 097 151 elements: row 255 of a tile stays inside the loads' 1 GiB window
bool gemm_mfma_supports(bool a_kmajor, bool b_kmajor, Epilogue epi);
template <class E>
bool launch_gemm_mfma(const GemmParams<E> &p, bool a_kmajor, bool b_kmajor, Epilogue epi, hipStream_t s);
// Its share of problems with fewer than 128 tiles of 256 x 256, both operands k-contiguous (gemm_small.hip); p.ldc, p.N multiples of 8
// and every tensor 16-byte aligned.  Uses p.partial for slices of a long k range where that is large enough.
template <int EPI, class E> void launch_gemm_small(const GemmParams<E> &p, hipStream_t s);
// Slices of the k range that it cuts a weight gradient into, given so many floats of scratch (1 = none).
int gemm_small_slices(int M, int N, int K, size_t partial_floats);
// out[m, n] = beta * out[m, n] + sum_z partial[z][m][n], slices in index order; N and ldc multiples of 4, 16-byte aligned
void launch_splitk_reduce(const float *partial, int slices, float *out, int M, int N, int ldc, float beta, hipStream_t s);
// Several weight gradients (EPI_ACCUM_F32, the same K, ldc = N a multiple of 4) in one launch: on the large-tile kernel from operands as
// stored, where gemm_group_slices() > 0 for them together, or on k-contiguous ones.  p[0].partial / partial_floats is scratch for all.
template <class E> void launch_gemm_stored_group(const GemmParams<E> *p, int n, hipStream_t s);
template <class E> void launch_gemm_transposed_group(const GemmParams<E> *p, int n, hipStream_t s);
template <class E> void launch_gemm_small_group(const GemmParams<E> *p, int n, hipStream_t s);
int gemm_group_slices(const int *M, const int *N, int n, int K);
bool gemm_stored_group_wins(const int *M, const int *N, int n, int K);         // over a launch each, for matrices that are enough work alone
// A group's parameters with the k range in so many slices (1: not cut), and the sum of the slices (nothing to do without)
template <class E> void prepare_gemm_group(GemmGroup<E> &group, const GemmParams<E> *p, int slices);
template <class E> void launch_splitk_reduce_group(const GemmGroup<E> &group, hipStream_t s);
// Into how many slices of the k range launch_gemm_mfma cuts an fp32-accumulating, k-contiguous GEMM whose output has
// too few 256 x 256 tiles to occupy the chip (1 = not at all); it then needs slices * M * N floats of scratch.
// k = 0 asks for the largest count any k would give (for sizing the scratch).
int gemm_splitk_slices(int M, int N, int K);
// Whether a weight gradient of this size runs on the large-tile kernel, which takes both operands as stored ([K][ld], ld >= 256);
// true for every larger K then, too.  The 16-bit kernels for smaller ones want them k-contiguous.
bool gemm_takes_stored_operands(int M, int N, int K);
// Columns of the 256-row tiles of a product with both operands k-contiguous and epilogue epi (pre: GELU that stores its input, too): 192, 128,
// or 0 for 256 or the small kernel
int gemm_narrow_width(int M, int N, int K, int epi, bool pre);

// ---- causal attention --------------------------------------------------------------------
// qkv: [tokens, 3 d] with columns [Q | K | V], head h at columns h*dh inside each third; tokens =
// n_seq * s, each sequence attends only to itself.  out: [tokens, d].  lse: [n_seq, heads, s] holds
// log(sum_j exp(score_ij)) of the scaled scores.  d = heads * dh.
// causal != 0: position i attends to j <= i (decoder); 0: to its whole sequence (encoder).
struct AttnShape {
    int n_seq, s, heads, dh, causal;
};
int attn_fwd_subblocks(const AttnShape &sh);     // of 32 queries, per wavefront of the fused forward kernel: 1 or 2
template <class T> void launch_attn_fwd_simple(const T *qkv, T *out, float *lse, AttnShape sh, hipStream_t s);
// dqkv: [tokens, 3 d]; delta: scratch [n_seq, heads, s] (row sums of dout * out).
template <class T>
void launch_attn_bwd_simple(const T *qkv, const T *out, const float *lse, const T *dout, T *dqkv, float *delta,
                            AttnShape sh, hipStream_t s);
// The same on fp32 tensors with the fp32 matrix instruction (attention_f32.hip), head sizes up to 128 and more than 48 positions.
bool attn_f32_supports(AttnShape sh);
void launch_attn_fwd_f32(const float *qkv, float *out, float *lse, AttnShape sh, hipStream_t s);
void launch_attn_bwd_f32(const float *qkv, const float *out, const float *lse, const float *dout, float *dqkv, float *delta,
                         AttnShape sh, hipStream_t s);
// MFMA kernels with LDS-resident online softmax (E = bf16 or f16).  Head sizes other than those
// attn_bf16_supports() accepts are routed to the one-wavefront kernels above.
bool attn_bf16_supports(int dh);
template <class E> void launch_attn_fwd_mfma(const E *qkv, E *out, float *lse, AttnShape sh, hipStream_t s);
template <class E>
void launch_attn_bwd_mfma(const E *qkv, const E *out, const float *lse, const E *dout, E *dqkv, float *delta,
                          AttnShape sh, hipStream_t s);

// The O that the fused dQ kernels take delta = sum_c dO O from - or, where its memory is also dQKV's, delta from a pass before them, and NULL.
template <class E> const E *delta_apart(const E *out, const E *dout, const E *dqkv, float *delta, AttnShape sh, hipStream_t s);
// Fused kernels for head sizes above 160 and up to 320, multiples of 8 (attention_wide.hip).
bool attn_wide_supports(int dh);
template <class E> void launch_attn_fwd_wide(const E *qkv, E *out, float *lse, AttnShape sh, hipStream_t s);
template <class E>
void launch_attn_bwd_wide(const E *qkv, const E *out, const float *lse, const E *dout, E *dqkv, float *delta,
                          AttnShape sh, hipStream_t s);

// The same attention for head sizes without a fused kernel, built from batched GEMMs and two row kernels
// (attention_gemm.hip).  Needs s and dh to be multiples of 8 and a workspace of at least
// attn_gemm_workspace_bytes(s, 1) bytes (256-byte aligned); more workspace, up to attn_gemm_workspace_bytes(s, heads),
// lets more heads share a launch.
size_t attn_gemm_workspace_bytes(int s, int heads);
bool attn_gemm_supports(AttnShape sh, size_t ws_bytes);
template <class E>
void launch_attn_fwd_gemm(const E *qkv, E *out, float *lse, AttnShape sh, void *ws, size_t ws_bytes, hipStream_t s);
template <class E>
void launch_attn_bwd_gemm(const E *qkv, const E *out, const float *lse, const E *dout, E *dqkv, float *delta,
                          AttnShape sh, void *ws, size_t ws_bytes, hipStream_t s);

}  // namespace lga
