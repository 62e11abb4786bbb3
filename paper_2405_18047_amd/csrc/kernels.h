// Internal launch interface between the stage executor and the gfx950 kernels.
// Nothing here is part of the public C ABI (see include/tbp.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tbp {

enum Layout { NN = 0, NT = 1, TN = 2 };

// How a product that involves the causal probability matrix restricts its work.  A K_END or K_BEGIN product contracts over
// whole row tiles of its own (16 to 256 rows), so it reads its first operand beyond the diagonal, up to the end of the row
// tile: there that operand has to hold zeros.  The softmax zero-fills the probabilities P from the diagonal to the next
// multiple of kCausalPad columns, as far as any tile reads.  The score gradients dS come out of a SKIP_UPPER product, which
// leaves out tiles above the diagonal by a tile size of its own and writes zeros as far as GemmArgs::causal_fill says.
enum Causal {
  CAUSAL_NONE = 0,
  CAUSAL_SKIP_UPPER = 1,  // output [S,S] tiles strictly above the diagonal are not computed (q k^T, do v^T)
  CAUSAL_K_END = 2,       // A = P or dS [S,S]: contraction stops at the end of the row tile (P v, dS k)
  CAUSAL_K_BEGIN = 3      // A = P^T or dS^T:   contraction starts at the row tile's first index (P^T do, dS^T q)
};
constexpr int kCausalPad = 256;

struct GemmArgs {
  int layout;            // Layout
  int M, N, K;
  float alpha;
  const void* A; long lda;
  const void* B; long ldb;
  void* C; long ldc;
  const void* R;         // optional residual added before rounding (storage-type output only), same ld as C
  int out_f32;           // C is fp32
  int accumulate;        // C += (fp32 output only)
  int batch;             // grid z; z -> (zo = z / batch_inner, zi = z % batch_inner)
  int batch_inner;
  long sAo, sAi, sBo, sBi, sCo, sCi;   // element strides of the outer / inner batch index
  int causal;            // Causal
  // Softmax backward fused into the epilogue of dP = do v^T (per-head batched product with a storage-type output):
  // when delta is set, R points at the probabilities P (same layout as C) and the kernel stores
  // dS = P * (alpha * acc - delta[row]) for columns <= row and exact zeros above the diagonal (causal) instead of dP.
  // delta[(zo * sDo + zi * sDi) + row * ldd] = rowsum(dP * P) = sum over the head's columns of do * o.
  const float* delta; long ldd, sDo, sDi;
  int delta_causal;
  // With SKIP_UPPER and delta_causal: rows are written (zeros above the diagonal) up to the next multiple of causal_fill
  // columns, a power of two: the largest gemm_row_tile of the products that read dS.  Tiles that lie wholly above the
  // diagonal but inside that range store their zeros without contracting anything.
  int causal_fill;
  // Optional scratch for products whose output has too few tiles to fill the chip (see gemm_split_plan): device memory of
  // at least gemm_split_plan(...).bytes bytes, 256-byte aligned; nothing in it has to be initialised.
  void* ws; size_t ws_bytes;
  // TN layout, storage-type operands only: A is stored in panels of kPanel output rows, element (k, m) at
  // A[(m / kPanel) * a_panel + k * lda + m % kPanel] with lda == kPanel, so that the K x kPanel slab an output tile
  // contracts over is one contiguous stream.  0: plain [K, lda] matrix.  Such a product runs on kPanel-wide tiles.
  long a_panel;
  // SwiGLU backward fused into the epilogue of dm = dx Wd^T ([M, N] = [tokens, f]), where gemm_swiglu_p1_fuses: gate and up, C
  // receives their derivatives; both [M, 2 N] with leading dimension ldc, up behind gate.
  const void* gu;
};
// An NN product whose columns c and c + distance go into one result (see gemm_pairs_fuse): with m set, gate and up columns of a
// SwiGLU (distance = f; m [M, distance] receives silu(gate) * up); otherwise heads of 2 * distance columns, the first `rotated`
// of which leave rotated (rope: table [seq][distance], row r at position r % seq).
struct PairEpilogue {
  int distance;
  void* m;
  const float2* rope;
  int seq, rotated;
};
constexpr int kPanel = 128;
// elements of one (sequence, head) entry of the fused attention's dS^T scratch, stored in such panels
constexpr size_t attn_ds_elems(int seq) { return (size_t)((seq + kPanel - 1) / kPanel) * seq * kPanel; }

// Split of the contraction over several workgroups per output tile: slice i (contraction indices i * slice ..) leaves an
// fp32 partial product [M][N] in the scratch buffer and a second launch adds the slices up in order (so the result does
// not depend on timing).  split == 1: not worth it / not applicable.
struct SplitPlan { int tile, split, slice; size_t bytes; };
constexpr size_t kSplitHead = 1024;           // unused: part of the size that tbp_gemm_workspace_bytes has always told callers
SplitPlan gemm_split_plan(int dtype, int layout, int M, int N, int K, int out_f32, int batch);
// Scratch that a caller who would have to allocate it is told to bring for one such product: 0 also where slices gain too little.
size_t gemm_workspace_bytes(int dtype, int layout, int M, int N, int K, int out_f32);
// How gemm() runs a storage-type bf16 NN / NT product of at most one round of 256 x 256 tiles that is given ws_bytes of scratch:
// output tile, workgroups per compute unit that its LDS allows, slices.  false: another product.
bool gemm_plan(int layout, int M, int N, int K, size_t ws_bytes, int* tile_rows, int* tile_cols, int* per_cu, int* slices);

inline GemmArgs gemm_args(int layout, int M, int N, int K, const void* A, long lda, const void* B, long ldb,
                          void* C, long ldc) {
  GemmArgs g{};
  g.layout = layout; g.M = M; g.N = N; g.K = K; g.alpha = 1.f;
  g.A = A; g.lda = lda; g.B = B; g.ldb = ldb; g.C = C; g.ldc = ldc;
  g.batch = 1; g.batch_inner = 1;
  return g;
}

// dtype: 0 = fp32 storage, 1 = bf16 storage (matches tbp_dtype).
hipError_t gemm(int dtype, const GemmArgs& g, hipStream_t s);
bool gemm_swiglu_p1_fuses(int dtype, const GemmArgs& g);
bool gemm_pairs_fuse(int dtype, const GemmArgs& g, int distance);
hipError_t gemm_pairs(const GemmArgs& g, const PairEpilogue& pair, hipStream_t s);
// Rows of the output tiles that gemm() runs a product with a causal contraction (K_END, K_BEGIN) on.
int gemm_row_tile(int dtype, const GemmArgs& g);

// One bf16 weight-gradient product C (=, +=) A^T B (TN layout, fp32 C, alpha = 1).
// Same operand rules as the bf16 TN product of gemm(): 16-byte aligned pointers, extents and leading dimensions
// multiples of 8.
struct GroupedProduct {
  const void* A; const void* B; float* C;     // A [K, M] (lda), B [K, N] (ldb), C [M, N] (ldc)
  int M, N, K;
  int lda, ldb, ldc;
};
constexpr int kMaxGrouped = 40;               // products per launch (the table travels as a kernel argument)
struct GroupedTable {
  int n;
  int first_block[kMaxGrouped];
  GroupedProduct prod[kMaxGrouped];
};
// n of them, with one K; pool: host scratch for n entries.
hipError_t gemm_dw(const GroupedProduct* prods, int n, int accumulate, GroupedProduct* pool, hipStream_t s);

hipError_t rmsnorm_fwd(int dtype, int rows, int d, float eps, const void* x, const void* g, void* y, hipStream_t s);
// The same, leaving a copy of x in x_copy and, if table is not null, the rotation table of (seq, head_dim, base) in it.
hipError_t rmsnorm_fwd_first(int dtype, int rows, int d, float eps, const void* x, const void* g, void* y, void* x_copy,
                             float2* table, int seq, int head_dim, float base, hipStream_t s);
constexpr int kNormPartialBlocks = 256;     // at most this many row-block partials of the gain gradient per call
// RMSNorm backward-p1.  The gain gradient dg = sum over rows of dy * x * r leaves the row kernel as
// rmsnorm_partial_rows(dtype, rows, d) <= kNormPartialBlocks partial rows [d] fp32 (one per workgroup, each a sum over
// that workgroup's rows in a fixed order); gain_partials_sum adds partial rows up.
int rmsnorm_partial_rows(int dtype, int rows, int d);
// dx = resid + dL/dx; partials (may be null: nothing is computed for the gain) receives the partial rows; resid_copy
// (may be null) a copy of resid.
hipError_t rmsnorm_p1_rows(int dtype, int rows, int d, float eps, const void* dy, const void* x, const void* g,
                           const void* resid, void* dx, float* partials, hipStream_t s, void* resid_copy = nullptr);
// out[d] (= or +=) sum of the first n_rows rows of partials [n_rows][d]  (n_rows == 0: zero, or out left alone)
hipError_t gain_partials_sum(const float* partials, int n_rows, int d, int accumulate, float* out, hipStream_t s);
// The same for several norms in one launch (the table travels as a kernel argument).
constexpr int kMaxGainSums = 64;
struct GainSums { int n; const float* parts[kMaxGainSums]; float* out[kMaxGainSums]; };
hipError_t gain_partials_sums(const GainSums& g, int n_rows, int d, int accumulate, hipStream_t s);
// Both in one call: rows, then the sum into dg_out (dg_out == nullptr: nothing is computed for the gain).
hipError_t rmsnorm_p1(int dtype, int rows, int d, float eps, const void* dy, const void* x, const void* g,
                      const void* resid, void* dx, float* dg_out, float* partials, hipStream_t s);
hipError_t rmsnorm_gain_p2(int dtype, int rows, int d, float eps, const void* dy, const void* x, int accumulate,
                           float* dg_out, float* partials, hipStream_t s);
hipError_t swiglu_fwd(int dtype, int rows, int f, const void* gu, void* m, hipStream_t s);
hipError_t swiglu_p1(int dtype, int rows, int f, const void* dm, const void* gu, void* dgu, hipStream_t s);
hipError_t rope_table(int seq, int head_dim, float base, float2* table, hipStream_t s);
hipError_t rope(int dtype, int rows, int seq, int n_heads, int head_dim, long ld, const float2* table, int inverse,
                void* x, hipStream_t s);
hipError_t softmax_fwd(int dtype, long n_rows_total, int seq, int causal, const float* scores, void* P, hipStream_t s);
hipError_t softmax_p1(int dtype, long n_rows_total, int seq, int causal, const void* P, void* dP, hipStream_t s);
// delta[t * n_heads + h] = sum_c a[t, h*dh + c] * b[t, h*dh + c]   (fp32; a, b are [rows, n_heads*head_dim])
hipError_t head_rowdot(int dtype, int rows, int n_heads, int head_dim, const void* a, const void* b, float* delta,
                       hipStream_t s);
// Fused attention (bf16 storage only, head_dim 64 or 128).  qkv: [batch*seq, ld_qkv] with column blocks q | k | v of
// n_heads*head_dim each (q and k already rotated); out: [batch*seq, ld_out]; lse: [batch, n_heads, seq] fp32, the log2
// of each row's sum of exp2(score / sqrt(head_dim) * log2 e).
hipError_t attention_fwd(int batch, int n_heads, int seq, int head_dim, int causal, const void* qkv, long ld_qkv,
                         void* out, long ld_out, float* lse, hipStream_t s);

// Does the backward compute dq by a pass that rebuilds S and dP rather than from dS^T written to memory (for which a stage then has no
// room)?  At head_dim 64 always: the two products that the pass adds are cheap there.  At head_dim 128 by the number of workgroups of 128
// keys and the length: small grids rebuild (their workgroups can be halved, a product over 128 x 128 tiles cannot), and so do long
// sequences on many workgroups (short ones write little dS^T per workgroup); between, where the pass has an unfilled second round, dS^T is
// faster.  Time of the whole backward on dS^T over rebuilt, 1160 shapes; causal: up to 256 workgroups 1.08-1.34, 257-512 up to S 512
// 1.02-1.08; S 513-896 on 257-320 0.93-1.00, above 1.04-1.10; longer than 512 on 321-576 0.90-1.04 (B 3, H 8, S 2088 112.6 us and 119.6),
// but longer than 3072 on 321-384 0.97-1.09, 1.05 on average (B 3, H 4, S 3936 211 us and 193); longer than 768 on 577-1023 1.00-1.11;
// unmasked: up to 128 workgroups 1.24-1.40, 129-256 0.82-1.10, 257-511 0.91-1.06; S 769-1408 on 512-640 0.91-1.06 (B 4, H 16, S 1104 179.9
// us and 190.6), above 1.01-1.10; on 641-768 up to S 896 0.97, above 0.99-1.08. us, dS^T / rebuilt, dh 64: B 1, H 16, S 1024 45 / 30, B 4,
// H 12, S 1000 unmasked 82 / 73, B 2, H 24, S 2048 167 / 138, B 4, H 85, S 264 73 / 58 (unmasked 80 / 72), B 31, H 32, S 128 61 / 55, B 26,
// H 32, S 40 34 / 30, B 5, H 40, S 504 75 / 64; dh 128, 1024 workgroups: B 2, H 32, S 2048 270 / 264, B 8, H 32, S 512 131 / 135.
//
// `rotates`: dq and dk have to leave rotated back, as a stage asks for, which the rebuilt form does on the way and dS^T by one more
// launch.  The rebuilt form then is ahead on most of those grids as well: 1200 shapes with that launch; causal 257-576 workgroups above S 512
// 1.00-1.19, 577-1023 above S 768 1.09-1.29; unmasked up to 128 workgroups 1.29-1.61, 512-1023 above S 768 1.05-1.17, 129-256 above S 1024 0.85-1.06.
inline bool attn_rebuilds_dq(int batch, int n_heads, int seq, int head_dim, int causal, bool rotates) {
  const long w = (long)batch * n_heads * ((seq + 127) / 128);
  if (head_dim == 64) return true;
  if (w >= 1024) return seq > 512;
  if (rotates) return causal ? w <= 512 || seq > 768 : w <= 128 || (w >= 512 && seq > 768);
  if (!causal) return w <= 128 || (w > 768 ? seq > 768 : w > 640 ? seq > 896 : w >= 512 && seq > 1408);
  if (w <= 256) return true;
  if (seq <= 512) return w <= 512;
  return w <= 320 ? seq > 896 : w <= 384 ? seq > 3072 : w > 576 && seq > 768;
}

// Backward-p1 of the same: dq, dk, dv into the column blocks of dqkv from qkv, the forward's output and lse and the
// output derivative d_out (dense rows: ld_out == n_heads*head_dim).  delta: scratch [batch*seq, n_heads] fp32;
// ds_t: scratch of batch * n_heads * attn_ds_elems(seq) storage-type elements (receives dS^T in panels of kPanel
// queries: per (sequence, head) [ceil(seq / kPanel)][seq keys][kPanel queries]; dq is then one batched product
// dS K), or nullptr: dq is computed by a second pass over the keys that rebuilds S and dP (no dS^T anywhere), as it is
// with attn_rebuilds_dq in any case (ds_t is then not touched).  rope_table (may be null): q and k are rotated, and dq and dk
// leave rotated back (`rotates`).
hipError_t attention_p1(int batch, int n_heads, int seq, int head_dim, int causal, const void* qkv, long ld_qkv,
                        const void* out, const void* d_out, long ld_out, const float* lse, void* dqkv, long ld_dqkv,
                        float* delta, void* ds_t, const float2* rope_table, hipStream_t s);

// Register-resident MFMA loop (measurement aid): blocks x 4 waves x iters x 16 MFMAs of 32x32x16.
// seed: 8 x 64 x 8 bf16 values; sink: blocks * 256 floats.
hipError_t mfma_ceiling(int blocks, int iters, const void* seed, float* sink, hipStream_t s);

// A kernel that wants more than 64 KiB of dynamic LDS must be told so once per DEVICE (the attribute belongs to the
// kernel's image on that device).  One instance per kernel instantiation; racing threads repeat a harmless call.
struct AttrOnce {
  static constexpr int kMaxDev = 64;
  bool done[kMaxDev] = {};
  hipError_t set(const void* kern, size_t smem) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < kMaxDev && done[dev]) return hipSuccess;
    e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e == hipSuccess && dev >= 0 && dev < kMaxDev) done[dev] = true;
    return e;
  }
};

// Index behind the run of consecutive micro-batches that starts at mbs[i] and that backward-p2 contracts over in one go.
// The rows of a run are one contraction length, an int in the kernels with room for a slot beyond: longer runs are cut.
constexpr long kMaxRunRows = 1L << 30;
inline int run_end(const int* mbs, int n, int i, int tokens) {
  int j = i + 1;
  while (j < n && mbs[j] == mbs[j - 1] + 1 && (long)(j + 1 - i) * tokens <= kMaxRunRows) j++;
  return j;
}

// Limits enforced by the host before any launch.
inline int max_d_model(int dtype) { return dtype == 1 ? 8192 : 4096; }
constexpr int kMaxSeq = 4096;

}  // namespace tbp
