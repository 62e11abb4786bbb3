// Fused scaled-dot-product attention for gfx950 (bf16 storage, fp32 accumulation, head_dim 64 or 128): the forward
// keeps neither scores nor probabilities, only the log-sum-exp of every row; backward-p1 recomputes the
// probabilities from it.  Attention is one of the operations with no backward-p2 and a significant backward-p1
// (Section 4.1), so everything here is on the critical path of the pipeline.
//
// Orientation.  With the 32x32x16 MFMA an accumulator lane owns ONE column and 16 rows of a 32x32 tile.  The
// kernels arrange every product so that the softmax row statistics belong to the lane's column:
//   forward, dQ pass   S^T = K Q^T   (column = query): row max / row sum of a query are a reduction over the lane's own
//                      registers plus one exchange with lane ^ 32; the running rescale of the output is a per-lane
//                      scalar;
//   dK/dV pass         S   = Q K^T   (column = key), the statistics come from memory (one value per register row).
// In both cases the probabilities (and score gradients) leave the accumulators straight into the B operand of the next
// product: B lane (column c, half g) wants 8 contraction indices, and accumulator registers 8u .. 8u+7 of the
// lane are rows 16u + {0..3, 8..11} + 4g of its column, so k-step u of the next product simply DEFINES its
// contraction order to be that row order and the A operand is fetched in the same order (transpose reads of four
// consecutive rows at 16u + 4g and at 16u + 8 + 4g).  No shuffles, no LDS round trip for P.
#include "kernels.h"
#include "gfx950.h"

namespace tbp {

struct AttnParams {
  const bf16_t* qkv; long ld_qkv;      // [B*S, >= 3*H*DH]: q | k | v column blocks of H*DH each
  bf16_t* out; long ld_out;            // [B*S, >= H*DH]
  float* lse;                          // [B, H, S]: log2 of the row's sum of exp2(score * scale * log2 e)
  int B, H, S, causal;
  float scale_log2e;
};

// LDS image of `rows` x DH bf16, filled by asynchronous copies (a wave-wide copy writes 1 KiB = 4 or 8 rows).
// The 16-byte granule G of row r sits in slot G ^ swz(r).  swz is a bit permutation of the row index chosen so that
// both access patterns are free of bank conflicts: 16 consecutive rows at one granule (row fragments, ds_read_b128)
// and 4 consecutive rows x 2 adjacent granules (transpose fragments, ds_read_b64_tr_b16).
template <int DH>
struct HeadTile {
  static constexpr int RB = DH * 2, GPRW = DH / 8, RPC = 1024 / RB;
  static __device__ __forceinline__ int swz(int r) {
    if constexpr (DH == 128) return ((r & 3) << 1) | ((r >> 2) & 1) | (r & 8);
    else return (((r >> 1) & 1) << 1) | ((r >> 2) & 1) | (((r >> 3) & 1) << 2);
  }
  static __device__ __forceinline__ int at(int r, int G) { return r * RB + ((G ^ swz(r)) << 4); }
  // Copy plan of lane p of chunk c: tile row and byte offset inside the source row block.
  static __device__ __forceinline__ void plan(int c, int p, long ld, int& row, unsigned& goff) {
    row = RPC * c + p / GPRW;
    const int G = (p % GPRW) ^ swz(row);
    goff = (unsigned)((long)row * ld * 2 + G * 16);
  }
  // Per-lane byte offsets of the fragment reads, computed once per kernel (the swizzle makes them non-affine in the
  // k-step, so they are kept in registers; everything else - image, 32-row block, k-step pair - is an immediate).
  //   rows[s]: A-operand fragment of MFMA rows 0..31 of the image, contraction = columns 16 s .. 16 s + 15.
  //   cols[t][0/1]: A-operand fragment of the TRANSPOSED image: MFMA rows = columns 32 t .. 32 t + 31, contraction =
  //            image rows 16 u + {0..3} + 4 (lane / 32) (first read) and 16 u + 8 + {0..3} + 4 (lane / 32) (second):
  //            the accumulator row order, see the file header.  16 u rows further is an immediate too.
  struct Offsets { int rows[DH / 16]; int cols[DH / 32][2]; };
  static __device__ __forceinline__ Offsets offsets(int lane) {
    Offsets o;
#pragma unroll
    for (int s = 0; s < DH / 16; s++) o.rows[s] = at(lane & 31, 2 * s + (lane >> 5));
    const int i = lane & 15, q = (lane >> 4) & 1, g = lane >> 5;
    const int r = 4 * g + (i >> 2);
#pragma unroll
    for (int t = 0; t < DH / 32; t++) {
      const int G = 2 * (2 * t + q) + ((i & 3) >> 1);
      o.cols[t][0] = at(r, G) + 8 * (i & 1);
      o.cols[t][1] = at(r + 8, G) + 8 * (i & 1);
    }
    return o;
  }
  static __device__ __forceinline__ bf16x8 rows_frag(lds_u8* img, const Offsets& o, int r0, int s) {   // r0 % 16 == 0
    return *reinterpret_cast<LDS_AS const bf16x8*>(img + o.rows[s] + r0 * RB);
  }
  static __device__ __forceinline__ bf16x8 cols_frag(lds_u8* img, const Offsets& o, int r0, int u, int t) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<LDS_AS s16x4*>(img + o.cols[t][0] + (r0 + 16 * u) * RB));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<LDS_AS s16x4*>(img + o.cols[t][1] + (r0 + 16 * u) * RB));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
};

__device__ __forceinline__ float xor32(float v) { return __shfl_xor(v, 32, 64); }

__device__ __forceinline__ bf16x8 pack8(const f32x16& c, int u) {
  bf16x8 b;
#pragma unroll
  for (int t = 0; t < 8; t++) b[t] = (bf16_t)c[8 * u + t];
  return b;
}

// ------------------------------------------------------------------------------------------ forward
// One workgroup = 4 waves x 32 queries of one (sequence, head); keys and values stream through LDS in blocks of 64,
// double-buffered, K one block ahead of V.  Per block and wave: online softmax of S^T (64 keys x 32 queries) per lane,
// O^T += V^T P^T, and S^T of the next block.
// Bound: per block and wave 32 MFMAs of 32 clocks, about 900 clocks of vector ALU (32 exponentials at 16 clocks, the rest at
// 4), and 32 KiB of LDS reads, which two waves per SIMD turn into 2000 clocks of each.  Computing a block's scores, softmax
// and PV product one after the other, the units hardly overlapped; with the scores of the next block computed beside the
// exponentials of this one, in a pinned order, B 2, H 32, S 2048, dh 128 takes 77 us instead of 90 (S 4096, B 1: 136 for
// 162; dh 64: 46 for 57; without the causal mask: 131 for 149; calls in a row on inputs that take turns).  64 queries per wave (half the LDS reads, one wave per
// SIMD) was tried: 72 us for 53 at dh 64, spilled registers at 128.
// AHEAD = false, for sequences of at most 256 keys (four blocks): a block's own scores first, then its softmax and PV product.
// There are few next blocks to compute ahead, and the scores after the last one, which nobody uses, and a barrier more at the
// start cost more than the overlap gives.  us, ahead / not: B 32, H 32, dh 128, S 64 17.3 / 16.7, S 128 28.1 / 27.0, S 256 63.9 / 63.2;
// B 1, H 8, dh 64, S 192 5.94 / 5.62, S 256 6.80 / 6.58; beyond that either is ahead by 1-3 % up to S 512 (B 8, H 16, dh 128, S 264
// 13.0 / 13.3, S 512 19.4 / 19.7).  (Skipping the last scores by a branch in the pinned order instead: spilled registers.)
// SPLIT = 2, for grids that leave compute units idle: 64 queries per workgroup, and two waves per 32 queries, each on one
// 32-key tile of every block, whose sums meet at the end: twice the workgroups with half the chain each, for twice the copies
// per query.  (Computing scores ahead gains nothing here: 20.7 and 21.1 us at B 1, H 32, dh 128, S 1024, 11.5 and 11.0 at S 512.)
template <int DH, bool AHEAD, int SPLIT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_fwd_kernel(AttnParams p) {
  using HT = HeadTile<DH>;
  constexpr int KS = DH / 16, DT = DH / 32, BKV = 64, BQ = 128 / SPLIT, QW = 4 / SPLIT, NT = 2 / SPLIT;
  constexpr int IMG = BKV * HT::RB, SLOT = 2 * IMG;
  constexpr int NCH = IMG / 1024 / 4;                 // copies per wave per operand per block

  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  lds_u8* const lds = LDS_PTR(unsigned char, smem_raw);
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;

  const int lane = threadIdx.x & 63, ql = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // workgroup ids run over (head, sequence) fastest and query blocks slowest, longest (last) query blocks first: with
  // causal masking the work of a block grows with its index, and the blocks still to start near the end are short ones
  const int qb = (int)gridDim.y - 1 - (int)blockIdx.y;
  const int h = (int)blockIdx.x % p.H, b = (int)blockIdx.x / p.H;
  const int wq = SPLIT == 1 ? wave : wave % QW, wk = SPLIT == 1 ? 0 : wave / QW;      // which 32 queries, which 32-key tile of every block (SPLIT 2)
  const int q0 = qb * BQ, qw0 = q0 + 32 * wq, query = qw0 + ql;
  const int d = p.H * DH;
  const long tok0 = (long)b * p.S;

  const typename HT::Offsets fo = HT::offsets(lane);
  // ---- the block's query rows: copied (coalesced) into the second slot, which nothing else uses until they have been read;
  // fetched per lane they would be 32-byte pieces of 32 rows per instruction
  {
    const u32x4 dq = make_desc(p.qkv + (tok0 + q0) * p.ld_qkv + h * DH, (uint32_t)((long)(p.S - q0) * p.ld_qkv * 2));
#pragma unroll
    for (int i = 0; i < 2 * NCH / SPLIT; i++) {
      int row; unsigned go;
      HT::plan(wave + 4 * i, lane, p.ld_qkv, row, go);
      dma16(lds0 + SLOT + (wave + 4 * i) * 1024, dq, q0 + row < p.S ? go : kOob);
    }
  }
  // ---- copy plan of this wave: chunks wave, wave + 4, ... of the K image and of the V image
  int c_row[NCH];
  unsigned c_off[NCH];
#pragma unroll
  for (int i = 0; i < NCH; i++) HT::plan(wave + 4 * i, lane, p.ld_qkv, c_row[i], c_off[i]);
  const int kv_end = p.causal ? (q0 + BQ < p.S ? q0 + BQ : p.S) : p.S;
  const int nblk = (kv_end + BKV - 1) / BKV;
  auto issue = [&](int j, int which) {      // which: 0 the K image, 1 the V image of block j
    const int kv0 = j * BKV;
    const bf16_t* src = p.qkv + (tok0 + kv0) * p.ld_qkv + (which ? 2 * d : d) + h * DH;
    const u32x4 desc = make_desc(src, (uint32_t)((long)(p.S - kv0) * p.ld_qkv * 2));      // rows of this sequence only
    const uint32_t base = lds0 + (j & 1) * SLOT + which * IMG + wave * 1024;
#pragma unroll
    for (int i = 0; i < NCH; i++) dma16(base + i * 4096, desc, (kv0 + c_row[i] < p.S) ? c_off[i] : kOob);
  };

  f32x16 ot[DT];
#pragma unroll
  for (int t = 0; t < DT; t++)
#pragma unroll
    for (int e = 0; e < 16; e++) ot[t][e] = 0.f;
  // m: reference point of the row's exponentials (the same in both lane halves); l: this lane half's share of the row sum
  float m = -INFINITY, l[2] = {0.f, 0.f};

  issue(0, 0);
  issue(0, 1);
  wait_vmem<0>();
  __syncthreads();
  // ---- this lane's query row as B operand of S^T = K Q^T: 8 consecutive head-dim values per k-step
  bf16x8 qf[KS];
#pragma unroll
  for (int s = 0; s < KS; s++) qf[s] = HT::rows_frag(lds + SLOT, fo, 32 * wq, s);
  f32x16 sa[NT], sb[NT];               // S^T of the block whose softmax is in work, and of the next one
  const int wk_rows = 32 * wk * HT::RB;          // (SPLIT 2: this wave's tile of the K and V images)
  auto scores = [&](f32x16 (&st)[NT], lds_u8* kimg) {
#pragma unroll
    for (int kt = 0; kt < NT; kt++)
#pragma unroll
      for (int e = 0; e < 16; e++) st[kt][e] = 0.f;
#pragma unroll
    for (int s = 0; s < KS; s++)
#pragma unroll
      for (int kt = 0; kt < NT; kt++)
        st[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(HT::rows_frag(kimg, fo, 32 * kt, s), qf[s], st[kt], 0, 0, 0);
  };
  if constexpr (AHEAD) {
    scores(sa, lds + wk_rows);
    __syncthreads();                   // every wave has its query row: the second slot is free
    if (nblk > 1) issue(1, 0);
  }

  // Block j: softmax of its scores (st) and O^T += V^T P^T, with the scores of block j + 1 (nx) computed on the way.
  // The order of the instructions is pinned: the MFMAs of the next block's scores and the first three quarters of the PV
  // MFMAs each carry a share of the exponentials, so that the matrix pipe and the vector ALU work side by side.
  auto block = [&](f32x16 (&st)[NT], f32x16 (&nx)[NT], int j) {
    wait_vmem<0>();
    __syncthreads();                   // K of block j + 1 and V of block j have landed; every wave is done with block j - 1
    if (AHEAD ? j + 2 < nblk : j + 1 < nblk) issue(AHEAD ? j + 2 : j + 1, 0);      // (not AHEAD: K of block j has landed)
    if (j + 1 < nblk) issue(j + 1, 1);
    const int kv0 = j * BKV + 32 * wk;
    if (p.causal && kv0 > qw0 + 31) return;            // every key of the block is after every query of this wave
    if (SPLIT == 2 && kv0 >= p.S) return;              // no key at all (and so none in any later block)
    lds_u8* const kimg = lds + ((j + 1) & 1) * SLOT + wk_rows;   // (after the last block: an older one, whose scores nobody uses)
    lds_u8* const vimg = lds + (j & 1) * SLOT + IMG + wk_rows;
    bf16x8 kf[2][NT];
    if constexpr (AHEAD) {
#pragma unroll
      for (int s = 0; s < 2; s++)
#pragma unroll
        for (int kt = 0; kt < NT; kt++) kf[s][kt] = HT::rows_frag(kimg, fo, 32 * kt, s);
    } else {
      scores(st, lds + (j & 1) * SLOT + wk_rows);
    }
    // keys beyond the query (causal) or beyond the sequence do not take part (blocks on the diagonal / at the end only)
    if ((p.causal && kv0 + 32 * NT - 1 > qw0) || kv0 + 32 * NT > p.S) {
      const int last = p.causal ? (query < p.S - 1 ? query : p.S - 1) : p.S - 1;      // last key this lane's query sees
      const int rel = last - kv0 - 4 * g;
#pragma unroll
      for (int kt = 0; kt < NT; kt++)
#pragma unroll
        for (int e = 0; e < 16; e++)
          st[kt][e] = (32 * kt + 8 * (e >> 2) + (e & 3) > rel) ? -INFINITY : st[kt][e];
    }
    // The reference point m of the exponentials only has to stay within a safe distance of the running maximum, not
    // on it: o / l and lse = m + log2 l are the same for any m.  It is moved (and what is accumulated rescaled) only
    // when some query's maximum has risen by more than kSlack octaves above it; until then p <= 2^kSlack, far inside
    // the range of fp32 sums and of the storage type.  With the maximum itself as reference nearly every block moves
    // some lane's maximum and pays 16 * DT multiplications per lane; this way typically only the first block does, and
    // the two halves of a row need not exchange their maxima to find out.
    constexpr float kSlack = 8.f;
    float mx = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < NT; kt++)
#pragma unroll
      for (int e = 0; e < 16; e++) mx = fmaxf(mx, st[kt][e]);
    mx *= p.scale_log2e;                                // scale > 0: the maximum commutes with it
    if (__any(mx > m + kSlack)) {
      const float mnew = fmaxf(m, fmaxf(mx, xor32(mx)));
      // First block: m = -inf, exp2(-inf) = 0.  (SPLIT 2: so also for a lane that is here because of its neighbours while its own
      // query's keys have all scored -inf so far: -inf - -inf would make NaN of the zeros that it holds.)
      const float alpha = __builtin_amdgcn_exp2f(m - (SPLIT == 2 && mnew == -INFINITY ? 0.f : mnew));
      l[0] *= alpha;
      l[1] *= alpha;
#pragma unroll
      for (int t = 0; t < DT; t++)
#pragma unroll
        for (int e = 0; e < 16; e++) ot[t][e] *= alpha;
      m = mnew;
    }
    // (SPLIT 2: a wave whose keys have all scored -inf so far has no reference point yet, and the query's other wave may: zeros)
    const float ref = SPLIT == 2 && m == -INFINITY ? 0.f : m;
    bf16x8 pb[2 * NT], vf[DT];
    auto elements = [&](int e0, int e1) {               // exponentials of elements e0 .. e1 - 1 of the lane's 16 NT
#pragma unroll
      for (int e = e0; e < e1; e++) {
        const float pe = __builtin_amdgcn_exp2f(__builtin_fmaf(st[e >> 4][e & 15], p.scale_log2e, -ref));
        st[e >> 4][e & 15] = pe;
        l[e & 1] += pe;
        if (e % 8 == 7) pb[e >> 3] = pack8(st[e >> 4], (e >> 3) & 1);
      }
    };
    // MFMAs of the scores; elements done beside them, the rest beside all PV k-steps but the last
    constexpr int NA = NT * KS, NE = 16 * NT, EA = NT == 2 ? 18 : 10, PK = 2 * NT, PE = PK - 1;
    static_assert(EA >= 8 && EA + (NE - EA) / PE >= 16 && (NT == 1 || EA + (NE - EA) * 2 / PE >= 24), "P must be ready in time");
    if constexpr (AHEAD) {
#pragma unroll
      for (int kt = 0; kt < NT; kt++)
#pragma unroll
        for (int e = 0; e < 16; e++) nx[kt][e] = 0.f;
    }
    __builtin_amdgcn_s_setprio(1);             // (the SIMD's other wave fills in: 1-4 % faster than without)
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (AHEAD) {
#pragma unroll
      for (int i = 0; i < NA; i++) {
        const int s = i / NT, kt = i % NT;
        nx[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s & 1][kt], qf[s], nx[kt], 0, 0, 0);
        if (s + 2 < KS) kf[s & 1][kt] = HT::rows_frag(kimg, fo, 32 * kt, s + 2);
        if (i >= NA - DT) vf[i - (NA - DT)] = HT::cols_frag(vimg, fo, 0, 0, i - (NA - DT));
        elements(EA * i / NA, EA * (i + 1) / NA);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll
      for (int t = 0; t < DT; t++) vf[t] = HT::cols_frag(vimg, fo, 0, 0, t);
      elements(0, EA);
    }
#pragma unroll
    for (int i = 0; i < PK * DT; i++) {
      const int ku = i / DT, t = i % DT;
      ot[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[t], pb[ku], ot[t], 0, 0, 0);
      if (ku < PE) vf[t] = HT::cols_frag(vimg, fo, 32 * ((ku + 1) >> 1), (ku + 1) & 1, t);
      if (ku < PE) elements(EA + (NE - EA) * i / (PE * DT), EA + (NE - EA) * (i + 1) / (PE * DT));
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_setprio(0);
  };
  for (int j = 0; j < nblk; j += 2) {
    block(sa, sb, j);
    if (j + 1 < nblk) block(sb, sa, j + 1);
  }

  // ---- o = O^T / l, transposed back on the way out.  A lane holds 4 consecutive head-dim values of its query per
  // register group (8 bytes, 32 rows per instruction if stored directly): each wave passes its rows through LDS
  // (free after one more barrier; rows padded to DH * 2 + 16 bytes against bank conflicts) and writes them
  // whole, 16 bytes per lane.
  __syncthreads();
  constexpr int EROW = DH * 2 + 16;
  static_assert(BQ * EROW <= 2 * SLOT, "the output tile must fit in the ring");
  lds_u8* const erow = lds + 32 * wq * EROW;
  float lq = (l[0] + l[1]) + xor32(l[0] + l[1]);
  if constexpr (SPLIT == 2) {
    // the two waves of a query: what the second one summed, brought to the common reference point, joins the first one's.
    // (A wave that saw no key of the query, or only such as score -inf, has m = -inf and zeros, and adds nothing.)
    static_assert(BQ * EROW + 1024 <= SLOT && QW * DT * 4096 <= SLOT, "output tile, statistics and partial sums side by side");
    LDS_AS float* const part = reinterpret_cast<LDS_AS float*>(lds + SLOT) + wq * (DT * 1024);
    LDS_AS float* const stat = reinterpret_cast<LDS_AS float*>(lds + BQ * EROW) + wq * 128;
    if (wk == 1) {
#pragma unroll
      for (int t = 0; t < DT; t++)
#pragma unroll
        for (int e = 0; e < 16; e++) part[(t * 16 + e) * 64 + lane] = ot[t][e];
      stat[lane] = m;
      stat[64 + lane] = lq;
    }
    __syncthreads();
    if (wk == 1) return;
    const float m1 = stat[lane], mc = fmaxf(m, m1);
    const float f0 = __builtin_amdgcn_exp2f(m - mc), f1 = __builtin_amdgcn_exp2f(m1 - mc);
    m = mc;
    lq = lq * f0 + stat[64 + lane] * f1;
#pragma unroll
    for (int t = 0; t < DT; t++)
#pragma unroll
      for (int e = 0; e < 16; e++) ot[t][e] = ot[t][e] * f0 + part[(t * 16 + e) * 64 + lane] * f1;
  }
  {
    const float inv = 1.f / lq;
#pragma unroll
    for (int t = 0; t < DT; t++)
#pragma unroll
      for (int e4 = 0; e4 < 4; e4++) {
        bf16x4 v;
#pragma unroll
        for (int r = 0; r < 4; r++) v[r] = (bf16_t)(ot[t][4 * e4 + r] * inv);
        *reinterpret_cast<LDS_AS bf16x4*>(erow + ql * EROW + (32 * t + 8 * e4 + 4 * g) * 2) = v;
      }
    if (g == 0 && query < p.S) p.lse[((long)b * p.H + h) * p.S + query] = m + __builtin_amdgcn_logf(lq);
  }
  {  // (LDS operations of a wave execute in order: the reads below see this wave's own writes above)
    constexpr int LPR = DH / 8, RPI = 64 / LPR;
    const int rl = lane / LPR, piece = lane % LPR;
#pragma unroll
    for (int r0 = 0; r0 < 32; r0 += RPI) {
      const int qrow = qw0 + r0 + rl;
      if (qrow < p.S)
        *reinterpret_cast<u32x4*>(p.out + (tok0 + qrow) * p.ld_out + h * DH + 8 * piece) =
            *reinterpret_cast<const LDS_AS u32x4*>(erow + (r0 + rl) * EROW + 16 * piece);
    }
  }
}

// ------------------------------------------------------------------------------------------ backward-p1: dK, dV, dS^T
// One workgroup = 128 keys of one (sequence, head), 32 per wave pair; queries, their output derivatives and their row
// statistics stream through LDS in steps of 64 queries, three steps deep.  Per 32 queries and wave pair:
//   S = Q K^T and dP = dO V^T (column = key; K and V rows of the lane's key stay in registers as B operands),
//   P = exp2(S c - lse), dS = P (dP - delta), then dV^T += dO^T P and dK^T += Q^T dS with P and dS fed from the
//   accumulators (see the file header).  dS^T is also written out ([key][query], storage type): dQ = dS K is a
//   contraction over keys, which this kernel splits over workgroups, and is left to a batched product.
struct AttnBwdParams {
  const bf16_t* qkv; long ld_qkv;
  const bf16_t* dout; long ld_do;      // [B*S, >= H*DH] derivative of the attention output
  const float* lse;                    // [B, H, S] from the forward
  const float* delta;                  // [B*S, H]: rowsum(dout * out) per (token, head)
  bf16_t* dqkv; long ld_dqkv;          // dk and dv blocks are written (columns H*DH.. and 2*H*DH..)
  const float2* rope;                  // rotation table [S][DH / 2]: dk is rotated back; or nullptr
  bf16_t* dst;                         // dS^T per (b, h) in panels of 128 queries: [ceil(S / 128)][S keys][128 queries]
  int B, H, S, causal;
  float scale, scale_log2e;
};

// The two kinds of work run on different waves.  A single wave issues in order: while it works through the ~200 vector
// instructions that turn S and dP into P and dS, the matrix pipe of its SIMD idles, and the other way round (a
// single-wave form of this kernel, software-pipelined three tiles deep, kept the matrix pipe 27 % busy and was 5 %
// slower).  A workgroup is 8 waves, two per SIMD, of which
//   waves 0..3 ("left")   compute S = Q K^T and dP = dO V^T for their 32 keys, then P and dS, write dS^T out and hand
//                         P and dS (already in B-operand form, 64 bytes per lane) over through LDS;
//   waves 4..7 ("right")  take P and dS of the previous tile from LDS and accumulate dV^T += dO^T P, dK^T += Q^T dS.
// The hardware interleaves the two instruction streams of a SIMD, so the vector work of one tile runs under the MFMAs
// of its neighbours.  One workgroup barrier per 32-query tile; the hand-over buffers and the query-step images are
// double / triple buffered so that neither side ever waits for the other beyond that barrier.  The right waves also
// issue all asynchronous copies (they have no other vector-memory operations, so their copy counter is exact).
// KEYS = 64, for grids that leave compute units idle: two left waves per 32 keys, each on one tile of a 64-query step, and the
// right waves take both tiles per iteration: half the iterations per workgroup, twice the workgroups (and the transposed
// fragments of Q and dO, read for half the keys, weigh twice as much: about 10 % slower per key and query).
// ROPE is fixed at compile time: a branch on the table in the stores kept the reads of a row from overlapping the stores of the one
// before, 185 us instead of 181 at B 2, H 32, S 2048, dh 128 without a table, and 123.6 instead of 120.7 in the dq pass.
template <int DH, bool WRITE_DST, int KEYS, bool ROPE>
__global__ __launch_bounds__(512) void attn_bwd_kv_split_kernel(AttnBwdParams p) {
  using HT = HeadTile<DH>;
  constexpr int KS = DH / 16, DT = DH / 32, BQ = 64;
  constexpr int IMG = BQ * HT::RB, SLOT = 2 * IMG + 1024;     // Q image, dO image, 64 x (lse, delta); three slots
  constexpr int NCH = IMG / 1024 / 4;                         // copies per right wave and image
  constexpr int OPS = 2 * NCH + 1;                            // vector-memory operations of one issue(), per right wave
  constexpr int HAND = 4 * 4096;                              // one hand-over buffer: 4 wave pairs x 64 lanes x 64 bytes
  constexpr int HALF = 32 * HT::RB;                           // the second tile's rows inside an image
  constexpr int KB = KEYS / 32, TPI = 4 / KB;                 // 32-key blocks of the workgroup; 32-query tiles per iteration
  static_assert((KEYS == 128 || KEYS == 64) && !(WRITE_DST && KEYS != 128), "key block");

  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  lds_u8* const lds = LDS_PTR(unsigned char, smem_raw);
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
  lds_u8* const hand = lds + 3 * SLOT;

  const int tid = threadIdx.x, lane = tid & 63, kl = lane & 31, g = lane >> 5;
  const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int right = wave8 >> 2, wave = wave8 & 3;             // role, and which 32 keys of the block
  const int kb = blockIdx.y;
  const int kblk = KB == 4 ? wave : wave % KB, tq_left = KB == 4 ? 0 : wave / KB;      // a left wave's 32 keys, and which tile of an iteration
  const int h = (int)blockIdx.x % p.H, b = (int)blockIdx.x / p.H;
  const int kv0 = kb * KEYS, kw0 = kv0 + 32 * kblk, key = kw0 + kl;
  const int d = p.H * DH;
  const long tok0 = (long)b * p.S;
  const long bh = (long)b * p.H + h;
  const typename HT::Offsets fo = HT::offsets(lane);
  const int step0 = p.causal ? kv0 / BQ : 0;                  // queries before the first key of the block see none of it
  const int nstep = (p.S + BQ - 1) / BQ;
  const int t0 = 2 * step0, nt = 2 * (nstep - step0) / TPI;   // first tile, number of iterations
  typedef LDS_AS float lds_f32;
  lds_u8* const my_hand = hand + wave * 4096 + lane * 16;     // + buffer * HAND + 1024 * {p0, p1, s0, s1}
  constexpr int KVIMG = KEYS * HT::RB;                        // image of the block's K (then V) rows
  lds_u8* const kvimg = lds + 2 * SLOT;
  static_assert(2 * KVIMG <= SLOT + 2 * HAND, "K and V images must fit in the third slot plus the hand-over area");

  if (!right) {
    // ------------------------------------------------------------------ left: S, dP, P, dS, dS^T out
    bf16x8 kfb[KS], vfb[KS];
    const long ds_elems = (long)attn_ds_elems(p.S);
    const u32x4 rst = make_desc(p.dst + bh * ds_elems, (uint32_t)(ds_elems * 2));
    // The tiles of dS^T (32 keys x 32 queries each) leave through a per-wave LDS buffer that collects the two tiles of a
    // 64-query step (rows padded to 144 bytes against bank conflicts): a lane holds 4 consecutive queries of its key row
    // per register group, which stored directly is 8 bytes per lane and 32 rows per instruction; read back row-major
    // after the second tile it is 16 bytes per lane and 128 contiguous bytes (a whole cache line of the panel) per key row.
    constexpr int STG_ROW = 144;
    lds_u8* const stg = hand + 2 * HAND + wave * (32 * STG_ROW);
    lds_u8* const stg_wr = stg + kl * STG_ROW + 8 * g;          // + 64 (tile & 1) + 16 e4
    unsigned st_row[4];
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int row = (lane + 64 * r) >> 3;
      st_row[r] = kw0 + row < p.S ? (unsigned)(((kw0 + row) * kPanel + 8 * (lane & 7)) * 2) : kOob;
    }
    __syncthreads();                                          // steps step0, step0 + 1 and the K / V rows have landed
    // the lane's key row and value row as B operands (8 consecutive head-dim values per k-step), from the images the
    // right waves copied into the third slot and the hand-over area, which nothing else uses yet
#pragma unroll
    for (int s = 0; s < KS; s++) {
      kfb[s] = HT::rows_frag(kvimg, fo, 32 * kblk, s);
      vfb[s] = HT::rows_frag(kvimg + KVIMG, fo, 32 * kblk, s);
    }
    __syncthreads();                                          // every left wave has its rows: the area is free again
    for (int it = 0; it <= nt; it++) {
      if (it < nt) {
        const int tile = t0 + TPI * it + tq_left, qt0 = tile * 32;
        lds_u8* const slot = lds + (((tile >> 1) - step0) % 3) * SLOT;
        lds_u8* const qimg = slot + (tile & 1) * HALF;
        lds_u8* const dimg = qimg + IMG;
        const lds_f32* const stat = reinterpret_cast<const lds_f32*>(slot + 2 * IMG) + 32 * (tile & 1);
        f32x16 sa, da;
#pragma unroll
        for (int e = 0; e < 16; e++) { sa[e] = 0.f; da[e] = 0.f; }
        // The order is pinned: left to itself the compiler fetches a fragment right before the MFMA that wants it, and
        // the latency of the LDS is then paid at every one of the KS steps.
        constexpr int PF = KS < 4 ? KS : 4;
        bf16x8 fq[KS], fd[KS];
        f32x4 ls[4], dl[4];
#pragma unroll
        for (int s = 0; s < PF; s++) { fq[s] = HT::rows_frag(qimg, fo, 0, s); fd[s] = HT::rows_frag(dimg, fo, 0, s); }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < KS; s++) {
          if (s + PF < KS) { fq[s + PF] = HT::rows_frag(qimg, fo, 0, s + PF); fd[s + PF] = HT::rows_frag(dimg, fo, 0, s + PF); }
          if (s >= KS - 4) {
            const int e4 = s - (KS - 4);
            ls[e4] = *reinterpret_cast<const LDS_AS f32x4*>(stat + 8 * e4 + 4 * g);
            dl[e4] = *reinterpret_cast<const LDS_AS f32x4*>(stat + BQ + 8 * e4 + 4 * g);
          }
          sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fq[s], kfb[s], sa, 0, 0, 0);
          da = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fd[s], vfb[s], da, 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
        // register e of the tile is query qt0 + 8 (e / 4) + 4 g + e % 4.  Only a tile on the diagonal has a query before
        // one of the wave's keys: the others skip the two instructions per element of the comparison.
        float pv[16], sv[16];
#pragma unroll
        for (int e = 0; e < 16; e++) pv[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sa[e], p.scale_log2e, -ls[e >> 2][e & 3]));
        if (p.causal && qt0 < kw0 + 31) {
          const int rel = key - qt0 - 4 * g;
#pragma unroll
          for (int e = 0; e < 16; e++) pv[e] = (8 * (e >> 2) + (e & 3) < rel) ? 0.f : pv[e];
        }
#pragma unroll
        for (int e = 0; e < 16; e++) sv[e] = pv[e] * (da[e] - dl[e >> 2][e & 3]);
        bf16x8 kp[2], ks[2];
#pragma unroll
        for (int u = 0; u < 2; u++)
#pragma unroll
          for (int t = 0; t < 8; t++) { kp[u][t] = (bf16_t)pv[8 * u + t]; ks[u][t] = (bf16_t)sv[8 * u + t]; }
        lds_u8* const out = my_hand + ((TPI == 1 ? tile : it) & 1) * HAND;      // (the same parity; by `it` the loops of KEYS 128 ran 3 % slower)
        *reinterpret_cast<LDS_AS bf16x8*>(out) = kp[0];
        *reinterpret_cast<LDS_AS bf16x8*>(out + 1024) = kp[1];
        *reinterpret_cast<LDS_AS bf16x8*>(out + 2048) = ks[0];
        *reinterpret_cast<LDS_AS bf16x8*>(out + 3072) = ks[1];
        // dS^T out: the two halves of each packed k-step are four consecutive queries of the lane's key row.  Nobody
        // reads it before the kernel ends, so the stores go out untracked: the barrier below must not wait for them
        // (tracked, their acknowledgements cost a quarter of the kernel's time).
        const u32x4 s0 = __builtin_bit_cast(u32x4, ks[0]), s1 = __builtin_bit_cast(u32x4, ks[1]);
        const u32x2 dsv[4] = {u32x2{s0[0], s0[1]}, u32x2{s0[2], s0[3]}, u32x2{s1[0], s1[1]}, u32x2{s1[2], s1[3]}};
        if constexpr (WRITE_DST) {
#pragma unroll
          for (int e4 = 0; e4 < 4; e4++) *reinterpret_cast<LDS_AS u32x2*>(stg_wr + 64 * (tile & 1) + 16 * e4) = dsv[e4];
        }
        // (LDS operations of a wave execute in order: the reads below see the writes above and those of the tile before)
        if (WRITE_DST && (tile & 1)) {
          const int qe = qt0 - 32;                              // first query of the step; the step lies inside one panel
          const long pan = ((long)(qe / kPanel) * p.S * kPanel + qe % kPanel) * 2;
#pragma unroll
          for (int r = 0; r < 4; r++) {
            const int idx = lane + 64 * r;
            const u32x4 v = *reinterpret_cast<const LDS_AS u32x4*>(stg + (idx >> 3) * STG_ROW + 16 * (idx & 7));
            store16_async(v, rst, qe + 8 * (lane & 7) < p.S ? st_row[r] : kOob, (uint32_t)__builtin_amdgcn_readfirstlane((int)pan));
          }
        }
      }
      __syncthreads();
    }
    __syncthreads();                                          // every right wave's copies have landed: the ring is free
    __syncthreads();                                          // the right waves have put dK and dV into LDS (below)
    return;
  }

  // -------------------------------------------------------------------- right: copies, dV^T, dK^T
  int c_row[NCH];
  unsigned cq_off[NCH], cd_off[NCH];
#pragma unroll
  for (int i = 0; i < NCH; i++) {
    HT::plan(wave + 4 * i, lane, p.ld_qkv, c_row[i], cq_off[i]);
    HT::plan(wave + 4 * i, lane, p.ld_do, c_row[i], cd_off[i]);
  }
  // Every call issues exactly OPS operations per wave (steps past the end write zeros into their slot and fetch
  // nothing), so a wait for "all but the last issue" is a fixed count.
  auto issue = [&](int i) {
    const int q0 = i * BQ;
    const bool live = i < nstep;
    const uint32_t slot = lds0 + ((i - step0) % 3) * SLOT;      // slots count from the block's first step
    const int qs = live ? q0 : 0;
    const u32x4 dq = make_desc(p.qkv + (tok0 + qs) * p.ld_qkv + h * DH, (uint32_t)((long)(p.S - qs) * p.ld_qkv * 2));
    const u32x4 dd = make_desc(p.dout + (tok0 + qs) * p.ld_do + h * DH, (uint32_t)((long)(p.S - qs) * p.ld_do * 2));
#pragma unroll
    for (int c = 0; c < NCH; c++) {
      const bool ok = live && q0 + c_row[c] < p.S;
      dma16(slot + wave * 1024 + c * 4096, dq, ok ? cq_off[c] : kOob);
      dma16(slot + IMG + wave * 1024 + c * 4096, dd, ok ? cd_off[c] : kOob);
    }
    // row statistics: wave 0 fetches lse[0..63], wave 1 delta[0..63]; waves 2 and 3 issue the same instruction out of
    // range (nothing moves) to keep the count uniform.  Their 256 bytes land behind the two statistics rows.
    const int q = q0 + lane;
    const u32x4 ds = (wave & 1) == 0 ? make_desc(p.lse + bh * p.S, (uint32_t)(p.S * 4))
                                     : make_desc(p.delta + tok0 * p.H + h, (uint32_t)(((long)(p.S - 1) * p.H + 1) * 4));
    const unsigned off = (live && wave < 2 && q < p.S) ? (unsigned)((wave & 1) == 0 ? q * 4 : (long)q * p.H * 4) : kOob;
    dma4(slot + 2 * IMG + wave * 256, ds, off);
  };
  // A right wave owns 32 head-dim columns (its index) of dV^T and dK^T for all four key blocks of the workgroup: it then
  // reads only its quarter of the Q and dO tiles as transposed fragments (the expensive reads) and all four left waves'
  // P and dS (cheap, lane-contiguous).  With head_dim 64 waves 2 and 3 have no columns and only copy.
  f32x16 dvt[KB], dkt[KB];
#pragma unroll
  for (int t = 0; t < KB; t++)
#pragma unroll
    for (int e = 0; e < 16; e++) { dvt[t][e] = 0.f; dkt[t][e] = 0.f; }
  const bool has_cols = wave < DT;
  int col0 = 0, col1 = 0;                                     // fragment offsets of this wave's column block
#pragma unroll
  for (int t = 0; t < DT; t++)
    if (t == wave) { col0 = fo.cols[t][0]; col1 = fo.cols[t][1]; }
  auto my_cols = [&](lds_u8* img, int u) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<LDS_AS s16x4*>(img + col0 + 16 * u * HT::RB));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<LDS_AS s16x4*>(img + col1 + 16 * u * HT::RB));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  {  // the block's K and V rows, for the left waves (coalesced here; fetched per lane they are 32-byte pieces of 32 rows)
    const bf16_t* kb0 = p.qkv + (tok0 + kv0) * p.ld_qkv + d + h * DH;
    const uint32_t bytes = (uint32_t)((long)(p.S - kv0) * p.ld_qkv * 2);
    const u32x4 dk = make_desc(kb0, bytes), dv = make_desc(kb0 + d, bytes);
#pragma unroll
    for (int i = 0; i < NCH * KEYS / 64; i++) {
      int row; unsigned go;
      HT::plan(wave + 4 * i, lane, p.ld_qkv, row, go);
      const unsigned off = kv0 + row < p.S ? go : kOob;
      dma16(lds0 + 2 * SLOT + (wave + 4 * i) * 1024, dk, off);
      dma16(lds0 + 2 * SLOT + KVIMG + (wave + 4 * i) * 1024, dv, off);
    }
  }
  issue(step0);
  issue(step0 + 1);
  wait_vmem<0>();
  __syncthreads();
  __syncthreads();                                            // the left waves have read their K and V rows
  for (int it = 0; it <= nt; it++) {
    const int tp = t0 + TPI * it;                             // the (first) tile the left waves are on
    if (it > 0 && has_cols) {
#pragma unroll
      for (int tq = 0; tq < TPI; tq++) {
        const int tile = tp - TPI + tq;
        lds_u8* const qimg = lds + (((tile >> 1) - step0) % 3) * SLOT + (tile & 1) * HALF;
        lds_u8* const dimg = qimg + IMG;
        // this wave's 32 head-dim columns of dO^T and Q^T (two k-steps of 16 queries), then every key block's P and dS, each
        // fetched one key block ahead of its MFMAs (pinned, as on the left)
        bf16x8 fo_d[2], fo_q[2], kp[2][2], ks[2][2];
        const lds_u8* const in = hand + ((TPI == 1 ? tile : it - 1) & 1) * HAND + tq * (KB * 4096) + lane * 16;
        auto fetch = [&](int kbk) {
#pragma unroll
          for (int u = 0; u < 2; u++) {
            kp[kbk & 1][u] = *reinterpret_cast<const LDS_AS bf16x8*>(in + kbk * 4096 + 1024 * u);
            ks[kbk & 1][u] = *reinterpret_cast<const LDS_AS bf16x8*>(in + kbk * 4096 + 2048 + 1024 * u);
          }
        };
#pragma unroll
        for (int u = 0; u < 2; u++) { fo_d[u] = my_cols(dimg, u); fo_q[u] = my_cols(qimg, u); }
        fetch(0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kbk = 0; kbk < KB; kbk++) {
          if (kbk + 1 < KB) fetch(kbk + 1);
#pragma unroll
          for (int u = 0; u < 2; u++) {
            dvt[kbk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fo_d[u], kp[kbk & 1][u], dvt[kbk], 0, 0, 0);
            dkt[kbk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fo_q[u], ks[kbk & 1][u], dkt[kbk], 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    if constexpr (TPI == 1) {
      // Step (tp + 1) / 2 + 1 is what the left waves start two barriers from now, when tp is odd: it was issued three
      // barriers ago and only the issue after it may still be in flight
      if (tp & 1) wait_vmem<OPS>();
      __syncthreads();
      // after this barrier nobody reads the step before tp / 2 any more (tp even): its slot takes step tp / 2 + 2
      if (!(tp & 1)) issue((tp >> 1) + 2);
    } else {
      // a whole step per iteration: the one after the left waves' was issued behind the barrier before, and the one before
      // it, which the right waves have just finished, leaves its slot to the step after next
      wait_vmem<0>();
      __syncthreads();
      issue(step0 + it + 2);
    }
  }
  wait_vmem<0>();                                             // (copies past the end: zeros, no traffic)
  __syncthreads();                                            // ... of every wave, before the ring is reused below

  // ---- dk = scale * dK^T transposed, dv = dV^T transposed.  A lane holds 4 consecutive head-dim values of one key per
  // register group; stored directly that is 8 bytes per lane scattered over 32 rows per instruction, and the 64 MB of
  // dK and dV of a launch then cost a tenth of the kernel's time.  The waves put their column blocks together in LDS
  // (the copy ring is free by now; rows padded to 272 bytes against bank conflicts) and each writes 32 whole key
  // rows, 16 bytes per lane, 256 contiguous bytes per row.
  constexpr int EROW = DH * 2 + 16;
  lds_u8* const edk = lds;
  lds_u8* const edv = lds + KEYS * EROW;
  static_assert(2 * KEYS * EROW <= 3 * SLOT, "dK and dV tiles must fit in the ring");
  if (has_cols) {
#pragma unroll
    for (int kbk = 0; kbk < KB; kbk++)
#pragma unroll
      for (int e4 = 0; e4 < 4; e4++) {
        bf16x4 vk, vv;
#pragma unroll
        for (int r = 0; r < 4; r++) { vk[r] = (bf16_t)(dkt[kbk][4 * e4 + r] * p.scale); vv[r] = (bf16_t)dvt[kbk][4 * e4 + r]; }
        const int off = (32 * kbk + kl) * EROW + (32 * wave + 8 * e4 + 4 * g) * 2;
        *reinterpret_cast<LDS_AS bf16x4*>(edk + off) = vk;
        *reinterpret_cast<LDS_AS bf16x4*>(edv + off) = vv;
      }
  }
  __syncthreads();
  {
    constexpr int LPR = DH / 8, RPI = 64 / LPR;               // lanes per row, rows per wave-wide store
    const int rl = lane / LPR, piece = lane % LPR;
#pragma unroll
    for (int r0 = 0; r0 < KEYS / 4; r0 += RPI) {
      const int row = KEYS / 4 * wave + r0 + rl;              // this wave's quarter of the key rows
      const int krow = kv0 + row;
      if (krow < p.S) {
        bf16_t* const out = p.dqkv + (tok0 + krow) * p.ld_dqkv + d + h * DH + 8 * piece;
        bf16x8 vk = *reinterpret_cast<const LDS_AS bf16x8*>(edk + row * EROW + 16 * piece);
        if constexpr (ROPE) {                                 // rotated back: the other half of the row is in LDS as well
          const bf16x8 other = *reinterpret_cast<const LDS_AS bf16x8*>(edk + row * EROW + 16 * (piece ^ (LPR / 2)));
          const float2* const tb = p.rope + (long)krow * (DH / 2) + 8 * (piece & (LPR / 2 - 1));
          const float sgn = piece < LPR / 2 ? 1.f : -1.f;
#pragma unroll
          for (int i = 0; i < 8; i += 2) {
            const f32x4 cs = *reinterpret_cast<const f32x4*>(tb + i);
            vk[i] = (bf16_t)((float)vk[i] * cs[0] + sgn * cs[1] * (float)other[i]);
            vk[i + 1] = (bf16_t)((float)vk[i + 1] * cs[2] + sgn * cs[3] * (float)other[i + 1]);
          }
        }
        *reinterpret_cast<bf16x8*>(out) = vk;
        *reinterpret_cast<u32x4*>(out + d) = *reinterpret_cast<const LDS_AS u32x4*>(edv + row * EROW + 16 * piece);
      }
    }
  }
}

// ------------------------------------------------------------------------------------------ backward-p1: dQ
// dQ = scale * dS K is a contraction over keys.  This pass is oriented like the forward (S^T = K Q^T: a lane owns one
// query, so lse and delta of the row are per-lane scalars): per block of 64 keys it recomputes S^T and dP^T = V dO^T,
// forms P^T = exp2(S^T c - lse) and dS^T = P^T (dP^T - delta) in the accumulators and feeds dS^T straight into
// dQ^T += K^T dS^T (the B-operand trick of the file header), accumulating dQ^T in registers over all key blocks.
// Three products per tile instead of one, but no dS^T is written to or read from memory, nothing is added
// atomically, and the result is bit-reproducible.  Workgroup = 4 waves x 32 queries, K and V blocks double-buffered
// through LDS exactly as in the forward; SPLIT = 2 as there.
// It runs before the pass over the queries, because it has a query's rows of dout in registers: delta = rowsum(dout * out) costs
// it one more image, which arrives beside the first key block, instead of a launch that reads both tensors.  Kernel times, us: B 2, H 32,
// S 2048, dh 128 105.0 and a row dot of 11.2 before, now 108.7; B 2, H 40, S 1816, dh 64, unmasked 117.5 and 7.0, now 119.2 (the lane's pieces
// of the row by plain loads beside the first copies, without image and barriers: no faster).
struct AttnDqParams {
  const bf16_t* qkv; long ld_qkv;
  const bf16_t* dout; long ld_do;
  const bf16_t* out;                   // [B*S, H*DH] the forward's output (rows as dout)
  const float* lse;                    // [B, H, S]
  float* delta;                        // [B*S, H]: written here (rowsum(dout * out)), read by the pass over the queries
  const float2* rope;                  // rotation table [S][DH / 2]: dq is rotated back; or nullptr
  bf16_t* dqkv; long ld_dqkv;          // dq block is written (columns h * DH ..)
  int B, H, S, causal;
  float scale, scale_log2e;
};

template <int DH, int SPLIT, bool ROPE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_bwd_dq_kernel(AttnDqParams p) {
  using HT = HeadTile<DH>;
  constexpr int KS = DH / 16, DT = DH / 32, BKV = 64, BQ = 128 / SPLIT, QW = 4 / SPLIT;
  constexpr int IMG = BKV * HT::RB, SLOT = 2 * IMG;
  constexpr int NCH = IMG / 1024 / 4;

  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  lds_u8* const lds = LDS_PTR(unsigned char, smem_raw);
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;

  const int lane = threadIdx.x & 63, ql = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qb = (int)gridDim.y - 1 - (int)blockIdx.y;             // longest (last) query blocks first
  const int h = (int)blockIdx.x % p.H, b = (int)blockIdx.x / p.H;
  const int wq = SPLIT == 1 ? wave : wave % QW, wk = SPLIT == 1 ? 0 : wave / QW;      // which 32 queries, which 32-key tile of every block (SPLIT 2)
  const int q0 = qb * BQ, qw0 = q0 + 32 * wq, query = qw0 + ql;
  const int d = p.H * DH;
  const long tok0 = (long)b * p.S;
  const long bh = (long)b * p.H + h;

  const typename HT::Offsets fo = HT::offsets(lane);
  // ---- the block's query rows into the second slot and their output derivatives into the first (coalesced copies)
  {
    const u32x4 dq = make_desc(p.qkv + (tok0 + q0) * p.ld_qkv + h * DH, (uint32_t)((long)(p.S - q0) * p.ld_qkv * 2));
    const u32x4 dd = make_desc(p.dout + (tok0 + q0) * p.ld_do + h * DH, (uint32_t)((long)(p.S - q0) * p.ld_do * 2));
#pragma unroll
    for (int i = 0; i < 2 * NCH / SPLIT; i++) {
      int row; unsigned go, gd;
      HT::plan(wave + 4 * i, lane, p.ld_qkv, row, go);
      HT::plan(wave + 4 * i, lane, p.ld_do, row, gd);
      const bool ok = q0 + row < p.S;
      dma16(lds0 + SLOT + (wave + 4 * i) * 1024, dq, ok ? go : kOob);
      dma16(lds0 + (wave + 4 * i) * 1024, dd, ok ? gd : kOob);
    }
  }
  int c_row[NCH];
  unsigned c_off[NCH];
#pragma unroll
  for (int i = 0; i < NCH; i++) HT::plan(wave + 4 * i, lane, p.ld_qkv, c_row[i], c_off[i]);
  const int kv_end = p.causal ? (q0 + BQ < p.S ? q0 + BQ : p.S) : p.S;
  const int nblk = (kv_end + BKV - 1) / BKV;
  auto issue = [&](int j) {
    const int kv0 = j * BKV;
    const bf16_t* kb = p.qkv + (tok0 + kv0) * p.ld_qkv + d + h * DH;
    const uint32_t bytes = (uint32_t)((long)(p.S - kv0) * p.ld_qkv * 2);
    const u32x4 dk = make_desc(kb, bytes), dv = make_desc(kb + d, bytes);
    const uint32_t base = lds0 + (j & 1) * SLOT + wave * 1024;
#pragma unroll
    for (int i = 0; i < NCH; i++) {
      const unsigned off = (kv0 + c_row[i] < p.S) ? c_off[i] : kOob;
      dma16(base + i * 4096, dk, off);
      dma16(base + IMG + i * 4096, dv, off);
    }
  };
  const bool qlive = query < p.S;
  const float lse_q = qlive ? p.lse[bh * p.S + query] : 0.f;

  f32x16 dqt[DT];
#pragma unroll
  for (int t = 0; t < DT; t++)
#pragma unroll
    for (int e = 0; e < 16; e++) dqt[t][e] = 0.f;

  wait_vmem<0>();
  __syncthreads();
  bf16x8 qf[KS], dof[KS];            // this lane's query row and output-derivative row as B operands
#pragma unroll
  for (int s = 0; s < KS; s++) {
    qf[s] = HT::rows_frag(lds + SLOT, fo, 32 * wq, s);
    dof[s] = HT::rows_frag(lds, fo, 32 * wq, s);
  }
  __syncthreads();                   // every wave has its rows: both slots are free for the key blocks
  issue(0);
  // ---- delta of this lane's query, rowsum(dout * out): the block's rows of the output arrive in the second slot beside the
  // first key block
  {
    const u32x4 dr = make_desc(p.out + (tok0 + q0) * p.ld_do + h * DH, (uint32_t)((long)(p.S - q0) * p.ld_do * 2));
#pragma unroll
    for (int i = 0; i < 2 * NCH / SPLIT; i++) {
      int row; unsigned go;
      HT::plan(wave + 4 * i, lane, p.ld_do, row, go);
      dma16(lds0 + SLOT + (wave + 4 * i) * 1024, dr, q0 + row < p.S ? go : kOob);
    }
  }
  wait_vmem<0>();
  __syncthreads();
  float dl_q = 0.f;
#pragma unroll
  for (int s = 0; s < KS; s++) {
    const bf16x8 o = HT::rows_frag(lds + SLOT, fo, 32 * wq, s);
#pragma unroll
    for (int i = 0; i < 8; i++) dl_q += (float)o[i] * (float)dof[s][i];
  }
  dl_q += xor32(dl_q);
  if (qlive && g == 0 && wk == 0) p.delta[(tok0 + query) * p.H + h] = dl_q;
  __syncthreads();                   // the second slot is free again
  for (int j = 0; j < nblk; j++) {
    wait_vmem<0>();
    __syncthreads();                 // block j has landed; every wave is done with the other slot
    if (j + 1 < nblk) issue(j + 1);
    const int kv0 = j * BKV;
    if (p.causal && kv0 > qw0 + 31) continue;
    lds_u8* const kimg = lds + (j & 1) * SLOT;
    lds_u8* const vimg = kimg + IMG;
    // keys beyond the query (causal) or beyond the sequence do not take part: their probability is zero
    const bool edge = (p.causal && kv0 + BKV - 1 > qw0) || kv0 + BKV > p.S;
    const int last = p.causal ? (query < p.S - 1 ? query : p.S - 1) : p.S - 1;
    const int rel = last - kv0 - 4 * g;
    // one 32-key tile at a time (both tiles at once would need 64 more accumulator registers than a wave has):
    // S^T and dP^T as two interleaved accumulation chains, fragments one k-step ahead; then dS^T in place and
    // dQ^T += K^T dS^T over the tile's two k-steps on DT independent accumulators
#pragma unroll 1
    for (int kt = SPLIT == 2 ? wk : 0; kt < (SPLIT == 2 ? wk + 1 : 2); kt++) {
      f32x16 st, dp;
#pragma unroll
      for (int e = 0; e < 16; e++) { st[e] = 0.f; dp[e] = 0.f; }
      // (the order is pinned: the compiler would fetch each fragment right before its MFMA)
      constexpr int PF = 3;
      bf16x8 kf[PF], vf[PF], ktf[DT];
#pragma unroll
      for (int s = 0; s < PF; s++) { kf[s] = HT::rows_frag(kimg, fo, 32 * kt, s); vf[s] = HT::rows_frag(vimg, fo, 32 * kt, s); }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < KS; s++) {
        st = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s % PF], qf[s], st, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[s % PF], dof[s], dp, 0, 0, 0);
        if (s + PF < KS) { kf[s % PF] = HT::rows_frag(kimg, fo, 32 * kt, s + PF); vf[s % PF] = HT::rows_frag(vimg, fo, 32 * kt, s + PF); }
        if (s >= KS - DT) ktf[s - (KS - DT)] = HT::cols_frag(kimg, fo, 32 * kt, 0, s - (KS - DT));
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int e = 0; e < 16; e++) {
        st[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(st[e], p.scale_log2e, -lse_q));
      }
      if (edge) {
#pragma unroll
        for (int e = 0; e < 16; e++) st[e] = (32 * kt + 8 * (e >> 2) + (e & 3) > rel) ? 0.f : st[e];
      }
#pragma unroll
      for (int e = 0; e < 16; e++) st[e] *= dp[e] - dl_q;    // dS^T
#pragma unroll
      for (int u = 0; u < 2; u++) {
        const bf16x8 sb = pack8(st, u);
#pragma unroll
        for (int t = 0; t < DT; t++) {
          dqt[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ktf[t], sb, dqt[t], 0, 0, 0);
          if (u == 0) ktf[t] = HT::cols_frag(kimg, fo, 32 * kt, 1, t);     // the second k-step's fragment, behind the MFMA that used the first
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  }

  __syncthreads();
  if constexpr (SPLIT == 2) {        // the two waves of a query add up, first the wave of the first tiles
    LDS_AS float* const part = reinterpret_cast<LDS_AS float*>(lds) + wq * (DT * 1024);
    static_assert(QW * DT * 4096 <= 2 * SLOT, "the partial sums must fit in the ring");
    if (wk == 1) {
#pragma unroll
      for (int t = 0; t < DT; t++)
#pragma unroll
        for (int e = 0; e < 16; e++) part[(t * 16 + e) * 64 + lane] = dqt[t][e];
    }
    __syncthreads();
    if (wk == 0) {
#pragma unroll
      for (int t = 0; t < DT; t++)
#pragma unroll
        for (int e = 0; e < 16; e++) dqt[t][e] += part[(t * 16 + e) * 64 + lane];
    }
    __syncthreads();
    if (wk == 1) return;
  }
  // ---- dq = scale * dQ^T (rotated back: a lane holds both halves of its query's row), transposed back through LDS and
  // written as whole rows (as the forward writes its output)
#pragma unroll
  for (int t = 0; t < DT; t++)
#pragma unroll
    for (int e = 0; e < 16; e++) dqt[t][e] *= p.scale;
  if constexpr (ROPE) {
    const float2* const tb = p.rope + (long)(qlive ? query : 0) * (DH / 2) + 4 * g;
#pragma unroll
    for (int t = 0; t < DT / 2; t++)
#pragma unroll
      for (int e4 = 0; e4 < 4; e4++) {
        const f32x4 c01 = *reinterpret_cast<const f32x4*>(tb + 32 * t + 8 * e4);
        const f32x4 c23 = *reinterpret_cast<const f32x4*>(tb + 32 * t + 8 * e4 + 2);
        const float cs[4] = {c01[0], c01[2], c23[0], c23[2]}, sn[4] = {c01[1], c01[3], c23[1], c23[3]};
#pragma unroll
        for (int r = 0; r < 4; r++) {
          const float x = dqt[t][4 * e4 + r], y = dqt[t + DT / 2][4 * e4 + r];
          dqt[t][4 * e4 + r] = x * cs[r] + y * sn[r];
          dqt[t + DT / 2][4 * e4 + r] = y * cs[r] - x * sn[r];
        }
      }
  }
  constexpr int EROW = DH * 2 + 16;
  static_assert(BQ * EROW <= 2 * SLOT, "the output tile must fit in the ring");
  lds_u8* const erow = lds + 32 * wq * EROW;
#pragma unroll
  for (int t = 0; t < DT; t++)
#pragma unroll
    for (int e4 = 0; e4 < 4; e4++) {
      bf16x4 v;
#pragma unroll
      for (int r = 0; r < 4; r++) v[r] = (bf16_t)dqt[t][4 * e4 + r];
      *reinterpret_cast<LDS_AS bf16x4*>(erow + ql * EROW + (32 * t + 8 * e4 + 4 * g) * 2) = v;
    }
  {  // (LDS operations of a wave execute in order: the reads below see this wave's own writes above)
    constexpr int LPR = DH / 8, RPI = 64 / LPR;
    const int rl = lane / LPR, piece = lane % LPR;
#pragma unroll
    for (int r0 = 0; r0 < 32; r0 += RPI) {
      const int qrow = qw0 + r0 + rl;
      if (qrow < p.S)
        *reinterpret_cast<u32x4*>(p.dqkv + (tok0 + qrow) * p.ld_dqkv + h * DH + 8 * piece) =
            *reinterpret_cast<const LDS_AS u32x4*>(erow + (r0 + rl) * EROW + 16 * piece);
    }
  }
}

// Workgroups of 128 queries (keys) of a launch; and is the chip short of them?  Up to one per compute unit it is; with the
// causal mask, whose longest workgroup works eight times as long as the shortest (or more), up to two.  (Lines set at head_dim 128; at 64
// halves would pay on somewhat larger grids too: B 3, H 24, S 512, causal, 288 workgroups, forward 11.5 / 10.0 us.)
static long query_groups(long heads, int seq) { return heads * ((seq + 127) / 128); }
static bool few_query_groups(long heads, int seq) { const long w = query_groups(heads, seq); return w <= 256 || (w <= 512 && seq > 896); }

template <int DH, bool AHEAD, int SPLIT>
static hipError_t launch_fwd(const AttnParams& p, hipStream_t s) {
  constexpr size_t smem = 2 * 2 * 64 * DH * 2;
  auto kern = attn_fwd_kernel<DH, AHEAD, SPLIT>;
  static AttrOnce once;
  if (hipError_t e = once.set(reinterpret_cast<const void*>(kern), smem); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)(p.H * p.B), (unsigned)((p.S * SPLIT + 127) / 128)), dim3(256), smem, s, p);
  return hipGetLastError();
}

hipError_t attention_fwd(int batch, int n_heads, int seq, int head_dim, int causal, const void* qkv, long ld_qkv,
                         void* out, long ld_out, float* lse, hipStream_t s) {
  if (batch <= 0 || n_heads <= 0 || seq <= 0) return hipSuccess;
  AttnParams p{};
  p.qkv = (const bf16_t*)qkv; p.ld_qkv = ld_qkv; p.out = (bf16_t*)out; p.ld_out = ld_out; p.lse = lse;
  p.B = batch; p.H = n_heads; p.S = seq; p.causal = causal;
  p.scale_log2e = 1.4426950408889634f / sqrtf((float)head_dim);
  if (head_dim != 128 && head_dim != 64) return hipErrorInvalidValue;
  // us, 128 / 64 queries per workgroup; causal: B 1, H 32, dh 128, S 256 9.0 / 7.6, S 512 13.5 / 11.0, S 1024 23.8 / 21.1, S 2048
  // 51.7 / 48.3; B 4, H 12, dh 64, S 1000 18.9 / 16.9; lost: B 4, H 32, dh 128, S 512 21.1 / 23.6, B 1, H 40, S 2048 55.3 / 62.9; unmasked:
  // B 1, H 16, dh 128, S 1024 21.8 / 17.4, twice the heads 26.5 / 24.9; S 64 4.1 / 4.3
  if (seq > 64 && (query_groups(batch * (long)n_heads, seq) <= 256 || (causal && few_query_groups(batch * (long)n_heads, seq))))
    return head_dim == 128 ? launch_fwd<128, false, 2>(p, s) : launch_fwd<64, false, 2>(p, s);
  if (head_dim == 128) return seq > 256 ? launch_fwd<128, true, 1>(p, s) : launch_fwd<128, false, 1>(p, s);
  return seq > 256 ? launch_fwd<64, true, 1>(p, s) : launch_fwd<64, false, 1>(p, s);
}

template <int DH, int SPLIT>
static hipError_t launch_bwd_dq(const AttnDqParams& p, hipStream_t s) {
  constexpr size_t smem = 2 * 2 * 64 * DH * 2;
  auto kern = p.rope ? attn_bwd_dq_kernel<DH, SPLIT, true> : attn_bwd_dq_kernel<DH, SPLIT, false>;
  static AttrOnce once[2];
  if (hipError_t e = once[p.rope != nullptr].set(reinterpret_cast<const void*>(kern), smem); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)(p.H * p.B), (unsigned)((p.S * SPLIT + 127) / 128)), dim3(256), smem, s, p);
  return hipGetLastError();
}

// 64 keys per workgroup instead of 128?  By modelled time, in units of 128 keys times 128 queries: a workgroup costs its units and
// 1.3 (start and drain, one workgroup per compute unit), units on 64 keys 10 % more; the launch takes as long as its rounds or,
// with the causal mask, as its longest workgroup or as all of them spread over the chip.  us of the whole backward, 128 / 64: causal,
// dh 128, B 1, H 32, S 256 23.5 / 20.0, S 1024 64.1 / 56.6, S 2048 142 / 147, B 4, H 32, S 256 31.3 / 31.8, B 1, H 8, S 4096 199 / 167;
// unmasked, B 1, H 16, dh 128, S 1024 59.0 / 50.4, twice the heads 68.4 / 72.1, B 4, H 12, dh 64, S 1000 80.7 / 73.4, B 1, H 40, dh 128,
// S 2048 326 / 320.
static bool short_key_blocks(long heads, int seq, int causal) {
  const double kStart = 1.3, kSlower = 1.1, nb = (seq + 127) / 128;
  const double w = heads * nb;
  if (!causal) return ceil(2 * w / 256) * (0.5 * kSlower * nb + kStart) < ceil(w / 256) * (nb + kStart);
  const double units = heads * nb * (nb + 1) / 2;
  const double whole = fmax(nb + kStart, (units + kStart * w) / 256);
  return fmax(0.5 * kSlower * nb + kStart, (kSlower * units + 2 * kStart * w) / 256) < whole;
}

template <int DH, bool WRITE_DST, int KEYS>
static hipError_t launch_bwd_kv_split(const AttnBwdParams& p, hipStream_t s) {
  constexpr size_t smem = 3 * (2 * 64 * DH * 2 + 1024) + 2 * 4 * 4096 + (WRITE_DST ? 4 * 32 * 144 : 0);     // three slots, two hand-over buffers, dS^T staging
  auto kern = p.rope && !WRITE_DST ? attn_bwd_kv_split_kernel<DH, WRITE_DST, KEYS, !WRITE_DST> : attn_bwd_kv_split_kernel<DH, WRITE_DST, KEYS, false>;
  static AttrOnce once[2];
  if (hipError_t e = once[p.rope != nullptr].set(reinterpret_cast<const void*>(kern), smem); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)(p.H * p.B), (unsigned)((p.S + KEYS - 1) / KEYS)), dim3(512), smem, s, p);
  return hipGetLastError();
}

hipError_t attention_p1(int batch, int n_heads, int seq, int head_dim, int causal, const void* qkv, long ld_qkv,
                        const void* out, const void* d_out, long ld_out, const float* lse, void* dqkv, long ld_dqkv,
                        float* delta, void* ds_t, const float2* rope_table, hipStream_t s) {
  if (batch <= 0 || n_heads <= 0 || seq <= 0) return hipSuccess;
  if (ld_out != (long)n_heads * head_dim || (head_dim != 64 && head_dim != 128)) return hipErrorInvalidValue;      // out and d_out are read with the one leading dimension
  AttnBwdParams p{};
  p.qkv = (const bf16_t*)qkv; p.ld_qkv = ld_qkv; p.dout = (const bf16_t*)d_out; p.ld_do = ld_out;
  p.lse = lse; p.delta = delta; p.dqkv = (bf16_t*)dqkv; p.ld_dqkv = ld_dqkv; p.dst = (bf16_t*)ds_t;
  p.B = batch; p.H = n_heads; p.S = seq; p.causal = causal;
  p.scale = 1.f / sqrtf((float)head_dim);
  p.scale_log2e = 1.4426950408889634f * p.scale;
  hipError_t e;
  if (!ds_t || attn_rebuilds_dq(batch, n_heads, seq, head_dim, causal, rope_table != nullptr)) {
    const long heads = (long)batch * n_heads;
    // us of the whole backward, 128 / 64 queries per workgroup of the dq pass; causal: B 1, H 32, dh 128, S 256 23.5 / 21.1, S 1024
    // 64.1 / 57.3, S 2048 142 / 138, B 4, H 12, dh 64, S 1000 50.5 / 48.3; lost: B 4, H 32, S 512 60.9 / 62.1; unmasked: B 1, H 16,
    // dh 128, S 1024 59.0 / 52.6, H 24, S 1000 62.8 / 62.5, B 4, H 12, dh 64, S 1000 80.7 / 80.9
    const bool short_queries = causal ? few_query_groups(heads, seq) : query_groups(heads, seq) <= 128;
    p.rope = rope_table;
    AttnDqParams q{};
    q.qkv = p.qkv; q.ld_qkv = ld_qkv; q.dout = p.dout; q.ld_do = ld_out; q.out = (const bf16_t*)out; q.lse = lse; q.delta = delta;
    q.rope = rope_table; q.dqkv = p.dqkv; q.ld_dqkv = ld_dqkv; q.B = batch; q.H = n_heads; q.S = seq; q.causal = causal;
    q.scale = p.scale; q.scale_log2e = p.scale_log2e;
    if (short_queries) e = head_dim == 128 ? launch_bwd_dq<128, 2>(q, s) : launch_bwd_dq<64, 2>(q, s);
    else e = head_dim == 128 ? launch_bwd_dq<128, 1>(q, s) : launch_bwd_dq<64, 1>(q, s);
    if (e != hipSuccess) return e;
    if (short_key_blocks(heads, seq, causal)) return head_dim == 128 ? launch_bwd_kv_split<128, false, 64>(p, s) : launch_bwd_kv_split<64, false, 64>(p, s);
    return head_dim == 128 ? launch_bwd_kv_split<128, false, 128>(p, s) : launch_bwd_kv_split<64, false, 128>(p, s);
  }
  if (e = head_rowdot(1, batch * seq, n_heads, head_dim, d_out, out, delta, s); e != hipSuccess) return e;
  if (e = launch_bwd_kv_split<128, true, 128>(p, s); e != hipSuccess) return e;      // (head_dim 64 is always rebuilt)
  // dq = scale * dS k = scale * (dS^T)^T k per (sequence, head): contraction over keys, causal: keys <= query
  const long d = (long)n_heads * head_dim;
  GemmArgs g = gemm_args(TN, seq, head_dim, seq, ds_t, kPanel, (const char*)qkv + d * 2, ld_qkv, dqkv, ld_dqkv);
  g.alpha = p.scale;
  g.a_panel = (long)seq * kPanel;
  g.batch = batch * n_heads; g.batch_inner = n_heads;
  g.sAi = (long)attn_ds_elems(seq); g.sAo = n_heads * g.sAi;
  g.sBo = (long)seq * ld_qkv; g.sBi = head_dim;
  g.sCo = (long)seq * ld_dqkv; g.sCi = head_dim;
  g.causal = causal ? CAUSAL_K_END : CAUSAL_NONE;
  if (e = gemm(1, g, s); e != hipSuccess || !rope_table) return e;
  return rope(1, batch * seq, seq, 2 * n_heads, head_dim, ld_dqkv, rope_table, 1, dqkv, s);
}

}  // namespace tbp
