// GEMM kernels for gfx950 (MI355X).
//
// bf16 path: C = alpha * op(A) op(B) on the 32x32x16 bf16 MFMA instruction, fp32 accumulation.
//   One workgroup = 4 multiplying wavefronts (2 x 2) and, on the NN / NT tiles up to 256 x 128, 4 that only copy; block tile
//   BM x BN (64 x 64 to 256 x 256, chosen per product by modelled time), contraction consumed in slices of 32 through a 4-slot
//   LDS ring, or in slices of 64 through two to six slots where the contraction index is contiguous in
//   memory, filled by asynchronous global -> LDS copies (no staging registers) that stay in flight while the previous
//   slices are multiplied.  The smallest outputs run on 32 x 32 tiles that the four waves share, each through its own ring.
//   Outputs with too few tiles cut the contraction over several workgroups per tile (scratch memory, a second launch).
//   An operand whose contraction index is contiguous in memory ("KC": A of NN/NT, B of NT) is kept in
//   LDS as [row][k] and read as 16-byte vectors; an operand whose contraction index is the slow,
//   strided one ("KS": A of TN, B of NN/TN, i.e. both operands of dW = X^T dY) is kept as [k][row]
//   exactly as it sits in memory and transposed on the way to the registers by the LDS
//   transpose-read instruction (ds_read_b64_tr_b16), so no operand is ever transposed in HBM.
//   Out-of-range lanes of a copy are redirected past the end of the buffer descriptor (they deliver zero),
//   which handles ragged M, N and K without branches.
// fp32 path: the 32x32x2 (small outputs: 16x16x4) fp32 MFMA with the same kind of copies; a plain FMA tile kernel with generic strides for
// operands that are not made of whole aligned 16-byte pieces.
#include "kernels.h"
#include "gfx950.h"

namespace tbp {

struct GemmParams {
  const void* A; const void* B; void* C; const void* R;
  long lda, ldb, ldc;
  long sAo, sAi, sBo, sBi, sCo, sCi;
  int M, N, K;
  int batch_inner;
  int tiles_m, tiles_n;
  float alpha;
  int accumulate;
  int causal;
  // fp32 kernel only: element strides of A(m,k) and B(k,n)
  long sam, sak, sbk, sbn;
  // fused softmax backward (see GemmArgs)
  const float* delta; long ldd, sDo, sDi;
  int delta_causal, causal_fill;
  long a_panel;                 // see GemmArgs
  // contraction cut into `split` slices of split_k indices, one workgroup per (tile, slice) (see SplitPlan); slice i leaves
  // its partial product at C + i * sCo
  int split, split_k;
  const void* gu;               // see GemmArgs
  PairEpilogue pair;            // paired columns (gemm_bf16_pairs_kernel)
};

constexpr int BK = 32;                     // contraction depth of one LDS slot
constexpr int STAGES = 4;                  // LDS ring: one slot being multiplied, three in flight


// Workgroup id -> (tile row, tile column).  Workgroups are handed to the 8 XCDs round-robin; the first
// step makes each XCD own a contiguous range of the tile sequence (so its private L2 sees neighbouring
// tiles), the second walks that sequence in groups of 8 tile rows so that concurrently running tiles
// share A and B panels.
__device__ __forceinline__ void tile_of_block(int pid, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int nt = tiles_m * tiles_n;
  const int xcd = pid & 7, q = pid >> 3;
  const int per = nt >> 3, rem = nt & 7;
  int id = xcd * per + (xcd < rem ? xcd : rem) + q;
  const int GROUP = 8;
  const int width = GROUP * tiles_n;
  const int grp = id / width;
  const int first = grp * GROUP;
  const int gsz = (tiles_m - first) < GROUP ? (tiles_m - first) : GROUP;
  const int r = id - grp * width;
  tm = first + r % gsz;
  tn = r / gsz;
}

// The same for a product whose contraction is cut into slices: the sequence that is dealt out to the XCDs in contiguous
// ranges runs over the tiles of the first slice, then of the second, and so on.  An XCD then works on one slice (or a
// stretch of one), so each L2 fetches only its slice of the operands, and of the larger one (the weights) no other XCD
// fetches the same part.
__device__ __forceinline__ void tile_of_block_split(int pid, int tiles_m, int tiles_n, int split, int& tm, int& tn, int& slice) {
  const int nt = tiles_m * tiles_n, total = nt * split;
  const int xcd = pid & 7, q = pid >> 3;
  const int per = total >> 3, rem = total & 7;
  const int seq = xcd * per + (xcd < rem ? xcd : rem) + q;
  slice = seq / nt;
  const int id = seq - slice * nt;
  const int GROUP = 8, width = GROUP * tiles_n;
  const int grp = id / width, first = grp * GROUP;
  const int gsz = (tiles_m - first) < GROUP ? (tiles_m - first) : GROUP;
  const int r = id - grp * width;
  tm = first + r % gsz;
  tn = r / gsz;
}

// SKIP_UPPER: is the tile at (m0, n0) left out?  Tiles wholly above the diagonal are, except for those within the range that
// has to hold zeros (see GemmArgs::causal_fill); `empty` tells of one of those that there is nothing to contract.
template <int BM>
__device__ __forceinline__ bool tile_skipped(const GemmParams& p, int m0, int n0, bool& empty) {
  empty = n0 >= m0 + BM;
  const int fill = p.causal_fill > BM ? p.causal_fill : BM;
  return n0 >= (m0 & -fill) + fill;
}

// LDS image of one operand tile (R rows/columns of the output x BK of the contraction), laid out so that
// (a) every 1 KiB piece is what one wave-wide 16-byte-per-lane copy writes (64 consecutive 16-byte granules),
// (b) the MFMA fragment reads are free of bank conflicts without padding:
//   KC (contraction index contiguous in memory): image [R][depth], 4 or 8 granules per row; granule g of row r sits
//       in slot g ^ ((r >> 2) & 3) (depth 32) or g ^ ((r >> 1) & 7) (depth 64): the 16 lanes served per clock (256
//       bytes) then touch 16 different 16-byte bank groups.  A fragment read is one ds_read_b128 per lane.
//   KS (contraction index strided in memory): image [BK][R] as in memory, R/8 granules per row; granule
//       pairs (32 bytes = 16 columns) are swizzled: pair q of row k sits in pair slot q ^ (k & 3) (tiles of 32 columns have
//       two pairs per row and need no swizzle: four rows cover the banks).  A fragment
//       read is two ds_read_b64_tr_b16 (transpose reads), each covering 4 k x 16 columns per 16-lane group:
//       within a group lane j addresses row k + j/4, columns 4*(j%4)..+3 and receives 4 consecutive k of column j.
template <int R, bool KC, int KD = BK>
struct OperandTile {
  static constexpr int BYTES = R * KD * 2;
  static constexpr int CHUNKS = BYTES / 1024;       // wave-wide copies per tile
  static constexpr int PER_WAVE = CHUNKS / 4;
  static constexpr int GPR = R / 8;                 // granules per image row (KS)
  static constexpr int GR = KD / 8;                 // granules per image row (KC): 4 (64-byte rows) or 8 (128-byte rows)
  static constexpr int RPB = 16 / GR;               // KC rows per 256 bytes (one pass over all banks)
  static_assert(CHUNKS % 4 == 0, "tile must split evenly over 4 waves");
  static_assert(KD == 32 || KD == 64, "slot depth");

  // KC swizzle: granule g of row r sits in slot g ^ ((r / RPB) % GR), so 16 consecutive rows at one logical granule
  // cover the 16 bank groups once.
  static __device__ __forceinline__ int kc_swz(int row) { return (row / RPB) & (GR - 1); }
  static __device__ __forceinline__ int ks_swz(int k) { return R >= 64 ? (k & 3) : 0; }

  // Global byte offset (relative to the tile origin) and contraction index covered by lane p of chunk c.
  static __device__ __forceinline__ void copy_plan(int c, int p, long ld, int origin, int extent, unsigned& goff,
                                                   int& kidx) {
    if constexpr (KC) {
      const int row = (64 / GR) * c + p / GR;
      const int g = (p % GR) ^ kc_swz(row);
      goff = (origin + row < extent) ? (unsigned)((long)row * ld * 2 + g * 16) : kOob;
      kidx = g * 8;
    } else {
      const int P = 64 * c + p;
      const int k = P / GPR, sl = P % GPR;
      const int g = ((((sl >> 1) ^ ks_swz(k)) << 1) | (sl & 1));
      goff = (origin + g * 8 < extent) ? (unsigned)((long)k * ld * 2 + g * 16) : kOob;
      kidx = k;
    }
  }
  // Per-lane byte offset inside the image of the fragment of MFMA tile 0 (rows/columns w0..w0+31), variant v:
  // KC: v = k-step (0 .. KD/16 - 1);  KS: v = parity of the MFMA tile index.
  static __device__ __forceinline__ int frag_base(int lane, int w0, int v) {
    if constexpr (KC) {
      const int row = w0 + (lane & 31);
      const int g = 2 * v + (lane >> 5);
      return row * (KD * 2) + ((g ^ kc_swz(row)) << 4);
    } else {
      const int k = 8 * (lane >> 5) + ((lane & 15) >> 2);
      const int q = w0 / 16 + ((lane >> 4) & 1) + 2 * v;
      return k * (R * 2) + ((q ^ ks_swz(k)) << 5) + 8 * (lane & 3);
    }
  }
  static constexpr int VARIANTS = KC ? KD / 16 : 2;
  static __device__ __forceinline__ constexpr int variant(int ks, int t) { return KC ? ks : (t & 1); }
  // Byte offset of (k-step ks, MFMA tile t) relative to frag_base(..., variant(ks, t)).
  static __device__ __forceinline__ constexpr int frag_step(int ks, int t) {
    return KC ? t * 32 * KD * 2 : ks * 16 * R * 2 + (t >> 1) * 128;
  }
};

template <int R, bool KC>
__device__ __forceinline__ bf16x8 read_frag(lds_u8* q) {
  if constexpr (KC) {
    return *reinterpret_cast<LDS_AS const bf16x8*>(q);
  } else {
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<LDS_AS s16x4*>(q));
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<LDS_AS s16x4*>(q + 4 * R * 2));
    s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
  }
}

// One output tile (tm_i, tn_i) of batch entry z of the product described by p.
// ACC: C += (fp32 output).  A template parameter, because the registers that the old values take cost the overwriting
// 256 x 256 kernel 2-3 %.
// KD = contraction depth of one LDS slot: 32 with a ring of 4 slots, or 64 with 2 slots.  The deeper slot is for
// operands whose contraction index is contiguous in memory: their copies then fetch 128 contiguous bytes per tile
// row, a whole cache line, where the 32-deep slot fetches every line in two halves one iteration apart and doubles
// the number of requests to the L2.
// COPIERS: a workgroup of 8 waves, of which 0..3 multiply and 4..7 do nothing but start the copies and wait for them.  A wave
// that does both issues in order: while the texture path takes its 1 KiB requests one by one, its MFMAs wait.  With a wave of
// each kind on every SIMD a 128 x 128 tile of 4096 indices takes 33.9 us instead of 36.3 ([1024, 4096] x 4096; copies alone 27,
// MFMAs alone 25), on 256 products of all kinds 4-15 %.  The 256 x 256 and 256 x 192 tiles have no registers for a second wave.
template <int BM, int BN, bool AKC, bool BKC, typename OutT, int KD = BK, bool SPLIT = false, int RING = 0, bool ACC = false, bool COPIERS = false>
__device__ __forceinline__ void gemm_bf16_tile(const GemmParams& p, int tm_i, int tn_i, int z) {
  // RING == 0: the default pipeline of the slot depth (32: ring of STAGES slots; 64: two slots); RING >= 3: the ring
  // pipeline with that many slots, for either depth
  constexpr bool RINGPIPE = KD == 32 || RING >= 3;
  constexpr int NS = COPIERS || RING >= 3 ? RING : (KD == 32 ? STAGES : 2);       // ring slots
  constexpr int KSTEPS = KD / 16;
  constexpr int WM = BM / 2, WN = BN / 2;       // per-wave tile
  constexpr int TM = WM / 32, TN = WN / 32;     // MFMA tiles per wave
  using TA = OperandTile<BM, AKC, KD>;
  using TB = OperandTile<BN, BKC, KD>;
  constexpr int STAGE_BYTES = TA::BYTES + TB::BYTES;
  constexpr int NA = TA::PER_WAVE, NB = TB::PER_WAVE;
  constexpr int L = NA + NB;                    // asynchronous copies per thread per slot

  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  lds_u8* const lds = LDS_PTR(unsigned char, smem_raw);
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave = COPIERS ? wave8 & 3 : wave8;
  const int wm = wave >> 1, wn = wave & 1;

  const int m0 = tm_i * BM, n0 = tn_i * BN;

  int k_lo = 0, k_hi = p.K;
  if (p.causal == CAUSAL_SKIP_UPPER) {
    bool empty;
    if (tile_skipped<BM>(p, m0, n0, empty)) return;
    if (empty) k_hi = 0;
  } else if (p.causal == CAUSAL_K_END) {
    k_hi = (m0 + BM < p.K) ? m0 + BM : p.K;
  } else if (p.causal == CAUSAL_K_BEGIN) {
    k_lo = m0;
  }
  if constexpr (SPLIT) {      // z: this workgroup's slice of the contraction, in whole slots (the last may be shorter)
    k_lo = z * p.split_k;
    k_hi = k_lo + p.split_k < p.K ? k_lo + p.split_k : p.K;
  }
  const int nk = (k_hi - k_lo + KD - 1) / KD;

  const int zo = SPLIT ? z : z / p.batch_inner, zi = SPLIT ? 0 : z - zo * p.batch_inner;
  const bf16_t* A = reinterpret_cast<const bf16_t*>(p.A) + zo * p.sAo + zi * p.sAi;
  const bf16_t* B = reinterpret_cast<const bf16_t*>(p.B) + zo * p.sBo + zi * p.sBi;

  // ---- this wave's share of the global -> LDS copies of one slot: chunks wave, wave + 4, ...
  unsigned a_goff[NA], b_goff[NB];
  int a_kidx[NA], b_kidx[NB];
#pragma unroll
  for (int i = 0; i < NA; i++) TA::copy_plan(wave + 4 * i, lane, p.lda, m0, p.M, a_goff[i], a_kidx[i]);
#pragma unroll
  for (int i = 0; i < NB; i++) TB::copy_plan(wave + 4 * i, lane, p.ldb, n0, p.N, b_goff[i], b_kidx[i]);
  // tile origin at k = 0 (an operand stored in panels is only ever given to the kernel whose BM is the panel width)
  const bf16_t* Ablk = AKC ? A + (long)m0 * p.lda : (p.a_panel ? A + (long)tm_i * p.a_panel : A + m0);
  const bf16_t* Bblk = BKC ? B + (long)n0 * p.ldb : B + n0;
  const long a_kstep = AKC ? 1 : p.lda;                          // elements per unit of k
  const long b_kstep = BKC ? 1 : p.ldb;

  // Copies of the next K tile into the next ring slot.  One code path serves full tiles, the ragged last tile
  // and tiles past the end ( every lane is redirected out of range, zeros land in a slot nobody reads
  // again, no memory traffic), so the main loop needs no branch around it.
  struct CopyJob { u32x4 dA, dB; uint32_t sa, sb; int krem; };
  // Running state of the copy stream (all wave-uniform): next tile's operand addresses, ring slot and remaining k.
  uint64_t a_next = reinterpret_cast<uint64_t>(Ablk + (long)k_lo * a_kstep);
  uint64_t b_next = reinterpret_cast<uint64_t>(Bblk + (long)k_lo * b_kstep);
  const uint64_t a_adv = (uint64_t)(KD * a_kstep * 2), b_adv = (uint64_t)(KD * b_kstep * 2);
  int slot_next = 0, krem_next = k_hi - k_lo;
  auto next_job = [&]() {
    CopyJob j;
    j.dA = make_desc(reinterpret_cast<const void*>(a_next));
    j.dB = make_desc(reinterpret_cast<const void*>(b_next));
    j.sa = lds0 + slot_next * STAGE_BYTES + wave * 1024;
    j.sb = j.sa + TA::BYTES;
    j.krem = krem_next;
    a_next += a_adv; b_next += b_adv;
    slot_next = (slot_next + 1 == NS) ? 0 : slot_next + 1;
    krem_next -= KD;
    return j;
  };
  auto copy_one = [&](const CopyJob& j, int c) {     // c-th of this wave's L copies of the job
    if (c < NA) dma16(j.sa + c * 4096, j.dA, a_kidx[c] < j.krem ? a_goff[c] : kOob);
    else dma16(j.sb + (c - NA) * 4096, j.dB, b_kidx[c - NA] < j.krem ? b_goff[c - NA] : kOob);
  };

  int a_base[TA::VARIANTS], b_base[TB::VARIANTS];
#pragma unroll
  for (int v = 0; v < TA::VARIANTS; v++) a_base[v] = TA::frag_base(lane, wm * WM, v);
#pragma unroll
  for (int v = 0; v < TB::VARIANTS; v++) b_base[v] = TB::frag_base(lane, wn * WN, v) + TA::BYTES;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;

  // ---- main loop, software-pipelined over the two k-steps of a slot and scheduled by hand:
  //   while (tile t, k-step 0) is multiplied the fragments of (t, k-step 1) are fetched from LDS; then the wait
  //   for tile t+1 and the workgroup barrier; while (t, k-step 1) is multiplied the fragments of (t+1, k-step 0)
  //   are fetched and the asynchronous copies of tile t+STAGES-1 are started.  Reads and copies are spread
  //   between the MFMAs (an MFMA occupies the matrix pipe for 32 cycles, the other instructions issue in its
  //   shadow); sched_barrier pins that order.
  // Ring invariant: while tile t is multiplied, tiles t+1 .. t+STAGES-2 are landed or in flight; slot
  // (t-1) % STAGES is refilled only after a barrier that every wave passes after its last read of tile t-1.
  // The loop body has no data-dependent join around LDS reads (a join makes the compiler merge wait states and
  // stall MFMAs on reads they do not need): the last iteration also fetches "tile nk" fragments, stale but
  // in-bounds LDS contents that are never used.
  constexpr int MM = TM * TN, UNITS = TM + TN;
  // Fragment fetch order = order of first use by the MFMA sequence (i-major): a0, then every b, then a1, a2, ...;
  // one fetch per MFMA from the start of the region, so the fragments the NEXT region needs first have the whole
  // region to arrive and the last fetches still have MM - UNITS MFMAs of cover.  The copies fill the second half.
  // job != null: copies c0 .. c1-1 of the job are issued, spread over MFMAs m0 .. MM-1 of the region
  auto region = [&](const bf16x8* fa, const bf16x8* fb, bf16x8* na, bf16x8* nb, lds_u8* st, int nks, const CopyJob* job,
                    int c0 = 0, int c1 = -1, int m0 = -1) {
    if (c1 < 0) c1 = L;
    if (m0 < 0) m0 = MM >= 2 * L ? MM - L : 0;
#pragma unroll
    for (int m = 0; m < MM; m++) {
      const int i = m / TN, j = m % TN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
      constexpr int UPM = (UNITS + MM - 1) / MM;           // fetches per MFMA (1 for the tiles used here)
#pragma unroll
      for (int q = 0; q < UPM; q++) {
        const int u = m * UPM + q;                         // position in the fetch order
        if (u < UNITS) {
          if (u == 0) na[0] = read_frag<BM, AKC>(st + a_base[TA::variant(nks, 0)] + TA::frag_step(nks, 0));
          else if (u <= TN) nb[u - 1] = read_frag<BN, BKC>(st + b_base[TB::variant(nks, u - 1)] + TB::frag_step(nks, u - 1));
          else na[u - TN] = read_frag<BM, AKC>(st + a_base[TA::variant(nks, u - TN)] + TA::frag_step(nks, u - TN));
        }
      }
      if (job) {
        const int n = c1 - c0;
#pragma unroll
        for (int c = c0 + ((m - m0) * n) / (MM - m0); m >= m0 && c < c0 + ((m - m0 + 1) * n) / (MM - m0); c++) copy_one(*job, c);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  static_assert(BK == 32 && ((!RINGPIPE && !COPIERS) || (NS - (COPIERS ? 1 : 2)) * L < 64), "the wait counter has 6 bits");
  bf16x8 fa0[TM], fb0[TN], fa1[TM], fb1[TN];
  auto first_fragments = [&]() {
#pragma unroll
    for (int i = 0; i < TM; i++) fa0[i] = read_frag<BM, AKC>(lds + a_base[TA::variant(0, i)] + TA::frag_step(0, i));
#pragma unroll
    for (int j = 0; j < TN; j++) fb0[j] = read_frag<BN, BKC>(lds + b_base[TB::variant(0, j)] + TB::frag_step(0, j));
  };
  if constexpr (COPIERS) {
    // All NS slots are in flight or landed at any time: the barrier before the last k-step of a slot, whose fragments are in
    // registers by then, publishes the next slot and gives this one back to the copying waves.  Both kinds of wave pass
    // 1 + nk barriers here (none if nk is 0) and one below.
    if (wave8 >= 4) {
      auto issue = [&]() {
        const CopyJob j = next_job();
#pragma unroll
        for (int c = 0; c < L; c++) copy_one(j, c);
      };
      if (nk > 0) {
#pragma unroll
        for (int t = 0; t < NS; t++) issue();
        wait_vmem<(NS - 1) * L>();            // tile 0 has landed (this wave's share)
        __syncthreads();
        for (int t = 0; t < nk; t++) {
          wait_vmem<(NS - 2) * L>();          // tile t + 1
          __syncthreads();
          issue();                            // tile t + NS into the slot of tile t
        }
        wait_vmem<0>();                       // the (empty) copies issued past the end
      }
      __syncthreads();
      return;
    }
    if (nk > 0) {
      __syncthreads();
      first_fragments();
      for (int t = 0; t < nk; t++) {
        lds_u8* const cur = lds + (t % NS) * STAGE_BYTES;
#pragma unroll
        for (int ks = 1; ks < KSTEPS; ks++) {
          if (ks & 1) region(fa0, fb0, fa1, fb1, cur, ks, nullptr);
          else region(fa1, fb1, fa0, fb0, cur, ks, nullptr);
        }
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        region(fa1, fb1, fa0, fb0, lds + ((t + 1) % NS) * STAGE_BYTES, 0, nullptr);
      }
    }
  } else if constexpr (RINGPIPE) {
    // Ring of NS slots, KSTEPS k-steps per slot (an even number: the two fragment register sets alternate).  While
    // k-step ks - 1 of tile t is multiplied, the fragments of k-step ks are fetched; before the last k-step of a slot
    // (its fragments are in registers by then) come the wait for tile t + 1 and the workgroup barrier, and during that
    // last k-step the fragments of (t + 1, k-step 0) are fetched and the copies of tile t + NS - 1 are started.
    if (nk > 0) {
#pragma unroll
      for (int t = 0; t < NS - 1; t++) {
        const CopyJob j = next_job();
#pragma unroll
        for (int c = 0; c < L; c++) copy_one(j, c);
      }
      wait_vmem<(NS - 2) * L>();              // tile 0 has landed (this wave's share)
      __syncthreads();
      first_fragments();
      for (int t = 0; t < nk; t++) {
        lds_u8* const cur = lds + (t % NS) * STAGE_BYTES;
#pragma unroll
        for (int ks = 1; ks < KSTEPS; ks++) {
          if (ks & 1) region(fa0, fb0, fa1, fb1, cur, ks, nullptr);
          else region(fa1, fb1, fa0, fb0, cur, ks, nullptr);
        }
        wait_vmem<(NS - 3) * L>();            // tile t+1 has landed (this wave's share)
        __syncthreads();                      // everyone's share of t+1 landed; everyone is done with tile t-1
        const CopyJob j = next_job();         // tile t + NS - 1
        __builtin_amdgcn_sched_barrier(0);
        region(fa1, fb1, fa0, fb0, lds + ((t + 1) % NS) * STAGE_BYTES, 0, &j);
      }
      wait_vmem<0>();                         // drain the (empty) copies issued past the end
    }
  } else {
    // 64-deep slots, two of them: four k-steps per iteration.  The barrier sits before the last k-step: by then every
    // wave has fetched its last fragments of slot t (they are multiplied from registers in the last k-step), so the
    // barrier both publishes slot t+1 and frees slot t for tile t+2.
    // That refill is issued in two halves: one in the k-step after the barrier, one in the first k-step of the next
    // iteration (it still has three k-steps to land), so the texture path sees no burst of 16 copies per wave.
    // Invariant at the top of iteration t: tile t is landed or fully in flight, the first half of tile t+1 is in
    // flight and j is the job of tile t+1.
    if (nk > 0) {
      {
        const CopyJob j0 = next_job();
#pragma unroll
        for (int c = 0; c < L; c++) copy_one(j0, c);
      }
      CopyJob j = next_job();
#pragma unroll
      for (int c = 0; c < L / 2; c++) copy_one(j, c);
      wait_vmem<L / 2>();                     // tile 0 has landed (this wave's share)
      __syncthreads();
      first_fragments();
      for (int t = 0; t < nk; t++) {
        lds_u8* const cur = lds + (t & 1) * STAGE_BYTES;
        lds_u8* const nxt = lds + ((t + 1) & 1) * STAGE_BYTES;
        region(fa0, fb0, fa1, fb1, cur, 1, &j, L / 2, L, 0);
        region(fa1, fb1, fa0, fb0, cur, 2, nullptr);
        region(fa0, fb0, fa1, fb1, cur, 3, nullptr);
        wait_vmem<0>();                       // tile t+1 has landed (this wave's share)
        __syncthreads();
        j = next_job();                       // tile t + 2 into the slot of tile t
        __builtin_amdgcn_sched_barrier(0);
        region(fa1, fb1, fa0, fb0, nxt, 0, &j, 0, L / 2, 0);
      }
      wait_vmem<0>();
    }
  }

  // ---- epilogue.  Accumulator element e of a 32x32 tile sits at row 8*(e/4) + 4*(lane/32) + e%4, column lane%32:
  // a lane owns single elements of many rows.  Each wave therefore passes its tile through LDS one 32-row strip at
  // a time (the ring is free by now) and reads it back row-major, so that every lane stores 16 contiguous bytes
  // and a wave-wide store covers whole rows of the tile.
  __syncthreads();                          // every wave is done with the ring
  OutT* C = reinterpret_cast<OutT*>(p.C) + zo * p.sCo + zi * p.sCi;
  const bf16_t* R = reinterpret_cast<const bf16_t*>(p.R);
  if (R) R += zo * p.sCo + zi * p.sCi;
  constexpr int SW = WN + 4;                // strip row stride in floats
  typedef LDS_AS float lds_f32;
  lds_f32* const strip = reinterpret_cast<lds_f32*>(lds + wave * (32 * SW * 4));
  static_assert(4 * 32 * SW * 4 <= NS * STAGE_BYTES, "strips must fit in the ring");
  constexpr int V = sizeof(OutT) == 4 ? 4 : 8;          // elements per 16-byte store
  // A strip is 32 rows of LPR 16-byte vectors; vector q (row q / LPR) is stored by lane q % 64 in pass q / 64, so
  // a wave-wide store covers whole rows when LPR divides 64 and consecutive rows otherwise (WN = 96).
  constexpr int LPR = WN / V, NVEC = 32 * LPR;
  static_assert(NVEC % 64 == 0, "a strip must be a whole number of wave-wide stores");
  if constexpr (sizeof(OutT) == 4 && !ACC) {
    // fp32 goes out as it lies in the accumulators: 32 lanes are 32 consecutive floats of a row, a whole cache line, so the way
    // through LDS below would gain no larger pieces.  All weight gradients of a 7B layer, K 512 297 -> 288 us, K 1024 450 -> 437,
    // K 2048 730 -> 719; of four MLP blocks of d 2048, K 2048 508 -> 497.
    const bool whole = m0 + BM <= p.M && n0 + BN <= p.N;
    const int row0 = m0 + wm * WM + 4 * (lane >> 5), col0 = n0 + wn * WN + (lane & 31);
    float* const out = reinterpret_cast<float*>(C) + (long)row0 * p.ldc + col0;
    if (whole) {
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int e = 0; e < 16; e++) {
          float* const row = out + (long)(i * 32 + 8 * (e >> 2) + (e & 3)) * p.ldc;
#pragma unroll
          for (int j = 0; j < TN; j++) row[j * 32] = p.alpha * acc[i][j][e];
        }
    } else {
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int e = 0; e < 16; e++) {
          const int r = i * 32 + 8 * (e >> 2) + (e & 3);
          float* const row = out + (long)r * p.ldc;
#pragma unroll
          for (int j = 0; j < TN; j++)
            if (row0 + r < p.M && col0 + j * 32 < p.N) row[j * 32] = p.alpha * acc[i][j][e];
        }
    }
    return;
  }
  // fp32 +=: the old value that store u of strip i adds is requested where store u of strip i - 1 has used its own, so a
  // whole strip of requests is in flight (without branches: lanes outside the output read the tile's first element).
  // Read in place, one at a time, they made an accumulating round of 256 large tiles 22 us longer than an overwriting one;
  // now 14.  [4096, 22016] x 256 (128 x 128 tiles) 260 -> 198 us, x 1024 374 -> 321, [2048, 11008] x 2048 141 -> 121 (with the
  // tile that is chosen now 193, 303, 108).
  constexpr int OLD = ACC ? NVEC / 64 : 1;
  static_assert(!ACC || sizeof(OutT) == 4, "only an fp32 output accumulates");
  u32x4 old[OLD];
  auto request_old = [&](int i, int u) {
    const int q = u * 64 + lane;
    const int grow = m0 + wm * WM + i * 32 + q / LPR, gcol = n0 + wn * WN + (q % LPR) * V;
    const bool in = grow < p.M && gcol < p.N;
    old[u] = *reinterpret_cast<const u32x4*>(C + (in ? (long)grow * p.ldc + gcol : (long)m0 * p.ldc + n0));
  };
  if constexpr (ACC) {
#pragma unroll
    for (int u = 0; u < OLD; u++) request_old(0, u);
  }
#pragma unroll
  for (int i = 0; i < TM; i++) {
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int e = 0; e < 16; e++)
        strip[(8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)) * SW + j * 32 + (lane & 31)] = p.alpha * acc[i][j][e];
    // what the strip needs from memory (old C for +=, residual or probabilities) is requested for the whole strip
    // first, so the stores below wait for one memory latency per strip instead of one per row group
    constexpr int NIT = NVEC / 64;                            // stores per strip, and per request batch:
    constexpr int GRP = NIT <= 8 ? NIT : (NIT % 8 == 0 ? 8 : (NIT % 6 == 0 ? 6 : (NIT % 5 == 0 ? 5 : 4)));
    static_assert(NIT % GRP == 0, "request batches must tile the strip");
    const bool need_pre = (sizeof(OutT) == 4) ? false : (R != nullptr);
    __builtin_amdgcn_sched_barrier(0);      // keep the next strip's requests from being hoisted over this one
#pragma unroll
    for (int g0 = 0; g0 < NIT; g0 += GRP) {
      u32x4 pre[GRP];
      float dl[GRP];
#pragma unroll
      for (int u = 0; u < GRP; u++) {
        const int q = (g0 + u) * 64 + lane;
        const int grow = m0 + wm * WM + i * 32 + q / LPR, gcol = n0 + wn * WN + (q % LPR) * V;
        if (need_pre && grow < p.M && gcol < p.N) {
          const long idx = (long)grow * p.ldc + gcol;
          pre[u] = *reinterpret_cast<const u32x4*>(R + idx);
          if (p.delta) dl[u] = p.delta[zo * p.sDo + zi * p.sDi + (long)grow * p.ldd];
        }
      }
#pragma unroll
      for (int u = 0; u < GRP; u++) {
        const int qv = (g0 + u) * 64 + lane;
        const int r = qv / LPR, sc = (qv % LPR) * V;
        const int grow = m0 + wm * WM + i * 32 + r, gcol = n0 + wn * WN + sc;
        if (grow < p.M && gcol < p.N) {     // N is a multiple of 8: a vector is inside or outside as a whole
          const long idx = (long)grow * p.ldc + gcol;
          float v[V];
#pragma unroll
          for (int q = 0; q < V; q += 4) {
            const f32x4 t4 = *reinterpret_cast<LDS_AS const f32x4*>(strip + r * SW + sc + q);
            v[q] = t4[0]; v[q + 1] = t4[1]; v[q + 2] = t4[2]; v[q + 3] = t4[3];
          }
          if constexpr (sizeof(OutT) == 4) {
            if constexpr (ACC) {
#pragma unroll
              for (int q = 0; q < 4; q++) v[q] += __uint_as_float(old[g0 + u][q]);
            }
            f32x4 w4;
            w4[0] = v[0]; w4[1] = v[1]; w4[2] = v[2]; w4[3] = v[3];
            *reinterpret_cast<f32x4*>(C + idx) = w4;
          } else {
            if (p.delta) {                  // dS = P * (dP - delta[row]); zero above the diagonal
#pragma unroll
              for (int q = 0; q < 4; q++) {
                const float p0 = __uint_as_float(pre[u][q] << 16), p1 = __uint_as_float(pre[u][q] & 0xffff0000u);
                v[2 * q] = (!p.delta_causal || gcol + 2 * q <= grow) ? p0 * (v[2 * q] - dl[u]) : 0.f;
                v[2 * q + 1] = (!p.delta_causal || gcol + 2 * q + 1 <= grow) ? p1 * (v[2 * q + 1] - dl[u]) : 0.f;
              }
            } else if (R) {
#pragma unroll
              for (int q = 0; q < 4; q++) {
                v[2 * q] += __uint_as_float(pre[u][q] << 16);
                v[2 * q + 1] += __uint_as_float(pre[u][q] & 0xffff0000u);
              }
            }
            bf16x8 o;
#pragma unroll
            for (int q = 0; q < 8; q++) o[q] = (bf16_t)v[q];
            *reinterpret_cast<bf16x8*>(C + idx) = o;
          }
        }
        if constexpr (ACC) {
          if (i + 1 < TM) request_old(i + 1, g0 + u);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

template <int BM, int BN, bool AKC, bool BKC, typename OutT, int KD, int RING = 0, bool ACC = false>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(GemmParams p) {
  int tm_i, tn_i, z = (int)blockIdx.z;
  if (gridDim.z == 1) {
    tile_of_block(blockIdx.x, p.tiles_m, p.tiles_n, tm_i, tn_i);
  } else {
    // Batched (per-head) products.  The hardware hands consecutive workgroup ids (x fastest, then z) to the 8 XCDs in
    // turn, and each XCD has its own L2: with the plain id -> (tile, batch entry) map the tiles of one batch entry,
    // which share its operands, would be spread over all 8 XCDs and every L2 would fetch those operands again.  When
    // the batch count is a multiple of 8 the map is therefore regrouped so that an XCD walks whole batch entries; a
    // causal contraction that grows with the tile row starts with the longest tiles of each entry.
    const int nt = (int)gridDim.x;
    int id;
    if ((gridDim.z & 7) == 0) {
      const int lin = (int)blockIdx.x + nt * (int)blockIdx.z;
      const int xcd = lin & 7, j = lin >> 3;
      z = xcd + 8 * (j / nt);
      id = j % nt;
      if (p.causal == CAUSAL_K_END) id = nt - 1 - id;
    } else {
      // otherwise rotating the map by the batch index at least keeps one XCD from getting all the long tiles
      id = ((int)blockIdx.x + 3 * z) % nt;
    }
    if (p.causal == CAUSAL_SKIP_UPPER && p.tiles_m == p.tiles_n && p.causal_fill <= BM) {
      // only the lower-triangular tiles are launched: id = tm (tm + 1) / 2 + tn
      tm_i = (int)((__builtin_sqrtf(8.f * (float)id + 1.f) - 1.f) * 0.5f);
      while (tm_i * (tm_i + 1) / 2 > id) tm_i--;
      while ((tm_i + 1) * (tm_i + 2) / 2 <= id) tm_i++;
      tn_i = id - tm_i * (tm_i + 1) / 2;
    } else {
      tm_i = id % p.tiles_m;
      tn_i = id / p.tiles_m;
    }
  }
  gemm_bf16_tile<BM, BN, AKC, BKC, OutT, KD, false, RING, ACC>(p, tm_i, tn_i, z);
}

// Batched product with a causal contraction end (rows of tile i contract over (i + 1) * BM indices) and one tile column:
// a workgroup takes tile nt - 1 - i and then tile i, so every workgroup does the same amount of work, nt + 1 units,
// there are half as many of them (each pays its start-up once per two tiles' worth of streaming) and no compute unit
// is left with a long tile at the end.  Batch entries are regrouped by XCD as in gemm_bf16_kernel.
template <int BM, int BN, bool AKC, bool BKC, typename OutT, int KD>
__global__ __launch_bounds__(256) void gemm_bf16_causal_pair_kernel(GemmParams p) {
  const int np = (int)gridDim.x, nt = p.tiles_m;              // np = ceil(nt / 2) workgroups per batch entry
  int z = (int)blockIdx.z, id = (int)blockIdx.x;
  if ((gridDim.z & 7) == 0) {
    const int lin = (int)blockIdx.x + np * (int)blockIdx.z;
    const int xcd = lin & 7, j = lin >> 3;
    z = xcd + 8 * (j / np);
    id = j % np;
  }
  const int reps = (nt - 1 - id > id) ? 2 : 1;                // the middle tile of an odd count stands alone
  for (int r = 0; r < reps; r++) {
    gemm_bf16_tile<BM, BN, AKC, BKC, OutT, KD>(p, r == 0 ? nt - 1 - id : id, 0, z);
    __syncthreads();                          // every wave has read its strip back: the ring may be refilled
  }
}

// Storage-type NN / NT products with waves of their own for the copies; WGS workgroups share a compute unit.
template <int BM, int BN, bool BKC, int RING, int WGS>
__global__ __launch_bounds__(512, 2 * WGS) void gemm_bf16_copiers_kernel(GemmParams p) {
  int tm_i, tn_i;
  tile_of_block(blockIdx.x, p.tiles_m, p.tiles_n, tm_i, tn_i);
  gemm_bf16_tile<BM, BN, true, BKC, bf16_t, 64, false, RING, false, true>(p, tm_i, tn_i, 0);
}
template <int BM, int BN, bool BKC, int RING, int WGS>
__global__ __launch_bounds__(512, 2 * WGS) void gemm_bf16_copiers_split_kernel(GemmParams p) {
  int tm_i, tn_i, slice;
  tile_of_block_split(blockIdx.x, p.tiles_m, p.tiles_n, p.split, tm_i, tn_i, slice);
  gemm_bf16_tile<BM, BN, true, BKC, float, 64, true, RING, false, true>(p, tm_i, tn_i, slice);
}

// One workgroup per (tile, slice of the contraction); the fp32 partial products are added up by split_sum_kernel.
template <int BM, int BN, bool AKC, bool BKC, int KD, int RING>
__global__ __launch_bounds__(256) void gemm_bf16_split_kernel(GemmParams p) {
  int tm_i, tn_i, slice;
  tile_of_block_split(blockIdx.x, p.tiles_m, p.tiles_n, p.split, tm_i, tn_i, slice);
  gemm_bf16_tile<BM, BN, AKC, BKC, float, KD, true, RING>(p, tm_i, tn_i, slice);
}

constexpr int kSmallSlots = 4;                 // ring slots per wave of the small-output kernel
constexpr int kPairSlots = 3;                  // the same with two images of B per slot

// d(silu(gate) * up) for an output derivative v
__device__ __forceinline__ void swiglu_backward(float v, float gate, float up, float& dgate, float& dup) {
  const float s = 1.f / (1.f + __expf(-gate));
  dgate = v * up * s * (1.f + gate * (1.f - s));
  dup = v * gate * s;
}

// Outputs of at most one 32 x 32 tile per compute unit (storage-type NN / NT products of short micro-batches).  What bounds
// such a product is latency: a workgroup has few slots to walk, and every barrier and every slot that is not yet in flight
// adds to them.  The four waves of a workgroup share one 32 x 32 tile and take the 64-deep slots of the contraction in
// turn, each through a ring of its own that it fills with its own copies: no barrier until the waves' partial sums meet in
// the LDS (added in wave order), and 12 slots on their way at once.
// Measured against 64 x 64 tiles (us): [128, 256] x 256 4.2 -> 3.7, x 768 6.0 -> 4.2, x 1376 8.4 -> 4.7, [256, 1024] x 5504
// 14.5 -> 11.9, [64, 4096] x 4096 22 -> 11; at more than one tile per compute unit it loses ([200, 1536] x 512 5.4 -> 6.9).
template <bool BKC, bool SWIGLU>
__global__ __launch_bounds__(256) void gemm_bf16_small_kernel(GemmParams p) {
  using TA = OperandTile<32, true, 64>;
  using TB = OperandTile<32, BKC, 64>;
  constexpr int KD = 64, NS = kSmallSlots, L = 8;
  static_assert(TA::BYTES == 4096 && TB::BYTES == 4096 && (NS - 2) * L < 64, "slot layout, wait counter");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  lds_u8* const lds = LDS_PTR(unsigned char, smem_raw);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  lds_u8* const ring = lds + wave * (NS * 8192);
  const uint32_t ring0 = (uint32_t)(uintptr_t)lds + wave * (NS * 8192);

  int tm_i, tn_i;
  tile_of_block(blockIdx.x, p.tiles_m, p.tiles_n, tm_i, tn_i);
  const int m0 = tm_i * 32, n0 = tn_i * 32;
  const bf16_t* A = reinterpret_cast<const bf16_t*>(p.A);
  const bf16_t* B = reinterpret_cast<const bf16_t*>(p.B);

  unsigned a_goff[4], b_goff[4];
  int a_kidx[4], b_kidx[4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    TA::copy_plan(i, lane, p.lda, m0, p.M, a_goff[i], a_kidx[i]);
    TB::copy_plan(i, lane, p.ldb, n0, p.N, b_goff[i], b_kidx[i]);
  }
  const long b_kstep = BKC ? 1 : p.ldb;
  const int k0 = wave * KD;                   // this wave's slots: k0, k0 + 4 KD, ...
  uint64_t a_next = reinterpret_cast<uint64_t>(A + (long)m0 * p.lda + k0);
  uint64_t b_next = reinterpret_cast<uint64_t>((BKC ? B + (long)n0 * p.ldb : B + n0) + (long)k0 * b_kstep);
  int slot_next = 0, krem = p.K - k0;
  const int nk = krem > 0 ? (krem + 4 * KD - 1) / (4 * KD) : 0;
  auto issue = [&]() {                        // past the end: every lane out of range, zeros, no traffic
    const u32x4 dA = make_desc(reinterpret_cast<const void*>(a_next)), dB = make_desc(reinterpret_cast<const void*>(b_next));
    const uint32_t base = ring0 + slot_next * 8192;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      dma16(base + i * 1024, dA, a_kidx[i] < krem ? a_goff[i] : kOob);
      dma16(base + 4096 + i * 1024, dB, b_kidx[i] < krem ? b_goff[i] : kOob);
    }
    a_next += (uint64_t)(4 * KD * 2);
    b_next += (uint64_t)(4 * KD * b_kstep * 2);
    slot_next = slot_next + 1 == NS ? 0 : slot_next + 1;
    krem -= 4 * KD;
  };
  const int col = n0 + (lane & 31);
  float gate[4], up[4];
  if constexpr (SWIGLU) {                     // what the epilogue reads, requested before everything else
    const bf16_t* const gu = reinterpret_cast<const bf16_t*>(p.gu);
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int row = m0 + 8 * wave + 4 * (lane >> 5) + q;
      const long idx = row < p.M && col < p.N ? (long)row * p.ldc + col : 0;
      gate[q] = (float)gu[idx];
      up[q] = (float)gu[idx + p.N];
    }
  }
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; e++) acc[e] = 0.f;
  if (nk > 0) {
#pragma unroll
    for (int t = 0; t < NS - 1; t++) issue();
    for (int t = 0; t < nk; t++) {
      wait_vmem<(NS - 2) * L>();              // this wave's slot t has landed
      asm volatile("" ::: "memory");          // (its fragments must not be fetched earlier)
      __builtin_amdgcn_sched_barrier(0);
      lds_u8* const ia = ring + (t % NS) * 8192;
      lds_u8* const ib = ia + 4096;
      issue();                                // slot t + NS - 1 in the place of slot t - 1, whose fragments have been used
      bf16x8 fa[4], fb[4];
#pragma unroll
      for (int v = 0; v < 4; v++) {
        fa[v] = read_frag<32, true>(ia + TA::frag_base(lane, 0, TA::variant(v, 0)) + TA::frag_step(v, 0));
        fb[v] = read_frag<32, BKC>(ib + TB::frag_base(lane, 0, TB::variant(v, 0)) + TB::frag_step(v, 0));
      }
      __builtin_amdgcn_sched_barrier(0);    // (all fetched before the first MFMA, one LDS latency per slot)
#pragma unroll
      for (int v = 0; v < 4; v++) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[v], fb[v], acc, 0, 0, 0);
    }
    wait_vmem<0>();                           // (the empty copies issued past the end)
  }
  __syncthreads();                            // every wave is done with its ring
  LDS_AS float* const part = reinterpret_cast<LDS_AS float*>(lds);
#pragma unroll
  for (int e = 0; e < 16; e++) part[(wave * 16 + e) * 64 + lane] = acc[e];
  __syncthreads();
  // each wave adds up and stores 8 rows: registers 4 w .. 4 w + 3 are rows 8 w + 4 (lane / 32) + 0..3
  const bf16_t* R = reinterpret_cast<const bf16_t*>(p.R);
  bf16_t* C = reinterpret_cast<bf16_t*>(p.C);
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const int e = 4 * wave + q, row = m0 + 8 * wave + 4 * (lane >> 5) + q;
    float v = part[e * 64 + lane];
#pragma unroll
    for (int w = 1; w < 4; w++) v += part[(w * 16 + e) * 64 + lane];
    if (row >= p.M || col >= p.N) continue;
    const long idx = (long)row * p.ldc + col;
    v *= p.alpha;
    if constexpr (SWIGLU) {
      float dg, du;
      swiglu_backward(v, gate[q], up[q], dg, du);
      C[idx] = (bf16_t)dg;
      C[idx + p.N] = (bf16_t)du;
      continue;
    }
    if (R) v += (float)R[idx];
    C[idx] = (bf16_t)v;
  }
}

// The same for a product whose columns c and c + (a fixed distance) go into one result: gate and up of the SwiGLU (the distance
// is the FFN width), or the two halves of a head that the rotary embedding turns (half the head width).  A workgroup takes 32
// columns and their 32 partners, a lane holds both, and what would be a launch of its own over [rows, columns] becomes a few
// instructions here, on values that have not been rounded yet.  Launches are what a micro-batch this small costs: SwiGLU and
// rotation were 2.8 of 72 us each in a layer of d 256, f 688 on 128 tokens.
__global__ __launch_bounds__(256) void gemm_bf16_pairs_kernel(GemmParams p) {
  using TA = OperandTile<32, true, 64>;
  using TB = OperandTile<32, false, 64>;
  constexpr int KD = 64, NS = kPairSlots, L = 12, SLOT = 12288;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  lds_u8* const lds = LDS_PTR(unsigned char, smem_raw);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  lds_u8* const ring = lds + wave * (NS * SLOT);
  const uint32_t ring0 = (uint32_t)(uintptr_t)lds + wave * (NS * SLOT);
  int tm_i, tn_i;
  tile_of_block(blockIdx.x, p.tiles_m, p.tiles_n, tm_i, tn_i);
  const PairEpilogue& pe = p.pair;
  // first column (its partner is `distance` further) and the end of the first columns of this group (a head, or all gate columns)
  const int m0 = tm_i * 32, group = tn_i * 32 / pe.distance;
  const int n0 = tn_i * 32 + group * pe.distance, n_end = (2 * group + 1) * pe.distance;
  const bf16_t* A = reinterpret_cast<const bf16_t*>(p.A);
  const bf16_t* B = reinterpret_cast<const bf16_t*>(p.B);
  unsigned a_goff[4], b_goff[4];
  int a_kidx[4], b_kidx[4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    TA::copy_plan(i, lane, p.lda, m0, p.M, a_goff[i], a_kidx[i]);
    TB::copy_plan(i, lane, p.ldb, n0, n_end, b_goff[i], b_kidx[i]);
  }
  const int k0 = wave * KD;                   // this wave's slots: k0, k0 + 4 KD, ...
  uint64_t a_next = reinterpret_cast<uint64_t>(A + (long)m0 * p.lda + k0);
  uint64_t b_next = reinterpret_cast<uint64_t>(B + n0 + (long)k0 * p.ldb);
  int slot_next = 0, krem = p.K - k0;
  const int nk = krem > 0 ? (krem + 4 * KD - 1) / (4 * KD) : 0;
  auto issue = [&]() {                        // past the end: every lane out of range, zeros, no traffic
    const u32x4 dA = make_desc(reinterpret_cast<const void*>(a_next)), dB = make_desc(reinterpret_cast<const void*>(b_next)),
                dP = make_desc(reinterpret_cast<const void*>(b_next + (uint64_t)pe.distance * 2));
    const uint32_t base = ring0 + slot_next * SLOT;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      dma16(base + i * 1024, dA, a_kidx[i] < krem ? a_goff[i] : kOob);
      dma16(base + 4096 + i * 1024, dB, b_kidx[i] < krem ? b_goff[i] : kOob);
      dma16(base + 8192 + i * 1024, dP, b_kidx[i] < krem ? b_goff[i] : kOob);
    }
    a_next += (uint64_t)(4 * KD * 2);
    b_next += (uint64_t)(4 * KD * p.ldb * 2);
    slot_next = slot_next + 1 == NS ? 0 : slot_next + 1;
    krem -= 4 * KD;
  };
  f32x16 acc[2];
#pragma unroll
  for (int e = 0; e < 16; e++) { acc[0][e] = 0.f; acc[1][e] = 0.f; }
  if (nk > 0) {
#pragma unroll
    for (int t = 0; t < NS - 1; t++) issue();
    for (int t = 0; t < nk; t++) {
      wait_vmem<(NS - 2) * L>();              // this wave's slot t has landed
      asm volatile("" ::: "memory");          // (its fragments must not be fetched earlier)
      __builtin_amdgcn_sched_barrier(0);
      lds_u8* const ia = ring + (t % NS) * SLOT;
      issue();                                // slot t + NS - 1 in the place of slot t - 1, whose fragments have been used
      bf16x8 fa[4], fb[4], fp[4];
#pragma unroll
      for (int v = 0; v < 4; v++) {
        fa[v] = read_frag<32, true>(ia + TA::frag_base(lane, 0, TA::variant(v, 0)) + TA::frag_step(v, 0));
        fb[v] = read_frag<32, false>(ia + 4096 + TB::frag_base(lane, 0, TB::variant(v, 0)) + TB::frag_step(v, 0));
        fp[v] = read_frag<32, false>(ia + 8192 + TB::frag_base(lane, 0, TB::variant(v, 0)) + TB::frag_step(v, 0));
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int v = 0; v < 4; v++) {
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[v], fb[v], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[v], fp[v], acc[1], 0, 0, 0);
      }
    }
    wait_vmem<0>();                           // (the empty copies issued past the end)
  }
  __syncthreads();                            // every wave is done with its ring
  LDS_AS float* const part = reinterpret_cast<LDS_AS float*>(lds);
#pragma unroll
  for (int h = 0; h < 2; h++)
#pragma unroll
    for (int e = 0; e < 16; e++) part[((h * 4 + wave) * 16 + e) * 64 + lane] = acc[h][e];
  __syncthreads();
  bf16_t* C = reinterpret_cast<bf16_t*>(p.C);
  const int col = n0 + (lane & 31);
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const int e = 4 * wave + q, row = m0 + 8 * wave + 4 * (lane >> 5) + q;
    float v[2];
#pragma unroll
    for (int h = 0; h < 2; h++) {
      v[h] = part[(h * 64 + e) * 64 + lane];
#pragma unroll
      for (int w = 1; w < 4; w++) v[h] += part[((h * 4 + w) * 16 + e) * 64 + lane];
    }
    if (row >= p.M || col >= n_end) continue;
    const long idx = (long)row * p.ldc + col;
    if (pe.m) {
      reinterpret_cast<bf16_t*>(pe.m)[(long)row * pe.distance + col] = (bf16_t)(v[0] / (1.f + __expf(-v[0])) * v[1]);
    } else if (group < pe.rotated) {
      const float2 t = pe.rope[(long)(row % pe.seq) * pe.distance + (col - 2 * group * pe.distance)];
      const float x = v[0], y = v[1];
      v[0] = x * t.x - y * t.y;
      v[1] = x * t.y + y * t.x;
    }
    C[idx] = (bf16_t)v[0];
    C[idx + pe.distance] = (bf16_t)v[1];
  }
}

// C = bf16(sum over the slices of parts[slice][M][N] (+ R)), slices added in order.
__global__ __launch_bounds__(256) void split_sum_kernel(const float* __restrict__ parts, int split, int M, int N,
                                                        const bf16_t* __restrict__ R, bf16_t* __restrict__ C, long ldc) {
  const int nv = N / 8;
  const long v = blockIdx.x * 256L + threadIdx.x;
  if (v >= (long)M * nv) return;
  const long row = v / nv, col = (v - row * nv) * 8, idx = row * ldc + col, step = (long)M * N;
  const float* q = parts + row * N + col;
  u32x4 r = {0, 0, 0, 0};
  if (R) r = *reinterpret_cast<const u32x4*>(R + idx);
  f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
#pragma unroll 4
  for (int i = 0; i < split; i++) {
    a += *reinterpret_cast<const f32x4*>(q + i * step);
    b += *reinterpret_cast<const f32x4*>(q + i * step + 4);
  }
  float o[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
  bf16x8 w;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    w[2 * i] = (bf16_t)(o[2 * i] + __uint_as_float(r[i] << 16));
    w[2 * i + 1] = (bf16_t)(o[2 * i + 1] + __uint_as_float(r[i] & 0xffff0000u));
  }
  *reinterpret_cast<bf16x8*>(C + idx) = w;
}

// Several independent weight-gradient products (TN layout, fp32 output) in one launch: the tiles of all products form
// one sequence of workgroups, so the compute units that run out of tiles of one product start on the next one
// instead of idling until the slowest tile of a round has finished, and there is one launch instead of one per weight.
// Each product's first workgroup id is a multiple of 8, which keeps the id -> XCD correspondence that the tile map
// relies on; the surplus ids do nothing.
// This pays for short contractions.  For long ones it loses: the 32 tiles an XCD runs at
// a time share operand panels through its L2 only while they walk the contraction in step, which they do when a
// launch starts them together and stop doing once tiles of different products and start times are mixed.
// Tiles of 256 x 256 and 128 x 128 run on a ring of four 32-deep slots (one workgroup per compute unit, and two), 64 x 64
// on four 64-deep ones (two).
template <int TILE, bool ACC>
__global__ __launch_bounds__(256) void gemm_tn_grouped_kernel(GroupedTable g) {
  int lo = 0, hi = g.n - 1;                   // last product whose first workgroup id is <= blockIdx.x
  const int bid = (int)blockIdx.x;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (g.first_block[mid] <= bid) lo = mid; else hi = mid - 1;
  }
  const GroupedProduct& q = g.prod[lo];
  const int pid = bid - g.first_block[lo];
  const int tiles_m = (q.M + TILE - 1) / TILE, tiles_n = (q.N + TILE - 1) / TILE;
  if (pid >= tiles_m * tiles_n) return;
  GemmParams p{};
  p.A = q.A; p.B = q.B; p.C = q.C;
  p.lda = q.lda; p.ldb = q.ldb; p.ldc = q.ldc;
  p.M = q.M; p.N = q.N; p.K = q.K;
  p.batch_inner = 1; p.tiles_m = tiles_m; p.tiles_n = tiles_n;
  p.alpha = 1.f; p.causal = CAUSAL_NONE;
  int tm_i, tn_i;
  tile_of_block(pid, tiles_m, tiles_n, tm_i, tn_i);
  gemm_bf16_tile<TILE, TILE, false, false, float, (TILE == 64 ? 64 : 32), false, (TILE == 64 ? 4 : 0), ACC>(p, tm_i, tn_i, 0);
}

// ------------------------------------------------------------------------------------------ ceiling
// Register-resident MFMA loop: 4 waves per compute unit, 16 independent 32x32x16 bf16 MFMAs per iteration on
// operands that never leave the registers.  It measures what the matrix pipes sustain under the chip's power
// management with no memory system involved: the practical ceiling the GEMM kernel is compared with.
__global__ __launch_bounds__(256) void mfma_ceiling_kernel(int iters, const bf16_t* __restrict__ seed,
                                                           float* __restrict__ sink) {
  const int lane = threadIdx.x & 63;
  bf16x8 a[4], b[4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    a[i] = *reinterpret_cast<const bf16x8*>(seed + (size_t)(i * 64 + lane) * 8);
    b[i] = *reinterpret_cast<const bf16x8*>(seed + (size_t)((4 + i) * 64 + lane) * 8);
  }
  f32x16 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int j = 0; j < 4; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;
  for (int it = 0; it < iters; it++) {
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
      for (int j = 0; j < 4; j++)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
  }
  float t = 0.f;
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int j = 0; j < 4; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) t += acc[i][j][e];
  sink[(size_t)blockIdx.x * 256 + threadIdx.x] = t;
}

hipError_t mfma_ceiling(int blocks, int iters, const void* seed, float* sink, hipStream_t s) {
  hipLaunchKernelGGL(mfma_ceiling_kernel, dim3(blocks), dim3(256), 0, s, iters, (const bf16_t*)seed, sink);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------ fp32
// fp32 products on the 32x32x2 fp32 MFMA instruction (inputs and accumulation in full fp32).
//
// What bounds it: one such MFMA multiplies 32 x 32 x 2 in 64 clocks (256 FLOP per clock and compute unit), so a matrix
// pipe needs 16 bytes of operands from the LDS per 64 clocks and nothing about the LDS is critical; what matters is that
// all 4 x 256 pipes have a tile to work on and that the copies are far enough ahead.
// The kernel is the bf16 one's little sister: operands arrive in the LDS by asynchronous copies, in a ring of NS slots
// of KD contraction indices, one barrier per slot.  A 16-byte LDS read is 4 consecutive contraction indices of a row:
// lane half g holds indices 8 v + 4 g + j, j = 0..3, and MFMA j of the four that follow multiplies indices {8 v + j,
// 8 v + 4 + j}; an operand that is strided in the contraction index is read one float per MFMA in the same order.
// With WK = 4 the four waves share one 32 x 32 tile and split every slot's contraction between them (their sums meet in
// the LDS at the end, added in wave order): small outputs then still give every matrix pipe work.
// Measured against the FMA kernel that ran these products before: [512, 1024] x 5504 (NT) 990 -> 63 us, [256, 256] x 688
// 126 -> 10 us with the launch; [4096, 4096] x 4096 reaches 138-140 TFLOP/s of the 157 that the instruction allows.
template <int R, bool KC, int KD>
struct OperandTileF32 {
  static constexpr int BYTES = R * KD * 4, CHUNKS = BYTES / 1024, PER_WAVE = CHUNKS / 4;
  static constexpr int GR = KD / 4;                 // KC: 16-byte granules per image row [R][KD]
  static constexpr int GPR = R / 4;                 // KS: granules per image row [KD][R]
  static constexpr int RPB = GR >= 16 ? 1 : 16 / GR;
  static_assert(CHUNKS % 4 == 0, "tile must split evenly over 4 waves");
  // KC: granule g of row r sits in slot g ^ (r / RPB) % GR (16 rows at one granule touch all 16 bank groups).
  static __device__ __forceinline__ int kc_swz(int row) { return (row / RPB) & (GR - 1); }
  // KS: image row `pos` holds contraction index ks_k(pos), so the two indices that one MFMA multiplies (8 v + j and
  // 8 v + 4 + j) are neighbours; rows of 256 bytes or more swap their 128-byte halves on odd positions so that the two
  // lane halves of a read never meet in a bank.
  static __device__ __forceinline__ int ks_k(int pos) { return (pos & ~7) | ((pos & 1) << 2) | ((pos >> 1) & 3); }
  static __device__ __forceinline__ constexpr int ks_flip(int pos) { return R >= 64 ? (pos & 1) << 3 : 0; }
  static __device__ __forceinline__ void copy_plan(int c, int p, long ld, int origin, int extent, unsigned& goff, int& kidx) {
    const int P = 64 * c + p;
    if constexpr (KC) {
      const int row = P / GR, g = (P % GR) ^ kc_swz(row);
      goff = (origin + row < extent) ? (unsigned)((long)row * ld * 4 + g * 16) : kOob;
      kidx = g * 4;
    } else {
      const int pos = P / GPR, g = (P % GPR) ^ ks_flip(pos), k = ks_k(pos);
      goff = (origin + g * 4 < extent) ? (unsigned)((long)k * ld * 4 + g * 16) : kOob;
      kidx = k;
    }
  }
  // the 4 contraction indices 8 v + 4 (lane / 32) + 0..3 of row r0 + lane % 32
  static __device__ __forceinline__ f32x4 frag(lds_u8* img, int lane, int r0, int v) {
    if constexpr (KC) {
      const int row = r0 + (lane & 31);
      return *reinterpret_cast<LDS_AS const f32x4*>(img + row * (KD * 4) + (((2 * v + (lane >> 5)) ^ kc_swz(row)) << 4));
    } else {
      const int g = lane >> 5, col = (r0 + (lane & 31)) ^ (ks_flip(g) * 4);
      LDS_AS const float* const q = reinterpret_cast<LDS_AS const float*>(img) + (8 * v + g) * R + col;
      f32x4 o;
#pragma unroll
      for (int j = 0; j < 4; j++) o[j] = q[2 * j * R];
      return o;
    }
  }
};

template <int BM, int BN, bool AKC, bool BKC, int WK, int KD, int NS, bool SWIGLU>
__global__ __launch_bounds__(256) void gemm_f32_mfma_kernel(GemmParams p) {
  using TA = OperandTileF32<BM, AKC, KD>;
  using TB = OperandTileF32<BN, BKC, KD>;
  constexpr int SW = WK == 4 ? 1 : 2;               // waves along each side of the tile
  constexpr int TM = BM / (32 * SW), TN = BN / (32 * SW);
  constexpr int NA = TA::PER_WAVE, NB = TB::PER_WAVE, L = NA + NB, SLOT = TA::BYTES + TB::BYTES;
  static_assert(WK == 1 || (WK == 4 && TM == 1 && TN == 1), "wave arrangement");
  static_assert(KD % (8 * WK) == 0 && NS >= 2 && (NS - 2) * L < 64, "slot depth, wait counter");

  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  lds_u8* const lds = LDS_PTR(unsigned char, smem_raw);
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = WK == 4 ? 0 : wave >> 1, wn = WK == 4 ? 0 : wave & 1, wk = WK == 4 ? wave : 0;

  int tm_i, tn_i;
  if (gridDim.z == 1) tile_of_block(blockIdx.x, p.tiles_m, p.tiles_n, tm_i, tn_i);
  else { tm_i = (int)blockIdx.x % p.tiles_m; tn_i = (int)blockIdx.x / p.tiles_m; }
  const int m0 = tm_i * BM, n0 = tn_i * BN;
  int k_lo = 0, k_hi = p.K;
  if (p.causal == CAUSAL_SKIP_UPPER) {
    bool empty;
    if (tile_skipped<BM>(p, m0, n0, empty)) return;
    if (empty) k_hi = 0;
  } else if (p.causal == CAUSAL_K_END) {
    k_hi = (m0 + BM < p.K) ? m0 + BM : p.K;
  } else if (p.causal == CAUSAL_K_BEGIN) {
    k_lo = m0;
  }
  const int nk = k_hi > k_lo ? (k_hi - k_lo + KD - 1) / KD : 0;
  const int z = blockIdx.z;
  const int zo = z / p.batch_inner, zi = z - zo * p.batch_inner;
  const float* A = reinterpret_cast<const float*>(p.A) + zo * p.sAo + zi * p.sAi;
  const float* B = reinterpret_cast<const float*>(p.B) + zo * p.sBo + zi * p.sBi;

  unsigned a_goff[NA], b_goff[NB];
  int a_kidx[NA], b_kidx[NB];
#pragma unroll
  for (int i = 0; i < NA; i++) TA::copy_plan(wave + 4 * i, lane, p.lda, m0, p.M, a_goff[i], a_kidx[i]);
#pragma unroll
  for (int i = 0; i < NB; i++) TB::copy_plan(wave + 4 * i, lane, p.ldb, n0, p.N, b_goff[i], b_kidx[i]);
  const long a_kstep = AKC ? 1 : p.lda, b_kstep = BKC ? 1 : p.ldb;
  uint64_t a_next = reinterpret_cast<uint64_t>((AKC ? A + (long)m0 * p.lda : A + m0) + (long)k_lo * a_kstep);
  uint64_t b_next = reinterpret_cast<uint64_t>((BKC ? B + (long)n0 * p.ldb : B + n0) + (long)k_lo * b_kstep);
  int slot_next = 0, krem = k_hi - k_lo;
  // Copies of the next slot.  Past the end every lane is redirected out of range: zeros, no memory traffic, and the
  // number of operations in flight stays uniform.
  auto issue = [&]() {
    const u32x4 dA = make_desc(reinterpret_cast<const void*>(a_next)), dB = make_desc(reinterpret_cast<const void*>(b_next));
    const uint32_t base = lds0 + slot_next * SLOT + wave * 1024;
#pragma unroll
    for (int i = 0; i < NA; i++) dma16(base + i * 4096, dA, a_kidx[i] < krem ? a_goff[i] : kOob);
#pragma unroll
    for (int i = 0; i < NB; i++) dma16(base + TA::BYTES + i * 4096, dB, b_kidx[i] < krem ? b_goff[i] : kOob);
    a_next += (uint64_t)(KD * a_kstep * 4);
    b_next += (uint64_t)(KD * b_kstep * 4);
    slot_next = slot_next + 1 == NS ? 0 : slot_next + 1;
    krem -= KD;
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;

  if (nk > 0) {
#pragma unroll
    for (int t = 0; t < NS - 1; t++) issue();
    for (int t = 0; t < nk; t++) {
      wait_vmem<(NS - 2) * L>();              // slot t has landed (this wave's share)
      __syncthreads();                        // ... everyone's share; everyone is done with slot t - 1
      issue();                                // slot t + NS - 1 in the place of slot t - 1
      lds_u8* const ia = lds + (t % NS) * SLOT;
      lds_u8* const ib = ia + TA::BYTES;
#pragma unroll
      for (int u = 0; u < KD / 8 / WK; u++) {
        const int v = u * WK + wk;
        f32x4 fa[TM], fb[TN];
#pragma unroll
        for (int i = 0; i < TM; i++) fa[i] = TA::frag(ia, lane, (wm * TM + i) * 32, v);
#pragma unroll
        for (int j = 0; j < TN; j++) fb[j] = TB::frag(ib, lane, (wn * TN + j) * 32, v);
#pragma unroll
        for (int q = 0; q < 4; q++)
#pragma unroll
          for (int i = 0; i < TM; i++)
#pragma unroll
            for (int j = 0; j < TN; j++)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][q], fb[j][q], acc[i][j], 0, 0, 0);
      }
    }
    wait_vmem<0>();                           // (the empty copies issued past the end)
  }
  if constexpr (WK > 1) {                     // the waves' partial tiles, added in wave order; one quarter of the rows each
    __syncthreads();
    LDS_AS float* const part = reinterpret_cast<LDS_AS float*>(lds);
    static_assert(WK * 1024 * 4 <= NS * SLOT, "the partial tiles must fit in the ring");
#pragma unroll
    for (int e = 0; e < 16; e++) part[(wk * 16 + e) * 64 + lane] = acc[0][0][e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 16; e++) acc[0][0][e] = 0.f;
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int e = 4 * wave + q;             // registers 4 w .. 4 w + 3 = rows 8 w + 4 (lane / 32) + 0..3
      float s = part[e * 64 + lane];
#pragma unroll
      for (int w = 1; w < WK; w++) s += part[(w * 16 + e) * 64 + lane];
      acc[0][0][q] = s;
    }
  }
  // ---- epilogue: a wave-wide store is two rows of 32 consecutive floats
  float* C = reinterpret_cast<float*>(p.C) + zo * p.sCo + zi * p.sCi;
  const float* R = reinterpret_cast<const float*>(p.R);
  if (R) R += zo * p.sCo + zi * p.sCi;
  const float* const delta = p.delta ? p.delta + zo * p.sDo + zi * p.sDi : nullptr;
  constexpr int NE = WK > 1 ? 4 : 16;               // registers of an MFMA tile that this wave stores
  auto row_of = [&](int i, int e) {
    return m0 + (wm * TM + i) * 32 + (WK > 1 ? 8 * wave + 4 * (lane >> 5) + e : 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3));
  };
  // What an epilogue reads (old values, a residual, or the probabilities and delta of the softmax backward) is requested for a
  // whole MFMA tile at a time: one value at a time, between stores that the compiler must take to alias the next load, old
  // values made an accumulating [2616, 4084] x 64 product 66 us (now 38), and P and delta the 16 x [512, 512] x 64 product of a
  // score gradient 40 us (now 15).  The overwriting kernel keeps a branch of its own: sharing this one cost it 20-30 %.
  if constexpr (SWIGLU) {                           // gate and up in, their derivatives out
    const float* const gu = reinterpret_cast<const float*>(p.gu);
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) {
        const int col = n0 + (wn * TN + j) * 32 + (lane & 31);
        float gate[NE], up[NE];
#pragma unroll
        for (int e = 0; e < NE; e++) {
          const int row = row_of(i, e);
          const long idx = row < p.M && col < p.N ? (long)row * p.ldc + col : 0;
          gate[e] = gu[idx];
          up[e] = gu[idx + p.N];
        }
#pragma unroll
        for (int e = 0; e < NE; e++) {
          const int row = row_of(i, e);
          float dg, du;
          swiglu_backward(p.alpha * acc[i][j][e], gate[e], up[e], dg, du);
          if (row < p.M && col < p.N) {
            C[(long)row * p.ldc + col] = dg;
            C[(long)row * p.ldc + col + p.N] = du;
          }
        }
      }
    return;
  }
  if ((p.accumulate || R) && !(p.accumulate && R && !delta)) {
    const float* const src = R ? R : C;
#pragma unroll
    for (int i = 0; i < TM; i++) {
      float dl[NE];
      if (delta) {
#pragma unroll
        for (int e = 0; e < NE; e++) {
          const int row = row_of(i, e);
          dl[e] = delta[(long)(row < p.M ? row : m0) * p.ldd];
        }
      }
#pragma unroll
      for (int j = 0; j < TN; j++) {
        const int col = n0 + (wn * TN + j) * 32 + (lane & 31);
        float old[NE];
#pragma unroll
        for (int e = 0; e < NE; e++) {              // (without branches: outside the output the tile's first element)
          const int row = row_of(i, e);
          old[e] = src[row < p.M && col < p.N ? (long)row * p.ldc + col : (long)m0 * p.ldc + n0];
        }
#pragma unroll
        for (int e = 0; e < NE; e++) {
          const int row = row_of(i, e);
          const float v = p.alpha * acc[i][j][e];
          if (row < p.M && col < p.N)
            C[(long)row * p.ldc + col] = !delta ? old[e] + v : (!p.delta_causal || col <= row) ? old[e] * (v - dl[e]) : 0.f;
        }
      }
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++) {
      const int col = n0 + (wn * TN + j) * 32 + (lane & 31);
#pragma unroll
      for (int e = 0; e < NE; e++) {
        const int row = row_of(i, e);
        if (row >= p.M || col >= p.N) continue;
        const long idx = (long)row * p.ldc + col;
        float v = p.alpha * acc[i][j][e];
        if (p.accumulate) {
          v += C[idx];
          v += R[idx];
        }
        C[idx] = v;
      }
    }
}

// Outputs of at most two 16 x 16 tiles per compute unit.  What bounds such a product on 32 x 32 tiles is the chain of MFMAs
// itself (64 clocks per two indices, and a quarter of the contraction per wave): a quarter of the tile is a quarter of the
// chain (the 16x16x4 MFMA takes 32 clocks per four indices) on four times as many workgroups.  As in the bf16 kernel for
// small outputs the four waves take the slots of the contraction (32 indices, 2 KiB per operand) in turn, each through a
// ring of its own, with no barrier until their partial sums meet in the LDS (added in wave order).
// Lane group g = lane / 16 holds contraction indices 16 v + 4 g + j, j = 0..3 (one 16-byte read where they are contiguous),
// and MFMA j of the four that follow multiplies the indices 16 v + {0, 4, 8, 12} + j; an operand that is strided in the
// contraction index keeps the four indices of one MFMA in neighbouring image rows (64 bytes each: no bank conflicts).
// Measured against 32 x 32 tiles (us): [256, 256] x 256 4.7 -> 3.3, x 768 7.2 -> 4.0, x 1376 10.6 -> 5.3, [64, 1024] x 2752
// 19.2 -> 9.5; at three tiles per compute unit it loses ([256, 688] x 256 4.7 -> 5.9, [256, 768] x 256 4.9 -> 6.3).
template <bool KC>
struct SmallTileF32 {
  static __device__ __forceinline__ void copy_plan(int c, int p, long ld, int origin, int extent, unsigned& goff, int& kidx) {
    const int P = 64 * c + p;
    if constexpr (KC) {                       // [16 rows][32]: granule g of row r in slot g ^ (r / 2) % 8
      const int row = P / 8, g = (P % 8) ^ ((row >> 1) & 7);
      goff = (origin + row < extent) ? (unsigned)((long)row * ld * 4 + g * 16) : kOob;
      kidx = g * 4;
    } else {                                  // [32][16 columns]
      const int pos = P / 4, g = P % 4, k = (pos & ~15) | ((pos & 3) << 2) | ((pos >> 2) & 3);
      goff = (origin + g * 4 < extent) ? (unsigned)((long)k * ld * 4 + g * 16) : kOob;
      kidx = k;
    }
  }
  static __device__ __forceinline__ f32x4 frag(lds_u8* img, int lane, int v) {
    const int row = lane & 15, g = lane >> 4;
    if constexpr (KC) {
      return *reinterpret_cast<LDS_AS const f32x4*>(img + row * 128 + (((4 * v + g) ^ ((row >> 1) & 7)) << 4));
    } else {
      LDS_AS const float* const q = reinterpret_cast<LDS_AS const float*>(img) + (16 * v + g) * 16 + row;
      f32x4 o;
#pragma unroll
      for (int j = 0; j < 4; j++) o[j] = q[64 * j];
      return o;
    }
  }
};

template <bool AKC, bool BKC, bool SWIGLU>
__global__ __launch_bounds__(256) void gemm_f32_small_kernel(GemmParams p) {
  using TA = SmallTileF32<AKC>;
  using TB = SmallTileF32<BKC>;
  constexpr int KD = 32, NS = kSmallSlots, L = 4, SLOT = 4096;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  lds_u8* const lds = LDS_PTR(unsigned char, smem_raw);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  lds_u8* const ring = lds + wave * (NS * SLOT);
  const uint32_t ring0 = (uint32_t)(uintptr_t)lds + wave * (NS * SLOT);

  int tm_i, tn_i;
  if (gridDim.z == 1) tile_of_block(blockIdx.x, p.tiles_m, p.tiles_n, tm_i, tn_i);
  else { tm_i = (int)blockIdx.x % p.tiles_m; tn_i = (int)blockIdx.x / p.tiles_m; }
  const int m0 = tm_i * 16, n0 = tn_i * 16;
  int k_lo = 0, k_hi = p.K;
  if (p.causal == CAUSAL_SKIP_UPPER) {
    bool empty;                               // (uniform over the workgroup)
    if (tile_skipped<16>(p, m0, n0, empty)) return;
    if (empty) k_hi = 0;
  } else if (p.causal == CAUSAL_K_END) {
    k_hi = (m0 + 16 < p.K) ? m0 + 16 : p.K;
  } else if (p.causal == CAUSAL_K_BEGIN) {
    k_lo = m0;
  }
  const int z = blockIdx.z;
  const int zo = z / p.batch_inner, zi = z - zo * p.batch_inner;
  const float* A = reinterpret_cast<const float*>(p.A) + zo * p.sAo + zi * p.sAi;
  const float* B = reinterpret_cast<const float*>(p.B) + zo * p.sBo + zi * p.sBi;

  unsigned a_goff[2], b_goff[2];
  int a_kidx[2], b_kidx[2];
#pragma unroll
  for (int i = 0; i < 2; i++) {
    TA::copy_plan(i, lane, p.lda, m0, p.M, a_goff[i], a_kidx[i]);
    TB::copy_plan(i, lane, p.ldb, n0, p.N, b_goff[i], b_kidx[i]);
  }
  const long a_kstep = AKC ? 1 : p.lda, b_kstep = BKC ? 1 : p.ldb;
  const int k0 = k_lo + wave * KD;            // this wave's slots: k0, k0 + 4 KD, ...
  uint64_t a_next = reinterpret_cast<uint64_t>((AKC ? A + (long)m0 * p.lda : A + m0) + (long)k0 * a_kstep);
  uint64_t b_next = reinterpret_cast<uint64_t>((BKC ? B + (long)n0 * p.ldb : B + n0) + (long)k0 * b_kstep);
  int slot_next = 0, krem = k_hi - k0;
  const int nk = krem > 0 ? (krem + 4 * KD - 1) / (4 * KD) : 0;
  auto issue = [&]() {                        // past the end: every lane out of range, zeros, no traffic
    const u32x4 dA = make_desc(reinterpret_cast<const void*>(a_next)), dB = make_desc(reinterpret_cast<const void*>(b_next));
    const uint32_t base = ring0 + slot_next * SLOT;
#pragma unroll
    for (int i = 0; i < 2; i++) {
      dma16(base + i * 1024, dA, a_kidx[i] < krem ? a_goff[i] : kOob);
      dma16(base + 2048 + i * 1024, dB, b_kidx[i] < krem ? b_goff[i] : kOob);
    }
    a_next += (uint64_t)(4 * KD * a_kstep * 4);
    b_next += (uint64_t)(4 * KD * b_kstep * 4);
    slot_next = slot_next + 1 == NS ? 0 : slot_next + 1;
    krem -= 4 * KD;
  };
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (nk > 0) {
#pragma unroll
    for (int t = 0; t < NS - 1; t++) issue();
    for (int t = 0; t < nk; t++) {
      wait_vmem<(NS - 2) * L>();              // this wave's slot t has landed
      asm volatile("" ::: "memory");          // (its fragments must not be fetched earlier)
      __builtin_amdgcn_sched_barrier(0);
      lds_u8* const ia = ring + (t % NS) * SLOT;
      issue();                                // slot t + NS - 1 in the place of slot t - 1, whose fragments have been used
      f32x4 fa[2], fb[2];
#pragma unroll
      for (int v = 0; v < 2; v++) { fa[v] = TA::frag(ia, lane, v); fb[v] = TB::frag(ia + 2048, lane, v); }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int v = 0; v < 2; v++)
#pragma unroll
        for (int j = 0; j < 4; j++) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[v][j], fb[v][j], acc, 0, 0, 0);
    }
    wait_vmem<0>();                           // (the empty copies issued past the end)
  }
  __syncthreads();                            // every wave is done with its ring
  LDS_AS float* const part = reinterpret_cast<LDS_AS float*>(lds);
#pragma unroll
  for (int e = 0; e < 4; e++) part[(wave * 4 + e) * 64 + lane] = acc[e];
  __syncthreads();
  // wave w adds up and stores register w of the tile: rows 4 (lane / 16) + w
  float v = part[wave * 64 + lane];
#pragma unroll
  for (int w = 1; w < 4; w++) v += part[(w * 4 + wave) * 64 + lane];
  const int row = m0 + 4 * (lane >> 4) + wave, col = n0 + (lane & 15);
  if (row >= p.M || col >= p.N) return;
  float* const C = reinterpret_cast<float*>(p.C) + zo * p.sCo + zi * p.sCi;
  const float* const R = p.R ? reinterpret_cast<const float*>(p.R) + zo * p.sCo + zi * p.sCi : nullptr;
  const long idx = (long)row * p.ldc + col;
  v *= p.alpha;
  if constexpr (SWIGLU) {
    const float* const gu = reinterpret_cast<const float*>(p.gu);
    float dg, du;
    swiglu_backward(v, gu[idx], gu[idx + p.N], dg, du);
    C[idx] = dg;
    C[idx + p.N] = du;
    return;
  }
  if (p.delta) {
    v = (!p.delta_causal || col <= row) ? R[idx] * (v - p.delta[zo * p.sDo + zi * p.sDi + (long)row * p.ldd]) : 0.f;
  } else {
    if (p.accumulate) v += C[idx];
    if (R) v += R[idx];
  }
  C[idx] = v;
}

// The general fp32 product, for operands that the copies above cannot move in 16-byte pieces:
// 64 x 64 x 16 tile, 256 threads, 4 x 4 outputs per thread; operands addressed through element strides so
// one kernel serves NN, NT and TN.
template <typename OutT>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmParams p) {
  constexpr int TB = 64, TK = 16;
  __shared__ float As[TK][TB + 4];
  __shared__ float Bs[TK][TB + 4];
  const int tid = threadIdx.x;
  const int tx = tid & 15, ty = tid >> 4;
  const int tm_i = blockIdx.x / p.tiles_n, tn_i = blockIdx.x - tm_i * p.tiles_n;
  const int m0 = tm_i * TB, n0 = tn_i * TB;
  int k_lo = 0, k_hi = p.K;
  if (p.causal == CAUSAL_SKIP_UPPER) {
    bool empty;
    if (tile_skipped<TB>(p, m0, n0, empty)) return;
    if (empty) k_hi = 0;
  } else if (p.causal == CAUSAL_K_END) {
    k_hi = (m0 + TB < p.K) ? m0 + TB : p.K;
  } else if (p.causal == CAUSAL_K_BEGIN) {
    k_lo = m0;
  }
  const int z = blockIdx.z;
  const int zo = z / p.batch_inner, zi = z - zo * p.batch_inner;
  const float* A = reinterpret_cast<const float*>(p.A) + zo * p.sAo + zi * p.sAi;
  const float* B = reinterpret_cast<const float*>(p.B) + zo * p.sBo + zi * p.sBi;
  float acc[4][4] = {};
  for (int k0 = k_lo; k0 < k_hi; k0 += TK) {
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const int e = tid + 256 * i;            // 1024 elements of each tile
      // A tile: consecutive threads along the contiguous direction of the layout
      int am, ak, bn, bk;
      if (p.sak == 1) { ak = e & 15; am = e >> 4; } else { am = e & 63; ak = e >> 6; }
      if (p.sbn == 1) { bn = e & 63; bk = e >> 6; } else { bk = e & 15; bn = e >> 4; }
      const bool aok = (m0 + am < p.M) && (k0 + ak < k_hi);
      const bool bok = (n0 + bn < p.N) && (k0 + bk < k_hi);
      As[ak][am] = aok ? A[(long)(m0 + am) * p.sam + (long)(k0 + ak) * p.sak] : 0.f;
      Bs[bk][bn] = bok ? B[(long)(k0 + bk) * p.sbk + (long)(n0 + bn) * p.sbn] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < TK; k++) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; i++) a[i] = As[k][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; j++) b[j] = Bs[k][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
  OutT* C = reinterpret_cast<OutT*>(p.C) + zo * p.sCo + zi * p.sCi;
  const float* R = reinterpret_cast<const float*>(p.R);
  if (R) R += zo * p.sCo + zi * p.sCi;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int row = m0 + ty * 4 + i;
    if (row >= p.M) continue;
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const int col = n0 + tx * 4 + j;
      if (col >= p.N) continue;
      const long idx = (long)row * p.ldc + col;
      float v = p.alpha * acc[i][j];
      if (p.delta) {
        const float dl = p.delta[zo * p.sDo + zi * p.sDi + (long)row * p.ldd];
        v = (!p.delta_causal || col <= row) ? R[idx] * (v - dl) : 0.f;
      } else {
        if (p.accumulate) v += C[idx];
        if (R) v += R[idx];
      }
      C[idx] = v;
    }
  }
}

// ------------------------------------------------------------------------------------------ host
template <int BM, int BN, bool AKC, bool BKC, typename OutT, int KD, int RING, bool ACC>
static hipError_t launch_bf16_acc(const GemmParams& p0, int batch, hipStream_t s) {
  GemmParams p = p0;
  p.tiles_m = (p.M + BM - 1) / BM;
  p.tiles_n = (p.N + BN - 1) / BN;
  constexpr size_t smem = (size_t)(RING >= 3 ? RING : (KD == 32 ? STAGES : 2)) * (BM + BN) * KD * sizeof(bf16_t);
  static_assert(smem <= 160 * 1024, "LDS budget of one gfx950 compute unit");
  auto kern = gemm_bf16_kernel<BM, BN, AKC, BKC, OutT, KD, RING, ACC>;
  static AttrOnce once;
  if (hipError_t e = once.set(reinterpret_cast<const void*>(kern), smem); e != hipSuccess) return e;
  unsigned nt = (unsigned)(p.tiles_m * p.tiles_n);
  if (batch > 1 && p.causal == CAUSAL_SKIP_UPPER && p.tiles_m == p.tiles_n && p.causal_fill <= BM)
    nt = (unsigned)(p.tiles_m * (p.tiles_m + 1) / 2);       // lower-triangular tiles only
  dim3 grid(nt, 1, (unsigned)batch);
  hipLaunchKernelGGL(kern, grid, dim3(256), smem, s, p);
  return hipGetLastError();
}
template <int BM, int BN, bool AKC, bool BKC, typename OutT, int KD, int RING = 0>
static hipError_t launch_bf16(const GemmParams& p, int batch, hipStream_t s) {
  if constexpr (sizeof(OutT) == 4)
    if (p.accumulate) return launch_bf16_acc<BM, BN, AKC, BKC, OutT, KD, RING, true>(p, batch, s);
  return launch_bf16_acc<BM, BN, AKC, BKC, OutT, KD, RING, false>(p, batch, s);
}

template <int BM, int BN, bool AKC, bool BKC, typename OutT, int KD>
static hipError_t launch_bf16_causal_pair(const GemmParams& p0, int batch, hipStream_t s) {
  GemmParams p = p0;
  p.tiles_m = (p.M + BM - 1) / BM;
  p.tiles_n = (p.N + BN - 1) / BN;
  if (p.tiles_n != 1 || p.causal != CAUSAL_K_END) return hipErrorInvalidValue;
  constexpr size_t smem = (size_t)(KD == 32 ? STAGES : 2) * (BM + BN) * KD * sizeof(bf16_t);
  auto kern = gemm_bf16_causal_pair_kernel<BM, BN, AKC, BKC, OutT, KD>;
  static AttrOnce once;
  if (hipError_t e = once.set(reinterpret_cast<const void*>(kern), smem); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)((p.tiles_m + 1) / 2), 1, (unsigned)batch), dim3(256), smem, s, p);
  return hipGetLastError();
}

// Tile and number of contraction slices of a storage-type NN / NT product (the linear layers of forward and backward-p1)
// whose output is at most one round of 256 x 256 tiles.  Two models of a product's time, fitted to different data:
// `coarse_plan` knows six tiles, with constants of its own for up to 128 rows, and errs little where it errs; `product_time` knows all
// of them and more of what a product's time depends on.  The plan is the coarse one unless the other model has a choice that it
// holds for 4 to 30 % faster, depending on how well it knows the two.  On 3900 products (M 16-4096, N 128-27648, K 64-27648, weights that no
// cache holds) the coarse one alone costs 2.5 % more than the fastest of all tiles and slices on average, `product_time` alone 0.7 % with
// a tail of 1.3-fold misses ([16, 2560] x 3264 (NN) 13.4 us for 9.6).  On 3717 products (M 64-4096, N and K 256-12288; weights from HBM / from
// the cache) the plan with scratch costs 1.5 / 1.4 % more than the fastest, the coarse one 4.6 / 3.9 %; against the 4-wave kernels and the
// coarse plan of before it is 5.8 / 6.4 % faster on average and more than 6 % slower on 3 / 15.
// us, with the 4-wave kernels and the coarse plan that were here / now: [256, 22016] x 4096 (NN) 71 / 58 (128 x 192), [360, 4096] x 11008
// (NT) 54 / 47 (192 x 192 in five slices), [256, 4096] x 4096 (NN) 19.6 / 16.7 (64 x 64), [2000, 1152] x 3456 (NT) 27.3 / 23.6 (128 x 128), [1024, 4096] x 11008 (NN)
// 90 / 87.
enum ProductTile { T32, T64, T128X64, T128, T128_PAIR, T128X192, T256X128, T192, T256_NARROW, T256 };
struct TileCost {
  int bm, bn, per_cu;
  double index, fixed;          // us per contraction index of a full round, and per round
  double idle;                  // per_cu 1: share of `index` that an empty chip saves; per_cu 2: us per index of two workgroups
  double nn, nt, start;         // TB/s at which the operands are fetched, by layout, and us
  double overlap;               // us by which a round beyond the first starts early
  double half_b, half_a;        // extra time per index for rows of B, of A (NN) that are no multiple of 64
  double sum, sum_mb;           // us for the sum of the slices, and per MB of partial products
  double second;                // per_cu 2: share of the second workgroup's time that the first compute units with two add
};
static const TileCost kTileCost[] = {
    {32, 32, 1, 0.00174, 3.33, 0.309, 4.78, 14.0, 2.68, 5.93, 0.278, 0.270, 5.35, 0.230, 0.},        // no slices
    {64, 64, 2, 0.00327, 3.74, 0.00805, 5.48, 8.70, 0.694, 1.39, 0.229, 0.0826, 2.03, 0.347, 1.},
    {128, 64, 1, 0.00533, 4.77, 0.358, 4.60, 10.6, 1.91, 1.63, 0.232, 0.195, 1.89, 0.266, 0.},
    {128, 128, 1, 0.00791, 5.21, 0.425, 6.21, 8.46, 1.83, 2.22, 0.201, 0.0773, 1.77, 0.272, 0.},
    {128, 128, 2, 0.00979, 4.51, 0.0187, 4.67, 14.0, 1.87, 0.515, 0.110, 0.0414, 1.65, 0.306, 0.837},
    {128, 192, 1, 0.0106, 6.66, 0.379, 6.27, 10.0, 4.52, 0.747, 0.196, 0.0480, 1.76, 0.264, 0.},
    {256, 128, 1, 0.0122, 8.65, 0.438, 13.9, 10.0, 5.13, 1.60, 0.149, 0.134, 1.64, 0.206, 0.},
    {192, 192, 1, 0.0140, 9.81, 0.340, 7.18, 10.5, 5.69, 1.35, 0.113, 0.0303, 1.56, 0.199, 0.},
    {256, 192, 1, 0.0193, 9.71, 0.478, 4.72, 13.0, 15.0, 0., 0.183, 0.0324, 2.25, 0.131, 0.},
    {256, 256, 1, 0.0241, 11.6, 0.413, 5.99, 7.64, 15.0, 0.142, 0.0678, 0.0832, 1.50, 0.140, 0.}};

// A round of 256 workgroups (one per compute unit; 512 with two) costs its contraction indices and a fixed part, less per index
// where compute units stay idle (the others' copies then go faster), and no less than reading both operands once (of the
// shorter of these two times an eighth shows).  A row length that is no multiple of 64 puts every 128-byte piece of a tile row
// across two cache lines.  Slices add a second launch and the partial products.
static double product_time(const TileCost& t, int layout, int M, int N, int K, long n, int slice, int split) {
  const double slower = 1. + ((layout == NN ? N : K) % 64 ? t.half_b : 0.) + (layout == NN && K % 64 ? t.half_a : 0.);
  // 256 x 128 tiles: long slices run at the power limit, which the tile that fetches the most bytes for its size meets first.  Time over what
  // the rest of the model says, slices of 2-4 K / 4-6 / 6-8 / 8-12 / over 12 K indices: 0.87 / 0.98 / 1.02 / 1.05 / 1.12, NT with rows at
  // multiples of less than 64 bytes 0.98 / 1.03 / 1.14 / 1.25 / 1.25-1.44; 256 x 256 tiles go from 0.93 to 1.0 ([592, 10616] x 10248 (NT)
  // 203 us, in two slices of 256 x 256 170; [2304, 3328] x 28416 (NN) 392 and 365).
  const double late = &t != &kTileCost[T256X128] || slice <= 4096 ? 1. : 1. + (layout == NT && K % 32 ? 0.25 : 0.12) * fmin(1., (slice - 4096) / 4096.);
  const double work = slice * t.index * slower * late;
  double time;
  if (t.per_cu == 1) {
    const long rest = n % 256;
    const double last = work * (1. - t.idle * (1. - (double)(n <= 256 ? n : rest) / 256)) + t.fixed;
    time = n <= 256 ? last : (double)(n / 256) * (work + t.fixed) + (rest ? last : 0.) - (double)((n - 1) / 256) * t.overlap;
  } else {
    const long rest = n % 512;
    const double one = work + t.fixed, two = slice * t.idle * slower + t.fixed;
    time = (double)(n / 512) * two - (n > 512 ? (double)((n - 1) / 512) * t.overlap : 0.);
    if (rest) time += rest <= 256 ? one : one + (two - one) * (t.second + (1. - t.second) * (double)(rest - 256) / 256);
  }
  const double memory = 2e-6 * ((double)N * K + (double)M * K) / (layout == NN ? t.nn : t.nt) * (1. + 0.5 * (slower - 1.)) + t.start;
  time = time > memory ? time + 0.12 * memory : memory + 0.12 * time;
  return split > 1 ? 1.03 * (time + t.sum + t.sum_mb * 4e-6 * split * M * N) : time;
}
static const int kSlices[] = {1, 2, 3, 4, 5, 6, 8, 12, 16};
static SplitPlan slices_of(int tile, int M, int N, int K, int sp) {
  const int slice = sp == 1 ? K : ((K + 63) / 64 + sp - 1) / sp * 64, split = sp == 1 ? 1 : (K + slice - 1) / slice;
  return SplitPlan{tile, split, slice, split > 1 ? kSplitHead + (size_t)split * M * N * sizeof(float) : 0};
}
static long tiles_of(int tile, int M, int N) {
  const TileCost& t = kTileCost[tile];
  return (long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
}
// The coarse model, in us.  Its constants are those of kernels without copying waves, which the tiles up to 128 x 128 ran on before:
// they price a product too high there, by a factor that differs little between these tiles.  Fitted to 2500 (shape, tile,
// slices) triples, M 64-2048, N 256-22016, K 256-22016: a round of 256 workgroups of
// K / slices indices costs `one` per index (`two` with two workgroups on a compute unit) and a fixed part, but at least the time
// of reading both operands once at 4.9 TB/s plus 8.4; slices add 3.8 and 0.30 per MB of partial products, and must gain 12 % (3 % up to 128 rows).
// Up to 128 rows the weight is read for one row of tiles, from HBM, and the tiles differ in the rate at which they
// fetch it: 5.9 TB/s on 128 x 128 tiles and 4.5 on 64 x 64 ones where its columns are contiguous (pieces of 256 and of 128 bytes),
// 4.9 on both where the contraction is; each has its own start (`start`, us), and rings of few slots take longer per index
// (`thin`).  Fitted to 510 products, M 8-128, N 256-24000, K 64-16000, weights that no cache holds.
// Rows of K that are no multiple of 64 cost the 64 x 64 tiles, which fetch the most per product, 8 % on a CU of their own and 38 %
// beside a second one.
static double coarse_time_of_32(int layout, int M, int N, int K) {
  return M > 128 ? 0.0018 * K + 3.0 : (layout == NN ? 0.0022 : 0.0014) * K + 2.9 + 0.26e-6 * N * K;
}
static SplitPlan coarse_plan(int layout, int M, int N, int K, bool allow_split) {
  struct Coarse { int tile; double one, two, fixed, thin, start; };
  static const Coarse tiles[] = {{T128, 0.0091, 0., 3.0, 1.04, 4.9}, {T256_NARROW, 0.0167, 0., 8.0, 0., 0.},
                                 {T256, 0.0197, 0., 9.7, 0., 0.}, {T128_PAIR, 0.0126, 0.0188, 1.5, 1.17, 5.4},
                                 {T64, 0.0047, 0.0071, 1.3, 1.3, 3.9}};
  const double bytes = 2e-6 * ((double)N * K + (double)M * K);
  const bool thin = M <= 128, nn = layout == NN, half_lines = K % 64 != 0;
  SplitPlan best = slices_of(T64, M, N, K, 1);
  double best_time = 1e30;
  if (tiles_of(T32, M, N) <= 256) {
    best_time = coarse_time_of_32(layout, M, N, K);
    best.tile = T32;
  }
  for (const Coarse& t : tiles) {
    if (kTileCost[t.tile].bm == 256 && M < 192) continue;
    const double per_index = thin ? t.thin : 1., memory = thin ? bytes / (!nn ? 4.9 : t.tile == T64 ? 4.5 : 5.9) + t.start : bytes / 4.9 + 8.4;
    for (int sp : kSlices) {
      if (sp > 1 && (!allow_split || K / sp < 256)) break;
      const SplitPlan plan = slices_of(t.tile, M, N, K, sp);
      const long n = tiles_of(t.tile, M, N) * plan.split;
      if (t.tile == T128_PAIR && n <= 256) continue;
      const bool slow = half_lines && t.tile == T64;
      const double one = plan.slice * t.one * per_index * (slow ? 1.08 : 1.) + t.fixed, two = plan.slice * t.two * per_index * (slow ? 1.38 : 1.) + t.fixed;
      double time;
      if (t.two == 0.) time = (double)((n + 255) / 256) * one;
      else time = (double)(n / 512) * two + (n % 512 == 0 ? 0. : n % 512 <= 256 ? one : two);
      time = (time < memory ? memory : time) + 0.02 * time;       // (equally memory-bound: the one that computes faster)
      if (plan.split > 1) time = (thin ? 1.03 : 1.12) * (time + 3.8 + 0.303e-6 * plan.split * M * N * sizeof(float));
      if (time < best_time) { best_time = time; best = plan; }
    }
  }
  return best;
}
static bool one_round(int M, int N) { return (long)((M + 255) / 256) * ((N + 255) / 256) <= 256; }
static SplitPlan search_plan(int layout, int M, int N, int K, bool allow_split) {
  const SplitPlan coarse = coarse_plan(layout, M, N, K, allow_split);
  SplitPlan best = coarse;
  const long coarse_wgs = tiles_of(coarse.tile, M, N) * coarse.split;
  double coarse_time = product_time(kTileCost[coarse.tile], layout, M, N, K, coarse_wgs, coarse.slice, coarse.split);
  // 32 x 32 tiles of few rows: the coarse model knows them better, those it chose ([24, 584] x 3912 (NT) 6.5 us, 9.9 modelled here, in eleven
  // slices of 64 x 64 8.4) as well as those in place of another choice ([72, 2240] x 5312 (NN) in the steps of an MLP 14.2 to 21.5 us, 13.0 modelled
  // here, 17.7 there; in six slices of 64 x 64 12.6 to 18.6 with their sum).
  if (coarse.tile == T32 && M <= 128) coarse_time = fmin(coarse_time, coarse_time_of_32(layout, M, N, K));
  const bool few_pairs = coarse.tile == T128_PAIR && coarse_wgs > 256 && coarse_wgs <= 288 && M > 850;
  // 64 x 64 tiles that it prices likewise (below) and that narrow outputs of split cache lines had better keep: N up to 256, time on the other
  // choice (128 x 64) over theirs 1.10-1.14 (K 1100-1400; from HBM 1.10), 1.06 (900-1100) and 1.06-1.10 (1400-1800); level or less for
  // other K, and for wider outputs (500 tall ones of 257 to 290 workgroups; [4648, 216] x 1552 (NT), 292 of them, 11.8 us and 13.6).
  // [5448, 192] x 1248 (NT) 10.4 us, on 128 x 64 13.5.
  if (coarse.tile == T64 && coarse.split == 1 && coarse_wgs > 256 && coarse_wgs <= 300 && N <= 256 && K % 64 && K >= 900 && K < 1800) return coarse;
  double best_time = 1e30;
  for (int i = T32; i <= T256; i++) {
    const TileCost& t = kTileCost[i];
    const long tiles = tiles_of(i, M, N);
    if (i == T32 && tiles > 256) continue;
    if (t.bm > 128 && M <= t.bm / 2) continue;
    if (i == T128X192 && layout == NT && K % 64) continue;        // (rows across two lines: up to 1.8 times the modelled time)
    for (int sp : kSlices) {
      if (sp > 1 && (!allow_split || i == T32 || K / sp < 256)) break;
      const SplitPlan plan = slices_of(i, M, N, K, sp);
      double time = product_time(t, layout, M, N, K, tiles * plan.split, plan.slice, plan.split);
      if (i == T32 && M <= 128) time = fmax(time, coarse_time_of_32(layout, M, N, K));
      // Its times of 32 x 32 tiles err most, those of the two largest of the new tiles least, but for up to 192 rows, where these are
      // mostly padding ([176, 9280] x 4160 (NN) 32.6 us on five slices of 192 x 192, modelled 32.3; 26.7 on 64 x 64, modelled 39.0; less so in NT,
      // [168, 9712] x 4440 on five such slices 1.2 times as fast as on 128 x 128).  Up to 128
      // rows the coarse plan is good, and 64 x 64 tiles that read a large weight unsliced in its place lose ([64, 11928] x 11320 (NT)
      // 100 us, two slices of 128 x 128 86).  Short slices on 256 x 128 are level with two 128 x 128 workgroups per compute unit where it
      // holds them for 7 % faster ([2032, 2624] x 848 (NT) 18.8 us and 18.4).
      // Where two 128 x 128 workgroups share up to 32 of the compute units, this model prices all of them like that: 257 to 288 workgroups
      // take 0.78 of its time (weights in the cache; 0.83 from HBM), 181 to 256 0.98 (1.11).  Outputs of more than 850 rows that leave them for 256 x 128
      // tiles modelled less than 25 % faster lose ([2496, 1592] x 1000 (NT) 18.5 us, modelled 24.0, on 256 x 128 20.7; 9 of 10 such by 1 to 10 %); lower ones,
      // and all that leave them for 128 x 192, gain.  (It prices 64 x 64 tiles likewise, but apart from narrow outputs, see above, 44 of 48 such
      // products that leave them are faster for it.)
      const double must = fmin(few_pairs && t.bm > 128 ? 0.75 : 1.,
                               coarse.tile == T32 ? 0.8 : M <= 128 ? (i == T64 && sp == 1 && coarse.tile != T64 ? 0.7 : 0.85)
                               : M <= 192 && t.bm >= 192 ? (layout == NN ? 0.8 : 0.9) : i == T256X128 && plan.slice < 1024 ? 0.85
                               : i == T256X128 || i == T192 ? 0.96 : 0.9);
      if (time < must * coarse_time && time < best_time) { best_time = time; best = plan; }
    }
  }
  return best;
}
// The search above costs 2 us of host time, a sixth of what a small product takes from call to call, and a program runs the same few
// products over and over: each thread keeps its last plans (a function of these five numbers alone), one per slot.  The plans of a product
// with and without scratch, which a workspace query and the call after it ask for in turn, have slots of their own (in one, they threw each
// other out: 3.1 us for the two, at worst 5.2, instead of 2.2).
static SplitPlan product_plan(int layout, int M, int N, int K, bool allow_split) {
  struct Slot { int layout, M, N, K; SplitPlan plan; };
  static thread_local Slot slots[2][128];                           // (M is 0 in a slot that holds nothing)
  uint32_t h = (uint32_t)M * 0x9E3779B1u + (uint32_t)N * 0x85EBCA6Bu + (uint32_t)K * 0xC2B2AE35u + (uint32_t)layout * 0x27D4EB2Fu;
  Slot& slot = slots[allow_split][(h ^ h >> 15) * 0x9E3779B1u >> 25];
  if (M <= 0 || slot.M != M || slot.N != N || slot.K != K || slot.layout != layout)
    slot = Slot{layout, M, N, K, search_plan(layout, M, N, K, allow_split)};
  return slot.plan;
}
// The plan where `ws_bytes` of scratch are at hand.
static SplitPlan plan_within(int layout, int M, int N, int K, size_t ws_bytes) {
  const SplitPlan plan = product_plan(layout, M, N, K, ws_bytes > 0);
  return plan.bytes > ws_bytes ? product_plan(layout, M, N, K, false) : plan;
}
SplitPlan gemm_split_plan(int dtype, int layout, int M, int N, int K, int out_f32, int batch) {
  const SplitPlan none{0, 1, 0, 0};
  if (dtype != 1 || out_f32 || batch != 1 || layout == TN || !one_round(M, N)) return none;
  const SplitPlan plan = product_plan(layout, M, N, K, true);
  return plan.split > 1 ? plan : none;
}

// What a caller is told to bring for one product.  A call that allocates its workspace and starts two kernels takes 14 us of host time
// and one without 10, so a product that is modelled to take less than 15.6 in one launch (16.7 on 32 x 32 tiles, less where the L2 holds the
// weight) is left whole unless the coarse model cuts it as well.  From call to call, us, in slices / whole: [160, 416] x 4168 (NN) 15 / 12,
// [136, 376] x 6696 (NT) 13.6 / 9.8, [176, 928] x 4712 (NN) 14.2 / 10.9; above the lines [280, 376] x 7048 (NN) 14.3 / 21.3, [312, 616] x 6296 (NN)
// 13.9 / 19.8.  Of 7400 drawn products 3 are slower for a workspace, and 7 that would gain more than 10 % by one go without.  (The stage, whose
// scratch is there in any case, goes by gemm_split_plan.)
size_t gemm_workspace_bytes(int dtype, int layout, int M, int N, int K, int out_f32) {
  const SplitPlan plan = gemm_split_plan(dtype, layout, M, N, K, out_f32, 1);
  if (plan.split == 1 || coarse_plan(layout, M, N, K, true).split > 1) return plan.bytes;
  const int whole = product_plan(layout, M, N, K, false).tile;
  const double time = product_time(kTileCost[whole], layout, M, N, K, tiles_of(whole, M, N), K, 1);
  return time < (whole == T32 ? 16.7 : 15.6) ? 0 : plan.bytes;
}
bool gemm_plan(int layout, int M, int N, int K, size_t ws_bytes, int* tile_rows, int* tile_cols, int* per_cu, int* slices) {
  if ((layout != NN && layout != NT) || M <= 0 || N <= 0 || !one_round(M, N)) return false;
  const SplitPlan plan = plan_within(layout, M, N, K, ws_bytes);
  const TileCost& t = kTileCost[plan.tile];
  *tile_rows = t.bm; *tile_cols = t.bn; *per_cu = t.per_cu; *slices = plan.split;
  return true;
}

template <bool BKC, bool SWIGLU = false>
static hipError_t launch_small(const GemmParams& p0, hipStream_t s) {
  GemmParams p = p0;
  p.tiles_m = (p.M + 31) / 32;
  p.tiles_n = (p.N + 31) / 32;
  constexpr size_t smem = (size_t)4 * kSmallSlots * 8192;
  auto kern = gemm_bf16_small_kernel<BKC, SWIGLU>;
  static AttrOnce once;
  if (hipError_t e = once.set(reinterpret_cast<const void*>(kern), smem); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)(p.tiles_m * p.tiles_n)), dim3(256), smem, s, p);
  return hipGetLastError();
}

template <int BM, int BN>
static GemmParams with_tiles(const GemmParams& p0) {
  GemmParams p = p0;
  p.tiles_m = (p.M + BM - 1) / BM;
  p.tiles_n = (p.N + BN - 1) / BN;
  return p;
}
// The slices of a product on `kern`, then their sum.
static hipError_t launch_slices(void (*kern)(GemmParams), unsigned threads, size_t smem, GemmParams p, const SplitPlan& plan, void* ws, hipStream_t s) {
  const void* const R = p.R;
  void* const C = p.C;
  const long ldc = p.ldc;
  p.split = plan.split; p.split_k = plan.slice;
  float* const parts = reinterpret_cast<float*>(static_cast<char*>(ws) + kSplitHead);
  p.C = parts; p.ldc = p.N; p.sCo = (long)p.M * p.N; p.sCi = 0; p.R = nullptr;
  p.sAo = p.sAi = p.sBo = p.sBi = 0;
  hipLaunchKernelGGL(kern, dim3((unsigned)(p.tiles_m * p.tiles_n * plan.split)), dim3(threads), smem, s, p);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  const long nv = (long)p.M * (p.N / 8);
  hipLaunchKernelGGL(split_sum_kernel, dim3((unsigned)((nv + 255) / 256)), dim3(256), 0, s, parts, plan.split, p.M, p.N,
                     static_cast<const bf16_t*>(R), static_cast<bf16_t*>(C), ldc);
  return hipGetLastError();
}

// Tiles whose waves copy and multiply (256 x 256 and 256 x 192, two 64-deep slots).
template <int BM, int BN, bool BKC>
static hipError_t launch_product(const GemmParams& p0, const SplitPlan& plan, void* ws, hipStream_t s) {
  if (plan.split == 1) return launch_bf16<BM, BN, true, BKC, bf16_t, 64, 0>(p0, 1, s);
  constexpr size_t smem = (size_t)2 * (BM + BN) * 64 * sizeof(bf16_t);
  auto kern = gemm_bf16_split_kernel<BM, BN, true, BKC, 64, 0>;
  static AttrOnce once;
  if (hipError_t e = once.set(reinterpret_cast<const void*>(kern), smem); e != hipSuccess) return e;
  return launch_slices(kern, 256, smem, with_tiles<BM, BN>(p0), plan, ws, s);
}
// Tiles with waves of their own for the copies, on RING 64-deep slots.
template <int BM, int BN, bool BKC, int RING, int WGS = 1>
static hipError_t launch_copiers(const GemmParams& p0, const SplitPlan& plan, void* ws, hipStream_t s) {
  const GemmParams p = with_tiles<BM, BN>(p0);
  constexpr size_t smem = (size_t)RING * (BM + BN) * 64 * sizeof(bf16_t);
  static_assert(WGS * smem <= 160 * 1024, "LDS budget of one gfx950 compute unit");
  auto kern = plan.split > 1 ? gemm_bf16_copiers_split_kernel<BM, BN, BKC, RING, WGS> : gemm_bf16_copiers_kernel<BM, BN, BKC, RING, WGS>;
  static AttrOnce once[2];
  if (hipError_t e = once[plan.split > 1].set(reinterpret_cast<const void*>(kern), smem); e != hipSuccess) return e;
  if (plan.split > 1) return launch_slices(kern, 512, smem, p, plan, ws, s);
  hipLaunchKernelGGL(kern, dim3((unsigned)(p.tiles_m * p.tiles_n)), dim3(512), smem, s, p);
  return hipGetLastError();
}
template <bool BKC>
static hipError_t dispatch_product(const GemmParams& p, const SplitPlan& plan, void* ws, hipStream_t s) {
  switch (plan.tile) {
    case T32: return launch_small<BKC>(p, s);
    case T64: return launch_copiers<64, 64, BKC, 4, 2>(p, plan, ws, s);
    case T128X64: return launch_copiers<128, 64, BKC, 6>(p, plan, ws, s);
    case T128: return launch_copiers<128, 128, BKC, 4>(p, plan, ws, s);
    case T128_PAIR: return launch_copiers<128, 128, BKC, 2, 2>(p, plan, ws, s);
    case T128X192: return launch_copiers<128, 192, BKC, 4>(p, plan, ws, s);
    case T256X128: return launch_copiers<256, 128, BKC, 3>(p, plan, ws, s);
    case T192: return launch_copiers<192, 192, BKC, 3>(p, plan, ws, s);
    case T256_NARROW: return launch_product<256, 192, BKC>(p, plan, ws, s);
    case T256: return launch_product<256, 256, BKC>(p, plan, ws, s);
  }
  return hipErrorInvalidValue;
}

// 256 x 192 tiles for outputs of more than one round of large tiles: taken when the fraction of the rounds' capacity that
// is useful output, discounted 7 % for the narrower tile's lower operand reuse, beats what 256 x 256 tiles give by 8 %.
// [1024, 22016] x 4096 is 344 large tiles (67 % of two rounds) but 460 of the narrower ones (90 %): 210 against 180 us.
static bool narrow_tiles_pay(int M, int N, int K) {
  if (M < 256 || N < 256 || K <= 256) return false;
  const long tiles_m = (M + 255) / 256;
  const long t256 = tiles_m * ((N + 255) / 256), t192 = tiles_m * ((N + 191) / 192);
  const double area = (double)M * N;
  const double now = area / ((double)((t256 + 255) / 256) * 256 * 65536);
  const double narrow = 0.93 * area / ((double)((t192 + 255) / 256) * 256 * 49152);
  return narrow > 1.08 * now;
}

// The first part of a product of more than one round of large tiles that is cut: whole rounds of them, in whole tile columns (or
// rows, if there are more of those).
static void cut_of(int M, int N, int& head_m, int& head_n) {
  const int tiles_m = (M + 255) / 256, tiles_n = (N + 255) / 256;
  const long whole = (long)tiles_m * tiles_n / 256 * 256;
  head_m = tiles_n >= tiles_m ? M : (int)(whole / tiles_n) * 256;
  head_n = tiles_n >= tiles_m ? (int)(whole / tiles_m) * 256 : N;
}
// Storage-type NN / NT products of one to six rounds of large tiles: how they run, by the modelled time of the parts.  What they
// would run on otherwise (256 x 192 tiles where narrow_tiles_pay, else cut or plain) stays unless a choice is 5 % faster.
// 3048 random products of one to three rounds in turn with what was here: 5.3 % faster on average, 2 of them more than 3 % slower; 1227 of
// three to six rounds 1.7 %, 1.  [1024, 22016] x 4096 (NN) 197 us on 256 x 192 tiles, cut into a round of
// large tiles and 88 tiles' worth of smaller ones 184.
enum Rounds { R_DEFAULT, R_CUT, R_256X128 };
static Rounds rounds_of(int layout, int M, int N, int K) {
  const long large = tiles_of(T256, M, N);
  if (large <= 256 || large >= 1600 || M < 256 || N < 256 || K <= 256) return R_DEFAULT;
  auto time = [&](int tile, int m, int n) { return product_time(kTileCost[tile], layout, m, n, K, tiles_of(tile, m, n), K, 1); };
  int head_m, head_n;
  cut_of(M, N, head_m, head_n);
  const int rest_m = head_m < M ? M - head_m : M, rest_n = head_n < N ? N - head_n : N;
  const bool cuts = large % 256 != 0 && head_m > 0 && head_n > 0 && (head_m < M || head_n < N);
  double cut = 1e30;
  if (cuts) cut = time(T256, head_m, head_n) + time(product_plan(layout, rest_m, rest_n, K, false).tile, rest_m, rest_n) + 2.;
  double now = time(T256, M, N);
  if (narrow_tiles_pay(M, N, K)) now = time(T256_NARROW, M, N);
  else if (cuts && large % 256 <= 192) now = cut;
  const double wide = time(T256X128, M, N);
  if (cut <= wide) return cut < 0.95 * now ? R_CUT : R_DEFAULT;
  return wide < 0.95 * now ? R_256X128 : R_DEFAULT;
}

// Slot depth by layout and tile size: operands with a contiguous contraction index get the 64-deep slots on the
// large tiles (whole cache lines per tile row: up to 8 % faster); on the small tiles, which run two or three
// workgroups per compute unit and overlap that way, the 4-slot ring of 32-deep slots stays ahead.
#ifndef TBP_KC_DEPTH_SMALL
#define TBP_KC_DEPTH_SMALL 32
#endif
// The weight-gradient layout (both operands strided in the contraction index) on 64-deep slots, half the barriers
// and waits per unit of K: measured 0 to 4 % slower than the ring of four 32-deep slots.
#ifndef TBP_TN_DEPTH
#define TBP_TN_DEPTH 32
#endif
// The 256 x 192 tiles: two 64-deep slots (rings of four or five 32-deep slots measured 5 to 10 % slower: K-contiguous
// operands then arrive in half cache lines; a third 64-deep slot does not fit the LDS).
#ifndef TBP_NARROW_KD
#define TBP_NARROW_KD 64
#define TBP_NARROW_RING 0
#endif
#ifndef TBP_SMALL_DEEP_RING
#define TBP_SMALL_DEEP_RING 4
#endif
#ifndef TBP_SMALL_DEEP_KD
#define TBP_SMALL_DEEP_KD 64
#endif
// Small tiles with a deep ring, for outputs of at most one small tile per compute unit that product_plan does not take: the
// last, nearly empty round of a large weight gradient, and causal products of a single head.  No second workgroup shares the
// CU to cover the first one's waits, and a 32-deep slot of a 128 x 128 tile is multiplied in 256 clocks, so the three slots
// that a ring of four keeps in flight cover under 800 clocks of memory latency; four 64-deep slots (128 KiB of LDS; eight 32-deep
// ones where the contraction index is strided in memory) cover three times 512.  Measured on [1024, 4096] outputs when they
// ran here (the same tile with copying waves, product_plan's T128, has taken them since): K = 12288 (NT) 126 -> 107 us, K = 22016 (NT) 237 -> 216 us, K = 11008
// (NN) 104 -> 93 us; a ring of eight 32-deep slots gains 3 %, three 64-deep slots lose 5 %, five (all 160 KiB) lose too.
template <typename OutT>
static hipError_t dispatch_small_deep(int layout, const GemmParams& p, hipStream_t s) {
  switch (layout) {
    case NN: return launch_bf16<128, 128, true, false, OutT, TBP_SMALL_DEEP_KD, TBP_SMALL_DEEP_RING>(p, 1, s);
    case NT: return launch_bf16<128, 128, true, true, OutT, TBP_SMALL_DEEP_KD, TBP_SMALL_DEEP_RING>(p, 1, s);
    case TN: return launch_bf16<128, 128, false, false, OutT, 32, 8>(p, 1, s);
  }
  return hipErrorInvalidValue;
}

template <int BM, int BN, typename OutT>
static hipError_t dispatch_layout(int layout, const GemmParams& p, int batch, hipStream_t s) {
  constexpr int KD = BM >= 256 ? 64 : TBP_KC_DEPTH_SMALL;
  switch (layout) {
    case NN: return launch_bf16<BM, BN, true, false, OutT, KD>(p, batch, s);
    case NT: return launch_bf16<BM, BN, true, true, OutT, KD>(p, batch, s);
    case TN: return launch_bf16<BM, BN, false, false, OutT, (BM >= 256 ? TBP_TN_DEPTH : 32)>(p, batch, s);
  }
  return hipErrorInvalidValue;
}

template <int TILE>
static hipError_t launch_tn_grouped(const GroupedProduct* prods, int n, int accumulate, hipStream_t s) {
  constexpr size_t smem = (size_t)4 * (TILE + TILE) * (TILE == 64 ? 64 : 32) * sizeof(bf16_t);
  auto kern = accumulate ? gemm_tn_grouped_kernel<TILE, true> : gemm_tn_grouped_kernel<TILE, false>;
  static AttrOnce once[2];
  if (hipError_t e = once[accumulate ? 1 : 0].set(reinterpret_cast<const void*>(kern), smem); e != hipSuccess) return e;
  for (int i = 0; i < n;) {
    GroupedTable g{};
    int blocks = 0;
    for (; i < n && g.n < kMaxGrouped; i++) {
      if (prods[i].M <= 0 || prods[i].N <= 0) continue;
      g.prod[g.n] = prods[i];
      g.first_block[g.n] = blocks;
      const int tiles = ((prods[i].M + TILE - 1) / TILE) * ((prods[i].N + TILE - 1) / TILE);
      blocks += (tiles + 7) & ~7;
      g.n++;
    }
    if (g.n == 0) continue;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), smem, s, g);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Modelled time (us) of n weight-gradient tiles over K contraction indices in one launch.  A round of workgroups costs (per
// index) K + (fixed part, which reads and writes the fp32 output; more of it where the whole output is larger than the
// on-package cache).  The small tiles run two workgroups per compute unit: `one` up to 256 of them, `two` for 512, and already
// 0.6 of the difference once some compute units have two.  The constants were fitted to make the right choice: over 459 stages
// (all weight gradients, K 64-6500) and 578 single products, each measured on all three tile sizes, overwriting and
// accumulating, the tile that the model picks costs 0.9 % more than the fastest on average (more than 10 % in one case of 50).
static double dw_time(int tile, long n, int K, int acc) {
  const bool large = n * tile * tile > (1L << 26);          // output above 256 MB
  if (tile == 256) return (double)((n + 255) / 256) * (0.0217 * K + (acc ? (large ? 26.8 : 25.5) : (large ? 11.8 : 13.0)));
  const double one = tile == 128 ? 0.0087 * K + (acc ? 6.9 : 6.3) : 0.0043 * K + (acc ? 5.1 : 4.6);
  const double two = tile == 128 ? 0.0171 * K + (acc ? (large ? 12.5 : 9.0) : (large ? 6.2 : 5.1)) : 0.0084 * K + 4.3;
  const long r = n % 512;
  return (double)(n / 512) * two + (r == 0 ? 0. : r <= 256 ? one : one + (two - one) * (0.6 + 0.4 * (double)(r - 256) / 256));
}
constexpr double kLargeTileStart = 4.3;         // us that an arrangement on large tiles takes longer to get going
constexpr double kEndLaunch = 9.7;              // us that a second launch for the last tiles costs beside their own time
static long dw_tiles(int tile, int M, int N) { return (long)((M + tile - 1) / tile) * ((N + tile - 1) / tile); }

// The first `tiles` tiles of a product, in whole tile columns (or rows, if there are more of those), and the rest.
static void cut_product(const GroupedProduct& q, long tiles, GroupedProduct& head, GroupedProduct& rest) {
  const int tiles_m = (q.M + 255) / 256, tiles_n = (q.N + 255) / 256;
  head = rest = q;
  if (tiles_n >= tiles_m) {
    const int n0 = (int)(tiles / tiles_m) * 256;
    head.N = n0 < q.N ? n0 : q.N;
    rest.N = q.N - head.N;
    rest.B = static_cast<const char*>(q.B) + (size_t)n0 * 2;
    rest.C = q.C + n0;
  } else {
    const int m0 = (int)(tiles / tiles_n) * 256;
    head.M = m0 < q.M ? m0 : q.M;
    rest.M = q.M - head.M;
    rest.A = static_cast<const char*>(q.A) + (size_t)m0 * 2;
    rest.C = q.C + (size_t)m0 * q.ldc;
  }
}

// Arrangements, taken by modelled time:
//   one grouped launch of 64 x 64 or 128 x 128 tiles: short contractions, where writing the output is most of the work and a
//     second workgroup on the compute unit covers it, and outputs that have too few larger tiles;
//   large tiles, all products pooled in one grouped launch.  If it ends with a nearly empty round, its last tiles run as a
//     launch of smaller tiles instead;
//   for long contractions, every product's whole rounds of 256 large tiles as a launch of its own (tiles that start in step
//     share operand panels through the L2), and only what does not fill a round of all products in the pool.
// Measured (us), all weight gradients of a stage, 128 x 128 / large pooled / large in whole rounds: 7B layer, K 456 333 / 266 /
// 304, K 1440 707 / 569 / 592, K 4096 - / 1416 / 1423, K 8192 - / 2735 / 2676, K 32768 - / 11712 / 10366; four MLP blocks of d 2048,
// K 6144 - / 1464 / 1449, K 32768 - / 8100 / 7324; two layers of d 768, f 2456, accumulating, K 368 40 / 55 / -.
// Large pooled over large in whole rounds, overwriting / accumulating: eight 7B layers, K 512 0.91 / 0.77, K 2048 0.99 / 0.89, K 3072
// 1.00 / 0.96, K 4096 1.02 / 1.00, K 6144 1.04 / 1.04; twelve of d 2048, f 5504, K 4096 0.99 / 0.99.
hipError_t gemm_dw(const GroupedProduct* prods, int n, int acc, GroupedProduct* pool, hipStream_t s) {
  const int whole_rounds_k = acc ? 4096 : 3072;             // contractions longer than this in whole rounds
  long n64 = 0, n128 = 0, pooled = 0, whole = 0;
  int K = 0;
  for (int i = 0; i < n; i++) {
    n64 += dw_tiles(64, prods[i].M, prods[i].N);
    n128 += dw_tiles(128, prods[i].M, prods[i].N);
    const long t = dw_tiles(256, prods[i].M, prods[i].N);
    whole += t / 256 * 256;
    pooled += t % 256;
    K = prods[i].K;
  }
  if (K <= whole_rounds_k) { pooled += whole; whole = 0; }
  const long last = pooled % 256;
  const double e64 = dw_time(64, 16 * last, K, acc), e128 = dw_time(128, 4 * last, K, acc), e_end = (e64 < e128 ? e64 : e128) + kEndLaunch;
  const bool small_end = pooled > 256 && last > 0 && e_end < 0.8 * dw_time(256, last, K, acc);
  const double t64 = dw_time(64, n64, K, acc), t128 = dw_time(128, n128, K, acc);
  const double t256 = dw_time(256, whole, K, acc) + dw_time(256, small_end ? pooled - last : pooled, K, acc) + (small_end ? e_end : 0.) + kLargeTileStart;
  if (t64 <= t128 && t64 <= t256) return launch_tn_grouped<64>(prods, n, acc, s);
  if (t128 <= t256) return launch_tn_grouped<128>(prods, n, acc, s);
  int np = 0;
  for (int i = 0; i < n; i++) {
    const long t = dw_tiles(256, prods[i].M, prods[i].N);
    GroupedProduct head{}, rest = prods[i];
    if (K > whole_rounds_k) cut_product(prods[i], t / 256 * 256, head, rest);
    if (head.M > 0 && head.N > 0) {
      GemmParams p{};
      p.A = head.A; p.B = head.B; p.C = head.C;
      p.lda = head.lda; p.ldb = head.ldb; p.ldc = head.ldc;
      p.M = head.M; p.N = head.N; p.K = head.K;
      p.batch_inner = 1; p.alpha = 1.f; p.accumulate = acc; p.causal = CAUSAL_NONE;
      if (hipError_t e = launch_bf16<256, 256, false, false, float, TBP_TN_DEPTH>(p, 1, s); e != hipSuccess) return e;
    }
    if (rest.M > 0 && rest.N > 0) pool[np++] = rest;
  }
  if (np == 0) return hipSuccess;
  GroupedProduct end{};
  if (small_end) {                            // the pool's last tiles, cut off its last product
    const GroupedProduct q = pool[np - 1];
    const long t = dw_tiles(256, q.M, q.N);
    if (t > last) cut_product(q, t - last, pool[np - 1], end);
  }
  if (hipError_t e = launch_tn_grouped<256>(pool, np, acc, s); e != hipSuccess) return e;
  if (end.M <= 0 || end.N <= 0) return hipSuccess;
  return e64 < e128 ? launch_tn_grouped<64>(&end, 1, acc, s) : launch_tn_grouped<128>(&end, 1, acc, s);
}

// fp32: whole 16-byte pieces of A and B (pointers, leading dimensions, batch strides and contiguous extents), and a tile's
// rows within a 31-bit buffer range.  C, the residual and ldc have no such rule.
static bool f32_mfma_ok(const GemmArgs& g) {
  const long a_cols = g.layout == TN ? g.M : g.K, b_cols = g.layout == NT ? g.K : g.N;
  const long mult4 = g.lda | g.ldb | a_cols | b_cols | (g.batch > 1 ? g.sAo | g.sAi | g.sBo | g.sBi : 0);
  return mult4 % 4 == 0 && (reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.B)) % 16 == 0 &&
         g.lda < (1 << 22) && g.ldb < (1 << 22);
}

template <int BM, int BN, bool AKC, bool BKC, int WK, int KD, int NS, bool SWIGLU = false>
static hipError_t launch_f32(const GemmParams& p0, int batch, hipStream_t s) {
  GemmParams p = p0;
  p.tiles_m = (p.M + BM - 1) / BM;
  p.tiles_n = (p.N + BN - 1) / BN;
  constexpr size_t smem = (size_t)NS * (BM + BN) * KD * sizeof(float);
  static_assert(smem <= 160 * 1024, "LDS budget of one gfx950 compute unit");
  auto kern = gemm_f32_mfma_kernel<BM, BN, AKC, BKC, WK, KD, NS, SWIGLU>;
  static AttrOnce once;
  if (hipError_t e = once.set(reinterpret_cast<const void*>(kern), smem); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)(p.tiles_m * p.tiles_n), 1, (unsigned)batch), dim3(256), smem, s, p);
  return hipGetLastError();
}

template <int BM, int BN, int WK, int KD, int NS>
static hipError_t launch_f32_layout(int layout, const GemmParams& p, int batch, hipStream_t s) {
  switch (layout) {
    case NN: return launch_f32<BM, BN, true, false, WK, KD, NS>(p, batch, s);
    case NT: return launch_f32<BM, BN, true, true, WK, KD, NS>(p, batch, s);
    case TN: return launch_f32<BM, BN, false, false, WK, KD, NS>(p, batch, s);
  }
  return hipErrorInvalidValue;
}

static hipError_t launch_f32_small(int layout, const GemmParams& p0, int batch, hipStream_t s) {
  GemmParams p = p0;
  p.tiles_m = (p.M + 15) / 16;
  p.tiles_n = (p.N + 15) / 16;
  constexpr size_t smem = (size_t)4 * kSmallSlots * 4096;
  auto kern = p.gu ? gemm_f32_small_kernel<true, true, true> : layout == NN ? gemm_f32_small_kernel<true, false, false>
              : layout == NT ? gemm_f32_small_kernel<true, true, false> : gemm_f32_small_kernel<false, false, false>;
  static AttrOnce once[4];
  if (hipError_t e = once[p.gu ? 3 : layout].set(reinterpret_cast<const void*>(kern), smem); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)(p.tiles_m * p.tiles_n), 1, (unsigned)batch), dim3(256), smem, s, p);
  return hipGetLastError();
}

// Tile of an fp32 product: the one with the shortest modelled time.  Every kind runs two workgroups per compute unit (64 KiB of
// LDS each), so a launch is rounds of 512 workgroups, `two` us each, and a last one that costs `one` if it has at most 256; both
// have a part per contraction index (the matrix pipes: 132 TFLOP/s on 128 x 128 tiles, 110 on the smaller ones, which move more
// operand bytes) and a fixed one (start, store).  Fitted to 471 products, M and N 64-6000, K 32-4096, each measured on all four
// tiles (5 % rms; 8 % on 16 x 16).  A larger tile has to be 5 % faster in the model, which is its error (without that [3360, 2944] x
// 440 (NT) ran on 128 x 128 tiles: 98 us, 90 on 64 x 64; [2072, 328] x 640 (NN) on 64 x 64: 17.1, 16.2 on 32 x 32).  The choice
// costs 0.4 % more than the fastest on average; a rule by rounds and rates alone, 4 % (it took 32 x 32 tiles for short
// contractions, [1544, 3268] x 64: 36 us; 64 x 64 tiles 19).
// us, 16 / 32 / 64 / 128: [512, 1024] x 5504 - / 63 / 105 / 349 (too few tiles for the large ones), [512, 5504] x 1024 - / 75 / 62 / 79,
// [2048, 2048] x 2048 - / 175 / 144 / 149, [4096, 4096] x 4096 - / 1245 / 1069 / 998.  Rings of three or four shallower slots
// measured within 5 % of these (128: three slots slower, 1049; 64: four 32-deep slots 1058; 32: four 64-deep slots 1260).
static int f32_tile(int M, int N, int K, int batch) {
  struct Tile { int t; double one_k, one, two_k, two, share; };
  static const Tile tiles[] = {{16, 0.0017, 0.9, 0.0040, 1.3, 0.7}, {32, 0.0054, 1.8, 0.0100, 2.8, 1.0},
                               {64, 0.0184, 2.4, 0.0347, 4.4, 1.0}, {128, 0.0614, 6.3, 0.1226, 10.9, 1.0}};
  int best = 0;
  double best_time = 1e30;
  for (const Tile& x : tiles) {
    const long n = (long)((M + x.t - 1) / x.t) * ((N + x.t - 1) / x.t) * batch, r = n % 512;
    if (x.t == 16 && n > 512) continue;             // ([2436, 100] x 3448 (TN), 1071 of them: 55 us, 32 x 32 tiles 41)
    const double one = x.one_k * K + x.one, two = x.two_k * K + x.two;
    const double share = x.share + (1.0 - x.share) * (double)(r - 256) / 256;       // (16 x 16: 0.7 of the difference at 257)
    const double time = (double)(n / 512) * two + (r == 0 ? 0. : r <= 256 ? one : one + (two - one) * share);
    if (time < 0.95 * best_time) { best_time = time; best = x.t; }
  }
  return best;
}
static hipError_t dispatch_f32(int layout, const GemmParams& p, int batch, hipStream_t s) {
  switch (f32_tile(p.M, p.N, p.K, batch)) {
    case 16: return launch_f32_small(layout, p, batch, s);
    case 32: return p.gu ? launch_f32<32, 32, true, true, 4, 128, 2, true>(p, batch, s) : launch_f32_layout<32, 32, 4, 128, 2>(layout, p, batch, s);
    case 64: return launch_f32_layout<64, 64, 1, 64, 2>(layout, p, batch, s);
  }
  return launch_f32_layout<128, 128, 1, 32, 2>(layout, p, batch, s);
}

// bf16: large tiles when the output is big enough to fill 256 compute units with them.  Short contractions (the per-head
// q k^T and do v^T, K = head_dim) are all prologue and epilogue: small tiles let two or three workgroups share a compute
// unit and overlap them.
static bool large_tiles(const GemmArgs& g) {
  return g.M >= 256 && g.N >= 256 && (long)((g.M + 255) / 256) * ((g.N + 255) / 256) * g.batch >= 192 && g.K > 256;
}

int gemm_row_tile(int dtype, const GemmArgs& g) {
  if (dtype == 0) return f32_mfma_ok(g) ? f32_tile(g.M, g.N, g.K, g.batch) : 64;
  return !g.a_panel && large_tiles(g) ? 256 : 128;
}

static SplitPlan plan_of(const GemmArgs& g) {
  return plan_within(g.layout, g.M, g.N, g.K, g.ws && reinterpret_cast<uintptr_t>(g.ws) % 256 == 0 ? g.ws_bytes : 0);
}

// Where the epilogue pays: fp32 products of at most two 32 x 32 tiles per compute unit (256 tokens, d 256, f 688: 5.6 us and 3.0 for the
// SwiGLU, now 6.4; 512 tokens, d 1024, f 2752 level) and bf16 ones on 32 x 32 tiles (128 tokens: 4.1 and 2.9, now 4.6).  On long micro-batches it gains nothing: the larger tiles have no second
// workgroup under whose work the three passes over memory could hide, and they run at the power limit.
bool gemm_swiglu_p1_fuses(int dtype, const GemmArgs& g) {
  if (g.layout != NT || g.batch != 1 || g.M <= 0 || g.N <= 0 || g.K <= 0) return false;
  if (dtype == 0) return f32_mfma_ok(g) && (long)((g.M + 31) / 32) * ((g.N + 31) / 32) <= 512 && f32_tile(g.M, g.N, g.K, 1) <= 32;
  return one_round(g.M, g.N) && plan_of(g).tile == T32;
}

// One launch for an NN product of at most 256 tiles of 32 x 32 and what follows it on pairs of its columns.
bool gemm_pairs_fuse(int dtype, const GemmArgs& g, int distance) {
  return dtype == 1 && g.layout == NN && g.batch == 1 && g.M > 0 && g.K > 0 && distance % 8 == 0 && g.N % (2 * distance) == 0 &&
         (distance % 32 == 0 || g.N == 2 * distance) && one_round(g.M, g.N) && plan_of(g).tile == T32;
}
hipError_t gemm_pairs(const GemmArgs& g, const PairEpilogue& pair, hipStream_t s) {
  GemmParams p{};
  p.A = g.A; p.B = g.B; p.C = g.C;
  p.lda = g.lda; p.ldb = g.ldb; p.ldc = g.ldc;
  p.M = g.M; p.N = g.N; p.K = g.K;
  p.pair = pair;
  p.tiles_m = (g.M + 31) / 32;
  p.tiles_n = (g.N / 2 + 31) / 32;
  constexpr size_t smem = (size_t)4 * kPairSlots * 12288;
  static AttrOnce once;
  if (hipError_t e = once.set(reinterpret_cast<const void*>(gemm_bf16_pairs_kernel), smem); e != hipSuccess) return e;
  hipLaunchKernelGGL(gemm_bf16_pairs_kernel, dim3((unsigned)(p.tiles_m * p.tiles_n)), dim3(256), smem, s, p);
  return hipGetLastError();
}

hipError_t gemm(int dtype, const GemmArgs& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return hipSuccess;     // empty product: nothing to write
  GemmParams p{};
  p.A = g.A; p.B = g.B; p.C = g.C; p.R = g.R;
  p.lda = g.lda; p.ldb = g.ldb; p.ldc = g.ldc;
  p.sAo = g.sAo; p.sAi = g.sAi; p.sBo = g.sBo; p.sBi = g.sBi; p.sCo = g.sCo; p.sCi = g.sCi;
  p.M = g.M; p.N = g.N; p.K = g.K;
  p.batch_inner = g.batch_inner > 0 ? g.batch_inner : 1;
  p.alpha = g.alpha; p.accumulate = g.accumulate; p.causal = g.causal;
  p.delta = g.delta; p.ldd = g.ldd; p.sDo = g.sDo; p.sDi = g.sDi; p.delta_causal = g.delta_causal;
  p.causal_fill = g.delta && g.delta_causal ? g.causal_fill : 0;
  p.gu = g.gu;
  if (g.gu) {
    if (!gemm_swiglu_p1_fuses(dtype, g)) return hipErrorInvalidValue;
    if (dtype == 1) return launch_small<true, true>(p, s);
  }
  if (dtype == 0) {
    if (g.a_panel) return hipErrorInvalidValue;
    switch (g.layout) {
      case NN: p.sam = g.lda; p.sak = 1; p.sbk = g.ldb; p.sbn = 1; break;
      case NT: p.sam = g.lda; p.sak = 1; p.sbk = 1; p.sbn = g.ldb; break;
      case TN: p.sam = 1; p.sak = g.lda; p.sbk = g.ldb; p.sbn = 1; break;
      default: return hipErrorInvalidValue;
    }
    if (f32_mfma_ok(g)) return dispatch_f32(g.layout, p, g.batch, s);
    p.tiles_m = (g.M + 63) / 64;
    p.tiles_n = (g.N + 63) / 64;
    dim3 grid((unsigned)(p.tiles_m * p.tiles_n), 1, (unsigned)g.batch);
    hipLaunchKernelGGL(gemm_f32_kernel<float>, grid, dim3(256), 0, s, p);   // fp32 storage: C is fp32 either way
    return hipGetLastError();
  }
  if (g.a_panel) {
    if (g.layout != TN || g.lda != kPanel || g.ws) return hipErrorInvalidValue;
    p.a_panel = g.a_panel;
    // (pairs only when they still give every compute unit its two workgroups)
    if (!g.out_f32 && g.causal == CAUSAL_K_END && g.N <= 128 && !g.delta &&
        (long)((g.M + kPanel - 1) / kPanel + 1) / 2 * g.batch >= 512)
      return launch_bf16_causal_pair<kPanel, 128, false, false, bf16_t, 32>(p, g.batch, s);
    return g.out_f32 ? launch_bf16<kPanel, 128, false, false, float, 32>(p, g.batch, s)
                     : launch_bf16<kPanel, 128, false, false, bf16_t, 32>(p, g.batch, s);
  }
  const int tiles_m = (g.M + 255) / 256, tiles_n = (g.N + 255) / 256;
  const long tiles_big = (long)tiles_m * tiles_n * g.batch;
  const bool big = large_tiles(g);
  if (!g.out_f32 && g.batch == 1 && g.causal == CAUSAL_NONE && !g.delta && g.layout != TN && one_round(g.M, g.N)) {
    const SplitPlan plan = plan_of(g);
    return g.layout == NN ? dispatch_product<false>(p, plan, g.ws, s) : dispatch_product<true>(p, plan, g.ws, s);
  }
  const bool linear = !g.out_f32 && g.batch == 1 && g.causal == CAUSAL_NONE && !g.delta && g.layout != TN;
  const Rounds rounds = linear ? rounds_of(g.layout, g.M, g.N, g.K) : R_DEFAULT;
  if (rounds == R_256X128) {
    const SplitPlan plan{T256X128, 1, g.K, 0};
    return g.layout == NN ? dispatch_product<false>(p, plan, nullptr, s) : dispatch_product<true>(p, plan, nullptr, s);
  }
  if (linear && rounds != R_CUT && narrow_tiles_pay(g.M, g.N, g.K))
    return g.layout == NN ? launch_bf16<256, 192, true, false, bf16_t, TBP_NARROW_KD, TBP_NARROW_RING>(p, 1, s)
                          : launch_bf16<256, 192, true, true, bf16_t, TBP_NARROW_KD, TBP_NARROW_RING>(p, 1, s);
  // a weight gradient by itself: large tiles (below, with the last round on smaller ones where it is at most three quarters
  // full) unless smaller ones are faster by the same model as in gemm_dw.  [7264, 7208] x 1896: 841 large tiles are three
  // rounds and 73 tiles, 210 us, 128 x 128 tiles 247; [4128, 920] x 3824: 264 tiles of 128 x 128 58, 64 x 64 69; [600, 544] x
  // 5880, accumulating: 64 x 64 29, 128 x 128 50.
  if (g.out_f32 && g.layout == TN && g.batch == 1 && g.causal == CAUSAL_NONE && g.K > 0) {
    const double t64 = dw_time(64, dw_tiles(64, g.M, g.N), g.K, g.accumulate), t128 = dw_time(128, dw_tiles(128, g.M, g.N), g.K, g.accumulate);
    double t256 = 1e30;
    if (big) {
      const long whole = tiles_big / 256 * 256, r = tiles_big - whole;
      t256 = dw_time(256, tiles_big, g.K, g.accumulate);
      if (whole > 0 && r > 0 && r <= 192)
        t256 = dw_time(256, whole, g.K, g.accumulate) + (r <= 128 ? dw_time(128, 4 * r, g.K, g.accumulate) : 0.75 * dw_time(256, r, g.K, g.accumulate));
    }
    t256 += kLargeTileStart;
    if (t64 <= t128 && t64 <= t256) return launch_bf16<64, 64, false, false, float, 64, 4>(p, 1, s);
    if (t128 <= t256) return launch_bf16<128, 128, false, false, float, 32>(p, 1, s);
  }
  auto run = [&](const GemmParams& q, bool use_big) -> hipError_t {
    if (!use_big && g.batch == 1 && q.K >= 1024 && (long)((q.M + 127) / 128) * ((q.N + 127) / 128) <= 256)
      return g.out_f32 ? dispatch_small_deep<float>(g.layout, q, s) : dispatch_small_deep<bf16_t>(g.layout, q, s);
    if (g.out_f32)
      return use_big ? dispatch_layout<256, 256, float>(g.layout, q, g.batch, s)
                     : dispatch_layout<128, 128, float>(g.layout, q, g.batch, s);
    return use_big ? dispatch_layout<256, 256, bf16_t>(g.layout, q, g.batch, s)
                   : dispatch_layout<128, 128, bf16_t>(g.layout, q, g.batch, s);
  };
  // Tail quantisation: with nt large tiles on 256 compute units the last round runs nt % 256 workgroups.  When
  // that round would be at most three quarters full, the output is cut along its longer side into a part made of
  // whole rounds of large tiles and a remainder: of a forward or backward-p1 product on the tiles that product_plan
  // picks; of a weight gradient, up to half a round's worth on 128 x 128 tiles (four times as many workgroups), more on
  // 256 x 192 tiles (4/3 as many workgroups: one nearly full round of tiles that take 3/4 of the time).
  const long rem = tiles_big % 256;
  const bool has_narrow = (g.out_f32 && g.layout == TN) || (!g.out_f32 && g.layout != TN && !g.delta);
  auto run_rest = [&](const GemmParams& q) -> hipError_t {
    if (!g.out_f32 && g.layout != TN && !g.delta) {
      const SplitPlan plan = product_plan(g.layout, q.M, q.N, q.K, false);
      return g.layout == NN ? dispatch_product<false>(q, plan, nullptr, s) : dispatch_product<true>(q, plan, nullptr, s);
    }
    const long t192 = (long)((q.M + 255) / 256) * ((q.N + 191) / 192);
    if (rem <= 128 || !has_narrow || t192 > 256) return run(q, rem > 128);
    return launch_bf16<256, 192, false, false, float, 32>(q, 1, s);
  };
  if (big && g.batch == 1 && g.causal == CAUSAL_NONE && tiles_big > 256 && rem != 0 &&
      (rem <= 128 || (has_narrow && rem <= 192) || rounds == R_CUT)) {
    const long whole = tiles_big - rem;
    const size_t ce = g.out_f32 ? 4 : 2;
    GemmParams a = p, b = p;
    if (tiles_n >= tiles_m) {                       // cut along N
      const int cols = (int)(whole / tiles_m);      // tile columns of the first part
      if (cols > 0 && cols < tiles_n) {
        const long n0 = (long)cols * 256;
        a.N = (int)n0;
        b.N = g.N - (int)n0;
        b.B = (const char*)p.B + (g.layout == NT ? n0 * g.ldb : n0) * 2;
        b.C = (char*)p.C + n0 * ce;
        if (p.R) b.R = (const char*)p.R + n0 * 2;
        hipError_t e = run(a, true);
        return e != hipSuccess ? e : run_rest(b);
      }
    } else {                                        // cut along M
      const int rows = (int)(whole / tiles_n);
      if (rows > 0 && rows < tiles_m) {
        const long m0 = (long)rows * 256;
        a.M = (int)m0;
        b.M = g.M - (int)m0;
        b.A = (const char*)p.A + (g.layout == TN ? m0 : m0 * g.lda) * 2;
        b.C = (char*)p.C + m0 * g.ldc * ce;
        if (p.R) b.R = (const char*)p.R + m0 * g.ldc * 2;
        hipError_t e = run(a, true);
        return e != hipSuccess ? e : run_rest(b);
      }
    }
  }
  return run(p, big);
}

}  // namespace tbp
