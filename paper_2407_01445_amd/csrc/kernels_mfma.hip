// bf16 MFMA kernels of the FCCO step for gfx950 (wave64, v_mfma_f32_32x32x16_bf16).
//
//  k_strips_edge_bf16  the strip tiles with a ragged edge (whole tiles: k_strips_bf16 in kernels_strips.hip):
//                   S^T tile = contrasts x anchors^T (256 x 256 per workgroup), then in registers
//                   l = exp((s - s_ii)/tau) (Sec. 3), per-anchor sums of l and of (s - s_ii) l (Proc. 1 and the
//                   nabla_3 l sums of Eqs. 8-10), and l rounded to bf16 stored as the operand of the gradient
//                   contraction.  The similarity matrix itself never reaches memory.  Anchors run along lanes, so
//                   the sums are lane-local and every store is a contiguous 1 KiB per wavefront.
//  k_fold_bf16      the local contrast-side term of Eqs. 3 / 5 / 7: c_other[q] l_other(q, p_r) / c_own[r] is added to
//                   the strip element (r, off + q), which weights the same row of X, so that one contraction yields
//                   sum_j l(r,j) x_j + (1/c_r) sum_q c_q l(q,p_r) x_q.
//  k_contract_bf16  C[r][n] = sum_c Efrag[r][c] X[c][n] over the contrast columns, split over c into fp32
//                   partial results (Eqs. 2/4/6 plus the local part of Eqs. 3/5/7).
//
// Stored exp strips ("Efrag"): for anchor block ab = r / 32 and column block cb = c / 16 one 1 KiB fragment, laid out
// exactly as the A operand of the 32x32x16 MFMA: lane L = (r % 32) + 32 h holds 8 bf16, slot e <-> column
// 16 cb + 8 (e / 4) + 4 h + (e % 4).  The same slot order is used for the rows of X in the contraction, so the
// permutation cancels.  Columns [0, ldE) are contrasts (global rows, zero beyond B).
//
// MFMA layout facts used (32x32x16, wave64): lane l supplies row/column (l & 31) of its operand and 8 contraction
// slots selected by (l >> 5); accumulator register v of lane l is D[8 (v >> 2) + 4 (l >> 5) + (v & 3)][l & 31].
//
// Main loop of the contraction (whole tiles): a ring of five 32 KiB LDS slots, each one 32-deep stage of both operands,
// filled by global_load_lds_dwordx4 (no VGPR staging) four stages ahead; one barrier per stage; LDS operand reads of
// the next 16-deep step are issued between the MFMAs of the current one.  Tiles that touch a ragged edge use guarded
// register loads into the same LDS images, one stage at a time.
#include "mfma_common.hpp"
#include "state_common.hpp"

namespace fc {

// ----------------------------------------------------------------------------------------------------------------
// Operand sources.  Each describes, for one workgroup tile, how a stage is brought into an LDS slot (dma: 8 wave
// loads per thread and stage, indices 0..3 = A operand, 4..7 = B operand; fill_guarded: the same image through
// registers with zero fill) and how a wave reads its MFMA operands from the slot.
//
// Strip kernel: both operands are K-contiguous row tiles.  A operand = 256 contrast rows, B operand = 256 anchor rows.
struct StripTile {
  static constexpr int NJ = 4;   // 32-column blocks of the B operand per wave
  const bf16_t *X, *A;   // wave-uniform: first contrast row / first anchor row of the tile
  int64_t ldx, lda;
  uint32_t oa[4], ob[4]; // per-lane byte offsets of the 4 + 4 wave loads of a stage (relative to X / A, stage 0)
  uint32_t la[4], lb[4]; // LDS byte offsets inside a slot (wave-uniform)
  int wr, wc_, lr, hk;   // wave row/col block, lane split
  int64_t x_rows, a_rows, d;   // valid rows below X / A, contraction length (guarded path)

  // Xc / An: row 0 of the contrast / anchor matrix; c0 / a0: first row of the tile; B / b: rows of the matrices.
  __device__ __forceinline__ void setup(const bf16_t* Xc, int64_t ldx_, int64_t c0, int64_t B, const bf16_t* An,
                                        int64_t lda_, int64_t a0, int64_t b, int64_t d_, int tid) {
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;   // wave-uniform, kept in SGPRs
    wr = wave >> 1; wc_ = wave & 1; lr = lane & 31; hk = lane >> 5;
    X = Xc + c0 * ldx_; ldx = ldx_; x_rows = B - c0;
    A = An + a0 * lda_; lda = lda_; a_rows = b - a0;
    d = d_;
    // The unguarded wave loads fetch, for a row of the tile that does not exist, the tile's last existing row instead
    // (x_rows, a_rows >= 1): whatever such a row contributes lands in elements that the guarded epilogue discards.
    const int x_last = (int)(x_rows < 256 ? x_rows : 256) - 1, a_last = (int)(a_rows < 256 ? a_rows : 256) - 1;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int j = wave * 4 + i;                      // wave load j covers rows 16 j .. 16 j + 15 of the tile
      const int row = 16 * j + (lane >> 2);
      const int chunk = (lane & 3) ^ rt_swz(row);      // logical chunk fetched into position (lane & 3)
      oa[i] = (uint32_t)((row < x_last ? row : x_last) * (int)ldx_ + chunk * 8) * 2u;
      ob[i] = (uint32_t)((row < a_last ? row : a_last) * (int)lda_ + chunk * 8) * 2u;
      la[i] = (uint32_t)(j * 1024);
      lb[i] = (uint32_t)(kOpBytes + j * 1024);
    }
  }
  __device__ __forceinline__ void dma(int i, int stage, uint32_t slot) const {
    if (i < 4) dma16(X + (int64_t)stage * BK, oa[i], slot + la[i]);
    else dma16(A + (int64_t)stage * BK, ob[i - 4], slot + lb[i - 4]);
  }
  __device__ __forceinline__ void fill_guarded(int stage, char* slot, int tid) const {
    const int chunk = tid & 3;
    const int64_t k = (int64_t)stage * BK + chunk * 8;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = (tid >> 2) + 64 * i;
      u32x4 va = {0u, 0u, 0u, 0u}, vb = {0u, 0u, 0u, 0u};
      if (k < d && row < x_rows) va = *(const u32x4*)(X + row * ldx + k);
      if (k < d && row < a_rows) vb = *(const u32x4*)(A + row * lda + k);
      *(u32x4*)(slot + rt_off(row, chunk)) = va;
      *(u32x4*)(slot + kOpBytes + rt_off(row, chunk)) = vb;
    }
  }
  __device__ __forceinline__ bf16x8 read_a(const char* slot, int t, int kk) const {
    return *(const bf16x8*)(slot + rt_off(wr * 128 + t * 32 + lr, kk * 2 + hk));
  }
  __device__ __forceinline__ bf16x8 read_b(const char* slot, int t, int kk) const {
    return *(const bf16x8*)(slot + kOpBytes + rt_off(wc_ * 128 + t * 32 + lr, kk * 2 + hk));
  }
  __device__ __forceinline__ u32x2 read_b_half(const char* slot, int t, int kk, int half) const {   // for the ring loop
    return *(const u32x2*)(slot + kOpBytes + rt_off(wc_ * 128 + t * 32 + lr, kk * 2 + hk) + 8 * half);
  }
};

// Contraction kernel: A operand = 8 anchor blocks x 2 column blocks of Efrag per stage (fragments are copied as they
// are), B operand = 32 rows x 64 NJ columns of X in its natural layout, read with transposing LDS reads.
// What bounds it: the matrix cores at the clock that the power limit leaves (1.2 PFLOP/s for 1024 of 32768 at 1024), and
// writing the partial tiles.  NJ = 4: 256 x 256 output tiles; NJ = 3: 256 x 192, three quarters of the MFMAs for 28 of 32 KiB
// a stage, for widths and batches that 256 columns cut badly (the rule and both sides are where the plan is made).
// LDS image of the B operand: rows of 64 NJ columns, 16-byte piece p of row k at piece position p ^ nswz(k), so that the
// 4 rows x 64 bytes of a transposing read cover all 64 banks.  256 columns (512 bytes a row): nt_swz.  192 columns: rows are
// 384 bytes apart, every other one half the banks further, and rows 2 and 3 of four take the other quarter.
// REMOTE (gathered state): the A operand is E + F / c_own, formed between the loads of both strips and the LDS image.
template <int NJ_, bool REMOTE>
struct ContractTile {
  static constexpr int NJ = NJ_;
  static constexpr int kCols = 64 * NJ, kPieces = 8 * NJ;
  const bf16_t* Efr;       // wave-uniform: fragment (ab0, column block 0) of the strip
  const bf16_t* Xn;        // wave-uniform: X + n0
  int64_t ldx;
  uint32_t oa[4], ob[NJ];  // per-lane byte offsets of the wave loads (A: relative to Efr; B: relative to row 0 of a stage)
  uint32_t la[4], lb[NJ];
  int wm, wn, lane;
  int64_t n0, N, B;   // guarded path
  const bf16_t* Ffr;  // REMOTE: the second strip as Efr, and 1 / c_own of the lane's row in the two anchor blocks that the
  float inv[2];       // wave brings in (fragments 0, 1 and 2, 3)

  static __device__ __forceinline__ int nswz(int k) { return NJ == 4 ? nt_swz(k) : ((k >> 1) & 1) << 2; }
  // row of the stage and logical piece that lane `lane` of wave load f (0 .. 4 NJ - 1) fetches
  __device__ __forceinline__ void b_piece(int f, int* k, int* piece) const {
    const unsigned at = (unsigned)(f * 64 + lane);
    *k = (int)(at / kPieces);
    *piece = (int)(at % kPieces) ^ nswz(*k);
  }
  __device__ __forceinline__ void setup(const bf16_t* E, int64_t nCB, int64_t ab0, const bf16_t* X_, int64_t ldx_,
                                        int64_t n0_, int64_t N_, int64_t B_, int tid) {
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform, kept in SGPRs
    lane = tid & 63; wm = wave >> 1; wn = wave & 1;
    Efr = E + ab0 * nCB * 512; Xn = X_ + n0_; ldx = ldx_;
    n0 = n0_; N = N_; B = B_;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int f = wave * 4 + i;                       // fragment f = 2 * (anchor block) + (column block in stage)
      oa[i] = (uint32_t)(((f >> 1) * (int)nCB + (f & 1)) * 512 + lane * 8) * 2u;
      la[i] = (uint32_t)(f * 1024);
    }
#pragma unroll
    for (int i = 0; i < NJ; ++i) {
      const int f = wave * NJ + i;
      int k, piece;
      b_piece(f, &k, &piece);
      ob[i] = (uint32_t)(k * (int)ldx_ + piece * 8) * 2u;
      lb[i] = (uint32_t)(kOpBytes + f * 1024);
    }
  }
  __device__ __forceinline__ void setup_remote(const bf16_t* F, int64_t nCB, int64_t ab0, const float* c_own, int64_t b, int tid) {
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Ffr = F + ab0 * nCB * 512;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int64_t r = (ab0 + wave * 2 + i) * 32 + (lane & 31);
      inv[i] = r < b ? 1.0f / c_own[r] : 0.f;
    }
  }
  // chunk i of a stage of either strip, and two of its elements put together
  __device__ __forceinline__ u32x4 load_e(int i, int stage) const {
    return *(const u32x4*)((const char*)(Efr + (int64_t)stage * 1024) + oa[i]);
  }
  __device__ __forceinline__ u32x4 load_f(int i, int stage) const {
    return *(const u32x4*)((const char*)(Ffr + (int64_t)stage * 1024) + oa[i]);
  }
  __device__ __forceinline__ uint32_t combine(int i, uint32_t e, uint32_t f) const {
    const float lo = fmaf(__uint_as_float(f << 16), inv[i >> 1], __uint_as_float(e << 16));
    const float hi = fmaf(__uint_as_float(f & 0xffff0000u), inv[i >> 1], __uint_as_float(e & 0xffff0000u));
    return pack_bf16x2(lo, hi);
  }
  __device__ __forceinline__ const bf16_t* stage_rows(int stage) const {   // X row of stage row 0, plus n0
    return Xn + (int64_t)stage * BK * ldx;
  }
  __device__ __forceinline__ void dma(int i, int stage, uint32_t slot) const {
    if (i < 4) dma16(Efr + (int64_t)stage * 1024, oa[i], slot + la[i]);
    else dma16(stage_rows(stage), ob[i - 4], slot + lb[i - 4]);
  }
  __device__ __forceinline__ void fill_guarded(int stage, char* slot, int tid) const {
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int f = wave * 4 + i;
      u32x4 v = load_e(i, stage);
      if constexpr (REMOTE) {
        const u32x4 w = load_f(i, stage);
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = combine(i, v[q], w[q]);
      }
      *(u32x4*)(slot + f * 1024 + lane * 16) = v;
    }
#pragma unroll
    for (int i = 0; i < NJ; ++i) {
      const int f = wave * NJ + i;
      int k, piece;
      b_piece(f, &k, &piece);
      const int64_t c = (int64_t)stage * BK + k;        // contrast column = row of X
      const bool ok = c < B && (n0 + piece * 8 < N);
      u32x4 v = {0u, 0u, 0u, 0u};
      if (ok) v = *(const u32x4*)((const char*)stage_rows(stage) + ob[i]);
      *(u32x4*)(slot + kOpBytes + f * 1024 + lane * 16) = v;
    }
  }
  __device__ __forceinline__ bf16x8 read_a(const char* slot, int t, int kk) const {
    return *(const bf16x8*)(slot + (((wm * 4 + t) * 2 + kk) * 1024 + lane * 16));
  }
  // slots e = 0..3 <-> rows 16 kk + 4 h + e, slots 4..7 <-> rows 16 kk + 8 + 4 h + (e - 4): two transposing reads
  // (half 0 / 1), each taking 4 rows x 16 columns per group of 16 lanes (source lane s: row s / 4, columns 4 (s % 4) ..).
  __device__ __forceinline__ u32x2 read_b_half(const char* slot, int t, int kk, int half) const {
    const int h = lane >> 5, s = lane & 15;
    const int n = wn * (kCols / 2) + t * 32 + ((lane >> 4) & 1) * 16 + 4 * (s & 3);   // first of 4 columns read by this lane
    const int k = 16 * kk + 8 * half + 4 * h + (s >> 2);
    const char* base = slot + kOpBytes + ((n & 7) << 1);
    lds_v4s* p = (lds_v4s*)(uintptr_t)lds_addr(base + k * (kPieces * 16) + (((n >> 3) ^ nswz(k)) << 4));
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(p));
  }
  __device__ __forceinline__ bf16x8 read_b(const char* slot, int t, int kk) const {
    return join_halves(read_b_half(slot, t, kk, 0), read_b_half(slot, t, kk, 1));
  }
};

#define FC_MM(ti, tj, A_, B_) acc[ti][tj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A_[ti], B_[tj], acc[ti][tj], 0, 0, 0)
// The same with the B operand held as the two halves that the transposing reads deliver.
#define FC_MMH(ti, tj, A_, BL_, BH_) \
  acc[ti][tj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A_[ti], join_halves(BL_[tj], BH_[tj]), acc[ti][tj], 0, 0, 0)

// One 32-deep stage of the ring: 16 MFMAs on the operands already in registers while the operands of the second
// 16-deep step are read; then "stage s+1 has landed" (vmcnt) + barrier, which also retires the slot of stage s-1; then
// 16 MFMAs while the first operands of stage s+1 are read.  A lone wavefront per SIMD issues in order: whatever sits
// between two MFMAs delays the second one once it takes longer than the first one runs (32 cycles), so the 4 + 8 LDS
// reads and the 4 wave loads of a half stage are dealt out ONE per MFMA.  The 8 wave loads of a stage x are spread
// over a whole stage time, so that the load unit sees a steady trickle instead of a burst: the four A-operand loads
// in the second half of stage x-4 (DMAA, into the slot just retired), the four B-operand loads in the first half of
// stage x-3 (DMAB).  cur / nxt / prv / pp: byte offsets of the slots of stages s, s+1, s-1, s-2 in a ring of five.
// WAIT: loads that may stay in flight at the barrier, those of stages s+2 and s+3: 2 L, L or 0 for L = 4 + NJ per stage.
// The barrier is the bare instruction: the LDS reads of the first half need not have returned (their slot is written
// again only after the NEXT stage's barrier, and their consumers wait for them by themselves), so there is no
// "wait for all LDS traffic" in front of it as __syncthreads() would put.
// One MFMA followed by one other statement.
#define FC_SLOT(ti, tj, AP, BLP, BHP, STMT) FC_MMH(ti, tj, AP, BLP, BHP); FC_PIN(); STMT; FC_PIN();
// 16 MFMAs on operand set (AP, BLP, BHP) while the set (AQ, BLQ, BHQ) is read from slot `src`, step KQ, in the order in
// which the following half stage consumes it (its MFMAs run over tj fastest), and D0 .. D3 are issued.
#define FC_HALF(AP, BLP, BHP, AQ, BLQ, BHQ, src, KQ, RD, D0, D1, D2, D3)                                            \
    FC_SLOT(0, 0, AP, BLP, BHP, if (RD) BLQ[0] = T.read_b_half(src, 0, KQ, 0))                                      \
    FC_SLOT(0, 1, AP, BLP, BHP, if (RD) BHQ[0] = T.read_b_half(src, 0, KQ, 1))                                      \
    FC_SLOT(0, 2, AP, BLP, BHP, if (RD) AQ[0] = T.read_a(src, 0, KQ))                                               \
    FC_SLOT(0, 3, AP, BLP, BHP, D0)                                                                                 \
    FC_SLOT(1, 0, AP, BLP, BHP, if (RD) BLQ[1] = T.read_b_half(src, 1, KQ, 0))                                      \
    FC_SLOT(1, 1, AP, BLP, BHP, if (RD) BHQ[1] = T.read_b_half(src, 1, KQ, 1))                                      \
    FC_SLOT(1, 2, AP, BLP, BHP, if (RD) BLQ[2] = T.read_b_half(src, 2, KQ, 0))                                      \
    FC_SLOT(1, 3, AP, BLP, BHP, D1)                                                                                 \
    FC_SLOT(2, 0, AP, BLP, BHP, if (RD) BHQ[2] = T.read_b_half(src, 2, KQ, 1))                                      \
    FC_SLOT(2, 1, AP, BLP, BHP, if (RD) BLQ[3] = T.read_b_half(src, 3, KQ, 0))                                      \
    FC_SLOT(2, 2, AP, BLP, BHP, if (RD) BHQ[3] = T.read_b_half(src, 3, KQ, 1))                                      \
    FC_SLOT(2, 3, AP, BLP, BHP, D2)                                                                                 \
    FC_SLOT(3, 0, AP, BLP, BHP, if (RD) AQ[1] = T.read_a(src, 1, KQ))                                               \
    FC_SLOT(3, 1, AP, BLP, BHP, if (RD) AQ[2] = T.read_a(src, 2, KQ))                                               \
    FC_SLOT(3, 2, AP, BLP, BHP, if (RD) AQ[3] = T.read_a(src, 3, KQ))                                               \
    FC_SLOT(3, 3, AP, BLP, BHP, D3)
// The same for three blocks of 32 columns: 12 MFMAs, 4 + 6 reads.
#define FC_HALF3(AP, BLP, BHP, AQ, BLQ, BHQ, src, KQ, RD, D0, D1, D2, D3)                                           \
    FC_SLOT(0, 0, AP, BLP, BHP, if (RD) BLQ[0] = T.read_b_half(src, 0, KQ, 0))                                      \
    FC_SLOT(0, 1, AP, BLP, BHP, if (RD) BHQ[0] = T.read_b_half(src, 0, KQ, 1))                                      \
    FC_SLOT(0, 2, AP, BLP, BHP, if (RD) AQ[0] = T.read_a(src, 0, KQ))                                               \
    FC_SLOT(1, 0, AP, BLP, BHP, if (RD) BLQ[1] = T.read_b_half(src, 1, KQ, 0); D0)                                  \
    FC_SLOT(1, 1, AP, BLP, BHP, if (RD) BHQ[1] = T.read_b_half(src, 1, KQ, 1))                                      \
    FC_SLOT(1, 2, AP, BLP, BHP, if (RD) BLQ[2] = T.read_b_half(src, 2, KQ, 0))                                      \
    FC_SLOT(2, 0, AP, BLP, BHP, if (RD) BHQ[2] = T.read_b_half(src, 2, KQ, 1))                                      \
    FC_SLOT(2, 1, AP, BLP, BHP, D1)                                                                                 \
    FC_SLOT(2, 2, AP, BLP, BHP, if (RD) AQ[1] = T.read_a(src, 1, KQ))                                               \
    FC_SLOT(3, 0, AP, BLP, BHP, if (RD) AQ[2] = T.read_a(src, 2, KQ))                                               \
    FC_SLOT(3, 1, AP, BLP, BHP, if (RD) AQ[3] = T.read_a(src, 3, KQ); D3)                                           \
    FC_SLOT(3, 2, AP, BLP, BHP, D2)
#define FC_STAGE(T, MORE, DMAB, DMAA, WAIT)                                                                         \
  {                                                                                                                 \
    const char* sl = ring + cur;                                                                                    \
    const uint32_t bslot = ring_addr + pp;                                                                          \
if constexpr (NJ == 4) {                                                                                        \
      FC_HALF(a0, bl0, bh0, a1, bl1, bh1, sl, 1, true, if (DMAB) T.dma(4, s0 + s + 3, bslot),                       \
              if (DMAB) T.dma(5, s0 + s + 3, bslot), if (DMAB) T.dma(6, s0 + s + 3, bslot),                         \
              if (DMAB) T.dma(7, s0 + s + 3, bslot))                                                                \
    } else {                                                                                                        \
      FC_HALF3(a0, bl0, bh0, a1, bl1, bh1, sl, 1, true, if (DMAB) T.dma(4, s0 + s + 3, bslot),                      \
               if (DMAB) T.dma(5, s0 + s + 3, bslot), if (DMAB) T.dma(6, s0 + s + 3, bslot), )                      \
    }                                                                                                               \
    wait_vmcnt<WAIT>();                                                                                             \
    __builtin_amdgcn_s_barrier();                                                                                   \
    FC_PIN();                                                                                                       \
    const char* nx = ring + nxt;                                                                                    \
    const uint32_t aslot = ring_addr + prv;                                                                         \
    if constexpr (NJ == 4) {                                                                                        \
      FC_HALF(a1, bl1, bh1, a0, bl0, bh0, nx, 0, MORE, if (DMAA) T.dma(0, s0 + s + 4, aslot),                       \
              if (DMAA) T.dma(1, s0 + s + 4, aslot), if (DMAA) T.dma(2, s0 + s + 4, aslot),                         \
              if (DMAA) T.dma(3, s0 + s + 4, aslot))                                                                \
    } else {                                                                                                        \
      FC_HALF3(a1, bl1, bh1, a0, bl0, bh0, nx, 0, MORE, if (DMAA) T.dma(0, s0 + s + 4, aslot),                      \
               if (DMAA) T.dma(1, s0 + s + 4, aslot), if (DMAA) T.dma(2, s0 + s + 4, aslot),                        \
               if (DMAA) T.dma(3, s0 + s + 4, aslot))                                                               \
    }                                                                                                               \
    pp = prv; prv = cur; cur = nxt;                                                                                 \
    nxt = (nxt + (uint32_t)kStageBytes == (uint32_t)kRingBytes) ? 0u : nxt + (uint32_t)kStageBytes;                 \
    ++s;                                                                                                            \
  }

// Issue the wave loads of the first stages [s0, ...) of a tile into ring slots 0 .. 3: stages 0 .. 2 whole and of
// stage 3 the A-operand half (its B-operand half follows in the first half of stage 0, as for every later stage);
// tiles of at most 4 stages are requested whole.
template <typename Tile>
__device__ __forceinline__ void ring_prologue(const Tile& T, uint32_t ring_addr, int s0, int S) {
#pragma unroll
  for (int p = 0; p < 4; ++p)
    if (p < S) {
#pragma unroll
      for (int i = 0; i < 4 + Tile::NJ; ++i)
        if (p < 3 || i < 4 || S == 4) T.dma(i, s0 + p, ring_addr + p * kStageBytes);
    }
}

// acc += (A operand tile) x (B operand tile)^T over stages [s0, s0 + S); the prologue must have been issued, and
// nothing else may have touched the ring since.  Vector memory operations complete in order, so every wait names
// the number of younger loads that may stay in flight.  On return no wave reads the ring any more.
template <typename Tile>
__device__ __forceinline__ void ring_mainloop(f32x16 (&acc)[4][Tile::NJ], const Tile& T, char* ring, uint32_t ring_addr,
                                              int s0, int S) {
  constexpr int NJ = Tile::NJ, L = 4 + NJ;
  // stage 0 has landed; stages 1, 2 and (half or all of) 3 may be in flight
  if (S >= 5) wait_vmcnt<2 * L + 4>(); else if (S == 4) wait_vmcnt<3 * L>(); else wait_vmcnt<0>();
  __syncthreads();
  bf16x8 a0[4], a1[4];
  u32x2 bl0[NJ], bh0[NJ], bl1[NJ], bh1[NJ];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    a0[t] = T.read_a(ring, t, 0);
    if (t < NJ) {
      bl0[t] = T.read_b_half(ring, t, 0, 0);
      bh0[t] = T.read_b_half(ring, t, 0, 1);
    }
  }
  uint32_t cur = 0u, nxt = (uint32_t)kStageBytes, prv = 4u * (uint32_t)kStageBytes, pp = 3u * (uint32_t)kStageBytes;
  int s = 0;
  while (s + 4 < S) FC_STAGE(T, true, true, true, 2 * L)               // s = 0 .. S-5
  while (s + 4 == S && S >= 5) FC_STAGE(T, true, true, false, 2 * L)   // s = S-4: the last B-operand loads
  while (s + 3 < S) FC_STAGE(T, true, false, false, 2 * L)             // S == 4 only
  while (s + 2 < S) FC_STAGE(T, true, false, false, L)
  while (s + 1 < S) FC_STAGE(T, true, false, false, 0)
  FC_STAGE(T, false, false, false, 0)
  __syncthreads();
}

// The contraction's loop with gathered state (ContractTile<NJ, true>): the B operand comes as above, the A operand through
// registers.  Stage s forms the A operand of stage s + 3 from chunks of both strips that were requested two stages before, writes
// it into its slot and requests those of stage s + 5 into the registers just freed: two sets, taken in turn.  A pair of
// elements (seven VALU instructions) goes behind every other MFMA.
// Any run of stages, S >= 1: an odd one begins with a stage of zeros (A operand) ahead of its first, and what lies behind the last
// stage is requested as that one, into registers and slots that nobody reads.  One body, for which the wait counts are
// constant.  With the stages at the end peeled, and their requests left out, runs of 14 stages took 22.4 us instead of 23.1, of 32
// 36.2 instead of 36.7, of 128 155 instead of 154; with the short runs in a loop of their own beside them the kernel spills.
// Runs below eight stages and last odd ones one at a time through guarded_mainloop take as long as four stages each: 1536 of 3072
// at 200 36.6 us, here 20.1; 704 of 5632 at 448, steps, 80 / 69.
// LDS: what a stage writes is complete before the barrier of the one after the next: later reads of this wave, which LDS serves
// in order, have been waited for by then.
// Why not a pass over both strips ahead of the contraction: it reads and writes 384 MiB for 1024 of 32768 pairs
// at width 1024, 63 us; the loop takes 155 us instead of 116, bound by the strips' way from memory (pairs in the second half
// stage only or spread over both make no difference).  Steps, pass / here, us: 1024 of 32768 at 1024 376 / 347, 512 of 32768 at
// 512 162 / 143, 1024 of 16384 at 384 140 / 110, 1024 of 5120 at 1024 101 / 94.
struct RemoteSet {
  u32x4 e[4], f[4];
};
template <typename Tile>
__device__ __forceinline__ void remote_request(const Tile& T, RemoteSet& r, int stage) {
#pragma unroll
  for (int i = 0; i < 4; ++i) { r.e[i] = T.load_e(i, stage); r.f[i] = T.load_f(i, stage); }
}
// Pair w of the set's 16; a chunk that is complete goes to its place in the slot and its registers to the stage `next`.
template <typename Tile>
__device__ __forceinline__ void remote_pair(const Tile& T, RemoteSet& r, int w, char* slot, int next, bool zero = false) {
  const int i = w >> 2;
  r.e[i][w & 3] = T.combine(i, r.e[i][w & 3], r.f[i][w & 3]);
  if ((w & 3) == 3) {
    *(u32x4*)(slot + T.la[i] + T.lane * 16) = zero ? u32x4{0u, 0u, 0u, 0u} : r.e[i];
    r.e[i] = T.load_e(i, next); r.f[i] = T.load_f(i, next);
  }
}
// The half stages with a pair of elements behind every other MFMA (of three: behind two): P(0) .. P(7).
#define FC_HALF_P(AP, BLP, BHP, AQ, BLQ, BHQ, src, KQ, RD, D0, D1, D2, D3, P)                                       \
    FC_SLOT(0, 0, AP, BLP, BHP, if (RD) BLQ[0] = T.read_b_half(src, 0, KQ, 0); P(0))                                \
    FC_SLOT(0, 1, AP, BLP, BHP, if (RD) BHQ[0] = T.read_b_half(src, 0, KQ, 1))                                      \
    FC_SLOT(0, 2, AP, BLP, BHP, if (RD) AQ[0] = T.read_a(src, 0, KQ); P(1))                                         \
    FC_SLOT(0, 3, AP, BLP, BHP, D0)                                                                                 \
    FC_SLOT(1, 0, AP, BLP, BHP, if (RD) BLQ[1] = T.read_b_half(src, 1, KQ, 0); P(2))                                \
    FC_SLOT(1, 1, AP, BLP, BHP, if (RD) BHQ[1] = T.read_b_half(src, 1, KQ, 1))                                      \
    FC_SLOT(1, 2, AP, BLP, BHP, if (RD) BLQ[2] = T.read_b_half(src, 2, KQ, 0); P(3))                                \
    FC_SLOT(1, 3, AP, BLP, BHP, D1)                                                                                 \
    FC_SLOT(2, 0, AP, BLP, BHP, if (RD) BHQ[2] = T.read_b_half(src, 2, KQ, 1); P(4))                                \
    FC_SLOT(2, 1, AP, BLP, BHP, if (RD) BLQ[3] = T.read_b_half(src, 3, KQ, 0))                                      \
    FC_SLOT(2, 2, AP, BLP, BHP, if (RD) BHQ[3] = T.read_b_half(src, 3, KQ, 1); P(5))                                \
    FC_SLOT(2, 3, AP, BLP, BHP, D2)                                                                                 \
    FC_SLOT(3, 0, AP, BLP, BHP, if (RD) AQ[1] = T.read_a(src, 1, KQ); P(6))                                         \
    FC_SLOT(3, 1, AP, BLP, BHP, if (RD) AQ[2] = T.read_a(src, 2, KQ))                                               \
    FC_SLOT(3, 2, AP, BLP, BHP, if (RD) AQ[3] = T.read_a(src, 3, KQ); P(7))                                         \
    FC_SLOT(3, 3, AP, BLP, BHP, D3)
#define FC_HALF3_P(AP, BLP, BHP, AQ, BLQ, BHQ, src, KQ, RD, D0, D1, D2, D3, P)                                      \
    FC_SLOT(0, 0, AP, BLP, BHP, if (RD) BLQ[0] = T.read_b_half(src, 0, KQ, 0); P(0))                                \
    FC_SLOT(0, 1, AP, BLP, BHP, if (RD) BHQ[0] = T.read_b_half(src, 0, KQ, 1); P(1))                                \
    FC_SLOT(0, 2, AP, BLP, BHP, if (RD) AQ[0] = T.read_a(src, 0, KQ))                                               \
    FC_SLOT(1, 0, AP, BLP, BHP, if (RD) BLQ[1] = T.read_b_half(src, 1, KQ, 0); P(2))                                \
    FC_SLOT(1, 1, AP, BLP, BHP, if (RD) BHQ[1] = T.read_b_half(src, 1, KQ, 1); P(3))                                \
    FC_SLOT(1, 2, AP, BLP, BHP, if (RD) BLQ[2] = T.read_b_half(src, 2, KQ, 0); D0)                                  \
    FC_SLOT(2, 0, AP, BLP, BHP, if (RD) BHQ[2] = T.read_b_half(src, 2, KQ, 1); P(4))                                \
    FC_SLOT(2, 1, AP, BLP, BHP, if (RD) AQ[1] = T.read_a(src, 1, KQ); P(5))                                         \
    FC_SLOT(2, 2, AP, BLP, BHP, D1)                                                                                 \
    FC_SLOT(3, 0, AP, BLP, BHP, if (RD) AQ[2] = T.read_a(src, 2, KQ); P(6))                                         \
    FC_SLOT(3, 1, AP, BLP, BHP, if (RD) AQ[3] = T.read_a(src, 3, KQ); P(7))                                         \
    FC_SLOT(3, 2, AP, BLP, BHP, D2)
// Stage s: SET holds the chunks of stage s + 3, of which the first half stage takes the first eight pairs and the second half
// the others.  At the barrier those loads may stay in flight that are younger than the B operand of stage s + 1: two sets' and
// the B operands of stages s + 2 and s + 3.
#define FC_PAIR(k, SET) remote_pair(T, SET, k, ring + wslot, later(5))
#define FC_STAGE_REMOTE(SET)                                                                                        \
  {                                                                                                                 \
    const char* sl = ring + cur;                                                                                    \
    const uint32_t bslot = ring_addr + pp, wslot = pp;                                                              \
    auto first = [&](int k) __attribute__((always_inline)) { FC_PAIR(k, SET); };                                    \
    auto second = [&](int k) __attribute__((always_inline)) { FC_PAIR(8 + k, SET); };                               \
    if constexpr (NJ == 4) {                                                                                        \
      FC_HALF_P(a0, bl0, bh0, a1, bl1, bh1, sl, 1, true, T.dma(4, later(3), bslot), T.dma(5, later(3), bslot),      \
                T.dma(6, later(3), bslot), T.dma(7, later(3), bslot), first)                                        \
    } else {                                                                                                        \
      FC_HALF3_P(a0, bl0, bh0, a1, bl1, bh1, sl, 1, true, T.dma(4, later(3), bslot), T.dma(5, later(3), bslot),     \
                 T.dma(6, later(3), bslot), , first)                                                                \
    }                                                                                                               \
    wait_vmcnt<16 + 2 * NJ>();                                                                                      \
    __builtin_amdgcn_s_barrier();                                                                                   \
    FC_PIN();                                                                                                       \
    const char* nx = ring + nxt;                                                                                    \
    if constexpr (NJ == 4) {                                                                                        \
      FC_HALF_P(a1, bl1, bh1, a0, bl0, bh0, nx, 0, true, , , , , second)                                            \
    } else {                                                                                                        \
      FC_HALF3_P(a1, bl1, bh1, a0, bl0, bh0, nx, 0, true, , , , , second)                                           \
    }                                                                                                               \
    pp = prv; prv = cur; cur = nxt;                                                                                 \
    nxt = (nxt + (uint32_t)kStageBytes == (uint32_t)kRingBytes) ? 0u : nxt + (uint32_t)kStageBytes;                 \
    ++s;                                                                                                            \
  }
template <typename Tile>
__device__ __forceinline__ void remote_mainloop(f32x16 (&acc)[4][Tile::NJ], const Tile& T, char* ring, uint32_t ring_addr,
                                                int s0, int S) {
  constexpr int NJ = Tile::NJ;
  const int pad = S & 1, last = S - 1;
  int s = -pad;
  auto later = [&](int n) __attribute__((always_inline)) { return s0 + (s + n < 0 ? 0 : (s + n < last ? s + n : last)); };
  RemoteSet x, y;            // even stages, odd stages
  remote_request(T, x, later(0));
  remote_request(T, y, later(1));
  FC_FENCE();
#pragma unroll
  for (int p = 0; p < 3; ++p)
#pragma unroll
    for (int i = 4; i < 4 + NJ; ++i) T.dma(i, later(p), ring_addr + p * kStageBytes);
#pragma unroll
  for (int w = 0; w < 16; ++w) remote_pair(T, x, w, ring, later(2), pad);
  FC_FENCE();
#pragma unroll
  for (int w = 0; w < 16; ++w) remote_pair(T, y, w, ring + kStageBytes, later(3));
  FC_FENCE();
#pragma unroll
  for (int w = 0; w < 16; ++w) remote_pair(T, x, w, ring + 2 * kStageBytes, later(4));
  FC_FENCE();
  wait_vmcnt<8>();           // the B operands of stages 0 .. 2 have landed: 16 loads of the two sets are younger
  __syncthreads();
  bf16x8 a0[4], a1[4];
  u32x2 bl0[NJ], bh0[NJ], bl1[NJ], bh1[NJ];
#pragma unroll
  for (int t = 0; t < 4; ++t) a0[t] = T.read_a(ring, t, 0);
#pragma unroll
  for (int t = 0; t < NJ; ++t) {
    bl0[t] = T.read_b_half(ring, t, 0, 0);
    bh0[t] = T.read_b_half(ring, t, 0, 1);
  }
  uint32_t cur = 0u, nxt = (uint32_t)kStageBytes, prv = 4u * (uint32_t)kStageBytes, pp = 3u * (uint32_t)kStageBytes;
  while (s < S) {
    FC_STAGE_REMOTE(y)
    FC_STAGE_REMOTE(x)
  }
  wait_vmcnt<0>();           // into slots that nobody has read
  __syncthreads();
}

// Same contraction for tiles with a ragged edge: one stage at a time through registers, zero fill outside.
template <typename Tile>
__device__ __forceinline__ void guarded_mainloop(f32x16 (&acc)[4][Tile::NJ], const Tile& T, char* ring, int s0, int S,
                                                 int tid) {
  bf16x8 a[4], bq[Tile::NJ];
  for (int s = 0; s < S; ++s) {
    __syncthreads();
    T.fill_guarded(s0 + s, ring, tid);
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        a[t] = T.read_a(ring, t, kk);
        if (t < Tile::NJ) bq[t] = T.read_b(ring, t, kk);
      }
#pragma unroll
      for (int ti = 0; ti < 4; ++ti)
#pragma unroll
        for (int tj = 0; tj < Tile::NJ; ++tj) FC_MM(ti, tj, a, bq);
    }
  }
  __syncthreads();
}

// Second pass over the accumulators of one wave of an edge tile when the whole batch is local (b == B, off == 0; the
// first pass is strip_epilogue with the image anchors' row parameters).  Every element s_pj also yields
// f = l2(j, p) = 2^((s - s_jj) log2(e)/tau2_j) of the TEXT anchor j = its contrast column; f goes to the second strip
// F[0] in the form of E[0] and is summed over the wave's anchors.  scol_k / scol_d: log2(e)/tau2_j and s_jj of the
// tile's 256 columns (0 beyond the batch); sredc_w[quantity][column inside the tile] receives the wave's column sums
// of f and of (s - s_jj) f.  Zero outside the batch and on the diagonal j == p (B_{j-} excludes j).  Accumulator
// (ti, tj, v) of lane (lr, hk): contrast c0 + cw + 32 ti + 8 (v >> 2) + 4 hk + (v & 3), anchor a0 + aw + 32 tj + lr.
__device__ __forceinline__ void edge_epilogue_cols(const StripArgs& a, f32x16 (&acc)[4][4], const float* scol_k,
                                                   const float* scol_d, float (*sredc_w)[256], int64_t a0, int64_t c0,
                                                   int cw, int aw, int lane) {
  const int lr = lane & 31, hk = lane >> 5;
  const int B = (int)a.B, b = (int)a.b;
  bf16_t* __restrict__ F = a.F[0];
  const int64_t ab0 = (a0 + aw) >> 5, cb0 = (c0 + cw) >> 4;
#pragma unroll
  for (int ti = 0; ti < 4; ++ti) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {            // the 16-byte fragment store j holds the groups g = 2 j, 2 j + 1
      const int cl = cw + ti * 32 + 16 * j + 4 * hk;     // column inside the tile of (g = 2 j, q = 0)
      const float4 k0 = *(const float4*)(scol_k + cl), k1 = *(const float4*)(scol_k + cl + 8);
      const float4 d0 = *(const float4*)(scol_d + cl), d1 = *(const float4*)(scol_d + cl + 8);
      const float ck[8] = {k0.x, k0.y, k0.z, k0.w, k1.x, k1.y, k1.z, k1.w};
      const float cdk[8] = {d0.x * k0.x, d0.y * k0.y, d0.z * k0.z, d0.w * k0.w,
                            d1.x * k1.x, d1.y * k1.y, d1.z * k1.z, d1.w * k1.w};
      float cs[16];                          // column sums of this lane: f of 8 columns, then t f of 8 columns
#pragma unroll
      for (int i = 0; i < 16; ++i) cs[i] = 0.f;
      const int64_t cb = cb0 + 2 * ti + j;
#pragma unroll
      for (int tj = 0; tj < 4; ++tj) {
        const int anchor = (int)a0 + aw + tj * 32 + lr;
        uint32_t pf[4];
#pragma unroll
        for (int gi = 0; gi < 2; ++gi) {
          const int g = 2 * j + gi;
          float t2[4], f[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) t2[q] = fmaf(acc_read(acc[ti][tj][4 * g + q]), ck[4 * gi + q], -cdk[4 * gi + q]);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int c = (int)c0 + cl + 8 * gi + q;
            const bool ok = (c < B) && (anchor < b) && (c != anchor);
            f[q] = ok ? __builtin_amdgcn_exp2f(t2[q]) : 0.f;
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            cs[4 * gi + q] += f[q];
            cs[8 + 4 * gi + q] = fmaf(t2[q], f[q], cs[8 + 4 * gi + q]);
          }
          pf[2 * gi] = pack_bf16x2(f[0], f[1]);
          pf[2 * gi + 1] = pack_bf16x2(f[2], f[3]);
          FC_PIN();
        }
        const u32x4 wf = {pf[0], pf[1], pf[2], pf[3]};
        if (16 * cb < a.ldE) *(u32x4*)(F + (((ab0 + tj) * a.nCBF + cb) * 64 + lane) * 8) = wf;
        FC_PIN();
      }
      // divide the second quantity by log2(e)/tau_j while each lane still knows its columns, then sum over the lanes
#pragma unroll
      for (int i = 0; i < 8; ++i) cs[8 + i] = ck[i] > 0.f ? cs[8 + i] * __builtin_amdgcn_rcpf(ck[i]) : 0.f;
      lanes32_sum(cs, lane);
      if ((lr & 1) == 0) {
        const int v = lr >> 1, gi = (v >> 2) & 1, q = v & 3;     // value v = 8 quantity + 4 gi + q
        sredc_w[v >> 3][cl + 8 * gi + q] = cs[0];
      }
      FC_PIN();
    }
  }
}

// Tiles with a ragged edge (anchors, contrasts or width not a multiple of the tile): one workgroup per tile, guarded
// epilogue.  The stages that lie wholly inside the width run through the ring of the contraction kernel with unguarded
// direct-to-LDS loads (rows that do not exist are replaced by the tile's last existing row, see StripTile::setup); a
// ragged last stage goes through registers with zero fill.  When the whole batch is local and the similarity matrix is
// formed once (StripArgs::square) the tile also yields the text anchors' exponentials and their sums down the columns.
// After the main loop the ring is free and holds the epilogue's scalars and cross-wave sums.
__global__ void __launch_bounds__(256) k_strips_edge_bf16(StripArgs a) {
  __shared__ __attribute__((aligned(1024))) char ring[kRingBytes];
  float* sk = (float*)ring;                                          // [256] log2(e)/tau of the tile's anchors
  float* sdiag = sk + 256;                                           // [256] s_pp
  float (*sred)[2][256] = (float (*)[2][256])(ring + 2048);          // [contrast half][quantity][anchor]
  float* scol = (float*)(ring + 6144);                               // square: [2][256] log2(e)/tau2_j, s_jj of the columns
  float (*sredc)[2][256] = (float (*)[2][256])(ring + 8192);         // square: [anchor half][quantity][column]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave >> 1, wc = wave & 1;
  const int t = blockIdx.x;
  const int per_strip = a.nAT * a.nCT;
  const int strip = t / per_strip, at = t % a.nAT, ct = (t / a.nAT) % a.nCT;
  const int64_t a0 = strip_anchor_first(a, at, a.square), c0 = (int64_t)ct * 256;
  if (strip_tile_is_interior(a, a0, c0)) return;
  const int S = (int)((a.d + BK - 1) / BK), S_ring = (int)(a.d / BK);
  StripTile T;
  T.setup(a.contrasts[strip], a.ld_contrast[strip], c0, a.B, a.anchors[strip], a.ld_anchor[strip], a0, a.b, a.d, tid);
  f32x16 acc[4][4];
  zero_acc(acc);
  if (S_ring > 0) {
    ring_prologue(T, lds_addr(ring), 0, S_ring);
    ring_mainloop(acc, T, ring, lds_addr(ring), 0, S_ring);
  }
  if (S_ring < S) guarded_mainloop(acc, T, ring, S_ring, S - S_ring, tid);
  {
    const int64_t m = a0 + tid;
    sk[tid] = m < a.b ? a.kscale[strip][m] : 0.f;
    sdiag[tid] = m < a.b ? a.diag[m] : 0.f;
    if (a.square) {                    // off == 0: text anchor j is global row j
      const int64_t j = c0 + tid;
      scol[tid] = j < a.b ? a.kscale[1][j] : 0.f;
      scol[256 + tid] = j < a.b ? a.diag[j] : 0.f;
    }
  }
  __syncthreads();
  strip_epilogue<true, 4, 4>(a, acc, sk, sdiag, sred[wr], strip, a0, c0, wr * 128, wc * 128, lane);
  if (a.square) edge_epilogue_cols(a, acc, scol, scol + 256, sredc[wc], a0, c0, wr * 128, wc * 128, lane);
  __syncthreads();
  const int64_t m = a0 + tid;
  if (m < a.b) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
      a.sums[((size_t)(2 * strip + q) * a.nparts + ct) * a.bstride + m] = sred[0][q][tid] + sred[1][q][tid];
  }
  // the text anchors' sums (quantities 2, 3): partial number = the anchor tile, position = the column
  const int64_t j = c0 + tid;
  if (a.square && j < a.b) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
      a.sums[((size_t)(2 + q) * a.nparts + at) * a.bstride + j] = sredc[0][q][tid] + sredc[1][q][tid];
  }
}

static void make_strip_args(const StepCtx& c, StripArgs* out, bool* any_interior, bool* any_edge);

void launch_strips_bf16(const StepCtx& c) {
  StripArgs a;
  bool any_interior, any_edge;
  make_strip_args(c, &a, &any_interior, &any_edge);
  if (any_interior) launch_strips_interior_bf16(a, c.s);
  if (any_edge) hipLaunchKernelGGL(k_strips_edge_bf16, dim3((unsigned)a.ntiles), dim3(256), 0, c.s, a);
}

// Measurement: the whole-tile strip kernel of the plain mode with parts compiled out and cycle counters (kAbl* in
// kernels_strips.hip).  Only for layouts in which every tile is whole and the mode is the plain one.
bool launch_strips_measure(const StepCtx& c, int ablation, uint64_t* cycles) {
  StripArgs a;
  bool any_interior, any_edge;
  make_strip_args(c, &a, &any_interior, &any_edge);
  if (!any_interior || any_edge || a.square || a.colp) return false;
  a.cycles = cycles;
  return launch_strips_measure_bf16(a, ablation, c.s);
}

static void make_strip_args(const StepCtx& c, StripArgs* out, bool* any_interior_out, bool* any_edge_out) {
  const Layout& L = c.L;
  const bf16_t* img = (const bf16_t*)c.buf.img_glob;
  const bf16_t* txt = (const bf16_t*)c.buf.txt_glob;
  StripArgs& a = *out;
  a.cycles = nullptr;
  a.anchors[0] = img + L.off * c.cfg.ld_img;  a.ld_anchor[0] = c.cfg.ld_img;
  a.anchors[1] = txt + L.off * c.cfg.ld_txt;  a.ld_anchor[1] = c.cfg.ld_txt;
  a.contrasts[0] = txt;                       a.ld_contrast[0] = c.cfg.ld_txt;
  a.contrasts[1] = img;                       a.ld_contrast[1] = c.cfg.ld_img;
  a.diag = (const float*)(c.ws + L.diag);
  a.kscale[0] = (const float*)(c.ws + L.k1);
  a.kscale[1] = (const float*)(c.ws + L.k2);
  a.E[0] = (bf16_t*)(c.ws + L.E[0]);
  a.E[1] = (bf16_t*)(c.ws + L.E[1]);
  a.nCB = L.ldE / 16;
  a.ldE = L.ldE;
  a.sums = (float*)(c.ws + L.sums);
  a.nparts = L.nparts; a.bstride = L.bstride; a.b = L.b; a.B = L.B; a.d = L.d; a.off = L.off;
  a.nAT = (int)((L.b + 255) / 256);
  a.nCT = (int)((L.B + 255) / 256);
  a.square = L.square;
  a.ntiles = (L.square ? 1 : 2) * a.nAT * a.nCT;
  a.colp = L.gathered ? (const float*)(c.ws + L.colp) : nullptr;
  a.F[0] = (L.gathered || L.square) ? (bf16_t*)(c.ws + L.F[0]) : nullptr;
  a.F[1] = L.gathered ? (bf16_t*)(c.ws + L.F[1]) : nullptr;
  a.nCBF = L.ldE / 16;
  const bool d_ok = L.d % 64 == 0 && L.d >= 128;
  bool any_interior = false, any_edge = !d_ok || (L.B % 256);
  for (int at = 0; at < a.nAT; ++at) {
    const bool in = strip_tile_is_interior(a, strip_anchor_first(a, at, a.square), 0);
    any_interior |= in && L.B >= 256;
    any_edge |= !in;
  }
  *any_interior_out = any_interior;
  *any_edge_out = any_edge;
}

// ----------------------------------------------------------------------------------------------------------------
// Local contrast-side term of Eqs. 3 / 5 / 7, folded into the stored strips.  For two local anchors r, q the image
// row of r receives c1_r l1(r, p_q) txt_{p_q} (anchor side, Eq. 2) and c2_q l2(q, p_r) txt_{p_q} (contrast side of
// the text anchor q, Eq. 3): the same row of X with the weight w = c1_r l1(r, p_q) + c2_q l2(q, p_r), which is also
// the weight of img_{p_r} in the text gradient of q.  The strips hold l1(r, .) and l2(q, .) at exactly these
// columns, so the block (rb, qb) replaces E0[r][off + q] by w / c1_r and E1[q][off + r] by w / c2_q (the contraction's
// result is multiplied by the row's own coefficient afterwards) and one contraction per side yields both terms.
//
// A 64 x 64 window of a strip (rows row0 .., columns col0 ..) is read as whole 16-byte fragment chunks and laid out
// as tile[row][column] in LDS; col0 need not be a multiple of 16, so up to 5 column blocks are touched, ten chunks a row,
// of which a thread takes two or three.  All of them, of both windows, are requested before the first is used: what bounds this
// kernel on a small batch is latency, and one after the other they were six trips to memory (1024 local anchors: 8.6 us a
// launch, now 7.3).  A chunk that does not exist is fetched as one that does.
struct FoldChunks { uint4 raw[3]; };
__device__ __forceinline__ void fold_load(const bf16_t* __restrict__ E, int64_t nCB, int64_t row0, int64_t col0, int64_t rows,
                                          FoldChunks& c) {
  const int64_t row = row0 + (threadIdx.x & 63) < rows ? row0 + (threadIdx.x & 63) : rows - 1;
  const int chunks = (col0 & 15) ? 10 : 8;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int ch = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) + 4 * k;
    if (k == 2 && ch >= chunks) break;
    const int64_t cb = (col0 >> 4) + (ch >> 1) < nCB ? (col0 >> 4) + (ch >> 1) : nCB - 1;
    c.raw[k] = *(const uint4*)(E + (((row >> 5) * nCB + cb) * 64 + (row & 31) + 32 * (ch & 1)) * 8);
  }
}
__device__ __forceinline__ void fold_place(const FoldChunks& c, int64_t nCB, int64_t row0, int64_t col0, int64_t rows,
                                           float (*tile)[65]) {
  const int rl = (int)(threadIdx.x & 63);
  if (row0 + rl >= rows) return;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int ch = (int)(threadIdx.x >> 6) + 4 * k;
    if (ch >= ((col0 & 15) ? 10 : 8) || (col0 >> 4) + (ch >> 1) >= nCB) continue;
    const uint32_t w[4] = {c.raw[k].x, c.raw[k].y, c.raw[k].z, c.raw[k].w};
    const int c0 = 16 * (ch >> 1) + 4 * (ch & 1) - (int)(col0 & 15);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int cl = c0 + 8 * (e >> 2) + (e & 3);
      const uint32_t bits = (e & 1) ? (w[e >> 1] & 0xffff0000u) : (w[e >> 1] << 16);
      if (cl >= 0 && cl < 64) tile[rl][cl] = __uint_as_float(bits);
    }
  }
}
// The way back: a chunk that lies wholly inside the window's valid columns is stored as 16 bytes, any other chunk
// element by element (its remaining elements belong to a neighbouring block, which may be storing them right now).
__device__ __forceinline__ void fold_store(bf16_t* __restrict__ E, int64_t nCB, int64_t row0, int64_t col0,
                                           int64_t rows, int cols, float (*tile)[65]) {
  const int64_t cb_first = col0 >> 4, cb_last = (col0 + 63) >> 4;
  for (int i = threadIdx.x; i < 64 * 10; i += 256) {
    const int rl = i & 63, ch = i >> 6;
    const int64_t cb = cb_first + (ch >> 1);
    const int h = ch & 1;
    const int64_t row = row0 + rl;
    if (cb > cb_last || row >= rows) continue;
    bf16_t* dst = E + (((row >> 5) * nCB + cb) * 64 + (row & 31) + 32 * h) * 8;
    const int64_t cl_lo = 16 * cb + 4 * h - col0, cl_hi = cl_lo + 8;   // slots 0..3 and 4..7
    if (cl_lo >= 0 && cl_hi + 3 < cols) {
      const u32x4 w = {pack_bf16x2(tile[rl][cl_lo], tile[rl][cl_lo + 1]), pack_bf16x2(tile[rl][cl_lo + 2], tile[rl][cl_lo + 3]),
                       pack_bf16x2(tile[rl][cl_hi], tile[rl][cl_hi + 1]), pack_bf16x2(tile[rl][cl_hi + 2], tile[rl][cl_hi + 3])};
      *(u32x4*)dst = w;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int64_t cl = (e < 4 ? cl_lo : cl_hi) + (e & 3);
        if (cl >= 0 && cl < cols) dst[e] = f2bf(tile[rl][cl]);
      }
    }
  }
}

// The state phase inside the fold kernels (Layout::fused_state; otherwise k_state has run and the coefficients are
// read).  A block needs the coefficients c1 of its 64 rows r0 .. and c2 of its 64 rows q0 ..: it sums the strip
// phase's partial sums of those anchors (4 threads per anchor and side, then LDS, always in the same order, so every
// block that forms an anchor's coefficient gets the same bits) and applies Eq. 1 to the u^t that the prep kernel
// gathered.  Blocks on the diagonal (r0 == q0) have both sides of their anchors and finish them: scatter of u^{t+1},
// coefficients and diagonal factor for the later phases, Eq. 9, the scalars' partial sums.
// sc: c1_r, c2_q, 1 / c1_r, 1 / c2_q; rows at or beyond b get 1.
struct FoldState {
  float part[4][4][64];   // [quantity][part lane][anchor]
};
__device__ __forceinline__ void fold_coefficients(const StateArgs& a, int64_t r0, int64_t q0, float (*sc)[64],
                                                  FoldState& fs) {
  const int al = threadIdx.x & 63, pl = threadIdx.x >> 6;
  const bool diag = r0 == q0;
  const int side = threadIdx.x >> 6;                       // threads 0..63: side 0 of row r0 + al, 64..127: side 1 of q0 + al
  const int64_t m = (side == 0 ? r0 : q0) + al;
  if (!a.fused) {                                          // the state kernel has left the coefficients
    if (threadIdx.x < 128) {
      const float c = m < a.b ? (side == 0 ? a.c1 : a.c2)[m] : 1.0f;
      sc[side][al] = c;
      sc[2 + side][al] = 1.0f / c;
    }
    return;
  }
  // per-anchor inputs of the threads that form the coefficients below, requested before the sums
  float uo = 0.f, tt = 0.07f, uo_other = 0.f, tt_other = 0.07f;
  if (threadIdx.x < 128 && m < a.b) {
    uo = (side == 0 ? a.uold1 : a.uold2)[m];
    tt = (side == 0 ? a.tau1 : a.tau2)[m];
    if (diag && side == 0) { uo_other = a.uold2[m]; tt_other = a.tau2[m]; }
  }
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int pt = pl; pt < a.nparts; pt += 4) {              // rows up to bstride exist (whole 256-anchor tiles)
    acc[0] += a.sums[((size_t)0 * a.nparts + pt) * a.bstride + r0 + al];
    acc[2] += a.sums[((size_t)2 * a.nparts + pt) * a.bstride + q0 + al];
    if (diag) {
      acc[1] += a.sums[((size_t)1 * a.nparts + pt) * a.bstride + r0 + al];
      acc[3] += a.sums[((size_t)3 * a.nparts + pt) * a.bstride + q0 + al];
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) fs.part[q][pl][al] = acc[q];
  __syncthreads();
  auto total = [&](int q) { return (fs.part[q][0][al] + fs.part[q][1][al]) + (fs.part[q][2][al] + fs.part[q][3][al]); };
  if (diag) {
    if (threadIdx.x < 64) {
      float c1 = 1.0f, c2 = 1.0f;
      double lsum = 0.0, hsum = 0.0;
      if (m < a.b) {
        const float s4[4] = {total(0), total(1), total(2), total(3)};
        state_finish_anchor<false>(a, m, s4, uo, uo_other, tt, tt_other, &c1, &c2, &lsum, &hsum);
      }
      sc[0][al] = c1; sc[1][al] = c2; sc[2][al] = 1.0f / c1; sc[3][al] = 1.0f / c2;
      // the 64 anchors' terms of the loss and of the h sums (Eqs. 8 / 10): one pair per diagonal block
      const double x = wave_sum_f64(lsum), y = wave_sum_f64(hsum);
      if (threadIdx.x == 0) { a.red[2 * blockIdx.x + 0] = x; a.red[2 * blockIdx.x + 1] = y; }
    }
  } else if (threadIdx.x < 128) {
    float c = 1.0f, u_new;
    if (m < a.b) c = anchor_coefficient(a, total(side == 0 ? 0 : 2), uo, tt, &u_new);
    sc[side][al] = c;
    sc[2 + side][al] = 1.0f / c;
  }
}

__global__ void __launch_bounds__(256) k_fold_bf16(bf16_t* __restrict__ E0, bf16_t* __restrict__ E1, int64_t nCB,
                                                   StateArgs a, int64_t off) {
  __shared__ float t0[64][65];   // [r][q]: l1(r, off + q), then w / c1_r
  __shared__ float t1[64][65];   // [q][r]: l2(q, off + r), then w / c2_q
  __shared__ float sc[4][64];    // c1_r, c2_q, 1 / c1_r, 1 / c2_q of the block's rows
  __shared__ FoldState fs;
  const int64_t b = a.b;
  const int64_t r0 = (int64_t)blockIdx.x * 64, q0 = (int64_t)blockIdx.y * 64;
  if (!a.fused) fold_coefficients(a, r0, q0, sc, fs);   // two loads per thread, requested first
  FoldChunks e0, e1;                            // independent of the coefficients: in flight while they are formed
  fold_load(E0, nCB, r0, off + q0, b, e0);
  fold_load(E1, nCB, q0, off + r0, b, e1);
  if (a.fused) fold_coefficients(a, r0, q0, sc, fs);
  fold_place(e0, nCB, r0, off + q0, b, t0);
  fold_place(e1, nCB, q0, off + r0, b, t1);
  __syncthreads();
  const int nr = (int)(b - r0 < 64 ? b - r0 : 64), nq = (int)(b - q0 < 64 ? b - q0 : 64);
  {
    const int ql = threadIdx.x & 63;
    const float cq = sc[1][ql], icq = sc[3][ql];
#pragma unroll 4
    for (int rl = threadIdx.x >> 6; rl < 64; rl += 4) {
      if (rl >= nr || ql >= nq) continue;
      const float w = fmaf(sc[0][rl], t0[rl][ql], cq * t1[ql][rl]);
      t0[rl][ql] = w * sc[2][rl];
      t1[ql][rl] = w * icq;
    }
  }
  __syncthreads();
  fold_store(E0, nCB, r0, off + q0, b, nq, t0);
  fold_store(E1, nCB, q0, off + r0, b, nr, t1);
}

// The same when the whole batch is local and the similarity matrix was formed once: F0[r][q] holds l2(q, p_r) in the
// layout of E0 (off == 0), so w = c1_r E0[r][q] + c2_q F0[r][q]; w / c1_r goes back to E0[r][q] and w / c2_q, transposed,
// to E1[q][r], which nothing has written before: a block writes all 64 columns of its rows of E1, zeros beyond the
// batch, so that every column of E1 up to its padded width holds a number for the contraction.
// What bounds it: memory, two strips read and two written (128 MiB for 4096 pairs).  off == 0, so a window is whole chunks:
// a thread forms w from the two chunks it loads (wave w: column block w of the window, two anchor blocks), stores the
// first result from its registers and passes only the second through LDS, as the bf16 that it stores.  With both windows
// laid out in LDS as fp32, element by element, a step of 4096 pairs at width 768 took 148.2 us; now 137.1.
// (Rows of the LDS window are 36 words apart: the writes of a wave's two halves, four rows apart, go to different banks.)
__global__ void __launch_bounds__(256) k_fold_square_bf16(bf16_t* __restrict__ E0, const bf16_t* __restrict__ F0,
                                                          bf16_t* __restrict__ E1, int64_t nCB, StateArgs a) {
  __shared__ __attribute__((aligned(16))) bf16_t t1[64][72];     // [q][r]: w / c2_q
  __shared__ __attribute__((aligned(16))) float sc[4][64];
  __shared__ FoldState fs;
  const int64_t b = a.b;
  const int64_t r0 = (int64_t)blockIdx.x * 64, q0 = (int64_t)blockIdx.y * 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int h = lane >> 5, ql = 16 * wave + 4 * h;     // the chunk's columns: ql + 0..3, ql + 8..11
  u32x4 ev[2], fv[2];
  if (!a.fused) fold_coefficients(a, r0, q0, sc, fs);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    ev[i] = fv[i] = u32x4{0u, 0u, 0u, 0u};
    if (r0 + 32 * i + (lane & 31) < b) {
      const int64_t at = ((((r0 >> 5) + i) * nCB + (q0 >> 4) + wave) * 64 + lane) * 8;
      ev[i] = *(const u32x4*)(E0 + at);
      fv[i] = *(const u32x4*)(F0 + at);
    }
  }
  if (a.fused) fold_coefficients(a, r0, q0, sc, fs);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int rl = 32 * i + (lane & 31);
    const bool row_ok = r0 + rl < b;
    const float cr = sc[0][rl], icr = sc[2][rl];
    uint32_t out[4];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const float4 cq4 = *(const float4*)&sc[1][ql + 8 * half], icq4 = *(const float4*)&sc[3][ql + 8 * half];
      const float cq[4] = {cq4.x, cq4.y, cq4.z, cq4.w}, icq[4] = {icq4.x, icq4.y, icq4.z, icq4.w};
      float w0[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t ew = ev[i][2 * half + (e >> 1)], fw = fv[i][2 * half + (e >> 1)];
        const float l1 = __uint_as_float((e & 1) ? (ew & 0xffff0000u) : (ew << 16));
        const float l2 = __uint_as_float((e & 1) ? (fw & 0xffff0000u) : (fw << 16));
        const int q = ql + 8 * half + e;
        const float w = row_ok && q0 + q < b ? fmaf(cr, l1, cq[e] * l2) : 0.f;
        w0[e] = w * icr;
        t1[q][rl] = f2bf(w * icq[e]);
      }
      out[2 * half] = pack_bf16x2(w0[0], w0[1]);
      out[2 * half + 1] = pack_bf16x2(w0[2], w0[3]);
    }
    if (row_ok) *(u32x4*)(E0 + ((((r0 >> 5) + i) * nCB + (q0 >> 4) + wave) * 64 + lane) * 8) = u32x4{out[0], out[1], out[2], out[3]};
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {       // E1: rows q, columns r = 16 wave + 4 h + 0..3, 8..11 of the window
    const int q = 32 * i + (lane & 31);
    if (q0 + q >= b) continue;
    const u32x2 lo = *(const u32x2*)&t1[q][ql], hi = *(const u32x2*)&t1[q][ql + 8];
    *(u32x4*)(E1 + ((((q0 >> 5) + i) * nCB + (r0 >> 4) + wave) * 64 + lane) * 8) = u32x4{lo[0], lo[1], hi[0], hi[1]};
  }
}

void launch_fold_bf16(const StepCtx& c) {
  const Layout& L = c.L;
  const unsigned nb = (unsigned)((L.b + 63) / 64);
  const StateArgs st = make_state_args(c);
  if (L.square)
    hipLaunchKernelGGL(k_fold_square_bf16, dim3(nb, nb), dim3(256), 0, c.s, (bf16_t*)(c.ws + L.E[0]),
                       (const bf16_t*)(c.ws + L.F[0]), (bf16_t*)(c.ws + L.E[1]), L.ldE / 16, st);
  else
    hipLaunchKernelGGL(k_fold_bf16, dim3(nb, nb), dim3(256), 0, c.s, (bf16_t*)(c.ws + L.E[0]), (bf16_t*)(c.ws + L.E[1]),
                       L.ldE / 16, st, L.off);
}

// ----------------------------------------------------------------------------------------------------------------
typedef __attribute__((address_space(1))) float global_f32;      // known to be global memory
typedef __attribute__((address_space(1))) f32x4 global_f32x4;
struct ContractJob {
  const bf16_t* E;    // fragment-ordered strip: l of the local anchors with the contrast-side weights folded in
  const bf16_t* X;    // the matrix whose rows the strip weights: texts for strip 0, images for strip 1
  float* C;           // [nsplit][tile][64 groups of 4 rows][64 NJ columns][4 rows]: whole tiles
  int64_t ldx;
  size_t split_stride;
  int64_t nCB;        // column blocks (of 16) per anchor block of E
  int stages, slice;  // 32-deep stages in all; stages per split
};
struct ContractArgs {
  ContractJob job[2];   // the two strips
  int64_t M, N, B;
  int nsplit, tiles_m, tiles_n;
  // gathered state: the second strip, fragment-ordered as E, and the coefficients of the local anchors
  const bf16_t* F[2];
  const float* c_own[2];
};

template <int NJ, bool REMOTE>
__global__ void __launch_bounds__(256) k_contract_bf16(ContractArgs g) {
  constexpr int W = 64 * NJ;       // columns of an output tile
  __shared__ __attribute__((aligned(1024))) char ring[kRingBytes];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const uint32_t ring_addr = lds_addr(ring);
  // Workgroups that share an XCD (id mod 8) take neighbours in the order split, side, column tile, row tile: the same slice of the
  // depth, whose rows of X and fragments of the strips its L2 then fetches once.  With the splits going round the ids every
  // XCD fetched every slice where their number is no multiple of eight: 1792 of 7168 at 1024 (3 splits) 83 us, now 54; 1408 of
  // 22528 at 512 (10) 77 / 66; gathered state 768 of 24576 at 1024 (10) 144 / 94, 2160 of 8640 at 952 (3) 140 / 96.
  const int tiles = g.tiles_m * g.tiles_n;
  const int p = ((int)blockIdx.x & 7) * ((int)gridDim.x >> 3) + ((int)blockIdx.x >> 3);
  if (p >= 2 * tiles * g.nsplit) return;
  const int split = p / (2 * tiles), of_split = p - split * 2 * tiles;
  const int ji = of_split >= tiles, tile = of_split - ji * tiles;
  const ContractJob& J = g.job[ji];
  const int64_t m0 = (int64_t)(tile % g.tiles_m) * 256, n0 = (int64_t)(tile / g.tiles_m) * W;
  const int s0 = split * J.slice;
  const int S = (s0 + J.slice <= J.stages ? J.slice : J.stages - s0);

  f32x16 acc[4][NJ];
  zero_acc(acc);
  if (S > 0) {
    ContractTile<NJ, REMOTE> T;
    T.setup(J.E, J.nCB, m0 >> 5, J.X, J.ldx, n0, g.N, g.B, tid);
    if constexpr (REMOTE) T.setup_remote(g.F[ji], J.nCB, m0 >> 5, g.c_own[ji], g.M, tid);
    // The unguarded loads of a stage take 32 whole rows of X and W columns from n0 on.  They stay inside the matrix
    // (B rows of ldx elements, the last one of N) for the stages below `safe`: rows beyond B never, and where the tile
    // is wider than what is left of a row (n0 + W > N) the words past the row's end are the next rows' - they exist
    // except behind the last rows, and what they put into the columns from N on reaches no output.  Those stages run
    // through the ring; the few that are left at the ragged end go one at a time with guards.
    int64_t rows_ok = g.B;
    if (n0 + W > g.N) rows_ok -= (n0 + W - g.N + J.ldx - 1) / J.ldx;
    const int safe = rows_ok > 0 ? (int)(rows_ok / BK) : 0;
    const int S_ring = s0 + S <= safe ? S : (safe > s0 ? safe - s0 : 0);
    if (S_ring > 0) {
      if constexpr (REMOTE) {
        remote_mainloop(acc, T, ring, ring_addr, s0, S_ring);
      } else {
        ring_prologue(T, ring_addr, s0, S_ring);
        ring_mainloop(acc, T, ring, ring_addr, s0, S_ring);
      }
    }
    if (S_ring < S) guarded_mainloop(acc, T, ring, s0 + S_ring, S - S_ring, tid);
  }
  // The partial result leaves as whole tiles of [64 groups of 4 rows][W columns][4 rows]: a lane holds C[m][n] for
  // n = n0 + wn W/2 + tj 32 + lr and the rows m = m0 + wm 128 + ti 32 + 8 q + 4 hk + t, t = 0..3, so its four values of one
  // q are one 16-byte word of that layout and a wave store covers two runs of 512 consecutive bytes.  The buffer holds
  // whole tiles, so nothing is guarded here; k_finalize_bf16 reads four rows at a time in the same order.  The scalar base
  // keeps its address space through the asm statement: as flat stores the kernel takes 0.5 - 1.5 us longer (832 of 13312 at
  // 240: 27.0 / 25.5, 1024 of 32768 at 1024: 117.5 / 116).
  const int lr = lane & 31, hk = lane >> 5;
  float* C = J.C + (size_t)split * J.split_stride + (size_t)tile * (256 * W);     // wave-uniform
  const uint32_t at = (uint32_t)(((wm * 32 + hk) * W + wn * (W / 2) + lr) * 4);
#pragma unroll
  for (int ti = 0; ti < 4; ++ti)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      global_f32* row = (global_f32*)C + (ti * 8 + q * 2) * (W * 4);
      asm volatile("" : "+s"(row));            // one scalar address per four rows, not one per store in vector registers
#pragma unroll
      for (int tj = 0; tj < NJ; ++tj) {
        const f32x4 v = {acc[ti][tj][4 * q], acc[ti][tj][4 * q + 1], acc[ti][tj][4 * q + 2], acc[ti][tj][4 * q + 3]};
        *(global_f32x4*)(row + at + tj * 128) = v;
      }
    }
}

void launch_contract_bf16(const StepCtx& c) {
  const Layout& L = c.L;
  ContractArgs g;
  for (int s = 0; s < 2; ++s) {
    ContractJob& J = g.job[s];
    J.E = (const bf16_t*)(c.ws + L.E[s]);
    g.F[s] = L.gathered ? (const bf16_t*)(c.ws + L.F[s]) : nullptr;
    g.c_own[s] = (const float*)(c.ws + (s == 0 ? L.c1 : L.c2));
    J.X = (const bf16_t*)(s == 0 ? c.buf.txt_glob : c.buf.img_glob);
    J.ldx = s == 0 ? c.cfg.ld_txt : c.cfg.ld_img;
    J.C = (float*)(c.ws + L.Opart[s]);
    J.split_stride = partial_split_floats(L.b, L.d, L.out_cols);
    J.nCB = L.ldE / 16;
    J.stages = (int)(L.ldE / BK);
    J.slice = (int)L.kslice;
  }
  g.M = L.b; g.N = L.d; g.B = L.B;
  g.nsplit = L.nsplit;
  g.tiles_m = (int)((L.b + 255) / 256);
  g.tiles_n = (int)((L.d + L.out_cols - 1) / L.out_cols);
  const unsigned grid = (2u * (unsigned)(g.nsplit * g.tiles_m * g.tiles_n) + 7) / 8 * 8;
  auto* kernel = L.gathered ? (L.out_cols == 192 ? k_contract_bf16<3, true> : k_contract_bf16<4, true>)
                            : (L.out_cols == 192 ? k_contract_bf16<3, false> : k_contract_bf16<4, false>);
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, c.s, g);
}

}  // namespace fc
