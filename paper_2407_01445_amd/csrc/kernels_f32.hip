// fp32-storage accuracy path of the FCCO step on the fp64 matrix cores (gfx950, wave64, v_mfma_f64_16x16x4_f64): the
// embeddings are fp32, every dot product, every sum over the contrasts and every gradient sum is carried in fp64, and what
// is stored between the phases (exponentials, coefficients) and every output is fp32.
//
//  k_strips_f64  the similarity strips of Proc. 1 on T x T tiles (T anchors against T contrasts): s in fp64, then
//                l = exp((s - s_ii) / tau) stored as fp32, and per anchor the sums of l and of (s - s_ii) l.
//  k_grad_f64    the gradients of Eqs. 2-7 as matrix products on T x T output tiles: the weights
//                w[r][j] = c_own[r] l_own(r, j) + (contrast side) are formed in fp64 while a stage is brought into LDS.
//  k_strips_f32_few, k_grad_f32_few  the same in plain loops, for two dozen pairs at most (at the end of this file).
//
// What bounds them: the fp64 pipes.  A 16x16x4 product takes 64 cycles of its SIMD (measured, dependent or not: 32 flop per
// cycle and SIMD, the fp64 vector rate as well), and no other vector instruction of the SIMD issues meanwhile (measured:
// a product and two conversions take 80 cycles, of two waves 159), so every conversion and address computation comes on
// top.  A dot product per wave - the form this path had before - reads both operands for every element and then spends
// six shuffles on its sum; products on tiles read each operand once per 16 x 16 block.  Measured, before and after:
//                                        strips                gradients
//   128 of 1024 pairs, d = 512, v3      417 ->  12.3 us       398 ->  14.6 us    (0.27 GFLOP each: 4 us at the fp64 rate)
//   1024 pairs, d = 512, v2             996 ->  28 us        1757 ->  46.6 us    (1.07 and 2.15 GFLOP: 14 and 28 us)
// (These two phases alone.  Where the strips prepare their anchors and the gradients run the state phase, as at 128 of 1024, the
// launches take 13.4 and 16.0 us and are the step's only ones.)
// When the whole batch is local (b == B) the text strip is the transpose of the image strip, so only one is formed and
// both sides' weights come from it.
//
// T = 64 where that fills the chip (a tile per compute unit), else T = 32: four times the workgroups at half the operand
// reuse, which the fp64 rate leaves room for (a 32 x 32 tile needs 16 bytes per cycle and compute unit of 64).
#include <string.h>

#include "mfma_common.hpp"
#include "state_common.hpp"

namespace fc {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// D = A B + C on 16 x 16 x 4: lane l gives A[l % 16][l / 16] and B[l / 16][l % 16]; element v of lane l is
// D[4 v + l / 16][l % 16].
__device__ __forceinline__ f64x4 mm_f64(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Four consecutive floats at any 4-byte boundary; the first `have` of them, zeros for the rest.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ f32x4 load4(const float* p) { return (f32x4)*(const f32x4u*)p; }
__device__ __forceinline__ f32x4 load4_guarded(const float* p, int64_t have) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (have > q) v[q] = p[q];
  return v;
}

struct F32StripArgs {
  const float* anchors[2];      // first local row of the anchor side
  const float* contrasts[2];    // row 0 of the contrast side
  int64_t ld_anchor[2], ld_contrast[2];
  int vec[2];                   // both operands of the strip can be fetched as whole 16-byte words (alignment, strides)
  const float* diag;
  const float* tau[2];
  float* E[2];                  // [b][ldE] l of the anchors; square: E[1] is [b][ldE] l2(j, p) at [p][j]
  float* F[2];                  // gathered: c_j l(j, p) of the remote anchors j
  int64_t ldE;
  const float* colp;            // gathered: column parameters (see k_prep), else nullptr
  int64_t ncol;
  float* sums;                  // nparts == 1: float [4][bstride]
  double* sums64;               // nparts > 1: [4][nparts][bstride]
  int nparts, per_part;         // partial sums per anchor and quantity; contrast tiles behind each
  int64_t bstride, b, B, d, off;
  int nAT, nCT, square;
  // PREP: what k_prep reads and leaves for the state phase
  const int64_t* idx;
  int64_t stride;
  const float *tau_glob, *tau_in[2], *u_in[2];     // tau_glob: nullptr with one temperature per sample (V2)
  float *tau_out[2], *u_out[2];
  unsigned* arrived;            // counters of the gradients, zeroed here
  int narrived;
};

constexpr int kFD = 32;                        // depth of a stage: 128 bytes per row

// LDS image of an operand of a stage (T rows x 128 bytes): 16-byte chunk c of row r at chunk position c ^ ((r >> 1) & 7), so
// that the 16 consecutive rows of an operand read cover a 256-byte bank window.  A lane reads whole chunks: its four
// values of k serve four products, whose k slots are then lane / 16 of four different chunks - the same ones for
// both operands, so the order of k does not matter.
__device__ __forceinline__ int fd_off(int row, int chunk) { return row * 128 + ((chunk ^ ((row >> 1) & 7)) << 4); }

// Eight waves, two per SIMD, so that one wave's LDS reads, conversions and barrier waits hide behind the other's products:
// two groups of 2 x 2 waves of T/2 x T/2, which take every other stage and add their accumulators up through the
// similarity tile.  A step of the loop is two stages; the ring holds four steps (T = 32: 64 KiB, T = 64: 128 KiB).
//
// PREP: the workgroup prepares its anchors itself and k_prep is not launched: s_ii of its rows (and, whole batch local, columns),
// 16 threads per row over 16-byte words;
// temperature and u^t by dataset index.
template <int T, bool PREP>
__global__ void __launch_bounds__(512, 2) k_strips_f64(F32StripArgs a) {
  constexpr int W = T / 32;                    // 16 x 16 blocks of a wave in either direction
  constexpr int kSlot = 2 * T * 128, kSteps = 4, kAhead = kSteps - 1, kSlots = 2 * kSteps;
  constexpr int kSpitch = T + 1;               // row pitch of the similarity tile in doubles
  constexpr int CPT = T == 32 ? 2 : 4;         // columns that a thread takes at a time in the row pass
  constexpr int TPR = 512 / T;                 // threads per anchor in the row pass = row groups of the column pass
  __shared__ __attribute__((aligned(1024))) char ring[kSlots * kSlot];
  static_assert(T * kSpitch * 8 + 2 * 512 * 8 <= kSlots * kSlot, "the tile and the column sums reuse the ring");
  double* S = (double*)ring;                                // after the main loop: [T][kSpitch]
  double (*csum)[TPR][T] = (double (*)[TPR][T])(ring + T * kSpitch * 8);    // [quantity][row group][column]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave >> 2, row0 = ((wave >> 1) & 1) * 16 * W, col0 = (wave & 1) * 16 * W;
  const int lr = lane & 15, g = lane >> 4;
  const uint32_t ring_addr = lds_addr(ring);
  warm_arguments<sizeof(F32StripArgs)>();
  const int part = (int)blockIdx.x % a.nparts, at = ((int)blockIdx.x / a.nparts) % a.nAT;
  const int strip = (int)blockIdx.x / (a.nparts * a.nAT);
  const int64_t a0 = (int64_t)at * T;
  const int stages = (int)((a.d + kFD - 1) / kFD), whole = a.vec[strip] ? (int)(a.d / kFD) : 0;
  // row pass: this thread's anchor
  const int prow = tid / TPR, pcol = (tid % TPR) * CPT;
  const int64_t r = a0 + prow;
  const bool live = r < a.b;
  double s_pp = 0.0, inv_tau = 0.0;
  if (!PREP && live) { s_pp = (double)a.diag[r]; inv_tau = 1.0 / (double)a.tau[strip][r]; }
  double sum_e = 0.0, sum_xe = 0.0;
  const int64_t lda = a.ld_anchor[strip], ldx = a.ld_contrast[strip];
  const float* A0 = a.anchors[strip] + a0 * lda;
  const int64_t a_rows = a.b - a0;
  // wave loads of a step: W per wave and operand, 8 rows each; a group requests its own stage
  uint32_t oa[W];
  if (whole) {      // rows that do not exist are fetched as the last one that does; what they yield is discarded
    const int last = (int)(a_rows < T ? a_rows : T) - 1;
#pragma unroll
    for (int i = 0; i < W; ++i) {
      const int row = 8 * ((wave & 3) * W + i) + (lane >> 3);
      oa[i] = (uint32_t)((row < last ? row : last) * (int)lda + (((lane & 7) ^ ((row >> 1) & 7)) << 2)) * 4u;
    }
  }
  const int ct_end = (part + 1) * a.per_part < a.nCT ? (part + 1) * a.per_part : a.nCT;
  // PREP: [rows, columns][s_ii, 1 / tau][T]; threads < 64 gather, of a row (tid < 32) or column tid % 32
  __shared__ double anchor[PREP ? 2 : 1][2][PREP ? T : 1];
  float my_tau = 1.f, my_u = 0.f;
  const int my_set = tid >> 5;                     // 0: the rows' side; 1 (whole batch local): the columns', side 1
  const int64_t my_r = (my_set ? (int64_t)part * T : a0) + (tid & 31);
  const bool gathers = PREP && tid < (a.square ? 64 : 32) && my_r < a.b, keeper = gathers && (my_set ? at : part) == 0;
  if constexpr (PREP) {
    static_assert(T == 32, "16 threads per row");
    if (gathers) {
      const int side = my_set ? 1 : strip;
      my_tau = a.tau_glob ? a.tau_glob[0] : 1.f;
      const int64_t n = a.idx[my_r] * a.stride;
      if (!a.tau_glob) my_tau = a.tau_in[side][n];
      if (keeper) my_u = a.u_in[side][n];
    }
    for (int i = (int)blockIdx.x * 512 + tid; i < a.narrived; i += (int)gridDim.x * 512) a.arrived[i] = 0u;
  }
  if constexpr (PREP) {
    for (int set = 0; set < (a.square ? 2 : 1); ++set) {
      const int row = tid >> 4, sub = tid & 15;
      const int64_t q = (set ? (int64_t)part * T : a0) + row;
      double dot = 0.0;
      if (q < a.b) {
        const float *pa = a.anchors[strip] + q * lda, *px = a.contrasts[strip] + (a.off + q) * ldx;
        for (int64_t k0 = 4 * sub; k0 < a.d; k0 += 512) {         // eight words of either row in flight at once
          f32x4 x[8], y[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int64_t k = k0 + 64 * i;
            x[i] = y[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
            if (k + 4 <= a.d) { x[i] = load4(pa + k); y[i] = load4(px + k); }
            else if (k < a.d) { x[i] = load4_guarded(pa + k, a.d - k); y[i] = load4_guarded(px + k, a.d - k); }
          }
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (k0 + 64 * i < a.d) {
#pragma unroll
              for (int e = 0; e < 4; ++e) dot += (double)x[i][e] * (double)y[i][e];
            }
        }
      }
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) dot += __shfl_xor(dot, o);
      if (sub == 0) anchor[set][0][row] = (double)(float)dot;
    }
  }
  for (int ct = part * a.per_part; ct < ct_end; ++ct) {
    const int64_t c0 = (int64_t)ct * T;
    const float* X0 = a.contrasts[strip] + c0 * ldx;
    const int64_t x_rows = a.B - c0;
    float diag_j = 0.f, tau_j = 1.f;                // square: the column that this thread finishes, requested ahead of everything
    if (!PREP && a.square) {
      const int64_t j = c0 + tid % T < a.B ? c0 + tid % T : a.B - 1;
      diag_j = a.diag[j];
      tau_j = a.tau[1][j];
    }
    f64x4 acc[W][W];
#pragma unroll
    for (int i = 0; i < W; ++i)
#pragma unroll
      for (int j = 0; j < W; ++j) acc[i][j] = (f64x4){0.0, 0.0, 0.0, 0.0};
    auto compute = [&](const char* slot) {
      f32x4 x[2][W], y[2][W];
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int t = 0; t < W; ++t) {
          x[kk][t] = *(const f32x4*)(slot + fd_off(row0 + t * 16 + lr, kk * 4 + g));
          y[kk][t] = *(const f32x4*)(slot + T * 128 + fd_off(col0 + t * 16 + lr, kk * 4 + g));
        }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int p = 0; p < W; ++p)
#pragma unroll
            for (int q = 0; q < W; ++q) acc[p][q] = mm_f64((double)x[kk][p][i], (double)y[kk][q][i], acc[p][q]);
    };
    if (whole) {
      const int last = (int)(x_rows < T ? x_rows : T) - 1;
      uint32_t ox[W];
#pragma unroll
      for (int i = 0; i < W; ++i) {
        const int row = 8 * ((wave & 3) * W + i) + (lane >> 3);
        ox[i] = (uint32_t)((row < last ? row : last) * (int)ldx + (((lane & 7) ^ ((row >> 1) & 7)) << 2)) * 4u;
      }
      const int steps = (whole + 1) / 2;
      // a second stage that does not exist is requested as the last one (nobody reads it): the count per step is constant
      auto request = [&](int step, int at) {
        const int stage = step * 2 + kg < whole ? step * 2 + kg : whole - 1;
        const uint32_t dst = ring_addr + (uint32_t)((at * 2 + kg) * kSlot + (wave & 3) * W * 1024);
#pragma unroll
        for (int i = 0; i < W; ++i) {
          dma16(wave_uniform(A0 + (int64_t)stage * kFD), oa[i], dst + i * 1024);
          dma16(wave_uniform(X0 + (int64_t)stage * kFD), ox[i], dst + T * 128 + i * 1024);
        }
      };
      for (int p = 0; p < kAhead && p < steps; ++p) request(p, p);
      int slot = 0, fill = kAhead;
      for (int s = 0; s < steps; ++s) {
        // step s has landed: vector memory operations complete in order, 2 W of them per younger step
        const int younger = steps - 1 - s < kAhead - 1 ? steps - 1 - s : kAhead - 1;
        if (younger == 0) __builtin_amdgcn_s_waitcnt(0x0f70);
        else if (younger == 1) __builtin_amdgcn_s_waitcnt(W == 1 ? 0x0f72 : 0x0f74);
        else __builtin_amdgcn_s_waitcnt(W == 1 ? 0x0f74 : 0x0f78);
        __builtin_amdgcn_s_barrier();
        FC_FENCE();
        if (s + kAhead < steps) request(s + kAhead, fill);
        if (s * 2 + kg < whole) compute(ring + (slot * 2 + kg) * kSlot);
        FC_FENCE();
        slot = slot + 1 == kSteps ? 0 : slot + 1;
        fill = fill + 1 == kSteps ? 0 : fill + 1;
      }
    }
    for (int s = whole; s < stages; ++s) {          // a ragged last stage, or rows that are not aligned: through registers
      __syncthreads();
      for (int u = tid; u < 2 * T * 8; u += 512) {
        const int op = u / (T * 8), row = (u / 8) % T, chunk = u % 8;
        const int64_t k = (int64_t)s * kFD + chunk * 4;
        const bool there = row < (op ? x_rows : a_rows);
        const float* src = (op ? X0 + row * ldx : A0 + row * lda) + k;
        const f32x4 v = there && k + 4 <= a.d ? load4(src) : load4_guarded(src, there ? a.d - k : 0);
        *(f32x4*)(ring + op * T * 128 + fd_off(row, chunk)) = v;
      }
      __syncthreads();
      if (kg == 0) compute(ring);
    }
    if (gathers) anchor[my_set][1][tid & 31] = 1.0 / (double)my_tau;
    __syncthreads();
    if constexpr (PREP) {
      s_pp = anchor[0][0][prow];
      inv_tau = anchor[0][1][prow];
    }
    for (int half = 0; half < 2; ++half) {
      if (kg == half) {
#pragma unroll
        for (int p = 0; p < W; ++p)
#pragma unroll
          for (int q = 0; q < W; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              double* at = S + (row0 + p * 16 + 4 * v + g) * kSpitch + col0 + q * 16 + lr;
              *at = half ? *at + acc[p][q][v] : acc[p][q][v];
            }
      }
      __syncthreads();
    }
    // row pass: l of the tile's anchors; the own column is not in B_{i-}
    if (live) {
      float* E = a.E[strip] + r * a.ldE + c0;
#pragma unroll
      for (int i = 0; i < T / (CPT * TPR); ++i) {
        const int c = pcol + i * CPT * TPR;
        float e4[CPT];
#pragma unroll
        for (int q = 0; q < CPT; ++q) {
          const double xs = S[prow * kSpitch + c + q] - s_pp;
          const double e = (c0 + c + q < a.B && c0 + c + q != a.off + r) ? exp(xs * inv_tau) : 0.0;
          sum_e += e;
          sum_xe += xs * e;
          e4[q] = (float)e;
        }
        if (c0 + c + CPT - 1 < a.B && a.ldE % CPT == 0) {
          if (CPT == 4) *(float4*)(E + c) = make_float4(e4[0], e4[1], e4[CPT - 2], e4[CPT - 1]);
          else *(float2*)(E + c) = make_float2(e4[0], e4[1]);
        } else {
#pragma unroll
          for (int q = 0; q < CPT; ++q)
            if (c0 + c + q < a.B) E[c + q] = e4[q];
        }
      }
    }
    // column pass: what the contrast column means as an anchor of its own
    if (a.square || a.colp) {                       // block-uniform
      const int col = tid % T, rg = tid / T;
      const int64_t j = c0 + col;
      if (a.square) {                               // l2(j, p) of text anchor j, and its sums over the images
        const bool there = j < a.B;
        const double s_jj = PREP ? anchor[PREP][0][PREP ? col : 0] : (double)diag_j;
        const double inv = PREP ? anchor[PREP][1][PREP ? col : 0] : 1.0 / (double)tau_j;
        double se = 0.0, sx = 0.0;
#pragma unroll
        for (int i = 0; i < T / TPR; ++i) {
          const int row = rg + i * TPR;
          const double xs = S[row * kSpitch + col] - s_jj;
          if (there && a0 + row < a.b) {
            const double e = a0 + row != j ? exp(xs * inv) : 0.0;
            a.E[1][(a0 + row) * a.ldE + j] = (float)e;
            se += e;
            sx += xs * e;
          }
        }
        csum[0][rg][col] = se;
        csum[1][rg][col] = sx;
      } else if (j < a.B) {                         // gathered: the weight c_j l(j, p_r) of a remote anchor j
        const float* cp = a.colp + (((int64_t)strip * (a.ncol >> 8) + (j >> 8)) * 4) * 256 + (j & 255);
        const double kj = (double)cp[0], dj = (double)cp[256], cj = (double)cp[512];
#pragma unroll
        for (int i = 0; i < T / TPR; ++i) {
          const int row = rg + i * TPR;
          if (a0 + row < a.b)
            a.F[strip][(a0 + row) * a.ldE + j] =
                cj == 0.0 ? 0.f : (float)(cj * exp2(S[row * kSpitch + col] * kj - dj));
        }
      }
    }
    __syncthreads();
    if (a.square && tid < 2 * T && c0 + tid % T < a.B) {    // square: one tile per part, partial number = anchor tile
      const int q = tid / T, col = tid % T;
      double s = 0.0;
#pragma unroll
      for (int i = 0; i < TPR; ++i) s += csum[q][i][col];
      if (a.nparts == 1) a.sums[(size_t)(2 + q) * a.bstride + c0 + col] = (float)s;
      else a.sums64[((size_t)(2 + q) * a.nparts + at) * a.bstride + c0 + col] = s;
    }
    __syncthreads();
  }
  if (keeper) {
    const int side = my_set ? 1 : strip;
    a.tau_out[side][my_r] = my_tau;
    a.u_out[side][my_r] = my_u;
  }
#pragma unroll
  for (int o = 1; o < TPR; o <<= 1) {
    sum_e += __shfl_xor(sum_e, o);
    sum_xe += __shfl_xor(sum_xe, o);
  }
  if (live && tid % TPR == 0) {
    // quantities 0, 1 belong to strip 0 (sum l1, sum x1 l1), 2, 3 to strip 1.  A single partial is the whole sum and is
    // rounded to fp32 here; several are kept in fp64 until the state phase has added them up.
    if (a.nparts == 1) {
      a.sums[(size_t)(2 * strip + 0) * a.bstride + r] = (float)sum_e;
      a.sums[(size_t)(2 * strip + 1) * a.bstride + r] = (float)sum_xe;
    } else {
      a.sums64[((size_t)(2 * strip + 0) * a.nparts + part) * a.bstride + r] = sum_e;
      a.sums64[((size_t)(2 * strip + 1) * a.nparts + part) * a.bstride + r] = sum_xe;
    }
  }
}

// Whole 16-byte words of rows `ld` apart; the lane offsets inside a tile are 32-bit.
static bool rows_are_vec(const void* p, int64_t ld) {
  return ((uintptr_t)p & 15) == 0 && ld % 4 == 0 && ld <= ((int64_t)1 << 22);
}

void launch_strips_f32(const StepCtx& c) {
  const Layout& L = c.L;
  const float* img = (const float*)c.buf.img_glob;
  const float* txt = (const float*)c.buf.txt_glob;
  F32StripArgs a;
  memset(&a, 0, sizeof(a));
  a.anchors[0] = img + L.off * c.cfg.ld_img;  a.ld_anchor[0] = c.cfg.ld_img;
  a.anchors[1] = txt + L.off * c.cfg.ld_txt;  a.ld_anchor[1] = c.cfg.ld_txt;
  a.contrasts[0] = txt;                       a.ld_contrast[0] = c.cfg.ld_txt;
  a.contrasts[1] = img;                       a.ld_contrast[1] = c.cfg.ld_img;
  a.vec[0] = a.vec[1] = rows_are_vec(img, c.cfg.ld_img) && rows_are_vec(txt, c.cfg.ld_txt);
  a.diag = (const float*)(c.ws + L.diag);
  a.tau[0] = (const float*)(c.ws + L.tau1);
  a.tau[1] = (const float*)(c.ws + L.tau2);
  for (int s = 0; s < 2; ++s) {
    a.E[s] = (float*)(c.ws + L.E[s]);
    a.F[s] = L.gathered ? (float*)(c.ws + L.F[s]) : nullptr;
  }
  a.ldE = L.ldE;
  a.colp = L.gathered ? (const float*)(c.ws + L.colp) : nullptr;
  a.ncol = L.ncol;
  a.sums = (float*)(c.ws + L.sums);
  a.sums64 = (double*)(c.ws + L.sums);
  a.nparts = L.nparts; a.per_part = L.per_part;
  a.bstride = L.bstride; a.b = L.b; a.B = L.B; a.d = L.d; a.off = L.off;
  const int T = L.strip_tile;
  a.nAT = (int)((L.b + T - 1) / T);
  a.nCT = (int)((L.B + T - 1) / T);
  a.square = L.square;
  const dim3 grid((unsigned)((L.square ? 1 : 2) * a.nAT * a.nparts));
  if (L.own_prep) {
    a.idx = c.buf.idx; a.stride = c.cfg.state_stride;
    a.tau_glob = c.cfg.version == FASTCLIP_V2 ? nullptr : c.buf.tau;
    a.tau_in[0] = c.buf.tau_img; a.tau_in[1] = c.buf.tau_txt;
    a.u_in[0] = c.buf.u_img; a.u_in[1] = c.buf.u_txt;
    a.tau_out[0] = (float*)(c.ws + L.tau1); a.tau_out[1] = (float*)(c.ws + L.tau2);
    a.u_out[0] = (float*)(c.ws + L.uold1); a.u_out[1] = (float*)(c.ws + L.uold2);
    a.arrived = (unsigned*)(c.ws + L.arrived); a.narrived = L.narrived;
  }
  auto* kernel = T == 64 ? k_strips_f64<64, false> : (L.own_prep ? k_strips_f64<32, true> : k_strips_f64<32, false>);
  hipLaunchKernelGGL(kernel, grid, dim3(512), 0, c.s, a);
}

// ------------------------------------------------------------------------------------------
// Gradients.  One range of the contraction's depth: A[m][k] = c_row E + c_col F.  E and F are stored as [m][k], or (trans)
// as [k][m]; c_row belongs to the stored row, c_col to the stored column (nullptr: 1).
struct GradRange {
  const float *E, *F;         // F may be nullptr
  const float *c_row, *c_col;
  const float* X;             // the rows that the weights multiply: row k of this range at X + k ldx
  int64_t K;
  int trans;
};
struct GradSide {
  GradRange range[2];
  int nrange;
  const float* partner;       // rows of the diagonal term: d[r] -= dcoef[r] partner[off + r]
  int64_t ldx;
  float* out;
};
struct GradF32Args {
  GradSide side[2];
  int64_t ldE, b, d, off;
  int tiles_m, tiles_n, nsplit, slice;     // stages per split
  double* part;                            // nsplit > 1: [nsplit][2][tiles][T * T]
  unsigned* arrived;                       // nsplit > 1: [2][tiles], zeroed by the prep kernel or the strips that take its place
  const float* dcoef;
  const double* red; int nred; int version; const float* tau; float rho; float* loss; float* d_tau;
  unsigned* scalars_arrived;               // STATE: 0 before the launch
  int finishers;                           // STATE: workgroups behind the tiles' that finish the anchors
};
constexpr size_t kGradStateAt = (sizeof(GradF32Args) + 7) / 8 * 8;      // the kernel's second argument

// A side's partial sums of anchor r and one quantity, `step` of them from `first` on, in fp64.
__device__ __forceinline__ double add_partials(const StateArgs& a, int quantity, int64_t r, int first, int step) {
  double s = 0.0;
  auto add = [&](const auto* p) {
    for (int p0 = first; p0 < a.nparts; p0 += 8 * step) {         // eight in flight at once
      double v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = (double)p[(size_t)(p0 + i * step < a.nparts ? p0 + i * step : p0) * a.bstride];
#pragma unroll
      for (int i = 0; i < 8; ++i) s += p0 + i * step < a.nparts ? v[i] : 0.0;
    }
  };
  const size_t at = (size_t)quantity * a.nparts * a.bstride + r;
  if (a.sums64) add(a.sums64 + at);
  else add(a.sums + at);
  return s;
}

// STATE.  The coefficients that a workgroup's tile and slice need: own[T] and drow[T] of its rows, other[nk] of the anchors k0 ..
// of the other side, zeros where there is no anchor.  Up to 512 at a time: a power of two of threads share an anchor's sum.
template <int T>
__device__ __forceinline__ void grad_coefficients(const StateArgs& a, int side, int64_t m0, int64_t k0, int nk, float* own, float* drow,
                                                  float* other, double* work) {
  const int items = 2 * T + nk, tid = threadIdx.x;
  int per = 2 * T;                                  // threads of a lane: the least power of two that holds the items, or all
  while (per < items && per < 512) per *= 2;
  const int lane = tid / per, lanes = 512 / per;
  // (the side differs between lanes: chosen among pointers that are there, not by a load from the arguments)
  const float *u1 = wave_uniform(a.uold1), *u2 = wave_uniform(a.uold2), *t1 = wave_uniform(a.tau1), *t2 = wave_uniform(a.tau2);
  for (int i0 = 0; i0 < items; i0 += 512) {
    const int i = i0 + (tid & (per - 1));
    const int s = i < T ? side : 1 - side;
    const int64_t r = i < 2 * T ? m0 + (i & (T - 1)) : k0 + i - 2 * T;
    const bool live = i < items && r < a.b;
    float u = 0.f, tau = 1.f;
    if (live && lane == 0) {
      u = (s ? u2 : u1)[r];
      tau = (s ? t2 : t1)[r];
    }
    double se = 0.0;
    if (live) se = add_partials(a, 2 * s, r, lane, lanes);
    if (lane > 0) work[tid] = se;
    __syncthreads();
    if (lane == 0) {
      float c = 0.f, ce = 0.f;
      if (live) {
        for (int q = 1; q < lanes; ++q) se += work[q * per + i];
        c = anchor_coefficient(a, (float)se, u, tau, &u);
        ce = __fmul_rn(c, (float)se);
      }
      if (i < T) own[i] = c;
      else if (i >= 2 * T && i < items) other[i - 2 * T] = c;
      // c1 M g1 + c2 M g2: a row's two sides are 32 lanes apart
      static_assert(T == 32, "one wave holds both sides of the rows");
      const float both = ce + __shfl_xor(ce, 32);
      if (i < T) drow[i] = both;
    }
    __syncthreads();
  }
}

// STATE.  The state phase of one side of 64 anchors by a workgroup of its own, eight threads per anchor; true in the wave that is
// to form the scalars.
__device__ __forceinline__ bool grad_finish(const GradF32Args& g, const StateArgs& a, int f, double* work, int* flag) {
  const int side = f & 1, tid = threadIdx.x, col = tid & 63, lane = tid >> 6;
  const int64_t r = (int64_t)(f >> 1) * 64 + col;
  const bool live = r < g.b, finisher = live && lane == 0;
  int64_t n = 0;
  float u_old = 0.f, tau = 1.f, m = 0.f, v = 0.f;
  if (finisher) {
    n = a.idx[r] * a.stride;
    u_old = (side ? a.uold2 : a.uold1)[r];
    tau = (side ? a.tau2 : a.tau1)[r];
    if (a.version == FASTCLIP_V2 && a.tau_upd.optimizer) {
      m = (side ? a.m_txt : a.m_img)[n];
      if (keeps_second_moment(a.tau_upd)) v = (side ? a.v_txt : a.v_img)[n];
    }
  }
  double se = live ? add_partials(a, 2 * side, r, lane, 8) : 0.0, sx = live ? add_partials(a, 2 * side + 1, r, lane, 8) : 0.0;
  work[tid] = se;
  work[512 + tid] = sx;
  __syncthreads();
  double lterm = 0.0, hterm = 0.0;
  if (finisher) {
#pragma unroll
    for (int q = 1; q < 8; ++q) { se += work[q * 64 + col]; sx += work[512 + q * 64 + col]; }
    state_finish_side<true>(a, side, r, n, (float)se, (float)sx, u_old, tau, m, v, &lterm, &hterm);
  }
  lterm = wave_sum_f64(lterm);
  hterm = wave_sum_f64(hterm);
  if (tid == 0) {
    double* red = a.red + 2 * f;
    store_agent(red, lterm);
    store_agent(red + 1, hterm);
  }
  return last_to_arrive(g.scalars_arrived, (unsigned)g.finishers, flag) && tid < 64;
}

// T x T output tile, stages of KD of the depth; per thread and stage U words of four weights and of four elements of X.
// The weights are formed in fp64 on the way into LDS, [k][m]; X stays fp32, [k][n].  The pitches put the four k rows that
// an operand read touches (lane / 16) into different banks, and the column of a weight is XORed with its k so that the
// writes of [m][k] words, whose lanes run along k, spread over the banks as well.
// Eight waves: two groups of 2 x 2 waves of T/2 x T/2 that take either half of every stage and add their accumulators up at
// the end (against 2 x 4 waves on whole stages a third fewer LDS reads per product at T = 64: 49 -> 46.6 us; stages of 64
// at T = 64 instead of 32 took 55 us).
template <int T, int KD>
struct GradTile {
  static constexpr int W = T / 32, MC = T / 4, KC = KD / 4, KI = KC / 2, U = T * KD / 2048;
  double (*As)[KD][T + 16];     // [2]
  float (*Xs)[KD][T + 16];      // [2]
  int tid, kg, row0, col0, lr, gk;
  int64_t m0, n0, ldE, ldx, b, d;
  // STATE: the coefficients in LDS, of the tile's rows (this side) and of the slice's anchors k (the other side, from k0 on)
  const float *own, *other;
  int64_t k0;

  // columns of a weight's LDS row k: m ^ swz(k); whole groups of four columns change places
  static __device__ __forceinline__ int swz(int k) { return ((k >> 2) & (T / 4 - 1)) * 4; }

  struct Words { f32x4 e[U], f[U], x[U], cc[U]; float cr[U]; };   // a thread's words of a stage; cr: c_row, cc: c_col of the columns

  // word i of thread tid is number u = tid + 512 i of a stage.  Weights stored as [m][k]: row m0 + u / KC, columns
  // 4 (u % KC) ..; as [k][m]: row u / MC, columns 4 (u % MC) ..; X: row u / MC, columns 4 (u % MC) ..
  template <bool TRANS, bool HAS_F, bool HAS_CC>
  __device__ __forceinline__ void store(const Words& w, int buf) const {
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int u = tid + 512 * i;
      double a[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        a[q] = (double)w.cr[i] * (double)w.e[i][q];
        if (HAS_F) a[q] += HAS_CC ? (double)w.cc[i][q] * (double)w.f[i][q] : (double)w.f[i][q];
      }
      if (TRANS) {
        double* dst = &As[buf][u / MC][((u % MC) * 4) ^ swz(u / MC)];
#pragma unroll
        for (int q = 0; q < 4; ++q) dst[q] = a[q];
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) As[buf][(u % KC) * 4 + q][(u / KC) ^ swz((u % KC) * 4)] = a[q];
      }
      *(f32x4*)&Xs[buf][u / MC][(u % MC) * 4] = w.x[i];
    }
  }
  // the stage's products; `between` runs behind product number KI - 3, whose successors run on while it issues
  template <typename Fn>
  __device__ __forceinline__ void products(f64x4 (&acc)[W][W], int cur, const Fn& between) const {
    double av[2][W];
    float xv[2][W];
    auto read = [&](int i) {
      const int k = 4 * (i + kg * KI) + gk, sw = swz(4 * (i + kg * KI));
#pragma unroll
      for (int t = 0; t < W; ++t) {
        xv[i & 1][t] = Xs[cur][k][col0 + t * 16 + lr];
        av[i & 1][t] = As[cur][k][(row0 + t * 16 + lr) ^ sw];
      }
    };
    read(0);
#pragma unroll
    for (int i = 0; i < KI; ++i) {
      if (i + 1 < KI) read(i + 1);
      FC_PIN();
#pragma unroll
      for (int q = 0; q < W; ++q) {
        const double xd = (double)xv[i & 1][q];
#pragma unroll
        for (int p = 0; p < W; ++p) acc[p][q] = mm_f64(av[i & 1][p], xd, acc[p][q]);
      }
      FC_PIN();
      if (i == KI - 3) { between(); FC_PIN(); }
    }
  }
  // Stages [s0, s1) of one range.  Those that lie wholly inside its depth run as a pipeline: stage s + 2 is requested into
  // one set of registers while stage s + 1 waits in the other to be written to LDS, without a branch in between (the
  // compiler then counts outstanding loads; behind a branch it waits for all of them, which made the kernel wait for
  // memory in every stage: 61 us instead of 49 us on the 1024 x 1024 x 512 step).  Rows and columns of the tile that do not exist are taken from
  // the last ones that do: what they yield is never stored.
  template <bool STATE, bool TRANS, bool HAS_F, bool HAS_CC>
  __device__ __forceinline__ void run(f64x4 (&acc)[W][W], const GradRange& R, int s0, int s1) const {
    const int whole = d % 4 == 0 ? (int)(R.K / KD) : 0;       // d % 4: a word of X would end behind the matrix
    const int p1 = s1 < whole ? s1 : whole;
    const int64_t m_last = TRANS ? (b - 1) & ~(int64_t)3 : b - 1;
    if (s0 < p1) {
      const float *pe[U], *pf[U], *px[U], *pc[U];             // pc: coefficients by k
      float c_fix[U];
      f32x4 cc_fix[U];
#pragma unroll
      for (int i = 0; i < U; ++i) {
        const int u = tid + 512 * i;
        const int64_t m_own = TRANS ? m0 + (u % MC) * 4 : m0 + u / KC, m = m_own < m_last ? m_own : m_last;
        const int64_t k = (int64_t)s0 * KD + (TRANS ? u / MC : (u % KC) * 4);
        const int64_t n_own = n0 + (u % MC) * 4, n = n_own < d - 4 ? n_own : d - 4;
        const int64_t at = TRANS ? k * ldE + m : m * ldE + k;
        pe[i] = R.E + at;
        pf[i] = HAS_F ? R.F + at : nullptr;
        px[i] = R.X + ((int64_t)s0 * KD + u / MC) * ldx + n;
        if constexpr (STATE) {
          pc[i] = other + (k - k0);
          c_fix[i] = TRANS ? 0.f : own[m - m0];
          if (TRANS && HAS_CC) cc_fix[i] = load4(own + (m_own - m0));
        } else {
          pc[i] = (TRANS ? R.c_row : R.c_col) + k;
          c_fix[i] = TRANS ? 0.f : R.c_row[m];
          if (TRANS && HAS_CC) cc_fix[i] = load4(R.c_col + m);
        }
      }
      const int64_t de = TRANS ? (int64_t)KD * ldE : KD, dx = (int64_t)KD * ldx;
      auto load = [&](Words& w, int s) {        // the last stage again once the stages have run out
        const int64_t go = (s < p1 ? s : p1 - 1) - s0;
#pragma unroll
        for (int i = 0; i < U; ++i) {
          w.e[i] = load4(pe[i] + go * de);
          if (HAS_F) w.f[i] = load4(pf[i] + go * de);
          w.x[i] = load4(px[i] + go * dx);
          w.cr[i] = TRANS ? pc[i][go * KD] : c_fix[i];
          if (HAS_CC) w.cc[i] = TRANS ? cc_fix[i] : load4(pc[i] + go * KD);
        }
      };
      Words w0, w1;
      load(w0, s0);
      load(w1, s0 + 1);
      store<TRANS, HAS_F, HAS_CC>(w0, 0);
      __syncthreads();
      for (int s = s0; s < p1; s += 2) {
        load(w0, s + 2);
        products(acc, 0, [&]() { store<TRANS, HAS_F, HAS_CC>(w1, 1); });
        __syncthreads();
        if (s + 1 == p1) break;
        load(w1, s + 3);
        products(acc, 1, [&]() { store<TRANS, HAS_F, HAS_CC>(w0, 0); });
        __syncthreads();
      }
    }
    for (int s = s0 > p1 ? s0 : p1; s < s1; ++s) {            // the ragged end, one stage at a time
      Words w;
#pragma unroll
      for (int i = 0; i < U; ++i) {
        const int u = tid + 512 * i;
        const int64_t m = TRANS ? m0 + (u % MC) * 4 : m0 + u / KC, n = n0 + (u % MC) * 4;
        const int64_t k = (int64_t)s * KD + (TRANS ? u / MC : (u % KC) * 4), kx = (int64_t)s * KD + u / MC;
        const int64_t have = TRANS ? (k < R.K ? b - m : 0) : (m < b ? R.K - k : 0);
        const int64_t at = TRANS ? k * ldE + m : m * ldE + k;
        w.e[i] = load4_guarded(R.E + at, have);
        if (HAS_F) w.f[i] = load4_guarded(R.F + at, have);
        if constexpr (STATE) {                                // zeros behind the last row and the last anchor
          w.cr[i] = TRANS ? other[k - k0] : own[m - m0];
          if (HAS_CC) w.cc[i] = load4(TRANS ? own + (m - m0) : other + (k - k0));
        } else {
          w.cr[i] = TRANS ? (k < R.K ? R.c_row[k] : 0.f) : (m < b ? R.c_row[m] : 0.f);
          if (HAS_CC) w.cc[i] = TRANS ? load4_guarded(R.c_col + m, b - m) : load4_guarded(R.c_col + k, R.K - k);
        }
        w.x[i] = load4_guarded(R.X + kx * ldx + n, kx < R.K ? d - n : 0);
      }
      store<TRANS, HAS_F, HAS_CC>(w, 0);
      __syncthreads();
      products(acc, 0, []() {});
      __syncthreads();
    }
  }
};

// With several splits of the depth the last workgroup of an output tile to arrive adds the partial tiles up in the order of
// the splits, so the result does not depend on who was last.  One more workgroup forms the step's scalars.
//
// STATE (where make_layout says so): the state phase rides along.  Every workgroup forms the coefficients that it needs, a trip to
// memory of some 1.5 us, and workgroups of their own, for which there is room beside the tiles' on a compute unit, finish the
// anchors and the scalars while the products run: a launch of 4 us less (64 pairs at width 32: 18.3 -> 14.8 us a step, 128 of
// 1024 at 512 34.8 -> 31.2).  (By the last workgroup of a row of strip tiles instead the step took longer, 19.5 and 36.1: store,
// count, gather, sums and logarithm come one after the other there.)  The order of the sums differs between the coefficients
// here and the anchors' own, in fp64.
template <int T, int KD, bool STATE>
__global__ void __launch_bounds__(512, 2) k_grad_f64(GradF32Args g, StateArgs state) {
  using Tile = GradTile<T, KD>;
  constexpr int W = Tile::W;
  __shared__ __attribute__((aligned(16))) double As[2][KD][T + 16];
  __shared__ __attribute__((aligned(16))) float Xs[2][KD][T + 16];
  __shared__ int last_flag;
  __shared__ __attribute__((aligned(16))) float own[STATE ? T : 1], drow[STATE ? T : 1], other[STATE ? kGradAnchors : 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  warm_arguments<sizeof(GradF32Args)>();
  const int tiles = g.tiles_m * g.tiles_n;
  if ((int)blockIdx.x >= 2 * tiles * g.nsplit) {
    bool scalars = tid < 64;
    if constexpr (STATE)
      scalars = grad_finish(late_argument<0>(g), late_argument<kGradStateAt>(state), (int)blockIdx.x - 2 * tiles * g.nsplit, &As[0][0][0],
                            &last_flag);
    if (scalars) write_scalars<STATE>(g.red, g.nred, g.b, g.version, g.tau, g.rho, g.loss, g.d_tau);
    return;
  }
  const int split = (int)blockIdx.x % g.nsplit, tile = ((int)blockIdx.x / g.nsplit) % tiles;
  const int side = (int)blockIdx.x / (g.nsplit * tiles);
  const GradSide& Sd = g.side[side];
  Tile t;
  t.As = As; t.Xs = Xs; t.tid = tid;
  t.kg = wave >> 2; t.row0 = ((wave >> 1) & 1) * 16 * W; t.col0 = (wave & 1) * 16 * W;
  t.lr = lane & 15; t.gk = lane >> 4;
  t.m0 = (int64_t)(tile % g.tiles_m) * T; t.n0 = (int64_t)(tile / g.tiles_m) * T;
  t.ldE = g.ldE; t.ldx = Sd.ldx; t.b = g.b; t.d = g.d;
  const int n_first = (int)((Sd.range[0].K + KD - 1) / KD);
  const int n_all = n_first + (Sd.nrange > 1 ? (int)((Sd.range[1].K + KD - 1) / KD) : 0);
  const int s_begin = split * g.slice, s_end = s_begin + g.slice < n_all ? s_begin + g.slice : n_all;

  // the diagonal terms of this thread's outputs (the first group's waves finish the tile).  Rows and columns that do not exist are
  // read as the last ones, so that no lane branches: behind its branches the compiler waited for these loads one by one, 2.7 us of
  // a 64 x 64 tile's 45.
  float dc[W][4] = {}, xp[W][W][4] = {};
  if (t.kg == 0) {
#pragma unroll
    for (int p = 0; p < W; ++p)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t row = t.m0 + t.row0 + p * 16 + 4 * v + t.gk, m = row < g.b ? row : g.b - 1;
        dc[p][v] = STATE ? 0.f : g.dcoef[m];
        const float* of_row = Sd.partner + (g.off + m) * t.ldx;
#pragma unroll
        for (int q = 0; q < W; ++q) {
          const int64_t col = t.n0 + t.col0 + q * 16 + t.lr;
          xp[p][q][v] = of_row[col < g.d ? col : g.d - 1];
        }
      }
  }
  f64x4 acc[W][W];
#pragma unroll
  for (int i = 0; i < W; ++i)
#pragma unroll
    for (int j = 0; j < W; ++j) acc[i][j] = (f64x4){0.0, 0.0, 0.0, 0.0};
  const int q_begin = s_begin > n_first ? s_begin - n_first : 0;               // stages over the other side's strip
  if constexpr (STATE) {
    const bool square = Sd.nrange == 1;
    const int first = square ? s_begin : q_begin, last = square ? s_end : (s_end > n_first ? s_end - n_first : 0);
    t.own = own; t.other = other; t.k0 = (int64_t)first * KD;
    grad_coefficients<T>(late_argument<kGradStateAt>(state), side, t.m0, t.k0, last > first ? (last - first) * KD : 0, own, drow, other,
                         &As[0][0][0]);
#pragma unroll
    for (int p = 0; p < W; ++p)
#pragma unroll
      for (int v = 0; v < 4; ++v) dc[p][v] = drow[t.row0 + p * 16 + 4 * v + t.gk];
  }
  if (s_begin < n_first) {
    const GradRange& R = Sd.range[0];
    const int e = s_end < n_first ? s_end : n_first;
    if (R.trans) t.template run<STATE, true, true, true>(acc, R, s_begin, e);            // square, text side
    else if (Sd.nrange == 1) t.template run<STATE, false, true, true>(acc, R, s_begin, e);      // square, image side
    else if (R.F) t.template run<STATE, false, true, false>(acc, R, s_begin, e);         // gathered state
    else t.template run<STATE, false, false, false>(acc, R, s_begin, e);
  }
  if (s_end > n_first) t.template run<STATE, true, false, false>(acc, Sd.range[1], q_begin, s_end - n_first);
  // the second group's accumulators join the first's (the staging buffers are free)
  double* meet = &As[0][0][0];
  if (t.kg == 1) {
#pragma unroll
    for (int p = 0; p < W; ++p)
#pragma unroll
      for (int q = 0; q < W; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) meet[((p * W + q) * 4 + v) * 256 + (tid & 255)] = acc[p][q][v];
  }
  __syncthreads();
  if (t.kg == 0) {
#pragma unroll
    for (int p = 0; p < W; ++p)
#pragma unroll
      for (int q = 0; q < W; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[p][q][v] += meet[((p * W + q) * 4 + v) * 256 + tid];
  }
  if (g.nsplit > 1) {
    double* P = g.part + ((size_t)(split * 2 + side) * tiles + tile) * (T * T) + tid;
    asm volatile("" : "+v"(P));      // one address per lane: immediate offsets reach the tile's 32 KiB
    if (t.kg == 0) {
#pragma unroll
      for (int p = 0; p < W; ++p)
#pragma unroll
        for (int q = 0; q < W; ++q)
#pragma unroll
          for (int v = 0; v < 4; ++v) store_agent(P + ((p * W + q) * 4 + v) * 256, (double)acc[p][q][v]);
    }
    if (!last_to_arrive(g.arrived + side * tiles + tile, (unsigned)g.nsplit, &last_flag)) return;
    if (t.kg == 0) {
#pragma unroll
      for (int i = 0; i < W; ++i)
#pragma unroll
        for (int j = 0; j < W; ++j) acc[i][j] = (f64x4){0.0, 0.0, 0.0, 0.0};
      const double* Q = g.part + ((size_t)side * tiles + tile) * (T * T) + tid;
      for (int sp = 0; sp < g.nsplit; ++sp, Q += (size_t)2 * tiles * (T * T)) {
#pragma unroll
        for (int p = 0; p < W; ++p)
#pragma unroll
          for (int q = 0; q < W; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[p][q][v] += load_agent(Q + ((p * W + q) * 4 + v) * 256);
      }
    }
  }
  if (t.kg == 0) {
#pragma unroll
    for (int p = 0; p < W; ++p)
#pragma unroll
      for (int q = 0; q < W; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int64_t m = t.m0 + t.row0 + p * 16 + 4 * v + t.gk, n = t.n0 + t.col0 + q * 16 + t.lr;
          if (m < g.b && n < g.d)
            Sd.out[m * g.d + n] = (float)(acc[p][q][v] - (double)dc[p][v] * (double)xp[p][q][v]);
        }
  }
}

void launch_grad_f32(const StepCtx& c) {
  const Layout& L = c.L;
  const float* img = (const float*)c.buf.img_glob;
  const float* txt = (const float*)c.buf.txt_glob;
  const float* coef[2] = {(const float*)(c.ws + L.c1), (const float*)(c.ws + L.c2)};
  GradF32Args g;
  memset(&g, 0, sizeof(g));
  for (int s = 0; s < 2; ++s) {
    GradSide& S = g.side[s];
    const float* X = s == 0 ? txt : img;
    S.partner = X;
    S.ldx = s == 0 ? c.cfg.ld_txt : c.cfg.ld_img;
    S.out = s == 0 ? c.buf.d_img : c.buf.d_txt;
    GradRange& R = S.range[0];
    R.X = X;
    R.K = L.B;
    if (L.square) {            // w[r][j] = c1_r l1(r, j) + c2_j l2(j, r), stored as [r][j] for both sides
      R.E = (const float*)(c.ws + L.E[0]);
      R.F = (const float*)(c.ws + L.E[1]);
      R.c_row = coef[0]; R.c_col = coef[1];
      R.trans = s;
      S.nrange = 1;
    } else {                   // all contrasts with this side's strip, then the local anchors of the other side's strip
      R.E = (const float*)(c.ws + L.E[s]);
      R.F = L.gathered ? (const float*)(c.ws + L.F[s]) : nullptr;
      R.c_row = coef[s];
      GradRange& Q = S.range[1];
      Q.E = (const float*)(c.ws + L.E[1 - s]) + L.off;
      Q.c_row = coef[1 - s];
      Q.trans = 1;
      Q.X = X + L.off * S.ldx;
      Q.K = L.b;
      S.nrange = 2;
    }
  }
  g.ldE = L.ldE; g.b = L.b; g.d = L.d; g.off = L.off;
  const int T = L.grad_tile;
  g.tiles_m = (int)((L.b + T - 1) / T); g.tiles_n = (int)((L.d + T - 1) / T);
  g.nsplit = L.nsplit; g.slice = (int)L.kslice;
  g.part = L.nsplit > 1 ? (double*)(c.ws + L.Opart[0]) : nullptr;
  g.arrived = (unsigned*)(c.ws + L.arrived);
  g.dcoef = (const float*)(c.ws + L.dcoef);
  g.red = (const double*)(c.ws + L.red); g.nred = L.nstate_blocks; g.version = c.cfg.version;
  g.tau = c.buf.tau; g.rho = c.cfg.rho; g.loss = c.buf.loss; g.d_tau = c.buf.d_tau;
  g.finishers = L.grad_state ? L.nstate_blocks : 0;
  g.scalars_arrived = L.grad_state ? g.arrived + L.narrived - 1 : nullptr;
  const dim3 grid((unsigned)(2 * g.tiles_m * g.tiles_n * g.nsplit + (L.grad_state ? g.finishers : 1)));
  auto* kernel = L.grad_state ? k_grad_f64<32, 64, true> : (T == 64 ? k_grad_f64<64, 32, false> : k_grad_f64<32, 64, false>);
  hipLaunchKernelGGL(kernel, grid, dim3(512), 0, c.s, g, make_state_args(c));
}

// ------------------------------------------------------------------------------------------
// Few pairs (at most kFewPairs, kFewNarrowPairs of narrow rows): both phases in plain loops.  There a 32 x 32 tile is mostly padding, and its products
// come one after the other in a single workgroup (per side of the output and 32 columns); a wavefront per dot product
// spreads the few that there are over the chip.  What bounds it: launches (four dependent ones) and, for wide rows, the
// loads' latency.  Steps, tiles / plain, us: 2 pairs at width 64: 17.8 / 17.1, at 1024 29.4 / 17.7, 1 of 2 at 1869
// (unaligned) 56.1 / 23.9, 10 at 1915 47.9 / 45.1, 12 of 16 at 77: 21.7 / 20.0, 23 at 2: 20.4 / 19.7; with more pairs the
// tiles: 23 at 303: 24.7 / 28.2, 64 at 32: 18.6 / 23.0, at 512 26 / 67.
//
// Strips (Proc. 1).  Block (r, side): anchor r against every contrast row j != p; side 0: image anchor vs texts (l1), side 1:
// text anchor vs images (l2).  One wavefront per contrast row, fp64 accumulation; stores l as fp32 and the two row sums.
__global__ void __launch_bounds__(256) k_strips_f32_few(const float* __restrict__ img, const float* __restrict__ txt,
                                                        int64_t ld_img, int64_t ld_txt, int64_t off, int64_t B,
                                                        int64_t d, const float* __restrict__ diag,
                                                        const float* __restrict__ tau1, const float* __restrict__ tau2,
                                                        float* __restrict__ E1, float* __restrict__ E2, int64_t ldE,
                                                        float* __restrict__ sums, int64_t bstride,
                                                        const float* __restrict__ colp, int64_t ncol,
                                                        float* __restrict__ F1, float* __restrict__ F2) {
  const int64_t r = blockIdx.x;
  const int side = blockIdx.y;
  const int64_t p = off + r;
  const float* anchor = side == 0 ? img + p * ld_img : txt + p * ld_txt;
  const float* X = side == 0 ? txt : img;
  const int64_t ldx = side == 0 ? ld_txt : ld_img;
  float* E = (side == 0 ? E1 : E2) + r * ldE;
  float* F = colp ? (side == 0 ? F1 : F2) + r * ldE : nullptr;   // gathered: c_j l(j, p) of every remote anchor j
  const double s_pp = (double)diag[r];
  const double tau = (double)(side == 0 ? tau1[r] : tau2[r]);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double sg = 0.0, sh = 0.0;
  for (int64_t j = wave; j < B; j += 4) {
    const float* x = X + j * ldx;
    double acc = 0.0;
    for (int64_t k = lane; k < d; k += 64) acc += (double)anchor[k] * (double)x[k];
    acc = wave_sum_f64(acc);
    const double xs = acc - s_pp;
    const double e = j == p ? 0.0 : exp(xs / tau);
    if (lane == 0) E[j] = (float)e;
    if (F && lane == 0) {
      const float* cp = colp + (((int64_t)side * (ncol >> 8) + (j >> 8)) * 4) * 256 + (j & 255);
      const double cj = (double)cp[512];
      F[j] = cj == 0.0 ? 0.f : (float)(cj * exp2(acc * (double)cp[0] - (double)cp[256]));
    }
    sg += e;
    sh += xs * e;
  }
  __shared__ double red[2][4];
  if (lane == 0) { red[0][wave] = sg; red[1][wave] = sh; }
  __syncthreads();
  if (threadIdx.x == 0) {
    // quantities 0,1 belong to side 0 (sum e1, sum x1 e1), 2,3 to side 1; nparts == 1 on this path
    sums[(size_t)(2 * side + 0) * bstride + r] = (float)(red[0][0] + red[0][1] + red[0][2] + red[0][3]);
    sums[(size_t)(2 * side + 1) * bstride + r] = (float)(red[1][0] + red[1][1] + red[1][2] + red[1][3]);
  }
}

void launch_strips_f32_few(const StepCtx& c) {
  const Layout& L = c.L;
  dim3 grid((unsigned)L.b, 2), block(256);
  hipLaunchKernelGGL(k_strips_f32_few, grid, block, 0, c.s, (const float*)c.buf.img_glob, (const float*)c.buf.txt_glob,
                     c.cfg.ld_img, c.cfg.ld_txt, L.off, L.B, L.d, (const float*)(c.ws + L.diag),
                     (const float*)(c.ws + L.tau1), (const float*)(c.ws + L.tau2), (float*)(c.ws + L.E[0]),
                     (float*)(c.ws + L.E[1]), L.ldE, (float*)(c.ws + L.sums), L.bstride,
                     L.gathered ? (const float*)(c.ws + L.colp) : nullptr, L.ncol,
                     L.gathered ? (float*)(c.ws + L.F[0]) : nullptr, L.gathered ? (float*)(c.ws + L.F[1]) : nullptr);
}

// Gradients (Eqs. 2-7 for the local rows).  Block (r, side) writes one output row:
//   side 0: d_img[r] = c1_r * sum_j l1(r,j) txt_j - (c1_r M g1_r + c2_r M g2_r) txt_p
//                      + sum_{r' != r} c2_{r'} l2(r', p) txt_{p'}
//   side 1: the mirror image.  The stored strips hold l with the anchor's own column zeroed.
__global__ void __launch_bounds__(256) k_grad_f32_few(const float* __restrict__ img, const float* __restrict__ txt,
                                                      int64_t ld_img, int64_t ld_txt, int64_t off, int64_t b, int64_t B,
                                                      int64_t d, const float* __restrict__ E1, const float* __restrict__ E2,
                                                      int64_t ldE, const float* __restrict__ c1, const float* __restrict__ c2,
                                                      const float* __restrict__ dcoef, float* __restrict__ d_img,
                                                      float* __restrict__ d_txt, const double* __restrict__ red, int nblocks,
                                                      int version, const float* __restrict__ tau, float rho,
                                                      float* __restrict__ loss, float* __restrict__ d_tau,
                                                      const float* __restrict__ F1, const float* __restrict__ F2,
                                                      const float* __restrict__ norm_img,
                                                      const float* __restrict__ norm_txt) {
  const int64_t r = blockIdx.x;
  const int side = blockIdx.y;
  const int64_t p = off + r;
  const float* Fown = F1 ? (side == 0 ? F1 : F2) + r * ldE : nullptr;   // gathered: remote anchors' weights
  const float* X = side == 0 ? txt : img;       // rows that the exp weights multiply
  const int64_t ldx = side == 0 ? ld_txt : ld_img;
  const float* Eown = (side == 0 ? E1 : E2) + r * ldE;       // l of this anchor over all contrasts
  const float* Eoth = side == 0 ? E2 : E1;                   // l of the other local anchors at column p
  const float* cown = side == 0 ? c1 : c2;
  const float* coth = side == 0 ? c2 : c1;
  float* out = (side == 0 ? d_img : d_txt) + r * d;
  int cw = 32;
  while (cw < 256 && cw < d) cw <<= 1;
  const int groups = 256 / cw;
  const int cl = threadIdx.x % cw, grp = threadIdx.x / cw;
  __shared__ double red2[256];
  for (int64_t c0 = 0; c0 < d; c0 += cw) {
    const int64_t col = c0 + cl;
    double acc = 0.0, acc6 = 0.0;
    if (col < d) {
      for (int64_t j = grp; j < B; j += groups) acc += (double)Eown[j] * (double)X[j * ldx + col];
      for (int64_t q = grp; q < b; q += groups)
        acc6 += (double)coth[q] * (double)Eoth[q * ldE + p] * (double)X[(off + q) * ldx + col];
      if (Fown)
        for (int64_t j = grp; j < B; j += groups) acc6 += (double)Fown[j] * (double)X[j * ldx + col];
    }
    red2[threadIdx.x] = (double)cown[r] * acc + acc6;
    __syncthreads();
    if (grp == 0 && col < d) {
      double t = 0.0;
      for (int g = 0; g < groups; ++g) t += red2[g * cw + cl];
      out[col] = (float)(t - (double)dcoef[r] * (double)X[p * ldx + col]);
    }
    __syncthreads();
  }
  if (norm_img) {
    // gradient through e^ = e / |e|: out := (out - e^ (e^ . out)) / |e|, e^ = this side's own row (see k_finalize_bf16)
    const float* ep = side == 0 ? img + p * ld_img : txt + p * ld_txt;
    double dot = 0.0;
    for (int64_t col = threadIdx.x; col < d; col += 256) dot += (double)out[col] * (double)ep[col];
    red2[threadIdx.x] = dot;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
      if ((int)threadIdx.x < w) red2[threadIdx.x] += red2[threadIdx.x + w];
      __syncthreads();
    }
    dot = red2[0];
    const double inv = 1.0 / (double)(side == 0 ? norm_img[r] : norm_txt[r]);
    for (int64_t col = threadIdx.x; col < d; col += 256)
      out[col] = (float)(((double)out[col] - dot * (double)ep[col]) * inv);
  }
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 64)
    write_scalars(red, nblocks, b, version, tau, rho, loss, d_tau);
}

void launch_grad_f32_few(const StepCtx& c) {
  const Layout& L = c.L;
  dim3 grid((unsigned)L.b, 2), block(256);
  hipLaunchKernelGGL(k_grad_f32_few, grid, block, 0, c.s, (const float*)c.buf.img_glob, (const float*)c.buf.txt_glob,
                     c.cfg.ld_img, c.cfg.ld_txt, L.off, L.b, L.B, L.d, (const float*)(c.ws + L.E[0]),
                     (const float*)(c.ws + L.E[1]), L.ldE, (const float*)(c.ws + L.c1), (const float*)(c.ws + L.c2),
                     (const float*)(c.ws + L.dcoef), c.buf.d_img, c.buf.d_txt, (const double*)(c.ws + L.red),
                     L.nstate_blocks, c.cfg.version, c.buf.tau, c.cfg.rho, c.buf.loss, c.buf.d_tau,
                     L.gathered ? (const float*)(c.ws + L.F[0]) : nullptr,
                     L.gathered ? (const float*)(c.ws + L.F[1]) : nullptr, c.buf.norm_img, c.buf.norm_txt);
}

}  // namespace fc
