// MFMA kernels of the FCCO step for batches whose 256 x 256 tiles would leave most of the chip idle (the shapes the paper
// trains at: 128 - 640 anchors per worker of a global batch of 1024 - 5120, width 512):
//
//  k_strips_t128_bf16    the similarity strips of Proc. 1 on tiles of 64 or 128 anchors by 128 contrasts: l = exp((s - s_ii) /
//                        tau), the per-anchor sums of l and (s - s_ii) l, l stored in the fragment order of the contraction;
//                        any ragged edge; where the anchors' rows are few, s_ii and the gathers by dataset index too;
//  k_contract_t128_bf16  everything behind them on output tiles of 32 x 32, 64 x 64 or 128 x 64: the state phase (Eq. 1,
//                        coefficients, Eq. 9, loss) where there is one round of workgroups, the gradient contractions of
//                        Eqs. 2 - 7 with the contrast-side term of the local anchors as further contraction depth, the
//                        outputs and the scalars.
//
// What bounds these batches is not bytes or flops but the chain of dependent launches and, inside a launch, the chain of
// dependent instructions: a launch costs about 3 us, and so does a kernel that waits for memory twice.  So the whole
// step behind the strips is one launch (it was a fold kernel with the state phase, a contraction and a finalize kernel),
// and either kernel keeps as much in flight as the LDS holds: the strips two steps of 128 in k, the contraction 16 KiB
// per wave, every wave on its own slice of the depth with its own LDS region, so that its main loop has no barrier.
//
// Column order.  For this contraction the stored strips and the sums number the contrasts from the worker's own rows on:
// column c is global row (off + c) mod B.  The local anchors are columns 0 .. b - 1 whatever `off` is, so the transposing
// reads of the contrast-side term are always aligned, and a row's own column is its own number.  (For the contraction of
// kernels_wide128.hip the same strips are stored by global row.)  Rows are addressed by 32-bit lane offsets from the
// matrix (B ld < 2^30 elements, checked in make_layout).
#include <string.h>

#include <type_traits>

#include "mfma_common.hpp"
#include "state_common.hpp"

namespace fc {

constexpr int kT = 128;                         // contrasts of a strip tile; its anchors: AT = 64 or 128
constexpr int kD = 64;                          // depth of a strip stage: whole 128-byte lines
constexpr int kPanel = kT * kD * 2;             // the contrasts of a stage: 16 KiB

// The wave's LDS reads have returned (lgkmcnt 0): what it read from may be written again.
__device__ __forceinline__ void wave_reads_done() {
  FC_FENCE();
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __builtin_amdgcn_wave_barrier();
  FC_FENCE();
}

// LDS image of a panel (128 rows x 128 bytes): 16-byte chunk c of row r at chunk position c ^ ((r >> 1) & 7), so that the 16
// consecutive rows of an operand read cover a 256-byte bank window.
__device__ __forceinline__ int p_swz(int row) { return (row >> 1) & 7; }

constexpr float kLog2e = 1.4426950408889634f;

struct T128StripJob {           // one strip
  const bf16_t *X, *A;          // contrast row 0, first local anchor row
  const float* kscale;          // log2(e) / tau of the anchors
  bf16_t *E, *F;                // stored strip; gathered state: second strip
  const float* colp;            // gathered state: [tile of 256 columns][4][256] column parameters
  float* sums;                  // [2][nparts][bstride]
  int ldx, lda;
  // PREP: the side's temperatures and u by dataset index, and where they go for the state phase
  const float *tau, *u;
  float *tau_out, *u_out;
};
struct T128StripArgs {
  T128StripJob job[2];
  const float* diag;            // s_pp per local anchor
  int nCB, ldE, nparts, bstride, b, B, d;
  int first, own;               // global row of column 0; column of local anchor 0
  // PREP
  const int64_t* idx;
  const float* tau_glob;        // nullptr: one temperature per sample (V2)
  int64_t stride;
  unsigned* arrived;            // counters of the contraction, zeroed here
  int narrived;
};

// One workgroup per tile (AT = 128: 128 anchors against 128 contrasts of one strip), eight waves = two groups of 2 x 2 waves of
// 64 x 64: either group takes every other 64-deep stage, so that a SIMD always has a second wave to issue from, an operand
// read serves two products, and the loop has half the barriers; afterwards the groups exchange halves of their
// accumulators and each finishes half of the tile's columns.  AT = 64, 32: the four waves of a group take 32 contrasts each.
// Measured with AT = 128 at 128 anchors of 1024 pairs, d = 512 (a shape that takes AT = 32 now, strips_t128_anchors), against four
// waves on 32-deep stages through a ring of five (k_strips_wide128_bf16): 12.0 -> 8.5 us, of which (in-kernel counters, 2.4
// GHz) 0.4 set-up, 1.1 until the first step is there, 2.6 in the four steps (1.7 of products), 0.7 exchange, 1.5
// exponentials, 0.5 sums.
//
// GATHERED: every element also yields the weight f = c_j 2^(s k_j - d_j) with which contrast column j, an anchor of another
// worker, moves the local row (Eqs. 3 / 5 / 7); it goes to a second strip of the same form.  A workgroup then takes two
// neighbouring contrast tiles one after the other and leaves one partial sum for both: with its second exponential a
// tile is longer, and at the sizes of this path one round of workgroups does for both.
//
// PREP: the workgroup prepares its anchors itself and k_prep is not launched: s_ii = <a_i, x_i> from the anchor rows that pass
// through LDS anyway and the partner rows, eight lanes per anchor and one 16-byte chunk each, summed as in k_prep (fp32 within a
// chunk, fp64 over the chunks), and temperature and u^t by dataset index.  The partner's chunk of a step is requested a
// step ahead and used behind the step's barrier, when everything requested before it has landed.
template <int AT, bool GATHERED, bool PREP>
__global__ void __launch_bounds__(512, 2) k_strips_t128_bf16(T128StripArgs a) {
  static_assert(!(GATHERED && PREP), "gathered state is prepared by k_prep");
  constexpr int NP = AT > 64 ? AT / 64 : 1;       // PREP: anchors per group of eight lanes
  constexpr int NJ = AT == 32 ? 1 : 2;            // 32-row blocks of anchors per wave
  constexpr int WC = AT / (32 * NJ), NI = WC;     // waves across the anchors; 32-row blocks of contrasts per wave
  constexpr int kStage = kPanel + AT * kD * 2, kStep = 2 * kStage;   // a step = one stage for either group of waves
  constexpr int NA = AT / 32, NL = 4 + NA;        // wave loads per step: 4 of the contrasts, 1, 2 or 4 of the anchors
  constexpr int CW = 32 * NI;                     // contrasts of a wave
  __shared__ __attribute__((aligned(1024))) char ring[2 * kStep];    // 80 / 96 / 128 KiB
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave >> 2, q4 = wave & 3, wr = q4 / WC, wc = q4 % WC, lr = lane & 31, hk = lane >> 5;
  const int ct = blockIdx.x, at = blockIdx.y, strip = blockIdx.z;    // no divisions: they are serial instructions at the start
  const int a0 = at * AT;
  const int B = a.B, b = a.b, first = a.first, own = a.own, d = a.d;
  const T128StripJob& J = a.job[strip];
  // pointers pinned in scalar registers: left in the argument segment they are loaded again behind every memory fence
  const bf16_t *Xm = wave_uniform(J.X), *Am = wave_uniform(J.A);
  const int ldx = J.ldx, lda = J.lda;
  const uint32_t ring_addr = lds_addr(ring);
  float total = 0.f;                              // tid < 2 AT: quantity tid / AT of anchor tid % AT
  auto tile = [&](int sub) {
  const int c0 = GATHERED ? ct * 256 + sub * kT : ct * kT;
  // wave loads of a stage: 8 rows x 128 bytes each, four per wave and operand.  A row that does not exist is fetched as
  // the last one that does; what it yields is masked in the epilogue.
  uint32_t ox[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int row = (i < 4 ? 8 * (4 * q4 + i) : 8 * (NA * q4 + i - 4)) + (lane >> 3);
    int g = first + (c0 + row < B ? c0 + row : B - 1);
    g -= g >= B ? B : 0;
    const int m = a0 + row < b ? a0 + row : b - 1;
    ox[i] = (uint32_t)(i < 4 ? g * ldx : m * lda) * 2u + (uint32_t)(((lane & 7) ^ p_swz(row)) * 16);
  }
  const int S = (d + kD - 1) / kD, steps = (S + 1) / 2;
  const int tail = (d % kD) / 8;                  // 16-byte chunks of the last stage that exist (0: all eight)
  // the epilogue's per-anchor scalars (a lane's anchors are a0 + 32 (NJ wc + tj) + lr), requested ahead of everything else
  float kk[NJ], dk[NJ];
#pragma unroll
  for (int tj = 0; tj < NJ; ++tj) {
    const int m = a0 + (wc * NJ + tj) * 32 + lr;
    kk[tj] = !PREP && m < b ? J.kscale[m] : 0.f;
    dk[tj] = !PREP && m < b ? a.diag[m] : 0.f;
  }
  // PREP: anchors 64 i + 8 wave + lane / 8 of the tile (AT = 32: the last four waves do the last anchor's again), chunk lane % 8 of
  // every stage
  const int prow = 8 * wave + (lane >> 3) < AT ? 8 * wave + (lane >> 3) : AT - 1, pch = lane & 7;
  uint32_t po[NP];
  u32x4 partner[2][NP], mine[2][NP];              // [stage of the step][anchor]
  double dot[NP];
  int64_t n = 0;                                  // tid < AT: the anchor's dataset index
  float tau = 1.f, u_old = 0.f;
  const bool keeper = ct == 0;                    // of the workgroups that prepare these anchors the one that leaves them in memory
  auto chunks_of = [&](int st) { return st >= S ? 0 : (tail && st == S - 1 ? tail : 8); };
  auto fetch_partner = [&](auto edge, int step) { // a chunk that does not exist is fetched as the first one, and not used
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      int st = 2 * step + g;
      uint32_t back = 0u;
      if constexpr (decltype(edge)::value) {
        back = pch < chunks_of(st) ? 0u : (uint32_t)pch * 16u;
        st = st < S ? st : S - 1;
      }
#pragma unroll
      for (int i = 0; i < NP; ++i) partner[g][i] = *(const u32x4*)((const char*)(Xm + st * kD) + (po[i] - back));
    }
  };
  auto read_mine = [&](int step) {
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int i = 0; i < NP; ++i)
        mine[g][i] = *(const u32x4*)(ring + (step & 1) * kStep + g * kStage + kPanel + (64 * i + prow) * 128 + ((pch ^ p_swz(prow)) << 4));
  };
  auto add_dots = [&](auto edge, int step) {
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const bool there = !decltype(edge)::value || pch < chunks_of(2 * step + g);
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        float part = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const uint32_t x = mine[g][i][w], y = partner[g][i][w];      // (bit_cast of a vector's element takes element 0)
          part = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, x), __builtin_bit_cast(bf16x2, y), part, false);
        }
        dot[i] += (double)(there ? part : 0.f);
      }
    }
  };
  auto gather = [&]() {                           // behind the index
    if (tid < AT && a0 + tid < b) {
      if (!a.tau_glob) tau = J.tau[n * a.stride];
      if (keeper) u_old = J.u[n * a.stride];
    }
  };
  if constexpr (PREP) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int m = a0 + 64 * i + prow;
      po[i] = (uint32_t)((first + own + (m < b ? m : b - 1)) * ldx) * 2u + (uint32_t)pch * 16u;
      dot[i] = 0.0;
    }
    if (tid < AT && a0 + tid < b) {
      n = a.idx[a0 + tid];
      if (a.tau_glob) tau = a.tau_glob[0];
    }
    fetch_partner(std::true_type{}, 0);
    const int wg = (strip * (int)gridDim.y + at) * (int)gridDim.x + ct, wgs = 2 * (int)gridDim.y * (int)gridDim.x;
    for (int i = wg * 512 + tid; i < a.narrived; i += wgs * 512) a.arrived[i] = 0u;
  }
  float col = 0.f;                                // GATHERED: the tile's column parameters, k_j, d_j, c_j of 128 columns
  if (GATHERED && tid < 3 * kT)
    col = J.colp[(ct * 4 + (tid >> 7)) * 256 + (c0 & 255) + (tid & (kT - 1))];
  // Load i (0 .. 3: contrasts, then anchors) of this wave for a step.  A stage that does not exist is requested as the last
  // one and not used: the number of loads per step is constant.
  const uint32_t my = ring_addr + (uint32_t)(kg * kStage);
  auto request = [&](auto edge, int step, int i) {
    int st = step * 2 + kg;
    uint32_t o = ox[i];
    const int row8 = i < 4 ? 4 * q4 + i : NA * q4 + i - 4;            // its rows: 8 row8 .. + 7 of the panel
    if constexpr (decltype(edge)::value) {
      st = st < S ? st : S - 1;
      if (tail && st == S - 1) {                  // a chunk beyond the row is fetched as the stage's first one, and not used
        const int row = 8 * row8 + (lane >> 3), c = (lane & 7) ^ p_swz(row);
        if (c >= tail) o -= (uint32_t)c * 16u;
      }
    }
    dma16((i < 4 ? Xm : Am) + st * kD, o, my + (uint32_t)((step & 1) * kStep + (i < 4 ? 0 : kPanel) + row8 * 1024));
  };
#pragma unroll
  for (int i = 0; i < NL; ++i) request(std::true_type{}, 0, i);
  if (steps > 1) {
#pragma unroll
    for (int i = 0; i < NL; ++i) request(std::true_type{}, 1, i);
  }
  f32x16 acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  if (steps == 1) FC_WAIT_VMCNT0();
  else wait_vmcnt<NL>();
  __syncthreads();
  FC_FENCE();
  const int rx = wr * CW + lr, ra = wc * NJ * 32 + lr;     // rows 32 further on share the swizzle
  // EDGE: the step holds the last stage (which may end inside, or not exist for group 1)
  auto read = [&](auto edge, int s, int kq, bf16x8 (&x)[NI], bf16x8 (&y)[NJ]) {
    const char* px = ring + (s & 1) * kStep + kg * kStage + rx * 128;
    const char* pa = ring + (s & 1) * kStep + kg * kStage + kPanel + ra * 128;
    const int c = 2 * kq + hk, st = s * 2 + kg;
    const int valid = st >= S ? 0 : (tail && st == S - 1 ? tail : 8);
    const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      u32x4 v = *(const u32x4*)(px + i * 4096 + ((c ^ p_swz(rx)) << 4));
      if constexpr (decltype(edge)::value) v = c < valid ? v : z;
      x[i] = __builtin_bit_cast(bf16x8, v);
    }
#pragma unroll
    for (int i = 0; i < NJ; ++i) {
      u32x4 v = *(const u32x4*)(pa + i * 4096 + ((c ^ p_swz(ra)) << 4));
      if constexpr (decltype(edge)::value) v = c < valid ? v : z;
      y[i] = __builtin_bit_cast(bf16x8, v);
    }
  };
  // The products on (x, y); loads r, r + 1 of step `next` are dealt out between them: a direct-to-LDS load holds its wave for
  // about a hundred cycles when all eight waves issue, which the SIMD's other wave fills with its products.
  auto multiply = [&](auto edge, const bf16x8 (&x)[NI], const bf16x8 (&y)[NJ], bool more, int next, int r) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int p = 0; p < NI; ++p) {              // NI products, then a load
        const int ti = NI == 2 ? h : 0, tj = NI == 2 ? p : h;
        if (tj < NJ) acc[ti][tj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[ti], y[tj], acc[ti][tj], 0, 0, 0);
      }
      FC_PIN();
      if (more && r + h < NL) request(edge, next, r + h);
      FC_PIN();
    }
  };
  // Step s: the loads from 2 on of step s + 1 go out between its first products (0 and 1 went out behind the barrier of step s - 1);
  // three quarters in, the step's panels have been read and the next step's have landed.
  auto step = [&](auto edge_here, auto edge_next, int s) {
    bf16x8 x0[NI], y0[NJ], x1[NI], y1[NJ];
    const bool fill = s > 0 && s + 1 < steps;
    read(edge_here, s, 0, x0, y0);
    read(edge_here, s, 1, x1, y1);
    if constexpr (PREP) read_mine(s);
    multiply(edge_next, x0, y0, fill, s + 1, 2);
    read(edge_here, s, 2, x0, y0);
    multiply(edge_next, x1, y1, fill, s + 1, 4);
    read(edge_here, s, 3, x1, y1);
    multiply(edge_next, x0, y0, fill, s + 1, 6);
    if (s + 1 < steps) {
      FC_WAIT_VMCNT0();
      __syncthreads();
      FC_FENCE();
    }
    multiply(std::true_type{}, x1, y1, s + 2 < steps, s + 2, 0);
    if constexpr (PREP) {                         // while the products run
      add_dots(edge_here, s);
      if (s == 0) gather();
      if (s + 1 < steps) fetch_partner(edge_next, s + 1);
    }
  };
  int s = 0;
  for (; s + 2 < steps; ++s) step(std::false_type{}, std::false_type{}, s);
  for (; s + 1 < steps; ++s) step(std::false_type{}, std::true_type{}, s);
  step(std::true_type{}, std::true_type{}, s);
  // ---- the groups exchange accumulator halves: group g finishes the columns 16 g .. 16 g + 15 of every 32 x 32 block
  __syncthreads();
  auto give = [&](auto group) {
    constexpr int FROM = decltype(group)::value ? 0 : 8;        // the half that the other group finishes
    float* mine = (float*)(ring + wave * 8192) + lane * 4;
#pragma unroll
    for (int ti = 0; ti < NI; ++ti)
#pragma unroll
      for (int tj = 0; tj < NJ; ++tj)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f32x4 w = {acc[ti][tj][FROM + 4 * h], acc[ti][tj][FROM + 4 * h + 1], acc[ti][tj][FROM + 4 * h + 2],
                           acc[ti][tj][FROM + 4 * h + 3]};
          *(f32x4*)(mine + ((ti * NJ + tj) * 2 + h) * 256) = w;
        }
  };
  if (kg) give(std::true_type{}); else give(std::false_type{});
  float* scol = (float*)(ring + 8 * 8192 + 4096);          // GATHERED: [3][128]; PREP: [2][AT], log2(e) / tau and s_ii
  if (GATHERED && tid < 3 * kT) scol[tid] = col;
  if constexpr (PREP) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
#pragma unroll
      for (int o = 1; o < 8; o <<= 1) dot[i] += __shfl_xor(dot[i], o);
      if (pch == 0) scol[AT + 64 * i + prow] = a0 + 64 * i + prow < b ? (float)dot[i] : 0.f;
    }
    if (tid < AT) scol[tid] = a0 + tid < b ? kLog2e / tau : 0.f;
    if (keeper && tid < AT && a0 + tid < b) { J.tau_out[a0 + tid] = tau; J.u_out[a0 + tid] = u_old; }
  }
  __syncthreads();
  if constexpr (PREP) {
#pragma unroll
    for (int tj = 0; tj < NJ; ++tj) {
      kk[tj] = scol[(wc * NJ + tj) * 32 + lr];
      dk[tj] = scol[AT + (wc * NJ + tj) * 32 + lr];
    }
  }
  const float* other = (const float*)(ring + (wave ^ 4) * 8192);
  float (*sred)[2][AT] = (float (*)[2][AT])(ring + 8 * 8192);        // [contrasts' wave, group][quantity][anchor in the tile]: 4 KiB
  bf16_t* __restrict__ E = J.E;
  bf16_t* __restrict__ F = J.F;
  // MASK: the tile reaches beyond the batch or the local anchors, or holds anchors' own columns (B_{i-} excludes i)
  auto finish = [&](auto masked, auto group) {
    constexpr bool MASK = decltype(masked)::value;
    constexpr int OWN = decltype(group)::value ? 8 : 0;
#pragma unroll
    for (int tj = 0; tj < NJ; ++tj) {
      const int al = (wc * NJ + tj) * 32 + lr, anchor = a0 + al;
      const float k = kk[tj], dkk = dk[tj] * k;
      float sg[4] = {0.f, 0.f, 0.f, 0.f}, sx[4] = {0.f, 0.f, 0.f, 0.f};   // independent chains
#pragma unroll
      for (int ti = 0; ti < NI; ++ti) {
        const int c_first = c0 + wr * CW + ti * 32 + kg * 16 + 4 * hk;
        uint32_t pk[4], pf[4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          f32x4 ck, cd, cc;
          if constexpr (GATHERED) {
            const float* cp = scol + c_first - c0 + 8 * h;
            ck = *(const f32x4*)cp; cd = *(const f32x4*)(cp + kT); cc = *(const f32x4*)(cp + 2 * kT);
          }
          float f[4];
          const f32x4 o = *(const f32x4*)(other + ((ti * NJ + tj) * 2 + h) * 256 + lane * 4);
          float e[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float s = acc[ti][tj][OWN + 4 * h + q] + o[q];
            const float x = fmaf(s, k, -dkk);
            if constexpr (GATHERED) {                 // the local rows' c is 0: no mask for the own column
              f[q] = cc[q] * __builtin_amdgcn_exp2f(fmaf(s, ck[q], -cd[q]));
              if (MASK) f[q] = anchor < b ? f[q] : 0.f;
            }
            e[q] = __builtin_amdgcn_exp2f(x);
            if (MASK) {
              const int c = c_first + 8 * h + q;
              e[q] = (c < B && anchor < b && c != own + anchor) ? e[q] : 0.f;
            }
            sg[q] += e[q];
            sx[q] = fmaf(x, e[q], sx[q]);
          }
          pk[2 * h] = pack_bf16x2(e[0], e[1]);
          pk[2 * h + 1] = pack_bf16x2(e[2], e[3]);
          if constexpr (GATHERED) { pf[2 * h] = pack_bf16x2(f[0], f[1]); pf[2 * h + 1] = pack_bf16x2(f[2], f[3]); }
        }
        const int cb = ((c0 + wr * CW) >> 4) + 2 * ti + kg;
        const u32x4 w = {pk[0], pk[1], pk[2], pk[3]};
        const int64_t word = (((int64_t)(a0 / 32 + wc * NJ + tj) * a.nCB + cb) * 64 + lane) * 8;
        if (!MASK || 16 * cb < a.ldE) {
          *(u32x4*)(E + word) = w;
          if constexpr (GATHERED) { const u32x4 wf = {pf[0], pf[1], pf[2], pf[3]}; *(u32x4*)(F + word) = wf; }
        }
      }
      const float g1 = (sg[0] + sg[1]) + (sg[2] + sg[3]), x1 = (sx[0] + sx[1]) + (sx[2] + sx[3]);
      const float g2 = g1 + __shfl_xor(g1, 32), x2 = x1 + __shfl_xor(x1, 32);
      if (hk == 0) {
        sred[wr * 2 + kg][0][al] = g2;
        sred[wr * 2 + kg][1][al] = k > 0.f ? x2 * __builtin_amdgcn_rcpf(k) : 0.f;   // sum of (s - s_pp) l
      }
    }
  };
  const bool whole = a0 + AT <= b && c0 + kT <= B && (own + a0 >= c0 + kT || c0 >= own + a0 + AT);
  if (kg) {
    if (whole) finish(std::false_type{}, std::true_type{}); else finish(std::true_type{}, std::true_type{});
  } else {
    if (whole) finish(std::false_type{}, std::false_type{}); else finish(std::true_type{}, std::false_type{});
  }
  __syncthreads();
  if (tid < 2 * AT) {
    const int q = tid / AT, m = tid % AT;
    float part = 0.f;
#pragma unroll
    for (int w = 0; w < 8 / WC; w += 2) part += sred[w][q][m] + sred[w + 1][q][m];
    total += part;
  }
  if (GATHERED) { __syncthreads(); FC_FENCE(); }
  };
  tile(0);
  if (GATHERED && ct * 256 + kT < B) tile(1);
  if (tid < 2 * AT) {
    const int q = tid / AT, m = tid % AT;
    if (a0 + m < b) J.sums[((size_t)q * a.nparts + ct) * a.bstride + a0 + m] = total;
  }
}

void launch_strips_t128_bf16(const StepCtx& c) {
  const Layout& L = c.L;
  const bf16_t* img = (const bf16_t*)c.buf.img_glob;
  const bf16_t* txt = (const bf16_t*)c.buf.txt_glob;
  T128StripArgs a;
  memset(&a, 0, sizeof(a));
  for (int i = 0; i < 2; ++i) {
    T128StripJob& J = a.job[i];
    J.X = i == 0 ? txt : img;
    J.ldx = (int)(i == 0 ? c.cfg.ld_txt : c.cfg.ld_img);
    J.A = i == 0 ? img + L.off * c.cfg.ld_img : txt + L.off * c.cfg.ld_txt;
    J.lda = (int)(i == 0 ? c.cfg.ld_img : c.cfg.ld_txt);
    J.kscale = (const float*)(c.ws + (i == 0 ? L.k1 : L.k2));
    J.E = (bf16_t*)(c.ws + L.E[i]);
    J.sums = (float*)(c.ws + L.sums) + (size_t)(2 * i) * L.nparts * L.bstride;
    if (L.gathered) {
      J.F = (bf16_t*)(c.ws + L.F[i]);
      J.colp = (const float*)(c.ws + L.colp) + (size_t)i * 4 * L.ncol;
    }
  }
  a.diag = (const float*)(c.ws + L.diag);
  a.nCB = (int)(L.ldE / 16); a.ldE = (int)L.ldE; a.nparts = L.nparts; a.bstride = (int)L.bstride;
  a.b = (int)L.b; a.B = (int)L.B; a.d = (int)L.d;
  a.first = L.wide ? 0 : (int)L.off; a.own = L.wide ? (int)L.off : 0;
  const int rows = strips_t128_anchors(L);
  if (L.own_prep) {
    a.idx = c.buf.idx; a.stride = c.cfg.state_stride;
    a.tau_glob = c.cfg.version == FASTCLIP_V2 ? nullptr : c.buf.tau;
    a.arrived = (unsigned*)(c.ws + L.arrived); a.narrived = L.narrived;
    for (int i = 0; i < 2; ++i) {
      a.job[i].tau = i == 0 ? c.buf.tau_img : c.buf.tau_txt;
      a.job[i].u = i == 0 ? c.buf.u_img : c.buf.u_txt;
      a.job[i].tau_out = (float*)(c.ws + (i == 0 ? L.tau1 : L.tau2));
      a.job[i].u_out = (float*)(c.ws + (i == 0 ? L.uold1 : L.uold2));
    }
  }
  auto* kernel = L.gathered ? (rows == 64 ? k_strips_t128_bf16<64, true, false> : k_strips_t128_bf16<128, true, false>)
                 : L.own_prep ? (rows == 32 ? k_strips_t128_bf16<32, false, true>
                                            : rows == 64 ? k_strips_t128_bf16<64, false, true> : k_strips_t128_bf16<128, false, true>)
                              : (rows == 32 ? k_strips_t128_bf16<32, false, false>
                                            : rows == 64 ? k_strips_t128_bf16<64, false, false> : k_strips_t128_bf16<128, false, false>);
  hipLaunchKernelGGL(kernel, dim3((unsigned)L.nparts, (unsigned)((L.b + rows - 1) / rows), 2), dim3(512), 0, c.s, a);
}

// ----------------------------------------------------------------------------------------------------------------
// Output tiles of 32 RB rows: RB = 1 (32 x 32), 2 (64 x 64) or 4 (128 x 64).  A wave's stage is KS 16-deep steps, NA KiB of the
// strip, 2 KiB of X and, with gathered state, the second strip; as many stages as fit 160 KiB beside the coefficients.
template <int RB> constexpr int kCB = RB == 1 ? 1 : 2;      // blocks of 32 columns
template <int RB> constexpr int kKS = RB == 1 ? 2 : 1;
template <int RB> constexpr int kNA = RB * kKS<RB>;
template <int RB, bool G> constexpr int kWStage = 1024 * (kNA<RB> * (G ? 2 : 1) + 2);
template <int RB, bool G> constexpr int kWSlots = RB < 4 && !G ? 4 : 3;
template <int RB, bool G> constexpr int kWRing = 8 * kWSlots<RB, G> * kWStage<RB, G>;   // 128 / 144 KiB
constexpr int kMaxQ = (kMaxLocalQ + 511) / 512;   // local anchors per thread whose coefficients a workgroup forms

struct T128Job {
  const bf16_t* E;       // fragment-ordered strip of this side
  const bf16_t* F;       // gathered state: the weights c_j l(j, p_r) of the remote anchors j, same form as E
  const bf16_t* Eo;      // ... of the other side, whose columns 0 .. b - 1 are the contrast-side term's weights
  const bf16_t* X;       // the matrix whose rows the strips weight (texts for side 0, images for side 1): also the rows of
                         // the diagonal terms, d_img[r] -= dcoef[r] txt[off + r]
  float* out;            // d_img / d_txt
  int64_t ldx;
};
// Division of numbers below 2^16 by a divisor below 2^16 whose reciprocal the host has formed (0: by 1).  An integer division is
// some forty dependent instructions at the start of a kernel that has nothing to hide them behind.
static inline unsigned reciprocal(int divisor) { return divisor > 1 ? (unsigned)(0xffffffffu / (unsigned)divisor + 1u) : 0u; }
__device__ __forceinline__ int div_small(int x, unsigned inv) { return inv ? (int)(((uint64_t)(unsigned)x * inv) >> 32) : x; }

struct T128Args {
  T128Job job[2];
  int b, d, B, off;
  int64_t nCB;
  int tiles_m, tiles_n, nsplit;
  unsigned inv_tiles, inv_tiles_n;      // reciprocal(2 tiles_m tiles_n), reciprocal(tiles_n)
  int nA, nB;            // stages over the contrasts / over the local anchors
  int sliceA, sliceB;    // ... per wave
  double* part;          // nsplit > 1: [tile][split][64 x 64 floats as pairs]
  unsigned* arrived;     // per 64 rows of an output tile; 0 before the launch
  unsigned* scalars_arrived;   // the same for the workgroups or waves whose terms the scalars are made of
  const double* red;
  int version;
  int nterms;            // pairs in the state phase's list of the scalars' terms
  int finishers;         // leading workgroups that run the state phase; 0: the first workgroups of side 0 do
  float rho;
  const float* tau;
  float *loss, *d_tau;
};

// Output tile (rows from m0, columns from n0) of one side: C = sum_c c_own E[r][c] X[c] + sum_q c_other[q] E_other[q][r] X[q] over
// the contrasts c and the local anchors q (Eq. 2 / 4 / 6 and the local part of Eqs. 3 / 5 / 7; column q is the row X[q] in
// both sums), minus the diagonal term.  The depth is cut into nsplit x 8 slices, one per wave of every workgroup of the
// tile; a wave adds up its part of the first sum, multiplies by the rows' coefficients and goes on with its part of the
// second.  Its operands go through LDS of its own, four 16-deep stages in flight, and nothing but its own waits is in the
// loop.  Then the eight waves' tiles are added up through LDS, and with several splits by the last workgroup to arrive.
//
// The state phase rides along: every workgroup forms the coefficients that it needs from the partial sums while its first
// stages are on their way.  The order of the sums is fixed but not the same everywhere (an output tile's rows as eight
// interleaved runs, local anchors as eight, four, two or one, the finishing workgroups one after the other), so the
// coefficient of an anchor in two workgroups, and the u^{t+1} behind it and the one that is stored, are equal up to the
// rounding of fp32 sums in another order; two steps on the same inputs give the same bits.  The anchors are finished
// (scatter, Eq. 9, loss) by workgroups of their own where compute units are left for them, else by the last waves of the
// workgroups of side 0, split 0 and the first columns, which are late by that (4 us in the chain of one of 12 us).  When there
// is more than one round of workgroups (plan_t128), k_state has run before and the coefficients are read.
//
// What bounds it: operands come at 64 bytes per clock and compute unit, so eight 16-deep stages of 64 x 64 tiles (32 KiB) take
// 512 cycles against 256 of products (650 - 880 measured), and about 5 us go into the start, the coefficients, the sum over
// the waves and the outputs.  128-row tiles (RB = 4) move a quarter less per product and are taken where 64-row ones need
// a second round of workgroups; the cost model is in plan_t128.  Steps before and after (fold + contraction + finalize
// kernels before; strips of 64 anchors included): 128 of 1024 pairs, d = 512: 34.7 -> 20.7 us, 256 of 8192: 47.8 -> 31.2,
// 1024 of 1024: 37.9 -> 30.1, 1000 of 4000, d = 760, rows of 768 (128-row tiles): 71.5 -> 61.9; 640 of 5120 with gathered state
// (a pass over both strips before): 72.5 -> 60.8.  With the workgroups in plain order every XCD fetched every slice of the
// depth: 640 of 5120 gathered 67 us.
// GATHERED: the remote anchors' weights multiply the same rows of X, so the first sum's operand is c_own E + F, formed as
// E + F / c_own (the sum is multiplied by c_own afterwards) between the reads and the products of a stage.
constexpr size_t kStateAt = (sizeof(T128Args) + 7) / 8 * 8;      // the kernel's second argument

// The state phase of 256 anchors by a workgroup of its own (one of g.finishers), a thread per side of an anchor: scatter, outputs,
// Eq. 9, the terms of the scalars, which the last of these workgroups adds up.
// True in the wave that is to form the scalars.
__device__ __forceinline__ bool t128_finish(const T128Args& g, const StateArgs& a, int* flag) {
  const int tid = threadIdx.x, side = __builtin_amdgcn_readfirstlane(tid >> 8), r = (int)blockIdx.x * 256 + (tid & 255);
  double lterm = 0.0, hterm = 0.0;
  if (r < g.b) {
    const int64_t n = a.idx[r] * a.stride;
    const float u = (side ? a.uold2 : a.uold1)[r], tau = (side ? a.tau2 : a.tau1)[r];
    float m = 0.f, v = 0.f;
    if (a.version == FASTCLIP_V2 && a.tau_upd.optimizer) {
      m = (side ? a.m_txt : a.m_img)[n];
      if (keeps_second_moment(a.tau_upd)) v = (side ? a.v_txt : a.v_img)[n];
    }
    const float* e = a.sums + (size_t)(2 * side) * a.nparts * a.bstride + r;
    const float* x = e + (size_t)a.nparts * a.bstride;
    float se = 0.f, sx = 0.f;
    for (int p0 = 0; p0 < a.nparts; p0 += 8) {          // eight partial sums of either quantity in flight at once
      float ve[8], vx[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const size_t o = (size_t)(p0 + i < a.nparts ? p0 + i : p0) * a.bstride;
        ve[i] = e[o];
        vx[i] = x[o];
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) { se += p0 + i < a.nparts ? ve[i] : 0.f; sx += p0 + i < a.nparts ? vx[i] : 0.f; }
    }
    state_finish_side<false>(a, side, r, n, se, sx, u, tau, m, v, &lterm, &hterm);
  }
  lterm = wave_sum_f64(lterm);
  hterm = wave_sum_f64(hterm);
  if ((tid & 63) == 0) {
    double* red = a.red + 2 * ((int64_t)blockIdx.x * 8 + (tid >> 6));
    store_agent(red, lterm);
    store_agent(red + 1, hterm);
  }
  return last_to_arrive(g.scalars_arrived, (unsigned)g.finishers, flag) && tid < 64;
}

template <int RB, bool GATHERED>
__device__ __forceinline__ bool t128_tile(const T128Args& g, const StateArgs& a, char* ring, float* crow, float (*drow)[32 * RB],
                                          float* cq, int* flag) {
  constexpr int kM = 32 * RB, kStageB = kWStage<RB, GATHERED>, kSlotsW = kWSlots<RB, GATHERED>;
  constexpr int CB = kCB<RB>, KS = kKS<RB>, NA = kNA<RB>, kD16 = 16 * KS, kO = 32 * CB, kX = 1024 * NA, kF = kX + 2048;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, hk = lane >> 5;
  // Workgroups that share an XCD (id mod 8) take neighbours in the order split, side, row tile, column tile: the same slice of
  // the depth and the same rows of the strips, which its L2 then fetches once.  The XCD counts, whatever workgroups lead the grid:
  // a side then stays on the XCDs that read the same matrix in the strips.  One XCD further on, 104 of 416 with gathered state
  // took 62.4 us at width 3360 instead of 52.1 (70.2 / 54.5 at 3352), 640 of 5120 at 512 55.4 instead of 54.5.
  const int wg = (int)blockIdx.x - g.finishers, p = ((int)blockIdx.x & 7) * (((int)gridDim.x - g.finishers) >> 3) + (wg >> 3);
  const int tiles = 2 * g.tiles_m * g.tiles_n;
  if (p >= tiles * g.nsplit) return false;
  const int split = div_small(p, g.inv_tiles), tile = p - split * tiles;
  const int sm = div_small(tile, g.inv_tiles_n), tn = tile - sm * g.tiles_n, side = sm >= g.tiles_m, tm = sm - side * g.tiles_m;
  const int m0 = tm * kM, n0 = tn * kO;
  const T128Job& J = g.job[side];
  // pinned in scalar registers: left in the argument segment they are loaded again behind every memory fence
  const int B = __builtin_amdgcn_readfirstlane(g.B), ldx = __builtin_amdgcn_readfirstlane((int)J.ldx);
  const bf16_t* X = wave_uniform(J.X);
  const int d = __builtin_amdgcn_readfirstlane(g.d);
  const int qbase = split * 8 * g.sliceB * kD16;     // this workgroup's local anchors q
  int nq = g.b - qbase < 8 * g.sliceB * kD16 ? g.b - qbase : 8 * g.sliceB * kD16;
  nq = nq < 0 ? 0 : nq;
  const int nq16 = (nq + kD16 - 1) & ~(kD16 - 1);    // coefficients that the stages over the local anchors read

  // ---- operand requests
  const int unit = split * 8 + wave;
  const int A0 = unit * g.sliceA, nAw = A0 >= g.nA ? 0 : (A0 + g.sliceA <= g.nA ? g.sliceA : g.nA - A0);
  const int Q0 = unit * g.sliceB, nBw = Q0 >= g.nB ? 0 : (Q0 + g.sliceB <= g.nB ? g.sliceB : g.nB - Q0);
  const int nst = nAw + nBw;
  const uint32_t wring = lds_addr(ring) + (uint32_t)(wave * kSlotsW * kStageB);
  const char* wslot = ring + wave * kSlotsW * kStageB;
  // X: two wave loads of 8 rows x 128 bytes; 16-byte piece p of stage row k at piece p ^ (4 ((k >> 1) & 1)), so that the 4 rows x
  // 64 bytes that a transposing read touches cover a bank window.  RB = 1: of 16 rows x 64 bytes, which do as they are.  Rows
  // wrap at B; pieces beyond the width are fetched as the row's first of the tile and reach no output.
  int grow[2];
  uint32_t xoff[2];
  const uint32_t wrap = (uint32_t)(B * ldx) * 2u, next_rows = (uint32_t)(kD16 * ldx) * 2u;
  auto open_rows = [&](int col) {              // columns col .. col + kD16 - 1
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int k = RB == 1 ? 16 * i + (lane >> 2) : 8 * i + (lane >> 3);
      const int pc = RB == 1 ? lane & 3 : (lane & 7) ^ (((k >> 1) & 1) << 2);
      int r = g.off + col + k;                 // below 2 B + 32: a division would take longer
      while (r >= B) r -= B;
      grow[i] = r;
      xoff[i] = (uint32_t)(r * ldx + (n0 + pc * 8 < d ? n0 + pc * 8 : n0)) * 2u;
    }
  };
  // Strip operand of the first sum: the fragments (m0 / 32 + i, stage), 1 KiB each; RB = 1: (m0 / 32, 2 stage + i).  Of the second:
  // 16 KS anchors q x kM columns r as chunks of 16 bytes, [column block][half][q] with q at q ^ (4 half) ^ (8 (column block & 1)),
  // again for the transposing reads' bank windows.
  const char* src = nullptr;                   // uniform; stage `at` comes from src + woff[i]
  uint32_t woff[NA];
  const uint32_t row_block = (uint32_t)g.nCB * 1024u;
  int at = 0;                                  // next stage to request
  auto open_own = [&]() {
    src = wave_uniform((const char*)J.E + ((int64_t)(m0 >> 5) * g.nCB + A0 * KS) * 1024);
#pragma unroll
    for (int i = 0; i < NA; ++i) woff[i] = (uint32_t)(lane * 16) + (uint32_t)i * (RB == 1 ? 1024u : row_block);
    open_rows(A0 * kD16);
  };
  const char* src_other = wave_uniform((const char*)J.Eo + ((int64_t)(KS == 2 ? Q0 : Q0 >> 1) * g.nCB + (m0 >> 4)) * 1024 +
                                       (KS == 2 ? 0 : (Q0 & 1) * 256));
  auto open_other = [&]() {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int cb = RB == 1 ? i : 2 * i + (lane >> 5), h = RB == 1 ? lane >> 5 : (lane >> 4) & 1;
      const int q = (lane & (kD16 - 1)) ^ (4 * h) ^ (8 * (cb & 1));
      woff[i] = (uint32_t)((cb * 64 + q + 32 * h) * 16);
    }
    open_rows(Q0 * kD16);
  };
  const int64_t to_f = GATHERED ? (const char*)wave_uniform(J.F) - (const char*)wave_uniform(J.E) : 0;
  uint32_t fill = wring;                       // slot of stage `at`
  auto request = [&]() {
#pragma unroll
    for (int i = 0; i < NA; ++i) dma16(src, woff[i], fill + (uint32_t)(i * 1024));
    if (GATHERED && at < nAw) {
#pragma unroll
      for (int i = 0; i < NA; ++i) dma16(src + to_f, woff[i], fill + (uint32_t)(kF + i * 1024));
    }
    dma16(X, xoff[0], fill + (uint32_t)kX);
    dma16(X, xoff[1], fill + (uint32_t)(kX + 1024));
    fill = fill + kStageB == wring + kSlotsW * kStageB ? wring : fill + kStageB;
    ++at;
    src = at == nAw ? src_other
                    : src + (at < nAw ? 1024u * KS : (KS == 2 ? row_block : (((Q0 + at - nAw) & 1) ? 256u : row_block - 256u)));
    if (at == nAw) {
      open_other();
    } else {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        grow[j] += kD16; xoff[j] += next_rows;
        if (grow[j] >= B) { grow[j] -= B; xoff[j] -= wrap; }
      }
    }
  };
  src = src_other;
  if (nAw > 0) open_own(); else open_other();
  if (nst > 0) request();

  // ---- the coefficients: of the rows (both sides, for the diagonal factor too) and of the q's (the other side).  Their inputs are
  // requested behind the first stage, the other stages behind the inputs' arrival: vector memory operations complete in order.
  auto request_more = [&]() {
    for (int s = 1; s < kSlotsW - 1 && s < nst; ++s) request();
  };
  const bool fused = a.fused;
  const bool finisher = fused && g.finishers == 0 && side == 0 && tn == 0 && split == 0;
  constexpr int kFin = RB == 1 ? 2 : RB;             // a finisher's last waves finish a side of (up to) 64 anchors each, images first
  const int fw = wave - (8 - kFin), fside = fw >= kFin / 2, frow = (fside ? fw - kFin / 2 : fw) * 64 + lane;
  const bool finishing = finisher && fw >= 0 && frow < kM && m0 + frow < g.b;
  double lterm = 0.0, hterm = 0.0;
  if (fused) {
    // Sums of the q's: groups of 256 anchors, one wave load per group and partial sum, dealt out to the waves: wave w takes group
    // w % groups_w (and that plus 8) and every slices-th partial sum.
    const int groups = (nq + 255) >> 8;
    const int lg = groups > 4 ? 3 : (groups > 2 ? 2 : (groups > 1 ? 1 : 0)), groups_w = 1 << lg, slices = 8 >> lg;
    // partial sums of a wave, [4 quantities][rows] and [2 groups][256], in the slot of its ring that is requested last (behind the
    // second barrier below)
    auto psum = [&](int w) { return (float*)(ring + (w * kSlotsW + kSlotsW - 1) * kStageB); };
    static_assert(kStageB >= (4 * kM + 512) * 4 && kMaxLocalQ <= 16 * 256, "the partial sums fit a slot");
    // Addresses are a wave-uniform base and a 32-bit byte offset per lane: what bounds this part is the number of instructions
    // (with 64-bit addresses per lane 6500 cycles from the first request to the sums in LDS).
    auto at = [](const float* base, uint32_t bytes) { return *(const float*)((const char*)base + bytes); };
    const int rside = RB == 1 ? hk : wave >= RB / 2, row = tid & (kM - 1);      // tid < 2 kM: side and row of a coefficient
    auto one_of = [&](const float* img, const float* txt) {       // RB = 1: the side differs between lanes
      return RB == 1 ? (rside ? txt : img) : wave_uniform(rside ? txt : img);
    };
    const bool rows_here = tid < 2 * kM && m0 + row < g.b;
    int64_t fn = 0;                                  // dataset index
    float fu = 0.f, ft = 1.f, fm = 0.f, fv = 0.f, ur = 0.f, tr = 1.f, uq[kMaxQ], tq[kMaxQ];
    const uint32_t last_anchor = (uint32_t)(g.b - 1);
    if (finisher && fw >= 0) {                       // anchors that do not exist as the last one
      const uint32_t m = (uint32_t)(m0 + frow) < last_anchor ? (uint32_t)(m0 + frow) : last_anchor;
      fn = *(const int64_t*)((const char*)a.idx + m * 8u);
      fu = at(wave_uniform(fside ? a.uold2 : a.uold1), m * 4u);
      ft = at(wave_uniform(fside ? a.tau2 : a.tau1), m * 4u);
    }
    if (wave < RB) {
      const uint32_t m = (uint32_t)(m0 + row) < last_anchor ? (uint32_t)(m0 + row) : last_anchor;
      ur = at(one_of(a.uold1, a.uold2), m * 4u);
      tr = at(one_of(a.tau1, a.tau2), m * 4u);
    }
    const float *u_other = wave_uniform(side ? a.uold1 : a.uold2), *t_other = wave_uniform(side ? a.tau1 : a.tau2);
    const int j0 = (tid - 2 * kM) & 511, jw = (wave * 64 - 2 * kM) & 511;    // q's behind the threads that have the rows
#pragma unroll
    for (int i = 0; i < kMaxQ; ++i) {
      uq[i] = 0.f; tq[i] = 1.f;
      if (jw + 512 * i < nq) {                       // wave-uniform
        const uint32_t m = (uint32_t)(qbase + j0 + 512 * i) < last_anchor ? (uint32_t)(qbase + j0 + 512 * i) : last_anchor;
        uq[i] = at(u_other, m * 4u);
        tq[i] = at(t_other, m * 4u);
      }
    }
    // four anchors per lane; what lies behind the anchors (up to bstride) is added up and not used
    const int bs = (int)a.bstride, nparts = a.nparts;
    const char* sums = (const char*)wave_uniform(a.sums);
    auto words_at = [&](int quantity, int m) { return (uint32_t)(quantity * nparts * bs + (m < bs ? m : bs - 4)) * 4u; };
    auto words = [&](int pt, uint32_t off) { return *(const f32x4*)(sums + (uint32_t)(pt * bs) * 4u + off); };
    // partial sums wave, wave + 8, .. of the rows (a lane's quantity: lane / 16; RB = 4: 2 (lane / 32) + i; RB = 1: lane / 8 % 4), and
    // wave / groups_w, + slices, .. of the wave's group of q's: up to 16 of the latter in flight at once
    constexpr int NR = RB == 4 ? 2 : 1;
    const int rq0 = RB == 4 ? 2 * (lane >> 5) : (RB == 1 ? (lane >> 3) & 3 : lane >> 4), r4 = 4 * (lane & (8 * RB - 1));
    uint32_t pr[NR];
    f32x4 sr[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      pr[i] = words_at(rq0 + i, m0 + r4);
      sr[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    const int last_part = nparts - 1;
    int ptr = wave;                                  // next partial sum of the rows
    for (int gi = 0, gr = wave & (groups_w - 1); gi == 0 || gr < groups; ++gi, gr += 8) {
      const uint32_t pq = words_at(2 * (1 - side), qbase + gr * 256 + 4 * lane);
      f32x4 sq = zero;
      // the next N partial sums of the q's, and the rows' that come up meanwhile (a slices-th as many)
      auto sweep = [&](auto count, int pt) {
        constexpr int N = decltype(count)::value;
        f32x4 vq[N], vr[NR][N];
#pragma unroll
        for (int e = 0; e < N; ++e) {
          vq[e] = zero;
#pragma unroll
          for (int i = 0; i < NR; ++i) vr[i][e] = zero;
          if (pt + e * slices <= last_part) vq[e] = words(pt + e * slices, pq);
          if ((e << 3) < (N << (3 - lg)) && ptr + 8 * e <= last_part) {
#pragma unroll
            for (int i = 0; i < NR; ++i)
              if (i == 0 || finisher) vr[i][e] = words(ptr + 8 * e, pr[i]);
          }
        }
        FC_PIN();
#pragma unroll
        for (int e = 0; e < N; ++e) {
          sq += vq[e];
#pragma unroll
          for (int i = 0; i < NR; ++i) sr[i] += vr[i][e];
        }
        ptr += ((N << (3 - lg)) + 7) & ~7;
      };
      for (int pt = wave >> lg; pt <= last_part;) {
        const int left = ((last_part - pt) >> (3 - lg)) + 1;     // slices: a power of two
        if (left > 8) { sweep(std::integral_constant<int, 16>{}, pt); pt += 16 * slices; }
        else if (left > 2) { sweep(std::integral_constant<int, 8>{}, pt); pt += 8 * slices; }
        else { sweep(std::integral_constant<int, 2>{}, pt); pt += 2 * slices; }
      }
      if (gr < groups) *(f32x4*)(psum(wave) + 4 * kM + gi * 256 + 4 * lane) = sq;
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) *(f32x4*)(psum(wave) + (rq0 + i) * kM + r4) = sr[i];
    if (finisher && fw >= 0) {
      const StateArgs& la = late_argument<kStateAt>(a);
      if (la.version == FASTCLIP_V2 && la.tau_upd.optimizer) {      // the temperature's moments, by now addressable
        fm = (fside ? la.m_txt : la.m_img)[fn * la.stride];
        if (keeps_second_moment(la.tau_upd)) fv = (fside ? la.v_txt : la.v_img)[fn * la.stride];
      }
    }
    request_more();
    __syncthreads();
    FC_FENCE();
    auto add8 = [](const float (&w)[8]) { return ((w[0] + w[1]) + (w[2] + w[3])) + ((w[4] + w[5]) + (w[6] + w[7])); };
    auto row_total = [&](int quantity, int al) {
      float w[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) w[i] = psum(i)[quantity * kM + al];
      return add8(w);
    };
    if (finisher && fw >= 0) {
      // nobody in this launch waits for its results but the wave that adds the terms up at the very end
      const StateArgs& la = late_argument<kStateAt>(a);
      if (finishing)
        state_finish_side<false>(la, fside, m0 + frow, fn * la.stride, row_total(2 * fside, frow), row_total(2 * fside + 1, frow),
                                 fu, ft, fm, fv, &lterm, &hterm);
    }
    float u;
    if (tid < 2 * kM) {
      float c = 0.f, ce = 0.f;
      if (rows_here) {
        const float s = row_total(2 * rside, row);
        c = anchor_coefficient(a, s, ur, tr, &u);
        ce = __fmul_rn(c, s);
      }
      if (rside == side) crow[row] = c;
      drow[rside][row] = ce;
    }
#pragma unroll
    for (int i = 0; i < kMaxQ; ++i) {
      const int j = j0 + 512 * i;
      if (jw + 512 * i >= nq16) break;               // wave-uniform
      float c = 0.f;
      if (j < nq) {
        const int gr = j >> 8, at = 4 * kM + (gr >> 3) * 256 + (j & 255);
        float w[8];                                  // all eight reads at once, also where there are fewer slices
#pragma unroll
        for (int sl = 0; sl < 8; ++sl) {
          w[sl] = psum((gr & (groups_w - 1)) + ((sl < slices ? sl : 0) << lg))[at];
          w[sl] = sl < slices ? w[sl] : 0.f;
        }
        c = anchor_coefficient(a, add8(w), uq[i], tq[i], &u);
      }
      if (j < nq16) cq[j] = c;
    }
    __syncthreads();
    FC_FENCE();
    if (finisher && fw >= 0) {
      // both sums over the wave in one run: the lower half of the lanes carries the loss terms, the upper half the h terms
      double v = (lane < 32 ? lterm : hterm) + __shfl_xor(lane < 32 ? hterm : lterm, 32);
#pragma unroll
      for (int o = 16; o > 0; o >>= 1) v += __shfl_xor(v, o);
      if (lr == 0) store_agent(const_cast<double*>(late_argument<0>(g).red) + 2 * (tm * kFin + fw) + hk, v);
    }
  } else {
    request_more();
    for (int i = tid; i < kM + nq16; i += 512) {
      if (i < kM) {
        crow[i] = m0 + i < g.b ? (side == 0 ? a.c1 : a.c2)[m0 + i] : 0.f;
        drow[0][i] = m0 + i < g.b ? a.dcoef[m0 + i] : 0.f;
        drow[1][i] = 0.f;
      } else {
        const int q = qbase + i - kM;
        cq[i - kM] = q < g.b ? (side == 0 ? a.c2 : a.c1)[q] : 0.f;
      }
    }
    __syncthreads();
    FC_FENCE();
  }

  // ---- main loop
  f32x16 acc[RB][CB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  // lane offsets of the operand reads inside a slot: transposing reads take 4 rows x 16 columns per group of 16 lanes, source
  // lane s row s / 4, columns 4 (s % 4) ..; the halves h = 0, 1 of a read are 8 rows apart
  const int s16 = lane & 15, c16 = (lane >> 4) & 1;
  uint32_t rx[2], rq[NA][2];                          // of column block t / row block t; RB = 1: of 16-deep step t
  constexpr uint32_t kXHalf = RB == 1 ? 512u : 1024u;
  const int k0 = 4 * hk + (s16 >> 2);                 // 8 rows further on: the same swizzles
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int nl = t * 32 + c16 * 16 + 4 * (s16 & 3);
    rx[t] = RB == 1 ? (uint32_t)(kX + (16 * t + k0) * 64 + (nl & 31) * 2)
                    : (uint32_t)(kX + k0 * 128 + (((nl >> 3) ^ (((k0 >> 1) & 1) << 2)) << 4) + ((nl & 7) << 1));
  }
#pragma unroll
  for (int t = 0; t < NA; ++t) {
    const int cb = RB == 1 ? c16 : 2 * t + c16, r4 = s16 & 3, hh = r4 & 1;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      rq[t][h] = (uint32_t)((cb * 2 + hh) * (16 * kD16) +
                            (((RB == 1 ? 16 * t : 0) + 8 * h + k0) ^ (4 * hh) ^ (8 * (cb & 1))) * 16 + (r4 >> 1) * 8);
  }
  auto tr = [](uint32_t addr) {
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(uintptr_t)addr));
  };
  float inv_c[RB];                                    // GATHERED: 1 / c_own of the operand's rows (lanes run over rows)
  if constexpr (GATHERED) {
#pragma unroll
    for (int t = 0; t < RB; ++t) {
      const float c = crow[t * 32 + lr];
      inv_c[t] = m0 + t * 32 + lr < g.b ? 1.0f / c : 0.f;
    }
  }
  uint32_t slot = wring;
  // Stages [i0, i1): read stage i, request the next into the slot that stage i - 1 was read from, multiply.  The requests
  // hide the reads' latency, and the products run on into the next stage's wait.
  auto run = [&](auto other_side, int i0, int i1) {
    constexpr bool OTHER = decltype(other_side)::value;
    const float* c = cq + (Q0 * kD16 - qbase) + 4 * hk;    // c_other[q], two runs of four q per lane and 16-deep step
    for (int i = i0; i < i1; ++i) {
      // stage i has landed: at most the younger ones, NA + 2 loads each (with a second strip two more), may be in flight
      if (kSlotsW == 4 && at - i == 3) __builtin_amdgcn_s_waitcnt(0x0f78);
      else if (at - i == 2 && GATHERED && i + 1 < nAw) __builtin_amdgcn_s_waitcnt(0x0f76);
      else if (at - i == 2) __builtin_amdgcn_s_waitcnt(NA == 2 ? 0x0f74 : 0x0f76);
      else __builtin_amdgcn_s_waitcnt(0x0f70);
      __builtin_amdgcn_wave_barrier();
      FC_FENCE();
      u32x4 w[NA];
      u32x4 wf[GATHERED && !OTHER ? NA : 1];
      u32x2 xl[2], xh[2];
#pragma unroll
      for (int t = 0; t < NA; ++t) {
        if constexpr (!OTHER) {
          w[t] = *(const u32x4*)(wslot + (slot - wring) + t * 1024 + lane * 16);
          if constexpr (GATHERED) wf[t] = *(const u32x4*)(wslot + (slot - wring) + kF + t * 1024 + lane * 16);
        } else {
          const u32x2 lo = tr(slot + rq[t][0]), hi = tr(slot + rq[t][1]);
          w[t] = (u32x4){lo[0], lo[1], hi[0], hi[1]};
        }
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        xl[t] = tr(slot + rx[t]);
        xh[t] = tr(slot + rx[t] + kXHalf);
      }
      f32x4 cl[KS], ch[KS];
      if constexpr (OTHER) {
#pragma unroll
        for (int k = 0; k < KS; ++k) { cl[k] = *(const f32x4*)(c + 16 * k); ch[k] = *(const f32x4*)(c + 16 * k + 8); }
        c += kD16;
      }
      slot = slot + kStageB == wring + kSlotsW * kStageB ? wring : slot + kStageB;
      FC_PIN();
      if (at < nst) request();
      wave_reads_done();                          // the stage's slot may be filled again
      if constexpr (GATHERED && !OTHER) {
#pragma unroll
        for (int t = 0; t < NA; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            w[t][e] = pack_bf16x2(fmaf(__uint_as_float(wf[t][e] << 16), inv_c[t], __uint_as_float(w[t][e] << 16)),
                                  fmaf(__uint_as_float(wf[t][e] & 0xffff0000u), inv_c[t], __uint_as_float(w[t][e] & 0xffff0000u)));
      }
      if constexpr (OTHER) {
#pragma unroll
        for (int t = 0; t < NA; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int k = RB == 1 ? t : 0;
            const float c0 = e < 2 ? cl[k][2 * e] : ch[k][2 * e - 4], c1 = e < 2 ? cl[k][2 * e + 1] : ch[k][2 * e - 3];
            w[t][e] = pack_bf16x2(__uint_as_float(w[t][e] << 16) * c0, __uint_as_float(w[t][e] & 0xffff0000u) * c1);
          }
      }
#pragma unroll
      for (int t = 0; t < 2 * RB; ++t) {
        const int wt = RB == 1 ? t : t >> 1, ti = RB == 1 ? 0 : t >> 1, tj = RB == 1 ? 0 : t & 1;
        acc[ti][tj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w[wt]),
                                                              join_halves(xl[t & 1], xh[t & 1]), acc[ti][tj], 0, 0, 0);
      }
    }
  };
  run(std::false_type{}, 0, nAw);
#pragma unroll
  for (int ti = 0; ti < RB; ++ti)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x4 c = *(const f32x4*)(crow + ti * 32 + 8 * q + 4 * hk);
#pragma unroll
      for (int tj = 0; tj < CB; ++tj)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[ti][tj][4 * q + v] *= c[v];
    }
  run(std::true_type{}, nAw, nst);

  const T128Args& lg = late_argument<0>(g);
  // The finishing waves count themselves once their stores are acknowledged at agent scope (they are long since); the answer is
  // looked at behind the outputs.
  unsigned scalars_before = 0;
  if (finisher && fw >= 0) {
    __builtin_amdgcn_s_waitcnt(0x0f70);
    FC_FENCE();
    if (lane == 0)
      scalars_before = __hip_atomic_fetch_add(lg.scalars_arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  float* out = const_cast<float*>(wave_uniform(side ? lg.job[1].out : lg.job[0].out));
  if constexpr (RB == 1) {
    // 32 x 32: a thread finishes two rows of a column, values 2 (lane & 1) .. of word `wave / 2` of lane 32 (wave & 1) + lane / 2
    const int row0 = 8 * (wave >> 1) + 4 * (wave & 1) + 2 * (lane & 1), n = n0 + (lane >> 1);
    bf16_t xd[2];
    float dc[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int m = m0 + row0 + e < lg.b ? m0 + row0 + e : lg.b - 1;
      xd[e] = X[(uint32_t)((lg.off + m) * ldx + (n < d ? n : 0))];
      dc[e] = drow[0][row0 + e] + drow[1][row0 + e];
    }
    __syncthreads();
    FC_FENCE();
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *(f32x4*)((float*)(ring + wave * 4096) + q * 256 + lane * 4) =
          (f32x4){acc[0][0][4 * q], acc[0][0][4 * q + 1], acc[0][0][4 * q + 2], acc[0][0][4 * q + 3]};
    __syncthreads();
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const float* p = (const float*)ring + (wave >> 1) * 256 + ((wave & 1) * 32 + (lane >> 1)) * 4 + 2 * (lane & 1);
    f32x2 w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = *(const f32x2*)(p + i * 1024);
    const f32x2 sum = ((w[0] + w[1]) + (w[2] + w[3])) + ((w[4] + w[5]) + (w[6] + w[7]));
    float* o = out + (uint32_t)((m0 + row0) * d + n);
#pragma unroll
    for (int e = 0; e < 2; ++e)
      if (n < d && m0 + row0 + e < lg.b) o[e * d] = sum[e] - dc[e] * bf2f(xd[e]);
  } else {
    // ---- the eight waves' tiles are added up; larger tiles 64 rows at a time: wave w finishes block w / 2 of them, its rows 16 (w % 2) .. + 15
    const int rl = (wave >> 2) * 32 + (wave & 1) * 16 + 4 * hk;          // row of e = 0; e = 4: 8 further on
    const int n = n0 + ((wave >> 1) & 1) * 32 + lr;
    const bool whole = m0 + kM <= lg.b && n0 + kO <= d;
#pragma unroll
    for (int mb = 0; mb < RB / 2; ++mb) {
      const int row0 = mb * 64 + rl;
      bf16_t xd[8];                              // the diagonal terms' rows, requested ahead of the sums
      f32x4 dc[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) dc[h] = *(const f32x4*)(drow[0] + row0 + 8 * h) + *(const f32x4*)(drow[1] + row0 + 8 * h);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        int m = m0 + row0 + 8 * (e >> 2) + (e & 3);
        m = m < lg.b ? m : lg.b - 1;
        xd[e] = X[(uint32_t)((lg.off + m) * ldx + (n < d ? n : 0))];
      }
      __syncthreads();
      FC_FENCE();
      {
        float* o = (float*)(ring + wave * 16384) + lane * 4;
#pragma unroll
        for (int ti = 0; ti < 2; ++ti)
#pragma unroll
          for (int tj = 0; tj < 2; ++tj)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const f32x16& v = acc[mb * 2 + ti][tj];
              *(f32x4*)(o + ((ti * 2 + tj) * 4 + q) * 256) = (f32x4){v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
            }
      }
      __syncthreads();
      f32x4 sum[2];
      {
        const float* p = (const float*)ring + wave * 512 + lane * 4;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          sum[h] = *(const f32x4*)(p + h * 256);
#pragma unroll
          for (int w = 1; w < 8; ++w) sum[h] += *(const f32x4*)(p + w * 4096 + h * 256);
        }
      }
      bool writer = true;
      if (lg.nsplit > 1) {
        const size_t slab = (size_t)lg.nsplit * (kO * kO / 2);
        double* all = lg.part + (size_t)(tile * (RB / 2) + mb) * slab + wave * 256 + lane;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const u32x2 w = {__float_as_uint(sum[p >> 1][2 * (p & 1)]), __float_as_uint(sum[p >> 1][2 * (p & 1) + 1])};
          store_agent(all + (size_t)split * (kO * kO / 2) + p * 64, __builtin_bit_cast(double, w));
        }
        writer = last_to_arrive(lg.arrived + tile * (RB / 2) + mb, (unsigned)lg.nsplit, flag);
        if (writer) {
          sum[0] = sum[1] = (f32x4){0.f, 0.f, 0.f, 0.f};
          for (int s0 = 0; s0 < lg.nsplit; s0 += 4) {      // the partial results of four splits in flight at once
            double w[4][4];
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
              for (int p = 0; p < 4; ++p)
                w[s][p] = load_agent(all + (size_t)(s0 + s < lg.nsplit ? s0 + s : s0) * (kO * kO / 2) + p * 64);
            FC_PIN();
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
              for (int p = 0; p < 4; ++p) {
                const u32x2 v = __builtin_bit_cast(u32x2, w[s][p]);
                sum[p >> 1][2 * (p & 1)] += s0 + s < lg.nsplit ? __uint_as_float(v[0]) : 0.f;
                sum[p >> 1][2 * (p & 1) + 1] += s0 + s < lg.nsplit ? __uint_as_float(v[1]) : 0.f;
              }
          }
        }
      }
      if (writer) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = sum[e >> 2][e & 3] - dc[e >> 2][e & 3] * bf2f(xd[e]);
        float* o = out + (uint32_t)((m0 + row0) * d + n);
        if (whole) {
#pragma unroll
          for (int e = 0; e < 8; ++e) o[(8 * (e >> 2) + (e & 3)) * d] = v[e];
        } else {
          const int rows = n < d ? lg.b - m0 - row0 : 0;
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (8 * (e >> 2) + (e & 3) < rows) o[(8 * (e >> 2) + (e & 3)) * d] = v[e];
        }
      }
    }
  }
  // scalars, by the wave that finished the last anchors
  if (fused) return finisher && fw >= 0 && (unsigned)__shfl((int)scalars_before, 0) + 1u == (unsigned)(kFin * lg.tiles_m);
  return side == 0 && tn == 0 && tm == 0 && split == 0 && wave == 7;
}

template <int RB, bool GATHERED>
__global__ void __launch_bounds__(512, 2) k_contract_t128_bf16(T128Args g, StateArgs a) {
  __shared__ __attribute__((aligned(1024))) char ring[kWRing<RB, GATHERED>];
  __shared__ __attribute__((aligned(16))) float crow[32 * RB], drow[2][32 * RB], cq[kMaxLocalQ];
  __shared__ int flag;
  warm_arguments<sizeof(T128Args) + sizeof(StateArgs)>();
  // (one place that calls write_scalars: see there)
  const bool last = (int)blockIdx.x < g.finishers ? t128_finish(late_argument<0>(g), late_argument<kStateAt>(a), &flag)
                                                  : t128_tile<RB, GATHERED>(g, a, ring, crow, drow, cq, &flag);
  const T128Args& lg = late_argument<0>(g);
  if (last) write_scalars<true>(lg.red, lg.nterms, lg.b, lg.version, lg.tau, lg.rho, lg.loss, lg.d_tau);
}

void launch_contract_t128_bf16(const StepCtx& c) {
  const Layout& L = c.L;
  T128Args g;
  memset(&g, 0, sizeof(g));
  for (int s = 0; s < 2; ++s) {
    T128Job& J = g.job[s];
    J.E = (const bf16_t*)(c.ws + L.E[s]);
    J.Eo = (const bf16_t*)(c.ws + L.E[1 - s]);
    J.F = L.gathered ? (const bf16_t*)(c.ws + L.F[s]) : nullptr;
    J.X = (const bf16_t*)(s == 0 ? c.buf.txt_glob : c.buf.img_glob);
    J.ldx = s == 0 ? c.cfg.ld_txt : c.cfg.ld_img;
    J.out = s == 0 ? c.buf.d_img : c.buf.d_txt;
  }
  g.b = (int)L.b; g.d = (int)L.d; g.B = (int)L.B; g.off = (int)L.off; g.nCB = L.ldE / 16;
  const int64_t out_cols = L.out_rows == 32 ? 32 : 64, depth = L.out_rows == 32 ? 32 : 16;      // columns of a tile; a stage
  g.tiles_m = (int)((L.b + L.out_rows - 1) / L.out_rows); g.tiles_n = (int)((L.d + out_cols - 1) / out_cols);
  g.nsplit = L.nsplit;
  g.inv_tiles = reciprocal(2 * g.tiles_m * g.tiles_n);
  g.inv_tiles_n = reciprocal(g.tiles_n);
  g.nA = (int)((L.B + depth - 1) / depth); g.nB = (int)((L.b + depth - 1) / depth);
  g.sliceA = (g.nA + L.nsplit * 8 - 1) / (L.nsplit * 8);
  g.sliceB = (g.nB + L.nsplit * 8 - 1) / (L.nsplit * 8);
  g.part = L.nsplit > 1 ? (double*)(c.ws + L.Opart[0]) : nullptr;
  g.arrived = (unsigned*)(c.ws + L.arrived);
  g.scalars_arrived = g.arrived + L.narrived - 1;
  g.tau = c.buf.tau; g.rho = c.cfg.rho; g.loss = c.buf.loss; g.d_tau = c.buf.d_tau;
  g.red = (const double*)(c.ws + L.red); g.version = c.cfg.version;
  auto* kernel = L.gathered ? k_contract_t128_bf16<2, true>
                 : L.out_rows == 32 ? k_contract_t128_bf16<1, false>
                                    : (L.out_rows == 64 ? k_contract_t128_bf16<2, false> : k_contract_t128_bf16<4, false>);
  const unsigned groups = (2u * (unsigned)(g.nsplit * g.tiles_m * g.tiles_n) + 7) / 8 * 8;
  // the state phase has workgroups of its own where compute units are left for them
  const unsigned finishers = (unsigned)((L.b + 255) / 256);
  g.finishers = L.fused_state && groups + finishers <= 256 ? (int)finishers : 0;
  g.nterms = !L.fused_state ? L.nstate_blocks : (g.finishers ? 8 * g.finishers : t128_finishing_waves(L.out_rows) * g.tiles_m);
  hipLaunchKernelGGL(kernel, dim3(groups + (unsigned)g.finishers), dim3(512), 0, c.s, g, make_state_args(c));
}

}  // namespace fc
