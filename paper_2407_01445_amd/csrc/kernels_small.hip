// Small kernels of the FCCO step: s_ii and temperature gather, the state update of Eq. 1 with
// the per-anchor coefficients, the finishing kernels of the MFMA path, the scalar outputs, and the index checker.
#include <string.h>

#include <type_traits>

#include "fc_internal.hpp"
#include "mfma_common.hpp"
#include "state_common.hpp"

namespace fc {

constexpr float kLog2e = 1.4426950408889634f;

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}
__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

__device__ inline float load_elem(const float* p) { return *p; }
__device__ inline float load_elem(const bf16_t* p) { return __uint_as_float((uint32_t)(*p) << 16); }

// ------------------------------------------------------------------------------------------
// prep: one wavefront per local anchor r.  s_pp = <img_p, txt_p> (the s_ii of Sec. 3), the
// temperatures that enter l1 / l2 of this anchor (Proc. 1: global tau, or tau_1[idx], tau_2[idx]),
// and k = log2(e) / tau for the exp2-based evaluation in the MFMA path.
__device__ inline double row_dot(const float* pi, const float* pt, int64_t d, int lane) {
  double acc = 0.0;
  for (int64_t k = lane; k < d; k += 64) acc += (double)pi[k] * (double)pt[k];
  return acc;
}
// bf16 rows: d and the row strides are multiples of 8 and the bases 16-byte aligned, so 8 elements per load
__device__ inline double row_dot(const bf16_t* pi, const bf16_t* pt, int64_t d, int lane) {
  double acc = 0.0;
  for (int64_t k = (int64_t)lane * 8; k < d; k += 512) {
    const uint4 a = *(const uint4*)(pi + k), b = *(const uint4*)(pt + k);
    const uint32_t aw[4] = {a.x, a.y, a.z, a.w}, bw[4] = {b.x, b.y, b.z, b.w};
    float part = 0.f;   // 8 exact bf16 x bf16 products
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      part = fmaf(__uint_as_float(aw[w] << 16), __uint_as_float(bw[w] << 16), part);
      part = fmaf(__uint_as_float(aw[w] & 0xffff0000u), __uint_as_float(bw[w] & 0xffff0000u), part);
    }
    acc += (double)part;
  }
  return acc;
}

// Gathered state (Alg. 1 line 8; Eqs. 3 / 5 / 7 over every global anchor; GATHERED): one wavefront per global row j, the local
// rows as above.  Remote anchor j contributes c_j l2(j, p) txt_j to the image gradient of a local row p and c_j l1(j, p) img_j
// to its text gradient, with l2(j, p) = exp((s_pj - s_jj) / tau2_j), l1(j, p) = exp((s_jp - s_jj) / tau1_j) and
// c_j = kappa_j / (|B_k| |B_j-| (eps + u_j^{t+1})): the strips already form s_pj and s_jp, so all they need per column j is
// log2(e)/tau_j, s_jj log2(e)/tau_j and c_j.  Local rows get c = 0: their u^{t+1} is only known after the state phase, and their
// share is the local contrast-side term of what follows it (the fold, or further depth of the contraction on the small
// tiles and on the fp32 path).  So do the padding columns beyond B.
// What bounds it: the launch and two dependent gathers for a small batch, reading both matrices (5.7 TB/s) for a large one.
// Local and remote rows are one launch, in which either's latency hides behind the other's; as two launches 640 of 5120 at
// width 512 took 4.7 + 4.0 us, 1024 of 32768 at 1024 4.8 + 23.7.
// Arguments: what only gathered state needs is in a struct of its own behind the rest, so that the plain kernel's are three lines,
// which come at once.  fp32, 64 pairs at width 32: 3.22 us with all fields in one struct, 3.14 so without the early touch of the
// three lines, 3.01 with it.
template <typename T>
struct PrepArgs {
  const T *img, *txt;
  int64_t ld_img, ld_txt, off, b, d;
  const int64_t* idx;
  const float *tau, *tau_img, *tau_txt, *u_img, *u_txt;
  int64_t stride;
  int version, narrived, threads;        // threads of the launch
  float *diag, *tau1, *tau2, *k1, *k2, *uold1, *uold2;
  unsigned* arrived;
};
template <typename T>
struct PrepGatheredArgs : PrepArgs<T> {
  int64_t B;
  const float *tau_glob_img, *tau_glob_txt, *u_glob_img, *u_glob_txt;
  float eps, bm;
  int64_t ncol;
  float* colp;
  int from_own;
};
static_assert(sizeof(PrepArgs<float>) <= 192, "three lines");

template <typename T, typename Args>
__global__ void __launch_bounds__(256) k_prep(Args a) {
  constexpr bool GATHERED = std::is_same<Args, PrepGatheredArgs<T>>::value;
  warm_arguments<sizeof(Args)>();
  const int lane = threadIdx.x & 63;
  const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  for (int i = (int)(blockIdx.x * 256 + threadIdx.x); i < a.narrived; i += a.threads) a.arrived[i] = 0u;
  int64_t rows = a.b, j = a.off + w;                              // global row
  if constexpr (GATHERED) { rows = a.ncol; j = w; }
  if (w >= rows) return;
  const int64_t r = j - a.off;                                    // local anchor
  const bool local = !GATHERED || (r >= 0 && r < a.b);            // wave-uniform
  bool exists = true;
  if constexpr (GATHERED) exists = j < a.B;
  float t1 = 0.f, t2 = 0.f, u1 = 0.f, u2 = 0.f;
  if (lane == 0 && exists) {
    // issue the gathers before the dot product so that the latencies overlap: by dataset index the temperatures, and u^t of
    // Eq. 1 for the state phase (nothing writes u before that phase); of a remote anchor what its worker has sent
    const float *u_img = a.u_img, *u_txt = a.u_txt, *tau_img = a.tau_img, *tau_txt = a.tau_txt;
    if constexpr (GATHERED) {
      if (!local) { u_img = a.u_glob_img; u_txt = a.u_glob_txt; tau_img = a.tau_glob_img; tau_txt = a.tau_glob_txt; }
    }
    const int64_t at = local ? a.idx[r] : 0;
    if (a.version != FASTCLIP_V2) t1 = t2 = a.tau[0];       // on its way together with the index
    const int64_t n = local ? at * a.stride : j;
    u1 = u_img[n];
    u2 = u_txt[n];
    if (a.version == FASTCLIP_V2) {
      t1 = tau_img[n];
      t2 = tau_txt[n];
    }
  }
  double s_jj = 0.0;
  if (exists) s_jj = wave_sum(row_dot(a.img + j * a.ld_img, a.txt + j * a.ld_txt, a.d, lane));
  if (lane != 0) return;
  float k1 = 0.f, k2 = 0.f;
  if (exists) { k1 = kLog2e / t1; k2 = kLog2e / t2; }
  if (local) {
    a.diag[r] = (float)s_jj;
    a.tau1[r] = t1;
    a.tau2[r] = t2;
    a.k1[r] = k1;
    a.k2[r] = k2;
    a.uold1[r] = u1;
    a.uold2[r] = u2;
  }
  if constexpr (GATHERED) {
    float c1 = 0.f, c2 = 0.f;
    if (local) k1 = k2 = 0.f;
    else if (exists) {
      c1 = 1.0f / (a.bm * (a.eps + u1));
      c2 = 1.0f / (a.bm * (a.eps + u2));
      if (a.version == FASTCLIP_V0) { c1 /= t1; c2 /= t2; }
    }
    // column of row j: its number, or (from_own) counted from the worker's own rows on
    const int64_t col = !a.from_own || !exists ? j : (j >= a.off ? j - a.off : j - a.off + a.B);
    const int64_t ntile = a.ncol >> 8, tile = col >> 8, in = col & 255;
    float* p0 = a.colp + ((0 * ntile + tile) * 4) * 256 + in;   // side 0: text anchors (tau_2, u_2)
    float* p1 = a.colp + ((1 * ntile + tile) * 4) * 256 + in;   // side 1: image anchors (tau_1, u_1)
    p0[0] = k2; p0[256] = (float)(s_jj * (double)k2); p0[512] = c2; p0[768] = 0.f;
    p1[0] = k1; p1[256] = (float)(s_jj * (double)k1); p1[512] = c1; p1[768] = 0.f;
  }
}

template <typename T, typename Args>
static void launch_prep_rows(const StepCtx& c, Args& a, int64_t rows) {
  const Layout& L = c.L;
  a.img = (const T*)c.buf.img_glob; a.txt = (const T*)c.buf.txt_glob;
  a.ld_img = c.cfg.ld_img; a.ld_txt = c.cfg.ld_txt; a.off = L.off; a.b = L.b; a.d = L.d;
  a.idx = c.buf.idx; a.tau = c.buf.tau; a.tau_img = c.buf.tau_img; a.tau_txt = c.buf.tau_txt;
  a.u_img = c.buf.u_img; a.u_txt = c.buf.u_txt; a.stride = c.cfg.state_stride; a.version = c.cfg.version;
  a.diag = (float*)(c.ws + L.diag);
  a.tau1 = (float*)(c.ws + L.tau1); a.tau2 = (float*)(c.ws + L.tau2);
  a.k1 = (float*)(c.ws + L.k1); a.k2 = (float*)(c.ws + L.k2);
  a.uold1 = (float*)(c.ws + L.uold1); a.uold2 = (float*)(c.ws + L.uold2);
  a.arrived = (unsigned*)(c.ws + L.arrived); a.narrived = L.narrived;
  const dim3 grid((unsigned)((rows + 3) / 4)), block(256);
  a.threads = (int)(grid.x * 256);
  hipLaunchKernelGGL((k_prep<T, Args>), grid, block, 0, c.s, a);
}

template <typename T>
static void launch_prep_of(const StepCtx& c) {
  const Layout& L = c.L;
  if (!L.gathered) {
    PrepArgs<T> a;
    launch_prep_rows<T>(c, a, L.b);
    return;
  }
  PrepGatheredArgs<T> a;
  a.B = L.B;
  a.tau_glob_img = c.buf.tau_glob_img; a.tau_glob_txt = c.buf.tau_glob_txt;
  a.u_glob_img = c.buf.u_glob_img; a.u_glob_txt = c.buf.u_glob_txt;
  a.eps = c.cfg.eps; a.bm = (float)L.b * (float)(L.B - 1);
  a.from_own = L.t128; a.ncol = L.ncol;
  a.colp = (float*)(c.ws + L.colp);
  launch_prep_rows<T>(c, a, L.ncol);
}

void launch_prep(const StepCtx& c) {
  if (c.L.bf16) launch_prep_of<bf16_t>(c);
  else launch_prep_of<float>(c);
}

// ------------------------------------------------------------------------------------------
// Cosine similarity at the boundary (Sec. 3): one wavefront per raw encoder row e: |e| with the squares summed in fp64,
// then e / |e| rounded once to the storage type of the step.  A row of zeros gives a row of zeros and norm 0.
__device__ inline void store_elem(float* p, float x) { *p = x; }
__device__ inline void store_elem(bf16_t* p, float x) { *p = __builtin_bit_cast(uint16_t, (__bf16)x); }

template <typename TI, typename TO>
__global__ void __launch_bounds__(256) k_normalize_rows(const TI* __restrict__ raw, int64_t ld_raw, int64_t b, int64_t d,
                                                        TO* __restrict__ unit, int64_t ld_unit, float* __restrict__ norm) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= b) return;
  const TI* src = raw + r * ld_raw;
  double acc = 0.0;
  for (int64_t k = lane; k < d; k += 64) {
    const double x = (double)load_elem(src + k);
    acc += x * x;
  }
  const double n = sqrt(wave_sum(acc));
  const float inv = n > 0.0 ? (float)(1.0 / n) : 0.f;
  TO* dst = unit + r * ld_unit;
  for (int64_t k = lane; k < d; k += 64) store_elem(dst + k, load_elem(src + k) * inv);
  if (lane == 0) norm[r] = (float)n;
}

// The same where rows are whole groups of four elements, aligned (16 bytes of fp32, 8 of bf16): a lane holds its up to kNormQuads
// groups of the row between the two passes, all of them in flight at once.  What bounds it is the chain load - sum over the
// wave - square root - store: element by element it was one memory latency per 64 elements and pass (256 rows of width
// 512: 5.9 -> 3.2 us a launch).
constexpr int kNormQuads = 4;
__device__ inline float4 load_quad(const float* p) { return *(const float4*)p; }
__device__ inline float4 load_quad(const bf16_t* p) {
  const uint2 w = *(const uint2*)p;
  return make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16),
                     __uint_as_float(w.y & 0xffff0000u));
}
__device__ inline void store_quad(float* p, float4 v) { *(float4*)p = v; }
__device__ inline void store_quad(bf16_t* p, float4 v) {
  uint2 w;
  w.x = (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)v.x) | ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)v.y) << 16);
  w.y = (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)v.z) | ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)v.w) << 16);
  *(uint2*)p = w;
}

template <typename TI, typename TO>
__global__ void __launch_bounds__(256) k_normalize_rows_quads(const TI* __restrict__ raw, int64_t ld_raw, int64_t b, int d,
                                                              TO* __restrict__ unit, int64_t ld_unit, float* __restrict__ norm) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= b) return;
  const TI* src = raw + r * ld_raw;
  float4 v[kNormQuads];
#pragma unroll
  for (int i = 0; i < kNormQuads; ++i) {
    const int k = 4 * (lane + 64 * i);
    v[i] = k < d ? load_quad(src + k) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  double acc = 0.0;
#pragma unroll
  for (int i = 0; i < kNormQuads; ++i) {
    const double x = v[i].x, y = v[i].y, z = v[i].z, w = v[i].w;
    acc += (x * x + y * y) + (z * z + w * w);
  }
  const double n = sqrt(wave_sum(acc));
  const float inv = n > 0.0 ? (float)(1.0 / n) : 0.f;
  TO* dst = unit + r * ld_unit;
#pragma unroll
  for (int i = 0; i < kNormQuads; ++i) {
    const int k = 4 * (lane + 64 * i);
    if (k < d) store_quad(dst + k, make_float4(v[i].x * inv, v[i].y * inv, v[i].z * inv, v[i].w * inv));
  }
  if (lane == 0) norm[r] = (float)n;
}

template <typename TI, typename TO>
static void normalize_rows(const void* raw, int64_t ld_raw, int64_t b, int64_t d, void* unit, int64_t ld_unit, float* norm,
                           hipStream_t s) {
  const dim3 grid((unsigned)((b + 3) / 4)), block(256);
  const bool quads = d % 4 == 0 && d <= 256 * kNormQuads && ld_raw % 4 == 0 && ld_unit % 4 == 0 &&
                     (uintptr_t)raw % (4 * sizeof(TI)) == 0 && (uintptr_t)unit % (4 * sizeof(TO)) == 0;
  if (quads)
    hipLaunchKernelGGL((k_normalize_rows_quads<TI, TO>), grid, block, 0, s, (const TI*)raw, ld_raw, b, (int)d, (TO*)unit, ld_unit,
                       norm);
  else
    hipLaunchKernelGGL((k_normalize_rows<TI, TO>), grid, block, 0, s, (const TI*)raw, ld_raw, b, d, (TO*)unit, ld_unit, norm);
}

void launch_normalize_rows(const void* raw, int raw_bf16, int64_t ld_raw, int64_t b, int64_t d, void* unit, int unit_bf16,
                           int64_t ld_unit, float* norm, hipStream_t s) {
  if (raw_bf16 && unit_bf16) normalize_rows<bf16_t, bf16_t>(raw, ld_raw, b, d, unit, ld_unit, norm, s);
  else if (raw_bf16) normalize_rows<bf16_t, float>(raw, ld_raw, b, d, unit, ld_unit, norm, s);
  else if (unit_bf16) normalize_rows<float, bf16_t>(raw, ld_raw, b, d, unit, ld_unit, norm, s);
  else normalize_rows<float, float>(raw, ld_raw, b, d, unit, ld_unit, norm, s);
}

// ------------------------------------------------------------------------------------------
// Global temperature (V0, V3): one thread.
__global__ void k_tau_scalar(TauUpd u, float* tau, float* m, float* v, const float* d_tau) {
  if (threadIdx.x == 0 && blockIdx.x == 0) tau_step(u, tau, m, v, d_tau[0]);
}

// Individual temperatures (V2): one thread per side (blockIdx.y) of a local anchor; gathers and scatters by dataset index.  What
// bounds it for a batch is the chain index - gathers - scatters; both sides by one thread are two of them (256 anchors: 3.7 us
// a launch, 2.9 by a thread per side).  So they are (one row
// of workgroups, sides == 1) where the sides share an array: the text's step goes on from what the image's has left there.
__global__ void __launch_bounds__(256) k_tau_sparse(TauUpd u, const int64_t* __restrict__ idx, int64_t b,
                                                    const float* __restrict__ g_img, const float* __restrict__ g_txt,
                                                    float* tau_img, float* tau_txt, float* m_img, float* v_img,
                                                    float* m_txt, float* v_txt, int sides) {
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r >= b) return;
  int side = blockIdx.y;
  do {
    const float g = (side ? g_txt : g_img)[r];
    const int64_t n = idx[r] * u.stride;
    float* v = side ? v_txt : v_img;
    tau_step(u, (side ? tau_txt : tau_img) + n, (side ? m_txt : m_img) + n, v ? v + n : nullptr, g);
    side += sides;
  } while (side < 2);
}

void launch_tau_scalar(const TauUpd& u, const fastclip_tau_state& st, const float* d_tau, hipStream_t s) {
  hipLaunchKernelGGL(k_tau_scalar, dim3(1), dim3(64), 0, s, u, st.tau, st.m, st.v, d_tau);
}

void launch_tau_sparse(const TauUpd& u, const fastclip_tau_state& st, const int64_t* idx, int64_t b,
                       const float* d_tau_img, const float* d_tau_txt, hipStream_t s) {
  const float *img[3] = {st.tau_img, st.m_img, st.v_img}, *txt[3] = {st.tau_txt, st.m_txt, st.v_txt};
  int sides = 2;
  for (const float* p : img)
    for (const float* q : txt)
      if (p && p == q) sides = 1;
  hipLaunchKernelGGL(k_tau_sparse, dim3((unsigned)((b + 255) / 256), (unsigned)sides), dim3(256), 0, s, u, idx, b, d_tau_img,
                     d_tau_txt, st.tau_img, st.tau_txt, st.m_img, st.v_img, st.m_txt, st.v_txt, sides);
}

// ------------------------------------------------------------------------------------------
// State phase (Alg. 1 line 7 and the per-anchor half of lines 9 and 12): Eq. 1 at the batch's samples, the coefficients
// of Eqs. 2-7, Eq. 9, the partial sums of the loss and of Eqs. 8 / 10, and - if asked for - the temperature step of the
// same samples.  A thread owns ONE SIDE of one anchor (threads 2 r and 2 r + 1 are the image and the text side of
// anchor r), so the two words that a record layout keeps next to each other are moved by neighbouring lanes of one
// memory instruction.  256 threads = `lanes` partial-sum lanes x (256 / lanes) anchor sides; the threads of partial-sum
// lane 0 finish the anchor sides.  With canonical 8-float records a finishing thread moves its side's four fields
// {u, tau, m, v} as one 16-byte word: a sample costs one 32-byte sector each way, read and written whole.
// se / sx of partial-sum lane 0 plus those of lanes 1 .. LANES - 1, which sit 256 / LANES entries apart
template <int LANES, typename T>
__device__ __forceinline__ void add_parts(const T (*part)[256], int sa, T& se, T& sx) {
  T e[LANES], x[LANES];
#pragma unroll
  for (int q = 1; q < LANES; ++q) { e[q] = part[0][q * (256 / LANES) + sa]; x[q] = part[1][q * (256 / LANES) + sa]; }
#pragma unroll
  for (int q = 1; q < LANES; ++q) { se += e[q]; sx += x[q]; }
}

// the accuracy path adds its partial sums (fp64 unless there is only one) up in fp64
template <bool PRECISE> struct SumType { typedef float type; };
template <> struct SumType<true> { typedef double type; };

template <bool PRECISE>
__global__ void __launch_bounds__(256) k_state(StateArgs a) {
  using sum_t = typename SumType<PRECISE>::type;
  __shared__ sum_t part[2][256];
  __shared__ double scal[2][4];
  warm_arguments<sizeof(StateArgs)>();
  const int SA = 256 / a.lanes;                       // anchor sides per tile of a block
  const int sa = threadIdx.x % SA, pl = threadIdx.x / SA;
  const int side = sa & 1;
  double lterm = 0.0, hterm = 0.0;                    // this thread's terms of the two scalars, over all its tiles
  // a block takes the tiles blockIdx.x, blockIdx.x + gridDim.x, ..: the step launches one block per tile, the phase on
  // its own a bounded number of blocks (so that the scalars' partial sums stay few)
  for (int64_t tile = blockIdx.x; tile < a.ntiles; tile += gridDim.x) {
    const int64_t r = tile * (SA >> 1) + (sa >> 1);
    const bool finisher = pl == 0 && r < a.b;
    // the finishing threads' own inputs are requested first: the gather by dataset index is the longest latency here
    int64_t n = 0;
    float u_old = 0.f, tau = 0.f, m = 0.f, v = 0.f;
    if (finisher) {
      n = a.idx[r] * a.stride;
      if (a.records) {
        const float4 w = *(const float4*)(a.u_img + n + 4 * side);
        u_old = w.x; tau = w.y; m = w.z; v = w.w;
      } else if (a.gather) {
        u_old = (side ? a.u_txt : a.u_img)[n];
        tau = a.version == FASTCLIP_V2 ? (side ? a.tau_txt : a.tau_img)[n] : a.tau_glob[0];
      } else {
        u_old = (side ? a.uold2 : a.uold1)[r];
        tau = (side ? a.tau2 : a.tau1)[r];
      }
    }
    sum_t se_t = 0, sx_t = 0;
    if (r < a.b) {
      // eight partial sums of each quantity per round (sixteen loads in flight), or four
      auto add_up = [&](const auto* s0) {
        const auto* s1 = s0 + (size_t)a.nparts * a.bstride;
        int pt = pl;
        for (; pt + 7 * a.lanes < a.nparts; pt += 8 * a.lanes) {
          sum_t e[8], x[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            e[q] = s0[(size_t)(pt + q * a.lanes) * a.bstride];
            x[q] = s1[(size_t)(pt + q * a.lanes) * a.bstride];
          }
#pragma unroll
          for (int q = 0; q < 8; q += 4) {
            se_t += (e[q] + e[q + 1]) + (e[q + 2] + e[q + 3]);
            sx_t += (x[q] + x[q + 1]) + (x[q + 2] + x[q + 3]);
          }
        }
        for (; pt + 3 * a.lanes < a.nparts; pt += 4 * a.lanes) {
          sum_t e[4], x[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            e[q] = s0[(size_t)(pt + q * a.lanes) * a.bstride];
            x[q] = s1[(size_t)(pt + q * a.lanes) * a.bstride];
          }
          se_t += (e[0] + e[1]) + (e[2] + e[3]);
          sx_t += (x[0] + x[1]) + (x[2] + x[3]);
        }
        for (; pt < a.nparts; pt += a.lanes) {
          se_t += s0[(size_t)pt * a.bstride];
          sx_t += s1[(size_t)pt * a.bstride];
        }
      };
      const size_t first = (size_t)(2 * side) * a.nparts * a.bstride + r;
      if (PRECISE && a.sums64) add_up(a.sums64 + first);
      else add_up(a.sums + first);
    }
    if (a.lanes > 1) {                                   // block-uniform
      part[0][threadIdx.x] = se_t;
      part[1][threadIdx.x] = sx_t;
      __syncthreads();
      if (pl == 0) {      // all LDS reads of a thread issued together (compile-time trip counts), then added in order
        switch (a.lanes) {
          case 2: add_parts<2>(part, sa, se_t, sx_t); break;
          case 4: add_parts<4>(part, sa, se_t, sx_t); break;
          case 8: add_parts<8>(part, sa, se_t, sx_t); break;
          case 16: add_parts<16>(part, sa, se_t, sx_t); break;
          default: add_parts<32>(part, sa, se_t, sx_t); break;
        }
      }
      __syncthreads();                                   // before the next tile overwrites part
    }
    const float se = (float)se_t, sx = (float)sx_t;
    float ce = 0.f;
    if (finisher) {
      const SideResult o = state_side<PRECISE>(a, se, sx, u_old, tau);
      ce = o.ce;
      lterm += o.lterm;
      hterm += o.hterm;
      const bool step_tau = a.version == FASTCLIP_V2 && a.tau_upd.optimizer;
      if (a.records) {
        if (step_tau) {
          tau_step_values(a.tau_upd, tau, m, v, o.gt);
          *(float4*)(a.u_img + n + 4 * side) = make_float4(o.u, tau, m, v);
        } else {
          a.u_img[n + 4 * side] = o.u;
        }
      } else {
        (side ? a.u_txt : a.u_img)[n] = o.u;
        if (step_tau) {
          float* pv = side ? a.v_txt : a.v_img;
          tau_step(a.tau_upd, (side ? a.tau_txt : a.tau_img) + n, (side ? a.m_txt : a.m_img) + n, pv ? pv + n : nullptr,
                   o.gt);
        }
      }
      (side ? a.c2 : a.c1)[r] = o.c;
      if (a.version == FASTCLIP_V2) (side ? a.d_tau_txt : a.d_tau_img)[r] = o.gt;
      float* g_out = side ? a.g_txt : a.g_img;
      if (g_out) g_out[r] = se * a.inv_M;
      float* u_out = side ? a.u_new_txt : a.u_new_img;
      if (u_out) u_out[r] = o.u;
    }
    const float ce_other = __shfl_xor(ce, 1);              // the two sides of an anchor are neighbouring lanes
    if (finisher && side == 0) a.dcoef[r] = ce + ce_other;  // c1 M g1 + c2 M g2
  }
  const double x = wave_sum_f64(lterm), y = wave_sum_f64(hterm);
  if ((threadIdx.x & 63) == 0) { scal[0][threadIdx.x >> 6] = x; scal[1][threadIdx.x >> 6] = y; }
  __syncthreads();
  if (threadIdx.x == 0) {
    a.red[2 * blockIdx.x + 0] = (scal[0][0] + scal[0][1]) + (scal[0][2] + scal[0][3]);
    a.red[2 * blockIdx.x + 1] = (scal[1][0] + scal[1][1]) + (scal[1][2] + scal[1][3]);
  }
}

// The per-sample arrays are the fields {u_1, tau_1, m_1, v_1, u_2, tau_2, m_2, v_2} of 32-byte aligned records.
bool state_records_are_canonical(const float* u_img, const float* u_txt, const fastclip_tau_state& t, int64_t stride) {
  return stride >= 8 && stride % 8 == 0 && ((uintptr_t)u_img & 31) == 0 && t.tau_img == u_img + 1 &&
         t.m_img == u_img + 2 && t.v_img == u_img + 3 && u_txt == u_img + 4 && t.tau_txt == u_img + 5 &&
         t.m_txt == u_img + 6 && t.v_txt == u_img + 7;
}

StateArgs make_state_args(const StepCtx& c) {
  const Layout& L = c.L;
  StateArgs a;
  a.idx = c.buf.idx; a.u_img = c.buf.u_img; a.u_txt = c.buf.u_txt;
  a.tau1 = (const float*)(c.ws + L.tau1); a.tau2 = (const float*)(c.ws + L.tau2);
  a.uold1 = (const float*)(c.ws + L.uold1); a.uold2 = (const float*)(c.ws + L.uold2);
  a.sums = (const float*)(c.ws + L.sums); a.nparts = L.nparts;
  a.sums64 = !L.bf16 && L.nparts > 1 ? (const double*)(c.ws + L.sums) : nullptr;
  a.bstride = L.bstride; a.b = L.b;
  a.fused = L.fused_state;
  a.stride = c.cfg.state_stride;
  a.M = (float)(L.B - 1); a.inv_M = 1.0f / a.M; a.bM = (float)L.b * a.M; a.gamma = c.cfg.gamma; a.eps = c.cfg.eps; a.rho = c.cfg.rho;
  a.tau_scale = c.cfg.tau_grad_scale; a.version = c.cfg.version;
  a.c1 = (float*)(c.ws + L.c1); a.c2 = (float*)(c.ws + L.c2); a.dcoef = (float*)(c.ws + L.dcoef);
  a.red = (double*)(c.ws + L.red);
  a.d_tau_img = c.buf.d_tau_img; a.d_tau_txt = c.buf.d_tau_txt; a.g_img = c.buf.g_img; a.g_txt = c.buf.g_txt;
  a.u_new_img = c.buf.u_new_img; a.u_new_txt = c.buf.u_new_txt;
  a.tau_upd = c.tau_upd;
  if (c.cfg.version != FASTCLIP_V2) a.tau_upd.optimizer = 0;
  a.tau_img = c.tau_st.tau_img; a.tau_txt = c.tau_st.tau_txt;
  a.m_img = c.tau_st.m_img; a.v_img = c.tau_st.v_img; a.m_txt = c.tau_st.m_txt; a.v_txt = c.tau_st.v_txt;
  a.lanes = state_lanes(L.nparts);
  a.ntiles = L.nstate_blocks;
  a.tau_glob = c.buf.tau;
  // with the temperature update on canonical records the kernel takes u^t and the temperatures from the records
  // themselves (the same values that the prep kernel gathered): one 16-byte word per side holds all it needs
  a.records = a.tau_upd.optimizer && state_records_are_canonical(a.u_img, a.u_txt, c.tau_st, a.stride);
  a.gather = a.records;
  return a;
}

void launch_state(const StepCtx& c) {
  auto* kernel = c.L.bf16 ? k_state<false> : k_state<true>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)c.L.nstate_blocks), dim3(256), 0, c.s, make_state_args(c));
}

// One wavefront: the scalars of a state phase that ran on its own.
__global__ void k_scalars(const double* red, int nblocks, int64_t b, int version, const float* tau, float rho,
                          float* loss, float* d_tau);

// The state phase on its own (fastclip_state_phase): n = cfg.b anchors whose four sums are given, everything else as
// in the step; the kernel gathers u^t and the temperatures itself.
void launch_state_phase(const fastclip_config& cfg, const fastclip_buffers& buf, const TauUpd& upd,
                        const fastclip_tau_state& tst, const float* sums, float* coef, double* red, int nblocks,
                        hipStream_t s) {
  StateArgs a;
  memset(&a, 0, sizeof(a));
  a.idx = buf.idx; a.u_img = buf.u_img; a.u_txt = buf.u_txt;
  a.sums = sums; a.nparts = 1; a.bstride = cfg.b; a.b = cfg.b;
  a.stride = cfg.state_stride;
  a.M = (float)(cfg.B - 1); a.inv_M = 1.0f / a.M; a.bM = (float)cfg.b * a.M; a.gamma = cfg.gamma; a.eps = cfg.eps; a.rho = cfg.rho;
  a.tau_scale = cfg.tau_grad_scale; a.version = cfg.version;
  a.c1 = coef; a.c2 = coef + cfg.b; a.dcoef = coef + 2 * cfg.b;
  a.red = red;
  a.d_tau_img = buf.d_tau_img; a.d_tau_txt = buf.d_tau_txt; a.g_img = buf.g_img; a.g_txt = buf.g_txt;
  a.u_new_img = buf.u_new_img; a.u_new_txt = buf.u_new_txt;
  a.tau_upd = upd;
  if (cfg.version != FASTCLIP_V2) a.tau_upd.optimizer = 0;
  a.tau_img = a.tau_upd.optimizer ? tst.tau_img : const_cast<float*>(buf.tau_img);
  a.tau_txt = a.tau_upd.optimizer ? tst.tau_txt : const_cast<float*>(buf.tau_txt);
  a.m_img = tst.m_img; a.v_img = tst.v_img; a.m_txt = tst.m_txt; a.v_txt = tst.v_txt;
  a.lanes = 1;
  a.ntiles = (cfg.b + 127) / 128;
  a.tau_glob = buf.tau;
  a.gather = 1;
  a.records = cfg.version == FASTCLIP_V2 && a.tau_upd.optimizer &&
              state_records_are_canonical(a.u_img, a.u_txt, tst, a.stride);
  auto* kernel = cfg.emb_dtype == FASTCLIP_BF16 ? k_state<false> : k_state<true>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)nblocks), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_scalars, dim3(1), dim3(64), 0, s, (const double*)red, nblocks, cfg.b, cfg.version, buf.tau,
                     cfg.rho, buf.loss, buf.d_tau);
}

// Eq. 1 alone, one thread per anchor (the same update as in k_state).
__global__ void __launch_bounds__(256) k_state_flat(const int64_t* __restrict__ idx, int64_t n, int64_t stride,
                                                    float gamma, float invM,
                                                    const float* __restrict__ s1, const float* __restrict__ s2,
                                                    float* __restrict__ u_img, float* __restrict__ u_txt,
                                                    float* __restrict__ o1, float* __restrict__ o2) {
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r >= n) return;
  const int64_t i = idx[r] * stride;
  const float u1 = ema_update(u_img[i], s1[r] * invM, gamma);
  const float u2 = ema_update(u_txt[i], s2[r] * invM, gamma);
  u_img[i] = u1;
  u_txt[i] = u2;
  o1[r] = u1;
  o2[r] = u2;
}

void launch_state_flat(const int64_t* idx, int64_t n, int64_t stride, float gamma, float M, const float* sum_img,
                       const float* sum_txt, float* u_img, float* u_txt, float* u_new_img, float* u_new_txt,
                       hipStream_t s) {
  hipLaunchKernelGGL(k_state_flat, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, idx, n, stride, gamma, 1.0f / M, sum_img,
                     sum_txt, u_img, u_txt, u_new_img, u_new_txt);
}

__global__ void k_scalars(const double* red, int nblocks, int64_t b, int version, const float* tau, float rho,
                          float* loss, float* d_tau) {
  write_scalars(red, nblocks, b, version, tau, rho, loss, d_tau);
}

// ------------------------------------------------------------------------------------------
// MFMA path, last phase.  d_img[r] = c1_r * (sum over splits of the contraction)[r] - dcoef_r txt_p, and the mirror
// image (the contraction already carries the contrast-side terms divided by c_r); block (0,0,0) also writes the
// scalars.  The split partials are whole tiles of [64 groups of 4 rows][cols columns][4 rows] (the order in
// which k_contract_bf16's accumulators leave in 16-byte words), so a block of one wavefront takes four rows and 256
// columns, 4 KiB of addresses per split (consecutive ones inside a tile), and a thread four columns.  A block is four
// wavefronts: four groups of rows (SHARE_SPLITS false), or, when that would leave most of the chip idle, one group
// of rows whose splits the four wavefronts share (wave w sums the splits w, w + 4, ..; the four sums meet in LDS and
// are added in the order of the waves).
template <bool SHARE_SPLITS>
__global__ void __launch_bounds__(256) k_finalize_bf16(const bf16_t* __restrict__ img, const bf16_t* __restrict__ txt,
                                                       int64_t ld_img, int64_t ld_txt, int64_t off, int64_t b, int64_t d,
                                                       const float* __restrict__ O1, const float* __restrict__ O2,
                                                       int nsplit, int cols, const float* __restrict__ c1,
                                                       const float* __restrict__ c2, const float* __restrict__ dcoef,
                                                       float* __restrict__ d_img, float* __restrict__ d_txt,
                                                       const double* __restrict__ red, int nblocks, int version,
                                                       const float* __restrict__ tau, float rho, float* __restrict__ loss,
                                                       float* __restrict__ d_tau) {
  __shared__ float4 meet[SHARE_SPLITS ? 3 : 1][4][64];     // [wave - 1][column of the thread][lane]
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t r0 = ((int64_t)blockIdx.x * (SHARE_SPLITS ? 1 : 4) + (SHARE_SPLITS ? 0 : wave)) * 4;   // rows r0 .. r0 + 3
  const int64_t n0 = (int64_t)blockIdx.z * 256 + (int64_t)lane * 4;     // columns n0 .. n0 + 3 (d % 8 == 0)
  const int side = blockIdx.y;
  const bool live = r0 < b && n0 < d;
  const int nr = (int)(b - r0 < 4 ? b - r0 : 4);
  const bf16_t* X = side == 0 ? txt : img;          // the diagonal term takes the other side's row
  const int64_t ldx = side == 0 ? ld_txt : ld_img;
  float cown[4], dc[4];                             // requested ahead of the partial sums: one memory latency, not two
  uint2 xr[4];
  float acc[4][4] = {};                             // [column][row]
  if (live) {
    if (!SHARE_SPLITS || wave == 0) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int64_t r = r0 + (t < nr ? t : 0);
        cown[t] = (side == 0 ? c1 : c2)[r];
        dc[t] = dcoef[r];
        xr[t] = *(const uint2*)(X + (off + r) * ldx + n0);
      }
    }
    const float* O = side == 0 ? O1 : O2;
    const size_t split_stride = partial_split_floats(b, d, cols);
    const int64_t tiles_m = (b + 255) / 256;
    const int n = (int)n0, tile_n = cols == 256 ? n >> 8 : n / 192;      // d < 2^24; four columns never straddle tiles
    const size_t at = (size_t)(tile_n * tiles_m + (r0 >> 8)) * (size_t)(256 * cols) +
                      (size_t)((((r0 & 255) >> 2) * cols + (n - tile_n * cols)) * 4);
#pragma unroll 4
    for (int s = SHARE_SPLITS ? wave : 0; s < nsplit; s += SHARE_SPLITS ? 4 : 1) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float4 v = *(const float4*)(O + (size_t)s * split_stride + at + 4 * j);
        acc[j][0] += v.x; acc[j][1] += v.y; acc[j][2] += v.z; acc[j][3] += v.w;
      }
    }
  }
  if (SHARE_SPLITS) {
    if (wave > 0) {
#pragma unroll
      for (int j = 0; j < 4; ++j) meet[wave - 1][j][lane] = make_float4(acc[j][0], acc[j][1], acc[j][2], acc[j][3]);
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int w = 0; w < 3; ++w)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float4 v = meet[w][j][lane];
        acc[j][0] += v.x; acc[j][1] += v.y; acc[j][2] += v.z; acc[j][3] += v.w;
      }
  }
  if (live) {
    float* out = (side == 0 ? d_img : d_txt) + r0 * d + n0;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (t >= nr) break;
      float4 o;
      o.x = cown[t] * acc[0][t] - dc[t] * __uint_as_float(xr[t].x << 16);
      o.y = cown[t] * acc[1][t] - dc[t] * __uint_as_float(xr[t].x & 0xffff0000u);
      o.z = cown[t] * acc[2][t] - dc[t] * __uint_as_float(xr[t].y << 16);
      o.w = cown[t] * acc[3][t] - dc[t] * __uint_as_float(xr[t].y & 0xffff0000u);
      *(float4*)(out + t * d) = o;
    }
  }
  if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x < 64)
    write_scalars(red, nblocks, b, version, tau, rho, loss, d_tau);
}

// Gradient through e^ = e / |e| (cosine similarity, Sec. 3), after the gradients with respect to e^ are complete:
// out := (out - e^ (e^ . out)) / |e|, e^ = the side's own row.  One block per anchor and side; on the accuracy path
// (T = float) in fp64.
template <typename T, typename A>
__global__ void __launch_bounds__(256) k_norm_backward(const T* __restrict__ img, const T* __restrict__ txt,
                                                       int64_t ld_img, int64_t ld_txt, int64_t off, int64_t d,
                                                       float* __restrict__ d_img, float* __restrict__ d_txt,
                                                       const float* __restrict__ norm_img,
                                                       const float* __restrict__ norm_txt) {
  __shared__ A part[4];
  const int64_t r = blockIdx.x;
  const int side = blockIdx.y;
  const T* ep = side == 0 ? img + (off + r) * ld_img : txt + (off + r) * ld_txt;
  float* out = (side == 0 ? d_img : d_txt) + r * d;
  A dot = 0;
  for (int64_t n = threadIdx.x; n < d; n += 256) dot += (A)out[n] * (A)load_elem(ep + n);
  dot = wave_sum(dot);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = dot;
  __syncthreads();
  dot = (part[0] + part[1]) + (part[2] + part[3]);
  const A inv = (A)1 / (A)(side == 0 ? norm_img : norm_txt)[r];
  for (int64_t n = threadIdx.x; n < d; n += 256) out[n] = (float)(((A)out[n] - dot * (A)load_elem(ep + n)) * inv);
}

// The same where rows are whole groups of four elements, aligned, and at most 1024 wide: a wavefront per anchor and side, whose
// lanes hold the row (k_normalize_rows_quads).  What bounds it is the chain load - sum - store: with the norm and the row a
// second time behind the sum it was three trips to memory, and a workgroup of four wavefronts per row.  What it adds to a step, us:
// 4096 bf16 rows of width 768 14.9 -> 10.0, 1024 fp32 rows of width 512 4.6 -> 2.3, 128 3.6 -> 2.9; one round of workgroups of bf16
// rows as before (256 of width 512 3.6).
template <typename T, typename A>
__global__ void __launch_bounds__(256) k_norm_backward_quads(const T* __restrict__ img, const T* __restrict__ txt, int64_t ld_img,
                                                             int64_t ld_txt, int64_t off, int64_t b, int d,
                                                             float* __restrict__ d_img, float* __restrict__ d_txt,
                                                             const float* __restrict__ norm_img, const float* __restrict__ norm_txt) {
  const int lane = threadIdx.x & 63, side = blockIdx.y;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= b) return;
  const T* ep = side == 0 ? img + (off + r) * ld_img : txt + (off + r) * ld_txt;
  float* out = (side == 0 ? d_img : d_txt) + r * d;
  const float norm = (side == 0 ? norm_img : norm_txt)[r];
  float4 o[kNormQuads], e[kNormQuads];
#pragma unroll
  for (int i = 0; i < kNormQuads; ++i) {
    const int k = 4 * (lane + 64 * i);
    o[i] = k < d ? load_quad((const float*)out + k) : make_float4(0.f, 0.f, 0.f, 0.f);
    e[i] = k < d ? load_quad(ep + k) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  A dot = 0;
#pragma unroll
  for (int i = 0; i < kNormQuads; ++i)
    dot += ((A)o[i].x * (A)e[i].x + (A)o[i].y * (A)e[i].y) + ((A)o[i].z * (A)e[i].z + (A)o[i].w * (A)e[i].w);
  dot = wave_sum(dot);
  const A inv = (A)1 / (A)norm;
#pragma unroll
  for (int i = 0; i < kNormQuads; ++i) {
    const int k = 4 * (lane + 64 * i);
    if (k < d)
      store_quad(out + k, make_float4((float)(((A)o[i].x - dot * (A)e[i].x) * inv), (float)(((A)o[i].y - dot * (A)e[i].y) * inv),
                                      (float)(((A)o[i].z - dot * (A)e[i].z) * inv), (float)(((A)o[i].w - dot * (A)e[i].w) * inv)));
  }
}

void launch_finalize_bf16(const StepCtx& c) {
  const Layout& L = c.L;
  const dim3 block(256);
  const unsigned col_tiles = (unsigned)((L.d + 255) / 256);
  // four row groups per block unless that makes fewer than two blocks per compute unit: then one, its splits shared
  const bool share = (uint64_t)((L.b + 15) / 16) * 2 * col_tiles < 512 && L.nsplit >= 4;
  const dim3 grid((unsigned)(share ? (L.b + 3) / 4 : (L.b + 15) / 16), 2, col_tiles);
  auto* kernel = share ? k_finalize_bf16<true> : k_finalize_bf16<false>;
  hipLaunchKernelGGL(kernel, grid, block, 0, c.s, (const bf16_t*)c.buf.img_glob, (const bf16_t*)c.buf.txt_glob,
                     c.cfg.ld_img, c.cfg.ld_txt, L.off, L.b, L.d, (const float*)(c.ws + L.Opart[0]),
                     (const float*)(c.ws + L.Opart[1]), L.nsplit, L.out_cols, (const float*)(c.ws + L.c1),
                     (const float*)(c.ws + L.c2), (const float*)(c.ws + L.dcoef), c.buf.d_img, c.buf.d_txt, (const double*)(c.ws + L.red),
                     L.nstate_blocks, c.cfg.version, c.buf.tau, c.cfg.rho, c.buf.loss, c.buf.d_tau);
}

void launch_norm_backward(const StepCtx& c) {
  const Layout& L = c.L;
  if (!c.buf.norm_img) return;
  const dim3 grid((unsigned)L.b, 2), block(256), of_quads((unsigned)((L.b + 3) / 4), 2);
  const size_t quad = 4 * (L.bf16 ? sizeof(bf16_t) : sizeof(float));
  const bool quads = L.d % 4 == 0 && L.d <= 256 * kNormQuads && c.cfg.ld_img % 4 == 0 && c.cfg.ld_txt % 4 == 0 &&
                     (uintptr_t)c.buf.img_glob % quad == 0 && (uintptr_t)c.buf.txt_glob % quad == 0;   // (d_img, d_txt: 16 bytes)
  if (quads && L.bf16)
    hipLaunchKernelGGL((k_norm_backward_quads<bf16_t, float>), of_quads, block, 0, c.s, (const bf16_t*)c.buf.img_glob,
                       (const bf16_t*)c.buf.txt_glob, c.cfg.ld_img, c.cfg.ld_txt, L.off, L.b, (int)L.d, c.buf.d_img, c.buf.d_txt,
                       c.buf.norm_img, c.buf.norm_txt);
  else if (quads)
    hipLaunchKernelGGL((k_norm_backward_quads<float, double>), of_quads, block, 0, c.s, (const float*)c.buf.img_glob,
                       (const float*)c.buf.txt_glob, c.cfg.ld_img, c.cfg.ld_txt, L.off, L.b, (int)L.d, c.buf.d_img, c.buf.d_txt,
                       c.buf.norm_img, c.buf.norm_txt);
  else if (L.bf16)
    hipLaunchKernelGGL((k_norm_backward<bf16_t, float>), grid, block, 0, c.s, (const bf16_t*)c.buf.img_glob,
                       (const bf16_t*)c.buf.txt_glob, c.cfg.ld_img, c.cfg.ld_txt, L.off, L.d, c.buf.d_img, c.buf.d_txt,
                       c.buf.norm_img, c.buf.norm_txt);
  else
    hipLaunchKernelGGL((k_norm_backward<float, double>), grid, block, 0, c.s, (const float*)c.buf.img_glob,
                       (const float*)c.buf.txt_glob, c.cfg.ld_img, c.cfg.ld_txt, L.off, L.d, c.buf.d_img, c.buf.d_txt,
                       c.buf.norm_img, c.buf.norm_txt);
}

// ------------------------------------------------------------------------------------------
// Index checker: open-addressing hash set of the b indices; flag word at ws[0].
__global__ void __launch_bounds__(256) k_idx_fill(int* flag, long long* table, size_t slots) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i == 0) *flag = 0;
  if (i < slots) table[i] = -1;
}

__global__ void __launch_bounds__(256) k_idx_insert(const int64_t* __restrict__ idx, int64_t b, int64_t N, int* flag,
                                                    unsigned long long* table, size_t slots, int shift) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= b) return;
  const int64_t v = idx[i];
  if (v < 0 || v >= N) { *flag = 1; return; }
  size_t h = (size_t)(((unsigned long long)v * 11400714819323198485ull) >> shift);
  for (size_t probe = 0; probe < slots; ++probe) {     // bounded: the table has at least 2b slots
    const unsigned long long old = atomicCAS(&table[h], ~0ull, (unsigned long long)v);
    if (old == ~0ull) return;
    if (old == (unsigned long long)v) { *flag = 1; return; }
    h = (h + 1) & (slots - 1);
  }
  *flag = 1;
}

void launch_check_indices(const int64_t* idx, int64_t b, int64_t N, void* ws, hipStream_t s) {
  size_t slots = 64;
  int log2s = 6;
  while (slots < (size_t)b * 2) { slots <<= 1; ++log2s; }
  int* flag = (int*)ws;
  long long* table = (long long*)((char*)ws + 256);
  hipLaunchKernelGGL(k_idx_fill, dim3((unsigned)((slots + 255) / 256)), dim3(256), 0, s, flag, table, slots);
  hipLaunchKernelGGL(k_idx_insert, dim3((unsigned)((b + 255) / 256)), dim3(256), 0, s, idx, b, N, flag,
                     (unsigned long long*)table, slots, 64 - log2s);
}

}  // namespace fc
