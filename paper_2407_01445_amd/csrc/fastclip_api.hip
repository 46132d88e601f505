// C ABI of libfastclip: argument validation, workspace carving, launch sequences.
// The arithmetic lives in the kernel translation units; nothing here runs on the CPU
// except checks, address arithmetic and the gamma schedule.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <mutex>

#include "fc_internal.hpp"

namespace fc {

static bool bad_float(float x) { return !(x == x) || isinf(x); }

static thread_local hipError_t g_last_hip_error = hipSuccess;
// Reads and clears the runtime's error state; remembers a failure for fastclip_last_hip_error.
static fastclip_status launch_status() {
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) return FASTCLIP_OK;
  g_last_hip_error = e;
  return FASTCLIP_ERR_LAUNCH;
}
static fastclip_status hip_failed(hipError_t e) {
  g_last_hip_error = e;
  return FASTCLIP_ERR_LAUNCH;
}

fastclip_status validate(const fastclip_config* cfg, const fastclip_buffers* bufs) {
  if (!cfg) return FASTCLIP_ERR_NULL;
  if (cfg->struct_size != sizeof(fastclip_config) || (cfg->flags & ~(FASTCLIP_GATHERED_STATE | FASTCLIP_FINE_TILES | FASTCLIP_SINGLE_PASS | FASTCLIP_TILES_128 | FASTCLIP_TILES_256)))
    return FASTCLIP_ERR_SHAPE;
  if (cfg->B < 2 || cfg->b < 1 || cfg->off < 0 || cfg->off + cfg->b > cfg->B || cfg->d < 1 ||
      cfg->ld_img < cfg->d || cfg->ld_txt < cfg->d || cfg->N < 1 || cfg->b > cfg->N || cfg->state_stride < 1 ||
      cfg->state_stride > 64)
    return FASTCLIP_ERR_SHAPE;
  if ((cfg->flags & FASTCLIP_TILES_128) && (cfg->flags & FASTCLIP_TILES_256)) return FASTCLIP_ERR_VALUE;
  if (cfg->version < FASTCLIP_V0 || cfg->version > FASTCLIP_V3) return FASTCLIP_ERR_VALUE;
  if (cfg->emb_dtype != FASTCLIP_F32 && cfg->emb_dtype != FASTCLIP_BF16) return FASTCLIP_ERR_VALUE;
  if (bad_float(cfg->gamma) || bad_float(cfg->eps) || bad_float(cfg->rho) || bad_float(cfg->tau_grad_scale))
    return FASTCLIP_ERR_VALUE;
  if (!(cfg->gamma > 0.0f && cfg->gamma <= 1.0f) || cfg->eps < 0.0f) return FASTCLIP_ERR_VALUE;
  const int64_t lim = (int64_t)1 << 24;
  if (cfg->B > lim || cfg->b > lim || cfg->d > lim || cfg->ld_img > ((int64_t)1 << 30) ||
      cfg->ld_txt > ((int64_t)1 << 30))
    return FASTCLIP_ERR_UNSUPPORTED;
  if (cfg->emb_dtype == FASTCLIP_BF16 && (cfg->d % 8 || cfg->ld_img % 8 || cfg->ld_txt % 8))
    return FASTCLIP_ERR_UNSUPPORTED;
  // the MFMA kernels address a tile panel (256 rows, or 8 anchor blocks of the stored strips) with 32-bit byte
  // offsets per lane
  const int64_t lim22 = (int64_t)1 << 22;
  if (cfg->emb_dtype == FASTCLIP_BF16 && (cfg->B + cfg->b > lim22 || cfg->ld_img > lim22 || cfg->ld_txt > lim22))
    return FASTCLIP_ERR_UNSUPPORTED;
  if (bufs) {
    if (!bufs->img_glob || !bufs->txt_glob || !bufs->idx || !bufs->u_img || !bufs->u_txt ||
        !bufs->d_img || !bufs->d_txt || !bufs->loss)
      return FASTCLIP_ERR_NULL;
    if (cfg->version == FASTCLIP_V2) {
      if (!bufs->tau_img || !bufs->tau_txt || !bufs->d_tau_img || !bufs->d_tau_txt) return FASTCLIP_ERR_NULL;
    } else {
      if (!bufs->tau) return FASTCLIP_ERR_NULL;
      if ((cfg->version == FASTCLIP_V0 || cfg->version == FASTCLIP_V3) && !bufs->d_tau) return FASTCLIP_ERR_NULL;
    }
    if ((bufs->norm_img == nullptr) != (bufs->norm_txt == nullptr)) return FASTCLIP_ERR_NULL;
    if ((cfg->flags & FASTCLIP_GATHERED_STATE) && cfg->b < cfg->B) {   // b == B: no remote anchors, arrays not read
      if (!bufs->u_glob_img || !bufs->u_glob_txt) return FASTCLIP_ERR_NULL;
      if (cfg->version == FASTCLIP_V2 && (!bufs->tau_glob_img || !bufs->tau_glob_txt)) return FASTCLIP_ERR_NULL;
    }
    if (cfg->emb_dtype == FASTCLIP_BF16 &&
        (((uintptr_t)bufs->img_glob & 15) || ((uintptr_t)bufs->txt_glob & 15)))
      return FASTCLIP_ERR_UNSUPPORTED;
    if (((uintptr_t)bufs->d_img & 15) || ((uintptr_t)bufs->d_txt & 15)) return FASTCLIP_ERR_UNSUPPORTED;
  }
  return FASTCLIP_OK;
}

fastclip_status validate_tau_update(int32_t version, const fastclip_tau_update* upd, const fastclip_tau_state* st) {
  if (!upd || !st) return FASTCLIP_ERR_NULL;
  if (upd->struct_size != sizeof(fastclip_tau_update) || upd->state_stride < 0 || upd->state_stride > 64)
    return FASTCLIP_ERR_SHAPE;
  if (version < FASTCLIP_V0 || version > FASTCLIP_V3) return FASTCLIP_ERR_VALUE;
  if (upd->optimizer < FASTCLIP_TAU_SGDM || upd->optimizer > FASTCLIP_TAU_ADAMW) return FASTCLIP_ERR_VALUE;
  const float f[7] = {upd->lr, upd->beta1, upd->beta2, upd->eps, upd->tau_min, upd->lr_drop_below, upd->lr_drop_factor};
  for (float x : f)
    if (bad_float(x)) return FASTCLIP_ERR_VALUE;
  if (upd->step < 1 || upd->lr < 0.0f || upd->eps < 0.0f || upd->beta1 < 0.0f || upd->beta1 >= 1.0f ||
      upd->beta2 < 0.0f || upd->beta2 >= 1.0f || upd->lr_drop_factor < 0.0f)
    return FASTCLIP_ERR_VALUE;
  const bool two = upd->optimizer == FASTCLIP_TAU_ADAMW || upd->optimizer == FASTCLIP_TAU_LAMB;
  if (version == FASTCLIP_V2) {
    if (!st->tau_img || !st->tau_txt || !st->m_img || !st->m_txt) return FASTCLIP_ERR_NULL;
    if (two && (!st->v_img || !st->v_txt)) return FASTCLIP_ERR_NULL;
  } else if (version != FASTCLIP_V1) {
    if (!st->tau || !st->m || (two && !st->v)) return FASTCLIP_ERR_NULL;
  }
  return FASTCLIP_OK;
}

TauUpd make_tau_upd(const fastclip_tau_update& upd) {
  TauUpd u;
  u.optimizer = upd.optimizer;
  u.lr = upd.lr; u.beta1 = upd.beta1; u.beta2 = upd.beta2; u.eps = upd.eps;
  // bias corrections 1 / (1 - beta^step) of Proc. "parameter_update", in double on the host
  u.corr1 = (float)(1.0 / (1.0 - pow((double)upd.beta1, (double)upd.step)));
  u.corr2 = (float)(1.0 / (1.0 - pow((double)upd.beta2, (double)upd.step)));
  u.tau_min = upd.tau_min; u.drop_below = upd.lr_drop_below; u.drop_factor = upd.lr_drop_factor;
  u.stride = upd.state_stride > 1 ? upd.state_stride : 1;
  return u;
}

// What a plan may put into the workspace for speed alone (see make_layout).
struct Room {
  int64_t split_bytes;     // partial results of splits
  bool partial_sums;       // fp32 path: partial sums of the strips, which its single pass needs too
  bool state_rides;        // fp32 path: the state phase inside the gradients, which has a counter and scalar partials of its own
};

// fp32 path: tile sizes, partial sums and the split of the gradients' depth.
static void plan_f32(const fastclip_config& cfg, const Room& room, Layout* L) {
  // 64 x 64 strip tiles once there is one per compute unit; below that 32 x 32, four times as many
  const int64_t strips = L->square ? 1 : 2;
  L->strip_tile = strips * ((cfg.b + 63) / 64) * ((cfg.B + 63) / 64) >= 256 ? 64 : 32;
  // Partial sums: one per contrast tile, at most 64 (the state phase reads them all); a whole local batch also sums down
  // its columns, one partial per anchor tile, and keeps one per tile on either side.
  const int64_t nCT = (cfg.B + L->strip_tile - 1) / L->strip_tile;
  int64_t per = L->square ? 1 : (nCT + 63) / 64;
  if (!room.partial_sums) per = nCT;
  L->per_part = (int)per;
  L->nparts = (int)((nCT + per - 1) / per);
  // Gradients: tile size and splits by the time of the fullest compute unit in cycles of a SIMD.  A stage is 1024 cycles of
  // matrix products on 32 x 32 tiles (64 deep) and 2048 on 64 x 64 tiles (32 deep), 1.3 times that as measured; a tile's
  // start and end cost 3000, the meeting of several splits 4000 + 500 per split.  Measured: 128 anchors of 1024 pairs of
  // width 512: 38.4 us per step with one split of 32 x 32 tiles, 33.2 with two (chosen), 34.4 with four; 1024 pairs: 94 us on
  // 32 x 32 tiles, 88 on 64 x 64 (chosen).
  double best_cost = 0.0;
  for (int T = 32; T <= 64; T += 32) {
    const int64_t kd = T == 32 ? 64 : 32;
    const int64_t stages = (cfg.B + kd - 1) / kd + (L->square ? 0 : (cfg.b + kd - 1) / kd);
    const int64_t tiles = 2 * ((cfg.b + T - 1) / T) * ((cfg.d + T - 1) / T);
    for (int64_t ns = 1; ns <= 16 && ns <= stages; ++ns) {
      const int64_t slice = (stages + ns - 1) / ns;
      if ((stages + slice - 1) / slice != ns) continue;
      if (ns > 1 && (tiles * ns > 2048 || ns * tiles * T * T * (int64_t)sizeof(double) > room.split_bytes)) break;
      const double rounds = (double)((tiles * ns + 255) / 256);
      const double cost = rounds * ((double)slice * (T == 32 ? 1330.0 : 2600.0) + 3000.0) +
                          (ns > 1 ? 4000.0 + 500.0 * (double)ns : 0.0);
      if (best_cost == 0.0 || cost < best_cost) {
        best_cost = cost;
        L->grad_tile = T; L->nsplit = (int)ns; L->kslice = slice;
      }
    }
  }
}

// Every 64 x 64 block of the fold needs the coefficients of 128 anchor sides.  Forming them inside the fold saves a
// launch, but every block then sums those anchors' partial sums again (b^2 / 32 anchor sides x nparts floats in
// all, against 2 b x nparts once): worth it only while that stays small.
static bool fold_forms_state(int64_t b, int nparts) {
  return nparts <= 64 && (double)b * (double)b / 32.0 * (double)nparts * 4.0 <= 2.0 * 1024 * 1024;
}

// 128 x 128-tile path: which contraction, its output tiles, the split of its depth over workgroups, and who runs the state
// phase.  False: the 256 x 256 tiles take less time (gathered state).
static bool plan_t128(const fastclip_config& cfg, const Room& room, Layout* L) {
  double best_cost = 0.0, in_a_row = 0.0;
  int64_t rounds = 0;
  for (int64_t rows = L->gathered ? 64 : 32; rows <= (L->gathered ? 64 : 128); rows *= 2) {
    const int64_t cols = rows == 32 ? 32 : 64, depth = rows == 32 ? 32 : 16;      // 32 x 32 tiles: stages of 32
    const int64_t nA = (cfg.B + depth - 1) / depth, nB = (cfg.b + depth - 1) / depth;
    const int64_t tiles = 2 * ((cfg.b + rows - 1) / rows) * ((cfg.d + cols - 1) / cols);
    for (int64_t ns = 1; ns <= (rows == 32 ? 1 : 16) && ns * 32 <= L->ldE; ++ns) {
      if (rows == 32 && tiles > 256) break;
      if (ns > 1 && (tiles * ns > 2048 || ns * tiles * rows * 64 * (int64_t)sizeof(float) > room.split_bytes)) break;
      const int64_t sA = (nA + ns * 8 - 1) / (ns * 8), sB = (nB + ns * 8 - 1) / (ns * 8);
      const int64_t nq = sB * 8 * depth < cfg.b ? sB * 8 * depth : cfg.b;
      const int64_t r = (tiles * ns + 255) / 256;
      // The state phase inside the contraction: every workgroup adds up the partial sums of its rows and of its q's, at the 57
      // bytes per clock of a compute unit, which takes less than a launch of its own (4.7 us) while it happens once.
      const bool fused = r == 1 || (rows == 64 && nq <= 256 && L->nparts <= 64);
      const double coef_us = (double)((nq + 2 * rows) * L->nparts * 4) / (57.0 * 2400.0);
      const double stages = (L->gathered ? 1.4 : 1.0) * (double)sA + (double)sB;   // a wave's, 16 deep; 1.4: with a second strip
      // compute units left for workgroups that finish the anchors?
      const bool full = (tiles * ns + 7) / 8 * 8 + (cfg.b + 255) / 256 > 256;
      // us: start, coefficients, sum over the waves and end of a workgroup; a stage of its eight waves (the load path of a
      // compute unit: 32 KiB, 48 for 128 rows or with a second strip; 16 deep, on 32 x 32 tiles 32 deep, for which latency is the
      // bound); partial results; the state phase as a launch of its own or by the workgroups of the first columns.  Steps on
      // 32 x 32 / 64 x 64 tiles (their best split), us, width 512: 128 of 1024 13.7 / 16.9, 256 of 2048 18.1 / 19.8, 256 of 4096
      // 23.3 / 23.3, 128 of 4096 22.4 / 20.5, 256 of 8192 36.7 / 30.6; width 256: 512 of 512 15.2 / 16.3, 512 of 2048 18.9 / 20.3,
      // 512 of 4096 25.6 / 25.4; 128 of 1024 at 1024 19.0 / 20.1.
      const double cost = (double)r * (rows == 32 ? 4.1 + 0.62 * stages : (rows == 64 ? 8.0 + 0.27 * stages : 9.5 + 0.38 * stages)) +
                          (ns > 1 ? 2.3 + 0.25 * (double)ns : 0.0) + (fused ? (nq > 256 || rows > 64 ? coef_us : 0.0) + (full ? 1.2 : 0.0) : 4.7);
      if (best_cost == 0.0 || cost < best_cost) {
        best_cost = cost;
        rounds = r; in_a_row = (double)r * stages;
        L->nsplit = (int)ns; L->out_rows = (int)rows; L->fused_state = fused;
      }
    }
  }
  if (L->gathered) {
    // The 256 x 256 tiles fetch a quarter of the bytes per product, at the price of a pass over both strips (fold), partial
    // results and their sum.  Up to 104 stages in a row the small tiles are the faster ones, small / large, us: 640 of 5120 at
    // width 768 (61 stages) 68 / 87, 1024 of 2048 at 1024 (61) 68 / 79, 256 of 8192 at 2048 (92) 106 / 118, 768 of 4096 at 1024
    // (102) 91 / 93.  Beyond, the large ones: 1024 of 4096 at 1024 (106) 98 / 96, 640 of 5120 at 1024 (122) 99 / 96, 512 of 8192
    // at 1280 (187) 131 / 111, 1024 of 4096 at 4096 (422) 363 / 203.  The large strip tiles take longer, up to twice, for a ragged
    // batch, and somewhat longer for rows that end inside a stage.  Ragged batches: 1000 of 4000 at 1024 (106) 103 / 145, 791 of
    // 3880 at 3072 (252) 227 / 237, 702 of 4212 at 3072 (261) 233 / 242, 1135 of 2322 at 4096 (320) 285 / 275, 1000 of 4000 at 3072
    // (317) 267 / 249.  Ragged rows: 700 of 4900 at 760 (121) 107 / 120, 768 of 5376 at 1000 (130) 128 / 133, 452 of 7969 at 1376
    // (140) 144 / 142, 1024 of 4096 at 1376 (158) 140 / 131, 768 of 4105 at 2408 (209) 212 / 174, 997 of 2991 at 3936 (333)
    // 303 / 205.  No room for splits: none for the partial results of the large tiles either.
    const double limit = cfg.d % 64 ? 140.0 : (cfg.B % 256 ? 270.0 : 104.0);
    return room.split_bytes == 0 || in_a_row <= limit;
  }
  // Contraction of kernels_wide128.hip behind the fold.
  // It is taken where the kernel above would need a second round of workgroups, except
  //  - with few local anchors (the fold saves little) or fewer than one workgroup per compute unit,
  //  - with a few workgroups over one per compute unit, two on some.  One split: where the kernel above has two rounds, and below
  //    384 workgroups with fewer than eight rows of tiles, or an odd number of them and, the more rows the more, contrasts that
  //    are not local.  More splits: below 416 workgroups with up to five rows of tiles, below 304 with up to seven,
  //  - with an odd number of workgroups (over 1 split) in a column of tiles: they go to the XCDs in turn, and then every L2
  //    sees the whole of the strips; not where most of the batch is local, which doubles the depth above, and the kernel above
  //    would have two rounds of its 128-row tiles (1896 of 1896 at 640, 3 splits of 15 rows of tiles: 80 / 71; but with two of
  //    64-row tiles 1344 of 1344 at 768, 11 rows: 51 / 55).
  // Step times, above / wide, us.  One round: 1000 of 1000 at 1024: 37 / 42, 1024 of 4096 at 1024: 67 / 70, 640 of 5120 at
  // 1280: 74 / 94.  Two: 1000 of 1000 at 1280: 54 / 48, 1536 of 1536 at 1024: 75 / 65, 2048 of 2048 at 768: 82 / 69 and at
  // 1024 (256 workgroups): 89 / 86, 1024 of 4096 at 2048: 122 / 105.  Four: 2048 of 2048 at 2048: 170 / 115.  Excepted, in
  // this order: 320 of 3300 at 4096: 98 / 102, 411 of 2055 at 2104: 65 / 70, 1408 of 1408 at 1280 (220): 67 / 70; 1435 of 1435
  // at 1288 (264): 91 / 96, 640 of 5120 at 4096 (320, 5 rows): 187 / 205, 576 of 576 at 4096 (320, 5) 75 / 89, 768 of 768 at
  // 3072 (288, 6) 75 / 82, 832 of 2496 at 2560 (280, 7) 130 / 142, 1137 of 2241 at 2560 (360, 9) 140 / 154, 1084 of 1164 at
  // 2560 (360, 9) 93 / 96, 1372 of 2010 at 1536 (264, 11) 106 / 113 (but 900 of 3600 at 2560 (320, 8) 166 / 154, 1212 of 1212
  // at 2048 (320, 10) 87 / 80, 1344 of 1344 at 1536 (264, 11) 89 / 82, 1383 of 1630 at 1536 (264, 11) 106 / 104, 1664 of 1664
  // at 1280 (260, 13) 112 / 94), 576 of 1092 at 2264 (2 splits, 360, 5) 63 / 75, 640 of 2453 at 2560 (2, 400, 5) 83 / 87, 690
  // of 1428 at 1472 (2, 288, 6) 50 / 55 (but 700 of 2800 at 2048 (2, 384, 6) 98 / 91, 512 of 3584 at 2560 (3, 480, 4) 91 /
  // 89); 1344 of 1546 at 736 (3 splits, 11 rows of tiles): 62 / 67, 800 of 4096 at 1536 (3, 7): 100 / 106.
  if (rounds < 2 || cfg.b < 448) return true;
  // Its depth in 32-deep stages goes over `split` workgroups per output tile.  Time in stages of a workgroup that has its
  // compute unit to itself: a second one there stretches both by 1.45, beyond 512 they run in rounds; a tile's start and end
  // cost 4; the finalize kernel 5 + 0.42 per MiB of partial results it reads.
  const int64_t depth = L->ldE / 32, wide_tiles = 2 * ((cfg.b + 127) / 128) * ((cfg.d + 127) / 128);
  int64_t split = 1;
  double wide_cost = 0.0;
  for (int64_t ns = 1; ns <= kMaxSplit && ns <= depth; ++ns) {
    const int64_t slice = (depth + ns - 1) / ns, wgs = wide_tiles * ns;
    if ((depth + slice - 1) / slice != ns) continue;                // every split must get at least one stage
    if (ns > 1 && wgs * 128 * 128 * (int64_t)sizeof(float) > room.split_bytes) break;
    const double stretch = wgs <= 256 ? 1.0 : (wgs <= 512 ? 1.0 + 0.45 * (double)(wgs - 256) / 256.0
                                                          : 1.45 * (double)((wgs + 511) / 512));
    const double cost = stretch * (double)slice + 4.0 + (ns > 1 ? 5.0 + 0.42 / 16.0 * (double)wgs : 0.0);
    if (ns == 1 || cost < wide_cost) { split = ns; wide_cost = cost; }
  }
  const int64_t rows_of_tiles = (cfg.b + 127) / 128, wgs = wide_tiles * split;
  const bool few_rows = rows_of_tiles < 8 || (rows_of_tiles % 2 && cfg.B > cfg.b + 64 + 192 * (rows_of_tiles - 9));
  const bool some_have_two = wgs > 256 && (split == 1 ? rounds == 2 || (wgs < 384 && few_rows)
                                                      : wgs < (rows_of_tiles < 6 ? 416 : (rows_of_tiles < 8 ? 304 : 0)));
  const bool no_shared_l2 = split > 1 && (split * rows_of_tiles) % 2 && (L->out_rows == 64 || 10 * cfg.b < 9 * cfg.B);
  if (wgs >= (cfg.b > 512 ? 256 : 257) && !some_have_two && !no_shared_l2) {
    L->wide = 1;
    L->nsplit = (int)split; L->kslice = (depth + split - 1) / split;
    L->fused_state = fold_forms_state(cfg.b, L->nparts);
    // Strips of one workgroup per compute unit are two bare rounds just above 256 tiles, and with an odd number of contrast tiles
    // the XCDs share no panels either.  Those / two workgroups per compute unit, us: strips of 1536 of 1536 at 1024 25.2 / 23.4,
    // of 960 of 2880 at 1440 (23 contrast tiles) 41 / 37, of 1344 of 2688 at 1120 (21) 37 / 32; steps of 1800 of 1800 at 512
    // 64.1 / 62.3.  With few anchors (768 of 4096, 384 tiles) and at 512 tiles the former are the faster ones all the same
    // (96.1 / 100.8 at 2048).
    const int64_t tiles = 2 * ((cfg.b + 127) / 128) * L->nparts;
    L->wide_strips = tiles > 256 && tiles < 512 && (4 * cfg.b > 3 * cfg.B || L->nparts % 2);
  }
  return true;
}

static void make_layout(const fastclip_config& cfg, const Room& room, Layout* L) {
  memset(L, 0, sizeof(*L));
  L->B = cfg.B; L->b = cfg.b; L->off = cfg.off; L->d = cfg.d; L->N = cfg.N;
  L->bf16 = cfg.emb_dtype == FASTCLIP_BF16;
  L->bstride = (int64_t)round_up((size_t)cfg.b, kTileContrasts);   // whole anchor tiles: the strip kernel works on 256 rows
  L->gathered = (cfg.flags & FASTCLIP_GATHERED_STATE) && cfg.b < cfg.B;
  L->ncol = (int64_t)round_up((size_t)cfg.B, kTileContrasts);
  L->few = !L->bf16 && (cfg.B <= kFewPairs || (cfg.B <= kFewNarrowPairs && cfg.d <= 128));
  // forming the similarity matrix once halves the MFMA work of the strip phase but doubles the epilogue of every
  // tile: it pays once the tiles outnumber the compute units (below that one tile's latency is the phase's time)
  const int64_t bt = (cfg.B + kTileContrasts - 1) / kTileContrasts;
  L->square = cfg.b == cfg.B && (L->bf16 ? 2 * bt * bt > 256 || (cfg.flags & FASTCLIP_SINGLE_PASS) : room.partial_sums && !L->few);
  // Fine tiles (opt-in) where 256 x 256 tiles would leave most of the chip idle: fewer large strip tiles than three
  // quarters of the compute units (one per compute unit is what the large-tile kernels are built for).
  const int64_t big_tiles = 2 * ((cfg.b + 255) / 256) * ((cfg.B + 255) / 256);
  L->fine = (cfg.flags & FASTCLIP_FINE_TILES) && L->bf16 && !L->gathered && !L->square && big_tiles < 192;
  // 128 x 128 tiles: asked for (wherever a quarter of the large tiles' workgroups would still not fill the chip), or
  // chosen when the large tiles would occupy at most half of the compute units.  Steps on small / large tiles, us, width 512:
  // 128 of 1024 (8 large tiles) 21 / 42, 1024 of 1024 (32) 30 / 49, 640 of 5120 (120) 47 / 58, 1024 of 4096 (128) 50 / 63, 2048 of
  // 2048 (128) 56 / 66; at width 1024 2048 of 2048 breaks even (86 / 85).  Above, small tiles are still the faster ones for ragged
  // batches (1200 of 4600, 180 large tiles: 71 / 103) and narrow rows (1024 of 5120, 160: 49 / 55 at 256, 61 / 69 at 512, 84 /
  // 84 at 1024) but not for large whole ones (2304 of 2304, 162: 84 / 79 at 512, 114 / 101 at 1024).
  const bool small_ok = L->bf16 && !L->square && !L->fine && !(cfg.flags & FASTCLIP_TILES_256);
  // (the kernels address rows by 32-bit byte offsets, number their output tiles in 16 bits and hold the coefficients of a
  // workgroup's local anchors in LDS)
  const int64_t ld_max = cfg.ld_img > cfg.ld_txt ? cfg.ld_img : cfg.ld_txt;
  L->t128 = small_ok && ((cfg.flags & FASTCLIP_TILES_128) ? big_tiles < 192 : big_tiles <= 128) &&
            cfg.B * ld_max < ((int64_t)1 << 30) && cfg.b <= kMaxLocalQ - 128 &&
            2 * ((cfg.b + 63) / 64) * ((cfg.d + 63) / 64) < 32768;
  size_t at = 0;
  auto take = [&](size_t bytes) { size_t o = at; at += round_up(bytes, 256); return o; };
  const size_t fb = sizeof(float) * (size_t)L->bstride;
  if (L->t128) {
    L->nparts = L->gathered ? (int)((cfg.B + 255) / 256) : (int)((cfg.B + 127) / 128);
    L->ldE = (int64_t)round_up((size_t)cfg.B, 64);
    if (!plan_t128(cfg, room, L)) L->t128 = L->out_rows = 0;
  }
  if (L->t128) {
    // planned
  } else if (L->fine) {
    L->nparts = (int)((cfg.B + 127) / 128);
    L->ldE = (int64_t)round_up((size_t)cfg.B, 64);
    // Split of the contraction over its column range, in 64-deep stages.  Cost model in units of one stage time: rounds
    // of 512 workgroups (two per compute unit) x (slice + 6 for the tile's start and end), and with more than one split
    // the finalize kernel: 27 for its launch + 0.02 per split and output tile.  One split needs no finalize kernel.
    const int64_t stages = L->ldE / 64;
    const int64_t tiles = ((cfg.b + 63) / 64) * ((cfg.d + 63) / 64) * 2;
    int64_t best = 1;
    double best_cost = 0.0;
    for (int64_t ns = 1; ns <= kMaxSplit && ns <= stages; ++ns) {
      const int64_t slice = (stages + ns - 1) / ns;
      const int64_t used = (stages + slice - 1) / slice;
      if (used != ns) continue;                                     // every split must get at least one stage
      const int64_t rounds = (tiles * ns + 511) / 512;
      const double cost = (double)rounds * (double)(slice + 6) + (ns > 1 ? 27.0 + 0.02 * (double)tiles * (double)ns : 0.0);
      if (ns == 1 || cost < best_cost) { best = ns; best_cost = cost; }
    }
    L->nsplit = (int)best;
    L->kslice = (stages + best - 1) / best;
  } else if (L->bf16) {
    L->nparts = (int)((cfg.B + kTileContrasts - 1) / kTileContrasts);
    L->ldE = (int64_t)round_up((size_t)cfg.B, 64);
    // Split of the contraction over its column range, and the columns of its output tiles.  A workgroup owns one output
    // tile of 256 rows of one side and `slice` stages; the 256 compute units take the workgroups in rounds.  Cost model in
    // units of the time of one stage of 256 columns: rounds x (slice + 12 for writing the partial tile) + 0.05 per split
    // and output tile for the finalize pass that adds the partial results up.
    // 192 columns, a stage of which takes 0.8 of one of 256, where that leaves less of a row's last tile or of the chip's last
    // round unused.  Steps with 256 / with the chosen 192 columns, us: 4096 of 4096 at 768 131 / 129, at 640 125 / 123, at 576
    // 122 / 112, at 384 105 / 97, at 128 86 / 81; 1024 of 8192 at 768 87.4 / 82.5, at 192 59.5 / 55.1; 512 of 32768 at 768
    // 148 / 126; 2048 of 16384 at 576 196 / 177; 3000 of 3000 at 768 143 / 139; 2560 of 2560 at 960 106 / 95.
    // Gathered state: the strips are twice as much whatever the columns, so a stage of 192 takes as long.
    const int64_t stages = L->ldE / 32;
    int64_t max_split = stages / 8;
    if (max_split > kMaxSplit) max_split = kMaxSplit;
    if (max_split < 1) max_split = 1;
    double best_cost = 0.0;
    // Plans of `cols` columns whose partial results take at most `most` floats (0: any); even: whose splits are all of an even
    // number of stages.
    auto consider = [&](int cols, size_t most, bool even) {
      const double width = cols == 256 || L->gathered ? 1.0 : 0.80;
      const int64_t tiles = ((cfg.b + 255) / 256) * ((cfg.d + cols - 1) / cols) * 2;
      for (int64_t ns = 1; ns <= max_split; ++ns) {
        int64_t slice = (stages + ns - 1) / ns;
        if (even) slice += slice & 1;
        const int64_t used = (stages + slice - 1) / slice;          // splits that really get stages
        const size_t partial = (size_t)used * partial_split_floats(cfg.b, cfg.d, cols);
        if (most && partial > most) break;
        const int64_t rounds = (tiles * used + 255) / 256;
        const double cost = (double)rounds * width * (double)(slice + 12) + 0.05 * (double)tiles * (double)used * (double)cols / 256.0;
        if (best_cost == 0.0 || cost < best_cost) {
          best_cost = cost;
          L->out_cols = cols; L->nsplit = (int)used; L->kslice = slice;
        }
      }
    };
    consider(256, 0, false);
    const size_t most = (size_t)L->nsplit * partial_split_floats(cfg.b, cfg.d, 256);   // 192 columns take no more workspace
    // Gathered state that does not fit the array of fastclip_step_static: longer runs, which some batches fit it with.
    const bool even = L->gathered && room.split_bytes == 0;
    if (even) {
      best_cost = 0.0;
      consider(256, most, true);
    }
    consider(192, most, even);
  } else {
    L->ldE = room.partial_sums ? (int64_t)round_up((size_t)cfg.B, 4) : cfg.B;
    if (L->few) L->nparts = L->nsplit = 1;
    else plan_f32(cfg, room, L);
  }
  if (L->t128 && !L->gathered && !L->wide_strips) {
    // Strips that prepare their anchors save the launch, about 3 us, and take longer by two or four 16-byte loads and LDS reads a
    // lane for every 128 of width, in every round of workgroups.  What that saves of a step, us, by width:
    // 32 anchors a tile, 128 of 1024 1.3 (512), 0.3 (1024), 0.2 (1152), -0.2 (1280), -0.7 (1536), -2.0 (2048), 512 of 512 0.7 (1024),
    // 0.0 (1280), -0.4 (1536); 64 anchors a tile, 128 of 1024 2.6 (256), 2.3 (512), 0.9 (1024), 0.5 (1152), 0.0 (1280), -0.9 (1536), -2.2 (2048), -5.2
    // (3072), 512 of 2048 2.3, 1.8, 0.5, 0.2, -0.3, -1.2, -2.5, -4.8; 128 anchors, 256 of 8192 1.6 (256), 1.4 (768), 0.7 (1152), 0.2
    // (1280), 0.1 (1536), -0.3 (2048), 384 of 4096 1.2 (512), 0.6 (1152), 0.5 (1280), -0.4 (1536); two rounds, 1000 of 4000 1.1
    // (256), 0.2 (448), -0.3 (512), -2.4 (768), 1280 of 2560 1.8, 0.0, 0.0, -0.4 (640); more rounds, no difference up to 384.
    const int64_t rows = strips_t128_anchors(*L), tiles = 2 * ((cfg.b + rows - 1) / rows) * L->nparts;
    L->own_prep = cfg.d <= (tiles <= 256 ? (rows <= 64 ? 1200 : 1400) : (tiles <= 512 ? 480 : 0));
  }
  if (!L->t128) L->fused_state = L->bf16 && fold_forms_state(cfg.b, L->nparts);
  // scalar partials: t128 without the fold leaves those of its finishing waves, eight of a workgroup of 256 anchors or the tiles'
  int64_t out_blocks = 0;
  if (L->t128 && !L->wide) {
    const int64_t of_tiles = t128_finishing_waves(L->out_rows) * ((cfg.b + L->out_rows - 1) / L->out_rows);
    out_blocks = 8 * ((cfg.b + 255) / 256);
    out_blocks = of_tiles > out_blocks ? of_tiles : out_blocks;
  }
  if (!L->bf16 && !L->few) {
    // Strips on 32 x 32 tiles that prepare their anchors save the launch and add the rows' dot products to every workgroup, twice
    // as many where the whole batch is local.  Steps without / so, us: 128 of 1024 at width 128 20.6 / 19.4, at 512 29.6 / 28.4, at
    // 1024 44.9 / 41.3, at 4096 125 / 119, 200 of 2000 at 1536 158 / 158; whole batches 64 at 32 14.7 / 14.4, 448 at 128 23.3 /
    // 22.7, 128 at 512 22.3 / 21.8, 512 at 512 36.6 / 36.5, but 128 at 768 25.9 / 26.5, 256 at 1024 37.6 / 38.4.
    // Two workgroups fit a compute unit; with more than 512, where they would prepare in rounds, it does not pay: 800 of 800 at 96
    // 42.6 / 43.8, 768 of 768 at 512 68.9 / 69.3.
    const int64_t strip_wgs = (L->square ? 1 : 2) * ((cfg.b + 31) / 32) * L->nparts;
    L->own_prep = L->strip_tile == 32 && !L->gathered && (!L->square || cfg.d <= 512) && strip_wgs <= 512;
    // The state phase inside the gradients: on 32 x 32 tiles, two workgroups of which fit a compute unit, where that leaves room for
    // those that finish the anchors (behind 512 others they would come last), and where a workgroup forms the coefficients of at
    // most 1024 of the other side's anchors, those of its slice, from at most 25000 partial sums.  Steps with k_state / so, us: 64 pairs at width 32 18.5 / 15.2,
    // 128 of 128 at 512 26.5 / 22.8, 448 of 448 at 512 (462 workgroups) 37.6 / 33.5, 1024 of 1024 at 64 37.1 / 35.0, 128 of 1024 at
    // 512 34.1 / 30.0; with more than 512 workgroups 512 of 512 at 512 37.2 / 38.5, 768 of 768 at 512 69.1 / 72.4; with 34816 and 68544 partial
    // sums (800 of 800 at 96, 22400: 44.3 / 42.6) 1024 of 2048 at 64 68.2 / 69.6, 1000 of 4000 at 128 153 / 158.
    const int64_t of_slice = L->square ? L->kslice * 64 : (L->kslice * 64 < cfg.b + 63 ? L->kslice * 64 : (cfg.b + 63) / 64 * 64);
    const int64_t tiles = 2 * ((cfg.b + 31) / 32) * ((cfg.d + 31) / 32), finishers = 2 * ((cfg.b + 63) / 64);
    L->grad_state = room.state_rides && L->grad_tile == 32 && of_slice <= kGradAnchors && (of_slice + 64) * L->nparts <= 25000 &&
                    tiles * L->nsplit + finishers <= 512;
  }
  L->nstate_blocks = L->grad_state ? (int)(2 * ((cfg.b + 63) / 64)) : L->fused_state ? (int)(out_blocks ? out_blocks : (cfg.b + 63) / 64) : state_blocks(cfg.b, L->nparts);
  L->diag = take(fb); L->tau1 = take(fb); L->tau2 = take(fb); L->k1 = take(fb); L->k2 = take(fb);
  L->uold1 = take(fb); L->uold2 = take(fb);
  L->sums = take(fb * 4 * (size_t)L->nparts * (!L->bf16 && L->nparts > 1 ? 2 : 1));
  L->c1 = take(fb); L->c2 = take(fb); L->dcoef = take(fb);
  const size_t red_bytes = sizeof(double) * 2 * (size_t)L->nstate_blocks;
  if (L->bf16) L->red = take(red_bytes);
  const size_t esz = L->bf16 ? sizeof(bf16_t) : sizeof(float);
  if (L->bf16) {
    // fragment-ordered strips: anchors padded to whole 256-row tiles
    const size_t rows = round_up((size_t)cfg.b, 256);
    for (int s = 0; s < 2; ++s) L->E[s] = take(esz * rows * (size_t)L->ldE);
    if (L->wide) {     // [nsplit][2 sides][b to 128][d to 128] floats, only with more than one split
      if (L->nsplit > 1)
        L->Opart[0] = take(sizeof(float) * (size_t)L->nsplit * 2 * round_up((size_t)cfg.b, 128) * round_up((size_t)cfg.d, 128));
    } else if (L->t128) {     // arrival counters of the output tiles and of the scalars; [2][tiles][nsplit][64 x 64] floats
      const int64_t tiles = L->nsplit > 1 ? 2 * (L->out_rows / 64) * ((cfg.b + L->out_rows - 1) / L->out_rows) * ((cfg.d + 63) / 64) : 0;
      L->narrived = (int)tiles + 1;
      L->arrived = take(sizeof(unsigned) * (size_t)L->narrived);
      if (L->nsplit > 1) L->Opart[0] = take(sizeof(float) * (size_t)L->nsplit * (size_t)tiles * 64 * 64);
    } else if (L->fine) {     // [nsplit][2 sides][b to 64][d to 64] floats, only with more than one split
      if (L->nsplit > 1)
        L->Opart[0] = take(sizeof(float) * (size_t)L->nsplit * 2 * round_up((size_t)cfg.b, 64) * round_up((size_t)cfg.d, 64));
    } else {
      for (int s = 0; s < 2; ++s)
        L->Opart[s] = take(sizeof(float) * (size_t)L->nsplit * partial_split_floats(cfg.b, cfg.d, L->out_cols));
    }
  } else {
    for (int s = 0; s < 2; ++s) L->E[s] = take(esz * (size_t)cfg.b * (size_t)L->ldE);
    L->red = take(red_bytes);    // behind the strips: a word of four columns that begins in their last row may end here
    if (L->nsplit > 1) {
      const int64_t T = L->grad_tile, tiles = 2 * ((cfg.b + T - 1) / T) * ((cfg.d + T - 1) / T);
      L->narrived = (int)tiles;
      L->Opart[0] = take(sizeof(double) * (size_t)L->nsplit * (size_t)tiles * (size_t)(T * T));
    }
  }
  if (!L->bf16) {
    L->narrived += L->grad_state;
    if (L->narrived) L->arrived = take(sizeof(unsigned) * (size_t)L->narrived);
  }
  if (L->square && L->bf16) L->F[0] = take(esz * round_up((size_t)cfg.b, 256) * (size_t)L->ldE);
  if (L->gathered) {
    L->colp = take(sizeof(float) * 2 * 4 * (size_t)L->ncol);
    if (L->bf16) {
      const size_t rows = round_up((size_t)cfg.b, 256);
      for (int s = 0; s < 2; ++s) L->F[s] = take(esz * rows * (size_t)L->ldE);
    } else {
      for (int s = 0; s < 2; ++s) L->F[s] = take(esz * (size_t)cfg.b * (size_t)L->ldE);
    }
  }
  L->total = at;
}

// A configuration of the fp32 path whose stored strips fit the array of fastclip_step_static fits it whole, so that every such
// configuration is taken there, and with the same layout whichever entry point runs it.  What the step has in its workspace
// for speed alone gives way in this order: the state phase inside the gradients (3 us, by less than 3 KiB), splits as far as their partial results do not fit (a few per cent mostly, at worst
// a quarter: 1000 of 8000 pairs at width 64 take 227 us, 177 with two splits; 2600 of 2600 at width 512 keep their single pass
// and take 577, with three splits 537, without the single pass 1460), then, where the strips alone leave less than the partial
// sums take (the last 5 % below the array's size), the partial sums and the single pass, at two to three times the time.
void make_layout(const fastclip_config& cfg, Layout* L) {
  constexpr int64_t kLimit = FASTCLIP_STATIC_SCRATCH_BYTES;
  make_layout(cfg, Room{INT64_MAX, true, true}, L);
  if (L->bf16 || (int64_t)L->total <= kLimit) return;
  Layout small;
  make_layout(cfg, Room{INT64_MAX, true, false}, &small);
  if ((int64_t)small.total <= kLimit) { *L = small; return; }
  make_layout(cfg, Room{0, true, false}, &small);
  if ((int64_t)small.total <= kLimit) {
    // beside the partial results a split plan has an arrival counter for each of its at most 1024 tiles
    make_layout(cfg, Room{kLimit - (int64_t)small.total - 4096, true, false}, L);
    if ((int64_t)L->total > kLimit) *L = small;
    return;
  }
  make_layout(cfg, Room{0, false, false}, &small);
  if ((int64_t)small.total <= kLimit) *L = small;
}

static fastclip_status run_step(const fastclip_config* cfg, const fastclip_buffers* bufs, void* workspace,
                                size_t workspace_bytes, void* stream, float* phase_ms,
                                const fastclip_tau_update* upd = nullptr, const fastclip_tau_state* tst = nullptr,
                                const Layout* planned = nullptr) {
  fastclip_status st = validate(cfg, bufs);
  if (st != FASTCLIP_OK) return st;
  if (!bufs) return FASTCLIP_ERR_NULL;
  StepCtx c;
  c.cfg = *cfg;
  c.buf = *bufs;
  memset(&c.tau_upd, 0, sizeof(c.tau_upd));
  memset(&c.tau_st, 0, sizeof(c.tau_st));
  if (upd || tst) {
    st = validate_tau_update(cfg->version, upd, tst);
    if (st != FASTCLIP_OK) return st;
    // the step must read the very temperatures that the update writes
    if (cfg->version == FASTCLIP_V2 ? (tst->tau_img != bufs->tau_img || tst->tau_txt != bufs->tau_txt)
                                    : (cfg->version != FASTCLIP_V1 && tst->tau != bufs->tau))
      return FASTCLIP_ERR_VALUE;
    // ... laid out as the step's own state arrays are
    if (cfg->version == FASTCLIP_V2 && (upd->state_stride > 1 ? upd->state_stride : 1) != cfg->state_stride)
      return FASTCLIP_ERR_VALUE;
    if (cfg->version != FASTCLIP_V1) { c.tau_upd = make_tau_upd(*upd); c.tau_st = *tst; }
  }
  if (planned) c.L = *planned;
  else make_layout(*cfg, &c.L);
  if (!workspace) return FASTCLIP_ERR_NULL;
  if (workspace_bytes < c.L.total || ((uintptr_t)workspace & 255)) return FASTCLIP_ERR_WORKSPACE;
  c.ws = (char*)workspace;
  c.s = (hipStream_t)stream;
  (void)hipGetLastError();

  hipEvent_t ev[FASTCLIP_N_PHASES + 1];
  int nev = 0;
  int phase_of[FASTCLIP_N_PHASES];
  auto mark = [&](int phase) {
    if (!phase_ms) return;
    if (nev == 0) { (void)hipEventCreate(&ev[0]); (void)hipEventRecord(ev[0], c.s); nev = 1; }
    if (phase >= 0) { (void)hipEventCreate(&ev[nev]); (void)hipEventRecord(ev[nev], c.s); phase_of[nev - 1] = phase; ++nev; }
  };
  mark(-1);
  if (!c.L.own_prep) { launch_prep(c); mark(FASTCLIP_PHASE_PREP); }
  if (c.L.t128) {
    if (c.L.wide_strips) launch_strips_wide128_bf16(c);
    else launch_strips_t128_bf16(c);
    mark(FASTCLIP_PHASE_STRIPS);
    if (!c.L.fused_state) { launch_state(c); mark(FASTCLIP_PHASE_STATE); }
    if (c.L.wide) {
      launch_fold_bf16(c);                mark(FASTCLIP_PHASE_LOCAL);   // with fused_state: the state phase as well
      launch_contract_wide128_bf16(c);    mark(FASTCLIP_PHASE_CONTRACT);  // outputs and scalars included
    } else {
      launch_contract_t128_bf16(c);       mark(FASTCLIP_PHASE_CONTRACT);  // outputs and scalars (and the state phase) included
    }
    launch_norm_backward(c);
  } else if (c.L.fine) {
    launch_strips_fine_bf16(c);           mark(FASTCLIP_PHASE_STRIPS);
    if (!c.L.fused_state) { launch_state(c); mark(FASTCLIP_PHASE_STATE); }
    launch_fold_bf16(c);                  mark(FASTCLIP_PHASE_LOCAL);   // with fused_state: the state phase as well
    launch_contract_fine_bf16(c);         mark(FASTCLIP_PHASE_CONTRACT);  // outputs and scalars included
    launch_norm_backward(c);
  } else if (c.L.bf16) {
    launch_strips_bf16(c);                mark(FASTCLIP_PHASE_STRIPS);
    if (!c.L.fused_state) { launch_state(c); mark(FASTCLIP_PHASE_STATE); }
    launch_fold_bf16(c);                  mark(FASTCLIP_PHASE_LOCAL);   // with fused_state: the state phase as well
    launch_contract_bf16(c);              mark(FASTCLIP_PHASE_CONTRACT);
    launch_finalize_bf16(c);
    launch_norm_backward(c);
  } else if (c.L.few) {
    launch_strips_f32_few(c);             mark(FASTCLIP_PHASE_STRIPS);
    launch_state(c);                      mark(FASTCLIP_PHASE_STATE);
    launch_grad_f32_few(c);
  } else {
    launch_strips_f32(c);                 mark(FASTCLIP_PHASE_STRIPS);
    if (!c.L.grad_state) { launch_state(c); mark(FASTCLIP_PHASE_STATE); }
    launch_grad_f32(c);
    launch_norm_backward(c);
  }
  // global temperature: stepped once its gradient is complete (V2 was stepped in the state phase)
  if (c.tau_upd.optimizer && c.cfg.version != FASTCLIP_V2) launch_tau_scalar(c.tau_upd, c.tau_st, c.buf.d_tau, c.s);
  mark(FASTCLIP_PHASE_FINALIZE);
  fastclip_status rc = launch_status();
  if (phase_ms) {
    for (int i = 0; i < FASTCLIP_N_PHASES; ++i) phase_ms[i] = 0.0f;
    const hipError_t es = hipStreamSynchronize(c.s);
    if (es != hipSuccess) rc = hip_failed(es);
    for (int i = 0; i + 1 < nev; ++i) {
      float ms = 0.0f;
      if (rc == FASTCLIP_OK && hipEventElapsedTime(&ms, ev[i], ev[i + 1]) == hipSuccess) phase_ms[phase_of[i]] += ms;
    }
    for (int i = 0; i < nev; ++i) (void)hipEventDestroy(ev[i]);
  }
  return rc;
}

// ---- fastclip_step_static: the step's workspace in device memory that the library's code object brings along -------
// One array per GPU (every device that loads the code object holds its own copy at its own address, until the process
// ends).  In host code the array's name is only a handle for hipGetSymbolAddress: the address that kernels and memory
// calls need is looked up once per device, with that device current, and kept.
static __device__ __align__(256) unsigned char scratch[FASTCLIP_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static void* g_scratch_ptr[kMaxDevices];   // device address of `scratch` on device i, nullptr until first used there

static fastclip_status static_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_failed(e);
  if (dev < 0 || dev >= kMaxDevices) return FASTCLIP_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return hip_failed(e != hipSuccess ? e : hipErrorInvalidSymbol);
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return FASTCLIP_OK;
}

}  // namespace fc

extern "C" {

fastclip_status fastclip_step_static(const fastclip_config* cfg, const fastclip_buffers* bufs, void* stream) {
  const fastclip_status st = fc::validate(cfg, bufs);
  if (st != FASTCLIP_OK) return st;
  fc::Layout L;
  fc::make_layout(*cfg, &L);
  // the small tiles without partial results, also for gathered state that is on the 256 x 256 tiles for the time they take; or
  // the longer runs that gathered state on the latter can do with
  if (L.total > (size_t)FASTCLIP_STATIC_SCRATCH_BYTES) fc::make_layout(*cfg, fc::Room{0, true, false}, &L);
  if (L.total > (size_t)FASTCLIP_STATIC_SCRATCH_BYTES) return FASTCLIP_ERR_WORKSPACE;
  void* ws = nullptr;
  const fastclip_status sp = fc::static_scratch(&ws);
  if (sp != FASTCLIP_OK) return sp;
  return fc::run_step(cfg, bufs, ws, (size_t)FASTCLIP_STATIC_SCRATCH_BYTES, stream, nullptr, nullptr, nullptr, &L);
}

size_t fastclip_workspace_bytes(const fastclip_config* cfg) {
  if (fc::validate(cfg, nullptr) != FASTCLIP_OK) return 0;
  fc::Layout L;
  fc::make_layout(*cfg, &L);
  return L.total;
}

fastclip_status fastclip_describe(const fastclip_config* cfg, fastclip_plan* plan) {
  if (!plan) return FASTCLIP_ERR_NULL;
  const fastclip_status st = fc::validate(cfg, nullptr);
  if (st != FASTCLIP_OK) return st;
  fc::Layout L;
  fc::make_layout(*cfg, &L);
  plan->tile = !L.bf16 ? 0 : (L.t128 ? 128 : (L.fine ? 64 : 256));
  plan->single_pass = L.square;
  plan->gathered = L.gathered;
  plan->fused_state = L.fused_state || L.grad_state;
  plan->nsplit = L.nsplit;
  plan->nparts = L.nparts;
  return FASTCLIP_OK;
}

fastclip_status fastclip_validate(const fastclip_config* cfg, const fastclip_buffers* bufs) {
  return fc::validate(cfg, bufs);
}

fastclip_status fastclip_step(const fastclip_config* cfg, const fastclip_buffers* bufs, void* workspace,
                              size_t workspace_bytes, void* stream) {
  return fc::run_step(cfg, bufs, workspace, workspace_bytes, stream, nullptr);
}

fastclip_status fastclip_step_timed(const fastclip_config* cfg, const fastclip_buffers* bufs, void* workspace,
                                    size_t workspace_bytes, void* stream, float* phase_ms) {
  if (!phase_ms) return FASTCLIP_ERR_NULL;
  return fc::run_step(cfg, bufs, workspace, workspace_bytes, stream, phase_ms);
}

fastclip_status fastclip_step_update_tau(const fastclip_config* cfg, const fastclip_buffers* bufs,
                                         const fastclip_tau_update* upd, const fastclip_tau_state* state,
                                         void* workspace, size_t workspace_bytes, void* stream) {
  if (!upd || !state) return FASTCLIP_ERR_NULL;
  return fc::run_step(cfg, bufs, workspace, workspace_bytes, stream, nullptr, upd, state);
}

// blocks of the state phase on its own: one per 128 anchors up to eight per compute unit of the largest part
static int state_phase_blocks(int64_t b) {
  const int tiles = fc::state_blocks(b, 1);
  return tiles < 2048 ? tiles : 2048;
}

size_t fastclip_state_phase_workspace_bytes(int64_t b) {
  if (b < 1 || b > ((int64_t)1 << 24)) return 0;
  return fc::round_up(sizeof(double) * 2 * (size_t)state_phase_blocks(b), 256);
}

fastclip_status fastclip_state_phase(const fastclip_config* cfg, const fastclip_buffers* bufs,
                                     const fastclip_tau_update* upd, const fastclip_tau_state* state,
                                     const float* sums, float* coef, void* workspace, size_t workspace_bytes,
                                     void* stream) {
  // the phase sees the batch only through M = B - 1 and its b anchors: none of the matrix limits of the step apply
  if (!cfg) return FASTCLIP_ERR_NULL;
  if (cfg->struct_size != sizeof(fastclip_config) || cfg->B < 2 || cfg->b < 1 || cfg->N < 1 || cfg->b > cfg->N ||
      cfg->state_stride < 1 || cfg->state_stride > 64)
    return FASTCLIP_ERR_SHAPE;
  if (cfg->version < FASTCLIP_V0 || cfg->version > FASTCLIP_V3 ||
      (cfg->emb_dtype != FASTCLIP_F32 && cfg->emb_dtype != FASTCLIP_BF16))
    return FASTCLIP_ERR_VALUE;
  if (fc::bad_float(cfg->gamma) || fc::bad_float(cfg->eps) || fc::bad_float(cfg->rho) ||
      fc::bad_float(cfg->tau_grad_scale) || !(cfg->gamma > 0.0f && cfg->gamma <= 1.0f) || cfg->eps < 0.0f)
    return FASTCLIP_ERR_VALUE;
  if (cfg->b > ((int64_t)1 << 24) || cfg->B > ((int64_t)1 << 24)) return FASTCLIP_ERR_UNSUPPORTED;
  fastclip_status st = FASTCLIP_OK;
  if (!bufs || !sums || !coef || !workspace) return FASTCLIP_ERR_NULL;
  if (!bufs->idx || !bufs->u_img || !bufs->u_txt || !bufs->loss) return FASTCLIP_ERR_NULL;
  if (cfg->version == FASTCLIP_V2) {
    if (!bufs->tau_img || !bufs->tau_txt || !bufs->d_tau_img || !bufs->d_tau_txt) return FASTCLIP_ERR_NULL;
  } else {
    if (!bufs->tau) return FASTCLIP_ERR_NULL;
    if (cfg->version != FASTCLIP_V1 && !bufs->d_tau) return FASTCLIP_ERR_NULL;
  }
  if ((upd == nullptr) != (state == nullptr)) return FASTCLIP_ERR_NULL;
  fc::TauUpd tu;
  memset(&tu, 0, sizeof(tu));
  fastclip_tau_state ts;
  memset(&ts, 0, sizeof(ts));
  if (upd) {
    st = fc::validate_tau_update(cfg->version, upd, state);
    if (st != FASTCLIP_OK) return st;
    if (cfg->version == FASTCLIP_V2 ? (state->tau_img != bufs->tau_img || state->tau_txt != bufs->tau_txt)
                                    : (cfg->version != FASTCLIP_V1 && state->tau != bufs->tau))
      return FASTCLIP_ERR_VALUE;
    if (cfg->version == FASTCLIP_V2 && (upd->state_stride > 1 ? upd->state_stride : 1) != cfg->state_stride)
      return FASTCLIP_ERR_VALUE;
    if (cfg->version != FASTCLIP_V1) { tu = fc::make_tau_upd(*upd); ts = *state; }
  }
  if (workspace_bytes < fastclip_state_phase_workspace_bytes(cfg->b) || ((uintptr_t)workspace & 255))
    return FASTCLIP_ERR_WORKSPACE;
  (void)hipGetLastError();
  fc::launch_state_phase(*cfg, *bufs, tu, ts, sums, coef, (double*)workspace, state_phase_blocks(cfg->b),
                         (hipStream_t)stream);
  if (tu.optimizer && cfg->version != FASTCLIP_V2) fc::launch_tau_scalar(tu, ts, bufs->d_tau, (hipStream_t)stream);
  return fc::launch_status();
}

fastclip_status fastclip_temperature_update(int32_t version, const fastclip_tau_update* upd,
                                            const fastclip_tau_state* state, const int64_t* idx, int64_t b,
                                            int64_t N, const float* d_tau, const float* d_tau_img,
                                            const float* d_tau_txt, void* stream) {
  const fastclip_status st = fc::validate_tau_update(version, upd, state);
  if (st != FASTCLIP_OK) return st;
  if (version == FASTCLIP_V1) return FASTCLIP_OK;
  (void)hipGetLastError();
  const fc::TauUpd u = fc::make_tau_upd(*upd);
  if (version == FASTCLIP_V2) {
    if (!idx || !d_tau_img || !d_tau_txt) return FASTCLIP_ERR_NULL;
    if (b < 0 || N < 1 || b > N || b > ((int64_t)1 << 31) - 1024) return FASTCLIP_ERR_SHAPE;
    if (b == 0) return FASTCLIP_OK;
    fc::launch_tau_sparse(u, *state, idx, b, d_tau_img, d_tau_txt, (hipStream_t)stream);
  } else {
    if (!d_tau) return FASTCLIP_ERR_NULL;
    fc::launch_tau_scalar(u, *state, d_tau, (hipStream_t)stream);
  }
  return fc::launch_status();
}

fastclip_status fastclip_measure_mfma_ceiling(int32_t workgroups, int32_t iters, void* workspace,
                                              size_t workspace_bytes, void* stream, float* ms, double* stats) {
  if (!workspace || !ms || !stats) return FASTCLIP_ERR_NULL;
  if (workgroups < 1 || workgroups > 4096 || iters < 1 || iters > (1 << 24)) return FASTCLIP_ERR_SHAPE;
  const size_t need = (size_t)workgroups * 8 * 2 * sizeof(uint64_t) + 512 * sizeof(float);
  if (workspace_bytes < need || ((uintptr_t)workspace & 255)) return FASTCLIP_ERR_WORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  uint64_t* out = (uint64_t*)workspace;
  float* sink = (float*)((char*)workspace + (size_t)workgroups * 8 * 2 * sizeof(uint64_t));
  (void)hipGetLastError();
  hipEvent_t e0, e1;
  hipError_t e = hipEventCreate(&e0);
  if (e != hipSuccess) return fc::hip_failed(e);
  e = hipEventCreate(&e1);
  if (e != hipSuccess) { (void)hipEventDestroy(e0); return fc::hip_failed(e); }
  fc::launch_mfma_ceiling(workgroups, iters, out, sink, s);     // untimed: first launch of the kernel
  (void)hipEventRecord(e0, s);
  fc::launch_mfma_ceiling(workgroups, iters, out, sink, s);
  (void)hipEventRecord(e1, s);
  fastclip_status rc = fc::launch_status();
  e = hipStreamSynchronize(s);
  if (e != hipSuccess) rc = fc::hip_failed(e);
  *ms = 0.f;
  if (rc == FASTCLIP_OK && hipEventElapsedTime(ms, e0, e1) != hipSuccess) rc = FASTCLIP_ERR_LAUNCH;
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc != FASTCLIP_OK) return rc;
  // per-wave counters of the timed launch: mean shader cycles and mean 100 MHz ticks of a wave's loop
  const size_t nw = (size_t)workgroups * 8;
  uint64_t* host = (uint64_t*)malloc(nw * 2 * sizeof(uint64_t));
  if (!host) return FASTCLIP_ERR_LAUNCH;
  e = hipMemcpy(host, out, nw * 2 * sizeof(uint64_t), hipMemcpyDeviceToHost);
  if (e != hipSuccess) { free(host); return fc::hip_failed(e); }
  double cyc = 0.0, ticks = 0.0;
  for (size_t i = 0; i < nw; ++i) { cyc += (double)host[2 * i]; ticks += (double)host[2 * i + 1]; }
  free(host);
  cyc /= (double)nw; ticks /= (double)nw;
  stats[0] = (double)workgroups * 8.0 * (double)iters * 8.0 * 32768.0;   // flop of the timed launch
  stats[1] = cyc;                                                       // shader cycles per wave
  stats[2] = ticks > 0.0 ? cyc / (ticks * 10.0) : 0.0;                  // GHz while the loop ran (ticks of 10 ns)
  stats[3] = cyc / ((double)iters * 8.0);                               // cycles per MFMA as one wave sees them
  return FASTCLIP_OK;
}

fastclip_status fastclip_measure_strips(const fastclip_config* cfg, const fastclip_buffers* bufs, void* workspace,
                                        size_t workspace_bytes, void* stream, int32_t ablation, int32_t reps, float* ms,
                                        double* stats) {
  if (!ms || !stats) return FASTCLIP_ERR_NULL;
  fastclip_status st = fc::validate(cfg, bufs);
  if (st != FASTCLIP_OK) return st;
  if (!bufs || !workspace) return FASTCLIP_ERR_NULL;
  if (reps < 1 || reps > 1000) return FASTCLIP_ERR_SHAPE;
  fc::StepCtx c;
  c.cfg = *cfg;
  c.buf = *bufs;
  memset(&c.tau_upd, 0, sizeof(c.tau_upd));
  memset(&c.tau_st, 0, sizeof(c.tau_st));
  fc::make_layout(*cfg, &c.L);
  const size_t ncyc = (size_t)256 * 2 * 4;
  if (workspace_bytes < c.L.total + ncyc * sizeof(uint64_t) || ((uintptr_t)workspace & 255)) return FASTCLIP_ERR_WORKSPACE;
  if (!c.L.bf16 || c.L.fine || c.L.t128 || c.L.square || c.L.gathered) return FASTCLIP_ERR_UNSUPPORTED;
  c.ws = (char*)workspace;
  c.s = (hipStream_t)stream;
  uint64_t* cycles = (uint64_t*)(c.ws + c.L.total);
  (void)hipGetLastError();
  hipError_t e = hipMemsetAsync(cycles, 0, ncyc * sizeof(uint64_t), c.s);
  if (e != hipSuccess) return fc::hip_failed(e);
  fc::launch_prep(c);                                   // s_ii and the temperatures that the epilogue reads
  if (!fc::launch_strips_measure(c, ablation, cycles)) return FASTCLIP_ERR_UNSUPPORTED;   // untimed first launch
  hipEvent_t e0, e1;
  e = hipEventCreate(&e0);
  if (e != hipSuccess) return fc::hip_failed(e);
  e = hipEventCreate(&e1);
  if (e != hipSuccess) { (void)hipEventDestroy(e0); return fc::hip_failed(e); }
  (void)hipEventRecord(e0, c.s);
  for (int i = 0; i < reps; ++i) (void)fc::launch_strips_measure(c, ablation, cycles);
  (void)hipEventRecord(e1, c.s);
  fastclip_status rc = fc::launch_status();
  e = hipStreamSynchronize(c.s);
  if (e != hipSuccess) rc = fc::hip_failed(e);
  *ms = 0.f;
  if (rc == FASTCLIP_OK && hipEventElapsedTime(ms, e0, e1) != hipSuccess) rc = FASTCLIP_ERR_LAUNCH;
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc != FASTCLIP_OK) return rc;
  *ms /= (float)reps;
  uint64_t* host = (uint64_t*)malloc(ncyc * sizeof(uint64_t));
  if (!host) return FASTCLIP_ERR_LAUNCH;
  e = hipMemcpy(host, cycles, ncyc * sizeof(uint64_t), hipMemcpyDeviceToHost);
  if (e != hipSuccess) { free(host); return fc::hip_failed(e); }
  // counters of the last launch: [workgroup][older | younger wave of SIMD 0][total cycles, epilogue cycles, 10 ns ticks, -]
  double tot[2] = {0.0, 0.0}, epi[2] = {0.0, 0.0}, ticks = 0.0;
  int used = 0;
  for (int w = 0; w < 256; ++w) {
    if (!host[(w * 2) * 4]) continue;
    ++used;
    for (int y = 0; y < 2; ++y) { tot[y] += (double)host[(w * 2 + y) * 4]; epi[y] += (double)host[(w * 2 + y) * 4 + 1]; }
    ticks += (double)host[(w * 2) * 4 + 2];
  }
  free(host);
  if (!used) return FASTCLIP_ERR_LAUNCH;
  const double tiles_per_wg = 2.0 * (double)((cfg->b + 255) / 256) * (double)((cfg->B + 255) / 256) / (double)used;
  stats[0] = tot[0] / used;                                 // cycles of the older wave of a SIMD, kernel entry to exit
  stats[1] = tot[1] / used;                                 // ... of the younger wave
  stats[2] = epi[0] / used;                                 // of which between the last stage of a tile and the next tile
  stats[3] = tiles_per_wg * (double)(cfg->d / 64);          // 64-deep stages per workgroup
  stats[4] = ticks > 0.0 ? tot[0] / (ticks * 10.0) : 0.0;   // shader clock in GHz while the kernel ran
  stats[5] = (double)used;                                  // workgroups
  return FASTCLIP_OK;
}

fastclip_status fastclip_normalize_rows(const void* raw, int32_t raw_dtype, int64_t ld_raw, int64_t b, int64_t d,
                                        void* unit, int32_t unit_dtype, int64_t ld_unit, float* norm, void* stream) {
  if (!raw || !unit || !norm) return FASTCLIP_ERR_NULL;
  if (b < 0 || d < 1 || ld_raw < d || ld_unit < d) return FASTCLIP_ERR_SHAPE;
  if ((raw_dtype != FASTCLIP_F32 && raw_dtype != FASTCLIP_BF16) || (unit_dtype != FASTCLIP_F32 && unit_dtype != FASTCLIP_BF16))
    return FASTCLIP_ERR_VALUE;
  if (b > ((int64_t)1 << 31) - 1024 || d > ((int64_t)1 << 24) || ld_raw > ((int64_t)1 << 30) || ld_unit > ((int64_t)1 << 30))
    return FASTCLIP_ERR_UNSUPPORTED;
  if (raw == unit && (raw_dtype != unit_dtype || ld_raw != ld_unit)) return FASTCLIP_ERR_VALUE;
  if (b == 0) return FASTCLIP_OK;
  (void)hipGetLastError();
  fc::launch_normalize_rows(raw, raw_dtype == FASTCLIP_BF16, ld_raw, b, d, unit, unit_dtype == FASTCLIP_BF16, ld_unit, norm,
                            (hipStream_t)stream);
  return fc::launch_status();
}

fastclip_status fastclip_measure_record_rmw(const int64_t* idx, int64_t n, int64_t N, float* records,
                                            int64_t record_floats, void* stream) {
  if (!idx || !records) return FASTCLIP_ERR_NULL;
  if (n < 0 || N < 1 || n > N || n > ((int64_t)1 << 30) || record_floats < 8 || record_floats % 8 ||
      record_floats > 64)
    return FASTCLIP_ERR_SHAPE;
  if ((uintptr_t)records & 31) return FASTCLIP_ERR_UNSUPPORTED;
  if (n == 0) return FASTCLIP_OK;
  (void)hipGetLastError();
  fc::launch_record_rmw(idx, n, records, record_floats, (hipStream_t)stream);
  return fc::launch_status();
}

const char* fastclip_phase_name(int phase) {
  switch (phase) {
    case FASTCLIP_PHASE_PREP: return "prep";
    case FASTCLIP_PHASE_STRIPS: return "strips";
    case FASTCLIP_PHASE_STATE: return "state";
    case FASTCLIP_PHASE_LOCAL: return "local";
    case FASTCLIP_PHASE_CONTRACT: return "contract";
    case FASTCLIP_PHASE_FINALIZE: return "finalize";
    default: return "unused";
  }
}

fastclip_status fastclip_state_update(const int64_t* idx, int64_t n, int64_t N, float gamma, float M,
                                      const float* sum_img, const float* sum_txt, float* u_img, float* u_txt,
                                      float* u_new_img, float* u_new_txt, void* stream) {
  return fastclip_state_update_strided(idx, n, N, 1, gamma, M, sum_img, sum_txt, u_img, u_txt, u_new_img, u_new_txt,
                                       stream);
}

fastclip_status fastclip_state_update_strided(const int64_t* idx, int64_t n, int64_t N, int64_t state_stride,
                                              float gamma, float M, const float* sum_img, const float* sum_txt,
                                              float* u_img, float* u_txt, float* u_new_img, float* u_new_txt,
                                              void* stream) {
  if (!idx || !sum_img || !sum_txt || !u_img || !u_txt || !u_new_img || !u_new_txt) return FASTCLIP_ERR_NULL;
  // the indices are distinct values in [0, N), so there cannot be more than N of them
  if (n < 0 || N < 1 || n > N || n > ((int64_t)1 << 31) - 1024 || state_stride < 1 || state_stride > 64)
    return FASTCLIP_ERR_SHAPE;
  if (fc::bad_float(gamma) || fc::bad_float(M) || !(gamma > 0.0f && gamma <= 1.0f) || !(M > 0.0f))
    return FASTCLIP_ERR_VALUE;
  if (n == 0) return FASTCLIP_OK;
  (void)hipGetLastError();
  fc::launch_state_flat(idx, n, state_stride, gamma, M, sum_img, sum_txt, u_img, u_txt, u_new_img, u_new_txt,
                        (hipStream_t)stream);
  return fc::launch_status();
}

static size_t table_slots(int64_t b) {
  size_t s = 64;
  while (s < (size_t)b * 2) s <<= 1;
  return s;
}

size_t fastclip_check_indices_workspace_bytes(int64_t b) {
  if (b < 0 || b > ((int64_t)1 << 28)) return 0;
  return 256 + table_slots(b) * sizeof(int64_t);
}

fastclip_status fastclip_check_indices(const int64_t* idx, int64_t b, int64_t N, void* workspace,
                                       size_t workspace_bytes, void* stream) {
  if (!idx || !workspace) return FASTCLIP_ERR_NULL;
  if (b < 0 || N < 1 || b > ((int64_t)1 << 28)) return FASTCLIP_ERR_SHAPE;
  if (workspace_bytes < fastclip_check_indices_workspace_bytes(b) || ((uintptr_t)workspace & 255))
    return FASTCLIP_ERR_WORKSPACE;
  if (b == 0) return FASTCLIP_OK;
  hipStream_t s = (hipStream_t)stream;
  (void)hipGetLastError();
  fc::launch_check_indices(idx, b, N, workspace, s);
  int flag = 0;
  if (fc::launch_status() != FASTCLIP_OK) return FASTCLIP_ERR_LAUNCH;
  hipError_t e = hipMemcpyAsync(&flag, workspace, sizeof(int), hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return fc::hip_failed(e);
  e = hipStreamSynchronize(s);
  if (e != hipSuccess) return fc::hip_failed(e);
  return flag ? FASTCLIP_ERR_INDEX : FASTCLIP_OK;
}

float fastclip_gamma_cosine(int64_t t, int64_t iters_per_epoch, int64_t decay_epochs, float gamma_min) {
  if (iters_per_epoch < 1) iters_per_epoch = 1;
  if (t < 0) t = 0;
  const int64_t epoch = t / iters_per_epoch;
  if (decay_epochs < 1 || epoch >= decay_epochs) return gamma_min;
  const double c = cos(M_PI * (double)epoch / (double)decay_epochs);
  return (float)(0.5 * (1.0 + c) * (1.0 - (double)gamma_min) + (double)gamma_min);
}

const char* fastclip_last_hip_error(void) { return hipGetErrorString(fc::g_last_hip_error); }

const char* fastclip_status_string(fastclip_status s) {
  switch (s) {
    case FASTCLIP_OK: return "ok";
    case FASTCLIP_ERR_NULL: return "a required pointer is NULL";
    case FASTCLIP_ERR_SHAPE: return "invalid shape or struct_size";
    case FASTCLIP_ERR_VALUE: return "invalid scalar, version or dtype";
    case FASTCLIP_ERR_WORKSPACE: return "workspace too small or misaligned";
    case FASTCLIP_ERR_UNSUPPORTED: return "unsupported size or alignment";
    case FASTCLIP_ERR_LAUNCH: return "HIP runtime error";
    case FASTCLIP_ERR_INDEX: return "index out of range or repeated";
    default: return "unknown status";
  }
}

}  // extern "C"
