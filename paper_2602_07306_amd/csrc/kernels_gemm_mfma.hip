// Chooses the tile configuration of the MFMA GEMM family by shape and dispatches to the kernels, which are
// instantiated per epilogue in kernels_gemm_mfma_{store,residual,swiglu,qkv_a..d,qkv_rows_a..c}.hip from gemm_mfma_impl.h.
#include <algorithm>

#include "pt_device.h"

template <int EPI, int CFG>
int pt_gemm_mfma_launch_one(const pt_gemm_args& g, hipStream_t s);

template <int EPI>
static int launch_epi(const pt_gemm_args& g, hipStream_t s, int cfg) {
  switch (cfg) {
    case 0: return pt_gemm_mfma_launch_one<EPI, 0>(g, s);
    case 1: return pt_gemm_mfma_launch_one<EPI, 1>(g, s);
    case 2: return pt_gemm_mfma_launch_one<EPI, 2>(g, s);
    case 3: return pt_gemm_mfma_launch_one<EPI, 3>(g, s);
    case 4: return pt_gemm_mfma_launch_one<EPI, 4>(g, s);
    case 5: return pt_gemm_mfma_launch_one<EPI, 5>(g, s);
    case 6: return pt_gemm_mfma_launch_one<EPI, 6>(g, s);
    case 7: return pt_gemm_mfma_launch_one<EPI, 7>(g, s);
    case 8: return pt_gemm_mfma_launch_one<EPI, 8>(g, s);
    case 9: return pt_gemm_mfma_launch_one<EPI, 9>(g, s);
    case 10: return pt_gemm_mfma_launch_one<EPI, 10>(g, s);
    default: return pt_gemm_mfma_launch_one<EPI, 11>(g, s);
  }
}

#define GM_BK 64

// Tile configuration override for tuning runs (pt_set_tuning): -1 = choose by shape.
int pt_tune_gemm_cfg = -1;

#define GM_NCFG 12
static const int kWaveN[GM_NCFG] = {128, 64, 64, 64, 128, 64, 128, 128, 128, 64, 128, 128};   // columns per wavefront

static bool cfg_fits(const pt_gemm_args& g, int cfg) {
  const int wn = kWaveN[cfg];
  if (g.epi == EPI_SWIGLU) return g.N % 64 == 0 && wn % 64 == 0;
  if (g.epi == EPI_QKV) {
    // every wavefront owns whole heads; the q / k / v sections start on wavefront borders
    if (g.hd != 64 && g.hd != 128) return false;
    return wn % g.hd == 0 && (g.H * g.hd) % wn == 0 && (g.Hkv * g.hd) % wn == 0;
  }
  return true;
}

// Expected time in us of a GEMM on tile configuration 0 (256 x 256), 2 (128 x 128) or 4 (128 x 256).  0 and 4 run in
// rounds of one tile per compute unit, each with an epilogue and a part per K step of 64, both longer the more of the chip
// works (`full`); the tiles of 2 share their unit two at a time.  Fitted inside the Mid model (4 tracks, K = 1024 and 4096;
// us, measured 0 / 2): gate/up 100 rows 30 / 20, 512 33 / 42, 600 50 / 50, 1000 56 / 73, 4096 202 / 271; QKV 512 30 / 27, 1000
// 36 / 41, 1300 58 / 51, 4096 88 / 125; out 1000 33 / 20, 3000 47 / 49, 4096 57 / 65; down 1000 77 / 44, 2000 83 / 73, 4096
// 113 / 150; head 300 41 / 44, 1000 72 / 98; the residual terms were fitted on an epilogue that took 1 to 7 us longer).  It
// orders them correctly there but for down around 1500 rows (4 takes 65 of its 70) and for Large (8 tracks, 512 rows: gate/up
// 195 / 282, out 62 / 53) and the one-GPU share (512 rows: gate/up 325 / 440, down 476 / 278).  4 wins where one round of it
// takes a residual GEMM that leaves 0 half empty and fills 2 twice (Mid down 1300 rows 59 against 76 / 71, Large down 512
// 139 against 171 / 164) and for QKV of few rows with heads of 128, too wide for a wavefront of 2 (Large 96 rows 48 / 56).
static double tile_us(const pt_gemm_args& g, int cfg) {
  const int bm = cfg == 0 ? 256 : 128, bn = cfg == 2 ? 128 : 256;
  const int64_t tiles = (int64_t)((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn) * g.batch;
  const double steps = (double)g.K / GM_BK;
  const int64_t n_cu = pt_device_cus();
  const double rounds = (double)((tiles + n_cu - 1) / n_cu), full = std::min(1.0, (double)tiles / n_cu);
  const bool res = g.epi == EPI_RESIDUAL, swiglu = g.epi == EPI_SWIGLU, qkv = g.epi == EPI_QKV;
  if (cfg == 0) return 8.0 + rounds * ((res ? 10.6 + 18.0 * full : swiglu ? 5.0 : 9.0) + (0.9 + 0.3 * full) * steps);
  if (cfg == 4) return rounds * (12.4 + (res ? 6.0 + 10.0 * full : 0.0) + 0.735 * steps) * (rounds > 1 ? 1.13 : 1.0);
  return 10.0 + rounds * ((res ? 5.3 : swiglu ? 0.5 : qkv ? 1.5 : 4.3) + 0.48 * steps);
}

// Grouped GEMM.  Above 32 rows in an average group: the largest tile, also where a group fills a small part of it.  Group
// sizes scatter, each tile past a group's first re-reads its weights, and the reads of the weights are the time: 4 tracks
// x 8 experts of width 2048 on K = 1024, gate/up and down in us with 256 rows: 106 + 58 (256 x 256) against 109 + 73
// (128 x 256), 175 + 82 (64 x 256) and 158 + 77 (32 x 256); 512 rows: 106 + 58 against 126 + 73 (128 x 256).
// With fewer rows a tile is nearly empty and its fixed cost counts.  gate/up: 256 x 256 still wins where a group's weights
// take long to read (same experts, 96 rows: 90 against 106 and 170; 8 tracks x 64 experts of width 256 on K = 2048: 277
// against 302 and 362), 32 x 256 where they are small and tiles fill the chip at least once (4 tracks on K = 1024, 96
// rows: 64 experts of width 256 111 against 120 us, 32 of width 512 108 against 115, 16 of 512 66 against 71; not with
// 64 of width 512, 198 against 189).  down: 32 x 256 under the same condition (64 experts of width 256: 90 against 113;
// 32 of 256: 53 against 64), else 128 x 256 (8 experts of width 2048: 48 against 57; 16 of 1024: 54 against 75; 8 tracks
// x 32 of 1024 on width 2048: 386 against 438).
static int choose_grouped(const pt_gemm_args& g) {
  if (g.grp_rows > 0 && g.grp_rows <= 32) {
    const int64_t weights = (int64_t)g.N * g.K;   // elements of a group's matrix
    const int64_t tiles = (int64_t)g.n_groups * g.batch * ((g.N + 255) / 256);
    const bool small = weights <= 512 * 1024 || (g.epi == EPI_SWIGLU && weights <= 1024 * 1024 && tiles <= 2 * pt_device_cus() && g.grp_rows <= 24);
    if (g.K <= 1024 && small && tiles >= pt_device_cus() && cfg_fits(g, 5)) return 5;
    if (g.epi == EPI_STORE_F32) return 4;
  }
  return cfg_fits(g, 0) ? 0 : -1;
}

// The tile configuration for a problem, or -1 if the family does not cover it (-2: nothing to do).
static int choose_cfg(const pt_gemm_args& g) {
  if (g.dtype != PT_BF16) return -1;
  if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return -2;
  if (g.K < 2 * GM_BK || g.K % (2 * GM_BK)) return -1;
  if ((g.lda & 7) || (g.ldb & 7) || (g.a_bstride & 7) || (g.w_bstride & 7)) return -1;
  if (((uintptr_t)g.A | (uintptr_t)g.W) & 15) return -1;
  if (g.blk_group && ((g.w_gstride & 7) || (g.M & 255))) return -1;   // expert segments are whole 256-row tiles
  if (g.a_rows && (g.a_bstride ? g.a_bstride : (int64_t)g.M * g.lda) * 2 >= ((int64_t)1 << 32)) return -1;   // 32-bit gather offsets
  if ((g.epi == EPI_STORE_F32 || g.epi == EPI_RESIDUAL) &&
      ((g.ldo & 3) || (g.N & 3) || (g.out_bstride & 3) || (g.res_bstride & 3) || (((uintptr_t)g.out | (uintptr_t)g.res) & 15))) return -1;
  if (g.epi == EPI_SWIGLU && ((g.olp_bstride & 7) || ((uintptr_t)g.olp & 15))) return -1;
  if (pt_tune_gemm_cfg >= 0 && pt_tune_gemm_cfg < GM_NCFG) return cfg_fits(g, pt_tune_gemm_cfg) ? pt_tune_gemm_cfg : -1;
  static const int m64[] = {3, 6, -1}, m32[] = {5, 7, -1};
  if (g.blk_group) return choose_grouped(g);
  if (g.M <= 64) {
    for (const int* c = g.M <= 32 ? m32 : m64; *c >= 0; ++c)
      if (cfg_fits(g, *c)) return *c;
    return -1;
  }
  // One tile of rows and more than three rounds of 2 at one tile per compute unit: the weights' way from HBM is the time, and 4
  // has most of them in flight while K is long (gate/up of 8 tracks, us on 4 / on 2: K = 2048, 832 tiles of 2, 96 rows 98 / 98, 128
  // rows 100 / 104; 960 tiles 107 / 108 and 110 / 114; 1024 (Large) 112 / 112 and 115 / 119; K = 4096, 960 tiles 192 / 202 and 197 /
  // 208.  Not at K = 1024: 960 tiles 59 / 56 and 60 / 59, 1024 tiles 62 / 57 and 62 / 60; and not in three rounds: K = 2048, 768
  // tiles 93 / 85 and 96 / 89).
  if (g.M <= 128 && g.K >= 2048 && (int64_t)((g.N + 127) / 128) * g.batch > 3 * (int64_t)pt_device_cus() && cfg_fits(g, 4)) return 4;
  int best = -1;
  double best_us = 1e30;
  for (int cfg : {0, 4, 2}) {
    const double us = cfg_fits(g, cfg) ? tile_us(g, cfg) : 1e30;
    if (us < best_us) { best_us = us; best = cfg; }
  }
  return best;
}

bool pt_gemm_mfma_covers(const pt_gemm_args& g) { return choose_cfg(g) >= 0; }

// Blocks of 32 rows inside one sequence, at positions from a multiple of 8 on.
static bool qkv_blocks_aligned(const pt_gemm_args& g) {
  return (g.row_map ? g.row_blocks != 0 : (g.S & 31) == 0) && (g.pos0 & 7) == 0;
}

// Configurations whose tile is at least 128 x 128 run the LDS-staged residual epilogue, which can also emit the
// scaled bf16 copy and the per-row sums of squares; one block of sums per wavefront column range.
int pt_gemm_mfma_fold_parts(const pt_gemm_args& g) {
  const int cfg = choose_cfg(g);
  // the square tiles, except the large one's QKV form for rows of any place
  if (g.epi == EPI_QKV || g.epi == EPI_SWIGLU)
    return cfg == 2 || (cfg == 0 && (g.epi == EPI_SWIGLU || qkv_blocks_aligned(g))) ? (int)PT_NF_MAX_SUMS : 0;
  if (g.epi != EPI_RESIDUAL) return 0;
  static const bool staged[GM_NCFG] = {true, true, true, false, true, false, false, false, true, true, true, true};
  if (cfg < 0 || !staged[cfg] || g.N % kWaveN[cfg]) return 0;
  return g.N / kWaveN[cfg];
}

// Residual GEMMs whose tiles leave compute units idle: every K slice is a launch's worth of tiles more, and the kernel
// that normalises adds the slices to the residual stream (it would run anyway).  The slices cost their traffic, taken at
// 4 TB/s.  Inside the models, out + down projection + normalising kernel in us a layer, without slices / as chosen: Mid (4 tracks,
// width 1024) 96 rows 16.6 + 39.4 + 1.5 / 11.4 + 17.2 + 14.6, 300 rows 16.1 + 35.8 + 6.2 / 16.6 + 22.2 + 9.4; Large (8 x 2048) 96 rows
// 29.5 + 83.7 + 16.1 / 22.2 + 58.9 + 20.1; one-GPU share (1 x 8192) 128 rows 78 + 279 + 29 / 41 + 100 + 41, 384 rows 81 + 281 + 37 /
// 82 + 208 + 46.
// What bounds a slice is the latency of its few K steps' weights on their way from HBM, hence estimates of their own, for
// either side.  They are fitted on 128 x 128 tiles staged through registers, which took longer; with the present ones they
// still choose no slices that cost more than none at 65 to 700 rows of these models and of a dense one of width 8192, but too
// few in places (Mid 256 rows, out projection not cut: a layer 99 us against 97 with four slices of both; Large 128 rows 284
// against 280; share 384 rows 840 against 834).
static double slice_us(const pt_gemm_args& g, int cfg, int slices) {
  const int bm = cfg == 0 ? 256 : 128, bn = cfg == 2 ? 128 : 256;
  const int64_t tiles = (int64_t)((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn) * g.batch * slices;
  const double steps = (double)g.K / (slices * GM_BK);
  const int64_t n_cu = pt_device_cus();
  const double rounds = (double)((tiles + n_cu - 1) / n_cu);
  if (cfg == 0) return rounds * (16.7 + 1.02 * steps);
  if (cfg == 4) return rounds * (12.4 + 0.735 * steps);
  return 9.5 + rounds * 0.585 * steps;
}

int pt_gemm_mfma_ksplit(const pt_gemm_args& g) {
  const int cfg = choose_cfg(g);
  if (cfg < 0 || g.epi != EPI_RESIDUAL || g.blk_group || !g.sk_part || ((uintptr_t)g.sk_part & 15) || pt_tune_gemm_cfg >= 0) return 1;
  const double traffic_us = (double)g.batch * g.M * g.N * 8.0 / 4e6;   // a slice written and read once
  double best_us = 1e30;
  for (int c : {0, 4, 2}) best_us = std::min(best_us, slice_us(g, c, 1));
  int best = 1;
  for (int slices = 2; slices <= 16; slices *= 2) {
    if (g.K % (slices * 2 * GM_BK) || (int64_t)slices * g.batch * g.M * g.N > g.sk_part_floats) break;
    const double us = slice_us(g, 2, slices) + slices * traffic_us;
    if (us < 0.9 * best_us) { best_us = us; best = slices; }
  }
  return best;
}

int pt_launch_gemm_mfma_split(const pt_gemm_args& g, int slices, hipStream_t s) {
  return launch_epi<EPI_STORE_F32>(pt_gemm_slices(g, slices), s, 2);
}

// The tile kernels with an LDS-staged QKV epilogue assume 32-row blocks inside one sequence at positions from a multiple
// of 8 on; any other rows run the form that looks up every row's place.
static int launch_qkv(const pt_gemm_args& g, hipStream_t s, int cfg) {
  if (qkv_blocks_aligned(g)) return launch_epi<EPI_QKV>(g, s, cfg);
  switch (cfg) {
    case 0: return pt_gemm_mfma_launch_one<EPI_QKV_ROWS, 0>(g, s);
    case 1: return pt_gemm_mfma_launch_one<EPI_QKV_ROWS, 1>(g, s);
    case 2: return pt_gemm_mfma_launch_one<EPI_QKV_ROWS, 2>(g, s);
    case 4: return pt_gemm_mfma_launch_one<EPI_QKV_ROWS, 4>(g, s);
    case 8: return pt_gemm_mfma_launch_one<EPI_QKV_ROWS, 8>(g, s);
    case 9: return pt_gemm_mfma_launch_one<EPI_QKV_ROWS, 9>(g, s);
    case 10: return pt_gemm_mfma_launch_one<EPI_QKV_ROWS, 10>(g, s);
    case 11: return pt_gemm_mfma_launch_one<EPI_QKV_ROWS, 11>(g, s);
    default: return launch_epi<EPI_QKV>(g, s, cfg);   // tiles without a staged epilogue: one form for all rows
  }
}

int pt_launch_gemm_mfma(const pt_gemm_args& g, hipStream_t s) {
  const int cfg = choose_cfg(g);
  if (cfg == -2) return 1;
  if (cfg < 0) return 0;
  if (g.nf_out && g.nf_parts != pt_gemm_mfma_fold_parts(g))
    return pt_set_error(PT_ERR_INVALID_ARGUMENT, "folded RMSNorm asked of a GEMM configuration that cannot emit it");
  if (!g.nf_out && g.nf_parts > 0 && (g.nf_parts > pt_gemm_mfma_fold_parts(g) || (g.nf_parts & 3) || (g.nf_ss_bstride & 3) || ((uintptr_t)g.nf_ss & 15)))
    return pt_set_error(PT_ERR_INVALID_ARGUMENT, "row sums handed to a GEMM configuration that cannot add them up");
  switch (g.epi) {
    case EPI_STORE_F32: return launch_epi<EPI_STORE_F32>(g, s, cfg);
    case EPI_RESIDUAL: return launch_epi<EPI_RESIDUAL>(g, s, cfg);
    case EPI_SWIGLU: return launch_epi<EPI_SWIGLU>(g, s, cfg);
    case EPI_QKV: return launch_qkv(g, s, cfg);
  }
  return 0;
}
