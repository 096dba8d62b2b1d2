// Host side of the Accordion hot-path library: configuration checks, workspace layout,
// tile tables, the step state machine and the kernel launches.  The C ABI is declared and
// documented in include/accordion.h.
#include "../../include/accordion.h"

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "acc_common.h"
#include "acc_powersgd.h"
#include "acc_regime.h"
#include "acc_topk.h"
#include "acc_batch.h"

using namespace acc;

namespace {

thread_local char g_init_error[256] = "no error";

inline int64_t align_up(int64_t v, int64_t a) { return (v + a - 1) / a * a; }

struct Region { int64_t off = 0, bytes = 0; };

// Everything that follows from the configuration alone (no GPU needed).
struct Plan {
  std::vector<LayerDev> layers;
  std::vector<FlatTile> ftiles;
  std::vector<MatTile> mtiles, qmtiles;
  std::vector<QTile> qtiles;
  std::vector<PTile> ptiles;
  std::vector<int32_t> vectiles;
  std::vector<int32_t> matlayers;
  int32_t rmax = 0;
  int32_t pmean_in_orth = 0, q_stream = 0;   // PowerSGD: see Ws, QStream
  bool u_stream = false;   // PowerSGD: unaligned rows are streamed (kUStreamBytes), where they are more than a sixteenth
  int32_t mrows = kMatRows, qrows = kQRows;   // PowerSGD: rows of the two kinds of matrix tiles
  int64_t N = 0, e_stride = 0;
  int64_t q_total = 0;   // floats of Q in the caller's layout (rows of rmax floats)
  int64_t q_dev = 0;     // floats of Q on the device: every row padded to kMaxRank floats
  int64_t p_total = 0, ppart_stride = 0, qpart_stride = 0, vec_total = 0;
  int64_t pay_stride = 0, q_stride = 0;
  int64_t n_t2slots = 0;    // TopK: slots of level-2 counts per worker (see t2_group_shift)
  bool pick3_big = false;   // TopK: some layer has more quarters than the small last pick kernel takes
  // workspace regions
  Region r_layers, r_ftiles, r_mtiles, r_qmtiles, r_qtiles, r_ptiles, r_vectiles, r_matlayers;
  Region r_level, r_norm_old, r_norm_prev, r_norm_curr, r_has_old, r_rank_used, r_words;
  Region r_A, r_e, r_norm_part, r_norm_part_m, r_afresh, r_sq_part, r_bstate;
  int64_t n_model = 0;   // elements that belong to a layer
  Region r_Q, r_Phat, r_Pwork, r_Ppart, r_Qpart, r_vecmean, r_pending;
  Region r_hist1, r_t2, r_qlist, r_sel, r_hist2m, r_lflag, r_b1hist, r_guess, r_qinfo, r_candval, r_candidx, r_gtq, r_eqq, r_gtpre, r_eqpre, r_payidx, r_payval, r_overlap, r_tpending;
  int64_t total_bytes = 0;
};

int fail(char* buf, int code, const char* msg) {
  std::snprintf(buf, 256, "%s", msg);
  return code;
}

// Rows of the matrix tiles.  A wave has a few rows in flight and waits for the first of them, so few tall
// tiles leave the chip idle and many flat ones spend their time on their own start (a tile's rows of Q, the
// sums of its columns).  First pass and decompression: 32 rows, 16 up to kFlatTileGroups workgroups (with the fused
// update on ResNet-18 shapes at W = 1, 1476 workgroups: a step 105.8 us at 32, 103.5 at 16; VGG-19 shapes at W = 1,
// 2626: 113.3 and 114.4; ResNet-18 at W = 4: 172.2 at 32, 180.8 at 64).  Right product: 128 rows, fewer while that leaves
// compute units without a workgroup (four small layers, 56 workgroups: a step 29.9 us at 128, 28.7 at 64, 28.8 at 32;
// ResNet-18 at W = 1 with the fused update, 356: 103.4 at 128, 105.3 at 64: twice the partial sums).  The workgroups
// counted are those of the whole step's launches, all workers in one: the tiles of the decompression, which runs once for
// all of them, and of the call-by-call path, one worker per launch, are the same ones, as the partial sums and the norms'
// tiles have to be.  (Call by call against 64- and 128-row tiles throughout: four small layers at W = 16 219 us a step and
// 436, odd sizes at W = 3 151 and 194, ResNet-18 shapes at W = 4 212 and 232, VGG-19 shapes at W = 8 664 and 781, the
// loops' share included.)
constexpr int kComputeUnits = 256;
constexpr int kFlatTileGroups = 8 * kComputeUnits;
constexpr int kOrthLoads = 24;   // three requests of kPartLoads; see make_plan_tiled

void choose_tiling(const acc_config* c, Plan& p) {
  auto workgroups = [&](int rows) {
    int64_t n = 0;
    for (int i = 0; i < c->n_layers; ++i) {
      const acc_layer& l = c->layers[i];
      if (l.is_matrix) n += (int64_t)((l.cols + kMatCols - 1) / kMatCols) * ((l.rows + rows - 1) / rows);
    }
    return n * c->n_workers;
  };
  p.mrows = workgroups(32) <= kFlatTileGroups ? 16 : 32;
  while (p.qrows > 32 && workgroups(p.qrows) < kComputeUnits) p.qrows /= 2;
}

// PowerSGD's tiles in the order in which workgroups take them (tile_of_block; in the tables, so that small sets pay nothing for it).
void run_order(std::vector<MatTile>& tiles) {
  const std::vector<MatTile> in_order = tiles;
  for (size_t b = 0; b < tiles.size(); ++b) tiles[b] = in_order[(size_t)tile_of_block((int)b, (int)tiles.size())];
}

// coarse: the tallest tiles, which need the least workspace.
int make_plan_tiled(const acc_config* c, Plan& p, char* err, bool coarse) {
  if (!c) return fail(err, ACC_EINVAL, "config is NULL");
  if (c->method != ACC_POWERSGD && c->method != ACC_TOPK && c->method != ACC_BATCH)
    return fail(err, ACC_EINVAL, "unknown method");
  if (c->n_layers <= 0 || c->n_layers > (1 << 20)) return fail(err, ACC_EINVAL, "n_layers out of range");
  if (!c->layers) return fail(err, ACC_EINVAL, "layers is NULL");
  if (c->n_workers < 1 || c->n_workers > ACC_MAX_WORKERS) return fail(err, ACC_EINVAL, "n_workers out of range");
  if (c->n_params <= 0 || c->n_params > (int64_t(1) << 40)) return fail(err, ACC_EINVAL, "n_params out of range");
  if (!(c->eta >= 0.0f) || !std::isfinite(c->eta)) return fail(err, ACC_EINVAL, "eta must be finite and >= 0");
  if (c->initial_level != 0 && c->initial_level != 1) return fail(err, ACC_EINVAL, "initial_level must be 0 or 1");
  if (c->detector != ACC_DETECT_NORM && c->detector != ACC_DETECT_MSDR) return fail(err, ACC_EINVAL, "unknown detector");
  if (c->detector == ACC_DETECT_MSDR && c->method == ACC_BATCH)
    return fail(err, ACC_EINVAL, "the MSDR detector is not available in batch-size mode");
  if (c->detector == ACC_DETECT_MSDR && !(c->eta < 1.0f)) return fail(err, ACC_EINVAL, "MSDR detector: eta must be below 1");
  if (c->method == ACC_POWERSGD) {
    if (c->rank_crit < 1 || c->rank_crit > ACC_MAX_RANK || c->rank_noncrit < 1 || c->rank_noncrit > ACC_MAX_RANK)
      return fail(err, ACC_EINVAL, "rank out of [1, ACC_MAX_RANK]");
  } else if (c->method == ACC_BATCH) {
    if (c->batch_multiplier < 1 || c->batch_multiplier > ACC_MAX_BATCH_MULTIPLIER)
      return fail(err, ACC_EINVAL, "batch_multiplier out of [1, ACC_MAX_BATCH_MULTIPLIER]");
    if (c->batch_monotone != 0 && c->batch_monotone != 1) return fail(err, ACC_EINVAL, "batch_monotone must be 0 or 1");
  } else {
    if (c->k_den < 1 || c->k_num_crit < 1 || c->k_num_noncrit < 1 || c->k_num_crit > c->k_den ||
        c->k_num_noncrit > c->k_den)
      return fail(err, ACC_EINVAL, "k fraction out of (0, 1]");
  }
  const int nl = c->n_layers;
  // layers: positive shapes, inside the flat buffer, pairwise disjoint
  std::vector<std::pair<int64_t, int64_t>> spans;
  spans.reserve(nl);
  for (int i = 0; i < nl; ++i) {
    const acc_layer& l = c->layers[i];
    if (l.rows < 1 || l.cols < 1) return fail(err, ACC_EINVAL, "layer with rows < 1 or cols < 1");
    if (l.is_matrix != 0 && l.is_matrix != 1) return fail(err, ACC_EINVAL, "is_matrix must be 0 or 1");
    const int64_t n = (int64_t)l.rows * l.cols;
    if (n >= (int64_t(1) << 31)) return fail(err, ACC_EINVAL, "layer has 2^31 or more elements");
    if (l.offset < 0 || l.offset + n > c->n_params) return fail(err, ACC_EINVAL, "layer outside [0, n_params)");
    spans.emplace_back(l.offset, l.offset + n);
  }
  std::sort(spans.begin(), spans.end());
  for (size_t i = 1; i < spans.size(); ++i)
    if (spans[i].first < spans[i - 1].second) return fail(err, ACC_EINVAL, "layers overlap");

  p.N = c->n_params;
  p.e_stride = align_up(p.N, 64);
  p.rmax = (c->method == ACC_POWERSGD) ? std::max(c->rank_crit, c->rank_noncrit) : 0;
  p.layers.resize(nl);
  if (c->method == ACC_POWERSGD && !coarse) choose_tiling(c, p);
  int64_t ntile = 0, orth_loads = 0;   // orth_loads: most partial sums of P that a thread of the orthogonalisation would add
  int64_t aligned_rows = 0;            // elements of the matrix layers whose rows are aligned
  for (int i = 0; i < nl; ++i) {
    const acc_layer& l = c->layers[i];
    LayerDev& d = p.layers[i];
    std::memset(&d, 0, sizeof(d));
    const int64_t n = (int64_t)l.rows * l.cols;
    d.offset = l.offset;
    d.rows = l.rows;
    d.cols = l.cols;
    d.is_matrix = (c->method == ACC_POWERSGD && l.is_matrix) ? 1 : 0;
    d.vec4 = (l.offset % 4 == 0 && l.cols % 4 == 0) ? 1 : 0;
    d.tile0 = (int32_t)ntile;
    d.ntiles = (int32_t)((n + kTile - 1) / kTile);
    d.qoff = 4 * (int64_t)d.tile0 + i;
    for (int t = 0; t < d.ntiles; ++t) {
      FlatTile ft;
      ft.layer = i;
      ft.start = t * kTile;
      ft.count = (int32_t)std::min<int64_t>(kTile, n - (int64_t)t * kTile);
      ft.qslot0 = (int32_t)(d.qoff + 4 * (int64_t)t);
      p.ftiles.push_back(ft);
    }
    ntile += d.ntiles;
    if (4 * (int64_t)d.ntiles > kLdsQuarters) p.pick3_big = true;
    d.t2slot0 = (int32_t)p.n_t2slots;
    p.n_t2slots += ((d.ntiles - 1) >> t2_group_shift(d.ntiles)) + 1;
    p.n_model += n;
    if (ntile > (int64_t(1) << 30)) return fail(err, ACC_EINVAL, "too many tiles");
    if (c->method == ACC_POWERSGD) {
      if (d.is_matrix) {
        const int cap = std::min(l.rows, l.cols);
        d.rank[0] = std::max(1, std::min(c->rank_noncrit, cap));
        d.rank[1] = std::max(1, std::min(c->rank_crit, cap));
        d.n_colchunks = (l.cols + kMatCols - 1) / kMatCols;
        d.mt0 = (int32_t)p.mtiles.size();
        if (d.vec4) aligned_rows += n;
        const int n_rb = (l.rows + p.mrows - 1) / p.mrows;
        d.n_rowblocks = (l.rows + p.qrows - 1) / p.qrows;
        d.q_off = p.q_dev;
        p.q_total += (int64_t)l.cols * p.rmax;
        p.q_dev += (int64_t)l.cols * kMaxRank;
        d.p_off = p.p_total;
        p.p_total += (int64_t)l.rows * p.rmax;
        d.ppart_off = p.ppart_stride;
        p.ppart_stride += (int64_t)d.n_colchunks * l.rows * p.rmax;
        d.qpart_off = p.qpart_stride;
        p.qpart_stride += (int64_t)d.n_rowblocks * l.cols * p.rmax;
        p.matlayers.push_back(i);
        for (int rb = 0; rb < d.n_rowblocks; ++rb)
          for (int cc = 0; cc < d.n_colchunks; ++cc) p.qmtiles.push_back(MatTile{i, rb * p.qrows, cc * kMatCols, 0});
        for (int rb = 0; rb < n_rb; ++rb)
          for (int cc = 0; cc < d.n_colchunks; ++cc) {
            MatTile mt;
            mt.layer = i;
            mt.row0 = rb * p.mrows;
            mt.col0 = cc * kMatCols;
            mt.id = (int32_t)p.mtiles.size();
            p.mtiles.push_back(mt);
          }
        for (int r0 = 0; r0 < l.rows; r0 += kPmeanRows) p.ptiles.push_back(PTile{i, r0});
        for (int cc = 0; cc < d.n_colchunks; ++cc) p.qtiles.push_back(QTile{i, cc * kMatCols});
        // an entry of P belongs to one thread, which adds its chunks and workers one after the other
        const int64_t entries = (int64_t)l.rows * std::max(d.rank[0], d.rank[1]);
        orth_loads = std::max(orth_loads, l.rows > kOrthThreads ? INT64_MAX
                                : (entries + kOrthThreads - 1) / kOrthThreads * d.n_colchunks * c->n_workers);
      } else {
        d.vec_off = p.vec_total;
        p.vec_total += n;
        for (int t = 0; t < d.ntiles; ++t) p.vectiles.push_back(d.tile0 + t);
      }
    } else if (c->method == ACC_TOPK) {
      auto kof = [&](int num) {
        const int64_t k = ((int64_t)n * num + c->k_den - 1) / c->k_den;
        return (int32_t)std::max<int64_t>(1, std::min<int64_t>(n, k));
      };
      d.k[0] = kof(c->k_num_noncrit);
      d.k[1] = kof(c->k_num_crit);
      d.pay_off = p.pay_stride;
      p.pay_stride += std::max(d.k[0], d.k[1]);
    }
  }
  // The orthogonalisation's one workgroup per layer sums the partials of P itself while none of its threads has
  // more than kOrthLoads of them to add at the higher rank: that is where it stops gaining there (the lower rank has
  // fewer and gains).  us per step so, and with the sums in a launch of their own, at the higher | the lower rank:
  // 16 loads (six layers of 256 x 4096, W = 1) 49.2, 50.5 | 45.1, 46.9; 24 (256 x 6144, W = 1) 64.8, 65.5 | 60.1, 62.2;
  // 24 (512 x 1536, W = 2) 67.9, 67.0 | 62.0, 63.3; 32 (256 x 8192, W = 1) 78.4, 78.4 | 73.6, 75.4; 36 (ResNet-18 shapes,
  // W = 1) 76.6, 74.9 | 69.5, 70.8; 576 (twelve layers of 10 x 9216, W = 16) 161, 118.5.
  p.pmean_in_orth = orth_loads <= kOrthLoads ? 1 : 0;
  // The right product, which reads Delta for the last time in the step, streams it unless the error memory may stay in the
  // 256 MB Infinity Cache beside what else a program does.  Read plainly, Delta stays there dirty, and the passes after it
  // wait for its lines to be evicted; read with the streaming hint, they go back to memory under this pass (e = g + e over
  // 3 x 179 MB in turn and a read of e after each: 91 + 26 us plain, 91 + 9 so).  us per step, plain -> streamed, three states in
  // turn | one state again and again | one state and 1 GB of a program's own traffic between its steps | the same and the gradients written
  // just before the step.  Aligned rows, where those of all workers take more than 72 MiB: ResNet-18 shapes W = 4 (170 MiB)
  // 172 -> 158 | 156 -> 158 | 172 -> 165 | 157 -> 153, W = 2 (85 MiB) 103.7 -> 102.5 | 101.1 -> 102.4 | 114 -> 109 | 105 -> 103, VGG-19 W = 1 (78 MiB)
  // 116 -> 115 | 113.7 -> 115.0 | 128 -> 123 | 119 -> 115, W = 4 (314 MiB) 319 -> 274 | 315 -> 272 | 321 -> 281 | 319 -> 282; LSTM W = 1 (196 MiB)
  // 541 -> 513 | 496 -> 503 | 535 -> 529 | 514 -> 507; the next smaller set measured is ResNet-18 W = 1 (43 MiB): 75.3 -> 76.0 three states in turn.
  // Unaligned rows (the odd-sized set, of which 6 % are aligned, its other passes streamed: kUStreamBytes), from 248 MiB of error memory on: W = 2 (58 MiB)
  // 85.0 -> 90.4 | 84.3 -> 90.0 | 99.8 -> 103.8 | 95.3 -> 98.2, W = 3 108.0 -> 112.8 | 104.7 -> 112.6 | 123.5 -> 130.9 | 117.6 -> 121.6, W = 6 (173 MiB)
  // 180.1 -> 179.1 | 162.8 -> 177.8 | 189.6 -> 207.9 | 180.0 -> 189.1, W = 8 (231 MiB) 224.0 -> 225.0 | 202.7 -> 222.2 | 233.4 -> 257.4 | 220.4 -> 236.3,
  // W = 9 (259 MiB) 255.1 -> 248.3 | 234.0 -> 246.4 | 274.9 -> 283.5 | 259.9 -> 269.1, W = 10 (288 MiB) 294.0 -> 272.7 | 285.7 -> 270.3 | 324.9 -> 307.8 |
  // 305.5 -> 298.8, W = 12 347 -> 322 | 343 -> 318 | 382 -> 355 | 371 -> 348.  Between 231 and 288 MiB the regimes disagree; both in the same
  // buffers: W = 8 225.6 -> 223.8 | 201.5 -> 220.8 | 222.9 -> 241.4 | 221.3 -> 232.9, W = 9 254.5 -> 246.9 | 235.5 -> 245.9 | 260.1 -> 267.2 | 260.4 -> 265.5, with the
  // update 274.9 -> 268.0 | 258.3 -> 266.7 | 281.0 -> 287.6 | 281.3 -> 286.0, call by call 388.6 -> 371.0 | 377.3 -> 369.2 | 405.6 -> 391.8 | 402.3 -> 388.7,
  // W = 10 290.8 -> 271.0 | 284.7 -> 269.7 | 299.9 -> 291.4 | 304.0 -> 297.2; ten layers of up to 2400 x 2400 W = 11 (316 MiB) 310.1 -> 301.9 | 289.6 -> 300.0 |
  // 317.1 -> 321.8 | 324.3 -> 328.8.  So at 248 MiB, where a call-by-call step gains in all of them, a batched one loses up to 5 % in three.
  p.q_stream = 4 * p.e_stride * c->n_workers > (int64_t(248) << 20) ? kQAllRows
               : 4 * aligned_rows * c->n_workers > (int64_t(72) << 20) ? kQAlignedRows : kQPlain;
  // (Of 12 M elements, aligned and unaligned rows, W = 4 | W = 2 with the update, plain -> streamed, three states in turn: a hundredth unaligned 187.8 -> 187.9 |
  // 144.3 -> 144.6, 3 % 188.7 -> 187.2 | 145.8 -> 146.7, 6 % 189.2 -> 187.9 | 145.8 -> 145.2, 12 % 190.2 -> 187.9 | 146.1 -> 145.2, 25 % 188.8 -> 186.3 |
  // 155.9 -> 148.3: below an eighth the two hardly differ, and a sixteenth keeps models with a few such layers on the smaller kernels.)
  const int64_t mat = p.n_model - p.vec_total;
  p.u_stream = 16 * (mat - aligned_rows) > mat && 4 * p.e_stride * c->n_workers > kUStreamBytes;
  run_order(p.mtiles);
  run_order(p.qmtiles);
  p.q_stride = 4 * ntile + nl;

  // workspace layout, 256-byte aligned regions
  int64_t off = 0;
  auto reg = [&](Region& r, int64_t bytes) {
    r.off = off;
    r.bytes = bytes;
    off = align_up(off + std::max<int64_t>(bytes, 0), 256);
  };
  const int64_t W = c->n_workers;
  reg(p.r_layers, (int64_t)sizeof(LayerDev) * nl);
  reg(p.r_ftiles, (int64_t)sizeof(FlatTile) * (int64_t)p.ftiles.size());
  reg(p.r_mtiles, (int64_t)sizeof(MatTile) * (int64_t)p.mtiles.size());
  reg(p.r_qmtiles, (int64_t)sizeof(MatTile) * (int64_t)p.qmtiles.size());
  reg(p.r_qtiles, (int64_t)sizeof(QTile) * (int64_t)p.qtiles.size());
  reg(p.r_ptiles, (int64_t)sizeof(PTile) * (int64_t)p.ptiles.size());
  reg(p.r_vectiles, 4 * (int64_t)p.vectiles.size());
  reg(p.r_matlayers, 4 * (int64_t)p.matlayers.size());
  reg(p.r_level, 4 * (int64_t)nl);
  reg(p.r_norm_old, 4 * (int64_t)nl);
  reg(p.r_norm_prev, 4 * (int64_t)nl);
  reg(p.r_norm_curr, 4 * (int64_t)nl);
  reg(p.r_has_old, 4 * (int64_t)nl);
  reg(p.r_rank_used, 4 * (int64_t)nl);
  reg(p.r_words, 8 * 7);
  reg(p.r_A, 4 * p.e_stride);
  reg(p.r_e, 4 * p.e_stride * W);
  reg(p.r_norm_part, 8 * ntile);
  reg(p.r_norm_part_m, 8 * (int64_t)p.mtiles.size());
  reg(p.r_afresh, 4);
  reg(p.r_sq_part, c->detector == ACC_DETECT_MSDR ? 8 * ntile : 0);
  reg(p.r_bstate, 4 * 8);
  if (c->method == ACC_POWERSGD) {
    reg(p.r_Q, 4 * p.q_dev);
    reg(p.r_Phat, 4 * p.p_total);
    reg(p.r_Pwork, 8 * p.p_total);
    reg(p.r_Ppart, 8 * p.ppart_stride * W);
    reg(p.r_Qpart, 8 * p.qpart_stride * W);
    reg(p.r_vecmean, 4 * p.vec_total);
    reg(p.r_pending, 4);
  } else if (c->method == ACC_TOPK) {
    reg(p.r_hist1, 4 * (int64_t)kHistBins * nl * W);
    reg(p.r_t2, 4 * (int64_t)kSub2 * p.n_t2slots * W);
    reg(p.r_qlist, 4 * (int64_t)kQListCap * p.q_stride * W);
    reg(p.r_sel, (int64_t)sizeof(SelState) * nl * W);
    reg(p.r_hist2m, 4 * (int64_t)kL2Bins * nl * W);
    reg(p.r_lflag, 4 * (int64_t)nl);
    reg(p.r_b1hist, 8 * 2 * (int64_t)nl * W);
    reg(p.r_guess, 4 * 2 * (int64_t)nl * W);
    reg(p.r_qinfo, (int64_t)sizeof(uint4) * p.q_stride * W);
    reg(p.r_candval, 4 * (int64_t)kCandCap * p.q_stride * W);
    reg(p.r_candidx, 2 * (int64_t)kCandCap * p.q_stride * W);
    reg(p.r_gtq, 4 * p.q_stride * W);
    reg(p.r_eqq, 4 * p.q_stride * W);
    reg(p.r_gtpre, 4 * p.q_stride * W);
    reg(p.r_eqpre, 4 * p.q_stride * W);
    reg(p.r_payidx, 4 * p.pay_stride * W);
    reg(p.r_payval, 4 * p.pay_stride * W);
    reg(p.r_overlap, 8 * (int64_t)nl);
    reg(p.r_tpending, 4);
  }
  p.total_bytes = off;
  return ACC_OK;
}

// Flatter tiles than the coarse ones need a little more workspace (tile tables, partial sums of Q): a workspace
// of `room` bytes that holds only the coarse ones gets those.  (Step with the fused update, ResNet-18 shapes at W = 1:
// 103.5 us with the flat ones, 108.9 with the coarse.)
int make_plan(const acc_config* c, Plan& p, char* err, size_t room) {
  const int rc = make_plan_tiled(c, p, err, false);
  if (rc != ACC_OK || c->method != ACC_POWERSGD || (size_t)p.total_bytes <= room) return rc;
  Plan coarse;
  if (make_plan_tiled(c, coarse, err, true) == ACC_OK && (size_t)coarse.total_bytes <= room) p = std::move(coarse);
  return ACC_OK;
}

}  // namespace

// Plain streaming copy used to calibrate hardware counters and to measure the copy bandwidth
// the memory system reaches: 256 threads, four 16-byte groups per thread, loads before stores.
constexpr int kProbeQuadsPerThread = 4;
__global__ __launch_bounds__(256) void probe_copy_kernel(float4* __restrict__ dst, const float4* __restrict__ src,
                                                         int64_t nquads) {
  const int64_t base = (int64_t)blockIdx.x * (256 * kProbeQuadsPerThread) + threadIdx.x;
  float4 v[kProbeQuadsPerThread];
#pragma unroll
  for (int i = 0; i < kProbeQuadsPerThread; ++i) {
    const int64_t q = base + (int64_t)i * 256;
    if (q < nquads) v[i] = src[q];
  }
#pragma unroll
  for (int i = 0; i < kProbeQuadsPerThread; ++i) {
    const int64_t q = base + (int64_t)i * 256;
    if (q < nquads) dst[q] = v[i];
  }
}

// ---- the workspace of callers that cannot allocate (accordion_init_static) ----------------------
// One array per GPU (every device that loads the library holds its own copy until the process
// ends).  Host code never uses the array's name as an address: the device address is taken once
// per device with hipGetSymbolAddress, that device being current, and kept.
static __device__ __align__(256) unsigned char scratch[ACC_STATIC_WORKSPACE_BYTES];

namespace {
constexpr int kMaxDevices = 64;
struct StaticSlot {
  void* ptr = nullptr;         // device address of `scratch` on this device
  acc_ctx* owner = nullptr;    // the context that uses it now (the last one created on it)
};
StaticSlot g_static[kMaxDevices];
std::mutex g_static_mutex;
}  // namespace

enum Stage {
  ST_psgd_ef_p_kernel = 0, ST_psgd_orth_kernel, ST_psgd_q_kernel, ST_psgd_qmean_kernel,
  ST_psgd_decomp_kernel, ST_psgd_residual_kernel, ST_topk_ef_hist_kernel, ST_topk_pick12_kernel,
  ST_topk_count3_kernel, ST_topk_pick3_kernel,
  ST_topk_compact_kernel, ST_topk_compact_mean_kernel, ST_topk_sparse_mean_kernel,
  ST_norm_partial_kernel, ST_regime_decide_kernel, ST_recount_words_kernel, ST_zero_accum_kernel,
  ST_psgd_decomp_update_kernel, ST_topk_compact_update_kernel, ST_topk_sparse_update_kernel,
  ST_batch_micro_kernel, ST_batch_micro_update_kernel, ST_batch_decide_kernel,
  ST_topk_overlap_kernel, ST_zero_u64_kernel, ST_msdr_sq_kernel, ST_msdr_decide_kernel,
  ST_psgd_clear_pending_kernel, ST_topk_residual_kernel, ST_topk_clear_pending_kernel,
  ST_topk_pick3_big_kernel, ST_psgd_pmean_kernel, ST_norm_refresh_kernel,
  ST_COUNT
};
static_assert(ST_COUNT <= ACC_N_STAGES, "more stages than the header announces");
static const char* const kStageNames[ST_COUNT] = {
  "psgd_ef_p_kernel", "psgd_orth_kernel", "psgd_q_kernel", "psgd_qmean_kernel",
  "psgd_decomp_kernel", "psgd_residual_kernel", "topk_ef_hist_kernel", "topk_pick12_kernel",
  "topk_count3_kernel", "topk_pick3_kernel",
  "topk_compact_kernel", "topk_compact_mean_kernel", "topk_sparse_mean_kernel",
  "norm_partial_kernel", "regime_decide_kernel", "recount_words_kernel", "zero_accum_kernel",
  "psgd_decomp_update_kernel", "topk_compact_update_kernel", "topk_sparse_update_kernel",
  "batch_micro_kernel", "batch_micro_update_kernel", "batch_decide_kernel",
  "topk_overlap_kernel", "zero_u64_kernel", "msdr_sq_kernel", "msdr_decide_kernel",
  "psgd_clear_pending_kernel", "topk_residual_kernel", "topk_clear_pending_kernel",
  "topk_pick3_big_kernel", "psgd_pmean_kernel", "norm_refresh_kernel"};

struct EventPair { hipEvent_t a, b; int stage; };

struct acc_ctx {
  // per-kernel timing
  int profiling = 0;               // 0 off, 1 every kernel, 2 only the fused error-feedback pass, 3 every fourth launch of it
  uint32_t prof_tick = 0;          // launches of that pass seen in mode 3
  std::vector<EventPair> pending, spare;
  double stage_ms[ST_COUNT] = {0};
  long long stage_n[ST_COUNT] = {0};
  acc_config cfg;
  std::vector<acc_layer> layers;
  Plan plan;
  Ws ws;
  char* base = nullptr;
  hipStream_t stream = nullptr;
  int static_dev = -1;             // >= 0: the workspace is the library's static array of that device
  // step state machine
  bool in_step = false;
  uint32_t step_id = 2;            // number of the current step (the device keeps 0 for "never")
  uint32_t p0_mask = 0, p1_mask = 0;
  bool agg0 = false, agg1 = false;
  GradPtrs grads;
  char err[256];
};

namespace {

#define ACC_HIP(ctx, call)                                                              \
  do {                                                                                  \
    hipError_t e_ = (call);                                                             \
    if (e_ != hipSuccess) {                                                             \
      std::snprintf((ctx)->err, 256, "%s failed: %s", #call, hipGetErrorString(e_));    \
      return ACC_EHIP;                                                                  \
    }                                                                                   \
  } while (0)

template <class T>
T* at(acc_ctx* c, const Region& r) { return reinterpret_cast<T*>(c->base + r.off); }

uint32_t all_workers_mask(const acc_ctx* c) {
  return c->cfg.n_workers == 32 ? 0xffffffffu : ((1u << c->cfg.n_workers) - 1u);
}

int check_launch(acc_ctx* c, const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    std::snprintf(c->err, 256, "launch of %s failed: %s", what, hipGetErrorString(e));
    return ACC_EHIP;
  }
  return ACC_OK;
}

// A context on the library's static workspace is usable only while it is the last one created on
// that device's array (a later accordion_init_static cleared and re-planned the memory).
int check_owner(acc_ctx* c) {
  if (c->static_dev < 0) return ACC_OK;
  std::lock_guard<std::mutex> lock(g_static_mutex);
  if (g_static[c->static_dev].owner == c) return ACC_OK;
  return fail(c->err, ACC_ESTATE, "the static workspace of this context was taken over by a later accordion_init_static");
}

#define ACC_USABLE(c)                          \
  do {                                         \
    if (!(c)) return ACC_EINVAL;               \
    const int rc_owner_ = check_owner(c);      \
    if (rc_owner_ != ACC_OK) return rc_owner_; \
  } while (0)

// Fold the finished event pairs into the per-stage totals (synchronises the stream).
int drain_profile(acc_ctx* c) {
  if (c->pending.empty()) return ACC_OK;
  if (hipStreamSynchronize(c->stream) != hipSuccess) return fail(c->err, ACC_EHIP, "hipStreamSynchronize failed");
  for (EventPair& p : c->pending) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, p.a, p.b) == hipSuccess) {
      c->stage_ms[p.stage] += ms;
      c->stage_n[p.stage] += 1;
    }
    c->spare.push_back(p);
  }
  c->pending.clear();
  return ACC_OK;
}

bool prof_begin(acc_ctx* c, int stage, EventPair& p) {
  if (!c->profiling) return false;
  if (c->profiling >= 2 && stage != ST_topk_ef_hist_kernel && stage != ST_psgd_ef_p_kernel &&
      stage != ST_batch_micro_kernel && stage != ST_batch_micro_update_kernel)
    return false;
  if (c->profiling == 3 && (c->prof_tick++ & 3u) != 0u) return false;
  if (c->pending.size() >= 8192) drain_profile(c);
  if (!c->spare.empty()) {
    p = c->spare.back();
    c->spare.pop_back();
  } else {
    if (hipEventCreate(&p.a) != hipSuccess) return false;
    if (hipEventCreate(&p.b) != hipSuccess) { (void)hipEventDestroy(p.a); return false; }
  }
  p.stage = stage;
  return true;
}

void prof_end(acc_ctx* c, EventPair& p) { c->pending.push_back(p); }

// stage: the kernel's name; kernel: the kernel itself (an instantiation of a template has no name of its own).
#define ACC_LAUNCH_AS(ctx, stage, kernel, grid, block, ...)                  \
  do {                                                                       \
    EventPair ep_;                                                           \
    const bool prof_ = prof_begin(ctx, ST_##stage, ep_);                     \
    if (prof_) {                                                             \
      /* the two events take the dispatch's own begin and end timestamps */  \
      hipExtLaunchKernelGGL((kernel), grid, block, 0, (ctx)->stream, ep_.a, ep_.b, 0, __VA_ARGS__); \
      prof_end(ctx, ep_);                                                    \
    } else {                                                                 \
      hipLaunchKernelGGL((kernel), grid, block, 0, (ctx)->stream, __VA_ARGS__); \
    }                                                                        \
    int rc_ = check_launch(ctx, #stage);                                     \
    if (rc_ != ACC_OK) return rc_;                                           \
  } while (0)
#define ACC_LAUNCH(ctx, name, grid, block, ...) ACC_LAUNCH_AS(ctx, name, name, grid, block, __VA_ARGS__)

// --- launches of each stage for workers [w0, w0 + nw) ------------------------------------

// What a step leaves to the 256 MB Infinity Cache until the next one: batched TopK steps the first kCachedError elements of the
// workers' error memories, fused updates the first kCachedUpdate of weights and velocity (or all or none, see update_cached).  The rest goes through streaming
// loads and stores.  Everything accessed plainly, whatever does not fit is evicted while the next pass reads, dirty line by dirty line:
// e = g + e over 3 x 179 MB in turn runs at 5.8 TB/s so, 6.2 streamed.  us per step, everything plain -> so, three states in turn | one state
// again and again | one state and 1 GB of a program's own traffic between its steps | the same and the gradients written just before:
//   error memory: ResNet-18 shapes W = 4 K = 10 % 194 -> 181 | 161 -> 162 | 185 -> 183 | 166 -> 161, K = 1 % 172 -> 153 | 142 -> 146 | 166 -> 164 |
//   147 -> 143; W = 2 119 -> 110 | 104 -> 105 | 121 -> 121 | 111 -> 111; VGG-19 W = 1 131 -> 124 | 116 -> 118 | 135 -> 135 | 124 -> 125,
//   W = 4 340 -> 307 | 332 -> 291 | 336 -> 316 | 341 -> 302; odd sizes W = 3 106 -> 96 | 93 -> 94 | 108 -> 109 | 100 -> 101; LSTM W = 1 327 -> 288 |
//   271 -> 263 | 318 -> 292 | 300 -> 265; two windows of five steps of ResNet-18 1681 -> 1679 | 1653 -> 1649 | 1882 -> 1844 | 1711 -> 1625, of four
//   of VGG-19 at K = 99 % and 2 %, W = 2 1431 -> 1465 | 1412 -> 1442 | 1614 -> 1617 | 1474 -> 1471.  32 MB instead of 64: ResNet-18 W = 4 169 | 164, but
//   those VGG-19 windows 1483; 96 MB 187 | 162; none 170 | 169.
//   weights and velocity (16 MB of them plain at every size; update_cached takes the small and the large contexts out), TopK: ResNet-18 W = 1 113 -> 95 | 89 -> 94 | 114 -> 109 | 107 -> 103, W = 4 215 -> 208 | 179 -> 184 | 212 -> 208 | 187 -> 185;
//   VGG-19 W = 1 186 -> 177 | 153 -> 158 | 186 -> 181 | 173 -> 169; LSTM W = 1 422 -> 393 | 418 -> 369 | 415 -> 400 | 381 -> 371; odd sizes W = 3 135 -> 128 |
//   111 -> 116 | 136 -> 136 | 125 -> 125; PowerSGD: ResNet-18 W = 1 103 -> 96 | 90 -> 96 | 106 -> 106 | 101 -> 101, W = 2 131 -> 127 | 121 -> 126 | 136 -> 135 |
//   130 -> 128; VGG-19 W = 1 170 -> 159 | 151 -> 158 | 171 -> 168 | 163 -> 161; LSTM W = 1 643 -> 624 | 642 -> 608 | 636 -> 634 | 612 -> 612.
// So a state that finds the caches as it left them, and fits them, pays up to 6 %; wherever a program does anything between two steps
// the policy gains or makes no difference.
constexpr int64_t kCachedError = (int64_t(64) << 20) / 4, kCachedUpdate = (int64_t(16) << 20) / 8;

// The first element of weights and velocity that a fused update streams.  TopK: none is left to the cache where they and the error memory take
// more than 192 MiB.  16 MB plain -> none, regimes as above; beyond: K = 25 % ResNet-18 W = 4 252.5 -> 247.8 | 231 -> 229 | 244 -> 241 | 236 -> 234,
// VGG-19 W = 1 201 -> 195 | 183 -> 186 | 200 -> 201 | 193 -> 194; K = 10 % ResNet-18 W = 4 211 -> 208 | 187.5 -> 189.8 | 204 -> 204 | 193.5 -> 194.6, W = 8
// 345 -> 338 | 316 -> 319 | 339 -> 341 | 335 -> 337, VGG-19 W = 1 181 -> 171 | 162 -> 164 | 177.5 -> 178 | 171.5 -> 172, W = 4 364 -> 355 | 334 -> 337 |
// 357 -> 357 | 353 -> 355, LSTM W = 1 388 -> 385 | 369 -> 372 | 396 -> 397 | 383.5 -> 385; below: ResNet-18 W = 1 K = 1 % 98.1 -> 99.6 | 97 -> 98.3 |
// 112 -> 111 | 107 -> 106, W = 2 K = 10 % (170 MiB) 144 -> 137 | 129 -> 131 | 142.6 -> 143 | 137 -> 138, odd sizes W = 3 (144 MiB) 133 -> 129 |
// 119 -> 122.5 | 133 -> 134 | 128 -> 129.  PowerSGD: 16 MB at every size, ResNet-18 W = 2 129 -> 130.5 | 129 -> 130.5 | 138 -> 139 | 135.5 -> 136.5, VGG-19 W = 1
// 157 -> 159 | 156 -> 158.5 | 167.5 -> 168.5 | 164.5 -> 165.5, W = 2 216 -> 216 | 212 -> 214.5 | 228 -> 229 | 221 -> 222, ResNet-18 W = 8 within 0.5 %.
// Small contexts, up to 76 MiB of error memory, weights and velocity, leave everything to the cache.  Plain -> 16 MB plain and the rest streamed,
// layers of 1024 x 512: TopK K = 25 % W = 1 2.6 M elements (30 MiB) 51.0 -> 55.5 | 50.8 -> 55.6 | 63 -> 63 | 62 -> 62, 5.2 M (60 MiB) 62.8 -> 66.6 | 62.5 -> 66.6 |
// 75.6 -> 75.2 | 74.3 -> 73.9, W = 2 3.7 M (56 MiB) 66.1 -> 71.6 | 65.8 -> 72.1 | 79 -> 79 | 77 -> 77; PowerSGD W = 1 3.7 M (42 MiB) 52.4 -> 54.4 | 52.4 -> 54.6 |
// 60 -> 60 | 59 -> 59, 6.3 M (72 MiB) 68.0 -> 70.6 | 67.3 -> 70.4 | 77 -> 78 | 76 -> 76; above, PowerSGD W = 2 5.2 M (80 MiB) 77.3 -> 76.7 | 74.1 -> 76.0 | 84 -> 84 |
// 82 -> 83, TopK K = 25 % 89 -> 85 | 80 -> 84 | 94.5 -> 93 | 92.5 -> 91, W = 1 8.4 M (96 MiB) 94 -> 86 | 83 -> 87 | 94 -> 96 | 92 -> 95.
int64_t update_cached(const acc_ctx* c) {
  const int64_t resident = 4 * c->plan.e_stride * (int64_t)c->cfg.n_workers + 8 * c->plan.N;
  if (resident <= (int64_t(76) << 20)) return c->plan.N;
  return c->cfg.method == ACC_TOPK && resident > (int64_t(192) << 20) ? 0 : kCachedUpdate;
}

// Tiles of a launch from which the counting kernel takes a tile per wave.  us per step, a quarter per wave -> a tile per wave:
// LSTM set W = 16 (100 000 tiles) 2409 -> 2381, K = 1 % 2085 -> 2055, W = 4 (25 000) 709 -> 707; ResNet-18 W = 8 (11 000) 300 -> 302,
// four small layers W = 2 36.6 -> 40.4.
constexpr int64_t kWideCountTiles = 20000;

// TopK selection of workers [w0, w0 + nw): the fused error-feedback pass, then the per-layer decisions
// (level-1/2 bins, re-staging after a missed guess, level-3/4 counts, threshold and prefixes).  e_reread: Delta is read
// again within the step, whatever the guess.
int launch_topk_select(acc_ctx* c, int w0, int nw, int e_reread) {
  const Ws& ws = c->ws;
  const dim3 tiles(ws.n_ftiles, nw);
  if (ws.e_stride * ws.W > kCachedError)
    ACC_LAUNCH_AS(c, topk_ef_hist_kernel, topk_ef_hist_large_kernel, tiles, dim3(256), ws, c->grads, w0, kCachedError, e_reread);
  else
    ACC_LAUNCH_AS(c, topk_ef_hist_kernel, topk_ef_hist_kernel, tiles, dim3(256), ws, c->grads, w0, kCachedError, e_reread);
  ACC_LAUNCH(c, topk_pick12_kernel, dim3(ws.L, nw), dim3(kPickThreads), ws, w0);
  if ((int64_t)ws.n_ftiles * nw >= kWideCountTiles)
    ACC_LAUNCH_AS(c, topk_count3_kernel, topk_count3_wide_kernel, dim3((ws.n_ftiles + 3) / 4, nw), dim3(256), ws, w0);
  else
    ACC_LAUNCH(c, topk_count3_kernel, tiles, dim3(256), ws, w0);
  ACC_LAUNCH(c, topk_pick3_kernel, dim3(ws.L, nw), dim3(kPickThreads), ws, w0, c->step_id);
  if (c->plan.pick3_big) ACC_LAUNCH(c, topk_pick3_big_kernel, dim3(ws.L, nw), dim3(kPickThreads), ws, w0, c->step_id);
  return ACC_OK;
}

// The MSDR detector also needs the squared norm of worker 0's raw gradient of every step.
int launch_detector_feed(acc_ctx* c, int w0) {
  const Ws& ws = c->ws;
  if (c->cfg.detector == ACC_DETECT_MSDR && w0 == 0)
    ACC_LAUNCH(c, msdr_sq_kernel, dim3(ws.n_ftiles), dim3(256), ws, c->grads.p[0]);
  return ACC_OK;
}

int launch_phase0(acc_ctx* c, int w0, int nw) {
  const Ws& ws = c->ws;
  {
    const int rc = launch_detector_feed(c, w0);
    if (rc != ACC_OK) return rc;
  }
  if (c->cfg.method == ACC_POWERSGD) {
    const int gx = ws.n_mtiles + (w0 == 0 ? ws.n_vectiles : 0);
    if (gx > 0 && c->plan.u_stream) ACC_LAUNCH_AS(c, psgd_ef_p_kernel, psgd_ef_p_stream_kernel, dim3(gx, nw), dim3(256), ws, c->grads, w0);
    else if (gx > 0) ACC_LAUNCH(c, psgd_ef_p_kernel, dim3(gx, nw), dim3(256), ws, c->grads, w0);
  } else {
    const int rc = launch_topk_select(c, w0, nw, 1);   // the compaction reads Delta once more
    if (rc != ACC_OK) return rc;
    ACC_LAUNCH(c, topk_compact_kernel, dim3(ws.n_ftiles, nw), dim3(256), ws, w0);
  }
  return ACC_OK;
}

int launch_agg0(acc_ctx* c) {
  const Ws& ws = c->ws;
  if (c->cfg.method == ACC_POWERSGD) {
    // the mean of the 1-D layers rides with the first of the two launches
    if (!ws.pmean_in_orth) ACC_LAUNCH(c, psgd_pmean_kernel, dim3(ws.n_ptiles + ws.n_vectiles), dim3(256), ws, c->grads);
    const int gx = ws.n_mat + (ws.pmean_in_orth ? ws.n_vectiles : 0);
    if (gx > 0) ACC_LAUNCH(c, psgd_orth_kernel, dim3(gx), dim3(kOrthThreads), ws, c->grads);
  }
  return ACC_OK;
}

int launch_phase1(acc_ctx* c, int w0, int nw) {
  const Ws& ws = c->ws;
  if (ws.n_qmtiles == 0) return ACC_OK;
  // a kernel for each: one that held both kinds of access was 45 KB of code instead of 28, which a step that follows a program's own
  // kernels has to fetch (ResNet-18 shapes at W = 1, plain either way: 83.3 us per step so, 80.8 with a kernel for each)
  const dim3 grid(ws.n_qmtiles, nw);
  switch (c->plan.q_stream) {
    case kQPlain: ACC_LAUNCH_AS(c, psgd_q_kernel, psgd_q_kernel<kQPlain>, grid, dim3(256), ws, w0); break;
    case kQAlignedRows: ACC_LAUNCH_AS(c, psgd_q_kernel, psgd_q_kernel<kQAlignedRows>, grid, dim3(256), ws, w0); break;
    default: ACC_LAUNCH_AS(c, psgd_q_kernel, psgd_q_kernel<kQAllRows>, grid, dim3(256), ws, w0); break;
  }
  return ACC_OK;
}

int launch_agg1(acc_ctx* c) {
  const Ws& ws = c->ws;
  if (ws.n_qtiles > 0) ACC_LAUNCH(c, psgd_qmean_kernel, dim3(ws.n_qtiles, kMatCols / kQmeanCols), dim3(256), ws);
  return ACC_OK;
}

bool misaligned(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

Sink sink_out(float* out) { return Sink{out, nullptr, nullptr, 0.f, 0.f, 0.f, 0}; }

// sink.wt != nullptr: the optimizer step consumes the averaged gradient instead of a store.
int launch_decompress(acc_ctx* c, const Sink& sink) {
  const Ws& ws = c->ws;
  if (c->cfg.method == ACC_POWERSGD) {
    const dim3 grid(ws.n_mtiles + ws.n_vectiles);
    if (c->plan.u_stream) {
      if (sink.wt) ACC_LAUNCH_AS(c, psgd_decomp_update_kernel, psgd_decomp_update_stream_kernel, grid, dim3(256), ws, sink);
      else ACC_LAUNCH_AS(c, psgd_decomp_kernel, psgd_decomp_stream_kernel, grid, dim3(256), ws, sink);
    } else {
      if (sink.wt) ACC_LAUNCH(c, psgd_decomp_update_kernel, grid, dim3(256), ws, sink);
      else ACC_LAUNCH(c, psgd_decomp_kernel, grid, dim3(256), ws, sink);
    }
  } else {
    if (sink.wt) ACC_LAUNCH(c, topk_sparse_update_kernel, dim3(ws.n_ftiles), dim3(256), ws, sink);
    else ACC_LAUNCH(c, topk_sparse_mean_kernel, dim3(ws.n_ftiles), dim3(256), ws, sink);
  }
  return ACC_OK;
}

// Batch-size mode: the running sums are accessed plainly as far as they and the accumulator fit the 256 MB Infinity Cache, the
// rest is streamed: a plain rest evicts what would have stayed, dirty line by dirty line.  One large batch of four
// micro-steps, us, everything plain -> so: VGG-19 W = 4 790 -> 639, ResNet-18 W = 8 804 -> 656, odd sizes W = 9 652 -> 530, LSTM W = 4 1377 -> 1238;
// eight of ResNet-18 W = 4 (224 MB) 741 -> 738.  160 MB instead: W = 8 689, ResNet-18 W = 4 752; 240 MB: within 1 %.
constexpr int64_t kCachedSums = (int64_t(224) << 20) / 4;

const char* const kBatchCallByCall =
    "batch-size mode has no call-by-call sequence: use accordion_step_all / accordion_step_all_update";

// One micro-step of the batch-size mode for all workers (c->grads is set).
int launch_batch_micro(acc_ctx* c, const Sink& sink) {
  const Ws& ws = c->ws;
  const uint32_t parity = c->step_id & 1u;
  const int64_t sums_cached = (kCachedSums - (ws.W > 1 ? ws.e_stride : 0)) / ws.W;
  if (sink.wt) ACC_LAUNCH(c, batch_micro_update_kernel, dim3(ws.n_ftiles), dim3(256), ws, c->grads, sink, parity, sums_cached);
  else ACC_LAUNCH(c, batch_micro_kernel, dim3(ws.n_ftiles), dim3(256), ws, c->grads, sink, parity, sums_cached);
  return ACC_OK;
}

int launch_topk_compact_mean(acc_ctx* c, const Sink& sink) {
  const Ws& ws = c->ws;
  const dim3 grid(ws.n_ftiles * kMeanSplit), block(kMeanWaves * kWave);
  const bool large = ws.delta_stream || ws.lists_stream;
  if (sink.wt) {
    if (large) ACC_LAUNCH_AS(c, topk_compact_update_kernel, topk_compact_update_large_kernel, grid, block, ws, sink);
    else ACC_LAUNCH(c, topk_compact_update_kernel, grid, block, ws, sink);
  } else {
    if (large) ACC_LAUNCH_AS(c, topk_compact_mean_kernel, topk_compact_mean_large_kernel, grid, block, ws, sink);
    else ACC_LAUNCH(c, topk_compact_mean_kernel, grid, block, ws, sink);
  }
  return ACC_OK;
}

// Arguments of the optimizer step: finite hyper-parameters, two distinct aligned device buffers.
int check_sgd(acc_ctx* c, const float* w, const float* v, float lr, float mu, float wd) {
  if (!w || !v) return fail(c->err, ACC_EINVAL, "weights_dev or velocity_dev is NULL");
  if (misaligned(w) || misaligned(v)) return fail(c->err, ACC_EINVAL, "weights_dev / velocity_dev is not 16-byte aligned");
  if (w == v) return fail(c->err, ACC_EINVAL, "weights_dev and velocity_dev are the same buffer");
  if (!(std::isfinite(lr) && std::isfinite(mu) && std::isfinite(wd)) || lr < 0.f || mu < 0.f || wd < 0.f)
    return fail(c->err, ACC_EINVAL, "lr, momentum and weight_decay must be finite and not negative");
  return ACC_OK;
}

// Make the error memory explicit: e_w = Delta_w - D for the workers whose residual is pending.
int materialise(acc_ctx* c) {
  const Ws& ws = c->ws;
  if (c->cfg.method == ACC_TOPK) {
    ACC_LAUNCH(c, topk_residual_kernel, dim3(ws.n_ftiles, ws.W), dim3(256), ws);
    ACC_LAUNCH(c, topk_clear_pending_kernel, dim3(1), dim3(64), ws);
    return ACC_OK;
  }
  if (c->cfg.method != ACC_POWERSGD) return ACC_OK;
  if (ws.n_mtiles > 0) ACC_LAUNCH(c, psgd_residual_kernel, dim3(ws.n_mtiles, ws.W), dim3(256), ws);
  ACC_LAUNCH(c, psgd_clear_pending_kernel, dim3(1), dim3(64), ws);
  return ACC_OK;
}

void end_step(acc_ctx* c) {
  c->in_step = false;
  c->step_id += 1;
  c->p0_mask = c->p1_mask = 0;
  c->agg0 = c->agg1 = false;
}

// Q between the caller's layout (every matrix layer's cols x rmax block, layers in order) and the
// device layout (rows padded to kMaxRank floats, so that a row is one aligned 16-byte load).
int copy_q(acc_ctx* c, float* host, bool to_host) {
  const Plan& p = c->plan;
  if (p.q_dev == 0) return ACC_OK;
  std::vector<float> dev((size_t)p.q_dev, 0.f);
  if (to_host) ACC_HIP(c, hipMemcpy(dev.data(), c->ws.Q, 4 * dev.size(), hipMemcpyDeviceToHost));
  size_t hp = 0;
  for (const int li : p.matlayers) {
    const LayerDev& L = p.layers[(size_t)li];
    for (int j = 0; j < L.cols; ++j)
      for (int k = 0; k < p.rmax; ++k) {
        float& d = dev[(size_t)L.q_off + (size_t)j * kMaxRank + k];
        if (to_host) host[hp] = d; else d = host[hp];
        ++hp;
      }
  }
  if (!to_host) ACC_HIP(c, hipMemcpy(c->ws.Q, dev.data(), 4 * dev.size(), hipMemcpyHostToDevice));
  return ACC_OK;
}

size_t state_bytes_of(const acc_ctx* c) {
  const Plan& p = c->plan;
  const size_t L = (size_t)c->cfg.n_layers;
  return 4 * ((size_t)p.N * (size_t)(c->cfg.n_workers + 1) + (size_t)p.q_total + 3 * L +
              (c->cfg.method == ACC_BATCH ? 1u : 0u));
}

}  // namespace

extern "C" {

int32_t accordion_workspace_bytes(const acc_config* cfg, size_t* out_bytes) {
  if (!out_bytes) return fail(g_init_error, ACC_EINVAL, "out_bytes is NULL");
  // the size by which a caller decides whether the static workspace serves: the coarse tiles' where only they fit it
  Plan p;
  const int rc = make_plan(cfg, p, g_init_error, ACC_STATIC_WORKSPACE_BYTES);
  if (rc != ACC_OK) return rc;
  *out_bytes = (size_t)p.total_bytes;
  return ACC_OK;
}

static int32_t init_common(const acc_config* cfg, void* workspace_dev, size_t workspace_bytes,
                           const float* q_init_host, void* hip_stream, acc_ctx** out, const char* too_small) {
  if (!out) return fail(g_init_error, ACC_EINVAL, "out is NULL");
  *out = nullptr;
  acc_ctx* c = new (std::nothrow) acc_ctx();
  if (!c) return fail(g_init_error, ACC_ENOSPACE, "out of host memory");
  auto bail = [&](int rc, const char* msg) {
    if (msg) std::snprintf(g_init_error, 256, "%s", msg);
    else std::snprintf(g_init_error, 256, "%s", c->err);
    delete c;
    return rc;
  };
  int rc = make_plan(cfg, c->plan, g_init_error, workspace_bytes);
  if (rc != ACC_OK) { delete c; return rc; }
  if (!workspace_dev) return bail(ACC_EINVAL, "workspace is NULL");
  if ((reinterpret_cast<uintptr_t>(workspace_dev) & 255u) != 0) return bail(ACC_EINVAL, "workspace is not 256-byte aligned");
  if (workspace_bytes < (size_t)c->plan.total_bytes) return bail(ACC_ENOSPACE, too_small);
  if (cfg->method == ACC_POWERSGD && c->plan.q_total > 0 && !q_init_host)
    return bail(ACC_EINVAL, "q_init_host is NULL");
  c->cfg = *cfg;
  c->layers.assign(cfg->layers, cfg->layers + cfg->n_layers);
  c->cfg.layers = c->layers.data();
  c->base = static_cast<char*>(workspace_dev);
  c->stream = static_cast<hipStream_t>(hip_stream);
  std::snprintf(c->err, 256, "no error");
  std::memset(&c->grads, 0, sizeof(c->grads));
  Plan& p = c->plan;

  Ws& ws = c->ws;
  std::memset(&ws, 0, sizeof(ws));
  ws.layers = at<LayerDev>(c, p.r_layers);
  ws.ftiles = at<FlatTile>(c, p.r_ftiles);
  ws.mtiles = at<MatTile>(c, p.r_mtiles);
  ws.qmtiles = at<MatTile>(c, p.r_qmtiles);
  ws.qtiles = at<QTile>(c, p.r_qtiles);
  ws.ptiles = at<PTile>(c, p.r_ptiles);
  ws.vectiles = at<int32_t>(c, p.r_vectiles);
  ws.matlayers = at<int32_t>(c, p.r_matlayers);
  ws.level = at<int32_t>(c, p.r_level);
  ws.norm_old = at<float>(c, p.r_norm_old);
  ws.norm_prev = at<float>(c, p.r_norm_prev);
  ws.norm_curr = at<float>(c, p.r_norm_curr);
  ws.has_old = at<int32_t>(c, p.r_has_old);
  ws.rank_used = at<int32_t>(c, p.r_rank_used);
  ws.words = at<unsigned long long>(c, p.r_words);
  ws.stats = ws.words + 4;
  ws.A = at<float>(c, p.r_A);
  ws.e = at<float>(c, p.r_e);
  ws.e_stride = p.e_stride;
  ws.norm_part = at<double>(c, p.r_norm_part);
  ws.norm_part_m = at<double>(c, p.r_norm_part_m);
  ws.a_fresh = at<uint32_t>(c, p.r_afresh);
  ws.sq_part = p.r_sq_part.bytes > 0 ? at<double>(c, p.r_sq_part) : nullptr;
  if (cfg->method == ACC_POWERSGD) {
    ws.Q = at<float>(c, p.r_Q);
    ws.Phat = at<float>(c, p.r_Phat);
    ws.Pwork = at<double>(c, p.r_Pwork);
    ws.Ppart = at<double>(c, p.r_Ppart);
    ws.ppart_stride = p.ppart_stride;
    ws.Qpart = at<double>(c, p.r_Qpart);
    ws.qpart_stride = p.qpart_stride;
    ws.vecmean = at<float>(c, p.r_vecmean);
    ws.pending = at<uint32_t>(c, p.r_pending);
  } else if (cfg->method == ACC_TOPK) {
    ws.hist1 = at<uint32_t>(c, p.r_hist1);
    ws.t2 = at<uint32_t>(c, p.r_t2);
    ws.qlist = at<uint32_t>(c, p.r_qlist);
    ws.sel = at<SelState>(c, p.r_sel);
    ws.hist2m = at<uint32_t>(c, p.r_hist2m);
    ws.lflag = at<uint32_t>(c, p.r_lflag);
    ws.b1hist = at<uint2>(c, p.r_b1hist);
    ws.guess = at<uint32_t>(c, p.r_guess);
    ws.qinfo = at<uint4>(c, p.r_qinfo);
    ws.cand_val = at<uint32_t>(c, p.r_candval);
    ws.cand_idx = at<uint16_t>(c, p.r_candidx);
    ws.gtq = at<uint32_t>(c, p.r_gtq);
    ws.eqq = at<uint32_t>(c, p.r_eqq);
    ws.gtpre = at<uint32_t>(c, p.r_gtpre);
    ws.eqpre = at<uint32_t>(c, p.r_eqpre);
    ws.pay_idx = at<int32_t>(c, p.r_payidx);
    ws.pay_val = at<float>(c, p.r_payval);
    ws.pay_stride = p.pay_stride;
    ws.overlap = at<unsigned long long>(c, p.r_overlap);
    ws.tpending = at<uint32_t>(c, p.r_tpending);
    // The compaction is the last to read Delta (where it does: band guesses) and the candidate lists.  Read with the streaming
    // hint, what lies dirty in the Infinity Cache goes back to memory under this pass instead of during the next one.  us per step, plain ->
    // streamed, three states in turn | one state again and again | one state and 1 GB of other traffic between its steps | the same and the
    // gradients written just before.  Delta: where the error memory exceeds the cache (LSTM set K = 99 %, W = 4, 941 -> 894 | 937 -> 892 |
    // 1018 -> 902 | 1025 -> 908; not below: ResNet-18 shapes K = 99 %, W = 4, 179 MB, 225 -> 219 | 199 -> 217 | 216 -> 228 | 197 -> 205, VGG-19 W = 2
    // 224 -> 218 | 195 -> 218 | 219 -> 230 | 203 -> 210; pairs, K = 30 %: odd sizes W = 8 (231 MiB) 311 -> 297 | 288 -> 287 | 311 -> 307 | 304 -> 302, VGG-19 W = 3
    // (235 MiB) 324 -> 314 | 303 -> 305 | 323 -> 324 | 322 -> 324, ResNet-18 W = 6 (256 MiB) 346 -> 331 | 331 -> 322 | 349 -> 341 | 352 -> 345).  The holes layout, whose payload
    // writes leave less room, later: K = 99 % odd sizes W = 8 284 -> 278 | 258 -> 276 | 274 -> 298 | 267 -> 279, VGG-19 W = 3 302 -> 302 | 274 -> 301 | 292 -> 321 |
    // 286 -> 307, ResNet-18 W = 6 330 -> 317 | 304 -> 314 | 328 -> 341 | 323 -> 333, windows of four steps at K = 99 % and 2 % 2116 -> 2126 | 2093 -> 2124 | 2129 -> 2149 |
    // 2103 -> 2124; odd sizes W = 10 (288 MiB) 370 -> 343 | 342 -> 341 | 371 -> 366 | 376 -> 373, windows 2392 -> 2347 | 2348 -> 2345 | 2394 -> 2374 | 2366 -> 2348.  Lists: where there are more than 64 M elements (K = 10 %: ResNet-18 W = 8 326 -> 313 |
    // 287 -> 292 | 316 -> 320 | 298 -> 303, VGG-19 W = 4 322 -> 308 | 284 -> 291 | 309 -> 317 | 293 -> 302, odd sizes W = 12 342 -> 330 | 301 -> 305 |
    // 329 -> 333 | 313 -> 318, LSTM W = 4 705 -> 704 | 686 -> 688 | 712 -> 714 | 708 -> 706: 4 % where nothing of a state stays in the cache, for 1 to 3 %
    // where some of it does; not below: LSTM W = 1, 51 M, 289 -> 296 | 263 -> 289 | 291 -> 310 | 265 -> 281, VGG-19 W = 1 123 -> 124 | 118 -> 123 |
    // 137 -> 142 | 126 -> 131).
    const int64_t elements = p.e_stride * cfg->n_workers;
    ws.delta_stream = 4 * elements > (int64_t(224) << 20) ? 1 : 0;
    ws.delta_stream_holes = 4 * elements > (int64_t(280) << 20) ? 1 : 0;
    ws.lists_stream = elements > (int64_t(64) << 20) ? 1 : 0;
  }
  ws.bstate = at<uint32_t>(c, p.r_bstate);
  ws.bmult = cfg->method == ACC_BATCH ? cfg->batch_multiplier : 1;
  ws.bmono = cfg->method == ACC_BATCH ? cfg->batch_monotone : 0;
  ws.n_model = p.n_model;
  ws.q_stride = p.q_stride;
  ws.n_qslots = p.q_stride * cfg->n_workers;
  ws.N = p.N;
  ws.W = cfg->n_workers;
  ws.L = cfg->n_layers;
  ws.rmax = p.rmax;
  ws.mrows = p.mrows;
  ws.pmean_in_orth = p.pmean_in_orth;
  ws.qrows = p.qrows;
  ws.n_ftiles = (int32_t)p.ftiles.size();
  ws.n_t2slots = (int32_t)p.n_t2slots;
  ws.n_mtiles = (int32_t)p.mtiles.size();
  ws.n_qmtiles = (int32_t)p.qmtiles.size();
  ws.n_qtiles = (int32_t)p.qtiles.size();
  ws.n_ptiles = (int32_t)p.ptiles.size();
  ws.n_vectiles = (int32_t)p.vectiles.size();
  ws.n_mat = (int32_t)p.matlayers.size();
  ws.xcd_runs = cfg->method == ACC_TOPK && p.e_stride * cfg->n_workers > (int64_t(1) << 28) ? 1 : 0;
  ws.eta = cfg->eta;

  const int nl_ = cfg->n_layers;
  auto init_dev = [&]() -> int {
    ACC_HIP(c, hipMemsetAsync(c->base, 0, (size_t)p.total_bytes, c->stream));
    ACC_HIP(c, hipStreamSynchronize(c->stream));
    auto up = [&](const Region& r, const void* src) -> hipError_t {
      if (r.bytes == 0) return hipSuccess;
      return hipMemcpy(c->base + r.off, src, (size_t)r.bytes, hipMemcpyHostToDevice);
    };
    ACC_HIP(c, up(p.r_layers, p.layers.data()));
    ACC_HIP(c, up(p.r_ftiles, p.ftiles.data()));
    ACC_HIP(c, up(p.r_mtiles, p.mtiles.data()));
    ACC_HIP(c, up(p.r_qmtiles, p.qmtiles.data()));
    ACC_HIP(c, up(p.r_qtiles, p.qtiles.data()));
    ACC_HIP(c, up(p.r_ptiles, p.ptiles.data()));
    ACC_HIP(c, up(p.r_vectiles, p.vectiles.data()));
    ACC_HIP(c, up(p.r_matlayers, p.matlayers.data()));
    std::vector<int32_t> lv((size_t)cfg->n_layers, cfg->initial_level);
    ACC_HIP(c, up(p.r_level, lv.data()));
    if (cfg->method == ACC_POWERSGD && p.q_total > 0) {
      const int rq = copy_q(c, const_cast<float*>(q_init_host), false);
      if (rq != ACC_OK) return rq;
    }
    if (cfg->method == ACC_TOPK) {
      std::vector<uint32_t> none((size_t)2 * nl_ * cfg->n_workers, kNoGuess);
      ACC_HIP(c, up(p.r_guess, none.data()));
    }
    ACC_LAUNCH(c, recount_words_kernel, dim3(1), dim3(256), c->ws, (int)cfg->method, -1);
    ACC_HIP(c, hipStreamSynchronize(c->stream));
    return ACC_OK;
  };
  rc = init_dev();
  if (rc != ACC_OK) return bail(rc, nullptr);
  *out = c;
  return ACC_OK;
}

int32_t accordion_init(const acc_config* cfg, void* workspace_dev, size_t workspace_bytes,
                       const float* q_init_host, void* hip_stream, acc_ctx** out) {
  return init_common(cfg, workspace_dev, workspace_bytes, q_init_host, hip_stream, out, "workspace too small");
}

int32_t accordion_init_static(const acc_config* cfg, const float* q_init_host, void* hip_stream, acc_ctx** out) {
  if (!out) return fail(g_init_error, ACC_EINVAL, "out is NULL");
  *out = nullptr;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
    return fail(g_init_error, ACC_EHIP, "hipGetDevice failed (or a device number beyond the library's table)");
  std::lock_guard<std::mutex> lock(g_static_mutex);
  StaticSlot& slot = g_static[dev];
  if (!slot.ptr) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      std::snprintf(g_init_error, 256, "hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
      return ACC_EHIP;
    }
    slot.ptr = p;
  }
  const int32_t rc = init_common(cfg, slot.ptr, (size_t)ACC_STATIC_WORKSPACE_BYTES, q_init_host, hip_stream, out,
                                 "configuration needs more than ACC_STATIC_WORKSPACE_BYTES of workspace: "
                                 "use accordion_init with a caller-owned workspace");
  if (rc != ACC_OK) return rc;
  (*out)->static_dev = dev;
  slot.owner = *out;                                       // an earlier context on this array is now stale
  return ACC_OK;
}

int32_t accordion_destroy(acc_ctx* ctx) {
  if (!ctx) return ACC_EINVAL;
  if (ctx->static_dev >= 0) {
    std::lock_guard<std::mutex> lock(g_static_mutex);
    if (g_static[ctx->static_dev].owner == ctx) g_static[ctx->static_dev].owner = nullptr;
  }
  (void)drain_profile(ctx);
  for (EventPair& p : ctx->spare) {
    (void)hipEventDestroy(p.a);
    (void)hipEventDestroy(p.b);
  }
  delete ctx;
  return ACC_OK;
}

const char* accordion_last_error(const acc_ctx* ctx) { return ctx ? ctx->err : g_init_error; }

int32_t accordion_compress_step(acc_ctx* c, int32_t worker, const float* grad_dev, int32_t phase) {
  ACC_USABLE(c);
  if (c->cfg.method == ACC_BATCH) return fail(c->err, ACC_EINVAL, kBatchCallByCall);
  if (worker < 0 || worker >= c->cfg.n_workers) return fail(c->err, ACC_EINVAL, "worker out of range");
  const uint32_t bit = 1u << worker;
  if (phase == 0) {
    if (!grad_dev) return fail(c->err, ACC_EINVAL, "grad_dev is NULL");
    if (misaligned(grad_dev)) return fail(c->err, ACC_EINVAL, "grad_dev is not 16-byte aligned");
    if (c->agg0) return fail(c->err, ACC_ESTATE, "phase 0 after aggregate(0); finish the step with decompress first");
    if (c->p0_mask & bit) return fail(c->err, ACC_ESTATE, "worker already compressed in this step");
    c->grads.p[worker] = grad_dev;
    const int rc = launch_phase0(c, worker, 1);
    if (rc != ACC_OK) return rc;
    c->in_step = true;
    c->p0_mask |= bit;
    return ACC_OK;
  }
  if (phase == 1) {
    if (c->cfg.method != ACC_POWERSGD) return fail(c->err, ACC_EINVAL, "phase 1 exists for PowerSGD only");
    if (!c->agg0 || c->agg1) return fail(c->err, ACC_ESTATE, "phase 1 needs aggregate(0) first and comes before aggregate(1)");
    if (c->p1_mask & bit) return fail(c->err, ACC_ESTATE, "worker already did phase 1 in this step");
    const int rc = launch_phase1(c, worker, 1);
    if (rc != ACC_OK) return rc;
    c->p1_mask |= bit;
    return ACC_OK;
  }
  return fail(c->err, ACC_EINVAL, "phase must be 0 or 1");
}

int32_t accordion_aggregate(acc_ctx* c, int32_t phase) {
  ACC_USABLE(c);
  if (c->cfg.method == ACC_BATCH) return fail(c->err, ACC_EINVAL, kBatchCallByCall);
  if (phase == 0) {
    if (c->agg0) return fail(c->err, ACC_ESTATE, "aggregate(0) already done");
    if (c->p0_mask != all_workers_mask(c)) return fail(c->err, ACC_ESTATE, "aggregate(0) needs phase 0 of every worker");
    const int rc = launch_agg0(c);
    if (rc != ACC_OK) return rc;
    c->agg0 = true;
    return ACC_OK;
  }
  if (phase == 1) {
    if (c->cfg.method != ACC_POWERSGD) return fail(c->err, ACC_EINVAL, "phase 1 exists for PowerSGD only");
    if (!c->agg0 || c->agg1) return fail(c->err, ACC_ESTATE, "aggregate(1) out of order");
    if (c->p1_mask != all_workers_mask(c)) return fail(c->err, ACC_ESTATE, "aggregate(1) needs phase 1 of every worker");
    const int rc = launch_agg1(c);
    if (rc != ACC_OK) return rc;
    c->agg1 = true;
    return ACC_OK;
  }
  return fail(c->err, ACC_EINVAL, "phase must be 0 or 1");
}

static int32_t decompress_into(acc_ctx* c, const Sink& sink) {
  if (c->cfg.method == ACC_BATCH) return fail(c->err, ACC_EINVAL, kBatchCallByCall);
  if (c->cfg.method == ACC_POWERSGD ? !c->agg1 : !c->agg0)
    return fail(c->err, ACC_ESTATE, "decompress before the aggregation of this step is complete");
  const int rc = launch_decompress(c, sink);
  if (rc != ACC_OK) return rc;
  end_step(c);
  return ACC_OK;
}

int32_t accordion_decompress(acc_ctx* c, float* out_dev) {
  ACC_USABLE(c);
  if (!out_dev) return fail(c->err, ACC_EINVAL, "out_dev is NULL");
  if (misaligned(out_dev)) return fail(c->err, ACC_EINVAL, "out_dev is not 16-byte aligned");
  return decompress_into(c, sink_out(out_dev));
}

int32_t accordion_decompress_update(acc_ctx* c, float* weights_dev, float* velocity_dev, float lr,
                                    float momentum, float weight_decay) {
  ACC_USABLE(c);
  const int rc = check_sgd(c, weights_dev, velocity_dev, lr, momentum, weight_decay);
  if (rc != ACC_OK) return rc;
  return decompress_into(c, Sink{nullptr, weights_dev, velocity_dev, lr, momentum, weight_decay, update_cached(c)});
}

static int32_t step_all_into(acc_ctx* c, const float* const* grads_host_array, const Sink& sink) {
  if (!grads_host_array) return fail(c->err, ACC_EINVAL, "grads_host_array is NULL");
  if (c->in_step) return fail(c->err, ACC_ESTATE, "a call-by-call step is in flight");
  const int W = c->cfg.n_workers;
  for (int w = 0; w < W; ++w) {
    if (!grads_host_array[w]) return fail(c->err, ACC_EINVAL, "a gradient pointer is NULL");
    if (misaligned(grads_host_array[w])) return fail(c->err, ACC_EINVAL, "a gradient pointer is not 16-byte aligned");
  }
  for (int w = 0; w < W; ++w) c->grads.p[w] = grads_host_array[w];
  int rc;
  if (c->cfg.method == ACC_BATCH) {
    rc = launch_batch_micro(c, sink);
  } else if (c->cfg.method == ACC_POWERSGD) {
    rc = launch_phase0(c, 0, W);
    if (rc == ACC_OK) rc = launch_agg0(c);
    if (rc == ACC_OK) rc = launch_phase1(c, 0, W);
    if (rc == ACC_OK) rc = launch_agg1(c);
    if (rc == ACC_OK) rc = launch_decompress(c, sink);
  } else {
    // the compaction of all workers and the mean of their kept values share one pass over Delta
    rc = launch_detector_feed(c, 0);
    if (rc == ACC_OK) rc = launch_topk_select(c, 0, W, 0);
    if (rc == ACC_OK) rc = launch_topk_compact_mean(c, sink);
  }
  end_step(c);
  return rc;
}

int32_t accordion_step_all(acc_ctx* c, const float* const* grads_host_array, float* out_dev) {
  ACC_USABLE(c);
  if (!out_dev) return fail(c->err, ACC_EINVAL, "out_dev is NULL");
  if (misaligned(out_dev)) return fail(c->err, ACC_EINVAL, "out_dev is not 16-byte aligned");
  return step_all_into(c, grads_host_array, sink_out(out_dev));
}

int32_t accordion_step_all_update(acc_ctx* c, const float* const* grads_host_array, float* weights_dev,
                                  float* velocity_dev, float lr, float momentum, float weight_decay) {
  ACC_USABLE(c);
  const int rc = check_sgd(c, weights_dev, velocity_dev, lr, momentum, weight_decay);
  if (rc != ACC_OK) return rc;
  return step_all_into(c, grads_host_array, Sink{nullptr, weights_dev, velocity_dev, lr, momentum, weight_decay, update_cached(c)});
}

int32_t accordion_set_stream(acc_ctx* c, void* hip_stream) {
  ACC_USABLE(c);
  if (c->in_step) return fail(c->err, ACC_ESTATE, "set_stream inside a step");
  const int rc = drain_profile(c);                           // pending timing events belong to the old stream
  if (rc != ACC_OK) return rc;
  c->stream = static_cast<hipStream_t>(hip_stream);
  return ACC_OK;
}

int32_t accordion_detect_regime(acc_ctx* c, float lr_curr, float lr_next) {
  ACC_USABLE(c);
  if (c->in_step) return fail(c->err, ACC_ESTATE, "detect_regime inside a step");
  const Ws& ws = c->ws;
  if (c->cfg.method == ACC_BATCH) {
    ACC_LAUNCH(c, norm_partial_kernel, dim3(ws.n_ftiles), dim3(256), ws);
    ACC_LAUNCH(c, batch_decide_kernel, dim3(1), dim3(256), ws, lr_curr, lr_next);
    return ACC_OK;
  }
  // the sums of squares of A are kept per tile by the pass that adds the gradient; "A <- 0" is a
  // flag that the counting kernel sets once every layer has been decided
  if (c->cfg.detector == ACC_DETECT_MSDR) ACC_LAUNCH(c, msdr_decide_kernel, dim3(ws.L), dim3(64), ws);
  else ACC_LAUNCH(c, regime_decide_kernel, dim3(ws.L), dim3(64), ws, lr_curr, lr_next);
  ACC_LAUNCH(c, recount_words_kernel, dim3(1), dim3(256), ws, (int)c->cfg.method, 1);
  return ACC_OK;
}

int32_t accordion_flush(acc_ctx* c) {
  ACC_USABLE(c);
  if (c->in_step) return fail(c->err, ACC_ESTATE, "flush inside a step");
  return materialise(c);
}

int32_t accordion_reset_accumulator(acc_ctx* c) {
  ACC_USABLE(c);
  if (c->in_step) return fail(c->err, ACC_ESTATE, "reset_accumulator inside a step");
  ACC_LAUNCH(c, zero_accum_kernel, dim3(c->ws.n_ftiles), dim3(256), c->ws, c->cfg.method == ACC_BATCH ? 1 : 0);
  return ACC_OK;
}

int32_t accordion_get_levels(acc_ctx* c, int32_t* levels_host) {
  ACC_USABLE(c);
  if (!levels_host) return fail(c->err, ACC_EINVAL, "levels_host is NULL");
  ACC_HIP(c, hipStreamSynchronize(c->stream));
  ACC_HIP(c, hipMemcpy(levels_host, c->ws.level, 4 * (size_t)c->cfg.n_layers, hipMemcpyDeviceToHost));
  return ACC_OK;
}

int32_t accordion_get_norms(acc_ctx* c, float* old_host, float* curr_host) {
  ACC_USABLE(c);
  if (!old_host || !curr_host) return fail(c->err, ACC_EINVAL, "host pointer is NULL");
  ACC_HIP(c, hipStreamSynchronize(c->stream));
  ACC_HIP(c, hipMemcpy(old_host, c->ws.norm_prev, 4 * (size_t)c->cfg.n_layers, hipMemcpyDeviceToHost));
  ACC_HIP(c, hipMemcpy(curr_host, c->ws.norm_curr, 4 * (size_t)c->cfg.n_layers, hipMemcpyDeviceToHost));
  return ACC_OK;
}

int32_t accordion_get_payload(acc_ctx* c, int32_t worker, int32_t layer, int32_t* idx_host,
                              float* val_host, int64_t capacity, int64_t* count_out) {
  ACC_USABLE(c);
  if (c->cfg.method != ACC_TOPK) return fail(c->err, ACC_EINVAL, "payloads exist for TopK only");
  if (worker < 0 || worker >= c->cfg.n_workers) return fail(c->err, ACC_EINVAL, "worker out of range");
  if (layer < 0 || layer >= c->cfg.n_layers) return fail(c->err, ACC_EINVAL, "layer out of range");
  if (!count_out) return fail(c->err, ACC_EINVAL, "count_out is NULL");
  ACC_HIP(c, hipStreamSynchronize(c->stream));
  SelState s;
  ACC_HIP(c, hipMemcpy(&s, c->ws.sel + (size_t)worker * c->cfg.n_layers + layer, sizeof(s), hipMemcpyDeviceToHost));
  const LayerDev& L = c->plan.layers[layer];
  const int64_t k = std::min<int64_t>(s.k, std::max(L.k[0], L.k[1]));
  *count_out = k;
  if (capacity < k) return fail(c->err, ACC_ENOSPACE, "payload buffers too small");
  if (k == 0) return ACC_OK;
  if (!idx_host || !val_host) return fail(c->err, ACC_EINVAL, "host pointer is NULL");
  const size_t o = (size_t)worker * c->plan.pay_stride + L.pay_off;
  ACC_HIP(c, hipMemcpy(val_host, c->ws.pay_val + o, 4 * (size_t)k, hipMemcpyDeviceToHost));
  const uint32_t n = (uint32_t)L.rows * (uint32_t)L.cols;
  const uint32_t nholes = n - (uint32_t)k;
  if (!payload_has_holes(n, (uint32_t)k)) {
    ACC_HIP(c, hipMemcpy(idx_host, c->ws.pay_idx + o, 4 * (size_t)k, hipMemcpyDeviceToHost));
    return ACC_OK;
  }
  // values + holes: the kept indices are the complement of the (ascending) hole list
  std::vector<int32_t> holes(nholes);
  if (nholes > 0)
    ACC_HIP(c, hipMemcpy(holes.data(), c->ws.pay_idx + o, 4 * (size_t)nholes, hipMemcpyDeviceToHost));
  int64_t out_pos = 0;
  uint32_t h = 0;
  for (uint32_t i = 0; i < n; ++i) {
    if (h < nholes && holes[h] == (int32_t)i) { ++h; continue; }
    if (out_pos < k) idx_host[out_pos] = (int32_t)i;
    ++out_pos;
  }
  if (out_pos != k || h != nholes) return fail(c->err, ACC_EHIP, "hole list of the payload is inconsistent");
  return ACC_OK;
}

int32_t accordion_payload_format(const acc_config* cfg, int32_t layer, int32_t level, int32_t* format,
                                 int64_t* kept, int64_t* words) {
  if (!cfg || !format || !kept || !words) return fail(g_init_error, ACC_EINVAL, "NULL argument");
  Plan p;
  const int rc = make_plan_tiled(cfg, p, g_init_error, false);
  if (rc != ACC_OK) return rc;
  if (cfg->method != ACC_TOPK) return fail(g_init_error, ACC_EINVAL, "payload formats exist for TopK only");
  if (layer < 0 || layer >= cfg->n_layers) return fail(g_init_error, ACC_EINVAL, "layer out of range");
  if (level != 0 && level != 1) return fail(g_init_error, ACC_EINVAL, "level must be 0 or 1");
  const LayerDev& L = p.layers[layer];
  const uint32_t n = (uint32_t)L.rows * (uint32_t)L.cols, k = (uint32_t)L.k[level];
  const bool holes = payload_has_holes(n, k);
  *format = holes ? ACC_PAYLOAD_VALUES_HOLES : ACC_PAYLOAD_INDEX_VALUE;
  *kept = k;
  *words = holes ? (int64_t)n : 2 * (int64_t)k;
  return ACC_OK;
}

int32_t accordion_get_factors(acc_ctx* c, int32_t layer, float* p_hat_host, float* q_host, int32_t* rank_out) {
  ACC_USABLE(c);
  if (c->cfg.method != ACC_POWERSGD) return fail(c->err, ACC_EINVAL, "factors exist for PowerSGD only");
  if (layer < 0 || layer >= c->cfg.n_layers) return fail(c->err, ACC_EINVAL, "layer out of range");
  const LayerDev& L = c->plan.layers[layer];
  if (!L.is_matrix) return fail(c->err, ACC_EINVAL, "layer is not a matrix");
  if (!p_hat_host || !q_host || !rank_out) return fail(c->err, ACC_EINVAL, "host pointer is NULL");
  ACC_HIP(c, hipStreamSynchronize(c->stream));
  int32_t r = 0;
  ACC_HIP(c, hipMemcpy(&r, c->ws.rank_used + layer, 4, hipMemcpyDeviceToHost));
  r = std::max(0, std::min(r, c->plan.rmax));
  *rank_out = r;
  const int rmax = c->plan.rmax;
  std::vector<float> tp((size_t)L.rows * rmax), tq((size_t)L.cols * kMaxRank);
  ACC_HIP(c, hipMemcpy(tp.data(), c->ws.Phat + L.p_off, 4 * tp.size(), hipMemcpyDeviceToHost));
  ACC_HIP(c, hipMemcpy(tq.data(), c->ws.Q + L.q_off, 4 * tq.size(), hipMemcpyDeviceToHost));
  for (int i = 0; i < L.rows; ++i)
    for (int k = 0; k < r; ++k) p_hat_host[(size_t)i * r + k] = tp[(size_t)i * rmax + k];
  for (int j = 0; j < L.cols; ++j)
    for (int k = 0; k < r; ++k) q_host[(size_t)j * r + k] = tq[(size_t)j * kMaxRank + k];
  return ACC_OK;
}

int32_t accordion_payload_words(acc_ctx* c, int64_t* last_step, int64_t* cumulative) {
  ACC_USABLE(c);
  if (!last_step || !cumulative) return fail(c->err, ACC_EINVAL, "host pointer is NULL");
  ACC_HIP(c, hipStreamSynchronize(c->stream));
  unsigned long long w[3] = {0, 0, 0};
  ACC_HIP(c, hipMemcpy(w, c->ws.words, sizeof(w), hipMemcpyDeviceToHost));
  *last_step = (int64_t)w[1];
  *cumulative = (int64_t)w[2];
  return ACC_OK;
}

int32_t accordion_topk_stats(acc_ctx* c, int64_t* restaged_layers, int64_t* swept_layers) {
  ACC_USABLE(c);
  if (c->cfg.method != ACC_TOPK) return fail(c->err, ACC_EINVAL, "TopK statistics exist for TopK only");
  if (!restaged_layers || !swept_layers) return fail(c->err, ACC_EINVAL, "host pointer is NULL");
  ACC_HIP(c, hipStreamSynchronize(c->stream));
  unsigned long long s[2] = {0, 0};
  ACC_HIP(c, hipMemcpy(s, c->ws.stats, sizeof(s), hipMemcpyDeviceToHost));
  *restaged_layers = (int64_t)s[0];
  *swept_layers = (int64_t)s[1];
  return ACC_OK;
}

int32_t accordion_topk_short_lists(acc_ctx* c, int64_t* short_layers) {
  ACC_USABLE(c);
  if (c->cfg.method != ACC_TOPK) return fail(c->err, ACC_EINVAL, "TopK statistics exist for TopK only");
  if (!short_layers) return fail(c->err, ACC_EINVAL, "host pointer is NULL");
  ACC_HIP(c, hipStreamSynchronize(c->stream));
  unsigned long long s = 0;
  ACC_HIP(c, hipMemcpy(&s, c->ws.stats + 2, sizeof(s), hipMemcpyDeviceToHost));
  *short_layers = (int64_t)s;
  return ACC_OK;
}

int32_t accordion_topk_overlap(acc_ctx* c, int32_t worker_a, int32_t worker_b, int64_t* common_host,
                               int64_t* kept_host) {
  ACC_USABLE(c);
  if (c->cfg.method != ACC_TOPK) return fail(c->err, ACC_EINVAL, "overlaps exist for TopK only");
  if (worker_a < 0 || worker_a >= c->cfg.n_workers || worker_b < 0 || worker_b >= c->cfg.n_workers)
    return fail(c->err, ACC_EINVAL, "worker out of range");
  if (!common_host || !kept_host) return fail(c->err, ACC_EINVAL, "host pointer is NULL");
  if (c->in_step) return fail(c->err, ACC_ESTATE, "overlap inside a step");
  if (c->step_id == 2) return fail(c->err, ACC_ESTATE, "no step has run yet: there are no payloads");
  const Ws& ws = c->ws;
  const int L = ws.L;
  ACC_LAUNCH(c, zero_u64_kernel, dim3((L + 255) / 256), dim3(256), ws.overlap, L);
  ACC_LAUNCH(c, topk_overlap_kernel, dim3(ws.n_ftiles), dim3(256), ws, (int)worker_a, (int)worker_b, ws.overlap);
  ACC_HIP(c, hipStreamSynchronize(c->stream));
  std::vector<unsigned long long> cnt((size_t)L);
  std::vector<SelState> sel((size_t)L);
  ACC_HIP(c, hipMemcpy(cnt.data(), ws.overlap, 8 * (size_t)L, hipMemcpyDeviceToHost));
  ACC_HIP(c, hipMemcpy(sel.data(), ws.sel + (size_t)worker_a * L, sizeof(SelState) * (size_t)L, hipMemcpyDeviceToHost));
  for (int i = 0; i < L; ++i) {
    common_host[i] = (int64_t)cnt[(size_t)i];
    kept_host[i] = (int64_t)sel[(size_t)i].k;
  }
  return ACC_OK;
}

int32_t accordion_batch_status(acc_ctx* c, int32_t* level, int32_t* pending_micro_steps,
                               int32_t* last_batch_micro_steps, int64_t* exchanges, int64_t* micro_steps) {
  ACC_USABLE(c);
  if (c->cfg.method != ACC_BATCH) return fail(c->err, ACC_EINVAL, "batch status exists for the batch-size mode only");
  if (!level || !pending_micro_steps || !last_batch_micro_steps || !exchanges || !micro_steps)
    return fail(c->err, ACC_EINVAL, "host pointer is NULL");
  ACC_HIP(c, hipStreamSynchronize(c->stream));
  uint32_t slot[4] = {0, 0, 0, 0};
  unsigned long long s[2] = {0, 0};
  ACC_HIP(c, hipMemcpy(slot, c->ws.bstate + 4 * (c->step_id & 1u), sizeof(slot), hipMemcpyDeviceToHost));
  ACC_HIP(c, hipMemcpy(s, c->ws.stats, sizeof(s), hipMemcpyDeviceToHost));
  ACC_HIP(c, hipMemcpy(level, c->ws.level, 4, hipMemcpyDeviceToHost));
  *pending_micro_steps = (int32_t)slot[0];
  *last_batch_micro_steps = (int32_t)slot[1];
  *exchanges = (int64_t)s[0];
  *micro_steps = (int64_t)s[1];
  return ACC_OK;
}

int32_t accordion_state_bytes(const acc_ctx* c, size_t* out_bytes) {
  if (!c || !out_bytes) return ACC_EINVAL;
  *out_bytes = state_bytes_of(c);
  return ACC_OK;
}

static int32_t state_copy(acc_ctx* c, char* host, bool to_host) {
  const Plan& p = c->plan;
  const size_t N4 = 4 * (size_t)p.N, L4 = 4 * (size_t)c->cfg.n_layers;
  auto cp = [&](void* dev, size_t bytes) -> hipError_t {
    if (bytes == 0) return hipSuccess;
    hipError_t e = to_host ? hipMemcpy(host, dev, bytes, hipMemcpyDeviceToHost)
                           : hipMemcpy(dev, host, bytes, hipMemcpyHostToDevice);
    host += bytes;
    return e;
  };
  for (int w = 0; w < c->cfg.n_workers; ++w) ACC_HIP(c, cp(c->ws.e + (size_t)w * p.e_stride, N4));
  uint32_t fresh = 0;                                        // the window has just restarted: A counts as zero
  if (to_host) ACC_HIP(c, hipMemcpy(&fresh, c->ws.a_fresh, 4, hipMemcpyDeviceToHost));
  if (fresh) {
    std::memset(host, 0, N4);
    host += N4;
  } else {
    ACC_HIP(c, cp(c->ws.A, N4));
  }
  if (c->cfg.method == ACC_POWERSGD) {
    const int rq = copy_q(c, reinterpret_cast<float*>(host), to_host);
    if (rq != ACC_OK) return rq;
    host += 4 * (size_t)p.q_total;
  }
  // batch-size mode: micro-steps summed so far, in the slot the next micro-step reads
  if (c->cfg.method == ACC_BATCH) ACC_HIP(c, cp(c->ws.bstate + 4 * (c->step_id & 1u), 4));
  ACC_HIP(c, cp(c->ws.norm_old, L4));
  ACC_HIP(c, cp(c->ws.has_old, L4));
  ACC_HIP(c, cp(c->ws.level, L4));
  return ACC_OK;
}

int32_t accordion_get_state(acc_ctx* c, void* state_host, size_t bytes) {
  ACC_USABLE(c);
  if (!state_host) return fail(c->err, ACC_EINVAL, "state_host is NULL");
  if (c->in_step) return fail(c->err, ACC_ESTATE, "get_state inside a step");
  if (bytes < state_bytes_of(c)) return fail(c->err, ACC_ENOSPACE, "state buffer too small");
  const int rc = materialise(c);
  if (rc != ACC_OK) return rc;
  ACC_HIP(c, hipStreamSynchronize(c->stream));
  return state_copy(c, static_cast<char*>(state_host), true);
}

int32_t accordion_set_state(acc_ctx* c, const void* state_host, size_t bytes) {
  ACC_USABLE(c);
  if (!state_host) return fail(c->err, ACC_EINVAL, "state_host is NULL");
  if (c->in_step) return fail(c->err, ACC_ESTATE, "set_state inside a step");
  if (bytes < state_bytes_of(c)) return fail(c->err, ACC_ENOSPACE, "state buffer too small");
  // levels must be 0 or 1: they index the per-layer rank / k tables in the kernels
  const size_t L = (size_t)c->cfg.n_layers;
  const int32_t* lv = reinterpret_cast<const int32_t*>(static_cast<const char*>(state_host) + state_bytes_of(c) - 4 * L);
  for (size_t i = 0; i < L; ++i)
    if (lv[i] != 0 && lv[i] != 1) return fail(c->err, ACC_EINVAL, "state holds a level other than 0 or 1");
  if (c->cfg.method == ACC_BATCH) {
    for (size_t i = 1; i < L; ++i)
      if (lv[i] != lv[0]) return fail(c->err, ACC_EINVAL, "batch-size mode has one level for the whole model");
    const int32_t* jp = reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(lv) - 8 * L - 4);
    if (*jp < 0 || *jp >= c->cfg.batch_multiplier)
      return fail(c->err, ACC_EINVAL, "state holds a micro-step count outside [0, batch_multiplier)");
  }
  ACC_HIP(c, hipStreamSynchronize(c->stream));
  const int32_t rc = state_copy(c, const_cast<char*>(static_cast<const char*>(state_host)), false);
  if (rc != ACC_OK) return rc;
  if (c->cfg.method == ACC_POWERSGD)                         // the memory just written is explicit
    ACC_LAUNCH(c, psgd_clear_pending_kernel, dim3(1), dim3(64), c->ws);
  if (c->cfg.method == ACC_TOPK) ACC_LAUNCH(c, topk_clear_pending_kernel, dim3(1), dim3(64), c->ws);
  if (c->plan.r_sq_part.bytes > 0) {                         // the MSDR window restarts with the import
    const int n8 = (int)(c->plan.r_sq_part.bytes / 8);
    ACC_LAUNCH(c, zero_u64_kernel, dim3((n8 + 255) / 256), dim3(256),
               reinterpret_cast<unsigned long long*>(c->ws.sq_part), n8);
  }
  // the imported A: its sums of squares per tile, and it is not "fresh"
  if (c->cfg.method != ACC_BATCH)
    ACC_LAUNCH(c, norm_refresh_kernel, dim3(c->ws.n_ftiles + c->ws.n_mtiles), dim3(256), c->ws);
  ACC_LAUNCH(c, recount_words_kernel, dim3(1), dim3(256), c->ws, (int)c->cfg.method, c->cfg.method != ACC_BATCH ? 0 : -1);
  ACC_HIP(c, hipStreamSynchronize(c->stream));
  return ACC_OK;
}

int32_t accordion_set_profiling(acc_ctx* c, int32_t enable) {
  if (!c) return ACC_EINVAL;
  const int rc = drain_profile(c);
  if (rc != ACC_OK) return rc;
  if (enable && !c->profiling) {
    for (int i = 0; i < ST_COUNT; ++i) { c->stage_ms[i] = 0.0; c->stage_n[i] = 0; }
  }
  c->profiling = (enable == 2 || enable == 3) ? enable : (enable != 0 ? 1 : 0);
  c->prof_tick = 0;
  return ACC_OK;
}

int32_t accordion_get_profile(acc_ctx* c, int32_t stage, double* total_ms, int64_t* launches) {
  if (!c) return ACC_EINVAL;
  if (stage < 0 || stage >= ST_COUNT) return fail(c->err, ACC_EINVAL, "stage out of range");
  if (!total_ms || !launches) return fail(c->err, ACC_EINVAL, "host pointer is NULL");
  const int rc = drain_profile(c);
  if (rc != ACC_OK) return rc;
  *total_ms = c->stage_ms[stage];
  *launches = c->stage_n[stage];
  return ACC_OK;
}

const char* accordion_stage_name(int32_t stage) {
  return (stage >= 0 && stage < ST_COUNT) ? kStageNames[stage] : nullptr;
}

int32_t accordion_probe_copy(float* dst_dev, const float* src_dev, int64_t n, void* hip_stream) {
  if (!dst_dev || !src_dev) return fail(g_init_error, ACC_EINVAL, "probe_copy: pointer is NULL");
  if (misaligned(dst_dev) || misaligned(src_dev)) return fail(g_init_error, ACC_EINVAL, "probe_copy: pointer is not 16-byte aligned");
  if (n <= 0 || n % 4 != 0 || n > (int64_t(1) << 36)) return fail(g_init_error, ACC_EINVAL, "probe_copy: n must be a positive multiple of 4");
  const int64_t nquads = n / 4;
  const int64_t per_block = 256 * kProbeQuadsPerThread;
  const int64_t blocks = (nquads + per_block - 1) / per_block;
  if (blocks > (int64_t(1) << 31) - 1) return fail(g_init_error, ACC_EINVAL, "probe_copy: n too large");
  hipLaunchKernelGGL(probe_copy_kernel, dim3((unsigned)blocks), dim3(256), 0, static_cast<hipStream_t>(hip_stream),
                     reinterpret_cast<float4*>(dst_dev), reinterpret_cast<const float4*>(src_dev), nquads);
  if (hipGetLastError() != hipSuccess) return fail(g_init_error, ACC_EHIP, "probe_copy: launch failed");
  return ACC_OK;
}

}  // extern "C"
