// PowerSGD kernels: error-feedback add fused with P = Delta Q, mean + Gram-Schmidt,
// Q = Delta^T P^, mean of Q, decompress + residual.  All products are HBM-bound at rank <= 4
// (2r flop per 4-byte element), so the kernels stream the matrix once per pass with 16-byte
// accesses and keep the thin factor in registers; no MFMA.
//
// The residual e_w = Delta_w - P^ Q~^T of a step is not written by that step: the error memory
// keeps Delta_w, and the next step's first pass forms e_w on the fly from the previous factors
// (which are still in place: Q~ is the warm start, P^ is overwritten only later in the step)
// before it adds the new gradient.  That saves one read and one write of the matrix per worker
// and step.  psgd_residual_kernel makes the memory explicit when somebody wants to look at it.
//
// Matrix tile: ws.mrows rows x 256 columns, one workgroup of 4 waves.  A lane owns 4 adjacent columns
// and a wave owns rows wave, wave + 4, ...; how a lane reaches its columns depends on the layer (RowMode).
#pragma once
#include "acc_common.h"

namespace acc {

// How the rows of a matrix layer are accessed.  kRowAligned: every row starts on a 16-byte boundary and
// holds whole groups of four.  kRowUnaligned: rows of at least four elements that start anywhere; a
// 16-byte access needs no more than 4-byte alignment on this part (64 lanes still cover one dense
// kilobyte), and the lane whose four columns reach past the row reads the row's last four instead and
// owns only what is its own.  kRowNarrow: fewer than four columns, element by element.
enum RowMode { kRowAligned = 0, kRowUnaligned = 1, kRowNarrow = 2 };

__device__ __forceinline__ int row_mode(const LayerDev& L) {
  return L.vec4 ? kRowAligned : (L.cols >= 4 ? kRowUnaligned : kRowNarrow);
}

// c: first column the lane accesses; own0: first of its four columns that it owns (0: all of them, 4 or
// more: none).  kRowNarrow: c = 0, own0 = number of columns for lane 0 and 0 for the others (owned: the
// columns below it).
struct LaneCols { int c, own0; };

template <int MODE>
__device__ __forceinline__ LaneCols lane_cols(int col0, int lane, int cols) {
  LaneCols lc;
  if (MODE == kRowNarrow) {
    lc.c = 0;
    lc.own0 = lane == 0 ? cols : 0;
  } else {
    const int col = col0 + 4 * lane;
    lc.c = min(col, cols - 4);
    lc.own0 = min(col - lc.c, 4);
  }
  return lc;
}

template <int MODE>
__device__ __forceinline__ bool owns(const LaneCols& lc, int v) {
  return MODE == kRowNarrow ? v < lc.own0 : (MODE == kRowAligned ? lc.own0 == 0 : v >= lc.own0);
}

// Streaming access for what a step touches once, so that Delta stays in the caches between the
// passes (first pass 119 -> 110 us on ResNet-18 shapes, W = 4).
constexpr bool kPsgdStreamG = true;     // gradients: read once per step
constexpr bool kPsgdStreamA = true;     // accumulator: read and written once per step
constexpr bool kPsgdStreamOut = true;   // averaged gradient: written once, read by nobody here

// Rows that do not start on a 16-byte boundary share their first and last cache line with their neighbours, which other
// workgroups read and write: streamed, such a line may have to be fetched twice, plain, the gradients push the error memory out of the caches.
// Since neighbouring tiles meet in one L2 (tile_of_block) streaming wins wherever the error memory is of a size for that to matter: in contexts of
// more than kUStreamBytes of it (the kernels with US) gradients, accumulator, D, weights and velocity of unaligned rows are streamed as those of
// aligned rows always are.  us per step, plain -> streamed, both in the same buffers, three states in turn | one state again and again | one state and 1 GB of
// other traffic between its steps | the same and the gradients written just before.  Odd sizes W = 2 (58 MiB) 92.3 -> 84.6 | 83.0 -> 83.8 | 94.5 -> 95.6 |
// 90.7 -> 93.5, W = 3 (86 MiB) 115.8 -> 108.1 | 104.1 -> 104.8 | 118.7 -> 117.8 | 113.3 -> 116.1, W = 4 138.0 -> 135.4 | 126.3 -> 125.9 | 141.4 -> 140.6 | 136.3 -> 138.9,
// W = 6 (173 MiB) 183.2 -> 179.7 | 170.5 -> 163.0 | 186.6 -> 181.5 | 187.5 -> 178.9, with the update W = 2 112.1 -> 103.5 | 98.8 -> 102.9 | 115.3 -> 116.1 | 111.5 -> 113.5,
// W = 6 201.6 -> 200.6 | 193.4 -> 182.9 | 205.3 -> 203.5 | 205.9 -> 200.3, call by call W = 2 107.7 -> 99.6 | 98.1 -> 99.3 | 112.5 -> 111.7 | 106.7 -> 110.1; ten layers of up to
// 2400 x 2400 W = 2 (57 MiB) 96.0 -> 90.0 | 85.8 -> 89.3 | 100.9 -> 100.1 | 98.2 -> 99.8; 30 of up to 700 x 1000 W = 3 (50 MiB) 79.1 -> 74.0 | 69.3 -> 73.2 | 85.0 -> 83.5 |
// 81.2 -> 82.0.  So above 150 MiB every regime gains; between the line and there a program that goes through several states or lets them grow cold gains 2 to 8 %,
// one whose steps follow each other or whose gradients still lie in the caches loses 1 to 3 % (up to 5 % with nothing between the steps); below the line
// W = 1 (29 MiB) 66.4 -> 62.9 | 59.0 -> 62.3 | 71.6 -> 69.8 | 69.2 -> 69.1, and layers of up to 600 x 800 W = 4 (11 MiB) 36.8 -> 39.3 | 36.3 -> 40.0 | 47.4 -> 45.5 |
// 45.6 -> 44.8.  With the accumulator plain W = 3 112.1 | 103.4 | 116.2 | 115.8, with the gradients plain 114.5 | 105.9 | 121.8 | 114.9.  Kernels of their own, so that small
// sets fetch no more code.
constexpr int64_t kUStreamBytes = int64_t(48) << 20;

// The lane's four elements of a row, loaded whatever the lane owns (every address lies inside the row);
// row: the row's first element.  STREAM: non-temporal.
template <int MODE, bool STREAM = false>
__device__ __forceinline__ void load_row(const float* __restrict__ row, int c, int cols, float (&d)[4]) {
  if (MODE != kRowNarrow) {
    const float4 t = STREAM ? ld16_stream(row + c) : ld16(row + c);
    d[0] = t.x; d[1] = t.y; d[2] = t.z; d[3] = t.w;
  } else {
#pragma unroll
    for (int v = 0; v < 4; ++v) d[v] = row[min(v, cols - 1)];
  }
}

// Stores what the lane owns.  STREAM: non-temporal, on unaligned rows only with US (see kUStreamBytes).
template <int MODE, bool STREAM = false, bool US = false>
__device__ __forceinline__ void store_row(float* __restrict__ row, const LaneCols& lc, const float (&d)[4]) {
  if (MODE == kRowAligned) {
    if (lc.own0 == 0) {
      if (STREAM) st16_stream(row + lc.c, make_float4(d[0], d[1], d[2], d[3]));
      else st16(row + lc.c, make_float4(d[0], d[1], d[2], d[3]));
    }
  } else if (MODE == kRowUnaligned) {
    if (lc.own0 == 0) {
      if (STREAM && US) st16_stream(row + lc.c, make_float4(d[0], d[1], d[2], d[3]));
      else st16(row + lc.c, make_float4(d[0], d[1], d[2], d[3]));
    } else {
#pragma unroll
      for (int v = 1; v < 4; ++v)
        if (v >= lc.own0) row[lc.c + v] = d[v];
    }
  } else {
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (owns<MODE>(lc, v)) row[v] = d[v];
  }
}

// The rows of Q (kMaxRank floats each on the device, zero beyond rmax) of the four columns a lane
// accesses: one aligned 16-byte load per row.  (Sixteen single-word loads at a 64-byte stride between
// lanes kept the texture path busy for longer than the rows of the tile themselves.)  What the lane
// does not own is set to zero by the caller (own_q_rows), once the loads are needed.
template <int MODE>
__device__ __forceinline__ void load_q_rows(const Ws& ws, const LayerDev& L, const LaneCols& lc,
                                            float (&q)[4][kMaxRank]) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int col = MODE == kRowNarrow ? min(v, L.cols - 1) : lc.c + v;
    const float4 t = *reinterpret_cast<const float4*>(ws.Q + L.q_off + (int64_t)col * kMaxRank);
    q[v][0] = t.x; q[v][1] = t.y; q[v][2] = t.z; q[v][3] = t.w;
  }
}

template <int MODE>
__device__ __forceinline__ void own_q_rows(const LaneCols& lc, float (&q)[4][kMaxRank]) {
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int k = 0; k < kMaxRank; ++k) q[v][k] = owns<MODE>(lc, v) ? q[v][k] : 0.f;
}

// ---- phase 0: Delta = g + e (in place of e), A += g (worker 0), P partial = Delta Q ---------

// (double)f, converted where it is written.  The conversions of the lane's rows of Q are loop-invariant and
// were kept across the row loop, 32 registers for what sixteen cheap instructions per row give.
__device__ __forceinline__ double cvt_here(float f) {
  double d;
  asm volatile("v_cvt_f64_f32 %0, %1" : "=v"(d) : "v"(f));
  return d;
}

// One entry of P^ Q~^T: sum_k p[k] q[k] over all kMaxRank columns, where the caller has set p[k]
// to 0 beyond the rank in use (a product with 0 leaves the sum as it is).  Every kernel that
// needs an entry of D forms it with this one expression, so that they agree bit for bit.
__device__ __forceinline__ float low_rank_entry(const float (&p)[kMaxRank], const float (&q)[kMaxRank]) {
  float s = p[0] * q[0];
  s = fmaf(p[1], q[1], s);
  s = fmaf(p[2], q[2], s);
  s = fmaf(p[3], q[3], s);
  return s;
}

// The rows a wave has requested together.  The first pass keeps two of these in flight: while one is
// worked on the next is on its way.  It is bound by memory where the chip is full and by latency where few
// workgroups share it; a wave that waited for each pair of rows before it asked for the next was slower at
// both ends, states beyond the caches: four small layers at W = 2 15.4 us, 8.2 so with 16-row tiles;
// ResNet-18 shapes at W = 4 120 us, 110.7 so (5.2 -> 5.65 TB/s); 40 layers of ragged rows at W = 3, where the
// 16-byte accesses replace 4-byte ones as well, 79.6 us, 71.2 so.
constexpr int kEfRows = 2;
struct EfRows { float g[kEfRows][4], e[kEfRows][4], a[kEfRows][4]; };

// The tile's pointers and lane geometry; Asrc: where A's old value is loaded from (the accumulation
// window has just restarted: the gradient once more, from the cache, and its value is ignored).
struct EfTile {
  const float* g;
  float* e;
  const float* Asrc;
  float* A;
  double* ppart;       // this layer's and chunk's share of the worker's P partials, row 0
  int cols, row_end;
  LaneCols lc;
};

// Rows i0 and i0 + 4 (a row beyond the tile: every lane asks for one and the same 16 bytes of the last
// row and nobody looks at them; a request behind a branch would make every wait a wait for all requests).
template <int MODE, bool HASA, bool US>
__device__ __forceinline__ void ef_load(const EfTile& t, int i0, EfRows& r) {
#pragma unroll
  for (int b = 0; b < kEfRows; ++b) {
    const int i = i0 + 4 * b;
    const int64_t rb = (int64_t)min(i, t.row_end - 1) * t.cols;
    const int c = i < t.row_end ? t.lc.c : 0;
    load_row<MODE, kPsgdStreamG && (MODE == kRowAligned || US)>(t.g + rb, c, t.cols, r.g[b]);
    load_row<MODE>(t.e + rb, c, t.cols, r.e[b]);
    if (HASA) load_row<MODE, kPsgdStreamA && (MODE == kRowAligned || US)>(t.Asrc + rb, c, t.cols, r.a[b]);
  }
}

// rp > 0: the memory still holds the previous step's Delta; its residual is Delta - P^ Q~^T with
// the previous P^ (its rows of the tile are in ps) and Q~ (= the warm start, first rp columns).
template <int R, int MODE, bool HASA, bool US>
__device__ __forceinline__ void ef_rows(const EfTile& t, int i0, EfRows& r, const float (&q)[4][kMaxRank], int rp,
                                        const float (*ps)[kMaxRank], int row0, int rmax, bool a_fresh, double& a_sq) {
  const int lane = threadIdx.x & 63;
  double part[R >= 3 ? 1 : kEfRows][R];                    // a row that does not exist contributes zeros
#pragma unroll
  for (int b = 0; b < (R >= 3 ? 1 : kEfRows); ++b)
#pragma unroll
    for (int k = 0; k < R; ++k) part[b][k] = 0.0;
#pragma unroll
  for (int b = 0; b < kEfRows; ++b) {
    const int i = i0 + 4 * b;
    if (i < t.row_end) {                                   // wave-uniform
      const int64_t rb = (int64_t)i * t.cols;
      if (rp > 0) {                                        // wave-uniform: the pending residual first
        float pp[kMaxRank];
#pragma unroll
        for (int k = 0; k < kMaxRank; ++k) pp[k] = ps[i - row0][k];
#pragma unroll
        for (int v = 0; v < 4; ++v) r.e[b][v] = r.e[b][v] - low_rank_entry(pp, q[v]);
      }
      float d[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) d[v] = owns<MODE>(t.lc, v) ? r.g[b][v] + r.e[b][v] : 0.f;
      store_row<MODE>(t.e + rb, t.lc, d);
      if (HASA) {
        float a[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) a[v] = owns<MODE>(t.lc, v) ? (a_fresh ? 0.f : r.a[b][v]) + r.g[b][v] : 0.f;
        store_row<MODE, kPsgdStreamA, US>(t.A + rb, t.lc, a);
#pragma unroll
        for (int v = 0; v < 4; ++v) a_sq += (double)a[v] * (double)a[v];
      }
      // the lane's share of the chunk's share of P_w's row, in fp64: products of fp32 values are
      // exact there, the sums carry an error far below the fp32 rounding of the stored P_w
      double dd[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) dd[v] = (double)d[v];
#pragma unroll
      for (int k = 0; k < R; ++k) {
        double s = dd[0] * cvt_here(q[0][k]);
        s = fma(dd[1], cvt_here(q[1][k]), s);
        s = fma(dd[2], cvt_here(q[2][k]), s);
        s = fma(dd[3], cvt_here(q[3][k]), s);
        part[R >= 3 ? 0 : b][k] = s;
      }
      if constexpr (R >= 3) {
        // Three or four values per row: folded row by row (as many instructions as folding both
        // rows together, half the registers).  The lower 32 lanes end with columns 0 and 1 of
        // P (even / odd rows of 16 lanes), the upper 32 with columns 2 and 3.
        const double y02 = fold32_d(part[0][0], part[0][2]);
        const double y13 = fold32_d(part[0][1], R > 3 ? part[0][R - 1] : 0.0);
        const double y = row_sum_d(fold16_d(y02, y13));
        const int kcol = 2 * (lane >> 5) + ((lane >> 4) & 1);
        if ((lane & 15) == 0 && kcol < R) t.ppart[(int64_t)i * rmax + kcol] = y;
      }
    }
  }
  if constexpr (R <= 2) {
    // One or two values per row: both rows' values are folded over the wave together (the upper
    // 32 lanes keep the second row, the odd rows of 16 lanes the second column of P), so that
    // the lane exchanges of a full butterfly per value (27 instructions each in fp64) shrink
    // to about 20 for all of them.
    const int hb = lane >> 5, rp16 = (lane >> 4) & 1;       // which row of the pair / which column
    const int i_mine = i0 + 4 * hb;
    double* dst = t.ppart + (int64_t)i_mine * rmax;
    const bool writer = (lane & 15) == 0 && i_mine < t.row_end;
    if constexpr (R == 1) {
      double y = fold32_d(part[0][0], part[1][0]);
      y = row_sum_d(y);
      y = fold16_d(y, y);                                    // both rows of 16 lanes of a half
      if (writer && rp16 == 0) dst[0] = y;
    } else {
      const double y0 = fold32_d(part[0][0], part[1][0]), y1 = fold32_d(part[0][1], part[1][1]);
      const double y = row_sum_d(fold16_d(y0, y1));         // even rows of 16 lanes: column 0, odd rows: column 1
      if (writer) dst[rp16] = y;
    }
  }
}

template <int R, int MODE, bool HASA, bool US>
__device__ __forceinline__ double ef_loop(const EfTile& t, int i0, EfRows& cur, const float (&q)[4][kMaxRank], int rp,
                                          const float (*ps)[kMaxRank], int row0, int rmax, bool a_fresh) {
  double a_sq = 0.0;     // worker 0: the lane's share of the tile's sum of squares of A
  for (; i0 < t.row_end; i0 += 4 * kEfRows) {
    EfRows nxt;
    ef_load<MODE, HASA, US>(t, i0 + 4 * kEfRows, nxt);
    ef_rows<R, MODE, HASA, US>(t, i0, cur, q, rp, ps, row0, rmax, a_fresh, a_sq);
    cur = nxt;
  }
  return a_sq;
}

template <int MODE, bool HASA, bool US>
__device__ __forceinline__ void ef_p_tile(const Ws& ws, const LayerDev& L, const MatTile& mt, const float* __restrict__ g,
                                          float* __restrict__ e, double* __restrict__ ppart, int level, int rp_used,
                                          uint32_t pending, uint32_t fresh, int w, float (*ps)[kMaxRank], double* red4) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  EfTile t;
  const bool a_fresh = HASA && fresh != 0u;                // uniform over the workgroup
  t.lc = lane_cols<MODE>(mt.col0, lane, L.cols);
  t.cols = L.cols;
  t.row_end = min(mt.row0 + ws.mrows, L.rows);
  t.g = g + L.offset;
  t.e = e + L.offset;
  t.A = HASA ? ws.A + L.offset : nullptr;
  t.Asrc = a_fresh ? t.g : t.A;
  t.ppart = ppart + L.ppart_off + (int64_t)(mt.col0 / kMatCols) * L.rows * ws.rmax;
  // requested together: the first rows, Q's rows, and the previous P^ rows of the tile (for LDS)
  const int i0 = mt.row0 + wave;
  EfRows first;
  ef_load<MODE, HASA, US>(t, i0, first);
  float q[4][kMaxRank];
  load_q_rows<MODE>(ws, L, t.lc, q);
  const int pr = threadIdx.x >> 2, pk = threadIdx.x & 3;
  const float ph = ws.Phat[L.p_off + (int64_t)min(mt.row0 + pr, L.rows - 1) * ws.rmax + min(pk, ws.rmax - 1)];
  const int rp = ((pending >> w) & 1u) ? rp_used : 0;      // rank of the previous step's factors
  const int r = level ? L.rank[1] : L.rank[0];
  ps[pr][pk] = pk < rp ? ph : 0.f;
  own_q_rows<MODE>(t.lc, q);
  __syncthreads();
  double a_sq;
  switch (r) {
    case 1: a_sq = ef_loop<1, MODE, HASA, US>(t, i0, first, q, rp, ps, mt.row0, ws.rmax, a_fresh); break;
    case 2: a_sq = ef_loop<2, MODE, HASA, US>(t, i0, first, q, rp, ps, mt.row0, ws.rmax, a_fresh); break;
    case 3: a_sq = ef_loop<3, MODE, HASA, US>(t, i0, first, q, rp, ps, mt.row0, ws.rmax, a_fresh); break;
    default: a_sq = ef_loop<4, MODE, HASA, US>(t, i0, first, q, rp, ps, mt.row0, ws.rmax, a_fresh); break;
  }
  if (HASA) {
    const double tsum = block_sum4_d(a_sq, red4);
    if (threadIdx.x == 0) ws.norm_part_m[mt.id] = tsum;
  }
}

// *ws.pending: bit w set = worker w's memory holds the previous Delta (see the top of this file).
// The mask lives on the device (set by the decompress pass, cleared when the residual is written
// out), so a captured graph of a step stays valid whatever happens between its replays.
template <bool US>
__device__ __forceinline__ void ef_p_body(const Ws& ws, const GradPtrs& gp, int w0) {
  __shared__ float ps[kMatRows][kMaxRank];
  __shared__ double red4[4];
  const int w = w0 + blockIdx.y;
  const float* __restrict__ g = gp.p[w];
  float* __restrict__ e = ws.e + (int64_t)w * ws.e_stride;
  if ((int)blockIdx.x >= ws.n_mtiles) {
    // 1-D layers: only the accumulation A += g of worker 0 happens here (and the tile's sum of squares)
    if (w != 0) return;
    const bool a_fresh = *ws.a_fresh != 0u;
    const int tile_id = ws.vectiles[blockIdx.x - ws.n_mtiles];
    const FlatTile ft = ws.ftiles[tile_id];
    const LayerDev& L = ws.layers[ft.layer];
    const TileGeom tg = tile_geom(L, ft);
    double a_sq = 0.0;
    for (int q = threadIdx.x; q < tg.nquads; q += kFlatThreads) {
      const int64_t base = tg.a0 + 4 * (int64_t)q;
      float4 a = a_fresh ? make_float4(0.f, 0.f, 0.f, 0.f) : ld_quad(ws.A, base, tg.hi);
      const float4 gv = ld_quad(g, base, tg.hi);
      a.x += gv.x; a.y += gv.y; a.z += gv.z; a.w += gv.w;
      st_quad(ws.A, base, tg.hi, a);
      a_sq += sq4(a);                                        // elements outside the tile were loaded as zeros
    }
    a_sq = block_sum4_d(a_sq, red4);
    if (threadIdx.x == 0) ws.norm_part[tile_id] = a_sq;
    return;
  }
  const uint32_t pending = *ws.pending, fresh = *ws.a_fresh;
  const MatTile t = ws.mtiles[blockIdx.x];
  const LayerDev& L = ws.layers[t.layer];
  const int level = ws.level[t.layer], rp_used = ws.rank_used[t.layer];
  double* ppart = ws.Ppart + (int64_t)w * ws.ppart_stride;
  // worker 0 also updates A
  switch (2 * row_mode(L) + (w == 0 ? 1 : 0)) {
    case 2 * kRowAligned: ef_p_tile<kRowAligned, false, false>(ws, L, t, g, e, ppart, level, rp_used, pending, fresh, w, ps, red4); break;
    case 2 * kRowAligned + 1: ef_p_tile<kRowAligned, true, false>(ws, L, t, g, e, ppart, level, rp_used, pending, fresh, w, ps, red4); break;
    case 2 * kRowUnaligned: ef_p_tile<kRowUnaligned, false, US>(ws, L, t, g, e, ppart, level, rp_used, pending, fresh, w, ps, red4); break;
    case 2 * kRowUnaligned + 1: ef_p_tile<kRowUnaligned, true, US>(ws, L, t, g, e, ppart, level, rp_used, pending, fresh, w, ps, red4); break;
    case 2 * kRowNarrow: ef_p_tile<kRowNarrow, false, false>(ws, L, t, g, e, ppart, level, rp_used, pending, fresh, w, ps, red4); break;
    default: ef_p_tile<kRowNarrow, true, false>(ws, L, t, g, e, ppart, level, rp_used, pending, fresh, w, ps, red4); break;
  }
}

__global__ __launch_bounds__(256) void psgd_ef_p_kernel(const Ws ws, const GradPtrs gp, int w0) { ef_p_body<false>(ws, gp, w0); }

__global__ __launch_bounds__(256) void psgd_ef_p_stream_kernel(const Ws ws, const GradPtrs gp, int w0) { ef_p_body<true>(ws, gp, w0); }

// ---- aggregate 0: P_bar = mean over workers (and column chunks), Gram-Schmidt -----------
//
// Precision.  Gram-Schmidt carries an error of its input into column k multiplied by the
// condition number of P_bar, and P_bar = Delta_bar Q is as badly conditioned as the warm start Q
// happens to be (a 2 x 2 Q with condition 2000 occurs among random starts).  So the whole chain
// that leads to P^ runs in fp64 and rounds to fp32 exactly where the method stores an fp32
// quantity: the products Delta Q are accumulated in fp64 per 256-column chunk (first pass), a
// worker's chunks are summed in fp64 and rounded (P_w), the workers' P_w are summed in fp64,
// divided by W and rounded (P_bar), the projections and norms of Gram-Schmidt are fp64 and the
// finished column is rounded (P^).  The passes over Delta are bound by memory either way.

constexpr int kOrthThreads = 1024;
constexpr int kOrthWaves = kOrthThreads / kWave;

// sum_w fl32(sum_b partial[w][b]) in fp64 (P_w and Q_w are fp32 quantities): workers and blocks in index
// order, U partial sums requested together, so that a thread waits for few round trips.  U blocks of one worker
// are a stretch of one stride; where fewer are left, the positions are walked one by one over the workers' ends,
// and the last one is asked for again instead of one beyond it.  Everything but src is wave-uniform.
template <int U>
__device__ __forceinline__ double sum_partials_by(const double* __restrict__ src, int64_t wstride, int64_t bstride, int W,
                                                  int nb) {
  const int64_t to_next_worker = wstride - (int64_t)(nb - 1) * bstride;
  double total = 0.0, s = 0.0;
  int64_t at = 0;                                          // position of partial[w][b]
  int w = 0, b = 0;
  while (w < W) {
    double v[U];
    if (b + U <= nb) {
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = src[at + u * bstride];
#pragma unroll
      for (int u = 0; u < U; ++u) s += v[u];
      b += U;
      at += U * bstride;
      if (b == nb) { total += (double)(float)s; s = 0.0; b = 0; ++w; at += to_next_worker - bstride; }
    } else {
      int lw = w, lb = b;                                  // next one to request
#pragma unroll
      for (int u = 0; u < U; ++u) {
        v[u] = src[at];
        if (lb + 1 < nb) { ++lb; at += bstride; }
        else if (lw + 1 < W) { lb = 0; ++lw; at += to_next_worker; }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (w < W) {
          s += v[u];
          if (++b == nb) { total += (double)(float)s; s = 0.0; b = 0; ++w; }
        }
      }
    }
  }
  return total;
}

// Bound by its round trips: eight requests at a time, fewer where there are fewer partial sums in all.  (Walked one by
// one throughout, the address arithmetic was a third of the time on many blocks, and eight requests for a single
// partial sum two thirds of it.  Mean of Q, us: 782 blocks at W = 4 293, 141 so; one block of 2 M columns 54.2, 19.5;
// mean of P: 10 rows of 36 chunks at W = 16 17.7, 11.7.  Sixteen and more at a time are 1 to 3 us slower per step.)
constexpr int kPartLoads = 8;
__device__ __forceinline__ double sum_partials(const double* __restrict__ src, int64_t wstride, int64_t bstride, int W,
                                               int nb) {
  const int64_t n = (int64_t)W * nb;
  if (n == 1) return 0.0 + (double)(float)(0.0 + src[0]);   // the sums start from +0
  if (n == 2) return sum_partials_by<2>(src, wstride, bstride, W, nb);
  if (n <= 4) return sum_partials_by<4>(src, wstride, bstride, W, nb);
  return sum_partials_by<kPartLoads>(src, wstride, bstride, W, nb);
}

// 1-D layers are sent raw: mean over the workers in worker order (fp64, rounded once) of one flat tile.
// Four elements per thread and four workers' gradients are requested together: they come from memory,
// and one after the other they were what the orthogonalisation launch waited for (3 of its 7 us).
__device__ __forceinline__ void vec_mean_tile(const Ws& ws, const GradPtrs& gp, int vt) {
  constexpr int E = 4, U = 4;
  const FlatTile ft = ws.ftiles[ws.vectiles[vt]];
  const LayerDev& L = ws.layers[ft.layer];
  const int64_t base = L.offset + ft.start;
  float* __restrict__ mean = ws.vecmean + L.vec_off + ft.start;
  for (int i0 = threadIdx.x; i0 < ft.count; i0 += E * blockDim.x) {
    double s[E];
#pragma unroll
    for (int x = 0; x < E; ++x) s[x] = 0.0;
    for (int w0 = 0; w0 < ws.W; w0 += U) {
      float g[U][E];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int x = 0; x < E; ++x)
          g[u][x] = gp.p[min(w0 + u, ws.W - 1)][base + min(i0 + x * (int)blockDim.x, ft.count - 1)];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int x = 0; x < E; ++x)
          if (w0 + u < ws.W) s[x] += (double)g[u][x];
    }
#pragma unroll
    for (int x = 0; x < E; ++x)
      if (i0 + x * (int)blockDim.x < ft.count) mean[i0 + x * blockDim.x] = (float)(s[x] / (double)ws.W);
  }
}

// P_bar[i][k] = fl32( (sum_w fl32(sum_c partial[w][c][i][k])) / W ).
// One workgroup per 16 rows of a layer; thread = (share, row, column of P), four shares per entry:
// share s sums the workers s, s + 4, ... (each worker's chunks in fp64, rounded to the fp32 value
// P_w), then the four shares are added in order.  Many small workgroups: the partial sums of a
// layer (1.2 MB for the largest ResNet-18 layer at four workers) are read by many compute units
// at once, and a thread waits for few dependent batches of loads.  Where a layer has few of them
// (Ws::pmean_in_orth) the orthogonalisation sums them itself and this launch is left out.
constexpr int kPmeanRows = 16;

__global__ __launch_bounds__(256) void psgd_pmean_kernel(const Ws ws, const GradPtrs gp) {
  __shared__ double share_sum[4][kPmeanRows * 4];
  if ((int)blockIdx.x >= ws.n_ptiles) {
    vec_mean_tile(ws, gp, blockIdx.x - ws.n_ptiles);
    return;
  }
  const PTile t = ws.ptiles[blockIdx.x];
  const LayerDev& L = ws.layers[t.layer];
  const int level = ws.level[t.layer];
  const int r = level ? L.rank[1] : L.rank[0];
  const int share = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), slot = threadIdx.x & 63;
  const int i = t.row0 + (slot >> 2), k = slot & 3;
  const bool live = i < L.rows && k < r;
  double total = 0.0;
  if (live && share < ws.W) {
    const double* base = ws.Ppart + L.ppart_off + (int64_t)i * ws.rmax + k + (int64_t)share * ws.ppart_stride;
    total = sum_partials(base, 4 * ws.ppart_stride, (int64_t)L.rows * ws.rmax, (ws.W - share + 3) >> 2, L.n_colchunks);
  }
  share_sum[share][slot] = total;
  __syncthreads();
  if (share == 0 && live) {
    const double sum = ((share_sum[0][slot] + share_sum[1][slot]) + share_sum[2][slot]) + share_sum[3][slot];
    ws.Phat[L.p_off + (int64_t)i * ws.rmax + k] = (float)(sum / (double)ws.W);
  }
}

// Sums over the threads of the orthogonalisation workgroup of M values each, the same for every
// thread.  `slot` alternates between calls so that one barrier per call is enough.
// Only the first nwaves waves of the workgroup are still running (the others have left).
template <int M>
__device__ __forceinline__ void block_sum_orth(double (&v)[M], double (*red)[kOrthWaves][kMaxRank], int& slot, int nwaves) {
#pragma unroll
  for (int m = 0; m < M; ++m) v[m] = wave_sum_d(v[m]);
  if (nwaves == 1) return;
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int m = 0; m < M; ++m) red[slot][wave][m] = v[m];
  }
  __syncthreads();
  // every row of 16 lanes reads the (at most sixteen) waves' sums and adds them up by lane exchanges: one
  // LDS round trip instead of one per wave
  const int from = threadIdx.x & (kOrthWaves - 1);
  static_assert(kOrthWaves == 16, "a row of lanes holds one sum per wave");
#pragma unroll
  for (int m = 0; m < M; ++m) v[m] = row_sum_d(from < nwaves ? red[slot][from][m] : 0.0);
  slot ^= 1;
}

// Modified Gram-Schmidt of column K and what it takes from the columns after it: |v_K|^2 and the
// products v_K . v_j come out of one reduction over the workgroup (r of them instead of r (r + 1) / 2:
// the reductions, each a barrier, are what this kernel spends its time on).
template <int R, int K, class SumF>
__device__ __forceinline__ void orth_column(double (&v)[R], SumF sum) {
  if constexpr (K < R) {
    double s[R - K];
#pragma unroll
    for (int j = K; j < R; ++j) s[j - K] = v[K] * v[j];
    sum(s);
    const double nrm = sqrt(s[0]);
    const bool some = nrm > 0.0;
    v[K] = some ? v[K] / nrm : 0.0;
#pragma unroll
    for (int j = K + 1; j < R; ++j) v[j] = fma(some ? -(s[j - K] / nrm) : 0.0, v[K], v[j]);
    orth_column<R, K + 1>(v, sum);
  }
}

// Modified Gram-Schmidt over the r columns of P_bar (fp32), in column order, in
// fp64; a column of zero length stays zero; P^ (fp32) replaces P_bar.  Layers of up to
// kOrthThreads rows live in registers, one row per thread; taller ones in an fp64 copy in
// global memory (each thread only ever touches its own rows).  P_bar is in ws.Phat, or -- Ws::pmean_in_orth,
// layers of up to kOrthThreads rows -- summed up here from the partials (pbar: LDS).
template <int R>
__device__ void orth_layer(const Ws& ws, const LayerDev& L, double (*red)[kOrthWaves][kMaxRank], float* pbar) {
  const int n = L.rows;
  const int tid = threadIdx.x;
  float* ph = ws.Phat + L.p_off;
  int slot = 0;
  if (n <= kOrthThreads) {
    if (ws.pmean_in_orth) {                                  // uniform
      for (int x = tid; x < n * R; x += kOrthThreads) {
        const double* src = ws.Ppart + L.ppart_off + (int64_t)(x / R) * ws.rmax + x % R;
        pbar[x] = (float)(sum_partials(src, ws.ppart_stride, (int64_t)n * ws.rmax, ws.W, L.n_colchunks) / (double)ws.W);
      }
      __syncthreads();
    }
    const int nwaves = (n + kWave - 1) / kWave;
    if (tid >= nwaves * kWave) return;                       // whole waves
    const bool holder = tid < n;
    double v[R];
    if (ws.pmean_in_orth) {
#pragma unroll
      for (int k = 0; k < R; ++k) v[k] = holder ? (double)pbar[tid * R + k] : 0.0;
    } else {
#pragma unroll
      for (int k = 0; k < R; ++k) v[k] = holder ? (double)ph[(int64_t)tid * ws.rmax + k] : 0.0;
    }
    orth_column<R, 0>(v, [&](auto& s) { block_sum_orth(s, red, slot, nwaves); });
    if (holder) {
#pragma unroll
      for (int k = 0; k < R; ++k) ph[(int64_t)tid * ws.rmax + k] = (float)v[k];
    }
  } else {
    double* pw = ws.Pwork + L.p_off;
    for (int i = tid; i < n; i += kOrthThreads)
#pragma unroll
      for (int k = 0; k < R; ++k) pw[(int64_t)i * ws.rmax + k] = (double)ph[(int64_t)i * ws.rmax + k];
    for (int k = 0; k < R; ++k) {
      for (int j = 0; j < k; ++j) {
        double d[1] = {0.0};
        for (int i = tid; i < n; i += kOrthThreads)
          d[0] = fma(pw[(int64_t)i * ws.rmax + j], pw[(int64_t)i * ws.rmax + k], d[0]);
        block_sum_orth(d, red, slot, kOrthWaves);
        for (int i = tid; i < n; i += kOrthThreads)
          pw[(int64_t)i * ws.rmax + k] = fma(-d[0], pw[(int64_t)i * ws.rmax + j], pw[(int64_t)i * ws.rmax + k]);
      }
      double nn[1] = {0.0};
      for (int i = tid; i < n; i += kOrthThreads) {
        const double x = pw[(int64_t)i * ws.rmax + k];
        nn[0] = fma(x, x, nn[0]);
      }
      block_sum_orth(nn, red, slot, kOrthWaves);
      const double nrm = sqrt(nn[0]);
      for (int i = tid; i < n; i += kOrthThreads) {
        const double x = (nrm > 0.0) ? pw[(int64_t)i * ws.rmax + k] / nrm : 0.0;
        pw[(int64_t)i * ws.rmax + k] = x;
        ph[(int64_t)i * ws.rmax + k] = (float)x;
      }
    }
  }
}

__global__ __launch_bounds__(kOrthThreads) void psgd_orth_kernel(const Ws ws, const GradPtrs gp) {
  __shared__ double red[2][kOrthWaves][kMaxRank];
  __shared__ float pbar[kOrthThreads * kMaxRank];
  // worker 0's first pass has added its gradient to A: the window is no longer fresh
  if (blockIdx.x == 0 && threadIdx.x == 0) *ws.a_fresh = 0u;
  if ((int)blockIdx.x >= ws.n_mat) {
    vec_mean_tile(ws, gp, blockIdx.x - ws.n_mat);
    return;
  }
  const int li = ws.matlayers[blockIdx.x];
  const LayerDev& L = ws.layers[li];
  const int level = ws.level[li];
  const int r = level ? L.rank[1] : L.rank[0];
  if (threadIdx.x == 0) ws.rank_used[li] = r;
  switch (r) {
    case 1: orth_layer<1>(ws, L, red, pbar); break;
    case 2: orth_layer<2>(ws, L, red, pbar); break;
    case 3: orth_layer<3>(ws, L, red, pbar); break;
    default: orth_layer<4>(ws, L, red, pbar); break;
  }
}

// ---- phase 1: Q partial = Delta^T P^ over one block of Ws::qrows rows ------------------------
//
// fp64 accumulation here too: where the memory dominates gradient + memory, Delta^T p^_k cancels
// to a small fraction of its terms for the columns of P^ that the new gradient determines, and an
// fp32 sum would lose those columns of Q (the oracle's contraction is fp64, rounded once).

// Tile: ws.qrows rows x 256 columns, one workgroup of 4 waves; a wave owns rows wave, wave + 4, ...
// and keeps the sums of its four columns per lane in registers; the four waves' sums meet in LDS.
// Bound by memory, or by latency where few workgroups share the chip, like the first pass: the next batch of
// rows is requested before the current one is used (ResNet-18 shapes 39.1 -> 32.0 us at W = 4, 16.0 -> 10.0 at
// W = 1; 2 rows per batch: 2 us more per step at W = 4; 8: within 1 us, for 32 more registers).  Rows beyond the tile
// are asked for only where a batch straddles its end, not by the first batch nor by one after the last (100 layers of
// 2 x 20000 at W = 4 118.5 -> 112.6 us, 200 of 512 x 9 33.0 -> 30.9).
constexpr int kQBatch = 4;   // rows a wave requests together; two such batches are in flight

// STREAM: Delta is requested with the streaming hint.  It is not read again before the next step, and a plain
// read leaves it in the Infinity Cache, dirty, for the next passes to evict; read so, its lines go back to memory here, at next
// to no cost.  Which rows of which contexts: see QStream.
// (From clamped addresses: a request behind a branch would make every wait in the loop a wait for all of them.)
template <int MODE, bool STREAM>
__device__ __forceinline__ void q_load(const float* __restrict__ e, int cols, int row_end, const LaneCols& lc, int i0,
                                       float (&d)[kQBatch][4]) {
#pragma unroll
  for (int b = 0; b < kQBatch; ++b) {
    const int i = i0 + 4 * b;                                // beyond the tile: one 16-byte address, see ef_load
    load_row<MODE, STREAM>(e + (int64_t)min(i, row_end - 1) * cols, i < row_end ? lc.c : 0, cols, d[b]);
  }
}

template <int R, int MODE, bool STREAM>
__device__ __forceinline__ void q_loop(const Ws& ws, const LayerDev& L, const MatTile& t, const float* __restrict__ e,
                                       double* __restrict__ qpart, double (*red)[16][64], const float (*ps)[kMaxRank],
                                       const LaneCols& lc, int row_end, float (&cur)[kQBatch][4]) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double acc[4][R];
#pragma unroll
  for (int v = 0; v < 4; ++v)
#pragma unroll
    for (int k = 0; k < R; ++k) acc[v][k] = 0.0;
  auto use = [&](int i0) {
#pragma unroll
    for (int b = 0; b < kQBatch; ++b) {
      const int i = i0 + 4 * b;
      if (i < row_end) {                                     // wave-uniform
        double p[R], dd[4];
#pragma unroll
        for (int k = 0; k < R; ++k) p[k] = (double)ps[i - t.row0][k];
#pragma unroll
        for (int v = 0; v < 4; ++v) dd[v] = (double)cur[b][v];
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int k = 0; k < R; ++k) acc[v][k] = fma(dd[v], p[k], acc[v][k]);
      }
    }
  };
  int i0 = t.row0 + wave;
  for (; i0 + 4 * kQBatch < row_end; i0 += 4 * kQBatch) {
    float nxt[kQBatch][4];
    q_load<MODE, STREAM>(e, L.cols, row_end, lc, i0 + 4 * kQBatch, nxt);
    use(i0);
#pragma unroll
    for (int b = 0; b < kQBatch; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) cur[b][v] = nxt[b][v];
  }
  use(i0);
  // the four waves' sums, in the fixed order (wave 0 + wave 2) + (wave 1 + wave 3)
  if (wave >= 2) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int k = 0; k < R; ++k) red[wave - 2][v * R + k][lane] = acc[v][k];
  }
  __syncthreads();
  if (wave < 2) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int k = 0; k < R; ++k) acc[v][k] += red[wave][v * R + k][lane];
  }
  __syncthreads();
  if (wave < 2) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int k = 0; k < R; ++k) red[wave][v * R + k][lane] = acc[v][k];
  }
  __syncthreads();
  // thread (wave, lane) finishes column slot v = wave of that lane, if the lane owns it
  {
    const int v = wave;
    const int cv = lc.c + v;
    if (owns<MODE>(lc, v)) {
      const int rb = t.row0 / ws.qrows;
      double* dst = qpart + L.qpart_off + ((int64_t)rb * L.cols + cv) * ws.rmax;
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const int s = v * R + k;
        dst[k] = red[0][s][lane] + red[1][s][lane];
      }
    }
  }
}

template <int MODE, bool STREAM>
__device__ __forceinline__ void q_tile(const Ws& ws, const LayerDev& L, const MatTile& t, const float* __restrict__ e_w,
                                       double* __restrict__ qpart, int level, double (*red)[16][64],
                                       float (*ps)[kMaxRank]) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const LaneCols lc = lane_cols<MODE>(t.col0, lane, L.cols);
  const float* __restrict__ e = e_w + L.offset;
  const int row_end = min(t.row0 + ws.qrows, L.rows);
  // the first rows of Delta and the tile's rows of P^ (for LDS) are requested together; the wait for the latter
  // covers the former, so branches cost nothing here
  float first[kQBatch][4];
#pragma unroll
  for (int b = 0; b < kQBatch; ++b) {
    const int i = t.row0 + wave + 4 * b;
    if (i < row_end) load_row<MODE, STREAM>(e + (int64_t)i * L.cols, lc.c, L.cols, first[b]);   // wave-uniform
  }
  const int r = level ? L.rank[1] : L.rank[0];
  for (int s = threadIdx.x; s < ws.qrows * kMaxRank; s += 256) {
    const int pr = s >> 2, pk = s & 3;
    const int i = t.row0 + pr;
    ps[pr][pk] = (i < L.rows && pk < r) ? ws.Phat[L.p_off + (int64_t)i * ws.rmax + pk] : 0.f;
  }
  __syncthreads();
  switch (r) {
    case 1: q_loop<1, MODE, STREAM>(ws, L, t, e, qpart, red, ps, lc, row_end, first); break;
    case 2: q_loop<2, MODE, STREAM>(ws, L, t, e, qpart, red, ps, lc, row_end, first); break;
    case 3: q_loop<3, MODE, STREAM>(ws, L, t, e, qpart, red, ps, lc, row_end, first); break;
    default: q_loop<4, MODE, STREAM>(ws, L, t, e, qpart, red, ps, lc, row_end, first); break;
  }
}

// Which rows the right product reads with the streaming hint (chosen on the host, see make_plan_tiled).
// A row that does not start on a cache line shares its first and last line with its neighbours, which other waves and other workgroups
// read: streamed, the line has to be fetched again, so such rows are streamed only where the error memory would not stay in the
// cache in any case.
enum QStream { kQPlain = 0, kQAlignedRows = 1, kQAllRows = 2 };

template <int QS>
__global__ __launch_bounds__(256) void psgd_q_kernel(const Ws ws, int w0) {
  __shared__ double red[2][16][64];
  __shared__ float ps[kQRows][kMaxRank];
  const int w = w0 + blockIdx.y;
  const MatTile t = ws.qmtiles[blockIdx.x];
  const LayerDev& L = ws.layers[t.layer];
  const int level = ws.level[t.layer];
  const float* __restrict__ e = ws.e + (int64_t)w * ws.e_stride;
  double* qpart = ws.Qpart + (int64_t)w * ws.qpart_stride;
  switch (row_mode(L)) {
    case kRowAligned: q_tile<kRowAligned, (QS >= kQAlignedRows)>(ws, L, t, e, qpart, level, red, ps); break;
    case kRowUnaligned: q_tile<kRowUnaligned, (QS >= kQAllRows)>(ws, L, t, e, qpart, level, red, ps); break;
    default: q_tile<kRowNarrow, false>(ws, L, t, e, qpart, level, red, ps); break;
  }
}

// ---- aggregate 1: Q_bar = mean over workers of (sum over row blocks) -------------------------

// Q_bar[c][k] = fl32( (sum_w fl32(sum_rb partial[w][rb][c][k])) / W ).  One thread per entry, four per
// column: a thread per column left a quarter of the workgroups and four times the loads to each.
constexpr int kQmeanCols = 64;   // columns of a workgroup: kMatCols / kQmeanCols of them take a QTile

__global__ __launch_bounds__(256) void psgd_qmean_kernel(const Ws ws) {
  const QTile t = ws.qtiles[blockIdx.x];
  const LayerDev& L = ws.layers[t.layer];
  const int level = ws.level[t.layer];
  const int r = level ? L.rank[1] : L.rank[0];
  const int c = t.col0 + blockIdx.y * kQmeanCols + (threadIdx.x >> 2), k = threadIdx.x & 3;
  if (c >= L.cols || k >= r) return;
  const double sum = sum_partials(ws.Qpart + L.qpart_off + (int64_t)c * ws.rmax + k, ws.qpart_stride,
                                  (int64_t)L.cols * ws.rmax, ws.W, L.n_rowblocks);
  ws.Q[L.q_off + (int64_t)c * kMaxRank + k] = (float)(sum / (double)ws.W);   // rows of Q are kMaxRank floats apart
}

// ---- decompress: D = P^ Q_bar^T (the residual stays implicit) ----------------------------------

// NT (the update): weights and velocity beyond Sink::wv_cached are streamed (unaligned rows: in contexts with US, see kUStreamBytes).
// WHAT 0: writes D of the tile to sink.out.  1: e = Delta - D in place.  2: D drives the optimizer step
// on sink.wt / sink.vel and is not stored.
enum DecompWhat { kDecompStore = 0, kDecompResidual = 1, kDecompUpdate = 2 };

template <int WHAT, int MODE, bool NT = false, bool US = false>
__device__ __forceinline__ void decomp_tile(const Ws& ws, const LayerDev& L, const MatTile& t, float* __restrict__ e,
                                            const Sink& sink, int r, float (*ps)[kMaxRank]) {
  constexpr bool RESIDUAL = WHAT == kDecompResidual;
  constexpr bool UPD = WHAT == kDecompUpdate;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const LaneCols lc = lane_cols<MODE>(t.col0, lane, L.cols);
  const int cols = L.cols;
  const int row_end = min(t.row0 + ws.mrows, L.rows);
  constexpr int B = 4;
  constexpr bool IN = RESIDUAL || UPD;                     // the pass reads something per element
  float* const src = (UPD ? sink.wt : e) + L.offset;       // not used when D is only stored
  float* const vel = UPD ? sink.vel + L.offset : nullptr;
  float* const out = IN ? nullptr : sink.out + L.offset;
  // rows i0, i0 + 4, ...; beyond the tile one 16-byte address, see ef_load
  auto request = [&](int i0, float (&d)[IN ? B : 1][4], float (&vv)[UPD ? B : 1][4]) {
    if (IN) {
#pragma unroll
      for (int b = 0; b < B; ++b) {
        const int i = i0 + 4 * b;
        const int64_t rb = (int64_t)min(i, row_end - 1) * cols;
        const int c = i < row_end ? lc.c : 0;
        load_row<MODE, UPD && NT>(src + rb, c, cols, d[IN ? b : 0]);
        if (UPD) load_row<MODE, NT>(vel + rb, c, cols, vv[UPD ? b : 0]);
      }
    }
  };
  // requested together: the first rows, Q's rows, and the tile's rows of P^ (zero-padded to four columns,
  // for LDS): the row loop then waits for no load but those of the rows ahead
  float d[IN ? B : 1][4], vv[UPD ? B : 1][4];
  request(t.row0 + wave, d, vv);
  float q[4][kMaxRank];
  load_q_rows<MODE>(ws, L, lc, q);
  {
    const int pr = threadIdx.x >> 2, pk = threadIdx.x & 3;
    const float ph = ws.Phat[L.p_off + (int64_t)min(t.row0 + pr, L.rows - 1) * ws.rmax + min(pk, ws.rmax - 1)];
    ps[pr][pk] = pk < r ? ph : 0.f;
  }
  __syncthreads();
  for (int i0 = t.row0 + wave; i0 < row_end; i0 += 4 * B) {
    float dn[IN ? B : 1][4], vn[UPD ? B : 1][4];
    request(i0 + 4 * B, dn, vn);
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int i = i0 + 4 * b;
      if (i < row_end) {
        const int64_t rb = (int64_t)i * cols;
        float p[kMaxRank];
#pragma unroll
        for (int k = 0; k < kMaxRank; ++k) p[k] = ps[i - t.row0][k];
        float D[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) D[v] = low_rank_entry(p, q[v]);
        if (RESIDUAL) {
          float res[4];
#pragma unroll
          for (int v = 0; v < 4; ++v) res[v] = d[IN ? b : 0][v] - D[v];
          store_row<MODE>(src + rb, lc, res);
        } else if (UPD) {
#pragma unroll
          for (int v = 0; v < 4; ++v) nesterov(D[v], d[IN ? b : 0][v], vv[UPD ? b : 0][v], sink.lr, sink.mu, sink.wd);
          store_row<MODE, NT, US>(src + rb, lc, d[IN ? b : 0]);
          store_row<MODE, NT, US>(vel + rb, lc, vv[UPD ? b : 0]);
        } else {
          store_row<MODE, kPsgdStreamOut, US>(out + rb, lc, D);
        }
      }
    }
#pragma unroll
    for (int b = 0; b < (IN ? B : 1); ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) d[b][v] = IN ? dn[b][v] : 0.f;
#pragma unroll
    for (int b = 0; b < (UPD ? B : 1); ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) vv[b][v] = UPD ? vn[b][v] : 0.f;
  }
}

template <int WHAT, bool US = false>
__device__ __forceinline__ void decomp_any(const Ws& ws, const LayerDev& L, const MatTile& t, float* __restrict__ e,
                                           const Sink& sink, int r, float (*ps)[kMaxRank]) {
  switch (row_mode(L)) {                                     // uniform over the workgroup
    case kRowAligned:
      if (WHAT == kDecompUpdate && L.offset + (int64_t)t.row0 * L.cols >= sink.wv_cached)
        decomp_tile<WHAT, kRowAligned, WHAT == kDecompUpdate>(ws, L, t, e, sink, r, ps);
      else
        decomp_tile<WHAT, kRowAligned>(ws, L, t, e, sink, r, ps);
      break;
    case kRowUnaligned:
      if (US && WHAT == kDecompUpdate && L.offset + (int64_t)t.row0 * L.cols >= sink.wv_cached)
        decomp_tile<WHAT, kRowUnaligned, US && WHAT == kDecompUpdate, US>(ws, L, t, e, sink, r, ps);
      else
        decomp_tile<WHAT, kRowUnaligned, false, US>(ws, L, t, e, sink, r, ps);
      break;
    default: decomp_tile<WHAT, kRowNarrow>(ws, L, t, e, sink, r, ps); break;
  }
}

// The averaged decompressed gradient: D on matrix layers, the plain mean on 1-D layers (which keep
// no memory: their e is cleared for every worker).
template <bool UPD, bool US>
__device__ __forceinline__ void decomp_body(const Ws& ws, const Sink& sink) {
  __shared__ float ps[kMatRows][kMaxRank];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *ws.pending = ws.W == 32 ? 0xffffffffu : ((1u << ws.W) - 1u);   // every e_w now holds Delta_w
    ws.words[1] = ws.words[0];
    ws.words[2] += ws.words[0];
  }
  if ((int)blockIdx.x >= ws.n_mtiles) {
    const FlatTile ft = ws.ftiles[ws.vectiles[blockIdx.x - ws.n_mtiles]];
    const LayerDev& L = ws.layers[ft.layer];
    for (int i = threadIdx.x; i < ft.count; i += kFlatThreads) {
      const int64_t a = L.offset + ft.start + i;
      for (int w = 0; w < ws.W; ++w) ws.e[(int64_t)w * ws.e_stride + a] = 0.f;
      const float d = ws.vecmean[L.vec_off + ft.start + i];
      if (UPD) {
        float wv = sink.wt[a], vv = sink.vel[a];
        nesterov(d, wv, vv, sink.lr, sink.mu, sink.wd);
        sink.wt[a] = wv;
        sink.vel[a] = vv;
      } else {
        sink.out[a] = d;
      }
    }
    return;
  }
  const MatTile t = ws.mtiles[blockIdx.x];
  const LayerDev& L = ws.layers[t.layer];
  const int r = ws.rank_used[t.layer];                     // written by the orthogonalisation of this step
  decomp_any<UPD ? kDecompUpdate : kDecompStore, US>(ws, L, t, nullptr, sink, r, ps);
}

__global__ __launch_bounds__(256) void psgd_decomp_kernel(const Ws ws, const Sink sink) {
  decomp_body<false, false>(ws, sink);
}

__global__ __launch_bounds__(256) void psgd_decomp_stream_kernel(const Ws ws, const Sink sink) {
  decomp_body<false, true>(ws, sink);
}

// The same pass with the optimizer step in place of the store of D.
__global__ __launch_bounds__(256) void psgd_decomp_update_kernel(const Ws ws, const Sink sink) {
  decomp_body<true, false>(ws, sink);
}

__global__ __launch_bounds__(256) void psgd_decomp_update_stream_kernel(const Ws ws, const Sink sink) {
  decomp_body<true, true>(ws, sink);
}

// e_w = Delta_w - D for the workers whose bit is set in *ws.pending, in place; the caller clears
// the mask with psgd_clear_pending_kernel afterwards.
__global__ __launch_bounds__(256) void psgd_residual_kernel(const Ws ws) {
  const uint32_t pending = *ws.pending;
  const int w = blockIdx.y;
  if (((pending >> w) & 1u) == 0u) return;
  float* __restrict__ e = ws.e + (int64_t)w * ws.e_stride;
  const MatTile t = ws.mtiles[blockIdx.x];
  const LayerDev& L = ws.layers[t.layer];
  const int r = ws.rank_used[t.layer];
  const Sink none = {nullptr, nullptr, nullptr, 0.f, 0.f, 0.f};
  __shared__ float ps[kMatRows][kMaxRank];
  decomp_any<kDecompResidual>(ws, L, t, e, none, r, ps);
}

__global__ void psgd_clear_pending_kernel(const Ws ws) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *ws.pending = 0u;
}

}  // namespace acc
