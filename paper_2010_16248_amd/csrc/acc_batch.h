// Batch-size mode of Accordion (Section 3 "Distributed SGD with adaptive batch size"; Section
// 4.2: the same algorithm on the gradient of the whole model; Section 5.1 "Hyperparameters":
// learning rate scaled with the batch; Appendix A "Additional Details for Batch Size experiment":
// the large batch is several backward passes summed before one exchange, and it only grows).
//
// One launch per micro-step (one backward pass of every worker on B_low samples):
//   A += g_0;   S_w = g_w (first micro-step of a batch) or S_w + g_w;
//   batch complete (1 micro-step inside a critical regime, `mult` outside):
//     D = (S_0 + S_1 + ... + S_{W-1}) / (W * micro-steps), stored or consumed by the optimizer step
//     with the learning rate lr * micro-steps; the sums need not be written then.
// The number of micro-steps summed so far lives on the device in two slots used alternately
// (slot = micro-step parity), so that the one thread that advances it never races with the
// workgroups that read it.
#pragma once
#include <type_traits>

#include "acc_common.h"

namespace acc {

constexpr int kBatchWorkers = 4;   // workers whose loads are in flight together
// The gradients stream in (read once), so that the running sums, the accumulator (of several workers; of one worker: see NTA)
// and, in the small-batch regime, the averaged gradient stay in the caches from one micro-step to the next:
// 118 -> 95 us per micro-step on ResNet-18 shapes, W = 4.  Streaming the rest as well brings
// nothing in the large-batch regime there and costs 3 us in the small-batch one.
constexpr bool kBatchStreamG = true;
constexpr bool kBatchStream = false;

// Slot layout (uint32 x 4): [0] micro-steps summed before this micro-step, [1] micro-steps of the
// batch the previous micro-step completed (0: none), [2], [3] spare.
__device__ __forceinline__ const uint32_t* batch_slot(const Ws& ws, uint32_t parity) {
  return ws.bstate + 4 * (parity & 1u);
}

// NTS, NTA: the running sums (see kCachedSums on the host side) / the accumulator (one worker, whatever the size) are accessed with the
// streaming hint.  NTA, us per four micro-steps plain -> streamed, three states in turn | one state | one state with 1 GB of a program's own
// traffic between its micro-steps | the same and the gradients written just before them; one large batch: 0.8 M
// elements 30.1 -> 30.5 | 23.5 -> 22.2 | 41 -> 38 | 37 -> 34, 4.3 M 68.7 -> 70.4 | 68.2 -> 69.0 | 95 -> 97 | 82 -> 78, 7.6 M 111 -> 109 | 109 -> 109 |
// 144 -> 143 | 131 -> 126, 51 M (LSTM) 731 -> 593 | 730 -> 574 | 719 -> 697 | 695 -> 592; four small batches: 0.8 M 31.6 -> 31.7 | 24.9 -> 25.0 | 41 -> 38 |
// 36 -> 36, 4.3 M 61.8 -> 65.2 | 61.3 -> 64.5 | 84 -> 91 | 69 -> 65, 11 M 130 -> 128 | 129 -> 126 | 162 -> 150 | 146 -> 130.  (Plain is the better one
// around 4 M elements while nothing lies between the micro-steps; a rule for that would be one size's.)
// NW: the number of workers, 0: any.  (Four loads from clamped indices whatever the number asked memory for the same lines again:
// ResNet-18 shapes at W = 1, eight micro-steps, 390 -> 298 us with the streamed accumulator; LSTM set W = 2, four micro-steps,
// 1055 -> 920.)  Where few workgroups wait for their loads the branches inside the loop were what counted: four small layers,
// four micro-steps, W = 2 43.4 -> 34.8 us, W = 16 189 -> 152.
template <bool AL, bool UPD, int NW = 0, bool NTS = false, bool NTA = false>
__device__ __forceinline__ void batch_tile(const Ws& ws, const GradPtrs& gp, const Sink& sink,
                                           const TileGeom& tg, uint32_t j, bool exch) {
  const int W = ws.W;
  const int64_t e_stride = ws.e_stride;
  float* const S = ws.e;
  float* const A = ws.A;
  const float denom = (float)((uint32_t)W * (j + 1u));
  const float lr_eff = sink.lr * (float)(j + 1u);
  const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
  // a loop for each case: a request behind a branch would be waited for before the next one goes out
  auto loop = [&](auto first_c, auto exch_c) {
    constexpr bool FIRST = decltype(first_c)::value, EXCH = decltype(exch_c)::value;
    for (int q = threadIdx.x; q < tg.nquads; q += kFlatThreads) {
      float4 a = ldq<AL, NTA>(A, tg.a0, tg.hi, q, true);
      float4 wq = zero4, vq = zero4;
      if (UPD && EXCH) {
        wq = ldq<AL, kBatchStream>(sink.wt, tg.a0, tg.hi, q, true);
        vq = ldq<AL, kBatchStream>(sink.vel, tg.a0, tg.hi, q, true);
      }
      float4 acc = zero4;
      // N workers from wb on, their loads in flight together
      auto workers = [&](int wb, auto n_workers) {
        constexpr int N = decltype(n_workers)::value;
        float4 g[N], s[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
          g[u] = ldq<AL, kBatchStreamG>(gp.p[wb + u], tg.a0, tg.hi, q, true);
          s[u] = FIRST ? zero4 : ldq<AL, NTS>(S + (int64_t)(wb + u) * e_stride, tg.a0, tg.hi, q, true);
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
          const int w = wb + u;
          if (w == 0) a = make_float4(a.x + g[u].x, a.y + g[u].y, a.z + g[u].z, a.w + g[u].w);
          float4 t = g[u];
          if (!FIRST) t = make_float4(s[u].x + t.x, s[u].y + t.y, s[u].z + t.z, s[u].w + t.w);
          if (EXCH) acc = (w == 0) ? t : make_float4(acc.x + t.x, acc.y + t.y, acc.z + t.z, acc.w + t.w);
          else stq<AL, NTS>(S + (int64_t)w * e_stride, tg.a0, tg.hi, q, t);
        }
      };
      if constexpr (NW > 0) {
        workers(0, std::integral_constant<int, NW>());
      } else {
        int wb = 0;
        for (; wb + kBatchWorkers <= W; wb += kBatchWorkers) workers(wb, std::integral_constant<int, kBatchWorkers>());
        static_assert(kBatchWorkers == 4, "the switch takes every number of workers that may be left");
        switch (W - wb) {                                  // uniform
          case 1: workers(wb, std::integral_constant<int, 1>()); break;
          case 2: workers(wb, std::integral_constant<int, 2>()); break;
          case 3: workers(wb, std::integral_constant<int, 3>()); break;
          default: break;
        }
      }
      stq<AL, NTA>(A, tg.a0, tg.hi, q, a);
      if (EXCH) {
        const float4 d = make_float4(acc.x / denom, acc.y / denom, acc.z / denom, acc.w / denom);
        if (UPD) {
          nesterov(d.x, wq.x, vq.x, lr_eff, sink.mu, sink.wd);
          nesterov(d.y, wq.y, vq.y, lr_eff, sink.mu, sink.wd);
          nesterov(d.z, wq.z, vq.z, lr_eff, sink.mu, sink.wd);
          nesterov(d.w, wq.w, vq.w, lr_eff, sink.mu, sink.wd);
          stq<AL, kBatchStream>(sink.wt, tg.a0, tg.hi, q, wq);
          stq<AL, kBatchStream>(sink.vel, tg.a0, tg.hi, q, vq);
        } else {
          stq<AL, kBatchStream>(sink.out, tg.a0, tg.hi, q, d);
        }
      }
    }
  };
  if (j == 0u && !exch) loop(std::true_type(), std::false_type());   // uniform
  else if (!exch) loop(std::false_type(), std::false_type());
  else if (j == 0u) loop(std::true_type(), std::true_type());
  else loop(std::false_type(), std::true_type());
}

template <bool UPD>
__device__ __forceinline__ void batch_micro_body(const Ws& ws, const GradPtrs& gp, const Sink& sink,
                                                 uint32_t parity, int64_t sums_cached) {
  const uint32_t j = batch_slot(ws, parity)[0];
  const uint32_t target = (ws.level[0] == 1) ? 1u : (uint32_t)ws.bmult;
  const bool exch = j + 1u >= target;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    uint32_t* next = ws.bstate + 4 * ((parity + 1u) & 1u);
    next[0] = exch ? 0u : j + 1u;
    next[1] = exch ? j + 1u : 0u;
    const unsigned long long sent = exch ? (unsigned long long)ws.n_model : 0ull;
    ws.words[1] = sent;
    ws.words[2] += sent;
    ws.stats[0] += exch ? 1ull : 0ull;                     // exchanges
    ws.stats[1] += 1ull;                                   // micro-steps
  }
  const FlatTile ft = ws.ftiles[blockIdx.x];
  const LayerDev& L = ws.layers[ft.layer];
  const TileGeom tg = tile_geom(L, ft);
  const bool nts = tg.a0 >= sums_cached;                   // uniform, like all that follows
  auto tile = [&](auto n_workers, auto nta) {
    if (nts) batch_tile<true, UPD, decltype(n_workers)::value, true, decltype(nta)::value>(ws, gp, sink, tg, j, exch);
    else batch_tile<true, UPD, decltype(n_workers)::value, false, decltype(nta)::value>(ws, gp, sink, tg, j, exch);
  };
  if (!tg.aligned) {
    batch_tile<false, UPD>(ws, gp, sink, tg, j, exch);
    return;
  }
  switch (ws.W) {
    case 1: tile(std::integral_constant<int, 1>(), std::true_type()); break;
    case 2: tile(std::integral_constant<int, 2>(), std::false_type()); break;
    case 3: tile(std::integral_constant<int, 3>(), std::false_type()); break;
    case 4: tile(std::integral_constant<int, 4>(), std::false_type()); break;
    default: tile(std::integral_constant<int, 0>(), std::false_type()); break;
  }
}

__global__ __launch_bounds__(256) void batch_micro_kernel(const Ws ws, const GradPtrs gp, const Sink sink,
                                                          uint32_t parity, int64_t sums_cached) {
  batch_micro_body<false>(ws, gp, sink, parity, sums_cached);
}

__global__ __launch_bounds__(256) void batch_micro_update_kernel(const Ws ws, const GradPtrs gp,
                                                                 const Sink sink, uint32_t parity, int64_t sums_cached) {
  batch_micro_body<true>(ws, gp, sink, parity, sums_cached);
}

// One workgroup: c = sqrt(sum of all tile partials) (the norm of the whole model's accumulated
// gradient), Algorithm 1 once, "the batch only grows" if asked for; the decision is written to
// every layer's entry so that the per-layer read-backs show it.
__global__ __launch_bounds__(256) void batch_decide_kernel(const Ws ws, float lr_curr, float lr_next) {
  __shared__ double red[4];
  __shared__ int s_level;
  __shared__ float s_old, s_c;
  const int tid = threadIdx.x;
  double s = 0.0;
  for (int t = tid; t < ws.n_ftiles; t += 256) s += ws.norm_part[t];
  s = wave_sum_f64(s);
  if ((tid & 63) == 0) red[tid >> 6] = s;
  __syncthreads();
  if (tid == 0) {
    const float c = (float)sqrt((red[0] + red[1]) + (red[2] + red[3]));
    const float old = ws.norm_old[0];
    const bool has_old = ws.has_old[0] != 0;
    bool crit;
    if (lr_next < lr_curr) crit = true;
    else if (!has_old) crit = true;
    else if (old == 0.0f) crit = true;
    else crit = (fabsf(old - c) / old) >= ws.eta;
    int level = crit ? 1 : 0;
    if (ws.bmono != 0 && ws.level[0] == 0) level = 0;
    s_level = level;
    s_old = old;
    s_c = c;
  }
  __syncthreads();
  for (int li = tid; li < ws.L; li += 256) {
    ws.level[li] = s_level;
    ws.norm_prev[li] = s_old;
    ws.norm_curr[li] = s_c;
    ws.norm_old[li] = s_c;
    ws.has_old[li] = 1;
  }
}

}  // namespace acc
