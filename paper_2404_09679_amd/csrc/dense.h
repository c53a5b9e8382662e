// The dense Adagrad step of one parameter, its gradient added up over the shards on the fly: used by the dense update (optim.hip)
// and, of fp32 models, by blocks of the sparse update's launch (coalesce.hip).
#pragma once

#include "common.h"

namespace antdt {

// Tab: the shards' number K and weights w.
template <typename Tab>
__device__ __forceinline__ float weighted_sum(const float* grads, int64_t stride, int64_t i, const Tab& tab) {
  // Every load is issued (a branch per load would serialise them); the value of a shard
  // with weight 0, which may never have been written, is replaced by 0 afterwards.
  float acc = 0.0f;
  int k = 0;
  for (; k + 3 < tab.K; k += 4) {  // four loads in flight, added in shard order
    float x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = grads[(int64_t)(k + q) * stride + i];
#pragma unroll
    for (int q = 0; q < 4; ++q) acc = fmaf(tab.w[k + q], tab.w[k + q] != 0.0f ? x[q] : 0.0f, acc);
  }
  for (; k < tab.K; ++k) {
    const float x = grads[(int64_t)k * stride + i];
    acc = fmaf(tab.w[k], tab.w[k] != 0.0f ? x : 0.0f, acc);
  }
  return acc;
}

// A: p, state, grads, stride, lr, eps.
template <typename A, typename Tab>
__device__ __forceinline__ void adagrad_elem(const A& a, const Tab& tab, int64_t i) {
  const float g = weighted_sum(a.grads, a.stride, i, tab);
  const float s1 = fmaf(g, g, a.state[i]);
  const float p1 = a.p[i] - a.lr * g / (sqrtf(s1) + a.eps);
  a.state[i] = s1;
  a.p[i] = p1;
}

}  // namespace antdt
