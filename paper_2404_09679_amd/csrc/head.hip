// Last (single-logit) layer, binary cross-entropy and the start of the backward
// pass of the worker step, plus the per-shard reductions that are sums over the
// samples of a shard (last-layer weight gradient, bias gradients, mean loss).
// Every reduction runs in a fixed order, so results are bitwise repeatable.
#include "common.h"

namespace antdt {
namespace {

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// One wavefront per sample: z = h . w + b, the sample's loss and dz, then dh = dz * w
// (zeroed where the hidden activation is not positive).
template <typename TH, typename TD>
__global__ __launch_bounds__(256) void head_kernel(HeadArgs a, ShardTab tab) {
  const int lane = threadIdx.x & 63;
  const int64_t first = tab.start[a.k_begin];
  const int64_t last = (int64_t)tab.start[a.k_end - 1] + tab.len[a.k_end - 1];
  const int64_t s = first + (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (s >= last) return;
  int k = a.k_begin;
  while (k + 1 < a.k_end && s >= (int64_t)tab.start[k] + tab.len[k]) ++k;
  const float inv_bk = 1.0f / (float)tab.len[k];
  const TH* h = reinterpret_cast<const TH*>(a.h) + s * a.ldh;
  float part = 0.0f;
  for (int j = lane; j < a.width; j += 64) part = fmaf(to_f32(h[j]), a.w[j], part);
  const float z = wave_sum(part) + a.b[0];
  const float y = a.labels[s];
  const float e = expf(-fabsf(z));
  const float loss = fmaxf(z, 0.0f) - z * y + log1pf(e);
  const float sig = z >= 0.0f ? 1.0f / (1.0f + e) : e / (1.0f + e);
  const float dz = (sig - y) * inv_bk;
  if (lane == 0) {
    a.z[s] = z;
    a.loss_s[s] = loss;
    a.dz[s] = dz;
  }
  TD* dh = reinterpret_cast<TD*>(a.dh) + s * a.lddh;
  for (int j = lane; j < a.dh_cols; j += 64) {
    float g = dz * a.w[j];
    if (a.relu && !(to_f32(h[j]) > 0.0f)) g = 0.0f;
    dh[j] = from_f32<TD>(g);
  }
}

// A block works on HEAD_TILE consecutive samples of one shard, four per wavefront; a lane holds the columns
// lane, lane + 64, ... of all four, 512 columns at a time (its loads are then in flight together, and widths
// up to 512 are read once).  Besides the loss, dz and dh it leaves the sums over its samples that the last
// layer's weight gradient, bias gradient and the shard's loss are made of, so that nothing has to read the
// activation again; the last block of a shard to finish adds up the shard's loss (in tile order: the
// result does not depend on which block that is).
// Bound by the chain of round trips (activation -> logit -> gradient), not by bytes.
template <typename TH, typename TD>
__global__ __launch_bounds__(256) void head_tile_kernel(HeadArgs a, ShardTab tab, HeadTiles ht) {
  constexpr int SPW = HEAD_TILE / 4;   // samples per wavefront
  constexpr int CPL = 8, CHUNK = 64 * CPL;
  __shared__ float col[4][CHUNK];
  __shared__ float sums[4][2];
  __shared__ int last;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile = ht.base[a.k_begin] + blockIdx.x;
  int k = a.k_begin;
  while (k + 1 < a.k_end && tile >= ht.base[k + 1]) ++k;
  const int t0 = (tile - ht.base[k]) * HEAD_TILE;            // first sample inside the shard
  const int count = min(tab.len[k] - t0, HEAD_TILE);         // samples of the tile (at least one)
  const int rows = min(max(count - wave * SPW, 0), SPW);     // samples of this wavefront
  const int64_t s0 = (int64_t)tab.start[k] + t0;
  int64_t row[SPW];                                          // (clamped into the tile)
#pragma unroll
  for (int r = 0; r < SPW; ++r) row[r] = s0 + min(wave * SPW + r, count - 1);
  const TH* h = reinterpret_cast<const TH*>(a.h);
  const float label = a.labels[s0 + min(wave * SPW + min(lane, SPW - 1), count - 1)];   // lanes 0 .. SPW-1: one sample each
  const float bias = a.b[0];

  float hv[SPW][CPL], w[CPL];
  auto load = [&](int j0) {
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      if (j0 + i * 64 >= a.width) {   // (the same for all lanes)
        w[i] = 0.0f;
#pragma unroll
        for (int r = 0; r < SPW; ++r) hv[r][i] = 0.0f;
      } else {
        const int j = j0 + i * 64 + lane, jc = min(j, a.width - 1);
        w[i] = a.w[jc];
#pragma unroll
        for (int r = 0; r < SPW; ++r) hv[r][i] = to_f32(h[row[r] * a.ldh + jc]);
        if (j >= a.width) {
          w[i] = 0.0f;
#pragma unroll
          for (int r = 0; r < SPW; ++r) hv[r][i] = 0.0f;
        }
      }
    }
  };
  float part[SPW] = {};
  for (int j0 = 0; j0 < a.width; j0 += CHUNK) {
    load(j0);
#pragma unroll
    for (int i = 0; i < CPL; ++i)
#pragma unroll
      for (int r = 0; r < SPW; ++r) part[r] = fmaf(hv[r][i], w[i], part[r]);
  }
  float mine = 0.0f;   // lane r < SPW: logit of sample r
#pragma unroll
  for (int r = 0; r < SPW; ++r) {
    const float z = wave_sum(part[r]);
    if (lane == r) mine = z;
  }
  const float z = mine + bias;
  const float e = expf(-fabsf(z));
  const float sig = z >= 0.0f ? 1.0f / (1.0f + e) : e / (1.0f + e);
  const bool on = lane < rows;
  const float dz_lane = on ? (sig - label) * (1.0f / (float)tab.len[k]) : 0.0f;
  const float loss_lane = on ? fmaxf(z, 0.0f) - z * label + log1pf(e) : 0.0f;
  float dz[SPW], sdz = 0.0f, sl = 0.0f;
#pragma unroll
  for (int r = 0; r < SPW; ++r) {
    dz[r] = __shfl(dz_lane, r, 64);
    sdz += dz[r];
    sl += __shfl(loss_lane, r, 64);
  }
  if (lane == 0) {
    sums[wave][0] = sdz;
    sums[wave][1] = sl;
  }
  float* part_out = a.part + (int64_t)tile * a.ldpart;
  for (int j0 = 0; j0 < a.width; j0 += CHUNK) {   // (dh_cols <= width)
    if (a.width > CHUNK) load(j0);
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      const int j = j0 + i * 64 + lane;
      float g = 0.0f;
#pragma unroll
      for (int r = 0; r < SPW; ++r)
        if (r < rows) {
          g = fmaf(hv[r][i], dz[r], g);
          const float d = (!a.relu || hv[r][i] > 0.0f) ? dz[r] * w[i] : 0.0f;
          if (j < a.dh_cols) reinterpret_cast<TD*>(a.dh)[row[r] * a.lddh + j] = from_f32<TD>(d);
        }
      if (j0 + i * 64 < a.width) col[wave][i * 64 + lane] = g;
    }
    __syncthreads();
    for (int q = threadIdx.x; q < CHUNK && j0 + q < a.width; q += 256)
      part_out[j0 + q] = (col[0][q] + col[1][q]) + (col[2][q] + col[3][q]);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    // The block that adds the losses up may run on another XCD: stores that go past this XCD's L2, waited for
    // before this block is counted.  (A release fence instead would write back all that L2 holds of the
    // products before this kernel.)
    __hip_atomic_store(part_out + a.width, (sums[0][0] + sums[1][0]) + (sums[2][0] + sums[3][0]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(part_out + a.width + 1, (sums[0][1] + sums[1][1]) + (sums[2][1] + sums[3][1]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const int tiles = ht.base[k + 1] - ht.base[k];
    last = __hip_atomic_fetch_add(a.done + k, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == tiles - 1;
  }
  if (blockIdx.x == 0 && a.k_begin + (int)threadIdx.x < a.k_end && tab.len[a.k_begin + threadIdx.x] == 0) {   // shards without samples
    a.loss_k[a.k_begin + threadIdx.x] = 0.0f;
    if (a.loss_out) a.loss_out[threadIdx.x] = 0.0f;
  }
  __syncthreads();
  if (!last || wave != 0) return;
  float l = 0.0f;
  for (int t = ht.base[k] + lane; t < ht.base[k + 1]; t += 64)
    l += __hip_atomic_load(a.part + (int64_t)t * a.ldpart + a.width + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  l = wave_sum(l);
  if (lane == 0) {
    __hip_atomic_store(a.done + k, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const float lk = l / (float)tab.len[k];
    a.loss_k[k] = lk;
    if (a.loss_out) a.loss_out[k - a.k_begin] = lk;
  }
}

// Losses of shards without samples, when no shard of the range has any.
__global__ __launch_bounds__(64) void head_no_samples_kernel(HeadArgs a) {
  for (int k = a.k_begin + (int)threadIdx.x; k < a.k_end; k += 64) {
    a.loss_k[k] = 0.0f;
    if (a.loss_out) a.loss_out[k - a.k_begin] = 0.0f;
  }
}

__global__ __launch_bounds__(64) void zero_words_kernel(int32_t* p, int n) {
  for (int i = threadIdx.x; i < n; i += 64) p[i] = 0;
}

// Block (64 columns x 4 sample lanes) of shard k = k_begin + blockIdx.y:
//   dW_last[j] = sum_s h[s, j] * dz[s];  block 0 also: db_last = sum_s dz[s], loss_k = mean loss.
template <typename TH>
__global__ __launch_bounds__(256) void head_reduce_kernel(HeadReduceArgs a, ShardTab tab) {
  __shared__ float red[4][64];
  const int k = a.k_begin + blockIdx.y;
  const int64_t s0 = tab.start[k];
  const int n = tab.len[k];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int j = blockIdx.x * 64 + tx;
  float* g = a.grads + (int64_t)k * a.P;
  float acc = 0.0f;
  if (j < a.width) {
    const TH* h = reinterpret_cast<const TH*>(a.h) + s0 * a.ldh + j;
    for (int s = ty; s < n; s += 4) acc = fmaf(to_f32(h[(int64_t)s * a.ldh]), a.dz[s0 + s], acc);
  }
  red[ty][tx] = acc;
  __syncthreads();
  if (ty == 0 && j < a.width) g[a.w_off + j] = (red[0][tx] + red[1][tx]) + (red[2][tx] + red[3][tx]);
  if (blockIdx.x == 0) {
    __syncthreads();
    float sdz = 0.0f, sl = 0.0f;
    for (int s = threadIdx.x; s < n; s += 256) {
      sdz += a.dz[s0 + s];
      sl += a.loss_s[s0 + s];
    }
    sdz = wave_sum(sdz);
    sl = wave_sum(sl);
    if (tx == 0) {
      red[0][ty] = sdz;
      red[1][ty] = sl;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      g[a.b_off] = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
      const float lk = n > 0 ? ((red[1][0] + red[1][1]) + (red[1][2] + red[1][3])) / (float)n : 0.0f;
      a.loss_k[k] = lk;
      if (a.loss_out) a.loss_out[k - a.k_begin] = lk;
    }
  }
}

// db[k][o] = sum over the samples of shard k of dh[s, o].
template <typename TD>
__global__ __launch_bounds__(256) void bias_grad_kernel(BiasGradArgs a, ShardTab tab) {
  __shared__ float red[4][64];
  const int k = a.k_begin + blockIdx.y;
  const int64_t s0 = tab.start[k];
  const int n = tab.len[k];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int j = blockIdx.x * 64 + tx;
  float acc = 0.0f;
  if (j < a.width) {
    const TD* d = reinterpret_cast<const TD*>(a.dh) + s0 * a.lddh + j;
    int s = ty;
    for (; s + 12 < n; s += 16) {
      const float v0 = to_f32(d[(int64_t)s * a.lddh]), v1 = to_f32(d[(int64_t)(s + 4) * a.lddh]);
      const float v2 = to_f32(d[(int64_t)(s + 8) * a.lddh]), v3 = to_f32(d[(int64_t)(s + 12) * a.lddh]);
      acc += (v0 + v1) + (v2 + v3);
    }
    for (; s < n; s += 4) acc += to_f32(d[(int64_t)s * a.lddh]);
  }
  red[ty][tx] = acc;
  __syncthreads();
  if (ty == 0 && j < a.width)
    a.grads[(int64_t)k * a.P + a.b_off + j] = (red[0][tx] + red[1][tx]) + (red[2][tx] + red[3][tx]);
}

}  // namespace

hipError_t launch_head(const HeadArgs& a, const ShardTab& tab, hipStream_t s) {
  const int64_t first = tab.start[a.k_begin];
  const int64_t last = (int64_t)tab.start[a.k_end - 1] + tab.len[a.k_end - 1];
  if (last <= first) return hipSuccess;
  dim3 grid((unsigned)((last - first + 3) / 4)), block(256);
  hipLaunchKernelGGL((head_kernel<float, float>), grid, block, 0, s, a, tab);
  return hipGetLastError();
}

hipError_t launch_head_tiles(const HeadArgs& a, const ShardTab& tab, hipStream_t s) {
  const HeadTiles ht = head_tiles(tab);
  const int tiles = ht.base[a.k_end] - ht.base[a.k_begin];
  if (tiles == 0) hipLaunchKernelGGL(head_no_samples_kernel, dim3(1), dim3(64), 0, s, a);
  else if (a.bf16_dh) hipLaunchKernelGGL((head_tile_kernel<bf16_t, bf16_t>), dim3(tiles), dim3(256), 0, s, a, tab, ht);
  else if (a.bf16_h) hipLaunchKernelGGL((head_tile_kernel<bf16_t, float>), dim3(tiles), dim3(256), 0, s, a, tab, ht);
  else hipLaunchKernelGGL((head_tile_kernel<float, float>), dim3(tiles), dim3(256), 0, s, a, tab, ht);
  return hipGetLastError();
}

hipError_t launch_zero_words(int32_t* p, int n, hipStream_t s) {
  hipLaunchKernelGGL(zero_words_kernel, dim3(1), dim3(64), 0, s, p, n);
  return hipGetLastError();
}

hipError_t launch_head_reduce(const HeadReduceArgs& a, const ShardTab& tab, hipStream_t s) {
  dim3 grid((a.width + 63) / 64, a.k_end - a.k_begin), block(256);
  hipLaunchKernelGGL(head_reduce_kernel<float>, grid, block, 0, s, a, tab);
  return hipGetLastError();
}

hipError_t launch_bias_grad(const BiasGradArgs& a, const ShardTab& tab, hipStream_t s) {
  dim3 grid((a.width + 63) / 64, a.k_end - a.k_begin), block(256);
  if (a.bf16_dh) hipLaunchKernelGGL(bias_grad_kernel<bf16_t>, grid, block, 0, s, a, tab);
  else hipLaunchKernelGGL(bias_grad_kernel<float>, grid, block, 0, s, a, tab);
  return hipGetLastError();
}

}  // namespace antdt
