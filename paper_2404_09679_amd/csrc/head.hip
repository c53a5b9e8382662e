// Last (single-logit) layer, binary cross-entropy and the start of the backward
// pass of the worker step, with the partial sums over samples that the last layer's
// gradients and the shards' mean losses are made of.
// Every reduction runs in a fixed order, so results are bitwise repeatable.
#include "common.h"

namespace antdt {
namespace {

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// A block works on HEAD_TILE consecutive samples of one shard, four per wavefront; a lane holds the columns
// lane, lane + 64, ... of all four, 512 columns at a time (its loads are then in flight together, and widths
// up to 512 are read once).  Besides the loss, dz and dh it leaves the sums over its samples that the last
// layer's weight gradient, bias gradient and the shard's loss are made of, so that nothing has to read the
// activation again.
// Bound by the chain of round trips (activation -> logit -> gradient), not by bytes.
template <typename TH, typename TD>
__global__ __launch_bounds__(256) void head_tile_kernel(HeadArgs a, ShardTab tab, HeadTiles ht) {
  constexpr int SPW = HEAD_TILE / 4;   // samples per wavefront
  constexpr int CPL = 8, CHUNK = 64 * CPL;
  __shared__ float col[4][CHUNK];
  __shared__ float sums[4][2];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile = ht.base[a.k_begin] + blockIdx.x;
  int k = a.k_begin;
  while (k + 1 < a.k_end && tile >= ht.base[k + 1]) ++k;
  const int t0 = (tile - ht.base[k]) * HEAD_TILE;            // first sample inside the shard
  const int count = min(tab.len[k] - t0, HEAD_TILE);         // samples of the tile (at least one)
  const int rows = min(max(count - wave * SPW, 0), SPW);     // samples of this wavefront
  const int64_t s0 = (int64_t)tab.start[k] + t0;
  // (fp32: dh may lie in h's place, so a wavefront reads its own samples only, or the weights if it has none)
  int64_t row[SPW];
  const TH* h[SPW];
#pragma unroll
  for (int r = 0; r < SPW; ++r) {
    row[r] = s0 + min(wave * SPW + min(r, max(rows - 1, 0)), count - 1);
    h[r] = sizeof(TH) == 4 && rows == 0 ? reinterpret_cast<const TH*>(a.w) : reinterpret_cast<const TH*>(a.h) + row[r] * a.ldh;
  }
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
        for (int r = 0; r < SPW; ++r) hv[r][i] = to_f32(h[r][jc]);
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
  const bool per_sample = sizeof(TD) == 4 && a.dz;   // (bf16 gradients: there is a hidden layer)
  if (per_sample && on) {   // (lane r < rows: the wavefront's sample r)
    a.dz[s0 + wave * SPW + lane] = dz_lane;
    a.loss_s[s0 + wave * SPW + lane] = loss_lane;
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
    if (per_sample) continue;
    __syncthreads();
    for (int q = threadIdx.x; q < CHUNK && j0 + q < a.width; q += 256)
      part_out[j0 + q] = (col[0][q] + col[1][q]) + (col[2][q] + col[3][q]);
    __syncthreads();
  }
  if (threadIdx.x == 0 && !per_sample) {
    part_out[a.width] = (sums[0][0] + sums[1][0]) + (sums[2][0] + sums[3][0]);
    part_out[a.width + 1] = (sums[0][1] + sums[1][1]) + (sums[2][1] + sums[3][1]);
  }
  if (blockIdx.x == 0 && (int)threadIdx.x < a.k_end - a.k_begin) {
    const int q = a.k_begin + threadIdx.x;
    LossJob j;
    j.sums = per_sample ? a.loss_s + tab.start[q] : a.part + (int64_t)ht.base[q] * a.ldpart + a.width + 1;
    j.loss_out = a.loss_out ? a.loss_out + threadIdx.x : nullptr;
    j.ldpart = per_sample ? 1 : a.ldpart;
    j.tiles = per_sample ? tab.len[q] : ht.base[q + 1] - ht.base[q];
    j.len = tab.len[q];
    a.job[q] = j;
  }
}

// Losses of shards without samples, when no shard of the range has any.
__global__ __launch_bounds__(64) void head_no_samples_kernel(HeadArgs a) {
  for (int k = a.k_begin + (int)threadIdx.x; k < a.k_end; k += 64)
    if (a.loss_out) a.loss_out[k - a.k_begin] = 0.0f;
}

__global__ __launch_bounds__(64) void losses_kernel(const LossJob* job) { add_up_losses(job + blockIdx.x); }

}  // namespace

hipError_t launch_head_tiles(const HeadArgs& a, const ShardTab& tab, hipStream_t s) {
  const HeadTiles ht = head_tiles(tab);
  const int tiles = ht.base[a.k_end] - ht.base[a.k_begin];
  if (tiles == 0) hipLaunchKernelGGL(head_no_samples_kernel, dim3(1), dim3(64), 0, s, a);
  else if (a.bf16_dh) hipLaunchKernelGGL((head_tile_kernel<bf16_t, bf16_t>), dim3(tiles), dim3(256), 0, s, a, tab, ht);
  else if (a.bf16_h) hipLaunchKernelGGL((head_tile_kernel<bf16_t, float>), dim3(tiles), dim3(256), 0, s, a, tab, ht);
  else hipLaunchKernelGGL((head_tile_kernel<float, float>), dim3(tiles), dim3(256), 0, s, a, tab, ht);
  return hipGetLastError();
}

hipError_t launch_losses(const LossJob* job, int shards, hipStream_t s) {
  hipLaunchKernelGGL(losses_kernel, dim3(shards), dim3(64), 0, s, job);
  return hipGetLastError();
}

}  // namespace antdt
