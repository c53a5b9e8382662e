// Last (single-logit) layer, binary cross-entropy and the start of the backward
// pass of the worker step, with the partial sums over samples that the last layer's
// gradients and the shards' mean losses are made of.
// Every reduction runs in a fixed order, so results are bitwise repeatable.
#include <type_traits>

#include "common.h"

namespace antdt {
namespace {

// Another lane's value (no trip through LDS, which a shuffle is).
template <int CTRL> __device__ __forceinline__ float moved(float x, std::integral_constant<int, CTRL>) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, true));
}

// Sum over the wavefront, in every lane: halves, then quarters, ...
__device__ __forceinline__ float wave_sum(float v) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  auto both = [](u32x2 p) { return __uint_as_float(p.x) + __uint_as_float(p.y); };
  v = both(__builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false));
  v = both(__builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false));
  v += moved(v, std::integral_constant<int, 0x128>());   // eight lanes round a row of sixteen
  v += moved(v, std::integral_constant<int, 0x124>());   // four (the halves of the row are the same by now)
  v += moved(v, std::integral_constant<int, 0x4E>());    // lane ^ 2
  v += moved(v, std::integral_constant<int, 0xB1>());    // lane ^ 1
  return v;
}
__device__ __forceinline__ float lane_value(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// Four neighbouring columns of a row as they lie in memory, and the store of four results.
template <typename T> struct Quad;
template <> struct Quad<float> {
  static constexpr int WORDS = 4;
  uint32_t d[4];
  __device__ __forceinline__ void load(const float* x) {
    const uint4 q = *reinterpret_cast<const uint4*>(x);
    d[0] = q.x; d[1] = q.y; d[2] = q.z; d[3] = q.w;
  }
  __device__ __forceinline__ float operator[](int e) const { return __uint_as_float(d[e]); }
};
template <> struct Quad<bf16_t> {
  static constexpr int WORDS = 2;
  uint32_t d[2];
  __device__ __forceinline__ void load(const bf16_t* x) {
    const uint2 q = *reinterpret_cast<const uint2*>(x);
    d[0] = q.x; d[1] = q.y;
  }
  __device__ __forceinline__ float operator[](int e) const { return __uint_as_float(e & 1 ? d[e >> 1] & 0xFFFF0000u : d[e >> 1] << 16); }
};
// The 4 x 4 of registers and rows of sixteen lanes turned: register r of row q takes register q of row r.
__device__ __forceinline__ void turn(uint32_t& a, uint32_t& b, uint32_t& c, uint32_t& d) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  auto swap = [](u32x2 p, uint32_t& x, uint32_t& y) {
    x = p.x;
    y = p.y;
  };
  swap(__builtin_amdgcn_permlane32_swap(a, c, false, false), a, c);
  swap(__builtin_amdgcn_permlane32_swap(b, d, false, false), b, d);
  swap(__builtin_amdgcn_permlane16_swap(a, b, false, false), a, b);
  swap(__builtin_amdgcn_permlane16_swap(c, d, false, false), c, d);
}
__device__ __forceinline__ void store4(float* x, const float (&v)[4]) { *reinterpret_cast<float4*>(x) = make_float4(v[0], v[1], v[2], v[3]); }
__device__ __forceinline__ void store4(bf16_t* x, const float (&v)[4]) { *reinterpret_cast<uint2*>(x) = make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3])); }

// A block works on HEAD_TILE consecutive samples of one shard, four per wavefront, 512 columns at a time.  Besides the loss, dz
// and dh it leaves the sums over its samples that the last layer's weight gradient, bias gradient and the shard's
// loss are made of, so that nothing has to read the activation again.
// Bound by the chain of round trips (activation -> logit -> gradient) and by its own instructions, each of which a launch
// fetches anew and runs about once: a column at a time they were 9 KB.
// VEC: widths and pitches are multiples of four (all bf16 models with a hidden layer), so columns are moved four at a time.
//
// The logit's products are added in one order whatever the path: 64 chains, chain c of the columns c, c + 64, c + 128, ..., and
// then the chains in halves (c and c ^ 32, c ^ 16, ... c ^ 1).  Any other order moves logits by their last bit, and bf16 models
// amplify that: single entries of dh then round to another bf16 neighbour (up to 3e-4 of a step).
//   Without VEC a lane is a chain, of each of the four samples.
//   VEC: sixteen lanes have a sample, four chains each (columns 4 (lane & 15) .. + 3 of every 64).  The sums over the samples and
//   dh need a column of all four samples in one lane; the registers are turned for them (loaded a second time in that order they
//   left a SIMD three wavefronts).  A launch, us, with columns loaded one at a time / twice / turned: 64 x 256 7.0 / 5.9 / 5.8,
//   4096 x 256 6.6 / 6.2 / 5.9, 15 625 x 256 10.8 / 12.9 / 10.0, 16 384 x 512 13.7 / 17.7 / 12.6.
template <typename TH, typename TD, bool VEC>
__global__ __launch_bounds__(256, sizeof(TH) == 2 ? 5 : 4) void head_tile_kernel(HeadArgs a, ShardTab tab, HeadTiles ht) {
  constexpr int SPW = HEAD_TILE / 4;   // samples per wavefront
  static_assert(SPW == 4, "sixteen lanes per sample");
  constexpr int PARTS = 2, CHUNK = 256 * PARTS;
  __shared__ float col[4][CHUNK];
  __shared__ float sums[4][2];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile = ht.base[a.k_begin] + blockIdx.x;
  // the shard: how many of the range's shards before the last end at or before the tile, counted by the lanes (one load of
  // the table instead of a chain of them)
  static_assert(ANTDT_MAX_SHARDS <= 64, "a table entry per lane");
  const int shard_end = ht.base[min(lane, ANTDT_MAX_SHARDS - 1) + 1];
  const int k = a.k_begin + __popcll(__ballot(lane >= a.k_begin && lane + 1 < a.k_end && shard_end <= tile));
  const int t0 = (tile - ht.base[k]) * HEAD_TILE;            // first sample inside the shard
  const int count = min(tab.len[k] - t0, HEAD_TILE);         // samples of the tile (at least one)
  const int rows = min(max(count - wave * SPW, 0), SPW);     // samples of this wavefront
  const int64_t s0 = (int64_t)tab.start[k] + t0;
  const int own = lane >> 4;                                 // the lane's sample (of the wavefront's)
  // (fp32: dh may lie in h's place, so a wavefront reads its own samples only, or the weights if it has none)
  auto sample_row = [&](int r) { return s0 + min(wave * SPW + min(r, max(rows - 1, 0)), count - 1); };
  auto activation = [&](int64_t at) {
    return sizeof(TH) == 4 && rows == 0 ? reinterpret_cast<const TH*>(a.w) : reinterpret_cast<const TH*>(a.h) + at * a.ldh;
  };
  int64_t row[SPW];
  const TH* h[SPW];
#pragma unroll
  for (int r = 0; r < SPW; ++r) {
    row[r] = sample_row(r);
    h[r] = activation(row[r]);
  }
  const float label = a.labels[s0 + min(wave * SPW + own, count - 1)];
  const float bias = a.b[0];

  // Columns of all four samples: column(i, e) of the 512 from j0 on.
  typedef Quad<typename std::conditional<VEC, TH, float>::type> Columns;
  Columns hv[PARTS][SPW];
  Quad<float> w[PARTS];
  auto column = [&](int i, int e) { return i * 256 + (VEC ? lane * 4 + e : e * 64 + lane); };
  auto load_w = [&](int j0) {
#pragma unroll
    for (int i = 0; i < PARTS; ++i) {
      if (j0 + i * 256 >= a.width) continue;   // (the same for all lanes)
      if (VEC) {
        w[i].load(a.w + min(j0 + column(i, 0), a.width - 4));
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) w[i].d[e] = j0 + column(i, e) < a.width ? __float_as_uint(a.w[j0 + column(i, e)]) : 0;
      }
    }
  };
  auto load_h = [&](int j0) {
#pragma unroll
    for (int i = 0; i < PARTS; ++i) {
      if (j0 + i * 256 >= a.width) continue;
#pragma unroll
      for (int r = 0; r < SPW; ++r) {
        if constexpr (VEC) {
          hv[i][r].load(h[r] + min(j0 + column(i, 0), a.width - 4));
          if (j0 + column(i, 0) >= a.width) hv[i][r] = {};   // (the four are inside or outside together)
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            hv[i][r].d[e] = j0 + column(i, e) < a.width ? __float_as_uint(to_f32(h[r][j0 + column(i, e)])) : 0;
        }
      }
    }
  };
  const bool loaded = a.width <= CHUNK;
  float z;   // logit of the lane's sample, without the bias
  if constexpr (VEC) {
    const TH* h_own = activation(sample_row(own));
    constexpr int STEPS = CHUNK / 64;
    float chain[4] = {};
    for (int j0 = 0; j0 < a.width; j0 += CHUNK) {
      Columns x[STEPS];
      Quad<float> y[STEPS];
#pragma unroll
      for (int i = 0; i < STEPS; ++i) {
        x[i] = {};
        y[i] = {};
        if (j0 + i * 64 < a.width) {   // (the same for all lanes)
          const int jc = min(j0 + i * 64 + (lane & 15) * 4, a.width - 4);
          x[i].load(h_own + jc);
          y[i].load(a.w + jc);
        }
      }
      if (loaded) load_w(0);
#pragma unroll
      for (int i = 0; i < STEPS; ++i) {
        if (j0 + i * 64 >= a.width) continue;
        if (j0 + i * 64 + (lane & 15) * 4 >= a.width) {
          x[i] = {};
          y[i] = {};
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) chain[e] = fmaf(x[i][e], y[i][e], chain[e]);
      }
      if (loaded) {
#pragma unroll
        for (int i = 0; i < PARTS; ++i) {
#pragma unroll
          for (int r = 0; r < SPW; ++r) hv[i][r] = x[i * 4 + r];
#pragma unroll
          for (int k = 0; k < Columns::WORDS; ++k) turn(hv[i][0].d[k], hv[i][1].d[k], hv[i][2].d[k], hv[i][3].d[k]);
        }
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {   // chains 4 q + e of the sixteen lanes q
      chain[e] += moved(chain[e], std::integral_constant<int, 0x128>());   // eight lanes round the row of sixteen: chains c and c ^ 32
      chain[e] += moved(chain[e], std::integral_constant<int, 0x124>());   // four (the halves of the row are the same by now): c ^ 16
      chain[e] += moved(chain[e], std::integral_constant<int, 0x4E>());    // lane ^ 2: c ^ 8
      chain[e] += moved(chain[e], std::integral_constant<int, 0xB1>());    // lane ^ 1: c ^ 4
    }
    z = (chain[0] + chain[2]) + (chain[1] + chain[3]);
  } else {
    float part[SPW] = {};
    for (int j0 = 0; j0 < a.width; j0 += CHUNK) {
      load_w(j0);
      load_h(j0);
#pragma unroll
      for (int i = 0; i < PARTS; ++i) {
        if (j0 + i * 256 >= a.width) continue;
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int r = 0; r < SPW; ++r) part[r] = fmaf(hv[i][r][e], w[i][e], part[r]);
      }
    }
    z = 0.0f;
#pragma unroll
    for (int r = 0; r < SPW; ++r) {
      const float sum = wave_sum(part[r]);
      if (own == r) z = sum;
    }
  }
  z += bias;
  const float e = expf(-fabsf(z));
  const float sig = (z >= 0.0f ? 1.0f : e) / (1.0f + e);
  const bool on = own < rows;
  const float dz_lane = on ? (sig - label) * (1.0f / (float)tab.len[k]) : 0.0f;
  float dz[SPW];
#pragma unroll
  for (int r = 0; r < SPW; ++r) dz[r] = lane_value(dz_lane, r * 16);
  const bool per_sample = sizeof(TD) == 4 && a.dz;   // (bf16 gradients: there is a hidden layer)
  float* part_out = a.part + (int64_t)tile * a.ldpart;
  for (int j0 = 0; j0 < a.width; j0 += CHUNK) {   // (dh_cols <= width)
    if (!loaded) {
      load_w(j0);
      load_h(j0);
    }
#pragma unroll
    for (int i = 0; i < PARTS; ++i) {
      if (j0 + i * 256 >= a.width) continue;   // (the same for all lanes)
      float g[4] = {};
#pragma unroll
      for (int r = 0; r < SPW; ++r)
        if (r < rows) {
          float d[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            g[e] = fmaf(hv[i][r][e], dz[r], g[e]);
            d[e] = (!a.relu || hv[i][r][e] > 0.0f) ? dz[r] * w[i][e] : 0.0f;
          }
          TD* out = reinterpret_cast<TD*>(a.dh) + row[r] * a.lddh + j0;
          if (VEC) {
            if (j0 + column(i, 0) < a.dh_cols) store4(out + column(i, 0), d);   // (dh_cols: a multiple of four)
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (j0 + column(i, e) < a.dh_cols) out[column(i, e)] = from_f32<TD>(d[e]);
          }
        }
      if (VEC) {
        store4(&col[wave][column(i, 0)], g);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) col[wave][column(i, e)] = g[e];
      }
    }
    const bool last = j0 + CHUNK >= a.width;
    if (last) {   // the losses, behind the stores of the gradient
      const float loss_lane = on ? fmaxf(z, 0.0f) - z * label + log1pf(e) : 0.0f;
      float sdz = 0.0f, sl = 0.0f;
#pragma unroll
      for (int r = 0; r < SPW; ++r) {
        sdz += dz[r];
        sl += lane_value(loss_lane, r * 16);
      }
      if (lane == 0) {
        sums[wave][0] = sdz;
        sums[wave][1] = sl;
      }
      if (per_sample && on && (lane & 15) == 0) {
        a.dz[s0 + wave * SPW + own] = dz_lane;
        a.loss_s[s0 + wave * SPW + own] = loss_lane;
      }
    }
    if (per_sample) continue;
    __syncthreads();
    for (int q = threadIdx.x; q < CHUNK && j0 + q < a.width; q += 256)
      part_out[j0 + q] = (col[0][q] + col[1][q]) + (col[2][q] + col[3][q]);
    if (!last) __syncthreads();
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
  else {
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(tiles), dim3(256), 0, s, a, tab, ht); };
    // (16-byte aligned: the activations lie in the workspace, their rows one behind the other; the weights where the layers before end)
    const bool vec = ((a.width | a.dh_cols | a.ldh | a.lddh) & 3) == 0 && (reinterpret_cast<uintptr_t>(a.w) & 15) == 0;
    if (a.bf16_dh) vec ? launch(head_tile_kernel<bf16_t, bf16_t, true>) : launch(head_tile_kernel<bf16_t, bf16_t, false>);
    else if (a.bf16_h) vec ? launch(head_tile_kernel<bf16_t, float, true>) : launch(head_tile_kernel<bf16_t, float, false>);
    else vec ? launch(head_tile_kernel<float, float, true>) : launch(head_tile_kernel<float, float, false>);
  }
  return hipGetLastError();
}

hipError_t launch_losses(const LossJob* job, int shards, hipStream_t s) {
  hipLaunchKernelGGL(losses_kernel, dim3(shards), dim3(64), 0, s, job);
  return hipGetLastError();
}

}  // namespace antdt
