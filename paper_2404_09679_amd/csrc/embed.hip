// Embedding-bag gather and sum- or mean-pool (worker side of the iteration, Section II:
// the forward pass on the local batch B_k), plus the procedural table fill.
#include <algorithm>

#include "common.h"

namespace antdt {

// 16-byte vector of table elements.
template <typename T> struct Vec16;
template <> struct Vec16<float> {
  static constexpr int N = 4;
  float4 v;
  __device__ __forceinline__ float get(int i) const { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }
};
template <> struct Vec16<bf16_t> {
  static constexpr int N = 8;
  uint4 v;
  __device__ __forceinline__ float get(int i) const {
    uint32_t w = i < 2 ? v.x : i < 4 ? v.y : i < 6 ? v.z : v.w;
    return (i & 1) ? __uint_as_float(w & 0xFFFF0000u) : __uint_as_float(w << 16);
  }
};

template <typename OT, int N> __device__ __forceinline__ void store_row(OT* dst, const float* v);
template <> __device__ __forceinline__ void store_row<float, 4>(float* dst, const float* v) {
  *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
}
template <> __device__ __forceinline__ void store_row<float, 8>(float* dst, const float* v) {
  reinterpret_cast<float4*>(dst)[0] = make_float4(v[0], v[1], v[2], v[3]);
  reinterpret_cast<float4*>(dst)[1] = make_float4(v[4], v[5], v[6], v[7]);
}
template <> __device__ __forceinline__ void store_row<bf16_t, 4>(bf16_t* dst, const float* v) {
  *reinterpret_cast<uint2*>(dst) = make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]));
}
template <> __device__ __forceinline__ void store_row<bf16_t, 8>(bf16_t* dst, const float* v) {
  *reinterpret_cast<uint4*>(dst) = make_uint4(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]), f2bf2(v[4], v[5]), f2bf2(v[6], v[7]));
}

// Dense-feature columns of up to 64 samples (below `end`): copied behind the pooled embeddings, the padding columns of
// the row are zeroed.
template <typename OT>
__device__ __forceinline__ void dense_columns(const PoolArgs& a, int sl0, int end) {
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  if (sl0 + tx >= end) return;
  const int64_t s = a.s0 + sl0 + tx;
  const int FD = a.F * a.D;
  OT* xrow = reinterpret_cast<OT*>(a.x) + s * a.ldx + FD;
  for (int c = ty; c < a.ldx - FD; c += 4) {
    const float v = c < a.num_dense ? a.dense[s * a.num_dense + c] : 0.0f;
    xrow[c] = from_f32<OT>(v);
  }
}

constexpr int MOST_ITERATIONS = 15;   // (bags that take as many or more count as equally long)

// Gather and sum-pool.  A block owns SPB consecutive samples of one field; a group of
// LPR = D*sizeof(T)/16 lanes owns one bag, so a wavefront works on 64/LPR bags at once.
// The group fetches LPR ids with one coalesced load, hands the rows' places round with lane
// exchanges and issues the LPR row loads (16 bytes per lane, one whole row per group)
// back to back before adding them, which keeps 64 rows in flight per wavefront; the next ids are
// requested before the rows are waited for.  Every lookup's sample index is recorded for the sort.
// ORDERED: a block hands its 64 samples out in order of the iterations they take, so that the bags a wavefront works on at once are
// about as long as each other: with 1 .. 50 lookups, the longest of eight in any order makes every second load of a wavefront
// one of few lanes (41.8 M lookups: 10.7 M load and 209 M vector instructions, in order 7.1 M and 152 M).
// Bound, where bags are long, by the rows' way from the L2s, 55 lines outstanding on a compute unit (41.8 M lookups of 128-byte
// bf16 rows 507 -> 489 us, 4.3 M of fp32 rows 70.6 -> 68.1; buffer loads that need no bounds took the vector instructions
// down to the additions and won nothing), else by round trips.  Like the sort's tiles, the blocks of a field go to one XCD: its
// rows are fetched into one L2 (fields interleaved two to sixteen at a time: 492 .. 530 us).
// WIDE: a table of 2^32 or more 16-byte pieces.
template <typename TT, typename OT, int LPR, int SPB, bool ORDERED, bool WIDE>
__global__ __launch_bounds__(256) void pool_tile_kernel(PoolArgs a, FieldPtr fp) {
  constexpr int EV = Vec16<TT>::N;
  constexpr int G = 256 / LPR;       // bags per round
  constexpr int ROUNDS = (SPB + G - 1) / G;
  const int tiles = (a.ns + SPB - 1) / SPB, total = tiles * (a.F + 1), share = (total + 7) >> 3;
  const int idx = (int)(blockIdx.x & 7) * share + (int)(blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= share || idx >= total) return;
  const int f = idx / tiles, sl0 = (idx - f * tiles) * SPB, sl1 = min(sl0 + SPB, a.ns);
  if (f == a.F) {
    dense_columns<OT>(a, sl0, sl1);
    return;
  }
  const int g = threadIdx.x / LPR, c = threadIdx.x % LPR;
  const int gl4 = ((threadIdx.x & 63) - c) * 4;  // first lane of this group inside the wavefront
  const int32_t* ids = a.ids + fp.p[f];
  int32_t* smp = a.lookup_sample ? a.lookup_sample + fp.p[f] : nullptr;
  const uint4* tab = reinterpret_cast<const uint4*>(reinterpret_cast<const TT*>(a.tables) + (int64_t)f * a.R * a.D) + c;
  const int last = (int)(a.R - 1);
  auto fetch = [&](int j, int end) { return j < end ? ids[j] : 0; };
  // The bags of round r (sample of the block, lookups): as they come, or (64 of them) in order of the iterations they take, the
  // longest first, every wavefront with long and short ones.
  int sample[ROUNDS], begin[ROUNDS], end[ROUNDS];
  const int32_t* off = a.offsets + (int64_t)f * (a.B + 1) + a.s0 + sl0;
  static_assert(!ORDERED || SPB == 64, "a lane per sample");
  if (ORDERED) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int b0 = 0, e0 = 0;
    if (sl0 + lane < sl1) {
      b0 = off[lane];
      e0 = off[lane + 1];
    }
    const int iterations = min((max(e0 - b0, 0) + LPR - 1) / LPR, MOST_ITERATIONS);
    int place = 0, longer = 0;
    for (int i = MOST_ITERATIONS; i >= 0; --i) {
      const uint64_t m = __ballot(iterations == i);
      if (iterations == i) place = longer + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
      longer += __popcll(m);
    }
    const int sorted = __builtin_amdgcn_ds_permute(place * 4, lane), sb = __builtin_amdgcn_ds_permute(place * 4, b0),
              se = __builtin_amdgcn_ds_permute(place * 4, e0);
    constexpr int PER_WAVE = 64 / LPR;   // bags of a wavefront and round
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const int from = ((r * 4 + (r & 1 ? 3 - w : w)) * PER_WAVE + (threadIdx.x & 63) / LPR) * 4;
      sample[r] = __builtin_amdgcn_ds_bpermute(from, sorted);
      begin[r] = __builtin_amdgcn_ds_bpermute(from, sb);
      end[r] = __builtin_amdgcn_ds_bpermute(from, se);
    }
  } else {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      sample[r] = r * G + g;
      begin[r] = end[r] = 0;
      if (sl0 + sample[r] < sl1) {
        begin[r] = off[sample[r]];
        end[r] = off[sample[r] + 1];
      }
    }
  }
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int ls = sample[r];
    const int64_t s = a.s0 + sl0 + ls;
    const int b0 = begin[r], e0 = end[r];
    float acc[EV];
#pragma unroll
    for (int e = 0; e < EV; ++e) acc[e] = 0.0f;
    int next = fetch(b0 + c, e0);
    for (int jb = b0; jb < e0; jb += LPR) {
      const int id = min(max(next, 0), last);   // keeps a bad id in bounds
      const uint32_t mine = WIDE ? (uint32_t)id : (uint32_t)id * LPR;
      if (smp && jb + c < e0) smp[jb + c] = (int32_t)s;
      next = fetch(jb + LPR + c, e0);
      Vec16<TT> v[LPR];
#pragma unroll
      for (int q = 0; q < LPR; ++q) {
        const uint32_t o = (uint32_t)__builtin_amdgcn_ds_bpermute(gl4 + q * 4, (int)mine);
        if (jb + q < e0) v[q].v = *reinterpret_cast<const decltype(v[q].v)*>(tab + (WIDE ? (uint64_t)o * LPR : (uint64_t)o));
      }
#pragma unroll
      for (int q = 0; q < LPR; ++q)
        if (jb + q < e0) {
#pragma unroll
          for (int e = 0; e < EV; ++e) acc[e] += v[q].get(e);
        }
    }
    if (a.mean_pool && e0 - b0 > 1) {
      const float len = (float)(e0 - b0);
#pragma unroll
      for (int e = 0; e < EV; ++e) acc[e] /= len;
    }
    if (sl0 + ls < sl1) store_row<OT, EV>(reinterpret_cast<OT*>(a.x) + s * a.ldx + f * a.D + c * EV, acc);
  }
}

// Fallback for other row sizes: one wavefront per (sample, field) bag, 64/LPR rows in
// flight, partial sums combined with a butterfly over the lane groups.
template <typename TT, typename OT>
__global__ __launch_bounds__(256) void pool_kernel(PoolArgs a, FieldPtr fp) {
  constexpr int EV = Vec16<TT>::N;
  const int lane = threadIdx.x & 63;
  const int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t sl = item / a.F;
  if (sl >= a.ns) return;
  const int f = (int)(item - sl * a.F);
  const int64_t s = a.s0 + sl;
  OT* xrow = reinterpret_cast<OT*>(a.x) + s * a.ldx;
  const int lpr = a.D / EV;  // lanes per row, power of two
  const int rpi = 64 / lpr;  // rows in flight
  const int sub = lane / lpr;
  const int c = lane - sub * lpr;
  const int32_t* off = a.offsets + (int64_t)f * (a.B + 1) + s;
  const int begin = off[0], end = off[1];
  const int32_t* ids = a.ids + fp.p[f];
  const TT* tab = reinterpret_cast<const TT*>(a.tables) + (int64_t)f * a.R * a.D + c * EV;
  if (a.lookup_sample)
    for (int j = begin + lane; j < end; j += 64) a.lookup_sample[fp.p[f] + j] = (int32_t)s;
  float acc[EV];
#pragma unroll
  for (int e = 0; e < EV; ++e) acc[e] = 0.0f;
  for (int j = begin + sub; j < end; j += rpi) {
    const int64_t row = min(max((int64_t)ids[j], (int64_t)0), a.R - 1);  // keeps a bad id in bounds
    Vec16<TT> v;
    v.v = *reinterpret_cast<const decltype(v.v)*>(tab + row * a.D);
#pragma unroll
    for (int e = 0; e < EV; ++e) acc[e] += v.get(e);
  }
  for (int o = lpr; o < 64; o <<= 1) {
#pragma unroll
    for (int e = 0; e < EV; ++e) acc[e] += __shfl_xor(acc[e], o, 64);
  }
  if (a.mean_pool && end - begin > 1) {
    const float len = (float)(end - begin);
#pragma unroll
    for (int e = 0; e < EV; ++e) acc[e] /= len;
  }
  if (sub == 0) store_row<OT, EV>(xrow + f * a.D + c * EV, acc);
}

template <typename OT>
__global__ __launch_bounds__(256) void pool_dense_kernel(PoolArgs a) {
  dense_columns<OT>(a, blockIdx.x * 64, a.ns);
}

template <typename TT, typename OT, int LPR, int SPB, bool ORDERED>
static void launch_pool_tiles(const PoolArgs& a, const FieldPtr& fp, hipStream_t s) {
  const dim3 grid(8 * (((a.ns + SPB - 1) / SPB * (a.F + 1) + 7) / 8)), block(256);
  if ((uint64_t)a.R * LPR >> 32) hipLaunchKernelGGL((pool_tile_kernel<TT, OT, LPR, SPB, ORDERED, true>), grid, block, 0, s, a, fp);
  else hipLaunchKernelGGL((pool_tile_kernel<TT, OT, LPR, SPB, ORDERED, false>), grid, block, 0, s, a, fp);
}

// 64 samples per block, or as many as the block takes at once (at most 32) where that leaves most of the places on the
// compute units empty and the round trips of one bag after the other are the kernel's time (a worker's step of 26 fields and small layers, us,
// 32 / 64 samples: 260 blocks of 64 47.4 / 48.6, 494 53.1 / 54.6, 832 57.3 / 58.1, 1040 67.0 / 67.1, 1664 82.9 / 83.1).
// The samples of a block in order (see pool_tile_kernel) from eight lookups a bag on, and where eight or more lanes take a row: shorter bags
// are of one length in iterations and pay for the order (the same, as they come / in order: 12 000 samples of 26 fields, bags of up to
// 8 / 20 / 50, rows of 8 lanes 59.8 / 60.3, 84.0 / 82.6, 145.5 / 143.9, of 16 lanes 101.4 / 102.5, 139 / 133, 230 / 214; bags of one, 100 fields,
// 4096 samples 174.8 / 177.4), and rows of 4 lanes, sixteen bags to a wavefront, lose by it at any length (100 fields, 12 000 samples, bags
// of up to 20 210 / 223).
template <typename TT, typename OT, int LPR>
static void launch_pool_row(const PoolArgs& a, const FieldPtr& fp, hipStream_t s) {
  if ((int64_t)((a.ns + 63) / 64) * a.F < 1024) launch_pool_tiles<TT, OT, LPR, (LPR > 8 ? 256 / LPR : 32), false>(a, fp, s);
  else if (LPR >= 8 && fp.p[a.F] >= (int64_t)8 * a.F * a.B) launch_pool_tiles<TT, OT, LPR, 64, (LPR >= 8)>(a, fp, s);
  else launch_pool_tiles<TT, OT, LPR, 64, false>(a, fp, s);
}

template <typename TT, typename OT>
static void launch_pool_typed(const PoolArgs& a, const FieldPtr& fp, hipStream_t s) {
  const int lpr = a.D / Vec16<TT>::N;
  if (lpr == 4) launch_pool_row<TT, OT, 4>(a, fp, s);
  else if (lpr == 8) launch_pool_row<TT, OT, 8>(a, fp, s);
  else if (lpr == 16) launch_pool_row<TT, OT, 16>(a, fp, s);
  else {
    const int64_t items = (int64_t)a.ns * a.F;
    hipLaunchKernelGGL((pool_kernel<TT, OT>), dim3((unsigned)((items + 3) / 4)), dim3(256), 0, s, a, fp);
    hipLaunchKernelGGL((pool_dense_kernel<OT>), dim3((a.ns + 63) / 64), dim3(256), 0, s, a);
  }
}

// Input check: flags[0] bit 0 = an id outside [0, R), bit 1 = offsets of a field that do not
// start at 0, decrease, or do not end at the field's lookup count; flags[1] = lowest offending
// field + 1.  Reads only what the host-side sizes cover, never through an offset.
__global__ __launch_bounds__(256) void validate_kernel(const int32_t* ids, const int32_t* offsets, FieldPtr fp,
                                                       int64_t B, int64_t R, int F, int32_t* flags) {
  const int f = blockIdx.y;
  const int64_t n = fp.p[f + 1] - fp.p[f];
  const int32_t* off = offsets + (int64_t)f * (B + 1);
  int bad = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int32_t id = ids[fp.p[f] + i];
    if (id < 0 || id >= R) bad |= 1;
  }
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i <= B; i += (int64_t)gridDim.x * 256) {
    const int64_t v = off[i];
    if (i == 0 && v != 0) bad |= 2;
    if (i == B && v != n) bad |= 2;
    if (i > 0 && v < off[i - 1]) bad |= 2;
  }
  if (bad) {
    atomicOr(&flags[0], bad);
    atomicMin(&flags[1], f + 1);
  }
}

__global__ void validate_reset_kernel(int32_t* flags) {
  if (threadIdx.x == 0) {
    flags[0] = 0;
    flags[1] = 0x7FFFFFFF;
  }
}

hipError_t launch_validate_reset(int32_t* flags, hipStream_t s) {
  hipLaunchKernelGGL(validate_reset_kernel, dim3(1), dim3(64), 0, s, flags);
  return hipGetLastError();
}

hipError_t launch_validate(const int32_t* ids, const int32_t* offsets, const FieldPtr& fp, int64_t B, int64_t R, int F,
                           int32_t* flags, hipStream_t s) {
  hipLaunchKernelGGL(validate_reset_kernel, dim3(1), dim3(64), 0, s, flags);
  int64_t work = B + 1;
  for (int f = 0; f < F; ++f) work = std::max<int64_t>(work, fp.p[f + 1] - fp.p[f]);
  const unsigned bx = (unsigned)std::min<int64_t>((work + 255) / 256, 1024);
  hipLaunchKernelGGL(validate_kernel, dim3(bx, F), dim3(256), 0, s, ids, offsets, fp, B, R, F, flags);
  return hipGetLastError();
}

hipError_t launch_pool(const PoolArgs& a, const FieldPtr& fp, hipStream_t s) {
  if (a.ns <= 0) return hipSuccess;
  if (a.table_bf16) {
    if (a.x_bf16) launch_pool_typed<bf16_t, bf16_t>(a, fp, s);
    else launch_pool_typed<bf16_t, float>(a, fp, s);
  } else {
    if (a.x_bf16) launch_pool_typed<float, bf16_t>(a, fp, s);
    else launch_pool_typed<float, float>(a, fp, s);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------------
__device__ __forceinline__ uint32_t fmix32(uint32_t x) {
  x ^= x >> 16;
  x *= 0x85EBCA6Bu;
  x ^= x >> 13;
  x *= 0xC2B2AE35u;
  x ^= x >> 16;
  return x;
}

template <typename TT>
__global__ __launch_bounds__(256) void fill_tables_kernel(TT* tables, int F, int64_t R, int D, float scale) {
  const int64_t total = (int64_t)F * R * D;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
    const int64_t row = i / D;
    const int d = (int)(i - row * D);
    const int64_t f = row / R;
    const uint32_t r = (uint32_t)(row - f * R);
    const uint32_t h1 = fmix32(r + 0x9E3779B9u * (uint32_t)(f + 1));
    const uint32_t h = fmix32(h1 ^ (0x85EBCA6Bu * (uint32_t)(d + 1)));
    const float t = __fsub_rn(__fmul_rn((float)(h >> 8), 1.1920928955078125e-07f), 1.0f);
    tables[i] = from_f32<TT>(__fmul_rn(scale, t));
  }
}

hipError_t launch_fill_tables(void* tables, int bf16, int F, int64_t R, int D, float scale, hipStream_t s) {
  dim3 grid(256 * 16), block(256);
  if (bf16) hipLaunchKernelGGL(fill_tables_kernel<bf16_t>, grid, block, 0, s, (bf16_t*)tables, F, R, D, scale);
  else hipLaunchKernelGGL(fill_tables_kernel<float>, grid, block, 0, s, (float*)tables, F, R, D, scale);
  return hipGetLastError();
}

}  // namespace antdt
