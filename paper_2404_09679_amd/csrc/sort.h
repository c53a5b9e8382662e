// The sort of a field's lookups in one block, and what it shares with the sort over many blocks: used by the launches of
// coalesce.hip, and beside the weight gradients of fp32 models (gemm.hip).
#pragma once

#include "common.h"

namespace antdt {

constexpr int MAX_BINS = 1024;

__device__ __forceinline__ uint64_t lanemask_lt() {
  const unsigned lane = threadIdx.x & 63;
  return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// LDS traffic between the lanes of one wavefront: executed in program order, only the compiler has to keep it so.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// x summed over the lanes up to this one.
__device__ __forceinline__ uint32_t wave_prefix(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);   // rows of 16 lanes: one lane down, ...
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);   // ... eight
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);   // last lane of a row to the next row (rows 1 and 3)
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);   // lane 31 to rows 2 and 3
  return x;
}

// Lanes (among the valid ones) that hold the same digit.  Per bit: the lane's bit spread over a word, one compare
// for the ballot, and one three-operand logic operation per half of the mask (these instructions are what
// bounds the sort's scatter).
__device__ __forceinline__ uint64_t same_digit(uint32_t d, int rb, bool valid) {
  const uint64_t all = __ballot(valid);
  uint32_t lo = (uint32_t)all, hi = (uint32_t)(all >> 32);
  for (int b = 0; b < rb; ++b) {
    const uint32_t mine = (uint32_t)__builtin_amdgcn_sbfe((int)d, b, 1);   // 0 or ~0
    const uint64_t bal = __ballot(mine != 0);
    lo &= ~(mine ^ (uint32_t)bal);
    hi &= ~(mine ^ (uint32_t)(bal >> 32));
  }
  return (uint64_t)lo | ((uint64_t)hi << 32);
}

// All passes of a field's sort in one block, for fields of up to SMALL_THREADS * IT lookups: keys and sample
// indices stay in registers between the passes (item i of wavefront w: position 64 (w per + i) + lane, all wavefronts
// holding the same number `per` of items a lane) and trade places through LDS.  Same ranking, hence the same stable
// order, as the passes over many blocks, in one launch instead of three per pass; a block's time is a few microseconds per pass and 8 items of a
// thread.
// (26 fields of 1000 lookups, two passes: 29 us of kernels and their gaps -> one launch of 10 us.)
constexpr int SMALL_THREADS = 1024, SMALL_WAVES = SMALL_THREADS / 64;
struct SmallSortLds {   // and, behind it or elsewhere, SMALL_THREADS * IT words
  uint16_t cnt[SMALL_WAVES][MAX_BINS];
  uint16_t dpre[MAX_BINS];
  uint32_t wsum[SMALL_WAVES];
};
template <int IT>
__device__ __forceinline__ void sort_small_field(SmallSortLds& lds, int32_t* stage, const int32_t* keys_in, const int32_t* pay_in, int32_t* keys_out,
                                                 int32_t* pay_out, int nnz, int passes, int rb) {
  if (nnz == 0) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int per = (nnz + SMALL_THREADS - 1) / SMALL_THREADS;   // <= IT
  const int first = w * (64 * per) + lane;
  auto mine = [&](int i) { return i < per && first + i * 64 < nnz; };
  int32_t key[IT], pay[IT];
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int pos = min(first + i * 64, nnz - 1);
    if (i < per) {
      key[i] = keys_in[pos];
      pay[i] = pay_in[pos];
    }
  }
  const int nb = 1 << rb;   // (at most one digit per thread)
  const uint64_t lt = lanemask_lt();
  for (int p = 0; p < passes; ++p) {
    const int shift = p * rb;
    for (int d = lane; d < nb; d += 64) lds.cnt[w][d] = 0;   // (each wavefront its own row)
    wave_lds_order();
    uint32_t rank[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      rank[i] = 0;
      if (i < per && w * (64 * per) + i * 64 < nnz) {   // (uniform)
        const bool valid = first + i * 64 < nnz;
        const uint32_t d = ((uint32_t)key[i] >> shift) & (nb - 1);
        const uint64_t m = same_digit(d, rb, valid);
        const uint32_t prior = lds.cnt[w][d];
        wave_lds_order();
        rank[i] = prior + (uint32_t)__popcll(m & lt);
        if (valid && (m & lt) == 0) lds.cnt[w][d] = (uint16_t)(prior + (uint32_t)__popcll(m));   // lowest lane of the group
        wave_lds_order();
      }
    }
    __syncthreads();
    // per digit: exclusive prefix over the wavefronts, then over the digits
    uint32_t tot = 0;
    if ((int)threadIdx.x < nb) {
      uint32_t c[SMALL_WAVES];
#pragma unroll
      for (int q = 0; q < SMALL_WAVES; ++q) c[q] = lds.cnt[q][threadIdx.x];
#pragma unroll
      for (int q = 0; q < SMALL_WAVES; ++q) {
        lds.cnt[q][threadIdx.x] = (uint16_t)tot;
        tot += c[q];
      }
    }
    const uint32_t incl = wave_prefix(tot);
    if (lane == 63) lds.wsum[w] = incl;
    __syncthreads();
    uint32_t before = 0;
    for (int q = 0; q < w; ++q) before += lds.wsum[q];
    if ((int)threadIdx.x < nb) lds.dpre[threadIdx.x] = (uint16_t)(before + incl - tot);
    __syncthreads();
    uint32_t place[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      if (i >= per) break;
      const uint32_t d = ((uint32_t)key[i] >> shift) & (nb - 1);
      place[i] = lds.dpre[d] + lds.cnt[w][d] + rank[i];
    }
    auto trade = [&](int32_t (&x)[IT]) {
#pragma unroll
      for (int i = 0; i < IT; ++i)
        if (mine(i)) stage[place[i]] = x[i];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < IT; ++i)
        if (mine(i)) x[i] = stage[first + i * 64];
      __syncthreads();
    };
    trade(key);
    trade(pay);
  }
#pragma unroll
  for (int i = 0; i < IT; ++i)
    if (mine(i)) {
      keys_out[first + i * 64] = key[i];
      pay_out[first + i * 64] = pay[i];
    }
}

// One pass of a field's sort by a block of a launch that does something else beside it (gemm.hip): up to PASS_KEYS lookups from memory to memory,
// in the same stable order.
constexpr int PASS_KEYS = 4096;
struct SortPass {
  const int32_t *keys_in, *pay_in;
  int32_t *keys_out, *pay_out;
  int32_t F, shift, rb;
  FieldPtr fp;
};
template <int THREADS>
struct SortPassLds {
  uint16_t cnt[THREADS / 64][MAX_BINS];
  uint16_t dpre[MAX_BINS];
  uint32_t wsum[THREADS / 64];
};
template <int THREADS>
__device__ __forceinline__ void sort_pass_field(const SortPass& sp, int f, SortPassLds<THREADS>& lds) {
  constexpr int IT = PASS_KEYS / THREADS, WAVES = THREADS / 64, DIGITS = MAX_BINS / THREADS;   // digits of a thread: DIGITS threadIdx.x + q
  const int64_t base = sp.fp.p[f];
  const int n = (int)min(sp.fp.p[f + 1] - base, (int64_t)PASS_KEYS);
  if (n == 0) return;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nb = 1 << sp.rb;
  const int per = (n + THREADS - 1) / THREADS;   // <= IT; item i of wavefront w: position 64 (w per + i) + lane
  const int first = w * (64 * per) + lane;
  int32_t key[IT], pay[IT];
#pragma unroll
  for (int i = 0; i < IT; ++i)
    if (i < per) {
      const int pos = min(first + i * 64, n - 1);
      key[i] = sp.keys_in[base + pos];
      pay[i] = sp.pay_in[base + pos];
    }
  for (int d = lane; d < nb; d += 64) lds.cnt[w][d] = 0;   // (each wavefront its own row)
  wave_lds_order();
  const uint64_t lt = lanemask_lt();
  uint32_t rank[IT];
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    rank[i] = 0;
    if (i < per && w * (64 * per) + i * 64 < n) {   // (uniform)
      const bool valid = first + i * 64 < n;
      const uint32_t d = ((uint32_t)key[i] >> sp.shift) & (uint32_t)(nb - 1);
      const uint64_t m = same_digit(d, sp.rb, valid);
      const uint32_t prior = lds.cnt[w][d];
      wave_lds_order();
      rank[i] = prior + (uint32_t)__popcll(m & lt);
      if (valid && (m & lt) == 0) lds.cnt[w][d] = (uint16_t)(prior + (uint32_t)__popcll(m));   // lowest lane of the group
      wave_lds_order();
    }
  }
  __syncthreads();
  // per digit: exclusive prefix over the wavefronts, then over the digits
  uint32_t tot[DIGITS], sum = 0;
#pragma unroll
  for (int q = 0; q < DIGITS; ++q) {
    const int d = (int)threadIdx.x * DIGITS + q;
    tot[q] = 0;
    if (d < nb) {
      uint32_t c[WAVES];
#pragma unroll
      for (int v = 0; v < WAVES; ++v) c[v] = lds.cnt[v][d];
#pragma unroll
      for (int v = 0; v < WAVES; ++v) {
        lds.cnt[v][d] = (uint16_t)tot[q];
        tot[q] += c[v];
      }
    }
    sum += tot[q];
  }
  const uint32_t incl = wave_prefix(sum);
  if (lane == 63) lds.wsum[w] = incl;
  __syncthreads();
  uint32_t before = incl - sum;
  for (int q = 0; q < w; ++q) before += lds.wsum[q];
#pragma unroll
  for (int q = 0; q < DIGITS; ++q) {
    const int d = (int)threadIdx.x * DIGITS + q;
    if (d < nb) lds.dpre[d] = (uint16_t)before;
    before += tot[q];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < IT; ++i)
    if (i < per && first + i * 64 < n) {
      const uint32_t d = ((uint32_t)key[i] >> sp.shift) & (uint32_t)(nb - 1);
      const uint32_t place = lds.dpre[d] + lds.cnt[w][d] + rank[i];
      if (place < (uint32_t)n) {
        sp.keys_out[base + place] = key[i];
        sp.pay_out[base + place] = pay[i];
      }
    }
}
inline bool passes_fit(int F, const FieldPtr& fp) {
  for (int f = 0; f < F; ++f)
    if (fp.p[f + 1] - fp.p[f] > PASS_KEYS) return false;
  return true;
}

// Lookups per thread (2, 4, 8 or 16) that the longest field takes, 0 if it does not fit one block.
inline int small_sort_items(int F, const FieldPtr& fp) {
  int64_t most = 0;
  for (int f = 0; f < F; ++f) most = fp.p[f + 1] - fp.p[f] > most ? fp.p[f + 1] - fp.p[f] : most;
  for (int it = 2; it <= 16; it *= 2)
    if (most <= (int64_t)SMALL_THREADS * it) return it;
  return 0;
}

}  // namespace antdt
