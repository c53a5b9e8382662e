// MLP matrix products of the worker step (forward, data gradient, weight gradient).
//   bf16 operands / fp32 accumulate: LDS-tiled kernels on the gfx950 matrix cores (mfma.h);
//   fp32 operands: matrix cores as well (v_mfma_f32_16x16x4_f32: fp32 products and sums), operands straight
//   from memory to registers.
#include <algorithm>

#include "mfma.h"
#include "sort.h"

namespace antdt {
namespace {

// Two packed bf16 values, each kept where the matching mask value is positive.
__device__ __forceinline__ uint32_t relu_mask2(uint32_t v, uint32_t mk) {
  const uint32_t lo = ((mk & 0x8000u) == 0 && (mk & 0x7FFFu) != 0) ? 0x0000FFFFu : 0u;
  const uint32_t hi = ((mk & 0x80000000u) == 0 && (mk & 0x7FFF0000u) != 0) ? 0xFFFF0000u : 0u;
  return v & (lo | hi);
}

// LDS traffic between the lanes of one wavefront: executed in program order, so only the compiler has
// to be kept from reordering it.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

template <int TM, int TN>
__device__ __forceinline__ void zero_acc(f32x16 (&acc)[TM][TN]) {
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
}

// C[m, n] = sum_k A(m, k) * B(n, k) with the epilogue of GemmArgs; A contiguous along k, B either way.
// Blocks are numbered so that an XCD (block i runs on XCD i mod 8) has a share of consecutive tiles, and tiles along the shorter side of C
// are neighbours: of the longer operand an XCD's L2 then fetches its own share only, of the shorter one all.  (Rows of C
// neighbours always, weights of 2 to 8 MB fetched by all eight: 512 x 3840 x 1024 12.2 us, so 9.3; 256 x 832 x 1024 5.7 / 4.8.)
// The results leave through LDS, 32 rows of a wavefront's tile at a time: a lane of the MFMA result holds
// groups of four neighbouring columns of one row, which would be 8-byte stores (16 with fp32 results) all
// over 32 rows; staged, they are 16-byte stores of whole row segments.
template <int TM, int TN, int WR, int WC, int BK, int STAGES, bool B_STRIDED, bool FAR, int WAVES>
__device__ __forceinline__ void gemm_bf16_tile(GemmArgs p, int pid, int nblk, int tiles_minor, bool m_minor, char* lds) {
  typedef BlockProduct<TM, TN, WR, WC, BK, STAGES, false, B_STRIDED, FAR, WAVES> P;
  pid = (pid & 7) * (nblk >> 3) + min(pid & 7, nblk & 7) + (pid >> 3);
  const int major = pid / tiles_minor, minor = pid - major * tiles_minor;
  const int m0 = (m_minor ? minor : major) * P::BM, n0 = (m_minor ? major : minor) * P::BN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int fr = lane & 31, fg = lane >> 5;

  // One bias column per lane, requested ahead of the product and added at its end: a sum that started from the
  // bias would round differently, and where activations are bf16 such a difference grows from layer to layer.
  constexpr int WN = 32 * TN;
  static_assert(WN <= 64, "one bias column per lane");
  float bias = 0.0f;
  if (p.epi == EPI_BIAS_RELU) bias = p.bias[min(n0 + wave % WC * WN + lane % WN, p.N - 1)];
  f32x16 acc[TM][TN];
  zero_acc(acc);
  P::run(reinterpret_cast<const bf16_t*>(p.A), reinterpret_cast<const bf16_t*>(p.B), p.lda, p.ldb, p.M, p.N, m0, n0, 0,
         p.K, lds, acc);
  if (WAVES > WR * WC && wave >= WR * WC) return;
  __builtin_assume(wave < WR * WC);   // (which the compiler cannot see)
  const int wr = wave / WC, wc = wave % WC;
  const int mw = m0 + wr * (32 * TM), nw = n0 + wc * WN;
  if (p.bf16_out) {
    constexpr int SP = WN + 8;
    static_assert(WR * WC * 32 * SP * 2 <= P::LDS_BYTES, "epilogue staging");
    bf16_t* st = reinterpret_cast<bf16_t*>(lds) + wave * (32 * SP);
    constexpr int CPR = WN / 8, RPI = 64 / CPR;   // 16-byte pieces per row, rows per wavefront instruction
    const int rr = lane / CPR, cc = (lane % CPR) * 8;
    bf16_t* C = reinterpret_cast<bf16_t*>(p.C);
    if (p.epi == EPI_BIAS_RELU) {
      float* sb = reinterpret_cast<float*>(st);
      if (lane < WN) sb[lane] = bias;
      wave_lds_fence();
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float4 b = *reinterpret_cast<const float4*>(sb + j * 32 + 8 * v + 4 * fg);
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            acc[i][j][4 * v] += b.x; acc[i][j][4 * v + 1] += b.y; acc[i][j][4 * v + 2] += b.z; acc[i][j][4 * v + 3] += b.w;
          }
        }
      wave_lds_fence();
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          float x[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = acc[i][j][4 * v + e];
          const int c = j * 32 + 8 * v + 4 * fg;
          if (p.epi == EPI_BIAS_RELU) {
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = fmaxf(x[e], 0.0f);
          }
          *reinterpret_cast<uint2*>(st + fr * SP + c) = make_uint2(f2bf2(x[0], x[1]), f2bf2(x[2], x[3]));
        }
      wave_lds_fence();
#pragma unroll
      for (int r0 = 0; r0 < 32; r0 += RPI) {
        const int r = r0 + rr, m = mw + i * 32 + r, n = nw + cc;
        if (m < p.M && n < p.N) {   // (N is a multiple of 8)
          uint4 val = *reinterpret_cast<const uint4*>(st + r * SP + cc);
          if (p.epi == EPI_RELU_MASK) {
            const uint4 mk = *reinterpret_cast<const uint4*>(reinterpret_cast<const bf16_t*>(p.mask) + (int64_t)m * p.ldmask + n);
            val = make_uint4(relu_mask2(val.x, mk.x), relu_mask2(val.y, mk.y), relu_mask2(val.z, mk.z), relu_mask2(val.w, mk.w));
          }
          *reinterpret_cast<uint4*>(C + (int64_t)m * p.ldc + n) = val;
        }
      }
      wave_lds_fence();
    }
  } else {
    constexpr int SP = WN + 4;
    static_assert(WR * WC * 32 * SP * 4 <= P::LDS_BYTES, "epilogue staging");
    float* st = reinterpret_cast<float*>(lds) + wave * (32 * SP);
    constexpr int CPR = WN / 4, RPI = 64 / CPR;
    const int rr = lane / CPR, cc = (lane % CPR) * 4;
    float* C = reinterpret_cast<float*>(p.C);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          *reinterpret_cast<float4*>(st + fr * SP + j * 32 + 8 * v + 4 * fg) =
              make_float4(acc[i][j][4 * v], acc[i][j][4 * v + 1], acc[i][j][4 * v + 2], acc[i][j][4 * v + 3]);
      wave_lds_fence();
#pragma unroll
      for (int r0 = 0; r0 < 32; r0 += RPI) {
        const int r = r0 + rr, m = mw + i * 32 + r, n = nw + cc;
        if (m < p.M && n < p.N)   // (N and ldc are multiples of 4)
          *reinterpret_cast<float4*>(C + (int64_t)m * p.ldc + n) = *reinterpret_cast<const float4*>(st + r * SP + cc);
      }
      wave_lds_fence();
    }
  }
}

template <int TM, int TN, int WR, int WC, int BK, int STAGES, bool B_STRIDED, bool FAR, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void gemm_bf16_kernel(GemmArgs p, int tiles_minor, bool m_minor) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int nblk = gridDim.x - p.loss_blocks;
  if ((int)blockIdx.x >= nblk) {
    add_up_losses(p.loss + (blockIdx.x - nblk));
    return;
  }
  gemm_bf16_tile<TM, TN, WR, WC, BK, STAGES, B_STRIDED, FAR, WAVES>(p, blockIdx.x, nblk, tiles_minor, m_minor, lds);
}

// The same with a pass of the sort of the coming aggregation in the first blocks, a field each: neither waits for the other, and a small
// step's products leave most compute units idle (96 samples of 845-1024-512-256, 26 fields of 1000 lookups: the sort in a launch of its
// own behind the products 8.7 us).
template <int TM, int TN, int WR, int WC, int BK, int STAGES, bool B_STRIDED, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void gemm_bf16_sort_kernel(GemmArgs p, int tiles_minor, bool m_minor, SortPass sp) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int block = (int)blockIdx.x - sp.F, nblk = (int)gridDim.x - sp.F - p.loss_blocks;
  if (block < 0) sort_pass_field<64 * WAVES>(sp, blockIdx.x, *reinterpret_cast<SortPassLds<64 * WAVES>*>(lds));
  else if (block >= nblk) add_up_losses(p.loss + (block - nblk));
  else gemm_bf16_tile<TM, TN, WR, WC, BK, STAGES, B_STRIDED, false, WAVES>(p, block, nblk, tiles_minor, m_minor, lds);
}

// Weight gradients of all hidden layers in one launch (see WgradArgs): block = one tile of one layer's
//   [dW_l ; db_l] = [act_l ; 1]^T dH_{l+1}
// over sample ranges; both operands are read as they lie in memory, [sample, width].
//   WGRAD_STORE   the range of `shard`: written to that shard's flat gradient;
//   otherwise     every range's sum from zero, added up with the ranges' weights in range order
//                 (g = fma(w_k, sum_k, g), the order in which the stand-alone dense update adds the shards'
//                 gradients), then Adagrad on the tile and the bf16 copy of the new weights.
//                 WGRAD_ONE: a single range: its sum is scaled in place (fma(w, sum, 0) = w * sum), and the
//                 second set of accumulators is not needed (fewer registers leave more room for the kernels
//                 running beside it).
// The bias gradient comes from the blocks of the first tile row, as a product with a row of ones.
enum WgradMode { WGRAD_STORE, WGRAD_ONE, WGRAD_MANY };

__device__ __forceinline__ float adagrad1(float p, float& s, float g, float lr, float eps) {
  s = fmaf(g, g, s);
  return p - lr * g / (sqrtf(s) + eps);
}

// The last layer (one output): the loss kernel has summed dz * h (and dz, the bias gradient) over its tiles of
// samples, or, of a model without a hidden layer, may have left dz per sample (the sums are then formed from the samples,
// T: type of the input); 64 columns per block, four lanes of tiles or samples per column.
template <WgradMode MODE, typename T>
__device__ __forceinline__ void last_layer(const WgradArgs& u, const KSegments& seg, int block, int shard, int tid, float (*red)[64]) {
  const int tx = tid & 63, ty = tid >> 6;
  const int j = block * 64 + tx;
  const bool on = j <= u.width;
  const int q0 = MODE == WGRAD_STORE ? shard : 0, q1 = MODE == WGRAD_STORE ? q0 + 1 : seg.n;
  float g = 0.0f;
  for (int q = q0; q < q1; ++q) {
    float sum = 0.0f;
    if (on && ty < 4 && u.dz) {
      const T* x = reinterpret_cast<const T*>(u.A[0]) + min(j, u.width - 1);
#pragma unroll 8
      for (int s = seg.ks[q] + ty; s < seg.ke[q]; s += 4) sum = fmaf(j < u.width ? to_f32(x[(int64_t)s * u.lda[0]]) : 1.0f, u.dz[s], sum);
    } else if (on && ty < 4) {
      const float* x = u.part + j;
      int t = seg.ts[q] + ty;
      for (; t + 28 < seg.te[q]; t += 32) {   // eight loads in flight
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = x[(int64_t)(t + 4 * i) * u.ldpart];
#pragma unroll
        for (int i = 0; i < 8; ++i) sum += v[i];
      }
      for (; t < seg.te[q]; t += 4) sum += x[(int64_t)t * u.ldpart];
    }
    if (ty < 4) red[ty][tx] = sum;
    __syncthreads();
    sum = (red[0][tx] + red[1][tx]) + (red[2][tx] + red[3][tx]);
    g = MODE == WGRAD_STORE ? sum : fmaf(seg.w[q], sum, g);
    __syncthreads();
  }
  if (!on || ty != 0) return;
  const int64_t idx = u.last_off + j;
  if (MODE == WGRAD_STORE) {
    u.grads[(int64_t)(u.k0 + shard) * u.stride + idx] = g;
  } else {
    float s1 = u.state[idx];
    u.p[idx] = adagrad1(u.p[idx], s1, g, u.lr, u.eps);
    u.state[idx] = s1;
  }
}

template <int TM, int TN, int WR, int WC, int BK, int STAGES, WgradMode MODE, bool FAR>
__device__ __forceinline__ void wgrad_tile(const WgradArgs& u, const KSegments& seg, int tile, int shard, char* lds) {
  typedef BlockProduct<TM, TN, WR, WC, BK, STAGES, true, true, FAR> P;
  if (tile >= u.tile_base[u.n_layers]) {
    last_layer<MODE, bf16_t>(u, seg, tile - u.tile_base[u.n_layers], shard, threadIdx.x, reinterpret_cast<float(*)[64]>(lds));
    return;
  }
  int li = 0;
  while (li + 1 < u.n_layers && tile >= u.tile_base[li + 1]) ++li;
  const int pid = tile - u.tile_base[li];
  const int M = u.M[li], N = u.N[li];
  const int m0 = (pid / u.tiles_n[li]) * P::BM, n0 = (pid % u.tiles_n[li]) * P::BN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave / WC, wc = wave % WC;
  const int fr = lane & 31, fg = lane >> 5;
  const bool ones = m0 == 0 && wr == 0;

  f32x16 tot[TM][TN], totb[1][TN];
  zero_acc(tot);
  zero_acc(totb);
  if (MODE != WGRAD_MANY) {
    const int q = MODE == WGRAD_STORE ? shard : 0;
    P::template run<true>(reinterpret_cast<const bf16_t*>(u.A[li]), reinterpret_cast<const bf16_t*>(u.B[li]), u.lda[li], u.ldb[li], M, N, m0, n0, seg.ks[q], seg.ke[q], lds, tot, totb[0], ones);
    if (MODE == WGRAD_ONE) {
      const float w = seg.w[0];
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
#pragma unroll
          for (int i = 0; i < TM; ++i) tot[i][j][e] *= w;
          totb[0][j][e] *= w;
        }
    }
  } else {
    for (int q = 0; q < seg.n; ++q) {
      f32x16 acc[TM][TN], accb[1][TN];
      zero_acc(acc);
      zero_acc(accb);
      P::template run<true>(reinterpret_cast<const bf16_t*>(u.A[li]), reinterpret_cast<const bf16_t*>(u.B[li]), u.lda[li], u.ldb[li], M, N, m0, n0, seg.ks[q], seg.ke[q], lds, acc, accb[0], ones);
      const float w = seg.w[q];
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
#pragma unroll
          for (int i = 0; i < TM; ++i) tot[i][j][e] = fmaf(w, acc[i][j][e], tot[i][j][e]);
          totb[0][j][e] = fmaf(w, accb[0][j][e], totb[0][j][e]);
        }
    }
  }

  // Epilogue: each wavefront stages its tile through its own slice of the (free) LDS, 32 rows at a time, so that
  // a lane ends up with four consecutive columns of one row: 16-byte loads and stores throughout.
  constexpr int WN = 32 * TN, SP = WN + 4;
  static_assert(WR * WC * 32 * SP * 4 <= P::LDS_BYTES, "epilogue staging");
  const int mw = m0 + wr * (32 * TM), nw = n0 + wc * WN;
  float* st = reinterpret_cast<float*>(lds) + wave * (32 * SP);
  constexpr int CPR = WN / 4, RPI = 64 / CPR;
  const int rr = lane / CPR, cc = (lane % CPR) * 4;
  const int64_t base = u.w_off[li];
  float* out = MODE == WGRAD_STORE ? u.grads + (int64_t)(u.k0 + shard) * u.stride + base : nullptr;
  float* Pm = u.p + base;
  float* S = u.state + base;
  bf16_t* Wb = u.wb[li];
  auto finish4 = [&](int64_t idx, const float4& g, bool weight) {
    if (MODE == WGRAD_STORE) {
      *reinterpret_cast<float4*>(out + idx) = g;
      return;
    }
    const float4 p0 = *reinterpret_cast<const float4*>(Pm + idx);
    float4 s1 = *reinterpret_cast<const float4*>(S + idx);
    float4 p1;
    p1.x = adagrad1(p0.x, s1.x, g.x, u.lr, u.eps);
    p1.y = adagrad1(p0.y, s1.y, g.y, u.lr, u.eps);
    p1.z = adagrad1(p0.z, s1.z, g.z, u.lr, u.eps);
    p1.w = adagrad1(p0.w, s1.w, g.w, u.lr, u.eps);
    *reinterpret_cast<float4*>(S + idx) = s1;
    *reinterpret_cast<float4*>(Pm + idx) = p1;
    if (weight) *reinterpret_cast<uint2*>(Wb + idx) = make_uint2(f2bf2(p1.x, p1.y), f2bf2(p1.z, p1.w));
  };
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        *reinterpret_cast<float4*>(st + fr * SP + j * 32 + 8 * v + 4 * fg) =
            make_float4(tot[i][j][4 * v], tot[i][j][4 * v + 1], tot[i][j][4 * v + 2], tot[i][j][4 * v + 3]);
    wave_lds_fence();
#pragma unroll
    for (int r0 = 0; r0 < 32; r0 += RPI) {
      const int r = r0 + rr, m = mw + i * 32 + r, n = nw + cc;
      if (m < M && n < N)   // (N is a multiple of 8: the four columns are inside together)
        finish4((int64_t)m * N + n, *reinterpret_cast<const float4*>(st + r * SP + cc), true);
    }
    wave_lds_fence();
  }
  if (ones && fr == 0) {   // every row of the product with ones is the same
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int n = nw + j * 32 + 8 * v + 4 * fg;
        if (n < N)
          finish4((int64_t)M * N + n, make_float4(totb[0][j][4 * v], totb[0][j][4 * v + 1], totb[0][j][4 * v + 2], totb[0][j][4 * v + 3]), false);
      }
  }
}

template <int TM, int TN, int WR, int WC, int BK, int STAGES, WgradMode MODE, bool FAR>
__global__ __launch_bounds__(64 * WR * WC) void wgrad_kernel(WgradArgs u, KSegments seg) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  wgrad_tile<TM, TN, WR, WC, BK, STAGES, MODE, FAR>(u, seg, blockIdx.x, blockIdx.y, lds);
}

// The per-shard weight gradients and, in further blocks, the gradient of the pooled input (GEMM: its tile) and the losses: neither
// waits for the other, and on one stream the second launch would wait for the first one's last block.
template <int TM, int TN, int WR, int WC, int BK, int STAGES>
__global__ __launch_bounds__(256) void wgrad_dgrad_kernel(WgradArgs u, KSegments seg, int tiles, GemmArgs p, int tiles_minor, bool m_minor) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  int i = blockIdx.x;
  if (i < tiles * seg.n) {
    wgrad_tile<1, 1, 2, 2, 64, 3, WGRAD_STORE, false>(u, seg, i % tiles, i / tiles, lds);
    return;
  }
  i -= tiles * seg.n;
  const int nblk = gridDim.x - tiles * seg.n - p.loss_blocks;
  if (i >= nblk) add_up_losses(p.loss + (i - nblk));
  else gemm_bf16_tile<TM, TN, WR, WC, BK, STAGES, false, false, 4>(p, i, nblk, tiles_minor, m_minor, lds);
}

// ---------------------------------------------------------------- fp32 products
// One wavefront computes TM x TN tiles of 16 x 16 with v_mfma_f32_16x16x4_f32 (fp32 throughout, twice the rate
// of the vector FMAs).  A step is 16 contraction slots, four MFMAs: lane (l & 15) of quarter l >> 4 supplies the
// slots 4 (l >> 4) .. + 3 of its row, one 16-byte load where the contraction index is contiguous, four loads
// of 16 neighbouring rows each where it is not.  No LDS: the models that use fp32 products are small, their
// products are bound by load latency and by how few tiles there are, so loads run D steps ahead and tiles
// stay small; what neighbouring wavefronts share comes from the L1.
// (Through LDS in 64 x 64 tiles, one step in flight: 1500 x 256 x 397 91 us, here 13; 1500 x 384 x 256 110 us, here 16;
// whole steps of an 845-1024-512-256 model with 512 / 4096 / 16384 samples 952 / 1145 / 3230 us, here 200 / 695 / 2400; of
// 653-2048-2048 with 4096 2550, here 2025.)
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));   // a 16-byte load takes any 4-byte-aligned address

// How an operand whose contraction index is contiguous is loaded: slot by slot (fewer than 4 slots), 16 bytes at a time
// from aligned rows (the last vector may reach into the row's padding), or from rows at any place.  845-1001-333
// model, 4096 / 16384 samples, a step: slot by slot 942 / 3103 us, from any place 590 / 1954; 845-1024-512-256 with
// 512 samples: aligned 201 us, as if at any place 207.
enum F32Load { F32_SLOTS, F32_ALIGNED, F32_ANY };

template <int T, bool KC, F32Load L>   // KC: contraction index contiguous
struct F32Operand {
  const float* row[T];
  int64_t ld;
  __device__ __forceinline__ F32Operand(const float* x, int64_t ld_, int r0, int rows, int lane) : ld(ld_) {
#pragma unroll
    for (int t = 0; t < T; ++t) {   // rows past the end repeat the last one (their products are not stored)
      const int r = min(r0 + 16 * t + (lane & 15), rows - 1);
      row[t] = KC ? x + (int64_t)r * ld : x + r;
    }
  }
  // Slots past the end are read at the last slot (or the last whole vector, or the last four) instead; `clip` moves the ones
  // that are inside to their places and clears the others.
  __device__ __forceinline__ void load(int step, int K, int lane, float (&f)[T][4]) const {
    const int k = step * 16 + 4 * (lane >> 4);
#pragma unroll
    for (int t = 0; t < T; ++t) {
      if (KC && L == F32_ALIGNED) {
        const float4 v = *reinterpret_cast<const float4*>(row[t] + min(k, (K - 1) & ~3));
        f[t][0] = v.x; f[t][1] = v.y; f[t][2] = v.z; f[t][3] = v.w;
      } else if (KC && L == F32_ANY) {
        const f32x4_any v = *reinterpret_cast<const f32x4_any*>(row[t] + min(k, K - 4));
        f[t][0] = v.x; f[t][1] = v.y; f[t][2] = v.z; f[t][3] = v.w;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) f[t][i] = row[t][KC ? (int64_t)min(k + i, K - 1) : (int64_t)min(k + i, K - 1) * ld];
      }
    }
  }
  static __device__ __forceinline__ void clip(int step, int K, int lane, float (&f)[T][4]) {
    const int k = step * 16 + 4 * (lane >> 4);
#pragma unroll
    for (int t = 0; t < T; ++t) {
      if (KC && L == F32_ANY) {
        const int over = k - (K - 4);   // 1 .. 3: slots the vector was read ahead of its place
        const bool by1 = over > 0 && (over & 1), by2 = over > 0 && (over & 2);
        const float g0 = by1 ? f[t][1] : f[t][0], g1 = by1 ? f[t][2] : f[t][1], g2 = by1 ? f[t][3] : f[t][2];
        f[t][0] = by2 ? g2 : g0;
        f[t][1] = by2 ? f[t][3] : g1;
        f[t][2] = g2;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) f[t][i] = k + i < K ? f[t][i] : 0.0f;
    }
  }
};

// acc = A B^T over the steps first, first + stride, ... of the K contraction slots; with `ones`, sum_b also
// receives the sums of B's rows (products with ones).  The four MFMAs of a step go to CH sums of their own, added up at
// the end: with four none waits for the one before, and chains a quarter as long round less (errors against 64
// bits of a 397-256-128 model's coalesced gradients 1.05e-7 with one, 7.7e-8 with four; 9.8e-8 in vector FMAs); the
// weight gradients, in four chains by wavefront already, keep one and the registers.  Result layout: lane l of acc[i][j] holds row l & 15
// and the columns 4 (l >> 4) .. + 3 of tile (i, j).
template <int TM, int TN, int D, int CH, bool ONES, typename OA, typename OB>
__device__ __forceinline__ void f32_product(const OA& oa, const OB& ob, int K, int first, int stride, int lane,
                                            f32x4 (&acc)[TM][TN], f32x4 (&sum_b)[TN], bool ones) {
  if (K <= 0) return;
  const int nk = (K + 15) / 16;
  f32x4 part[CH][TM][TN] = {}, part_b[CH][TN] = {};
  float a[D][TM][4], b[D][TN][4];
#pragma unroll
  for (int q = 0; q < D; ++q) {
    oa.load(first + q * stride, K, lane, a[q]);
    ob.load(first + q * stride, K, lane, b[q]);
  }
  for (int s = first; s < nk; s += D * stride) {
#pragma unroll
    for (int q = 0; q < D; ++q) {
      const int step = s + q * stride;
      if (step * 16 + 16 > K) {   // (uniform) partly or wholly past the end
        OA::clip(step, K, lane, a[q]);
        OB::clip(step, K, lane, b[q]);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            part[e % CH][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[q][j][e], a[q][i][e], part[e % CH][i][j], 0, 0, 0);
        if (ONES && ones) {
#pragma unroll
          for (int j = 0; j < TN; ++j)
            part_b[e % CH][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[q][j][e], 1.0f, part_b[e % CH][j], 0, 0, 0);
        }
      }
      oa.load(step + D * stride, K, lane, a[q]);
      ob.load(step + D * stride, K, lane, b[q]);
    }
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
#pragma unroll
    for (int i = 0; i < TM; ++i) acc[i][j] = CH == 4 ? (part[0][i][j] + part[1 % CH][i][j]) + (part[2 % CH][i][j] + part[3 % CH][i][j]) : part[0][i][j];
    if (ONES) sum_b[j] = CH == 4 ? (part_b[0][j] + part_b[1 % CH][j]) + (part_b[2 % CH][j] + part_b[3 % CH][j]) : part_b[0][j];
  }
}

// C[m, n] = sum_k A[m * lda + k] B(n, k) with the epilogue of GemmArgs: the tile of one wavefront.
template <int TM, int TN, int D, bool BKC, F32Load L>
__device__ __forceinline__ void gemm_f32_tile(GemmArgs p, int tiles_n, int id) {
  const int lane = threadIdx.x & 63;
  const int m0 = id / tiles_n * (16 * TM), n0 = id % tiles_n * (16 * TN);
  const F32Operand<TM, true, L> oa(reinterpret_cast<const float*>(p.A), p.lda, m0, p.M, lane);
  const F32Operand<TN, BKC, L> ob(reinterpret_cast<const float*>(p.B), p.ldb, n0, p.N, lane);
  f32x4 acc[TM][TN] = {}, none[TN];
  f32_product<TM, TN, D, 4, false>(oa, ob, p.K, 0, 1, lane, acc, none, false);
  float* C = reinterpret_cast<float*>(p.C);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int m = m0 + 16 * i + (lane & 15);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int n = n0 + 16 * j + 4 * (lane >> 4) + e;
        if (m >= p.M || n >= p.N) continue;
        float v = acc[i][j][e];
        if (p.epi == EPI_BIAS_RELU) v = fmaxf(v + p.bias[n], 0.0f);
        else if (p.epi == EPI_RELU_MASK) v = reinterpret_cast<const float*>(p.mask)[(int64_t)m * p.ldmask + n] > 0.0f ? v : 0.0f;
        C[(int64_t)m * p.ldc + n] = v;
      }
    }
}

// Four wavefronts per block, each a tile of its own (neighbours along n first: they share the rows of A).
template <int TM, int TN, int D, bool BKC, F32Load L>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs p, int tiles_n, int tiles) {
  const int nblk = gridDim.x - p.loss_blocks;
  if ((int)blockIdx.x >= nblk) {
    add_up_losses(p.loss + (blockIdx.x - nblk));
    return;
  }
  const int id = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (id < tiles) gemm_f32_tile<TM, TN, D, BKC, L>(p, tiles_n, id);
}

// Per-shard weight gradients of an fp32 model: tile blockIdx.x, shard blockIdx.y (wgrad_kernel's WGRAD_STORE).  The
// four wavefronts of a block share one tile and take every fourth step of the contraction (over samples:
// there are few tiles and the contraction is long); their sums are added in LDS.  397-256-128 model, 1500 samples
// of five shards: 16 us, against 177 us for the four products and bias sums of one layer each before.
// (By 256 threads; `tid`: this one's number among them.  Two barriers either way.)
template <int TM, int TN> struct WgradF32Lds {
  static constexpr int BM = 16 * TM, BN = 16 * TN, PITCH = BN + 4;
  float red[4][(BM + 1) * PITCH];   // row BM: the bias gradient
};
template <int TM, int TN, int D>
__device__ __forceinline__ void wgrad_f32_tile(const WgradArgs& u, const KSegments& seg, int tile, int q, int tid, WgradF32Lds<TM, TN>& lds) {
  typedef WgradF32Lds<TM, TN> Lds;
  constexpr int BM = Lds::BM, BN = Lds::BN, PITCH = Lds::PITCH;
  auto& red = lds.red;
  if (tile >= u.tile_base[u.n_layers]) {
    last_layer<WGRAD_STORE, float>(u, seg, tile - u.tile_base[u.n_layers], q, tid, reinterpret_cast<float(*)[64]>(&red[0][0]));
    return;
  }
  int li = 0;
  while (li + 1 < u.n_layers && tile >= u.tile_base[li + 1]) ++li;
  const int pid = tile - u.tile_base[li];
  const int M = u.M[li], N = u.N[li];
  const int m0 = (pid / u.tiles_n[li]) * BM, n0 = (pid % u.tiles_n[li]) * BN;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool ones = m0 == 0;
  f32x4 acc[TM][TN] = {}, accb[TN] = {};
  const float* A = reinterpret_cast<const float*>(u.A[li]) + (int64_t)seg.ks[q] * u.lda[li];
  const float* B = reinterpret_cast<const float*>(u.B[li]) + (int64_t)seg.ks[q] * u.ldb[li];
  const F32Operand<TM, false, F32_SLOTS> oa(A, u.lda[li], m0, M, lane);
  const F32Operand<TN, false, F32_SLOTS> ob(B, u.ldb[li], n0, N, lane);
  f32_product<TM, TN, D, 1, true>(oa, ob, seg.ke[q] - seg.ks[q], wave, 4, lane, acc, accb, ones);
  float* mine = red[wave];
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int c = 16 * j + 4 * (lane >> 4);
#pragma unroll
    for (int i = 0; i < TM; ++i) *reinterpret_cast<f32x4*>(mine + (16 * i + (lane & 15)) * PITCH + c) = acc[i][j];
    if ((lane & 15) == 0) *reinterpret_cast<f32x4*>(mine + BM * PITCH + c) = accb[j];   // (all its rows are the same)
  }
  __syncthreads();
  float* out = u.grads + (int64_t)(u.k0 + q) * u.stride + u.w_off[li];
  for (int e = tid; e < (BM + (ones ? 1 : 0)) * BN; e += 256) {
    const int r = e / BN, c = e % BN, n = n0 + c;
    const int m = r == BM ? M : m0 + r;   // the bias lies behind the weights
    if (n >= N || (r < BM && m >= M)) continue;
    const int o = r * PITCH + c;
    out[(int64_t)m * N + n] = (red[0][o] + red[1][o]) + (red[2][o] + red[3][o]);
  }
  __syncthreads();
}

template <int TM, int TN, int D>
__global__ __launch_bounds__(256) void wgrad_f32_kernel(WgradArgs u, KSegments seg) {
  __shared__ __attribute__((aligned(16))) WgradF32Lds<TM, TN> lds;
  wgrad_f32_tile<TM, TN, D>(u, seg, blockIdx.x, blockIdx.y, threadIdx.x, lds);
}

// The gradient of the pooled input (and the losses) in further blocks of the launch of the weight gradients: neither waits for the other.
struct DgradF32 {
  GemmArgs p;
  int32_t tiles_n, tiles;   // of gemm_f32_tile, one per wavefront; 0: none
  int32_t aligned;          // F32_ALIGNED, else F32_ANY
};
template <int GT, int GD>   // GT: 16 x 16 pieces of a wavefront's tile, each way; 0: no such blocks (their registers cost the others 8 - 15 us of 150 - 200)
__device__ __forceinline__ void dgrad_f32_block(DgradF32 d, int block, int waves) {
  const int id = block * waves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nblk = (d.tiles + waves - 1) / waves;
  if (block >= nblk) {
    if (block - nblk < d.p.loss_blocks) add_up_losses(d.p.loss + (block - nblk));
    return;
  }
  if (id >= d.tiles) return;
  if (d.aligned) gemm_f32_tile<GT, GT, GD, true, F32_ALIGNED>(d.p, d.tiles_n, id);
  else gemm_f32_tile<GT, GT, GD, true, F32_ANY>(d.p, d.tiles_n, id);
}

template <int TM, int TN, int D, int GT, int GD>
__global__ __launch_bounds__(256) void wgrad_dgrad_f32_kernel(WgradArgs u, KSegments seg, int tiles, DgradF32 d) {
  __shared__ __attribute__((aligned(16))) WgradF32Lds<TM, TN> lds;
  const int i = blockIdx.x;
  if (i < tiles * seg.n) wgrad_f32_tile<TM, TN, D>(u, seg, i % tiles, i / tiles, threadIdx.x, lds);
  else dgrad_f32_block<GT, GD>(d, i - tiles * seg.n, 4);
}

// The same with the sort of the coming aggregation beside it, a field to a block ahead of the others, which do four tiles each:
// neither waits for the other, both leave most compute units idle, and one stream runs its launches one after the other
// (1500 samples, 397-256-128, 12 fields of 9000 lookups: 15 + 23 us apart, 256 samples, 141-64-32, 8 fields of 640: 5 + 6; together 31 and 8).
template <int TM, int TN, int D, int IT, int GT, int GD>
__global__ __launch_bounds__(SMALL_THREADS) void wgrad_f32_sort_kernel(WgradArgs u, KSegments seg, int tiles, SortBuffers sb, FieldPtr fp, int F,
                                                                       int passes, int rb, DgradF32 d) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  if ((int)blockIdx.x < F) {
    const int64_t base = fp.p[blockIdx.x];
    sort_small_field<IT>(*reinterpret_cast<SmallSortLds*>(lds), reinterpret_cast<int32_t*>(lds + sizeof(SmallSortLds)), sb.ids + base, sb.pay0 + base,
                         sb.key[0] + base, sb.pay[0] + base, (int)(fp.p[blockIdx.x + 1] - base), passes, rb);
    return;
  }
  const int block = (int)blockIdx.x - F, wblocks = (tiles * seg.n + 3) / 4;
  if constexpr (GT > 0) {
    if (block >= wblocks) {
      dgrad_f32_block<GT, GD>(d, block - wblocks, SMALL_THREADS / 64);
      return;
    }
  }
  const int sub = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), i = block * 4 + sub;
  if (i < tiles * seg.n) {
    wgrad_f32_tile<TM, TN, D>(u, seg, i % tiles, i / tiles, threadIdx.x & 255, reinterpret_cast<WgradF32Lds<TM, TN>*>(lds)[sub]);
  } else {   // (the others' barriers)
    __syncthreads();
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void cast_bf16_kernel(CastArgs a) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n_dst; i += stride)
    a.dst[i] = i < a.n_src ? f2bf(a.src[i]) : (bf16_t)0;
}

template <int TM, int TN, int WR, int WC, int BK, int STAGES, bool BS, bool FAR = false, int WAVES = WR * WC>
hipError_t launch_bf16(const GemmArgs& a, hipStream_t s) {
  typedef BlockProduct<TM, TN, WR, WC, BK, STAGES, false, BS, FAR, WAVES> P;
  static std::atomic<uint64_t> allowed{0};
  const hipError_t ok = allow_lds(gemm_bf16_kernel<TM, TN, WR, WC, BK, STAGES, BS, FAR, WAVES>, P::LDS_BYTES, 0, allowed);
  if (ok != hipSuccess) return ok;
  const int tiles_m = (a.M + P::BM - 1) / P::BM, tiles_n = (a.N + P::BN - 1) / P::BN;
  const bool m_minor = a.M < a.N;
  hipLaunchKernelGGL((gemm_bf16_kernel<TM, TN, WR, WC, BK, STAGES, BS, FAR, WAVES>), dim3(tiles_m * tiles_n + a.loss_blocks), dim3(P::THREADS),
                     P::LDS_BYTES, s, a, m_minor ? tiles_m : tiles_n, m_minor);
  return hipGetLastError();
}

template <int TM, int TN, int WR, int WC, int BK, int STAGES, bool BS, int WAVES>
hipError_t launch_bf16_or_sort(const GemmArgs& a, const SortPass* sp, hipStream_t s) {
  if (!sp) return launch_bf16<TM, TN, WR, WC, BK, STAGES, BS, false, WAVES>(a, s);
  typedef BlockProduct<TM, TN, WR, WC, BK, STAGES, false, BS, false, WAVES> P;
  constexpr int bytes = std::max(P::LDS_BYTES, (int)sizeof(SortPassLds<P::THREADS>));
  static std::atomic<uint64_t> allowed{0};
  const hipError_t ok = allow_lds(gemm_bf16_sort_kernel<TM, TN, WR, WC, BK, STAGES, BS, WAVES>, bytes, 0, allowed);
  if (ok != hipSuccess) return ok;
  const int tiles_m = (a.M + P::BM - 1) / P::BM, tiles_n = (a.N + P::BN - 1) / P::BN;
  const bool m_minor = a.M < a.N;
  hipLaunchKernelGGL((gemm_bf16_sort_kernel<TM, TN, WR, WC, BK, STAGES, BS, WAVES>), dim3(sp->F + tiles_m * tiles_n + a.loss_blocks), dim3(P::THREADS),
                     bytes, s, a, m_minor ? tiles_m : tiles_n, m_minor, *sp);
  return hipGetLastError();
}

// Tiles of a product of bf16 operands.
enum Bf16Tiles { TILES_FAR, TILES_256, TILES_128, TILES_128_DEEP, TILES_64, TILES_32_X_64, TILES_32, TILES_32_LOADERS };
Bf16Tiles bf16_tiles(const GemmArgs& a) {
  // A tile holds up to 256 rows of an operand (128 contraction slots of a strided one); its pieces are addressed by 32-bit
  // offsets where those reach.
  if (std::max(a.lda, a.ldb) * (256 * 2) >> 32) return TILES_FAR;
  const bool strided = !a.b_kc;   // (BS)
  auto blocks = [&](int bm, int bn) { return (int64_t)((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn); };
  // The largest tile that gives most of the 256 compute units a block wins (it reads the fewest operand bytes); below that
  // blocks that all find a place at once do, with few of them those that get their loads away fastest.  Measured (us; M x N x K):
  //   256 x 256 / 128 x 128:                            16384 x 1024 x 6400 187 / 226; 16384 x 3840 x 1024 151 / 183; 15625 x 1024 x 848 33 / 35;
  //   128 x 128 with two (two blocks to a compute unit) / three stages / 64 x 64:  8192 x 1024 x 848 19.2 / 20.4 / 27; 4096 x 1024 x 848
  //     15.0 / 11.7 / 16.6; 4096 x 832 x 1024 15.9 / 13.1 / 17; 2560 x 1024 x 848 14.5 / 10.9 / 12.9; 2048 x 1024 x 848 14.4 / 10.7 / 10.0; input-like
  //     operands (BS false) 3072 x 1024 x 512 10.3 / 9.0 / 8.6, 3072 x 832 x 1024 15.2 / 12.2 / 12.1, 768 x 3840 x 1024 15.8 / 12.6 / 12.8;
  //   64 x 64 / 32 x 64, loads by eight wavefronts / 32 x 32, by four / by its own:  1024 x 1024 x 848 7.1 / 8.4 / 10.7 / 11.7;
  //     512 x 1024 x 848 7.1 / 5.8 / 7.5 / 7.4; 1024 x 512 x 1024 6.8 / 5.9 / 6.3 / 6.2; 256 x 1024 x 848 6.3 / 5.6 / 5.7 / 5.8; 96 x 1024 x 848 6.3 / 5.4 /
  //     5.0 / 5.4; 64 x 256 x 512 4.5 / 4.2 / 3.9 / 4.1; BS false: 896 x 832 x 1024 7.5 / 8.4 / 7.5 / 6.8; 512 x 1024 x 512 5.2 / 4.8 / 4.8 / 4.8;
  //     64 x 832 x 1024 6.4 / 5.6 / 5.0 / 5.1.  (256 instead of 128 slots a stage, by four: 5.0, 3.7 and 4.5 us at 96, 64 and 64 samples, launched over and over,
  //     but a worker step on 64 samples 44.8 us, with 128 44.5: every launch fetches its instructions anew.)
  // 256 x 256 from 200 blocks on instead of 150 was measured over 75 models and calls of 150 .. 199 such blocks (a step, or a
  // worker's: 3000 samples of 3840-1024-512 222 -> 240 us, 166 -> 173; 9800 of 845-1024-512-256 287 -> 295, 210 -> 218): 1 .. 8 %
  // slower but for five, of 3.8 M lookups in tables of half a million rows and more, where the tiles wait for compute
  // units that the weight gradients hold (2501 samples of 3840-1024-512 392 -> 380).
  if (blocks(256, 256) >= 150) return TILES_256;
  if (blocks(128, 128) > 256) return TILES_128;
  if (blocks(128, 128) >= (strided ? 150 : 200)) return TILES_128_DEEP;
  if (blocks(32, 32) <= 256) return TILES_32_LOADERS;
  if (strided && blocks(32, 64) <= 256) return TILES_32_X_64;
  if (!strided && blocks(32, 32) <= 768) return TILES_32;
  return TILES_64;
}

// sp: a pass of the sort for the same launch, or NULL (see gemm_takes_sort).
template <bool BS>
hipError_t launch_bf16_sized(const GemmArgs& a, const SortPass* sp, hipStream_t s) {
  switch (bf16_tiles(a)) {
    case TILES_FAR: return launch_bf16<1, 1, 1, 1, 128, 3, BS, true>(a, s);
    case TILES_256: return launch_bf16<4, 2, 2, 4, 64, 2, BS>(a, s);
    case TILES_128: return launch_bf16<2, 1, 2, 4, 64, 2, BS>(a, s);
    case TILES_128_DEEP: return launch_bf16<2, 1, 2, 4, 64, 3, BS>(a, s);
    case TILES_64: return launch_bf16_or_sort<1, 1, 2, 2, 64, 3, BS, 4>(a, sp, s);
    case TILES_32_LOADERS: return launch_bf16_or_sort<1, 1, 1, 1, 128, 3, BS, 4>(a, sp, s);
    case TILES_32_X_64:
      if constexpr (BS) return launch_bf16_or_sort<1, 1, 1, 2, 128, 3, BS, 8>(a, sp, s);
      break;
    case TILES_32:
      if constexpr (!BS) return launch_bf16<1, 1, 1, 1, 128, 3, BS>(a, s);
      break;
  }
  return hipErrorInvalidValue;
}

bool f32_aligned(const void* x, int64_t ld) { return (ld & 3) == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0; }

template <int TM, int TN, int D>
hipError_t launch_f32_tile(const GemmArgs& a, hipStream_t s) {
  const int tiles_n = (a.N + 16 * TN - 1) / (16 * TN), tiles = (a.M + 16 * TM - 1) / (16 * TM) * tiles_n;
  const dim3 grid((tiles + 3) / 4 + a.loss_blocks), block(256);
  const F32Load load = f32_aligned(a.A, a.lda) && (!a.b_kc || f32_aligned(a.B, a.ldb)) ? F32_ALIGNED : a.K >= 4 ? F32_ANY : F32_SLOTS;
  auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, s, a, tiles_n, tiles); };
  if (load == F32_ALIGNED) a.b_kc ? launch(gemm_f32_kernel<TM, TN, D, true, F32_ALIGNED>) : launch(gemm_f32_kernel<TM, TN, D, false, F32_ALIGNED>);
  else if (load == F32_ANY) a.b_kc ? launch(gemm_f32_kernel<TM, TN, D, true, F32_ANY>) : launch(gemm_f32_kernel<TM, TN, D, false, F32_ANY>);
  else a.b_kc ? launch(gemm_f32_kernel<TM, TN, D, true, F32_SLOTS>) : launch(gemm_f32_kernel<TM, TN, D, false, F32_SLOTS>);
  return hipGetLastError();
}

// 32 x 32 per wavefront (half the operand bytes of 16 x 16) where that still leaves enough wavefronts; with 16 x 16 the operands'
// requests are the bound (six steps in flight instead of four: 12.3 -> 13.3 us).  A step, us, 16 x 16 / 32 x 32: input gradients
// in 512 / 528 / 564 / 756 / 1536 tiles of 32 193 / 195, 99.8 / 96.2, 107 / 103, 107 / 103, 147 / 136; forward products in 752 / 768 / 1024
// (256 columns) / 1024 (1001) tiles 122.7 / 124.2, 234.8 / 233.3, 136.0 / 134.3, 226 / 212.  Every tile shape adds up the products in the same order.
bool f32_wide(const GemmArgs& a) { return (int64_t)((a.M + 31) / 32) * ((a.N + 31) / 32) > (a.b_kc ? 512 : 767); }
hipError_t launch_f32(const GemmArgs& a, hipStream_t s) {
  if (f32_wide(a)) return launch_f32_tile<2, 2, 2>(a, s);
  return launch_f32_tile<1, 1, 4>(a, s);
}

template <int TM, int TN, int D, int IT, int GT, int GD>
hipError_t launch_wgrad_f32_sort(const WgradArgs& u, const KSegments& seg, int tiles, const SortPlan& pl, const SortBuffers& sb, const FieldPtr& fp,
                                 const DgradF32& d, hipStream_t s) {
  constexpr int sort_bytes = (int)sizeof(SmallSortLds) + SMALL_THREADS * IT * 4, tile_bytes = 4 * (int)sizeof(WgradF32Lds<TM, TN>);
  constexpr int bytes = sort_bytes > tile_bytes ? sort_bytes : tile_bytes, waves = SMALL_THREADS / 64;
  static std::atomic<uint64_t> allowed{0};
  const hipError_t ok = allow_lds(wgrad_f32_sort_kernel<TM, TN, D, IT, GT, GD>, bytes, 0, allowed);
  if (ok != hipSuccess) return ok;
  const int blocks = pl.F + (tiles * seg.n + 3) / 4 + (d.tiles + waves - 1) / waves + d.p.loss_blocks;
  hipLaunchKernelGGL((wgrad_f32_sort_kernel<TM, TN, D, IT, GT, GD>), dim3(blocks), dim3(SMALL_THREADS), bytes, s, u, seg, tiles, sb, fp,
                     pl.F, pl.passes, pl.radix_bits, d);
  return hipGetLastError();
}

template <int TM, int TN, int D, int GT, int GD>
hipError_t launch_wgrad_f32_tile(const WgradArgs& a, const KSegments& seg, const SortPlan* pl, const SortBuffers* sb, const FieldPtr* fp,
                                 const GemmArgs* dgrad, hipStream_t s) {
  WgradArgs u = a;
  u.tile_base[0] = 0;
  for (int l = 0; l < u.n_layers; ++l) {
    u.tiles_n[l] = (u.N[l] + 16 * TN - 1) / (16 * TN);
    u.tile_base[l + 1] = u.tile_base[l] + (u.M[l] + 16 * TM - 1) / (16 * TM) * u.tiles_n[l];
  }
  const int tiles = u.tile_base[u.n_layers] + (u.width + 64) / 64;
  DgradF32 d = {};
  if constexpr (GT > 0) {
    d.p = *dgrad;
    d.tiles_n = (d.p.N + 16 * GT - 1) / (16 * GT);
    d.tiles = (d.p.M + 16 * GT - 1) / (16 * GT) * d.tiles_n;
    d.aligned = f32_aligned(d.p.A, d.p.lda) && f32_aligned(d.p.B, d.p.ldb);
  }
  if (pl) {
    switch (small_sort_items(pl->F, *fp)) {
      case 2: return launch_wgrad_f32_sort<TM, TN, D, 2, GT, GD>(u, seg, tiles, *pl, *sb, *fp, d, s);
      case 4: return launch_wgrad_f32_sort<TM, TN, D, 4, GT, GD>(u, seg, tiles, *pl, *sb, *fp, d, s);
      case 8: return launch_wgrad_f32_sort<TM, TN, D, 8, GT, GD>(u, seg, tiles, *pl, *sb, *fp, d, s);
      case 16: return launch_wgrad_f32_sort<TM, TN, D, 16, GT, GD>(u, seg, tiles, *pl, *sb, *fp, d, s);
      default: return hipErrorInvalidValue;
    }
  }
  if constexpr (GT > 0)
    hipLaunchKernelGGL((wgrad_dgrad_f32_kernel<TM, TN, D, GT, GD>), dim3(tiles * seg.n + (d.tiles + 3) / 4 + d.p.loss_blocks), dim3(256), 0, s, u, seg, tiles, d);
  else
    hipLaunchKernelGGL((wgrad_f32_kernel<TM, TN, D>), dim3(tiles, seg.n), dim3(256), 0, s, u, seg);
  return hipGetLastError();
}

int64_t wgrad_f32_tiles(const WgradArgs& a, int size) {   // of `size` rows and columns, of the hidden layers
  int64_t n = 0;
  for (int l = 0; l < a.n_layers; ++l) n += (int64_t)((a.M[l] + size - 1) / size) * ((a.N[l] + size - 1) / size);
  return n;
}
bool wgrad_f32_wide(const WgradArgs& a, int ranges) { return wgrad_f32_tiles(a, 32) * ranges >= 512; }

hipError_t launch_wgrad_f32(const WgradArgs& a, const KSegments& seg, const SortPlan* pl, const SortBuffers* sb, const FieldPtr* fp, const GemmArgs* dgrad,
                            hipStream_t s) {
  auto tiles = [&](auto gt, auto gd) {
    constexpr int GT = decltype(gt)::value, GD = decltype(gd)::value;
    if (wgrad_f32_wide(a, seg.n)) return launch_wgrad_f32_tile<2, 2, 2, GT, GD>(a, seg, pl, sb, fp, dgrad, s);
    return launch_wgrad_f32_tile<1, 1, 4, GT, GD>(a, seg, pl, sb, fp, dgrad, s);
  };
  typedef std::integral_constant<int, 0> None;
  if (!dgrad) return tiles(None(), None());
  if (f32_wide(*dgrad)) return tiles(std::integral_constant<int, 2>(), std::integral_constant<int, 2>());
  return tiles(std::integral_constant<int, 1>(), std::integral_constant<int, 4>());
}

template <int TM, int TN, int WR, int WC, int BK, int STAGES, WgradMode MODE, bool FAR = false>
hipError_t launch_wgrad_tile(const WgradArgs& a, const KSegments& seg, int groups, hipStream_t s) {
  typedef BlockProduct<TM, TN, WR, WC, BK, STAGES, true, true, FAR> P;
  static std::atomic<uint64_t> allowed{0};
  const hipError_t ok = allow_lds(wgrad_kernel<TM, TN, WR, WC, BK, STAGES, MODE, FAR>, P::LDS_BYTES, 0, allowed);
  if (ok != hipSuccess) return ok;
  WgradArgs u = a;
  u.tile_base[0] = 0;
  for (int l = 0; l < u.n_layers; ++l) {
    u.tiles_n[l] = (u.N[l] + P::BN - 1) / P::BN;
    u.tile_base[l + 1] = u.tile_base[l] + ((u.M[l] + P::BM - 1) / P::BM) * u.tiles_n[l];
  }
  hipLaunchKernelGGL((wgrad_kernel<TM, TN, WR, WC, BK, STAGES, MODE, FAR>), dim3(u.tile_base[u.n_layers] + (u.width + 64) / 64, groups),
                     dim3(P::THREADS), P::LDS_BYTES, s, u, seg);
  return hipGetLastError();
}

bool wgrad_far(const WgradArgs& a) {   // 64 samples of a tile beyond 32-bit offsets
  for (int l = 0; l < a.n_layers; ++l)
    if ((int64_t)std::max(a.lda[l], a.ldb[l]) * (64 * 2) >> 32) return true;
  return false;
}
// Every block walks all samples, so a large tile means few operand bytes per output but also few blocks.
// Measured alone (us; tiles of 128 x 128 with eight wavefronts / 64 x 64): 6400-1024-512 model, 16384 samples,
// one range (432 large tiles) 320 / 509; 3840-1024-512, 2501 samples, 16 ranges (272) 128 / 83;
// 845-1024-512-256, 4096 samples, one range (96) 61 / 39; 15625 samples, 8 ranges 269 / 167.
bool wgrad_large_tiles(const WgradArgs& a, int groups) {
  int n = 0;
  for (int l = 0; l < a.n_layers; ++l) n += ((a.M[l] + 127) / 128) * ((a.N[l] + 127) / 128);
  return n * groups >= 400;
}

template <WgradMode MODE>
hipError_t launch_wgrad_sized(const WgradArgs& a, const KSegments& seg, int groups, hipStream_t s) {
  if (wgrad_far(a)) return launch_wgrad_tile<1, 1, 2, 2, 64, 3, MODE, true>(a, seg, groups, s);
  if (wgrad_large_tiles(a, groups)) return launch_wgrad_tile<2, 1, 2, 4, 64, 2, MODE>(a, seg, groups, s);
  return launch_wgrad_tile<1, 1, 2, 2, 64, 3, MODE>(a, seg, groups, s);
}

template <int TM, int TN, int WR, int WC, int BK, int STAGES>
hipError_t launch_wgrad_dgrad_tile(const WgradArgs& a, const KSegments& seg, const GemmArgs& g, hipStream_t s) {
  typedef BlockProduct<1, 1, 2, 2, 64, 3, true, true> PW;
  typedef BlockProduct<TM, TN, WR, WC, BK, STAGES, false, false, false, 4> PG;
  static_assert(PW::THREADS == 256 && PG::THREADS == 256, "blocks of one launch");
  constexpr int bytes = std::max(PW::LDS_BYTES, PG::LDS_BYTES);
  static std::atomic<uint64_t> allowed{0};
  const hipError_t ok = allow_lds(wgrad_dgrad_kernel<TM, TN, WR, WC, BK, STAGES>, bytes, 0, allowed);
  if (ok != hipSuccess) return ok;
  WgradArgs u = a;
  u.tile_base[0] = 0;
  for (int l = 0; l < u.n_layers; ++l) {
    u.tiles_n[l] = (u.N[l] + PW::BN - 1) / PW::BN;
    u.tile_base[l + 1] = u.tile_base[l] + ((u.M[l] + PW::BM - 1) / PW::BM) * u.tiles_n[l];
  }
  const int tiles = u.tile_base[u.n_layers] + (u.width + 64) / 64;
  const int tiles_m = (g.M + PG::BM - 1) / PG::BM, tiles_n = (g.N + PG::BN - 1) / PG::BN;
  const bool m_minor = g.M < g.N;
  hipLaunchKernelGGL((wgrad_dgrad_kernel<TM, TN, WR, WC, BK, STAGES>), dim3(tiles * seg.n + tiles_m * tiles_n + g.loss_blocks), dim3(256), bytes, s,
                     u, seg, tiles, g, m_minor ? tiles_m : tiles_n, m_minor);
  return hipGetLastError();
}

}  // namespace

bool gemm_takes_sort(const GemmArgs& a) {   // (large tiles, and small ones of one wavefront, don't)
  if (a.M <= 0 || a.N <= 0 || !a.bf16_in) return false;
  const Bf16Tiles tiles = bf16_tiles(a);
  return tiles == TILES_64 || tiles == TILES_32_X_64 || tiles == TILES_32_LOADERS;
}
hipError_t launch_gemm(const GemmArgs& a, const SortPass* sp, hipStream_t s) {
  if (sp && !gemm_takes_sort(a)) return hipErrorInvalidValue;
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  if (!a.bf16_in) return launch_f32(a, s);
  return a.b_kc ? launch_bf16_sized<false>(a, sp, s) : launch_bf16_sized<true>(a, sp, s);
}

hipError_t launch_wgrad(const WgradArgs& a, const KSegments& seg, bool store, hipStream_t s) {
  if (store && seg.n <= 0) return hipSuccess;
  for (int l = 0; l < a.n_layers; ++l)
    if (a.M[l] <= 0 || a.N[l] <= 0 || (a.bf16 && (a.N[l] & 7))) return hipErrorInvalidValue;
  if (!a.bf16) return store ? launch_wgrad_f32(a, seg, nullptr, nullptr, nullptr, nullptr, s) : hipErrorInvalidValue;
  if (store) return launch_wgrad_sized<WGRAD_STORE>(a, seg, seg.n, s);
  return seg.n == 1 ? launch_wgrad_sized<WGRAD_ONE>(a, seg, 1, s) : launch_wgrad_sized<WGRAD_MANY>(a, seg, 1, s);
}

// Beside the sort the tiles lie four to a block that has the sort's LDS too, so fewer of them share a compute unit: that costs them
// about 6 us per 1000 blocks, and 15 - 20 us per million tiles (of 32) x samples where there are few (less where they fill several rounds
// of blocks: 4096 samples in eight shards, 12 fields of 12 000, 512-256 217 / 204).  What it saves is the
// sort's time, 4.5 / 8 / 16 / 25 us with 2 / 4 / 8 / 16 lookups a thread.  A step, us, one after the other / together (fp32, one stream;
// 512 samples in 1 / 4 / 12 shards, 26 fields of 1000 lookups): 256-128 81 / 77, 81 / 79, 89 / 90; 512-256 101 / 104, 100 / 101, 118 / 123;
// 1024-512-256 172 / 180, 176 / 181, 226 / 250; of 15 000 lookups: 121 / 111, 121 / 112, 130 / 113; 141 / 125, 142 / 126, 161 / 146; 215 / 198,
// 219 / 203, 269 / 271.  100 fields of 1300, 1024-512-256 in four shards 317 / 340; eight of 10 000, 2048-1024 in eight 356 / 373.
bool wgrad_takes_sort(const WgradArgs& a, int ranges, int64_t samples, int F, const FieldPtr& fp) {
  const int64_t saved = std::min(small_sort_items(F, fp), 12);   // (0: a field does not fit a block)
  if (a.bf16 || saved == 0) return false;
  const int64_t tiles = wgrad_f32_tiles(a, wgrad_f32_wide(a, ranges) ? 32 : 16) * ranges;
  const int64_t work = wgrad_f32_tiles(a, 32) * samples;
  return tiles <= 1280 * saved && work <= 100000 * saved * (tiles >= 2048 ? 4 : 3) / 3;
}

hipError_t launch_wgrad_and_sort(const WgradArgs& a, const KSegments& seg, const SortPlan& pl, const SortBuffers& sb, const FieldPtr& fp,
                                 const GemmArgs* dgrad, hipStream_t s) {
  for (int l = 0; l < a.n_layers; ++l)
    if (a.M[l] <= 0 || a.N[l] <= 0) return hipErrorInvalidValue;
  if (a.bf16 || seg.n <= 0) return hipErrorInvalidValue;
  return launch_wgrad_f32(a, seg, &pl, &sb, &fp, dgrad, s);
}

// One launch for both (us, apart / together; a worker step whose weight gradients belong to it): bf16, 1024-512-256, on 8 / 64 / 500 / 1531 / 3072 samples
// 43.2 / 39.4, 44.4 / 39.4, 51.4 / 43.9, 69.6 / 64.2, 126 / 121.  fp32, a whole step: 4096 / 16384 samples of 845-1024-512-256 692 / 675, 2228 / 2142;
// 4096 of 653-256-128 192 / 182; not where small tiles of the one, which want many wavefronts, would wait behind thousands of wide blocks of the other
// (512 of 845-1024-512-256 198 / 212).  In the launch that has the sort, blocks of 1024 threads with the sort's LDS and registers, only where all find a
// place at once, one or (small tiles, up to eight lookups a thread) two to a compute unit: 256 samples of 141-64-32 47.8 / 45.7, 1500 of 397-256-128
// 101.4 / 97.9, 1024 of 525-64-32 67.7 / 65.2; beyond it 4096 of 653-256-128 in eight shards 153 / 161.
bool wgrad_takes_dgrad(const WgradArgs& a, int ranges, const GemmArgs& g, int F, const FieldPtr* sorted) {
  if (ranges <= 0 || g.M <= 0 || g.N <= 0 || !g.b_kc) return false;
  if (a.bf16) {
    if (!g.bf16_in || sorted || wgrad_far(a) || wgrad_large_tiles(a, ranges) || std::max(g.lda, g.ldb) * (256 * 2) >> 32) return false;
    return (int64_t)((g.M + 127) / 128) * ((g.N + 127) / 128) < 200;   // (see bf16_tiles: else tiles of other blocks)
  }
  if (g.bf16_in || g.K < 4) return false;
  const bool wide = f32_wide(g), wgrad_wide = wgrad_f32_wide(a, ranges);
  const int size = wide ? 32 : 16;
  const int64_t tiles = (wgrad_f32_tiles(a, wgrad_wide ? 32 : 16) + (a.width + 64) / 64) * ranges;
  const int64_t dtiles = (int64_t)((g.M + size - 1) / size) * ((g.N + size - 1) / size);
  if (!sorted) return wide || !wgrad_wide || tiles + dtiles / 4 <= 1024;
  const int64_t blocks = F + (tiles + 3) / 4 + (dtiles + 15) / 16 + g.loss_blocks;
  return blocks <= (wide || wgrad_wide || small_sort_items(F, *sorted) > 8 ? 256 : 512);
}

hipError_t launch_wgrad_and_dgrad(const WgradArgs& a, const KSegments& seg, const GemmArgs& g, hipStream_t s) {
  for (int l = 0; l < a.n_layers; ++l)
    if (a.M[l] <= 0 || a.N[l] <= 0 || (a.bf16 && (a.N[l] & 7))) return hipErrorInvalidValue;
  if (!wgrad_takes_dgrad(a, seg.n, g, 0, nullptr)) return hipErrorInvalidValue;
  if (!a.bf16) return launch_wgrad_f32(a, seg, nullptr, nullptr, nullptr, &g, s);
  if ((int64_t)((g.M + 31) / 32) * ((g.N + 31) / 32) <= 256) return launch_wgrad_dgrad_tile<1, 1, 1, 1, 128, 3>(a, seg, g, s);
  return launch_wgrad_dgrad_tile<1, 1, 2, 2, 64, 3>(a, seg, g, s);
}

hipError_t launch_cast_bf16(const CastArgs& a, hipStream_t s) {
  if (a.n_dst <= 0) return hipSuccess;
  int64_t blocks = (a.n_dst + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(cast_bf16_kernel, dim3((unsigned)blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace antdt
