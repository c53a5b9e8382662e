// Shared declarations of the gfx950 kernels and their host-side launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "antdt.h"

#include <atomic>
#include <string>

namespace antdt {

void set_last_error(const std::string& msg);  // message returned by antdt_last_error(NULL)

typedef uint16_t bf16_t;  // raw bfloat16 bit pattern

__device__ __forceinline__ float bf2f(bf16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// Two floats -> two packed bfloat16 (lo in the low half), round to nearest even, NaN stays NaN: one instruction
// (v_cvt_pk_bf16_f32; checked against the integer formula for all 2^32 floats).
__device__ __forceinline__ uint32_t f2bf2(float lo, float hi) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const f32x2 v = {lo, hi};
  const bf16x2 h = __builtin_convertvector(v, bf16x2);
  return __builtin_bit_cast(uint32_t, h);
}

__device__ __forceinline__ bf16_t f2bf(float f) { return (bf16_t)f2bf2(f, f); }

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t x) { return bf2f(x); }
template <typename T> __device__ __forceinline__ T from_f32(float x);
template <> __device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float x) { return f2bf(x); }

// Small tables passed to kernels by value (kernel-argument segment), so that no
// host-to-device copy is needed per call.
struct FieldPtr {
  int64_t p[ANTDT_MAX_FIELDS + 1];  // start of each field's lookups inside ids
};
struct ShardTab {
  int32_t K;
  int32_t start[ANTDT_MAX_SHARDS];
  int32_t len[ANTDT_MAX_SHARDS];
  float w[ANTDT_MAX_SHARDS];  // aggregation weight B_k / sum of included B_k (0 if excluded)
};
struct WeightTab {   // ranges of samples of one aggregation weight, in sample order
  int32_t start[ANTDT_MAX_SHARDS];
  float w[ANTDT_MAX_SHARDS];
};
struct TileBase {
  int32_t t[ANTDT_MAX_FIELDS + 1];  // prefix sum of sort tiles per field
};

// Kernels whose blocks need more than 64 KB of LDS have to be allowed it, once per device; `done`: the devices (a bit
// each) on which that has been done for this kernel.
template <typename F>
inline hipError_t allow_lds(F kernel, int dynamic_bytes, int static_bytes, std::atomic<uint64_t>& done) {
  if (dynamic_bytes + static_bytes <= 64 * 1024) return hipSuccess;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = 1ull << (dev & 63);
  if (done.load(std::memory_order_relaxed) & bit) return hipSuccess;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, dynamic_bytes);
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_relaxed);
  return e;
}

// Kernel classes for the optional event timing.  (Ids are part of the C interface: classes whose kernels are gone
// keep their places and count no launches.)
enum KernelId {
  KID_POOL = 0,
  KID_GEMM_FWD,
  KID_GEMM_DGRAD,      // gone: counted under KID_GEMM_BWD
  KID_GEMM_WGRAD,      // (of an fp32 model with the sort, where it joins)
  KID_HEAD,
  KID_HEAD_REDUCE,     // gone: blocks of the input-gradient and the weight-gradient launch
  KID_BIAS_GRAD,       // gone: part of the weight gradients
  KID_SORT_HIST,
  KID_SORT_SCAN,
  KID_SORT_SCATTER,
  KID_SEG_HEADS,
  KID_SEG_SCAN,
  KID_SEG_EMIT,
  KID_SEG_REDUCE,
  KID_SEG_REDUCE_LONG,
  KID_DENSE_AGG,
  KID_SPARSE_ADAGRAD,
  KID_DENSE_ADAGRAD,
  KID_ADAM,
  KID_TRANSPOSE,       // gone
  KID_GEMM_BWD,
  KID_WGRAD_ADAGRAD,
  KID_COUNT
};

struct Profiler;  // defined in ctx.hip
int prof_begin(Profiler* p, int kid, hipStream_t s);   // returns the bracket's index, -1 if not timed
void prof_end(Profiler* p, int idx, hipStream_t s);
void prof_count(Profiler* p, int idx, int launches);   // launches covered by the bracket (default 1)

// A pair of events on stream `s` around the launches made while the scope is open.
struct ProfScope {
  Profiler* p;
  int idx = -1;
  hipStream_t s;
  ProfScope(Profiler* p_, int kid, hipStream_t s_) : p(p_), s(s_) {
    if (p) idx = prof_begin(p, kid, s);
  }
  ~ProfScope() { close(); }
  // One bracket around several back-to-back launches: the bracket itself costs a few
  // microseconds on the stream, which would swamp kernels of 10-20 us if each had its own.
  void launches(int n) {
    if (p && idx >= 0) prof_count(p, idx, n);
  }
  void close() {  // end the bracket before the scope does
    if (p && idx >= 0) prof_end(p, idx, s);
    p = nullptr;
  }
};

// ---------------------------------------------------------------- embed.hip
struct PoolArgs {
  const void* tables;
  const int32_t* ids;
  const int32_t* offsets;
  const float* dense;
  void* x;
  int32_t* lookup_sample; // optional [nnz]: global sample index of every lookup (sort payload)
  int32_t F, D, num_dense, ldx, B, s0, ns;
  int64_t R;
  int32_t table_bf16, x_bf16;
  int32_t mean_pool;      // divide every bag's sum by its number of lookups
};
hipError_t launch_pool(const PoolArgs& a, const FieldPtr& fp, hipStream_t s);
hipError_t launch_validate(const int32_t* ids, const int32_t* offsets, const FieldPtr& fp, int64_t B, int64_t R, int F,
                           int32_t* flags, hipStream_t s);
hipError_t launch_validate_reset(int32_t* flags, hipStream_t s);
hipError_t launch_fill_tables(void* tables, int bf16, int F, int64_t R, int D, float scale,
                              hipStream_t s);

// ----------------------------------------------------------------- gemm.hip
enum Epilogue { EPI_BIAS_RELU = 0, EPI_RELU_MASK = 1, EPI_PLAIN = 2 };

// C[m, n] = sum_k A(m, k) * B(n, k): A(m,k) = A[m*lda + k]; B(n,k) = B[n*ldb + k] (b_kc) or B[k*ldb + n].
struct GemmArgs {
  const void* A;
  const void* B;
  void* C;
  const float* bias;   // EPI_BIAS_RELU: [N]
  const void* mask;    // EPI_RELU_MASK: activations [M, ldmask], C = acc where mask > 0 else 0
  int64_t lda, ldb, ldc, ldmask;
  int32_t M, N, K;
  int32_t b_kc, epi;
  int32_t bf16_in;     // operands (and mask) are bf16, else fp32
  int32_t bf16_out;    // C is bf16, else fp32
  // Further blocks of the launch add up the losses that the loss kernel left per tile of samples, one shard each (nobody
  // waits for them, and counting the loss kernel's blocks to have its last one do it kept the chain waiting 3 us).
  int32_t loss_blocks;
  const struct LossJob* loss;   // [loss_blocks]
};
struct SortPass;   // sort.h
bool gemm_takes_sort(const GemmArgs& a);   // the launch has room for a pass of the sort
hipError_t launch_gemm(const GemmArgs& a, const SortPass* sp, hipStream_t s);   // sp: a pass of the sort for such a launch, or NULL

// Sample ranges (shards; neighbours of equal weight merged) in sample order, with their aggregation
// weights, and the partial sums that the loss kernel left for them.
struct KSegments {
  int32_t n;
  int32_t ks[ANTDT_MAX_SHARDS], ke[ANTDT_MAX_SHARDS];   // samples [ks, ke)
  int32_t ts[ANTDT_MAX_SHARDS], te[ANTDT_MAX_SHARDS];   // tiles of the loss kernel [ts, te)
  float w[ANTDT_MAX_SHARDS];
};
// Keys per sort tile (one block of 512 threads, ANTDT_SORT_TILE / 512 keys per thread).
constexpr int ANTDT_SORT_TILE = 2048;
struct SortPlan {
  int32_t F;
  int32_t passes, radix_bits;      // digit width per pass
  int32_t total_tiles;
  int64_t rows, samples;           // row ids and sample indices lie below
  int64_t width;                   // pooled inputs of a sample
  bool beside;                     // runs beside other work
};
struct SortBuffers {
  const int32_t* ids;
  const int32_t* pay0;             // sample index of every lookup (payload of the first pass)
  const int32_t* offsets;          // [F][samples + 1] bag boundaries, of a sort that finds the samples by itself (see sort_finds_samples), or NULL
  int32_t* key[2];
  int32_t* pay[2];
  uint32_t* hist;                  // [total_tiles << radix_bits]
  uint32_t* digit_total;            // [F << radix_bits]
  int32_t* slots;                  // scratch, a word per slot of the windows (window_slots), or NULL: none that is free
};
// Weight gradients of all layers in one launch (see wgrad_kernel, wgrad_f32_kernel): per range written to
// the shards' flat gradients, or aggregated and applied (Adagrad) on the spot, in which case neither
// the per-shard nor the aggregated gradient goes to memory.
struct WgradArgs {
  int32_t n_layers;                    // hidden layers
  int32_t bf16;                        // type of A and B
  const void* A[ANTDT_MAX_LAYERS];     // activations [samples, lda], M columns
  const void* B[ANTDT_MAX_LAYERS];     // pre-activation gradients [samples, ldb], N columns
  int32_t M[ANTDT_MAX_LAYERS], N[ANTDT_MAX_LAYERS], lda[ANTDT_MAX_LAYERS], ldb[ANTDT_MAX_LAYERS];
  int64_t w_off[ANTDT_MAX_LAYERS];     // W_l inside the flat parameters, [M, N] then the bias [N]
  bf16_t* wb[ANTDT_MAX_LAYERS];        // bf16 models: copy of W_l, [rows padded, N]
  int32_t tile_base[ANTDT_MAX_LAYERS + 1];
  int32_t tiles_n[ANTDT_MAX_LAYERS];
  // last layer (one output): the loss kernel's sums over its tiles of samples
  const float* part;                   // [tiles, ldpart] sum of dz * h per column; column `width`: sum of dz
  const float* dz;                     // models without a hidden layer: [samples] instead of those sums (A[0]: the input), or NULL
  int64_t ldpart, last_off;            // offset of the last layer in the flat parameters (bias behind the weights)
  int32_t width;
  float* p;
  float* state;
  float lr, eps;
  float* grads;                        // per-shard flat gradients [K, stride] (when storing), ranges = shards k0 ..
  int64_t stride;
  int32_t k0;
};
hipError_t launch_wgrad(const WgradArgs& a, const KSegments& seg, bool store, hipStream_t s);
// Per-shard gradients and, in the same launch, the gradient of the pooled input: where wgrad_takes_dgrad says so (`sorted`: the launch sorts
// those F fields too, else NULL).
bool wgrad_takes_dgrad(const WgradArgs& a, int ranges, const GemmArgs& g, int F, const FieldPtr* sorted);
hipError_t launch_wgrad_and_dgrad(const WgradArgs& a, const KSegments& seg, const GemmArgs& g, hipStream_t s);
// Per-shard gradients of an fp32 model and, in the same launch, the sort (launch_sort with every field in one block, result in
// key / pay [0]) and, unless NULL, the gradient of the pooled input (as above).
hipError_t launch_wgrad_and_sort(const WgradArgs& a, const KSegments& seg, const SortPlan& pl, const SortBuffers& sb, const FieldPtr& fp,
                                 const GemmArgs* dgrad, hipStream_t s);
bool wgrad_takes_sort(const WgradArgs& a, int ranges, int64_t samples, int F, const FieldPtr& fp);   // it pays

struct CastArgs {  // fp32 [rows, cols] -> bf16 [rows_pad, cols], extra rows zero
  const float* src;
  bf16_t* dst;
  int64_t n_src, n_dst;
};
hipError_t launch_cast_bf16(const CastArgs& a, hipStream_t s);

// ----------------------------------------------------------------- head.hip
struct HeadArgs {
  const void* h;        // [B, ldh] last hidden activation (or the pooled input when there is none)
  const float* w;       // [width] last-layer weight
  const float* b;       // [1]
  const float* labels;  // [B]
  void* dh;             // [B, lddh] gradient w.r.t. h (masked by h > 0 when `relu`), or fp32 dX
  int64_t ldh, lddh;
  int32_t width, dh_cols, relu, bf16_h, bf16_dh;
  int32_t k_begin, k_end;
  // the sums over the samples are formed along the way, per tile of samples of one shard
  float* part;          // [tiles, ldpart] sum of dz * h per column; column `width`: sum of dz, `width` + 1: of the losses
  int64_t ldpart;
  float* dz;            // [B] d(mean shard loss)/d logit of every sample, and [B] its loss, instead of those sums (or NULL)
  float* loss_s;
  struct LossJob* job;  // [K] those of the range's shards are written by the first block, for the launch that adds up the losses
  float* loss_out;      // caller's buffer or NULL; element (k - k_begin)
};
// Tiles of the loss kernel: HEAD_TILE consecutive samples of one shard.  tile_base[k] = first tile of shard k.
constexpr int HEAD_TILE = 16;
struct HeadTiles {
  int32_t base[ANTDT_MAX_SHARDS + 1];
};
inline HeadTiles head_tiles(const ShardTab& tab) {
  HeadTiles t;
  t.base[0] = 0;
  for (int k = 0; k < ANTDT_MAX_SHARDS; ++k)
    t.base[k + 1] = t.base[k] + (k < tab.K ? (tab.len[k] + HEAD_TILE - 1) / HEAD_TILE : 0);
  return t;
}
hipError_t launch_head_tiles(const HeadArgs& a, const ShardTab& tab, hipStream_t s);
hipError_t launch_losses(const LossJob* job, int shards, hipStream_t s);   // stand-alone, for models without a hidden layer

// The mean loss of a shard: its tiles' sums in a fixed order (lanes take every 64th tile).  One job per shard: worker
// steps of different shards may run on different streams at the same time.
struct LossJob {
  const float* sums;    // the first tile's sum of losses, ldpart further on the next one's
  float* loss_out;
  int64_t ldpart;
  int32_t tiles, len;   // samples: len
};
__device__ __forceinline__ void add_up_losses(const LossJob* job) {   // (the first wavefront of a block)
  if (threadIdx.x >= 64) return;
  // (pointers from memory are not known to be global ones, and a flat access makes the compiler wait for all loads in the rest of the kernel)
  typedef __attribute__((address_space(1))) float global_float;
  const global_float* sums = (const global_float*)job->sums;
  float l = 0.0f;
  for (int t = (int)threadIdx.x; t < job->tiles; t += 64) l += sums[(int64_t)t * job->ldpart];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o, 64);
  if (threadIdx.x == 0 && job->loss_out) *(global_float*)job->loss_out = job->len > 0 ? l / (float)job->len : 0.0f;
}

// ------------------------------------------------------------- coalesce.hip
// Pass `pass` of a sort whose fields fit sort_pass_field, for a launch of something else to take.
void plan_sort_pass(const SortPlan& pl, const SortBuffers& sb, const FieldPtr& fp, int pass, SortPass& sp);
// Whether launch_sort can do without sample indices, and work them out of the bags' boundaries (of a whole batch).
bool sort_finds_samples(const SortPlan& pl, const SortBuffers& sb, const FieldPtr& fp);
// Sorts every field's lookups by row id (stable); the result is in key / pay [*sorted_buf].
hipError_t launch_sort(const SortPlan& pl, const SortBuffers& sb, const FieldPtr& fp, const TileBase& tb, Profiler* prof, hipStream_t s,
                       int* sorted_buf);

// Slots of the windows: window i of a field that starts at lookup p has slot p / 128 + i.  A field of n > 256 lookups has
// ceil(n / 256) <= floor(n / 128) windows at most, so no two fields' windows meet and none lies past the last
// lookup's; a field in one window needs no slot (and has none).
inline int64_t window_slots(int64_t lookups) { return lookups >> 7; }

struct SegArgs {
  const int32_t* key;              // sorted row ids, field-major at fp.p[f]
  const int32_t* pay;              // sample index of each sorted lookup
  // run table (for the views only)
  int32_t* tile_heads;             // [total_tiles + 1] heads per tile -> exclusive prefix
  int32_t* ubase;                  // [F + 1] first unique of each field; ubase[F] = U
  int32_t* uniq;                   // [U] row id of each run
  int32_t* segabs;                 // [U + 1] start of each run in the sorted arrays (all fields)
  int32_t* segoff;                 // [U + F], per-field offsets; field f's slice starts at ubase[f] + f
  float* G;                        // [U, D] coalesced gradient (written when not updating)
  int32_t window;                  // sorted lookups per block of the reduction: 256 or 512, or (every field in one window) 1024 or 2048
  int32_t* goes_out;               // [slots] the last run of the window starts there, is long and goes on in the next one
  float* partial;                  // [slots, 2, D] sums over the window: of the run that comes in, of the run that goes out
  const float* dx;                 // [B, lddx]
  int64_t lddx;
  const int32_t* offsets;          // [F][B + 1] bag boundaries of the batch (read when mean_pool)
  int32_t mean_pool;               // bags are averaged: a lookup's gradient is dX / bag length
  int32_t F, D, B, total_tiles;
  // parameter update fused into the reduction (update != 0)
  int32_t update, table_bf16, rowwise;
  void* tables;
  float* state;
  int64_t R;
  float lr, eps, inv_dim;          // inv_dim: 1 / D
  int32_t weights;                 // (set by launch_seg_reduce) ranges of the table of weights; the first one's weight
  float weight;
};
hipError_t launch_expand_samples(const int32_t* offsets, int32_t* lookup_sample, const FieldPtr& fp, int F, int B, hipStream_t s);
hipError_t launch_segments(const SegArgs& a, const FieldPtr& fp, const TileBase& tb, Profiler* prof, hipStream_t s);
hipError_t launch_mask_pack(const int32_t* ids, const int32_t* lookup_sample, const int32_t* offsets, int64_t B, int F,
                            const FieldPtr& fp, const ShardTab& tab, int64_t* cbase, int32_t* ids_out,
                            int32_t* pay_out, hipStream_t s);
// The dense update of an fp32 model in further blocks of that launch (of the one over the windows): n parameters, K rows of gradients.
struct DenseJob {
  float* p;
  float* state;
  const float* grads;              // [K, stride]
  int64_t stride, n;               // n = 0: none
  float lr, eps;
  int32_t K;
  float w[ANTDT_MAX_SHARDS];
};
hipError_t launch_seg_reduce(const SegArgs& a, const FieldPtr& fp, const TileBase& tb, const ShardTab& tab, const DenseJob& dense, Profiler* prof,
                             hipStream_t s);

// ---------------------------------------------------------------- optim.hip
struct DenseAggArgs {
  const float* grads;  // [K, stride] per-shard flat gradients
  float* g;            // [P]
  int64_t P, stride;
};
hipError_t launch_dense_agg(const DenseAggArgs& a, const ShardTab& tab, hipStream_t s);

// Dense Adagrad on the flat MLP parameters with the gradient aggregated on the fly
// (g = sum_k w_k grads[k]).  Hidden-layer weight matrices of bf16 models are walked in 64x64 tiles
// and their bf16 operand copies refreshed in the same pass; everything else (biases, the last
// layer, fp32 models) goes through plain ranges.
struct DenseAdagradArgs {
  float* p;
  float* state;
  const float* grads;  // [K, stride]
  int64_t stride;
  float lr, eps;
  int32_t n_mat;
  int64_t w_off[ANTDT_MAX_LAYERS];
  int32_t rows[ANTDT_MAX_LAYERS], cols[ANTDT_MAX_LAYERS];
  bf16_t* wb[ANTDT_MAX_LAYERS];
  int32_t tile_base[ANTDT_MAX_LAYERS + 1];
  int32_t n_rng;
  int64_t rng_off[ANTDT_MAX_LAYERS + 1], rng_len[ANTDT_MAX_LAYERS + 1];
  int32_t rng_block[ANTDT_MAX_LAYERS + 2];  // first block of each range, relative to the first range block
};
hipError_t launch_dense_adagrad(const DenseAdagradArgs& a, const ShardTab& tab, hipStream_t s);

struct AdamArgs {
  float* p;
  float* m;
  float* v;
  const float* g[16];
  float w[16];
  int32_t K;
  int64_t n;
  float lr, b1, b2, c1, c2, eps, inv_bc1, inv_bc2;  // c = 1 - b, formed in double on the host
};
hipError_t launch_adam(const AdamArgs& a, hipStream_t s);
hipError_t launch_stream_copy(float* dst, const float* src, int64_t n, hipStream_t s);

}  // namespace antdt
