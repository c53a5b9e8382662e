// Block-level bf16 matrix product on the gfx950 matrix cores, shared by the MLP kernels.
//
//   acc[i][j] += sum_{k in [ks, ke)} A(m, k) * B(n, k)      (v_mfma_f32_32x32x16_bf16, fp32 accumulation)
//
// An operand is stored in one of two ways:
//   contiguous  K runs fastest:        X(r, k) = x[r * ld + k]   (activations in the forward product, ...)
//   strided     the other index does:  X(r, k) = x[k * ld + r]   (weights W[in, out] in the forward product,
//                                       activations and gradients [sample, width] in the weight gradient)
// so that no operand needs a transposed copy in memory: a strided operand's tile goes to LDS as it
// lies in memory, and `ds_read_b64_tr_b16` hands its columns to the lanes.
//
// Tiles move from memory straight to LDS (global_load_lds, 16 bytes per lane, no registers), S stages
// deep: while stage t is multiplied, stages t+1 .. t+S-1 are in flight; one barrier per stage.  LDS rows
// are unpadded (the load writes 64 consecutive 16-byte slots per wavefront); the slots of a row are
// permuted instead, on the side of the memory address, so that every fragment read touches each
// bank once.
#pragma once

#include <type_traits>

#include "common.h"

namespace antdt {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

// 16 zero bytes: where a lane's 16-byte piece lies past the end of the contraction it is read from here.
static __device__ __attribute__((aligned(16))) uint32_t mfma_zero16[4];

// One 16-byte piece per lane from memory to LDS slot `lds + 16 * lane` (`lds` is wavefront-uniform).
__device__ __forceinline__ void load_lds16(const void* src, uint32_t lds) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"{m0}"(lds), "v"(src) : "memory");
}
__device__ __forceinline__ void load_lds16(const void* base, uint64_t off, uint32_t lds) {
  load_lds16(reinterpret_cast<const char*>(base) + off, lds);
}
// The same from base + off (base wavefront-uniform).
__device__ __forceinline__ void load_lds16(const void* base, uint32_t off, uint32_t lds) {
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"{m0}"(lds), "v"(off), "s"(base) : "memory");
}
template <int N> __device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void block_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
}

// BR rows (m or n) x BK contraction slots of one operand.
template <int BR, int BK, bool STRIDED>
struct OperandTile {
  static constexpr int BYTES = BR * BK * 2;
  static constexpr int PITCH = (STRIDED ? BR : BK) / 8;   // 16-byte slots per LDS row
  static constexpr int SLOTS = BR * BK / 8;

  // Where piece c of LDS row r sits.  Contiguous operands are read down a column of pieces (16 rows at a
  // time), strided ones four rows by four neighbouring pieces: either way 16 slots that have to differ
  // modulo 16 (256 bytes, all banks).
  static __device__ __forceinline__ int swizzle(int r) {
    if (!STRIDED) return PITCH >= 16 ? (r & 15) : ((r >> 1) & 7);
    return PITCH >= 16 ? ((r & 3) << 2) : PITCH == 8 ? (((r >> 1) & 1) << 2) : 0;
  }

  // Byte offset, inside the tile, of what this lane reads for the fragment of 32 rows starting at a
  // multiple of 32 and contraction step kk = 0; `half`: the second four contraction slots of a strided
  // operand.  Fragments of other rows and steps are at constant distances except for the permutation,
  // which depends on the step only for contiguous operands.
  static __device__ __forceinline__ bf16x8 fragment(const char* tile, int r0, int kk, int lane) {
    if (!STRIDED) {
      const int r = r0 + (lane & 31);
      const int c = (kk >> 3) + (lane >> 5);
      return *reinterpret_cast<const bf16x8*>(tile + (r * PITCH + (c ^ swizzle(r))) * 16);
    } else {
      // a group of 16 lanes reads a block of four contraction slots x 16 rows; lane j of the group supplies
      // the address of slot j / 4, rows 4 (j % 4) .. + 3 and receives row j of the block
      typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
      const int j = lane & 15, k = kk + (lane >> 5) * 8 + (j >> 2);
      const int c = (r0 >> 3) + ((lane >> 4) & 1) * 2 + ((j & 3) >> 1);
      const char* p = tile + (k * PITCH + (c ^ swizzle(k))) * 16 + (j & 1) * 8;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * PITCH * 16));
      union {
        s16x4 s[2];
        bf16x8 v;
      } u;
      u.s[0] = lo;
      u.s[1] = hi;
      return u.v;
    }
  }
};

// The tiles of one block: WR x WC wavefronts of TM x TN MFMA tiles each.  Every shape adds up the products in the
// same order, so that a sample's results do not depend on how many samples are computed with it.
// FAR: pieces of a tile may lie 4 GiB or more from its origin (operands wider than 2^31 / rows of the tile).
// WAVES: wavefronts of the block; those behind the first WR x WC only request pieces (one wavefront gets a load away every 64 cycles or
// so, so a tile of one wavefront alone waits for its own requests).
template <int TM, int TN, int WR, int WC, int BK, int STAGES, bool A_STRIDED, bool B_STRIDED, bool FAR = false, int WAVES = WR * WC>
struct BlockProduct {
  typedef typename std::conditional<FAR, uint64_t, uint32_t>::type Offset;
  static constexpr int THREADS = 64 * WAVES;
  static constexpr int BM = 32 * TM * WR, BN = 32 * TN * WC;
  typedef OperandTile<BM, BK, A_STRIDED> TA;
  typedef OperandTile<BN, BK, B_STRIDED> TB;
  static constexpr int STAGE_BYTES = TA::BYTES + TB::BYTES;
  static constexpr int LDS_BYTES = STAGES * STAGE_BYTES;
  static constexpr int VA = TA::SLOTS / THREADS, VB = TB::SLOTS / THREADS;  // pieces per thread and stage
  static_assert(VA * THREADS == TA::SLOTS && VB * THREADS == TB::SLOTS, "tile / thread count");
  static_assert(BK % 16 == 0, "contraction slots per stage");

  // Rows of the operands that exist: indices are clamped to them (a clamped row's products are never stored).
  // ks, ke: multiples of 8 unless both operands are strided.
  static __device__ __forceinline__ void run(const bf16_t* A, const bf16_t* B, int64_t lda, int64_t ldb, int rows_a,
                                             int rows_b, int m0, int n0, int ks, int ke, char* lds,
                                             f32x16 (&acc)[TM][TN]) {
    f32x16 none[TN];
    run<false>(A, B, lda, ldb, rows_a, rows_b, m0, n0, ks, ke, lds, acc, none, false);
  }
  // ONES: where `ones` (wavefront-uniform) is set, sum_b[j] additionally receives the products of B's rows with
  // a row of ones, i.e. sum_k B(n, k): the bias gradient next to a weight gradient.
  template <bool ONES>
  static __device__ __forceinline__ void run(const bf16_t* A, const bf16_t* B, int64_t lda, int64_t ldb, int rows_a,
                                             int rows_b, int m0, int n0, int ks, int ke, char* lds,
                                             f32x16 (&acc)[TM][TN], f32x16 (&sum_b)[TN], bool ones) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = wave % (WR * WC) / WC, wc = wave % WC;   // (the modulo says that a single wavefront is number 0)
    const uint32_t lds0 = lds_address(lds) + wave * 1024;
    // Byte offsets of this thread's pieces from the tile's origin, the same for every stage; the origin
    // moves along the contraction (scalar arithmetic only).
    Offset oa[VA], ob[VB];
    int ka[VA], kb[VB];   // contraction slot (relative to the stage) of each piece
#pragma unroll
    for (int i = 0; i < VA; ++i) piece<TA, A_STRIDED>(tid + i * THREADS, lda, rows_a, m0, oa[i], ka[i]);
#pragma unroll
    for (int i = 0; i < VB; ++i) piece<TB, B_STRIDED>(tid + i * THREADS, ldb, rows_b, n0, ob[i], kb[i]);
    const char* pa = reinterpret_cast<const char*>(A_STRIDED ? A + (int64_t)ks * lda + m0 : A + (int64_t)m0 * lda + ks);
    const char* pb = reinterpret_cast<const char*>(B_STRIDED ? B + (int64_t)ks * ldb + n0 : B + (int64_t)n0 * ldb + ks);
    const int64_t step_a = (A_STRIDED ? lda * BK : BK) * 2, step_b = (B_STRIDED ? ldb * BK : BK) * 2;
    const int len = ke - ks;
    const int nk = len > 0 ? (len + BK - 1) / BK : 0;

    int left = len;                // contraction slots not requested yet
    uint32_t fill = lds0;          // buffer of the next stage to request
    auto issue = [&]() {
      if (left >= BK) {
#pragma unroll
        for (int i = 0; i < VA; ++i) load_lds16(pa, oa[i], fill + i * (THREADS * 16));
#pragma unroll
        for (int i = 0; i < VB; ++i) load_lds16(pb, ob[i], fill + TA::BYTES + i * (THREADS * 16));
      } else {                     // last, partly filled stage: zeros past the end
        const char* zero = reinterpret_cast<const char*>(mfma_zero16);
#pragma unroll
        for (int i = 0; i < VA; ++i) load_lds16(ka[i] < left ? pa + oa[i] : zero, fill + i * (THREADS * 16));
#pragma unroll
        for (int i = 0; i < VB; ++i) load_lds16(kb[i] < left ? pb + ob[i] : zero, fill + TA::BYTES + i * (THREADS * 16));
      }
      pa += step_a;
      pb += step_b;
      left -= BK;
      fill = fill == lds0 + (STAGES - 1) * STAGE_BYTES ? lds0 : fill + STAGE_BYTES;
    };
    constexpr int PER_STAGE = VA + VB;
#pragma unroll
    for (int t = 0; t < STAGES - 1; ++t)
      if (t < nk) issue();
    uint32_t read = 0;             // buffer of stage t
    for (int t = 0; t < nk; ++t) {
      // this wavefront's pieces of stage t have arrived when only those of the later stages are outstanding
      if (t + STAGES - 2 < nk) wait_loads<(STAGES - 2) * PER_STAGE>();
      else wait_loads<0>();
      block_barrier();          // ... and so have everyone's; stage t-1 has been read by everyone
      if (WAVES > WR * WC && wave >= WR * WC) {
        if (left > 0) issue();
        continue;
      }
      // The fragments of the next contraction step are requested before the current one is multiplied, and
      // the next stage behind the first multiplications: with one or two wavefronts per SIMD nothing else
      // would hide those instructions.
      const char* la = lds + read;
      const char* lb = la + TA::BYTES;
      constexpr int Q = BK / 16;
      bf16x8 af[2][TM], bf[2][TN];
      auto fetch = [&](int q, bf16x8 (&a)[TM], bf16x8 (&b)[TN]) {
        const int kk = q * 16;
#pragma unroll
        for (int i = 0; i < TM; ++i) a[i] = TA::fragment(la, (wr * TM + i) * 32, kk, lane);
#pragma unroll
        for (int j = 0; j < TN; ++j) b[j] = TB::fragment(lb, (wc * TN + j) * 32, kk, lane);
      };
      fetch(0, af[0], bf[0]);
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        if (q + 1 < Q) fetch(q + 1, af[(q + 1) & 1], bf[(q + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        // operands swapped: lane (lane & 31) of the result holds one row m, its 16 elements are the columns
        // 8 (e / 4) + 4 (lane / 32) + e % 4 of a 32-column tile
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[q & 1][j], af[q & 1][i], acc[i][j], 0, 0, 0);
        if (ONES && ones) {
          const __bf16 one = (__bf16)1.0f;
          const bf16x8 row = {one, one, one, one, one, one, one, one};
#pragma unroll
          for (int j = 0; j < TN; ++j)
            sum_b[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[q & 1][j], row, sum_b[j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (q == 0 && left > 0) issue();
      }
      read = read == (STAGES - 1) * STAGE_BYTES ? 0 : read + STAGE_BYTES;
    }
    block_barrier();   // the buffers are free
  }

 private:
  // Piece `slot` of an operand's tile whose first row is r0: its offset from the tile's origin and its
  // contraction slot.
  template <typename T, bool STRIDED>
  static __device__ __forceinline__ void piece(int slot, int64_t ld, int rows, int r0, Offset& off, int& k) {
    const int r = slot / T::PITCH, c = (slot % T::PITCH) ^ T::swizzle(r);
    if (!STRIDED) {
      k = c * 8;
      off = (Offset)(min(r, rows - 1 - r0) * ld + k) * 2;
    } else {   // (the row length is a multiple of 8, so the last whole piece of a row is in bounds)
      k = r;
      off = (Offset)(r * ld + min(c * 8, ((rows - 1) & ~7) - r0)) * 2;
    }
  }
};

}  // namespace antdt
