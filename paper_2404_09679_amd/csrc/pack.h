// How the lookups of a shard's field are dealt to the threads that pack them (see mask_pack_kernel).  Plain C++, so that the host
// can walk it too.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define PACK_FUNCTION __host__ __device__ __forceinline__
#else
#define PACK_FUNCTION inline
#endif

namespace antdt {

constexpr int PACK_THREADS = 256, PACK_BLOCKS = 8, PACK_ITEMS = 4, PACK_LOOKUPS = PACK_THREADS * PACK_ITEMS;

// Every round of a thread among the `n` lookups: body(i), for the lookups i, i + PACK_THREADS, ... PACK_ITEMS of them (those
// below n).  A field may hold almost 2^31 lookups and a step is 8192: the index passes 2^31 behind the last round.
template <typename Body> PACK_FUNCTION void pack_rounds(int block, int thread, int64_t n, Body body) {
  for (int64_t i = (int64_t)block * PACK_LOOKUPS + thread; i < n; i += PACK_BLOCKS * PACK_LOOKUPS) body(i);
}

}  // namespace antdt
