// Server-side coalescing of the pushed sparse gradients (Section II: the servers combine
// the gradients of all workers): per field, a stable sort of (row id, sample index) pairs
// (LSD radix, of large batches by ranges of rows), detection of the runs of equal ids
// (unique ids + segment offsets), and the weighted segmented reduction
//   G[u, :] = sum over the run of w(sample) * dX[sample, field slice].
// No floating-point atomics are used, so the sums are bitwise repeatable.  The reduction can
// apply the row-sparse Adagrad step of each row at once (the parameter update of Section II).
#include <algorithm>
#include <type_traits>

#include "dense.h"
#include "pack.h"
#include "sort.h"

namespace antdt {
namespace {

constexpr int SORT_THREADS = 512;
constexpr int SORT_WAVES = SORT_THREADS / 64;
constexpr int SORT_TILE = ANTDT_SORT_TILE;            // keys per block
constexpr int SORT_ITEMS = SORT_TILE / SORT_THREADS;

// Blocks of a launch of one block per tile (see tile_of_block).
__host__ __device__ inline unsigned tile_grid(int total_tiles) { return 8u * ((total_tiles + 7) / 8); }

// Tile T of all fields' tiles -> (field, tile of the field): how many fields end at or before it, counted by the
// lanes of the wavefront (one load of the table instead of a chain of them).
__device__ __forceinline__ void field_of_tile(const TileBase& tb, int T, int& f, int& t) {
  const int lane = threadIdx.x & 63;
  static_assert(ANTDT_MAX_FIELDS == 128, "two table entries per lane");
  const int t0 = tb.t[1 + lane], t1 = tb.t[65 + lane];
  f = __builtin_amdgcn_readfirstlane(__popcll(__ballot(t0 <= T)) + __popcll(__ballot(t1 <= T)));
  t = T - tb.t[f];
}

// Block -> (field, tile, part of the tile) for the kernels that walk the lookups of the fields tile by tile,
// `parts` blocks per tile.  The hardware hands block i to XCD i mod 8, and every XCD has an L2 of its own: the
// blocks whose index is x modulo 8 take the x-th eighth of all tiles, so that every pass over a field's lookups
// runs on one XCD (two where a field crosses an eighth).  The scattered 4-byte stores of a sort pass are then
// assembled into full lines in that L2 (spread over eight L2s, each wrote its partial lines back: 3.7 times
// the payload), and the next pass over the field finds them there; so does the reduction with the field's
// slice of the pooled gradients.
__device__ __forceinline__ bool tile_of_block(const TileBase& tb, int F, int parts, int& f, int& t, int& part) {
  const int total = tb.t[F], share = (total + 7) >> 3;
  const int slot = (int)(blockIdx.x >> 3) / parts;
  const int T = (int)(blockIdx.x & 7) * share + slot;
  if (slot >= share || T >= total) return false;
  part = (int)(blockIdx.x >> 3) % parts;
  field_of_tile(tb, T, f, t);
  return true;
}

// ----------------------------------------------------------------- sort
// The sort by buckets (see sort_buckets_kernel): a field's rows are cut into ranges of about as many lookups each, one pass over many
// blocks puts the lookups into them, and a block each sorts them in LDS.
constexpr int BUCKET_THREADS = 512, BUCKET_WAVES = BUCKET_THREADS / 64, BUCKET_ITEMS = 16, BUCKET_KEYS = BUCKET_THREADS * BUCKET_ITEMS;
constexpr int BUCKET_BITS = 8;                     // of a pass inside a bucket, at most; a bucket has up to 2^16 rows
constexpr int MAX_BUCKETS = 256, BUCKET_CELLS = 256;
struct FieldBuckets {
  int32_t first[MAX_BUCKETS + 4];                  // first row of each bucket (one without rows: the number of rows)
  uint16_t cell[BUCKET_CELLS];                     // buckets of the first and the last row (high half) of an equal part of the rows
};
struct BucketPlan {
  int32_t rb;           // log2 of the number of buckets of a field
  int32_t range_bits;   // log2 of the most rows of a bucket; range_bits + sample_bits <= 32
  int32_t sample_bits;
  int32_t cell_bits;    // log2 of the rows of a cell
  int32_t last_row;
  const int32_t* offsets;   // [F][B + 1] where the samples of the lookups are to be worked out from these, or NULL
  int32_t B;
  FieldBuckets* fields;
  int32_t* large;       // [0]: number of buckets of more than BUCKET_KEYS lookups and one row, then those (field, bucket)
  int32_t most_large;   // no more of them
  // (ids that are no rows go where the update takes them to be: the first row, the last one)
  __device__ __forceinline__ int32_t in_range(int32_t key) const { return min(max(key, 0), last_row); }
  __device__ __forceinline__ uint32_t bucket(const FieldBuckets& fb, int32_t key) const {
    const uint32_t c = fb.cell[key >> cell_bits];
    uint32_t lo = c & 0xFF, hi = c >> 8;
    while (lo < hi) {
      const uint32_t mid = (lo + hi + 1) >> 1;
      if (fb.first[mid] <= key) lo = mid;
      else hi = mid - 1;
    }
    return lo;
  }
};
// Samples of 256 neighbouring lookups of a field, from position p0 (one of the field's) on, by a wavefront: lane l receives those of
// p0 + 64 i + l (past the field's end: any).  off: the field's bag boundaries, off[0] = 0, off[B] its lookups; mark: 256 words of LDS.
__device__ __forceinline__ void samples_of(const int32_t* off, int B, int p0, uint32_t* mark, int32_t (&sample)[4]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < 4; ++i) mark[i * 64 + lane] = 0;
  int lo = 0, hi = B;   // the bag of p0: off[lo] <= p0 < off[hi]
  while (hi - lo > 1) {
    const int step = (hi - lo + 64) / 65, at = lo + (lane + 1) * step;
    const int below = __popcll(__ballot(at < hi && off[min(at, hi)] <= p0));
    hi = min(hi, lo + (below + 1) * step);
    lo += below * step;
  }
  wave_lds_order();
  for (int s = lo + 1; s < B; s += 64) {   // bags that begin among the lookups behind p0, empty ones too
    const int begin = off[min(s + lane, B)] - p0;
    if (s + lane < B && begin > 0 && begin < 256) atomicAdd(&mark[begin], 1u);
    if (__ballot(begin >= 256)) break;
  }
  wave_lds_order();
  uint32_t bags = (uint32_t)lo;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t upto = bags + wave_prefix(mark[i * 64 + lane]);
    sample[i] = (int32_t)upto;
    bags = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
  }
  wave_lds_order();
}

template <int THREADS>
__device__ __forceinline__ void load_buckets(FieldBuckets& to, const FieldBuckets& from) {
  constexpr int WORDS = sizeof(FieldBuckets) / 4;
  for (int i = threadIdx.x; i < WORDS; i += THREADS) reinterpret_cast<uint32_t*>(&to)[i] = reinterpret_cast<const uint32_t*>(&from)[i];
}

// The threads' values (x: a word each) in ascending order, by the first N threads; steps within a wavefront need no memory.
template <int N>
__device__ __forceinline__ int32_t bitonic_sort(int32_t v, int32_t* x) {
  const int i = threadIdx.x;
#pragma unroll
  for (int k = 2; k <= N; k <<= 1)
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) {
      int32_t o;
      if (j >= 64) {
        if (i < N) x[i] = v;
        __syncthreads();
        o = i < N ? x[i ^ j] : v;
        __syncthreads();
      } else {
        o = __shfl_xor(v, j, 64);
      }
      v = ((i & j) == 0) == ((i & k) == 0) ? min(v, o) : max(v, o);
    }
  if (i < N) x[i] = v;
  __syncthreads();
  return v;
}
// Sum of the values of the threads before this one (wsum: a word per wavefront), and of all.
__device__ __forceinline__ uint32_t block_prefix(uint32_t x, uint32_t* wsum, int waves, uint32_t& all, bool again = true) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t incl = wave_prefix(x);
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  uint32_t before = 0;
  all = 0;
  for (int q = 0; q < waves; ++q) {
    const uint32_t c = wsum[q];
    before += q < w ? c : 0;
    all += c;
  }
  if (again) __syncthreads();   // (another one may follow)
  return before + incl - x;
}

// Cuts a field's rows into buckets, by SAMPLE_KEYS of its lookups: a row that seems to have half of BUCKET_KEYS lookups or more is a bucket by
// itself (they are in order once they are together), the others are cut where equal shares of their lookups end, and every 2^range_bits rows.
// (Which cuts are made changes no result.)
// The sample: a lookup of each of SAMPLE_KEYS equal stretches, at a place that looks random.  At even distances all of them would be at one place of
// their bags where bags have one length and their number is a multiple of SAMPLE_KEYS, and see few of the rows if ids have an order in a bag
// (16384 bags of 50 ascending ids of 50000 rows: 730000 of a field's 819200 lookups in one range, now 12000; the scatter and the ranges' sort
// of three such fields 3128 us, in random order 65; a step now 219, in random order 231).
constexpr int SAMPLE_KEYS = 1024, HOT_KEYS = 4;
__device__ __forceinline__ int64_t sampled_lookup(int64_t n, int f, int i) {
  uint32_t h = (uint32_t)(f * SAMPLE_KEYS + i + 1);   // (MurmurHash3's finaliser)
  h = (h ^ (h >> 16)) * 0x85EBCA6Bu;
  h = (h ^ (h >> 13)) * 0xC2B2AE35u;
  h ^= h >> 16;
  const int64_t first = n * i / SAMPLE_KEYS, end = n * (i + 1) / SAMPLE_KEYS;
  return first + (int64_t)(((uint64_t)h * (uint64_t)(end - first)) >> 32);   // (first where the stretch is empty: below n)
}
__global__ __launch_bounds__(SAMPLE_KEYS) void sort_cuts_kernel(const int32_t* keys, FieldPtr fp, BucketPlan bp) {
  __shared__ int32_t key[SAMPLE_KEYS], cut[SAMPLE_KEYS];
  __shared__ uint8_t hot[SAMPLE_KEYS];
  __shared__ uint32_t wsum[SAMPLE_KEYS / 64];
  __shared__ FieldBuckets fb;
  const int f = blockIdx.x, i = threadIdx.x;
  if (f == 0 && i == 0) bp.large[0] = 0;
  const int64_t n = fp.p[f + 1] - fp.p[f];
  if (n == 0) return;
  const int32_t k = bitonic_sort<SAMPLE_KEYS>(bp.in_range(keys[fp.p[f] + sampled_lookup(n, f, i)]), key);
  auto bound = [&](int32_t v) {   // sampled keys below v
    int lo = 0, hi = SAMPLE_KEYS;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (key[mid] < v) lo = mid + 1;
      else hi = mid;
    }
    return lo;
  };
  const int head = bound(k), many = 1 << bp.rb, fixed = (bp.last_row >> bp.range_bits) + 1;
  uint32_t all, hots;
  const int hot_keys = min((int)((int64_t)SAMPLE_KEYS * (BUCKET_KEYS / 2) / n) + HOT_KEYS, SAMPLE_KEYS);
  const bool is_hot = head == i && i + hot_keys <= SAMPLE_KEYS && key[i + hot_keys - 1] == k;
  const uint32_t hot_place = block_prefix(is_hot, wsum, SAMPLE_KEYS / 64, hots);
  const uint32_t most_hot = (uint32_t)(many - fixed) / 4;
  hot[i] = is_hot && hot_place < most_hot;
  hots = min(hots, most_hot);
  __syncthreads();
  const bool cold = !hot[head];
  const uint32_t cold_place = block_prefix(cold, wsum, SAMPLE_KEYS / 64, all);
  const int cuts = many - fixed - 2 * (int)hots;                 // (at least half of those that are not fixed)
  const int step = max(((int)all + cuts - 1) / cuts, 1);
  cut[i] = 0x7FFFFFFF;
  __syncthreads();
  const bool quantile = cold && cold_place % (uint32_t)step == 0;
  if (i < fixed) cut[i] = i << bp.range_bits;
  if (hot[i]) {
    cut[fixed + 2 * (int)hot_place] = k;
    cut[fixed + 2 * (int)hot_place + 1] = k + 1;
  }
  if (quantile) cut[fixed + 2 * (int)hots + (int)(cold_place / (uint32_t)step)] = k;
  __syncthreads();
  bitonic_sort<MAX_BUCKETS>(i < MAX_BUCKETS ? cut[i] : 0, cut);   // (no more than `many` of them)
  const int rows = bp.last_row + 1;
  const bool first = i < many && cut[i] < rows && (i == 0 || cut[i] != cut[i - 1]);
  const uint32_t place = block_prefix(first, wsum, SAMPLE_KEYS / 64, all);
  if (i < MAX_BUCKETS + 4) fb.first[i] = rows;
  __syncthreads();
  if (first) fb.first[place] = cut[i];
  __syncthreads();
  auto last_at = [&](int32_t row) {   // the bucket of a row
    int lo = 0, hi = (int)all - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (fb.first[mid] <= row) lo = mid;
      else hi = mid - 1;
    }
    return lo;
  };
  if (i < BUCKET_CELLS) {
    const int64_t r0 = (int64_t)i << bp.cell_bits, r1 = r0 + (1 << bp.cell_bits) - 1;
    fb.cell[i] = (uint16_t)(last_at((int32_t)min(r0, (int64_t)bp.last_row)) | last_at((int32_t)min(r1, (int64_t)bp.last_row)) << 8);
  }
  __syncthreads();
  load_buckets<SAMPLE_KEYS>(bp.fields[f], fb);
}

// Histogram layout: hist[(tile_base[f] + tile) << rb | digit] (digits of a tile contiguous);
// digit_total[f << rb | digit] = number of the field's keys with the digit.

// Digit histogram of one tile.  Hot rows make many lanes count one digit, and LDS adds to one address go one after
// the other: every digit has copies of its counter, and the lanes take turns with them (42 M lookups of 21 bits: 60 / 102 / 121
// us a pass with one counter, the keys more and more in order; 54 with eight, the blocks' loads and their latency).
// BUCKETS: their numbers are the digits.
template <bool BUCKETS>
__global__ __launch_bounds__(SORT_THREADS) void sort_hist_kernel(const int32_t* keys, uint32_t* hist,
                                                                 FieldPtr fp, TileBase tb, int F, int shift, int rb, BucketPlan bp) {
  constexpr int LOG_COUNTERS = 12, LOG_COPIES = 3;
  __shared__ uint32_t h[1 << LOG_COUNTERS];
  __shared__ typename std::conditional<BUCKETS, FieldBuckets, int>::type fb;
  int f, t, part;
  if (!tile_of_block(tb, F, 1, f, t, part)) return;
  const int nb = 1 << rb;
  const int cb = min(LOG_COPIES, LOG_COUNTERS - rb);   // log2 of the copies
  const int64_t base = fp.p[f];
  const int count = min((int)(fp.p[f + 1] - base) - t * SORT_TILE, SORT_TILE);
  const int32_t* in = keys + base + (int64_t)t * SORT_TILE;
  int32_t k[SORT_ITEMS];
#pragma unroll
  for (int i = 0; i < SORT_ITEMS; ++i) k[i] = in[min(i * SORT_THREADS + (int)threadIdx.x, count - 1)];   // (all loads first)
  for (int d = threadIdx.x; d < nb << cb; d += SORT_THREADS) h[d] = 0;
  if constexpr (BUCKETS) load_buckets<SORT_THREADS>(fb, bp.fields[f]);
  __syncthreads();
  const int copy = threadIdx.x & ((1 << cb) - 1);
#pragma unroll
  for (int i = 0; i < SORT_ITEMS; ++i)
    if (i * SORT_THREADS + (int)threadIdx.x < count) {
      uint32_t d;
      if constexpr (BUCKETS) {
        d = bp.bucket(fb, bp.in_range(k[i]));
      } else {
        d = ((uint32_t)k[i] >> shift) & (nb - 1);
      }
      atomicAdd(&h[(d << cb) + copy], 1u);
    }
  __syncthreads();
  uint32_t* out = hist + ((int64_t)(tb.t[f] + t) << rb);
  for (int d = threadIdx.x; d < nb; d += SORT_THREADS) {
    uint32_t sum = 0;
    for (int c = 0; c < 1 << cb; ++c) sum += h[(d << cb) + ((c + d) & ((1 << cb) - 1))];   // (turned: neighbours read different banks)
    out[d] = sum;
  }
}

// The counts of a digit are replaced by their exclusive prefix over the tiles, and their total goes to digit_total.  A block has up to
// SCAN_DIGITS digits of a field; a thread has a digit and one stretch of the tiles, which it walks twice (their sum; their
// prefixes).  Bound by the chain of loads, and by what one compute unit can fetch (the counts were written by other XCDs): one
// block per field, a chain of loads for each digit, took 18.8 us for 204 tiles of 128 digits, now 11.6, and 11 for 80 of
// 1024, now 7.5.
constexpr int SCAN_THREADS = 1024, SCAN_DIGITS = 128;
template <bool BUCKETS>
__global__ __launch_bounds__(SCAN_THREADS) void sort_scan_kernel(uint32_t* hist, uint32_t* digit_total, TileBase tb, int rb, BucketPlan bp) {
  __shared__ uint32_t sums[SCAN_THREADS];
  const int nb = 1 << rb, digits = min(nb, SCAN_DIGITS), groups = nb / digits;
  const int f = (int)blockIdx.x / groups;
  const int tiles = tb.t[f + 1] - tb.t[f];
  const int parts = SCAN_THREADS / digits, dl = threadIdx.x & (digits - 1), part = threadIdx.x / digits;
  const int d = ((int)blockIdx.x - f * groups) * digits + dl;
  const int t0 = tiles * part / parts, t1 = tiles * (part + 1) / parts;
  uint32_t* h = hist + ((int64_t)tb.t[f] << rb) + d;
  auto walk = [&](uint32_t run, bool store) {
    for (int t = t0; t < t1; t += 4) {
      uint32_t c[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) c[q] = h[(int64_t)min(t + q, t1 - 1) << rb];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (t + q < t1) {
          if (store) h[(int64_t)(t + q) << rb] = run;
          run += c[q];
        }
    }
    return run;
  };
  sums[threadIdx.x] = walk(0, false);
  __syncthreads();
  uint32_t run = 0, total = 0;
  for (int q = 0; q < parts; ++q) {
    const uint32_t c = sums[q * digits + dl];
    if (q < part) run += c;
    total += c;
  }
  walk(run, true);
  if (part == 0) {
    digit_total[((int64_t)f << rb) + d] = total;
    if (BUCKETS && total > (uint32_t)BUCKET_KEYS && bp.fields[f].first[d + 1] - bp.fields[f].first[d] > 1) {
      const int at = atomicAdd(bp.large, 1);
      if (at < bp.most_large) bp.large[1 + at] = f << 16 | d;   // (in any order: each is a block's work)
    }
  }
}

// Stable scatter of one tile.  Wave w owns the contiguous slice w of the tile and walks it in
// rounds of 64 keys; lanes holding equal digits find each other with one
// ballot per digit bit, the per-wave running count of the digit lives in LDS.
// Bound by memory where fields are large (42 M keys in 7-bit digits: 678 MB of compulsory traffic in 134 us, a copy's rate), by
// vector instructions else (75 an item, a third of them the ballots).  Us a pass, with counters in flat accesses, 32 bits wide,
// and prefixes by LDS exchange / now: 42 M keys 172 / 134, 4.3 M in 10-bit digits 29.7 / 26, 1.1 M 13.1 / 11.3.
// FULL: all the tile's keys exist.  BUCKETS: place inside the bucket's rows and sample leave as one word (packed), or, of a bucket of one row,
// key and sample.
constexpr int DPT = MAX_BINS / SORT_THREADS;   // digits per thread: threadIdx.x + q SORT_THREADS
struct ScatterLds {
  union {
    uint16_t cnt[SORT_WAVES][MAX_BINS];   // (a tile's counts fit 16 bits)
    int32_t staged[2][SORT_TILE];         // then: the tile sorted by digit (keys, samples)
  };
  uint32_t gbase[MAX_BINS];
  uint16_t dpre[MAX_BINS];
  uint32_t wsum[2][DPT][SORT_WAVES];
};
template <bool FULL, bool BUCKETS, typename Buckets>
__device__ __forceinline__ void scatter_tile(ScatterLds& lds, const int32_t* keys_in, const int32_t* pay_in, int32_t* keys_out, int32_t* pay_out,
                                             int32_t* packed, const uint32_t* hb, const uint32_t* totals, int count, int nnz, int shift, int rb,
                                             const BucketPlan& bp, Buckets& fb, const FieldBuckets* table,
                                             int f, int tile0) {
  constexpr int ITEMS = SORT_ITEMS;
  const int nb = 1 << rb;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int first = w * (64 * ITEMS) + lane;   // item i: position first + 64 i of the tile
  // The first position of a digit's keys of this tile in the output: digits before it in the field, and the digit's keys in
  // earlier tiles.  Loaded up front with coalesced loads, looked up in LDS.
  uint32_t earlier[DPT], total[DPT];
#pragma unroll
  for (int q = 0; q < DPT; ++q) {
    const int d = (int)threadIdx.x + q * SORT_THREADS;
    earlier[q] = hb[min(d, nb - 1)];
    total[q] = totals[min(d, nb - 1)];
  }
  int32_t key[ITEMS], pay[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {  // all loads first (clamped), so that they overlap
    const int pos = FULL ? first + i * 64 : min(first + i * 64, count - 1);
    key[i] = keys_in[pos];
    if (!BUCKETS || !bp.offsets) pay[i] = pay_in[pos];
  }
  if constexpr (BUCKETS) load_buckets<SORT_THREADS>(fb, *table);
  if constexpr (BUCKETS) {
    static_assert(ITEMS == 4 && sizeof(lds.cnt[0]) >= 256 * 4, "lookups of a wavefront");
    if (bp.offsets && w * (64 * ITEMS) < count)
      samples_of(bp.offsets + (int64_t)f * (bp.B + 1), bp.B, tile0 + w * (64 * ITEMS), reinterpret_cast<uint32_t*>(lds.cnt[w]), pay);
  }
  for (int d = lane; d < nb; d += 64) lds.cnt[w][d] = 0;   // (each wavefront its own row)
  wave_lds_order();
  if (BUCKETS) __syncthreads();
  const uint64_t lt = lanemask_lt();
  uint32_t rank[ITEMS];
  uint32_t digits[ITEMS];
  auto digit = [&](int32_t k) { return ((uint32_t)k >> shift) & (uint32_t)(nb - 1); };
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    if (BUCKETS) key[i] = bp.in_range(key[i]);
    if constexpr (BUCKETS) digits[i] = bp.bucket(fb, key[i]);
    else digits[i] = digit(key[i]);
  }
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const bool valid = FULL || first + i * 64 < count;
    const uint32_t d = digits[i];
    const uint64_t m = same_digit(d, rb, valid);
    const uint32_t prior = lds.cnt[w][d];
    wave_lds_order();
    rank[i] = prior + (uint32_t)__popcll(m & lt);
    if (valid && (m & lt) == 0) lds.cnt[w][d] = (uint16_t)(prior + (uint32_t)__popcll(m));  // lowest lane of the group
    wave_lds_order();
  }
  __syncthreads();
  // Per digit: the counts of the wavefronts become exclusive prefixes (keys of the digit in
  // earlier wavefronts of the tile), their sum the tile's count of the digit; an exclusive scan of
  // these counts in digit order gives every key its place in the tile sorted by digit, one of the totals of the
  // field the place of the digit in the field.
  uint32_t tot[DPT], incl[DPT], incl_total[DPT];
#pragma unroll
  for (int q = 0; q < DPT; ++q) {
    tot[q] = incl[q] = incl_total[q] = 0;
    if (q * SORT_THREADS + (w << 6) < nb) {   // (uniform)
      const int d = threadIdx.x + q * SORT_THREADS;
      if (d < nb) {
#pragma unroll
        for (int ww = 0; ww < SORT_WAVES; ++ww) {
          const uint32_t c = lds.cnt[ww][d];
          lds.cnt[ww][d] = (uint16_t)tot[q];
          tot[q] += c;
        }
      }
      incl[q] = wave_prefix(tot[q]);
      incl_total[q] = wave_prefix(d < nb ? total[q] : 0);
    }
    if (lane == 63) {
      lds.wsum[0][q][w] = incl[q];
      lds.wsum[1][q][w] = incl_total[q];
    }
  }
  __syncthreads();
  {
    uint32_t before = 0, before_total = 0;  // keys with a digit handled by an earlier (q, wavefront): of the tile, of the field
#pragma unroll
    for (int q = 0; q < DPT; ++q) {
      if (q * SORT_THREADS < nb) {   // (uniform)
        uint32_t mine = before, mine_total = before_total;
        for (int ww = 0; ww < SORT_WAVES; ++ww) {
          const uint32_t c = lds.wsum[0][q][ww], ct = lds.wsum[1][q][ww];
          if (ww < w) {
            mine += c;
            mine_total += ct;
          }
          before += c;
          before_total += ct;
        }
        const int d = threadIdx.x + q * SORT_THREADS;
        if (d < nb) {
          const uint32_t place = mine + incl[q] - tot[q];  // of the digit's first key in the sorted tile
          lds.dpre[d] = (uint16_t)place;
          lds.gbase[d] = mine_total + incl_total[q] - total[q] + earlier[q] - place;   // output position = gbase[d] + place in the sorted tile
          // (positions are 31 bits wide: the highest one says that the bucket has one row)
          if constexpr (BUCKETS) lds.gbase[d] = (lds.gbase[d] & 0x7FFFFFFFu) | (fb.first[d + 1] - fb.first[d] == 1 ? 0x80000000u : 0);
        }
      }
    }
  }
  __syncthreads();
  uint32_t lp[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint32_t d = digits[i];
    lp[i] = lds.dpre[d] + lds.cnt[w][d] + rank[i];
  }
  __syncthreads();  // the counters are dead: their memory stages the tile sorted by digit
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    if ((FULL || first + i * 64 < count) && lp[i] < (uint32_t)SORT_TILE) {
      if constexpr (BUCKETS) {
        lds.staged[0][lp[i]] = (int32_t)((uint32_t)(key[i] - fb.first[digits[i]]) << bp.sample_bits | ((uint32_t)pay[i] & ((1u << bp.sample_bits) - 1)));
        lds.staged[1][lp[i]] = (int32_t)digits[i];
      } else {
        lds.staged[0][lp[i]] = key[i];
        lds.staged[1][lp[i]] = pay[i];
      }
    }
  }
  __syncthreads();
  // Consecutive threads hold consecutive keys of the sorted tile: keys of one digit go to consecutive
  // positions of the output, so that their 4-byte stores merge into one request per run.
#pragma unroll
  for (int q = 0; q < ITEMS; ++q) {
    const int j = q * SORT_THREADS + threadIdx.x;
    if (FULL || j < count) {
      const int32_t k = lds.staged[0][j];
      if constexpr (BUCKETS) {
        const int d = lds.staged[1][j];
        const uint32_t base = lds.gbase[d], dst = (base + (uint32_t)j) & 0x7FFFFFFFu;
        if (dst >= (uint32_t)nnz) continue;
        if ((int32_t)base >= 0) {
          packed[dst] = k;
        } else {
          keys_out[dst] = fb.first[d];
          pay_out[dst] = k;
        }
      } else {
        const uint32_t dst = lds.gbase[digit(k)] + (uint32_t)j;
        if (dst < (uint32_t)nnz) {
          keys_out[dst] = k;
          pay_out[dst] = lds.staged[1][j];
        }
      }
    }
  }
}

template <bool BUCKETS>
__global__ __launch_bounds__(SORT_THREADS, 8) void sort_scatter_kernel(
    const int32_t* keys_in, const int32_t* pay_in, int32_t* keys_out, int32_t* pay_out, int32_t* packed, const uint32_t* hist,
    const uint32_t* digit_total, FieldPtr fp, TileBase tb, int F, int shift, int rb, BucketPlan bp) {
  __shared__ ScatterLds lds;
  __shared__ typename std::conditional<BUCKETS, FieldBuckets, int>::type fb;
  static_assert(4 * (sizeof(lds) + sizeof(fb)) <= 160 * 1024, "four blocks to fill a compute unit's places for wavefronts");
  int f, t, part;
  if (!tile_of_block(tb, F, 1, f, t, part)) return;
  const int64_t base = fp.p[f], start = base + (int64_t)t * SORT_TILE;
  const int nnz = (int)(fp.p[f + 1] - base), count = min(SORT_TILE, nnz - t * SORT_TILE);
  const uint32_t* hb = hist + ((int64_t)(tb.t[f] + t) << rb);
  const uint32_t* totals = digit_total + ((int64_t)f << rb);
  if (count == SORT_TILE) scatter_tile<true, BUCKETS>(lds, keys_in + start, pay_in + start, keys_out + base, pay_out + base, packed + base, hb, totals, count, nnz, shift, rb, bp, fb, bp.fields + f, f,
                                                    t * SORT_TILE);
  else scatter_tile<false, BUCKETS>(lds, keys_in + start, pay_in + start, keys_out + base, pay_out + base, packed + base, hb, totals, count, nnz, shift, rb, bp, fb, bp.fields + f, f,
                                                    t * SORT_TILE);
}

// A block sorts a bucket's lookups (place of the row in the bucket, sample; in sample order) by the rows and takes the words apart.  Up to
// BUCKET_KEYS of them stay in LDS, in passes of up to BUCKET_BITS bits; what more there are (cuts are made by a sample) go
// through memory, BUCKET_KEYS at a time, by the first blocks of the launch.
// A lookup is read and written twice on the way from the batch to its place, as one word in between, where a pass over all of them reads it
// twice and writes it once (42 M lookups: 1.0 GB instead of 2.5).  Bound by the ballots (a bit of a lookup costs four instructions a
// wavefront either way).  42 M lookups of Zipf(1.2) ids, us: cuts 17, histogram 79, scan 12, scatter 153, buckets 184.  By the ids' highest bits instead, the
// buckets of hot rows kept single blocks busy: 522; 1024 threads with 8 lookups each: 337 where ids are even (512 with 16: 214).  Four
// tiles a block in the histogram, or the buckets' numbers kept as bytes for the scatter: 77 and 98 there, 154 and 141 in the scatter.
struct BucketLds {
  uint16_t cnt[BUCKET_WAVES][1 << BUCKET_BITS];
  uint32_t base[1 << BUCKET_BITS];           // place of a digit's first key of those in hand
  uint32_t count[2][1 << BUCKET_BITS];       // large buckets: where the digit's next key goes, of each pass
  uint32_t wsum[BUCKET_WAVES];
  int32_t stage[BUCKET_KEYS];
};
// Ranks of the n keys in hand (item i of wavefront w: position 64 (w per + i) + lane) among those of their digit in their wavefront;
// lds.cnt: keys of the digit in the wavefronts before.  Returns the block's keys of digit threadIdx.x.
__device__ __forceinline__ uint32_t rank_keys(BucketLds& lds, const uint32_t (&x)[BUCKET_ITEMS], int n, int per, int shift, int bits,
                                              uint32_t (&rank)[BUCKET_ITEMS]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nb = 1 << bits;
  const int first = w * (64 * per) + lane;
  const uint64_t lt = lanemask_lt();
  for (int d = lane; d < nb; d += 64) lds.cnt[w][d] = 0;   // (each wavefront its own row)
  wave_lds_order();
#pragma unroll
  for (int i = 0; i < BUCKET_ITEMS; ++i) {
    rank[i] = 0;
    if (i < per && w * (64 * per) + i * 64 < n) {   // (uniform)
      const bool valid = first + i * 64 < n;
      const uint32_t d = (x[i] >> shift) & (uint32_t)(nb - 1);
      const uint64_t m = same_digit(d, bits, valid);
      const uint32_t prior = lds.cnt[w][d];
      wave_lds_order();
      rank[i] = prior + (uint32_t)__popcll(m & lt);
      if (valid && (m & lt) == 0) lds.cnt[w][d] = (uint16_t)(prior + (uint32_t)__popcll(m));   // lowest lane of the group
      wave_lds_order();
    }
  }
  __syncthreads();
  uint32_t tot = 0;
  if ((int)threadIdx.x < nb) {
    uint32_t c[BUCKET_WAVES];
#pragma unroll
    for (int q = 0; q < BUCKET_WAVES; ++q) c[q] = lds.cnt[q][threadIdx.x];
#pragma unroll
    for (int q = 0; q < BUCKET_WAVES; ++q) {
      lds.cnt[q][threadIdx.x] = (uint16_t)tot;
      tot += c[q];
    }
  }
  return tot;
}
__device__ __forceinline__ void sort_bucket(BucketLds& lds, const BucketPlan& bp, const uint32_t* in, int32_t* keys_out, int32_t* pay_out, int n,
                                            int row0, int rows) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int per = (n + BUCKET_THREADS - 1) / BUCKET_THREADS;   // <= BUCKET_ITEMS
  const int first = w * (64 * per) + lane;
  auto mine = [&](int i) { return i < per && first + i * 64 < n; };
  uint32_t x[BUCKET_ITEMS] = {};
#pragma unroll
  for (int i = 0; i < BUCKET_ITEMS; ++i)
    if (i < per) x[i] = in[min(first + i * 64, n - 1)];
  const int low = 32 - __clz(rows - 1), passes = (low + BUCKET_BITS - 1) / BUCKET_BITS, most = (low + passes - 1) / passes;
  for (int from = 0; from < low; from += most) {
    const int bits = min(low - from, most), shift = bp.sample_bits + from, nb = 1 << bits;
    uint32_t rank[BUCKET_ITEMS], all;
    const uint32_t tot = rank_keys(lds, x, n, per, shift, bits, rank);
    const uint32_t before = block_prefix(tot, lds.wsum, BUCKET_WAVES, all, false);   // (the sums are read by all before the next barrier)
    if ((int)threadIdx.x < nb) lds.base[threadIdx.x] = before;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < BUCKET_ITEMS; ++i)
      if (mine(i)) {
        const uint32_t d = (x[i] >> shift) & (uint32_t)(nb - 1);
        lds.stage[lds.base[d] + lds.cnt[w][d] + rank[i]] = (int32_t)x[i];
      }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < BUCKET_ITEMS; ++i)
      if (mine(i)) x[i] = (uint32_t)lds.stage[first + i * 64];   // (three barriers before the next pass writes there)
  }
#pragma unroll
  for (int i = 0; i < BUCKET_ITEMS; ++i)
    if (mine(i)) {
      keys_out[first + i * 64] = row0 + (int32_t)(x[i] >> bp.sample_bits);
      pay_out[first + i * 64] = (int32_t)(x[i] & ((1u << bp.sample_bits) - 1));
    }
}
// More than BUCKET_KEYS lookups: two passes from `in` to `between` to the results.
__device__ __forceinline__ void sort_large_bucket(BucketLds& lds, const BucketPlan& bp, const uint32_t* in, uint32_t* between, int32_t* keys_out,
                                                  int32_t* pay_out, int n, int row0, int rows) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int low = 32 - __clz(rows - 1);
  const int bits[2] = {(low + 1) / 2, low / 2}, shift[2] = {bp.sample_bits, bp.sample_bits + bits[0]};
  for (int d = threadIdx.x; d < 2 << BUCKET_BITS; d += BUCKET_THREADS) (&lds.count[0][0])[d] = 0;
  __syncthreads();
  for (int c0 = 0; c0 < n; c0 += BUCKET_KEYS) {   // keys of every digit
    uint32_t x[BUCKET_ITEMS];
#pragma unroll
    for (int i = 0; i < BUCKET_ITEMS; ++i) x[i] = in[min(c0 + i * BUCKET_THREADS + (int)threadIdx.x, n - 1)];
#pragma unroll
    for (int i = 0; i < BUCKET_ITEMS; ++i) {
      const bool valid = c0 + i * BUCKET_THREADS + (int)threadIdx.x < n;
#pragma unroll
      for (int p = 0; p < 2; ++p) {   // one addition for the lanes of a digit: hot rows make them many
        const uint32_t d = (x[i] >> shift[p]) & ((1u << bits[p]) - 1);
        const uint64_t m = same_digit(d, bits[p], valid);
        if (valid && (m & lanemask_lt()) == 0) atomicAdd(&lds.count[p][d], (uint32_t)__popcll(m));
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const uint32_t tot = (int)threadIdx.x < 1 << BUCKET_BITS ? lds.count[p][threadIdx.x & ((1 << BUCKET_BITS) - 1)] : 0;
    uint32_t all;
    const uint32_t before = block_prefix(tot, lds.wsum, BUCKET_WAVES, all);
    if ((int)threadIdx.x < 1 << BUCKET_BITS) lds.count[p][threadIdx.x] = before;
  }
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const uint32_t* from = p == 0 ? in : between;
    for (int c0 = 0; c0 < n; c0 += BUCKET_KEYS) {
      const int nc = min(n - c0, BUCKET_KEYS), per = (nc + BUCKET_THREADS - 1) / BUCKET_THREADS, first = w * (64 * per) + lane;
      uint32_t x[BUCKET_ITEMS] = {}, rank[BUCKET_ITEMS];
#pragma unroll
      for (int i = 0; i < BUCKET_ITEMS; ++i)
        if (i < per) x[i] = from[c0 + min(first + i * 64, nc - 1)];
      const uint32_t tot = rank_keys(lds, x, nc, per, shift[p], bits[p], rank);
      if ((int)threadIdx.x < 1 << bits[p]) {
        const uint32_t at = lds.count[p][threadIdx.x];
        lds.base[threadIdx.x] = at;
        lds.count[p][threadIdx.x] = at + tot;
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < BUCKET_ITEMS; ++i)
        if (i < per && first + i * 64 < nc) {
          const uint32_t d = (x[i] >> shift[p]) & ((1u << bits[p]) - 1);
          const uint32_t dst = lds.base[d] + lds.cnt[w][d] + rank[i];
          if (dst >= (uint32_t)n) continue;   // (never)
          if (p == 0) {
            between[dst] = x[i];
          } else {
            keys_out[dst] = row0 + (int32_t)(x[i] >> bp.sample_bits);
            pay_out[dst] = (int32_t)(x[i] & ((1u << bp.sample_bits) - 1));
          }
        }
      __syncthreads();   // (counters and bases are the next ones')
    }
    // (what other wavefronts wrote is read next: they are of this block, and its compute unit, whose barrier waits for their stores)
  }
}
__global__ __launch_bounds__(BUCKET_THREADS) void sort_buckets_kernel(const int32_t* in, int32_t* between, int32_t* keys_out, int32_t* pay_out,
                                                                      const uint32_t* digit_total, FieldPtr fp, int F, int large_blocks,
                                                                      BucketPlan bp) {
  __shared__ BucketLds lds;
  auto place = [&](int f, int b, int64_t& at, int& n) {   // the bucket's lookups: those of the field's buckets before it come first
    const uint32_t* totals = digit_total + ((int64_t)f << bp.rb);
    const int lane = threadIdx.x & 63;
    uint32_t t[MAX_BUCKETS / 64], before = 0;
#pragma unroll
    for (int q = 0; q < MAX_BUCKETS / 64; ++q) t[q] = totals[min(q * 64 + lane, b)];
#pragma unroll
    for (int q = 0; q < MAX_BUCKETS / 64; ++q) before += q * 64 + lane < b ? t[q] : 0;
    before = (uint32_t)__builtin_amdgcn_readlane((int)wave_prefix(before), 63);
    at = fp.p[f] + before;
    n = max(min((int64_t)totals[b], fp.p[f + 1] - at), (int64_t)0);
  };
  int64_t at;
  int n;
  if ((int)blockIdx.x < large_blocks) {
    const int count = min(bp.large[0], bp.most_large);
    for (int i = blockIdx.x; i < count; i += large_blocks) {
      const int f = bp.large[1 + i] >> 16, b = bp.large[1 + i] & 0xFFFF;
      place(f, b, at, n);
      const int row0 = bp.fields[f].first[b], rows = bp.fields[f].first[b + 1] - row0;
      sort_large_bucket(lds, bp, reinterpret_cast<const uint32_t*>(in) + at, reinterpret_cast<uint32_t*>(between) + at, keys_out + at, pay_out + at, n, row0,
                        rows);
    }
    return;
  }
  // (the buckets of a field on the XCD that its tiles were scattered on, see tile_of_block)
  const int block = (int)blockIdx.x - large_blocks, total = F << bp.rb, share = (total + 7) >> 3, i = (block & 7) * share + (block >> 3);
  if ((block >> 3) >= share || i >= total) return;
  const int f = i >> bp.rb, b = i - (f << bp.rb);
  if (fp.p[f + 1] == fp.p[f]) return;
  const int row0 = bp.fields[f].first[b], rows = bp.fields[f].first[b + 1] - row0;
  if (rows <= 1) return;   // (the partition has put these where they belong)
  place(f, b, at, n);
  if (n == 0 || n > BUCKET_KEYS) return;
  sort_bucket(lds, bp, reinterpret_cast<const uint32_t*>(in) + at, keys_out + at, pay_out + at, n, row0, rows);
}

// Block = field.
template <int IT>
__global__ __launch_bounds__(SMALL_THREADS) void sort_small_kernel(const int32_t* keys_in, const int32_t* pay_in, int32_t* keys_out,
                                                                   int32_t* pay_out, FieldPtr fp, int passes, int rb) {
  __shared__ SmallSortLds lds;
  extern __shared__ int32_t stage[];   // [SMALL_THREADS * IT]
  const int64_t base = fp.p[blockIdx.x];
  sort_small_field<IT>(lds, stage, keys_in + base, pay_in + base, keys_out + base, pay_out + base, (int)(fp.p[blockIdx.x + 1] - base), passes, rb);
}

template <int IT>
hipError_t launch_sort_small_items(const SortPlan& pl, const SortBuffers& sb, const FieldPtr& fp, Profiler* prof, hipStream_t s) {
  constexpr int bytes = SMALL_THREADS * IT * 4;
  static std::atomic<uint64_t> allowed{0};
  const hipError_t ok = allow_lds(sort_small_kernel<IT>, bytes, 36 * 1024, allowed);
  if (ok != hipSuccess) return ok;
  ProfScope ps(prof, KID_SORT_SCATTER, s);
  hipLaunchKernelGGL((sort_small_kernel<IT>), dim3(pl.F), dim3(SMALL_THREADS), bytes, s,
                     sb.ids, sb.pay0, sb.key[0], sb.pay[0], fp, pl.passes, pl.radix_bits);
  return hipGetLastError();
}

// Sample index of every lookup, from the offsets alone: what the gather records along the way, for a sort that does not
// wait for the gather.  Eight lanes per bag.  It runs beside the gather, which the two then share the memory with: 17 MB of
// sample indices in 61 us (11 with the chip to itself), 167 MB in 404 us (the gather 490).
__global__ __launch_bounds__(256) void expand_samples_kernel(const int32_t* offsets, int32_t* lookup_sample, FieldPtr fp, int B) {
  const int f = blockIdx.y, c = threadIdx.x & 7;
  const int s = blockIdx.x * 32 + (threadIdx.x >> 3);
  if (s >= B) return;
  const int32_t* off = offsets + (int64_t)f * (B + 1) + s;
  const int nnz = (int)(fp.p[f + 1] - fp.p[f]);
  const int e = min(off[1], nnz);
  int32_t* out = lookup_sample + fp.p[f];
  for (int j = max(off[0], 0) + c; j < e; j += 8) out[j] = s;
}

// ------------------------------------------------- leaving shards out
// When the servers disregard the gradients of some workers (the backup-workers baseline of
// Section VII-A.3), only the lookups of the remaining shards are coalesced.  A shard is a
// contiguous range of samples, hence a contiguous range of every field's lookups: the ranges
// of the included shards (weight != 0) are packed side by side, field after field.

// cbase[f] = number of included lookups in the fields before f (cbase[F] = their total).
__global__ __launch_bounds__(256) void mask_count_kernel(const int32_t* offsets, int64_t B, int F, ShardTab tab,
                                                         int64_t* cbase) {
  __shared__ int64_t cnt[ANTDT_MAX_FIELDS];
  for (int f = threadIdx.x; f < F; f += 256) {
    const int32_t* off = offsets + (int64_t)f * (B + 1);
    int64_t c = 0;
    for (int k = 0; k < tab.K; ++k)
      if (tab.w[k] != 0.0f) c += off[tab.start[k] + tab.len[k]] - off[tab.start[k]];
    cnt[f] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t run = 0;
    for (int f = 0; f < F; ++f) {
      cbase[f] = run;
      run += cnt[f];
    }
    cbase[F] = run;
  }
}

// Blocks (k, f, *) copy the ids and sample indices of shard k's lookups in field f, PACK_LOOKUPS each in turn: bound by the chain
// of loads (one block for all of them: 5 shards x 26 fields of 5300 lookups 16 us).
__global__ __launch_bounds__(PACK_THREADS) void mask_pack_kernel(const int32_t* ids, const int32_t* lookup_sample,
                                                                 const int32_t* offsets, int64_t B, FieldPtr fp, ShardTab tab,
                                                                 const int64_t* cbase, int32_t* ids_out, int32_t* pay_out) {
  const int k = blockIdx.x, f = blockIdx.y;
  if (tab.w[k] == 0.0f) return;
  const int32_t* off = offsets + (int64_t)f * (B + 1);
  int64_t dst = cbase[f];
  for (int q = 0; q < k; ++q)
    if (tab.w[q] != 0.0f) dst += off[tab.start[q] + tab.len[q]] - off[tab.start[q]];
  const int64_t src = fp.p[f] + off[tab.start[k]];
  const int64_t n = off[tab.start[k] + tab.len[k]] - off[tab.start[k]];
  pack_rounds(blockIdx.z, threadIdx.x, n, [&](int64_t i0) {
    int32_t id[PACK_ITEMS], smp[PACK_ITEMS];
#pragma unroll
    for (int q = 0; q < PACK_ITEMS; ++q) {
      const int64_t i = min(i0 + q * PACK_THREADS, n - 1);
      id[q] = ids[src + i];
      smp[q] = lookup_sample[src + i];
    }
#pragma unroll
    for (int q = 0; q < PACK_ITEMS; ++q)
      if (i0 + q * PACK_THREADS < n) {
        ids_out[dst + i0 + q * PACK_THREADS] = id[q];
        pay_out[dst + i0 + q * PACK_THREADS] = smp[q];
      }
  });
}

// ------------------------------------------------------------- segments
__device__ __forceinline__ bool is_head(const int32_t* key, int pos) {
  return pos == 0 || key[pos] != key[pos - 1];
}

// Number of run heads in each tile of the sorted keys.
__global__ __launch_bounds__(SORT_THREADS) void seg_heads_kernel(SegArgs a, FieldPtr fp, TileBase tb) {
  __shared__ int wsum[SORT_WAVES];
  int f, t, part;
  if (!tile_of_block(tb, a.F, 1, f, t, part)) return;
  const int32_t* key = a.key + fp.p[f];
  const int nnz = (int)(fp.p[f + 1] - fp.p[f]);
  int c = 0;
#pragma unroll
  for (int i = 0; i < SORT_ITEMS; ++i) {
    const int pos = t * SORT_TILE + i * SORT_THREADS + threadIdx.x;
    if (pos < nnz && is_head(key, pos)) ++c;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    int s = 0;
    for (int i = 0; i < SORT_WAVES; ++i) s += wsum[i];
    a.tile_heads[tb.t[f] + t] = s;
  }
}

// One block: exclusive prefix over all tiles (-> first unique of every tile and field) and the terminal
// segment offset of every field.
__global__ __launch_bounds__(1024) void seg_scan_kernel(SegArgs a, FieldPtr fp, TileBase tb) {
  __shared__ int wsum[16];
  const int n = a.total_tiles;
  const int chunk = (n + 1023) / 1024;
  const int lo = min(n, (int)threadIdx.x * chunk), hi = min(n, lo + chunk);
  int sum = 0;
  for (int i = lo; i < hi; ++i) sum += a.tile_heads[i];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(incl, o, 64);
    if (lane >= o) incl += v;
  }
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  int wbase = 0, total = 0;
  for (int i = 0; i < 16; ++i) {
    if (i < w) wbase += wsum[i];
    total += wsum[i];
  }
  int run = wbase + incl - sum;
  for (int i = lo; i < hi; ++i) {
    const int c = a.tile_heads[i];
    a.tile_heads[i] = run;
    run += c;
  }
  if (threadIdx.x == 0) {
    a.tile_heads[n] = total;
    a.segabs[total] = (int32_t)fp.p[a.F];
  }
  __threadfence_block();
  __syncthreads();
  for (int f = threadIdx.x; f <= a.F; f += 1024) a.ubase[f] = a.tile_heads[tb.t[f]];
  for (int f = threadIdx.x; f < a.F; f += 1024)
    a.segoff[a.tile_heads[tb.t[f + 1]] + f] = (int32_t)(fp.p[f + 1] - fp.p[f]);
}

// Unique ids and segment offsets.  Thread j of a tile owns 8 consecutive sorted positions.
__global__ __launch_bounds__(SORT_THREADS) void seg_emit_kernel(SegArgs a, FieldPtr fp, TileBase tb) {
  __shared__ int wsum[SORT_WAVES];
  int f, t, part;
  if (!tile_of_block(tb, a.F, 1, f, t, part)) return;
  const int32_t* key = a.key + fp.p[f];
  const int nnz = (int)(fp.p[f + 1] - fp.p[f]);
  const int p0 = t * SORT_TILE + threadIdx.x * SORT_ITEMS;
  unsigned flags = 0;
#pragma unroll
  for (int i = 0; i < SORT_ITEMS; ++i)
    if (p0 + i < nnz && is_head(key, p0 + i)) flags |= 1u << i;
  const int c = __popc(flags);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int incl = c;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(incl, o, 64);
    if (lane >= o) incl += v;
  }
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  int rank = a.tile_heads[tb.t[f] + t] + incl - c;
  for (int i = 0; i < w; ++i) rank += wsum[i];
#pragma unroll
  for (int i = 0; i < SORT_ITEMS; ++i)
    if (flags & (1u << i)) {
      a.uniq[rank] = key[p0 + i];
      a.segabs[rank] = (int32_t)fp.p[f] + p0 + i;
      a.segoff[rank + f] = p0 + i;
      ++rank;
    }
}

// ------------------------------------------------- weighted run sums (+ update)
struct RowSum {   // a lane's four columns (4c .. 4c + 3, c: the lane inside its group of D/4)
  float v[4];
};

// Aggregation weights by sample: the ranges of samples of one weight (neighbouring shards of equal weight are one), held by
// the lanes.  (An array of a weight per sample was read at random: a cache line for each lookup of a window of short
// runs, a sixth of the lines that the reduction of 42 M lookups asked L2 for: 1021 -> 963 us a launch, 4.3 M lookups with eight
// weights 150 -> 138.)
struct SampleWeights {
  int32_t n, start;   // ranges; where this lane's begins
  float w;            // its weight (of a single range: in every lane)
  __device__ __forceinline__ SampleWeights(const SegArgs& a, const WeightTab& t) : n(a.weights), start(0x7FFFFFFF), w(a.weight) {
    const int lane = threadIdx.x & 63;
    if (n > 1 && lane < n) {
      start = t.start[lane];
      w = t.w[lane];
    }
  }
  // (by whole wavefronts)
  __device__ __forceinline__ float of(int s) const {
    if (n == 1) return w;
    int i = 0;
    for (int step = 1 << (31 - __clz(n - 1)); step > 0; step >>= 1)   // (n <= 64: i + step is a lane)
      if (s >= __builtin_amdgcn_ds_bpermute((i + step) * 4, start)) i += step;
    return __int_as_float(__builtin_amdgcn_ds_bpermute(i * 4, __float_as_int(w)));
  }
};

// Weight of one lookup of sample s: the shard weight, divided by the length of the sample's bag
// in this field when the bags are mean-pooled (the bag is not empty: the lookup is in it).
template <bool MEAN>
__device__ __forceinline__ float lookup_weight(const SampleWeights& sw, const int32_t* off, int s) {
  const float w = sw.of(s);
  if (!MEAN) return w;
  return w / (float)max(off[s + 1] - off[s], 1);
}

// What the sums need of a sorted lookup, worked out once per lookup when it is staged (and not by each of the D/4
// lanes that then use it): its sample's byte offset in dX, and its weight.
struct __attribute__((aligned(16))) Lookup {
  uint64_t offset;
  float w;
  int32_t unused;
};

// g += w(lookup) * dX[sample, field slice] over `n` staged lookups, added in order, four in flight; dx: this lane's
// columns of sample 0.
__device__ __forceinline__ void accumulate_run(const char* dx, const Lookup* look, int n, RowSum& g) {
  for (int i = 0; i < n; i += 4) {
    float w[4];
    float4 x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (i + q < n) {
        const Lookup l = look[i + q];
        w[q] = l.w;
        x[q] = *reinterpret_cast<const float4*>(dx + l.offset);
      }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (i + q < n) {
        g.v[0] = fmaf(w[q], x[q].x, g.v[0]);
        g.v[1] = fmaf(w[q], x[q].y, g.v[1]);
        g.v[2] = fmaf(w[q], x[q].z, g.v[2]);
        g.v[3] = fmaf(w[q], x[q].w, g.v[3]);
      }
  }
}

__device__ __forceinline__ void add_floats(RowSum& g, const float* x) {
  const float4 v = *reinterpret_cast<const float4*>(x);
  g.v[0] += v.x; g.v[1] += v.y; g.v[2] += v.z; g.v[3] += v.w;
}
__device__ __forceinline__ void store_floats(float* x, const RowSum& g) {
  *reinterpret_cast<float4*>(x) = make_float4(g.v[0], g.v[1], g.v[2], g.v[3]);
}

// x summed over the lane's group of lps (a power of two) lanes; every lane of the group gets the same bits.
__device__ __forceinline__ float group_sum(float x, int lps) {
  auto moved = [](float v, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), decltype(ctrl)::value, 0xF, 0xF, true));
  };
  if (lps > 1) x += moved(x, std::integral_constant<int, 0xB1>());    // lane ^ 1
  if (lps > 2) x += moved(x, std::integral_constant<int, 0x4E>());    // lane ^ 2
  if (lps > 4) x += moved(x, std::integral_constant<int, 0x141>());   // the other four of eight (mirrored: they hold the same)
  if (lps > 8) x += moved(x, std::integral_constant<int, 0x140>());   // the other eight of sixteen
  if (lps > 16) x += __shfl_xor(x, 16, 64);
  if (lps > 32) x += __shfl_xor(x, 32, 64);
  return x;
}

// Square root and quotient for operands far from the ends of the exponent range (the general ones spend two thirds of
// their instructions on those): the hardware's estimates, a Newton step, and for the quotient Markstein's correction by the
// remainder ("Computation of elementary functions on the IBM RISC System/6000 processor", 1990), which rounds right if the
// reciprocal does and neither quotient nor remainder leaves the range.  Rounded right on this hardware are the roots of all floats from
// 2^-90 to 2^90 and the reciprocals of all from 2^-46 to 2^47 (each compared), so with roots and numerators bounded as in
// TableRow::update, quotients within 2^-125 .. 2^124, these are the bits of the general ones (1.7e10 pairs compared: the same).
__device__ __forceinline__ float sqrt_mid(float x) {
  const float y = __builtin_amdgcn_rsqf(x), r = x * y;
  return fmaf(fmaf(-r, r, x), 0.5f * y, r);
}
__device__ __forceinline__ float rcp_mid(float d) {
  const float r = __builtin_amdgcn_rcpf(d);
  return fmaf(fmaf(-d, r, 1.0f), r, r);
}
__device__ __forceinline__ float div_mid(float n, float d, float rcp) {   // (fixed up: NaN stays NaN, infinity infinite, 0 / d is 0)
  const float q = n * rcp;
  return __builtin_amdgcn_div_fixupf(fmaf(fmaf(-q, d, n), rcp, q), d, n);
}
__device__ __forceinline__ uint32_t beyond_mid(float x) {   // below MID_SPAN: 2^-90 <= x < 2^90 (not a NaN)
  return __float_as_uint(x) - ((127u - 90u) << 23);
}
constexpr uint32_t MID_SPAN = 180u << 23;
__device__ __forceinline__ uint32_t magnitude_or_zero(float x) {   // from MID_LEAST on: 2^-75 <= |x|, or 0
  return (__float_as_uint(x) << 1) - 1;
}
constexpr uint32_t MID_LEAST = ((127u - 75u) << 24) - 1;

// A lane's columns of one table row and of its accumulators, as they lie in memory, and the row-sparse Adagrad step:
//   element-wise: S += g^2;                 p -= lr * g / (sqrt(S) + eps)
//   row-wise:     S[r] += mean_d g[r,d]^2;  p -= lr * g / (sqrt(S[r]) + eps)
// bf16 tables are written back round-to-nearest-even.
template <typename TT, bool ROWWISE> struct TableRow {
  uint4 p;          // (bf16: x and y only)
  float4 s;
  float srow;
  __device__ __forceinline__ void load(const SegArgs& a, int64_t row, int c) {
    const TT* src = reinterpret_cast<const TT*>(a.tables) + row * a.D + c * 4;
    if (sizeof(TT) == 4) {
      p = *reinterpret_cast<const uint4*>(src);
    } else {
      const uint2 v = *reinterpret_cast<const uint2*>(src);
      p.x = v.x;
      p.y = v.y;
    }
    if (ROWWISE) srow = a.state[row];
    else s = *reinterpret_cast<const float4*>(a.state + row * a.D + c * 4);
  }
  __device__ __forceinline__ void update(const SegArgs& a, int64_t row, int c, int lps, const RowSum& g) const {
    float sv[4];
    uint32_t beyond;
    if (ROWWISE) {
      const float sq = group_sum((g.v[0] * g.v[0] + g.v[1] * g.v[1]) + (g.v[2] * g.v[2] + g.v[3] * g.v[3]), lps);
      sv[0] = srow + sq * a.inv_dim;   // (D is a power of two)
      if (c == 0) a.state[row] = sv[0];
      beyond = beyond_mid(sv[0]);
    } else {
      sv[0] = fmaf(g.v[0], g.v[0], s.x);
      sv[1] = fmaf(g.v[1], g.v[1], s.y);
      sv[2] = fmaf(g.v[2], g.v[2], s.z);
      sv[3] = fmaf(g.v[3], g.v[3], s.w);
      *reinterpret_cast<float4*>(a.state + row * a.D + c * 4) = make_float4(sv[0], sv[1], sv[2], sv[3]);
      beyond = max(max(beyond_mid(sv[0]), beyond_mid(sv[1])), max(beyond_mid(sv[2]), beyond_mid(sv[3])));
    }
    float p0[4], p1[4];
    if (sizeof(TT) == 4) {
      p0[0] = __uint_as_float(p.x); p0[1] = __uint_as_float(p.y); p0[2] = __uint_as_float(p.z); p0[3] = __uint_as_float(p.w);
    } else {
      p0[0] = __uint_as_float(p.x << 16); p0[1] = __uint_as_float(p.x & 0xFFFF0000u);
      p0[2] = __uint_as_float(p.y << 16); p0[3] = __uint_as_float(p.y & 0xFFFF0000u);
    }
    constexpr int NS = ROWWISE ? 1 : 4;
    float n[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) n[e] = a.lr * g.v[e];
    const uint32_t least = min(min(magnitude_or_zero(n[0]), magnitude_or_zero(n[1])), min(magnitude_or_zero(n[2]), magnitude_or_zero(n[3])));
    // Accumulators and gradients of any run under way.  (A root is below 2^45, a gradient of 256 columns below 2^49 then.)
    if ((__ballot(beyond >= MID_SPAN) | __ballot(least < MID_LEAST)) == 0 && a.eps < 0x1p45f && a.lr < 0x1p30f) {
      float den[NS], rcp[NS];
#pragma unroll
      for (int e = 0; e < NS; ++e) {
        den[e] = sqrt_mid(sv[e]) + a.eps;
        rcp[e] = rcp_mid(den[e]);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) p1[e] = p0[e] - div_mid(n[e], den[e % NS], rcp[e % NS]);
    } else {
      float den[NS];
#pragma unroll
      for (int e = 0; e < NS; ++e) den[e] = sqrtf(sv[e]) + a.eps;
#pragma unroll
      for (int e = 0; e < 4; ++e) p1[e] = p0[e] - n[e] / den[e % NS];
    }
    TT* dst = reinterpret_cast<TT*>(a.tables) + row * a.D + c * 4;
    if (sizeof(TT) == 4) *reinterpret_cast<float4*>(dst) = make_float4(p1[0], p1[1], p1[2], p1[3]);
    else *reinterpret_cast<uint2*>(dst) = make_uint2(f2bf2(p1[0], p1[1]), f2bf2(p1[2], p1[3]));
  }
};

// Slot of a field's first window (see window_slots).
__device__ __forceinline__ int64_t window_slot(int64_t field_start) { return field_start >> 7; }

// First run of field f that starts at absolute position `pos` of the sorted lookups or behind it (run table present).
__device__ __forceinline__ int64_t run_index(const SegArgs& a, int f, int pos) {
  int lo = a.ubase[f], hi = a.ubase[f + 1] - 1;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (a.segabs[mid] < pos) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// Sums of the runs of equal ids and, when `UPDATE`, the Adagrad step of each row at once (the coalesced
// gradient never goes to memory); otherwise the sums are written to G.
//
// A block takes a window of W sorted lookups, straight from the sort: keys and sample indices of the window
// (and of LONG_RUN lookups on either side) go to LDS, the block finds the runs' heads there, and groups of
// D/4 lanes take one item of work each: a whole run of up to LONG_RUN lookups that starts in the window (it may
// end behind it), summed in sorted (= sample) order, or, of longer runs, a piece of at most LONG_RUN lookups
// that ends at a multiple of LONG_RUN in the window.  The pieces' sums meet in LDS in order; what of a run leaves the window
// goes to memory (two slots per window: the run that comes in, the run that goes out) and is added up by seg_finish_kernel (nothing leaves it
// where a window holds its field: 1024 threads, see fill_seg_args in ctx.hip).  No run table is needed (counting, scanning and
// writing one, with lists of the long runs, were six launches and 10-250 us between sort and reduction), only keys, sample indices and
// the rows themselves are read, and the chain of dependent accesses is down to LDS -> row and pooled gradients.
// A window that lies inside one run (60 % of them with 42 M lookups of Zipf(1.2) ids) needs none of this: sum_window.
// Bound by the requests for pooled-gradient rows that a compute unit can have outstanding (about 64 lines; they come from
// L2 and the memory-side cache) and by vector instructions (67 % of the cycles; windows inside a run have a way of their own and the
// update goes without the general square root and division; the pooled-gradient rows of a sample that looks a
// row up several times are read once there).  Row and accumulators are requested ahead of the item's pooled gradients, not
// an item ahead: that took 8 registers more, and eight wavefronts per SIMD hide as much.  Us per launch, before / now:
// 42 M lookups of 128-byte bf16 rows 1228 / 1016 (963 with the weights in registers, see SampleWeights; of that 880 in the
// windows of short runs; 978 with the update's numerators bounded), 3.8 M 141 / 119 (122), 4.3 M of 128-byte fp32 rows 161 / 148 (138),
// 1.1 M 46.6 / 41.7 (42).
// Streaming loads and stores of the rows: 42 M 1003, but 1.1 M of a batch that returns 53 (they leave the memory-side cache).
constexpr int LONG_RUN = 16;

// Sum over the W lookups of a window that lies inside one run; every lane group of the first wavefront returns it.  Nothing
// is to be found there, so each wavefront works on lookups of its own (its part of `look`), without the others until the
// sums meet.  Lookups of one row by one sample are neighbours (the sort is stable) and become one pair with a
// multiple of the weight.
template <int W, int THREADS>
__device__ __forceinline__ RowSum sum_window(const char* dx, Lookup* look, const int (&smp)[W / THREADS], const float (&weight)[W / THREADS],
                                             int64_t pitch, float* wave_sums, int D, int lps, int c) {
  constexpr int ROUNDS = W / THREADS;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Lookup* mine = look + wave * (64 * ROUNDS);
  int n = 0;
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const bool start = lane == 0 || smp[r] != __shfl_up(smp[r], 1, 64);
    const uint64_t starts = __ballot(start);
    if (start) {
      const uint64_t rest = lane == 63 ? 0 : starts >> (lane + 1);
      Lookup l;
      l.offset = (uint64_t)smp[r] * (uint64_t)pitch;
      l.w = weight[r] * (float)(rest ? __ffsll((unsigned long long)rest) : 64 - lane);
      l.unused = 0;
      mine[n + __popcll(starts & lanemask_lt())] = l;
    }
    n += __popcll(starts);
  }
  wave_lds_order();
  const int ngroups = 64 / lps;
  RowSum sum = {};
  for (int i = lane / lps; i < n; i += 4 * ngroups) {
    float w[4];
    float4 x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (i + q * ngroups < n) {
        const Lookup l = mine[i + q * ngroups];
        w[q] = l.w;
        x[q] = *reinterpret_cast<const float4*>(dx + l.offset);
      }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (i + q * ngroups < n) {
        sum.v[0] = fmaf(w[q], x[q].x, sum.v[0]);
        sum.v[1] = fmaf(w[q], x[q].y, sum.v[1]);
        sum.v[2] = fmaf(w[q], x[q].z, sum.v[2]);
        sum.v[3] = fmaf(w[q], x[q].w, sum.v[3]);
      }
  }
  for (int o = lps; o < 64; o <<= 1) {
#pragma unroll
    for (int e = 0; e < 4; ++e) sum.v[e] += __shfl_xor(sum.v[e], o, 64);
  }
  if (lane < lps) store_floats(wave_sums + wave * D + c * 4, sum);
  __syncthreads();
  sum = {};
#pragma unroll
  for (int q = 0; q < THREADS / 64; ++q) add_floats(sum, wave_sums + q * D + c * 4);
  return sum;
}

template <typename TT, bool ROWWISE, bool UPDATE, bool MEAN, int W, int THREADS>
__global__ __launch_bounds__(THREADS, ROWWISE ? 8 : 1) void seg_window_kernel(SegArgs a, FieldPtr fp, TileBase tb, WeightTab wt, DenseJob dense) {
  constexpr int PARTS = SORT_TILE / W, ROUNDS = W / THREADS, WAVES = THREADS / 64;
  constexpr int BITS = W <= 512 ? 9 : 11, POS = (1 << BITS) - 1, HEAD = 1 << BITS, PIECE = 2 << BITS;   // entries of `order`
  static_assert(W <= 2048 && LONG_RUN == 16, "list entries and the search for long runs");
  __shared__ int32_t key_[W + 2 * LONG_RUN];        // positions -LONG_RUN .. W + LONG_RUN - 1 relative to the window
  __shared__ Lookup look[W + LONG_RUN];
  __shared__ uint16_t order[W];                     // work items: runs of up to four lookups from the front (position, length), others from the end
  __shared__ int16_t lead[W / LONG_RUN + 1];        // pieces' runs: [0] the one that comes in, [1 + j] starts in the j-th LONG_RUN positions
  __shared__ int counts[ROUNDS][WAVES];
  __shared__ int goes_out;
  __shared__ uint64_t heads[UPDATE ? 1 : W / 64];   // (sums written out: the place of a run is the window's first one's + heads before)
  __shared__ int64_t first_run;
  // [2 W / LONG_RUN][D], piece 2 j: starts at LONG_RUN j inside its run, 2 j + 1: at the run's head
  extern __shared__ __attribute__((aligned(16))) float piece_sum[];
  // The blocks behind those of the windows: the dense update of an fp32 model (a launch of 4 - 13 us by itself; a step of 256 samples of 141-64-32
  // 45.7 -> 42.6 us, 1500 of 397-256-128 97.9 -> 93.4, 512 of 845-1024-512-256 198 -> 187).
  if (UPDATE) {
    const int windows = (int)tile_grid(tb.t[a.F]) * PARTS;
    if ((int)blockIdx.x >= windows) {
      const int64_t i = (int64_t)((int)blockIdx.x - windows) * THREADS + threadIdx.x;
      if (i < dense.n) adagrad_elem(dense, dense, i);
      return;
    }
  }
  int f, t, part;
  if (!tile_of_block(tb, a.F, PARTS, f, t, part)) return;
  const int64_t base = fp.p[f];
  const int nnz = (int)(fp.p[f + 1] - base);
  const int P = t * SORT_TILE + part * W;
  const int tid = threadIdx.x;
  if (P >= nnz) return;
  const int64_t slot = window_slot(base) + t * PARTS + part;
  const SampleWeights weights(a, wt);
  const int32_t* off = MEAN ? a.offsets + (int64_t)f * (a.B + 1) : nullptr;
  const int32_t *keys = a.key + base, *pay = a.pay + base;
  const int32_t first_key = __builtin_amdgcn_readfirstlane(keys[P]), last_key = __builtin_amdgcn_readfirstlane(keys[min(P + W, nnz) - 1]);
  int32_t k_own[ROUNDS], k_side = 0;
  int smp[ROUNDS], smp_tail = 0;
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int pos = min(P + r * THREADS + tid, nnz - 1);
    k_own[r] = keys[pos];
    smp[r] = pay[pos];
  }
  if (tid < 2 * LONG_RUN) k_side = keys[min(max(tid < LONG_RUN ? P + tid - LONG_RUN : P + W + tid - LONG_RUN, 0), nnz - 1)];
  if (tid < LONG_RUN) smp_tail = pay[min(P + W + tid, nnz - 1)];
  float weight[ROUNDS], weight_tail = 0.0f;
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    smp[r] = min(max(smp[r], 0), a.B - 1);
    weight[r] = lookup_weight<MEAN>(weights, off, smp[r]);
  }
  const int lps = a.D >> 2;
  const int ngroups = THREADS / lps;
  const int g = tid / lps, c = tid - g * lps;
  const char* dx = reinterpret_cast<const char*>(a.dx + f * a.D + c * 4);
  if (P + W <= nnz && first_key == last_key) {   // (the same for all threads)
    const bool in = P > 0 && keys[P - 1] == first_key, out = P + W < nnz && keys[P + W] == first_key;
    const int64_t row = (int64_t)f * a.R + min(max(first_key, 0), (int)(a.R - 1));
    TableRow<TT, ROWWISE> tr;
    if (UPDATE && !in && !out && tid < lps) tr.load(a, row, c);
    const RowSum sum = sum_window<W, THREADS>(dx, look, smp, weight, a.lddx * 4, piece_sum, a.D, lps, c);
    if (tid < lps) {
      if (in || out) store_floats(a.partial + (slot * 2 + (in ? 0 : 1)) * a.D + c * 4, sum);
      else if (UPDATE) tr.update(a, row, c, lps, sum);
      else store_floats(a.G + run_index(a, f, (int)base + P) * a.D + c * 4, sum);
    }
    if (tid == 0 && nnz > W) a.goes_out[slot] = !in && out;
    return;
  }
  if (tid < 64) {   // (a whole wavefront, for LONG_RUN lookups)
    smp_tail = min(max(smp_tail, 0), a.B - 1);
    weight_tail = lookup_weight<MEAN>(weights, off, smp_tail);
  }
  auto stage = [&](int i, int sample, float w) {
    Lookup l;
    l.offset = (uint64_t)sample * (uint64_t)(a.lddx * 4);
    l.w = w;
    l.unused = 0;
    look[i] = l;
  };
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    key_[LONG_RUN + r * THREADS + tid] = k_own[r];
    stage(r * THREADS + tid, smp[r], weight[r]);
  }
  if (tid < 2 * LONG_RUN) key_[tid < LONG_RUN ? tid : W + tid] = k_side;
  if (tid < LONG_RUN) stage(W + tid, smp_tail, weight_tail);
  if (tid <= W / LONG_RUN) lead[tid] = -1;
  if (tid == 0) {
    goes_out = 0;
    if (!UPDATE) first_run = run_index(a, f, (int)base + P);
  }
  __syncthreads();
  const int32_t* key = key_ + LONG_RUN;   // key[q]: position P + q
  auto same = [&](int q, int32_t k) { return P + q < nnz && key[q] == k; };   // (0 <= P + q)
  // Items: heads, and multiples of LONG_RUN inside long runs.  A run is long if two of its keys are LONG_RUN apart;
  // for a position q inside a run: if one of the pairs (q - LONG_RUN, q) ... (q, q + LONG_RUN) is equal.
  uint32_t entry[ROUNDS];
  bool few[ROUNDS], other[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int q = r * THREADS + tid;
    const bool valid = P + q < nnz;
    const int32_t k = key[q];
    const bool head = valid && (P + q == 0 || key[q - 1] != k);
    const bool ahead = same(q + LONG_RUN, k);
    const uint64_t behind = __ballot(valid && P + q >= LONG_RUN && key[q - LONG_RUN] == k);
    const bool long_inside = ahead || ((behind >> (tid & 48)) & 0xFFFFu) != 0;
    few[r] = head && !same(q + 4, k);
    other[r] = head ? !few[r] : valid && (q & (LONG_RUN - 1)) == 0 && long_inside;
    entry[r] = few[r] ? q | (((int)same(q + 1, k) + (int)same(q + 2, k) + (int)same(q + 3, k)) << BITS)
                      : q | (head ? HEAD : 0) | (!head || ahead ? PIECE : 0);
    const uint64_t mf = __ballot(few[r]), mo = __ballot(other[r]);
    if ((tid & 63) == 0) counts[r][tid >> 6] = __popcll(mf) | (__popcll(mo) << 16);
    if (!UPDATE) {
      const uint64_t mh = __ballot(head);
      if ((tid & 63) == 0) heads[q >> 6] = mh;
    }
  }
  __syncthreads();
  int sum_counts = 0;
  {
    const uint64_t lt = lanemask_lt();
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const uint64_t mf = __ballot(few[r]), mo = __ballot(other[r]);
      int before = sum_counts;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        if (w < (tid >> 6)) before += counts[r][w];
        sum_counts += counts[r][w];
      }
      if (few[r]) order[(before & 0xFFFF) + __popcll(mf & lt)] = (uint16_t)entry[r];
      if (other[r]) order[W - 1 - (before >> 16) - __popcll(mo & lt)] = (uint16_t)entry[r];
    }
  }
  __syncthreads();
  const int n_few = sum_counts & 0xFFFF, n_other = sum_counts >> 16;
  auto row_of = [&](int q) { return (int64_t)f * a.R + min(max(key[q], 0), (int)(a.R - 1)); };
  auto finish = [&](int64_t row, const RowSum& sum, const TableRow<TT, ROWWISE>& tr, int q) {
    if (UPDATE) {
      tr.update(a, row, c, lps, sum);
    } else {
      int64_t u = first_run + __popcll(heads[q >> 6] & ((1ull << (q & 63)) - 1));
      for (int i = 0; i < (q >> 6); ++i) u += __popcll(heads[i]);
      store_floats(a.G + u * a.D + c * 4, sum);
    }
  };
  // The long items first, so that the lane groups of a wavefront have items of about the same length.
  auto entry_of = [&](int i) { return i < n_other ? (int)order[W - 1 - i] : (int)order[i - n_other]; };
  for (int i = g; i < n_other + n_few; i += ngroups) {
    const int en = entry_of(i), q0 = en & POS;
    TableRow<TT, ROWWISE> tr;
    if (UPDATE && !(i < n_other && (en & PIECE))) tr.load(a, row_of(q0), c);
    int n = (en >> BITS) + 1;
    bool head = true, piece = false;
    if (i < n_other) {
      head = en & HEAD;
      piece = en & PIECE;
      n = LONG_RUN - (q0 & (LONG_RUN - 1));   // of a long run that starts here: up to the next multiple
      if (!head || !piece) {                  // the run's keys from here on, LONG_RUN at most (sorted: bisection)
        const int32_t k = key[q0];
        n = 1;
#pragma unroll
        for (int st = 8; st > 0; st >>= 1)
          if (same(q0 + n + st - 1, k)) n += st;
      }
    }
    RowSum sum = {};
    accumulate_run(dx, look + q0, n, sum);
    if (piece) {
      store_floats(piece_sum + (2 * (q0 / LONG_RUN) + (head ? 1 : 0)) * a.D + c * 4, sum);
      if (c == 0 && (head || q0 == 0)) lead[head ? 1 + q0 / LONG_RUN : 0] = (int16_t)q0;
    } else {
      finish(row_of(q0), sum, tr, q0);
    }
  }
  __syncthreads();
  for (int l = g; l < W / LONG_RUN + 1; l += ngroups) {
    const int q0 = lead[l];
    if (q0 < 0) continue;
    const int32_t k = key[q0];
    const bool out = same(W, k);
    const int64_t row = row_of(q0);
    TableRow<TT, ROWWISE> tr;
    if (UPDATE && l > 0 && !out) tr.load(a, row, c);
    RowSum sum = {};
    add_floats(sum, piece_sum + (2 * (q0 / LONG_RUN) + (l > 0 ? 1 : 0)) * a.D + c * 4);
    for (int j = q0 / LONG_RUN + 1; j < W / LONG_RUN && same(j * LONG_RUN, k); ++j) add_floats(sum, piece_sum + 2 * j * a.D + c * 4);
    if (l > 0 && !out) {
      finish(row, sum, tr, q0);
    } else {
      store_floats(a.partial + (slot * 2 + (l > 0 ? 1 : 0)) * a.D + c * 4, sum);   // (a run over two windows: the field has slots)
      if (l > 0) goes_out = 1;
    }
  }
  __syncthreads();
  if (tid == 0 && nnz > W) a.goes_out[slot] = goes_out;
}

// Runs that leave the window they start in, one wavefront each: the sum of the first window's part, then those
// of the windows the run comes into, lane groups taking turns (fixed order: repeatable bit for bit).
template <typename TT, bool ROWWISE, bool UPDATE>
__global__ __launch_bounds__(256) void seg_finish_kernel(SegArgs a, FieldPtr fp, TileBase tb, int W) {
  const int parts = SORT_TILE / W;
  const int win = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (win >= a.total_tiles * parts) return;
  int f, t;
  field_of_tile(tb, win / parts, f, t);
  const int64_t base = fp.p[f];
  const int nnz = (int)(fp.p[f + 1] - base);
  const int next = t * SORT_TILE + (win % parts + 1) * W;   // where the following window starts
  if (next >= nnz) return;
  const int64_t slot = window_slot(base) + t * parts + win % parts;
  if (!a.goes_out[slot]) return;
  const int lane = threadIdx.x & 63;
  const int32_t k = a.key[base + next - 1];
  int n = 0;   // following windows that start inside the run
  for (;;) {
    const int64_t pos = next + (int64_t)(n + lane) * W;
    const bool in = pos < nnz && a.key[base + min(pos, (int64_t)nnz - 1)] == k;
    const uint64_t out = ~__ballot(in);
    if (out) {
      n += __ffsll((unsigned long long)out) - 1;
      break;
    }
    n += 64;
  }
  const int lps = a.D >> 2, ngroups = 64 / lps;
  const int g = lane / lps, c = lane - g * lps;
  const int64_t row = (int64_t)f * a.R + min(max(k, 0), (int)(a.R - 1));
  TableRow<TT, ROWWISE> tr;
  if (UPDATE) tr.load(a, row, c);
  RowSum sum = {};
  const float* part = a.partial + slot * 2 * a.D + c * 4;
  if (g == 0) add_floats(sum, part + a.D);
#pragma unroll 4
  for (int i = 1 + g; i <= n; i += ngroups) add_floats(sum, part + (int64_t)i * 2 * a.D);
  for (int o = lps; o < 64; o <<= 1) {
#pragma unroll
    for (int e = 0; e < 4; ++e) sum.v[e] += __shfl_xor(sum.v[e], o, 64);
  }
  if (g != 0) return;
  if (UPDATE) {
    tr.update(a, row, c, lps, sum);
  } else {   // the run's head: the first position of the key in the window
    int lo = next - W, hi = next - 1;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (a.key[base + mid] < k) lo = mid + 1;
      else hi = mid;
    }
    store_floats(a.G + run_index(a, f, (int)base + lo) * a.D + c * 4, sum);
  }
}

template <typename TT, bool ROWWISE, bool UPDATE, bool MEAN, int W, int THREADS = 256>
hipError_t launch_reduce_window(const SegArgs& a, const FieldPtr& fp, const TileBase& tb, const WeightTab& wt, const DenseJob& dense, Profiler* prof,
                                hipStream_t s) {
  const unsigned parts = SORT_TILE / W;
  const int bytes = 2 * W / LONG_RUN * a.D * 4;
  const unsigned blocks = tile_grid(a.total_tiles) * parts + (unsigned)((dense.n + THREADS - 1) / THREADS);
  {
    static std::atomic<uint64_t> allowed{0};
    constexpr int ONE_FIELD = W > 512 ? 48 * 1024 : 0;   // (static LDS of the wide windows)
    const hipError_t ok = allow_lds(seg_window_kernel<TT, ROWWISE, UPDATE, MEAN, W, THREADS>, ONE_FIELD ? 2 * W / LONG_RUN * 64 * 4 : bytes,
                                    ONE_FIELD, allowed);
    if (ok != hipSuccess) return ok;
    ProfScope ps(prof, UPDATE ? KID_SPARSE_ADAGRAD : KID_SEG_REDUCE, s);
    hipLaunchKernelGGL((seg_window_kernel<TT, ROWWISE, UPDATE, MEAN, W, THREADS>), dim3(blocks), dim3(THREADS),
                       bytes, s, a, fp, tb, wt, dense);
  }
  if (W < 1024) {   // (no run leaves a window that holds its field)
    ProfScope ps(prof, KID_SEG_REDUCE_LONG, s);
    hipLaunchKernelGGL((seg_finish_kernel<TT, ROWWISE, UPDATE>), dim3((a.total_tiles * parts + 3) / 4), dim3(256), 0, s, a, fp, tb, W);
  }
  return hipGetLastError();
}

template <typename TT, bool ROWWISE, bool UPDATE, bool MEAN>
hipError_t launch_reduce_pooling(const SegArgs& a, const FieldPtr& fp, const TileBase& tb, const WeightTab& wt, const DenseJob& dense, Profiler* prof,
                                 hipStream_t s) {
  if (a.window == 2048) return launch_reduce_window<TT, ROWWISE, UPDATE, MEAN, 2048, 1024>(a, fp, tb, wt, dense, prof, s);
  if (a.window == 1024) return launch_reduce_window<TT, ROWWISE, UPDATE, MEAN, 1024, 1024>(a, fp, tb, wt, dense, prof, s);
  if (a.window == 512) return launch_reduce_window<TT, ROWWISE, UPDATE, MEAN, 512>(a, fp, tb, wt, dense, prof, s);
  return launch_reduce_window<TT, ROWWISE, UPDATE, MEAN, 256>(a, fp, tb, wt, dense, prof, s);
}

template <typename TT, bool ROWWISE, bool UPDATE>
hipError_t launch_reduce_variant(const SegArgs& a, const FieldPtr& fp, const TileBase& tb, const WeightTab& wt, const DenseJob& dense, Profiler* prof,
                                 hipStream_t s) {
  if (a.mean_pool) return launch_reduce_pooling<TT, ROWWISE, UPDATE, true>(a, fp, tb, wt, dense, prof, s);
  return launch_reduce_pooling<TT, ROWWISE, UPDATE, false>(a, fp, tb, wt, dense, prof, s);
}

}  // namespace

static hipError_t launch_sort_pass(const SortPlan& pl, const SortBuffers& sb, int pass, const FieldPtr& fp,
                            const TileBase& tb, Profiler* prof, hipStream_t s) {
  const int shift = pass * pl.radix_bits;
  const int32_t* kin = pass == 0 ? sb.ids : sb.key[(pass - 1) & 1];
  const int32_t* pin = pass == 0 ? sb.pay0 : sb.pay[(pass - 1) & 1];
  dim3 grid(tile_grid(pl.total_tiles));
  {
    ProfScope ps(prof, KID_SORT_HIST, s);
    hipLaunchKernelGGL(sort_hist_kernel<false>, grid, dim3(SORT_THREADS), 0, s, kin, sb.hist, fp, tb, pl.F, shift, pl.radix_bits, BucketPlan());
  }
  {
    ProfScope ps(prof, KID_SORT_SCAN, s);
    const int groups = std::max(1, (1 << pl.radix_bits) / SCAN_DIGITS);
    hipLaunchKernelGGL(sort_scan_kernel<false>, dim3(pl.F * groups), dim3(SCAN_THREADS), 0, s, sb.hist, sb.digit_total, tb, pl.radix_bits, BucketPlan());
  }
  {
    ProfScope ps(prof, KID_SORT_SCATTER, s);
    hipLaunchKernelGGL(sort_scatter_kernel<false>, grid, dim3(SORT_THREADS), 0, s, kin, pin, sb.key[pass & 1],
                       sb.pay[pass & 1], sb.key[0], sb.hist, sb.digit_total, fp, tb, pl.F, shift, pl.radix_bits, BucketPlan());
  }
  return hipGetLastError();
}

static int bits_of(int64_t n) {   // of the numbers below n
  int b = 0;
  while (b < 62 && (1ll << b) < n) ++b;
  return b;
}
// Whether the sort goes by buckets, and how: from as many lookups on as pay for its launches' chain.  Alone, by passes / by buckets, us: 42 M lookups
// (1.2 M rows, 3 passes) 614 / 449, 4.1 M (1 M rows, 2 passes) 93 / 91, 3.8 M (0.5 M rows) 79 / 82; a step of 4.1 M on one stream 551 / 552, of 3.8 M
// 420 / 424, of 2.2 M 383 / 387.  Beside the gather and the MLP it takes less memory traffic from them, us a step: 2.2 M 341 / 336, 3.8 M 372 / 361, 4.1 M
// 507 / 496, 42 M 2738 / 2536; 1.5 M 251 / 253.  The buckets follow a sample of the lookups, so neither how the hot rows lie matters (ids in
// order of their frequency: 3.8 M 362 / 340, 20 M 1490 / 1387) nor an order of the ids in their bags (60 fields of 4096 bags of 50 lookups, at random / ascending /
// padded with row 0: 561 / 500, 560 / 499, 551 / 485).
// Two passes cost little, most of all of short digits, and the sort by buckets is then the longer chain: it pays where it is long all the same, or
// where it saves memory traffic from a gather that takes long.  A step with the sort beside it, by passes / by buckets:
//   Digits of up to 9 bits (2^18 rows): 20 fields of 4096 samples, 256-128, 2.5 / 4.5 / 6.5 / 10 / 16 M lookups 136 / 149, 163 / 176, 198 / 212, 288 / 287,
//   451 / 408, 1024-512-256 179 / 187, 210 / 212, 247 / 249, 335 / 309, 494 / 450; three of 8192 3.2 / 6.5 M 202 / 238, 295 / 319; everything on one stream, eight
//   fields, 6.2 / 9.5 M 280 / 298, 384 / 376.  Many pooled inputs: 39 fields of 16 columns, 16384 samples, 64 in fp32, 4.5 M 247 / 258; 26 of 32, 16384, 256-128,
//   3.2 / 6.5 M 249 / 204, 300 / 249; 60 of 64, 4096, 64 in fp32, 4.5 M 395 / 308.
//   Of 10 bits: three fields of 8192 samples, 256-128, 2.1 / 3.2 / 4.5 M 183 / 196, 222 / 236, 249 / 253; six of 4096 3.2 M 181 / 192; eight of 8192 2.1 / 3.2 / 4.5 M
//   147 / 145, 175 / 160, 198 / 174.
static constexpr int64_t BUCKETS_MIN = 6000000, BUCKETS_MIN_BESIDE = 2000000, BUCKETS_MIN_SHORT = 8000000, BUCKETS_MIN_TWO = 3500000,
                         MANY_POOLED = 12000000;
static int64_t buckets_min(const SortPlan& pl) {
  const int64_t least = pl.beside ? BUCKETS_MIN_BESIDE : BUCKETS_MIN;
  if (pl.passes > 2 || (pl.beside && pl.samples * pl.width >= MANY_POOLED)) return least;
  return std::max(least, pl.radix_bits <= 9 ? BUCKETS_MIN_SHORT : BUCKETS_MIN_TWO);
}
static bool plan_buckets(const SortPlan& pl, const SortBuffers& sb, const FieldPtr& fp, BucketPlan& bp) {
  if (!sb.slots || pl.passes < 2 || fp.p[pl.F] < buckets_min(pl)) return false;
  int64_t most = 0;
  for (int f = 0; f < pl.F; ++f) most = std::max(most, fp.p[f + 1] - fp.p[f]);
  bp.sample_bits = bits_of(pl.samples);
  bp.range_bits = std::min(2 * BUCKET_BITS, 32 - bp.sample_bits);
  bp.last_row = (int32_t)(pl.rows - 1);
  bp.offsets = sb.offsets;
  bp.B = (int32_t)pl.samples;
  bp.cell_bits = std::max(bits_of(pl.rows) - bits_of(BUCKET_CELLS), 0);
  bp.rb = std::min({bits_of(std::max<int64_t>(most / 3000, 32)), pl.radix_bits, bits_of(MAX_BUCKETS)});   // (the histograms' space)
  const int64_t fixed = ((int64_t)bp.last_row >> std::max(bp.range_bits, 0)) + 1;
  if (bp.range_bits < BUCKET_BITS || 2 * fixed > (1 << bp.rb)) return false;
  // the buckets' tables and the list of the large ones
  constexpr int64_t WORDS = sizeof(FieldBuckets) / 4;
  bp.fields = reinterpret_cast<FieldBuckets*>(sb.slots);
  bp.large = sb.slots + WORDS * pl.F;
  bp.most_large = (int32_t)(fp.p[pl.F] / (BUCKET_KEYS + 1));
  return WORDS * pl.F + 1 + bp.most_large <= window_slots(fp.p[pl.F]);
}
static hipError_t launch_sort_buckets(const SortPlan& pl, const SortBuffers& sb, const FieldPtr& fp, const TileBase& tb, const BucketPlan& bp,
                                      Profiler* prof, hipStream_t s) {
  const dim3 grid(tile_grid(pl.total_tiles));
  {
    ProfScope ps(prof, KID_SORT_HIST, s);
    hipLaunchKernelGGL(sort_cuts_kernel, dim3(pl.F), dim3(SAMPLE_KEYS), 0, s, sb.ids, fp, bp);
    hipLaunchKernelGGL(sort_hist_kernel<true>, grid, dim3(SORT_THREADS), 0, s, sb.ids, sb.hist, fp, tb, pl.F, 0, bp.rb, bp);
    ps.launches(2);
  }
  {
    ProfScope ps(prof, KID_SORT_SCAN, s);
    const int groups = std::max(1, (1 << bp.rb) / SCAN_DIGITS);
    hipLaunchKernelGGL(sort_scan_kernel<true>, dim3(pl.F * groups), dim3(SCAN_THREADS), 0, s, sb.hist, sb.digit_total, tb, bp.rb, bp);
  }
  ProfScope ps(prof, KID_SORT_SCATTER, s);
  hipLaunchKernelGGL(sort_scatter_kernel<true>, grid, dim3(SORT_THREADS), 0, s, sb.ids, sb.pay0, sb.key[0], sb.pay[0], sb.key[1], sb.hist,
                     sb.digit_total, fp, tb, pl.F, 0, bp.rb, bp);
  const int large_blocks = std::min((bp.most_large + 7) / 8 * 8, 1024);   // (the others keep their XCDs)
  hipLaunchKernelGGL(sort_buckets_kernel, dim3(large_blocks + 8 * (((pl.F << bp.rb) + 7) / 8)), dim3(BUCKET_THREADS), 0, s, sb.key[1], sb.pay[1],
                     sb.key[0], sb.pay[0], sb.digit_total, fp, pl.F, large_blocks, bp);
  ps.launches(2);
  return hipGetLastError();
}

void plan_sort_pass(const SortPlan& pl, const SortBuffers& sb, const FieldPtr& fp, int pass, SortPass& sp) {
  sp.keys_in = pass == 0 ? sb.ids : sb.key[(pass - 1) & 1];
  sp.pay_in = pass == 0 ? sb.pay0 : sb.pay[(pass - 1) & 1];
  sp.keys_out = sb.key[pass & 1];
  sp.pay_out = sb.pay[pass & 1];
  sp.F = pl.F; sp.shift = pass * pl.radix_bits; sp.rb = pl.radix_bits;
  sp.fp = fp;
}
bool sort_finds_samples(const SortPlan& pl, const SortBuffers& sb, const FieldPtr& fp) {
  BucketPlan bp = {};
  return small_sort_items(pl.F, fp) == 0 && plan_buckets(pl, sb, fp, bp);
}

hipError_t launch_sort(const SortPlan& pl, const SortBuffers& sb, const FieldPtr& fp, const TileBase& tb, Profiler* prof, hipStream_t s,
                       int* sorted_buf) {
  *sorted_buf = 0;
  if (pl.total_tiles == 0) return hipSuccess;
  // One block per field as long as a field fits one: two passes over 1000 / 9000 lookups of a field take 10 / 24 us, the
  // six launches 29 / 30 and the host four times as long.
  switch (small_sort_items(pl.F, fp)) {
    case 2: return launch_sort_small_items<2>(pl, sb, fp, prof, s);
    case 4: return launch_sort_small_items<4>(pl, sb, fp, prof, s);
    case 8: return launch_sort_small_items<8>(pl, sb, fp, prof, s);
    case 16: return launch_sort_small_items<16>(pl, sb, fp, prof, s);
  }
  BucketPlan bp = {};
  if (plan_buckets(pl, sb, fp, bp)) return launch_sort_buckets(pl, sb, fp, tb, bp, prof, s);
  for (int p = 0; p < pl.passes; ++p) {
    const hipError_t e = launch_sort_pass(pl, sb, p, fp, tb, prof, s);
    if (e != hipSuccess) return e;
  }
  *sorted_buf = (pl.passes - 1) & 1;
  return hipSuccess;
}

hipError_t launch_expand_samples(const int32_t* offsets, int32_t* lookup_sample, const FieldPtr& fp, int F, int B, hipStream_t s) {
  if (B <= 0) return hipSuccess;
  hipLaunchKernelGGL(expand_samples_kernel, dim3((B + 31) / 32, F), dim3(256), 0, s, offsets, lookup_sample, fp, B);
  return hipGetLastError();
}

hipError_t launch_segments(const SegArgs& a, const FieldPtr& fp, const TileBase& tb, Profiler* prof, hipStream_t s) {
  dim3 grid(tile_grid(a.total_tiles));
  if (a.total_tiles > 0) {
    ProfScope ps(prof, KID_SEG_HEADS, s);
    hipLaunchKernelGGL(seg_heads_kernel, grid, dim3(SORT_THREADS), 0, s, a, fp, tb);
  }
  {
    ProfScope ps(prof, KID_SEG_SCAN, s);
    hipLaunchKernelGGL(seg_scan_kernel, dim3(1), dim3(1024), 0, s, a, fp, tb);
  }
  if (a.total_tiles > 0) {
    ProfScope ps(prof, KID_SEG_EMIT, s);
    hipLaunchKernelGGL(seg_emit_kernel, grid, dim3(SORT_THREADS), 0, s, a, fp, tb);
  }
  return hipGetLastError();
}

hipError_t launch_mask_pack(const int32_t* ids, const int32_t* lookup_sample, const int32_t* offsets, int64_t B, int F,
                            const FieldPtr& fp, const ShardTab& tab, int64_t* cbase, int32_t* ids_out,
                            int32_t* pay_out, hipStream_t s) {
  hipLaunchKernelGGL(mask_count_kernel, dim3(1), dim3(256), 0, s, offsets, B, F, tab, cbase);
  hipLaunchKernelGGL(mask_pack_kernel, dim3(tab.K, F, PACK_BLOCKS), dim3(PACK_THREADS), 0, s, ids, lookup_sample, offsets, B, fp, tab, cbase,
                     ids_out, pay_out);
  return hipGetLastError();
}

hipError_t launch_seg_reduce(const SegArgs& args, const FieldPtr& fp, const TileBase& tb, const ShardTab& tab, const DenseJob& dense, Profiler* prof,
                             hipStream_t s) {
  if (args.total_tiles == 0) return hipSuccess;
  SegArgs a = args;
  WeightTab wt = {};
  a.weights = 0;
  for (int k = 0; k < tab.K; ++k) {
    if (tab.len[k] == 0 || (a.weights > 0 && wt.w[a.weights - 1] == tab.w[k])) continue;
    wt.start[a.weights] = a.weights ? tab.start[k] : 0;
    wt.w[a.weights++] = tab.w[k];
  }
  a.weights = std::max(a.weights, 1);
  a.weight = wt.w[0];
  if (!a.update) return launch_reduce_variant<float, false, false>(a, fp, tb, wt, dense, prof, s);
  if (a.table_bf16) {
    if (a.rowwise) return launch_reduce_variant<bf16_t, true, true>(a, fp, tb, wt, dense, prof, s);
    return launch_reduce_variant<bf16_t, false, true>(a, fp, tb, wt, dense, prof, s);
  }
  if (a.rowwise) return launch_reduce_variant<float, true, true>(a, fp, tb, wt, dense, prof, s);
  return launch_reduce_variant<float, false, true>(a, fp, tb, wt, dense, prof, s);
}

}  // namespace antdt
