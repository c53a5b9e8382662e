// C boundary: context, workspace layout, call-order checks and the launch
// sequences of worker_step / aggregate / apply_update (see include/antdt.h).
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "common.h"
#include "sort.h"

namespace antdt {

struct ProfRec {
  hipEvent_t start, stop;
  int kid;
  int n = 1;  // launches inside the bracket
  bool closed = false;
};
struct Profiler {
  int mode = 0, sel = -1;
  std::vector<ProfRec> recs;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> pool;
  double total_ms[KID_COUNT] = {};
  int64_t launches[KID_COUNT] = {};
};

static bool prof_times(const Profiler* p, int kid) {
  return p->mode != 0 && !(p->mode == 2 && kid != p->sel) && !(p->mode == 3 && !((p->sel >> kid) & 1));
}
int prof_begin(Profiler* p, int kid, hipStream_t s) {
  if (!prof_times(p, kid)) return -1;
  ProfRec r;
  r.kid = kid;
  if (!p->pool.empty()) {
    r.start = p->pool.back().first;
    r.stop = p->pool.back().second;
    p->pool.pop_back();
  } else {
    // timing events: no cache write-back at the record (it would disturb what is being timed)
    if (hipEventCreateWithFlags(&r.start, hipEventDisableSystemFence) != hipSuccess) return -1;
    if (hipEventCreateWithFlags(&r.stop, hipEventDisableSystemFence) != hipSuccess) return -1;
  }
  (void)hipEventRecord(r.start, s);
  p->recs.push_back(r);
  return (int)p->recs.size() - 1;
}
void prof_count(Profiler* p, int idx, int launches) { p->recs[idx].n = launches; }
void prof_end(Profiler* p, int idx, hipStream_t s) {
  p->recs[idx].closed = true;
  (void)hipEventRecord(p->recs[idx].stop, s);
}

static void prof_drain(Profiler* p) {
  for (auto& r : p->recs) {
    float ms = 0.f;
    if (r.closed && hipEventSynchronize(r.stop) == hipSuccess &&
        hipEventElapsedTime(&ms, r.start, r.stop) == hipSuccess) {
      p->total_ms[r.kid] += ms;
      p->launches[r.kid] += r.n;
    }
    p->pool.push_back({r.start, r.stop});
  }
  p->recs.clear();
}

static const char* kKernelNames[KID_COUNT] = {
    "pool",        "gemm_fwd",   "gemm_dgrad",     "gemm_wgrad",  "head",
    "head_reduce", "bias_grad",  "sort_hist",      "sort_scan",   "sort_scatter",
    "seg_heads",   "seg_scan",   "seg_emit",       "seg_reduce",  "seg_reduce_long",
    "dense_agg",   "sparse_adagrad", "dense_adagrad", "adam", "transpose", "gemm_bwd", "wgrad_adagrad"};

}  // namespace antdt

using namespace antdt;

static thread_local std::string g_last_error;

namespace antdt {
void set_last_error(const std::string& msg) { g_last_error = msg; }
}

enum Stage { ST_CREATED = 0, ST_BOUND, ST_BATCH, ST_AGGREGATED };

struct antdt_ctx {
  antdt_model m;
  std::string err;
  Stage stage = ST_CREATED;
  Profiler prof;
  // derived sizes
  int L = 0, FD = 0, in0 = 0, ldx = 0;
  int act_bf16 = 0;
  size_t act_size = 4;
  int64_t P = 0, Pstride = 0;  // Pstride: P rounded up to 4 (per-shard gradient pitch)
  bool gdense_valid = false;
  int64_t w_off[ANTDT_MAX_LAYERS], b_off[ANTDT_MAX_LAYERS];
  int width[ANTDT_MAX_LAYERS + 1];  // width[l] = layer_sizes[l]
  int sort_passes = 1, radix_bits = 1;
  int64_t max_tiles_total = 0;
  bool g_valid = false;
  size_t ws_bytes = 0;
  // caller's buffers
  void* tables = nullptr;
  float* table_state = nullptr;
  float* params = nullptr;
  float* pstate = nullptr;
  // workspace carve-up
  char* x = nullptr;
  char* h[ANTDT_MAX_LAYERS] = {};
  char* dh[ANTDT_MAX_LAYERS] = {};
  float* dx = nullptr;
  float *shard_grads = nullptr, *g_dense = nullptr, *G = nullptr;
  bf16_t* wb[ANTDT_MAX_LAYERS] = {};     // bf16 W_l as [in (padded), out]: operand of the forward product and the data gradient
  bf16_t* wb0_alt = nullptr;             // second buffer for W_0: a dense update beside the launch stream writes the new
                                         // copy there while the input-gradient product may still read the old one
  float* head_part = nullptr;            // loss kernel's sums per tile of samples [tiles, ldpart]
  int64_t ldpart = 0;
  bool sums_per_sample = false;          // head_part: d loss / d logit [max_batch], losses [max_batch] (see carve)
  LossJob* loss_job = nullptr;           // [K] what it leaves to the launch that adds up the losses
  int32_t* lookup_sample = nullptr;
  int32_t *key[2] = {}, *pay[2] = {}, *tile_heads = nullptr, *ubase = nullptr, *uniq = nullptr;
  int32_t *segoff = nullptr, *pack_pay = nullptr, *segabs = nullptr, *goes_out = nullptr;
  float* partial = nullptr;
  uint32_t *hist = nullptr, *digit_total = nullptr;
  // batch
  const int32_t* ids = nullptr;
  const int32_t* offsets = nullptr;
  const float* dense = nullptr;
  const float* labels = nullptr;
  int64_t B = 0;
  FieldPtr fp;
  TileBase tb;
  int total_tiles = 0;
  // the lookups that the current aggregation coalesces: all of the batch (the four above), or
  // the packed lookups of the included shards when some are left out
  FieldPtr afp;
  TileBase atb;
  int atotal_tiles = 0;
  int64_t* cbase = nullptr;
  int32_t* vflags = nullptr;  // result of antdt_validate_batch
  // shards
  ShardTab tab;
  bool have_shards = false;
  int64_t shard_B = 0;
  bool stepped[ANTDT_MAX_SHARDS] = {};
  bool included[ANTDT_MAX_SHARDS] = {};
  double shard_scale[ANTDT_MAX_SHARDS];  // per-worker factor on the aggregation weight (1 unless set)
  bool weights_dirty = false;            // the factors changed after the weights were last formed
  // Weight gradients formed inside the dense update (bf16 products with a weight-gradient stream):
  // the worker step only leaves their operands behind and an event (ev_dh[0]) that says they are
  // complete; per-shard gradients are computed when a view asks for them.
  bool eager_wgrad = false;              // option: the worker step computes the per-shard weight gradients itself
  bool batched = false;                  // the last worker step covered all shards
  bool left_out = false;                 // the aggregation of its gradients left shards out
  bool wgrad_deferred = false;           // this worker step left the weight gradients to apply_update / the views
  bool shard_grads_done = false;         // the per-shard dense gradients of this worker step are (being) written
  bool grads_viewed[ANTDT_MAX_SHARDS] = {};  // a view handed out the shard's gradients of its last worker step
  bool captured = false;                 // a stream capture has recorded calls of this binding (see note_capture)
  bool operands_captured = false;        // ev_dh[0] was last recorded into a capture
  hipStream_t operands_stream = nullptr; // the stream it was last recorded on (only compared)
  int sorted_buf = 0;
  // side stream on which the coalescing structure of a batch is built while the MLP runs
  hipStream_t side = nullptr;
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;
  // second side stream: the weight-gradient products, which nothing needs before the dense
  // update, run there beside the sparse reduction
  hipStream_t wside = nullptr;
  hipEvent_t ev_dh[ANTDT_MAX_LAYERS + 1] = {};  // [0]: the operands of the weight gradients are complete; [L]: all before the dense update
  hipEvent_t ev_wgrad = nullptr;                // all weight gradients of the last worker step are written
  bool wgrad_pending = false;
  // The last batched step that sorted in its weight-gradient launch did not do so for nothing: an aggregation of all shards
  // followed.  Where none did (shards left out, only the gradients wanted) the next step leaves the sort to the aggregation.
  bool joined_sort_used = true;
  bool slots_apart = false;       // the loss kernel's sums and jobs end before the windows' slots (see carve)
  bool samples_missing = false;   // a batched step left the lookups' sample indices to its sort, which needs none (see sample_indices)
  bool replays_leave_samples = false;   // a capture has recorded such a step
  bool presorted = false;     // the coalescing structure of the current batch and split is built (or being built)
  bool side_pending = false;  // work is in flight on the side stream that no other stream has waited for yet
  // bound by antdt_bind_static: the workspace is the library's static device buffer and every
  // kernel goes to the caller's stream (no library-owned stream or event exists or is created)
  bool static_bound = false;
  bool no_streams = false;   // option: everything on the caller's stream although the library's streams exist
  int static_device = -1;
};

// The library's own streams, or none when the context works on the caller's stream only.  Going to another stream
// and back costs the host about 25 us (the waits on events), so it has to hide that much GPU work, and the step has to be one whose
// kernels take longer than the host's calls.
//   Sort: from 100 000 lookups (26 fields, 1024-512-256, dense update on the launch stream, sort on the side or not, us per step:
//   22 000 / 36 000 / 52 000 / 82 000 / 115 000 / 164 000 / 273 000 lookups 80 / 73, 83 / 79, 85 / 82, 89 / 85, 90 / 91, 93 / 99, 101 / 115;
//   3200-1024-512 with D = 64 at 70 000, dense update on the side: 100 / 90), and below where a long field makes it long (more than 4096
//   lookups: 14 us and more in one block) and the MLP hides it: bf16 models from 2e8 samples x parameters (four fields; 1000 samples,
//   1024-512-256, 42 000 lookups 88 / 102; 4096, 256-128, 49 000 89 / 98; 12 000, 512-256, 48 000 150 / 164; less: 2000, 256-128, 84 000 99 / 90),
//   fp32 models from 8192 samples (256-128, 48 000 lookups 173 / 190) or, where the sort has no place in the weight-gradient launch, from 1e8
//   (2000, 512-256, 84 000 115 / 130, 256-128 101 / 102; with a place: 4096, 256-128, 49 000 109 / 102).
//   Dense update beside the sparse one: where there are many lookups or many weights (26 fields, 1024-512-256, beside or after:
//   164 000 / 273 000 / 355 000 / 546 000 / 682 000 / 874 000 lookups 111 / 93, 112 / 101, 115 / 109, 134 / 126, 140 / 144, 158 / 168;
//   3840-1024-512 at 50 000: 102 / 122).  With 100 000 lookups and more also where the kernels take long and those beside each other get on:
//   the weight gradients formed in pieces (see cut_ranges; 8192 samples, 1024-512-256, 213 000 lookups 187 / 199; 12 000, 512-256 with D = 64,
//   312 000 254 / 280), or by few blocks over at least 8192 samples (four fields, 12 000, 512-256, 504 000 163 / 180; 26 of D = 16, 256-128,
//   8192 105 / 114, 512-256, 9000 134 / 149), or by those of a large model over no more than 5000 (26 fields, 4096, 1024-512-256, 106 000
//   140 / 146; 39 of D = 16, 5000 158 / 164).  Otherwise the blocks hold the compute units that the input gradient waits for (26 fields,
//   512-256, 9000, 351 000 199 / 160; D = 64, 8192, 213 000 229 / 190).
//   After one worker step per shard not: six workers, 1024-512-256, with
//   300 000 / 500 000 / 700 000 / 1.6 M / 4.1 M lookups 367 / 322, 398 / 345, 424 / 376, 539 / 500, 838 / 816 us; eight, 3840-1024-512
//   with 0.9 / 3.8 / 12 M 550 / 505, 846 / 845, 1504 / 1497 us.  Unless shards were left out: the host has then waited for the
//   stream and is no longer ahead of it (one of six workers left out, 700 000 / 1.6 M / 4.1 M lookups 374 / 380, 473 / 482,
//   804 / 829 us, fewer lookups alike; one of eight with 0.9 / 3.8 M 486 / 508, 778 / 822).  fp32 models never (176 / 171 us
//   at 430 000 lookups).
static bool sort_joins(antdt_ctx* c);
static bool wgrad_in_pieces(const antdt_ctx* c);
static hipStream_t side_stream(antdt_ctx* c) {
  if (c->static_bound || c->no_streams) return nullptr;
  const int64_t lookups = c->fp.p[c->m.num_fields];
  bool enough = lookups >= 100000;
  if (!enough && lookups >= 16384) {
    int64_t most = 0;
    for (int f = 0; f < c->m.num_fields; ++f) most = std::max(most, c->fp.p[f + 1] - c->fp.p[f]);
    const double work = (double)c->B * (double)c->P;
    enough = most > 4096 && (c->act_bf16 ? work >= 2e8 : c->B >= 8192 || (work >= 1e8 && !sort_joins(c)));
  }
  return enough ? c->side : nullptr;
}
static hipStream_t wgrad_stream(const antdt_ctx* c) {
  if (c->static_bound || c->no_streams || !c->act_bf16 || !(c->batched || c->left_out)) return nullptr;
  const int64_t lookups = c->fp.p[c->m.num_fields];
  bool enough = lookups >= 600000 || c->P >= 2000000;
  if (!enough && c->batched && lookups >= 100000 && c->B >= 3000) {
    int64_t blocks = 0;
    for (int l = 0; l + 1 < c->L; ++l) blocks += (int64_t)((c->width[l] + 63) / 64) * ((c->width[l + 1] + 63) / 64);
    enough = (c->B <= 5000 && c->P >= 1250000) || (c->B >= 8192 && blocks <= 100) || wgrad_in_pieces(c);
  }
  return enough ? c->wside : nullptr;
}

// A captured call is replayed behind the library's back, with the addresses it was captured with: from the first one on
// (until the context is bound again) W_0's copy keeps its place, and per-shard gradients that a view computed are not
// taken for those of the last replay.
static bool note_capture(antdt_ctx* c, hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  const bool capturing = hipStreamIsCapturing(s, &st) == hipSuccess && st != hipStreamCaptureStatusNone;
  c->captured = c->captured || capturing;
  return capturing;
}

static int fail(antdt_ctx* c, int code, const std::string& msg) {
  if (c) c->err = msg;
  g_last_error = msg;
  return code;
}
#define HIP_TRY(c, expr)                                                                   \
  do {                                                                                     \
    hipError_t e__ = (expr);                                                               \
    if (e__ != hipSuccess)                                                                 \
      return fail(c, ANTDT_HIP_ERROR, std::string(#expr) + ": " + hipGetErrorString(e__)); \
  } while (0)

// Events that order the library's own streams on one device.  Without the system-scope fence a
// record does not write the caches back for the host or other devices (work on this device
// still sees everything the recorded work wrote): on the launch stream that fence costs about
// 2 us per record and evicts what the next kernel would have found in L2.
static constexpr unsigned SYNC_EVENT_FLAGS = hipEventDisableTiming | hipEventDisableSystemFence;

static inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
// Whether one of two classes is being timed: launches that would do the work of both are then made apart.
static inline bool prof_apart(const Profiler* p, int a, int b) { return p && (prof_times(p, a) || prof_times(p, b)); }
static inline Profiler* prof_of(antdt_ctx* c) { return c->prof.mode ? &c->prof : nullptr; }

static bool is_pow2(int64_t v) { return v > 0 && (v & (v - 1)) == 0; }

// Lays the workspace out; with base == nullptr only the size is computed.
static size_t carve(antdt_ctx* c, char* base) {
  size_t off = 0;
  auto take = [&](size_t bytes) -> char* {
    char* p = base ? base + off : nullptr;
    off = align_up(off + bytes, 256);
    return p;
  };
  const antdt_model& m = c->m;
  const int64_t Bm = m.max_batch, K = m.max_shards, N = m.max_nnz;
  c->x = take((size_t)Bm * c->ldx * c->act_size);
  for (int l = 1; l < c->L; ++l) {
    c->h[l] = take((size_t)Bm * c->width[l] * c->act_size);
    // (the loss kernel is the last to read the last activation, and leaves the gradient in its place: fp32 models need no
    // more than before these sums existed; bf16 models keep both, a place of its own costs them nothing)
    if (l == c->L - 1 && !c->act_bf16) c->dh[l] = c->h[l];
    else c->dh[l] = take((size_t)Bm * c->width[l] * c->act_size);
  }
  c->dx = (float*)take((size_t)Bm * c->FD * 4);
  c->shard_grads = (float*)take((size_t)K * c->Pstride * 4);
  if (c->act_bf16) {
    for (int l = 0; l + 1 < c->L; ++l) {
      const int64_t rows = l == 0 ? c->ldx : c->width[l];
      c->wb[l] = (bf16_t*)take((size_t)rows * c->width[l + 1] * 2);
      if (l == 0) c->wb0_alt = (bf16_t*)take((size_t)rows * c->width[l + 1] * 2);
    }
  }
  c->lookup_sample = (int32_t*)take((size_t)N * 4);
  for (int i = 0; i < 2; ++i) {
    c->key[i] = (int32_t*)take((size_t)N * 4);
    c->pay[i] = (int32_t*)take((size_t)N * 4);
  }
  c->hist = (uint32_t*)take((size_t)(c->max_tiles_total << c->radix_bits) * 4);
  c->digit_total = (uint32_t*)take((size_t)(m.num_fields << c->radix_bits) * 4);
  const bool share = !c->act_bf16 && c->L == 1;   // (see below)
  const size_t jobs = (size_t)K * sizeof(LossJob), counts = (size_t)(ANTDT_MAX_FIELDS + 1) * 8;
  char* small = take(counts + 8 + (share ? 0 : jobs));
  c->cbase = (int64_t*)small;
  c->vflags = (int32_t*)(small ? small + counts : nullptr);
  c->loss_job = (LossJob*)(small ? small + counts + 8 : nullptr);
  // The loss kernel's sums and jobs.  Of an fp32 model without a hidden layer they share memory with what only an
  // aggregation and what follows it use: the worker step itself reads them last (in bf16 models apply_update does).  What else runs
  // beside a worker step keeps away from there (see slots_apart).
  // Where that is too small for sums over tiles (few lookups, many dense features), or where those of a bf16 model
  // without a hidden layer would take more than its inputs (most shards hold one sample), they are kept per sample instead,
  // and the last layer's gradient is added up from the samples.
  const size_t tiles = (size_t)std::min(Bm, Bm / HEAD_TILE + K);   // (every tile has a sample)
  const size_t shared = off;
  if (share) c->loss_job = (LossJob*)take(jobs);
  const size_t sums = off;
  c->sums_per_sample = c->act_bf16 && c->L == 1 && tiles * c->ldpart * 4 > (size_t)Bm * c->ldx * 2;
  c->head_part = (float*)take(c->sums_per_sample ? (size_t)Bm * 8 : tiles * c->ldpart * 4);
  size_t behind = off;
  if (share) off = shared;
  c->g_dense = (float*)take((size_t)c->P * 4);
  c->tile_heads = (int32_t*)take((size_t)(c->max_tiles_total + 1) * 4);
  c->ubase = (int32_t*)take((size_t)(m.num_fields + 1) * 4);
  c->uniq = (int32_t*)take((size_t)N * 4);
  c->segoff = (int32_t*)take((size_t)(N + m.num_fields + 1) * 4);
  c->pack_pay = (int32_t*)take((size_t)N * 4);
  c->segabs = (int32_t*)take((size_t)(N + 1) * 4);
  c->partial = (float*)take((size_t)window_slots(N) * 2 * m.dim * 4);
  c->G = (float*)take((size_t)N * m.dim * 4);
  // (last: a batched step's sort has its tables there, beside the worker step, which the sums above seldom reach)
  const size_t slots = off;
  c->goes_out = (int32_t*)take((size_t)window_slots(N) * 4);
  if (share && behind > off) {
    c->sums_per_sample = true;
    behind = align_up(sums + (size_t)Bm * 8, 256);
  }
  c->slots_apart = !share || behind <= slots;
  return std::max(off, behind);
}

// ----------------------------------------------------------------------------------------
// Scratch of antdt_bind_static, the entry point for callers that cannot allocate.  The array's
// name is only a host-side handle; kernels and copies get the address that
// hipGetSymbolAddress reports for the device that is current, looked up once per device (each
// device holds its own copy of the array at its own address).
static __device__ __align__(256) unsigned char scratch[ANTDT_STATIC_SCRATCH_BYTES];

static constexpr int MAX_DEVICES = 64;
static std::mutex g_scratch_mutex;
static void* g_scratch_ptr[MAX_DEVICES] = {};
static antdt_ctx* g_scratch_owner[MAX_DEVICES] = {};  // context whose workspace the buffer currently is

// A context that gives the static buffer up (rebound to a caller's workspace, or destroyed).
static void release_static(antdt_ctx* c) {
  if (!c->static_bound) return;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (c->static_device >= 0 && c->static_device < MAX_DEVICES && g_scratch_owner[c->static_device] == c)
    g_scratch_owner[c->static_device] = nullptr;
  c->static_bound = false;
  c->static_device = -1;
}

// Makes `s` wait for whatever the side stream is still doing (it writes the sort buffers and reads the sample index of every
// lookup): before anything rebuilds or overwrites those.  Whether that structure is still valid is a separate question.
static int join_side(antdt_ctx* c, hipStream_t s) {
  if (c->side_pending) {
    HIP_TRY(c, hipStreamWaitEvent(s, c->ev_join, 0));
    c->side_pending = false;
  }
  return ANTDT_OK;
}

// Makes `s` wait for the weight-gradient products of the last worker step (they run on their
// own stream): before anything reads the per-shard dense gradients or overwrites their operands.
static int join_wgrad(antdt_ctx* c, hipStream_t s) {
  if (c->wgrad_pending) {
    HIP_TRY(c, hipStreamWaitEvent(s, c->ev_wgrad, 0));
    c->wgrad_pending = false;
  }
  return ANTDT_OK;
}

extern "C" {

const char* antdt_last_error(const antdt_ctx* ctx) { return ctx ? ctx->err.c_str() : g_last_error.c_str(); }

const char* antdt_kernel_name(int32_t kid) { return (kid >= 0 && kid < KID_COUNT) ? kKernelNames[kid] : nullptr; }

int antdt_create(const antdt_model* model, antdt_ctx** out) {
  if (!model || !out) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_create: null argument");
  const antdt_model& m = *model;
  auto bad = [&](const char* what) { return fail(nullptr, ANTDT_INVALID_ARG, std::string("antdt_create: ") + what); };
  if (m.num_fields < 1 || m.num_fields > ANTDT_MAX_FIELDS) return bad("num_fields out of range");
  if (m.rows_per_field < 1 || m.rows_per_field >= (1ll << 31)) return bad("rows_per_field out of range");
  if (m.table_dtype != ANTDT_F32 && m.table_dtype != ANTDT_BF16) return bad("table_dtype");
  if (m.gemm_dtype != ANTDT_F32 && m.gemm_dtype != ANTDT_BF16) return bad("gemm_dtype");
  if (m.adagrad_state != ANTDT_STATE_ELEMENTWISE && m.adagrad_state != ANTDT_STATE_ROWWISE) return bad("adagrad_state");
  const int64_t row_bytes = (int64_t)m.dim * (m.table_dtype == ANTDT_BF16 ? 2 : 4);
  if (m.dim < 4 || m.dim > 256 || row_bytes < 16 || !is_pow2(row_bytes))
    return bad("dim: 4..256, a power of two (a row's gradient is summed by at most one wavefront, four columns per lane)");
  if (m.num_dense < 0) return bad("num_dense");
  if (m.num_layers < 1 || m.num_layers > ANTDT_MAX_LAYERS) return bad("num_layers out of range");
  if ((int64_t)m.layer_sizes[0] != (int64_t)m.num_fields * m.dim + m.num_dense) return bad("layer_sizes[0] != num_fields*dim + num_dense");
  if (m.layer_sizes[m.num_layers] != 1) return bad("last layer must have one output");
  for (int l = 1; l < m.num_layers; ++l) {
    if (m.layer_sizes[l] < 1) return bad("layer size");
    if (m.gemm_dtype == ANTDT_BF16 && m.layer_sizes[l] % 8) return bad("bf16 GEMMs need hidden widths that are multiples of 8");
  }
  if (m.max_shards < 1 || m.max_shards > ANTDT_MAX_SHARDS) return bad("max_shards out of range");
  if (m.max_batch < 1 || m.max_batch >= (1ll << 31)) return bad("max_batch out of range");
  if (m.max_nnz < 0 || m.max_nnz >= (1ll << 31) - 4096) return bad("max_nnz out of range");
  if (m.pooling != ANTDT_POOL_SUM && m.pooling != ANTDT_POOL_MEAN) return bad("pooling: ANTDT_POOL_SUM or ANTDT_POOL_MEAN");
  if (!(m.lr >= 0.f) || !(m.eps > 0.f)) return bad("lr must be >= 0 and eps > 0");

  antdt_ctx* c = new antdt_ctx();
  c->m = m;
  for (int k = 0; k < ANTDT_MAX_SHARDS; ++k) c->shard_scale[k] = 1.0;
  c->L = m.num_layers;
  c->FD = m.num_fields * m.dim;
  c->in0 = m.layer_sizes[0];
  c->ldx = (c->in0 + 7) / 8 * 8;
  c->act_bf16 = m.gemm_dtype == ANTDT_BF16;
  c->act_size = c->act_bf16 ? 2 : 4;
  c->ldpart = (int64_t)m.layer_sizes[c->L - 1] + 2;
  int64_t off = 0;
  for (int l = 0; l <= c->L; ++l) c->width[l] = m.layer_sizes[l];
  for (int l = 0; l < c->L; ++l) {
    c->w_off[l] = off;
    off += (int64_t)c->width[l] * c->width[l + 1];
    c->b_off[l] = off;
    off += c->width[l + 1];
  }
  c->P = off;
  c->Pstride = (off + 3) / 4 * 4;
  int bits = 1;
  while ((1ll << bits) < m.rows_per_field) ++bits;
  c->sort_passes = (bits + 9) / 10;
  c->radix_bits = (bits + c->sort_passes - 1) / c->sort_passes;
  c->max_tiles_total = m.max_nnz / ANTDT_SORT_TILE + m.num_fields + 1;
  c->ws_bytes = carve(c, nullptr);
  memset(&c->tab, 0, sizeof(c->tab));
  *out = c;
  return ANTDT_OK;
}

int antdt_destroy(antdt_ctx* ctx) {
  if (!ctx) return ANTDT_OK;
  release_static(ctx);
  prof_drain(&ctx->prof);
  if (ctx->side) {
    (void)hipStreamSynchronize(ctx->side);
    (void)hipStreamDestroy(ctx->side);
    (void)hipEventDestroy(ctx->ev_fork);
    (void)hipEventDestroy(ctx->ev_join);
  }
  if (ctx->wside) {
    (void)hipStreamSynchronize(ctx->wside);
    (void)hipStreamDestroy(ctx->wside);
    (void)hipEventDestroy(ctx->ev_wgrad);
    for (auto& e : ctx->ev_dh)
      if (e) (void)hipEventDestroy(e);
  }
  for (auto& e : ctx->prof.pool) {
    (void)hipEventDestroy(e.first);
    (void)hipEventDestroy(e.second);
  }
  delete ctx;
  return ANTDT_OK;
}

int antdt_workspace_bytes(const antdt_ctx* ctx, size_t* bytes) {
  if (!ctx || !bytes) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_workspace_bytes: null argument");
  *bytes = ctx->ws_bytes;
  return ANTDT_OK;
}

// What a fresh workspace has to hold before the first iteration.
static int init_workspace(antdt_ctx* c, hipStream_t s) {
  if (!c->act_bf16) return ANTDT_OK;
  for (int l = 0; l + 1 < c->L; ++l) {
    CastArgs a;
    a.src = c->params + c->w_off[l];
    a.dst = c->wb[l];
    a.n_src = (int64_t)c->width[l] * c->width[l + 1];
    a.n_dst = (int64_t)(l == 0 ? c->ldx : c->width[l]) * c->width[l + 1];
    HIP_TRY(c, launch_cast_bf16(a, s));
    if (l == 0) {  // (its padding rows must be zero as well)
      a.dst = c->wb0_alt;
      HIP_TRY(c, launch_cast_bf16(a, s));
    }
  }
  return ANTDT_OK;
}

int antdt_bind(antdt_ctx* c, void* tables, float* table_state, float* mlp_params, float* mlp_state,
               void* workspace, size_t workspace_bytes, void* stream) {
  if (!c) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_bind: null context");
  if (!tables || !table_state || !mlp_params || !mlp_state || !workspace)
    return fail(c, ANTDT_INVALID_ARG, "antdt_bind: null buffer");
  if (workspace_bytes < c->ws_bytes) return fail(c, ANTDT_WORKSPACE_TOO_SMALL, "antdt_bind: workspace too small");
  if (((uintptr_t)workspace & 255) || ((uintptr_t)tables & 15) || ((uintptr_t)table_state & 15) ||
      ((uintptr_t)mlp_params & 15) || ((uintptr_t)mlp_state & 15))
    return fail(c, ANTDT_INVALID_ARG, "antdt_bind: misaligned buffer (workspace 256 B, others 16 B)");
  release_static(c);
  c->tables = tables;
  c->table_state = table_state;
  c->params = mlp_params;
  c->pstate = mlp_state;
  carve(c, (char*)workspace);
  c->captured = false;
  c->replays_leave_samples = false;
  memset(c->grads_viewed, 0, sizeof(c->grads_viewed));
  if (!c->side) {
    HIP_TRY(c, hipStreamCreateWithFlags(&c->side, hipStreamNonBlocking));
    HIP_TRY(c, hipEventCreateWithFlags(&c->ev_fork, SYNC_EVENT_FLAGS));
    HIP_TRY(c, hipEventCreateWithFlags(&c->ev_join, SYNC_EVENT_FLAGS));
  }
  if (!c->wside) {
    HIP_TRY(c, hipStreamCreateWithFlags(&c->wside, hipStreamNonBlocking));
    HIP_TRY(c, hipEventCreateWithFlags(&c->ev_wgrad, SYNC_EVENT_FLAGS));
    for (int l = 0; l <= c->L; ++l) HIP_TRY(c, hipEventCreateWithFlags(&c->ev_dh[l], SYNC_EVENT_FLAGS));
  }
  c->stage = ST_BOUND;
  return init_workspace(c, (hipStream_t)stream);
}

int antdt_bind_static(antdt_ctx* c, void* tables, float* table_state, float* mlp_params, float* mlp_state,
                      void* stream) {
  if (!c) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_bind_static: null context");
  if (!tables || !table_state || !mlp_params || !mlp_state)
    return fail(c, ANTDT_INVALID_ARG, "antdt_bind_static: null buffer");
  if (((uintptr_t)tables & 15) || ((uintptr_t)table_state & 15) || ((uintptr_t)mlp_params & 15) ||
      ((uintptr_t)mlp_state & 15))
    return fail(c, ANTDT_INVALID_ARG, "antdt_bind_static: misaligned buffer (16 B)");
  if (c->ws_bytes > (size_t)ANTDT_STATIC_SCRATCH_BYTES)
    return fail(c, ANTDT_WORKSPACE_TOO_SMALL,
                "antdt_bind_static: the model needs " + std::to_string(c->ws_bytes) +
                    " bytes of scratch, the library's static buffer holds " +
                    std::to_string((size_t)ANTDT_STATIC_SCRATCH_BYTES) + " (use antdt_bind with a workspace)");
  int dev = -1;
  HIP_TRY(c, hipGetDevice(&dev));
  if (dev < 0 || dev >= MAX_DEVICES) return fail(c, ANTDT_UNSUPPORTED, "antdt_bind_static: device index out of range");
  void* base = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {  // once per device, with that device current
      void* p = nullptr;
      const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (e != hipSuccess || !p)
        return fail(c, ANTDT_HIP_ERROR, std::string("antdt_bind_static: hipGetSymbolAddress: ") + hipGetErrorString(e));
      g_scratch_ptr[dev] = p;
    }
    base = g_scratch_ptr[dev];
    // The buffer serves one context at a time: the context that held it must be bound again
    // before its next iteration (its calls fail with BAD_STATE until then).
    antdt_ctx* prev = g_scratch_owner[dev];
    if (prev && prev != c) {
      prev->stage = ST_CREATED;
      prev->static_bound = false;
      prev->static_device = -1;
    }
    g_scratch_owner[dev] = c;
  }
  if (((uintptr_t)base & 255)) return fail(c, ANTDT_HIP_ERROR, "antdt_bind_static: static buffer is not 256-byte aligned");
  // A context that was bound with antdt_bind before may still have work on its own streams.
  if (c->side) HIP_TRY(c, hipStreamSynchronize(c->side));
  if (c->wside) HIP_TRY(c, hipStreamSynchronize(c->wside));
  c->side_pending = false;
  c->wgrad_pending = false;
  c->presorted = false;
  c->static_bound = true;
  c->static_device = dev;
  c->tables = tables;
  c->table_state = table_state;
  c->params = mlp_params;
  c->pstate = mlp_state;
  carve(c, (char*)base);
  c->captured = false;
  c->replays_leave_samples = false;
  memset(c->grads_viewed, 0, sizeof(c->grads_viewed));
  c->stage = ST_BOUND;
  c->have_shards = false;
  return init_workspace(c, (hipStream_t)stream);
}

// Tile decomposition of per-field lookup ranges.
static void plan_tiles(int F, const FieldPtr& fp, TileBase& tb, int& total_tiles) {
  memset(&tb, 0, sizeof(tb));
  for (int f = 0; f < F; ++f)
    tb.t[f + 1] = tb.t[f] + (int)((fp.p[f + 1] - fp.p[f] + ANTDT_SORT_TILE - 1) / ANTDT_SORT_TILE);
  for (int f = F + 1; f <= ANTDT_MAX_FIELDS; ++f) tb.t[f] = tb.t[F];
  total_tiles = tb.t[F];
}

static void coalesce_whole_batch(antdt_ctx* c) {
  c->afp = c->fp;
  c->atb = c->tb;
  c->atotal_tiles = c->total_tiles;
}

int antdt_set_batch(antdt_ctx* c, const int32_t* ids, const int64_t* field_ptr, const int32_t* offsets,
                    const float* dense, const float* labels, int64_t B, void* stream) {
  if (!c) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_set_batch: null context");
  if (c->stage < ST_BOUND) return fail(c, ANTDT_BAD_STATE, "antdt_set_batch: call antdt_bind first");
  if (B < 0 || B > c->m.max_batch) return fail(c, ANTDT_INVALID_ARG, "antdt_set_batch: B out of range");
  if (!field_ptr || !offsets || (B > 0 && (!labels || (c->m.num_dense > 0 && !dense))))
    return fail(c, ANTDT_INVALID_ARG, "antdt_set_batch: null buffer");
  const int F = c->m.num_fields;
  if (field_ptr[0] != 0) return fail(c, ANTDT_INVALID_ARG, "antdt_set_batch: field_ptr[0] != 0");
  for (int f = 0; f < F; ++f)
    if (field_ptr[f + 1] < field_ptr[f]) return fail(c, ANTDT_INVALID_ARG, "antdt_set_batch: field_ptr decreases");
  if (field_ptr[F] > c->m.max_nnz) return fail(c, ANTDT_INVALID_ARG, "antdt_set_batch: more lookups than max_nnz");
  if (field_ptr[F] > 0 && !ids) return fail(c, ANTDT_INVALID_ARG, "antdt_set_batch: null ids");
  memset(&c->fp, 0, sizeof(c->fp));
  for (int f = 0; f < F; ++f) c->fp.p[f + 1] = field_ptr[f + 1];
  for (int f = F + 1; f <= ANTDT_MAX_FIELDS; ++f) c->fp.p[f] = c->fp.p[F];
  plan_tiles(F, c->fp, c->tb, c->total_tiles);
  coalesce_whole_batch(c);
  c->ids = ids;
  c->offsets = offsets;
  c->dense = dense;
  c->labels = labels;
  c->B = B;
  c->stage = ST_BATCH;
  {
    const int rc = join_side(c, (hipStream_t)stream);
    if (rc) return rc;
  }
  c->presorted = false;
  c->samples_missing = false;
  memset(c->stepped, 0, sizeof(c->stepped));
  return ANTDT_OK;
}

int antdt_validate_batch(antdt_ctx* c, void* stream) {
  if (!c) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_validate_batch: null context");
  if (c->stage < ST_BATCH) return fail(c, ANTDT_BAD_STATE, "antdt_validate_batch: call antdt_set_batch first");
  hipStream_t s = (hipStream_t)stream;
  HIP_TRY(c, launch_validate(c->ids, c->offsets, c->fp, c->B, c->m.rows_per_field, c->m.num_fields, c->vflags, s));
  int32_t fl[2] = {0, 0};
  HIP_TRY(c, hipMemcpyAsync(fl, c->vflags, sizeof(fl), hipMemcpyDeviceToHost, s));
  HIP_TRY(c, hipStreamSynchronize(s));
  if (fl[0] == 0) return ANTDT_OK;
  std::string what = "antdt_validate_batch: field " + std::to_string(fl[1] - 1) + " (lowest offending):";
  if (fl[0] & 1) what += " an id outside [0, rows_per_field)";
  if (fl[0] & 2) what += std::string(fl[0] & 1 ? ";" : "") + " offsets that do not start at 0, decrease, or do not end at the field's lookup count";
  return fail(c, ANTDT_INVALID_ARG, what);
}

int antdt_assign_shard(antdt_ctx* c, int64_t B, int32_t K, const int64_t* sizes, const double* speed,
                       int64_t* start_out, int64_t* len_out) {
  if (!c) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_assign_shard: null context");
  if (K < 1 || K > c->m.max_shards) return fail(c, ANTDT_INVALID_ARG, "antdt_assign_shard: K out of range");
  if (B < 0 || B > c->m.max_batch) return fail(c, ANTDT_INVALID_ARG, "antdt_assign_shard: B out of range");
  std::vector<int64_t> len(K, 0);
  if (sizes) {
    int64_t tot = 0;
    for (int k = 0; k < K; ++k) {
      if (sizes[k] < 0) return fail(c, ANTDT_INVALID_ARG, "antdt_assign_shard: negative shard size");
      len[k] = sizes[k];
      tot += sizes[k];
    }
    if (tot != B) return fail(c, ANTDT_INVALID_ARG, "antdt_assign_shard: sizes do not sum to B");
  } else if (speed) {
    // Eq. 3: minimise z subject to z >= B_k / v_k, sum_k B_k = B.  Every worker can take
    // floor(B v_k / sum v) - 1 samples without exceeding the continuous optimum B / sum v;
    // the rest is handed out one sample at a time to the worker whose load after the
    // addition is smallest (ties: lowest k), which is optimal for a max of linear costs.
    long double tot_v = 0;
    for (int k = 0; k < K; ++k) {
      if (!(speed[k] > 0.0) || !isfinite(speed[k])) return fail(c, ANTDT_INVALID_ARG, "antdt_assign_shard: speed must be finite and > 0");
      tot_v += speed[k];
    }
    int64_t given = 0;
    for (int k = 0; k < K; ++k) {
      int64_t b = (int64_t)floorl((long double)B * speed[k] / tot_v) - 1;
      if (b < 0) b = 0;
      len[k] = b;
      given += b;
    }
    for (; given < B; ++given) {
      int best = 0;
      for (int k = 1; k < K; ++k) {
        // (len[k]+1)/v_k < (len[best]+1)/v_best, cross-multiplied
        const long double lhs = (long double)(len[k] + 1) * speed[best];
        const long double rhs = (long double)(len[best] + 1) * speed[k];
        if (lhs < rhs) best = k;
      }
      ++len[best];
    }
  } else {
    const int64_t q = B / K, r = B % K;
    for (int k = 0; k < K; ++k) len[k] = q + (k < r ? 1 : 0);
  }
  memset(&c->tab, 0, sizeof(c->tab));
  c->tab.K = K;
  int64_t s = 0;
  for (int k = 0; k < K; ++k) {
    c->tab.start[k] = (int32_t)s;
    c->tab.len[k] = (int32_t)len[k];
    if (start_out) start_out[k] = s;
    if (len_out) len_out[k] = len[k];
    s += len[k];
  }
  for (int k = K; k < ANTDT_MAX_SHARDS; ++k) c->tab.start[k] = (int32_t)s;
  c->have_shards = true;
  c->presorted = false;
  c->shard_B = B;
  memset(c->stepped, 0, sizeof(c->stepped));
  memset(c->grads_viewed, 0, sizeof(c->grads_viewed));
  if (c->stage == ST_AGGREGATED) c->stage = ST_BATCH;
  return ANTDT_OK;
}

static void fill_seg_args(antdt_ctx* c, SegArgs& a) {
  const antdt_model& m = c->m;
  memset(&a, 0, sizeof(a));
  a.key = c->key[c->sorted_buf]; a.pay = c->pay[c->sorted_buf];
  a.tile_heads = c->tile_heads; a.ubase = c->ubase; a.uniq = c->uniq; a.segabs = c->segabs; a.segoff = c->segoff;
  a.goes_out = c->goes_out; a.partial = c->partial;
  a.G = c->G; a.dx = c->dx; a.lddx = c->FD;
  a.offsets = c->offsets; a.mean_pool = m.pooling == ANTDT_POOL_MEAN;
  a.F = m.num_fields; a.D = m.dim; a.B = (int32_t)c->B; a.total_tiles = c->atotal_tiles;
  // 512 lookups per block need half the blocks but, with LDS growing with D, leave fewer of them on a compute unit.  The
  // launch, 512 against 256: 4.3 M lookups with D = 32 160 us against 172, with D = 64 3.8 M 173 against 143, 42 M 1486 against
  // 1239; 1.1 M with D = 32 50 against 45.  A step of 26 fields, 1024-512-256: D = 32 with 1.5 / 2.8 / 4.2 / 7 M lookups
  // 243 / 242, 410 / 420, 547 / 558, 865 / 894; D = 16 with 1.5 / 2.8 / 5 M 212 / 214, 354 / 361, 570 / 605; D = 8 with 2.8 / 7 M
  // 309 / 309, 647 / 659.
  a.window = c->afp.p[m.num_fields] >= (4 << 20) && m.dim <= 32 ? 512 : 256;
  // Fields that fit one window (1024 or 2048 lookups, 1024 threads) take one each: no run goes on in another one, and the launch
  // that adds those up is not needed.  A step, us, windows of 256 / of the whole field: 26 fields of 500 / 1000 / 1400 / 2000 lookups
  // 74.1 / 68.8, 80.4 / 73.7, 85.6 / 82.9, 86.9 / 87.0; 8 fields of 640 (fp32) 53.8 / 50.1; 26 of 1900 with D = 64 86.3 / 86.3.  (Wider
  // rows: the pieces' sums no longer fit LDS.)
  int64_t most = 0;
  for (int f = 0; f < m.num_fields; ++f) most = std::max(most, c->afp.p[f + 1] - c->afp.p[f]);
  if (m.dim <= 64 && most <= 2048) a.window = most <= 1024 ? 1024 : 2048;
  a.tables = c->tables; a.state = c->table_state; a.R = m.rows_per_field; a.lr = m.lr; a.eps = m.eps; a.inv_dim = 1.0f / (float)m.dim;
  a.table_bf16 = m.table_dtype == ANTDT_BF16; a.rowwise = m.adagrad_state == ANTDT_STATE_ROWWISE;
}

static void set_weights(antdt_ctx* c) {
  const int K = c->tab.K;
  int64_t tot = 0;
  for (int k = 0; k < K; ++k)
    if (c->included[k]) tot += c->tab.len[k];
  for (int k = 0; k < ANTDT_MAX_SHARDS; ++k)
    c->tab.w[k] = (k < K && c->included[k] && tot > 0)
                      ? (float)(c->shard_scale[k] * ((double)c->tab.len[k] / (double)tot)) : 0.0f;
  c->weights_dirty = false;
}

// beside: the sort runs beside the worker step (on the side stream).
static void fill_sort(antdt_ctx* c, const int32_t* ids, const int32_t* pay0, SortPlan& pl, SortBuffers& sb, bool beside = false) {
  const antdt_model& m = c->m;
  pl.F = m.num_fields; pl.passes = c->sort_passes; pl.radix_bits = c->radix_bits;
  pl.total_tiles = c->atotal_tiles;
  pl.rows = m.rows_per_field; pl.samples = c->B; pl.width = c->FD; pl.beside = beside;
  sb.ids = ids;
  sb.key[0] = c->key[0]; sb.key[1] = c->key[1]; sb.pay[0] = c->pay[0]; sb.pay[1] = c->pay[1];
  sb.hist = c->hist;
  sb.digit_total = c->digit_total;
  sb.slots = beside && !c->slots_apart ? nullptr : c->goes_out;   // (the reduction's, which follows)
  sb.pay0 = pay0;
  sb.offsets = nullptr;
}

// Sort the lookups by row id: everything of the server side that depends only on the batch's ids.
static int build_coalescing(antdt_ctx* c, const int32_t* ids, const int32_t* pay0, hipStream_t s) {
  SortPlan pl;
  SortBuffers sb;
  fill_sort(c, ids, pay0, pl, sb, c->side && s == c->side);
  if (!pay0) sb.offsets = c->offsets;
  HIP_TRY(c, launch_sort(pl, sb, c->afp, c->atb, prof_of(c), s, &c->sorted_buf));
  return ANTDT_OK;
}

// Whether the sort beside a batched step finds the samples of the lookups by itself: by buckets it reads the lookups in the batch's order
// once, and works them out of the bags' boundaries on the way.  Saves writing and reading them, but moves the sort further into the gather,
// which wants the memory too (with a launch for the samples ahead / so, a step, us: 42 M lookups 2537 / 2499, 9 M 685 / 674; 6 M
// 518 / 532, 4.1 M 501 / 503, 3.8 M 361 / 356, 3.2 M 413 / 427; behind the gather 42 M 2547 / 2517, 3.8 M 359 / 375).
static constexpr int64_t FINDS_MIN = 8000000;
static bool sort_beside_finds_samples(antdt_ctx* c) {
  if (c->fp.p[c->m.num_fields] < FINDS_MIN) return false;
  SortPlan pl;
  SortBuffers sb;
  coalesce_whole_batch(c);
  fill_sort(c, c->ids, nullptr, pl, sb, true);
  return sort_finds_samples(pl, sb, c->afp);
}

// The sample index of every lookup, where the last batched step may have left none: also if that was a replay (of other bags perhaps), or will be,
// when this capture is replayed.  What is captured here has not run.
static int sample_indices(antdt_ctx* c, hipStream_t s) {
  const bool capturing = note_capture(c, s), leaves = capturing && c->fp.p[c->m.num_fields] >= FINDS_MIN;
  if (!c->samples_missing && !c->replays_leave_samples && !leaves) return ANTDT_OK;
  HIP_TRY(c, launch_expand_samples(c->offsets, c->lookup_sample, c->fp, c->m.num_fields, (int)c->B, s));
  c->samples_missing = c->samples_missing && capturing;
  return ANTDT_OK;
}

static void fill_wgrad_args(antdt_ctx* c, WgradArgs& u) {
  memset(&u, 0, sizeof(u));
  u.n_layers = c->L - 1;
  u.bf16 = c->act_bf16;
  for (int l = 0; l + 1 < c->L; ++l) {
    u.A[l] = l == 0 ? c->x : c->h[l]; u.lda[l] = l == 0 ? c->ldx : c->width[l];
    u.B[l] = c->dh[l + 1]; u.ldb[l] = c->width[l + 1];
    u.M[l] = c->width[l]; u.N[l] = c->width[l + 1];
    u.w_off[l] = c->w_off[l]; u.wb[l] = c->wb[l];
  }
  u.part = c->head_part; u.ldpart = c->ldpart;
  if (c->sums_per_sample) {
    u.dz = c->head_part; u.A[0] = c->x; u.lda[0] = c->ldx;
  }
  u.width = c->width[c->L - 1]; u.last_off = c->w_off[c->L - 1];
  u.p = c->params; u.state = c->pstate; u.lr = c->m.lr; u.eps = c->m.eps;
  u.grads = c->shard_grads; u.stride = c->Pstride;
}

// Whether the sort of a batched step runs in the launch of the weight gradients (where it goes to no stream of its own).
static bool sort_joins(antdt_ctx* c) {
  WgradArgs u;
  fill_wgrad_args(c, u);
  return wgrad_takes_sort(u, c->tab.K, c->B, c->m.num_fields, c->fp);
}

// Per-shard gradients of all dense layers for shards [k0, k1), one launch on `ws`; with `dgrad` it forms the gradient of the pooled
// input too, with `sort` that of an fp32 model also sorts the batch's lookups.
static int shard_weight_gradients(antdt_ctx* c, int k0, int k1, hipStream_t ws, bool sort = false, const GemmArgs* dgrad = nullptr) {
  WgradArgs u;
  fill_wgrad_args(c, u);
  u.k0 = k0;
  const HeadTiles ht = head_tiles(c->tab);
  KSegments seg;
  memset(&seg, 0, sizeof(seg));
  seg.n = k1 - k0;
  for (int q = 0; q < seg.n; ++q) {
    seg.ks[q] = c->tab.start[k0 + q]; seg.ke[q] = seg.ks[q] + c->tab.len[k0 + q];
    seg.ts[q] = ht.base[k0 + q]; seg.te[q] = ht.base[k0 + q + 1];
  }
  ProfScope ps(prof_of(c), KID_GEMM_WGRAD, ws);
  if (sort) {
    SortPlan pl;
    SortBuffers sb;
    fill_sort(c, c->ids, c->lookup_sample, pl, sb);
    HIP_TRY(c, launch_wgrad_and_sort(u, seg, pl, sb, c->afp, dgrad, ws));
    c->sorted_buf = 0;
  } else if (dgrad) {
    HIP_TRY(c, launch_wgrad_and_dgrad(u, seg, *dgrad, ws));
  } else {
    HIP_TRY(c, launch_wgrad(u, seg, true, ws));
  }
  return ANTDT_OK;
}

// The per-shard dense gradients of a worker step that left them to the dense update: computed
// now, on the weight-gradient stream, for a view (or the stand-alone aggregation) that wants
// them in memory.  Shards that were not stepped get whatever their rows hold (never read back).
static int compute_shard_grads(antdt_ctx* c, bool capturing) {
  if (!c->wgrad_deferred || (c->shard_grads_done && !c->captured)) return ANTDT_OK;
  hipStream_t ws = c->wside;
  if (!c->operands_captured || capturing) HIP_TRY(c, hipStreamWaitEvent(ws, c->ev_dh[0], 0));   // (else the replay is complete)
  {
    const int rc = shard_weight_gradients(c, 0, c->tab.K, ws);
    if (rc) return rc;
  }
  HIP_TRY(c, hipEventRecord(c->ev_wgrad, ws));
  c->wgrad_pending = true;
  c->shard_grads_done = true;
  return ANTDT_OK;
}

// Dense update from gradients in memory: g = sum over the rows of `tab` with their weights, then Adagrad and the bf16
// copies of the weights (W_0's to `wb0`).
static int dense_update(antdt_ctx* c, const ShardTab& tab, bf16_t* wb0, hipStream_t s) {
  DenseAdagradArgs a;
  memset(&a, 0, sizeof(a));
  a.p = c->params; a.state = c->pstate; a.grads = c->shard_grads; a.stride = c->Pstride; a.lr = c->m.lr; a.eps = c->m.eps;
  int nr = 0, rblocks = 0;
  auto add_range = [&](int64_t off, int64_t len) {
    a.rng_off[nr] = off; a.rng_len[nr] = len; a.rng_block[nr] = rblocks;
    rblocks += (int)((len + 255) / 256);
    ++nr;
  };
  if (c->act_bf16) {
    for (int l = 0; l + 1 < c->L; ++l) {
      a.w_off[l] = c->w_off[l]; a.rows[l] = c->width[l]; a.cols[l] = c->width[l + 1];
      a.wb[l] = l == 0 ? wb0 : c->wb[l];
      a.tile_base[l + 1] = a.tile_base[l] + ((c->width[l] + 63) / 64) * ((c->width[l + 1] + 63) / 64);
      add_range(c->b_off[l], c->width[l + 1]);
    }
    a.n_mat = c->L - 1;
    add_range(c->w_off[c->L - 1], c->P - c->w_off[c->L - 1]);
  } else {
    add_range(0, c->P);
  }
  a.n_rng = nr;
  a.rng_block[nr] = rblocks;
  ProfScope ps(prof_of(c), KID_DENSE_ADAGRAD, s);
  HIP_TRY(c, launch_dense_adagrad(a, tab, s));
  return ANTDT_OK;
}

// Cuts the sample ranges into pieces (one row of the gradient buffer each, the longest first) if the weight gradients
// are better formed piece by piece, on large tiles, and added up by the update than by blocks that each walk all
// samples.  With few tiles and many samples the latter have to be small tiles to be enough for the compute
// units, and read each operand twice as often (845-1024-512-256, 15625 samples of eight unequal shards: 168 us against
// 85 + 19 for the update; the whole step with 1.1 M (4.3 M) lookups 483 -> 381 (624 -> 517) us, of 9000 samples 314 -> 273 (391 -> 369), 6500
// in one range 218 -> 202).  Every piece costs a write and a read of all gradients, which takes about a thousand samples to pay (6500
// samples in 7 pieces 284 / 294 us, 2573-1024-512 with 6500 in 12 pieces 471 / 507, 11000 in 12 779 / 777: measured on earlier kernels).
static int cut_ranges(const antdt_ctx* c, const KSegments& seg, KSegments& pieces) {
  int64_t samples = 0, tiles = 0;
  for (int q = 0; q < seg.n; ++q) samples += seg.ke[q] - seg.ks[q];
  for (int l = 0; l + 1 < c->L; ++l) tiles += (int64_t)((c->width[l] + 127) / 128) * ((c->width[l + 1] + 127) / 128);
  if (tiles >= 400) return 0;
  auto count = [&](int64_t len) {
    int64_t n = 0;
    for (int q = 0; q < seg.n; ++q) n += (seg.ke[q] - seg.ks[q] + len - 1) / len;
    return n;
  };
  int64_t len = 1536;
  while (count(len) > c->m.max_shards) len += len / 4;   // (ends: there are no more ranges than shards)
  if (tiles * count(len) < 400 || samples < 1024 * count(len)) return 0;
  memset(&pieces, 0, sizeof(pieces));
  std::pair<int, int> order[ANTDT_MAX_SHARDS];   // (-length, place in the list of all pieces)
  KSegments all;
  memset(&all, 0, sizeof(all));
  for (int q = 0; q < seg.n; ++q)
    for (int k = seg.ks[q]; k < seg.ke[q]; k += (int)len) {
      const int i = all.n++;
      all.ks[i] = k; all.ke[i] = std::min(seg.ke[q], k + (int)len); all.w[i] = seg.w[q];
      all.ts[i] = seg.ts[q]; all.te[i] = k == seg.ks[q] ? seg.te[q] : seg.ts[q];   // (the last layer's sums: with the first piece)
      order[i] = {-(all.ke[i] - all.ks[i]), i};
    }
  std::sort(order, order + all.n);
  for (pieces.n = 0; pieces.n < all.n; ++pieces.n) {
    const int i = pieces.n, j = order[i].second;
    pieces.ks[i] = all.ks[j]; pieces.ke[i] = all.ke[j]; pieces.w[i] = all.w[j];
    pieces.ts[i] = all.ts[j]; pieces.te[i] = all.te[j];
  }
  return pieces.n;
}

// Whether the split's ranges would be cut (shards of equal length weigh the same unless they have factors).
static bool wgrad_in_pieces(const antdt_ctx* c) {
  KSegments seg, pieces;
  memset(&seg, 0, sizeof(seg));
  for (int k = 0; k < c->tab.K; ++k) {
    const int ks = c->tab.start[k], ke = ks + c->tab.len[k];
    if (seg.n > 0 && c->tab.len[k] == c->tab.len[k - 1]) {
      seg.ke[seg.n - 1] = ke;
    } else {
      seg.ks[seg.n] = ks; seg.ke[seg.n++] = ke;
    }
  }
  return cut_ranges(c, seg, pieces) > 0;
}

// Lookups from which the sort does not wait for the gather: the sample index of every lookup then comes from a launch of
// its own on the sort's stream, one more for the host (or is not needed, see FINDS_MIN; behind / beside the gather, us per step: 26 fields, 1.1 M lookups 193 / 200,
// 1.8 M 267 / 282, 2.5 M 361 / 357, 3.3 M 435 / 438, 4.3 M 521 / 515; 60 fields, 2.0 M 238 / 238, 3.8 M 397 / 385; 100, 42 M 2879 / 2820).
static constexpr int64_t EARLY_MIN = 3000000;

// Forward and backward of shards [k0, k1) as one batched sequence of launches.
static int worker_range(antdt_ctx* c, int k0, int k1, float* loss_out, hipStream_t s) {
  if (c->stage < ST_BATCH) return fail(c, ANTDT_BAD_STATE, "antdt_worker_step: call antdt_set_batch first");
  if (!c->have_shards || c->shard_B != c->B)
    return fail(c, ANTDT_BAD_STATE, "antdt_worker_step: antdt_assign_shard with the batch's B is required");
  {  // an earlier batched step whose aggregate never came (or whose split was replaced): let its side work finish
    const int rc = join_side(c, s);
    if (rc) return rc;
    c->presorted = false;
  }
  {  // this step overwrites the operands of the previous step's weight-gradient products
    const int rc = join_wgrad(c, s);
    if (rc) return rc;
  }
  Profiler* pr = prof_of(c);
  const antdt_model& m = c->m;
  const ShardTab& tab = c->tab;
  const int64_t s0 = tab.start[k0];
  const int64_t ns = (int64_t)tab.start[k1 - 1] + tab.len[k1 - 1] - s0;
  const int L = c->L;
  const size_t es = c->act_size;
  c->presorted = false;
  c->batched = k0 == 0 && k1 == tab.K;
  c->left_out = false;
  const bool capturing = note_capture(c, s);
  const bool beside = c->batched && side_stream(c);
  const bool finds = beside && sort_beside_finds_samples(c), early = beside && c->fp.p[m.num_fields] >= EARLY_MIN;
  if (early) HIP_TRY(c, hipEventRecord(c->ev_fork, s));
  {
    PoolArgs a;
    a.tables = c->tables; a.ids = c->ids; a.offsets = c->offsets; a.dense = c->dense; a.x = c->x;
    a.F = m.num_fields; a.D = m.dim; a.num_dense = m.num_dense; a.ldx = c->ldx; a.B = (int32_t)c->B;
    a.s0 = (int32_t)s0; a.ns = (int32_t)ns; a.R = m.rows_per_field;
    a.table_bf16 = m.table_dtype == ANTDT_BF16; a.x_bf16 = c->act_bf16;
    a.mean_pool = m.pooling == ANTDT_POOL_MEAN;
    a.lookup_sample = early ? nullptr : c->lookup_sample;
    ProfScope ps(pr, KID_POOL, s);
    HIP_TRY(c, launch_pool(a, c->fp, s));
  }
  if (c->batched) c->samples_missing = finds;
  c->replays_leave_samples = c->replays_leave_samples || (finds && capturing);
  if (beside) {
    // All shards in one pass: the sort of the coming aggregate depends on the batch alone, so it runs beside the MLP
    // and, of large batches, beside the gather too (see EARLY_MIN).
    for (int k = 0; k < tab.K; ++k) c->included[k] = true;
    set_weights(c);
    if (!early) HIP_TRY(c, hipEventRecord(c->ev_fork, s));
    HIP_TRY(c, hipStreamWaitEvent(c->side, c->ev_fork, 0));
    coalesce_whole_batch(c);
    if (early && !finds) HIP_TRY(c, launch_expand_samples(c->offsets, c->lookup_sample, c->fp, m.num_fields, (int)c->B, c->side));
    const int rc = build_coalescing(c, c->ids, finds ? nullptr : c->lookup_sample, c->side);
    if (rc) return rc;
    HIP_TRY(c, hipEventRecord(c->ev_join, c->side));
    c->presorted = true;
    c->side_pending = true;
  }
  auto act = [&](int l) -> char* { return l == 0 ? c->x : c->h[l]; };
  auto ld = [&](int l) -> int64_t { return l == 0 ? c->ldx : c->width[l]; };
  auto weight = [&](int l) -> const void* {
    return c->act_bf16 ? (const void*)c->wb[l] : (const void*)(c->params + c->w_off[l]);
  };
  auto forward = [&](int l) {   // hidden layer l + 1
    GemmArgs g;
    memset(&g, 0, sizeof(g));
    g.A = act(l) + s0 * ld(l) * es; g.lda = ld(l);
    g.C = c->h[l + 1] + s0 * c->width[l + 1] * es; g.ldc = c->width[l + 1];
    g.bias = c->params + c->b_off[l];
    g.M = (int32_t)ns; g.N = c->width[l + 1];
    if (c->act_bf16) {  // (the padding rows of W_0's copy are zero)
      g.K = (int32_t)ld(l);
      g.B = c->wb[l]; g.ldb = c->width[l + 1]; g.b_kc = 0;
    } else {
      g.K = c->width[l];
      g.B = c->params + c->w_off[l]; g.ldb = c->width[l + 1]; g.b_kc = 0;
    }
    g.epi = EPI_BIAS_RELU; g.bf16_in = c->act_bf16; g.bf16_out = c->act_bf16;
    return g;
  };
  auto backward = [&](int l) {   // gradient w.r.t. act_l: through W_l, then the ReLU of layer l-1 (none for the input)
    GemmArgs g;
    memset(&g, 0, sizeof(g));
    g.A = c->dh[l + 1] + s0 * c->width[l + 1] * es; g.lda = c->width[l + 1];
    g.B = weight(l); g.ldb = c->width[l + 1]; g.b_kc = 1;
    g.M = (int32_t)ns; g.K = c->width[l + 1];
    g.bf16_in = c->act_bf16;
    if (l > 0) {
      g.C = c->dh[l] + s0 * c->width[l] * es; g.ldc = c->width[l]; g.N = c->width[l];
      g.mask = c->h[l] + s0 * c->width[l] * es; g.ldmask = c->width[l];
      g.epi = EPI_RELU_MASK; g.bf16_out = c->act_bf16;
    } else {
      g.C = c->dx + s0 * c->FD; g.ldc = c->FD; g.N = c->FD;
      g.epi = EPI_PLAIN; g.bf16_out = 0;
      if (loss_out) {
        g.loss = c->loss_job + k0;
        g.loss_blocks = k1 - k0;
      }
    }
    return g;
  };
  // Backward.  The data-gradient chain dH_{l+1} -> dH_l first; nothing needs the weight gradients before the dense
  // update.  With bf16 products they are not computed here at all, unless the caller asked for them or the
  // library may have no streams of its own: apply_update forms them inside the dense update (aggregated over
  // the shards in registers, never written per shard), and this step only records when their operands are
  // complete; the per-shard gradients of the contract are computed when a view asks for them.  Otherwise
  // (fp32 models: they are small) one launch behind the chain: beside the input gradient on another stream it would
  // hide less than the hop costs (one worker's step on 64 / 1531 samples: 87 / 109 us that way, 54 / 78 here).
  bool defer = !c->eager_wgrad;
  for (int k = 0; k < tab.K; ++k)   // (also when another shard's step of this iteration did: apply_update goes one way for all)
    defer = defer || ((k < k0 || k >= k1) && c->stepped[k] && c->wgrad_deferred);
  const bool deferred = defer && c->act_bf16 && c->wside && !c->static_bound;
  // All shards of an fp32 model whose sort goes to no other stream: it runs beside the weight gradients
  const bool sort = !deferred && c->batched && !beside && c->total_tiles > 0 && c->joined_sort_used && sort_joins(c);
  // The gradient of the pooled input, which only the aggregation reads, shares the launch of weight gradients that are formed here, where
  // that takes it (and nobody times the two classes apart).
  bool joins = false;
  if (L > 1 && !deferred && !prof_apart(pr, KID_GEMM_BWD, KID_GEMM_WGRAD)) {
    WgradArgs u;
    fill_wgrad_args(c, u);
    joins = wgrad_takes_dgrad(u, k1 - k0, backward(0), m.num_fields, sort ? &c->fp : nullptr);
  }
  // All shards of a bf16 model whose sort goes to no other stream, no field longer than a block takes in a pass: the passes run beside the products,
  // one in a launch (behind / beside them, a step, us: 1024-512-256, 26 fields of 670 / 1000 / 2000 / 3200 / 3800 lookups 75.4 / 69.7, 72.8 / 67.6,
  // 84.6 / 81.0, 90.1 / 87.5, 91.3 / 90.8, three passes of 1000 79.1 / 73.7; ten fields of 4100 91.1 / 90.8; 256-128, 26 of 1600 70.5 / 68.0;
  // 1024-512, 30 of 3000 90.0 / 87.8).  Where as many products have room for one: large tiles have none, and a pass in a launch of its own takes
  // longer than all of them in one block a field (in one block / by pass: 1024, 24 fields of 64 columns, 4095 samples 134 / 149, three passes 138 / 161; 256, 20
  // of 2000 samples, three passes and two products 80 / 87).
  bool passes_join = c->act_bf16 && c->batched && !beside && c->total_tiles > 0 && c->joined_sort_used &&
                     L > 1 && ns > 0 && passes_fit(m.num_fields, c->fp) && !prof_apart(pr, KID_GEMM_FWD, KID_SORT_SCATTER) &&
                     !prof_apart(pr, KID_GEMM_BWD, KID_SORT_SCATTER);
  if (passes_join) {
    int room = 0;
    for (int l = 0; l + 1 < L; ++l) room += gemm_takes_sort(forward(l)) + ((l > 0 || !joins) && gemm_takes_sort(backward(l)));
    passes_join = room >= c->sort_passes;
  }
  SortPlan sort_plan;
  SortBuffers sort_buffers;
  SortPass sort_pass;
  int sort_next = 0;   // pass
  if (passes_join) {
    coalesce_whole_batch(c);
    fill_sort(c, c->ids, c->lookup_sample, sort_plan, sort_buffers);
    plan_sort_pass(sort_plan, sort_buffers, c->fp, 0, sort_pass);
  }
  auto product = [&](const GemmArgs& g) {
    const bool sorts = passes_join && sort_next < c->sort_passes && gemm_takes_sort(g);
    const hipError_t e = launch_gemm(g, sorts ? &sort_pass : nullptr, s);
    if (sorts && ++sort_next < c->sort_passes) plan_sort_pass(sort_plan, sort_buffers, c->fp, sort_next, sort_pass);
    return e;
  };
  // the matrix products of each pass are timed as one bracket when they run back to back
  ProfScope fwd_scope(L > 1 ? pr : nullptr, KID_GEMM_FWD, s);
  fwd_scope.launches(L - 1);
  for (int l = 0; l + 1 < L; ++l) HIP_TRY(c, product(forward(l)));
  fwd_scope.close();
  {
    HeadArgs a;
    memset(&a, 0, sizeof(a));
    a.h = act(L - 1); a.ldh = ld(L - 1); a.width = c->width[L - 1];
    a.w = c->params + c->w_off[L - 1]; a.b = c->params + c->b_off[L - 1];
    a.labels = c->labels;
    a.bf16_h = c->act_bf16;
    if (L > 1) {
      a.dh = c->dh[L - 1]; a.lddh = c->width[L - 1]; a.dh_cols = c->width[L - 1]; a.relu = 1; a.bf16_dh = c->act_bf16;
    } else {
      a.dh = c->dx; a.lddh = c->FD; a.dh_cols = c->FD; a.relu = 0; a.bf16_dh = 0;
    }
    a.k_begin = k0; a.k_end = k1;
    a.part = c->head_part; a.ldpart = c->ldpart;
    if (c->sums_per_sample) {
      a.dz = c->head_part; a.loss_s = c->head_part + m.max_batch;
    }
    a.job = c->loss_job; a.loss_out = loss_out;
    ProfScope ps(pr, KID_HEAD, s);
    HIP_TRY(c, launch_head_tiles(a, tab, s));
    if (L == 1 && loss_out && ns > 0) HIP_TRY(c, launch_losses(c->loss_job + k0, k1 - k0, s));   // (else beside the input gradient)
  }
  c->wgrad_deferred = deferred;
  c->shard_grads_done = false;
  // The event behind the last operand of the weight gradients (with up to one hidden layer the loss kernel
  // writes it, else the data gradient of layer 1).
  if (deferred) {
    // Steps of other shards since the last update on another stream: the library's stream waits for their operands before
    // the event stands for this step's (in a capture on one stream the caller's own order is all there is).
    bool others = false;
    for (int k = 0; k < tab.K; ++k) others = others || c->stepped[k];
    if (others && c->operands_stream != s && c->operands_captured == capturing && !(capturing && !wgrad_stream(c)))
      HIP_TRY(c, hipStreamWaitEvent(c->wside, c->ev_dh[0], 0));
    c->operands_stream = s;
  }
  c->operands_captured = capturing;
  if (deferred && L <= 2) HIP_TRY(c, hipEventRecord(c->ev_dh[0], s));
  ProfScope bwd_scope(L > 1 ? pr : nullptr, KID_GEMM_BWD, s);
  bwd_scope.launches(L - 1);
  for (int l = L - 2; l >= 0; --l) {
    if (l > 0 || !joins) HIP_TRY(c, product(backward(l)));
    if (l == 1 && deferred) HIP_TRY(c, hipEventRecord(c->ev_dh[0], s));
  }
  bwd_scope.close();
  if (passes_join) {
    c->sorted_buf = (c->sort_passes - 1) & 1;
    c->joined_sort_used = false;
    for (int k = 0; k < tab.K; ++k) c->included[k] = true;
    set_weights(c);
    c->presorted = true;
  }
  if (!deferred) {
    if (sort) {
      c->joined_sort_used = false;
      for (int k = 0; k < tab.K; ++k) c->included[k] = true;
      set_weights(c);
      coalesce_whole_batch(c);
    }
    const GemmArgs dgrad = joins ? backward(0) : GemmArgs{};
    const int rc = shard_weight_gradients(c, k0, k1, s, sort, joins ? &dgrad : nullptr);
    if (rc) return rc;
    c->presorted = c->presorted || sort;
  }
  for (int k = k0; k < k1; ++k) {
    c->stepped[k] = true;
    c->grads_viewed[k] = false;
  }
  if (c->stage == ST_AGGREGATED) c->stage = ST_BATCH;
  return ANTDT_OK;
}

int antdt_worker_step(antdt_ctx* c, int32_t k, float* loss_out, void* stream) {
  if (!c) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_worker_step: null context");
  if (!c->have_shards || k < 0 || k >= c->tab.K) return fail(c, ANTDT_INVALID_ARG, "antdt_worker_step: shard index out of range");
  return worker_range(c, k, k + 1, loss_out, (hipStream_t)stream);
}

int antdt_worker_step_all(antdt_ctx* c, float* loss_out, void* stream) {
  if (!c) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_worker_step_all: null context");
  if (!c->have_shards) return fail(c, ANTDT_BAD_STATE, "antdt_worker_step_all: call antdt_assign_shard first");
  return worker_range(c, 0, c->tab.K, loss_out, (hipStream_t)stream);
}

int antdt_aggregate(antdt_ctx* c, const uint8_t* shard_mask, void* stream) {
  if (!c) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_aggregate: null context");
  if (c->stage < ST_BATCH || !c->have_shards || c->shard_B != c->B)
    return fail(c, ANTDT_BAD_STATE, "antdt_aggregate: set_batch, assign_shard and worker_step come first");
  hipStream_t s = (hipStream_t)stream;
  const int K = c->tab.K;
  for (int k = 0; k < K; ++k) {
    c->included[k] = !shard_mask || shard_mask[k];
    if (c->included[k]) {
      if (c->tab.len[k] > 0 && !c->stepped[k])
        return fail(c, ANTDT_BAD_STATE, "antdt_aggregate: an included shard has no worker_step result");
    }
  }
  bool all = true;  // leaving out an empty shard changes nothing
  for (int k = 0; k < K; ++k) all = all && (c->included[k] || c->tab.len[k] == 0);
  {  // also when what is sorted there is stale (a new split): its buffers are rebuilt below
    const int rc = join_side(c, s);
    if (rc) return rc;
  }
  if (c->presorted && all) {
    // the batched worker step has sorted, on the side stream or in its weight-gradient launch (the weights are no part of it)
    if (c->weights_dirty) set_weights(c);
  } else if (all) {
    set_weights(c);
    coalesce_whole_batch(c);
    int rc = sample_indices(c, s);
    if (rc) return rc;
    rc = build_coalescing(c, c->ids, c->lookup_sample, s);
    if (rc) return rc;
  } else {
    // Some shards are left out: pack the lookups of the others (the unique-id buffer serves as
    // staging; the sort has consumed it before a view's run table is written there), fetch the
    // per-field counts (the one place where the host waits for the stream) and coalesce those.
    set_weights(c);
    const int F = c->m.num_fields;
    int32_t* ids_in = c->uniq;
    int32_t* pay_in = c->pack_pay;
    const int rcs = sample_indices(c, s);
    if (rcs) return rcs;
    HIP_TRY(c, launch_mask_pack(c->ids, c->lookup_sample, c->offsets, c->B, F, c->fp, c->tab, c->cbase, ids_in,
                                pay_in, s));
    int64_t cb[ANTDT_MAX_FIELDS + 1];
    HIP_TRY(c, hipMemcpyAsync(cb, c->cbase, (size_t)(F + 1) * 8, hipMemcpyDeviceToHost, s));
    HIP_TRY(c, hipStreamSynchronize(s));
    memset(&c->afp, 0, sizeof(c->afp));
    for (int f = 0; f <= F; ++f) {
      if (cb[f] < 0 || cb[f] > c->fp.p[F] || (f > 0 && cb[f] < cb[f - 1]))
        return fail(c, ANTDT_INVALID_ARG, "antdt_aggregate: offsets of the batch are not monotone");
      c->afp.p[f] = cb[f];
    }
    for (int f = F + 1; f <= ANTDT_MAX_FIELDS; ++f) c->afp.p[f] = c->afp.p[F];
    plan_tiles(F, c->afp, c->atb, c->atotal_tiles);
    const int rc = build_coalescing(c, ids_in, pay_in, s);
    if (rc) return rc;
  }
  c->left_out = !all;
  if (all) c->joined_sort_used = true;
  c->presorted = false;
  c->g_valid = false;
  c->gdense_valid = false;  // the dense sum is formed inside the optimizer kernel (or on request)
  c->stage = ST_AGGREGATED;
  return ANTDT_OK;
}

int antdt_set_shard_scale(antdt_ctx* c, const double* scale, int32_t K) {
  if (!c) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_set_shard_scale: null context");
  if (scale && (K < 1 || K > c->m.max_shards)) return fail(c, ANTDT_INVALID_ARG, "antdt_set_shard_scale: K out of range");
  if (scale)
    for (int k = 0; k < K; ++k)
      if (!(scale[k] >= 0.0) || !isfinite(scale[k]))
        return fail(c, ANTDT_INVALID_ARG, "antdt_set_shard_scale: factors must be finite and >= 0");
  for (int k = 0; k < ANTDT_MAX_SHARDS; ++k) c->shard_scale[k] = (scale && k < K) ? scale[k] : 1.0;
  c->weights_dirty = true;  // those in `tab` are stale: antdt_aggregate forms them anew, also where the sort was made ahead of time
  return ANTDT_OK;
}

int antdt_set_eager_weight_gradients(antdt_ctx* c, int32_t on) {
  if (!c) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_set_eager_weight_gradients: null context");
  c->eager_wgrad = on != 0;
  return ANTDT_OK;
}

int antdt_set_library_streams(antdt_ctx* c, int32_t on) {
  if (!c) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_set_library_streams: null context");
  bool stepped = false;
  for (int k = 0; k < ANTDT_MAX_SHARDS; ++k) stepped = stepped || c->stepped[k];
  if (c->side_pending || c->wgrad_pending || stepped)
    return fail(c, ANTDT_BAD_STATE, "antdt_set_library_streams: call it between iterations (after antdt_apply_update or antdt_bind)");
  c->no_streams = on == 0;
  return ANTDT_OK;
}

int antdt_set_lr(antdt_ctx* c, float lr) {
  if (!c) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_set_lr: null context");
  if (!(lr >= 0.f) || !isfinite(lr)) return fail(c, ANTDT_INVALID_ARG, "antdt_set_lr: lr must be finite and >= 0");
  c->m.lr = lr;
  return ANTDT_OK;
}

int antdt_apply_update(antdt_ctx* c, void* stream) {
  if (!c) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_apply_update: null context");
  if (c->stage != ST_AGGREGATED) return fail(c, ANTDT_BAD_STATE, "antdt_apply_update: call antdt_aggregate first");
  hipStream_t s = (hipStream_t)stream;
  Profiler* pr = prof_of(c);
  // The dense update touches nothing the sparse update touches, so it runs on the
  // weight-gradient stream (behind those products, which it needs anyway) beside the sparse
  // update; `s` joins it before this call's work on `s` is complete.
  hipStream_t ds = wgrad_stream(c) ? wgrad_stream(c) : s;
  const bool capturing = note_capture(c, s);
  // Beside the launch stream the input-gradient product of this step, enqueued behind the event that `ds` waits for, may
  // still be reading the bf16 copy of W_0: the new one goes to the other buffer, which is the current one from then
  // on (the products of deeper layers ran before the event).  On one stream, and for a captured iteration, whose
  // replays would never see the buffers change places, it is overwritten behind everything on `s`.
  const bool other_w0 = c->wgrad_deferred && ds != s && !c->captured;
  if (ds != s && !other_w0) {
    // (the dense update overwrites weights or copies that the worker step's last products on `s` read)
    HIP_TRY(c, hipEventRecord(c->ev_dh[c->L], s));  // everything enqueued on `s` so far (loss, last layer's gradient)
    HIP_TRY(c, hipStreamWaitEvent(ds, c->ev_dh[c->L], 0));
  }
  // Of an fp32 model the dense update (see dense_update) is a few blocks more of the sparse one's launch, unless nothing was looked up
  // or the two are timed apart.
  DenseJob dense = {};
  if (!c->act_bf16 && c->atotal_tiles > 0 && !prof_apart(pr, KID_SPARSE_ADAGRAD, KID_DENSE_ADAGRAD)) {
    dense.p = c->params; dense.state = c->pstate; dense.grads = c->shard_grads; dense.stride = c->Pstride; dense.n = c->P;
    dense.lr = c->m.lr; dense.eps = c->m.eps; dense.K = c->tab.K;
    memcpy(dense.w, c->tab.w, sizeof(dense.w));
  }
  {  // weighted run sums with the Adagrad step of every touched row applied on the spot
    SegArgs a;
    fill_seg_args(c, a);
    a.update = 1;
    HIP_TRY(c, launch_seg_reduce(a, c->afp, c->atb, c->tab, dense, pr, s));
  }
  if (c->wgrad_deferred) {
    // Weight gradients, their aggregation over the shards and the dense update in one kernel
    // (the per-shard and the aggregated gradient stay in registers; see cut_ranges for the other
    // way), behind the event that says the worker step's activations and pre-activation gradients are
    // complete.
    if (other_w0) {
      HIP_TRY(c, hipStreamWaitEvent(ds, c->ev_dh[0], 0));
    } else if (ds == s) {  // (per-shard gradients that a view asked for may still be in flight on the library's stream)
      const int rcj = join_wgrad(c, s);
      if (rcj) return rcj;
    }
    WgradArgs u;
    fill_wgrad_args(c, u);
    bf16_t* wb0 = other_w0 ? c->wb0_alt : c->wb[0];
    u.wb[0] = wb0;
    const HeadTiles ht = head_tiles(c->tab);
    KSegments seg;
    memset(&seg, 0, sizeof(seg));
    for (int k = 0; k < c->tab.K; ++k) {
      const float w = c->tab.w[k];
      if (w == 0.0f || c->tab.len[k] == 0) continue;
      const int ks = c->tab.start[k], ke = ks + c->tab.len[k];
      if (seg.n > 0 && seg.w[seg.n - 1] == w && seg.ke[seg.n - 1] == ks) {
        seg.ke[seg.n - 1] = ke;  // neighbours of equal weight: one range
        seg.te[seg.n - 1] = ht.base[k + 1];
      } else {
        seg.ks[seg.n] = ks; seg.ke[seg.n] = ke; seg.w[seg.n] = w;
        seg.ts[seg.n] = ht.base[k]; seg.te[seg.n] = ht.base[k + 1];
        ++seg.n;
      }
    }
    KSegments pieces;
    bool free_rows = !c->shard_grads_done;   // (gradients that a view handed out stay where they are)
    for (int k = 0; k < c->tab.K; ++k) free_rows = free_rows && !c->grads_viewed[k];
    if (free_rows && cut_ranges(c, seg, pieces) > 0) {
      {
        ProfScope ps(pr, KID_GEMM_WGRAD, ds);
        HIP_TRY(c, launch_wgrad(u, pieces, true, ds));
      }
      ShardTab tab;
      memset(&tab, 0, sizeof(tab));
      tab.K = pieces.n;
      for (int i = 0; i < pieces.n; ++i) tab.w[i] = pieces.w[i];
      const int rc = dense_update(c, tab, wb0, ds);
      if (rc) return rc;
      // a view may form the per-shard gradients in the same buffer, on the library's stream, behind this event
      if (ds == s) {
        HIP_TRY(c, hipEventRecord(c->ev_dh[0], s));
        c->operands_captured = capturing;
      }
    } else {
      ProfScope ps(pr, KID_WGRAD_ADAGRAD, ds);
      HIP_TRY(c, launch_wgrad(u, seg, false, ds));
    }
    if (other_w0) std::swap(c->wb[0], c->wb0_alt);
    if (ds != s) {
      HIP_TRY(c, hipEventRecord(c->ev_wgrad, ds));
      HIP_TRY(c, hipStreamWaitEvent(s, c->ev_wgrad, 0));
    }
    c->wgrad_pending = false;  // `s` now waits for everything on that stream
  } else if (dense.n == 0) {
    const int rc = dense_update(c, c->tab, c->wb[0], ds);
    if (rc) return rc;
    if (ds != s) {
      HIP_TRY(c, hipEventRecord(c->ev_wgrad, ds));
      HIP_TRY(c, hipStreamWaitEvent(s, c->ev_wgrad, 0));
      c->wgrad_pending = false;  // `s` now waits for everything on that stream
    }
  }
  c->stage = ST_BATCH;
  memset(c->stepped, 0, sizeof(c->stepped));
  return ANTDT_OK;
}

int antdt_dense_aggregate_adam(float* p, float* mm, float* v, const float* const* grads, const float* weights,
                               int32_t K, int64_t n, double lr, double beta1, double beta2, double eps,
                               int64_t step, void* stream) {
  if (K < 1 || K > 16) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_dense_aggregate_adam: K must be 1..16");
  if (n < 0 || step < 1) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_dense_aggregate_adam: n >= 0 and step >= 1 required");
  if (n == 0) return ANTDT_OK;  // nothing to do; empty buffers may be null
  if (!p || !mm || !v || !grads || !weights) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_dense_aggregate_adam: null argument");
  AdamArgs a;
  memset(&a, 0, sizeof(a));
  a.p = p; a.m = mm; a.v = v; a.K = K; a.n = n;
  uintptr_t al = (uintptr_t)p | (uintptr_t)mm | (uintptr_t)v;
  for (int k = 0; k < K; ++k) {
    if (!grads[k]) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_dense_aggregate_adam: null gradient buffer");
    a.g[k] = grads[k];
    a.w[k] = weights[k];
    al |= (uintptr_t)grads[k];
  }
  if (al & 15) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_dense_aggregate_adam: buffers must be 16-byte aligned");
  a.lr = (float)lr; a.b1 = (float)beta1; a.b2 = (float)beta2; a.eps = (float)eps;
  a.c1 = (float)(1.0 - beta1); a.c2 = (float)(1.0 - beta2);
  a.inv_bc1 = (float)(1.0 / (1.0 - pow(beta1, (double)step)));
  a.inv_bc2 = (float)(1.0 / (1.0 - pow(beta2, (double)step)));
  HIP_TRY(nullptr, launch_adam(a, (hipStream_t)stream));
  return ANTDT_OK;
}

int antdt_stream_copy(float* dst, const float* src, int64_t n, void* stream) {
  if (n < 0 || n >= (1ll << 40) || (n > 0 && (!dst || !src)) || (((uintptr_t)dst | (uintptr_t)src) & 15))
    return fail(nullptr, ANTDT_INVALID_ARG, "antdt_stream_copy: null or misaligned pointer, or n out of range");
  HIP_TRY(nullptr, launch_stream_copy(dst, src, n, (hipStream_t)stream));
  return ANTDT_OK;
}

int antdt_fill_tables(void* tables, int32_t dtype, int32_t F, int64_t R, int32_t D, float scale, void* stream) {
  if (!tables || F < 1 || R < 1 || D < 1 || (dtype != ANTDT_F32 && dtype != ANTDT_BF16))
    return fail(nullptr, ANTDT_INVALID_ARG, "antdt_fill_tables: invalid argument");
  HIP_TRY(nullptr, launch_fill_tables(tables, dtype == ANTDT_BF16, F, R, D, scale, (hipStream_t)stream));
  return ANTDT_OK;
}

int antdt_view_pooled(antdt_ctx* c, int32_t k, const void** x, int64_t* rows, int64_t* ldo, int32_t* dtype) {
  if (!c || !x || !rows || !ldo || !dtype) return fail(c, ANTDT_INVALID_ARG, "antdt_view_pooled: null argument");
  if (!c->have_shards || k < 0 || k >= c->tab.K) return fail(c, ANTDT_INVALID_ARG, "antdt_view_pooled: shard index out of range");
  if (c->stage < ST_BATCH) return fail(c, ANTDT_BAD_STATE, "antdt_view_pooled: nothing computed yet");
  *x = c->x + (int64_t)c->tab.start[k] * c->ldx * c->act_size;
  *rows = c->tab.len[k];
  *ldo = c->ldx;
  *dtype = c->act_bf16 ? ANTDT_BF16 : ANTDT_F32;
  return ANTDT_OK;
}

int antdt_view_shard_grads(antdt_ctx* c, int32_t k, const float** dense, const float** dx, int64_t* ld_dx) {
  if (!c || !dense || !dx || !ld_dx) return fail(c, ANTDT_INVALID_ARG, "antdt_view_shard_grads: null argument");
  if (!c->have_shards || k < 0 || k >= c->tab.K) return fail(c, ANTDT_INVALID_ARG, "antdt_view_shard_grads: shard index out of range");
  if (c->stage < ST_BATCH) return fail(c, ANTDT_BAD_STATE, "antdt_view_shard_grads: nothing computed yet");
  {
    const int rcg = compute_shard_grads(c, false);
    if (rcg) return rcg;
  }
  if (c->wgrad_pending) {  // the weight gradients are written on their own stream: wait for it here
    HIP_TRY(c, hipStreamSynchronize(c->wside));
    c->wgrad_pending = false;
  }
  c->grads_viewed[k] = true;
  *dense = c->shard_grads + (int64_t)k * c->Pstride;
  *dx = c->dx + (int64_t)c->tab.start[k] * c->FD;
  *ld_dx = c->FD;
  return ANTDT_OK;
}

int antdt_view_dense_grad(antdt_ctx* c, const float** g, void* stream) {
  if (!c || !g) return fail(c, ANTDT_INVALID_ARG, "antdt_view_dense_grad: null argument");
  if (c->stage != ST_AGGREGATED) return fail(c, ANTDT_BAD_STATE, "antdt_view_dense_grad: valid between antdt_aggregate and antdt_apply_update");
  {
    const int rcg = compute_shard_grads(c, note_capture(c, (hipStream_t)stream));
    if (rcg) return rcg;
    const int rcj = join_wgrad(c, (hipStream_t)stream);
    if (rcj) return rcj;
  }
  if (!c->gdense_valid) {  // written out on request only; apply_update forms the same sum on the fly
    DenseAggArgs d;
    d.grads = c->shard_grads; d.g = c->g_dense; d.P = c->P; d.stride = c->Pstride;
    ProfScope ps(prof_of(c), KID_DENSE_AGG, (hipStream_t)stream);
    HIP_TRY(c, launch_dense_agg(d, c->tab, (hipStream_t)stream));
    c->gdense_valid = true;
  }
  *g = c->g_dense;
  return ANTDT_OK;
}

int antdt_view_coalesced(antdt_ctx* c, int32_t f, const int32_t** unique_ids, const int32_t** seg_offsets,
                         const int32_t** seg_samples, int64_t* num_unique, int64_t* nnz, const float** G,
                         void* stream) {
  if (!c || !unique_ids || !seg_offsets || !seg_samples || !num_unique || !nnz || !G)
    return fail(c, ANTDT_INVALID_ARG, "antdt_view_coalesced: null argument");
  if (f < 0 || f >= c->m.num_fields) return fail(c, ANTDT_INVALID_ARG, "antdt_view_coalesced: field out of range");
  if (c->stage < ST_BATCH) return fail(c, ANTDT_BAD_STATE, "antdt_view_coalesced: call antdt_aggregate first");
  if (c->stage != ST_AGGREGATED) return fail(c, ANTDT_BAD_STATE, "antdt_view_coalesced: valid between antdt_aggregate and antdt_apply_update");
  if (!c->g_valid) {  // the run table and the coalesced sums are only written out on request
    SegArgs a;
    fill_seg_args(c, a);
    a.update = 0;
    HIP_TRY(c, launch_segments(a, c->afp, c->atb, prof_of(c), (hipStream_t)stream));
    HIP_TRY(c, launch_seg_reduce(a, c->afp, c->atb, c->tab, DenseJob{}, prof_of(c), (hipStream_t)stream));
    c->g_valid = true;
  }
  int32_t ub[2];
  HIP_TRY(c, hipMemcpyAsync(ub, c->ubase + f, sizeof(ub), hipMemcpyDeviceToHost, (hipStream_t)stream));
  HIP_TRY(c, hipStreamSynchronize((hipStream_t)stream));
  *unique_ids = c->uniq + ub[0];
  *seg_offsets = c->segoff + ub[0] + f;
  *seg_samples = c->pay[c->sorted_buf] + c->afp.p[f];
  *num_unique = ub[1] - ub[0];
  *nnz = c->afp.p[f + 1] - c->afp.p[f];
  *G = c->G + (int64_t)ub[0] * c->m.dim;
  return ANTDT_OK;
}

int antdt_profile(antdt_ctx* c, int32_t mode, int32_t kernel_id) {
  if (!c) return fail(nullptr, ANTDT_INVALID_ARG, "antdt_profile: null context");
  if (mode < 0 || mode > 3 || (mode == 2 && (kernel_id < 0 || kernel_id >= KID_COUNT)))
    return fail(c, ANTDT_INVALID_ARG, "antdt_profile: invalid mode or kernel id");
  c->prof.mode = mode;
  c->prof.sel = kernel_id;
  return ANTDT_OK;
}

int antdt_profile_overhead(antdt_ctx* c, void* stream, int32_t n, double* empty_ms, double* tiny_ms) {
  if (!c || !empty_ms || !tiny_ms || n < 1 || n > 4096)
    return fail(c, ANTDT_INVALID_ARG, "antdt_profile_overhead: null argument or n outside 1..4096");
  if (c->stage < ST_BOUND) return fail(c, ANTDT_BAD_STATE, "antdt_profile_overhead: call antdt_bind first");
  hipStream_t s = (hipStream_t)stream;
  std::vector<hipEvent_t> ev((size_t)n * 4);
  for (auto& e : ev) HIP_TRY(c, hipEventCreateWithFlags(&e, hipEventDisableSystemFence));
  for (int i = 0; i < n; ++i) {  // the flags kernel is the smallest one the library has
    HIP_TRY(c, launch_validate_reset(c->vflags, s));
    HIP_TRY(c, hipEventRecord(ev[4 * i + 0], s));
    HIP_TRY(c, hipEventRecord(ev[4 * i + 1], s));
    HIP_TRY(c, launch_validate_reset(c->vflags, s));
    HIP_TRY(c, hipEventRecord(ev[4 * i + 2], s));
    HIP_TRY(c, launch_validate_reset(c->vflags, s));
    HIP_TRY(c, hipEventRecord(ev[4 * i + 3], s));
  }
  HIP_TRY(c, hipStreamSynchronize(s));
  double e_sum = 0.0, t_sum = 0.0;
  for (int i = 0; i < n; ++i) {
    float a = 0.f, b = 0.f;
    HIP_TRY(c, hipEventElapsedTime(&a, ev[4 * i + 0], ev[4 * i + 1]));
    HIP_TRY(c, hipEventElapsedTime(&b, ev[4 * i + 2], ev[4 * i + 3]));
    e_sum += a;
    t_sum += b;
  }
  for (auto& e : ev) (void)hipEventDestroy(e);
  *empty_ms = e_sum / n;
  *tiny_ms = t_sum / n;
  return ANTDT_OK;
}

int antdt_profile_read(antdt_ctx* c, int32_t kid, int64_t* launches, double* total_ms) {
  if (!c || !launches || !total_ms) return fail(c, ANTDT_INVALID_ARG, "antdt_profile_read: null argument");
  if (kid < 0 || kid >= KID_COUNT) return fail(c, ANTDT_INVALID_ARG, "antdt_profile_read: kernel id out of range");
  prof_drain(&c->prof);
  *launches = c->prof.launches[kid];
  *total_ms = c->prof.total_ms[kid];
  c->prof.launches[kid] = 0;
  c->prof.total_ms[kid] = 0.0;
  return ANTDT_OK;
}

}  // extern "C"
