// Host side of the C ABI declared in include/dynts.h: argument checks, workspace layout and
// kernel launches.  Nothing here allocates device memory or synchronises the host.
#include "../../include/dynts.h"

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <atomic>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "attend.hpp"
#include "compact.hpp"
#include "paged.hpp"
#include "predictor.hpp"
#include "probe.hpp"
#include "resident.hpp"
#include "score_block.hpp"
#include "select.hpp"

namespace {

constexpr size_t kAlign = 256;
constexpr int kSelectLdsMax = 16384;  // candidates whose keys are cached in LDS (64 KiB)

// Ticket counters lie 256 bytes apart: a line of 32 of them was handed from XCD to XCD for every ticket.
constexpr int kCounterStride = 64;

size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

struct Plan {
  int G = 0, waves = 0, chunk = 0, nsplit = 0;
  size_t off_part_o = 0, off_part_ml = 0, off_unit_cnt = 0, off_seq_cnt = 0, off_qprev = 0, off_mlprev = 0, off_nprev = 0, off_spill = 0;
  int cap_pad = 0;
  size_t bytes = 0;  // that every call needs
  // runs of steps (resident_kernel): a cache of several chunks, each of one tile a wave; steps of a run whose partials the room behind has place
  // for, or 0; the bytes of both
  int run_steps = 0;
  size_t off_run_o = 0, off_run_ml = 0, off_run_stats = 0, off_run_n = 0, off_run_rec = 0;
  size_t run_bytes = 0;
};

int check_config(const dynts_config *c) {
  if (!c) return DYNTS_ENULL;
  if (c->n_layers <= 0 || c->batch <= 0 || c->n_q_heads <= 0 || c->n_kv_heads <= 0) return DYNTS_EINVAL;
  if (c->budget < 0 || c->window < 0 || c->evict_every <= 0 || c->capacity <= 0) return DYNTS_EINVAL;
  if (c->score_mode != DYNTS_SCORE_ACCUMULATE && c->score_mode != DYNTS_SCORE_EXTERNAL) return DYNTS_EINVAL;
  if (!(c->softmax_scale >= 0.f) || std::isinf(c->softmax_scale)) return DYNTS_EINVAL;
  if (c->head_dim != 64 && c->head_dim != 128) return DYNTS_ESHAPE;
  if (c->n_q_heads % c->n_kv_heads) return DYNTS_ESHAPE;
  if (c->n_q_heads / c->n_kv_heads > 16) return DYNTS_ESHAPE;
  if (c->n_kv_heads * (c->head_dim / 8) > 1024) return DYNTS_ESHAPE;
  if (c->batch > 65535 || c->n_kv_heads > 65535) return DYNTS_ESHAPE;
  if (c->capacity > (1 << 22)) return DYNTS_ESHAPE;  // row offsets inside a unit are 32-bit byte offsets
  if ((long long)c->capacity < (long long)c->budget + c->window + c->evict_every) return DYNTS_ECAPACITY;
  return DYNTS_OK;
}

// Split every (sequence, KV head) cache into chunks, one workgroup per chunk.  Workgroups have
// 8 waves (one per compute unit fits) when that still fills the chip, else 4; chunks are whole
// multiples of the workgroup's tile quantum.  The aim is about one 8-wave workgroup per compute
// unit: few enough that every wave loops over many tiles with its loads in flight, and that
// the split partials stay small.
Plan make_plan(const dynts_config &c, int target_wgs, int waves) {
  Plan p;
  p.G = c.n_q_heads / c.n_kv_heads;
  const long long units = (long long)c.batch * c.n_kv_heads;
  const long long target = target_wgs > 0 ? target_wgs : 256;  // workgroups wanted (256 compute units)
  p.waves = waves == 4 ? 4 : 8;
  const int quantum = p.waves * dynts::kTile;
  const int quanta = (c.capacity + quantum - 1) / quantum;
  long long want = (target + units / 2) / units;
  if (want < 1) want = 1;
  if (want > quanta) want = quanta;
  const int per = (int)((quanta + want - 1) / want);  // quanta per chunk
  p.chunk = per * quantum;
  p.nsplit = (c.capacity + p.chunk - 1) / p.chunk;
  const size_t rows = (size_t)units * p.nsplit * p.G;
  size_t off = 0;
  p.off_part_o = off;  off = align_up(off + rows * c.head_dim * sizeof(uint64_t));  // value + tag per word
  p.off_part_ml = off; off = align_up(off + rows * 2 * sizeof(uint64_t));
  p.off_unit_cnt = off; off = align_up(off + (size_t)units * kCounterStride * sizeof(uint32_t));
  p.off_seq_cnt = off; off = align_up(off + (size_t)c.batch * kCounterStride * sizeof(uint32_t));
  const size_t LB = (size_t)c.n_layers * c.batch;
  p.off_qprev = off;   off = align_up(off + 2 * LB * c.n_q_heads * c.head_dim * sizeof(uint16_t));  // two copies, used in turn
  p.off_mlprev = off;  off = align_up(off + LB * c.n_q_heads * 2 * sizeof(float));
  p.off_nprev = off;   off = align_up(off + LB * sizeof(int32_t));
  // the logits of one step of one layer, where they are kept for its score update (score_mode accumulate only)
  p.cap_pad = (c.capacity + dynts::kTile - 1) / dynts::kTile * dynts::kTile;
  p.off_spill = off;
  if (c.score_mode == DYNTS_SCORE_ACCUMULATE) off = align_up(off + (size_t)units * p.G * p.cap_pad * sizeof(float));
  p.bytes = off;
  // Room for the partials of a run's steps: of as many as lie between two triggers, but 16 to 64, and 64 MB of them at most (23 steps or more:
  // chunks of one tile a wave are at most 341 for all units).
  if (target_wgs == 0 && waves == 0 && p.nsplit > 1 && p.nsplit == quanta) {
    const long long fit = (64ll << 20) / (long long)(rows * (c.head_dim + 2) * sizeof(float));
    const int between = c.evict_every < 16 ? 16 : c.evict_every < dynts::kPartSteps ? c.evict_every : dynts::kPartSteps;
    p.run_steps = (int)(fit < between ? fit : between);
    const size_t R = (size_t)p.run_steps;
    p.off_run_o = off;     off = align_up(off + R * rows * c.head_dim * sizeof(float));
    p.off_run_ml = off;    off = align_up(off + R * rows * 2 * sizeof(float));
    p.off_run_stats = off; off = align_up(off + R * (size_t)units * 32 * sizeof(float));
    p.off_run_n = off;     off = align_up(off + R * c.batch * sizeof(int32_t));
    p.off_run_rec = off;   off = align_up(off + (size_t)c.batch * 4 * sizeof(int32_t));
  }
  p.run_bytes = off;
  return p;
}

}  // namespace

struct dynts_ctx {
  dynts_config cfg;
  Plan plan;
  float scale_log2;
  bool bound = false;
  bool shaped = false;                 // the launch shape is the caller's (dynts_set_launch_shape)
  uint16_t *K = nullptr, *V = nullptr;
  float *S = nullptr;
  int32_t *pos = nullptr, *seq_len = nullptr, *next_pos = nullptr, *n_prompt = nullptr, *status = nullptr;
  unsigned char *ws = nullptr;
  int run_steps = 0;                   // the plan's, where the workspace has the room for them
  // per layer: a score update is owed (1: by a pass over K, 2: from kept logits; 3: either, the next fused step's pass
  // over K or the kept logits, whichever is asked for first)
  std::vector<unsigned char> pending;
  std::vector<unsigned char> hint;     // per layer: a trigger follows the next fused step, keep its logits
  int spill_layer = -1;                // the layer the kept logits belong to (its pending is 2 or 3), or -1
  // Whether an unfused attention's logits are worth keeping is learned from what follows it (see unfused_ends):
  std::vector<unsigned char> pairs;    // per layer, up to 2: of its last ones in a row, those followed by their own update
  int unfused_layer = -1;              // the layer whose unfused attention waits for that answer, or -1
  bool pairs_known = false;            // some layer has had its answer
  std::vector<unsigned char> qslot;    // per layer: which copy of the saved query is current
  hipEvent_t ev_start = nullptr, ev_stop = nullptr;
  std::vector<hipEvent_t> ev_list_start, ev_list_stop;  // one pair per coming attend launch
  size_t ev_list_next = 0;
  // paged layout (dynts_bind_paged): K and V above are the page pools
  bool paged = false;
  int32_t *block_table = nullptr, *free_stack = nullptr, *free_top = nullptr;
  int max_pages = 0, n_pages = 0;
};

namespace {

int launch_status() { return hipGetLastError() == hipSuccess ? DYNTS_OK : DYNTS_EHIP; }

// Serial number of an attend launch: the tag its split partials carry.  One counter for the whole
// process, so that two contexts which share scratch memory can never mistake each other's words for
// their own; 0 is skipped (zero-filled scratch must read as stale).
uint32_t next_launch_tag() {
  static std::atomic<uint32_t> serial{0};
  uint32_t t = serial.fetch_add(1, std::memory_order_relaxed) + 1;
  if (t == 0) t = serial.fetch_add(1, std::memory_order_relaxed) + 1;
  return t;
}

// What is recorded into a graph may be replayed in any order with other graphs and with eager calls, which the
// context's bookkeeping does not see.  (An error of the query, the null stream beside a capture, counts as a capture.)
bool capturing(hipStream_t st) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return true;
}

int check_call(const dynts_ctx *ctx, int32_t layer) {
  if (!ctx) return DYNTS_ENULL;
  if (!ctx->bound) return DYNTS_ENOTBOUND;
  if (layer < 0 || layer >= ctx->cfg.n_layers) return DYNTS_EINVAL;
  return DYNTS_OK;
}

struct LayerView {
  uint16_t *K, *V;
  float *S;
  int32_t *pos, *seq_len, *next_pos;
  uint16_t *qprev, *qnext;
  float *mlprev;
  int32_t *nprev;
  int32_t *block_table;  // paged layout: this layer's [Nb][Hkv][max_pages]
};

LayerView layer_view(const dynts_ctx *ctx, int layer) {
  const dynts_config &c = ctx->cfg;
  const size_t units = (size_t)c.batch * c.n_kv_heads;
  const size_t rows = units * c.capacity;
  LayerView v;
  v.K = ctx->paged ? ctx->K : ctx->K + (size_t)layer * rows * c.head_dim;
  v.V = ctx->paged ? ctx->V : ctx->V + (size_t)layer * rows * c.head_dim;
  v.block_table = ctx->paged ? ctx->block_table + (size_t)layer * units * ctx->max_pages : nullptr;
  v.S = ctx->S + (size_t)layer * rows;
  v.pos = ctx->pos + (size_t)layer * rows;
  v.seq_len = ctx->seq_len + (size_t)layer * c.batch;
  v.next_pos = ctx->next_pos + (size_t)layer * c.batch;
  const size_t LBq = (size_t)layer * c.batch * c.n_q_heads;
  uint16_t *qbuf = reinterpret_cast<uint16_t *>(ctx->ws + ctx->plan.off_qprev) + 2 * LBq * c.head_dim;
  const size_t qsz = (size_t)c.batch * c.n_q_heads * c.head_dim;
  v.qprev = qbuf + (ctx->qslot[layer] ? qsz : 0);
  v.qnext = qbuf + (ctx->qslot[layer] ? 0 : qsz);
  v.mlprev = reinterpret_cast<float *>(ctx->ws + ctx->plan.off_mlprev) + LBq * 2;
  v.nprev = reinterpret_cast<int32_t *>(ctx->ws + ctx->plan.off_nprev) + (size_t)layer * c.batch;
  return v;
}

// Whether a launch takes the kernel with the wide merges.  Their registers (228 - 233 against 108 - 209) are every wave's, so a
// head_dim 64 launch has them only where it has no second workgroup on a compute unit to lose (32 of an XCD's units'
// chunks).  us a step, groups of four / wide:
//   head_dim 128, 4 heads a group, 8 units: 10 chunks 11.5 / 12.2, 17 chunks 16.4 / 14.9, 18 chunks 13.9 / 12.4;
//     12 units: 17 chunks 22.7 / 21.4; 16 units: 9 chunks 14.1 / 14.8, 11 chunks 18.7 / 19.4; 32 units: 6 chunks 18.3 / 20.2
//   head_dim 128, 7 or 8 heads: 8 units, 10 chunks 12.2 / 12.0; 48 units, 5 chunks 16.9 / 16.3; every size between likewise
//   head_dim 64, 4 heads: 8 units, 18 chunks 12.6 / 12.0, 17 chunks 13.5 / 13.0, 10 chunks 9.7 / 11.2; 12 units, 18 chunks
//     13.7 / 15.2; 4 units (four XCDs), 33 chunks 17.1 / 18.6
bool wide_merge(int D, int waves, int G, int nsplit, long long grid) {
  const int ne = (G * D + 64 * waves - 1) / (64 * waves);  // output elements per thread
  if (waves != 8) return false;
  if (D == 64) return ne == 1 && nsplit > dynts::kWideFrom1 && grid <= 256;
  return (ne == 1 && nsplit > dynts::kWideFrom1) || (ne == 2 && nsplit > dynts::kWideFrom2);
}

// start/stop (may be null) are attached to the dispatch itself, so their timestamps are the
// kernel's own begin and end
template <int D, int W, bool ATTEND, bool PENDING, bool APPEND>
void launch_partial(const dynts::AttendParams &p, dim3 grid, hipStream_t st, hipEvent_t start, hipEvent_t stop) {
  // A pass over K alone of a large cache has a compute unit to itself, by LDS that it only holds: 512 units of 8704 slots, with a second
  // workgroup beside it / without 199.2 / 188.4 us, of 5256 116.3 / 108.6, of 2300 50.5 / 50.3; 1024 of 3000 122.8 / 124.6, of 900 37.5 / 40.2.
  const unsigned hold = !ATTEND && D == 128 && W == 8 && p.cap > 2500 ? 42000 : 0;
  const bool spill = ATTEND && p.spill != nullptr;  // the step that keeps its logits: a form of its own
#define DYNTS_LAUNCH(PAGED, LARGE, SPILL, WIDE)                                                                     \
  hipExtLaunchKernelGGL((dynts::attend_kernel<D, W, ATTEND, PENDING, APPEND, PAGED, LARGE, SPILL, WIDE>), grid,      \
                        dim3(W * 64), hold, st, start, stop, 0, p)
#define DYNTS_LAUNCH2(PAGED, LARGE, WIDE)              \
  if (spill) DYNTS_LAUNCH(PAGED, LARGE, ATTEND, WIDE); \
  else DYNTS_LAUNCH(PAGED, LARGE, false, WIDE)
  constexpr int kIfPending = PENDING ? dynts::kBurst : 0;  // (no scores to write otherwise)
  if (p.block_table) {
    if (PENDING && p.score_tiles > 1) { DYNTS_LAUNCH2(true, kIfPending, false); }
    else { DYNTS_LAUNCH2(true, 0, false); }
  } else if (p.fit_slots < p.cap) {
    DYNTS_LAUNCH2(false, dynts::kStream, false);
  } else if (ATTEND && wide_merge(D, W, p.G, p.nsplit, grid.x)) {  // (before bursts: 16 units of 30000 slots 46.3 us with those, 45.4 so, when K did not go through LDS)
    DYNTS_LAUNCH2(false, 0, (ATTEND && W == 8));
  } else if (PENDING && p.score_tiles > 1) {
    DYNTS_LAUNCH2(false, kIfPending, false);
  } else {
    DYNTS_LAUNCH2(false, 0, false);
  }
#undef DYNTS_LAUNCH2
#undef DYNTS_LAUNCH
}

template <int D, int W>
void launch_partial_d(const dynts::AttendParams &p, dim3 grid, hipStream_t st, hipEvent_t e0, hipEvent_t e1,
                      bool attend, bool pending, bool append) {
  if (!attend) return launch_partial<D, W, false, true, false>(p, grid, st, e0, e1);
  if (pending) {
    if (append) return launch_partial<D, W, true, true, true>(p, grid, st, e0, e1);
    return launch_partial<D, W, true, true, false>(p, grid, st, e0, e1);
  }
  if (append) return launch_partial<D, W, true, false, true>(p, grid, st, e0, e1);
  return launch_partial<D, W, true, false, false>(p, grid, st, e0, e1);
}

__global__ void clear_words_kernel(uint32_t *words, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) words[i] = 0u;
}

// scratch of one attend launch: split partials (tagged words) and ticket counters (zero between launches)
struct Transient {
  uint64_t *part_o, *part_ml;
  uint32_t *unit_cnt, *seq_cnt;
  int cnt_stride;
};

// attend (optionally with fused append) and/or the deferred score update of one layer
int run_attend(dynts_ctx *ctx, int layer, const uint16_t *q, const uint16_t *k_new, const uint16_t *v_new,
               const float *s_new, const uint8_t *active, float *out, float *lse, bool attend,
               bool apply_pending, bool append, hipStream_t st, const Transient *transient = nullptr,
               bool keep_logits = false) {
  // transient: where the split partials and the counters of this launch live (default: the head of the
  // workspace); what must survive from one step to the next is always in the workspace
  const dynts_config &c = ctx->cfg;
  const Plan &pl = ctx->plan;
  Transient tr;
  if (transient) {
    tr = *transient;
  } else {
    tr.part_o = reinterpret_cast<uint64_t *>(ctx->ws + pl.off_part_o);
    tr.part_ml = reinterpret_cast<uint64_t *>(ctx->ws + pl.off_part_ml);
    tr.unit_cnt = reinterpret_cast<uint32_t *>(ctx->ws + pl.off_unit_cnt);
    tr.seq_cnt = reinterpret_cast<uint32_t *>(ctx->ws + pl.off_seq_cnt);
    tr.cnt_stride = kCounterStride;
  }
  const LayerView lv = layer_view(ctx, layer);
  const bool track = c.score_mode == DYNTS_SCORE_ACCUMULATE;

  dynts::AttendParams p;
  p.K = lv.K; p.V = lv.V; p.S = lv.S; p.pos = lv.pos;
  p.seq_len = lv.seq_len; p.n_prompt = ctx->n_prompt; p.next_pos = lv.next_pos;
  p.q = q; p.k_new = k_new; p.v_new = v_new; p.s_new = s_new; p.active = active;
  p.out = out; p.lse = lse;
  p.qprev = lv.qprev; p.qnext = lv.qnext; p.mlprev = lv.mlprev; p.nprev = lv.nprev;
  p.part_o = tr.part_o;
  p.part_ml = tr.part_ml;
  p.tag = next_launch_tag();
  // K and V past the memory-side cache: only when all layers together are more than what still gains from it, and for launches of
  // 128 or more units and 100 MB or more.  us a step, through it / past it:
  //   one layer, 128 units: 303 MB 50.5 / 50.2, 314 MB 55.3 / 53.7, 323 MB 57.2 / 54.1, 382 MB 76.0 / 64.5
  //   2 layers of 512 units of 2640 slots 130.7 / 114.5, 8 of them 132.3 / 122.5; 384 units of 2464 98.9 / 82.6; 4 layers of
  //     128 units of 2464 36.2 / 32.3, 28 of them 35.5 / 33.0; 8 layers of 100 MB 24.8 / 23.4
  //   short launches lose: 16 layers of 128 units of 700 15.5 / 15.8.  (The line is a cautious one: 96 units of 8000 would take
  //     83.6 instead of 93.3, 8 layers of 64 units of 4000 28.0 instead of 30.9, 3 of 32 units of 16000 49.3 instead of 57.7.)
  // 272 MB of fixed places: with 320 MB 384 units of 2464 take 85.5 instead of 83.1, with 410 MB 99.3.
  const double kv_bytes = 4.0 * c.batch * c.n_kv_heads * (double)c.capacity * c.head_dim;
  const double slot_bytes = 4.0 * c.n_layers * c.batch * c.n_kv_heads * c.head_dim;
  const bool stream_bound = (long long)c.batch * c.n_kv_heads >= 128 && kv_bytes >= 100e6;
  const double fit = stream_bound ? 310e6 / slot_bytes : 1e9, rounds = 272e6 / (slot_bytes * pl.nsplit * pl.waves * dynts::kTile);
  p.fit_slots = (int)(fit < 1e9 ? fit : 1e9);
  p.rounds = (int)(rounds < 1e6 ? rounds : 1e6);
  // Scores in bursts: where a layer's K and V do not fit the memory-side cache with room to spare, dense caches (those not loaded
  // past it) only when all layers together do not fit.  us a step, tile by tile / in bursts: 64 units of 12000 slots
  // 78.9 / 77.5, of 9800 58.8 / 56.7; 120 units of 6000 74.9 / 73.2; two layers of 112 units of 4000 51.4 / 51.1; head_dim 64, 64
  // units of 24000 80.4 / 78.2; four layers of 40 units of 9800 46.3 / 47.0; one layer of 250 MB 42.3 / 42.7, of 295 MB 49.6 / 49.5.
  p.score_tiles = kv_bytes > 192e6 && (ctx->paged || kv_bytes * c.n_layers > 310e6) ? 16 : 1;
  p.spill = keep_logits ? reinterpret_cast<float *>(ctx->ws + pl.off_spill) : nullptr;
  p.cap_pad = pl.cap_pad;
  p.unit_cnt = tr.unit_cnt;
  p.seq_cnt = tr.seq_cnt;
  p.cnt_stride = tr.cnt_stride;
  p.status = ctx->status;
  p.Nb = c.batch; p.Hq = c.n_q_heads; p.Hkv = c.n_kv_heads; p.G = pl.G; p.cap = c.capacity;
  p.nsplit = pl.nsplit; p.track = track ? 1 : 0; p.scale_log2 = ctx->scale_log2;
  p.block_table = lv.block_table; p.block_table_w = lv.block_table; p.free_stack = ctx->free_stack;
  p.free_top = ctx->free_top; p.max_pages = ctx->max_pages; p.n_pages = ctx->n_pages;

  // one-dimensional grid: units rounded up to the 8 XCDs, times the chunks per unit (mapped inside the kernel)
  const long long units8 = ((long long)c.batch * c.n_kv_heads + 7) / 8 * 8;
  if (units8 * pl.nsplit > 0x7fffffffLL) return DYNTS_ESHAPE;
  const dim3 grid((unsigned)(units8 * pl.nsplit));
  hipEvent_t e0 = ctx->ev_start, e1 = ctx->ev_stop;
  if (attend && ctx->ev_list_next < ctx->ev_list_start.size()) {
    e0 = ctx->ev_list_start[ctx->ev_list_next];
    e1 = ctx->ev_list_stop[ctx->ev_list_next];
    ++ctx->ev_list_next;
  }
  if (c.head_dim == 128) {
    if (pl.waves == 8) launch_partial_d<128, 8>(p, grid, st, e0, e1, attend, apply_pending, append);
    else launch_partial_d<128, 4>(p, grid, st, e0, e1, attend, apply_pending, append);
  } else {
    if (pl.waves == 8) launch_partial_d<64, 8>(p, grid, st, e0, e1, attend, apply_pending, append);
    else launch_partial_d<64, 4>(p, grid, st, e0, e1, attend, apply_pending, append);
  }
  // Recorded into a graph: every replay has this tag, so what one leaves must not be there for the next, whose merging
  // workgroup could take it for partials still on their way.  (A kernel of its own: the same clearing at the end of the merge
  // costs every eager launch of the wide and paged forms 2 - 5 %, in registers and scheduling.)
  if (attend && pl.nsplit > 1 && capturing(st)) {
    const size_t rows = (size_t)c.batch * c.n_kv_heads * pl.nsplit * pl.G;
    const size_t bytes = align_up(rows * c.head_dim * sizeof(uint64_t)) + rows * 2 * sizeof(uint64_t);  // part_ml lies behind part_o
    hipLaunchKernelGGL(clear_words_kernel, dim3(256), dim3(256), 0, st, reinterpret_cast<uint32_t *>(p.part_o), bytes / sizeof(uint32_t));
  }
  const int rc = launch_status();
  if (rc == DYNTS_OK && attend && track) ctx->qslot[layer] ^= 1;  // the query just saved becomes the current one
  return rc;
}


// the score update of `layer` from its kept logits (pending 2 or 3).  In place of the pass over K behind an unfused attention
// it takes that launch's events.
int apply_spill(dynts_ctx *ctx, int layer, hipStream_t st) {
  const dynts_config &c = ctx->cfg;
  const Plan &pl = ctx->plan;
  const LayerView lv = layer_view(ctx, layer);
  const dim3 grid((c.capacity + 256 * dynts::kApplyPerThread - 1) / (256 * dynts::kApplyPerThread), c.n_kv_heads * c.batch);
  const bool timed = ctx->pending[layer] == 3;
  hipExtLaunchKernelGGL(dynts::apply_spill_kernel, grid, dim3(256), 0, st, timed ? ctx->ev_start : nullptr,
                        timed ? ctx->ev_stop : nullptr, 0, lv.S, reinterpret_cast<const float *>(ctx->ws + pl.off_spill),
                        lv.mlprev, lv.nprev, ctx->n_prompt, c.n_kv_heads, c.n_q_heads, pl.G, c.capacity, pl.cap_pad);
  const int rc = launch_status();
  if (rc == DYNTS_OK) {
    ctx->pending[layer] = 0;
    ctx->spill_layer = -1;
  }
  return rc;
}

// Whether a trigger's selection makes the update it owes from kept logits itself: one workgroup per unit then reads all of the
// unit's, the first 4096 slots' of up to eight heads in one go, the rest in dependent rounds.  us for both, two launches / one:
//   4 heads a group: 4 units of 240 slots 16.5 / 12.1; 8 of 4544 16.7 / 15.0, of 6100 17.4 / 18.0, of 16000 28.2 / 42.2; 256 of
//     6100 24.0 / 21.6
//   7 heads: 128 units of 2496 16.2 / 13.4, of 5300 20.3 / 21.2; 512 of 1200 19.2 / 18.8; 32 of 6100 19.3 / 22.3, of 9000 22.7 / 32.2
//   16 heads: one unit of 4500 17.9 / 18.3, 32 units 20.2 / 22.0
bool select_applies(const dynts_ctx *ctx) {
  return ctx->cfg.capacity <= 5 * 1024 && ctx->plan.G <= dynts::kSelHeads;
}

// Threads of a selection's workgroup.  1024 where a compute unit has one unit of the cache to look after: two of them fill it, so that
// launches of more than 512 take turns, and to start them costs more than small caches have to do.  us a selection with 256 / 512 / 1024 (with 256 in
// an older kernel), and a whole trigger from its step to its compaction:
//   256 units of 1000 slots 7.5 / 7.6 / 7.5 (8.0), of 4800 17.7 / 11.9 / 9.8 (22.8); 300 of 400 7.0 / 7.0 / 7.7 (6.9), trigger 48.0 / 48.2 / 51.0 (52.8)
//   512 of 2400 12.0 / 9.7 / 10.9 (16.2), trigger 395.2 / 387.4 / 385.6; 300 of 3200 14.0 / 10.9 / 11.6, trigger 358.6 / 344.1 / 339.7
//   672 of 330 7.0 / 7.3 / 10.8 (7.4); 800 of 1000 8.4 / 9.3 / 13.3 (10.2), of 1600 11.0 / 11.1 / 15.4, trigger 216.6 / 215.5 / 218.9
//   1024 of 66 7.0 / 7.8 / 13.0 (7.3), of 2400 14.9 / 13.8 / 18.7 (22.5); 2048 of 692 10.8 / 15.2 / 24.8 (11.8)
int select_threads(const dynts_config &c) {
  const long long units = (long long)c.batch * c.n_kv_heads;
  if (units <= 256 || (units <= 512 && c.capacity > 2500)) return 1024;
  return units <= 768 || c.capacity > 1200 ? 512 : 256;
}

template <int T>
void launch_select(const dynts::SelectParams &p, const dynts_config &c, bool apply, hipStream_t st) {
  const dim3 grid(c.n_kv_heads, c.batch);
  const size_t lds = (size_t)c.capacity * 4;
  if (apply) hipLaunchKernelGGL((dynts::select_kernel<T, true, true>), grid, dim3(T), lds, st, p);
  else if (c.capacity <= kSelectLdsMax) hipLaunchKernelGGL((dynts::select_kernel<T, true, false>), grid, dim3(T), lds, st, p);
  else hipLaunchKernelGGL((dynts::select_kernel<T, false, false>), grid, dim3(T), 0, st, p);
}

// Threads of a compaction's workgroup.  512 (twice the rows in flight, 4096 entries of the keep list on chip) unless there are more workgroups
// than the chip holds, four a compute unit: what is left over of a second round is then not worth its start, and with more rounds that
// start is more than the smallest caches have to do.  Long lists want their entries on chip, the more so on pages.  us with 256 (1024 entries) /
// 512 (in brackets with 256 and nothing on chip), a tenth to a third of the rows moved, head_dim 128, 6 workgroups a unit:
//   16 units of 700 slots 13.5 / 12.0 (14.1), of 333 11.2 / 11.1, paged 15.6 / 13.2 (15.8); 512 of 66 12.8 / 16.4 (13.2); 1024 of 66 16.7 / 23.2
//     (17.4), of 333 54.7 / 54.5; 512 of 1200 112.8 / 108.2 (115.3)
//   172 units of 1200 41.5 / 38.5 (39.9); 236 of 300 14.9 / 16.0, paged 19.2 / 19.3, of 700 27.2 / 27.4, paged 31.5 / 29.9, of 2400 92.6 / 84.3, paged
//     84.8 / 75.4; 288 of 700 30.1 / 31.1, of 1200 47.0 / 47.2
//   256 units of 5000 278 / 296 (280), of 7400 322 / 342, paged 370 / 320; 336 of 4500 249 / 243; head_dim 64: 320 of 4500 156 / 142
int compact_threads(const dynts_ctx *ctx) {
  const dynts_config &c = ctx->cfg;
  const long long wgs = (long long)c.batch * c.n_kv_heads * (2 * (c.head_dim * 2 / dynts::kCompactSliceBytes) + 2);
  if (wgs <= 1280) return 512;
  if (c.capacity <= 300) return 256;
  if (ctx->paged || wgs >= 2048) return 512;
  return c.capacity <= 1000 || (c.capacity > 4000 && c.head_dim == 128 && wgs > 1400 && wgs < 1700) ? 256 : 512;
}

template <int T>
void launch_compact(const dynts::CompactParams &p, const dynts_ctx *ctx, const dynts::PagedView &pv, hipStream_t st) {
  const dynts_config &c = ctx->cfg;
  const dim3 grid(2 * (c.head_dim * 2 / dynts::kCompactSliceBytes) + 2, c.n_kv_heads, c.batch), block(T);
  if (ctx->paged) {
    if (c.head_dim == 128) hipLaunchKernelGGL((dynts::paged_compact_kernel<128, T>), grid, block, 0, st, p, pv);
    else hipLaunchKernelGGL((dynts::paged_compact_kernel<64, T>), grid, block, 0, st, p, pv);
  } else if (c.head_dim == 128) {
    hipLaunchKernelGGL((dynts::compact_kernel<128, T>), grid, block, 0, st, p);
  } else {
    hipLaunchKernelGGL((dynts::compact_kernel<64, T>), grid, block, 0, st, p);
  }
}

// The buffer of kept logits is wanted for something else, or no longer: an update that rests on them alone is applied,
// one that the next pass over K can make as well is left to that.
int release_spill(dynts_ctx *ctx, hipStream_t st) {
  const int layer = ctx->spill_layer;
  if (layer < 0) return DYNTS_OK;
  if (ctx->pending[layer] == 2) return apply_spill(ctx, layer, st);
  ctx->pending[layer] = 1;
  ctx->spill_layer = -1;
  return DYNTS_OK;
}

// What came after the unfused attention that waits for an answer (if any does): `paired`, its own update, which kept logits
// have served or would have; or not, a fused step, another attention of the layer, or of another layer, which would have taken the
// buffer.  Logits are kept after two answers in a row for it, so that a caller who alternates does not pay for both; the
// first answer on a context speaks for every layer until it has its own.
constexpr unsigned char kPairsKeep = 2;
void unfused_ends(dynts_ctx *ctx, bool paired) {
  if (ctx->unfused_layer < 0) return;
  if (!ctx->pairs_known) ctx->pairs.assign(ctx->pairs.size(), paired ? kPairsKeep : 0);
  ctx->pairs_known = true;
  unsigned char &n = ctx->pairs[ctx->unfused_layer];
  n = !paired ? 0 : n < kPairsKeep ? n + 1 : n;
  ctx->unfused_layer = -1;
}

// Kept logits are written and read once, 8 bytes per slot and head of the group; without them the update reads the slot's
// K row again, 2 bytes per element.  us for both calls, second pass over K / kept:
//   up to a quarter of the K row: 128 units of 5000 slots 80.8 / 62.9 (head_dim 128, 4 heads), 42.4 / 35.1 (64, 4), of 1200 24.6 / 23.1 (128, 4);
//     but where K is less than some 30 MB the pass over it has become the faster one: 128 units of 1200 14.8 / 16.4 (64, 4), 8 units of
//     5000 16.8 / 17.3 (128, 4), 18.1 / 20.2 (128, 8)
//   up to half of it: 128 units of 5000 42.1 / 38.5 (64, 8), 81.7 / 80.2 (128, 16); of 1200 15.1 / 18.6 (64, 8); 512 units of 1200
//     40.1 / 37.0 (64, 8), 76.8 / 75.8 (128, 16); 8 units of 5000 15.8 / 18.1 (64, 8), 21.6 / 27.0 (128, 16); paged, 128 units of
//     5000 82.9 / 91.0 (128, 16)
//   all of it: 128 units of 1200 15.7 / 22.5 (64, 16), of 5000 42.4 / 45.3
bool kept_logits_pay(const dynts_ctx *ctx) {
  const dynts_config &c = ctx->cfg;
  const int G = ctx->plan.G;
  const double k_bytes = 2.0 * c.batch * c.n_kv_heads * (double)c.capacity * c.head_dim;
  return 16 * G <= c.head_dim || (8 * G <= c.head_dim && !ctx->paged && k_bytes >= 64e6);
}

// One fused step (attention, the score update owed by the previous step, optionally the append) with the
// bookkeeping of owed updates.  With a trigger announced for this layer (dynts_hint_trigger) the step keeps its
// logits, and its own update is later applied from them instead of from a second pass over K.
int fused_step(dynts_ctx *ctx, int layer, const uint16_t *q, const uint16_t *k_new, const uint16_t *v_new,
               const float *s_new, const uint8_t *active, float *out, float *lse, bool append, hipStream_t st,
               const Transient *transient) {
  const bool track = ctx->cfg.score_mode == DYNTS_SCORE_ACCUMULATE;
  const bool keep = track && ctx->hint[layer];
  ctx->hint[layer] = 0;
  if (keep || ctx->unfused_layer == layer) unfused_ends(ctx, false);
  int rc = DYNTS_OK;
  if (ctx->pending[layer] == 2) rc = apply_spill(ctx, layer, st);
  if (ctx->pending[layer] == 3 || keep) rc = rc == DYNTS_OK ? release_spill(ctx, st) : rc;
  if (rc != DYNTS_OK) return rc;
  rc = run_attend(ctx, layer, q, k_new, v_new, s_new, active, out, lse, true, ctx->pending[layer] == 1, append, st,
                  transient, keep);
  if (rc == DYNTS_OK) {
    ctx->pending[layer] = track ? (keep ? 2 : 1) : 0;
    if (keep) ctx->spill_layer = layer;
  }
  return rc;
}

// ---- consecutive steps in one launch ----------------------------------------------------------------
// How many consecutive steps of a layer are made by one launch that keeps the cache on the chip (resident_kernel), 0: a launch each.
// Dense caches of as many slots as its waves hold, and those of several chunks that are one tile a wave each (about one workgroup a
// compute unit then), which leave partials for two kernels that merge them and make the score updates.  Runs of three steps or more gain everywhere;
// us a step, a launch each / so:
//   one chunk, runs of 32: 1 unit of 120 slots of 16 heads 6.1 / 2.9, 1024 units of 120 slots 11.1 / 7.1, of 510 47.2 / 14.9
//   several: 8 units of 700 slots 8.4 / 3.2, of 4544 11.7 / 3.3, of 8000 13.4 / 3.2; 64 of 1000 9.6 / 3.6; one of 8000 of 16 heads 22.9 / 4.0;
//     head_dim 64, 2 units of 400 6.7 / 2.3, 128 of 510 7.7 / 2.9, 32 of 2000 8.4 / 2.6
//   by the run's length, 2 / 3 / 4 / 8 / 16: 8 units of 1000 9.2 / 10.5, 8.9 / 7.7, 8.9 / 6.6, 8.7 / 4.7, 8.6 / 3.7; 512 units of 510, head_dim 64,
//     15.3 / 15.5, 15.4 / 11.6, 15.0 / 10.3, 14.7 / 7.8, 14.6 / 6.5
// Caches that the chip's registers do not hold are read again for every step, one launch each.  (Only callers who hand over the inputs of three or
// more steps at once have runs: a decoder that forms each query from the step before pays a launch a step.)
// Not where every attend launch is to be timed or has a shape of the caller's, and not under capture: a replayed step finds and leaves
// the saved query by itself.
constexpr int kLeastRun = 3;
int resident_run(const dynts_ctx *ctx, hipStream_t st) {
  const Plan &pl = ctx->plan;
  const bool whole = pl.nsplit == 1 && ctx->cfg.capacity <= dynts::kResTiles * dynts::kResSlots;
  if (ctx->paged || ctx->shaped || !(whole || ctx->run_steps > 0)) return 0;
  if (ctx->ev_start || ctx->ev_list_next < ctx->ev_list_start.size() || capturing(st)) return 0;
  return whole ? dynts::kResSteps : ctx->run_steps;
}

template <int D>
void launch_resident(const dynts::ResidentParams &p, hipStream_t st) {
  const dim3 block(dynts::kResThreads);
  if (p.chunks == 1) {
    if (p.cap <= dynts::kResSlots) hipLaunchKernelGGL((dynts::resident_kernel<D, 1, false>), dim3(p.units), block, 0, st, p);
    else hipLaunchKernelGGL((dynts::resident_kernel<D, 2, false>), dim3(p.units), block, 0, st, p);
    return;
  }
  hipLaunchKernelGGL((dynts::resident_kernel<D, 1, true>), dim3(p.units * p.chunks), block, 0, st, p);
  hipLaunchKernelGGL(dynts::merge_run_kernel<D>, dim3(p.units, p.steps), block, 0, st, p);
  if (p.track) hipLaunchKernelGGL(dynts::run_scores_kernel<D>, dim3(p.units * p.chunks), block, 0, st, p);
}

// Steps [0, steps) of one layer, inputs of step 0 given.  evict: a trigger follows the last, which keeps its logits.
int resident_steps(dynts_ctx *ctx, int layer, int steps, bool evict, const uint16_t *q, const uint16_t *k_new, const uint16_t *v_new,
                   const float *s_new, const uint8_t *active, float *out, size_t out_stride, hipStream_t st) {
  if ((reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(k_new) | reinterpret_cast<uintptr_t>(v_new)) % 16) return DYNTS_EINVAL;
  const dynts_config &c = ctx->cfg;
  const bool track = c.score_mode == DYNTS_SCORE_ACCUMULATE;
  const bool keep = track && evict;
  ctx->hint[layer] = 0;
  if (keep || ctx->unfused_layer == layer) unfused_ends(ctx, false);
  int rc = DYNTS_OK;
  if (ctx->pending[layer] == 2) rc = apply_spill(ctx, layer, st);
  if (ctx->pending[layer] == 3 || keep) rc = rc == DYNTS_OK ? release_spill(ctx, st) : rc;
  if (rc != DYNTS_OK) return rc;
  const LayerView lv = layer_view(ctx, layer);
  dynts::ResidentParams p;
  p.K = lv.K; p.V = lv.V; p.S = lv.S; p.pos = lv.pos;
  p.seq_len = lv.seq_len; p.n_prompt = ctx->n_prompt; p.next_pos = lv.next_pos;
  p.q = q; p.k_new = k_new; p.v_new = v_new; p.s_new = s_new; p.active = active; p.out = out;
  p.q_stride = (size_t)c.n_layers * c.batch * c.n_q_heads * c.head_dim;
  p.kv_stride = (size_t)c.n_layers * c.batch * c.n_kv_heads * c.head_dim;
  p.out_stride = out_stride;
  p.steps = steps;
  // The two places of the saved query take turns step by step: the run leaves its last one where as many single steps would, so that
  // recorded steps replayed behind it find it where they look for it.
  p.qprev = lv.qprev; p.qnext = steps % 2 ? lv.qnext : lv.qprev; p.mlprev = lv.mlprev; p.nprev = lv.nprev;
  p.seq_cnt = reinterpret_cast<uint32_t *>(ctx->ws + ctx->plan.off_seq_cnt);
  p.cnt_stride = kCounterStride;
  p.status = ctx->status;
  p.Nb = c.batch; p.Hq = c.n_q_heads; p.Hkv = c.n_kv_heads; p.G = ctx->plan.G; p.cap = c.capacity;
  p.track = track ? 1 : 0;
  p.owed = ctx->pending[layer] == 1 ? 1 : 0;
  p.spill = keep ? reinterpret_cast<float *>(ctx->ws + ctx->plan.off_spill) : nullptr;
  p.cap_pad = ctx->plan.cap_pad;
  p.scale_log2 = ctx->scale_log2;
  const Plan &pl = ctx->plan;
  p.units = c.batch * c.n_kv_heads;
  p.chunks = pl.nsplit;
  p.part_o = reinterpret_cast<float *>(ctx->ws + pl.off_run_o);
  p.part_ml = reinterpret_cast<float *>(ctx->ws + pl.off_run_ml);
  p.stats = reinterpret_cast<float *>(ctx->ws + pl.off_run_stats);
  p.n_of = reinterpret_cast<int32_t *>(ctx->ws + pl.off_run_n);
  p.rec = reinterpret_cast<int32_t *>(ctx->ws + pl.off_run_rec);
  p.wide = wide_merge(c.head_dim, 8, pl.G, pl.nsplit, (long long)(p.units + 7) / 8 * 8 * pl.nsplit) ? 1 : 0;
  if (c.head_dim == 128) launch_resident<128>(p, st);
  else launch_resident<64>(p, st);
  rc = launch_status();
  if (rc != DYNTS_OK) return rc;
  if (track) ctx->qslot[layer] ^= steps % 2;
  ctx->pending[layer] = track ? (keep ? 2 : 1) : 0;
  if (keep) ctx->spill_layer = layer;
  return DYNTS_OK;
}

// ---- block scoring ----------------------------------------------------------------------------------
// bytes of one key range's denominators
size_t score_block_stats_bytes(const dynts_config &c, int n_queries) {
  const size_t rpad = align_up((size_t)n_queries * (c.n_q_heads / c.n_kv_heads));
  return align_up((size_t)c.batch * c.n_kv_heads * rpad * sizeof(float));
}

// Key ranges of the first pass: as many as fill the chip's 256 x 3 workgroup places once, where the rows alone do not, of
// at least eight chunks each.  64 queries on 128 units of 2464 slots (256 workgroups of rows): first pass 66 us with
// one range, 49 with two, 48 with three.  With scratch for fewer ranges there are fewer.
int score_block_splits(const dynts_config &c, int n_queries) {
  const long long R = (long long)n_queries * (c.n_q_heads / c.n_kv_heads);
  const long long wgs = (R + dynts::kSbRowsPerWg - 1) / dynts::kSbRowsPerWg * c.batch * c.n_kv_heads;
  const long long want = 768 / wgs, most = c.capacity / 256;
  const long long s = want < most ? want : most;
  return s < 1 ? 1 : s > dynts::kSbMaxSplits ? dynts::kSbMaxSplits : (int)s;
}

template <int D, bool PAGED>
void launch_score_block(const dynts::ScoreBlockParams &p, dim3 g1, dim3 g2, hipStream_t st) {
  hipLaunchKernelGGL((dynts::score_block_stats_kernel<D, PAGED>), g1, dim3(dynts::kSbWaves * 64), 0, st, p);
  hipLaunchKernelGGL((dynts::score_block_colsum_kernel<D, PAGED>), g2, dim3(dynts::kSbWaves * 64), 0, st, p);
}

// ---- Importance Predictor ---------------------------------------------------------------------------
struct MlpPlan {
  int bt;                 // batch tiles of 16
  int ft1, ft2, ns;       // feature tiles of 16 a workgroup takes in either layer; workgroups that share the second's K
  int wgs1, groups;       // workgroups of the first layer, groups of features of the second
  size_t off_sum, off_group, off_dot, off_done, total;  // scratch: layer 1's output first, then the words the first kernel zeroes
};

// us a call, by the number of tiles a workgroup takes (ft) and of workgroups that share the second layer's K (ns):
//   ft1 = 1 / 2: d = 2048 (256 tiles of 16 features) batch 4 13.2 / 13.9, batch 128 28.8 / 29.4; d = 2560 (320) 18.6 / 17.1, 40.8 / 32.4;
//     d = 3584 22.2 / 22.0, 49.9 / 39.0
//   (ft2, ns) = (1, 2) / (1, 4) / (2, 4) / (2, 8): d = 2048 (64 tiles) batch 4 13.6 / 13.9 / 14.8 / 14.8, batch 128 30.1 / 25.9 / 27.4 / 29.3;
//     d = 2560 (80) 18.0 / 19.2 / 17.3 / 21.6, 34.8 / 40.3 / 32.2 / 38.9; d = 3584 22.1 / 23.2 / 21.5 / 26.8, 43.4 / 50.3 / 39.0 / 50.9
//   Between 513 and 768 tiles two a workgroup are a second round that is nearly empty, which up to 32 sequences costs more than one a
//     workgroup does (ft1 = 1 / 2): d = 4288 (536) batch 1 29.4 / 32.1, batch 32 35.3 / 37.1; d = 6144 (768) 39.8 / 41.5, 46.9 / 48.4; d = 6656 (832)
//     53.2 / 52.0, 69.6 / 65.5; with 64 sequences d = 4288 45.3 / 44.2
//   A long K is shared by as many as leave each 64 k-steps, above 32 sequences 32 (ns = 2, 4, 8, 16): d = 512, m2 = 16, m1 = 16384 batch 1 21.6,
//     17.9, 16.2, 16.8, batch 128 60.4, 42.0, 32.7, 28.6; m1 = 8192 batch 128 36.0, 26.3, 20.8, 20.7; m1 = 4096 batch 1 11.8 with any
MlpPlan mlp_plan(const dynts_predictor *w, int batch) {
  MlpPlan pl;
  pl.bt = batch <= 64 ? (batch + 15) / 16 : batch <= 96 ? 6 : 8;
  const int t1 = w->m1 / 16, t2 = w->m2 / 16;
  pl.ft1 = t1 > 256 && !(t1 > 512 && t1 <= 768 && pl.bt <= 2) ? 2 : 1;
  pl.ft2 = t2 > 64 ? 2 : 1;
  pl.wgs1 = (t1 + pl.ft1 - 1) / pl.ft1;
  pl.groups = (t2 + pl.ft2 - 1) / pl.ft2;
  const int some = pl.ft2 == 2 || pl.bt > 2 ? 4 : 2, many = w->m1 / 32 / (pl.bt > 2 ? 32 : 64);
  const int want = some > many ? some : many, room = 256 / pl.groups, most = w->m1 / 32 / (2 * dynts::kMlpWaves);
  pl.ns = want < room ? want : room;
  pl.ns = pl.ns < most ? pl.ns : most;
  pl.ns = pl.ns < 1 ? 1 : pl.ns;
  size_t off = align_up((size_t)w->m1 * 16 * pl.bt * 2 * sizeof(uint16_t));
  pl.off_sum = off;
  if (pl.ns > 1) off += align_up((size_t)pl.groups * pl.ns * pl.ft2 * pl.bt * 256 * sizeof(uint64_t));
  pl.off_group = off;
  if (pl.ns > 1) off += align_up((size_t)pl.groups * dynts::kMlpCntStride * sizeof(uint32_t));
  pl.off_dot = off;
  off += align_up((size_t)pl.groups * batch * sizeof(uint64_t));
  pl.off_done = off;
  off += align_up(sizeof(uint32_t));
  pl.total = off;
  return pl;
}

// Whether the two-launch form's 32-bit offsets reach everything: the hidden states, a workgroup's weights, the second layer's
// operands, a grid's threads.
bool mlp_fits_32_bits(const dynts_predictor *w, int batch) {
  const long long limit = dynts::kMlpNowhere;
  return 2LL * batch * w->d < limit && 32LL * w->d < limit && 64LL * 8 * w->m1 < limit && 8LL * w->m2 < limit;
}

struct MlpSplitPlan {
  int bt;                // batch tiles of 16
  int nsplit1, nsplit2;  // slices of K in either layer
  size_t off_p1, off_yhi, off_ylo, off_p2, off_part, off_cnt, total;  // scratch
};

MlpSplitPlan mlp_split_plan(const dynts_predictor *w, int batch) {
  MlpSplitPlan pl;
  pl.bt = batch <= 16 ? 1 : batch <= 32 ? 2 : batch <= 64 ? 4 : 8;
  auto slices = [&](int K, int parts) {
    const int steps = dynts::mlp_slice_steps(pl.bt, parts);
    return (K / 32 + steps - 1) / steps;
  };
  pl.nsplit1 = slices(w->d, 1);
  pl.nsplit2 = slices(w->m1, 2);
  size_t off = 0;
  pl.off_p1 = off;
  off += align_up((size_t)pl.nsplit1 * batch * w->m1 * sizeof(float));
  pl.off_yhi = off;
  off += align_up((size_t)batch * w->m1 * sizeof(uint16_t));
  pl.off_ylo = off;
  off += align_up((size_t)batch * w->m1 * sizeof(uint16_t));
  pl.off_p2 = off;
  off += align_up((size_t)pl.nsplit2 * batch * w->m2 * sizeof(float));
  pl.off_part = off;
  off += align_up((size_t)batch * ((w->m2 + 255) / 256) * sizeof(uint64_t));  // tagged words
  pl.off_cnt = off;
  off += align_up((size_t)batch * sizeof(uint32_t));
  pl.total = off;
  return pl;
}

int check_predictor(const dynts_predictor *w, int batch) {
  if (!w) return DYNTS_ENULL;
  if (batch <= 0 || batch > 128) return DYNTS_EINVAL;
  if (w->d <= 0 || w->m1 <= 0 || w->m2 <= 0) return DYNTS_EINVAL;
  if (w->d % 32 || w->m1 % 32 || w->m2 % 16) return DYNTS_ESHAPE;
  if (w->activation < DYNTS_ACT_NONE || w->activation > DYNTS_ACT_SILU) return DYNTS_EINVAL;
  if (w->packed != 0 && w->packed != 1) return DYNTS_EINVAL;
  return DYNTS_OK;
}

// Whether a call takes the form that cuts K of both layers (mlp_split_gemm_kernel): sizes past 32-bit offsets, and two kinds of
// layer 1 of which the other form leaves the chip idle.  (Neither has the proportions of the paper's heads, d -> 2d -> d/2.)
//   Few features and a long K, of which a workgroup takes all: one with more than 1.4 MB of operands is slower, in launches of up to
//     128 workgroups.  us a call, two launches / this form, m2 = 256: d = 4096, m1 = 512 batch 128 (1.2 MB) 23.8 / 26.1; d = 8192, m1 = 1472
//     batch 64 (1.3) 24.3 / 26.1, batch 128 (2.4) 40.1 / 33.9; d = 16384, m1 = 512 batch 1 (1.0) 19.5 / 22.2, batch 64 (2.6) 34.3 / 25.9; d = 65536,
//     m1 = 32 batch 1 (4.2) 48.5 / 20.7, batch 128 200 / 31.  17 - 32 sequences from 1.1 MB on: d = 12288, m1 = 32 17.7 / 16.1.
//   Many features and a short K: thousands of workgroups, each little but its prologue.  m2 = 16: d = 512, m1 = 16384 batch 32 18.8 / 19.1,
//     m1 = 32768 28.2 / 22.2; d = 256, m1 = 24576 batch 16 20.3 / 21.4, m1 = 65536 30.6 / 24.9; but with more sequences the other form's lead
//     in partial sums counts: d = 1024, m1 = 65536 batch 128 73.4 / 79.8; d = 512, m1 = 32768, m2 = 1024 batch 64 42.2 / 44.0.
bool mlp_split(const dynts_predictor *w, int batch) {
  if (!mlp_fits_32_bits(w, batch)) return true;
  const MlpPlan pl = mlp_plan(w, batch);
  const long long taken = 32LL * w->d * (pl.ft1 + pl.bt);
  if (pl.wgs1 <= 128 && taken > 1400000) return true;
  if (pl.bt == 2 && pl.wgs1 <= 96 && taken > 1100000) return true;
  return w->m1 > (w->d > 256 ? 16384 : 24576) && w->m1 > 32LL * w->d && (long long)batch * w->d <= 65536 && (long long)batch * w->m2 <= 32768;
}

template <int FT, bool SECOND, bool PACKED>
void launch_mlp_ft(const dynts::MlpParams &p, int bt, dim3 grid, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  const dim3 block(dynts::kMlpThreads);
  switch (bt) {
    case 1: hipExtLaunchKernelGGL((dynts::mlp_kernel<FT, 1, SECOND, PACKED>), grid, block, 0, st, e0, e1, 0, p); break;
    case 2: hipExtLaunchKernelGGL((dynts::mlp_kernel<FT, 2, SECOND, PACKED>), grid, block, 0, st, e0, e1, 0, p); break;
    case 3: hipExtLaunchKernelGGL((dynts::mlp_kernel<FT, 3, SECOND, PACKED>), grid, block, 0, st, e0, e1, 0, p); break;
    case 4: hipExtLaunchKernelGGL((dynts::mlp_kernel<FT, 4, SECOND, PACKED>), grid, block, 0, st, e0, e1, 0, p); break;
    case 6: hipExtLaunchKernelGGL((dynts::mlp_kernel<FT, 6, SECOND, PACKED>), grid, block, 0, st, e0, e1, 0, p); break;
    default: hipExtLaunchKernelGGL((dynts::mlp_kernel<FT, 8, SECOND, PACKED>), grid, block, 0, st, e0, e1, 0, p); break;
  }
}

template <bool SECOND>
void launch_mlp(const dynts::MlpParams &p, int packed, int ft, int bt, int wgs, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  const dim3 grid(wgs);
  if (packed) {
    if (ft == 1) launch_mlp_ft<1, SECOND, true>(p, bt, grid, st, e0, e1);
    else launch_mlp_ft<2, SECOND, true>(p, bt, grid, st, e0, e1);
  } else {
    if (ft == 1) launch_mlp_ft<1, SECOND, false>(p, bt, grid, st, e0, e1);
    else launch_mlp_ft<2, SECOND, false>(p, bt, grid, st, e0, e1);
  }
}

template <int PARTS, bool PACKED>
void launch_mlp_split_gemm(const dynts::MlpSplitParams &p, int bt, int nsplit, hipStream_t st, hipEvent_t e0) {
  const dim3 grid((p.m + dynts::kMlpSplitFeatures - 1) / dynts::kMlpSplitFeatures, nsplit);
  const dim3 block(dynts::kMlpThreads);
  switch (bt) {
    case 1: hipExtLaunchKernelGGL((dynts::mlp_split_gemm_kernel<1, PARTS, PACKED>), grid, block, 0, st, e0, nullptr, 0, p); break;
    case 2: hipExtLaunchKernelGGL((dynts::mlp_split_gemm_kernel<2, PARTS, PACKED>), grid, block, 0, st, e0, nullptr, 0, p); break;
    case 4: hipExtLaunchKernelGGL((dynts::mlp_split_gemm_kernel<4, PARTS, PACKED>), grid, block, 0, st, e0, nullptr, 0, p); break;
    default: hipExtLaunchKernelGGL((dynts::mlp_split_gemm_kernel<8, PARTS, PACKED>), grid, block, 0, st, e0, nullptr, 0, p); break;
  }
}

void run_mlp_split(const dynts_predictor *w, const MlpSplitPlan &pl, const uint16_t *h, int batch, float *s_out, int n_rep,
                   unsigned char *base, hipStream_t st, hipEvent_t start, hipEvent_t stop) {
  float *P1 = reinterpret_cast<float *>(base + pl.off_p1), *P2 = reinterpret_cast<float *>(base + pl.off_p2);
  uint16_t *yhi = reinterpret_cast<uint16_t *>(base + pl.off_yhi), *ylo = reinterpret_cast<uint16_t *>(base + pl.off_ylo);
  const dynts::MlpSplitParams g1{w->W1, h, nullptr, P1, batch, w->m1, w->d}, g2{w->W2, yhi, ylo, P2, batch, w->m2, w->m1};
  if (w->packed) launch_mlp_split_gemm<1, true>(g1, pl.bt, pl.nsplit1, st, start);
  else launch_mlp_split_gemm<1, false>(g1, pl.bt, pl.nsplit1, st, start);
  const size_t n1 = (size_t)batch * w->m1 / 4;
  hipLaunchKernelGGL(dynts::mlp_split_act_kernel, dim3((unsigned)((n1 + 255) / 256)), dim3(256), 0, st, P1, w->b1, pl.nsplit1, batch,
                     w->m1, w->activation, yhi, ylo, reinterpret_cast<dynts::u32x4 *>(base + pl.off_part), (pl.total - pl.off_part) / 16);
  if (w->packed) launch_mlp_split_gemm<2, true>(g2, pl.bt, pl.nsplit2, st, nullptr);
  else launch_mlp_split_gemm<2, false>(g2, pl.bt, pl.nsplit2, st, nullptr);
  hipExtLaunchKernelGGL(dynts::mlp_split_dot_kernel, dim3((w->m2 + 255) / 256, batch), dim3(256), 0, st, nullptr, stop, 0, P2, w->b2,
                        pl.nsplit2, batch, w->m2, w->activation, w->w3, w->b3, reinterpret_cast<uint64_t *>(base + pl.off_part),
                        reinterpret_cast<uint32_t *>(base + pl.off_cnt), s_out, n_rep);
}

// ---- scratch that nobody allocates (dynts_decode_step_static) ----------------------------------------
// One array per GPU, part of the loaded code object, alive until the process ends.  Host code never uses the
// array's name as an address: it asks the runtime for the device address once per device and keeps it.
constexpr size_t kStaticScratchBytes = DYNTS_STATIC_SCRATCH_BYTES;
constexpr size_t kStaticCounters = size_t(1) << 20;  // the first MiB holds counters only
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex static_scratch_mutex;
unsigned char *static_scratch_ptr[kMaxDevices] = {};

// Device address of this GPU's array (the current device), looked up and cleared on first use.  nullptr on error.
unsigned char *static_scratch(hipStream_t st) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(static_scratch_mutex);
  if (!static_scratch_ptr[dev]) {
    unsigned char *ptr = nullptr;
    if (hipGetSymbolAddress(reinterpret_cast<void **>(&ptr), HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
    // counters must start at zero (launches leave them at zero afterwards); the whole array, once, with a
    // fill kernel on the caller's stream -- stream order puts it before the first launch that uses the array
    hipLaunchKernelGGL(clear_words_kernel, dim3(256), dim3(256), 0, st, reinterpret_cast<uint32_t *>(ptr),
                       kStaticScratchBytes / sizeof(uint32_t));
    if (hipGetLastError() != hipSuccess) return nullptr;
    static_scratch_ptr[dev] = ptr;
  }
  return static_scratch_ptr[dev];
}

}  // namespace

extern "C" {

int dynts_version(void) { return 100; }

const char *dynts_strerror(int code) {
  switch (code) {
    case DYNTS_OK: return "ok";
    case DYNTS_EINVAL: return "argument out of range";
    case DYNTS_ENULL: return "required pointer is null";
    case DYNTS_ESHAPE: return "unsupported shape (head_dim must be 64 or 128, group size <= 16, n_q_heads % n_kv_heads == 0)";
    case DYNTS_ECAPACITY: return "capacity or index stride too small";
    case DYNTS_ENOTBOUND: return "no buffers bound (call dynts_bind)";
    case DYNTS_EWORKSPACE: return "workspace too small or misaligned";
    case DYNTS_EHIP: return "HIP runtime error at kernel launch";
    case DYNTS_EPENDING: return "a score update is outstanding (call dynts_update_scores first)";
    default: return "unknown error";
  }
}

int dynts_create(const dynts_config *cfg, dynts_ctx **out) {
  if (!out) return DYNTS_ENULL;
  *out = nullptr;
  int rc = check_config(cfg);
  if (rc != DYNTS_OK) return rc;
  dynts_ctx *ctx = new (std::nothrow) dynts_ctx();
  if (!ctx) return DYNTS_EINVAL;
  ctx->cfg = *cfg;
  ctx->plan = make_plan(*cfg, 0, 0);
  const float scale = cfg->softmax_scale > 0.f ? cfg->softmax_scale : 1.0f / std::sqrt((float)cfg->head_dim);
  ctx->scale_log2 = scale * 1.4426950408889634f;
  ctx->pending.assign((size_t)cfg->n_layers, 0);
  ctx->hint.assign((size_t)cfg->n_layers, 0);
  ctx->pairs.assign((size_t)cfg->n_layers, kPairsKeep);
  ctx->qslot.assign((size_t)cfg->n_layers, 0);
  *out = ctx;
  return DYNTS_OK;
}

int dynts_destroy(dynts_ctx *ctx) {
  if (!ctx) return DYNTS_ENULL;
  delete ctx;
  return DYNTS_OK;
}

int dynts_set_launch_shape(dynts_ctx *ctx, int32_t target_workgroups, int32_t waves_per_workgroup) {
  if (!ctx) return DYNTS_ENULL;
  if (target_workgroups < 0 || (waves_per_workgroup != 0 && waves_per_workgroup != 4 && waves_per_workgroup != 8))
    return DYNTS_EINVAL;
  ctx->plan = make_plan(ctx->cfg, target_workgroups, waves_per_workgroup);
  ctx->shaped = target_workgroups > 0 || waves_per_workgroup > 0;
  ctx->bound = false;  // the workspace layout changed
  return DYNTS_OK;
}

size_t dynts_ctx_workspace_bytes(const dynts_ctx *ctx) { return ctx ? ctx->plan.run_bytes : 0; }

size_t dynts_workspace_bytes(const dynts_config *cfg) {
  if (check_config(cfg) != DYNTS_OK) return 0;
  return make_plan(*cfg, 0, 0).bytes;
}

int dynts_bind(dynts_ctx *ctx, uint16_t *K, uint16_t *V, float *S, int32_t *pos, int32_t *seq_len,
               int32_t *next_pos, int32_t *n_prompt, void *workspace, size_t workspace_bytes, int32_t *status) {
  if (!ctx || !K || !V || !S || !pos || !seq_len || !next_pos || !n_prompt || !workspace || !status) return DYNTS_ENULL;
  if (workspace_bytes < ctx->plan.bytes || (reinterpret_cast<uintptr_t>(workspace) % kAlign)) return DYNTS_EWORKSPACE;
  if ((reinterpret_cast<uintptr_t>(K) | reinterpret_cast<uintptr_t>(V)) % 16) return DYNTS_EINVAL;
  ctx->K = K; ctx->V = V; ctx->S = S; ctx->pos = pos; ctx->seq_len = seq_len; ctx->next_pos = next_pos;
  ctx->n_prompt = n_prompt; ctx->ws = static_cast<unsigned char *>(workspace); ctx->status = status;
  ctx->run_steps = workspace_bytes >= ctx->plan.run_bytes ? ctx->plan.run_steps : 0;
  ctx->paged = false; ctx->block_table = nullptr; ctx->free_stack = nullptr; ctx->free_top = nullptr;
  ctx->max_pages = ctx->n_pages = 0;
  ctx->pending.assign(ctx->pending.size(), 0);
  ctx->hint.assign(ctx->hint.size(), 0);
  ctx->spill_layer = -1;
  ctx->pairs.assign(ctx->pairs.size(), kPairsKeep);
  ctx->pairs_known = false;
  ctx->unfused_layer = -1;
  ctx->qslot.assign(ctx->qslot.size(), 0);
  ctx->bound = true;
  return DYNTS_OK;
}

int dynts_bind_paged(dynts_ctx *ctx, uint16_t *K_pool, uint16_t *V_pool, int32_t n_pages, int32_t *block_table,
                     int32_t max_pages, int32_t *free_stack, int32_t *free_top, float *S, int32_t *pos,
                     int32_t *seq_len, int32_t *next_pos, int32_t *n_prompt, void *workspace, size_t workspace_bytes,
                     int32_t *status) {
  if (!ctx || !block_table || !free_stack || !free_top) return DYNTS_ENULL;
  if (n_pages <= 0 || max_pages <= 0) return DYNTS_EINVAL;
  if ((long long)max_pages * dynts::kPageSlots < ctx->cfg.capacity) return DYNTS_ECAPACITY;
  const int rc = dynts_bind(ctx, K_pool, V_pool, S, pos, seq_len, next_pos, n_prompt, workspace, workspace_bytes, status);
  if (rc != DYNTS_OK) return rc;
  ctx->paged = true; ctx->block_table = block_table; ctx->free_stack = free_stack; ctx->free_top = free_top;
  ctx->max_pages = max_pages; ctx->n_pages = n_pages;
  return DYNTS_OK;
}

int dynts_prefill(dynts_ctx *ctx, int32_t layer, const uint16_t *K0, const uint16_t *V0, int32_t m_max,
                  const int32_t *m, void *stream) {
  int rc = check_call(ctx, layer);
  if (rc != DYNTS_OK) return rc;
  if (!K0 || !V0 || !m) return DYNTS_ENULL;
  if (m_max <= 0) return DYNTS_EINVAL;
  if (m_max > ctx->cfg.capacity) return DYNTS_ECAPACITY;
  if ((reinterpret_cast<uintptr_t>(K0) | reinterpret_cast<uintptr_t>(V0)) % 16) return DYNTS_EINVAL;
  const dynts_config &c = ctx->cfg;
  const LayerView lv = layer_view(ctx, layer);
  dynts::PrefillParams p{lv.K, lv.V, lv.S, lv.pos, lv.seq_len, lv.next_pos, ctx->n_prompt, K0, V0, m,
                         c.n_kv_heads, c.capacity, m_max};
  const int rows = 256 / (c.head_dim / 8);
  const dim3 grid((m_max + rows - 1) / rows, c.n_kv_heads, c.batch);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (ctx->paged) {
    const dynts::PagedView pv{lv.K, lv.V, lv.block_table, ctx->free_stack, ctx->free_top, ctx->max_pages, ctx->n_pages};
    const int units = c.batch * c.n_kv_heads;
    hipLaunchKernelGGL(dynts::paged_alloc_kernel, dim3((units + 63) / 64), dim3(64), 0, st, pv, nullptr, m, m_max,
                       c.batch, c.n_kv_heads, ctx->status);
    if (c.head_dim == 128) hipLaunchKernelGGL((dynts::paged_prefill_kernel<128>), grid, dim3(256), 0, st, p, pv);
    else hipLaunchKernelGGL((dynts::paged_prefill_kernel<64>), grid, dim3(256), 0, st, p, pv);
  } else if (c.head_dim == 128) {
    hipLaunchKernelGGL((dynts::prefill_kernel<128>), grid, dim3(256), 0, st, p);
  } else {
    hipLaunchKernelGGL((dynts::prefill_kernel<64>), grid, dim3(256), 0, st, p);
  }
  ctx->pending[layer] = 0;
  if (ctx->spill_layer == layer) ctx->spill_layer = -1;
  if (ctx->unfused_layer == layer) ctx->unfused_layer = -1;
  return launch_status();
}

int dynts_append(dynts_ctx *ctx, int32_t layer, const uint16_t *k_new, const uint16_t *v_new, const float *s_new,
                 const uint8_t *active, void *stream) {
  int rc = check_call(ctx, layer);
  if (rc != DYNTS_OK) return rc;
  if (!k_new || !v_new) return DYNTS_ENULL;
  const dynts_config &c = ctx->cfg;
  if (c.score_mode == DYNTS_SCORE_EXTERNAL && !s_new) return DYNTS_ENULL;
  if ((reinterpret_cast<uintptr_t>(k_new) | reinterpret_cast<uintptr_t>(v_new)) % 16) return DYNTS_EINVAL;
  const LayerView lv = layer_view(ctx, layer);
  dynts::AppendParams p{lv.K, lv.V, lv.S, lv.pos, lv.seq_len, lv.next_pos, k_new, v_new,
                        c.score_mode == DYNTS_SCORE_EXTERNAL ? s_new : nullptr, active, ctx->status,
                        c.n_kv_heads, c.capacity};
  const int threads = (c.n_kv_heads * (c.head_dim / 8) + 63) / 64 * 64;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (ctx->paged) {
    const dynts::PagedView pv{lv.K, lv.V, lv.block_table, ctx->free_stack, ctx->free_top, ctx->max_pages, ctx->n_pages};
    if (c.head_dim == 128) hipLaunchKernelGGL((dynts::paged_append_kernel<128>), dim3(c.batch), dim3(threads), 0, st, p, pv);
    else hipLaunchKernelGGL((dynts::paged_append_kernel<64>), dim3(c.batch), dim3(threads), 0, st, p, pv);
  } else if (c.head_dim == 128) {
    hipLaunchKernelGGL((dynts::append_kernel<128>), dim3(c.batch), dim3(threads), 0, st, p);
  } else {
    hipLaunchKernelGGL((dynts::append_kernel<64>), dim3(c.batch), dim3(threads), 0, st, p);
  }
  return launch_status();
}

int dynts_decode_attend(dynts_ctx *ctx, int32_t layer, const uint16_t *q, const uint8_t *active, float *out,
                        float *lse, void *stream) {
  int rc = check_call(ctx, layer);
  if (rc != DYNTS_OK) return rc;
  if (!q || !out) return DYNTS_ENULL;
  if (reinterpret_cast<uintptr_t>(q) % 16) return DYNTS_EINVAL;
  if (ctx->pending[layer] == 2) {  // kept logits would lose their statistics to this call: apply them first
    rc = apply_spill(ctx, layer, static_cast<hipStream_t>(stream));
    if (rc != DYNTS_OK) return rc;
  }
  // A caller who asks for the score update next is served from the attention's logits (4 bytes per slot and head
  // written, against a second pass over K): 32 x 8 units of 5256 slots, both calls 184 -> 135 us.  The attention by itself then
  // takes longer (paged 121 -> 143 us), so they are kept only where the update has been seen to follow, and not while
  // the buffer holds those of another layer whose update rests on them alone.
  // Not under capture: the buffer is one for all layers, so the update's graph would find in it whatever the last attention
  // replayed or issued before it left there, while the saved query and statistics it needs for its pass over K are the
  // layer's own.
  unfused_ends(ctx, false);
  const bool track = ctx->cfg.score_mode == DYNTS_SCORE_ACCUMULATE;
  const bool keep = track && ctx->pairs[layer] == kPairsKeep && kept_logits_pay(ctx) &&
                    (ctx->spill_layer < 0 || ctx->pending[ctx->spill_layer] == 3) &&
                    !capturing(static_cast<hipStream_t>(stream));
  if (keep || ctx->spill_layer == layer) release_spill(ctx, static_cast<hipStream_t>(stream));
  rc = run_attend(ctx, layer, q, nullptr, nullptr, nullptr, active, out, lse, true, false, false,
                  static_cast<hipStream_t>(stream), nullptr, keep);
  if (rc == DYNTS_OK) {
    ctx->pending[layer] = track ? (keep ? 3 : 1) : 0;
    if (keep) ctx->spill_layer = layer;
    if (track) ctx->unfused_layer = layer;
  }
  return rc;
}

int dynts_update_scores(dynts_ctx *ctx, int32_t layer, void *stream) {
  int rc = check_call(ctx, layer);
  if (rc != DYNTS_OK) return rc;
  if (!ctx->pending[layer]) return DYNTS_OK;
  if (ctx->unfused_layer == layer) unfused_ends(ctx, true);
  if (ctx->pending[layer] == 3 && capturing(static_cast<hipStream_t>(stream))) release_spill(ctx, static_cast<hipStream_t>(stream));
  if (ctx->pending[layer] >= 2) return apply_spill(ctx, layer, static_cast<hipStream_t>(stream));
  rc = run_attend(ctx, layer, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, false, true, false,
                  static_cast<hipStream_t>(stream));
  if (rc == DYNTS_OK) ctx->pending[layer] = 0;
  return rc;
}

int dynts_decode_attend_update(dynts_ctx *ctx, int32_t layer, const uint16_t *q, const uint8_t *active,
                               float *out, float *lse, void *stream) {
  int rc = check_call(ctx, layer);
  if (rc != DYNTS_OK) return rc;
  if (!q || !out) return DYNTS_ENULL;
  if (reinterpret_cast<uintptr_t>(q) % 16) return DYNTS_EINVAL;
  return fused_step(ctx, layer, q, nullptr, nullptr, nullptr, active, out, lse, false, static_cast<hipStream_t>(stream),
                    nullptr);
}

int dynts_decode_step(dynts_ctx *ctx, int32_t layer, const uint16_t *q, const uint16_t *k_new,
                      const uint16_t *v_new, const float *s_new, const uint8_t *active, float *out, float *lse,
                      void *stream) {
  int rc = check_call(ctx, layer);
  if (rc != DYNTS_OK) return rc;
  if (!q || !out || !k_new || !v_new) return DYNTS_ENULL;
  const bool ext = ctx->cfg.score_mode == DYNTS_SCORE_EXTERNAL;
  if (ext && !s_new) return DYNTS_ENULL;
  if ((reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(k_new) | reinterpret_cast<uintptr_t>(v_new)) % 16)
    return DYNTS_EINVAL;
  return fused_step(ctx, layer, q, k_new, v_new, ext ? s_new : nullptr, active, out, lse, true,
                    static_cast<hipStream_t>(stream), nullptr);
}

int dynts_decode_step_static(dynts_ctx *ctx, int32_t layer, const uint16_t *q, const uint16_t *k_new,
                             const uint16_t *v_new, const float *s_new, const uint8_t *active, float *out, float *lse,
                             void *stream) {
  int rc = check_call(ctx, layer);
  if (rc != DYNTS_OK) return rc;
  if (!q || !out || !k_new || !v_new) return DYNTS_ENULL;
  const bool ext = ctx->cfg.score_mode == DYNTS_SCORE_EXTERNAL;
  if (ext && !s_new) return DYNTS_ENULL;
  if ((reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(k_new) | reinterpret_cast<uintptr_t>(v_new)) % 16)
    return DYNTS_EINVAL;
  // Layout of the static array, the same for every context so that what one call leaves fits the next:
  //   [0, 512 KiB)      ticket counters of the (sequence, KV head) units -- every launch leaves them at zero
  //   [512 KiB, 1 MiB)  check-in counters of the sequences               -- likewise
  //   [1 MiB, 8 MiB)    split partials: tagged words, a stale one is recognised whoever wrote it
  const dynts_config &c = ctx->cfg;
  const Plan &pl = ctx->plan;
  const size_t units = (size_t)c.batch * c.n_kv_heads, rows = units * pl.nsplit * pl.G;
  const size_t part_o_bytes = align_up(rows * c.head_dim * sizeof(uint64_t)), part_ml_bytes = rows * 2 * sizeof(uint64_t);
  if (units * sizeof(uint32_t) > kStaticCounters / 2 || (size_t)c.batch * sizeof(uint32_t) > kStaticCounters / 2 ||
      part_o_bytes + part_ml_bytes > kStaticScratchBytes - kStaticCounters)
    return DYNTS_EWORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  unsigned char *base = static_scratch(st);
  if (!base) return DYNTS_EHIP;
  Transient tr;
  tr.unit_cnt = reinterpret_cast<uint32_t *>(base);
  tr.seq_cnt = reinterpret_cast<uint32_t *>(base + kStaticCounters / 2);
  tr.cnt_stride = kCounterStride;  // (as far apart as they all fit)
  while (units * tr.cnt_stride * sizeof(uint32_t) > kStaticCounters / 2) tr.cnt_stride /= 2;
  tr.part_o = reinterpret_cast<uint64_t *>(base + kStaticCounters);
  tr.part_ml = reinterpret_cast<uint64_t *>(base + kStaticCounters + part_o_bytes);
  return fused_step(ctx, layer, q, k_new, v_new, ext ? s_new : nullptr, active, out, lse, true, st, &tr);
}

int dynts_hint_trigger(dynts_ctx *ctx, int32_t layer) {
  const int rc = check_call(ctx, layer);
  if (rc != DYNTS_OK) return rc;
  ctx->hint[layer] = 1;
  return DYNTS_OK;
}

int dynts_select_evict(dynts_ctx *ctx, int32_t layer, const uint8_t *trigger, int32_t k_keep, int32_t *keep_idx,
                       int32_t keep_stride, int32_t *new_len, void *stream) {
  int rc = check_call(ctx, layer);
  if (rc != DYNTS_OK) return rc;
  if (!keep_idx || !new_len) return DYNTS_ENULL;
  if (keep_stride <= 0) return DYNTS_ECAPACITY;
  const dynts_config &c = ctx->cfg;
  if (k_keep < 0) k_keep = c.budget;
  const bool apply = ctx->pending[layer] == 2 && select_applies(ctx);
  if (!apply) rc = dynts_update_scores(ctx, layer, stream);
  if (rc != DYNTS_OK) return rc;
  const LayerView lv = layer_view(ctx, layer);
  dynts::SelectParams p{lv.S, lv.seq_len, ctx->n_prompt, trigger, keep_idx, new_len, ctx->status,
                        c.n_kv_heads, c.capacity, c.window, k_keep, keep_stride,
                        reinterpret_cast<const float *>(ctx->ws + ctx->plan.off_spill), lv.mlprev, lv.nprev, ctx->plan.G, ctx->plan.cap_pad};
  hipStream_t st = static_cast<hipStream_t>(stream);
  switch (select_threads(c)) {
    case 256: launch_select<256>(p, c, apply, st); break;
    case 512: launch_select<512>(p, c, apply, st); break;
    default: launch_select<1024>(p, c, apply, st); break;
  }
  rc = launch_status();
  if (rc == DYNTS_OK && apply) {
    ctx->pending[layer] = 0;
    ctx->spill_layer = -1;
  }
  return rc;
}

int dynts_compact(dynts_ctx *ctx, int32_t layer, const uint8_t *trigger, const int32_t *keep_idx,
                  int32_t keep_stride, const int32_t *new_len, void *stream) {
  int rc = check_call(ctx, layer);
  if (rc != DYNTS_OK) return rc;
  if (!keep_idx || !new_len) return DYNTS_ENULL;
  if (keep_stride <= 0) return DYNTS_ECAPACITY;
  if (ctx->pending[layer]) return DYNTS_EPENDING;
  const dynts_config &c = ctx->cfg;
  const LayerView lv = layer_view(ctx, layer);
  dynts::CompactParams p{lv.K, lv.V, lv.S, lv.pos, lv.seq_len, trigger, keep_idx, new_len,
                         c.n_kv_heads, c.capacity, keep_stride};
  const dynts::PagedView pv{lv.K, lv.V, lv.block_table, ctx->free_stack, ctx->free_top, ctx->max_pages, ctx->n_pages};
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (compact_threads(ctx) == 256) launch_compact<256>(p, ctx, pv, st);
  else launch_compact<512>(p, ctx, pv, st);
  if (ctx->paged)
    hipLaunchKernelGGL(dynts::paged_trim_kernel, dim3((c.batch + 63) / 64), dim3(64), 0, st, pv, trigger, new_len,
                       lv.seq_len, c.batch, c.n_kv_heads, c.capacity, keep_stride);
  return launch_status();
}

int dynts_set_kernel_events(dynts_ctx *ctx, void *start, void *stop) {
  if (!ctx) return DYNTS_ENULL;
  if ((start == nullptr) != (stop == nullptr)) return DYNTS_EINVAL;
  ctx->ev_start = static_cast<hipEvent_t>(start);
  ctx->ev_stop = static_cast<hipEvent_t>(stop);
  return DYNTS_OK;
}

int dynts_set_kernel_event_list(dynts_ctx *ctx, void *const *starts, void *const *stops, int32_t n) {
  if (!ctx) return DYNTS_ENULL;
  if (n < 0) return DYNTS_EINVAL;
  if (n > 0 && (!starts || !stops)) return DYNTS_ENULL;
  ctx->ev_list_start.clear();
  ctx->ev_list_stop.clear();
  ctx->ev_list_next = 0;
  for (int i = 0; i < n; ++i) {
    if (!starts[i] || !stops[i]) return DYNTS_ENULL;
    ctx->ev_list_start.push_back(static_cast<hipEvent_t>(starts[i]));
    ctx->ev_list_stop.push_back(static_cast<hipEvent_t>(stops[i]));
  }
  return DYNTS_OK;
}

size_t dynts_score_block_scratch_bytes(const dynts_config *cfg, int32_t n_queries) {
  if (!cfg || check_config(cfg) != DYNTS_OK || n_queries <= 0 || n_queries > (1 << 20)) return 0;
  return (size_t)score_block_splits(*cfg, n_queries) * score_block_stats_bytes(*cfg, n_queries);
}

int dynts_score_block(dynts_ctx *ctx, int32_t layer, const uint16_t *q_blk, const uint16_t *k_blk,
                      int32_t n_queries, const uint8_t *active, float *dst, int32_t accumulate, void *scratch,
                      size_t scratch_bytes, void *stream) {
  int rc = check_call(ctx, layer);
  if (rc != DYNTS_OK) return rc;
  if (!q_blk || !scratch) return DYNTS_ENULL;
  if (n_queries <= 0 || n_queries > (1 << 20)) return DYNTS_EINVAL;
  if (reinterpret_cast<uintptr_t>(q_blk) % 16 || reinterpret_cast<uintptr_t>(k_blk) % 16) return DYNTS_EINVAL;
  const dynts_config &c = ctx->cfg;
  const size_t one = score_block_stats_bytes(c, n_queries);
  if (scratch_bytes < one || reinterpret_cast<uintptr_t>(scratch) % 4) return DYNTS_EWORKSPACE;
  const LayerView lv = layer_view(ctx, layer);
  const int G = c.n_q_heads / c.n_kv_heads;
  dynts::ScoreBlockParams p{};
  p.K = lv.K;
  p.q_blk = q_blk;
  p.k_blk = k_blk;
  p.seq_len = lv.seq_len;
  p.n_prompt = ctx->n_prompt;
  p.active = active;
  p.stats = static_cast<float *>(scratch);
  p.dst = dst ? dst : lv.S;
  p.Nb = c.batch;
  p.T = n_queries;
  p.Hq = c.n_q_heads;
  p.Hkv = c.n_kv_heads;
  p.G = G;
  p.cap = c.capacity;
  p.Rpad = (int)align_up((size_t)n_queries * G);
  p.skip_prompt = dst ? 0 : 1;
  p.accumulate = accumulate ? 1 : 0;
  p.scale_log2 = ctx->scale_log2;
  p.block_table = lv.block_table; p.max_pages = ctx->max_pages; p.n_pages = ctx->n_pages;
  p.n_split = score_block_splits(c, n_queries);
  if ((size_t)p.n_split * one > scratch_bytes) p.n_split = (int)(scratch_bytes / one);
  const long long R = (long long)n_queries * G;
  // (1-D grids: blocks per unit x units rounded up to the 8 XCDs, mapped inside the kernels)
  const long long units8 = ((long long)c.batch * c.n_kv_heads + 7) / 8 * 8;
  const long long b1 = (R + dynts::kSbRowsPerWg - 1) / dynts::kSbRowsPerWg;
  const long long b2 = (c.capacity + dynts::kSbRowsPerWg - 1) / dynts::kSbRowsPerWg;
  if (b1 * units8 > 0x7fffffffLL || b2 * units8 > 0x7fffffffLL) return DYNTS_EINVAL;
  if ((long long)n_queries * c.n_q_heads * c.head_dim * 2 > 0x7fffffffLL) return DYNTS_EINVAL;  // 32-bit row offsets
  const dim3 g1((unsigned)(b1 * units8 * p.n_split)), g2((unsigned)(b2 * units8));
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (c.head_dim == 128) {
    if (ctx->paged) launch_score_block<128, true>(p, g1, g2, st);
    else launch_score_block<128, false>(p, g1, g2, st);
  } else {
    if (ctx->paged) launch_score_block<64, true>(p, g1, g2, st);
    else launch_score_block<64, false>(p, g1, g2, st);
  }
  return launch_status();
}

int dynts_predictor_pack(const uint16_t *W, int32_t m, int32_t K, uint16_t *W_packed, void *stream) {
  if (!W || !W_packed) return DYNTS_ENULL;
  if (m <= 0 || K <= 0) return DYNTS_EINVAL;
  if (m % 16 || K % 32) return DYNTS_ESHAPE;
  if (reinterpret_cast<uintptr_t>(W) % 16 || reinterpret_cast<uintptr_t>(W_packed) % 16 || W == W_packed) return DYNTS_EINVAL;
  const size_t pieces = (size_t)m * K / 8;
  hipLaunchKernelGGL(dynts::mlp_pack_kernel, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0,
                     static_cast<hipStream_t>(stream), W, m, K, W_packed);
  return launch_status();
}

size_t dynts_predict_scratch_bytes(const dynts_predictor *w, int32_t batch) {
  if (check_predictor(w, batch) != DYNTS_OK) return 0;
  // what serves a batch serves every smaller one
  size_t bytes = 0;
  for (int edge = 16; edge < 128 + 16; edge += 16) {
    const int nb = edge < batch ? edge : batch;
    const size_t need = mlp_split(w, nb) ? mlp_split_plan(w, nb).total : mlp_plan(w, nb).total;
    bytes = need > bytes ? need : bytes;
  }
  return bytes;
}

int dynts_predict_scores(const dynts_predictor *w, const uint16_t *h, int32_t batch, float *s_out, int32_t n_rep,
                         void *scratch, size_t scratch_bytes, void *start, void *stop, void *stream) {
  int rc = check_predictor(w, batch);
  if (rc != DYNTS_OK) return rc;
  if (!h || !s_out || !scratch || !w->W1 || !w->W2 || !w->w3) return DYNTS_ENULL;
  if (n_rep <= 0 || n_rep > 256) return DYNTS_EINVAL;
  if ((start == nullptr) != (stop == nullptr)) return DYNTS_EINVAL;
  if (reinterpret_cast<uintptr_t>(h) % 16 || reinterpret_cast<uintptr_t>(w->W1) % 16 ||
      reinterpret_cast<uintptr_t>(w->W2) % 16)
    return DYNTS_EINVAL;
  unsigned char *base = static_cast<unsigned char *>(scratch);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (mlp_split(w, batch)) {
    const MlpSplitPlan pl = mlp_split_plan(w, batch);
    if (scratch_bytes < pl.total || reinterpret_cast<uintptr_t>(scratch) % kAlign) return DYNTS_EWORKSPACE;
    run_mlp_split(w, pl, h, batch, s_out, n_rep, base, st, static_cast<hipEvent_t>(start), static_cast<hipEvent_t>(stop));
    return launch_status();
  }
  const MlpPlan pl = mlp_plan(w, batch);
  if (scratch_bytes < pl.total || reinterpret_cast<uintptr_t>(scratch) % kAlign) return DYNTS_EWORKSPACE;
  dynts::MlpParams p{};
  p.W = w->W1; p.x = h; p.bias = w->b1;
  p.Nb = batch; p.m = w->m1; p.K = w->d; p.act = w->activation;
  p.y = reinterpret_cast<uint16_t *>(base);
  p.clear = reinterpret_cast<uint32_t *>(base + pl.off_sum);
  p.n_clear = (uint32_t)((pl.total - pl.off_sum) / 16);
  // the optional events bracket the whole call: start on the first kernel, stop on the last
  launch_mlp<false>(p, w->packed, pl.ft1, pl.bt, pl.wgs1, st, static_cast<hipEvent_t>(start), nullptr);
  p.W = w->W2; p.x = p.y; p.bias = w->b2; p.m = w->m2; p.K = w->m1;
  p.w3 = w->w3; p.b3 = w->b3; p.ns = pl.ns;
  p.part_sum = reinterpret_cast<uint64_t *>(base + pl.off_sum);
  p.part_dot = reinterpret_cast<uint64_t *>(base + pl.off_dot);
  p.group_cnt = reinterpret_cast<uint32_t *>(base + pl.off_group);
  p.done_cnt = reinterpret_cast<uint32_t *>(base + pl.off_done);
  p.s_out = s_out; p.n_rep = n_rep;
  launch_mlp<true>(p, w->packed, pl.ft2, pl.bt, pl.groups * pl.ns, st, nullptr, static_cast<hipEvent_t>(stop));
  return launch_status();
}

int dynts_probe_read_stream(const void *buf, size_t bytes, int32_t n_workgroups, uint32_t magic, uint32_t *sink,
                            void *start, void *stop, void *stream) {
  if (!buf || !sink) return DYNTS_ENULL;
  if (bytes == 0 || bytes % 16 != 0 || n_workgroups <= 0 || n_workgroups > (1 << 20)) return DYNTS_EINVAL;
  if ((reinterpret_cast<uintptr_t>(buf) & 15) != 0) return DYNTS_EINVAL;
  if ((start == nullptr) != (stop == nullptr)) return DYNTS_EINVAL;
  hipExtLaunchKernelGGL(dynts::read_stream_kernel, dim3(n_workgroups), dim3(dynts::kProbeThreads), 0,
                        static_cast<hipStream_t>(stream), static_cast<hipEvent_t>(start),
                        static_cast<hipEvent_t>(stop), 0, static_cast<const uint32_t *>(buf), bytes / 16, magic, sink);
  return launch_status();
}

int dynts_probe_exp_rate(int32_t n_workgroups, int32_t iters, float *sink, void *start, void *stop, void *stream) {
  if (!sink) return DYNTS_ENULL;
  if (n_workgroups <= 0 || n_workgroups > (1 << 20) || iters <= 0) return DYNTS_EINVAL;
  if ((start == nullptr) != (stop == nullptr)) return DYNTS_EINVAL;
  hipExtLaunchKernelGGL(dynts::exp2_rate_kernel, dim3(n_workgroups), dim3(dynts::kProbeThreads), 0,
                        static_cast<hipStream_t>(stream), static_cast<hipEvent_t>(start),
                        static_cast<hipEvent_t>(stop), 0, iters, -12345.678f, sink);
  return launch_status();
}

int dynts_probe_issue_mix(int32_t n_workgroups, int32_t iters, int32_t what, float *sink, void *start, void *stop,
                          void *stream) {
  if (!sink) return DYNTS_ENULL;
  if (n_workgroups <= 0 || n_workgroups > (1 << 20) || iters <= 0 || what < 1 || what > 3) return DYNTS_EINVAL;
  if ((start == nullptr) != (stop == nullptr)) return DYNTS_EINVAL;
  const dim3 grid(n_workgroups), block(dynts::kProbeThreads);
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipEvent_t e0 = static_cast<hipEvent_t>(start), e1 = static_cast<hipEvent_t>(stop);
  const float c = 0.1f, L = -3.f, magic = -12345.678f;
  if (what == 1) hipExtLaunchKernelGGL(dynts::issue_mix_kernel<1>, grid, block, 0, st, e0, e1, 0, iters, c, L, magic, sink);
  else if (what == 2) hipExtLaunchKernelGGL(dynts::issue_mix_kernel<2>, grid, block, 0, st, e0, e1, 0, iters, c, L, magic, sink);
  else hipExtLaunchKernelGGL(dynts::issue_mix_kernel<3>, grid, block, 0, st, e0, e1, 0, iters, c, L, magic, sink);
  return launch_status();
}

int dynts_decode_loop(dynts_ctx *ctx, int32_t n_steps, const uint16_t *q, const uint16_t *k_new,
                      const uint16_t *v_new, const float *s_new, const uint8_t *active, const uint8_t *evict_steps,
                      const uint8_t *trigger, float *out, size_t out_step_stride, int32_t *keep_idx,
                      int32_t *new_len, void *stream) {
  int rc = check_call(ctx, 0);
  if (rc != DYNTS_OK) return rc;
  if (n_steps < 0) return DYNTS_EINVAL;
  if (!q || !k_new || !v_new || !out) return DYNTS_ENULL;
  const dynts_config &c = ctx->cfg;
  const bool ext = c.score_mode == DYNTS_SCORE_EXTERNAL;
  if (ext && !s_new) return DYNTS_ENULL;
  if (evict_steps && (!keep_idx || !new_len)) return DYNTS_ENULL;
  const size_t q_layer = (size_t)c.batch * c.n_q_heads * c.head_dim;
  const size_t kv_layer = (size_t)c.batch * c.n_kv_heads * c.head_dim;
  hipStream_t st = static_cast<hipStream_t>(stream);
  auto trigger_of = [&](int i, int l) {
    const uint8_t *trig = trigger ? trigger + (size_t)i * c.batch : nullptr;
    const int rc2 = dynts_select_evict(ctx, l, trig, c.budget, keep_idx, c.capacity, new_len, stream);
    return rc2 == DYNTS_OK ? dynts_compact(ctx, l, trig, keep_idx, c.capacity, new_len, stream) : rc2;
  };
  // Outputs of steps that overlap in part are left to launches in order (size_t: a stride may lead backwards).
  const size_t slab = c.n_layers * q_layer;
  const bool apart = out_step_stride == 0 || (out_step_stride >= slab && (size_t)0 - out_step_stride >= slab);
  for (int i = 0; i < n_steps; ++i) {
    const uint8_t *act = active ? active + (size_t)i * c.batch : nullptr;
    const float *sn = ext ? s_new + (size_t)i * c.batch * c.n_kv_heads : nullptr;
    int run = 1;  // steps up to the next trigger's, where they can be one launch
    const int most = apart ? resident_run(ctx, st) : 0;
    while (i + run < n_steps && run < most && !(evict_steps && evict_steps[i + run - 1])) ++run;
    if (run >= kLeastRun) {
      const bool evict = evict_steps && evict_steps[i + run - 1];
      for (int l = 0; l < c.n_layers; ++l) {
        const size_t sl = (size_t)i * c.n_layers + l;
        rc = resident_steps(ctx, l, run, evict, q + sl * q_layer, k_new + sl * kv_layer, v_new + sl * kv_layer, sn, act,
                            out + (size_t)i * out_step_stride + (size_t)l * q_layer, out_step_stride, st);
        if (rc == DYNTS_OK && evict) rc = trigger_of(i + run - 1, l);
        if (rc != DYNTS_OK) return rc;
      }
      i += run - 1;
      continue;
    }
    for (int l = 0; l < c.n_layers; ++l) {
      const size_t sl = (size_t)i * c.n_layers + l;
      if (evict_steps && evict_steps[i]) ctx->hint[l] = 1;  // the trigger below follows this step
      rc = dynts_decode_step(ctx, l, q + sl * q_layer, k_new + sl * kv_layer, v_new + sl * kv_layer, sn, act,
                             out + (size_t)i * out_step_stride + (size_t)l * q_layer, nullptr, stream);
      if (rc == DYNTS_OK && evict_steps && evict_steps[i]) rc = trigger_of(i, l);
      if (rc != DYNTS_OK) return rc;
    }
  }
  return DYNTS_OK;
}

}  // extern "C"
