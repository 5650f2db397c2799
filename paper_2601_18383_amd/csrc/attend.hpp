// Decode attention + deferred importance-score accumulation for gfx950 (wave64, MFMA).
//
// The cache of one (sequence, KV head) is shared out over nsplit workgroups of W waves (8 by
// default).  Wave number wi of the nsplit*W takes the 32-slot tile that starts at slot 32*wi -- its
// loads are issued before the kernel knows the sequence length (kStream: and then more tiles at fixed
// places, AttendParams::rounds) -- and then an equal, contiguous
// share of the slots behind those first tiles, 32 at a time, with the next tile's loads already
// in flight while it works on the current one:
//   * K rows are read whole, 1 KB a load instruction, and turned into MFMA operands through a wave-private LDS tile (lane (r, kg)
//     gets row r, columns 32*ks + 8*kg .. +7): read from memory in that order, 16 rows x 64 bytes an instruction, a
//     compute unit takes in 38 B/ns instead of 140, and the first tiles alone took it 2 us.
//     One v_mfma_f32_16x16x32_bf16 per 32 columns
//     gives the logits of 16 slots x 16 (padded) query heads of the group, so a K tile is read
//     once for the whole GQA group (Eq. attn-score).
//   * the same K registers are multiplied with the PREVIOUS step's query (operands swapped, so
//     a lane ends up with 4 heads of one slot); with that step's final softmax statistics this
//     gives its attention weights exactly, which are summed over the group and added to S
//     (Eq. importance-score, running form).  The score update thus rides on this step's pass
//     over K instead of a second pass or a spill of logits.
//   * V rows are staged through a wave-private LDS tile (coalesced 16-byte loads in,
//     ds_read_b64_tr_b16 transposing reads out) to form the V^T MFMA operand; the softmax
//     weights are split into bf16 hi + lo parts so P.V keeps ~16 bits of each weight
//     (Eq. attn-o); accumulation is fp32 throughout.
//   * online-softmax state (running max, sum, output) is per wave; the waves of a workgroup are
//     combined in LDS.  With nsplit == 1 the result is finished on the spot; otherwise the partial
//     goes to the workspace and the LAST workgroup of the (sequence, KV head) to arrive
//     (device-scope counter) merges the partials, writes `out`, and saves the query and the
//     statistics that the next step's score update needs.  Every workgroup checks in on a
//     per-sequence counter behind its first tile (kStream: in front of it); the last one to do so advances seq_len / next_pos.
//     No second kernel, no host round trip.
//   * the loop waits for no more than it uses: loads are waited for by their number, so every way through a tile issues the same ones in the
//     same order (no branch around V's part, one loop per way of loading, page numbers by the scalar cache).  Where the wait for the next
//     tile's K rows had been one for its V rows, and on pages one for everything: 64 steps and a trigger on 128 units of 2464 slots 1970 -> 1922 us, on
//     pages 2009 -> 1975; 8 steps of four layers of 512 units of 1184 1850 -> 1772; 16 of two layers of 512 of 2624 3580 -> 3535.
//   * with APPEND the new token's K/V row is written to its slot by one workgroup and enters the
//     softmax as the initial state of the first wave (max = q.k_new, sum = 1, output = v_new), so
//     no wave has to wait for the row to become visible.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace dynts {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef short i16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kTile = 32;           // cache slots one wave handles per iteration
constexpr float kLowest = -3.4028234663852886e38f;  // the lowest finite value
// A workgroup has W waves (4 or 8).

struct AttendParams {
  uint16_t *K, *V;          // layer base, [Nb][Hkv][cap][D]
  float *S;                 // [Nb][Hkv][cap]
  int32_t *pos;             // [Nb][Hkv][cap]
  int32_t *seq_len;         // [Nb]
  const int32_t *n_prompt;  // [Nb]
  int32_t *next_pos;        // [Nb]
  const uint16_t *q;        // [Nb][Hq][D]
  const uint16_t *k_new, *v_new;  // [Nb][Hkv][D] (fused append) or null
  const float *s_new;       // [Nb][Hkv] or null
  const uint8_t *active;    // [Nb] or null
  float *out;               // [Nb][Hq][D]
  float *lse;               // [Nb][Hq] or null
  const uint16_t *qprev;    // [Nb][Hq][D] query of the deferred update (read)
  uint16_t *qnext;          // [Nb][Hq][D] where this call's query is kept for the next deferred update
  float *mlprev;            // [Nb][Hq][2] (max in log2 units, sum) of the deferred update
  int32_t *nprev;           // [Nb] slots the deferred update covers (0 = none)
  uint64_t *part_o;         // [Nb][Hkv][nsplit][G][D]  (tag << 32 | fp32 bits)
  uint64_t *part_ml;        // [Nb][Hkv][nsplit][G][2]
  uint32_t tag;             // this launch's serial number (never 0)
  int score_tiles;          // updated scores are written out every so many tiles of a wave (1 .. 16)
  // When this step's own score update is expected to be asked for by itself (a trigger is known to follow, or it is the
  // unfused attention of a caller who asks for its update next), the step's scaled logits (log2 units) are kept,
  // [Nb][Hkv][cap_pad / 32][G][32] fp32 (see spill_at), so that its score update can be applied from them (apply_spill_kernel,
  // select_kernel) instead of by a second pass over K.  Null: not kept.
  float *spill;
  int cap_pad;              // cap rounded up to a whole tile
  uint32_t *unit_cnt;       // [Nb][Hkv][cnt_stride] ticket counters, zero between launches
  uint32_t *seq_cnt;        // [Nb][cnt_stride]      arrival counters, zero between launches
  int cnt_stride;           // words from one counter to the next
  int32_t *status;
  int Nb, Hq, Hkv, G, cap, nsplit;
  int track;                // 1: scores are accumulated from attention (save q and statistics)
  float scale_log2;         // softmax scale * log2(e)
  // Dense layout, K and V of all layers together beyond the 256 MB memory-side cache (the STREAM kernels): a cache that is
  // read whole, step after step, through a cache it does not fit evicts every row before its next use.  So the slots
  // below 32 * waves * rounds of each unit go through it and stay, the ones behind are loaded past it (non-temporal
  // loads), once a sequence has more than fit_slots.  (rounds = 0: the first tiles do not fit either; they are loaded through the caches all the same.)
  int fit_slots;            // slots per unit up to which everything fits
  int rounds;               // tiles of a wave at fixed places
  // paged layout only: K and V are page pools [n_pages][kPageSlots][D]; slot j of a unit lives in page
  // block_table[unit][j / kPageSlots], row j % kPageSlots
  const int32_t *block_table;  // layer base, [Nb][Hkv][max_pages]
  int32_t *block_table_w;      // the same, for the appender
  int32_t *free_stack;         // [n_pages] page ids; entries below *free_top are free
  int32_t *free_top;
  int max_pages, n_pages;
};

// Chunks of a unit are merged four at a time; in the WIDE kernels with one output element per thread more than kWideFrom1
// of them 32 at a time, with two (head_dim 128 only) more than kWideFrom2 of them eight at a time.
constexpr int kWideFrom1 = 16, kWideFrom2 = 4;

// Where the kept logit of head g of a unit's slot j lies: tile by tile, so that those of consecutive tiles are one run of memory.
__device__ __forceinline__ size_t spill_at(size_t unit, int cap_pad, int G, int g, int j) {
  return (unit * (size_t)cap_pad + (size_t)(j & ~(kTile - 1))) * (size_t)G + (size_t)(kTile * g + (j & (kTile - 1)));
}

constexpr int kStream = 1, kBurst = 2;  // forms of the kernel for large caches

constexpr int kPageSlots = 64;  // slots per page: two tiles, so a tile never straddles pages


__device__ __forceinline__ u32x4 load_u32x4(const uint16_t *p) { return *reinterpret_cast<const u32x4 *>(p); }
__device__ __forceinline__ void store_u32x4(uint16_t *p, u32x4 v) { *reinterpret_cast<u32x4 *>(p) = v; }

// (two branches that differ only in how they load would be merged into one)
#define DYNTS_OWN_BRANCH asm volatile("; past the caches")

// The first `rows` rows of a unit's cache (or of a page) as a buffer: a load past them reads zeros and fetches nothing, so that
// the prefetch behind a wave's last tile needs no branch (behind one every wait would be a wait for all loads), no clamp, and
// no memory.
using RowBuffer = __amdgpu_buffer_rsrc_t;
template <int D>
__device__ __forceinline__ RowBuffer row_buffer(const uint16_t *base, int rows) {
  // (uniform, and told so to the compiler: it would load each time in a loop over the values that lanes might have)
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(base), 0, __builtin_amdgcn_readfirstlane((rows > 0 ? rows : 0) * (2 * D)), 0x00027000);
}

// The 32 rows of the tile at t: contiguous memory, 1 KB a load instruction.  (Read in the order in which the MFMA operands want
// them, 16 rows x 64 bytes, a compute unit takes in 38 B/ns instead of 140.)  NT: past the caches (see AttendParams::fit_slots).
template <int D, bool NT = false>
__device__ __forceinline__ void load_tile(u32x4 (&f)[kTile * D / 512], RowBuffer rows, int t, int lane) {
  const uint32_t off = (uint32_t)t * (uint32_t)(2 * D) + 16u * (uint32_t)lane;
#pragma unroll
  for (int it = 0; it < kTile * D / 512; ++it)
    f[it] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rows, off + 1024u * it, 0, NT ? 2 : 0));
}
// Cross-workgroup traffic inside one launch (split partials, arrival counters) consists of relaxed
// agent-scope atomics only, which compile to sc1 accesses that are written through to, and read
// from, the level all XCDs share.  A split partial is handed over WITHOUT any ordering between
// different words: every 32-bit value travels in one 64-bit word together with the launch's tag
// (a serial number no earlier launch of this process used), stored and loaded with single 64-bit
// atomic accesses, so a word is either this launch's value or recognisably stale.  The workgroup
// that draws the last ticket of a (sequence, KV head) merges: it re-reads a word until its tag is
// this launch's.  (The replays of a launch recorded into a graph share one tag: there the words are cleared behind the
// launch, see run_attend.)  That loop ends: a workgroup draws its ticket only when it is running, it issues its
// stores without ever waiting for another workgroup, and issued stores become visible.  There is no
// fence, no wait for store acknowledgements and no cache-wide write-back; no ordinary cached access
// ever touches these words during a launch.
__device__ __forceinline__ void tagged_store(uint64_t *p, float v, uint32_t tag) {
  __hip_atomic_store(p, ((uint64_t)tag << 32) | (uint64_t)__float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t tagged_load(const uint64_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Draw a ticket from a device counter, the answer to be looked at later.  The address is made to look
// lane-dependent: for a uniform address the compiler rewrites the operation into its wave-aggregated
// form, whose broadcast of the result waits for the atomic -- and for every load issued before it --
// on the spot.
__device__ __forceinline__ uint32_t draw_ticket(uint32_t *counter) {
  uint32_t zero = 0;
  asm volatile("" : "+v"(zero));
  return __hip_atomic_fetch_add(counter + zero, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool tag_is(uint64_t w, uint32_t tag) { return (uint32_t)(w >> 32) == tag; }
__device__ __forceinline__ float tagged_value(uint64_t w) { return __uint_as_float((uint32_t)w); }

// 2^x by the hardware instruction alone (v_exp_f32, ~1 ulp).  Arguments here are <= 0 up to
// rounding; results below 2^-126 flush to zero, which is far under what the sums resolve.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LARGE: the caches do not fit the memory-side cache.  kStream (dense layout), see AttendParams::fit_slots.  kBurst: updated
// scores leave in bursts through LDS (see flush_scores) instead of tile by tile.  (Not both: loads past the cache made
// paged launches 5 % slower, and with them bursts gained nothing in the dense layout.)
// SPILL: the step keeps its logits (AttendParams::spill).
// WIDE: with the merges of 32 and of 8 chunks at a time (see merge below), whose registers every wave of the kernel pays for.
// Registers: two waves a SIMD.  Steps on large paged caches of head_dim 64 need four (128 registers, where the compiler would take 131), two workgroups a
// compute unit, as the other eight-wave forms of head_dim 64 have by themselves.  us a step, 131 / 128 registers (in brackets with K in operand order from memory,
// 144): 260 units of 8000 slots 166.7 / 128.4 (145.6), 384 of 5000 114.8 / 103.4 (107.2), 800 of 4000 191.4 / 170.4 (178.7), 520 of 4000
// 141.7 / 134.8 (127.9: eight workgroups wait for a place), 256 of 8000 103.2 / 103.4 (102.3).
constexpr int min_waves(int D, int W, bool append, bool paged, int large, bool spill) {
  return append && paged && D == 64 && W == 8 && large == kBurst && !spill ? 4 : 2;
}

template <int D, int W, bool ATTEND, bool PENDING, bool APPEND, bool PAGED = false, int LARGE = 0, bool SPILL = false,
          bool WIDE = false>
__global__ __launch_bounds__(W * 64, min_waves(D, W, APPEND, PAGED, LARGE, SPILL)) void attend_kernel(const AttendParams p) {
  constexpr int kWaves = W, kThreads = W * 64;
  constexpr int KS = D / 32;              // MFMA k-steps per K row
  constexpr int CB = D / 16;              // 16-column blocks of the output
  constexpr int PIECES = D / 8;           // 16-byte pieces per row
  constexpr int VROWS = 64 / PIECES;      // rows covered by one wave-wide 16-byte load
  constexpr int VIT = kTile / VROWS;
  constexpr int VSTRIDE = 2 * D + 32;     // bytes per staged V row (+32: transposing reads hit distinct banks)
  constexpr int KSTRIDE = 2 * D + 32;     // bytes per staged K or query row (+32: the 16 lanes that a 16-byte read serves at a time hit distinct banks)
  constexpr int OSTRIDE = D + 4;          // floats per row of the cross-wave output reduction
  constexpr bool STREAM = LARGE == kStream, BURST = LARGE == kBurst;
  static_assert(!(STREAM && PAGED), "pages are loaded through the caches");
  static_assert(kTile * VSTRIDE >= 16 * OSTRIDE * 4, "LDS tile is reused for the reduction");
  // A pass over K alone turns it 16 rows at a time: with room for whole tiles (83 KB at head_dim 128) no second workgroup fits on a compute
  // unit beside one, which short caches of many units need.  us, 32 / 16 rows at a time (in brackets with K in operand order from memory): 1024 units of
  // 66 slots 12.7 / 10.2 (11.5), of 300 17.9 / 15.1 (17.0), of 900 40.6 / 38.0 (42.0); 512 of 300 11.0 / 9.4 (10.9); 2048 of 300 42.1 / 29.1
  // (31.3); 512 of 2640 56.5 / 57.4 (65.7); 128 of 2464 15.8 / 15.5 (16.0)
  constexpr int KROWS = ATTEND ? kTile : 16, QPREV = ATTEND ? 16 : 0;  // (and holds the previous step's query rows only)
  constexpr int kStage = ATTEND ? kTile * VSTRIDE : KROWS * KSTRIDE;   // bytes of LDS a wave turns its tiles in
  __shared__ __align__(16) unsigned char smem[kWaves * kStage];
  __shared__ float sm_m[kWaves][16];
  __shared__ float sm_l[kWaves][16];
  __shared__ float sm_max[16];
  __shared__ uint32_t sm_flag;
  __shared__ int32_t sm_hdr[5];
  __shared__ __align__(16) unsigned char sm_q[(QPREV + 16) * KSTRIDE];  // this step's query rows, the previous step's
  __shared__ __align__(16) float sm_ml[32];                       // statistics of the previous step
  __shared__ __align__(16) unsigned char sm_new[APPEND ? 4 * D : 16];  // the appended token's K and V row
  // updated scores of up to kScoreTiles consecutive tiles per wave, written out together (see flush_scores)
  constexpr int kScoreTiles = 16;
  __shared__ __align__(16) float sm_score[PENDING && BURST ? kWaves : 1][PENDING && BURST ? kScoreTiles * kTile : 4];

  // logits of consecutive tiles per wave, written out together (see flush_logits)
  constexpr int kLogitRows = 32;  // heads times tiles
  __shared__ __align__(16) float sm_logit[SPILL ? kWaves : 1][SPILL ? kLogitRows * kTile : 4];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kg = lane >> 4;
  const int g = r16;  // query head (within the group) of this lane's logits
  // Workgroup -> (unit, chunk).  Consecutive workgroup ids go to the 8 XCDs in turn; the chunks of one
  // (sequence, KV head) unit get ids that are 8 apart, so that they normally run on ONE XCD and their
  // hand-off of partials travels through that XCD's L2 (measured: a round trip between workgroups costs
  // about 0.55 us inside an XCD, 0.7 - 0.9 us across).  Nothing depends on the placement but speed.
  // grid = round_up(units, 8) * nsplit; the padding workgroups leave at once.
  const int wg = blockIdx.x, per_grp = 8 * p.nsplit;
  const int grp = __builtin_amdgcn_readfirstlane(wg / per_grp);
  const int split = (wg - grp * per_grp) >> 3, u_lin = grp * 8 + (wg & 7);
  if (u_lin >= p.Nb * p.Hkv) return;
  // (a division leaves uniform values in vector registers, and every address formed from them)
  const int b = __builtin_amdgcn_readfirstlane(u_lin / p.Hkv), h = u_lin - b * p.Hkv;
  const int G = p.G;

  const size_t unit = (size_t)b * p.Hkv + h;
  // dense: this unit's rows; paged: the pools
  uint16_t *Kb = PAGED ? p.K : p.K + unit * (size_t)p.cap * D;
  uint16_t *Vb = PAGED ? p.V : p.V + unit * (size_t)p.cap * D;
  const int32_t *tb = PAGED ? p.block_table + unit * (size_t)p.max_pages : nullptr;
  // Looked up through the scalar cache: as a vector load, whose answer comes behind those of all loads in flight, a lookup a tile had the
  // wave wait for its next tile's rows.  (One entry may be written meanwhile, that of the page which the appended row opens.  A wave whose first tile
  // lies there may find the old or the new value, once or each time: every use clamps it into the pool, and the tile's rows lie past the
  // sequence, so they are masked.  The compiler takes the table as constant and may look an entry up again for each use of it.)
  const auto *tb_scalar = (const __attribute__((address_space(4))) int32_t *)tb;
  // Paged addressing of one tile: the tile start is first pulled back into the tile that holds row end-1
  // (so every clamped row stays in ONE page); the tile is then loaded relative to that page: base = pool +
  // page * 64 rows, rows and the clamp counted from the page's first slot.
  auto page_of = [&](int tp) -> int {
    int pi = tp / kPageSlots;
    pi = pi < p.max_pages ? pi : p.max_pages - 1;
    // never followed out of the pool (least, then greatest, so that the value looked up has one use: see above)
    const int pg = __builtin_elementwise_min(tb_scalar[pi], p.n_pages - 1);
    return __builtin_elementwise_max(pg, 0);
  };
  auto clamp_tile = [&](int tt, int end) -> int {
    const int last_tile = (end - 1) & ~(kTile - 1);
    return tt < last_tile ? tt : last_tile;
  };
  auto page_base = [&](int pg) -> size_t { return (size_t)pg * kPageSlots * D; };  // element offset of a page
  float *Sb = p.S + unit * (size_t)p.cap;
  unsigned char *vst = smem + wave * kStage;
  const int vrow_l = lane / PIECES, vpiece = lane % PIECES;
  // Work split of one (sequence, KV head) over its nsplit * W waves: wave wi first takes tile wi
  // (a position known before the sequence length is, so its loads can leave at once); the slots
  // past those first tiles are then cut into contiguous ranges of whole tiles, one per wave, from
  // the actual length, so the waves move (nearly) the same number of bytes whatever the length.
  const int NW = p.nsplit * kWaves;
  const int wi = split * kWaves + wave;
  int t = kTile * wi;

  // ---- request everything the prologue needs in one go -----------------------------------
  // Loads return in order, so the few scalars (lengths, activity) go first; right behind them
  // the first tile, whose addresses depend on kernel arguments only (rows clamped to the end
  // of the allocation; what lies past the sequence is masked once its length is known); then
  // the query and the statistics.
  //
  // The per-sequence words.  seq_len, nprev and next_pos are REWRITTEN during this launch, by the last
  // workgroup of the sequence to check in, so only wave 0 reads them (the wave of the thread that checks
  // in, which it does after these loads have returned); the other waves get them through LDS behind the
  // barrier below.  Lanes 0..4 of wave 0 fetch one word each with a vector load, so nothing waits here
  // (uniform addresses would become scalar loads that the wave must wait for before its tile loads).
  int hdr_word = 1;  // lane 4 without a mask: active
  if (tid < 4) {
    const int32_t *src = tid == 0 ? p.seq_len : (tid == 1 ? p.nprev : (tid == 2 ? p.next_pos : p.n_prompt));
    hdr_word = src[b];
  } else if (tid == 4 && p.active) {
    hdr_word = (int)p.active[b];
  }
  // The query rows, the previous step's and its statistics, and the appended token's rows: fetched once per workgroup, a piece
  // a thread, and handed round through LDS.
  const size_t qrow0 = ((size_t)b * p.Hq + (size_t)h * G) * D;
  constexpr int NQ = (2 * 16 * PIECES + kThreads - 1) / kThreads;
  u32x4 qpiece[NQ];
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    const int i = tid + j * kThreads, row = i / PIECES % 16;
    qpiece[j] = u32x4{0u, 0u, 0u, 0u};  // (rows past the group's heads)
    if (row < G) {
      if (i < 16 * PIECES) {
        if (ATTEND) qpiece[j] = load_u32x4(p.q + qrow0 + 8 * (size_t)i);
      } else if (PENDING && i < 2 * 16 * PIECES) {
        qpiece[j] = load_u32x4(p.qprev + qrow0 + 8 * (size_t)(i - 16 * PIECES));
      }
    }
  }
  float ml_word = 0.f;
  if (PENDING && wave == kWaves - 2 && lane < 2 * G) ml_word = p.mlprev[((size_t)b * p.Hq + (size_t)h * G) * 2 + lane];
  const bool new_wave = APPEND && split == 0 && wave == 0;               // starts from the appended token
  const bool row_wave = APPEND && split == 0 && wave == kWaves - 1;      // writes its row into the cache
  u32x4 new_piece = u32x4{0u, 0u, 0u, 0u};
  if (row_wave && lane < 2 * PIECES) new_piece = load_u32x4((lane < PIECES ? p.k_new : p.v_new) + unit * D + 8 * (lane % PIECES));
  __builtin_amdgcn_sched_barrier(0);
  u32x4 kr[VIT], vf[VIT];
  float s_old = 0.f;
  // (paged: the first tile's page is looked up right away and its 32 rows fetched whole: a tile lies inside one page, and a page id
  // is clamped into the pool, so the addresses are valid whatever the length turns out to be)
  const size_t b0 = PAGED ? page_base(page_of(t)) : 0;
  const int t0 = PAGED ? t & (kPageSlots - 1) : t;
  const RowBuffer k_first = row_buffer<D>(Kb + b0, PAGED ? kPageSlots : p.cap);
  load_tile<D>(kr, k_first, t0, lane);
  if (PENDING) {
    const int tok = t + (lane & (kTile - 1));
    s_old = Sb[tok < p.cap ? tok : p.cap - 1];
  }
  __builtin_amdgcn_sched_barrier(0);

  // Hand them round.  The K tile's loads are still in flight across this barrier.  (V's leave behind it, when the length is
  // known: a wave has to issue what it asks for in front of the barrier, and the rows past the sequence come as zeros.)
  if (tid < 5) sm_hdr[tid] = hdr_word;
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    const int i = tid + j * kThreads;
    if (i < (PENDING ? 2 : 1) * 16 * PIECES && (ATTEND || i >= 16 * PIECES))
      *reinterpret_cast<u32x4 *>(sm_q + (i / PIECES - 16 + QPREV) * KSTRIDE + 16 * (i % PIECES)) = qpiece[j];
  }
  if (PENDING && wave == kWaves - 2 && lane < 32) sm_ml[lane] = ml_word;
  if (row_wave && lane < 2 * PIECES) *reinterpret_cast<u32x4 *>(sm_new + 16 * lane) = new_piece;
  __syncthreads();
  // query fragments: lane (g, kg) holds q[g][32*ks + 8*kg .. +7]
  bf16x8 qf[KS], qpf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const unsigned char *src = sm_q + g * KSTRIDE + 64 * ks + 16 * kg;
    if (ATTEND) qf[ks] = *reinterpret_cast<const bf16x8 *>(src);
    if (PENDING) qpf[ks] = *reinterpret_cast<const bf16x8 *>(src + QPREV * KSTRIDE);
  }
  // statistics of the deferred update for heads 4*kg .. 4*kg+3 (the rows this lane gets from
  // the swapped-operand MFMA)
  float mprev[4], inv_lprev[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    mprev[i] = PENDING ? sm_ml[8 * kg + 2 * i] : 0.f;  // (0 past the group's heads)
    inv_lprev[i] = PENDING ? sm_ml[8 * kg + 2 * i + 1] : 0.f;
  }
  // (the same in every lane, and told so to the compiler: ranges, branches and buffers formed from them are scalar then)
  const int len_raw = __builtin_amdgcn_readfirstlane(sm_hdr[0]);
  const int prev_raw = PENDING ? __builtin_amdgcn_readfirstlane(sm_hdr[1]) : 0;
  const int pos_new_all = APPEND ? __builtin_amdgcn_readfirstlane(sm_hdr[2]) : 0;
  const int M = __builtin_amdgcn_readfirstlane(sm_hdr[3]);
  const int act_raw = __builtin_amdgcn_readfirstlane(sm_hdr[4]);

  // ---- what this launch does for sequence b (identical in every workgroup of b) ---------
  // n_rows cache slots are attended from the cache; when a token is appended in the same
  // pass its row is taken from k_new / v_new up front (below), so the tiles never see it.
  const bool act = act_raw != 0;
  int n_old = len_raw;
  n_old = n_old < 0 ? 0 : (n_old > p.cap ? p.cap : n_old);
  const bool appending = ATTEND && APPEND && act && n_old < p.cap;
  const int n_rows = ATTEND && act && (!APPEND || appending) ? n_old : 0, n_now = appending ? n_old + 1 : n_rows;
  if (ATTEND && APPEND && act && !appending && tid == 0 && split == 0 && h == 0) atomicOr(p.status, 1);
  int n_prev = prev_raw;
  n_prev = n_prev < 0 ? 0 : (n_prev > p.cap ? p.cap : n_prev);
  const int n_vis = n_rows > n_prev ? n_rows : n_prev;
  if (ATTEND) {
    const RowBuffer v_first = row_buffer<D>(Vb + b0, PAGED ? (n_rows - (t - t0) < kPageSlots ? n_rows - (t - t0) : kPageSlots) : n_rows);
    load_tile<D>(vf, v_first, t0, lane);
  }
  // workgroups of this unit that produce an attention partial (chunk 0 always does when the
  // sequence is attended: it owns the appended token), and that have any work at all
  // (a workgroup has work iff its first wave's first tile starts inside the sequence)
  constexpr int kFirst = kWaves * kTile;  // slots covered by a workgroup's first tiles
  auto wgs_for = [&](int n) { int c = (n + kFirst - 1) / kFirst; return c < p.nsplit ? c : p.nsplit; };
  const int chunks_now = n_now > 0 ? (wgs_for(n_rows) > 1 ? wgs_for(n_rows) : 1) : 0;
  const int chunks_prev = wgs_for(n_prev);
  const int chunks_vis = chunks_now > chunks_prev ? chunks_now : chunks_prev;
#pragma unroll
  for (int i = 0; i < 4; ++i)  // inv_l = 0 switches padded heads and idle sequences off
    inv_lprev[i] = (PENDING && 4 * kg + i < G && n_prev > 0) ? 1.0f / inv_lprev[i] : 0.f;

  // Every workgroup of the sequence checks in once its reads of seq_len / nprev / next_pos have come
  // back: thread 0 checks in, and its own wave made those reads and has already consumed their values
  // (they went through LDS above), so the atomic is issued after they completed.  The last workgroup
  // to check in advances the three words -- by then no workgroup of the sequence has a read of them
  // outstanding.  It is issued behind the first tile (answers come back in order: a wait for one of the first loads would be
  // a wait for the atomic as well) and its answer is looked at when the waves have been combined.  In the kStream form, whose two loops both may
  // begin with the first tile, it is issued in front of that tile: 8 steps of four layers of 512 units of 1184 slots 1772 us so, 1779 with it
  // behind all tiles, 1830 with the first tile of either loop by itself and the check-in behind it (two layers of 512 units of 2624: the same three times).
  uint32_t seq_ticket = 0xffffffffu;
  auto seq_checkin = [&]() {
    if (ATTEND && tid == 0) seq_ticket = draw_ticket(p.seq_cnt + (size_t)b * p.cnt_stride);
  };
  auto seq_settle = [&]() {
    if (ATTEND && tid == 0 && seq_ticket == (uint32_t)p.nsplit * p.Hkv - 1) {
      __hip_atomic_store(p.seq_cnt + (size_t)b * p.cnt_stride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (p.track) p.nprev[b] = n_now;
      if (APPEND && appending) {
        p.seq_len[b] = n_now;
        p.next_pos[b] = pos_new_all + 1;
      }
    }
  };

  if (split >= chunks_vis) {
    seq_checkin();
    seq_settle();
    return;
  }
  // this wave's contiguous range [ra, rb) behind the first tiles
  const int rounds = STREAM && p.rounds > 1 ? p.rounds : 1;
  const int base = kTile * NW * rounds;
  int per = n_vis > base ? (n_vis - base + NW - 1) / NW : 0;
  // whole tiles per wave: only the last wave with work ends on a partial tile (measured 1-3 % faster than
  // byte-equal ranges that end mid-tile everywhere), and in the paged layout no tile straddles two pages
  per = (per + kTile - 1) & ~(kTile - 1);
  // (handed out from the last wave down: the range that comes up short or empty goes to the unit's first
  // waves, of which wave 0 also takes the appended token; 0.5 % on the many-unit workloads)
  const int ra = base + (NW - 1 - wi) * per;
  const int rb = ra + per < n_vis ? ra + per : n_vis;

  // keep this call's query for the next deferred score update (its own buffer: the old one is
  // still being read by the other workgroups of this launch)
  if (ATTEND && p.track && split == 0 && n_now > 0) {
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      const int i = tid + j * kThreads;
      if (i < 16 * PIECES && i / PIECES < G) store_u32x4(p.qnext + qrow0 + 8 * (size_t)i, qpiece[j]);
    }
  }

  float m_run = -INFINITY, l_run = 0.f;
  f32x4 oacc[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) oacc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};

  // ---- fused append ------------------------------------------------------------------------
  // One wave of the unit takes the appended token: its logit is q.k_new for every head, its
  // weight relative to itself is 1, so the running state starts as (max = logit, sum = 1,
  // output = v_new).  Another wave writes the row into the cache.  All of it overlaps the
  // wait for the first tile.
  if (new_wave && appending) {
    f32x4 a0 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {  // every operand row is k_new
      const bf16x8 kn = *reinterpret_cast<const bf16x8 *>(sm_new + 64 * ks + 16 * kg);
      a0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kn, qf[ks], a0, 0, 0, 0);
    }
    m_run = a0[0] * p.scale_log2;
    l_run = kg == 0 ? 1.f : 0.f;  // per-lane partial sums are added over kg at the end
    if (SPILL && kg == 0 && g < G) p.spill[spill_at(unit, p.cap_pad, G, g, n_old)] = m_run;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
      const bf16x4 v4 = *reinterpret_cast<const bf16x4 *>(sm_new + 2 * D + 32 * cb + 8 * kg);
      oacc[cb] = f32x4{(float)v4[0], (float)v4[1], (float)v4[2], (float)v4[3]};
    }
  }
  if (row_wave && appending) {
    size_t new_row = (size_t)n_old * D;  // element offset of the new row from Kb / Vb
    bool have_row = true;
    if (PAGED) {
      // the slot's page: a fresh one from the free stack when the slot opens a page
      int pg = 0;
      if (lane == 0) {
        const int pi = n_old / kPageSlots;
        if (n_old % kPageSlots == 0) {
          const int idx = atomicSub(p.free_top, 1) - 1;
          if (idx >= 0) {
            pg = p.free_stack[idx];
            p.block_table_w[unit * (size_t)p.max_pages + pi] = pg;
          } else {  // pool exhausted: give the ticket back, drop the row, say so
            atomicAdd(p.free_top, 1);
            atomicOr(p.status, 4);
            pg = -1;
          }
        } else {
          pg = tb[pi];
        }
      }
      pg = __builtin_amdgcn_readfirstlane(pg);
      have_row = pg >= 0 && pg < p.n_pages;
      new_row = ((size_t)(have_row ? pg : 0) * kPageSlots + n_old % kPageSlots) * D;
    }
    if (lane < 2 * PIECES && have_row) store_u32x4((lane < PIECES ? Kb : Vb) + new_row + 8 * (lane % PIECES), new_piece);
    if (lane == 0) {
      Sb[n_old] = p.s_new ? p.s_new[unit] : 0.f;
      p.pos[unit * (size_t)p.cap + n_old] = pos_new_all;
    }
  }

  // A prefetch must not pull another wave's rows: the buffers end where this wave's own range does (or, with no range, its last
  // tile at a fixed place), V's at the end of the sequence.
  int t_fix = t;  // this wave's last tile at a fixed place
  if (STREAM) {
    for (int f = 1; f < rounds; ++f) t_fix = t_fix + kTile * NW < n_vis ? t_fix + kTile * NW : t_fix;
  }
  const int own_end = ra < rb ? rb : (t_fix + kTile < n_vis ? t_fix + kTile : n_vis);
  const int v_end = own_end < n_rows ? own_end : n_rows;
  const RowBuffer k_rows = row_buffer<D>(Kb, own_end), v_rows = row_buffer<D>(Vb, v_end);
  const bool past_caches = STREAM && n_vis > p.fit_slots;
  // paged: the page of the next tile to fetch is looked up one tile ahead of its use
  int pg_nxt = 0;
  if (PAGED) pg_nxt = page_of(clamp_tile(ra, own_end));

  // ---- updated scores leave in bursts (kBurst) ----------------------------------------------------
  // A tile updates 32 scores (128 bytes).  Written tile by tile these are small writes scattered through
  // the read stream, which beyond the memory-side cache cost the memory system far more than their bytes (measured: 4 % of
  // the launch for 1.2 % of the traffic; within it they are absorbed, and bursts at the end of a workgroup only lengthen its
  // tail).  So a wave parks them in LDS and writes a run of consecutive tiles with 16 bytes per lane at once: when the
  // run breaks, when score_tiles have gathered, and when the wave is
  // done.  sc_base: first slot of the run, sc_n: tiles in it, [sc_lo, sc_hi): the slots that may be written
  // (thinking slots below the end of the deferred update and of this wave's share).
  float *sbuf = sm_score[PENDING && BURST ? wave : 0];
  int sc_base = 0, sc_n = 0, sc_lo = 0, sc_hi = 0;
  auto flush_scores = [&]() {
    if (!PENDING || !BURST || sc_n == 0) return;
    wave_lds_fence();
    for (int c0 = 0; c0 < sc_n * kTile; c0 += 256) {
      const int off = c0 + 4 * lane;
      if (off < sc_n * kTile) {
        const f32x4 v = *reinterpret_cast<const f32x4 *>(sbuf + off);
        const int s0 = sc_base + off;
        float *dst = Sb + s0;
        if (s0 >= sc_lo && s0 + 4 <= sc_hi && (reinterpret_cast<uintptr_t>(dst) & 15) == 0) {
          *reinterpret_cast<f32x4 *>(dst) = v;
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (s0 + i >= sc_lo && s0 + i < sc_hi) dst[i] = v[i];
        }
      }
    }
    wave_lds_fence();  // the buffer is written again
    sc_n = 0;
  };

  // ---- kept logits leave in bursts, too -----------------------------------------------------------
  // Parked in LDS in the order in which they lie in memory; a run of consecutive tiles (32 / G of them at most) is written with
  // 1 KB a store instruction.  lg_base: first slot of the run, lg_n: tiles in it, lg_hi: end of the slots it may write (the slot
  // behind may be the appended token's, kept by its own wave).
  float *lbuf = sm_logit[SPILL ? wave : 0];
  int lg_base = 0, lg_n = 0, lg_hi = 0;
  auto flush_logits = [&]() {
    if (!SPILL || lg_n == 0) return;
    wave_lds_fence();
    float *dst = p.spill + spill_at(unit, p.cap_pad, G, 0, lg_base);
    const bool whole = lg_base + kTile * lg_n <= lg_hi;
    for (int off = 4 * lane; off < lg_n * G * kTile; off += 256) {
      const f32x4 v = *reinterpret_cast<const f32x4 *>(lbuf + off);
      const int s0 = lg_base + off / (G * kTile) * kTile + off % kTile;
      if (whole || s0 + 4 <= lg_hi) {
        *reinterpret_cast<f32x4 *>(dst + off) = v;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (s0 + i < lg_hi) dst[off + i] = v[i];
      }
    }
    wave_lds_fence();  // the buffer is written again
    lg_n = 0;
  };

  // ---- one 32-slot tile of this wave -------------------------------------------------------
  // Branch-free apart from two wave-uniform guards; the next tile's loads are issued
  // unconditionally (clamped), so the loop never drains its outstanding loads.
  // t: first slot of the tile; hi: end of the slots of this tile that belong to this wave;
  // tn: first slot of the wave's next tile (any value when there is none: the loads are clamped)
  auto tile = [&](auto PAST, int t, int hi, int tn) {
    constexpr bool past = decltype(PAST)::value;
    const int att_hi = hi < n_rows ? hi : n_rows;
    const int pend_hi = hi < n_prev ? hi : n_prev;

    // the tile's K rows into operand order through the wave's LDS tile: lane (r, kg) gets row r, columns 32*ks + 8*kg .. +7.
    // (A wave's LDS accesses are carried out in order, so K and V of one tile after another share the room.)
    bf16x8 kf[2][KS];
#pragma unroll
    for (int row0 = 0; row0 < kTile; row0 += KROWS) {
#pragma unroll
      for (int it = 0; it < KROWS / VROWS; ++it)
        *reinterpret_cast<u32x4 *>(vst + (VROWS * it + vrow_l) * KSTRIDE + 16 * vpiece) = kr[row0 / VROWS + it];
      wave_lds_fence();
#pragma unroll
      for (int s = 0; s < KROWS / 16; ++s)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          kf[row0 / 16 + s][ks] = *reinterpret_cast<const bf16x8 *>(vst + (16 * s + r16) * KSTRIDE + 64 * ks + 16 * kg);
      if (KROWS < kTile) wave_lds_fence();
    }
    // logits for the current query (A = K rows, B = q) and for the previous one (swapped:
    // accp[s][i] = logit(slot t + 16 s + r16, head 4 kg + i))
    f32x4 acc[2], accp[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
      accp[s] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (ATTEND) acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[s][ks], qf[ks], acc[s], 0, 0, 0);
        if (PENDING) accp[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qpf[ks], kf[s][ks], accp[s], 0, 0, 0);
      }
    }
    const float s_cur = s_old;
    // where the next tile is fetched from; in the paged layout relative to its page
    int nt = tn;
    RowBuffer k_next = k_rows, v_next = v_rows;
    if (PAGED) {
      const int page_start = tn & ~(kPageSlots - 1), left_k = own_end - page_start, left_v = v_end - page_start;
      const size_t nb = page_base(pg_nxt);
      nt = tn - page_start;
      k_next = row_buffer<D>(Kb + nb, left_k < kPageSlots ? left_k : kPageSlots);
      v_next = row_buffer<D>(Vb + nb, left_v < kPageSlots ? left_v : kPageSlots);
      pg_nxt = page_of(clamp_tile(tn + kTile, own_end));
    }
    load_tile<D, past>(kr, k_next, nt, lane);
    if (PENDING) {
      const int tok = tn + (lane & (kTile - 1));
      s_old = Sb[tok < p.cap ? tok : p.cap - 1];
    }

    // ---- deferred score update: S[slot] += sum over the group of alpha_prev[g][slot] --------
    if (PENDING && t < pend_hi) {
      float part[2];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        float a = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) a += fast_exp2(accp[s][i] * p.scale_log2 - mprev[i]) * inv_lprev[i];
        if (G > 4) a += __shfl_xor(a, 16);
        if (G > 8) a += __shfl_xor(a, 32);
        part[s] = a;
      }
      if (G <= 8) {  // lanes of row group 0 (and 1) hold the sums; hand sub-tile 1 to row group 1
        const float other = __shfl(part[1], r16);
        if (kg == 1) part[1] = other;
      }
      // lane < 32 holds the new score of slot t + lane (sub-tile kg, row r16): write it, or park it
      const float s_upd = s_cur + (kg == 0 ? part[0] : part[1]);
      if (!BURST) {
        const int tok = t + lane;
        if (lane < kTile && tok < pend_hi && tok >= M) Sb[tok] = s_upd;
      } else {
        if (sc_n > 0 && (t != sc_base + kTile * sc_n || sc_n >= p.score_tiles)) flush_scores();
        if (sc_n == 0) {
          sc_base = t;
          sc_lo = t > M ? t : M;
        }
        if (lane < kTile) sbuf[kTile * sc_n + lane] = s_upd;
        ++sc_n;
        sc_hi = pend_hi;
      }
    }

    // ---- attention for the current query --------------------------------------------------
    // (also of a tile behind the slots it attends, which the owed update alone may have: its weights are 0.  Around a branch the wait
    // for the next tile's K rows would be one for its V rows, too: loads are waited for by their number, and the way with fewer counts.)
    if (ATTEND) {
      // acc[s][i] = logit(slot t + 16 s + 4 kg + i, head g)
      float x[8];
      float mx = -INFINITY;
      if (t + kTile <= att_hi) {  // wave-uniform: a full tile needs no masks
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          x[e] = acc[e >> 2][e & 3] * p.scale_log2;
          mx = fmaxf(mx, x[e]);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int tok = t + 16 * (e >> 2) + 4 * kg + (e & 3);
          x[e] = tok < att_hi ? acc[e >> 2][e & 3] * p.scale_log2 : -INFINITY;
          mx = fmaxf(mx, x[e]);
        }
      }
      if (SPILL && t < att_hi) {
        if (lg_n > 0 && (t != lg_base + kTile * lg_n || (lg_n + 1) * G > kLogitRows)) flush_logits();
        if (lg_n == 0) lg_base = t;
        if (g < G) {  // this lane's 8 logits of head g: slots t + 16 s + 4 kg .. +3
#pragma unroll
          for (int s2 = 0; s2 < 2; ++s2)
            *reinterpret_cast<f32x4 *>(lbuf + (lg_n * G + g) * kTile + 16 * s2 + 4 * kg) = f32x4{x[4 * s2], x[4 * s2 + 1], x[4 * s2 + 2], x[4 * s2 + 3]};
        }
        ++lg_n;
        lg_hi = att_hi;
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float m_run_next = fmaxf(m_run, mx);
      const float m_new = m_run_next == -INFINITY ? 0.f : m_run_next;  // (-inf: no slot so far)
      const float corr = fast_exp2(m_run - m_new);  // m_run = -inf on the first tile -> 0
      m_run = m_run_next;
      bf16x8 ph, pl;
      float psum = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float pe = fast_exp2(x[e] - m_new);
        psum += pe;
        const __bf16 hi = (__bf16)pe;
        ph[e] = hi;
        pl[e] = (__bf16)(pe - (float)hi);
      }
      l_run = l_run * corr + psum;
      {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) oacc[cb] *= corr;
      }
      // stage this tile's V rows in the wave's LDS tile, then fetch the next tile's
#pragma unroll
      for (int it = 0; it < VIT; ++it)
        *reinterpret_cast<u32x4 *>(vst + (VROWS * it + vrow_l) * VSTRIDE + 16 * vpiece) = vf[it];
      wave_lds_fence();
      load_tile<D, past>(vf, v_next, nt, lane);
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        // V^T operand: lane (c = 16 cb + r16, kg) gets V[t + 16 s + 4 kg + i][c] as element 4 s + i.
        // ds_read_b64_tr_b16: within 16 lanes, lane i's element e comes from source lane
        // 4 e + i/4, element i%4; so source lane j points at row (j / 4), columns 4 (j % 4) .. +3.
        const unsigned char *src = vst + (4 * kg + (r16 >> 2)) * VSTRIDE + 2 * (16 * cb + 4 * (r16 & 3));
        i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) i16x4 *)(src));
        i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) i16x4 *)(src + 16 * VSTRIDE));
        i16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        const bf16x8 vt = __builtin_bit_cast(bf16x8, both);
        oacc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt, ph, oacc[cb], 0, 0, 0);
        oacc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vt, pl, oacc[cb], 0, 0, 0);
      }
      wave_lds_fence();
    }
  };

  constexpr std::false_type kThrough{};
  constexpr std::true_type kPast{};
  if constexpr (!STREAM) {
    if (t < n_vis) tile(kThrough, t, t + kTile < n_vis ? t + kTile : n_vis, ra);
    seq_checkin();
    for (t = ra; t < rb; t += kTile) tile(kThrough, t, rb, t + kTile);
  } else {
    // The tiles at fixed places, then the wave's range: one loop over those whose next tile is loaded through the caches, one over the others.
    // (Both ways of loading in one loop leave their rows in different registers, and to bring those together is to wait for the loads.)
    auto behind = [&](int at) { return at < t_fix ? at + kTile * NW : at == t_fix ? ra : at + kTile; };
    auto end_of = [&](int at) { return at > t_fix ? rb : at + kTile < n_vis ? at + kTile : n_vis; };
    seq_checkin();
    if (t < n_vis) {
      const int through_end = past_caches ? t_fix : t_fix < rb ? rb : t_fix + 1;
      for (; t < through_end; t = behind(t)) tile(kThrough, t, end_of(t), behind(t));
      if (past_caches)
        for (; t <= t_fix || t < rb; t = behind(t)) tile(kPast, t, end_of(t), behind(t));
    }
  }
  flush_scores();
  flush_logits();

  if (!ATTEND) return;
  // with several chunks per unit: draw this workgroup's ticket now, so that the round trip of the atomic
  // overlaps the combine below.  (The holder of the last ticket merges, whenever it gets there.)
  uint32_t unit_ticket = 0;
  if (chunks_vis > 1 && tid == 0) unit_ticket = draw_ticket(p.unit_cnt + unit * p.cnt_stride);
  const bool has_partial = split < chunks_now;  // workgroup-uniform; false: the chunk only carried a deferred update
  if (chunks_vis == 1 && !has_partial) {
    seq_settle();
    return;
  }

  constexpr int NE = (16 * D + kThreads - 1) / kThreads;  // output elements per thread at the largest group size
  const int ne = (G * D + kThreads - 1) / kThreads;
  const size_t ubase = unit * p.nsplit * (size_t)G;

  // ---- combine the waves -----------------------------------------------------------------
  // (sm_l holds a wave's sum relative to the workgroup's maximum, sm_max that maximum, behind the second barrier)
  float *ored = reinterpret_cast<float *>(smem);
  if (has_partial) {
  l_run += __shfl_xor(l_run, 16);
  l_run += __shfl_xor(l_run, 32);
  if (kg == 0) sm_m[wave][g] = m_run;
  __syncthreads();
  float mstar = sm_m[0][g];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) mstar = fmaxf(mstar, sm_m[w][g]);
  const float f = (m_run == -INFINITY) ? 0.f : fast_exp2(m_run - mstar);
  if (g < G) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      f32x4 v = oacc[cb] * f;
      *reinterpret_cast<f32x4 *>(ored + (wave * 16 + g) * OSTRIDE + 16 * cb + 4 * kg) = v;
    }
  }
  if (kg == 0) {
    sm_l[wave][g] = l_run * f;
    if (wave == 0) sm_max[g] = mstar;
  }
  __syncthreads();
  }
  auto sum_of = [&](int gg) {  // softmax sum of this workgroup's slots
    float ls = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) ls += sm_l[w][gg];
    return ls;
  };

  seq_settle();

  const size_t orow0 = (size_t)b * p.Hq + (size_t)h * G;  // first query head of this group
  if (chunks_vis == 1) {
    // the chunk is the whole cache: finish here
    for (int idx = tid; idx < G * D; idx += kThreads) {
      const int gg = idx / D, c = idx % D;
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) sum += ored[(w * 16 + gg) * OSTRIDE + c];
      p.out[(orow0 + gg) * D + c] = sum / sum_of(gg);
    }
    if (tid < G) {
      const float ls = sum_of(tid);
      if (p.lse) p.lse[orow0 + tid] = (sm_max[tid] + log2f(ls)) * 0.6931471805599453f;
      if (p.track) {
        p.mlprev[(orow0 + tid) * 2] = sm_max[tid];
        p.mlprev[(orow0 + tid) * 2 + 1] = ls;
      }
    }
    return;
  }

  // ---- several chunks: publish the partial, the holder of the last ticket merges ----------------
  float own_o[NE];
#pragma unroll
  for (int k = 0; k < NE; ++k) own_o[k] = 0.f;
  if (has_partial) {
    const size_t pbase = (unit * p.nsplit + split) * (size_t)G;
#pragma unroll
    for (int k = 0; k < NE; ++k) {
      const int idx = tid + k * kThreads;
      if (k < ne && idx < G * D) {
        const int gg = idx / D, c = idx % D;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) sum += ored[(w * 16 + gg) * OSTRIDE + c];
        own_o[k] = sum;
        tagged_store(&p.part_o[(pbase + gg) * D + c], sum, p.tag);
      }
    }
    if (tid < G) {
      tagged_store(&p.part_ml[(pbase + tid) * 2 + 0], sm_max[tid], p.tag);
      tagged_store(&p.part_ml[(pbase + tid) * 2 + 1], sum_of(tid), p.tag);
    }
  }
  // the ticket was drawn when this workgroup's first wave left its tile loop; its answer is looked at now
  if (tid == 0) sm_flag = unit_ticket;
  __syncthreads();
  const bool merger = sm_flag == (uint32_t)chunks_vis - 1;
  if (!merger) return;
  if (tid == 0) __hip_atomic_store(p.unit_cnt + unit * p.cnt_stride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (chunks_now == 0) return;

  // Merging: thread tid owns output elements tid + k * kThreads, k < E, in its own partial and in the merge; chunks are
  // merged N at a time.  Asking for a group means: threads 0 .. 16 * N - 1 request the (max, sum) of one (head, chunk) each, every
  // thread its elements of the group's partials; this workgroup's own partial never
  // comes from memory.  A round of asking takes a trip to the level all XCDs share, so with few elements per thread and many
  // chunks as many are asked for at once as the same registers hold.  The chunks' weights are formed once per head, across the
  // lanes that hold its statistics.
  constexpr int kMostChunks = WIDE ? kThreads / 16 : 4;  // whose statistics are asked for at once, one thread per (head, chunk)
  __shared__ __align__(16) float sm_w[16][kMostChunks];
  __shared__ float sm_old[16], sm_sum[16];  // weight of the groups before, sum so far
  auto merge = [&](auto E_, auto N_) {
    constexpr int E = decltype(E_)::value, N = decltype(N_)::value;
    static_assert(N <= kMostChunks && 16 * N <= kThreads, "one thread per (chunk, head)");
    uint64_t ask_o[E][N], ask_m, ask_l;
    // (uniform.  At head_dim 64 it spares groups of up to eight heads the second element, 0.5 - 2 % of a launch of 10 to 33
    // chunks; at head_dim 128 it costs the eight-chunk merges 1 %)
    auto has = [&](int k) { return D == 128 || WIDE || k < ne; };
    const int my_g = tid / N, my_j = tid % N;  // whose statistics this thread asks for
    const bool asks = tid < 16 * N && my_g < G;
    auto ask_group = [&](int s0) {
      ask_m = ask_l = (uint64_t)p.tag << 32;  // nothing to wait for
      if (asks && s0 + my_j < chunks_now && !(has_partial && s0 + my_j == split)) {
        const uint64_t *src = &p.part_ml[(ubase + (size_t)(s0 + my_j) * G + my_g) * 2];
        ask_m = tagged_load(src);
        ask_l = tagged_load(src + 1);
      }
#pragma unroll
      for (int k = 0; k < E; ++k) {
        const int idx = tid + k * kThreads;
#pragma unroll
        for (int j = 0; j < N; ++j) {
          const int sj = s0 + j;
          ask_o[k][j] = (uint64_t)p.tag << 32;
          if (has(k) && idx < G * D && sj < chunks_now && !(has_partial && sj == split))
            ask_o[k][j] = tagged_load(&p.part_o[(ubase + (size_t)sj * G + idx / D) * D + idx % D]);
        }
      }
    };
    auto group_fresh = [&]() {
      uint32_t differs = ((uint32_t)(ask_m >> 32) ^ p.tag) | ((uint32_t)(ask_l >> 32) ^ p.tag);
#pragma unroll
      for (int k = 0; k < E; ++k)
#pragma unroll
        for (int j = 0; j < N; ++j) differs |= (uint32_t)(ask_o[k][j] >> 32) ^ p.tag;
      return differs == 0;
    };
    // (finite: chunks without a finite logit weigh exp2(-inf - m_all) = 0 then, also where no other one has come before them)
    float m_all = kLowest, l_all = 0.f, o_e[E];
#pragma unroll
    for (int k = 0; k < E; ++k) o_e[k] = 0.f;
    for (int s0 = 0; s0 < chunks_now; s0 += N) {
      ask_group(s0);
      while (!group_fresh()) ask_group(s0);  // a word that is not this launch's yet is on its way: ask again
      if (asks) {
        const int sj = s0 + my_j;
        const bool mine = has_partial && sj == split, any = sj < chunks_now;
        const float mj = !any ? -INFINITY : mine ? sm_max[my_g] : tagged_value(ask_m);
        const float lj = !any ? 0.f : mine ? sum_of(my_g) : tagged_value(ask_l);
        float mn = mj;
#pragma unroll
        for (int x = 1; x < N; x *= 2) mn = fmaxf(mn, __shfl_xor(mn, x));
        mn = fmaxf(mn, m_all);
        const float old = fast_exp2(m_all - mn), wj = fast_exp2(mj - mn);
        float l = wj * lj;
#pragma unroll
        for (int x = 1; x < N; x *= 2) l += __shfl_xor(l, x);
        l_all = fmaf(l_all, old, l);
        m_all = mn;
        sm_w[my_g][my_j] = wj;
        if (my_j == 0) {
          sm_old[my_g] = old;
          sm_sum[my_g] = l_all;
        }
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < E; ++k) {
        const int idx = tid + k * kThreads;
        if (has(k) && idx < G * D) {
          const int gg = idx / D;
          float o = o_e[k] * sm_old[gg];
#pragma unroll
          for (int j = 0; j < N; j += 4) {
            const f32x4 w = *reinterpret_cast<const f32x4 *>(&sm_w[gg][j]);
#pragma unroll
            for (int i = 0; i < 4; ++i)
              o = fmaf((has_partial && s0 + j + i == split) ? own_o[k] : tagged_value(ask_o[k][j + i]), w[i], o);
          }
          o_e[k] = o;
        }
      }
      if (s0 + N < chunks_now) __syncthreads();  // the weights' LDS is written again
    }
    if (asks && my_j == 0) {
      if (p.lse) p.lse[orow0 + my_g] = (m_all + log2f(l_all)) * 0.6931471805599453f;
      if (p.track) {
        p.mlprev[(orow0 + my_g) * 2] = m_all;
        p.mlprev[(orow0 + my_g) * 2 + 1] = l_all;
      }
    }
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int idx = tid + k * kThreads;
      if (idx < G * D) p.out[orow0 * D + idx] = o_e[k] / sm_sum[idx / D];
    }
  };
  // (where the host chooses the wide merges: wide_merge in dynts.hip)
  if constexpr (WIDE) {
    if (ne == 1 && chunks_now > kWideFrom1) return merge(std::integral_constant<int, 1>{}, std::integral_constant<int, 32>{});
    if constexpr (D == 128) {
      if (ne == 2 && chunks_now > kWideFrom2) return merge(std::integral_constant<int, 2>{}, std::integral_constant<int, 8>{});
    }
  }
  merge(std::integral_constant<int, NE>{}, std::integral_constant<int, 4>{});
}

// The score update of a step whose logits were kept (AttendParams::spill): S[slot] += sum over the group of
// 2^(logit - max) / sum, for the thinking slots that step attended, with that step's final softmax
// statistics -- the same arithmetic as the deferred update inside attend_kernel, fed from 4 * G bytes per slot
// instead of a K row.  grid (ceil(cap / (256 * kApplyPerThread)), Hkv * Nb), 256 threads.
constexpr int kApplyPerThread = 4;
__global__ __launch_bounds__(256) void apply_spill_kernel(float *S, const float *spill, const float *mlprev,
                                                          const int32_t *nprev, const int32_t *n_prompt, int Hkv, int Hq,
                                                          int G, int cap, int cap_pad) {
  const int unit = blockIdx.y, b = unit / Hkv, h = unit - b * Hkv;
  const int n = nprev[b] < cap ? nprev[b] : cap, M = n_prompt[b];
  const int j0 = (blockIdx.x * 256 + threadIdx.x) * kApplyPerThread;
  if (j0 >= n || j0 + kApplyPerThread <= M) return;
  float add[kApplyPerThread];
#pragma unroll
  for (int i = 0; i < kApplyPerThread; ++i) add[i] = 0.f;
  for (int g = 0; g < G; ++g) {
    const float *ml = mlprev + ((size_t)b * Hq + (size_t)h * G + g) * 2;
    const float m = ml[0], inv_l = 1.0f / ml[1];
    const f32x4 x = *reinterpret_cast<const f32x4 *>(spill + spill_at((size_t)unit, cap_pad, G, g, j0));
#pragma unroll
    for (int i = 0; i < kApplyPerThread; ++i) add[i] = fmaf(fast_exp2(x[i] - m), inv_l, add[i]);
  }
  float *Su = S + (size_t)unit * cap;
#pragma unroll
  for (int i = 0; i < kApplyPerThread; ++i)
    if (j0 + i < n && j0 + i >= M) Su[j0 + i] += add[i];
}

}  // namespace dynts
