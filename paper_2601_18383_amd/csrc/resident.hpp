// Consecutive decode steps of one layer on a cache that the chip holds, in one launch (dynts_decode_loop between two triggers).
//
// A step on a small cache takes 5 to 13 us a launch whatever it computes: the launch itself, the sequence's words, K, V behind them, the
// combination of the waves, the hand-over between workgroups, each a trip to memory that the next one waits for.  So here the
// cache stays on the chip: one workgroup of eight waves per (sequence, KV head), and a wave keeps T tiles of 32 slots as MFMA operands in its registers
// through all steps of the launch.  A step then reads its query and its new row, which are asked for two steps ahead, and writes
// its output; a new row is put into the registers of the wave whose tile its slot lies in, and rows, scores and positions go to memory
// once, at the end.
//
// Caches of several chunks of 256 slots (PART) have a workgroup per chunk, which never waits for another one: it leaves its partials of every step,
// merge_run_kernel merges those of all steps at once, and run_scores_kernel makes the updates, a wave a tile of K.
//
// The arithmetic is attend_kernel's to the last bit, so that it makes no difference which of the two made a step: which wave takes which
// tile, the new token as the first wave's initial state, tiles of a wave one after the other, chunks merged in the same groups.  So are the
// things it leaves: the last step's update is owed (query, statistics, slots), or its logits are kept for the trigger that follows.
//
// What bounds it now: a chain of some 400 dependent instructions a wave and step, two waves a SIMD -- logits, maximum, weights, products, two
// barriers around the waves' combination, division, scores.  What that chain waits for is kept short: reads of LDS are asked for in groups
// before the first is used, the new row is put in between the barriers, with masks (its wave is waited for), and a score tile's two halves go side by
// side.  Each read and half waited for by itself, a launch of 64 steps on 18 chunks took 147 us and takes 129; 16 steps of head_dim 64 33.0 and 31.4.
// One barrier instead of two, each wave weighing all eight waves' outputs, took 0.2 to 0.4 us a step more.
// us a step, a launch each / so, runs of 32 steps: head_dim 64, 4 heads a group, 2 units of 250 slots 5.46 / 1.86, 128 of 510 (two chunks) 7.6 / 2.9;
// head_dim 128, 4 heads, 8 units of 250 6.6 / 2.5, of 1000 8.5 / 3.2, of 4544 (18 chunks) 11.7 / 3.3; 7 heads, 512 units of 510 26.3 / 7.5.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attend.hpp"

namespace dynts {

constexpr int kResWaves = 8, kResThreads = 64 * kResWaves;
constexpr int kResSlots = kResWaves * kTile;  // slots that one tile a wave holds
constexpr int kResTiles = 2;                  // tiles a wave keeps at most
constexpr int kResSteps = 1024;               // steps of a launch at most,
constexpr int kPartSteps = 64;                // and of one that leaves partials

struct ResidentParams {
  uint16_t *K, *V;          // layer base, [Nb][Hkv][cap][D]
  float *S;                 // [Nb][Hkv][cap]
  int32_t *pos;             // [Nb][Hkv][cap]
  int32_t *seq_len;         // [Nb]
  const int32_t *n_prompt;  // [Nb]
  int32_t *next_pos;        // [Nb]
  // step i's: base + i * stride elements
  const uint16_t *q;        // [Nb][Hq][D], q_stride
  const uint16_t *k_new, *v_new;  // [Nb][Hkv][D], kv_stride
  const float *s_new;       // [Nb][Hkv] or null, Nb * Hkv
  const uint8_t *active;    // [Nb] or null, Nb
  float *out;               // [Nb][Hq][D], out_stride (0, or so large that no two steps' overlap)
  size_t q_stride, kv_stride, out_stride;
  int steps;
  // the deferred update (see AttendParams): the one owed from before (owed != 0), and where the last step's is kept
  const uint16_t *qprev;
  uint16_t *qnext;          // (behind an even number of steps the same place: written when every chunk's workgroup has read it)
  float *mlprev;
  int32_t *nprev;
  uint32_t *seq_cnt;        // [Nb][cnt_stride] arrival counters, zero between launches
  int cnt_stride;
  int32_t *status;
  int Nb, Hq, Hkv, G, cap;
  int track;                // scores are accumulated from attention
  int owed;                 // an update is owed from before this launch
  float *spill;             // the last step's logits are kept (see AttendParams), or null
  int cap_pad;
  float scale_log2;
  // caches of several chunks: a launch of their steps leaves
  int units, chunks;        // Nb * Hkv; of 256 slots
  float *part_o, *part_ml;  // [steps][units][chunks][G][D], [..][G][2]: the chunks' partials (see attend_kernel)
  float *stats;             // [steps][units][16][2]: (max, 1 / sum) of the steps' softmax (merge_run_kernel)
  int32_t *n_of;            // [steps][Nb]: slots that the step attended in the cache, -1: the sequence was not attended
  int32_t *rec;             // [Nb][4]: slots before and behind the run, next position, whether the last step attended
  int wide;                 // merges of 32 and of 8 chunks at a time (wide_merge in dynts.hip)
};

// A lane's x and that of the lane 16 (32) further on in the pair of rows (halves) of the wave: no trip through LDS.
struct Pair {
  float low, high;
};
__device__ __forceinline__ Pair over_16(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ Pair over_32(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}
// over a wave's four rows of 16 lanes, in every lane
__device__ __forceinline__ float max_over_rows(float x) {
  Pair p = over_16(x);
  p = over_32(fmaxf(p.low, p.high));
  return fmaxf(p.low, p.high);
}
__device__ __forceinline__ float sum_over_rows(float x) {
  Pair p = over_16(x);
  p = over_32(p.low + p.high);
  return p.low + p.high;
}

template <int D, int T, bool PART>
__global__ __launch_bounds__(kResThreads, 2) void resident_kernel(const ResidentParams p) {
  static_assert(!PART || T == 1, "a chunk is a tile a wave");
  constexpr bool FULL = D == 128 && T == 2;  // no register of the 256 is left in the loop (32 steps and their trigger on 512 units of 510 slots, 7
                                             // heads: 264 us with two values more, in scratch memory, 262 so; the other forms have room)
  constexpr int KS = D / 32, CB = D / 16, PIECES = D / 8;
  constexpr int VROWS = 64 / PIECES, VIT = kTile / VROWS;  // rows of one wave-wide 16-byte load
  constexpr int STRIDE = 2 * D + 32;                       // bytes per staged row (see attend_kernel)
  constexpr int OSTRIDE = D + 4;
  constexpr int NE = (16 * D + kResThreads - 1) / kResThreads;  // output elements per thread at the largest group
  static_assert(kTile * STRIDE >= 16 * OSTRIDE * 4, "the tiles' LDS is reused for the outputs");
  __shared__ __align__(16) unsigned char smem[kResWaves * kTile * STRIDE];
  constexpr int IN = 18 * STRIDE;  // a step's query rows, its K and its V row
  __shared__ __align__(16) unsigned char sm_in[2 * IN];  // of even and of odd steps
  __shared__ __align__(16) float sm_m[16][kResWaves], sm_l[16][kResWaves];
  struct Stats { float m[16], l[16], inv_l[16]; };            // of a step's softmax: maximum, sum, its inverse
  __shared__ __align__(16) Stats sm_stats[kResWaves];         // (each wave its own: no barrier)
  __shared__ int32_t sm_hdr[5];
  __shared__ int16_t sm_step[kResSlots * T];                  // the step that appended each new row
  __shared__ uint8_t sm_active[kResSteps + 4];                // of each step

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kg = lane >> 4, g = r16;
  // (a division leaves uniform values in vector registers, and every address formed from them)
  const int unit = PART ? __builtin_amdgcn_readfirstlane(blockIdx.x / p.chunks) : blockIdx.x, chunk = PART ? blockIdx.x - unit * p.chunks : 0;
  const int b = __builtin_amdgcn_readfirstlane(unit / p.Hkv), h = unit - b * p.Hkv, G = p.G;
  uint16_t *Kb = p.K + (size_t)unit * p.cap * D, *Vb = p.V + (size_t)unit * p.cap * D;
  float *Sb = p.S + (size_t)unit * p.cap;
  const size_t row0 = (size_t)b * p.Hq + (size_t)h * G;  // the group's first query head

  // ---- a step's inputs, asked for two steps ahead: 16 bytes a thread of its query rows, its K and its V row --------
  // (no branch and no wait but for what is used: threads without a piece repeat the first)
  const int n_pieces = (G + 2) * PIECES, my_row = tid / PIECES;
  const bool has_piece = tid < n_pieces;
  const uint16_t *src = p.q + row0 * D + (my_row < G ? 8 * tid : 0);
  if (has_piece && my_row >= G) src = (my_row == G ? p.k_new : p.v_new) + (size_t)unit * D + 8 * (tid % PIECES);
  const size_t src_stride = has_piece && my_row >= G ? p.kv_stride : p.q_stride;
  unsigned char *put = sm_in + (my_row < G ? my_row : 16 + my_row - G) * STRIDE + 16 * (tid % PIECES);
  auto fetch = [&](int i, u32x4 &piece) {  // (called for one step after the other; behind the last, for the last again)
    piece = load_u32x4(src);
    if (i + 1 < p.steps) src += src_stride;
  };
  auto stage = [&](int i, const u32x4 &piece) {
    if (has_piece) *reinterpret_cast<u32x4 *>(put + (i & 1) * IN) = piece;
  };
  for (int i = tid; i < p.steps; i += kResThreads) sm_active[i] = p.active ? p.active[(size_t)i * p.Nb + b] : 1;

  // The words of the sequence are rewritten by the last of its workgroups to check in, which each does when its wave 0 has them.
  if (tid < 5) {
    const int32_t *w = tid == 0 ? p.seq_len : tid == 1 ? p.nprev : tid == 2 ? p.next_pos : p.n_prompt;
    sm_hdr[tid] = tid < 4 ? w[b] : 0;
  }
  u32x4 piece_a, piece_b;
  fetch(0, piece_a);
  for (int i = tid; i < 2 * (16 - G) * PIECES; i += kResThreads)  // (rows past the group's heads)
    *reinterpret_cast<u32x4 *>(sm_in + (i & 1) * IN + (G + (i >> 1) / PIECES) * STRIDE + 16 * ((i >> 1) % PIECES)) = u32x4{0u, 0u, 0u, 0u};
  __syncthreads();
  uint32_t seq_ticket = 0xffffffffu;
  if (!PART && tid == 0) seq_ticket = draw_ticket(p.seq_cnt + (size_t)b * p.cnt_stride);
  int n = __builtin_amdgcn_readfirstlane(sm_hdr[0]);
  n = n < 0 ? 0 : (n > p.cap ? p.cap : n);
  const int n_entry = n, M = __builtin_amdgcn_readfirstlane(sm_hdr[3]);
  if (PART && chunk > 0 && kResSlots * chunk > n + p.steps) return;  // no step gets so far

  // Tile j of this wave starts at slot first(j).  (A wave's second tile lies where attend_kernel has it, counted from the end.)
  auto first = [&](int j) { return kResSlots * chunk + kTile * (j == 0 ? wave : 2 * kResWaves - 1 - wave); };

  // ---- the cache, as operands (see attend_kernel); rows past the sequence are zeros ---------------------------------
  bf16x8 kf[T][2][KS];
  i16x8 vt[T][CB];
  float s_reg[T];  // lane < 32: score of slot first(tile) + lane
  unsigned char *vst = smem + wave * kTile * STRIDE;
#pragma unroll
  for (int j = 0; j < T; ++j) {
    const int t = first(j);
    u32x4 kr[VIT], vr[VIT];
    load_tile<D>(kr, row_buffer<D>(Kb, n), t, lane);
    load_tile<D>(vr, row_buffer<D>(Vb, n), t, lane);
    const int tok = t + (lane & (kTile - 1));
    s_reg[j] = tok < n ? Sb[tok] : 0.f;
#pragma unroll
    for (int it = 0; it < VIT; ++it)
      *reinterpret_cast<u32x4 *>(vst + (VROWS * it + lane / PIECES) * STRIDE + 16 * (lane % PIECES)) = kr[it];
    wave_lds_fence();
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        kf[j][s][ks] = *reinterpret_cast<const bf16x8 *>(vst + (16 * s + r16) * STRIDE + 64 * ks + 16 * kg);
    wave_lds_fence();
#pragma unroll
    for (int it = 0; it < VIT; ++it)
      *reinterpret_cast<u32x4 *>(vst + (VROWS * it + lane / PIECES) * STRIDE + 16 * (lane % PIECES)) = vr[it];
    wave_lds_fence();
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {  // lane (c = 16 cb + r16, kg): V[t + 16 s + 4 kg + i][c] as element 4 s + i
      const unsigned char *at = vst + (4 * kg + (r16 >> 2)) * STRIDE + 2 * (16 * cb + 4 * (r16 & 3));
      const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)(at));
      const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)(at + 16 * STRIDE));
      vt[j][cb] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
    wave_lds_fence();
  }

  // S[slot] += sum over the group of 2^(logit - m) / l for the thinking slots below lim of tile j; m, inv_l: of heads 4 kg .. 4 kg + 3
  auto score_tile = [&](int j, const bf16x8 (&qv)[KS], const f32x4 &m, const f32x4 &inv_l, int lim) {
    if (first(j) >= lim) return;
    f32x4 e[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};  // [s]: logit of slot 16 s + r16, head 4 kg + i
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int s = 0; s < 2; ++s) e[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qv[ks], kf[j][s][ks], e[s], 0, 0, 0);
    float part[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {  // (both sub-tiles, and then the group's size once)
      part[s] = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) part[s] += fast_exp2(e[s][i] * p.scale_log2 - m[i]) * inv_l[i];
    }
    if (G > 8) {
      part[0] = sum_over_rows(part[0]);
      part[1] = sum_over_rows(part[1]);
    } else if (G > 4) {
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const Pair r = over_16(part[s]);
        part[s] = r.low + r.high;
      }
    } else {
      part[1] = over_16(part[1]).low;  // (the first row's lanes hold the sums; the second takes sub-tile 1)
    }
    const int tok = first(j) + lane;
    if (lane < kTile && tok < lim && tok >= M) s_reg[j] += kg == 0 ? part[0] : part[1];
  };

  // ---- the update owed from before ------------------------------------------------------------------------------
  if (p.owed) {
    int n_prev = __builtin_amdgcn_readfirstlane(sm_hdr[1]);
    n_prev = n_prev < 0 ? 0 : (n_prev > n ? n : n_prev);
    if (n_prev > 0) {
      f32x4 m = {0.f, 0.f, 0.f, 0.f}, inv_l = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (4 * kg + i < G) {
          m[i] = p.mlprev[(row0 + 4 * kg + i) * 2];
          inv_l[i] = 1.0f / p.mlprev[(row0 + 4 * kg + i) * 2 + 1];
        }
      }
      bf16x8 qp[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        qp[ks] = __builtin_bit_cast(bf16x8, g < G ? load_u32x4(p.qprev + (row0 + g) * D + 32 * ks + 8 * kg) : u32x4{0u, 0u, 0u, 0u});
#pragma unroll
      for (int j = 0; j < T; ++j) score_tile(j, qp, m, inv_l, n_prev);
    }
  }
  __syncthreads();  // the tiles' LDS becomes the outputs'; every wave has its operands
  __builtin_amdgcn_s_waitcnt(0x0f70);  // (every load so far: one that the loop might still be owed would be waited for in each round)
  if (FULL && tid == 0) sm_hdr[4] = (int32_t)seq_ticket;
  stage(0, piece_a);
  fetch(1, piece_b);
  fetch(2, piece_a);
  __syncthreads();

  float *ored = reinterpret_cast<float *>(smem);
  bool last_attended = false;
  int n_dropped = 0;
  int act_next = sm_active[0];
  float *const out_rows = p.out + row0 * D;
  Stats &stats = sm_stats[wave];

  auto load_q = [&](bf16x8 (&qf)[KS], const unsigned char *in) {  // lane (g, kg): q[g][32 ks + 8 kg .. +7]
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8 *>(in + g * STRIDE + 64 * ks + 16 * kg);
  };
  // Step i; LAST: the launch's last, whose update is left owed (all the others, steps below `most`, make theirs).
  const int most = p.steps - 1;
  auto step = [&](auto LAST, int i, u32x4 &next) {
    constexpr bool last = decltype(LAST)::value;
    // ---- what this step does (the same in the whole workgroup) ---------------------------------------------
    const unsigned char *in = sm_in + (i & 1) * IN;
    const bool act = __builtin_amdgcn_readfirstlane(last ? (int)sm_active[most] : act_next) != 0 && (last || i < most);
    act_next = sm_active[i + 1];
    const int n_rows = __builtin_amdgcn_readfirstlane(n);
    const bool attended = act && n_rows < p.cap;
    n_dropped += act && !attended ? 1 : 0;
    if (last) last_attended = attended;
    n = attended ? n_rows + 1 : n_rows;
    const bool here = attended && (!PART || chunk == 0 || kResSlots * chunk < n_rows);  // (the new token is the first chunk's)
    if (PART && h == 0 && chunk == 0 && tid == 0) p.n_of[(size_t)i * p.Nb + b] = attended ? n_rows : -1;
    float m_run = -INFINITY, l_run = 0.f;
    f32x4 oacc[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) oacc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (here) {
      bf16x8 qf[KS];
      load_q(qf, in);
      if (chunk == 0 && wave == 0) {  // the new token (see attend_kernel)
        f32x4 a0 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const bf16x8 kn = *reinterpret_cast<const bf16x8 *>(in + 16 * STRIDE + 64 * ks + 16 * kg);
          a0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kn, qf[ks], a0, 0, 0, 0);
        }
        m_run = a0[0] * p.scale_log2;
        l_run = kg == 0 ? 1.f : 0.f;
        if (last && p.spill && kg == 0 && g < G) p.spill[spill_at((size_t)unit, p.cap_pad, G, g, n_rows)] = m_run;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
          const bf16x4 v4 = *reinterpret_cast<const bf16x4 *>(in + 17 * STRIDE + 32 * cb + 8 * kg);
          oacc[cb] = f32x4{(float)v4[0], (float)v4[1], (float)v4[2], (float)v4[3]};
        }
      }
      // ---- this wave's slots -------------------------------------------------------------------------------
#pragma unroll
      for (int j = 0; j < T; ++j) {
        const int t = first(j);
        if (t >= n_rows) continue;
        f32x4 acc[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[j][s][ks], qf[ks], acc[s], 0, 0, 0);
        }
        float x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = acc[k >> 2][k & 3] * p.scale_log2;
        if (t + kTile > n_rows) {
          DYNTS_OWN_BRANCH;
          const int rows = n_rows - t - 4 * kg;  // (against constants: eight slot numbers a tile are not kept over the loop)
#pragma unroll
          for (int k = 0; k < 8; ++k) x[k] = 16 * (k >> 2) + (k & 3) < rows ? x[k] : -INFINITY;
        }
        float mx = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
        if (last && p.spill && g < G) {
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const int tok = t + 16 * (k >> 2) + 4 * kg + (k & 3);
            if (tok < n_rows) p.spill[spill_at((size_t)unit, p.cap_pad, G, g, tok)] = x[k];
          }
        }
        mx = max_over_rows(mx);
        const float m_next = fmaxf(m_run, mx);
        const float m_new = m_next == -INFINITY ? 0.f : m_next;  // (-inf: no logit above it so far)
        const float corr = fast_exp2(m_run - m_new);
        if (j > 0 || (chunk == 0 && wave == 0)) {  // (else there is nothing to correct)
          DYNTS_OWN_BRANCH;
#pragma unroll
          for (int cb = 0; cb < CB; ++cb) oacc[cb] *= corr;
        }
        m_run = m_next;
        bf16x8 ph, pl;
        float psum = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const float pe = fast_exp2(x[k] - m_new);
          psum += pe;
          const __bf16 hi = (__bf16)pe;
          ph[k] = hi;
          pl[k] = (__bf16)(pe - (float)hi);
        }
        l_run = l_run * corr + psum;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          const bf16x8 v = __builtin_bit_cast(bf16x8, vt[j][cb]);
          oacc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, ph, oacc[cb], 0, 0, 0);
          oacc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, pl, oacc[cb], 0, 0, 0);
        }
      }
      l_run = sum_over_rows(l_run);
      if (kg == 0) sm_m[g][wave] = m_run;
    }
    __syncthreads();  // maxima; this step's inputs have been read
    if (!last) {
      stage(i + 1, next);
      fetch(i + 3, next);
    }
    const f32x4 ma = *reinterpret_cast<const f32x4 *>(&sm_m[g][0]), mb = *reinterpret_cast<const f32x4 *>(&sm_m[g][4]);
    const float mstar = fmaxf(fmaxf(fmaxf(ma[0], ma[1]), fmaxf(ma[2], ma[3])), fmaxf(fmaxf(mb[0], mb[1]), fmaxf(mb[2], mb[3])));
    if (here) {
      const float f = m_run == -INFINITY ? 0.f : fast_exp2(m_run - mstar);
      if (g < G) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) *reinterpret_cast<f32x4 *>(ored + (wave * 16 + g) * OSTRIDE + 16 * cb + 4 * kg) = oacc[cb] * f;
      }
      if (kg == 0) sm_l[g][wave] = l_run * f;
    }
    if (attended) {
      // ---- the new row, into the operands of the wave that has its slot ----------------------------------
      // (the others wait for this one: all its reads before the first is used, masks and no branches)
      if (tid == 0) sm_step[n_rows - n_entry] = i;
#pragma unroll
      for (int j = 0; j < T; ++j) {
        if ((n_rows & ~(kTile - 1)) != first(j)) continue;
        DYNTS_OWN_BRANCH;
        const int r = n_rows & (kTile - 1), dw_at = 2 * (r >> 4) + ((r & 3) >> 1);
        u32x4 k_row[KS];
        uint32_t v_row[CB];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) k_row[ks] = *reinterpret_cast<const u32x4 *>(in + 16 * STRIDE + 64 * ks + 16 * kg);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) v_row[cb] = *reinterpret_cast<const uint16_t *>(in + 17 * STRIDE + 2 * (16 * cb + r16));
        asm volatile("" ::: "memory");
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const bool mine = r16 == (r & 15) && s == r >> 4;
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) kf[j][s][ks] = mine ? __builtin_bit_cast(bf16x8, k_row[ks]) : kf[j][s][ks];
        }
        const uint32_t half = kg != ((r & 15) >> 2) ? 0u : (r & 1) ? 0xffff0000u : 0x0000ffffu;
        uint32_t put_at[4];
#pragma unroll
        for (int dw = 0; dw < 4; ++dw) put_at[dw] = dw == dw_at ? half : 0u;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          const uint32_t x = v_row[cb] | (v_row[cb] << 16);
          u32x4 v = __builtin_bit_cast(u32x4, vt[j][cb]);
#pragma unroll
          for (int dw = 0; dw < 4; ++dw) v[dw] = (v[dw] & ~put_at[dw]) | (x & put_at[dw]);
          vt[j][cb] = __builtin_bit_cast(i16x8, v);
        }
        if (lane == r) s_reg[j] = 0.f;
      }
    }
    __syncthreads();
    // (every read before the first sum, those of the outputs before the wait for the statistics)
    const f32x4 la = *reinterpret_cast<const f32x4 *>(&sm_l[g][0]), lb = *reinterpret_cast<const f32x4 *>(&sm_l[g][4]);
    const float lsum = ((((((la[0] + la[1]) + la[2]) + la[3]) + lb[0]) + lb[1]) + lb[2]) + lb[3];
    float o[NE];
#pragma unroll
    for (int k = 0; k < NE; ++k) {
      const int idx = tid + k * kResThreads, gg = idx / D;
      o[k] = 0.f;
      if (k == 0 || k * kResThreads < G * D) {
        float part[kResWaves];
#pragma unroll
        for (int w = 0; w < kResWaves; ++w) part[w] = ored[(w * 16 + gg) * OSTRIDE + idx % D];
        asm volatile("" ::: "memory");
#pragma unroll
        for (int w = 0; w < kResWaves; ++w) o[k] += part[w];
      }
    }
    if (!PART) {
      if (here && kg == 0) {
        stats.m[g] = mstar;
        stats.l[g] = lsum;
        stats.inv_l[g] = g < G ? 1.0f / lsum : 0.f;
      }
      wave_lds_fence();
    }
    // (a buffer that ends behind the group's heads, or is empty: no branch, so that a wait for a step's inputs is no wait for stores)
    const size_t part_row = (((size_t)i * p.units + unit) * p.chunks + chunk) * G;
    const RowBuffer out = __builtin_amdgcn_make_buffer_rsrc(PART ? p.part_o + part_row * D : out_rows + (size_t)i * p.out_stride, 0,
                                                            __builtin_amdgcn_readfirstlane(here ? G * D * 4 : 0), 0x00027000);
#pragma unroll
    for (int k = 0; k < NE; ++k) {
      const int idx = tid + k * kResThreads;
      if (!PART && (k == 0 || k * kResThreads < G * D)) o[k] /= stats.l[idx / D];
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o[k]), out, 4u * (uint32_t)idx, 0, 0);
    }
    if (PART) {
      const RowBuffer ml = __builtin_amdgcn_make_buffer_rsrc(p.part_ml + part_row * 2, 0, __builtin_amdgcn_readfirstlane(here ? G * 8 : 0), 0x00027000);
      const uint32_t off = wave == 0 && kg == 0 ? 8u * g : 1u << 30;  // (16 lanes; the others lie past the end)
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(mstar), ml, off, 0, 0);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(lsum), ml, off + 4u, 0, 0);
    } else if (here && p.track && !last) {
      const f32x4 m = *reinterpret_cast<const f32x4 *>(&stats.m[4 * kg]), inv_l = *reinterpret_cast<const f32x4 *>(&stats.inv_l[4 * kg]);
      bf16x8 qf[KS];
      load_q(qf, in);
#pragma unroll
      for (int j = 0; j < T; ++j) score_tile(j, qf, m, inv_l, n);
    }
    if (!PART) wave_lds_fence();  // the statistics are written again
  };
  for (int i = 0; i < most; i += 2) {     // (behind an odd number of steps one in which nothing happens: a branch around it
    step(std::false_type{}, i, piece_b);  // would have its inputs copied, and waited for, in every round)
    step(std::false_type{}, i + 1, piece_a);
  }
  step(std::true_type{}, most, piece_a);

  // ---- to memory: scores, new rows, positions, what the next deferred update needs, the sequence's words -----------
  // (PART: run_scores_kernel makes the run's updates and begins the new slots' scores)
  int at_end = FULL ? 64 * wave + lane : tid;  // (formed anew, so that nothing derived from it is kept over the loop)
  if (FULL) asm volatile("" : "+v"(at_end));
#pragma unroll
  for (int j = 0; j < T; ++j) {
    const int tok = first(j) + lane;
    if (lane < kTile && p.track && (PART ? p.owed && tok < n_entry && tok >= M : tok < n && (tok >= n_entry || tok >= M))) Sb[tok] = s_reg[j];
  }
  const int n_new = n - n_entry, pos0 = sm_hdr[2];
  const int lo = PART ? kResSlots * chunk - n_entry : 0, r_lo = lo > 0 ? lo : 0, r_hi = PART && lo + kResSlots < n_new ? lo + kResSlots : n_new;
  for (int i = at_end; i < 2 * (r_hi - r_lo) * PIECES; i += kResThreads) {
    const bool v = i >= (r_hi - r_lo) * PIECES;
    const int at = v ? i - (r_hi - r_lo) * PIECES : i, r = r_lo + at / PIECES, piece = 8 * (at % PIECES);
    const size_t from = (size_t)sm_step[r] * p.kv_stride + (size_t)unit * D + piece;
    store_u32x4((v ? Vb : Kb) + (size_t)(n_entry + r) * D + piece, load_u32x4((v ? p.v_new : p.k_new) + from));
  }
  for (int r = r_lo + at_end; r < r_hi; r += kResThreads) {
    p.pos[(size_t)unit * p.cap + n_entry + r] = pos0 + r;
    if (!p.track) Sb[n_entry + r] = p.s_new ? p.s_new[(size_t)sm_step[r] * p.Nb * p.Hkv + unit] : 0.f;
  }
  const bool owes = p.track && last_attended;
  if (!PART && owes) {  // (PART: merge_run_kernel)
    for (int i = at_end; i < G * PIECES; i += kResThreads)
      store_u32x4(p.qnext + row0 * D + 8 * (size_t)i, *reinterpret_cast<const u32x4 *>(sm_in + ((p.steps - 1) & 1) * IN + (i / PIECES) * STRIDE + 16 * (i % PIECES)));
    if (at_end < G) {
      p.mlprev[(row0 + at_end) * 2] = stats.m[at_end];
      p.mlprev[(row0 + at_end) * 2 + 1] = stats.l[at_end];
    }
  }
  if (n_dropped > 0 && h == 0 && chunk == 0 && at_end == 0) atomicOr(p.status, 1);
  if (PART) {
    if (h == 0 && chunk == 0 && at_end < 4) p.rec[4 * b + at_end] = at_end == 0 ? n_entry : at_end == 1 ? n : at_end == 2 ? pos0 + n_new : (int)last_attended;
    return;
  }
  if (at_end == 0 && (FULL ? (uint32_t)sm_hdr[4] : seq_ticket) == (uint32_t)p.Hkv - 1) {
    __hip_atomic_store(p.seq_cnt + (size_t)b * p.cnt_stride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (p.track) p.nprev[b] = owes ? n : 0;
    if (n_new > 0) {
      p.seq_len[b] = n;
      p.next_pos[b] = pos0 + n_new;
    }
  }
}

// ---- the partials of a run's steps, merged: outputs, statistics, what the next deferred update needs, the sequences' words ---------------------------
// grid (units, steps), 512 threads; the groups of chunks and the order of every sum are attend_kernel's.
template <int D>
__global__ __launch_bounds__(kResThreads) void merge_run_kernel(const ResidentParams p) {
  constexpr int NE = (16 * D + kResThreads - 1) / kResThreads, kMostChunks = kResThreads / 16;
  __shared__ __align__(16) float sm_w[16][kMostChunks];
  __shared__ float sm_old[16], sm_sum[16];
  const int unit = blockIdx.x, i = blockIdx.y, tid = threadIdx.x, G = p.G;
  const int b = __builtin_amdgcn_readfirstlane(unit / p.Hkv);
  if (i == 0 && unit == b * p.Hkv && tid == 0) {
    const int32_t *rec = p.rec + 4 * b;
    if (p.track) p.nprev[b] = rec[3] ? rec[1] : 0;
    if (rec[1] > rec[0]) {
      p.seq_len[b] = rec[1];
      p.next_pos[b] = rec[2];
    }
  }
  const int n_rows = p.n_of[(size_t)i * p.Nb + b];
  if (n_rows < 0) return;
  int chunks = (n_rows + kResSlots - 1) / kResSlots;
  chunks = chunks < 1 ? 1 : (chunks > p.chunks ? p.chunks : chunks);
  const size_t row = ((size_t)i * p.units + unit) * p.chunks;
  const float *po = p.part_o + row * G * D, *pml = p.part_ml + row * G * 2;
  const size_t orow0 = (size_t)unit * G;  // (= b * Hq + h * G)
  const bool last = i + 1 == p.steps;
  // the last step's query, a piece of 16 bytes a thread: kept with its statistics
  const bool keeps_q = last && p.track && tid < G * (D / 8);
  u32x4 q_piece = u32x4{0u, 0u, 0u, 0u};
  if (keeps_q) q_piece = load_u32x4(p.q + (size_t)i * p.q_stride + orow0 * D + 8 * (size_t)tid);
  auto merge = [&](auto N_) {
    constexpr int N = decltype(N_)::value;
    const int my_g = tid / N, my_j = tid % N;
    const bool asks = tid < 16 * N && my_g < G;
    float m_all = kLowest, l_all = 0.f, o_e[NE];  // (see attend_kernel)
#pragma unroll
    for (int k = 0; k < NE; ++k) o_e[k] = 0.f;
    for (int s0 = 0; s0 < chunks; s0 += N) {
      float part[NE][N];
#pragma unroll
      for (int k = 0; k < NE; ++k) {
        const int idx = tid + k * kResThreads;
#pragma unroll
        for (int j = 0; j < N; ++j) part[k][j] = idx < G * D && s0 + j < chunks ? po[(size_t)(s0 + j) * G * D + idx] : 0.f;
      }
      if (asks) {
        const int sj = s0 + my_j;
        const bool any = sj < chunks;
        const float mj = any ? pml[((size_t)sj * G + my_g) * 2] : -INFINITY;
        const float lj = any ? pml[((size_t)sj * G + my_g) * 2 + 1] : 0.f;
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
      for (int k = 0; k < NE; ++k) {
        const int idx = tid + k * kResThreads;
        if (idx < G * D) {
          const int gg = idx / D;
          float o = o_e[k] * sm_old[gg];
#pragma unroll
          for (int j = 0; j < N; ++j) o = fmaf(part[k][j], sm_w[gg][j], o);
          o_e[k] = o;
        }
      }
      __syncthreads();  // the weights' LDS is written again
    }
    if (tid < 16 * N && my_j == 0) {  // (of rows past the group's heads: no weight)
      float *st = p.stats + (((size_t)i * p.units + unit) * 16 + my_g) * 2;
      st[0] = asks ? m_all : 1e30f;
      st[1] = asks ? 1.0f / l_all : 0.f;
      if (asks && last && p.track) {
        p.mlprev[(orow0 + my_g) * 2] = m_all;
        p.mlprev[(orow0 + my_g) * 2 + 1] = l_all;
      }
    }
    if (keeps_q) store_u32x4(p.qnext + orow0 * D + 8 * (size_t)tid, q_piece);
    // Where every step's outputs go to one place, those of the last step that attended the sequence stay: the steps' workgroups have no
    // order.  (Looked up here: in front of the merge its loads wait behind it, 11.6 instead of 7.4 us for 64 steps of 18 chunks.)
    if (p.out_stride == 0)
      for (int s = i + 1; s < p.steps; ++s)
        if (p.n_of[(size_t)s * p.Nb + b] >= 0) return;
    float *out = p.out + (size_t)i * p.out_stride + orow0 * D;
#pragma unroll
    for (int k = 0; k < NE; ++k) {
      const int idx = tid + k * kResThreads;
      if (idx < G * D) out[idx] = o_e[k] / sm_sum[idx / D];
    }
  };
  const int ne = (G * D + kResThreads - 1) / kResThreads;
  if (p.wide && ne == 1 && chunks > kWideFrom1) merge(std::integral_constant<int, 32>{});
  else if (p.wide && D == 128 && ne == 2 && chunks > kWideFrom2) merge(std::integral_constant<int, 8>{});
  else merge(std::integral_constant<int, 4>{});
}

// ---- the score updates of a run's steps but the last (whose is owed), from the cache as the run left it -----------------
// grid units * chunks, 512 threads: a wave its tile of K.  Queries and statistics reach the waves through LDS, eight steps at a time: fetched by
// every wave for itself, in operand order, they alone took 0.6 us a step.
template <int D>
__global__ __launch_bounds__(kResThreads) void run_scores_kernel(const ResidentParams p) {
  constexpr int KS = D / 32, PIECES = D / 8, VROWS = 64 / PIECES, VIT = kTile / VROWS, STRIDE = 2 * D + 32;
  constexpr int kSteps = 8, kBuf = kSteps * 16 * STRIDE;  // steps at a time
  constexpr int NP = (16 * PIECES * kSteps + kResThreads - 1) / kResThreads;
  static_assert(kResWaves * kTile * STRIDE == 2 * kBuf && kPartSteps <= 64, "the tiles' LDS is reused for the queries; a lane per step");
  __shared__ __align__(16) unsigned char smem[kResWaves * kTile * STRIDE];
  __shared__ __align__(16) float sm_stats[2][kSteps * 32];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kg = lane >> 4, g = r16, G = p.G;
  const int unit = __builtin_amdgcn_readfirstlane(blockIdx.x / p.chunks), chunk = blockIdx.x - unit * p.chunks;
  const int b = __builtin_amdgcn_readfirstlane(unit / p.Hkv);
  const int n_entry = p.rec[4 * b], n = p.rec[4 * b + 1], M = p.n_prompt[b];
  if (kResSlots * chunk >= n) return;
  const int t = kResSlots * chunk + kTile * wave, tok = t + lane;
  float *Sb = p.S + (size_t)unit * p.cap;
  float s = lane < kTile && tok < n_entry ? Sb[tok] : 0.f;
  // (lane i: slots of step i; -1: nothing to add)
  const int n_lane = lane + 1 < p.steps ? p.n_of[(size_t)lane * p.Nb + b] : -1;
  bf16x8 kf[2][KS];
  {
    u32x4 kr[VIT];
    load_tile<D>(kr, row_buffer<D>(p.K + (size_t)unit * p.cap * D, n), t, lane);
    unsigned char *vst = smem + wave * kTile * STRIDE;
#pragma unroll
    for (int it = 0; it < VIT; ++it)
      *reinterpret_cast<u32x4 *>(vst + (VROWS * it + lane / PIECES) * STRIDE + 16 * (lane % PIECES)) = kr[it];
    wave_lds_fence();
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kf[x][ks] = *reinterpret_cast<const bf16x8 *>(vst + (16 * x + r16) * STRIDE + 64 * ks + 16 * kg);
  }
  __syncthreads();
  for (int i = tid; i < 2 * kSteps * (16 - G) * PIECES; i += kResThreads) {  // (rows past the group's heads)
    const int row = i / PIECES, in_step = row % (16 - G);
    *reinterpret_cast<u32x4 *>(smem + (row / (16 - G) * 16 + G + in_step) * STRIDE + 16 * (i % PIECES)) = u32x4{0u, 0u, 0u, 0u};
  }
  // eight steps' queries and statistics, a piece of 16 bytes a thread
  u32x4 piece[NP];
  float stat = 0.f;
  const uint16_t *qb = p.q + (size_t)unit * G * D;
  auto fetch = [&](int i0) {
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int at = tid + k * kResThreads, st = at / (G * PIECES), i = i0 + st;
      if (st < kSteps && i < p.steps) piece[k] = load_u32x4(qb + (size_t)i * p.q_stride + 8 * (at - st * (G * PIECES)));
    }
    if (tid < kSteps * 32 && i0 + tid / 32 < p.steps) stat = p.stats[((size_t)(i0 + tid / 32) * p.units + unit) * 32 + tid % 32];
  };
  fetch(0);
  for (int i0 = 0; i0 < p.steps - 1; i0 += kSteps) {
    const int buf = (i0 / kSteps) & 1;
    unsigned char *qs = smem + buf * kBuf;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int at = tid + k * kResThreads, st = at / (G * PIECES), in_step = at - st * (G * PIECES);
      if (st < kSteps) *reinterpret_cast<u32x4 *>(qs + (16 * st + in_step / PIECES) * STRIDE + 16 * (in_step % PIECES)) = piece[k];
    }
    if (tid < kSteps * 32) sm_stats[buf][tid] = stat;
    __syncthreads();
    fetch(i0 + kSteps);
    if (t >= n) continue;
    // Two steps side by side, whose chains of products, exponentials and sums then hide one another's latencies; added one after the other.
#pragma unroll 2
    for (int at = 0; at < kSteps; at += 2) {
      f32x4 e[2][2];
      float part[2][2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
#pragma unroll
        for (int x = 0; x < 2; ++x) e[j][x] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const bf16x8 qf = *reinterpret_cast<const bf16x8 *>(qs + (16 * (at + j) + g) * STRIDE + 64 * ks + 16 * kg);
#pragma unroll
          for (int x = 0; x < 2; ++x) e[j][x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qf, kf[x][ks], e[j][x], 0, 0, 0);
        }
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const f32x4 *st = reinterpret_cast<const f32x4 *>(&sm_stats[buf][32 * (at + j) + 8 * kg]);  // of heads 4 kg .. 4 kg + 3
        const f32x4 a = st[0], c = st[1], m = {a[0], a[2], c[0], c[2]}, inv_l = {a[1], a[3], c[1], c[3]};
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          float sum = 0.f;
#pragma unroll
          for (int k = 0; k < 4; ++k) sum += fast_exp2(e[j][x][k] * p.scale_log2 - m[k]) * inv_l[k];
          part[j][x] = sum;
        }
      }
      if (G > 8) {
#pragma unroll
        for (int j = 0; j < 4; ++j) part[j >> 1][j & 1] = sum_over_rows(part[j >> 1][j & 1]);
      } else if (G > 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const Pair r = over_16(part[j >> 1][j & 1]);
          part[j >> 1][j & 1] = r.low + r.high;
        }
      } else {
#pragma unroll
        for (int j = 0; j < 2; ++j) part[j][1] = over_16(part[j][1]).low;
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int i = i0 + at + j, n_rows = __builtin_amdgcn_readlane(n_lane, i < 64 ? i : 63);
        const float add = kg == 0 ? part[j][0] : part[j][1];
        if (tok <= n_rows && tok >= M) s += add;  // (the new slot too)
      }
    }
  }
  if (lane < kTile && tok < n && (tok >= n_entry || tok >= M)) Sb[tok] = s;
}

}  // namespace dynts
