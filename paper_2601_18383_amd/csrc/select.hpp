// Top-k selection inside the selection window (Sec. 4.2) for gfx950: one workgroup per
// (sequence, KV head).  A radix select over order-preserving integer keys, 8 bits a pass, finds the
// k-th largest score exactly; ties at the cut go to the lowest slots (= lowest positions,
// slots are kept in position order); counts of ballots turn the keep flags into the ascending
// list of retained slots.
//
// With APPLY the workgroup first makes the score update the trigger still owes, from the step's kept logits: the scores then pass
// from the update to the selection in the same launch.
//
// What bounds it: a chain of dependent steps on few workgroups.  So everything that can be asked for before the sequence's
// length is known leaves at once (with 1024 threads the first 4096 scores and logits of the unit); up to 16 waves share the passes
// (fewer where units outnumber the compute units: select_threads in dynts.hip); a pass
// counts into eight copies of its histogram (scores of one trigger share their leading bits: in one copy all 64 lanes of a wave wait for the
// same word), adds the copies up, and every wave finds the cut's bin for itself; and it ends as soon as the whole bin is kept.
// 128 units of 2496 slots, 7 heads a group: 9.6 us with the update, where 256 threads took 13.2 us behind 5.7 us of update.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attend.hpp"

namespace dynts {

constexpr int kSelCopies = 8, kSelPitch = 256 + 1;  // copies of the histogram, words from one to the next (+1: other banks)
constexpr int kSelHeads = 8;    // heads of a group whose kept logits a workgroup takes (APPLY)
constexpr int kSelEarly = 4;    // rounds of kSelThreads slots that are asked for before the length is known
constexpr int kSelCounts = 256;  // counts of flags, one per wave and round of candidates, that are added up together

struct SelectParams {
  float *S;                 // [Nb][Hkv][cap]
  const int32_t *seq_len;   // [Nb]
  const int32_t *n_prompt;  // [Nb]
  const uint8_t *trigger;   // [Nb] or null
  int32_t *keep_idx;        // [Nb][Hkv][keep_stride]
  int32_t *new_len;         // [Nb]
  int32_t *status;          // bit 1 latched when keep_stride is too small for a sequence
  int Hkv, cap, window, k_keep, keep_stride;
  // APPLY: kept logits (see spill_at), statistics [Nb][Hq][2] and slots of the step they belong to
  const float *spill, *mlprev;
  const int32_t *nprev;     // [Nb]
  int G, cap_pad;
};

// fp32 -> uint32 whose unsigned order is the IEEE order; -0 and +0 map to the same key
__device__ __forceinline__ uint32_t score_key(float s) {
  uint32_t u = __float_as_uint(s);
  if ((u << 1) == 0u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// inclusive prefix sum over the wave's lanes
__device__ __forceinline__ int wave_inclusive_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // from 1, 2, 4, 8 lanes below in the row of 16
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // rows 1 and 3: the last lane of the row before
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // rows 2 and 3: lane 31
  return x;
}

template <int kSelThreads, bool USE_LDS, bool APPLY>
__global__ __launch_bounds__(kSelThreads) void select_kernel(const SelectParams p) {
  static_assert(USE_LDS || !APPLY, "the updated scores are handed on through LDS");
  constexpr int kSelWaves = kSelThreads / 64, kSelRounds = kSelCounts / kSelWaves;
  static_assert(kSelThreads >= 256 && kSelWaves % 4 == 0 && kSelCounts % kSelWaves == 0, "a thread per bin; four waves' counts a lane");
  extern __shared__ uint32_t keys[];  // candidate keys when USE_LDS
  __shared__ uint32_t hist[kSelCopies * kSelPitch];
  __shared__ __align__(16) uint32_t total[256];
  __shared__ __align__(16) int cnt_gt[kSelCounts], cnt_eq[kSelCounts];  // per round and wave
  __shared__ float sm_m[kSelHeads], sm_inv[kSelHeads];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.x, b = blockIdx.y;
  const size_t unit = (size_t)b * p.Hkv + h;
  float *Su = p.S + unit * (size_t)p.cap;
  const int G = p.G;

  // ---- whatever does not hang on the length ----------------------------------------------
  float s_early[kSelEarly], x_early[APPLY ? kSelEarly : 1][kSelHeads];
  if (USE_LDS) {
#pragma unroll
    for (int c = 0; c < kSelEarly; ++c) {
      const int j = c * kSelThreads + tid;
      s_early[c] = j < p.cap ? Su[j] : 0.f;
    }
  }
  float m_l = 0.f, l_l = 1.f;
  if (APPLY) {
    if (tid < G) {
      const float *ml = p.mlprev + (unit * G + tid) * 2;
      m_l = ml[0];
      l_l = ml[1];
    }
#pragma unroll
    for (int c = 0; c < kSelEarly; ++c) {
      const int j = c * kSelThreads + tid;
#pragma unroll
      for (int g = 0; g < kSelHeads; ++g) x_early[c][g] = g < G && j < p.cap ? p.spill[spill_at(unit, p.cap_pad, G, g, j)] : 0.f;
    }
  }
  for (int i = tid; i < kSelCopies * kSelPitch; i += kSelThreads) hist[i] = 0;
  if (tid < kSelCounts) cnt_gt[tid] = cnt_eq[tid] = 0;

  int n = p.seq_len[b];
  n = n < 0 ? 0 : (n > p.cap ? p.cap : n);
  int M = p.n_prompt[b];
  const int M_raw = M;
  M = M < 0 ? 0 : (M > n ? n : M);
  const int lo = M;
  const int hi = (n - p.window > lo) ? n - p.window : lo;
  const int nc = hi - lo;
  const int kk = nc < p.k_keep ? nc : p.k_keep;
  const int out_len = M + kk + (n - hi);
  const bool triggered = !p.trigger || p.trigger[b];
  const bool listed = triggered && out_len <= p.keep_stride;  // else the retained slots cannot be listed: the sequence stays
  const bool choose = listed && kk > 0 && kk < nc;

  // ---- the owed update, S[slot] += sum over the group of 2^(logit - max) / sum, and the candidates' keys ------
  if (USE_LDS) {
    int n_prev = 0;
    if (APPLY) {
      n_prev = p.nprev[b];
      n_prev = n_prev < p.cap ? n_prev : p.cap;
      if (tid < G) {
        sm_m[tid] = m_l;
        sm_inv[tid] = 1.0f / l_l;
      }
      __syncthreads();
    }
    const int end = choose ? (hi > n_prev ? hi : n_prev) : n_prev;
    auto settle = [&](int j, float s, const float *early) {
      if (APPLY && j < n_prev && j >= M_raw) {
        float add = 0.f;
#pragma unroll
        for (int g = 0; g < kSelHeads; ++g)
          if (g < G) add = fmaf(fast_exp2((early ? early[g] : p.spill[spill_at(unit, p.cap_pad, G, g, j)]) - sm_m[g]), sm_inv[g], add);
        s += add;
        Su[j] = s;
      }
      if (j >= lo && j < hi && choose) keys[j - lo] = score_key(s);
    };
#pragma unroll
    for (int c = 0; c < kSelEarly; ++c)
      if (c * kSelThreads + tid < end) settle(c * kSelThreads + tid, s_early[c], x_early[APPLY ? c : 0]);
    for (int j = kSelEarly * kSelThreads + tid; j < end; j += kSelThreads) settle(j, Su[j], nullptr);
  }

  if (h == 0 && tid == 0) {
    p.new_len[b] = listed ? out_len : n;
    if (triggered && !listed) atomicOr(p.status, 2);
  }
  if (!listed) return;
  int32_t *ku = p.keep_idx + unit * (size_t)p.keep_stride;
  for (int i = tid; i < M; i += kSelThreads) ku[i] = i;
  for (int i = tid; i < n - hi; i += kSelThreads) ku[M + kk + i] = hi + i;
  if (kk == 0) return;
  if (kk == nc) {
    for (int i = tid; i < nc; i += kSelThreads) ku[M + i] = lo + i;
    return;
  }
  auto key = [&](int j) -> uint32_t { return USE_LDS ? keys[j] : score_key(Su[lo + j]); };
  __syncthreads();  // keys, histogram and counts are there

  // ---- radix select: the kk-th largest key, 8 bits per pass from the top ---------------
  uint32_t prefix = 0;
  int remaining = kk;
  uint32_t *const own_hist = hist + (tid & (kSelCopies - 1)) * kSelPitch;
#pragma unroll 1
  for (int shift = 24; shift >= 0; shift -= 8) {
    const uint32_t himask = shift == 24 ? 0u : (0xFFFFFFFFu << (shift + 8));
    for (int j = tid; j < nc; j += kSelThreads) {
      const uint32_t u = key(j);
      if ((u & himask) == prefix) atomicAdd(&own_hist[(u >> shift) & 255u], 1u);
    }
    __syncthreads();
    constexpr int PER = kSelThreads >= 512 ? 2 : 1;  // threads a bin, which share its copies
    if (tid < 256 * PER) {                 // (zeroed for the next pass)
      uint32_t c = 0;
      uint32_t *src = hist + (tid % PER) * (kSelCopies / PER) * kSelPitch + tid / PER;
#pragma unroll
      for (int k = 0; k < kSelCopies / PER; ++k) {
        c += src[k * kSelPitch];
        src[k * kSelPitch] = 0;
      }
      if (PER == 2) c += __shfl_xor(c, 1);
      if (tid % PER == 0) total[tid / PER] = c;
    }
    __syncthreads();
    // lane L holds bins 255-4L .. 252-4L, walked from the top
    const u32x4 t4 = *reinterpret_cast<const u32x4 *>(&total[252 - 4 * lane]);
    const int c0 = t4[3], c1 = t4[2], c2 = t4[1], c3 = t4[0];
    const int incl = wave_inclusive_scan(c0 + c1 + c2 + c3), excl = incl - (c0 + c1 + c2 + c3);
    const int r = remaining - excl;
    const int step = r <= c0 ? 0 : r <= c0 + c1 ? 1 : r <= c0 + c1 + c2 ? 2 : 3;
    const int above = excl + (step > 0 ? c0 : 0) + (step > 1 ? c1 : 0) + (step > 2 ? c2 : 0);
    const int in_bin = step == 0 ? c0 : step == 1 ? c1 : step == 2 ? c2 : c3;
    const int cut = __builtin_ctzll(__ballot(excl < remaining && remaining <= incl));  // (exactly one lane)
    const uint32_t bin = 255u - 4u * (uint32_t)cut - (uint32_t)__builtin_amdgcn_readlane(step, cut);
    prefix |= bin << shift;
    remaining -= __builtin_amdgcn_readlane(above, cut);
    if (remaining == __builtin_amdgcn_readlane(in_bin, cut)) {  // the whole bin is kept
      remaining = 0;
      prefix -= 1;  // (some candidate is not kept, so a key below the bin exists)
      break;
    }
  }
  const uint32_t T = prefix;      // kept: keys above T,
  const int take_eq = remaining;  // and of the slots with that key so many, lowest slots first

  // ---- flags -> ascending output: candidate j = round * kSelThreads + tid, kSelRounds rounds at a time -----
  int base_gt = 0, base_eq = 0;
  const uint64_t below = ((uint64_t)1 << lane) - 1;
  for (int j_first = 0; j_first < nc; j_first += kSelRounds * kSelThreads) {
    const int left = nc - j_first, rounds = (left + kSelThreads - 1) / kSelThreads < kSelRounds ? (left + kSelThreads - 1) / kSelThreads : kSelRounds;
    if (j_first > 0) {  // (the counts of the rounds before have been read)
      __syncthreads();
      if (tid < kSelCounts) cnt_gt[tid] = cnt_eq[tid] = 0;
      __syncthreads();
    }
    for (int c = 0; c < rounds; ++c) {
      const int j = j_first + c * kSelThreads + tid;
      const uint32_t u = j < nc ? key(j) : 0u;
      const uint64_t gt = __ballot(j < nc && u > T), eq = __ballot(j < nc && u == T);
      if (lane == 0) {
        cnt_gt[c * kSelWaves + wave] = __popcll(gt);
        cnt_eq[c * kSelWaves + wave] = __popcll(eq);
      }
    }
    __syncthreads();
    // lane L: counts 4 L .. 4 L + 3, of four waves of one round
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    const i32x4 g4 = *reinterpret_cast<const i32x4 *>(&cnt_gt[4 * lane]), e4 = *reinterpret_cast<const i32x4 *>(&cnt_eq[4 * lane]);
    const int g_in = wave_inclusive_scan(g4[0] + g4[1] + g4[2] + g4[3]), e_in = wave_inclusive_scan(e4[0] + e4[1] + e4[2] + e4[3]);
    const int sub = wave & 3;
    const int g_at = g_in - g4[3] - (sub < 3 ? g4[2] : 0) - (sub < 2 ? g4[1] : 0) - (sub < 1 ? g4[0] : 0);
    const int e_at = e_in - e4[3] - (sub < 3 ? e4[2] : 0) - (sub < 2 ? e4[1] : 0) - (sub < 1 ? e4[0] : 0);
    for (int c = 0; c < rounds; ++c) {
      const int j = j_first + c * kSelThreads + tid;
      const uint32_t u = j < nc ? key(j) : 0u;
      const bool is_gt = j < nc && u > T, is_eq = j < nc && u == T;
      const int at = (c * kSelWaves + wave) >> 2;
      const int gt_before = base_gt + __builtin_amdgcn_readlane(g_at, at) + __popcll(__ballot(is_gt) & below);
      const int eq_before = base_eq + __builtin_amdgcn_readlane(e_at, at) + __popcll(__ballot(is_eq) & below);
      const int off = gt_before + (eq_before < take_eq ? eq_before : take_eq);
      if ((is_gt || (is_eq && eq_before < take_eq)) && off < kk) ku[M + off] = lo + j;  // (off < kk always)
    }
    base_gt += __builtin_amdgcn_readlane(g_in, 63);
    base_eq += __builtin_amdgcn_readlane(e_in, 63);
  }
}

}  // namespace dynts
