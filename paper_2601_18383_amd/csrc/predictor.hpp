// Importance Predictor head (Sec. 4.1; App. A "Predictor Overhead"; App. C: 3584->7168->1792->1 and
// 4096->8192->2048->1): a three-layer MLP on the final hidden state of the current token of every
// sequence, s = w3 . act(W2 act(W1 h + b1) + b2) + b3, one score per token.  At decode batch sizes
// this is a skinny GEMM whose cost is reading the weights once (3 d^2 bf16 values, ~100 MB): HBM-bound.
//
// Two launches, one per hidden layer, of one kernel: a workgroup takes FT tiles of 16 features and its eight waves share out
// K between them, each with an accumulator for all features and sequences; the waves' sums are added through LDS.
//   * Layer 1 takes a workgroup's whole K, so that nothing has to be added across workgroups: it applies bias and activation
//     and writes the second layer's operand as bf16 hi + lo parts (two MFMAs per weight fragment there: nothing is rounded
//     to bf16 between the layers).
//   * Layer 2 has four times fewer features, so ns workgroups share the K of a group of features.  Their sums travel as tagged
//     words (see attend.hpp) and the workgroup that draws the group's last ticket adds them in index order, applies bias and
//     activation and forms the group's part of the dot product with w3; the one that draws the last ticket of all adds
//     those.  The words are zeroed by the first kernel, so that a tag is this call's whatever lay in the scratch.
//   * Weights are the MFMA A operand, loaded straight into operand registers.
//   * What a compute unit can take in counts as much as the memory: 140 B/ns where consecutive lanes read consecutive 16 bytes,
//     75 where a lane's 16 bytes lie 64 apart (packed weights), 38 where they lie in 16 rows (operand order of a row-major
//     matrix).  So layer 1 reads the hidden states 8 rows x 128 bytes at a time and turns them into operands through LDS of the
//     wave's own, and writes its output in the order in which layer 2's lanes read it.
//   * Offsets are 32 bits wide; sizes past them, and layers that leave the chip idle so (mlp_split in dynts.hip), take the form that
//     cuts K of both layers (mlp_split_gemm_kernel).
//   * k-steps are dealt out to the waves in turn: with contiguous shares, a power of two apart, all of them met on the same memory
//     channels (d = 4096, batch 32: 31.3 -> 27.7 us).
// us a call on the same weights again and again (77 MB, which the memory-side cache holds; 11.5 us at the rate of a plain read
// stream), d = 3584, with partial sums of both layers reduced by kernels of
// their own / so: batch 1 27.9 / 21.7, batch 32 30.0 / 24.5, batch 64 37.1 / 28.8, batch 128 65.3 / 39.0; d = 1024: 20.7 / 11.6,
// 20.8 / 12.7, -, 27.1 / 17.8.  Weights that come from HBM, eight heads in turn: d = 3584, batch 32 28.4 instead of 24.3, 128 49.2 instead of 39.2.  Of the 24.5, by timestamps and so to within a
// microsecond: layer 1 11.3, gap 1.3, layer 2's loop 9, two hand-offs with what lies between 3.4.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attend.hpp"

namespace dynts {

constexpr int kMlpWaves = 8;
constexpr int kMlpThreads = kMlpWaves * 64;

struct MlpParams {
  const uint16_t *W;    // [m][K] bf16, row-major or packed (mlp_pack_kernel)
  const uint16_t *x;    // layer 1: [Nb][K] bf16; layer 2: what layer 1 wrote (y)
  const float *bias;    // [m] or null
  int Nb, m, K, act;
  // layer 1
  uint16_t *y;          // [m/32][BT][2][4][16][8]: the second layer's B operands, hi and lo parts, 16 bytes per lane
  uint32_t *clear;      // the second layer's tagged words and counters, zeroed here
  uint32_t n_clear;     // in 16-byte pieces
  // layer 2
  const uint16_t *w3;   // [m]
  const float *b3;      // [1] or null
  int ns;               // workgroups that share the K of a group of features
  uint64_t *part_sum;   // [groups][ns][16 FT * 16 BT]: tagged partial sums
  uint64_t *part_dot;   // [groups][Nb]: tagged parts of the final dot product
  uint32_t *group_cnt;  // [groups][kMlpCntStride] tickets of the workgroups that share a group
  uint32_t *done_cnt;   // tickets of the groups
  float *s_out;         // [Nb][n_rep]
  int n_rep;
};

__device__ __forceinline__ float mlp_act(float x, int act) {
  if (act == 1) return x > 0.f ? x : 0.f;
  if (act == 2) return x / (1.f + __expf(-x));
  return x;
}

// round-to-nearest-even bf16 of a finite float
__device__ __forceinline__ uint16_t f32_to_bf16(float x) {
  uint32_t u = __float_as_uint(x);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf16_to_f32(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }

constexpr int kMlpCntStride = 64;  // counters lie 256 bytes apart (see attend.hpp)
constexpr uint32_t kMlpTag = 1;  // of a word written by this call's second kernel (the first zeroed it)

// What a wave keeps in flight: k-steps (32 elements of K) of weights, and of activations (layer 1: pairs of k-steps)
constexpr int mlp_w_depth(int bt) { return bt > 4 ? 2 : bt > 2 ? 4 : 8; }
constexpr int mlp_x_depth(int bt, bool second) {
  return second ? (bt > 4 ? 1 : bt > 2 ? 2 : bt == 2 ? 4 : 8) : (bt > 4 ? 1 : bt > 1 ? 2 : 4);
}

// 16 bytes of a buffer whose size is part of its descriptor: what lies past the end reads as zero and fetches nothing, so that
// the last steps' prefetches need no branch, which would make every wait behind it a wait for all loads.
using MlpBuffer = __amdgpu_buffer_rsrc_t;
__device__ __forceinline__ MlpBuffer mlp_buffer(const void *base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, 0x00027000);
}
__device__ __forceinline__ u32x4 mlp_load(MlpBuffer buf, uint32_t off) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(buf, off, 0, 0));
}
constexpr uint32_t kMlpNowhere = 0x80000000u;  // an offset past the end of every buffer

template <int FT, int BT, bool SECOND, bool PACKED>
__global__ __launch_bounds__(kMlpThreads, 2) void mlp_kernel(const MlpParams p) {
  constexpr int PARTS = SECOND ? 2 : 1;
  constexpr int DW = mlp_w_depth(BT), DX = mlp_x_depth(BT, SECOND);
  constexpr int NT = FT * BT;            // output tiles of 16 x 16
  constexpr int XROW = 128 + 16;         // LDS pitch of a sequence's 64 activations, bytes
  constexpr int XBYTES = SECOND ? 0 : 16 * BT * XROW, RBYTES = NT * 1024;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kMlpWaves * (XBYTES > RBYTES ? XBYTES : RBYTES)];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kg = lane >> 4;
  const int ns = SECOND ? p.ns : 1;
  // (uniform values that a division would leave in vector registers, and every address formed from them)
  const int group = SECOND ? __builtin_amdgcn_readfirstlane(blockIdx.x / ns) : blockIdx.x, split = blockIdx.x - group * ns;
  const int tile0 = group * FT, n_tiles = p.m / 16, n_all = p.K / 32;

  // This workgroup's k-steps [k0, k1), dealt out to its waves in turn (layer 1: by pairs, so that a row's piece is a whole
  // 128-byte line): what the workgroup asks for at a time is contiguous, and no two waves are a power of two apart.
  constexpr int UNIT = SECOND ? 1 : 2;
  const uint32_t n_units = (uint32_t)(n_all + UNIT - 1) / UNIT;
  const int u0 = __builtin_amdgcn_readfirstlane(n_units * (uint32_t)split / (uint32_t)ns);
  const int u1 = __builtin_amdgcn_readfirstlane(n_units * (uint32_t)(split + 1) / (uint32_t)ns);
  const int k0 = u0 * UNIT, k1 = u1 * UNIT < n_all ? u1 * UNIT : n_all;
  const int n = (u1 - u0 - wave + kMlpWaves - 1) / kMlpWaves * UNIT;  // (not positive: none)
  auto rel = [&](int st) { return (uint32_t)(SECOND ? wave + kMlpWaves * st : 2 * (wave + kMlpWaves * (st >> 1)) + (st & 1)); };

  // weights: this workgroup's share of each of its feature tiles
  MlpBuffer wbuf[FT];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft) {
    int tile = tile0 + ft;
    tile = tile < n_tiles ? tile : n_tiles - 1;  // (repeats the last; not written)
    const char *base = reinterpret_cast<const char *>(p.W);
    wbuf[ft] = PACKED ? mlp_buffer(base + ((size_t)tile * n_all + k0) * 1024, (uint32_t)(k1 - k0) * 1024u)
                      : mlp_buffer(base + (size_t)tile * 32 * p.K, (uint32_t)p.K * 32u);
  }
  const uint32_t w_off = PACKED ? 64u * r16 + 16u * kg : (uint32_t)r16 * (uint32_t)(2 * p.K) + (uint32_t)k0 * 64u + 16u * kg;
  bf16x8 wf[DW][FT];
  auto load_w = [&](int slot, int st) {
    const uint32_t off = PACKED ? w_off + rel(st) * 1024u : (int)rel(st) < k1 - k0 ? w_off + rel(st) * 64u : kMlpNowhere;
#pragma unroll
    for (int ft = 0; ft < FT; ++ft) wf[slot][ft] = __builtin_bit_cast(bf16x8, mlp_load(wbuf[ft], off));
  };
#pragma unroll
  for (int j = 0; j < DW; ++j) load_w(j, j);
  // What the end of the kernel needs is asked for here, too: a first read of it there would cost a trip to memory.
  // Element e of a thread's share of the sums: layer 1 takes f32x4 pieces, layer 2 single values.
  constexpr int NE = SECOND ? (NT * 256 + kMlpThreads - 1) / kMlpThreads : (NT * 64 + kMlpThreads - 1) / kMlpThreads;
  auto feature = [&](int j) {  // first feature of element j
    const int e = tid + j * kMlpThreads;
    return SECOND ? 16 * (tile0 + (e >> 8) / BT) + 4 * ((e & 255) >> 6) + (e & 3) : 16 * (tile0 + (e >> 6) / BT) + 4 * ((e & 63) >> 4);
  };
  constexpr int ALL = NT * (SECOND ? 256 : 64);
  auto in = [&](int j) { return ALL % kMlpThreads == 0 || tid + j * kMlpThreads < ALL; };
  auto has = [&](int j) { return in(j) && feature(j) < p.m; };
  // (of a thread's elements BSTEP in a row share a feature: in layer 2 their sequences differ)
  constexpr int NB = !SECOND ? NE : FT == 1 ? 1 : BT % 2 == 0 ? 2 : NE, BSTEP = NE / NB;
  f32x4 bias[NB];
  float w3[NB], b3 = 0.f;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    bias[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    w3[i] = 0.f;
    if (has(i * BSTEP)) {
      const int f = feature(i * BSTEP);
      if (p.bias) {
#pragma unroll
        for (int k = 0; k < (SECOND ? 1 : 4); ++k) bias[i][k] = p.bias[f + k];
      }
      if (SECOND) w3[i] = bf16_to_f32(p.w3[f]);
    }
  }
  if (SECOND && p.b3) b3 = p.b3[0];

  f32x4 acc[FT][BT];
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int bt = 0; bt < BT; ++bt) acc[ft][bt] = f32x4{0.f, 0.f, 0.f, 0.f};

  if constexpr (SECOND) {
    const MlpBuffer xbuf = mlp_buffer(reinterpret_cast<const char *>(p.x) + (size_t)k0 * (BT * 2048), (uint32_t)(k1 - k0) * (BT * 2048u));
    bf16x8 xf[DX][BT][PARTS];
    auto load_x = [&](int slot, int bt, int st) {
      const uint32_t off = rel(st) * (BT * 2048u) + 16u * lane;
#pragma unroll
      for (int part = 0; part < PARTS; ++part)
        xf[slot][bt][part] = __builtin_bit_cast(bf16x8, mlp_load(xbuf, off + (bt * PARTS + part) * 1024));
    };
#pragma unroll
    for (int j = 0; j < DX; ++j)
#pragma unroll
      for (int bt = 0; bt < BT; ++bt) load_x(j, bt, j);
    auto round = [&](int sb) {
#pragma unroll
      for (int j = 0; j < DW; ++j) {
        // (a tile's next activations are asked for as soon as its products have been issued; past the last step both
        // operands are zero)
#pragma unroll
        for (int bt = 0; bt < BT; ++bt) {
#pragma unroll
          for (int part = 0; part < PARTS; ++part)
#pragma unroll
            for (int ft = 0; ft < FT; ++ft)
              acc[ft][bt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[j][ft], xf[j % DX][bt][part], acc[ft][bt], 0, 0, 0);
          load_x(j % DX, bt, sb + j + DX);
          __builtin_amdgcn_sched_barrier(0);
        }
        load_w(j, sb + j + DW);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // (The first round by itself: a wait counts loads in the order in which either path to it issued them, and the ones above come in
    // another order than a round's own; a loop entered with them would wait for weights it has just asked for.  us a call, so before / now, other
    // weights each call: from the memory-side cache d = 2048, 16 sequences 13.9 / 13.5, 128 24.7 / 23.9; from HBM d = 3584, 32 27.9 / 27.5, 128 48.9 / 47.8,
    // d = 4096, 32 31.4 / 31.2.  Asked for in a round's order instead, weights behind the biases, the cached ones take 12.9 and 24.6, but those from HBM
    // 28.8, 48.6 and 32.6: there every moment counts by which the first weights leave earlier.)
    round(0);
    for (int sb = DW; sb < n; sb += DW) round(sb);
  } else {
    // A load covers 8 sequences x 128 bytes, which a wave turns into operands through LDS of its own
    unsigned char *xs = smem + wave * XBYTES;
    const MlpBuffer xbuf = mlp_buffer(p.x, (uint32_t)p.Nb * (uint32_t)(2 * p.K));
    const uint32_t col0 = (uint32_t)k0 * 64 + 16u * (lane & 7), col_end = (uint32_t)k1 * 64;
    uint32_t x_row[2 * BT];
#pragma unroll
    for (int i = 0; i < 2 * BT; ++i) {
      int row = 8 * i + (lane >> 3);
      row = row < p.Nb ? row : p.Nb - 1;
      x_row[i] = (uint32_t)row * (uint32_t)(2 * p.K);
    }
    u32x4 raw[DX][2 * BT];
    auto load_x = [&](int slot, int pr) {  // pair pr of this wave
      uint32_t col = col0 + rel(2 * pr) * 64;
      col = col < col_end ? col : kMlpNowhere;
#pragma unroll
      for (int i = 0; i < 2 * BT; ++i) raw[slot][i] = mlp_load(xbuf, x_row[i] + col);
    };
#pragma unroll
    for (int j = 0; j < DX; ++j) load_x(j, j);
    // the second layer's words, zeroed while the first loads are on their way
    for (uint32_t i = blockIdx.x * kMlpThreads + tid; i < p.n_clear; i += gridDim.x * kMlpThreads)
      reinterpret_cast<u32x4 *>(p.clear)[i] = u32x4{0u, 0u, 0u, 0u};
    auto round = [&](int sb) {
#pragma unroll
      for (int j = 0; j < DW; ++j) {
        if (j % 2 == 0) {
          wave_lds_fence();
#pragma unroll
          for (int i = 0; i < 2 * BT; ++i)
            *reinterpret_cast<u32x4 *>(xs + (8 * i + (lane >> 3)) * XROW + 16 * (lane & 7)) = raw[j / 2 % DX][i];
          wave_lds_fence();
          load_x(j / 2 % DX, sb / 2 + j / 2 + DX);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int bt = 0; bt < BT; ++bt) {
          const bf16x8 xf = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(xs + (16 * bt + r16) * XROW + 64 * (j % 2) + 16 * kg));
#pragma unroll
          for (int ft = 0; ft < FT; ++ft) acc[ft][bt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[j][ft], xf, acc[ft][bt], 0, 0, 0);
        }
        load_w(j, sb + j + DW);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    round(0);  // (by itself, see above)
    for (int sb = DW; sb < n; sb += DW) round(sb);
    __syncthreads();  // the waves' buffers are used again below
  }

  // ---- the waves' sums together --------------------------------------------------------------------
  // acc[ft][bt][i] of lane (r16, kg): feature 16 (tile0 + ft) + 4 kg + i, sequence 16 bt + r16
  float *red = reinterpret_cast<float *>(smem);  // [wave][ft][bt][lane][i]
  uint32_t ticket = 0;
  if (SECOND && tid == 0) ticket = draw_ticket(ns > 1 ? p.group_cnt + group * kMlpCntStride : p.done_cnt);
#pragma unroll
  for (int ft = 0; ft < FT; ++ft)
#pragma unroll
    for (int bt = 0; bt < BT; ++bt) *reinterpret_cast<f32x4 *>(red + (wave * NT + ft * BT + bt) * 256 + 4 * lane) = acc[ft][bt];
  __syncthreads();

  if constexpr (!SECOND) {
#pragma unroll
    for (int j = 0; j < NE; ++j) {
      if (!has(j)) continue;
      const int e = tid + j * kMlpThreads, bt = (e >> 6) % BT, f = feature(j);
      f32x4 v = *reinterpret_cast<const f32x4 *>(red + 4 * e);
#pragma unroll
      for (int w = 1; w < kMlpWaves; ++w) v += *reinterpret_cast<const f32x4 *>(red + w * NT * 256 + 4 * e);
      uint16_t hi[4], lo[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float y = mlp_act(v[i] + bias[j / BSTEP][i], p.act);
        hi[i] = f32_to_bf16(y);
        lo[i] = f32_to_bf16(y - bf16_to_f32(hi[i]));
      }
      uint16_t *dst = p.y + ((size_t)((f >> 5) * BT + bt) * 2) * 512 + ((f & 31) >> 3) * 128 + (e & 15) * 8 + (f & 7);
      *reinterpret_cast<uint2 *>(dst) = make_uint2(hi[0] | ((uint32_t)hi[1] << 16), hi[2] | ((uint32_t)hi[3] << 16));
      *reinterpret_cast<uint2 *>(dst + 512) = make_uint2(lo[0] | ((uint32_t)lo[1] << 16), lo[2] | ((uint32_t)lo[3] << 16));
    }
  } else {
    __shared__ float sm_dot[NT][4][16];
    __shared__ float sm_sum[kMlpThreads];
    __shared__ uint32_t sm_ticket[2];
    float v[NE];
#pragma unroll
    for (int j = 0; j < NE; ++j) {
      const int e = tid + j * kMlpThreads;
      v[j] = 0.f;
      if (in(j)) {
#pragma unroll
        for (int w = 0; w < kMlpWaves; ++w) v[j] += red[w * NT * 256 + e];
      }
    }
    if (ns > 1) {
      const size_t gb = (size_t)group * ns * (NT * 256);
#pragma unroll
      for (int j = 0; j < NE; ++j) {
        const int e = tid + j * kMlpThreads;
        if (in(j)) tagged_store(&p.part_sum[gb + (size_t)split * (NT * 256) + e], v[j], kMlpTag);
      }
      if (tid == 0) sm_ticket[0] = ticket;
      __syncthreads();
      if (sm_ticket[0] != (uint32_t)ns - 1) return;  // the holder of a group's last ticket goes on
      if (tid == 0) ticket = draw_ticket(p.done_cnt);
      float t[NE];
#pragma unroll
      for (int j = 0; j < NE; ++j) t[j] = 0.f;
      constexpr int SG = NE <= 4 ? 8 : 4;  // partial sums asked for at a time; added in index order
      for (int s0 = 0; s0 < ns; s0 += SG) {
        uint64_t w[SG][NE];
        bool ok;
        do {
          ok = true;
#pragma unroll
          for (int i = 0; i < SG; ++i)
#pragma unroll
            for (int j = 0; j < NE; ++j) {
              const int e = tid + j * kMlpThreads, s = s0 + i;
              w[i][j] = (uint64_t)kMlpTag << 32;
              if (s < ns && s != split && in(j)) w[i][j] = tagged_load(&p.part_sum[gb + (size_t)s * (NT * 256) + e]);
            }
#pragma unroll
          for (int i = 0; i < SG; ++i)
#pragma unroll
            for (int j = 0; j < NE; ++j) ok = ok && tag_is(w[i][j], kMlpTag);
        } while (!ok);
#pragma unroll
        for (int i = 0; i < SG; ++i)
#pragma unroll
          for (int j = 0; j < NE; ++j) t[j] += s0 + i == split ? v[j] : tagged_value(w[i][j]);
      }
#pragma unroll
      for (int j = 0; j < NE; ++j) v[j] = t[j];
    }
    // w3 . act(sum + bias) over this group's features
#pragma unroll
    for (int j = 0; j < NE; ++j) {
      const int e = tid + j * kMlpThreads, q = e >> 8;
      float t = has(j) ? w3[j / BSTEP] * mlp_act(v[j] + bias[j / BSTEP][0], p.act) : 0.f;
      t += __shfl_xor(t, 1);
      t += __shfl_xor(t, 2);
      if ((tid & 3) == 0 && in(j)) sm_dot[q][(e & 255) >> 6][(e & 63) >> 2] = t;
    }
    if (tid == 0) sm_ticket[1] = ticket;
    __syncthreads();
    const int n_groups = gridDim.x / ns;
    if (tid < p.Nb) {
      float t = 0.f;
#pragma unroll
      for (int ft = 0; ft < FT; ++ft)
#pragma unroll
        for (int k = 0; k < 4; ++k) t += sm_dot[ft * BT + (tid >> 4)][k][tid & 15];
      tagged_store(&p.part_dot[(size_t)group * p.Nb + tid], t, kMlpTag);
    }
    if (sm_ticket[1] != (uint32_t)n_groups - 1) return;  // the holder of the last ticket of all finishes
    constexpr int KT = kMlpThreads / (16 * BT);
    const int b = tid % (16 * BT), k = tid / (16 * BT);
    float t = 0.f;
    if (b < p.Nb && k < KT) {
      constexpr int U = 16;
      for (int g0 = k; g0 < n_groups; g0 += U * KT) {
        uint64_t w[U];
        bool ok;
        do {
          ok = true;
#pragma unroll
          for (int u = 0; u < U; ++u) {
            w[u] = (uint64_t)kMlpTag << 32;
            if (g0 + u * KT < n_groups) w[u] = tagged_load(&p.part_dot[(size_t)(g0 + u * KT) * p.Nb + b]);
          }
#pragma unroll
          for (int u = 0; u < U; ++u) ok = ok && tag_is(w[u], kMlpTag);
        } while (!ok);
#pragma unroll
        for (int u = 0; u < U; ++u) t += tagged_value(w[u]);
      }
    }
    sm_sum[tid] = t;
    __syncthreads();
    for (int o = tid; o < p.Nb * p.n_rep; o += kMlpThreads) {
      const int ob = o / p.n_rep;
      float s = sm_sum[ob];
#pragma unroll
      for (int i = 1; i < KT; ++i) s += sm_sum[i * 16 * BT + ob];
      p.s_out[o] = s + b3;
    }
  }
}

// Row-major bf16 weights [m][K] -> tiles of 16 rows x 32 columns stored contiguously, [m/16][K/32][16][32]:
// what one MFMA A-operand load of a wave reads becomes one contiguous kilobyte.  One-off, at load time.
// grid (ceil(m * K / 8 / 256)), 256 threads, 16 bytes per thread.
__global__ __launch_bounds__(256) void mlp_pack_kernel(const uint16_t *W, int m, int K, uint16_t *Wp) {
  const size_t piece = (size_t)blockIdx.x * 256 + threadIdx.x;  // 16-byte piece of the packed array
  if (piece >= (size_t)m * K / 8) return;
  const size_t e = piece * 8;                  // element index in the packed array
  const int c = (int)(e % 32), r = (int)((e / 32) % 16);
  const size_t ts = e / 512;                   // tile * n_steps + step
  const int n_steps = K / 32;
  const size_t tile = ts / n_steps, step = ts % n_steps;
  *reinterpret_cast<u32x4 *>(Wp + e) =
      *reinterpret_cast<const u32x4 *>(W + (tile * 16 + r) * (size_t)K + step * 32 + c);
}

// ---- the same head for sizes past 32-bit offsets, and for few features on a long K or many on a short one -----------------
// P[split][b][o] = sum_{k in split} W[o][k] * x[b][k] for either layer, then a kernel that adds the parts: four launches, every
// address 64 bits wide.  K is cut into as many slices as it has, so that a narrow layer fills the chip, too.

constexpr int kMlpSplitFeatures = 16 * kMlpWaves;  // a workgroup's: 16 a wave

struct MlpSplitParams {
  const uint16_t *W;    // [m][K] bf16
  const uint16_t *x0;   // [Nb][K] bf16 (hi part)
  const uint16_t *x1;   // [Nb][K] bf16 lo part, or null
  float *P;             // [nsplit][Nb][m] partial sums
  int Nb, m, K;
};

// k-steps (32 elements of K) one workgroup covers: its whole slice of the activations sits in 64 KB of LDS
// (128 KB for batches above 32, where the partial sums would otherwise outweigh the weights)
constexpr int mlp_slice_steps(int bt, int parts) { return (bt >= 4 ? 128 : 64) / (parts * bt); }

// BT = batch tiles of 16 (batch padded to 16 BT), PARTS = 1 (bf16 input) or 2 (hi + lo).
// grid (ceil(m / 128), ceil(K / 32 / S)), 512 threads, S = mlp_slice_steps(BT, PARTS).
// A workgroup fetches its slice of the activations once (all loads in flight together), parks it in
// LDS, meets at ONE barrier, and then only streams weights: a ring of DEPTH weight fragments per lane
// is kept in flight, so HBM latency is paid once per workgroup, not once per chunk.
template <int BT, int PARTS, bool PACKED>
__global__ __launch_bounds__(kMlpThreads) void mlp_split_gemm_kernel(const MlpSplitParams p) {
  constexpr int NBP = 16 * BT;                       // padded batch
  constexpr int S = mlp_slice_steps(BT, PARTS);      // k-steps per workgroup
  constexpr int DEPTH = S < 16 ? S : 16;             // weight fragments in flight per lane
  constexpr int LROW = S * 64 + 16;                  // padded LDS pitch of one batch row, bytes
  constexpr int PIECES = S * 4;                      // 16-byte pieces per batch row
  constexpr int NLD = PARTS * NBP * PIECES / kMlpThreads;  // = 8 staging loads per thread
  static_assert(PARTS * NBP * PIECES % kMlpThreads == 0, "staging must divide evenly");
  __shared__ __attribute__((aligned(16))) char lds[PARTS * NBP * LROW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, kg = lane >> 4;
  const int f0 = blockIdx.x * kMlpSplitFeatures + wave * 16;
  const bool has_rows = f0 < p.m;
  const int n_steps_all = p.K / 32;
  const int s0 = blockIdx.y * S;
  int s1 = s0 + S;
  s1 = s1 < n_steps_all ? s1 : n_steps_all;
  if (s0 >= s1) return;  // uniform
  const int n_steps = s1 - s0;

  // this lane's weight fragments.  Row-major weights: 16 bytes of row f0 + r16 per k-step, i.e. 16 rows a
  // whole weight row apart per load instruction.  Packed weights ([m/16][K/32][16][32], see
  // mlp_pack_kernel): the 1 KB a load instruction needs is contiguous, and so is the whole slice.
  // (Rows past the last repeat it; their results are not written.)
  int frow = f0 + r16;
  frow = frow < p.m ? frow : p.m - 1;
  const char *Wrow =
      PACKED ? reinterpret_cast<const char *>(p.W + ((size_t)(frow >> 4) * n_steps_all + s0) * 512 + (frow & 15) * 32) + 16 * kg
             : reinterpret_cast<const char *>(p.W + (size_t)frow * p.K + (size_t)s0 * 32) + 16 * kg;
  constexpr size_t kStepBytes = PACKED ? 1024 : 64;
  // first weight fragments on their way before anything else (steps past the slice repeat its last)
  bf16x8 wf[DEPTH];
#pragma unroll
  for (int j = 0; j < DEPTH; ++j) {
    const int st = j < n_steps ? j : n_steps - 1;
    wf[j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(Wrow + (size_t)st * kStepBytes));
  }

  // the slice of the activations: piece q = (part, batch row, 16-byte piece), coalesced along K
  {
    u32x4 stage[NLD];
#pragma unroll
    for (int k = 0; k < NLD; ++k) {
      const int q = tid + kMlpThreads * k;
      const int part = q / (NBP * PIECES), rem = q - part * (NBP * PIECES);
      int row = rem / PIECES;
      const int piece = rem - row * PIECES;
      row = row < p.Nb ? row : p.Nb - 1;
      int e = s0 * 32 + 8 * piece;
      e = e < s1 * 32 ? e : s1 * 32 - 8;  // past the slice: repeat its last piece (never multiplied)
      const uint16_t *src = (PARTS == 2 && part == 1) ? p.x1 : p.x0;
      stage[k] = *reinterpret_cast<const u32x4 *>(src + (size_t)row * p.K + e);
    }
#pragma unroll
    for (int k = 0; k < NLD; ++k) {
      const int q = tid + kMlpThreads * k;
      const int part = q / (NBP * PIECES), rem = q - part * (NBP * PIECES);
      const int row = rem / PIECES, piece = rem - row * PIECES;
      *reinterpret_cast<u32x4 *>(lds + (part * NBP + row) * LROW + 16 * piece) = stage[k];
    }
  }
  __syncthreads();
  if (!has_rows) return;

  f32x4 acc[BT];
#pragma unroll
  for (int bt = 0; bt < BT; ++bt) acc[bt] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int sb = 0; sb < n_steps; sb += DEPTH) {
#pragma unroll
    for (int j = 0; j < DEPTH; ++j) {
      const int st = sb + j;
      if (st < n_steps) {  // uniform
#pragma unroll
        for (int bt = 0; bt < BT; ++bt) {
#pragma unroll
          for (int part = 0; part < PARTS; ++part) {
            const bf16x8 xf = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(
                lds + (part * NBP + 16 * bt + r16) * LROW + 64 * st + 16 * kg));
            acc[bt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[j], xf, acc[bt], 0, 0, 0);
          }
        }
      }
      if (S > DEPTH) {  // refill this ring slot with the fragment DEPTH steps ahead
        int nx = st + DEPTH;
        nx = nx < n_steps ? nx : n_steps - 1;
        wf[j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(Wrow + (size_t)nx * kStepBytes));
      }
    }
  }

  // acc[bt][i]: feature f0 + 4 kg + i, batch 16 bt + r16
  const int f = f0 + 4 * kg;
#pragma unroll
  for (int bt = 0; bt < BT; ++bt) {
    const int b = 16 * bt + r16;
    if (b < p.Nb && f < p.m) {  // m is a multiple of 16, so the four features are all valid
      float *dst = p.P + ((size_t)blockIdx.y * p.Nb + b) * p.m + f;
      *reinterpret_cast<f32x4 *>(dst) = acc[bt];
    }
  }
}

// y = act(sum over splits of P + bias), written as bf16 hi and lo parts for the next layer.
// grid (ceil(Nb * m / 4 / 256)), 256 threads, 4 features per thread.
__global__ __launch_bounds__(256) void mlp_split_act_kernel(const float *P, const float *bias, int nsplit, int Nb,
                                                             int m, int act, uint16_t *y_hi, uint16_t *y_lo,
                                                             u32x4 *clear, size_t n_clear) {
  // (the final kernel's tagged words and counters: stream order puts this first)
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n_clear; i += (size_t)gridDim.x * 256) clear[i] = u32x4{0u, 0u, 0u, 0u};
  const size_t idx = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (idx >= (size_t)Nb * m) return;
  const int o = (int)(idx % m);
  f32x4 v = *reinterpret_cast<const f32x4 *>(P + idx);
#pragma unroll 4
  for (int s = 1; s < nsplit; ++s) v += *reinterpret_cast<const f32x4 *>(P + (size_t)s * Nb * m + idx);
  uint16_t hi[4], lo[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float y = mlp_act(v[i] + (bias ? bias[o + i] : 0.f), act);
    hi[i] = f32_to_bf16(y);
    lo[i] = f32_to_bf16(y - bf16_to_f32(hi[i]));
  }
  *reinterpret_cast<uint2 *>(y_hi + idx) = make_uint2(hi[0] | ((uint32_t)hi[1] << 16), hi[2] | ((uint32_t)hi[3] << 16));
  *reinterpret_cast<uint2 *>(y_lo + idx) = make_uint2(lo[0] | ((uint32_t)lo[1] << 16), lo[2] | ((uint32_t)lo[3] << 16));
}

// s[b] = w3 . act(sum over splits of P[.][b][:] + bias) + b3, written n_rep times.
// grid (ceil(m / 256), Nb), 256 threads: a workgroup takes 256 features of one sequence and leaves its part of
// the dot product in part[b][blockIdx.x] as a tagged word; the workgroup that draws the last ticket of a
// sequence adds the parts in index order, re-reading a word until it carries the tag, so the result
// does not depend on the arrival order and no store has to be waited for.
__global__ __launch_bounds__(256) void mlp_split_dot_kernel(const float *P, const float *bias, int nsplit, int Nb,
                                                             int m, int act, const uint16_t *w3, const float *b3,
                                                             uint64_t *part, uint32_t *row_cnt,
                                                             float *s_out, int n_rep) {
  __shared__ float red[4];
  __shared__ int is_last;
  const int b = blockIdx.y, tid = threadIdx.x, o = blockIdx.x * 256 + tid;
  float t = 0.f;
  if (o < m) {
    float v = 0.f;
#pragma unroll 8
    for (int s = 0; s < nsplit; ++s) v += P[((size_t)s * Nb + b) * m + o];
    t = bf16_to_f32(w3[o]) * mlp_act(v + (bias ? bias[o] : 0.f), act);
  }
#pragma unroll
  for (int sh = 32; sh >= 1; sh >>= 1) t += __shfl_xor(t, sh);
  if ((tid & 63) == 0) red[tid >> 6] = t;
  __syncthreads();
  if (tid == 0) {
    tagged_store(part + (size_t)b * gridDim.x + blockIdx.x, (red[0] + red[1]) + (red[2] + red[3]), kMlpTag);
    is_last = atomicAdd(row_cnt + b, 1u) == gridDim.x - 1;
  }
  __syncthreads();
  if (!is_last) return;
  if (tid < n_rep) {
    float tot = 0.f;
    for (unsigned k = 0; k < gridDim.x; ++k) {
      uint64_t w;
      do w = tagged_load(part + (size_t)b * gridDim.x + k);
      while (!tag_is(w, kMlpTag));
      tot += tagged_value(w);
    }
    s_out[(size_t)b * n_rep + tid] = tot + (b3 ? b3[0] : 0.f);
  }
}

}  // namespace dynts
