// Importance score from a block of T queries at once (Eq. importance-score with the sum over the
// answer tokens written out; App. B.1: the answer-by-thinking sub-matrix of the attention weights,
// summed over heads and over the answer dimension).  A dense [T*G x n] contraction per
// (sequence, KV head), done on the matrix cores in two passes over Q.K^T:
//   pass 1 (stats):  for every query row the log2 of its softmax denominator over the cached slots
//                    and, causally, the block's own keys  ->  L[row]  (one float per row);
//   pass 2 (colsum): logits again, p = 2^(logit - L[row]), summed over the rows for every cached
//                    slot  ->  dst[slot].
// Recomputing the logits costs a second pass of MFMAs; keeping them would cost 4 bytes per
// (row, slot) of HBM traffic each way, which at these shapes is several times slower.
//
// Both passes have the same shape.  A wave keeps 64 rows of one operand in registers (pass 1: query
// rows, pass 2: cached keys) as B fragments of v_mfma_f32_32x32x16_bf16 (lane (c, hf) = (lane % 32, lane / 32)
// holds elements 16*ks + 8*hf .. +7 of row c; A and B alike).  The other operand is streamed: the workgroup's
// 256 threads fetch 32 rows at a time, eight threads to a row (whole 128-byte lines), park them in one of two
// padded LDS buffers, and every wave reads its A fragments back from there (row pitch +16 bytes: the rows a
// ds_read_b128 touches fall into different banks).  The next chunk's loads are in flight while a chunk is
// multiplied; one barrier per chunk.  The product is  streamed rows (A)  x  stationary columns (B): a lane ends
// up with 16 streamed rows (8*(i/4) + 4*hf + i%4) of ONE stationary column, so
//   * pass 1 keeps a private shift and sum per lane and query column and merges the two lane halves
//     once, at the end;
//   * pass 2 keeps one private column sum per lane and key and adds the two halves once, at the end.
//
// What bounds them: the instruction stream.  A logit needs a multiply-add, a 2^x and an add in each pass beside
// its share of the MFMA, and the two pipes overlap only in part (dynts_probe_issue_mix, just these without memory: 0.355 us
// per 32 x 64 chunk and SIMD; MFMAs alone 0.267, vector instructions alone 0.211), so everything else that is issued
// per chunk counts.  32x32 tiles take half the MFMA issue slots and LDS reads per product of 16x16 ones, and one row
// per staging thread leaves one address to advance.  A block of 512 queries over 2464 slots
// (128 units, 28 query heads on 4): 664 -> 597 us a call against 16x16 tiles with a running maximum, 67 % of that mix's
// rate; 64 queries: 126 -> 98 us.  What lies between: with operands that do not toggle, zeros or one constant, the same instructions take 462 us (87 %);
// the 29 % on top are the clock that random products leave (64 queries: 77 and 90 us).  Tried and slower: products of one tile interleaved by hand with the exponentials of
// another in one wave (600 -> 640 us and more: registers).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "attend.hpp"

namespace dynts {

constexpr int kSbWaves = 4;        // waves per workgroup
constexpr int kSbTiles = 2;        // stationary 32-row tiles per wave
constexpr int kSbRowsPerWave = 32 * kSbTiles;
constexpr int kSbRowsPerWg = kSbRowsPerWave * kSbWaves;
constexpr int kSbChunk = 32;       // streamed rows per chunk
constexpr int kSbLRows = kSbWaves * 64;  // rows whose denominators are staged at a time (one per thread)
constexpr int kSbMaxSplits = 4;    // key ranges of the first pass

typedef float f32x16 __attribute__((ext_vector_type(16)));

struct ScoreBlockParams {
  const uint16_t *K;        // layer base, [Nb][Hkv][cap][D]
  const uint16_t *q_blk;    // [Nb][T][Hq][D]
  const uint16_t *k_blk;    // [Nb][T][Hkv][D] or null
  const int32_t *seq_len;   // [Nb]
  const int32_t *n_prompt;  // [Nb]
  const uint8_t *active;    // [Nb] or null
  float *stats;             // [Nb][Hkv][n_split][Rpad]  log2 of the softmax denominator per query row and key range
  float *dst;               // [Nb][Hkv][cap]
  int Nb, T, Hq, Hkv, G, cap, Rpad;
  int n_split;              // key ranges (workgroups) the first pass cuts a unit's keys into
  int skip_prompt;          // 1: slots below n_prompt[b] are left alone (dst is the score array)
  int accumulate;           // 1: dst += sums, 0: dst = sums
  float scale_log2;         // softmax scale * log2(e)
  // paged layout: K is the page pool, slot j of a unit is row j % 64 of page block_table[unit][j / 64]
  const int32_t *block_table;  // layer base [Nb][Hkv][max_pages], or null (dense layout)
  int max_pages, n_pages;
};

// byte offset from K of cached key row `row` of a unit (dense rows, or through the block table)
template <int D, bool PAGED>
__device__ __forceinline__ size_t sb_key_row(const ScoreBlockParams &p, size_t unit, int row) {
  if (PAGED) {
    int pi = row / kPageSlots;
    pi = pi < p.max_pages ? pi : p.max_pages - 1;
    int pg = p.block_table[unit * (size_t)p.max_pages + pi];
    pg = pg < 0 ? 0 : (pg >= p.n_pages ? p.n_pages - 1 : pg);
    return ((size_t)pg * kPageSlots + row % kPageSlots) * (2 * D);
  }
  return (unit * (size_t)p.cap + row) * (2 * D);
}

// MFMA operand fragments of one row (global memory or LDS): 16 bytes per k-step of 16 at the lane's half.
template <int D>
__device__ __forceinline__ void load_row_frags(bf16x8 (&f)[D / 16], const char *row, int hf) {
  const char *base = row + 16 * hf;
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks)
    f[ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(base + 32 * ks));
}

template <int D>
struct SbStage {
  static constexpr int NL = D / 64;              // 16-byte loads per thread and chunk, 128 bytes apart
  static constexpr int LROW = 2 * D + 16;        // padded row pitch in LDS, bytes
  static constexpr int kBufBytes = kSbChunk * LROW;
};

// The products of one chunk: 32 streamed rows (in LDS) x the wave's 64 stationary columns.
template <int D>
__device__ __forceinline__ void sb_multiply(f32x16 (&acc)[kSbTiles], const char *buf, const bf16x8 (&st)[kSbTiles][D / 16],
                                            int c, int hf) {
  bf16x8 a[D / 16];
  load_row_frags<D>(a, buf + c * SbStage<D>::LROW, hf);
#pragma unroll
  for (int t = 0; t < kSbTiles; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
  __builtin_amdgcn_s_setprio(1);  // (a wave's products first: 1 % of both passes)
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
    for (int t = 0; t < kSbTiles; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks], st[t][ks], acc[t], 0, 0, 0);
  __builtin_amdgcn_s_setprio(0);
}

// Sum over a lane's 16 products of 2^(c * product + add_i), in a balanced tree: the running sums then take one rounding per
// chunk instead of one per row.
template <typename Add>
__device__ __forceinline__ float sb_exp_sum(const f32x16 &acc, float c, Add add) {
  float q[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float e0 = fast_exp2(fmaf(acc[4 * j], c, add(4 * j))), e1 = fast_exp2(fmaf(acc[4 * j + 1], c, add(4 * j + 1)));
    const float e2 = fast_exp2(fmaf(acc[4 * j + 2], c, add(4 * j + 2))), e3 = fast_exp2(fmaf(acc[4 * j + 3], c, add(4 * j + 3)));
    q[j] = (e0 + e1) + (e2 + e3);
  }
  return (q[0] + q[1]) + (q[2] + q[3]);
}

// Workgroup -> (unit, block).  Consecutive workgroup ids go to the 8 XCDs in turn; this mapping
// keeps all blocks of one (sequence, KV head) unit on one XCD, so the operand they all stream is
// fetched into one L2 instead of eight.  Returns false for the padding of the last group of units.
__device__ __forceinline__ bool sb_map(int n_blk, int n_units, int &unit, int &blk) {
  const int id = blockIdx.x, xcd = id & 7, slot = id >> 3;
  unit = (slot / n_blk) * 8 + xcd;
  blk = slot % n_blk;
  return unit < n_units;
}

// ---- pass 1: log2 of the softmax denominator of every query row ---------------------------------
// 1-D grid of ceil(R / 256) * n_split * round_up(units, 8) workgroups, 256 threads.
//
// The shift that keeps the exponentials in range is not a running maximum: it is raised only when a logit lies above it.
// A chunk is folded with the shift at hand, and a chunk's sum that is too large for keys below the shift (or infinite;
// the first always is, its shift is far below any logit) sends the wave back to the chunk's logits, which are still in
// registers, with their true maximum.  A maximum over every logit costs a sixth of the vector instructions.
template <int D, bool PAGED>
__global__ __launch_bounds__(kSbWaves * 64, 3) void score_block_stats_kernel(const ScoreBlockParams p) {
  using St = SbStage<D>;
  __shared__ __attribute__((aligned(16))) char lds[2][St::kBufBytes];
  const int R = p.T * p.G;
  int unit, blk;
  const int n_blk = (R + kSbRowsPerWg - 1) / kSbRowsPerWg;
  if (!sb_map(n_blk * p.n_split, p.Nb * p.Hkv, unit, blk)) return;
  const int split = blk % p.n_split;
  blk /= p.n_split;
  const int b = unit / p.Hkv, h = unit - b * p.Hkv;
  if (p.active && !p.active[b]) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 31, hf = lane >> 5;
  const int row0 = blk * kSbRowsPerWg + wave * kSbRowsPerWave;
  // (the same in every lane of a wave, and told so to the compiler; a wave without rows still helps staging and
  // meets the barriers)
  const bool has_rows = __builtin_amdgcn_readfirstlane((int)(row0 < R)) != 0;
  int n = p.seq_len[b];
  n = n < 0 ? 0 : (n > p.cap ? p.cap : n);
  const char *Qb = reinterpret_cast<const char *>(p.q_blk + ((size_t)b * p.T * p.Hq + (size_t)h * p.G) * D);
  const float c = p.scale_log2;

  // stationary: this wave's query rows (column col of tile qt is row row0 + 32 qt + col)
  bf16x8 qf[kSbTiles][D / 16];
  int vis_blk[kSbTiles];  // block keys [0, vis_blk) are visible to this lane's query column
#pragma unroll
  for (int qt = 0; qt < kSbTiles; ++qt) {
    int r = row0 + 32 * qt + col;
    r = r < R ? r : R - 1;
    const int i = r / p.G, g = r - i * p.G;
    vis_blk[qt] = i + 1;
    load_row_frags<D>(qf[qt], Qb + ((size_t)i * p.Hq + g) * (size_t)(2 * D), hf);
  }

  // the exponents' addend (minus the shift, a whole number of log2 units) and the sum of 2^(c * dot + addend), private to the lane
  float nm[kSbTiles], l[kSbTiles];
#pragma unroll
  for (int qt = 0; qt < kSbTiles; ++qt) {
    nm[qt] = 1e30f;
    l[qt] = 0.f;
  }
  // A lane's 16 keys below the shift sum to 16 at most; from kLimit on some key lies above it.
  constexpr float kLimit = 16.5f;

  // Folds the chunk's logits into (nm, l).  masked: keys at or beyond lim[qt] do not exist for this query column.
  auto fold = [&](f32x16 (&acc)[kSbTiles], bool masked, int key0, const int (&lim)[kSbTiles]) {
    if (masked) {
#pragma unroll
      for (int qt = 0; qt < kSbTiles; ++qt)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (key0 + 8 * (i >> 2) + 4 * hf + (i & 3) >= lim[qt]) acc[qt][i] = -INFINITY;
    }
    float s[kSbTiles];
#pragma unroll
    for (int qt = 0; qt < kSbTiles; ++qt) {
      const float add = nm[qt];
      s[qt] = sb_exp_sum(acc[qt], c, [&](int) { return add; });
    }
    if (__any(fmaxf(s[0], s[1]) >= kLimit)) {
#pragma unroll
      for (int qt = 0; qt < kSbTiles; ++qt) {
        float mx = acc[qt][0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, acc[qt][i]);
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float nn = fminf(floorf(-mx * c), nm[qt]);
        l[qt] *= fast_exp2(nn - nm[qt]);
        s[qt] = sb_exp_sum(acc[qt], c, [&](int) { return nn; });
        nm[qt] = nn;
      }
    }
#pragma unroll
    for (int qt = 0; qt < kSbTiles; ++qt) l[qt] += s[qt];
  };

  // Streaming of chunks [c0, c1) of `rows` rows; rows beyond the last repeat it (the fold masks them).  own: rows of
  // the block's keys, pitch bytes apart, else the unit's cached key rows.  Every thread runs this.  Keys below see_all
  // are visible to all of the wave's rows, keys from see_any on to none (both the same in every lane).
  const int st_row = tid >> 3;
  const uint32_t st_piece = 16u * (uint32_t)(tid & 7);
  char *const park = lds[0] + st_row * St::LROW + st_piece;
  u32x4 stage[St::NL];
  auto stream = [&](auto OWN, const char *src, uint32_t pitch, int rows, int c0, int c1, int see_all, int see_any,
                    const int (&lim)[kSbTiles]) {
    constexpr bool own = decltype(OWN)::value;
    if (c0 >= c1) return;
    uint32_t off = (uint32_t)(c0 * kSbChunk + st_row) * pitch + st_piece;
    const uint32_t last = (uint32_t)(rows - 1) * pitch + st_piece;
    auto fetch = [&](int ch) {
      const char *rp;
      if (PAGED && !own) {  // a chunk lies inside one page
        const int first = ch * kSbChunk;
        int r = st_row < rows - 1 - first ? st_row : rows - 1 - first;
        rp = src + sb_key_row<D, true>(p, (size_t)unit, first) + ((uint32_t)r * (uint32_t)(2 * D) + st_piece);
      } else {
        rp = src + (off < last ? off : last);
        off += kSbChunk * pitch;
      }
#pragma unroll
      for (int k = 0; k < St::NL; ++k) stage[k] = *reinterpret_cast<const u32x4 *>(rp + 128 * k);
    };
    auto put = [&](int buf) {
#pragma unroll
      for (int k = 0; k < St::NL; ++k) *reinterpret_cast<u32x4 *>(park + buf * St::kBufBytes + 128 * k) = stage[k];
    };
    // Per chunk: one barrier; the next chunk, fetched an iteration ago, goes to the other buffer (read last before the
    // barrier); the one after it is fetched.
    fetch(c0);
    put(0);
    if (c0 + 1 < c1) fetch(c0 + 1);
    int buf = 0;
    for (int ch = c0; ch < c1; ++ch) {
      __syncthreads();
      if (ch + 1 < c1) put(buf ^ 1);
      if (ch + 2 < c1) fetch(ch + 2);
      if (ch * kSbChunk < see_any) {
        f32x16 acc[kSbTiles];
        sb_multiply<D>(acc, lds[buf], qf, col, hf);
        if ((ch + 1) * kSbChunk > see_all) fold(acc, true, ch * kSbChunk, lim);
        else fold(acc, false, 0, lim);
      }
      buf ^= 1;
    }
    __syncthreads();  // the buffers are filled again by the next stream
  };

  // The keys this workgroup sees: the cached slots (every query column sees all n of them), then the block's own keys,
  // causally: key i' is visible to query row (i, g) iff i' <= i, so keys [0, i_hi) to some row here.  Chunks of both
  // are numbered through and cut into n_split equal ranges.
  int i_hi = 0;
  if (p.k_blk) {
    int last = blk * kSbRowsPerWg + kSbRowsPerWg - 1;
    last = last < R ? last : R - 1;
    i_hi = last / p.G + 1;
  }
  const int nc = (n + kSbChunk - 1) / kSbChunk, no = (i_hi + kSbChunk - 1) / kSbChunk;
  const int lo = (int)((long long)(nc + no) * split / p.n_split), hi = (int)((long long)(nc + no) * (split + 1) / p.n_split);
  {
    int lim[kSbTiles];
#pragma unroll
    for (int qt = 0; qt < kSbTiles; ++qt) lim[qt] = n;
    const char *src = reinterpret_cast<const char *>(p.K) + (PAGED ? 0 : sb_key_row<D, false>(p, (size_t)unit, 0));
    stream(std::false_type{}, src, (uint32_t)(2 * D), n, lo, hi < nc ? hi : nc, n, has_rows ? n : 0, lim);
  }
  if (p.k_blk) {
    const char *src = reinterpret_cast<const char *>(p.k_blk + ((size_t)b * p.T * p.Hkv + h) * D);
    const int last = row0 + kSbRowsPerWave - 1 < R ? row0 + kSbRowsPerWave - 1 : R - 1;
    const int see_all = __builtin_amdgcn_readfirstlane(row0 / p.G + 1);
    const int see_any = __builtin_amdgcn_readfirstlane(has_rows ? last / p.G + 1 : 0);
    stream(std::true_type{}, src, (uint32_t)p.Hkv * (uint32_t)(2 * D), i_hi, lo > nc ? lo - nc : 0, hi - nc, see_all, see_any, vis_blk);
  }
  if (!has_rows) return;

  // Merge the two lane halves of every query column, write L = log2(l) - nm.  nm is a whole number, so the exponent of l
  // joins it without rounding and only the logarithm of l's mantissa is rounded, at the size of L.
#pragma unroll
  for (int qt = 0; qt < kSbTiles; ++qt) {
    const float no2 = __shfl_xor(nm[qt], 32), lo2 = __shfl_xor(l[qt], 32);
    const float nn = fminf(nm[qt], no2);
    const float lt = l[qt] * fast_exp2(nn - nm[qt]) + lo2 * fast_exp2(nn - no2);
    const float whole = (float)__builtin_amdgcn_frexp_expf(lt) - nn;
    const int r = row0 + 32 * qt + col;
    if (hf == 0 && r < R)
      p.stats[((size_t)unit * p.n_split + split) * (size_t)p.Rpad + r] = whole + __builtin_amdgcn_logf(__builtin_amdgcn_frexp_mantf(lt));
  }
}

// ---- pass 2: attention received by every cached slot, summed over the block's query rows ----------
// 1-D grid of ceil(cap / 256) * round_up(units, 8) workgroups, 256 threads.
template <int D, bool PAGED>
__global__ __launch_bounds__(kSbWaves * 64, 3) void score_block_colsum_kernel(const ScoreBlockParams p) {
  using St = SbStage<D>;
  __shared__ __attribute__((aligned(16))) char lds[2][St::kBufBytes];
  __shared__ __attribute__((aligned(16))) float ldsL[2][kSbLRows];
  int unit, blk;
  if (!sb_map((p.cap + kSbRowsPerWg - 1) / kSbRowsPerWg, p.Nb * p.Hkv, unit, blk)) return;
  const int b = unit / p.Hkv, h = unit - b * p.Hkv;
  if (p.active && !p.active[b]) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 31, hf = lane >> 5;
  const int R = p.T * p.G;
  int n = p.seq_len[b];
  n = n < 0 ? 0 : (n > p.cap ? p.cap : n);
  int first = 0;
  if (p.skip_prompt) {
    first = p.n_prompt[b];
    first = first < 0 ? 0 : first;
  }
  // uniform over the workgroup: nothing of this block is wanted
  if (blk * kSbRowsPerWg >= n || (blk + 1) * kSbRowsPerWg <= first) return;
  const int key0 = blk * kSbRowsPerWg + wave * kSbRowsPerWave;
  // (the same in every lane of a wave, and told so to the compiler: a plain branch instead of lane masks)
  const bool has_keys = __builtin_amdgcn_readfirstlane((int)(key0 < n && key0 + kSbRowsPerWave > first)) != 0;  // else: staging and barriers only
  const char *Qb = reinterpret_cast<const char *>(p.q_blk + ((size_t)b * p.T * p.Hq + (size_t)h * p.G) * D);
  const float *Lb = p.stats + (size_t)unit * p.n_split * (size_t)p.Rpad;
  const float c = p.scale_log2;

  // stationary: this wave's cached keys (column col of tile kt is slot key0 + 32 kt + col)
  bf16x8 kf[kSbTiles][D / 16];
#pragma unroll
  for (int kt = 0; kt < kSbTiles; ++kt) {
    int row = key0 + 32 * kt + col;
    row = row < n ? row : n - 1;
    load_row_frags<D>(kf[kt], reinterpret_cast<const char *>(p.K) + sb_key_row<D, PAGED>(p, (size_t)unit, row), hf);
  }
  float sum[kSbTiles];
#pragma unroll
  for (int kt = 0; kt < kSbTiles; ++kt) sum[kt] = 0.f;

  // streamed: the R query rows, 32 per chunk through LDS, and their log2 denominators, 256 rows at a time (one per
  // thread; left to one wave per chunk they held the other three up at the barrier, 8 % of the kernel).  A row beyond
  // the last repeats the last row's data and gets L = +inf, so it contributes 2^(-inf) = 0.
  // A thread stages row r = i * G + g; a chunk further on that is step_i tokens and step_g heads.
  const int st_row = tid >> 3;
  const uint32_t st_piece = 16u * (uint32_t)(tid & 7);
  char *const park = lds[0] + st_row * St::LROW + st_piece;
  const uint32_t stride_i = (uint32_t)p.Hq * (uint32_t)(2 * D);
  const int step_i = kSbChunk / p.G, step_g = kSbChunk - step_i * p.G;
  const uint32_t step_off = (uint32_t)step_i * stride_i + (uint32_t)step_g * (uint32_t)(2 * D);
  const uint32_t wrap_off = stride_i - (uint32_t)p.G * (uint32_t)(2 * D);
  int g = st_row % p.G;
  uint32_t off = (uint32_t)(st_row / p.G) * stride_i + (uint32_t)g * (uint32_t)(2 * D) + st_piece;
  const uint32_t last = (uint32_t)(p.T - 1) * stride_i + (uint32_t)(p.G - 1) * (uint32_t)(2 * D) + st_piece;
  u32x4 stage[St::NL];
  float stageL[kSbMaxSplits];
#pragma unroll
  for (int s = 0; s < kSbMaxSplits; ++s) stageL[s] = -INFINITY;
  int l_row = 0;  // the row whose L this thread has fetched
  auto fetch = [&]() {
    const char *rp = Qb + (off < last ? off : last);  // (offsets grow with the row)
#pragma unroll
    for (int k = 0; k < St::NL; ++k) stage[k] = *reinterpret_cast<const u32x4 *>(rp + 128 * k);
    off += step_off;
    g += step_g;
    if (g >= p.G) {
      g -= p.G;
      off += wrap_off;
    }
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int k = 0; k < St::NL; ++k) *reinterpret_cast<u32x4 *>(park + buf * St::kBufBytes + 128 * k) = stage[k];
  };
  auto fetch_L = [&](int group) {
    l_row = group * kSbLRows + tid;
    const uint32_t at = (uint32_t)(l_row < R ? l_row : R - 1);
    stageL[0] = Lb[at];
    if (p.n_split > 1) {
#pragma unroll
      for (int s = 1; s < kSbMaxSplits; ++s)
        if (s < p.n_split) stageL[s] = Lb[at + (uint32_t)(s * p.Rpad)];
    }
  };
  auto put_L = [&](int buf) {
    float L = stageL[0];
    if (p.n_split > 1) {  // the key ranges' denominators together
      float mx = L, t = 0.f;
#pragma unroll
      for (int s = 1; s < kSbMaxSplits; ++s) mx = fmaxf(mx, stageL[s]);
#pragma unroll
      for (int s = 0; s < kSbMaxSplits; ++s) t += fast_exp2(stageL[s] - mx);
      L = mx + __builtin_amdgcn_logf(t);
    }
    ldsL[buf][tid] = l_row < R ? L : INFINITY;
  };

  const int n_chunks = (R + kSbChunk - 1) / kSbChunk;
  constexpr int kGroup = kSbLRows / kSbChunk;  // chunks per group of denominators
  fetch();
  fetch_L(0);
  put(0);
  put_L(0);
  if (n_chunks > 1) fetch();
  int buf = 0;
  for (int ch = 0; ch < n_chunks; ++ch) {
    __syncthreads();
    if (ch + 1 < n_chunks) put(buf ^ 1);
    if (ch + 2 < n_chunks) fetch();
    const int in_group = ch % kGroup, group = ch / kGroup;
    if (in_group == 0 && ch + kGroup < n_chunks) fetch_L(group + 1);
    if (in_group == kGroup - 1 && ch + 1 < n_chunks) put_L((group + 1) & 1);
    if (has_keys) {
      f32x16 acc[kSbTiles];
      f32x4 L[4];  // of the rows 8 j + 4 hf .. +3 this lane's products belong to
#pragma unroll
      for (int j = 0; j < 4; ++j) L[j] = *reinterpret_cast<const f32x4 *>(&ldsL[group & 1][in_group * kSbChunk + 8 * j + 4 * hf]);
      sb_multiply<D>(acc, lds[buf], kf, col, hf);
#pragma unroll
      for (int kt = 0; kt < kSbTiles; ++kt)
        sum[kt] += sb_exp_sum(acc[kt], c, [&](int i) { return -L[i >> 2][i & 3]; });
    }
    buf ^= 1;
  }
  if (!has_keys) return;

  // add the two halves' rows; lane (col, hf) writes slot key0 + 32 hf + col
  float tot[kSbTiles];
#pragma unroll
  for (int kt = 0; kt < kSbTiles; ++kt) {
    tot[kt] = sum[kt] + __shfl_xor(sum[kt], 32);
  }
  const float v = hf == 0 ? tot[0] : tot[1];
  const int slot = key0 + 32 * hf + col;
  if (slot < n && slot >= first) {
    float *d = p.dst + (size_t)unit * (size_t)p.cap + slot;
    *d = p.accumulate ? *d + v : v;
  }
}

}  // namespace dynts
