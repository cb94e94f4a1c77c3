// Epilogue shared by the scoring kernels (Sec. 3.4.1): from the similarities omega of one point, held as
// matrix-core accumulators, to the stored scores, the arg-max label and the kernel regression of Eq. 4.
#pragma once

#include "aura_device.hpp"

namespace aura {

typedef float scores_f32x4 __attribute__((ext_vector_type(4)));
typedef float scores_f32x16 __attribute__((ext_vector_type(16)));

constexpr int kScoreTileM = 32;   // materials per matrix-core tile
constexpr int kScoreMaxP = 8;
constexpr int kScoreMaxK = 128;

// The property table in LDS as the epilogues read it: ys[p][m] with the materials padded to whole tiles by zeros, so that the values
// of a lane's four consecutive materials are one 16-byte read.  ys holds kScoreTileM * MT * P floats, 16-byte aligned; called by all
// `threads` threads, followed by a barrier.
template <int MT>
__device__ __forceinline__ void stage_properties(float* __restrict__ ys, const float* __restrict__ y, int K, int P, int thread,
                                                 int threads) {
  constexpr int kPad = kScoreTileM * MT;
  for (int t = thread; t < kPad * P; t += threads) {
    const int p = t / kPad, m = t % kPad;
    ys[t] = m < K ? y[m * P + p] : 0.0f;
  }
}

// Label and Eq. 4.  Lane l = 32 g + (point within the wave's 32): accumulator element r of tile mt is the similarity of the
// lane's point to material mt*32 + 8*(r/4) + 4*g + r%4, so the two lanes l and l ^ 32 hold all K scores of one
// point between them.  `ys`: see stage_properties.  store: whether the lane writes its point's results; all 64 lanes call this.
// The accumulators are used up.
// unseen_zero: a point whose similarities are all exactly zero (the fused row of a point that no view sees is all
// zero) gets zero properties instead of what Eq. 4 gives for equal similarities, the mean of y.
// One straight line of instructions, with places beyond K holding -inf (weight 0): as a branch per material, eight per
// material over P and an LDS read waited for in each, Eq. 4 held up whatever scored: single pass over 40 objects of 50 000 points and
// 24 materials 622 -> 588 us (its scoring wave was what the other waves waited for), 1.68 M voxels and 128 materials 1183 -> 1130,
// 123 457 points and 45 materials 184 -> 173 (with the stores of finish_scores_staged for any K), 200 000 queries densified 318 ->
// 307.
// QUADS: the first groups of eight places, four per lane group, that K may reach into.
template <int MT, int QUADS>
__device__ __forceinline__ void finish_quads(scores_f32x16 (&acc)[MT], long long n, bool store, int g, int K, int P, float inv_T,
                                             const float* __restrict__ ys, float* __restrict__ prop, int* __restrict__ label,
                                             bool unseen_zero) {
  constexpr int kRows = 4 * QUADS;   // accumulator elements that can hold a material: acc[r / 16][r % 16]
  auto material = [&](int r) { return 8 * (r >> 2) + 4 * g + (r & 3); };
  bool any_nonzero = false;
  if (unseen_zero) {   // uniform
#pragma unroll
    for (int r = 0; r < kRows; ++r) any_nonzero = any_nonzero || (material(r) < K && acc[r >> 4][r & 15] != 0.0f);
    any_nonzero = any_nonzero || __shfl_xor((int)any_nonzero, 32, kWave) != 0;
  }
  float best = -INFINITY;
  int at = 0;   // material index without the lane group's 4 g
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    if ((mt + 1) * kScoreTileM > K) {   // uniform: the tile has places beyond K
#pragma unroll
      for (int r = 16 * mt; r < min(16 * mt + 16, kRows); ++r)
        if (material(r) >= K) acc[mt][r & 15] = -INFINITY;
    }
#pragma unroll
    for (int r = 16 * mt; r < min(16 * mt + 16, kRows); ++r)   // ascending material index within the lane: the lowest index wins ties
      if (acc[mt][r & 15] > best) {
        best = acc[mt][r & 15];
        at = 8 * (r >> 2) + (r & 3);
      }
  }
  {
    const HalfPair b = half_pair(best), i = half_pair(__int_as_float(at + 4 * g));
    const int lo = __float_as_int(i.lo), hi = __float_as_int(i.hi);
    const bool first = b.lo > b.hi || (b.lo == b.hi && lo < hi);
    best = fmaxf(b.lo, b.hi);
    if (label && store && g == 0) label[n] = first ? lo : hi;
  }
  if (!prop) return;
  float den = 0.0f;
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    const float e = weight_exp((acc[r >> 4][r & 15] - best) * inv_T);
    acc[r >> 4][r & 15] = e;
    den += e;
  }
  const HalfPair d = half_pair(den);
  den = d.lo + d.hi;
  const scores_f32x4* __restrict__ yv = reinterpret_cast<const scores_f32x4*>(ys) + g;
  for (int p = 0; p < P; ++p, yv += kScoreTileM * MT / 4) {
    float num = 0.0f;
#pragma unroll
    for (int q = 0; q < QUADS; ++q) {
      const scores_f32x4 v = yv[2 * q];
#pragma unroll
      for (int e = 0; e < 4; ++e) num = __builtin_fmaf(acc[q >> 2][4 * (q & 3) + e], v[e], num);
    }
    const HalfPair s = half_pair(num);
    if (store && g == 0) prop[n * P + p] = unseen_zero && !any_nonzero ? 0.0f : (s.lo + s.hi) / den;
  }
}

// Stores the scores of the lane's point as they are, then label and Eq. 4.  All 64 lanes call this; those whose point does not exist
// with store == false.
template <int MT>
__device__ __forceinline__ void finish_scores(scores_f32x16 (&acc)[MT], long long n, bool store, int g, int K, int P, float inv_T,
                                              const float* __restrict__ ys, float* __restrict__ scores,
                                              float* __restrict__ prop, int* __restrict__ label, bool unseen_zero = false) {
  float* __restrict__ srow = scores + n * K;
  const bool vec_store = (K & 3) == 0 && ((reinterpret_cast<uintptr_t>(scores) & 15) == 0);
  if (store) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m0 = mt * kScoreTileM + 8 * q + 4 * g;
        if (vec_store) {
          if (m0 < K) {
            scores_f32x4 v = {acc[mt][4 * q], acc[mt][4 * q + 1], acc[mt][4 * q + 2], acc[mt][4 * q + 3]};
            *reinterpret_cast<scores_f32x4*>(srow + m0) = v;
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (m0 + e < K) srow[m0 + e] = acc[mt][4 * q + e];
        }
      }
  }
  finish_quads<MT, 4 * MT>(acc, n, store, g, K, P, inv_T, ys, prop, label, unseen_zero);
}

// The same for a whole wave whose 32 points are consecutive in memory (n0 .. n0 + rows - 1 exist), with the scores
// going through a small LDS buffer of the wave's own (kScoreStageFloats floats) so that they reach memory in long runs:
// in the accumulator layout a store instruction writes 32 bytes of each of 32 rows, and those partial-line writes cost
// the scoring kernels up to a fifth of their time (6.4 M points x 24 materials: 0.53 of 2.9 ms).  ROWS rows at a time
// (16, or 8 where LDS is short) are laid out as [row][material] in the buffer and copied out sixteen bytes per lane,
// eight neighbouring lanes per row; four bytes per lane where K is no multiple of four.  All 64 lanes call this, also those whose
// point does not exist.
constexpr int kScoreStagePitch = 36;   // floats: rows start 4 banks apart
template <int ROWS>
constexpr int score_stage_floats() { return ROWS * kScoreStagePitch; }

// SHORT: up to 16 materials fill half of the only tile's places, and label and Eq. 4 go over those alone.  Over all of them the step
// of 20 000 points, 512 fp32 channels and 12 materials had become slower than with a branch per material (57.5 -> 58.2 us, 55.9 now),
// 117 371 queries densified with 6 materials 67.6 -> 68.3 (67.9).  Same bits.  Only where these lines are the end of a
// wave with few others beside it: in k_tile_scores the second copy of them costs more than it saves (6.4 M points and 24 materials 143
// -> 150 us), in the scoring wave of k_tile_fused too (step of 200 000 points and 32 materials 220.2 -> 221.5).
template <int MT, int ROWS, bool SHORT = false>
__device__ __forceinline__ void finish_scores_staged(scores_f32x16 (&acc)[MT], long long n0, int rows, int lane, int K,
                                                     int P, float inv_T, const float* __restrict__ ys,
                                                     float* __restrict__ scores, float* __restrict__ prop,
                                                     int* __restrict__ label, bool unseen_zero, float* stage) {
  const int pt = lane & 31, g = lane >> 5;
  const bool vec = (K & 3) == 0 && ((reinterpret_cast<uintptr_t>(scores) & 15) == 0);   // 16 bytes per lane, else four
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int cols = min(kScoreTileM, K - mt * kScoreTileM);
    if (cols <= 0) continue;                                    // uniform
    // pieces of a row: cols / 4 vectors or cols floats; idx / per_row by a multiplication, exact for idx < 512 and per_row <= 32
    const int per_row = vec ? cols >> 2 : cols;
    const uint32_t inv = 65536u / (uint32_t)per_row + 1u;
#pragma unroll
    for (int part = 0; part < 32 / ROWS; ++part) {
      if (pt / ROWS == part) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<scores_f32x4*>(stage + (pt % ROWS) * kScoreStagePitch + 8 * q + 4 * g) =
              scores_f32x4{acc[mt][4 * q], acc[mt][4 * q + 1], acc[mt][4 * q + 2], acc[mt][4 * q + 3]};
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const int here = min(ROWS, rows - part * ROWS) * per_row;   // pieces of the rows that exist
      float* __restrict__ out = scores + (n0 + part * ROWS) * K + mt * kScoreTileM;
      if (vec) {
        for (int idx = lane; idx < here; idx += kWave) {
          const int r = (int)((uint32_t)idx * inv >> 16), c4 = idx - r * per_row;
          *reinterpret_cast<scores_f32x4*>(out + (long long)r * K + 4 * c4) =
              *reinterpret_cast<const scores_f32x4*>(stage + r * kScoreStagePitch + 4 * c4);
        }
      } else {
        for (int idx = lane; idx < here; idx += kWave) {
          const int r = (int)((uint32_t)idx * inv >> 16), c = idx - r * per_row;
          out[(long long)r * K + c] = stage[r * kScoreStagePitch + c];
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
  const long long n = n0 + (pt < rows ? pt : 0);
  if (SHORT && MT == 1 && K <= 16) finish_quads<MT, 2>(acc, n, pt < rows, g, K, P, inv_T, ys, prop, label, unseen_zero);   // uniform
  else finish_quads<MT, 4 * MT>(acc, n, pt < rows, g, K, P, inv_T, ys, prop, label, unseen_zero);
}

// Eq. 4 on equal similarities, for a point that no view sees: the epilogue's sums in its order with every weight 1, hence its bits (or
// zeros, with unseen_zero).  By one wave; out holds kScoreMaxP values, in LDS.
__device__ __forceinline__ void unseen_properties(int K, int P, const float* __restrict__ y, bool unseen_zero, int lane, float* out) {
  const int g = lane >> 5;
  float den = 0.0f, num[kScoreMaxP];
#pragma unroll
  for (int p = 0; p < kScoreMaxP; ++p) num[p] = 0.0f;
  for (int mt = 0; mt * kScoreTileM < K; ++mt)
    for (int r = 0; r < 16; ++r) {
      const int m = mt * kScoreTileM + 8 * (r >> 2) + 4 * g + (r & 3);
      if (m < K) {
        den += 1.0f;
#pragma unroll
        for (int p = 0; p < kScoreMaxP; ++p)
          if (p < P) num[p] = __builtin_fmaf(1.0f, y[m * P + p], num[p]);
      }
    }
  den += __shfl_xor(den, 32, kWave);
#pragma unroll
  for (int p = 0; p < kScoreMaxP; ++p) {
    const float t = num[p] + __shfl_xor(num[p], 32, kWave);
    if (lane == 0) out[p] = unseen_zero ? 0.0f : t / den;
  }
}

// What finish_scores_staged writes for 32 consecutive points whose similarities are all exactly +0 (a tile that no view
// sees), without its exponentials: scores 0, label 0, and the properties Eq. 4 gives for equal similarities - the same
// sums in the same order (every weight is exp(0 * inv_T) = 1, so a fused multiply-add by it is an addition), hence the
// same bits - or zeros with unseen_zero.  All 64 lanes call this; the caller has checked that 0 * inv_T is 0.
template <int MT>
__device__ __forceinline__ void finish_zero_rows(long long n0, int rows, int lane, int K, int P, const float* __restrict__ ys,
                                                 float* __restrict__ scores, float* __restrict__ prop, int* __restrict__ label,
                                                 bool unseen_zero) {
  const int pt = lane & 31, g = lane >> 5;
  float* __restrict__ base = scores + n0 * K;
  const long long total = (long long)rows * K;
  if ((K & 3) == 0 && ((reinterpret_cast<uintptr_t>(base) & 15) == 0)) {
    for (long long i = 4 * lane; i < total; i += 4 * kWave) *reinterpret_cast<scores_f32x4*>(base + i) = scores_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  } else {
    for (long long i = lane; i < total; i += kWave) base[i] = 0.0f;
  }
  if (label && g == 0 && pt < rows) label[n0 + pt] = 0;
  if (!prop) return;
  float den = 0.0f, num[kScoreMaxP];
#pragma unroll
  for (int p = 0; p < kScoreMaxP; ++p) num[p] = 0.0f;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = mt * kScoreTileM + 8 * (r / 4) + 4 * g + (r & 3);
      if (m < K) {
        den += 1.0f;
#pragma unroll
        for (int p = 0; p < kScoreMaxP; ++p)
          if (p < P) num[p] = __builtin_fmaf(1.0f, ys[p * kScoreTileM * MT + m], num[p]);
      }
    }
  den += __shfl_xor(den, 32, kWave);
#pragma unroll
  for (int p = 0; p < kScoreMaxP; ++p) {
    if (p < P) {
      const float t = num[p] + __shfl_xor(num[p], 32, kWave);
      if (g == 0 && pt < rows) prop[(n0 + pt) * P + p] = unseen_zero ? 0.0f : t / den;
    }
  }
}

}  // namespace aura
