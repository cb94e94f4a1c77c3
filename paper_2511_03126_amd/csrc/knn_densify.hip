// aura_knn_densify: Sec. 3.4.1 Eq. 5 - material vectors of dense query points from their k nearest
// source points in feature space (cosine similarity of the fused features), similarity-weighted mean,
// then the kernel regression of Eq. 4 on the interpolated vector.
//
// The similarities of all queries to all sources are one dense contraction [Ns x D] . [D x Nq], done on
// the matrix cores exactly like the material scores (sources on the M side, points on the N side, fp32
// operands as two bf16 terms, three partial products): a lane ends up with half the similarities of ONE
// query, lane l ^ 32 with the other half.  The selection of the k largest is k rounds of "largest value
// left" over the lane's registers plus one exchange with the partner lane (of equal values the lower
// source index first); both lanes of a pair keep the same list, in LDS.  The weighted mean of the neighbours'
// vectors is then evaluated directly in the accumulator layout of the scoring epilogue, which stores it
// and applies Eq. 4.
//
// The source features are divided by their norms before they are split into operand order, so the
// accumulators are <q, s / |s|>: the order of a query's similarities does not depend on its own norm, which
// only scales the weights at the end.
//
// What bounds it: with three waves per SIMD the vector and matrix units are busy for 30 and 33 % of the time and a third of a wave's
// time is waiting for rows and sources, which come at 2.9 TB/s.  200 000 queries, 150 sources, 768 channels, 32 materials, k = 5: 205
// us (before, rows and sources through registers, two waves per SIMD, 271), the whole call 218 (288).  us per call before / now:
// 100 materials 380 / 244 (their sums and the similarities no longer hold registers at the same time), 250 sources 382 / 298, with 120
// materials 531 / 322, 90 sources 256 / 172, 400 000 queries of 1024 channels 569 / 461, 20 000 of 768 60 / 49, 3000 49 / 44.
#include "aura_device.hpp"
#include "launch.hpp"
#include "scores_core.hpp"
#include "scores_epilogue.hpp"
#include "scores_staged.hpp"

namespace aura {

typedef float sc_f32x2 __attribute__((ext_vector_type(2)));

constexpr int kKnnMaxK = 16;       // neighbours per query
constexpr int kKnnMaxSources = 256;
constexpr int kKnnWaves = 4;       // per workgroup; they wait for each other at every half step, those of others fill the gaps
// Waves per SIMD: three where the accumulators of the similarities leave room for the rest in 168 registers.
constexpr int knn_waves_per_simd(int MT, bool aligned) { return aligned && MT <= 5 ? 3 : 2; }
// Bytes of LDS per workgroup: what as many of them as the registers allow can have of 160 KiB (handed out in pieces of 1280 bytes).
// What the similarities need is less for few sources; the rest keeps more material vectors close.
constexpr int knn_lds_bytes(int MT, bool aligned) { return knn_waves_per_simd(MT, aligned) == 3 ? 53760 : 81920; }

struct KnnArgs {
  const float* fq;          // [Nq][D]
  long long Nq;
  int D, Ns, K, P, k;
  const sc_bf16x8* a_split; // split source features
  int steps;
  const float* ws;          // [Ns][K]
  const float* y;
  float inv_T;
  float* wq;                // [Nq][K]
  float* prop;
  int* label;
  int* nn_idx;              // [Nq][k] or nullptr
  long long n_tiles;        // tiles of 32 queries
  int n_ranges;             // contiguous ranges of tiles (see the kernel)
};

// The source features divided by their norms (a zero vector stays zero: similarity 0 to everything), split into
// two bf16 terms in the operand order of scores_core.hpp.  One workgroup per source slot (slots beyond Ns are zero): a
// thread reads the eight neighbouring channels of a piece (step, lane group, half), and writes what the slot's operand lane holds of
// them once the sum of all squares is there; up to 2048 channels are read once.  (One wave per source took a chain of reads: 150 sources
// of 768 channels 12.9 us, now 4.9, which is what any launch takes.)
constexpr int kSplitThreads = 256;
__global__ __launch_bounds__(kSplitThreads) void k_split_sources(const float* __restrict__ fs, int Ns, int D, int MT, int steps,
                                                                 __bf16* __restrict__ out) {
  __shared__ float s_part[kSplitThreads / kWave];
  const int m = blockIdx.x, tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int pieces = steps * 4;
  const float* __restrict__ row = fs + (long long)m * D;
  const bool vec = (D & 3) == 0 && (reinterpret_cast<uintptr_t>(fs) & 15) == 0;   // uniform
  auto load = [&](int piece, float (&x)[8]) {
    const int c = 8 * piece;
    if (m < Ns && vec && c + 8 <= D) {
      const sc_f32x4 u = *reinterpret_cast<const sc_f32x4*>(row + c), v = *reinterpret_cast<const sc_f32x4*>(row + c + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) { x[e] = u[e]; x[4 + e] = v[e]; }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = m < Ns && c + e < D ? row[c + e] : 0.0f;
    }
  };
  float first[8], ss = 0.0f;
  load(tid, first);   // (a piece beyond the last: zeros)
#pragma unroll
  for (int e = 0; e < 8; ++e) ss = __builtin_fmaf(first[e], first[e], ss);
  for (int piece = tid + kSplitThreads; piece < pieces; piece += kSplitThreads) {
    float x[8];
    load(piece, x);
#pragma unroll
    for (int e = 0; e < 8; ++e) ss = __builtin_fmaf(x[e], x[e], ss);
  }
  ss = wave_sum(ss);
  if (lane == 0) s_part[wave] = ss;
  __syncthreads();
  ss = (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]);
  const float scale = ss > 0.0f ? 1.0f / sqrtf(ss) : 0.0f;
  for (int piece = tid; piece < pieces; piece += kSplitThreads) {
    float x[8];
    if (piece == tid) {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = first[e];
    } else {
      load(piece, x);
    }
    const int s = piece >> 2, g = (piece >> 1) & 1, j = piece & 1;   // channels score_chan_of(s, j, g, 0 .. 7)
    sc_bf16x8 hi, lo;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float v = x[e] * scale;
      const __bf16 h = (__bf16)v;
      hi[e] = h;
      lo[e] = (__bf16)(v - (float)h);
    }
    sc_bf16x8* to = reinterpret_cast<sc_bf16x8*>(out) + ((long long)(s * MT + m / 32) * 2 + j) * 2 * kWave + g * 32 + (m & 31);
    to[0] = hi;
    to[kWave] = lo;
  }
}

// MT: tiles of 32 sources; MTK: tiles of 32 materials.
template <int MT, int MTK, bool ROWS_ALIGNED>
__global__ __launch_bounds__(kKnnWaves * kWave)
    __attribute__((amdgpu_waves_per_eu(knn_waves_per_simd(MT, ROWS_ALIGNED), knn_waves_per_simd(MT, ROWS_ALIGNED))))
void k_knn_densify(KnnArgs a) {
  // While the similarities are made: the sources' places, then the rows'.  Afterwards: the properties of the materials; per wave the
  // winners of its queries, and in their place the score rows on their way to memory; the sources' material vectors, when they fit.
  constexpr StagedShape kShape = staged_shape(MT, kKnnWaves, knn_lds_bytes(MT, ROWS_ALIGNED));
  constexpr int kLdsBytes = knn_lds_bytes(MT, ROWS_ALIGNED);
  static_assert(!ROWS_ALIGNED || staged_bytes(MT, kShape) <= kLdsBytes);
  __shared__ __attribute__((aligned(1024))) char s_mem[kLdsBytes];
  const int pick_floats = max(64 * min(a.k, a.Ns), score_stage_floats<16>());
  float* const ys = reinterpret_cast<float*>(s_mem);
  float* const s_pick = ys + kScoreTileM * MTK * kScoreMaxP;
  float* const s_ws = s_pick + kKnnWaves * pick_floats;
  const int ws_floats = kLdsBytes / 4 - kScoreTileM * MTK * kScoreMaxP - kKnnWaves * pick_floats;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int g = lane / 32;
  const int ke = min(a.k, a.Ns);
  // The tiles are divided evenly into a.n_ranges contiguous ranges (one per compute unit), and workgroup b takes the
  // (b / n_ranges)-th four tiles of range b % n_ranges: all workgroups but a range's last are full, and the ranges'
  // last workgroups, with few waves each, run side by side at the end, instead of a few full workgroups running
  // alone after all the others.
  const int range = blockIdx.x % a.n_ranges;
  const long long t0 = a.n_tiles * range / a.n_ranges + (long long)(blockIdx.x / a.n_ranges) * kKnnWaves;
  const long long t_end = a.n_tiles * (range + 1) / a.n_ranges;
  if (t0 >= t_end) return;   // uniform over the workgroup, before its first barrier
  const long long tile = t0 + wave;
  const bool active = tile < t_end;                    // a wave without a tile still takes part in the staging
  const long long n0 = active ? tile * 32 : 0;
  const int rows = (int)min((long long)32, a.Nq - n0);
  const long long n = n0 + (lane & 31);
  const bool valid = active && (lane & 31) < rows;

  ScoreSums<MT, TermB> sum;
  sc_f32x16 (&acc)[MT] = sum.acc;
  float ss;
  if constexpr (ROWS_ALIGNED)   // whole macro steps, 16-byte aligned rows: through LDS
    ss = score_products_staged<MT, TermB, true, kKnnWaves, kShape.rows, kShape.sources>(a.fq + n0 * a.D, a.D, rows - 1, a.steps, a.a_split,
                                                                             wave, lane, s_mem, sum, active);
  else
    ss = score_products<MT, false, true>(a.fq + (valid ? n : a.Nq - 1) * a.D, a.D, a.steps, a.a_split, lane, acc);
  ss += __shfl_xor(ss, 32, kWave);
  const float q_inv = ss > 0.0f ? 1.0f / sqrtf(ss) : 0.0f;
  // The vectors of the sources, `pitch` floats apart: a multiple of four, so that a lane's four neighbouring materials are one read, and
  // an odd one, so that the vectors begin in different banks (32 materials back to back: 64 % of the LDS unit's time were conflicts).
  const int pitch = 4 * (((a.K + 3) >> 2) | 1);
  const bool ws_in_lds = a.Ns * pitch <= ws_floats;   // uniform
  if (ws_in_lds) {
    for (int j = wave; j < a.Ns; j += kKnnWaves)
      for (int m = lane; m < a.K; m += kWave) copy_lanes<4>(a.ws + (long long)j * a.K + (m - lane), 4u * lane, s_ws + j * pitch + (m - lane));
  }
  if (a.prop) stage_properties<MTK>(ys, a.y, a.K, a.P, threadIdx.x, blockDim.x);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  // Slots beyond Ns can never be selected (they can only be in the last two tiles: MT = ceil(Ns / 32), or 8 for 7).
#pragma unroll
  for (int mt = (MT > 2 ? MT - 2 : 0); mt < MT; ++mt)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int j = mt * 32 + 8 * (r >> 2) + 4 * g + (r & 3);
      if (j >= a.Ns) acc[mt][r] = -INFINITY;
    }

  if (!active) return;   // no barrier below; only LDS of the wave's own (its part of s_out) and what was filled before the loop

  // ---- the k nearest sources, in order.  The accumulators are <q, s/|s|>, the cosine
  // similarities times |q|: the same order.  A round scans the lane's values in four independent chains (each in
  // ascending source index, so the first of equal values stays; a single chain is one long run of dependent
  // instructions), merges them, and exchanges with the partner lane; both lanes of a pair find the same winner, which waits in
  // LDS with its weight until the similarities' registers are free for Eq. 5.
  sc_f32x2* const pick = reinterpret_cast<sc_f32x2*>(s_pick + wave * pick_floats) + (lane & 31);   // round t: pick[32 t]
  float den = 0.0f;
#pragma unroll 1
  for (int t = 0; t < ke; ++t) {
    float cb[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    int cj[4] = {0x7fffffff, 0x7fffffff, 0x7fffffff, 0x7fffffff};   // source index without the lane group's 4 g: a constant per element
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (acc[mt][r] > cb[r & 3]) { cb[r & 3] = acc[mt][r]; cj[r & 3] = mt * 32 + 8 * (r >> 2) + (r & 3); }
    auto merge = [](float& v, int& j, float ov, int oj) {   // larger value; of equal values the lower index
      if (ov > v || (ov == v && oj < j)) { v = ov; j = oj; }
    };
    merge(cb[0], cj[0], cb[1], cj[1]);
    merge(cb[2], cj[2], cb[3], cj[3]);
    merge(cb[0], cj[0], cb[2], cj[2]);
    float best = cb[0];
    int bj = cj[0] == 0x7fffffff ? cj[0] : cj[0] + 4 * g;
    merge(best, bj, __shfl_xor(best, 32, kWave), __shfl_xor(bj, 32, kWave));
    // Nothing compares greater when every similarity left is NaN (a NaN in the features): the round must still name
    // a source, because it addresses the sources' vectors.
    if ((unsigned)bj >= (unsigned)a.Ns) { bj = 0; best = 0.0f; }
    const float phi = best * q_inv;   // the cosine similarity
    den += phi;
    if (g == 0) pick[32 * t] = sc_f32x2{phi, __int_as_float(bj)};
    if (a.nn_idx && g == 0 && valid) a.nn_idx[n * a.k + t] = bj;
    const int bj_lane = bj - 4 * g;   // the winner's index as this lane's elements count
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (mt * 32 + 8 * (r >> 2) + (r & 3) == bj_lane) acc[mt][r] = -INFINITY;
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();

  // ---- Eq. 5 in the layout of the scoring epilogue: element r of tile mt is material mt*32 + 8*(r/4) + 4*g + r%4; a material index
  // beyond K reads the last material (in LDS: the last four) instead, into an element that the epilogue never looks at.
  const int k_last = a.K - 1;
  const bool ws_quads = (a.K & 3) == 0 && (reinterpret_cast<uintptr_t>(a.ws) & 15) == 0;
  auto read_vector = [&](int j, int mt, float (&v)[16]) {
    int kl = k_last;
    asm volatile("" : "+v"(kl));   // the clamped material indices are made again every time instead of living in 16 registers per tile
    if (ws_in_lds) {   // uniform.  (Two branches, so that the reads of the LDS copy are LDS instructions and not generic ones.)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const sc_f32x4 u = *reinterpret_cast<const sc_f32x4*>(s_ws + j * pitch + 4 * min(mt * 8 + 2 * q + g, kl >> 2));
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * q + e] = u[e];
      }
    } else if (ws_quads) {   // uniform
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const sc_f32x4 u = *reinterpret_cast<const sc_f32x4*>(a.ws + (long long)j * a.K + 4 * min(mt * 8 + 2 * q + g, kl >> 2));
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * q + e] = u[e];
      }
    } else {
      const float* __restrict__ src = a.ws + (long long)j * a.K;
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] = src[min(mt * 32 + 8 * (r >> 2) + 4 * g + (r & 3), kl)];
    }
  };
  sc_f32x16 out[MTK];
#pragma unroll
  for (int mt = 0; mt < MTK; ++mt)
#pragma unroll
    for (int r = 0; r < 16; ++r) out[mt][r] = 0.0f;
  sc_f32x2 next = pick[0];
  const int nearest = __float_as_int(next[1]);
#pragma unroll 1
  for (int t = 0; t < ke; ++t) {
    const float phi = next[0];
    const int bj = __float_as_int(next[1]);
    next = pick[32 * min(t + 1, ke - 1)];
#pragma unroll
    for (int mt = 0; mt < MTK; ++mt) {
      float v[16];
      read_vector(bj, mt, v);
#pragma unroll
      for (int r = 0; r < 16; ++r) out[mt][r] = __builtin_fmaf(phi, v[r], out[mt][r]);
    }
  }
  if (a.nn_idx && g == 0 && valid) {
    for (int t = ke; t < a.k; ++t) a.nn_idx[n * a.k + t] = -1;
  }
  if (fabsf(den) < 1e-12f) {   // no usable weights (a query without features, for one): the nearest source's vector
#pragma unroll
    for (int mt = 0; mt < MTK; ++mt) {
      float v[16];
      read_vector(nearest, mt, v);
#pragma unroll
      for (int r = 0; r < 16; ++r) out[mt][r] = v[r];
    }
  } else {
    const float inv_den = 1.0f / den;
#pragma unroll
    for (int mt = 0; mt < MTK; ++mt)
#pragma unroll
      for (int r = 0; r < 16; ++r) out[mt][r] *= inv_den;
  }
  finish_scores_staged<MTK, 16, true>(out, n0, rows, lane, a.K, a.P, a.inv_T, ys, a.wq, a.prop, a.label, false,
                                  s_pick + wave * pick_floats);
}

// ------------------------------------------------------------------------------------ host

static size_t knn_round256(size_t x) { return (x + 255) & ~(size_t)255; }
static int knn_source_tiles(int Ns) {
  const int mt = (Ns + 31) / 32;
  return mt <= 6 ? mt : 8;
}

bool knn_supported(int Ns, int K, int k, int P) {
  return Ns >= 1 && Ns <= kKnnMaxSources && K >= 1 && K <= kScoreMaxK && k >= 1 && k <= kKnnMaxK && P >= 0 && P <= kScoreMaxP;
}

size_t knn_workspace_bytes(int D, int Ns) {
  return knn_round256(split_embeddings_bytes(D, knn_source_tiles(Ns))) + knn_round256((size_t)Ns * sizeof(float));
}

template <int MT, int MTK>
static hipError_t launch_knn(const KnnArgs& a, bool aligned, hipStream_t stream) {
  int dev = 0, cus = 256;
  if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  KnnArgs b = a;
  b.n_ranges = (int)(a.n_tiles < cus ? a.n_tiles : cus);
  const long long longest = (a.n_tiles + b.n_ranges - 1) / b.n_ranges;   // tiles of the longest range
  const dim3 grid((unsigned)(((longest + kKnnWaves - 1) / kKnnWaves) * b.n_ranges)), block(kKnnWaves * kWave);
  if (aligned)
    hipLaunchKernelGGL((k_knn_densify<MT, MTK, true>), grid, block, 0, stream, b);
  else
    hipLaunchKernelGGL((k_knn_densify<MT, MTK, false>), grid, block, 0, stream, b);
  return hipGetLastError();
}

template <int MT>
static hipError_t launch_knn_mtk(const KnnArgs& a, bool aligned, hipStream_t stream) {
  const int mtk = (a.K + 31) / 32;
  if (mtk <= 1) return launch_knn<MT, 1>(a, aligned, stream);
  if (mtk == 2) return launch_knn<MT, 2>(a, aligned, stream);
  return launch_knn<MT, 4>(a, aligned, stream);
}

hipError_t launch_knn_densify(const float* fq, long long Nq, int D, const float* fs, int Ns, const float* ws, int K,
                              int k, const float* y, int P, float temperature, float* wq, float* prop, int* label,
                              int* nn_idx, void* workspace, hipStream_t stream) {
  if (Nq == 0) return hipSuccess;
  const int MT = knn_source_tiles(Ns);
  char* base = static_cast<char*>(workspace);
  void* split = base;
  const int steps = (D + kScoreStepK - 1) / kScoreStepK;
  hipLaunchKernelGGL(k_split_sources, dim3((unsigned)(MT * 32)), dim3(kSplitThreads), 0, stream, fs, Ns, D, MT, steps,
                     static_cast<__bf16*>(split));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  KnnArgs a{fq, Nq, D, Ns, K, P, k, static_cast<const sc_bf16x8*>(split), steps, ws,
            y, inverse_temperature(temperature), wq, prop, label, nn_idx, (Nq + 31) / 32, 1};
  // (through LDS a row's place among a wave's 32 is 32 bits wide: score_products_staged)
  const bool aligned = (D & 31) == 0 && D <= kStagedChannels && (reinterpret_cast<uintptr_t>(fq) & 15) == 0;
  switch (MT) {
    case 1: return launch_knn_mtk<1>(a, aligned, stream);
    case 2: return launch_knn_mtk<2>(a, aligned, stream);
    case 3: return launch_knn_mtk<3>(a, aligned, stream);
    case 4: return launch_knn_mtk<4>(a, aligned, stream);
    case 5: return launch_knn_mtk<5>(a, aligned, stream);
    case 6: return launch_knn_mtk<6>(a, aligned, stream);
    default: return launch_knn_mtk<8>(a, aligned, stream);
  }
}

}  // namespace aura
