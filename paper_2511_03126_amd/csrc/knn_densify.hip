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
#include <type_traits>

#include "aura_device.hpp"
#include "launch.hpp"
#include "scores_core.hpp"
#include "scores_epilogue.hpp"

namespace aura {

typedef float sc_f32x2 __attribute__((ext_vector_type(2)));

constexpr int kKnnMaxK = 16;       // neighbours per query
constexpr int kKnnMaxSources = 256;
constexpr int kKnnWaves = 4;       // per workgroup; those of one wait for each other at every half step, those of others fill the gaps
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

// From memory straight to LDS: 16 (4) bytes per lane, from base + off to lds + 16 (4) * lane.  (m0 holds the place in LDS.)
template <int BYTES>
__device__ __forceinline__ void copy_lanes(const void* base, uint32_t off, const void* lds) {
  const uint32_t at = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)lds);
  uint32_t saved_m0;
  if constexpr (BYTES == 16)
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b32 m0, %0"
                 : "=&s"(saved_m0) : "s"(at), "v"(off), "s"(base) : "memory");
  else
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %2, %3\n\ts_mov_b32 m0, %0"
                 : "=&s"(saved_m0) : "s"(at), "v"(off), "s"(base) : "memory");
}

// The same four times, 16 bytes per lane, 1 KiB apart in LDS.
__device__ __forceinline__ void copy_four(const void* base, const uint32_t (&off)[4], const void* lds) {
  const uint32_t at = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)lds);
  uint32_t saved_m0;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %6\n\t"
               "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %3, %6\n\t"
               "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %4, %6\n\t"
               "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %5, %6\n\ts_mov_b32 m0, %0"
               : "=&s"(saved_m0) : "s"(at), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base) : "memory", "scc");
}

// The contraction of scores_core.hpp, rows and split source features (they are as many bytes as the rows of 160 queries, and every
// wave needs all of them) on their way to the matrix cores through LDS, where copy_lanes puts them: whole 128-byte lines, no
// registers while they are on their way, hence three waves per SIMD beside the
// accumulators (with 512 bytes of LDS too many for the third workgroup, and the bank conflicts of unpadded material vectors, the call of
// 200 000 queries took 282 us; without either 227).
//
// A step is 32 channels, in two halves of 16.  A wave's rows of a step are 4 KiB of its own, two steps deep; the sources of a half
// are MT * 2 KiB for the whole workgroup, two halves deep.  At the top of a half, one barrier: this half's sources have arrived, and
// nobody reads those of the half before it any more, so the next ones are requested into their place; the rows of the step after next
// are requested as soon as this step's are in registers.  Requests return in order: a half waits for what it needs, and the rows
// requested last stay on their way (two halves, as long as the memory takes at its full rate).
// Row n's piece c of a step (16 bytes) lies at place c ^ (n % 8) of the row's 128 bytes: eight neighbouring lanes, which read
// the same piece of eight rows, meet in no bank.
// Needs D to be a multiple of 32 and 16-byte aligned rows (no partial step); all threads of the workgroup must call
// this together; a wave without queries of its own (`work` false, uniform over the wave) only copies its share of the
// sources and passes the barriers.  Nothing is on its way, and nobody reads LDS, when it returns.
// rows: first of the wave's 32 queries; last_row: the last one that exists (from 0; the others read it again).
template <int MT>
__device__ __forceinline__ float score_products_staged(const float* __restrict__ rows, int D, int last_row, int steps,
                                                       const sc_bf16x8* __restrict__ a_split, int wave, int lane,
                                                       char* s_src, char* s_rows, sc_f32x16 (&acc)[MT], bool work) {
  const int n = lane & 31, g = lane / 32;
  float ss = 0.0f;
  uint32_t row_off[4];   // of the lane's part of copy q: row 8 q + lane / 8
#pragma unroll
  for (int q = 0; q < 4; ++q)
    row_off[q] = (uint32_t)min(8 * q + (lane >> 3), last_row) * (uint32_t)D * 4u + (uint32_t)(((lane & 7) ^ (lane >> 3)) * 16);
  auto request_rows = [&](int s) { copy_four(rows + s * kScoreStepK, row_off, s_rows + (s & 1) * 4096); };
  auto request_sources = [&](int s, int j) {
    const char* base = reinterpret_cast<const char*>(a_split) + ((size_t)s * MT * 2 + j) * 2048;
    for (int i = wave; i < 2 * MT; i += kKnnWaves)
      copy_lanes<16>(base + (i >> 1) * 4096 + (i & 1) * 1024, (uint32_t)lane * 16u, s_src + j * MT * 2048 + i * 1024);
  };
  sc_f32x4 r[4];
  auto half = [&](int s, auto jc) {
    constexpr int j = decltype(jc)::value;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (j == 0) request_sources(s, 1);
    else if (s + 1 < steps) request_sources(s + 1, 0);
    if (!work) return;
    if constexpr (j == 0) {
      const char* mine = s_rows + (s & 1) * 4096 + n * 128;
#pragma unroll
      for (int q = 0; q < 4; ++q) r[q] = *reinterpret_cast<const sc_f32x4*>(mine + (((4 * g + q) ^ (n & 7)) * 16));
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]) :: "memory");
      if (s + 2 < steps) request_rows(s + 2);
    }
    sc_bf16x8 bh, bl;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float x = r[2 * j + (e >> 2)][e & 3];
      ss = __builtin_fmaf(x, x, ss);
      const __bf16 h = (__bf16)x;
      bh[e] = h;
      bl[e] = (__bf16)(x - (float)h);
    }
    const sc_bf16x8* src = reinterpret_cast<const sc_bf16x8*>(s_src + j * MT * 2048) + lane;
    // two tiles at a time: their accumulators take turns, so that no product waits for the one before it
#pragma unroll
    for (int m = 0; m < MT; m += 2) {
      const bool two = m + 1 < MT;
      const sc_bf16x8 h0 = src[2 * m * kWave], l0 = src[(2 * m + 1) * kWave];
      const sc_bf16x8 h1 = src[(two ? 2 * m + 2 : 2 * m) * kWave], l1 = src[(two ? 2 * m + 3 : 2 * m + 1) * kWave];
      acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(h0, bh, acc[m], 0, 0, 0);
      if (two) acc[two ? m + 1 : m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(h1, bh, acc[two ? m + 1 : m], 0, 0, 0);
      acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(h0, bl, acc[m], 0, 0, 0);
      if (two) acc[two ? m + 1 : m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(h1, bl, acc[two ? m + 1 : m], 0, 0, 0);
      acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(l0, bh, acc[m], 0, 0, 0);
      if (two) acc[two ? m + 1 : m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(l1, bh, acc[two ? m + 1 : m], 0, 0, 0);
    }
  };
  if (work) request_rows(0);
  request_sources(0, 0);
  if (work && steps > 1) request_rows(1);
  const bool rows_behind = work && steps > 1;
  if (rows_behind) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  for (int s = 0; s < steps; ++s) {   // uniform over the workgroup: every wave passes the same barriers
    half(s, std::integral_constant<int, 0>{});
    if (work && s + 2 < steps) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");   // (the rows of step s + 2 stay on their way)
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    half(s, std::integral_constant<int, 1>{});
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  return ss;
}

// MT: tiles of 32 sources; MTK: tiles of 32 materials.
template <int MT, int MTK, bool ROWS_ALIGNED>
__global__ __launch_bounds__(kKnnWaves * kWave)
    __attribute__((amdgpu_waves_per_eu(knn_waves_per_simd(MT, ROWS_ALIGNED), knn_waves_per_simd(MT, ROWS_ALIGNED))))
void k_knn_densify(KnnArgs a) {
  // While the similarities are made: the sources' places, then the rows'.  Afterwards: the properties of the materials; per wave the
  // winners of its queries, and in their place the score rows on their way to memory; the sources' material vectors, when they fit.
  constexpr int kSrcBytes = ROWS_ALIGNED ? 2 * MT * 2048 : 0, kRowBytes = ROWS_ALIGNED ? 2 * 4096 : 0;
  constexpr int kLdsBytes = knn_lds_bytes(MT, ROWS_ALIGNED);
  static_assert(kSrcBytes + kKnnWaves * kRowBytes <= kLdsBytes);
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

  sc_f32x16 acc[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[mt][r] = 0.0f;
  float ss;
  if constexpr (ROWS_ALIGNED)   // whole macro steps, 16-byte aligned rows: through LDS
    ss = score_products_staged<MT>(a.fq + n0 * a.D, a.D, rows - 1, a.steps, a.a_split, wave, lane, s_mem,
                                   s_mem + kSrcBytes + wave * kRowBytes, acc, active);
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
  const bool aligned = (D & 31) == 0 && (reinterpret_cast<uintptr_t>(fq) & 15) == 0;
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
