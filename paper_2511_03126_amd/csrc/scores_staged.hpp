// The contraction of scores_core.hpp with both operands on their way through LDS.
#pragma once

#include <type_traits>

#include "scores_core.hpp"

namespace aura {

// How far ahead: steps of a wave's rows, and halves of a step's sources (or embeddings), that have a place in LDS; waves: of a workgroup.
struct StagedShape { int waves, rows, sources; };
constexpr int staged_source_bytes(int MT, StagedShape d) { return d.sources * MT * 2048; }
constexpr int staged_bytes(int MT, StagedShape d) { return staged_source_bytes(MT, d) + d.waves * d.rows * 4096; }
// Two steps of rows, and as many halves of sources as `bytes` then hold, up to four.
constexpr StagedShape staged_shape(int MT, int waves, int bytes) {
  const int halves = (bytes - 2 * 4096 * waves) / (MT * 2048);
  return StagedShape{waves, 2, halves < 4 ? halves : 4};
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

template <int N>
__device__ __forceinline__ void wait_requests() { asm volatile("s_waitcnt vmcnt(%0)" :: "i"(N) : "memory"); }

// Channels up to which the 32 rows of a wave end within 4 GiB.
constexpr int kStagedChannels = 1 << 25;

// The contraction of scores_core.hpp, rows and split source features (they are as many bytes as the rows of 160 queries, and every
// wave needs all of them) on their way to the matrix cores through LDS, where copy_lanes puts them: whole 128-byte lines, no
// registers while they are on their way, hence more waves per SIMD beside the accumulators.
//
// A step is 32 channels, in two halves of 16.  A wave's rows of a step are 4 KiB of its own; the sources of a half are MT * 2 KiB for
// the whole workgroup.  At the top of a half, one barrier: this half's sources have arrived, and nobody reads those of the half before
// it any more, so those of DS - 1 halves later are requested into their place; the rows of DR steps later are requested as soon as
// this step's are in registers.  Requests return in order: a half waits for what it needs, and what was requested behind that stays
// on its way.
// Row n's piece c of a step (16 bytes) lies at place c ^ (n % 8) of the row's 128 bytes: eight neighbouring lanes, which read
// the same piece of eight rows, meet in no bank.
// Needs D to be a multiple of 32, up to kStagedChannels, and 16-byte aligned rows (no partial step); all threads of the workgroup must call
// this together; a wave without queries of its own (`work` false, uniform over the wave) only copies its share of the
// sources and passes the barriers.  Nothing is on its way, and nobody reads LDS, when it returns.
// rows: first of the wave's 32 queries; last_row: the last one that exists (from 0; the others read it again).
template <int MT, typename T, bool WANT_SS, int WAVES, int DR, int DS>
__device__ __forceinline__ float score_products_staged(const float* __restrict__ rows, int D, int last_row, int steps,
                                                       const void* __restrict__ a_split, int wave, int lane,
                                                       char* s_mem, ScoreSums<MT, T>& sum, bool work) {
  constexpr StagedShape kShape{WAVES, DR, DS};
  char* const s_src = s_mem;
  char* const s_rows = s_mem + staged_source_bytes(MT, kShape) + wave * (DR * 4096);
  const int n = lane & 31, g = lane / 32;
  float ss = 0.0f;
  uint32_t row_off[4];   // of the lane's part of copy q: row 8 q + lane / 8
#pragma unroll
  for (int q = 0; q < 4; ++q)
    row_off[q] = (uint32_t)min(8 * q + (lane >> 3), last_row) * (uint32_t)D * 4u + (uint32_t)(((lane & 7) ^ (lane >> 3)) * 16);
  const int halves = 2 * steps;
  auto request_rows = [&](int s) { copy_four(rows + s * kScoreStepK, row_off, s_rows + (s % DR) * 4096); };
  auto request_sources = [&](int h) {
    const char* base = reinterpret_cast<const char*>(a_split) + ((size_t)(h >> 1) * MT * 2 + (h & 1)) * 2048;
    char* to = s_src + (h % DS) * MT * 2048;
    for (int i = wave; i < 2 * MT; i += WAVES) copy_lanes<16>(base + (i >> 1) * 4096 + (i & 1) * 1024, (uint32_t)lane * 16u, to + i * 1024);
  };
  // Waits for this half's sources and, of an even half, the step's rows.  What may stay on its way: the sources of the DS - 2 halves
  // behind this one, and the rows that were requested in the halves since (after the sources, in even halves).
  constexpr int kFew = 2 * MT / WAVES, kMore = 2 * MT % WAVES;   // copies of a wave per half: one more for the first kMore waves
  auto wait_half = [&](int h, auto jc) {
    constexpr int j = decltype(jc)::value;
    // even halves from h - DS + 1 (that one's rows were requested after its sources) to h - 1
    constexpr int kRowRequests = (DS - 1 + j) / 2;
    static_assert(DS >= 2 && DR >= kRowRequests + 1 - j && (DS - 2) * (kFew + 1) + 4 * kRowRequests < 64);
    if (h + 2 * DR > halves || h + DS > halves) {   // less was requested towards the end
      wait_requests<0>();
    } else if (h < DS - 1) {   // sources from before the loop, and the rows of the steps behind it
      if (work) wait_requests<4 * (DR - 1)>();
      else wait_requests<0>();
    } else if (!work) {
      if (wave < kMore) wait_requests<(DS - 2) * (kFew + 1)>();
      else wait_requests<(DS - 2) * kFew>();
    } else {
      if (wave < kMore) wait_requests<(DS - 2) * (kFew + 1) + 4 * kRowRequests>();
      else wait_requests<(DS - 2) * kFew + 4 * kRowRequests>();
    }
  };
  sc_f32x4 r[4];
  auto half = [&](int s, auto jc) {
    constexpr int j = decltype(jc)::value;
    const int h = 2 * s + j;
    wait_half(h, jc);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (h + DS - 1 < halves) request_sources(h + DS - 1);
    if (!work) return;
    if constexpr (j == 0) {
      const char* mine = s_rows + (s % DR) * 4096 + n * 128;
#pragma unroll
      for (int q = 0; q < 4; ++q) r[q] = *reinterpret_cast<const sc_f32x4*>(mine + (((4 * g + q) ^ (n & 7)) * 16));
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]) :: "memory");
      if (s + DR < steps) request_rows(s + DR);
    }
    Term8<T> bh, bl;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float x = r[2 * j + (e >> 2)][e & 3];
      if (WANT_SS) ss = __builtin_fmaf(x, x, ss);
      T h, l;
      split_terms<T>(x, h, l);
      bh[e] = h;
      bl[e] = l;
    }
    const Term8<T>* src = reinterpret_cast<const Term8<T>*>(s_src + (h % DS) * MT * 2048) + lane;
    // two tiles at a time: their accumulators take turns, so that no product waits for the one before it
#pragma unroll
    for (int m = 0; m < MT; m += 2) {
      constexpr int kLast = MT - 1;
      const bool two = m < kLast;
      const int m1 = two ? m + 1 : m;
      const Term8<T> h0 = src[2 * m * kWave], l0 = src[(2 * m + 1) * kWave], h1 = src[2 * m1 * kWave], l1 = src[(2 * m1 + 1) * kWave];
      sum.acc[m] = score_mma(h0, bh, sum.acc[m]);
      if (two) sum.acc[m1] = score_mma(h1, bh, sum.acc[m1]);
      sum.low(m) = score_mma(h0, bl, sum.low(m));
      if (two) sum.low(m1) = score_mma(h1, bl, sum.low(m1));
      sum.low(m) = score_mma(l0, bh, sum.low(m));
      if (two) sum.low(m1) = score_mma(l1, bh, sum.low(m1));
    }
  };
  if (work) request_rows(0);
#pragma unroll
  for (int h = 0; h < DS - 1; ++h)
    if (h < halves) request_sources(h);
  if (work) {
#pragma unroll
    for (int s = 1; s < DR; ++s)
      if (s < steps) request_rows(s);
  }
  for (int s = 0; s < steps; ++s) {   // uniform over the workgroup: every wave passes the same barriers
    half(s, std::integral_constant<int, 0>{});
    half(s, std::integral_constant<int, 1>{});
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  return ss;
}

}  // namespace aura
