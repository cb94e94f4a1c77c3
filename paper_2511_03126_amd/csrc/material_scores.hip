// aura_material_scores: Sec. 3.4.1 - similarity omega_k = <fused, temb_k> and the kernel
// regression of Eq. 4, plus the arg-max material label.
//
// The contraction [K x D] . [D x N] runs on the matrix cores (v_mfma_f32_32x32x16_bf16) with the
// materials on the M side and the points on the N side, so that one lane ends up holding half of
// the scores of ONE point: the softmax over materials is then an in-register reduction plus a
// single exchange between lane l and lane l ^ 32.  fp32 operands are split into two bf16 terms
// (x = hi + lo) and three partial products hi*hi + hi*lo + lo*hi are accumulated in fp32, which
// keeps the error of a score of unit vectors near 1e-6.
//
// The kernel is bound by reading fused[N][D] once from HBM (arithmetic intensity 2K/(4+4K/D)
// flop per byte, far below the machine balance): the matrix cores are the right instruction,
// not the bound.  The text embeddings are split once per call by a small preparation kernel into
// the workspace, already in the per-lane operand order, and stay resident in L2.
#include <algorithm>
#include <type_traits>

#include "aura_device.hpp"
#include "launch.hpp"
#include "scores_core.hpp"
#include "scores_epilogue.hpp"
#include "scores_staged.hpp"

namespace aura {

typedef sc_bf16x8 bf16x8;
typedef sc_f32x4 f32x4;
typedef sc_f32x16 f32x16;

constexpr int kTileM = 32;      // materials per MFMA tile
constexpr int kTileN = 32;      // points per wave
constexpr int kStepK = 32;      // channels per macro step: lane group g = lane / 32 owns 16 of them
constexpr int kMaxP = 8;

struct ScoreArgs {
  const float* fused;
  long long N;
  int D, K, P;
  const float* y;
  float inv_T;
  int unseen_zero;
  float* scores;
  float* prop;
  int* label;
  const bf16x8* a_split;   // workspace: [S][MT][2 (j)][2 (hi, lo)][64 lanes] x 8 terms (bf16, or fp16 where the kernel says)
  int steps;               // S = ceil(D / 32)
};

template <typename T>
__global__ __launch_bounds__(256) void k_split_embeddings(const float* __restrict__ temb, int K, int D, int MT,
                                                          int steps, T* __restrict__ out) {
  long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;   // one thread per (slot, lane)
  long long total = (long long)steps * MT * 2 * kWave;
  if (t >= total) return;
  int lane = t % kWave;
  int j = (t / kWave) % 2;
  int mt = (t / (kWave * 2)) % MT;
  int s = t / ((long long)kWave * 2 * MT);
  int m = mt * kTileM + lane % 32, g = lane / 32;
  T* hi = out + ((((long long)(s * MT + mt) * 2 + j) * 2 + 0) * kWave + lane) * 8;
  T* lo = out + ((((long long)(s * MT + mt) * 2 + j) * 2 + 1) * kWave + lane) * 8;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    int c = score_chan_of(s, j, g, e);
    float x = (m < K && c < D) ? temb[(long long)m * D + c] : 0.0f;
    split_terms<T>(x, hi[e], lo[e]);
  }
}

template <int MT, bool ROWS_ALIGNED>
__global__ __launch_bounds__(256) void k_material_scores(ScoreArgs a) {
  __shared__ __attribute__((aligned(16))) float ys[kTileM * MT * kMaxP];
  if (a.prop) stage_properties<MT>(ys, a.y, a.K, a.P, threadIdx.x, blockDim.x);
  __syncthreads();

  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const long long n0 = ((long long)blockIdx.x * 4 + wave) * kTileN;
  if (n0 >= a.N) return;
  const int g = lane / 32;
  const long long n = n0 + (lane & 31);
  const bool valid = n < a.N;
  const float* __restrict__ row = a.fused + (valid ? n : a.N - 1) * a.D;

  f32x16 acc[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[mt][r] = 0.0f;

  score_products<MT, ROWS_ALIGNED, false>(row, a.D, a.steps, a.a_split, lane, acc);

  finish_scores<MT>(acc, valid ? n : a.N - 1, valid, g, a.K, a.P, a.inv_T, ys, a.scores, a.prop, a.label, a.unseen_zero != 0);
}

// The same contraction for whole macro steps and 16-byte aligned rows, software-pipelined: what step s + 1 needs - the
// lane's 64 bytes of its row and the split embeddings of the step (MT * 4 KiB, L2 hits) - is
// requested before the products of step s and kept in a second set of registers (the loop is unrolled by two, so
// that nothing that is still on its way has to be copied).  The memory counter returns reads in order: the requests
// for the next step are always the youngest, so waiting for this step's operands never waits for them.  Without the
// pipeline a wave asked for a step only when it needed it, and the kernel reached 4.0 of the 5.3 TB/s that the same
// read pattern reaches without arithmetic.
template <int MT, typename T>
__global__ __launch_bounds__(256) void k_material_scores_few(ScoreArgs a) {
  __shared__ __attribute__((aligned(16))) float ys[kTileM * MT * kMaxP];
  __shared__ __attribute__((aligned(16))) float s_stage[4][score_stage_floats<16>()];
  if (a.prop) stage_properties<MT>(ys, a.y, a.K, a.P, threadIdx.x, blockDim.x);
  __syncthreads();

  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const long long n0 = ((long long)blockIdx.x * 4 + wave) * kTileN;
  if (n0 >= a.N) return;
  const long long n = n0 + (lane & 31);
  const float* __restrict__ row = a.fused + (n < a.N ? n : a.N - 1) * a.D + (lane / 32) * 16;
  ScoreSums<MT, T> sum;

  struct Rows { f32x4 v[4]; };
  struct Emb { Term8<T> hi[MT][2], lo[MT][2]; };
  auto load_rows = [&](int s, Rows& r) {
#pragma unroll
    for (int q = 0; q < 4; ++q) r.v[q] = *reinterpret_cast<const f32x4*>(row + s * kStepK + 4 * q);
  };
  auto load_emb = [&](int s, Emb& e) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const Term8<T>* slot = reinterpret_cast<const Term8<T>*>(a.a_split) + ((long long)(s * MT + mt) * 2 + j) * 2 * kWave + lane;
        e.hi[mt][j] = slot[0];
        e.lo[mt][j] = slot[kWave];
      }
  };
  auto products = [&](const Rows& r, const Emb& e) {
    Term8<T> bh[2], bl[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const float x = r.v[2 * j + (c >> 2)][c & 3];
        T h, l;
        split_terms<T>(x, h, l);
        bh[j][c] = h;
        bl[j][c] = l;
      }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        sum.acc[mt] = score_mma(e.hi[mt][j], bh[j], sum.acc[mt]);
        sum.low(mt) = score_mma(e.hi[mt][j], bl[j], sum.low(mt));
        sum.low(mt) = score_mma(e.lo[mt][j], bh[j], sum.low(mt));
      }
  };

  const int last = a.steps - 1;
  Rows r0, r1;
  Emb e0, e1;
  load_rows(0, r0);
  load_emb(0, e0);
  for (int s = 0; s < a.steps; s += 2) {
    // step s from set 0 while step s + 1 arrives in set 1 (past the end: the last step again, read and not used)
    load_emb(min(s + 1, last), e1);
    load_rows(min(s + 1, last), r1);
    __builtin_amdgcn_sched_barrier(0);
    products(r0, e0);
    __builtin_amdgcn_sched_barrier(0);
    if (s + 1 < a.steps) {   // uniform
      load_emb(min(s + 2, last), e0);
      load_rows(min(s + 2, last), r0);
      __builtin_amdgcn_sched_barrier(0);
      products(r1, e1);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  sum.join();
  finish_scores_staged<MT, 16>(sum.acc, n0, (int)std::min<long long>(kTileN, a.N - n0), lane, a.K, a.P, a.inv_T, ys, a.scores,
                               a.prop, a.label, a.unseen_zero != 0, s_stage[wave]);
}

// Few rows: what such a call takes is launches and the chain of a wave's steps, not bytes.  A workgroup has 32 rows.  Its first
// waves read rows and embeddings, two macro steps at a time and three such pairs ahead, split them into two terms (no kernel
// has to run before this one) and leave the operands in LDS; a wave per 32 materials multiplies them, the steps in their order:
// the products of a score are added up as every other kernel here adds them, so a row's scores do not depend on how many
// rows the call has (and it takes no longer than a quarter of the steps to each of four waves and a sum of four parts did: 2001 rows
// of 384 channels and 10 materials 7.0 and 7.1 us, 10 000 of 512 and 32 materials 14.9 and 16.1; two launches 14.6 and 18.1).
template <int MT, typename T>
__global__ __launch_bounds__((2 + 3 * MT) * kWave) void k_material_scores_split(ScoreArgs a, const float* __restrict__ temb) {
  constexpr int kReaders = 2 * (1 + MT);   // wave w: operand w / 2 (the rows, then 32 materials each), step w % 2 of a pair
  constexpr int kAhead = 3;
  __shared__ __attribute__((aligned(16))) float ys[kTileM * MT * kMaxP];
  __shared__ __attribute__((aligned(16))) Term8<T> s_op[2][2][1 + MT][2][2][kWave];   // [pair][step][operand][j][hi, lo]
  __shared__ f32x4 s_part[MT > 1 ? MT - 1 : 1][4][kWave];
  __shared__ __attribute__((aligned(16))) float s_stage[score_stage_floats<16>()];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const long long n0 = (long long)blockIdx.x * kTileN;
  const int pairs = (a.steps + 1) / 2;
  if (a.prop) stage_properties<MT>(ys, a.y, a.K, a.P, threadIdx.x, blockDim.x);
  if (wave < kReaders) {
    const int op = wave >> 1, half = wave & 1;
    // (a row or material beyond the last one: the last again, into sums that nobody reads)
    const float* __restrict__ src = (op == 0 ? a.fused + std::min<long long>(n0 + (lane & 31), a.N - 1) * a.D
                                             : temb + (long long)min((op - 1) * kTileM + (lane & 31), a.K - 1) * a.D) + (lane / 32) * 16;
    struct Piece { f32x4 v[4]; } p[kAhead];   // the lane's 16 channels of a step
    auto load = [&](int pair, Piece& b) {     // (past the end: the last step, read and not used)
      const int at = min(2 * pair + half, a.steps - 1) * kStepK;
#pragma unroll
      for (int q = 0; q < 4; ++q) b.v[q] = *reinterpret_cast<const f32x4*>(src + at + 4 * q);
    };
    auto hand_over = [&](int pair, Piece& b) {
      Term8<T>(&out)[2][2][kWave] = s_op[pair & 1][half][op];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        Term8<T> hi, lo;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          T h, l;
          split_terms<T>(b.v[2 * j + (c >> 2)][c & 3], h, l);
          hi[c] = h;
          lo[c] = l;
        }
        out[j][0][lane] = hi;
        out[j][1][lane] = lo;
      }
      load(pair + kAhead, b);
      __syncthreads();
    };
#pragma unroll
    for (int e = 0; e < kAhead; ++e) load(e, p[e]);
    for (int i = 0; i < pairs; i += kAhead) {   // uniform over the workgroup: one barrier per pair here and below
#pragma unroll
      for (int e = 0; e < kAhead; ++e)
        if (i + e < pairs) hand_over(i + e, p[e]);
    }
    if constexpr (MT > 1) __syncthreads();
    return;
  }
  const int mt = wave - kReaders;
  ScoreSums<1, T> sum;
  auto products = [&](int s) {
    const Term8<T>(&row)[2][2][kWave] = s_op[(s >> 1) & 1][s & 1][0];
    const Term8<T>(&emb)[2][2][kWave] = s_op[(s >> 1) & 1][s & 1][1 + mt];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const Term8<T> bh = row[j][0][lane], bl = row[j][1][lane], eh = emb[j][0][lane], el = emb[j][1][lane];
      sum.acc[0] = score_mma(eh, bh, sum.acc[0]);
      sum.low(0) = score_mma(eh, bl, sum.low(0));
      sum.low(0) = score_mma(el, bh, sum.low(0));
    }
  };
  __syncthreads();   // the first pair is in LDS
  for (int i = 0; i < pairs; ++i) {
    products(2 * i);
    if (2 * i + 1 < a.steps) products(2 * i + 1);
    if (i + 1 < pairs) __syncthreads();   // the next pair is there, and this one's place is free
  }
  sum.join();
  f32x16 acc[MT];
  acc[0] = sum.acc[0];
  if constexpr (MT > 1) {
    if (mt > 0) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        s_part[mt - 1][q][lane] = f32x4{acc[0][4 * q], acc[0][4 * q + 1], acc[0][4 * q + 2], acc[0][4 * q + 3]};
    }
    __syncthreads();
    if (mt > 0) return;
#pragma unroll
    for (int t = 1; t < MT; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 part = s_part[t - 1][q][lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[t][4 * q + e] = part[e];
      }
  }
  finish_scores_staged<MT, 16, true>(acc, n0, (int)std::min<long long>(kTileN, a.N - n0), lane, a.K, a.P, a.inv_T, ys, a.scores,
                               a.prop, a.label, a.unseen_zero != 0, s_stage);
}

// 65 to 128 materials and few rows: the split embeddings of a step (16 KiB) pass through LDS, double buffered, once per workgroup of
// four waves and 128 points, the rows through registers (whole macro steps, 16-byte aligned rows).  With one wave per SIMD what counts is
// the chain of a step, which is shorter here than that of k_material_scores_staged (20 000 rows of 512 channels, 100 materials 25.5 us, 30
// there).  A step: the next block, requested a step ago, goes to LDS, the block after it and the rows of the step after next are requested,
// then the products; one barrier.
template <typename T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(TermOf<T>::kScaled ? 2 : 3, TermOf<T>::kScaled ? 2 : 3)))
void k_material_scores_wide(ScoreArgs a) {
  constexpr int MT = 4;
  constexpr int kBlock = MT * 2 * 2 * kWave;   // 16-byte operand slots of a step
  constexpr int kCopies = kBlock / 256;        // per thread
  __shared__ __attribute__((aligned(16))) float ys[kTileM * MT * kMaxP];
  __shared__ __attribute__((aligned(16))) Term8<T> s_a[2][kBlock];
  __shared__ __attribute__((aligned(16))) float s_stage[4][score_stage_floats<16>()];
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave, g = lane / 32;
  if (a.prop) stage_properties<MT>(ys, a.y, a.K, a.P, tid, 256);
  const long long n0 = ((long long)blockIdx.x * 4 + wave) * kTileN;   // a wave beyond the last row takes part in the copies
  const long long n = min(n0 + (lane & 31), a.N - 1);
  const float* __restrict__ row = a.fused + n * a.D + g * 16;
  const int last = a.steps - 1;                // requests past the end repeat the last step (read, not used)

  ScoreSums<MT, T> sum;
  struct Rows { f32x4 v[4]; };
  Term8<T> copy[kCopies];
  auto load_rows = [&](int s, Rows& r) {
#pragma unroll
    for (int q = 0; q < 4; ++q) r.v[q] = *reinterpret_cast<const f32x4*>(row + min(s, last) * kStepK + 4 * q);
  };
  auto load_block = [&](int s) {
#pragma unroll
    for (int u = 0; u < kCopies; ++u) copy[u] = reinterpret_cast<const Term8<T>*>(a.a_split)[(long long)min(s, last) * kBlock + u * 256 + tid];
  };
  auto step = [&](int s, Rows& r) {
    Term8<T>* next = s_a[(s + 1) & 1];
#pragma unroll
    for (int u = 0; u < kCopies; ++u) next[u * 256 + tid] = copy[u];
    load_block(s + 2);
    Term8<T> bh[2], bl[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const float x = r.v[2 * j + (c >> 2)][c & 3];
        T h, l;
        split_terms<T>(x, h, l);
        bh[j][c] = h;
        bl[j][c] = l;
      }
    __builtin_amdgcn_sched_barrier(0);
    load_rows(s + 2, r);
    __builtin_amdgcn_sched_barrier(0);
    const Term8<T>* cur = s_a[s & 1] + lane;
    // two tiles at a time: their accumulators take turns, so that no product waits for the one before it
    constexpr int kPair = 2;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int m0 = 0; m0 < MT; m0 += kPair) {
        Term8<T> ah[kPair], al[kPair];
#pragma unroll
        for (int i = 0; i < kPair; ++i) {
          ah[i] = cur[((m0 + i) * 2 + j) * 2 * kWave];
          al[i] = cur[(((m0 + i) * 2 + j) * 2 + 1) * kWave];
        }
#pragma unroll
        for (int i = 0; i < kPair; ++i) sum.acc[m0 + i] = score_mma(ah[i], bh[j], sum.acc[m0 + i]);
#pragma unroll
        for (int i = 0; i < kPair; ++i) sum.low(m0 + i) = score_mma(ah[i], bl[j], sum.low(m0 + i));
#pragma unroll
        for (int i = 0; i < kPair; ++i) sum.low(m0 + i) = score_mma(al[i], bh[j], sum.low(m0 + i));
      }
    __syncthreads();   // the next step's block is in place, and nobody reads this step's any more
  };
  Rows r0, r1;
  load_block(0);
#pragma unroll
  for (int u = 0; u < kCopies; ++u) s_a[0][u * 256 + tid] = copy[u];
  load_block(1);
  load_rows(0, r0);
  load_rows(1, r1);
  __syncthreads();
  for (int s = 0; s < a.steps; s += 2) {   // uniform over the workgroup
    step(s, r0);
    if (s + 1 < a.steps) step(s + 1, r1);
  }
  if (n0 >= a.N) return;
  sum.join();
  finish_scores_staged<MT, 16>(sum.acc, n0, (int)std::min<long long>(kTileN, a.N - n0), lane, a.K, a.P, a.inv_T, ys, a.scores,
                               a.prop, a.label, a.unseen_zero != 0, s_stage[wave]);
}

// The row stream of many rows: rows and split embeddings on their way through LDS (scores_staged.hpp), four waves and 128 rows per
// workgroup (whole macro steps, 16-byte aligned rows).  WAVES: per SIMD; what LDS holds per workgroup follows from it.  Bound by the rows
// from memory: 5.3 TB/s with 32 materials, 4.4 with 128, where the embeddings are as many bytes from L2 as the rows.  us, before (the
// embeddings resident in the LDS of one workgroup of 16 or 8 waves, or through registers and LDS as in k_material_scores_wide) / now:
// 1 M rows of 512 channels and 32 materials 451 / 408, 64 materials 481 / 444, 1.6 M and 24 726 / 640, 300 007 of 1024 channels and 100
// materials 386 / 360, 1.68 M and 128 1890 / 1760, 200 000 of 768 channels and 64 materials 172 / 148.  One workgroup of twelve waves per
// compute unit, which fetches the embeddings once instead of three times: 360 -> 371; two with sources four halves deep 366; operands
// of the next pair of tiles read ahead: the same.  (Right behind the kernel that wrote the rows it gains as much, 473 -> 435 for 1 M rows, but
// where such steps follow each other without a pause the fusion then takes 30 us longer: 1461 -> 1464 and, in another session,
// 1447 -> 1453 us a step; 1515 -> 1489 for a step alone.)
constexpr int kStagedWaves = 4;
constexpr long long kOneRound = 256 * kStagedWaves * kTileN;   // rows of one workgroup per compute unit
template <int MT, typename T, int WAVES>
__global__ __launch_bounds__(kStagedWaves * kWave) __attribute__((amdgpu_waves_per_eu(WAVES, WAVES)))
void k_material_scores_staged(ScoreArgs a) {
  constexpr StagedShape kShape = staged_shape(MT, kStagedWaves, 163840 / WAVES / 1280 * 1280);
  // While the products are made: embeddings, then rows.  Afterwards: the properties, then each wave's score rows on their way to memory.
  __shared__ __attribute__((aligned(1024))) char s_mem[staged_bytes(MT, kShape)];
  float* const ys = reinterpret_cast<float*>(s_mem);
  float* const s_stage = ys + kTileM * MT * kMaxP;
  static_assert((kTileM * MT * kMaxP + kStagedWaves * score_stage_floats<16>()) * sizeof(float) <= sizeof(s_mem));
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const long long t0 = ((long long)blockIdx.x * kStagedWaves + wave) * kTileN;
  const bool work = t0 < a.N;   // a wave beyond the last row takes part in the copies
  const long long n0 = work ? t0 : 0;
  const int rows = (int)std::min<long long>(kTileN, a.N - n0);
  ScoreSums<MT, T> sum;
  score_products_staged<MT, T, false, kStagedWaves, kShape.rows, kShape.sources>(a.fused + n0 * a.D, a.D, rows - 1, a.steps, a.a_split, wave, lane,
                                                                   s_mem, sum, work);
  if (a.prop) stage_properties<MT>(ys, a.y, a.K, a.P, threadIdx.x, kStagedWaves * kWave);
  __syncthreads();
  if (!work) return;
  sum.join();
  finish_scores_staged<MT, 16>(sum.acc, n0, rows, lane, a.K, a.P, a.inv_T, ys, a.scores, a.prop, a.label, a.unseen_zero != 0,
                               s_stage + wave * score_stage_floats<16>());
}

size_t split_embeddings_bytes(int D, int MT) {
  return (size_t)((D + kStepK - 1) / kStepK) * MT * 2 * 2 * kWave * 8 * sizeof(__bf16);
}

hipError_t launch_split_embeddings(const float* emb, int n_rows, int D, int MT, void* out, hipStream_t stream) {
  const int S = (D + kStepK - 1) / kStepK;
  const long long total = (long long)S * MT * 2 * kWave;
  hipLaunchKernelGGL((k_split_embeddings<TermB>), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, emb, n_rows, D,
                     MT, S, static_cast<__bf16*>(out));
  return hipGetLastError();
}

static int tiles_m(int K) { return (K + kTileM - 1) / kTileM; }
static int steps_k(int D) { return (D + kStepK - 1) / kStepK; }

size_t scores_split_bytes(int D, int K) {
  int MT = tiles_m(K);
  if (MT == 3) MT = 4;
  return (size_t)steps_k(D) * MT * 2 * 2 * kWave * 8 * sizeof(__bf16);
}

// the split embeddings, then room for an fp32 copy of embeddings that arrive as 16-bit values
size_t scores_workspace_bytes(int D, int K) {
  return scores_split_bytes(D, K) + (((size_t)K * D * sizeof(float) + 255) & ~(size_t)255);
}

// Text embeddings given as bf16 (dtype 1) or fp16 (dtype 2) values, widened exactly to fp32.
__global__ __launch_bounds__(256) void k_widen_embeddings(const uint16_t* __restrict__ src, int dtype, long long n,
                                                          float* __restrict__ dst) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint16_t b = src[i];
  dst[i] = dtype == 1 ? __uint_as_float((uint32_t)b << 16) : (float)__builtin_bit_cast(_Float16, b);
}

hipError_t launch_widen_embeddings(const void* src, int dtype, long long n, float* dst, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_widen_embeddings, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream,
                     static_cast<const uint16_t*>(src), dtype, n, dst);
  return hipGetLastError();
}

// Terms of type fp16: 16-byte aligned rows of whole macro steps only (launch_material_scores).
template <int MT, typename T>
static hipError_t launch_mt(const ScoreArgs& a, bool aligned, hipStream_t stream) {
  const dim3 grid((unsigned)((a.N + 4 * kTileN - 1) / (4 * kTileN))), block(256);
  if (aligned && a.D % kStepK == 0) {
    // Both operands through LDS from the second workgroup of 128 rows per compute unit on, where others fill the gaps of one (us per call,
    // through registers / LDS; 24 600 rows: 768 channels and 100 materials 32.4 / 38.2, 64 27.2 / 29.4, 32 21.6 / 23.6, 1024 channels and
    // 100 38.4 / 46.7; 33 000 rows: 46.6 / 44.6, 44.6 / 33.6, 36.2 / 26.9, 54.7 / 54.7; 60 000 rows: 49.3 / 49.0, 46.4 / 38.6,
    // 36.8 / 34.4, 69.6 / 65.2; 384 channels alike).
    if (a.N > kOneRound) {
      if constexpr (MT == 2) {
        // Rows a multiple of 4 KiB apart begin in the same channel of L2, wait for each other there, and want more requests ahead rather
        // than more waves (64 materials, four / three waves per SIMD, us: 400 000 rows of 1024 channels 414 / 369, 500 000 525 / 468;
        // 1 M of 512 444 / 444, 100 000 of 512 46.8 / 51.1, 70 000 of 384 31.5 / 34.1).
        if (a.D % 1024 == 0) {
          hipLaunchKernelGGL((k_material_scores_staged<MT, T, 3>), grid, block, 0, stream, a);
          return hipGetLastError();
        }
      }
      hipLaunchKernelGGL((k_material_scores_staged<MT, T, MT <= 2 ? 4 : (TermOf<T>::kScaled ? 2 : 3)>), grid, block, 0, stream, a);
      return hipGetLastError();
    }
    if constexpr (MT == 4) hipLaunchKernelGGL((k_material_scores_wide<T>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL((k_material_scores_few<MT, T>), grid, block, 0, stream, a);
    return hipGetLastError();
  }
  if constexpr (std::is_same_v<T, TermB>) {
    if (aligned)
      hipLaunchKernelGGL((k_material_scores<MT, true>), grid, block, 0, stream, a);
    else
      hipLaunchKernelGGL((k_material_scores<MT, false>), grid, block, 0, stream, a);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

// Which calls of up to 64 materials take k_material_scores_split: those of up to two of its workgroups per compute unit (512
// of 32 rows), of up to three with at most 16 materials and 1024 channels.  Every workgroup reads and splits the embeddings, and
// each round of workgroups adds to the time; the two launches take as long for 500 rows as for 30 000.  us per call, two
// launches / one (rows x channels, materials):
//   2001 x 384, 10     14.6 / 7.0     5000 x 512, 50     22.4 / 13.1     10 000 x 1024, 64   34.6 / 32.9
//   16 384 rows        x 32, 1   7.5 / 5.4     x 64, 64   13.8 / 13.6    x 512, 64   24.0 / 22.9    x 1024, 16   26.5 / 18.0
//                      x 2048, 64   56.3 / 54.0      x 4096, 32   87.0 / 65.0
//   16 385 rows        x 256, 32   13.9 / 12.9       x 64, 64   13.9 / 19.7          x 512, 64   24.0 / 32.3
//   24 576 rows        x 32, 16   8.5 / 8.5    x 512, 16   17.9 / 16.3   x 512, 20   18.9 / 17.7   x 1024, 16   26.6 / 25.0
//                      x 1024, 20   27.3 / 26.6      x 2048, 16   44.0 / 46.5
//   24 577 rows        x 256, 16   13.1 / 13.2       x 512, 16   17.9 / 19.3         x 1024, 16   26.7 / 31.2
static bool few_rows(long long N, int D, int K) { return N <= 16384 || (N <= 24576 && K <= 16 && D <= 1024); }

hipError_t launch_material_scores(const float* fused, long long N, int D, const float* temb, int K,
                                  const float* y, int P, float temperature, float* scores, float* prop,
                                  int* label, void* workspace, hipStream_t stream, int unseen_zero, bool f16_terms) {
  if (N == 0) return hipSuccess;
  int MT = tiles_m(K);
  if (MT == 3) MT = 4;
  const int S = steps_k(D);
  ScoreArgs a{fused, N, D, K, P, y, inverse_temperature(temperature), unseen_zero, scores, prop, label,
              static_cast<const bf16x8*>(workspace), S};
  const bool aligned = (D & 3) == 0 && (reinterpret_cast<uintptr_t>(fused) & 15) == 0;
  if (MT <= 2 && few_rows(N, D, K) && aligned && D % kStepK == 0 && (reinterpret_cast<uintptr_t>(temb) & 15) == 0) {
    const dim3 grid((unsigned)((N + kTileN - 1) / kTileN)), block((2 + 3 * MT) * kWave);
    if (f16_terms) {
      if (MT == 1) hipLaunchKernelGGL((k_material_scores_split<1, TermH>), grid, block, 0, stream, a, temb);
      else hipLaunchKernelGGL((k_material_scores_split<2, TermH>), grid, block, 0, stream, a, temb);
    } else {
      if (MT == 1) hipLaunchKernelGGL((k_material_scores_split<1, TermB>), grid, block, 0, stream, a, temb);
      else hipLaunchKernelGGL((k_material_scores_split<2, TermB>), grid, block, 0, stream, a, temb);
    }
    return hipGetLastError();
  }
  {
    long long total = (long long)S * MT * 2 * kWave;
    const dim3 grid((unsigned)((total + 255) / 256)), block(256);
    if (f16_terms)
      hipLaunchKernelGGL((k_split_embeddings<TermH>), grid, block, 0, stream, temb, K, D, MT, S, static_cast<TermH*>(workspace));
    else
      hipLaunchKernelGGL((k_split_embeddings<TermB>), grid, block, 0, stream, temb, K, D, MT, S, static_cast<TermB*>(workspace));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (f16_terms) {
    if (!aligned || D % kStepK != 0) return hipErrorInvalidValue;
    switch (MT) {
      case 1: return launch_mt<1, TermH>(a, aligned, stream);
      case 2: return launch_mt<2, TermH>(a, aligned, stream);
      default: return launch_mt<4, TermH>(a, aligned, stream);
    }
  }
  switch (MT) {
    case 1: return launch_mt<1, TermB>(a, aligned, stream);
    case 2: return launch_mt<2, TermB>(a, aligned, stream);
    default: return launch_mt<4, TermB>(a, aligned, stream);
  }
}

}  // namespace aura
