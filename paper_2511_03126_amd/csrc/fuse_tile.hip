// aura_fuse_features, matrix-core path (Sec. 3.1 "Feature Aggregation", Eq. 2).
//
// Eq. 2 with bilinear sampling is a weighted sum of feature cells:
//     sum_v M_vis(x_i, v) F_v(pi(x_i, v)) = sum_c  w[i][c] * F[c],
// where c runs over (view, cell) pairs and w[i][c] is the bilinear weight of cell c for point i
// (zero unless the view sees the point and c is one of the four cells around the projection).
// For a tile of 32 spatially neighbouring points only about a hundred cells carry a non-zero
// weight, so the sum is a small dense product
//     [32 points x L cells] . [L cells x D channels]
// that runs on the matrix cores with the stored 16-bit features as they are.  The gather
// formulation reads every cell row once per point and view (4 D elements per pair) and spends
// its time widening and multiplying on the vector ALUs; here each cell of the list is read once
// per tile.
//
// Two kernels:
//
// k_tile_prepare (one workgroup of 256 threads per tile, little register state, many tiles in
// flight per CU so that the projection -> depth-read -> list chain of one tile hides behind the
// others):
//   A  every (point, view) pair is projected and tested (Eq. 1, the shared fp32 decision
//      functions).  Per view, the bounding box of the touched cells is found with a half-wave
//      reduction.
//   B  views whose box fits 32 x 32 cells mark the touched cells in a 1024-bit map (exact list,
//      no duplicates, no untouched cells); larger boxes (points far apart) give each visible
//      pair four private entries.  A scan over the views lays the per-view lists end to end.
//   C  per chunk of the list: the weights are scattered into a [32][cells] matrix in LDS, split
//      into two 16-bit terms (hi + lo, about 16 mantissa bits), and copied out as k-steps of 16
//      cells in the operand layout of the matrix-core instruction.  Every tile owns a fixed number
//      of k-steps of storage; a tile that needs more (points far apart) is fused by a plain
//      gather after the others, so which way a tile goes depends on the tile alone and results are
//      reproducible bit for bit.
//
// k_tile_product (one workgroup per tile, wave s owns channels [256 s, 256 s + 256)): per k-step
// each lane reads two 8-byte pieces (4 channels each, 128 channels apart) of 8 cell rows straight
// from global memory (the rows of a tile's neighbours keep them in L2), regroups them with byte
// permutes into the 8 B-operands and issues v_mfma_f32_32x32x16 with the hi and the lo weights.
// No barrier inside the loop; reads run two k-steps ahead of the products.  Then mean, L2 norm
// (half-wave reduction, across the waves through LDS) and streaming stores.
// Accumulator t = 4 h + j, register r of lane l is point 8 (r/4) + 4 (l/32) + r%4, channel
// 256 s + 128 h + 4 (l%32) + j: a store instruction writes 16 bytes per lane and the 32 lanes of
// a half wave cover 512 contiguous bytes of a row (full cache lines; writing 16 of every 32
// bytes, as a lane owning 8 consecutive channels would, halves the achieved write bandwidth).
//
// List entries that only pad the last k-step have zero weights, so feature maps must be finite.
#include <algorithm>

#include "aura_device.hpp"
#include "fuse_args.hpp"
#include "fuse_tile_core.hpp"
#include "fuse_tile_groups.hpp"
#include "fuse_tile_lists.hpp"
#include "launch.hpp"
#include "scores_epilogue.hpp"
#include "timing.hpp"

namespace aura {

constexpr int kViewBatch = 32;                 // views handled per pass over the point tile
constexpr int kPrepThreads = 256;
constexpr int kSlots = kPrepThreads / kTilePts;   // views processed side by side (one per half wave)
constexpr int kNIT = kViewBatch / kSlots;      // (point, view) pairs per thread and batch
#ifndef AURA_CHUNK
#define AURA_CHUNK 12
#endif
#ifndef AURA_PREP_WPE
#define AURA_PREP_WPE 4
#endif
constexpr int kChunkSteps = AURA_CHUNK;        // k-steps of the weight matrix held in LDS
constexpr int kChunk = kChunkSteps * kStepCells;
constexpr int kPitch = kChunk + 8;             // row pitch in 16-bit elements (rows start 4 banks apart)

static_assert(kSlots * kTilePts == kPrepThreads && kNIT * kSlots == kViewBatch, "thread mapping");
// One (point, view) pair after Eq. 1 and the cell selection.
struct PairRec {
  int xy;        // y0 << 16 | x0 of the first cell, -1: the view does not see the point
  float ax, ay;  // weights of the second cell per axis
};

// DT: 1 bf16, 2 fp16 feature maps (decides the 16-bit format of the weights).  SEL: the views of each point are
// given (FuseArgs::in_mask) instead of decided by the depth test; a variant of its own so that the usual path does
// not carry the test.
template <int DT, bool SEL>
__global__ __launch_bounds__(kPrepThreads) __attribute__((amdgpu_waves_per_eu(AURA_PREP_WPE)))
void k_tile_prepare(FuseArgs a, TileWs ws, ObjTable tab) {
  __shared__ int s_win[kViewBatch][2];                 // first cell (x, y) of the view's map
  __shared__ int s_mode[kViewBatch];                   // 0 nothing seen, 1 cell map, 2 private entries
  __shared__ uint32_t s_vmask[kViewBatch];             // which of the 32 points the view sees
  __shared__ __attribute__((aligned(16))) uint32_t s_bits[kViewBatch][kWinSide];   // map of touched cells, row = word
  __shared__ __attribute__((aligned(16))) uint16_t s_wbase[kViewBatch][kWinSide];  // set bits before each row
  __shared__ int s_base[kViewBatch + 1];               // first list index of each view
  __shared__ __attribute__((aligned(16))) uint32_t s_cell[kChunk];
  __shared__ __attribute__((aligned(16))) uint16_t s_whi[kTilePts][kPitch];
  __shared__ __attribute__((aligned(16))) uint16_t s_wlo[kTilePts][kPitch];
  __shared__ int s_cnt[kTilePts];

  const ObjRange ob = tab.o[blockIdx.y];
  const int nblk = (ob.n_pts + kTilePts - 1) / kTilePts;
  if ((int)blockIdx.x >= nblk) return;
  const int blk = xcd_contiguous(blockIdx.x, nblk);
  TileHdr* __restrict__ hdr = ws.hdr + ob.tile_begin + blk;
  const long long slot0 = (long long)(ob.tile_begin + blk) * ws.quota;   // first k-step the tile owns
  const int tid = threadIdx.x, lane = tid % kWave;
  const int Hf = a.feat.Hf, Wf = a.feat.Wf;
  const uint32_t row_bytes = (uint32_t)a.feat.D * 2u;
  const int p = tid % kTilePts;          // point of this thread
  const int slot = tid / kTilePts;       // view slot of this thread
  const int li0 = blk * kTilePts;
  const bool p_valid = li0 + p < ob.n_pts;
  const long long ip = ob.pt_begin + li0 + (p_valid ? p : 0);
  const float px = a.xyz[3 * ip], py = a.xyz[3 * ip + 1], pz = a.xyz[3 * ip + 2];

  if (tid < kTilePts) s_cnt[tid] = 0;
  int used = 0;   // k-steps written so far (the view batches follow one another in the tile's run)
  bool exhausted = false;

  for (int vb0 = 0; vb0 < ob.n_views; vb0 += kViewBatch) {
    const int nvb = min(kViewBatch, ob.n_views - vb0);
    __syncthreads();   // the previous batch is done with the tables (and s_cnt is initialised)
    *reinterpret_cast<u32x4*>(&s_bits[tid / 8][4 * (tid % 8)]) = u32x4{0u, 0u, 0u, 0u};

    // ---- A: project and test; bounding box of the touched cells per view
    PairRec pr[kNIT];
    int my_cnt = 0;
    // All projections of the batch first, then all depth texels, then the tests: a thread's four pairs are four chains
    // of camera row -> projection -> texel address -> texel, and in one loop each chain waited for the one before it
    // (11 K of a tile's 26 K cycles with 32 views).
    Proj pjs[kNIT];
    bool frs[kNIT];
    float deps[kNIT];
#pragma unroll
    for (int it = 0; it < kNIT; ++it) {
      const int v = ob.view_begin + vb0 + min(it * kSlots + slot, nvb - 1);   // (a slot beyond the batch: its last view again)
      pjs[it] = project(a.vis.cam + (long long)v * 16, px, py, pz);
      frs[it] = in_frustum(a.vis, pjs[it]);
    }
#pragma unroll
    for (int it = 0; it < kNIT; ++it) {
      const int v = ob.view_begin + vb0 + min(it * kSlots + slot, nvb - 1);
      deps[it] = 1.0f;
      if (a.vis.depth) deps[it] = a.vis.depth[(long long)v * a.vis.H * a.vis.W + (frs[it] ? depth_texel(a.vis, pjs[it]) : 0)];
    }
#pragma unroll
    for (int it = 0; it < kNIT; ++it) {
      pr[it].xy = -1;
      pr[it].ax = pr[it].ay = 0.0f;
      if (it * kSlots >= nvb) continue;   // uniform
      const int vl = it * kSlots + slot;
      const Proj pj = pjs[it];
      const bool fr = frs[it];
      const float dep = deps[it];
      bool seen = vl < nvb && p_valid && fr && (a.vis.frustum_only || passes_depth(a.vis, pj, dep));
      if constexpr (SEL) seen = seen && view_kept(a, ip, vb0 + min(vl, nvb - 1));
      s16x2 lo2 = {0x7fff, 0x7fff}, hi2 = {-1, -1};   // (x, y) of the first / second cell
      if (seen) {
        const Tap tx = tap_axis(pj.u, a.feat.pitch_x, Wf), ty = tap_axis(pj.v, a.feat.pitch_y, Hf);
        pr[it].ax = tx.a;
        pr[it].ay = ty.a;
        pr[it].xy = (ty.i0 << 16) | tx.i0;
        lo2 = s16x2{(short)tx.i0, (short)ty.i0};
        hi2 = s16x2{(short)tx.i1, (short)ty.i1};
        ++my_cnt;
      }
      const unsigned long long seen_mask = __ballot(seen);
      lo2 = half_wave_reduce<true>(lo2);
      hi2 = half_wave_reduce<false>(hi2);
      if (p == kTilePts - 1 && vl < nvb) {
        const bool any = hi2[0] >= 0;
        const int ww = hi2[0] - lo2[0] + 1, wh = hi2[1] - lo2[1] + 1;
        s_win[vl][0] = lo2[0];
        s_win[vl][1] = lo2[1];
        s_mode[vl] = !any ? 0 : (ww <= kWinSide && wh <= kWinSide ? 1 : 2);
        s_vmask[vl] = (uint32_t)(seen_mask >> (lane & 32));
      }
    }
    if (my_cnt) atomicAdd(&s_cnt[p], my_cnt);
    __syncthreads();
    if (a.out_vis && tid < kTilePts && p_valid) {
      // the mask of Eq. 1 for this batch of views, from the per-view bit masks: point tid's bytes, four per store
      // where the row pitch allows
      uint8_t* __restrict__ vrow = a.out_vis + (ob.pt_begin + li0 + tid) * a.vis_pitch + vb0;
      if ((a.vis_pitch & 3) == 0) {
        for (int v4 = 0; v4 < nvb; v4 += 4) {
          uint32_t w = 0;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (v4 + e < nvb) w |= ((s_vmask[v4 + e] >> tid) & 1u) << (8 * e);
          if (v4 + 4 <= nvb) {
            *reinterpret_cast<uint32_t*>(vrow + v4) = w;
          } else {
            for (int e = 0; v4 + e < nvb; ++e) vrow[v4 + e] = (uint8_t)((w >> (8 * e)) & 1u);
          }
        }
      } else {
        for (int v = 0; v < nvb; ++v) vrow[v] = (uint8_t)((s_vmask[v] >> tid) & 1u);
      }
    }

    // ---- B: mark the touched cells of every view that uses a map
#pragma unroll
    for (int it = 0; it < kNIT; ++it) {
      if (pr[it].xy < 0) continue;
      const int vl = it * kSlots + slot;
      if (s_mode[vl] != 1) continue;
      const int x0 = pr[it].xy & 0xffff, y0 = pr[it].xy >> 16;
      const int bit = (y0 - s_win[vl][1]) * kWinSide + (x0 - s_win[vl][0]);
      const bool has_x1 = x0 + 1 < Wf, has_y1 = y0 + 1 < Hf;   // at the border the second cell has weight 0
      atomicOr(&s_bits[vl][bit >> 5], 1u << (bit & 31));
      if (has_x1) atomicOr(&s_bits[vl][(bit + 1) >> 5], 1u << ((bit + 1) & 31));
      if (has_y1) atomicOr(&s_bits[vl][(bit + kWinSide) >> 5], 1u << ((bit + kWinSide) & 31));
      if (has_x1 && has_y1) atomicOr(&s_bits[vl][(bit + kWinSide + 1) >> 5], 1u << ((bit + kWinSide + 1) & 31));
    }
    __syncthreads();
    if (tid < kWave) {   // list length of every view, exclusive scan over the views
      int n = 0;
      if (lane < nvb) {
        if (s_mode[lane] == 1) {
#pragma unroll 8
          for (int w = 0; w < kWinSide; ++w) {
            s_wbase[lane][w] = (uint16_t)n;
            n += __popc(s_bits[lane][w]);
          }
        } else if (s_mode[lane] == 2) {
          n = 4 * __popc(s_vmask[lane]);
        }
      }
      int inc = n;
#pragma unroll
      for (int o = 1; o < kViewBatch; o <<= 1) {
        const int up = __shfl_up(inc, o, kWave);
        if (lane >= o) inc += up;
      }
      if (lane < kViewBatch) s_base[lane] = inc - n;
      if (lane == kViewBatch - 1) s_base[kViewBatch] = inc;
    }
    __syncthreads();
    const int L = s_base[kViewBatch];
    const int nsteps = (L + kStepCells - 1) / kStepCells;
    if (used + nsteps > ws.quota) {   // uniform
      exhausted = true;
      break;
    }
    const int off = used;
    used += nsteps;

    // ---- C: chunks of the list -> weight matrix in LDS -> k-steps in global memory
    for (int c0 = 0; c0 < L; c0 += kChunk) {
      const int Lc = min(kChunk, L - c0);
      const int ksteps = (Lc + kStepCells - 1) / kStepCells;
      if (c0 > 0) __syncthreads();   // the previous chunk has been copied out
      for (int q = tid; q < kTilePts * ksteps * 2; q += kPrepThreads) {   // zero the matrix, 16 bytes per store
        const int row = q / (ksteps * 2), col = (q % (ksteps * 2)) * 8;
        const u32x4 z = {0u, 0u, 0u, 0u};
        *reinterpret_cast<u32x4*>(&s_whi[row][col]) = z;
        *reinterpret_cast<u32x4*>(&s_wlo[row][col]) = z;
      }
      // entries that pad the last k-step point at a cell that exists (their weights are zero)
      if (tid >= Lc && tid < ksteps * kStepCells) s_cell[tid] = (uint32_t)((ob.view_begin + vb0) * Hf * Wf) * row_bytes;
      __syncthreads();
      // weights and cells of every visible pair (a cell that several points touch gets the same value from each of
      // them; walking over the set bits of the maps instead kept a few threads busy for 4 K of a tile's 25 K cycles)
#pragma unroll
      for (int it = 0; it < kNIT; ++it) {
        if (pr[it].xy < 0) continue;
        const int vl = it * kSlots + slot;
        const int x0 = pr[it].xy & 0xffff, y0 = pr[it].xy >> 16;
        const float ax = pr[it].ax, ay = pr[it].ay;
        const bool has_x1 = x0 + 1 < Wf, has_y1 = y0 + 1 < Hf;
        const float wgt[4] = {(1.0f - ax) * (1.0f - ay), ax * (1.0f - ay), (1.0f - ax) * ay, ax * ay};
        const bool on[4] = {true, has_x1, has_y1, has_x1 && has_y1};
        int idx[4];
        if (s_mode[vl] == 1) {
          const int bit = (y0 - s_win[vl][1]) * kWinSide + (x0 - s_win[vl][0]);
          const int bs[4] = {bit, bit + 1, bit + kWinSide, bit + kWinSide + 1};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int b = on[k] ? bs[k] : bit;
            idx[k] = s_base[vl] + s_wbase[vl][b >> 5] + __popc(s_bits[vl][b >> 5] & ((1u << (b & 31)) - 1u)) - c0;
            if (on[k] && idx[k] >= 0 && idx[k] < Lc)
              s_cell[idx[k]] = (uint32_t)(((ob.view_begin + vb0 + vl) * Hf + y0 + (k >> 1)) * Wf + x0 + (k & 1)) * row_bytes;
          }
        } else {
          const int first = s_base[vl] + 4 * __popc(s_vmask[vl] & ((1u << p) - 1u)) - c0;
          const int cell0 = (ob.view_begin + vb0 + vl) * Hf;
          const int x1 = has_x1 ? x0 + 1 : x0, y1 = has_y1 ? y0 + 1 : y0;
          const int cx[4] = {x0, x1, x0, x1}, cy[4] = {y0, y0, y1, y1};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            idx[k] = first + k;
            if (idx[k] >= 0 && idx[k] < Lc) s_cell[idx[k]] = (uint32_t)((cell0 + cy[k]) * Wf + cx[k]) * row_bytes;
          }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (on[k] && idx[k] >= 0 && idx[k] < Lc) {
            uint16_t hi, lo;
            split_weight<DT>(wgt[k], hi, lo);
            s_whi[p][idx[k]] = hi;
            s_wlo[p][idx[k]] = lo;
          }
        }
      }
      __syncthreads();
      // copy out: per k-step 16 cell offsets and the two operand matrices (64 lanes x 16 bytes each)
      TileStep* __restrict__ out = ws.steps + slot0 + off + c0 / kStepCells;
      for (int q = tid; q < ksteps * 128; q += kPrepThreads) {
        const int s = q >> 7, part = (q >> 6) & 1, l = q & 63, g = l >> 5, m = l & 31;
        const uint16_t* src = part ? &s_wlo[m][kStepCells * s + 8 * g] : &s_whi[m][kStepCells * s + 8 * g];
        const u32x4 val = *reinterpret_cast<const u32x4*>(src);
        u32x4* dst = part ? &out[s].a_lo[l] : &out[s].a_hi[l];
        *reinterpret_cast<u32x4*>(dst) = val;
      }
      if (tid < ksteps * kStepCells) out[tid / kStepCells].cell[tid % kStepCells] = s_cell[tid];
    }
  }

  if (a.out_vis && tid < kTilePts && li0 + tid < ob.n_pts) {   // mask columns beyond the object's views
    for (int j = ob.n_views; j < a.vis_pitch; ++j) a.out_vis[(ob.pt_begin + li0 + tid) * a.vis_pitch + j] = 0;
  }
  __syncthreads();
  if (exhausted) {
    if (tid == 0) hdr->nsteps = -1;
    if (tid < kWave) push_tile(ws, ob.tile_begin + blk, blockIdx.y, lane);   // the product kernel fuses it by a gather
    return;
  }
  if (tid == 0) hdr->nsteps = used;
  if (tid < kTilePts) {
    hdr->cnt[tid] = s_cnt[tid];
    if (a.out_count && li0 + tid < ob.n_pts) a.out_count[ob.pt_begin + li0 + tid] = s_cnt[tid];
  }
}

// ------------------------------------------------------------------------------------ product

// What the prepare kernel wrote is constant for the product kernel: reading the tile header
// through the constant address space keeps the wave-uniform read on the scalar unit even inside
// the tile loop, where the compiler must otherwise assume that the stores of fused rows alias it.
typedef const uint32_t __attribute__((address_space(4))) * const_words;

__device__ __forceinline__ int load_nsteps(const TileHdr* h) {
  return (int)((const_words)(uintptr_t)&h->nsteps)[0];
}

// A tile's k-steps are staged in LDS before they are used (two buffers of kStage k-steps): the
// weight operands were written by the prepare kernel and come from far memory, the copy for the
// next tile is issued when the current tile starts and is hidden behind it.  The copy is a
// direct global -> LDS load (no registers): one instruction moves 64 x 16 contiguous bytes.
//
// The copy instruction is written as inline assembly on purpose.  Issued through the compiler's
// builtin, a copy that is still in flight makes every later wait for a vector read a wait for ALL
// outstanding reads (the compiler cannot tell which LDS reads the copy may feed), which serialises
// the row reads of the product loop.  Hidden from that bookkeeping, the copies only make the
// hardware counter larger than the compiler assumes; reads complete in order, so its waits remain
// sufficient.  The workgroup waits for the copies explicitly (wait_copies) before the barrier that
// publishes a buffer.
// The one-kernel form's stage: what fits LDS beside the rest with as many workgroups per compute unit as the registers
// allow (see fused_waves_per_simd), so that few tiles outgrow it (with 4, 8 and 16 k-steps for 256, 512 and
// more channels, 123 457 points of 11 views took 469 us, 200 000 of 8 views and 256 channels 1080 us; 197 and 187 us now).
template <int S, int NP, bool SC>
constexpr int fused_stage_steps() {
  constexpr int waves = S + NP + (SC ? 1 : 0);
  return waves > 4 ? 32 : (S == 1 ? 8 : (S == 2 ? (SC ? 12 : 16) : 16));
}

template <int S>
constexpr int stage_steps_for() { return S == 1 ? 4 : (S == 2 ? 8 : 16); }   // S: units of 256 channels   // keeps 8 waves per compute unit in LDS

__device__ __forceinline__ void copy_64x16(const char* g, char* lds) {
  // m0 = LDS byte address of the 1 KiB piece; lane l's 16 bytes land at m0 + 16 l
  const uint32_t lds_addr = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds);
  uint32_t saved_m0;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, off\n\ts_mov_b32 m0, %0"
               : "=&s"(saved_m0) : "s"(lds_addr), "v"(g) : "memory");
}

__device__ __forceinline__ void wait_copies() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

template <int S>
__device__ __forceinline__ void stage_steps(char* lds, const TileStep* __restrict__ src, int nsteps, int span, int lane) {
  const int bytes = nsteps * (int)sizeof(TileStep);
  const char* g = reinterpret_cast<const char*>(src);
  for (int piece = span; piece * 1024 < bytes; piece += S) {
    const int off = piece * 1024 + lane * 16;
    if (off < bytes) copy_64x16(g + off, lds + piece * 1024);
  }
}

__device__ __forceinline__ void lds_a(const char* lds, int k, int lane, StepA& r) {
  const TileStep* st = reinterpret_cast<const TileStep*>(lds) + k;
  r.hi = st->a_hi[lane];
  r.lo = st->a_lo[lane];
}

__device__ __forceinline__ void lds_c(const char* lds, int k, int g, StepC& r) {
  const TileStep* st = reinterpret_cast<const TileStep*>(lds) + k;
  r.lo = *reinterpret_cast<const u32x4*>(&st->cell[8 * g]);
  r.hi = *reinterpret_cast<const u32x4*>(&st->cell[8 * g + 4]);
}

template <int H>
__device__ __forceinline__ void load_q(const char* __restrict__ feat, const StepC& c, uint32_t lane_off, StepQ<H>& r) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const uint32_t cell = e < 4 ? c.lo[e] : c.hi[e - 4];
#pragma unroll
    for (int h = 0; h < H; ++h) r.q[h][e] = *reinterpret_cast<const u32x2*>(feat + (cell + lane_off + h * kHalf * 2));
  }
}

// Sums of squares of the wave's channels per point: one for each of its pieces of 128 channels, in ss.  (A sum per piece, so that
// the norm's additions do not depend on how the channels are dealt out to waves.)
template <int H>
__device__ __forceinline__ void piece_squares(const f32x16 (&acc)[4 * H], int lane, float (*ss)[kTilePts]) {
  float v[16 * H];
#pragma unroll
  for (int h = 0; h < H; ++h)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float sq = 0.0f;
#pragma unroll
      for (int t = 4 * h; t < 4 * h + 4; ++t) sq = __builtin_fmaf(acc[t][r], acc[t][r], sq);
      v[16 * h + r] = sq;
    }
  const float sum = half_wave_sums<H>(v, lane);
  const int i = lane_value<H>(lane & 31), r = i & 15;
  ss[i >> 4][8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)] = sum;
}

struct ProdArgs {
  const char* feat;
  int D;
  const TileHdr* hdr;
  const TileStep* steps;
  unsigned* counters;   // [objects of the launch][8]
  int quota;
  float* fused;
  float* factor;        // [N] or nullptr: what each point's raw tile product was multiplied by
  float norm_eps;
  int mean_only;
  int pace;             // k_tile_fused: shortest time between two tiles of a workgroup, in ticks of the 100 MHz counter
  int given_groups;     // k_tile_fused: the first workgroups of the launch, which begin with tiles that they need not ask for
  const unsigned* unlisted;   // k_tile_fused, may be nullptr: the word that holds kAllSeen where this launch has anything to do
};

// DT: 1 bf16, 2 fp16 feature maps.  S waves per workgroup, each owning H pieces of 128 channels:
// D == 128 * H * S.  PF: k-steps whose cell rows are requested ahead of their products.
//
// A workgroup walks over several tiles.  While a tile is multiplied, the k-steps of the next one
// are copied into the other LDS buffer; per k-step the weight operands and cell offsets come from
// LDS and the cell rows (shared with the neighbouring tiles, so mostly L2 hits) are read PF
// k-steps ahead of their product.  The k-steps are taken in groups of PF without a branch inside, so
// that the wait counters before each product allow for exactly the reads issued after its operands.
// A tile has one barrier (after its products); nothing in the tile loop waits for a round trip to memory
// that was started in the same tile:
//   * the ticket of a tile (see below) is asked for three tiles ahead,
//   * the length of its list is read two tiles ahead (a vector read: a scalar read would share its
//     counter with the LDS reads and stall them),
//   * its k-steps are copied one tile ahead,
//   * its first rows are requested right after the previous tile's stores.
// Memory operations inside the loop are unconditional (reads for a tile that does not exist go to cell 0,
// stores of rows that do not exist are dropped by the buffer bounds check): behind a branch the compiler
// has to assume the worst about outstanding operations and waits for all of them.
//
// Tile order: the workgroups with the same id modulo 8 run on the same XCD; XCD c owns one
// contiguous range of the object's tiles and its workgroups take the next tile of that range from
// a counter (tiles differ in length, a fixed split leaves a tail), so that at any time the tiles in
// flight on an XCD are neighbours and share cell rows in its L2.
constexpr int kProdGroupsMax = 768;   // two workgroups fit a compute unit at a time; the rest take over as the first run out of tiles

// The opening reads of a tile whose k-steps are staged at `sb` (n of them, possibly none): the rows of its
// first PF k-steps and the weights of its first k-step.  With nothing staged the reads go to cell 0 and are
// not used.
template <int H, int PF>
__device__ __forceinline__ void open_tile(const char* sb, int n_staged, const char* __restrict__ feat, uint32_t lane_off,
                                          int lane, int g, StepA (&wa)[2], StepQ<H> (&rq)[PF]) {
  const uint32_t on = n_staged > 0 ? 0xffffffffu : 0u;
  const int l0 = max(n_staged - 1, 0);
#pragma unroll
  for (int j = 0; j < PF; ++j) {
    StepC c;
    lds_c(sb, min(j, l0), g, c);
    c.lo &= on;
    c.hi &= on;
    load_q(feat, c, lane_off, rq[j]);
  }
  lds_a(sb, 0, lane, wa[0]);
}

template <int DT, int S, int H, int PF>
__global__ __launch_bounds__(kWave* S) __attribute__((amdgpu_waves_per_eu(H == 1 ? 3 : 2, H == 1 ? 3 : 2)))
void k_tile_product(FuseArgs fa, ProdArgs a, TileWs ws, ObjTable tab) {
  constexpr int kSpan = kHalf * H;   // channels per wave
  constexpr int kStage = stage_steps_for<S * H / 2>();
  __shared__ __attribute__((aligned(16))) char s_steps[2][kStage * sizeof(TileStep)];
  __shared__ float s_ss[2][S * H][kTilePts];   // [tile parity]: a wave may write the next tile's sums while another still reads
  __shared__ int s_take[2];
  __shared__ int s_job[4];   // see drain_tiles

  const ObjRange ob = tab.o[blockIdx.y];
  const int nblk = (ob.n_pts + kTilePts - 1) / kTilePts;
  const int groups = min(nblk, (int)gridDim.x);   // workgroups that work on this object
  if ((int)blockIdx.x >= groups) return;
  // The XCD's tiles and its counter (see XcdTiles: chunks of consecutive tiles taken in turn by the XCDs).
  const int xcd = blockIdx.x % kXcd;
  const XcdTiles mine(nblk, xcd);
  const int len = mine.len;
  auto tile_at = [&](int t) { return mine.at(t); };
  unsigned* __restrict__ ctr = a.counters + blockIdx.y * kXcd + xcd;
  const TileHdr* __restrict__ hdrs = a.hdr + ob.tile_begin;

  const int tid = threadIdx.x, lane = tid % kWave;
  const int span = __builtin_amdgcn_readfirstlane(tid / kWave);   // wave index: uniform, kept in a scalar register
  const int m = lane & 31, g = lane >> 5;
  const int D = a.D;
  const uint32_t lane_off = (uint32_t)(span * kSpan + 4 * m) * 2u;   // byte offset of the lane's first piece

  StepA wa[2];      // weight operands of the current and the next k-step
  StepC wc;         // cell offsets of the k-step whose rows are requested next
  StepQ<H> rq[PF];  // cell rows of the next PF k-steps

  // The first three tiles.  In the loop, a tile's ticket is asked for three tiles ahead, the length of its
  // list is read two tiles ahead and its k-steps are copied one tile ahead, so that none of the three
  // round trips is waited for.
  if (tid == 0) s_take[0] = (int)atomicAdd(ctr, 3u);
  const unsigned gathered = ws.status[1];   // tiles on the lists: the prepare kernel has pushed them all, and where there are
                                            // none nobody looks (a look at the end cost 2 us of 45)
  __syncthreads();
  const int t0 = s_take[0];
  int blk = t0 < len ? tile_at(t0) : -1;
  int nxt = t0 + 1 < len ? tile_at(t0 + 1) : -1;    // -1: no further tile
  int nxt2 = t0 + 2 < len ? tile_at(t0 + 2) : -1;
  int buf = 0;
  int n = blk >= 0 ? load_nsteps(hdrs + blk) : 0;
  int n_next = nxt >= 0 ? load_nsteps(hdrs + nxt) : 0;
  int pend_n = hdrs[max(nxt2, 0)].nsteps;   // list length of the tile after the next, picked up one tile later
  stage_steps<S>(s_steps[0], a.steps + (long long)(ob.tile_begin + max(blk, 0)) * a.quota, min(max(n, 0), kStage), span, lane);
  wait_copies();
  __syncthreads();
  open_tile<H, PF>(s_steps[0], min(max(n, 0), kStage), a.feat, lane_off, lane, g, wa, rq);

  while (blk >= 0) {
    const TileStep* __restrict__ st = a.steps + (long long)(ob.tile_begin + blk) * a.quota;
    // ask for the tile three tiles ahead (the answer is picked up after this tile's products)
    int asked = 0;
    if (tid == 0 && nxt2 >= 0) asked = (int)atomicAdd(ctr, 1u);
    // the next tile's k-steps go to the other buffer while this tile is multiplied
    stage_steps<S>(s_steps[buf ^ 1], a.steps + (long long)(ob.tile_begin + max(nxt, 0)) * a.quota,
                   nxt >= 0 ? min(max(n_next, 0), kStage) : 0, span, lane);
    const int my_cnt = hdrs[blk].cnt[tid % kTilePts];   // views that see point (lane % 32) of this tile

    f32x16 acc[4 * H];
#pragma unroll
    for (int t = 0; t < 4 * H; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[t][r] = 0.0f;

    const char* sb = s_steps[buf];
    for (int base = 0; base < n; base += kStage) {
      const int cnt = min(kStage, n - base), l0 = cnt - 1;
      if (base > 0) {
        // a tile with more k-steps than a buffer holds (rare): refill the buffer in place
        __syncthreads();
        stage_steps<S>(s_steps[buf], st + base, cnt, span, lane);
        wait_copies();
        __syncthreads();
        open_tile<H, PF>(sb, cnt, a.feat, lane_off, lane, g, wa, rq);
      }
      // k-steps in groups of PF without a branch inside: rows of k-step s + j + PF are requested right after
      // the products of k-step s + j have freed their registers (requests past the end repeat the last k-step)
      int s = 0;
      for (; s + PF <= cnt; s += PF) {
#pragma unroll
        for (int j = 0; j < PF; ++j) {
          lds_c(sb, min(s + j + PF, l0), g, wc);
          lds_a(sb, min(s + j + 1, l0), lane, wa[(j + 1) & 1]);
          mma_step<DT, H>(wa[j & 1], rq[j], acc);
          __builtin_amdgcn_sched_barrier(0);   // keep the reads behind the products that free their registers
          load_q(a.feat, wc, lane_off, rq[j]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // the last cnt - s < PF k-steps: their rows are there (or on the way), nothing more to request
#pragma unroll
      for (int j = 0; j < PF - 1; ++j) {
        if (s + j < cnt) {
          lds_a(sb, min(s + j + 1, l0), lane, wa[(j + 1) & 1]);
          mma_step<DT, H>(wa[j & 1], rq[j], acc);
        }
      }
    }

    // ---- sums of squares of the wave's channels, per point
    piece_squares<H>(acc, lane, &s_ss[buf][span * H]);
    if (tid == 0) s_take[buf] = asked;
    const int n_next2 = __builtin_amdgcn_readfirstlane(pend_n);
    wait_copies();
    __syncthreads();   // the one barrier of a tile: sums, ticket and the next tile's k-steps are in LDS; every
                       // wave is done with this tile's buffer

    // the tile three ahead: its list length is requested now and read after the next tile's products
    const int t3 = s_take[buf];
    const int nxt3 = (nxt2 >= 0 && t3 < len) ? tile_at(t3) : -1;
    pend_n = hdrs[max(nxt3, 0)].nsteps;

    // ---- mean and L2 norm: one factor per point, inv_count / max(norm of the mean, eps), applied to the raw
    // sums.  Lane l of every wave computes the factor of point l % 32; a lane fetches the factors of its 16
    // rows from those lanes.
    float factor;
    {
      float tot = 0.0f;
#pragma unroll
      for (int w = 0; w < S * H; ++w) tot += s_ss[buf][w][m];
      factor = point_factor(my_cnt, tot, a.norm_eps, a.mean_only);
    }
    {   // the factor of every point of the tile, for the scoring kernel (lanes 0..31 of the first wave; all
        // other lanes, and every lane when no factor array was given, fall outside the buffer)
      const int rows_f = a.factor ? min(kTilePts, ob.n_pts - blk * kTilePts) : 0;
      const __amdgpu_buffer_rsrc_t fout = __builtin_amdgcn_make_buffer_rsrc(a.factor + (a.factor ? ob.pt_begin + blk * kTilePts : 0), 0,
                                                                            rows_f * 4, 0x00020000);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(factor), fout, tid < kTilePts ? 4 * tid : 0x7ffffff0, 0, 0);
    }
    {
      // Buffer stores: the wave's part of the tile (rows of D floats, starting at a wave-uniform
      // address) is described by a buffer resource whose size covers the rows that exist, so a lane
      // only needs one 32-bit offset register and rows beyond the object's last point (or all rows, for
      // a tile without k-steps: n < 0, see push_tile) are dropped by the bounds check instead of by
      // branches.
      const int li0 = blk * kTilePts;
      float* obase = a.fused ? a.fused + (ob.pt_begin + li0) * D + span * kSpan : nullptr;
      uint32_t row_bytes = (uint32_t)D * 4u;
      // opaque to the optimiser: otherwise the 32 per-row offsets below, which do not change from tile
      // to tile, are kept in registers across the whole tile loop and push other values into scratch
      asm volatile("" : "+s"(row_bytes));
      const int rows = (n >= 0 && a.fused) ? min(kTilePts, ob.n_pts - li0) : 0;   // no rows wanted: every store is dropped
      const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(obase, 0, (int)(rows * row_bytes), 0x00020000);
      const uint32_t lane_out = (uint32_t)(4 * g) * row_bytes + (uint32_t)(4 * m) * 4u;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row0 = 8 * (r >> 2) + (r & 3);
        const float scale = __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (row0 + 4 * g), __float_as_int(factor)));
#pragma unroll
        for (int h = 0; h < H; ++h) {
          const f32x4 v = {acc[4 * h][r] * scale, acc[4 * h + 1][r] * scale, acc[4 * h + 2][r] * scale, acc[4 * h + 3][r] * scale};
          // the scalar-offset operand stays 0: with a register there, a store directly followed by
          // an instruction that overwrites its data registers was seen to write stale lanes
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), out,
                                                 (int)(lane_out + (uint32_t)row0 * row_bytes) + h * kHalf * 4, 0, /*streaming*/ 2);
        }
      }
    }
    // The next tile's opening reads.  They are issued after the stores: the counter of outstanding memory
    // operations is in order, and with the stores behind them the compiler's wait before the first product
    // would cover every read at once instead of one k-step at a time.
    __builtin_amdgcn_sched_barrier(0);
    open_tile<H, PF>(s_steps[buf ^ 1], nxt >= 0 ? min(max(n_next, 0), kStage) : 0, a.feat, lane_off, lane, g, wa, rq);

    blk = nxt;
    nxt = nxt2;
    nxt2 = nxt3;
    n = n_next;
    n_next = n_next2;
    buf ^= 1;
  }
  if (gathered != 0u) drain_tiles<DT, true, kGatherSweeps>(fa, ws, tab, blockIdx.y * gridDim.x + blockIdx.x, s_job, span, S, lane);
}

// ------------------------------------------------------------------------------------ one kernel
//
// k_tile_fused: the product kernel with one more wave per workgroup, the producer, that does the prepare kernel's work
// for the workgroup's NEXT tile while the S product waves multiply the current one.  The producer writes the k-steps
// straight into the other LDS buffer, in the layout the product waves read (no trip through memory, unless the scoring
// kernel wants them), so the projection -> depth read -> list -> weight chain of a tile hides behind the stores of the
// tile before it.  The tile's one barrier is shared: after it the buffer the products came from belongs to the producer
// and the buffer it filled belongs to the product waves.  The producer has no barrier of its own: it is one wave, and
// orders its LDS traffic with wave-level fences.  Tiles go to workgroups through the per-XCD counters as before; the
// producer asks for a ticket one tile ahead.  A tile whose list does not fit the buffer goes to the list of push_tile.

constexpr int kPBatch = 16;   // views per pass of the producer waves, at most: two per trip, one per half wave
constexpr int kMaxProducers = 4;
constexpr int kCamRows = 32;  // camera rows of the object kept in LDS for the producer
constexpr int kOneKernelViews = 8;
// A single producer is launched for up to kOneKernelViews views, so it makes four trips.  (With the eight of a full pass, of which
// the last four were never made, what a trip holds was kept for all of them and the compiler's code was the longer for it: single
// pass over 40 objects of 50 000 points and two to four views 660 -> 617 us, 64 of 100 000 and 4 views 1796 -> 1554, with rows as
// before.)
template <int NP>
constexpr int kPassViews = NP == 1 ? kOneKernelViews : kPBatch;

typedef const float __attribute__((address_space(3))) * lds_floats;

struct ProducerScratch {
  // (the rows' pitches keep 16-byte pieces aligned and put the same row of all views into different LDS banks)
  uint32_t bits[kPBatch][kWinSide + 4];   // map of touched cells per view, row = word
  uint16_t wbase[kPBatch][kWinSide + 8];  // set bits before each row
  int base[kPBatch + 1];              // first list index of each view
  int win[kPBatch][2];
  int mode[kPBatch];
  uint32_t vmask[kPBatch];
};

template <int NP>
struct TileSlot {    // what the product waves need to know about a staged tile
  int tile;          // index within the object; -1: no further tile
  int nsteps;        // -1: no k-steps, see push_tile
  int pad_[2];
  int cnt[NP][kTilePts];   // views that see each point, per producer wave
  uint32_t vmask[kCamRows];           // per view of the object: which of the tile's 32 points it sees (Eq. 1)
};

// The point that lane `lane` of a producer wave handles in tile `blk` (lane % 32; the tile's first point where the
// object has no such point).
__device__ __forceinline__ float3 tile_point(const FuseArgs& a, const ObjRange& ob, int blk, int lane) {
  const int p = lane & 31, li0 = blk * kTilePts;
  const long long ip = ob.pt_begin + li0 + (li0 + p < ob.n_pts ? p : 0);
  return float3{a.xyz[3 * ip], a.xyz[3 * ip + 1], a.xyz[3 * ip + 2]};
}

// Meeting point of the NP producer waves of a workgroup (the workgroup barrier belongs to the tile hand-over, which
// the product waves take part in).  Every wave publishes the number of the meeting after its LDS traffic and waits
// until the others have published it too; both producers pass the same meetings in the same order.  The wait is
// bounded: a producer that never arrives (a programming error) ends in wrong results, not in a hung machine - and in
// a set bit in the call's status word (TileWs::status), which the host can read back, so that wrong results never
// go unnoticed.  The waiting waves look again as soon as the last look is back (no sleep in between: the meeting is
// on the tile's critical path, and a look is one LDS read for all four flags).
// The flags are reached through a pointer that says LDS.  Through a generic pointer these volatile accesses compile to
// flat instructions, and a flat read is only complete when every global read of the wave in flight is too (the next
// tile's points, depth texels): each look then cost a round trip to memory, some thousands of cycles per tile.
constexpr unsigned kStatusMeetingMissed = 1u;
typedef volatile int __attribute__((address_space(3))) * lds_flags;

template <int NP>
__device__ __forceinline__ void producers_meet(lds_flags flags, int w, int& seq, int lane, unsigned* status) {
  wave_sync();
  if constexpr (NP > 1) {
    ++seq;
    if (lane == 0) flags[w] = seq;
    static_assert(NP <= 4, "the four flags are read as one 16-byte vector");
    typedef int flags4 __attribute__((ext_vector_type(4)));
    typedef const volatile flags4 __attribute__((address_space(3))) * lds_flags4;
    bool all = false;
    for (int spins = 0; spins < (1 << 16) && !all; ++spins) {
      const flags4 f = *(lds_flags4)flags;   // one LDS round trip per look
      all = true;
#pragma unroll
      for (int o = 0; o < NP; ++o) all = all && (f[o] - seq >= 0);
    }
    if (!all && lane == 0) atomicOr(status, kStatusMeetingMissed);
    wave_sync();
  }
}

// What a producer wave knows about its pairs of one batch of views before the tests: projection, whether it lands in
// the image, the depth texel (requested, maybe still on its way) and, with a given selection, whether the view is kept.
template <int NP>
struct ProjectedBatch {
  Proj pj[kPassViews<NP> / 2 / NP];
  float dep[kPassViews<NP> / 2 / NP];
  bool fr[kPassViews<NP> / 2 / NP], kept[kPassViews<NP> / 2 / NP];
};

// First every projection and the request for its depth texel (and mask byte), nothing that waits for them: a wave has
// nobody to hide a read behind, so the reads of all its pairs are in flight together - and, for the first batch of a
// tile, while the wave still works on the tile before.
template <bool SEL, int NP>
__device__ __forceinline__ void project_batch(const FuseArgs& a, const ObjRange& ob, int blk, float3 pt, int vb0,
                                              lds_floats cam_lds, int w, int lane, ProjectedBatch<NP>& f) {
  constexpr int kTrips = kPassViews<NP> / 2 / NP;
  const int p = lane & 31, h = lane >> 5;
  const int nvb = min(kPassViews<NP>, ob.n_views - vb0);
  const int li0 = blk * kTilePts;
  const long long ip = ob.pt_begin + li0 + (li0 + p < ob.n_pts ? p : 0);
#pragma unroll
  for (int j = 0; j < kTrips; ++j) {
    const int it = w + NP * j;
    f.dep[j] = 1.0f;
    f.fr[j] = false;
    f.kept[j] = true;
    f.pj[j] = Proj{0.0f, 0.0f, 0.0f};
    if (2 * it >= nvb) break;   // uniform
    const int vl = min(2 * it + h, nvb - 1);
    const int v = ob.view_begin + vb0 + vl;
    // the camera rows come from the LDS copy, through a pointer that says so: a generic read would wait for every
    // read in flight, the depth texels of the trips before included
    f.pj[j] = project(cam_lds + (vb0 + vl) * 16, pt.x, pt.y, pt.z);
    f.fr[j] = in_frustum(a.vis, f.pj[j]);
    if (a.vis.depth) f.dep[j] = a.vis.depth[(long long)v * a.vis.H * a.vis.W + (f.fr[j] ? depth_texel(a.vis, f.pj[j]) : 0)];
    if constexpr (SEL) f.kept[j] = view_kept(a, ip, vb0 + vl);
  }
}

// Builds tile `blk` of object `ob` into `stage` (room for `k_stage` k-steps) and `slot`.  pt: the lane's point; pre:
// the projected first batch of views (project_batch).  Called by all 64 lanes of
// each of the NP producer waves (w = 0 .. NP - 1), which share the views of the tile: wave w takes the trips
// it = w, w + NP, ... (two views per trip, one per half wave).  cam_lds: the object's camera rows in LDS.
// Bound by its own chain: a producer is one wave, and what a tile costs it is instructions and LDS round trips, one behind the
// other (of 10 to 17 K cycles per tile, a quarter goes to projections and depth texels, a quarter to cells and weights).  Hence
// two cells of a row are marked, and looked up, together; the rows of a map, of which the first few hold everything, are dealt
// out to waves and lanes in turn; trips beyond the object's views end the loop; views that see nothing of the tile stop before
// the list; and the depth texels of the next batch of views are requested while this one is worked on.  Together: 1.68 M voxels
// of 24 views, nine tiles of ten seen by nobody, single pass 1352 -> 1179 us; 40 objects of 50 000 points and two to four views
// 716 -> 680; 64 objects of 100 000 points and 4 views with rows 2997 -> 2933; 200 000 points of 16 views with rows 245 -> 241;
// 123 457 points of 11 views 190 -> 186.  (The same in k_tile_prepare was slower: 1 M points of 32 views 1615 -> 1644 us.)
template <int DT, bool SEL, int NP>
__device__ __forceinline__ void produce_tile(const FuseArgs& a, const ObjRange& ob, int blk,
                                             float3 pt, ProjectedBatch<NP>& pre, char* stage, int k_stage, int& dirty,
                                             TileSlot<NP>* slot, ProducerScratch* sc, lds_floats cam_lds, lds_flags flags,
                                             const TileWs& ws, int obj, int* pushed, int w, int& seq, int lane) {
  unsigned* status = ws.status;
  constexpr int kTrips = kPassViews<NP> / 2 / NP;   // trips of one wave per batch of views
  const int p = lane & 31, h = lane >> 5;
  const int Hf = a.feat.Hf, Wf = a.feat.Wf;
  const uint32_t row_bytes = (uint32_t)a.feat.D * 2u;
  const int li0 = blk * kTilePts;
  const bool p_valid = li0 + p < ob.n_pts;
  TileStep* st = reinterpret_cast<TileStep*>(stage);
  int used = 0, cnt = 0;
  bool exhausted = false;

  // zero weights, shared by the waves: complete for everybody at the first meeting, before any weight lands.  Only
  // the k-steps that the buffer's last tile wrote (`dirty` of them) can hold anything but zeros.
  for (int q = w * kWave + lane; q < dirty * 128; q += NP * kWave)
    reinterpret_cast<u32x4*>(reinterpret_cast<char*>(&st[q >> 7]) + 64)[q & 127] = u32x4{0u, 0u, 0u, 0u};

  for (int vb0 = 0; vb0 < ob.n_views; vb0 += kPassViews<NP>) {
    const int nvb = min(kPassViews<NP>, ob.n_views - vb0);
    if (vb0 > 0) producers_meet<NP>(flags, w, seq, lane, status);   // the previous batch is done with the tables
    // the maps of this wave's views (view 2 it + h of trip it): 32 words each
#pragma unroll
    for (int j = 0; j < kTrips; ++j) {
      const int it = w + NP * j;
      if (2 * it >= nvb) break;   // uniform
      reinterpret_cast<u32x4*>(&sc->bits[2 * it + ((lane >> 3) & 1)][0])[lane & 7] = u32x4{0u, 0u, 0u, 0u};
    }
    wave_sync();

    // ---- A: project and test; bounding box of the touched cells per view.  The projections and the requests for the
    // depth texels of the first batch were made a tile ago (project_batch), those of a later batch behind the tests of
    // the batch before it.
    PairRec pr[kTrips];
    Proj (&pj)[kTrips] = pre.pj;
    float (&dep)[kTrips] = pre.dep;
    bool (&fr)[kTrips] = pre.fr, (&kept)[kTrips] = pre.kept;
#pragma unroll
    for (int j = 0; j < kTrips; ++j) {
      const int it = w + NP * j;
      pr[j].xy = -1;
      pr[j].ax = pr[j].ay = 0.0f;
      if (2 * it >= nvb) break;   // uniform
      const int vl = 2 * it + h;
      const bool seen = vl < nvb && p_valid && fr[j] && kept[j] && (a.vis.frustum_only || passes_depth(a.vis, pj[j], dep[j]));
      s16x2 lo2 = {0x7fff, 0x7fff}, hi2 = {-1, -1};
      if (seen) {
        const Tap tx = tap_axis(pj[j].u, a.feat.pitch_x, Wf), ty = tap_axis(pj[j].v, a.feat.pitch_y, Hf);
        pr[j].ax = tx.a;
        pr[j].ay = ty.a;
        pr[j].xy = (ty.i0 << 16) | tx.i0;
        lo2 = s16x2{(short)tx.i0, (short)ty.i0};
        hi2 = s16x2{(short)tx.i1, (short)ty.i1};
        ++cnt;
      }
      const unsigned long long seen_mask = __ballot(seen);
      lo2 = half_wave_reduce<true>(lo2);
      hi2 = half_wave_reduce<false>(hi2);
      if (p == kTilePts - 1 && vl < nvb) {
        const bool any = hi2[0] >= 0;
        const int ww = hi2[0] - lo2[0] + 1, wh = hi2[1] - lo2[1] + 1;
        sc->win[vl][0] = lo2[0];
        sc->win[vl][1] = lo2[1];
        sc->mode[vl] = !any ? 0 : (ww <= kWinSide && wh <= kWinSide ? 1 : 2);
        sc->vmask[vl] = (uint32_t)(seen_mask >> (lane & 32));
      }
    }
    wave_sync();
    // the next batch's depth texels arrive while this batch's lists and weights are made
    if (vb0 + kPassViews<NP> < ob.n_views) project_batch<SEL, NP>(a, ob, blk, pt, vb0 + kPassViews<NP>, cam_lds, w, lane, pre);

    // ---- B: mark the touched cells of this wave's views that use a map: two cells of a row at a time (a map is as wide as
    // a row, so the second one is in the same word)
#pragma unroll
    for (int j = 0; j < kTrips; ++j) {
      if (2 * (w + NP * j) >= nvb) break;   // uniform
      if (pr[j].xy < 0) continue;
      const int vl = 2 * (w + NP * j) + h;
      if (sc->mode[vl] != 1) continue;
      const int x0 = pr[j].xy & 0xffff, y0 = pr[j].xy >> 16;
      const int my = y0 - sc->win[vl][1], mx = x0 - sc->win[vl][0];
      const uint32_t cells = (x0 + 1 < Wf ? 3u : 1u) << mx;
      atomicOr(&sc->bits[vl][my], cells);
      if (y0 + 1 < Hf) atomicOr(&sc->bits[vl][my + 1], cells);
    }
    producers_meet<NP>(flags, w, seq, lane, status);   // the maps, boxes and masks of all views are complete

    // the mask of Eq. 1 for this batch of views goes out with the tile: a product wave writes it to memory (a store
    // of a producer would hold up its next wait for a read: one counter covers both)
    if (w == 0 && a.out_vis && lane < nvb) slot->vmask[vb0 + lane] = sc->vmask[lane];
    // views that see none of the tile's points have no cells: no list, no k-steps (uniform, the same in every producer wave)
    if (__ballot(lane < nvb && sc->mode[lane] != 0) == 0) continue;
    {   // list length of every view, exclusive scan over the views: every producer wave does it (same values).
        // lane = (view, quarter of the map's rows): set bits before each row within the quarter, then the quarters'
        // totals through lane exchanges
      static_assert(kPBatch == 16 && kWinSide == 32, "lane = 16 views x 4 quarters of 8 rows");
      const int v = lane & 15, qd = lane >> 4;
      const bool map = v < nvb && sc->mode[v] == 1;
      int before[8], n = 0;
      const u32x4 rows[2] = {*reinterpret_cast<const u32x4*>(&sc->bits[v][8 * qd]), *reinterpret_cast<const u32x4*>(&sc->bits[v][8 * qd + 4])};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        before[e] = n;
        n += map ? __popc(rows[e >> 2][e & 3]) : 0;
      }
      const int n0 = __shfl(n, v, kWave), n1 = __shfl(n, v + 16, kWave), n2 = __shfl(n, v + 32, kWave), n3 = __shfl(n, v + 48, kWave);
      const int off = (qd > 0 ? n0 : 0) + (qd > 1 ? n1 : 0) + (qd > 2 ? n2 : 0);
      if (map) {
        u32x4 pairs;
#pragma unroll
        for (int e = 0; e < 4; ++e) pairs[e] = (uint32_t)(off + before[2 * e]) | (uint32_t)(off + before[2 * e + 1]) << 16;
        *reinterpret_cast<u32x4*>(&sc->wbase[v][8 * qd]) = pairs;
      }
      int total = n0 + n1 + n2 + n3;                                   // lanes 0 .. 15: the view's list length
      if (v < nvb && sc->mode[v] == 2) total = 4 * __popc(sc->vmask[v]);
      // running sum over the 16 views = over the first row of 16 lanes, with lane shifts inside the row (a lane without
      // a source adds 0): no trip through the LDS unit, which every exchange between arbitrary lanes would cost
      int inc = lane < kPBatch ? total : 0;
      inc = row_shift_add<0x111>(inc);   // row_shr:1
      inc = row_shift_add<0x112>(inc);   // row_shr:2
      inc = row_shift_add<0x114>(inc);   // row_shr:4
      inc = row_shift_add<0x118>(inc);   // row_shr:8
      if (lane < kPBatch) sc->base[lane] = inc - total;
      if (lane == kPBatch - 1) sc->base[kPBatch] = inc;
    }
    wave_sync();
    const int L = sc->base[kPBatch];
    const int nsteps = (L + kStepCells - 1) / kStepCells;
    if (used + nsteps > k_stage) {   // uniform, and the same in every producer wave
      exhausted = true;
      break;
    }
    TileStep* __restrict__ out = st + used;
    used += nsteps;

    // ---- C: the cells of the list, then the weights in the operand layout
    if (w == 0 && lane < nsteps * kStepCells - L) {   // entries that pad the last k-step point at a cell that exists
      const int idx = L + lane;
      out[idx >> 4].cell[idx & 15] = (uint32_t)((ob.view_begin + vb0) * Hf * Wf) * row_bytes;
    }
    {   // cells of the views with a map.  A map holds a few rows from its first one on, so the rows go to waves and lanes in
        // turn: wave w has rows w, w + NP, ..., and every view 4, 8 or 16 lanes that take those in turn
      constexpr int kWaveRows = kWinSide / NP, kRows = kWaveRows / 4;   // kRows: per lane, with four lanes per view
      const int lg = nvb <= 4 && kWaveRows >= 16 ? 4 : (nvb <= 8 ? 3 : 2);   // uniform
      const int vl = lane >> lg, first = lane & ((1 << lg) - 1);
      if (vl < nvb && sc->mode[vl] == 1) {
        const int cell0 = (ob.view_begin + vb0 + vl) * Hf + sc->win[vl][1], wx = sc->win[vl][0], base = sc->base[vl];
        uint32_t rows[kRows];
#pragma unroll
        for (int e = 0; e < kRows; ++e) {
          const int r = first + (e << lg);
          rows[e] = r < kWaveRows ? sc->bits[vl][w + NP * r] : 0u;
        }
#pragma unroll
        for (int e = 0; e < kRows; ++e) {
          uint32_t bits = rows[e];
          if (bits == 0u) continue;
          const int wd = w + NP * (first + (e << lg));
          int q = base + sc->wbase[vl][wd];
          while (bits) {
            const int bit = __builtin_ctz(bits);
            bits &= bits - 1;
            out[q >> 4].cell[q & 15] = (uint32_t)((cell0 + wd) * Wf + wx + bit) * row_bytes;
            ++q;
          }
        }
      }
    }
    // list positions of the four cells of every pair first (LDS reads only), then the stores: with both in one loop
    // the reads of a pair would wait behind the stores of the pair before it
    int idx[kTrips][4];
#pragma unroll
    for (int j = 0; j < kTrips; ++j) {
#pragma unroll
      for (int k = 0; k < 4; ++k) idx[j][k] = 0;
      if (2 * (w + NP * j) >= nvb) break;   // uniform
      if (pr[j].xy < 0) continue;
      const int vl = 2 * (w + NP * j) + h;
      const int x0 = pr[j].xy & 0xffff, y0 = pr[j].xy >> 16;
      if (sc->mode[vl] == 1) {
        // (the second cell of a row directly follows the first in the list; at the border it has no place and is not used)
        const int my = y0 - sc->win[vl][1], mx = x0 - sc->win[vl][0], my1 = y0 + 1 < Hf ? my + 1 : my;
        const uint32_t left = (1u << mx) - 1u;
        const int base = sc->base[vl];
        idx[j][0] = base + sc->wbase[vl][my] + __popc(sc->bits[vl][my] & left);
        idx[j][2] = base + sc->wbase[vl][my1] + __popc(sc->bits[vl][my1] & left);
        idx[j][1] = idx[j][0] + 1;
        idx[j][3] = idx[j][2] + 1;
      } else {
        const int first = sc->base[vl] + 4 * __popc(sc->vmask[vl] & ((1u << p) - 1u));
#pragma unroll
        for (int k = 0; k < 4; ++k) idx[j][k] = -1 - (first + k);   // negative: a private entry, its cell is still to be written
      }
    }
    wave_sync();
#pragma unroll
    for (int j = 0; j < kTrips; ++j) {
      if (2 * (w + NP * j) >= nvb) break;   // uniform
      if (pr[j].xy < 0) continue;
      const int vl = 2 * (w + NP * j) + h;
      const int x0 = pr[j].xy & 0xffff, y0 = pr[j].xy >> 16;
      const float ax = pr[j].ax, ay = pr[j].ay;
      const bool has_x1 = x0 + 1 < Wf, has_y1 = y0 + 1 < Hf;
      const float wgt[4] = {(1.0f - ax) * (1.0f - ay), ax * (1.0f - ay), (1.0f - ax) * ay, ax * ay};
      const bool on[4] = {true, has_x1, has_y1, has_x1 && has_y1};
      if (idx[j][0] < 0) {
        const int cell0 = (ob.view_begin + vb0 + vl) * Hf;
        const int x1 = has_x1 ? x0 + 1 : x0, y1 = has_y1 ? y0 + 1 : y0;
        const int cx[4] = {x0, x1, x0, x1}, cy[4] = {y0, y0, y1, y1};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          idx[j][k] = -1 - idx[j][k];
          out[idx[j][k] >> 4].cell[idx[j][k] & 15] = (uint32_t)((cell0 + cy[k]) * Wf + cx[k]) * row_bytes;
        }
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (on[k]) {
          uint16_t hi, lo;
          split_weight<DT>(wgt[k], hi, lo);
          const int c = idx[j][k] & 15;
          TileStep* stp = out + (idx[j][k] >> 4);
          reinterpret_cast<uint16_t*>(&stp->a_hi[(c >> 3) * kTilePts + p])[c & 7] = hi;
          reinterpret_cast<uint16_t*>(&stp->a_lo[(c >> 3) * kTilePts + p])[c & 7] = lo;
        }
      }
    }
  }

  const int mine = cnt + __shfl_xor(cnt, 32, kWave);   // views of this wave that see point lane % 32
  wave_sync();
  if (w == 0 && lane == 0) {
    slot->tile = blk;
    slot->nsteps = exhausted ? -1 : used;
  }
  if (exhausted && w == 0) {
    push_tile(ws, ob.tile_begin + blk, obj, lane);
    if (lane == 0) *pushed = 1;
  }
  if (lane < kTilePts) slot->cnt[w][lane] = mine;
  dirty = used;   // the same in every producer wave
}

// The scoring wave's part of a tile (Sec. 3.4.1): omega^T = G^T . W^T over the k-steps staged at `sb`, whose weight
// operand is exactly the B operand here; three partial products per k-step (hi * hi, hi * lo, lo * hi).  The rows of G
// of kScoreAhead k-steps are requested together (the wave has nobody to hide a read behind) and multiplied later.
// Accumulator element r of lane l is material 8 (r / 4) + 4 (l / 32) + r % 4 of point l % 32, before the point's factor.
constexpr int kScoreAhead = 8;

struct ScoreRows {
  uint32_t gv[kScoreAhead][8];
};

// What the scoring wave hands to a product wave for storing: a wave that stores to memory waits for the stores'
// acknowledgement before its next read comes back (one counter covers both), and the scoring wave lives on its reads.
struct __attribute__((aligned(16))) ScoreOut {
  float scores[kTilePts * kScoreTileM];   // [32][K]
  float prop[kTilePts * kScoreMaxP];      // [32][P]
  int label[kTilePts];
  int blk;                                // tile index within the object; -1: nothing to store
  int pad_[3];
};

// Requests G for those of the k-steps s0 .. s0 + kScoreAhead - 1 that exist (n staged ones).
__device__ __forceinline__ void request_rows(const char* sb, int n, int s0, const TileScoring& sc, uint32_t row_units, int lane,
                                             ScoreRows& rows) {
  const int pt = lane & 31, g = lane >> 5;
  const TileStep* st = reinterpret_cast<const TileStep*>(sb);
#pragma unroll
  for (int j = 0; j < kScoreAhead; ++j) {
    if (s0 + j >= n) break;   // uniform
    const TileStep* sj = st + s0 + j;
    const u32x4 c0 = *reinterpret_cast<const u32x4*>(&sj->cell[8 * g]);
    const u32x4 c1 = *reinterpret_cast<const u32x4*>(&sj->cell[8 * g + 4]);
#pragma unroll
    for (int e = 0; e < 8; ++e)
      rows.gv[j][e] = sc.G[(long long)cell_index(e < 4 ? c0[e] : c1[e - 4], row_units) * sc.Kpad + pt];
  }
}

template <int DT>
__device__ __forceinline__ void multiply_rows(const char* sb, int n, int s0, const ScoreRows& rows, int lane, f32x16& acc) {
  const TileStep* st = reinterpret_cast<const TileStep*>(sb);
#pragma unroll
  for (int j = 0; j < kScoreAhead; ++j) {
    if (s0 + j < n) {
      const u32x4 w_hi = st[s0 + j].a_hi[lane], w_lo = st[s0 + j].a_lo[lane];
      u32x4 g_hi, g_lo;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        g_hi[q] = __builtin_amdgcn_perm(rows.gv[j][2 * q + 1], rows.gv[j][2 * q], 0x05040100u);
        g_lo[q] = __builtin_amdgcn_perm(rows.gv[j][2 * q + 1], rows.gv[j][2 * q], 0x07060302u);
      }
      acc = mma<DT>(g_hi, w_hi, acc);
      acc = mma<DT>(g_hi, w_lo, acc);
      acc = mma<DT>(g_lo, w_hi, acc);
    }
  }
}

// Stores what the scoring wave left in `o` (if anything): scores, properties and labels of the tile's points are
// contiguous in memory.  Called by all lanes of one wave.
__device__ __forceinline__ void store_scores(const ScoreOut& o, const TileScoring& sc, const ObjRange& ob, int lane) {
  const int blk = o.blk;
  if (blk < 0) return;
  const long long p0 = ob.pt_begin + (long long)blk * kTilePts;
  const int rows = min(kTilePts, ob.n_pts - blk * kTilePts);
  for (int q = lane; q < rows * sc.K; q += kWave) sc.scores[p0 * sc.K + q] = o.scores[q];
  if (sc.prop)
    for (int q = lane; q < rows * sc.P; q += kWave) sc.prop[p0 * sc.P + q] = o.prop[q];
  if (sc.label && lane < rows) sc.label[p0 + lane] = o.label[lane];
}

// With one producer two workgroups share a compute unit, two waves per SIMD, and a product wave has two pieces of 128 channels
// (H = 2, 128 accumulator registers).  With four producers there is one workgroup, and the product waves are what a tile waits
// for: their k-steps are a chain of reads from L2 and beyond.  So they have one piece each there (H = 1): twice as many of them,
// on all SIMDs, three waves per SIMD where they are more than eight in all, each with half the products and half the rows in
// flight (us with two pieces / one; 16 views, 330 000 points: 512 channels 319 / 285, 24 materials 275 / 230, plain fusion 214 / 192;
// 768 channels 364 / 336, 288 / 270, 247 / 236; 1024 channels 427 / 400, plain 302 / 292; 60 000 points of 20 views 156 / 140, 163 /
// 159, 187 / 182; three k-steps ahead instead of two gain nothing).
template <int S, int NP, bool SC>
constexpr int fused_waves_per_simd() { return S + NP + (SC ? 1 : 0) <= 8 ? 2 : 3; }

// S product waves and NP producer waves per workgroup; with SC one more wave, which scores the tiles (K <= 32).
template <int DT, int S, int H, int PF, bool SEL, int NP, bool SC>
__global__ __launch_bounds__(kWave* (S + NP + (SC ? 1 : 0)))
    __attribute__((amdgpu_waves_per_eu(fused_waves_per_simd<S, NP, SC>(), fused_waves_per_simd<S, NP, SC>())))
void k_tile_fused(FuseArgs fa, ProdArgs a, TileWs ws, int keep, ObjTable tab) {
  constexpr int kSpan = kHalf * H;
  constexpr int kStage = fused_stage_steps<S, NP, SC>();
  __shared__ __attribute__((aligned(16))) char s_steps[2][kStage * sizeof(TileStep)];
  __shared__ TileSlot<NP> s_slot[2];
  __shared__ __attribute__((aligned(16))) ProducerScratch s_sc;
  __shared__ float s_ss[2][S * H][kTilePts];
  __shared__ __attribute__((aligned(16))) float s_cam[kCamRows][16];   // the object's camera rows, for the producers
  __shared__ int s_plan[4];      // the workgroup's tickets, k-th tile in slot k & 3
  __shared__ __attribute__((aligned(16))) int s_flags[kMaxProducers];   // meeting numbers of the producer waves
  __shared__ int s_job[4];       // see drain_tiles
  __shared__ int s_drain;        // whether this workgroup looks at the lists of push_tile at its end
  __shared__ __attribute__((aligned(16))) float s_ys[SC ? kScoreTileM * kScoreMaxP : 1];   // the properties, see stage_properties
  __shared__ ScoreOut s_out[SC ? 2 : 1];                        // scores of the tile before the last, on their way to memory

  const ObjRange ob = tab.o[blockIdx.y];
  if (a.unlisted && *a.unlisted != kAllSeen) return;   // uniform
  const int nblk = (ob.n_pts + kTilePts - 1) / kTilePts;
  const int groups = min(nblk, (int)gridDim.x);
  if ((int)blockIdx.x >= groups) return;
  const int xcd = blockIdx.x % kXcd;
  const XcdTiles mine(nblk, xcd);
  const int len = mine.len;
  // Tickets of the XCD: its workgroups take the first four tiles each without asking (those behind the launch's first given_groups ask for
  // them too), and the counter counts the tiles behind them.  An atomic operation on a word takes 11.5 ns, on other words of the same 32
  // bytes as well, 5 ns on others of the same 128 bytes: the 1024 that 256 workgroups had begun with were 12 us.  One object has a word
  // for each XCD in 32 bytes of its own, several have eight words each.  us before / now: one object, single pass, 60 000 points of 5 views 56 / 46, 20 000 of 4 views and 1024 channels 56.6 / 43.7, 50 000 of 10 views
  // 65 / 55, 123 457 of 11 views, 45 materials 150 / 141, 200 000 of 16 views 145 / 138; step of 200 000 points, 768 channels 206 / 203; 64
  // objects of 100 000 points 2920 / 2892.
  unsigned* __restrict__ ctr = a.counters + (gridDim.y == 1 ? launch_ticket_word(xcd, 1) : blockIdx.y * kXcd + xcd);
  constexpr int kGiven = 4;
  const int given = max(0, min(groups, a.given_groups - (int)(blockIdx.y * gridDim.x)));   // of the object's workgroups
  const int team = (given - xcd + kXcd - 1) / kXcd, member = (int)blockIdx.x / kXcd;   // those of the XCD; which of its workgroups this is

  const int tid = threadIdx.x, lane = tid % kWave;
  // Wave index: the product waves come first, then the scoring wave if there is one, then the NP producers (waves go
  // to the four SIMDs in turn: every producer then shares its SIMD with a wave that leaves the vector ALU mostly alone).
  const int span = __builtin_amdgcn_readfirstlane(tid / kWave);
  constexpr int kFirstProducer = S + (SC ? 1 : 0);
  const bool producer = span >= kFirstProducer;
  const lds_floats cam_lds = (lds_floats)&s_cam[0][0];   // the launch code takes this kernel for up to kCamRows views
  const int m = lane & 31, g = lane >> 5;
  const int D = a.D;
  const uint32_t lane_off = (uint32_t)(span * kSpan + 4 * m) * 2u;
  const unsigned group = blockIdx.y * gridDim.x + blockIdx.x;
  if (tid == 0) s_drain = 0;
  const int room = min(kStage, ws.quota);   // k-steps a tile may have: the same bound as where they go to memory
  // Zero weights everywhere, by all waves (the barrier that follows in every branch publishes them); from then on the
  // producers clear what a buffer's last tile wrote.  A launch of one object is short, and its last producer asks for the camera rows
  // before it helps.
  auto clear_stage = [&]() {
    for (int q = tid; q < room * (int)(sizeof(TileStep) / 16); q += kWave * (S + NP + (SC ? 1 : 0))) {
      reinterpret_cast<u32x4*>(s_steps[0])[q] = u32x4{0u, 0u, 0u, 0u};
      reinterpret_cast<u32x4*>(s_steps[1])[q] = u32x4{0u, 0u, 0u, 0u};
    }
  };

  const bool several = gridDim.y > 1;   // objects
  if (several) clear_stage();
  if (producer) {
    // With eight waves or more in the workgroup every producer shares its SIMD with product waves: the producers go first where
    // both are ready (measured on 1024 channels with 24 views, when that was eight waves: 12 % faster).
    if constexpr (S + NP >= 8) __builtin_amdgcn_s_setprio(1);
    // ... and so does a call without rows wait for its one producer (40 objects of two to four views 681 -> 669 us)
    else if (NP == 1 && a.fused == nullptr) __builtin_amdgcn_s_setprio(1);
    const int w = span - kFirstProducer;
    int seq = 0;
    // The last producer wave (the one with the fewest views where they don't come out even) takes the tickets (the counters are
    // zeroed once per call, before its first launch) and publishes them in s_plan, slot k & 3 for the k-th tile of the workgroup, two
    // tiles ahead of the one being built: at the top of a trip every producer knows the tile it builds now and the one after it.
    // Values of len or more mean that the XCD's range is used up.
    auto ticket = [&]() {
      int t = 0;
      if (lane == 0) t = (int)atomicAdd(ctr, 1u) + kGiven * team;
      return t;
    };
    int t_raw = 0;   // the ticket of tile k + 3 while tile k + 1 is built (lane 0 of the producer that takes them)
    if (w == NP - 1) {
      for (int q = lane; q < ob.n_views * 16; q += kWave) s_cam[q >> 4][q & 15] = fa.vis.cam[(long long)ob.view_begin * 16 + q];
      int t0 = member, t1 = member + team, t2 = member + 2 * team;
      t_raw = member + 3 * team;
      if ((int)blockIdx.x >= given) {   // uniform
        t0 = ticket();
        t1 = ticket();
        t2 = ticket();
        t_raw = ticket();
      }
      if (!several) clear_stage();
      if (lane == 0) {
        s_plan[0] = t0;
        s_plan[1] = t1;
        s_plan[2] = t2;
        for (int o = 0; o < kMaxProducers; ++o) s_flags[o] = 0;
      }
    }
    if (w != NP - 1 && !several) clear_stage();
    __syncthreads();   // camera rows, the first plans and the meeting flags are in LDS
    const int last_tile = nblk - 1;
    auto planned = [&](int t) { return t < len; };
    auto tile_at = [&](int t) { return mine.at(t); };
    // a plan past the end reads (and projects) a tile that exists; it is never built
    auto tile_of = [&](int t) { return min(mine.at(t), last_tile); };
    // Who looks at the lists: the workgroups that pushed, which may be the last to, and those among the launch's last
    // workgroups that find, when they run out of tiles, that somebody has (a workgroup in a launch of many thousands that ends
    // early is replaced by the next one).  The producer asks while the product waves are busy with the last tile: asked by
    // everybody at the end it cost 3 us (7812 points of 16 views and 1024 channels 46.8 us, 42.5 without).
    auto looks = [&]() {
      return group + kFusedGroupsMax >= gridDim.x * gridDim.y &&
             __hip_atomic_load(ws.status + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
    };
    ProjectedBatch<NP> pre;
    int dirty0 = 0, dirty1 = 0;   // k-steps of each stage buffer that hold weights of an earlier tile
    float3 pt;   // the lane's point of the tile that the next trip builds
    {
      const int t0 = s_plan[0], t1 = s_plan[1];
      const float3 pt0 = tile_point(fa, ob, tile_of(t0), lane);
      const float3 pt1 = tile_point(fa, ob, tile_of(t1), lane);
      project_batch<SEL, NP>(fa, ob, tile_of(t0), pt0, 0, cam_lds, w, lane, pre);
      if (planned(t0)) {
        produce_tile<DT, SEL, NP>(fa, ob, tile_at(t0), pt0, pre, s_steps[0], room, dirty0, &s_slot[0], &s_sc, cam_lds,
                                  (lds_flags)&s_flags[0], ws, blockIdx.y, &s_drain, w, seq, lane);
      } else if (w == 0 && lane == 0) {
        s_slot[0].tile = -1;
        s_slot[0].nsteps = 0;
        if (looks()) s_drain = 1;
      }
      project_batch<SEL, NP>(fa, ob, tile_of(t1), pt1, 0, cam_lds, w, lane, pre);
      pt = pt1;
    }
    __syncthreads();
    // Producers and product waves run loops with the same number of barriers: one trip per tile, ended by the barrier
    // after which the buffers change hands.  All leave when the slot they look at says that there is no further tile
    // (written before the last barrier, so every wave of the workgroup sees the same value).
    int buf = 0, k = 1;   // the trip builds the k-th tile of the workgroup
    while (s_slot[buf].tile >= 0) {
      const int t = s_plan[k & 3], tn = s_plan[(k + 1) & 3];
      const float3 pt_next = tile_point(fa, ob, tile_of(tn), lane);   // requested now, looked at after this tile is built
      if (planned(t)) {
        produce_tile<DT, SEL, NP>(fa, ob, tile_at(t), pt, pre, s_steps[buf ^ 1], room, buf ? dirty0 : dirty1, &s_slot[buf ^ 1], &s_sc, cam_lds,
                                  (lds_flags)&s_flags[0], ws, blockIdx.y, &s_drain, w, seq, lane);
      } else if (w == 0 && lane == 0) {
        s_slot[buf ^ 1].tile = -1;
        s_slot[buf ^ 1].nsteps = 0;
        if (looks()) s_drain = 1;
      }
      pt = pt_next;
      project_batch<SEL, NP>(fa, ob, tile_of(tn), pt, 0, cam_lds, w, lane, pre);   // its depth texels arrive during the barrier
      if (w == NP - 1) {   // the plan of tile k + 2: its slot (k + 2) & 3 held tile k - 2, which nobody looks at any more
        const int t3 = __builtin_amdgcn_readfirstlane(t_raw);
        if (lane == 0) s_plan[(k + 2) & 3] = t3;
        if (t3 < len) t_raw = ticket();
      }
      __syncthreads();
      buf ^= 1;
      ++k;
    }
  } else if (SC && span == S) {
    if constexpr (SC) {
      // The scoring wave follows the product waves through the tiles, one barrier behind.  During a tile it multiplies
      // the staged weights with G.  After the tile's barrier the product waves' sums of squares are in LDS: the factor
      // of every point follows as in the product waves, and the scores, labels and properties of the tile go to LDS
      // (a product wave stores them during the next tile) while the rows of G for the next tile are on their way.
      const TileScoring& sc = fa.scoring;
      constexpr uint32_t row_units = S * H / 2;   // D / 256
      if (sc.prop) stage_properties<1>(s_ys, sc.y, sc.K, sc.P, lane, kWave);
      if (lane == 0) s_out[0].blk = s_out[1].blk = -1;
      if (!several) clear_stage();
      __syncthreads();
      __syncthreads();
      int buf = 0;
      int blk_prev = -1, n_prev = 0, cnt_prev = 0;   // the tile whose products are in acc
      f32x16 acc[1];
      while (true) {
        const int blk = s_slot[buf].tile;
        const int n = blk >= 0 ? s_slot[buf].nsteps : 0;
        int my_cnt = 0;
#pragma unroll
        for (int o = 0; o < NP; ++o) my_cnt += s_slot[buf].cnt[o][m];
        ScoreRows rows;
        if (n > 0) request_rows(s_steps[buf], n, 0, sc, row_units, lane, rows);

        if (blk_prev >= 0) {   // the tile before: its sums are in the other half of s_ss
          const int li = blk_prev * kTilePts + m;
          const bool valid = li < ob.n_pts;
          const long long ip = ob.pt_begin + (valid ? li : ob.n_pts - 1);
          // (a tile without k-steps, n_prev < 0, gets its scores in gather_point)
          float tot = 0.0f;
#pragma unroll
          for (int wv = 0; wv < S * H; ++wv) tot += s_ss[buf ^ 1][wv][m];
          const float factor = point_factor(cnt_prev, tot, a.norm_eps, a.mean_only);
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[0][r] *= factor;
          if (blk >= 0) {   // a product wave stores the results during the next tile
            ScoreOut& o = s_out[buf ^ 1];
            if (n_prev >= 0)   // uniform
              finish_scores<1>(acc, (long long)m, valid, g, sc.K, sc.P, sc.inv_T, s_ys, o.scores, sc.prop ? o.prop : nullptr,
                               sc.label ? o.label : nullptr, sc.unseen_zero != 0);
            if (lane == 0) o.blk = n_prev >= 0 ? blk_prev : -1;
          } else if (n_prev >= 0) {   // the workgroup's last tile: nobody is left to hand it to
            finish_scores<1>(acc, ip, valid, g, sc.K, sc.P, sc.inv_T, s_ys, sc.scores, sc.prop, sc.label, sc.unseen_zero != 0);
          }
        }
        if (blk < 0) break;

#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][r] = 0.0f;
        for (int s0 = 0; s0 < n; s0 += kScoreAhead) {
          if (s0 > 0) request_rows(s_steps[buf], n, s0, sc, row_units, lane, rows);
          multiply_rows<DT>(s_steps[buf], n, s0, rows, lane, acc[0]);
        }
        __syncthreads();
        blk_prev = blk;
        n_prev = n;
        cnt_prev = my_cnt;
        buf ^= 1;
      }
    }
  } else {
    if (!several) clear_stage();
    __syncthreads();
    __syncthreads();

    StepA wa[2];
    StepC wc;
    StepQ<H> rq[PF];
    int buf = 0;
    unsigned long long started = 0;   // when the tile in work began, by the first wave's look at the counter
    if (s_slot[0].tile >= 0)
      open_tile<H, PF>(s_steps[0], min(max(s_slot[0].nsteps, 0), kStage), a.feat, lane_off, lane, g, wa, rq);

    while (true) {
      const int blk = s_slot[buf].tile;   // uniform over the workgroup: written before the last barrier
      if (blk < 0) break;
      const int n = s_slot[buf].nsteps;
      int my_cnt = 0;                      // views that see point (lane % 32) of this tile
#pragma unroll
      for (int o = 0; o < NP; ++o) my_cnt += s_slot[buf].cnt[o][m];
      f32x16 acc[4 * H];
#pragma unroll
      for (int t = 0; t < 4 * H; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.0f;

      const char* sb = s_steps[buf];
      {
        const int cnt = max(n, 0), l0 = cnt - 1;
        int s = 0;
        for (; s + PF <= cnt; s += PF) {
#pragma unroll
          for (int j = 0; j < PF; ++j) {
            lds_c(sb, min(s + j + PF, l0), g, wc);
            lds_a(sb, min(s + j + 1, l0), lane, wa[(j + 1) & 1]);
            mma_step<DT, H>(wa[j & 1], rq[j], acc);
            __builtin_amdgcn_sched_barrier(0);
            load_q(a.feat, wc, lane_off, rq[j]);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
#pragma unroll
        for (int j = 0; j < PF - 1; ++j) {
          if (s + j < cnt) {
            lds_a(sb, min(s + j + 1, l0), lane, wa[(j + 1) & 1]);
            mma_step<DT, H>(wa[j & 1], rq[j], acc);
          }
        }
      }

      // What goes to memory besides the fused rows.  After the products, not before: the memory counter is in order
      // and covers stores as well, so a store issued ahead of the first product (behind a condition, which makes the
      // compiler count it as possibly absent) would have to be acknowledged before the cell rows requested earlier count
      // as arrived - one store round trip per tile on the critical path.
      if (n >= 0 && span == 0 && tid < kTilePts && fa.out_count && blk * kTilePts + tid < ob.n_pts)
        fa.out_count[ob.pt_begin + blk * kTilePts + tid] = my_cnt;
      if constexpr (SC) {   // what the scoring wave finished during the last tile (the tile before that one)
        if (span == (S > 1 ? 1 : 0)) store_scores(s_out[buf], fa.scoring, ob, lane);
      }
      if (keep && tid == 0) ws.hdr[ob.tile_begin + blk].nsteps = n;   // the scoring kernel reads the header from memory
      if (fa.out_vis && lane < kTilePts && blk * kTilePts + lane < ob.n_pts) {
        // The visibility mask (Eq. 1) of the tile, as aura_project_visibility writes it: lane = point, and the product
        // waves share the views, eight at a time (eight bytes of the point's row).  A tile without
        // k-steps has its mask from gather_point, up to the columns beyond the object's views.
        uint8_t* __restrict__ vrow = fa.out_vis + (ob.pt_begin + blk * kTilePts + lane) * fa.vis_pitch;
        const uint32_t* vm = s_slot[buf].vmask;
        if (n >= 0) {
          const bool pairs = (fa.vis_pitch & 7) == 0 && (reinterpret_cast<uintptr_t>(fa.out_vis) & 7) == 0;
          const bool words = (fa.vis_pitch & 3) == 0 && (reinterpret_cast<uintptr_t>(fa.out_vis) & 3) == 0;
          // who takes the first eight views, the next eight, ...: the last wave, the first, then the others, with the
          // second wave (which stores the scores where the workgroup has a scoring wave) at the end
          const int turn = S <= 2 ? span : (span == S - 1 ? 0 : (span == 0 ? 1 : (span == 1 ? S - 1 : span)));
          for (int v0 = 8 * turn; v0 < ob.n_views; v0 += 8 * S) {
            uint32_t wd[2] = {0u, 0u};
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (v0 + e < ob.n_views) wd[e >> 2] |= ((vm[v0 + e] >> lane) & 1u) << (8 * (e & 3));
            if (pairs && v0 + 8 <= ob.n_views) {
              *reinterpret_cast<u32x2*>(vrow + v0) = u32x2{wd[0], wd[1]};
            } else {
#pragma unroll
              for (int q = 0; q < 2; ++q) {
                if (words && v0 + 4 * q + 4 <= ob.n_views) {
                  *reinterpret_cast<uint32_t*>(vrow + v0 + 4 * q) = wd[q];
                } else {
                  for (int e = 0; e < 4 && v0 + 4 * q + e < ob.n_views; ++e) vrow[v0 + 4 * q + e] = (uint8_t)((wd[q] >> (8 * e)) & 1u);
                }
              }
            }
          }
        }
        if (span == S - 1)
          for (int j = ob.n_views; j < fa.vis_pitch; ++j) vrow[j] = 0;
      }
      if (keep && n > 0) {
        // The scoring kernel wants the k-steps in memory: the product waves, which have issue slots to spare, copy the
        // staged tile out (the producers do not: their vector ALU work is what the tile waits for).
        u32x4* __restrict__ dst = reinterpret_cast<u32x4*>(ws.steps + (long long)(ob.tile_begin + blk) * ws.quota);
        const u32x4* src = reinterpret_cast<const u32x4*>(sb);
        for (int q = span * kWave + lane; q < n * (int)(sizeof(TileStep) / 16); q += S * kWave) dst[q] = src[q];
      }
      if (n > 0) {   // uniform
        piece_squares<H>(acc, lane, &s_ss[buf][span * H]);
      } else if (lane < kTilePts) {   // nobody sees the tile's points
#pragma unroll
        for (int h = 0; h < H; ++h) s_ss[buf][span * H + h][lane] = 0.0f;
      }
      if constexpr (!SC) {
        if (a.pace != 0 && span == 0) {   // see launch_tile (the other waves wait at the barrier; a counter that runs on ends it)
          while (__builtin_amdgcn_s_memrealtime() - started < (unsigned long long)a.pace) __builtin_amdgcn_s_sleep(4);
          started = __builtin_amdgcn_s_memrealtime();
        }
      }
      __syncthreads();   // the one barrier of a tile: the sums are in LDS, the producers have staged the next tile, and
                         // every product wave is done with this tile's buffer

      float factor;
      {
        float tot = 0.0f;
#pragma unroll
        for (int wv = 0; wv < S * H; ++wv) tot += s_ss[buf][wv][m];
        factor = point_factor(my_cnt, tot, a.norm_eps, a.mean_only);
      }
      {
        const int rows_f = a.factor ? min(kTilePts, ob.n_pts - blk * kTilePts) : 0;
        const __amdgpu_buffer_rsrc_t fout = __builtin_amdgcn_make_buffer_rsrc(a.factor + (a.factor ? ob.pt_begin + blk * kTilePts : 0), 0,
                                                                              rows_f * 4, 0x00020000);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(factor), fout, tid < kTilePts ? 4 * tid : 0x7ffffff0, 0, 0);
      }
      if (a.fused) {
        // (uniform.  A call without rows has nothing to scale or to store: the 32 stores of a wave and tile that the bounds
        // check would drop still pass the address unit, in front of the producer's reads.  With the norm of tiles that
        // nobody sees left out as well, 40 objects of 50 000 points, single pass, 771 -> 716 us; 123 457 points of 11 views
        // 198 -> 190; 1.68 M voxels of 24 views 1378 -> 1352; calls with rows as before.)
        const int li0 = blk * kTilePts;
        float* obase = a.fused + (ob.pt_begin + li0) * D + span * kSpan;
        uint32_t row_bytes = (uint32_t)D * 4u;
        asm volatile("" : "+s"(row_bytes));
        const int rows = n >= 0 ? min(kTilePts, ob.n_pts - li0) : 0;
        const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(obase, 0, (int)(rows * row_bytes), 0x00020000);
        const uint32_t lane_out = (uint32_t)(4 * g) * row_bytes + (uint32_t)(4 * m) * 4u;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row0 = 8 * (r >> 2) + (r & 3);
          const float scale = __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (row0 + 4 * g), __float_as_int(factor)));
#pragma unroll
          for (int h = 0; h < H; ++h) {
            const f32x4 v = {acc[4 * h][r] * scale, acc[4 * h + 1][r] * scale, acc[4 * h + 2][r] * scale, acc[4 * h + 3][r] * scale};
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), out,
                                                   (int)(lane_out + (uint32_t)row0 * row_bytes) + h * kHalf * 4, 0, /*streaming*/ 2);
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      buf ^= 1;
      {
        const int nn = s_slot[buf].tile >= 0 ? min(max(s_slot[buf].nsteps, 0), kStage) : 0;
        open_tile<H, PF>(s_steps[buf], nn, a.feat, lane_off, lane, g, wa, rq);
      }
    }
    if constexpr (SC) {   // the tile before the workgroup's last one (the scoring wave stores the last one itself)
      if (span == (S > 1 ? 1 : 0)) store_scores(s_out[buf], fa.scoring, ob, lane);
    }
  }
  if (s_drain != 0) {
    constexpr int kSweeps = fused_waves_per_simd<S, NP, SC>() == 2 ? kGatherSweeps : (kSpan * S + 511) / 512;
    drain_tiles<DT, !SEL, kSweeps>(fa, ws, tab, group, s_job, span, (int)(blockDim.x / kWave), lane);
  }
}

__global__ void k_clear_words(unsigned* words, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) words[i] = 0u;
}

// ------------------------------------------------------------------------------------ host

static long long tile_count_bound(long long N, int B) { return N / kTilePts + B; }

static int steps_quota(int B, int n_views) {
  // k-steps of storage per tile: two per view of an object, within [4, 32] (measured need on
  // spatially sorted points: 0.3 to 0.4 per view for coarse grids, up to 1 for pixel-sized cells)
  const long long per_obj = (n_views + B - 1) / B;
  return (int)(2 * per_obj < 4 ? 4 : (2 * per_obj > 32 ? 32 : 2 * per_obj));
}

static_assert(kMaxObjPerLaunch % kXcd == 0, "launches begin with a group of eight objects' counters");
static size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }

size_t fuse_tile_workspace_bytes(long long N, int B, int n_views) {
  const size_t tiles = (size_t)tile_count_bound(N, B);
  return round256(tiles * sizeof(TileHdr)) + (size_t)counter_words(B) * sizeof(unsigned) + 256 +
         tiles * (size_t)steps_quota(B, n_views) * sizeof(TileStep);
}

TileWs fuse_tile_workspace(void* workspace, long long N, int B, int n_views) {
  char* base = static_cast<char*>(workspace);
  TileWs ws;
  ws.hdr = reinterpret_cast<TileHdr*>(base);
  base += round256((size_t)tile_count_bound(N, B) * sizeof(TileHdr));
  ws.counters = reinterpret_cast<unsigned*>(base);
  base += (size_t)counter_words(B) * sizeof(unsigned);
  ws.status = reinterpret_cast<unsigned*>(base);
  base += 256;
  ws.steps = reinterpret_cast<TileStep*>(base);
  ws.quota = steps_quota(B, n_views);
  ws.obj_base = 0;
  return ws;
}

int fuse_tile_clear_words(int B) { return counter_words(B) + 256 / (int)sizeof(unsigned); }

hipError_t launch_fuse_tile_clear(const TileWs& ws, int B, hipStream_t stream) {
  const int n = fuse_tile_clear_words(B);
  hipLaunchKernelGGL(k_clear_words, dim3((n + 255) / 256), dim3(256), 0, stream, ws.counters, n);
  return hipGetLastError();
}

size_t fuse_tile_status_offset(long long N, int B) {
  return round256((size_t)tile_count_bound(N, B) * sizeof(TileHdr)) + (size_t)counter_words(B) * sizeof(unsigned);
}

bool fuse_tile_supported(int dtype, int D, int Hf, int Wf, long long feat_bytes) {
  // cell coordinates travel as 16-bit pairs and cell rows as 32-bit byte offsets inside the kernels
  return (dtype == 1 || dtype == 2) && Hf <= 32767 && Wf <= 32767 && D % 256 == 0 && D / 256 >= 1 && D / 256 <= 6 &&
         D / 256 != 5 && feat_bytes <= 0xffffffffll;
}

// K-steps of a tile, estimated from what sorted points on closed surfaces need: 0.3 per view and 17 more per point that there is for each
// cell of a view (330 000 points, 16 views of 32 x 32 cells 5.8, 123 457 of 11 views of 37 x 37 5.3, 60 000 of 20 13.6).
static double tile_steps(const FuseArgs& a, int views, int n_obj, long long tiles) {
  return views * (0.3 + 17.0 * a.feat.Hf * a.feat.Wf * n_obj / ((double)kTilePts * std::max(1ll, tiles)));
}

// How many producer waves the one-kernel form takes for this launch; 0: the two kernels.  units: channels / 256.  One producer wave
// keeps up with the product waves for a few views per object; beyond that four share the views of a tile and a compute unit
// holds one workgroup of up to twelve waves (see fused_waves_per_simd), which is the faster form of few views too where the launch
// is one object.
// Cells of at least 4 x 4 pixels: a tile needs 0.3 to 0.4 k-steps per view on spatially sorted points.  Smaller cells need up to
// one and more, too many for the short stage of the one-producer form and its producer, and the more views the longer the
// producers take.  Where the lines of one object lie (us, two kernels / one with four producers; 400 000 points unless said, "fine":
// cells of one or two pixels):
//   256 channels, fine     50 000 points, 8 views, step 412 / 252 (one producer 648), 100 000 191 / 152 (754), 300 000, 6 views 243 /
//                          193; 16 views, cells of 2 pixels, step 386 / 339, 1 pixel 436 / 380, single pass of 24 materials 350 /
//                          267; 20 views 417 / 442 (2 pixels), 468 / 450 (1 pixel); 32 views, single pass 502 / 574, 725 / 725
//   256 channels, coarse   10 views, step 303 / 243, plain 246 / 185; 16 views 332 / 282, 254 / 214; 20 views 352 / 385, 266 / 308
//   512 channels, fine     100 000 points, 6 views, one producer 227, four 206, 8 views, 2 pixels, single pass 154 / 105; 16 views,
//                          step 636 / 536; 32 views, 1 pixel, step 838 / 657, plain 615 / 442; 2 pixels, step 708 / 609, single pass,
//                          40 materials 574 / 604, 24 materials 530 / 483; 1 M points, 32 views, step 1611 / 1456; 800 000 points, 5
//                          views, step 438 (one producer) / 470
//   768 channels, fine     32 views, 1 pixel, step 901 / 722, plain 685 / 511; 2 pixels, single pass 600 / 544; 1024 channels, 28
//                          views 1002 / 800; 24 views of few points (most tiles outgrow their k-steps): 10 000 192 / 219, 25 000 311
//                          / 235
// Few views (up to eight): four producers for one object and for two, one producer / four, 200 000 points: 256 channels, 5 views,
// step 146 / 138, plain 104 / 96; 512 channels 154 / 144, 108 / 98, single pass 149 / 136; 768 channels 197 / 167, 152 / 112, 153 /
// 144; 1024 channels (two kernels / four producers) 272 / 200, 223 / 154, 193 / 156; 60 000 points of 8 views, 512 channels 108 / 91,
// 65 / 50; 30 000 of 5 views 82 / 51; 2 objects of 60 000 points, 6 views, 768 channels 138 / 95.  Not for many points of many views,
// which make the producers' trips longer than the product waves' turn: 700 000 points of 8 views, 512 channels, step 382 / 401, 256
// channels, single pass 375 / 390.
// More objects share the machine, and one workgroup per compute unit leaves every start of a workgroup uncovered, which two cover:
//   1024 channels always (two kernels / four producers): 20 objects of 60 000 points and 4 views, step 1301 / 971, plain 1213 / 892,
//     single pass 800 / 449; 64 of 5000 and 3 views 391 / 312, 336 / 255, 290 / 244
//   768 channels with rows: 24 of 50 000, 4 views, step 785 / 653, plain 691 / 647; 8 of 30 000, 6 views 203 / 161, 170 / 150; 50 of
//     40 000, 8 views, plain 1067 / 1044, but step 1378 / 1470; 64 of 4000, 4 views, step, 24 materials 265 / 233, 60 materials 288 /
//     292; without rows 24 of 50 000 377 / 460
//   512 channels with rows, up to four: 4 of 150 000, 4 views, step 295 / 261, plain 263 / 252; 6 of 30 000, step 125 / 130; without
//     rows 131 / 143
//   256 channels: 4 of 150 000, plain 155 / 239
static int one_kernel_producers(const FuseArgs& a, int views_per_obj, int units, int n_obj, long long tiles) {
  const bool coarse = a.feat.pitch_x >= 4.0f && a.feat.pitch_y >= 4.0f;
  const bool many_materials = a.scoring.G && a.scoring.Kpad > kScoreTileM;
  if (a.two_kernels || views_per_obj > kCamRows) return 0;
  if (n_obj == 1) {
    if (views_per_obj > kPBatch && units == 1) return 0;
    if (!coarse && views_per_obj > kPBatch && units == 2 && !a.fused && many_materials) return 0;
    if (!coarse && views_per_obj > kPBatch && units >= 3 && tiles < 512) return 0;
  } else if (!coarse && views_per_obj > (units >= 3 ? 16 : 4 * units)) {
    return 0;
  }
  if (views_per_obj <= kOneKernelViews) {
    if (n_obj <= 2) {
      const bool one = (units == 2 && a.fused && tiles > (coarse ? 12000 : 10000) && views_per_obj > (coarse ? 5 : 3)) ||
                       (units == 1 && many_materials && tiles > 12000 && views_per_obj > 5 && coarse);
      if (units <= 4 && !one) return 4;
    } else {
      if (units == 4) return 4;
      if (units == 3 && a.fused && (!a.scoring.G || ((views_per_obj <= 6 || tiles <= 32768) && (!many_materials || n_obj <= 32)))) return 4;
      if (units == 2 && a.fused && n_obj <= 4) return 4;
    }
    // One producer, where two workgroups fit a compute unit.
    if (units + 1 > 4) return 0;
    // Up to three views of 512 channels, or seven of 768, the two kernels are ahead until the launch has tiles enough to
    // hide the pipeline's start in every workgroup, many small objects later, and later again where no rows are stored (times
    // in us, two kernels / one):
    //   20 objects of 3 views, 512 channels    100 000 points 82 / 90, 200 000 145 / 139, 400 000 267 / 193
    //   ... single pass, 60 materials          200 000 points 159 / 192, 400 000 238 / 260, 800 000 396 / 396
    //   20 objects of 6 views, 768 channels, single pass   200 000 points 199 / 215, 400 000 306 / 290
    long long from = 0;   // tiles
    if (units == 3 && views_per_obj < 8 && n_obj > 8 && !a.fused) from = 8000;
    if (units == 2 && views_per_obj < 4 && n_obj > 8) from = a.fused ? 4000 : 25000;
    return tiles >= from ? 1 : 0;
  }
  if (units > 4 || (units == 1 && n_obj > 1)) return 0;
  // (where the scoring kernel wants the k-steps in memory the product waves copy them out: measured 3 to 7 % faster than
  // the two kernels on 768 channels with 16 views and on 1024 channels with 24 views)
  return 4;
}

// Whether the one-kernel form of this launch scores its tiles itself: a scoring wave must fit the workgroup (up to 768 channels beside
// four producers, 512 beside one) and one matrix-core tile must hold the materials.
static bool scoring_wave_fits(const FuseArgs& a, int producers, int units, double steps, int quota) {
  if (!a.out_factor || !a.scoring.G || a.scoring.Kpad != kScoreTileM || a.in_mask) return false;
  if (producers == 4) return 2 * units + 4 + 1 <= 12;
  // With one producer wave (two workgroups of up to four waves per compute unit) it pays where no rows are stored: with rows the call is
  // bound by their stores either way, and the separate scoring kernel keeps the fusion kernel shorter (64 objects of 100 000 points and 4
  // views, combined call, 3.12 ms against 3.16 ms).  us with / without, single pass: 512 channels, 16 x 3000 points, 8 views 71 / 84; 40 x
  // 3000, 4 views of 24 x 24 cells 116 / 128; 64 x 3000 151 / 179; 13 x 8615, 4 views of 37 x 37 97 / 114; 30 x 22 933, 4 views of 112 x 112
  // 556 / 591; 256 channels, 51 x 2211, 3 views of 32 x 32 222 / 250.
  if (units + 1 + 1 > 4 || a.fused) return false;
  // Not where tiles may have more k-steps than the stage beside a scoring wave holds (12 instead of 16) and need them: 512 channels, 8 views of
  // 24 x 24 cells, 35 x 2038 points 146 / 132, 13 x 1639 190 / 150; 33 x 18 457, of 56 x 56 817 / 610.
  return quota < 16 || steps <= 16.0;
}

// Whether k_tile_sift goes ahead of this launch: calls that store no rows, of sizes where the tiles that it finds are worth its
// launch and the lists.  (With rows the stores set the time, and the unseen rows' are best mixed with the others': 64 objects of
// 100 000 points and 4 views with rows 2927 us, 3296 sifted.)  us without / with it, single pass, 24 materials unless said, a tile per wave
// behind it both times:
//   one object, voxels of a solid   14 M, 12 views, 512 channels 2222 / 1007; 1.68 M, 24 views, 1024 channels, 128 materials 565 / 538; 1.45 M,
//     8 views, 768 channels 263 / 130; 951 000, 6 views, 512 channels 183 / 101; 400 000, 12 views, 768 channels 140 / 125; 300 000 129 / 122;
//     265 000, 24 views, 1024 channels, 100 materials 258 / 260; fewer 200 000, 6 views, 512 channels 66 / 64; 150 000, 12 views, 768
//     channels 100 / 107
//   ... seen from all around (every tile seen: all it costs)   262 200, 6 views, 512 channels 99 / 104, 16 views 167 / 172; 330 000, 24 views, 1024
//     channels, 60 materials 428 / 440; 1 M, 16 views, 512 channels 353 / 358; 14 M, 12 views 2844 / 2882; 400 000, 6 views, 256 channels, 40
//     materials 127 / 132
//   objects x points of frontal views   64 x 100 000, 4 views 693 / 684; 30 x 100 000 291 / 280; 12 x 110 000 155 / 146; 8 x 100 000 161 / 134; 4
//     x 200 000 157 / 130; 3 x 400 000 216 / 148; 6 x 150 000, 8, 768 channels 198 / 186; solids 9 x 123 000, 3 views 119 / 96, 2 x 265 000, 4 111 /
//     68; from all around 30 x 100 000, 6 441 / 473; 4 x 200 000 170 / 194
//   ... of fewer than 2500 tiles each   40 x 50 000 ragged, 2 to 4 278 / 285; 12 x 60 000, 4 112 / 120; 12 x 40 000, 4, 768 channels 105 / 111; 30 x
//     45 000 167 / 175; from all around 20 x 60 000, 6, 768 channels 233 / 259; 64 x 12 000, 4 155 / 176; 20 x 30 000, 8 150 / 177
//   ... of few such objects the ones gain what the others lose   frontal 3 x 102 000, 8 views 89 / 72; 2 x 112 000, 6, 1024 channels 73 / 67; from all
//     around 2 x 184 000, 8, 1024 channels, 100 materials 185 / 191; solids 3 x 128 000, 12, 256 channels 117 / 133, 3 x 80 000, 5, 1024 channels 100 / 84
constexpr long long kSiftOneObject = 8192, kSiftSeveral = 12288;   // tiles
static bool sift_tiles(const FuseArgs& a, int n_obj, long long tiles) {
  // The results of a tile that nobody sees are known to be zero (point_factor): not where a weight of exp(0 * inf) would make them
  // something else.
  if (a.fused || !a.scoring.G || a.in_mask || !(0.0f * a.scoring.inv_T == 0.0f)) return false;
  if (n_obj == 1) return tiles >= kSiftOneObject;
  return tiles >= kSiftSeveral && tiles >= 2500ll * n_obj;
}

// Which calls without rows take k_tile_fused of tile_waves.hip, a tile per wave.  Its waves hide each other's waits, so it wants many
// tiles, and it keeps a tile's k-steps in a wave's share of LDS, so it wants them short (tile_steps).  us by producers / by waves, 24 materials:
//   one object, up to eight views   60 000 points, 5 views, 512 channels 46 / 35; 20 000 of 4 views, 1024 channels 44 / 38; 80 000, 7
//     views of 37 x 37 cells, 768 channels 65 / 59; 120 000, 8 views of 56 x 56, 1024 channels 116 / 103; 800 000, 6 views, 256
//     channels 399 / 194; but 30 000, 6 views, 768 channels 42 / 48; 40 000, 8 views of 37 x 37 45 / 61; 100 000, 8 views of 112 x 112,
//     30 materials 127 / 138
//   one object, more views   400 000, 10 views 211 / 172, 24 views 364 / 308; 1 M, 16 views 512 / 369, 20 views, 1024 channels 887 /
//     567; 330 000, 16 views 204 / 196; 300 000, 24 views of 112 x 112 331 / 320; 270 000, 32 views of 56 x 56, 256 channels 442 / 325;
//     with fewer tiles than the sieve takes 200 000, 16 views, 768 channels 160 / 204; 100 000, 10 views 77 / 82
//   several objects, 512 channels and more   40 x 50 000 ragged, 2 to 4 views 457 / 289; 64 x 100 000, 4 987 / 562; 2 x 60 000, 12 96 / 75; 5
//     x 100 000, 16 439 / 257; 6 x 60 000, 20 365 / 277; 24 x 50 000, 6, 1024 channels, 128 materials 685 / 458; but 3 x 40 000, 24 views
//     of 37 x 37, 768 channels 175 / 226.  The more k-steps the less, and less where the views look at the same points (on a frontal arc,
//     where the estimate is short) than from all around: over 480 batches, waves / producers, on an arc 8 to 12 k-steps 0.89 (0.5 to
//     1.5), 12 to 18 0.99 (to 1.7), more 1.15 (to 2.5); from all around 0.68, 0.69, 0.83 (to 1.7).  Of up to eight views and fewer than 3000
//     tiles, where eight k-steps are the line, 8 to 10 on an arc 1.25 (6 x 9851, 2 to 7 views of 24 x 24, 768 channels, 60 materials 143 /
//     210; 4 x 16 637, 2 to 5 of 37 x 37, 60 materials 141 / 199), up to 8 0.83, from all around 8 to 10 0.75
//     (with 1250 tiles per object and 12 288 in all whatever their lists: 16 x 67 000, 20 views of 37 x 37, 1024 channels 1205 / 1101; 10 x 41 000, 10
//     of 112 x 112 845 / 717; 6 x 79 000, 10 of 112 x 112, 100 materials 754 / 659; but 8 x 70 000, 32 of 32 x 32, 1024 channels 710 / 805)
//   ... 256 channels, whose one producer has a stage of eight k-steps   16 x 3000, 8 views of 16 x 16 135 / 60; 30 x 6000, 8 of 24 x 24 338 / 109; 64
//     x 3000, 8 of 24 x 24 927 / 227; 53 x 22 641, 24 of 37 x 37 1145 / 617; 39 x 1782, 7 of 16 x 16, 100 materials 357 / 103; 55 x 9056, 32 of
//     16 x 16 471 / 342; up to 40 k-steps (3 x 8331, 24 of 24 x 24, 45 of them 168 / 234), with many tiles any number (35 x 11 559, 8 of 56 x
//     56 2672 / 517; 5 of 112 x 112, 3 x 54 203 230 / 197)
//   ... whose tiles need more k-steps than they own, half as many again by the estimate, so that most are fused point by point: few of them are better
//     left to the producers (6 x 6181, 2 views of 37 x 37, 1024 channels 92 / 148; 55 x 1590, 2 of 16 x 16, 256 channels, 100 materials 132 /
//     171; 18 x 3257, 3 of 24 x 24 149 / 195), many not (34 x 20 938, 2 of 56 x 56, 463 / 239; 21 x 11 986, 1024 channels 269 / 206)
// Long lists in one object of many views: where the sieve has sampled none but seen tiles, they are as long as the estimate, and the
// launch with four producers follows, which leaves at once where there is a list (*both; 300 000 points, 32 views of 56 x 56, 1024
// channels, seen from all around 510 / 682, voxels of a solid 271 / 256; the launch that leaves costs 5).  Beyond ten k-steps where cells are
// coarse; for smaller ones the estimate is too long, and it is twelve with cells of three pixels and 36 with one or two, up to 32
// materials and 16 384 tiles (producers / waves, 24 materials, cells of 3 pixels: 288 000 points, 25 views, 512 channels 415 / 477, 299 000 of
// 12, 768 channels 252 / 277, 388 000 of 25, 1024 channels 700 / 760; of 1 pixel: 420 000 of 23, 512 channels 644 / 722, 330 000 of 16, 768
// channels 513 / 531, 378 000 of 24 827 / 972, 324 000 of 23, 1024 channels 1110 / 1275; but 387 000 of 31, 512 channels, 40 k-steps 772 / 714, 360 000
// of 23, 100 materials 1031 / 972, 700 000 of 24, 1024 channels, 40 materials 1362 / 1295).
static bool tile_per_wave(const FuseArgs& a, int views, int units, int n_obj, long long tiles, double steps, int quota, bool sifted,
                          bool* both) {
  *both = false;
  if (a.fused || !a.scoring.G || a.in_mask || a.two_kernels || views > kWaveViews || units > 4) return false;
  if (n_obj > 1) {
    const bool many = tiles >= 5000;
    const double most = units > 1 ? (views <= kOneKernelViews && tiles < 3000 ? 8.0 : 12.0) : (many ? 1e9 : 40.0);
    return (tiles >= kSiftSeveral && tiles >= 1250ll * n_obj) || (steps <= most && (many || steps <= 1.5 * quota));
  }
  if (views <= kOneKernelViews) return tiles >= kSiftOneObject || steps <= 2.0 + tiles / 800.0;
  if (tiles < kSiftOneObject) return false;
  const float pitch = std::min(a.feat.pitch_x, a.feat.pitch_y);
  const bool few_materials = a.scoring.Kpad == kScoreTileM;
  const bool longer = pitch >= 4.0f ? steps > 10.0 && (units > 2 || (units == 2 && few_materials))
                                    : steps > (pitch >= 3.0f ? 12.0 : 36.0) && units >= 2 && few_materials && tiles < 16384;
  *both = sifted && longer;
  return sifted || !longer;
}

template <int DT, int S, int H, int PF>
static hipError_t launch_tile(const FuseArgs& a, const TileWs& ws, const ObjTable& tab, int n_obj, int max_pts,
                              hipStream_t stream, FuseOutcome* did) {
  const int max_tiles = (max_pts + kTilePts - 1) / kTilePts;
  ProdArgs pa{static_cast<const char*>(a.feat.feat), a.feat.D, ws.hdr, ws.steps, ws.counters + (size_t)ws.obj_base * kXcd,
              ws.quota, a.fused, a.out_factor, a.norm_eps, a.mean_only, 0, 0, nullptr};
  int max_views = 0;
  long long tiles = 0;
  for (int t = 0; t < n_obj; ++t) {
    max_views = std::max(max_views, tab.o[t].n_views);
    tiles += (tab.o[t].n_pts + kTilePts - 1) / kTilePts;
  }
  const double steps = tile_steps(a, max_views, n_obj, tiles);
  const TimedLaunch timed(stream);
  const bool sifted = !a.two_kernels && sift_tiles(a, n_obj, tiles);
  bool both = false;
  if (tile_per_wave(a, max_views, S, n_obj, tiles, steps, ws.quota, sifted, &both)) {
    if (sifted) {
      const hipError_t e = launch_tile_sift(a, ws, tab, n_obj, max_tiles, stream);
      if (e != hipSuccess) return e;
    }
    const hipError_t e = launch_tile_waves(a, ws, tab, n_obj, max_views, tiles, sifted, both, stream);
    if (e != hipSuccess || !both) {
      if (did) did->scored = true;
      return e;
    }
    pa.unlisted = pa.counters + kSeenWord;
    if (did) did->unlisted_only = true;
  }
  const int np = one_kernel_producers(a, max_views, S, n_obj, tiles);
  constexpr bool kOneProducer = S + 1 <= 4, kFourProducers = 2 * S + 4 <= 12;   // what it can answer (launched below)
  static_assert(H == 2, "four producers take waves of half the channels");
  if (np > 0) {
    // With one producer wave two workgroups fit a compute unit, with four one; several objects in one launch share the
    // machine.  Where the workgroup has just the two waves four fit: worth it for several objects (10 objects of 300 000
    // points, 8 views, combined call: 161 us with two, 143 with four), not for one (more than 32 materials, 400 000 points of 8
    // views: single pass 224 us with two, 230 with four, step 226 and 235; 1 M points of 6 views 503 and 503, 514 and 525).
    const bool scoring = scoring_wave_fits(a, np, S, steps, ws.quota);
    const int groups_max = np > 1 ? kFusedGroupsMax / 2 : (S == 1 && !scoring && n_obj > 1 ? 2 * kFusedGroupsMax : kFusedGroupsMax);
    const int keep = a.out_factor != nullptr && !scoring;   // the scoring kernel follows and reads the k-steps
    // Several objects in one launch: many more workgroups per object than are resident at a time (fuse_tile_groups.hpp: 64 objects
    // of 100 000 points and 4 views with eight per object: the workgroups' end times were spread over the last quarter of the
    // kernel; fusion call 2.79 ms, 2.44 with 64 per object, 2.41 with 128, 2.43 with 256 and 384).  The combined call, whose
    // workgroups also write the k-steps for the scoring kernel: 3.10 -> 2.94 ms with 64 and slower beyond.
    const int per_object = n_obj <= 1 ? 0
                         : (keep || scoring) ? std::min(64, max_tiles / 8 / kXcd * kXcd)
                                             : fused_groups_per_object(S, np, n_obj, groups_max, max_tiles);
    // Where nothing but the row stores sets the time, the workgroups must not run ahead of the memory: tiles that nobody sees
    // are stored as fast as they can be issued, and the more of that, the less of it memory takes (the faster producers made
    // such calls slower).  A workgroup then starts no tile sooner than 4.6 us after the last: its 64 KiB, times the 512 resident
    // workgroups, are 7.3 TB/s, a little above what a fill reaches.  us without / with it (in brackets with the slower producers):
    //   channels 512, objects x points, views   64 x 100 000, 4   2412 / 2317 (2357)     16 x 100 000, 4   648 / 625 (656)
    //     64 x 25 000, 4   620 / 598 (615)      40 x 50 000, 2 to 4   788 / 721 (784)    20 x 100 000, 3   793 / 759 (793)
    //     40 x 30 000, 3   489 / 454 (461)      40 x 30 000, 2   493 / 453 (477)         20 x 30 000, 2   260 / 252 (253)
    //     16 x 60 000, 1   392 / 379 (408)
    // Not for others.  More views: the producers are what it waits for (paced, 512 channels, 32 x 60 000, 8 views 721 -> 734).  Few
    // tiles or few objects: part of the machine is idle at the end, and the rest must not be held back (8 x 20 000, 3 views 102 ->
    // 110; 6 x 300 000, 4 views 708 -> 781).  256 channels 498 -> 508.
    // One object with four producers, one workgroup per compute unit: the same rate again, whatever the number of tiles (1.68 M
    // voxels of 24 views, nine tiles of ten seen by nobody, 1024 channels 1232 / 1101 (1151), 512 channels 801 / 802 (984); 700 000
    // voxels, 12 views, 768 channels 397 / 342 (365), 24 views, 1024 channels 525 / 476 (491); 30 000 points, 12 views, 1024 channels
    // 59 / 57 (60)).  Not several objects: 16 x 40 000, 10 views, 768 channels 391 -> 401.
    // 1.2 us since the product waves have 128 channels (1.15 / 1.2 us): 1.68 M voxels, 24 views, 1024 channels 1138 / 1091; 700 000,
    // 12 views, 1024 channels 513 / 487, 768 channels 356 / 342; 500 000 points, 4 views, 1024 channels 368 / 346; 700 000, 5 views,
    // 768 channels 339 / 343; with 1.3 us 1120, 476, 365, 347, 366, without any 1218, 519, 395, 373, 370.
    if (!keep && !scoring && np > 1 && n_obj == 1) pa.pace = 120 * S;
    if (!keep && !scoring && np == 1 && S == 2 && n_obj >= 16 && max_views <= 4 && tiles >= 32 * kFusedGroupsMax) pa.pace = 460;
    const int groups = std::max(kXcd, std::min(max_tiles, std::max((groups_max / n_obj + kXcd - 1) / kXcd * kXcd, per_object)));
    pa.given_groups = given_groups(std::min(groups, max_tiles) * n_obj, groups_max);
    const dim3 grid(std::min(groups, max_tiles), n_obj), block(kWave * ((np > 1 ? 2 * S : S) + np + (scoring ? 1 : 0)));
#define AURA_FUSED(s_, h_, sel, np_, sc) \
  hipLaunchKernelGGL((k_tile_fused<DT, s_, h_, PF, sel, np_, sc>), grid, block, 0, stream, a, pa, ws, keep, tab)
    if (scoring) {
      pa.factor = nullptr;   // nobody reads the factors back
      if (np == 1) {
        if constexpr (kOneProducer && S + 1 + 1 <= 4) { AURA_FUSED(S, H, false, 1, true); }
      } else {
        if constexpr (kFourProducers && 2 * S + 4 + 1 <= 12) { AURA_FUSED(2 * S, 1, false, 4, true); }
      }
      if (did) did->scored = true;
    } else if (np == 1) {
      if constexpr (kOneProducer) {
        if (a.in_mask) {   // (768 channels with rows and no scores take four producers)
          if constexpr (S < 3) { AURA_FUSED(S, H, true, 1, false); }
        } else { AURA_FUSED(S, H, false, 1, false); }
      }
    } else if constexpr (kFourProducers) {
      if (a.in_mask) { AURA_FUSED(2 * S, 1, true, 4, false); }
      else { AURA_FUSED(2 * S, 1, false, 4, false); }
    }
#undef AURA_FUSED
    return hipGetLastError();
  }
  if (a.in_mask)
    hipLaunchKernelGGL((k_tile_prepare<DT, true>), dim3(max_tiles, n_obj), dim3(kPrepThreads), 0, stream, a, ws, tab);
  else
    hipLaunchKernelGGL((k_tile_prepare<DT, false>), dim3(max_tiles, n_obj), dim3(kPrepThreads), 0, stream, a, ws, tab);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // several objects in one launch share the machine: fewer workgroups per object
  const int groups = std::max(kXcd, std::min(max_tiles, (kProdGroupsMax / n_obj + kXcd - 1) / kXcd * kXcd));
  hipLaunchKernelGGL((k_tile_product<DT, S, H, PF>), dim3(std::min(groups, max_tiles), n_obj), dim3(kWave * S), 0, stream, a, pa, ws, tab);
  return hipGetLastError();
}

hipError_t launch_fuse_tile(const FuseArgs& a, const TileWs& ws, const ObjTable& tab, int n_obj, int max_pts,
                            hipStream_t stream, FuseOutcome* did) {
  if (did) *did = FuseOutcome{};
  // waves x pieces of 128 channels per wave x k-steps of rows requested ahead, for each supported D
#define AURA_TILE_CASE(d, s, h, pf)                                                           \
  case d:                                                                                     \
    return a.feat.dtype == 1 ? launch_tile<1, s, h, pf>(a, ws, tab, n_obj, max_pts, stream, did)   \
                             : launch_tile<2, s, h, pf>(a, ws, tab, n_obj, max_pts, stream, did)
  switch (a.feat.D) {
    AURA_TILE_CASE(256, 1, 2, 2);
    AURA_TILE_CASE(512, 2, 2, 2);
    AURA_TILE_CASE(768, 3, 2, 2);
    AURA_TILE_CASE(1024, 4, 2, 2);
    AURA_TILE_CASE(1536, 6, 2, 2);
    default: return hipErrorInvalidValue;
  }
#undef AURA_TILE_CASE
}

}  // namespace aura
