// k_tile_fused for calls that keep no fused rows (aura_fuse_score_integrate): every wave takes tiles of its own from the projection
// to the stored scores.
//
// Without rows to store a tile is a short piece of work - 50 cells and 32 points, some 2000 vector instructions - made of a
// long chain: points, projections, depth texels, lists in LDS, feature rows, similarities, Eq. 4.  Nothing in it is bound by a
// rate of the machine, so what counts is how many chains are in flight.  With the work dealt out to producer, product and scoring waves
// (fuse_tile.hip, where rows are stored) a compute unit holds two tiles, and its vector units work 40 % of the time; here it holds
// twelve (objects of up to eight views) or eight, which never wait for each other.
//
// Per tile (lane = point % 32 in the projection, two views at a time, one per half of the wave):
//   A  every (point, view) pair is projected and tested (Eq. 1); all depth texels are requested before the first is looked at
//   B  per pair of views: the touched cells are marked in two 32 x 32-bit maps, rows counted by a scan over the half wave's lanes;
//      a point's four cells then know their places in the tile's list.  Views whose box is larger give each pair four entries of
//      its own.  The list is that of k_tile_prepare, cell for cell, so the sums have the bits of the two kernels.
//   C  the weights, in two 16-bit terms, as k-steps in the operand layout of the matrix cores, in the wave's own LDS
//   D  per 128 channels the product of weights and cell rows (fuse_tile_core.hpp) and its squares, for the norm: nothing else of
//      the row is needed
//   E  the scores as a product of the same weights with the per-cell similarities, as in k_tile_scores, and their epilogue
// A tile with more k-steps than the wave's LDS holds goes through C to E piece by piece: the pieces are made again for every 128
// channels, in the same order.  One with more than its quota (points in no order) goes to the lists of fuse_tile_lists.hpp.
#include <algorithm>

#include "aura_device.hpp"
#include "fuse_args.hpp"
#include "fuse_tile_core.hpp"
#include "fuse_tile_lists.hpp"
#include "launch.hpp"
#include "scores_epilogue.hpp"

namespace aura {

constexpr int kTeam = 4;   // waves of a workgroup: what they share is the table of properties and the lists at the end

// MANY: objects of more than eight views.
template <bool MANY>
constexpr int wave_steps() { return MANY ? 7 : 5; }   // k-steps in a wave's LDS
template <bool MANY>
constexpr int waves_per_simd() { return MANY ? 2 : 3; }
constexpr int kPairs = 4;              // pairs of views that a wave works on at a time
constexpr int kGroupViews = 2 * kPairs;
constexpr int kListViews = 16;         // the list is filled up to whole k-steps behind every 16 views, as the producers of fuse_tile.hip do

template <bool MANY>
struct __attribute__((aligned(16))) WaveScratch {
  TileStep step[wave_steps<MANY>()];                            // (cell: number of the cell, not its offset)
  float cam[MANY ? kWaveViews : kGroupViews][16];               // camera rows of the wave's object
  uint32_t bits[kPairs][2][kWinSide + 4];                       // maps of touched cells
  uint32_t vmask[MANY ? kWaveViews : kGroupViews];              // which of the tile's points each view sees
};

typedef const float __attribute__((address_space(3))) * wave_floats;
typedef const FuseArgs __attribute__((address_space(4))) * const_args;

// Inclusive sum over the lanes of each half of the wave.
__device__ __forceinline__ int half_wave_scan(int v) {
  v = row_shift_add<0x111>(v);   // row_shr:1
  v = row_shift_add<0x112>(v);
  v = row_shift_add<0x114>(v);
  v = row_shift_add<0x118>(v);
  return v + __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
}

// n zero bytes from p on, by one wave.
__device__ __forceinline__ void wave_zero(void* dst, long long n, int lane) {
  char* p = static_cast<char*>(dst);
  const int head = (int)min((long long)(-reinterpret_cast<uintptr_t>(p) & 15), n);
  if (lane < head) p[lane] = 0;
  p += head;
  n -= head;
  for (long long o = 16 * lane; o + 16 <= n; o += 16 * kWave) *reinterpret_cast<u32x4*>(p + o) = u32x4{0u, 0u, 0u, 0u};
  const int tail = (int)(n & 15);
  if (lane < tail) p[n - tail + lane] = 0;
}

// The products of one k-step with 128 channels; FIRST: into sums that are zero.
template <int DT, bool FIRST>
__device__ __forceinline__ void wave_products(const StepA& w, const StepQ<1>& r, f32x16 (&acc)[4]) {
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    u32x4 b;
#pragma unroll
    for (int e2 = 0; e2 < 4; ++e2)
      b[e2] = __builtin_amdgcn_perm(r.q[0][2 * e2 + 1][t >> 1], r.q[0][2 * e2][t >> 1], (t & 1) ? 0x07060302u : 0x05040100u);
    const f32x16 zero = {};
    acc[t] = mma<DT>(w.hi, b, FIRST ? zero : acc[t]);
    acc[t] = mma<DT>(w.lo, b, acc[t]);
  }
}

// Omega^T += G^T . W^T over k-steps from .. to - 1 (three partial products per k-step, see k_tile_scores).
template <int DT, int MT>
__device__ __forceinline__ void wave_scores(const TileStep* st, int from, int to, const TileScoring& sc, int lane, f32x16* acc) {
  const int pt = lane & 31, g = lane >> 5;
  struct Rows { uint32_t v[MT][8]; } g0, g1;
  auto request = [&](int s, Rows& r) {
    const u32x4 c0 = *reinterpret_cast<const u32x4*>(&st[s].cell[8 * g]);
    const u32x4 c1 = *reinterpret_cast<const u32x4*>(&st[s].cell[8 * g + 4]);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t at = __umul24(e < 4 ? c0[e] : c1[e - 4], 4u * (uint32_t)sc.Kpad) + 4u * pt;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) r.v[mt][e] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(sc.G) + (at + 128u * mt));
    }
  };
  auto products = [&](int s, const Rows& r) {
    const u32x4 w_hi = st[s].a_hi[lane], w_lo = st[s].a_lo[lane];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      u32x4 g_hi, g_lo;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        g_hi[q] = __builtin_amdgcn_perm(r.v[mt][2 * q + 1], r.v[mt][2 * q], 0x05040100u);
        g_lo[q] = __builtin_amdgcn_perm(r.v[mt][2 * q + 1], r.v[mt][2 * q], 0x07060302u);
      }
      acc[mt] = mma<DT>(g_hi, w_hi, acc[mt]);
      acc[mt] = mma<DT>(g_hi, w_lo, acc[mt]);
      acc[mt] = mma<DT>(g_lo, w_hi, acc[mt]);
    }
  };
  if constexpr (MT == 4) {   // (no registers for a second set)
    for (int s = from; s < to; ++s) {
      request(s, g0);
      products(s, g0);
    }
    return;
  }
  if (from >= to) return;
  request(from, g0);
  for (int s = from; s < to; s += 2) {   // the next k-step's rows are on their way
    if (s + 1 < to) request(s + 1, g1);
    products(s, g0);
    if (s + 1 < to) {
      if (s + 2 < to) request(s + 2, g0);
      products(s + 1, g1);
    }
  }
}

// DT: 1 bf16, 2 fp16 feature maps.  MT: 1: up to 32 materials; 4: more (two or four tiles of them: 33 to 64 materials run with the
// registers of four, `half_tiles`).  Three waves per SIMD leave 168 registers per lane, and up to eight views spill beyond them: 28 bytes of
// scratch per lane with one tile of materials, 140 with four (144 with SIFTED); two waves per SIMD (MANY) spill nothing.  SIFTED: after
// k_tile_sift, only the tiles on the objects' lists.
template <int DT, bool MANY, int MT, bool SIFTED>
__global__ __launch_bounds__(kTeam* kWave) __attribute__((amdgpu_waves_per_eu(waves_per_simd<MANY>(), waves_per_simd<MANY>())))
void k_tile_fused(FuseArgs fa, TileWs ws, int n_obj, int lists_only, ObjTable tab) {
  constexpr int kSteps = wave_steps<MANY>();
  __shared__ WaveScratch<MANY> s_wave[kTeam];
  __shared__ __attribute__((aligned(16))) float s_ys[kScoreTileM * MT * kScoreMaxP];
  __shared__ float s_unseen[kScoreMaxP];   // properties of a point that nobody sees
  __shared__ int s_job[4];                 // see drain_tiles
  __shared__ int s_drain;                  // whether this workgroup looks at the lists of push_tile at its end

  const TileScoring& sc = fa.scoring;
  const int tid = threadIdx.x;
  int lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  WaveScratch<MANY>& my = s_wave[wave];
  const bool half_tiles = MT == 4 && sc.Kpad == 64;   // uniform

  if (tid == 0) s_drain = 0;
  if (sc.prop) {
    if (half_tiles) stage_properties<2>(s_ys, sc.y, sc.K, sc.P, tid, kTeam * kWave);
    else stage_properties<MT>(s_ys, sc.y, sc.K, sc.P, tid, kTeam * kWave);
    if (wave == 1) unseen_properties(sc.K, sc.P, sc.y, sc.unseen_zero != 0, lane, s_unseen);
  }

  // The tiles of all objects in one row, object after object: lane b holds where object b's begin.  (SIFTED: those on its list,
  // unless it has none because nearly all are seen.)
  bool all_tiles = true;   // lane b: object b has no list
  int first = 0, total;
  {
    int n = 0;
    if (lane < n_obj) {
      n = (tab.o[lane].n_pts + kTilePts - 1) / kTilePts;
      if constexpr (SIFTED) {
        const unsigned listed = ws.counters[8 * (ws.obj_base + lane) + kSeenWord];
        all_tiles = listed == kAllSeen;
        if (!all_tiles) n = (int)listed;
        else if (lists_only) n = 0;
      }
    }
    int inc = half_wave_scan(n);
    const int lower = __builtin_amdgcn_readlane(inc, 31);
    if (lane >= 32) inc += lower;
    first = lane < n_obj ? inc - n : 0x7fffffff;
    total = __builtin_amdgcn_readlane(inc, 63);
  }
  const unsigned long long unlisted = __ballot(all_tiles);

  // Tiles are handed out by tickets, the first two of every wave without asking.  An atomic operation on a word takes 11 to 15 ns, in the
  // same 32 bytes one after the other, and in the same 128 bytes 5 ns apiece (eight words beside each other, asked by 3072 waves at
  // the start: 39 us; in lines of their own 9.5): each XCD's word is in 32 bytes of its own, of the eight words per object.
  const int xcd = blockIdx.x % kXcd;
  const XcdTiles mine(total, xcd);
  const int waves = (int)gridDim.x / kXcd * kTeam;   // of the XCD
  unsigned* __restrict__ ctr = ws.counters + 8 * ws.obj_base + launch_ticket_word(xcd, n_obj);
  auto ticket = [&]() {
    int t = 0;
    if (lane == 0) t = (int)atomicAdd(ctr, 1u) + 2 * waves;
    return t;
  };
  __syncthreads();

  // What is on its way for the tiles ahead: the ticket of the one after the next, the next one's number, and its points.
  int t_ahead = (int)blockIdx.x / kXcd * kTeam + wave;
  bool asked = false;
  int obj_next = 0, entry = -1;   // the next tile: its object, its number within it (-1: none)
  auto look_up = [&]() {          // the tile of the ticket that has arrived; and asks for the one behind it
    const int t = __builtin_amdgcn_readfirstlane(t_ahead);
    if (t >= mine.len) {
      // (who looks at the lists at the end: the workgroups that pushed, and those that find now that somebody has)
      if (lane == 0 && __hip_atomic_load(ws.status + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) s_drain = 1;
      entry = -1;
      return;
    }
    const int at = mine.at(t);
    obj_next = n_obj == 1 ? 0 : __builtin_popcountll(__ballot(first <= at)) - 1;
    const int pos = at - __builtin_amdgcn_readlane(first, obj_next);
    entry = pos;
    if constexpr (SIFTED) {
      if (!((unlisted >> obj_next) & 1)) entry = ws.hdr[tab.o[obj_next].tile_begin + pos].listed;
    }
    t_ahead = asked ? ticket() : t + waves;
    asked = true;
  };
  look_up();

  const_args args = (const_args)__builtin_amdgcn_kernarg_segment_ptr();
  const wave_floats cam = (wave_floats)&my.cam[0][0];
  int cam_obj = -1, obj, tile;
  float3 pt;
  auto next_points = [&]() {   // moves on to the tile whose number has arrived, and requests its points
    obj = obj_next;
    tile = __builtin_amdgcn_readfirstlane(entry);
    if (tile < 0) return;
    const int li0 = tile * kTilePts;
    const int p = lane & 31;
    const float* x = fa.xyz + 3 * (tab.o[obj].pt_begin + (li0 + p < tab.o[obj].n_pts ? li0 + p : 0));
    pt = float3{x[0], x[1], x[2]};
  };
  next_points();
  if (tile >= 0) look_up();

  while (tile >= 0) {
    // opaque to the optimiser: otherwise some hundred addresses that follow from the lane alone are kept across the tile loop, in
    // scratch memory
    asm volatile("" : "+v"(lane), "+s"(args));
    const FuseArgs& fa = *(const FuseArgs*)args;
    const TileScoring& sc = fa.scoring;
    const int Hf = fa.feat.Hf, Wf = fa.feat.Wf;
    const uint32_t row_bytes = (uint32_t)fa.feat.D * 2u;
    const int pieces = fa.feat.D / kHalf;
    const char* __restrict__ feat = static_cast<const char*>(fa.feat.feat);
    const bool zero_known = 0.0f * sc.inv_T == 0.0f;   // (otherwise the epilogue says what equal similarities give)
    const int p = lane & 31, h = lane >> 5;
    const ObjRange ob = tab.o[obj];
    const int blk = tile, li0 = blk * kTilePts, rows = min(kTilePts, ob.n_pts - li0);
    const long long i0 = ob.pt_begin + li0;
    const int nv = ob.n_views;
    const int here = obj;
    if (obj != cam_obj) {   // uniform
      cam_obj = obj;
      for (int q = lane; q < nv * 16; q += kWave) my.cam[q >> 4][q & 15] = fa.vis.cam[(long long)ob.view_begin * 16 + q];
      wave_sync();
    }

    const float3 at_pt = pt;
    next_points();
    if (tile >= 0) look_up();

    // ---- A: projections of eight views, and the requests for their depth texels
    Proj pj[kPairs];
    float dep[kPairs];
    bool fr[kPairs];
    auto project_views = [&](int v0) {
#pragma unroll
      for (int j = 0; j < kPairs; ++j) {
        dep[j] = 1.0f;
        fr[j] = false;
        pj[j] = Proj{0.0f, 0.0f, 0.0f};
        if (v0 + 2 * j >= nv) continue;   // uniform
        const int vl = min(v0 + 2 * j + h, nv - 1);
        pj[j] = project(cam + vl * 16, at_pt.x, at_pt.y, at_pt.z);
        fr[j] = in_frustum(fa.vis, pj[j]);
        if (fa.vis.depth)
          dep[j] = fa.vis.depth[(long long)(ob.view_begin + vl) * fa.vis.H * fa.vis.W + (fr[j] ? depth_texel(fa.vis, pj[j]) : 0)];
      }
    };
    project_views(0);

    int length = 0, cnt = 0, n = 0;   // cells on the list; views that see the point; k-steps
    u32x4* const lds_steps = reinterpret_cast<u32x4*>(&my.step[0]);
    u32x4* const far_steps = reinterpret_cast<u32x4*>(ws.steps + (long long)(ob.tile_begin + blk) * ws.quota);   // those beyond kSteps
    constexpr int kVecs = sizeof(TileStep) / 16;
    auto pad_list = [&]() {   // entries that pad the last k-step: a cell that exists, with weight 0
      if (lane < n * kStepCells - length) {
        TileStep* const steps = n > kSteps ? reinterpret_cast<TileStep*>(far_steps) : &my.step[0];
        steps[n - 1].cell[(length + lane) & 15] = (uint32_t)(ob.view_begin * Hf * Wf);
      }
    };
    for (int v0 = 0; v0 < nv; v0 += kGroupViews) {
      if (MANY && v0 > 0 && v0 % kListViews == 0) {
        pad_list();
        length = n * kStepCells;
      }
      // ---- B: tests; every seen pair's places in the list
      int xy[kPairs], org[kPairs];   // first cell (y0 << 16 | x0, -1: not seen) and the first one of the view's map
      float ax[kPairs], ay[kPairs];
      bool map[kPairs];
      unsigned long long mask[kPairs], any = 0;
#pragma unroll
      for (int j = 0; j < kPairs; ++j) {
        xy[j] = -1;
        org[j] = 0;
        ax[j] = ay[j] = 0.0f;
        map[j] = false;
        const bool seen = v0 + 2 * j + h < nv && p < rows && fr[j] && (fa.vis.frustum_only || passes_depth(fa.vis, pj[j], dep[j]));
        mask[j] = __ballot(seen);
        any |= mask[j];
        if (lane == 0) *reinterpret_cast<u32x2*>(&my.vmask[v0 + 2 * j]) = u32x2{(uint32_t)mask[j], (uint32_t)(mask[j] >> 32)};
        if (mask[j] == 0) continue;   // uniform
        s16x2 lo2 = {0x7fff, 0x7fff}, hi2 = {-1, -1};   // (x, y) of the first / second cell
        if (seen) {
          const Tap tx = tap_axis(pj[j].u, fa.feat.pitch_x, Wf), ty = tap_axis(pj[j].v, fa.feat.pitch_y, Hf);
          ax[j] = tx.a;
          ay[j] = ty.a;
          xy[j] = (ty.i0 << 16) | tx.i0;
          lo2 = s16x2{(short)tx.i0, (short)ty.i0};
          hi2 = s16x2{(short)tx.i1, (short)ty.i1};
          ++cnt;
        }
        lo2 = half_wave_reduce<true>(lo2);
        hi2 = half_wave_reduce<false>(hi2);
        // the halves' boxes, on the scalar unit
        auto box = [&](int at, bool& fits) {
          const int l = __builtin_amdgcn_readlane(__builtin_bit_cast(int, lo2), at), u = __builtin_amdgcn_readlane(__builtin_bit_cast(int, hi2), at);
          fits = (short)u - (short)l < kWinSide && (u >> 16) - (l >> 16) < kWinSide;   // (nobody seen: negative)
          return l;
        };
        bool map_a, map_b;
        const int box_a = box(31, map_a), box_b = box(63, map_b);
        org[j] = h ? box_b : box_a;
        map[j] = h ? map_b : map_a;
      }
      // the next views' depth texels arrive while these views' cells are listed
      if (MANY && v0 + kGroupViews < nv) project_views(v0 + kGroupViews);
      if (any == 0) continue;   // uniform

#pragma unroll
      for (int j = 0; j < kPairs; ++j) my.bits[j][h][p] = 0u;
      wave_sync();
      auto row_of = [&](int j) { return (xy[j] >> 16) - (org[j] >> 16); };
      auto col_of = [&](int j) { return (xy[j] & 0xffff) - (int)(short)org[j]; };
#pragma unroll
      for (int j = 0; j < kPairs; ++j) {
        if (xy[j] >= 0 && map[j]) {
          const uint32_t cells = ((xy[j] & 0xffff) + 1 < Wf ? 3u : 1u) << col_of(j);
          atomicOr(&my.bits[j][h][row_of(j)], cells);
          if ((xy[j] >> 16) + 1 < Hf) atomicOr(&my.bits[j][h][row_of(j) + 1], cells);
        }
      }
      wave_sync();
      // the rows' set bits before each row, by the lanes of the half; then every point looks its two rows up
      uint32_t place[kPairs];   // of the first cell of the upper and (from bit 16) of the lower row; bit 15: private entries
      const int before_group = n;
#pragma unroll
      for (int j = 0; j < kPairs; ++j) {
        place[j] = 0u;
        if (mask[j] == 0) continue;   // uniform
        const bool mark = xy[j] >= 0 && map[j];
        const int r0 = mark ? row_of(j) : 0, r1 = mark && (xy[j] >> 16) + 1 < Hf ? r0 + 1 : r0;
        const uint32_t row = my.bits[j][h][p], row0 = my.bits[j][h][r0], row1 = my.bits[j][h][r1];
        const int set = __popc(row), inc = half_wave_scan(set);
        const int before0 = __builtin_amdgcn_ds_bpermute(4 * (32 * h + r0), inc - set);
        const int before1 = __builtin_amdgcn_ds_bpermute(4 * (32 * h + r1), inc - set);
        const unsigned long long maps = __ballot(map[j]);
        const uint32_t mask_a = (uint32_t)mask[j], mask_b = (uint32_t)(mask[j] >> 32);
        const int len_a = (uint32_t)maps != 0u ? __builtin_amdgcn_readlane(inc, 31) : 4 * __popc(mask_a);
        const int len_b = (uint32_t)(maps >> 32) != 0u ? __builtin_amdgcn_readlane(inc, 63) : 4 * __popc(mask_b);
        const int base = h ? length + len_a : length;
        const uint32_t left = (1u << (col_of(j) & 31)) - 1u;
        const uint32_t own = base + 4 * __popc((h ? mask_b : mask_a) & ((1u << p) - 1u));
        place[j] = map[j] ? (uint32_t)(base + before0 + __popc(row0 & left)) | (uint32_t)(base + before1 + __popc(row1 & left)) << 16
                          : own | (own + 2) << 16 | 0x8000u;
        length += len_a + len_b;
      }
      n = (length + kStepCells - 1) / kStepCells;
      if (n > ws.quota) break;   // uniform

      // ---- C: zero weights in the k-steps that have come in use, then these views' weights and cells
      for (int q = 128 * before_group + lane; q < 128 * min(n, kSteps); q += kWave) lds_steps[(q >> 7) * kVecs + 4 + (q & 127)] = u32x4{0u, 0u, 0u, 0u};
      if (n > kSteps) {   // uniform
        for (int q = kVecs * max(before_group, kSteps) + lane; q < kVecs * n; q += kWave) far_steps[q] = u32x4{0u, 0u, 0u, 0u};
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      }
      wave_sync();
#pragma unroll
      for (int j = 0; j < kPairs; ++j) {
        if (xy[j] < 0) continue;
        const int x0 = xy[j] & 0xffff, y0 = xy[j] >> 16;
        const bool has_x1 = x0 + 1 < Wf, has_y1 = y0 + 1 < Hf, apart = (place[j] & 0x8000u) != 0u;
        const float wgt[4] = {(1.0f - ax[j]) * (1.0f - ay[j]), ax[j] * (1.0f - ay[j]), (1.0f - ax[j]) * ay[j], ax[j] * ay[j]};
        const bool on[4] = {true, has_x1, has_y1, has_x1 && has_y1};
        const int cell0 = ((ob.view_begin + v0 + 2 * j + h) * Hf + y0) * Wf + x0;
        const int dx = has_x1 ? 1 : 0, dy = has_y1 ? Wf : 0;
        const int cell[4] = {cell0, cell0 + dx, cell0 + dy, cell0 + dx + dy};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int at = (int)(k < 2 ? place[j] & 0x7fffu : place[j] >> 16) + (k & 1);
          uint16_t hi, lo;
          split_weight<DT>(wgt[k], hi, lo);
          auto put = [&](TileStep* steps) {
            TileStep& st = steps[at >> 4];
            const int c = at & 15;
            st.cell[c] = (uint32_t)cell[k];
            if (on[k]) {
              reinterpret_cast<uint16_t*>(&st.a_hi[(c >> 3) * kTilePts + p])[c & 7] = hi;
              reinterpret_cast<uint16_t*>(&st.a_lo[(c >> 3) * kTilePts + p])[c & 7] = lo;
            }
          };
          if (on[k] || apart) {
            if (at < kStepCells * kSteps) put(&my.step[0]);
            else put(reinterpret_cast<TileStep*>(far_steps));
          }
        }
      }
    }
    if (n > ws.quota) {   // uniform
      if (fa.out_vis && lane < rows) {   // mask columns beyond the object's views (the others: gather_point)
        uint8_t* __restrict__ vrow = fa.out_vis + (i0 + lane) * fa.vis_pitch;
        for (int v = nv; v < fa.vis_pitch; ++v) vrow[v] = 0;
      }
      push_tile(ws, ob.tile_begin + blk, here, lane);
      if (lane == 0) s_drain = 1;
      continue;
    }
    if (n == 0 && zero_known) {   // uniform: nobody sees the tile's points
      wave_zero(sc.scores + i0 * sc.K, (long long)rows * sc.K * 4, lane);
      if (fa.out_vis) wave_zero(fa.out_vis + i0 * fa.vis_pitch, (long long)rows * fa.vis_pitch, lane);
      if (lane < rows) {
        if (fa.out_count) fa.out_count[i0 + lane] = 0;
        if (sc.label) sc.label[i0 + lane] = 0;
      }
      if (sc.prop)
        for (int o = lane; o < rows * sc.P; o += kWave) sc.prop[i0 * sc.P + o] = s_unseen[o % sc.P];
      continue;
    }

    pad_list();
    if (n > kSteps) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    wave_sync();

    // ---- D: per 128 channels the product and its squares
    const int m = min(kSteps, n);   // k-steps in LDS
    const TileStep* const far = reinterpret_cast<const TileStep*>(far_steps);
    float sum = 0.0f;   // squares of the channels of point lane_value(lane) (see half_wave_sums)
    auto rows_of = [&](const u32x4& c0, const u32x4& c1, int c, StepQ<1>& r) {   // channels 128 c .. of the lane's eight cells
      const uint32_t lane_off = (uint32_t)(c * kHalf + 4 * p) * 2u;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        r.q[0][e] = *reinterpret_cast<const u32x2*>(feat + (__umul24(e < 4 ? c0[e] : c1[e - 4], row_bytes) + lane_off));
    };
    auto request = [&](const TileStep& st, int c, StepQ<1>& r) {
      rows_of(*reinterpret_cast<const u32x4*>(&st.cell[8 * h]), *reinterpret_cast<const u32x4*>(&st.cell[8 * h + 4]), c, r);
    };
    auto weights = [&](const TileStep& st) { return StepA{st.a_hi[lane], st.a_lo[lane]}; };
    auto add_squares = [&](const f32x16 (&acc)[4]) {
      float v[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float sq = 0.0f;
#pragma unroll
        for (int t = 0; t < 4; ++t) sq = __builtin_fmaf(acc[t][r], acc[t][r], sq);
        v[r] = sq;
      }
      sum += half_wave_sums<1>(v, lane);
    };
    // (the rows of the next channels are on their way while the squares of these are added up)
    f32x16 acc[4];
    StepQ<1> q0, q1;
    if (n == 1) {   // uniform; pieces is even
      request(my.step[0], 0, q0);
      for (int c = 0; c < pieces; c += 2) {
        const StepA w = weights(my.step[0]);
        request(my.step[0], c + 1, q1);
        wave_products<DT, true>(w, q0, acc);
        add_squares(acc);
        if (c + 2 < pieces) request(my.step[0], c + 2, q0);
        wave_products<DT, true>(w, q1, acc);
        add_squares(acc);
      }
    } else if (n > 1) {
      request(my.step[0], 0, q0);
      request(my.step[1], 0, q1);
      for (int c = 0; c < pieces; ++c) {
        wave_products<DT, true>(weights(my.step[0]), q0, acc);
        for (int s = 1; s < m; s += 2) {
          if (s + 1 < m) request(my.step[s + 1], c, q0);
          wave_products<DT, false>(weights(my.step[s]), q1, acc);
          if (s + 1 < m) {
            if (s + 2 < m) request(my.step[s + 2], c, q1);
            wave_products<DT, false>(weights(my.step[s + 1]), q0, acc);
          }
        }
        if (n > kSteps) {   // uniform; those in memory
          if constexpr (MANY) {
            // the cells four, the rows two and the weights one k-step ahead (300 000 points of 32 views of 56 x 56 cells 801 -> 682 us; with up to
            // eight views there are no registers for it: 120 000 points of 8 such views 103 -> 126)
            const int last = n - 1;
            u32x4 cells[2][2];
            auto far_cells = [&](int s, u32x4 (&r)[2]) {
              const u32x4* from = reinterpret_cast<const u32x4*>(&far[min(s, last)].cell[8 * h]);
              r[0] = from[0];
              r[1] = from[1];
            };
            far_cells(kSteps, cells[0]);
            far_cells(kSteps + 1, cells[1]);
            StepA w = weights(far[kSteps]);
            rows_of(cells[0][0], cells[0][1], c, q0);
            far_cells(kSteps + 2, cells[0]);
            rows_of(cells[1][0], cells[1][1], c, q1);
            far_cells(kSteps + 3, cells[1]);
            for (int s = kSteps; s < n; s += 2) {
              const StepA w1 = weights(far[min(s + 1, last)]);
              wave_products<DT, false>(w, q0, acc);
              rows_of(cells[0][0], cells[0][1], c, q0);
              far_cells(s + 4, cells[0]);
              if (s + 1 < n) {
                w = weights(far[min(s + 2, last)]);
                wave_products<DT, false>(w1, q1, acc);
                rows_of(cells[1][0], cells[1][1], c, q1);
                far_cells(s + 5, cells[1]);
              }
            }
          } else {
            for (int s = kSteps; s < n; ++s) {
              request(far[s], c, q0);
              wave_products<DT, false>(weights(far[s]), q0, acc);
            }
          }
        }
        if (c + 1 < pieces) {
          request(my.step[0], c + 1, q0);
          request(my.step[1], c + 1, q1);
        }
        add_squares(acc);
      }
    }

    // ---- E: the scores
    f32x16 omega[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 16; ++r) omega[mt][r] = 0.0f;
    auto add_scores = [&](const TileStep* st, int from, int to) {
      if (half_tiles) {
        if constexpr (MT == 4) wave_scores<DT, 2>(st, from, to, sc, lane, omega);
      } else {
        wave_scores<DT, MT>(st, from, to, sc, lane, omega);
      }
    };
    add_scores(my.step, 0, m);
    if (n > kSteps) add_scores(far, kSteps, n);

    // ---- the factor of the lane's point: mean and L2 norm
    const int seen_by = cnt + __shfl_xor(cnt, 32, kWave);
    float factor;
    {
      const int r = lane_value<1>(p);
      float* tot = reinterpret_cast<float*>(&my.bits[0][0][0]);
      wave_sync();
      tot[8 * (r >> 2) + 4 * h + (r & 3)] = sum;
      wave_sync();
      factor = point_factor(seen_by, tot[p], fa.norm_eps, fa.mean_only);
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 16; ++r) omega[mt][r] *= factor;

    // ---- what goes to memory
    if (h == 0 && p < rows && fa.out_count) fa.out_count[i0 + p] = seen_by;
    if (fa.out_vis && p < rows) {
      // lane = point, and the halves take eight views in turn
      uint8_t* __restrict__ vrow = fa.out_vis + (i0 + p) * fa.vis_pitch;
      const bool pairs = (fa.vis_pitch & 7) == 0 && (reinterpret_cast<uintptr_t>(fa.out_vis) & 7) == 0;
      const bool words = (fa.vis_pitch & 3) == 0 && (reinterpret_cast<uintptr_t>(fa.out_vis) & 3) == 0;
      for (int v0 = 8 * h; v0 < nv; v0 += 16) {
        uint32_t wd[2] = {0u, 0u};
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (v0 + e < nv) wd[e >> 2] |= ((my.vmask[v0 + e] >> p) & 1u) << (8 * (e & 3));
        if (pairs && v0 + 8 <= nv) {
          *reinterpret_cast<u32x2*>(vrow + v0) = u32x2{wd[0], wd[1]};
        } else {
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            if (words && v0 + 4 * q + 4 <= nv) {
              *reinterpret_cast<uint32_t*>(vrow + v0 + 4 * q) = wd[q];
            } else {
              for (int e = 0; e < 4 && v0 + 4 * q + e < nv; ++e) vrow[v0 + 4 * q + e] = (uint8_t)((wd[q] >> (8 * e)) & 1u);
            }
          }
        }
      }
      if (h == 1)
        for (int v = nv; v < fa.vis_pitch; ++v) vrow[v] = 0;
    }
    wave_sync();
    float* stage = reinterpret_cast<float*>(&my.step[0]);
    static_assert(score_stage_floats<16>() * sizeof(float) <= sizeof(my.step), "the rows' way to memory leads through the k-steps' place");
    if (half_tiles) {
      if constexpr (MT == 4) {
        f32x16 two[2] = {omega[0], omega[1]};
        finish_scores_staged<2, 16>(two, i0, rows, lane, sc.K, sc.P, sc.inv_T, s_ys, sc.scores, sc.prop, sc.label, sc.unseen_zero != 0, stage);
      }
    } else {
      finish_scores_staged<MT, 16>(omega, i0, rows, lane, sc.K, sc.P, sc.inv_T, s_ys, sc.scores, sc.prop, sc.label, sc.unseen_zero != 0, stage);
    }
    wave_sync();
  }

  __syncthreads();
  if (s_drain != 0) drain_tiles<DT, true, 2>(fa, ws, tab, blockIdx.x, s_job, wave, kTeam, lane);
}

// ------------------------------------------------------------------------------------ host

template <int DT, bool MANY, int MT>
static hipError_t launch_waves(const FuseArgs& a, const TileWs& ws, const ObjTable& tab, int n_obj, long long tiles, bool sifted,
                               bool lists_only, hipStream_t stream) {
  const long long groups = std::min<long long>((tiles + kTeam * kXcd - 1) / (kTeam * kXcd) * kXcd, 256 * waves_per_simd<MANY>());
  const dim3 grid((unsigned)groups), block(kTeam * kWave);
  if (sifted) hipLaunchKernelGGL((k_tile_fused<DT, MANY, MT, true>), grid, block, 0, stream, a, ws, n_obj, (int)lists_only, tab);
  else hipLaunchKernelGGL((k_tile_fused<DT, MANY, MT, false>), grid, block, 0, stream, a, ws, n_obj, (int)lists_only, tab);
  return hipGetLastError();
}

hipError_t launch_tile_waves(const FuseArgs& a, const TileWs& ws, const ObjTable& tab, int n_obj, int max_views, long long tiles,
                             bool sifted, bool lists_only, hipStream_t stream) {
#define AURA_WAVES(dt)                                                                                              \
  if (a.scoring.Kpad == kScoreTileM) {                                                                              \
    if (max_views <= kGroupViews) return launch_waves<dt, false, 1>(a, ws, tab, n_obj, tiles, sifted, lists_only, stream);                     \
    return launch_waves<dt, true, 1>(a, ws, tab, n_obj, tiles, sifted, lists_only, stream);                                       \
  }                                                                                                                 \
  if (max_views <= kGroupViews) return launch_waves<dt, false, 4>(a, ws, tab, n_obj, tiles, sifted, lists_only, stream);                       \
  return launch_waves<dt, true, 4>(a, ws, tab, n_obj, tiles, sifted, lists_only, stream)
  if (a.feat.dtype == 1) { AURA_WAVES(1); }
  AURA_WAVES(2);
#undef AURA_WAVES
}

}  // namespace aura
