// Tiles that need more k-steps than they own, in the matrix-core fusion kernels: the lists they go to and the gather that fuses them.
#pragma once

#include "aura_device.hpp"
#include "fuse_args.hpp"
#include "fuse_tile_core.hpp"

namespace aura {

// The slow way out when a tile needs more k-steps than it owns (points far apart): one wave fuses a point by a gather
// (lanes over channels, 512 channels per sweep, the whole row in registers; the rows of two views in flight together).
// The row is stored when the call has a place for it (FuseArgs::fused).  When the call wants scores as well
// (FuseArgs::scoring), they are taken here from the row in registers, so that no later kernel needs the row: omega_k is
// the fp32 dot product with the fp32 text embedding (largest error 1.2e-7 on 10 601 points of 512 channels; blended from
// the per-cell similarities, which hold two 16-bit terms, it was 1.2e-6 for bf16 maps), then Eq. 4 and the label with
// lanes over the materials.
constexpr int kGatherSweeps = 3;   // 512 channels each: D <= 1536 on this path

template <int DT>
__device__ __forceinline__ void widen_16(uint32_t w, float& lo, float& hi) {
  if constexpr (DT == 1) {
    lo = __uint_as_float(w << 16);
    hi = __uint_as_float(w & 0xffff0000u);
  } else {
    lo = (float)__builtin_bit_cast(_Float16, (uint16_t)(w & 0xffffu));
    hi = (float)__builtin_bit_cast(_Float16, (uint16_t)(w >> 16));
  }
}

// SCORES: whether such a call can want scores.  SWEEPS: of 512 channels each.  In the kernels of three waves per SIMD, whose 168
// registers three sweeps outgrow, as many as the channels fill (three with 100 bytes of scratch memory / two: 200 000 points in no
// order, 16 views, 768 channels 2447 / 2237 us; as one kernel of two waves per SIMD it was 2357); elsewhere three (16 ragged objects
// of 3000 points and 256 channels 813 us, 902 with one).
template <int DT, bool SCORES, int SWEEPS>
__device__ __forceinline__ void gather_point(const FuseArgs& a, const ObjRange& ob, int li, int lane) {
  const TileScoring& sc = a.scoring;
  const int D = a.feat.D, Hf = a.feat.Hf, Wf = a.feat.Wf;
  const long long i = ob.pt_begin + li;
  const float x = a.xyz[3 * i], y = a.xyz[3 * i + 1], z = a.xyz[3 * i + 2];
  float acc[SWEEPS][8];
#pragma unroll
  for (int s = 0; s < SWEEPS; ++s)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[s][e] = 0.0f;
  int cnt = 0;
  for (int vb = 0; vb < ob.n_views; vb += kWave) {
    bool seen = false;
    int x0 = 0, y0 = 0;
    float ax = 0.0f, ay = 0.0f;
    if (vb + lane < ob.n_views) {
      const int v = ob.view_begin + vb + lane;
      const Proj p = project(a.vis.cam + (long long)v * 16, x, y, z);
      const float* dv = a.vis.depth ? a.vis.depth + (long long)v * a.vis.H * a.vis.W : nullptr;
      seen = visible(a.vis, dv, p) && view_kept(a, i, vb + lane);
      if (a.out_vis) a.out_vis[i * a.vis_pitch + vb + lane] = seen ? 1 : 0;
      if (seen) {
        const Tap tx = tap_axis(p.u, a.feat.pitch_x, Wf), ty = tap_axis(p.v, a.feat.pitch_y, Hf);
        x0 = tx.i0; ax = tx.a;
        y0 = ty.i0; ay = ty.a;
      }
    }
    unsigned long long m = __ballot(seen);
    cnt += __popcll(m);
    while (m) {
      // two views; of a single one left the second is the first again, its weights zero and its rows not added
      const int src0 = __builtin_ctzll(m);
      m &= m - 1;
      const bool two = m != 0;
      const int src1 = two ? __builtin_ctzll(m) : src0;
      m &= m - 1;
      float wgt[2][4];
      long long cell[2][4];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int src = q ? src1 : src0;
        const int sx0 = __builtin_amdgcn_readlane(x0, src), sy0 = __builtin_amdgcn_readlane(y0, src);
        const float sax = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ax), src));
        const float say = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ay), src));
        const int sx1 = sx0 + 1 < Wf ? sx0 + 1 : Wf - 1, sy1 = sy0 + 1 < Hf ? sy0 + 1 : Hf - 1;
        wgt[q][0] = (1.0f - sax) * (1.0f - say); wgt[q][1] = sax * (1.0f - say);
        wgt[q][2] = (1.0f - sax) * say;          wgt[q][3] = sax * say;
        const long long first = (long long)(ob.view_begin + vb + src) * Hf * Wf;
        cell[q][0] = first + sy0 * Wf + sx0; cell[q][1] = first + sy0 * Wf + sx1;
        cell[q][2] = first + sy1 * Wf + sx0; cell[q][3] = first + sy1 * Wf + sx1;
      }
      u32x4 raw[SWEEPS][2][4];
#pragma unroll
      for (int s = 0; s < SWEEPS; ++s) {
        if (s * 8 * kWave >= D) break;   // uniform
        const int ch = min(s * 8 * kWave + 8 * lane, D - 8);
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int c = 0; c < 4; ++c)
            raw[s][q][c] = *reinterpret_cast<const u32x4*>(static_cast<const char*>(a.feat.feat) + (cell[q][c] * D + ch) * 2);
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (q == 1 && !two) break;   // uniform
#pragma unroll
        for (int s = 0; s < SWEEPS; ++s) {
          if (s * 8 * kWave >= D) break;   // uniform
#pragma unroll
          for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              float lo, hi;
              widen_16<DT>(raw[s][q][c][j], lo, hi);
              acc[s][2 * j] = __builtin_fmaf(wgt[q][c], lo, acc[s][2 * j]);
              acc[s][2 * j + 1] = __builtin_fmaf(wgt[q][c], hi, acc[s][2 * j + 1]);
            }
        }
      }
    }
  }
  // mean over the visible views (Eq. 2), then the L2 normalisation
  const float inv = cnt > 0 ? 1.0f / (float)cnt : 0.0f;
  float ss = 0.0f;
#pragma unroll
  for (int s = 0; s < SWEEPS; ++s) {
    const bool own = s * 8 * kWave + 8 * lane < D;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      acc[s][e] = own ? acc[s][e] * inv : 0.0f;
      ss = __builtin_fmaf(acc[s][e], acc[s][e], ss);
    }
  }
  if (!a.mean_only && cnt > 0) {   // uniform
    const float scale = 1.0f / fmaxf(sqrtf(wave_sum(ss)), a.norm_eps);
#pragma unroll
    for (int s = 0; s < SWEEPS; ++s)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[s][e] *= scale;
  }
  if (a.fused) {
    float* __restrict__ out_row = a.fused + i * D;
#pragma unroll
    for (int s = 0; s < SWEEPS; ++s) {
      const int ch = s * 8 * kWave + 8 * lane;
      if (ch < D) {
        *reinterpret_cast<f32x4*>(out_row + ch) = f32x4{acc[s][0], acc[s][1], acc[s][2], acc[s][3]};
        *reinterpret_cast<f32x4*>(out_row + ch + 4) = f32x4{acc[s][4], acc[s][5], acc[s][6], acc[s][7]};
      }
    }
  }
  if (a.out_count && lane == 0) a.out_count[i] = cnt;

  if (SCORES && sc.G) {
    // Sec. 3.4.1 for this point, eight materials at a time (their reads in flight together): a dot product per lane over
    // its channels, then the sums over the wave.  Lane l keeps the similarities of materials l and l + 64.
    // With two sweeps (768 and 1024 channels, three waves per SIMD) the next eight materials' first reads go ahead of the sums: 168
    // registers do not hold the reads of both sweeps at a time as 256 do (points in no order, without / with: 12 objects of 33 333
    // points, 768 channels and 60 materials 1213 / 1120 us, 200 000 points and 128 materials 4752 / 4227).  Not elsewhere: sorted
    // points of 32 pixel maps 1460 -> 1467 us.
    constexpr bool kAhead = SWEEPS == 2;
    float mine[2] = {-INFINITY, -INFINITY};
    auto request = [&](f32x4 (&t)[8][2], int m0, int s) {
      const int ch = min(s * 8 * kWave + 8 * lane, D - 8);
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const f32x4* e = reinterpret_cast<const f32x4*>(sc.temb + (long long)min(m0 + q, sc.K - 1) * D + ch);
        t[q][0] = e[0];
        t[q][1] = e[1];
      }
    };
    f32x4 t[8][2];
    if constexpr (kAhead) request(t, 0, 0);
    for (int m0 = 0; m0 < sc.K; m0 += 8) {
      float dot[8] = {};
#pragma unroll
      for (int s = 0; s < SWEEPS; ++s) {
        if (s * 8 * kWave >= D) break;   // uniform
        if (s > 0 || !kAhead) request(t, m0, s);
        if (s * 8 * kWave + 8 * lane < D) {
#pragma unroll
          for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              dot[q] = __builtin_fmaf(acc[s][e], t[q][0][e], dot[q]);
              dot[q] = __builtin_fmaf(acc[s][4 + e], t[q][1][e], dot[q]);
            }
        }
      }
      if constexpr (kAhead) request(t, m0 + 8, 0);   // (past the last material: the last one again)
      // the eight sums in one: in each of three rounds a lane passes on the half it will not hold, and from there every
      // eight lanes hold one material
#pragma unroll
      for (int n = 4, o = kWave / 2; n > 0; n >>= 1, o >>= 1) {
        const bool upper = (lane & o) != 0;
#pragma unroll
        for (int q = 0; q < n; ++q) dot[q] = (upper ? dot[n + q] : dot[q]) + __shfl_xor(upper ? dot[q] : dot[n + q], o, kWave);
      }
#pragma unroll
      for (int o = 4; o > 0; o >>= 1) dot[0] += __shfl_xor(dot[0], o, kWave);
      const float here = __shfl(dot[0], 8 * (lane & 7), kWave);   // material m0 + lane % 8
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (m0 == ((lane + kWave * h) & ~7) && lane + kWave * h < sc.K) mine[h] = here;
    }
    float best = fmaxf(mine[0], mine[1]);
    int bidx = mine[1] > mine[0] ? lane + 64 : lane;   // a lane without a material holds -inf
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
      const float ob_ = __shfl_xor(best, o, kWave);
      const int oi = __shfl_xor(bidx, o, kWave);
      if (ob_ > best || (ob_ == best && oi < bidx)) { best = ob_; bidx = oi; }   // lowest index wins ties
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int m = lane + 64 * h;
      if (m < sc.K) sc.scores[i * sc.K + m] = mine[h];
    }
    if (sc.label && lane == 0) sc.label[i] = bidx;
    if (sc.prop) {
      float e[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) e[h] = lane + 64 * h < sc.K ? weight_exp((mine[h] - best) * sc.inv_T) : 0.0f;
      const float den = wave_sum(e[0] + e[1]);
      // all similarities exactly zero (nobody sees the point): zero properties where the caller asks for that
      const bool zero_row = sc.unseen_zero && __ballot((lane < sc.K && mine[0] != 0.0f) || (lane + 64 < sc.K && mine[1] != 0.0f)) == 0;
      for (int p = 0; p < sc.P; ++p) {
        float num = 0.0f;
#pragma unroll
        for (int h = 0; h < 2; ++h)
          if (lane + 64 * h < sc.K) num = __builtin_fmaf(e[h], sc.y[(lane + 64 * h) * sc.P + p], num);
        num = wave_sum(num);
        if (lane == 0) sc.prop[i * sc.P + p] = zero_row ? 0.0f : num / den;
      }
    }
  }
}

// Tiles without k-steps go to lists that the workgroups of the launch empty together when they have run out of tiles.
// Fused on the spot by the waves that found out, a single such tile held its workgroup up for hundreds of microseconds
// (32 points one after the other), and with it the end of the kernel (8 tiles of 8000 points, 20 views, 768 channels:
// 671 us for the step, 169 us with the lists).
// kLists stacks: word kListWord + l of TileWs::status holds the tile last pushed to list l, plus one (0: empty).  Of
// TileHdr::cnt, which such a tile does not use, word 0 holds the entry below it, word 1 its object and word 2 how many of its
// kParts parts have been taken.  Parts are taken by adding to that word, which every comer can do at once; only whoever
// finds all of them taken moves the head to the entry below.  (Popped part by part, by exchanges on the heads that fail
// whenever another one came first, the 6250 tiles of 200 000 points in no order took 18.8 ms, 2.5 ms now; 566 of 1504 tiles of
// 16 objects of 3000 points, 8 views and 256 channels 2520 us, 360 us now.)  A tile is
// pushed once per launch, so a head never returns to an entry that it has left, and the exchanges cannot be fooled by a
// reused one.  Nobody waits: a workgroup that finds the lists empty leaves, and one that pushed, or that took parts, looks
// at the lists again afterwards: all parts of all tiles are taken, and the lists empty, when the last one leaves.
// Everything the workgroups share goes through agent-scope atomics, which act on memory that all XCDs see, so no cache has
// to be written back or dropped: the words of an entry are complete (s_waitcnt) before the exchange that publishes it, and
// their readers take their address from what the exchange left.
constexpr int kParts = 8, kPartPts = kTilePts / kParts;
constexpr int kLists = 32, kListWord = 32;
// A workgroup of two or three waves takes four parts where this many tiles have been pushed: there the words that everybody adds to
// are what the lists wait for.  As many parts as waves / four, points in no order: 16 objects of 3000 points, 8 views and 256
// channels, one producer, 884 / 799 us (850 before the gather became faster), 20 of 10 000 and 4 views 2390 / 2081 (2345), 40 of
// 5000, 4 views, 512 channels, plain fusion 2504 / 2221.  With few tiles on the lists they are better spread over all who look:
// 8 sorted objects of 10 000 points 119 / 147.
constexpr unsigned kManyPushed = 1024;

__device__ __forceinline__ void push_tile(const TileWs& ws, int tile, int obj, int lane) {   // one lane of a wave
  if (lane == 0) {
    int* words = ws.hdr[tile].cnt;
    unsigned* head = ws.status + kListWord + tile % kLists;
    __hip_atomic_store(&words[1], obj, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&words[2], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned top = __hip_atomic_load(head, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bool done = false;
    while (!done) {
      __hip_atomic_store(&words[0], (int)top, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      done = __hip_atomic_compare_exchange_strong(head, &top, (unsigned)tile + 1u, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    atomicAdd(ws.status + 1, 1u);   // second status word: tiles fused by the gather
  }
}

// Called by all waves of a workgroup together, at the end of its life: the first wave takes as many parts as there are waves (see
// kManyPushed), four points each (those 16 objects, combined call: 359 us; half as many parts 420 us, whole tiles 407 us), and all
// share their points.  `turn`: the list where the workgroup looks first; `job`: four words of LDS.
template <int DT, bool SCORES, int SWEEPS>
__device__ __forceinline__ void drain_tiles(const FuseArgs& a, const TileWs& ws, const ObjTable& tab, unsigned turn, int* job,
                                            int wave, int n_waves, int lane) {
  static_assert(kLists == 32, "lanes 0 .. 31 look at one list each");
  const int rot = (int)(turn % kLists);
  while (true) {
    if (wave == 0) {
      const unsigned pushed = __hip_atomic_load(ws.status + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int want = min(kParts, max(n_waves, pushed >= kManyPushed ? 4 : 0));
      int parts = 0, tile = 0, obj = 0, first = 0;
      while (true) {
        unsigned top = 0u;
        if (lane < kLists) top = __hip_atomic_load(ws.status + kListWord + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t full = (uint32_t)__ballot(top != 0u);
        if (full == 0u) break;   // every list is empty
        const uint32_t rotated = rot ? (full >> rot) | (full << (kLists - rot)) : full;
        const int list = (rot + __builtin_ctz(rotated)) % kLists;   // the first list at or after `rot` that holds something
        tile = __builtin_amdgcn_readlane((int)top, list) - 1;
        int* words = ws.hdr[tile].cnt;
        int below = 0;
        if (lane == 0) {
          first = __hip_atomic_fetch_add(&words[2], want, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          below = __hip_atomic_load(&words[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          obj = __hip_atomic_load(&words[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        first = __builtin_amdgcn_readfirstlane(first);
        parts = min(want, kParts - first);
        if (parts > 0) break;
        if (lane == 0) {
          unsigned entry = (unsigned)tile + 1u;
          __hip_atomic_compare_exchange_strong(ws.status + kListWord + list, &entry, (unsigned)below, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);   // (another one was faster: as good)
        }
        parts = 0;
      }
      if (lane == 0) {
        job[0] = parts;
        job[1] = tile;
        job[2] = first;
        job[3] = obj;
      }
    }
    __syncthreads();
    const int parts = __builtin_amdgcn_readfirstlane(job[0]), tile = __builtin_amdgcn_readfirstlane(job[1]);
    const int first = __builtin_amdgcn_readfirstlane(job[2]), obj = __builtin_amdgcn_readfirstlane(job[3]);
    __syncthreads();   // everybody has read the job before the next one is written
    if (parts == 0) return;
    const ObjRange ob = tab.o[obj];
    const int li0 = (tile - ob.tile_begin) * kTilePts + first * kPartPts;
    for (int li = li0 + wave; li < min(li0 + parts * kPartPts, ob.n_pts); li += n_waves) gather_point<DT, SCORES, SWEEPS>(a, ob, li, lane);
  }
}

}  // namespace aura
