// aura_fuse_features: Sec. 3.1 "Feature Aggregation", Eq. 2, with the L2 normalisation that the
// cosine similarity of Sec. 3.4.1 implies.
//
// Gather kernel: one wave per point, lanes across the D channels.
//   phase 1  lanes across the views of the point's object: each lane projects the point into one
//            view, evaluates Eq. 1 and prepares the two cell indices and blend weights per axis;
//            a ballot collects the visible views.
//   phase 2  for every visible view (wave-uniform loop over the ballot bits) the four cell rows are
//            read as contiguous D-vectors, widened to fp32 and blended into per-lane accumulators.
//   finish   mean over the visible views, one wave-level sum of squares, scale, streaming store.
// HBM traffic is the compulsory output row (4 D bytes per point) plus each feature cell once;
// the repeated cell reads are served by the caches, which is why points should arrive spatially
// sorted and why workgroup ids are mapped so that each XCD walks a contiguous range of points.
#include <algorithm>
#include <type_traits>

#include "aura_device.hpp"
#include "fuse_args.hpp"
#include "launch.hpp"
#include "timing.hpp"

namespace aura {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

constexpr int kFuseWaves = 4;
constexpr int kFusePtsPerWave = 8;   // at most: see launch_one

__device__ __forceinline__ void widen_pair(uint32_t w, int dtype_is_bf16, float& lo, float& hi) {
  if (dtype_is_bf16) {
    lo = __uint_as_float(w << 16);
    hi = __uint_as_float(w & 0xffff0000u);
  } else {
    f16x2 h = __builtin_bit_cast(f16x2, w);
    lo = (float)h[0];
    hi = (float)h[1];
  }
}

// Reads VEC consecutive elements `off` bytes behind `base` (wave-uniform; an unsigned 32-bit offset per lane keeps the
// 64-bit part of the address on the scalar unit) and widens them to fp32.
// DT: 0 fp32, 1 bf16, 2 fp16.  The address is VEC * sizeof(element) aligned by construction.
template <int DT, int VEC>
__device__ __forceinline__ void load_widen(const char* __restrict__ base, uint32_t off, float (&out)[VEC]) {
  if constexpr (DT == 0) {
    const float* p = reinterpret_cast<const float*>(base + off);
    if constexpr (VEC == 4) {
      f32x4 v = *reinterpret_cast<const f32x4*>(p);
      out[0] = v[0]; out[1] = v[1]; out[2] = v[2]; out[3] = v[3];
    } else if constexpr (VEC == 2) {
      f32x2 v = *reinterpret_cast<const f32x2*>(p);
      out[0] = v[0]; out[1] = v[1];
    } else {
      static_assert(VEC == 1, "fp32 rows are read 1, 2 or 4 elements at a time");
      out[0] = *p;
    }
  } else {
    const uint16_t* p = reinterpret_cast<const uint16_t*>(base + off);
    if constexpr (VEC == 8) {
      u32x4 v = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
      for (int j = 0; j < 4; ++j) widen_pair(v[j], DT == 1, out[2 * j], out[2 * j + 1]);
    } else if constexpr (VEC == 4) {
      u32x2 v = *reinterpret_cast<const u32x2*>(p);
      widen_pair(v[0], DT == 1, out[0], out[1]);
      widen_pair(v[1], DT == 1, out[2], out[3]);
    } else if constexpr (VEC == 2) {
      widen_pair(*reinterpret_cast<const uint32_t*>(p), DT == 1, out[0], out[1]);
    } else {
      static_assert(VEC == 1, "16-bit rows are read 1, 2, 4 or 8 elements at a time");
      float hi;
      widen_pair((uint32_t)*p, DT == 1, out[0], hi);
    }
  }
}

template <int VEC>
__device__ __forceinline__ void store_stream(float* __restrict__ p, const float (&v)[VEC]) {
  if constexpr (VEC % 4 == 0) {
#pragma unroll
    for (int j = 0; j < VEC; j += 4) {
      f32x4 q = {v[j], v[j + 1], v[j + 2], v[j + 3]};
      __builtin_nontemporal_store(q, reinterpret_cast<f32x4*>(p + j));
    }
  } else if constexpr (VEC == 2) {
    f32x2 q = {v[0], v[1]};
    __builtin_nontemporal_store(q, reinterpret_cast<f32x2*>(p));
  } else {
#pragma unroll
    for (int j = 0; j < VEC; ++j) p[j] = v[j];
  }
}

// The bilinear blend of one visible view: weights of the four cells and the start of their rows.
struct ViewTaps {
  const char* row[4];
  float w[4];
};

// DT element type, VEC elements per lane per load, PASSES loads per cell row.
// EXACT:   D == 64 * VEC * PASSES, the whole row lives in registers.
// MASKED:  D below that and a multiple of VEC: lanes beyond D repeat the row's last VEC channels and drop out of the sums
//          and the stores.
// GENERIC: any D; channels are processed 64 * VEC * PASSES at a time (outer loop), the unnormalised mean is stored first
//          and rescaled in a second sweep.
enum class RowWidth { EXACT, MASKED, GENERIC };

// A wave takes pts_per_wave consecutive points, one after the other.  What bounds a call of a few thousand points is that
// chain (point -> projections -> depth texels -> cell rows -> norm): with 8 points per wave and one channel per lane and
// load, 2001 points of 5 views and 384 channels took 97 us on 63 workgroups; one point per wave, 16-byte loads and the
// rows of two views in flight together bring the call's other stages and it from 122 to 43 us.
// PAIRS: two views at a time.  For calls that fill the chip many times over it is one: the second view's rows cost registers
// and with them waves (317 202 points, 6 views of 512 fp32 channels: 434 us staged with pairs, 415 without).
template <int DT, int VEC, int PASSES, RowWidth WIDTH, bool PAIRS>
__global__ __launch_bounds__(kFuseWaves* kWave) void k_fuse_gather(FuseArgs a, int pts_per_wave, ObjTable tab) {
  if (a.clear_status && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 4) a.clear_status[threadIdx.x] = 0u;
  const ObjRange ob = tab.o[blockIdx.y];
  const int pts_per_block = kFuseWaves * pts_per_wave;
  const int nblk = (ob.n_pts + pts_per_block - 1) / pts_per_block;
  if ((int)blockIdx.x >= nblk) return;
  const int blk = xcd_contiguous(blockIdx.x, nblk);
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  constexpr int CH = kWave * VEC * PASSES;
  constexpr bool GENERIC = WIDTH == RowWidth::GENERIC, EXACT = WIDTH == RowWidth::EXACT;
  static_assert(!GENERIC || (VEC == 1 && PASSES == 1), "one channel per lane and sweep");
  const int D = EXACT ? CH : a.feat.D, Hf = a.feat.Hf, Wf = a.feat.Wf;
  const long long view_elems = (long long)Hf * Wf * D;
  constexpr long long elt = DT == 0 ? 4 : 2;
  uint32_t off[PASSES];   // byte offset of the lane's channels within a row
#pragma unroll
  for (int p = 0; p < PASSES; ++p)
    off[p] = (uint32_t)(GENERIC ? lane : (EXACT ? p * kWave * VEC + lane * VEC : min(p * kWave * VEC + lane * VEC, D - VEC))) * (uint32_t)elt;

  for (int k = 0; k < pts_per_wave; ++k) {
    const int li = blk * pts_per_block + wave * pts_per_wave + k;
    if (li >= ob.n_pts) break;
    const long long i = ob.pt_begin + li;
    const float x = a.xyz[3 * i], y = a.xyz[3 * i + 1], z = a.xyz[3 * i + 2];
    float* __restrict__ out_row = a.fused + i * D;
    float ss = 0.0f;
    int cnt = 0;

    for (int cb = 0; cb < (GENERIC ? D : CH); cb += CH) {
      float acc[PASSES][VEC];
#pragma unroll
      for (int p = 0; p < PASSES; ++p)
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[p][e] = 0.0f;
      cnt = 0;

      for (int vb = 0; vb < ob.n_views; vb += kWave) {
        // phase 1: lane j handles view vb + j
        bool seen = false;
        int x0 = 0, y0 = 0;
        float ax = 0.0f, ay = 0.0f;
        if (vb + lane < ob.n_views) {
          const int v = ob.view_begin + vb + lane;
          const Proj p = project(a.vis.cam + (long long)v * 16, x, y, z);
          const float* dv = a.vis.depth ? a.vis.depth + (long long)v * a.vis.H * a.vis.W : nullptr;
          seen = visible(a.vis, dv, p) && view_kept(a, i, vb + lane);
          if (seen) {
            const Tap tx = tap_axis(p.u, a.feat.pitch_x, Wf), ty = tap_axis(p.v, a.feat.pitch_y, Hf);
            x0 = tx.i0; ax = tx.a;
            y0 = ty.i0; ay = ty.a;
          }
        }
        if (a.out_vis && vb + lane < a.vis_pitch && cb == 0) a.out_vis[i * a.vis_pitch + vb + lane] = seen ? 1 : 0;
        unsigned long long m = __ballot(seen);
        cnt += __popcll(m);
        // phase 2: wave-uniform loop over the visible views, with PAIRS two at a time so that the rows of both are in flight
        auto taps_of = [&](int src) {
          const int sx0 = __builtin_amdgcn_readlane(x0, src), sy0 = __builtin_amdgcn_readlane(y0, src);
          const float sax = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ax), src));
          const float say = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ay), src));
          const int sx1 = sx0 + 1 < Wf ? sx0 + 1 : Wf - 1, sy1 = sy0 + 1 < Hf ? sy0 + 1 : Hf - 1;
          const char* vbase = static_cast<const char*>(a.feat.feat) +
                              (long long)(ob.view_begin + vb + src) * view_elems * elt;
          // (32 x 32 bit products: a 64-bit one would leave the scalar unit, and the row addresses with it)
          auto row_of = [&](int y, int x) { return vbase + (long long)(y * Wf + x) * D * (DT == 0 ? 4 : 2); };
          ViewTaps t;
          t.w[0] = (1.0f - sax) * (1.0f - say); t.w[1] = sax * (1.0f - say);
          t.w[2] = (1.0f - sax) * say;          t.w[3] = sax * say;
          t.row[0] = row_of(sy0, sx0); t.row[1] = row_of(sy0, sx1);
          t.row[2] = row_of(sy1, sx0); t.row[3] = row_of(sy1, sx1);
          return t;
        };
        auto blend = [&](auto n_views_c) {
          constexpr int NV = decltype(n_views_c)::value;
          ViewTaps t[NV];
#pragma unroll
          for (int q = 0; q < NV; ++q) {
            t[q] = taps_of(__builtin_ctzll(m));
            m &= m - 1;
          }
#pragma unroll
          for (int p = 0; p < PASSES; ++p) {
            if (GENERIC && cb + lane >= D) continue;
            uint32_t o = EXACT ? off[0] : off[p] + (GENERIC ? (uint32_t)cb * (uint32_t)elt : 0u);
            asm("" : "+v"(o));   // stays a 32-bit offset to a scalar base (widened outside the loop it becomes 64-bit vector adds)
            float v[NV][4][VEC];
#pragma unroll
            for (int q = 0; q < NV; ++q)
#pragma unroll
              for (int c = 0; c < 4; ++c) load_widen<DT, VEC>(t[q].row[c] + (EXACT ? p * kWave * VEC * (int)elt : 0), o, v[q][c]);
#pragma unroll
            for (int q = 0; q < NV; ++q)
#pragma unroll
              for (int e = 0; e < VEC; ++e) {
                float s = acc[p][e];
#pragma unroll
                for (int c = 0; c < 4; ++c) s = __builtin_fmaf(t[q].w[c], v[q][c][e], s);
                acc[p][e] = s;
              }
          }
        };
        if constexpr (PAIRS) {
          while (m & (m - 1)) blend(std::integral_constant<int, 2>{});
        }
        while (m) blend(std::integral_constant<int, 1>{});
      }

      // mean over the visible views (Eq. 2); a point nobody sees keeps zeros
      const float inv = cnt > 0 ? 1.0f / (float)cnt : 0.0f;
#pragma unroll
      for (int p = 0; p < PASSES; ++p) {
        const bool mine = GENERIC || EXACT || p * kWave * VEC + lane * VEC < D;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          acc[p][e] = mine ? acc[p][e] * inv : 0.0f;
          ss = __builtin_fmaf(acc[p][e], acc[p][e], ss);
        }
      }
      if constexpr (!GENERIC) {
        float scale = 1.0f;
        if (!a.mean_only && cnt > 0) {   // uniform
          const float nrm = sqrtf(wave_sum(ss));
          scale = 1.0f / fmaxf(nrm, a.norm_eps);
        }
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
#pragma unroll
          for (int e = 0; e < VEC; ++e) acc[p][e] *= scale;
          const int ch = p * kWave * VEC + lane * VEC;
          if (EXACT || ch < D) store_stream<VEC>(out_row + ch, acc[p]);
        }
      } else {
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
          const int ch = cb + p * kWave * VEC + lane * VEC;
          if (ch < D) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) out_row[ch + e] = acc[p][e];
          }
        }
      }
    }

    if constexpr (GENERIC) {
      if (!a.mean_only && cnt > 0) {
        const float nrm = sqrtf(wave_sum(ss));
        const float scale = 1.0f / fmaxf(nrm, a.norm_eps);
        // every lane rescales exactly the channels it stored above (VEC == 1, PASSES == 1)
        for (int ch = lane; ch < D; ch += kWave) out_row[ch] *= scale;
      }
    }
    for (int j = (ob.n_views + kWave - 1) / kWave * kWave + lane; a.out_vis && j < a.vis_pitch; j += kWave)
      a.out_vis[i * a.vis_pitch + j] = 0;   // mask columns beyond the views' last 64
    if (a.out_count && lane == 0) a.out_count[i] = cnt;
  }
}

template <int DT, int VEC, int PASSES, RowWidth WIDTH>
static hipError_t launch_width(const FuseArgs& a, const ObjTable& tab, int n_obj, int max_pts, hipStream_t stream) {
  // points per wave: one until the launch has 32 waves per compute unit, up to eight beyond
  long long pts = 0;
  for (int t = 0; t < n_obj; ++t) pts += tab.o[t].n_pts;
  const int pts_per_wave = (int)std::min<long long>(kFusePtsPerWave, std::max<long long>(1, pts / 8192));
  const int pts_per_block = kFuseWaves * pts_per_wave;
  dim3 grid((unsigned)(((long long)max_pts + pts_per_block - 1) / pts_per_block), n_obj), block(kFuseWaves * kWave);
  const TimedLaunch timed(stream);
  if (pts_per_wave < kFusePtsPerWave)
    hipLaunchKernelGGL((k_fuse_gather<DT, VEC, PASSES, WIDTH, true>), grid, block, 0, stream, a, pts_per_wave, tab);
  else
    hipLaunchKernelGGL((k_fuse_gather<DT, VEC, PASSES, WIDTH, false>), grid, block, 0, stream, a, pts_per_wave, tab);
  return hipGetLastError();
}

template <int DT, int VEC, int PASSES>
static hipError_t launch_one(const FuseArgs& a, const ObjTable& tab, int n_obj, int max_pts, hipStream_t stream) {
  return a.feat.D == kWave * VEC * PASSES ? launch_width<DT, VEC, PASSES, RowWidth::EXACT>(a, tab, n_obj, max_pts, stream)
                                          : launch_width<DT, VEC, PASSES, RowWidth::MASKED>(a, tab, n_obj, max_pts, stream);
}

// The row in registers for every D that is a whole number of 16-byte pieces (8 bytes for 16-bit rows of up to 256
// channels, so that all lanes have work) and fits: up to 2048 16-bit or 1536 fp32 channels.
template <int DT>
static hipError_t dispatch_d(const FuseArgs& a, const ObjTable& tab, int n_obj, int max_pts, hipStream_t stream) {
  const int D = a.feat.D;
  if constexpr (DT == 0) {
    if (D % 4 == 0) {
      switch ((D + 255) / 256) {
        case 1: return launch_one<DT, 4, 1>(a, tab, n_obj, max_pts, stream);
        case 2: return launch_one<DT, 4, 2>(a, tab, n_obj, max_pts, stream);
        case 3: return launch_one<DT, 4, 3>(a, tab, n_obj, max_pts, stream);
        case 4: return launch_one<DT, 4, 4>(a, tab, n_obj, max_pts, stream);
        case 5: case 6: return launch_one<DT, 4, 6>(a, tab, n_obj, max_pts, stream);
        default: break;
      }
    }
  } else {
    if (D % 4 == 0 && D <= 256) return launch_one<DT, 4, 1>(a, tab, n_obj, max_pts, stream);
    if (D == 768) return launch_one<DT, 4, 3>(a, tab, n_obj, max_pts, stream);
    if (D % 8 == 0) {
      switch ((D + 511) / 512) {
        case 1: return launch_one<DT, 8, 1>(a, tab, n_obj, max_pts, stream);
        case 2: return launch_one<DT, 8, 2>(a, tab, n_obj, max_pts, stream);
        case 3: return launch_one<DT, 8, 3>(a, tab, n_obj, max_pts, stream);
        case 4: return launch_one<DT, 8, 4>(a, tab, n_obj, max_pts, stream);
        default: break;
      }
    }
  }
  return launch_width<DT, 1, 1, RowWidth::GENERIC>(a, tab, n_obj, max_pts, stream);
}

hipError_t launch_fuse_features(const VisArgs& vis, const FeatArgs& feat, const float* xyz, float* fused,
                                int* out_count, float norm_eps, int mean_only, const TileWs* tile_ws,
                                const ObjTable& tab, int n_obj, int max_pts, hipStream_t stream, float* out_factor,
                                uint8_t* out_vis, int vis_pitch, const uint8_t* in_mask, int in_mask_pitch, int two_kernels,
                                const TileScoring* scoring, FuseOutcome* did, unsigned* clear_status) {
  if (did) *did = FuseOutcome{};
  if (n_obj == 0 || max_pts == 0) return hipSuccess;
  FuseArgs a{vis, feat, xyz, fused, out_count, norm_eps, mean_only, tile_ws ? out_factor : nullptr,
             out_vis, vis_pitch, in_mask, in_mask_pitch, two_kernels, clear_status,
             tile_ws && scoring ? *scoring : TileScoring{}};
  if (tile_ws) return launch_fuse_tile(a, *tile_ws, tab, n_obj, max_pts, stream, did);
  switch (feat.dtype) {
    case 0: return dispatch_d<0>(a, tab, n_obj, max_pts, stream);
    case 1: return dispatch_d<1>(a, tab, n_obj, max_pts, stream);
    default: return dispatch_d<2>(a, tab, n_obj, max_pts, stream);
  }
}

}  // namespace aura
