// aura_select_views: Sec. 3.2.2, view importance-based filtering.
//
// For every visible (point, view) pair (Eq. 1, the shared fp32 decision functions):
//     S_dist = 1 / (1 + z),   S_angle = max(0, v . (-n)),   S_total = S_dist * S_angle,
// z the depth of the point in the camera frame, v the unit vector from the camera centre to the point, n the
// point's unit normal.  The k visible views with the largest S_total are kept, of equal scores the lower view
// index first.
//
// k_select_views: one thread per point, looping over the views of the point's object (camera rows by wave-uniform scalar
// reads, one depth texel per pair), the k best so far in registers.  k_select_views_wave, for sampled sets: one wave per
// point, a lane per view, the place of a view among the others counted.  The ray is taken in the camera frame, where it is
// Xc = R x + t itself: v . n = Xc . (R n) / |Xc|.  Traffic: 24 B per point in, 8 k + mask_pitch + 4 B out.
#include "aura_device.hpp"
#include "launch.hpp"

namespace aura {

struct SelArgs {
  VisArgs vis;
  const float* xyz;
  const float* normals;
  int k;
  int* sel_view;       // [N][k]
  float* sel_score;    // [N][k] or nullptr
  uint8_t* sel_mask;   // [N][mask_pitch] or nullptr
  int mask_pitch;
  int* n_sel;          // [N] or nullptr
};

// S_total of a visible pair: p the projection of the point (x, y, z) by the camera row c, (nx, ny, nz) its normal.  Every sum is
// written out as the multiply-adds it is (left to the compiler, the two kernels took different ones, and a point's scores
// depended on how many points the call had).
__device__ __forceinline__ float view_score(const float* __restrict__ c, const Proj& p, float x, float y, float z, float nx, float ny,
                                            float nz) {
  const float xc = __builtin_fmaf(c[2], z, __builtin_fmaf(c[1], y, __builtin_fmaf(c[0], x, c[9])));
  const float yc = __builtin_fmaf(c[5], z, __builtin_fmaf(c[4], y, __builtin_fmaf(c[3], x, c[10])));
  const float zc = p.z;
  const float rnx = __builtin_fmaf(c[2], nz, __builtin_fmaf(c[1], ny, c[0] * nx));   // the normal in the camera frame
  const float rny = __builtin_fmaf(c[5], nz, __builtin_fmaf(c[4], ny, c[3] * nx));
  const float rnz = __builtin_fmaf(c[8], nz, __builtin_fmaf(c[6], nx, c[7] * ny));
  const float len = sqrtf(__builtin_fmaf(zc, zc, __builtin_fmaf(xc, xc, yc * yc)));
  const float facing = __builtin_fmaf(zc, rnz, __builtin_fmaf(rnx, xc, rny * yc));
  const float s_angle = fmaxf(0.0f, -facing / len);
  return s_angle / (1.0f + zc);
}

// One wave per point, lane = view of the object (at most 64).  All of a point's projections and depth reads are in flight
// together; a visible view's place is the number of visible views that come before it (larger score, of equal scores the
// lower view), so there is no list and no order to keep.  A thread per point is a chain of projections, depth reads and
// insertions in one or two workgroups: 16 000 points and less, 16 views 17.0 -> 9.5 us, 64 views 61 -> 16.3, 4 views 9.4 and
// 9.7; 150 points, GPU time alone, 16 views 11.2 -> 3.0 us, 64 views 45.8 -> 3.2.
__global__ __launch_bounds__(256) void k_select_views_wave(SelArgs a, ObjTable tab) {
  const ObjRange ob = tab.o[blockIdx.y];
  const int lane = threadIdx.x % kWave;
  const int li = __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave);
  if (li >= ob.n_pts) return;
  const long long i = ob.pt_begin + li;
  const float x = a.xyz[3 * i], y = a.xyz[3 * i + 1], z = a.xyz[3 * i + 2];
  const float nx = a.normals[3 * i], ny = a.normals[3 * i + 1], nz = a.normals[3 * i + 2];
  bool seen = false;
  float s = 0.0f;
  if (lane < ob.n_views) {
    const int v = ob.view_begin + lane;
    const float* __restrict__ c = a.vis.cam + (long long)v * 16;
    const Proj p = project(c, x, y, z);
    seen = visible(a.vis, a.vis.depth ? a.vis.depth + (long long)v * a.vis.H * a.vis.W : nullptr, p);
    if (seen) s = view_score(c, p, x, y, z, nx, ny, nz);
  }
  const unsigned long long visible_views = __ballot(seen);
  const bool ranked = seen && s > -1.0f;   // -1: the score of a place that nobody has taken
  const unsigned long long all = __ballot(ranked);
  int place = 0;
  for (unsigned long long m = all; m; m &= m - 1) {
    const int j = __builtin_ctzll(m);
    const float other = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s), j));
    place += other > s || (other == s && j < lane) ? 1 : 0;
  }
  if (ranked && place < a.k) {
    a.sel_view[i * a.k + place] = lane;
    if (a.sel_score) a.sel_score[i * a.k + place] = s;
  }
  if (lane >= __popcll(all) && lane < a.k) {   // places that nobody took
    a.sel_view[i * a.k + lane] = -1;
    if (a.sel_score) a.sel_score[i * a.k + lane] = 0.0f;
  }
  if (a.n_sel && lane == 0) a.n_sel[i] = min(__popcll(visible_views), a.k);
  if (a.sel_mask) {
    const bool kept = ranked && place < a.k;
    for (int j = lane; j < a.mask_pitch; j += kWave) a.sel_mask[i * a.mask_pitch + j] = j == lane && kept ? 1 : 0;
  }
}

// Views whose depth texels are requested together: a thread's chain of projection -> depth read per view is what it waits for.
constexpr int kSelectAhead = 8;

// Points up to which a wave takes each: beyond, a lane per view leaves most lanes of few views idle (thread / wave, us: 32 000
// points of 4 views 8.7 / 10.0, of 16 views 17.1 / 12.6; 64 000 of 4 views 8.7 / 17.3, of 16 views 17.2 / 20.4).
constexpr long long kSelectWavePoints = 16384;

__global__ __launch_bounds__(256) void k_select_views(SelArgs a, ObjTable tab) {
  const ObjRange ob = tab.o[blockIdx.y];
  const int li = blockIdx.x * blockDim.x + threadIdx.x;
  if (li >= ob.n_pts) return;
  const long long i = ob.pt_begin + li;
  const float x = a.xyz[3 * i], y = a.xyz[3 * i + 1], z = a.xyz[3 * i + 2];
  const float nx = a.normals[3 * i], ny = a.normals[3 * i + 1], nz = a.normals[3 * i + 2];
  float best_s[kSelectMaxK];
  int best_v[kSelectMaxK];
#pragma unroll
  for (int t = 0; t < kSelectMaxK; ++t) {
    best_s[t] = -1.0f;   // below every score of a visible view
    best_v[t] = -1;
  }
  int seen = 0;
  for (int j0 = 0; j0 < ob.n_views; j0 += kSelectAhead) {
    Proj ps[kSelectAhead];
    bool frs[kSelectAhead];
    float deps[kSelectAhead];
#pragma unroll
    for (int e = 0; e < kSelectAhead; ++e) {
      const int v = ob.view_begin + min(j0 + e, ob.n_views - 1);   // (past the end: the last view again, unused)
      ps[e] = project(a.vis.cam + (long long)v * 16, x, y, z);
      frs[e] = in_frustum(a.vis, ps[e]);
      deps[e] = 1.0f;
      if (a.vis.depth) deps[e] = a.vis.depth[(long long)v * a.vis.H * a.vis.W + (frs[e] ? depth_texel(a.vis, ps[e]) : 0)];
    }
#pragma unroll
    for (int e = 0; e < kSelectAhead; ++e) {
      const int j = j0 + e;
      if (j >= ob.n_views) break;   // uniform
      const float* __restrict__ c = a.vis.cam + (long long)(ob.view_begin + j) * 16;
      const Proj p = ps[e];
      if (!(frs[e] && (a.vis.frustum_only || passes_depth(a.vis, p, deps[e])))) continue;
      ++seen;
      float s = view_score(c, p, x, y, z, nx, ny, nz);
      int sv = j;
      // insert into the sorted list: a later view only moves ahead of an entry with a strictly smaller score; from
      // there on every entry moves down one place
      bool moving = false;
#pragma unroll
      for (int t = 0; t < kSelectMaxK; ++t) {
        moving = moving || s > best_s[t];
        if (t < a.k && moving) {
          const float ts = best_s[t];
          const int tv = best_v[t];
          best_s[t] = s;
          best_v[t] = sv;
          s = ts;
          sv = tv;
        }
      }
    }
  }
#pragma unroll
  for (int t = 0; t < kSelectMaxK; ++t) {
    if (t < a.k) {
      a.sel_view[i * a.k + t] = best_v[t];
      if (a.sel_score) a.sel_score[i * a.k + t] = best_v[t] >= 0 ? best_s[t] : 0.0f;
    }
  }
  if (a.n_sel) a.n_sel[i] = seen < a.k ? seen : a.k;
  if (a.sel_mask) {
    uint8_t* __restrict__ row = a.sel_mask + i * a.mask_pitch;
    for (int j = 0; j < a.mask_pitch; ++j) {
      bool kept = false;
#pragma unroll
      for (int t = 0; t < kSelectMaxK; ++t) kept = kept || (t < a.k && best_v[t] == j);
      row[j] = kept ? 1 : 0;
    }
  }
}

hipError_t launch_select_views(const VisArgs& vis, const float* xyz, const float* normals, int k, int* sel_view,
                               float* sel_score, uint8_t* sel_mask, int mask_pitch, int* n_sel, const ObjTable& tab,
                               int n_obj, int max_pts, hipStream_t stream) {
  if (n_obj == 0 || max_pts == 0) return hipSuccess;
  SelArgs a{vis, xyz, normals, k, sel_view, sel_score, sel_mask, mask_pitch, n_sel};
  int max_views = 0;
  for (int b = 0; b < n_obj; ++b) max_views = tab.o[b].n_views > max_views ? tab.o[b].n_views : max_views;
  if (max_views <= kWave && (long long)max_pts * n_obj <= kSelectWavePoints) {
    hipLaunchKernelGGL(k_select_views_wave, dim3((max_pts + 3) / 4, n_obj), dim3(256), 0, stream, a, tab);
    return hipGetLastError();
  }
  const dim3 grid((max_pts + 255) / 256, n_obj), block(256);
  hipLaunchKernelGGL(k_select_views, grid, block, 0, stream, a, tab);
  return hipGetLastError();
}

}  // namespace aura
