// The sieve in front of k_tile_fused: which tiles does any view see?
//
// A tile that nobody sees (the inside of a voxelised solid: eight of ten; the far side of an object with frontal views: every
// second one) needs no k-steps and no products: its mask, counts, scores and labels are zero, its properties those of equal
// similarities.  Here a wave tests two tiles at a time, with many waves in flight, and only until the
// first hit; it begins with the view that saw its last tiles, so a tile that is seen costs little more than one projection per
// point.  The unseen tiles' results are written here, as plain runs of stores; the others go to their object's list, in groups of
// neighbours, and k_tile_fused (tile_waves.hip) works through that.
#include <type_traits>

#include "aura_device.hpp"
#include "fuse_args.hpp"
#include "scores_epilogue.hpp"

namespace aura {

typedef const float __attribute__((address_space(4))) * const_floats;

constexpr int kSiftWaves = 4;
constexpr int kSiftPairs = 4;   // pairs of tiles per wave
constexpr int kSiftTiles = 2 * kSiftWaves * kSiftPairs;   // tiles of a workgroup
constexpr int kSiftAhead = 4;   // views whose depth texels are in flight together

// Writes n zero bytes from p on, by all threads of a workgroup.
__device__ __forceinline__ void zero_bytes(void* dst, long long n) {
  const int tid = threadIdx.x;
  char* p = static_cast<char*>(dst);
  const int head = (int)min((long long)(-reinterpret_cast<uintptr_t>(p) & 15), n);
  if (tid < head) p[tid] = 0;
  p += head;
  n -= head;
  for (long long o = 16 * tid; o + 16 <= n; o += 16 * kSiftWaves * kWave) *reinterpret_cast<u32x4_t*>(p + o) = u32x4_t{0u, 0u, 0u, 0u};
  const int tail = (int)(n & 15);
  if (tid < tail) p[n - tail + tid] = 0;
}

__global__ __launch_bounds__(kSiftWaves* kWave) void k_tile_sift(FuseArgs a, TileWs ws, ObjTable tab) {
  __shared__ uint32_t s_seen[2][kSiftWaves];   // per wave: of the sample's two tiles, and of its own (bit t: tile t)
  __shared__ int s_at;
  __shared__ float s_prop[kScoreMaxP];         // properties of a point that nobody sees
  const ObjRange ob = tab.o[blockIdx.y];
  const int nblk = (ob.n_pts + kTilePts - 1) / kTilePts;
  const int group0 = blockIdx.x * kSiftTiles;
  if (group0 >= nblk) return;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), lane = threadIdx.x % kWave;
  unsigned* __restrict__ seen_word = ws.counters + 8 * (ws.obj_base + (int)blockIdx.y) + kSeenWord;
  const TileScoring& sc = a.scoring;

  auto point = [&](int tile) {   // of the pair that begins with `tile` (beyond the object: its last one)
    const long long li = min((long long)tile * kTilePts + lane, (long long)ob.n_pts - 1);
    const float* x = a.xyz + 3 * (ob.pt_begin + li);
    return float3{x[0], x[1], x[2]};
  };
  // The order of the views: four interleaved runs, so that every four of them look from all around.
  const int quarter = (ob.n_views + 3) >> 2;
  auto view_at = [&](int c) { return min((c & 3) * quarter + (c >> 2), ob.n_views - 1); };
  // Which of the two tiles of a pair are among `need` and seen by one of the kViews views v(0), v(1), ...; hint: the last that did.
  auto look = [&](const float3& pt, bool valid, uint32_t need, int& hint, auto views, auto v) -> uint32_t {
    constexpr int kViews = decltype(views)::value;
    Proj pj[kViews];
    bool fr[kViews];
    float dep[kViews];
#pragma unroll
    for (int e = 0; e < kViews; ++e) {
      const long long view = ob.view_begin + v(e);
      pj[e] = project((const_floats)(uintptr_t)(a.vis.cam + view * 16), pt.x, pt.y, pt.z);
      fr[e] = in_frustum(a.vis, pj[e]);
      dep[e] = 1.0f;
      if (a.vis.depth) dep[e] = a.vis.depth[view * a.vis.H * a.vis.W + (fr[e] ? depth_texel(a.vis, pj[e]) : 0)];
    }
    uint32_t hits = 0;
#pragma unroll
    for (int e = 0; e < kViews; ++e) {
      const unsigned long long m = __ballot(valid && fr[e] && (a.vis.frustum_only || passes_depth(a.vis, pj[e], dep[e])));
      const uint32_t now = (((uint32_t)m != 0u ? 1u : 0u) | ((uint32_t)(m >> 32) != 0u ? 2u : 0u)) & need;
      if ((now & ~hits) != 0u) hint = v(e);
      hits |= now;
    }
    return hits;
  };
  constexpr std::integral_constant<int, kSiftAhead> several{};

  // ---- A sample first, the same in every workgroup of the object: a pair of tiles per wave, up to eight views.  Where all are seen
  // so are nearly all of the object's, and the list is not worth making: k_tile_fused takes every tile, as without the sieve.
  {
    const int pairs = (nblk + 1) >> 1, tile = 2 * (int)((2 * wave + 1) * (long long)pairs / (2 * kSiftWaves));
    const uint32_t all = tile + 1 < nblk ? 3u : 1u;
    const float3 pt = point(tile);
    const bool valid = tile * kTilePts + lane < ob.n_pts;
    uint32_t hits = 0;
    int hint = 0;
    for (int c = 0; c < min(ob.n_views, 2 * kSiftAhead) && hits != all; c += kSiftAhead)
      hits |= look(pt, valid, all & ~hits, hint, several, [&](int e) { return view_at(c + e); });
    if (lane == 0) s_seen[0][wave] = hits == all ? 1u : 0u;
  }
  __syncthreads();
  uint32_t sampled = 1u;
#pragma unroll
  for (int w = 0; w < kSiftWaves; ++w) sampled &= s_seen[0][w];
  if (__builtin_amdgcn_readfirstlane((int)sampled) != 0) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *seen_word = kAllSeen;
    return;
  }

  // ---- which tiles are seen
  const int first = group0 + 2 * kSiftPairs * wave;   // the wave's first tile
  uint32_t mine = 0;
  int hint = 0;
  float3 pt = point(first);
  for (int q = 0; q < kSiftPairs; ++q) {
    const int tile = first + 2 * q;
    if (tile >= nblk) break;   // uniform
    const float3 next = point(min(tile + 2, nblk - 1));
    const bool valid = tile * kTilePts + lane < ob.n_pts;
    const uint32_t all = tile + 1 < nblk ? 3u : 1u;
    uint32_t hits = 0;
    if (q > 0 && ob.n_views > 0) {   // the view that saw the tiles before
      const int before = hint;
      hits = look(pt, valid, all, hint, std::integral_constant<int, 1>{}, [&](int) { return before; });
    }
    for (int c = 0; c < 4 * quarter && hits != all; c += kSiftAhead)
      hits |= look(pt, valid, all & ~hits, hint, several, [&](int e) { return view_at(c + e); });
    mine |= hits << (2 * q);
    pt = next;
  }
  if (lane == 0) s_seen[1][wave] = mine;
  __syncthreads();
  static_assert(kSiftTiles == 32, "a tile of the workgroup is a bit of a word");
  uint32_t seen = 0;
#pragma unroll
  for (int w = 0; w < kSiftWaves; ++w) seen |= s_seen[1][w] << (2 * kSiftPairs * w);
  seen = (uint32_t)__builtin_amdgcn_readfirstlane((int)seen);
  const int n_here = min(kSiftTiles, nblk - group0);
  uint32_t others = ~seen & (n_here < 32 ? (1u << n_here) - 1u : ~0u);

  // ---- the seen ones on the list
  if (threadIdx.x == 0 && seen != 0u) s_at = (int)atomicAdd(seen_word, (unsigned)__popc(seen));
  if (wave == 1 && others != 0u && sc.prop) {
    unseen_properties(sc.K, sc.P, sc.y, sc.unseen_zero != 0, lane, s_prop);
  }
  __syncthreads();
  if (threadIdx.x < kSiftTiles && ((seen >> threadIdx.x) & 1u))
    ws.hdr[ob.tile_begin + s_at + __popc(seen & ((1u << threadIdx.x) - 1u))].listed = group0 + threadIdx.x;

  // ---- what is known about the others, a run of neighbours at a time: all waves write one stretch of memory
  while (others != 0u) {   // uniform
    const int t = __builtin_ctz(others);
    const uint32_t rest = ~(others >> t);   // (the zeros shifted in end a run that reaches the last bit)
    const int run = rest != 0u ? __builtin_ctz(rest) : 32;
    others = run + t < 32 ? others & (~0u << (run + t)) : 0u;
    const int tile = group0 + t;
    const int rows = min(run * kTilePts, ob.n_pts - tile * kTilePts);
    const long long i0 = ob.pt_begin + (long long)tile * kTilePts;
    zero_bytes(sc.scores + i0 * sc.K, (long long)rows * sc.K * 4);
    if (a.out_vis) zero_bytes(a.out_vis + i0 * a.vis_pitch, (long long)rows * a.vis_pitch);
    if (a.out_count) zero_bytes(a.out_count + i0, (long long)rows * 4);
    if (sc.label) zero_bytes(sc.label + i0, (long long)rows * 4);
    if (sc.prop)
      for (int o = threadIdx.x; o < rows * sc.P; o += kSiftWaves * kWave) sc.prop[i0 * sc.P + o] = s_prop[o % sc.P];
  }
}

hipError_t launch_tile_sift(const FuseArgs& a, const TileWs& ws, const ObjTable& tab, int n_obj, int max_tiles, hipStream_t stream) {
  hipLaunchKernelGGL(k_tile_sift, dim3((max_tiles + kSiftTiles - 1) / kSiftTiles, n_obj), dim3(kSiftWaves * kWave), 0, stream, a, ws, tab);
  return hipGetLastError();
}

}  // namespace aura
