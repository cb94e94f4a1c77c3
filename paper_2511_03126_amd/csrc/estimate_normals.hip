// aura_estimate_normals: the normals of the sampled points, which the view importance score needs (Sec. 3.2.2, first
// step of the view filtering).
//
// For every sampled point q: the k points of the object's cloud nearest to q, the plane through them (eigenvector of
// the smallest eigenvalue of their covariance), turned to point away from the object's centre.
//
// One workgroup per query.  Which points are nearest is decided on the fp32 distance d = (dx dx + dy dy) + dz dz
// (every operation rounded, no contraction), of equal distances the lower index first.
//
// Usual path (k up to 256), one sweep over the cloud:
//   1. an upper bound of the k-th smallest distance that is exact by construction: the k-th smallest distance among
//      every stride-th quad of points, or point (at most 16384 points, kept in LDS; the k-th smallest of a subset can only be larger);
//   2. one sweep over the whole cloud collects the points within that bound (about k * stride of them) in LDS
//      (a cloud that fits the list goes there whole, without a bound);
//   3. among those, the k-th smallest distance by a radix select over the bit pattern of d (non-negative floats order
//      like their bits: histograms of the next 11 / 11 / 10 bits among the candidates left) and, when more points share
//      that distance than are still needed, the same select over their indices;
//   4. the selected points in index order: r and r r^T (r = p - q, exact in fp64) summed in that order by one
//      thread, then the covariance and a cyclic Jacobi iteration on the 3 x 3 matrix.
// General path (larger k, or more candidates than the LDS list holds, e.g. thousands of points at one distance): the
// radix select over the whole cloud (three sweeps), then one sweep for the sums.
// The queries of a call run side by side; the cloud comes from L2 (a few MB) or the last-level cache.
#include "aura_device.hpp"
#include "launch.hpp"
#include "normals_subset.hpp"

namespace aura {

constexpr int kNrmBlock = 1024;   // a sweep over the cloud is shared by 16 waves
constexpr int kNrmBins = 2048;
// The strided subset that bounds the k-th distance (normals_subset.hpp) lies far apart in memory: a read of a wave touches a
// cache line per lane, 16384 single points three times that.  Quads of neighbouring points (48 bytes, three 16-byte loads) take
// a quarter of the lines and a sixteenth of the loads; the sweep reads quads too (with the matrices of the last step in
// registers, 150 queries of 30 neighbours against 200 000 points 56 -> 46.6 us, against 1 M points 174 -> 154, against 8000, all
// of them candidates, 26 -> 20).
static_assert(kNrmSub <= 2 * kNrmCand, "the subset lies where the candidates go later");
constexpr int kNrmSel = 256;      // largest k of the one-sweep path

struct NrmObjDev {
  long long pt_begin;
  int n_pts;
  int q_begin;
  int n_q;
  float centre[3];
};

struct NrmTable {
  NrmObjDev o[kMaxObjPerLaunch];
};

struct NrmArgs {
  const float* xyz;
  const float* queries;
  int k;
  float* normals;   // [M][3]
  float* evals;     // [M][3] or nullptr: eigenvalues of the covariance, ascending
};

__device__ __forceinline__ uint32_t dist_bits(const float* __restrict__ p, float qx, float qy, float qz) {
#pragma clang fp contract(off)
  const float dx = p[0] - qx, dy = p[1] - qy, dz = p[2] - qz;
  float t = dx * dx + dy * dy;
  t = t + dz * dz;
  return __float_as_uint(t);
}

// Four consecutive points.  The loads are 16 bytes wide at any 4-byte address, which global loads allow.
struct __attribute__((packed, aligned(4))) PointQuad {
  float v[12];
};

__device__ __forceinline__ void quad_dist(const PointQuad& q, float qx, float qy, float qz, uint32_t (&d)[4]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float p[3] = {q.v[3 * e], q.v[3 * e + 1], q.v[3 * e + 2]};
    d[e] = dist_bits(p, qx, qy, qz);
  }
}

// Among the elements i of [0, n) with eligible(i), the `want` smallest by key(i) (want >= 1, at most the number of
// eligible elements): those below the key returned and *need of the *n_equal that have it.  All threads of the workgroup call it
// and get the same answer.
// EARLY: it ends with the pass that finds a bin which belongs to the `want` smallest as a whole, with the bin's largest key (*need =
// *n_equal; no key is larger and still in the bin).  Mostly that is the second of three, the bins of 22 bits of a distance are 1e-4
// wide.  A pass over a list in LDS is five barriers: 150 queries, three passes / ending early, us: 200 000 points and k = 30 41.9 /
// 39.3, k = 200 61.0 / 58.3, 1 M points 144.9 / 140.6, 50 000 26.7 / 24.5, 2000 13.8 / 12.5.  Not over the whole cloud, where it
// measured 180 / 214 (200 000 points, k = 300) and 974 / 884 (1 M, k = 1000) with the same loads and waits in the passes; why is not known.
template <bool EARLY, typename Key, typename Eligible>
__device__ uint32_t radix_select(int n, int want, Key key, Eligible eligible, uint32_t* s_hist, int* s_pick, int* n_equal,
                                 int* need) {
  uint32_t prefix = 0, mask = 0;
  int remaining = want;
  const int shifts[3] = {21, 10, 0}, widths[3] = {11, 11, 10};
  for (int pass = 0; pass < 3; ++pass) {
    const int shift = shifts[pass], nb = 1 << widths[pass];
    for (int b = threadIdx.x; b < kNrmBins; b += kNrmBlock) s_hist[b] = 0;
    __syncthreads();
    // four points per thread and trip, so that their reads are in flight together
    // (unsigned: past the end of the largest cloud, 2^31 - 1 points, the index has to stay above n)
    for (uint32_t i0 = threadIdx.x; i0 < (uint32_t)n; i0 += 4 * kNrmBlock) {
      uint32_t kv[4];
      bool cand[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t i = i0 + e * kNrmBlock;
        cand[e] = i < (uint32_t)n && eligible((int)i);
        kv[e] = cand[e] ? key((int)i) : 0u;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (cand[e] && (kv[e] & mask) == prefix) atomicAdd(&s_hist[(kv[e] >> shift) & (uint32_t)(nb - 1)], 1u);
    }
    __syncthreads();
    // the bin that holds the remaining-th candidate: thread t sums its kPer consecutive bins, a scan over the threads
    // finds the thread, which then walks its bins
    constexpr int kPer = kNrmBins / kNrmBlock;
    uint32_t mine = 0;
#pragma unroll
    for (int e = 0; e < kPer; ++e) mine += s_hist[threadIdx.x * kPer + e];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    uint32_t inc = mine;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t up = __shfl_up(inc, o, kWave);
      if (lane >= o) inc += up;
    }
    __shared__ uint32_t s_wave[kNrmBlock / kWave];
    if (lane == kWave - 1) s_wave[wave] = inc;
    __syncthreads();
    uint32_t before = inc - mine;
    for (int w = 0; w < wave; ++w) before += s_wave[w];
    if ((uint32_t)remaining > before && (uint32_t)remaining <= before + mine) {   // exactly one thread
      uint32_t run = before;
#pragma unroll
      for (int e = 0; e < kPer; ++e) {
        const uint32_t c = s_hist[threadIdx.x * kPer + e];
        if ((uint32_t)remaining > run && (uint32_t)remaining <= run + c) {
          s_pick[0] = threadIdx.x * kPer + e;
          s_pick[1] = (int)run;
          s_pick[2] = (int)c;
        }
        run += c;
      }
    }
    __syncthreads();
    prefix |= (uint32_t)s_pick[0] << shift;
    mask |= (uint32_t)(nb - 1) << shift;
    remaining -= s_pick[1];
    *n_equal = s_pick[2];
    __syncthreads();   // s_pick and s_hist are free again
    if (EARLY && remaining == *n_equal) {   // uniform
      prefix |= ~mask;
      break;
    }
  }
  *need = remaining;
  return prefix;
}

__device__ __forceinline__ double nrm_block_sum(double v, double* sh) {
  v = wave_sum(v);
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  __syncthreads();
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < kNrmBlock / kWave; ++w) t += sh[w];
  return t;
}

// One Jacobi rotation in the plane (p, q): app, aqq, apq the matrix there, arp and arq the third row's entries, vp and vq the
// columns of the eigenvectors.  The rotation's tangent t = sign(theta) / (|theta| + sqrt(theta^2 + 1)), theta = d / b, is taken
// without the division for theta.  (Entries are products of fp32 differences: their squares neither overflow nor vanish in
// fp64.)
__device__ __forceinline__ void rotate(double& app, double& aqq, double& apq, double& arp, double& arq, double (&vp)[3], double (&vq)[3]) {
  if (apq == 0.0) return;
  const double d = aqq - app, b = 2.0 * apq;
  const double t = (d < 0.0 ? -b : b) / (fabs(d) + sqrt(d * d + b * b));
  const double cs = 1.0 / sqrt(t * t + 1.0), sn = t * cs;
  app -= t * apq;
  aqq += t * apq;
  apq = 0.0;
  const double rp = arp, rq = arq;
  arp = cs * rp - sn * rq;
  arq = sn * rp + cs * rq;
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    const double p = vp[r], q = vq[r];
    vp[r] = cs * p - sn * q;
    vq[r] = sn * p + cs * q;
  }
}

// Eigenvalues (ascending in w) and the eigenvector of the smallest one of the symmetric matrix
// [a00 a01 a02; a01 a11 a12; a02 a12 a22], by cyclic Jacobi rotations.  One thread's chain: everything has a register of its
// own (as arrays indexed by loops the matrices were in scratch memory, a round trip per entry).
__device__ __forceinline__ void smallest_eigenvector(const double (&c)[6], double (&w)[3], double (&n)[3]) {
  double a00 = c[0], a01 = c[1], a02 = c[2], a11 = c[3], a12 = c[4], a22 = c[5];
  double v0[3] = {1, 0, 0}, v1[3] = {0, 1, 0}, v2[3] = {0, 0, 1};
#pragma unroll 1
  for (int sweep = 0; sweep < 24; ++sweep) {
    const double off = fabs(a01) + fabs(a02) + fabs(a12);
    const double diag = fabs(a00) + fabs(a11) + fabs(a22);
    if (off <= 1e-300 || off <= 1e-17 * diag) break;
    rotate(a00, a11, a01, a02, a12, v0, v1);
    rotate(a00, a22, a02, a01, a12, v0, v2);
    rotate(a11, a22, a12, a01, a02, v1, v2);
  }
  auto ascending = [](double& x, double& y, double (&vx)[3], double (&vy)[3]) {
    if (x > y) {
      const double t = x;
      x = y;
      y = t;
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const double u = vx[r];
        vx[r] = vy[r];
        vy[r] = u;
      }
    }
  };
  ascending(a00, a11, v0, v1);
  ascending(a11, a22, v1, v2);
  ascending(a00, a11, v0, v1);
  w[0] = a00; w[1] = a11; w[2] = a22;
  const double len = sqrt(v0[0] * v0[0] + v0[1] * v0[1] + v0[2] * v0[2]);
#pragma unroll
  for (int r = 0; r < 3; ++r) n[r] = v0[r] / len;
}

// From the sums of r and r r^T over the kk selected points to the stored normal (one thread).
__device__ __forceinline__ void finish_normal(const NrmArgs& a, const NrmObjDev& ob, long long m, float qx, float qy, float qz, int kk,
                              const double (&s1)[3], const double (&s2)[6]) {
  const double inv = 1.0 / (double)kk;
  const double mx = s1[0] * inv, my = s1[1] * inv, mz = s1[2] * inv;
  const double cov[6] = {s2[0] * inv - mx * mx, s2[1] * inv - mx * my, s2[2] * inv - mx * mz,
                         s2[3] * inv - my * my, s2[4] * inv - my * mz, s2[5] * inv - mz * mz};
  double w[3], nv[3];
  smallest_eigenvector(cov, w, nv);
  const double ox = (double)qx - (double)ob.centre[0], oy = (double)qy - (double)ob.centre[1], oz = (double)qz - (double)ob.centre[2];
  const double sgn = nv[0] * ox + nv[1] * oy + nv[2] * oz < 0.0 ? -1.0 : 1.0;
  for (int c = 0; c < 3; ++c) {
    a.normals[3 * m + c] = (float)(sgn * nv[c]);
    if (a.evals) a.evals[3 * m + c] = (float)w[c];
  }
}

__global__ __launch_bounds__(kNrmBlock) void k_estimate_normals(NrmArgs a, NrmTable tab) {
  __shared__ uint32_t s_hist[kNrmBins];
  __shared__ int s_pick[3];
  __shared__ double s_red[kNrmBlock / kWave];
  const NrmObjDev ob = tab.o[blockIdx.y];
  if ((int)blockIdx.x >= ob.n_q) return;
  const long long m = ob.q_begin + blockIdx.x;
  const float qx = a.queries[3 * m], qy = a.queries[3 * m + 1], qz = a.queries[3 * m + 2];
  const float* __restrict__ pts = a.xyz + 3 * ob.pt_begin;
  const int n = ob.n_pts;
  const int kk = a.k < n ? a.k : n;
  if (kk == 0) {   // an object without points
    if (threadIdx.x < 3) {
      a.normals[3 * m + threadIdx.x] = 0.0f;
      if (a.evals) a.evals[3 * m + threadIdx.x] = 0.0f;
    }
    return;
  }
  auto dist = [&](int i) { return dist_bits(pts + 3 * (long long)i, qx, qy, qz); };
  int n_equal, need;
  double s1[3] = {0, 0, 0}, s2[6] = {0, 0, 0, 0, 0, 0};   // sums of r and r r^T (in the first thread)
  bool summed = false;
  if (kk <= kNrmSel) {
    __shared__ __attribute__((aligned(16))) uint32_t s_list[2 * kNrmCand];                  // the subset's distances, later the candidates:
    uint32_t* const s_cd = s_list;                             // distance bits ...
    int* const s_ci = reinterpret_cast<int*>(s_list + kNrmCand);   // ... and point index
    __shared__ int s_cn, s_ns;
    __shared__ int s_sel[kNrmSel];        // the k selected points, unordered, then in index order
    __shared__ float s_pt[kNrmSel][3];
    auto quad = [&](int first) { return *reinterpret_cast<const PointQuad*>(pts + 3 * (long long)first); };
    constexpr int kTrip = 4;   // quads per thread and trip: reads in flight together
    if (n <= kNrmCand) {       // (uniform)
      for (int i = threadIdx.x; i < n; i += kNrmBlock) {
        s_cd[i] = dist(i);
        s_ci[i] = i;
      }
      if (threadIdx.x == 0) { s_cn = n; s_ns = 0; }
    } else {
      const NrmSubset sub = nrm_subset(n, kk);   // uniform
      if (sub.run == 4) {
        for (int j0 = threadIdx.x; j0 < sub.count; j0 += kTrip * kNrmBlock) {
          PointQuad q[kTrip];
#pragma unroll
          for (int e = 0; e < kTrip; ++e) q[e] = quad(4 * sub.stride * min(j0 + e * kNrmBlock, sub.count - 1));
#pragma unroll
          for (int e = 0; e < kTrip; ++e) {
            uint32_t d[4];
            quad_dist(q[e], qx, qy, qz, d);
            if (j0 + e * kNrmBlock < sub.count) *reinterpret_cast<uint4*>(s_list + 4 * (j0 + e * kNrmBlock)) = uint4{d[0], d[1], d[2], d[3]};
          }
        }
      } else {
        for (int j0 = threadIdx.x; j0 < sub.count; j0 += 8 * kNrmBlock) {
          uint32_t d[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) d[e] = dist(min(j0 + e * kNrmBlock, sub.count - 1) * sub.stride);
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (j0 + e * kNrmBlock < sub.count) s_list[j0 + e * kNrmBlock] = d[e];
        }
      }
      __syncthreads();
      const uint32_t bound = radix_select<true>(sub.run * sub.count, kk, [&](int j) { return s_list[j]; }, [](int) { return true; },
                                          s_hist, s_pick, &n_equal, &need);
      if (threadIdx.x == 0) { s_cn = 0; s_ns = 0; }
      __syncthreads();
      const int n_quads = nrm_quads(n);
      for (int g0 = threadIdx.x; g0 < n_quads; g0 += kTrip * kNrmBlock) {
        PointQuad q[kTrip];
        NrmQuad at[kTrip];
#pragma unroll
        for (int e = 0; e < kTrip; ++e) {
          at[e] = nrm_quad(g0 + e * kNrmBlock, n);
          q[e] = quad(at[e].first);
        }
#pragma unroll
        for (int e = 0; e < kTrip; ++e) {
          uint32_t d[4];
          quad_dist(q[e], qx, qy, qz, d);
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            if (d[c] <= bound && c >= at[e].skip) {
              const int pos = atomicAdd(&s_cn, 1);
              if (pos < kNrmCand) { s_cd[pos] = d[c]; s_ci[pos] = at[e].first + c; }
            }
          }
        }
      }
    }
    __syncthreads();
    const int cn = s_cn;
    if (cn <= kNrmCand) {   // uniform; otherwise the general path below
      const uint32_t tau = radix_select<true>(cn, kk, [&](int j) { return s_cd[j]; }, [](int) { return true; }, s_hist, s_pick,
                                        &n_equal, &need);
      int last_idx = 0x7fffffff;   // points at distance tau are taken up to this index
      if (need < n_equal) {
        int e2, n2;
        last_idx = (int)radix_select<true>(cn, need, [&](int j) { return (uint32_t)s_ci[j]; }, [&](int j) { return s_cd[j] == tau; },
                                     s_hist, s_pick, &e2, &n2);
      }
      for (int j = threadIdx.x; j < cn; j += kNrmBlock)
        if (s_cd[j] < tau || (s_cd[j] == tau && s_ci[j] <= last_idx)) s_sel[atomicAdd(&s_ns, 1)] = s_ci[j];   // exactly kk
      __syncthreads();
      // index order: the rank of a selected point is the number of selected points before it
      int mine = -1, rank = 0;
      if ((int)threadIdx.x < kk) {
        mine = s_sel[threadIdx.x];
        for (int j = 0; j < kk; ++j) rank += s_sel[j] < mine ? 1 : 0;
      }
      __syncthreads();
      if (mine >= 0) {
        const float* __restrict__ pm = pts + 3 * (long long)mine;
        s_pt[rank][0] = pm[0]; s_pt[rank][1] = pm[1]; s_pt[rank][2] = pm[2];
      }
      __syncthreads();
      if (threadIdx.x == 0) {
#pragma unroll 4
        for (int j = 0; j < kk; ++j) {   // (several points' reads in flight; the sums keep their order)
          const double rx = (double)s_pt[j][0] - (double)qx, ry = (double)s_pt[j][1] - (double)qy, rz = (double)s_pt[j][2] - (double)qz;
          s1[0] += rx; s1[1] += ry; s1[2] += rz;
          s2[0] += rx * rx; s2[1] += rx * ry; s2[2] += rx * rz;
          s2[3] += ry * ry; s2[4] += ry * rz; s2[5] += rz * rz;
        }
      }
      summed = true;
    }
  }
  if (!summed) {   // uniform
    const uint32_t tau = radix_select<false>(n, kk, dist, [](int) { return true; }, s_hist, s_pick, &n_equal, &need);
    int last_idx = 0x7fffffff;   // points at distance tau are taken up to this index
    if (need < n_equal) {
      int e2, n2;
      last_idx = (int)radix_select<false>(n, need, [](int i) { return (uint32_t)i; }, [&](int i) { return dist(i) == tau; }, s_hist,
                                   s_pick, &e2, &n2);
    }
    for (uint32_t i0 = threadIdx.x; i0 < (uint32_t)n; i0 += 4 * kNrmBlock) {   // (unsigned as in radix_select)
      float px[4], py[4], pz[4];
      bool in[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t i = min(i0 + e * kNrmBlock, (uint32_t)n - 1u);
        const float* __restrict__ p = pts + 3 * (long long)i;
        px[e] = p[0]; py[e] = p[1]; pz[e] = p[2];
        in[e] = i0 + e * kNrmBlock < (uint32_t)n;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = (int)(i0 + e * kNrmBlock);
        const float pe[3] = {px[e], py[e], pz[e]};
        const uint32_t d = dist_bits(pe, qx, qy, qz);
        if (in[e] && (d < tau || (d == tau && i <= last_idx))) {
          const double rx = (double)px[e] - (double)qx, ry = (double)py[e] - (double)qy, rz = (double)pz[e] - (double)qz;
          s1[0] += rx; s1[1] += ry; s1[2] += rz;
          s2[0] += rx * rx; s2[1] += rx * ry; s2[2] += rx * rz;
          s2[3] += ry * ry; s2[4] += ry * rz; s2[5] += rz * rz;
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) s1[c] = nrm_block_sum(s1[c], s_red);
#pragma unroll
    for (int c = 0; c < 6; ++c) s2[c] = nrm_block_sum(s2[c], s_red);
  }
  if (threadIdx.x == 0) finish_normal(a, ob, m, qx, qy, qz, kk, s1, s2);
}

hipError_t launch_estimate_normals(const float* xyz, const float* queries, const NrmObj* objs, int n_obj, int k,
                                   float* normals, float* evals, hipStream_t stream) {
  NrmTable tab{};
  int max_q = 0;
  for (int b = 0; b < n_obj; ++b) {
    NrmObjDev& d = tab.o[b];
    d.pt_begin = objs[b].pt_begin; d.n_pts = objs[b].n_pts; d.q_begin = objs[b].q_begin; d.n_q = objs[b].n_q;
    for (int c = 0; c < 3; ++c) d.centre[c] = objs[b].centre[c];
    max_q = d.n_q > max_q ? d.n_q : max_q;
  }
  if (max_q == 0) return hipSuccess;
  NrmArgs a{xyz, queries, k, normals, evals};
  hipLaunchKernelGGL(k_estimate_normals, dim3(max_q, n_obj), dim3(kNrmBlock), 0, stream, a, tab);
  return hipGetLastError();
}

}  // namespace aura
