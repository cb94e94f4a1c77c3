// aura_voxel_downsample: Sec. 3.2.1 "Adaptive Sampling".
//
// The voxel size follows the object, s_voxel = cbrt(V_bound / N_target); the object's boundary box is cut into cubes
// of that side and every occupied cube is replaced by the mean position of its points.  The grid of an object is
// small (a few hundred to a few thousand cubes for N_target ~ 150), so it is held densely:
//   k_vox_zero    clears the cubes' sums and counts
//   k_vox_bin     cube index of every point (fp32 decision chain), coordinates as 64-bit fixed point, added up per cube
//                 in a workgroup's LDS table and from there in memory (integer sums: the result does not depend on the
//                 order in which they land)
//   k_vox_count   occupied cubes per block of 2048 cubes
//   k_vox_emit    per block: the occupied cubes of the blocks before it, from there the position of every occupied cube in
//                 the output list, mean position, count; object offsets
//   k_vox_point   per point: the list position of its cube
// Every object's cubes start at a multiple of 2048, so blocks never straddle objects.  All traffic is a few bytes per
// point plus the grid: the call is bound by launch latency.
#include "aura_device.hpp"
#include "launch.hpp"

namespace aura {

constexpr int kVoxBlock = 256;
constexpr int kVoxCellsPerThread = 8;
constexpr int kVoxCellsPerBlock = kVoxBlock * kVoxCellsPerThread;   // 2048

struct VoxCell {
  long long sum[3];   // fixed-point coordinate sums
  long long cnt;
};

struct VoxObjDev {
  long long pt_begin;
  int n_pts;
  float lo[3];
  float s;
  int dims[3];
  int cell_begin;     // first cube of the object in the concatenated grid (a multiple of 2048)
};

struct VoxTable {
  VoxObjDev o[kMaxObjPerLaunch];
};

struct VoxArgs {
  const float* xyz;
  VoxCell* cells;      // [total cells]
  int* cell_slot;      // [total cells]: list position of an occupied cube
  int* block_cnt;      // [blocks]: occupied cubes
  int n_blocks;
  int shift;           // fixed-point scale 2^shift
  float* out_xyz;      // [capacity][3]
  int* out_count;      // [capacity] or nullptr
  long long capacity;
  int* out_offsets;    // [B + 1]
  int* voxel_of_point; // [N] or nullptr
  int n_obj;
};

__device__ __forceinline__ int vox_axis(float x, float lo, float s, int n) {
#pragma clang fp contract(off)
  const float t = x - lo;
  const float fl = floorf(t / s);
  return (fl >= (float)(n - 1)) ? n - 1 : ((fl > 0.0f) ? (int)fl : 0);
}

__device__ __forceinline__ int vox_cell(const VoxObjDev& ob, const float* __restrict__ p) {
  const int ix = vox_axis(p[0], ob.lo[0], ob.s, ob.dims[0]);
  const int iy = vox_axis(p[1], ob.lo[1], ob.s, ob.dims[1]);
  const int iz = vox_axis(p[2], ob.lo[2], ob.s, ob.dims[2]);
  return ob.cell_begin + (iz * ob.dims[1] + iy) * ob.dims[0] + ix;
}

__global__ __launch_bounds__(kVoxBlock) void k_vox_zero(VoxArgs a) {
  typedef uint32_t vox_u32x4 __attribute__((ext_vector_type(4)));
  vox_u32x4* __restrict__ z = reinterpret_cast<vox_u32x4*>(a.cells);
  const long long n = (long long)a.n_blocks * kVoxCellsPerBlock * (long long)(sizeof(VoxCell) / 16);
  for (long long i = (long long)blockIdx.x * kVoxBlock + threadIdx.x; i < n; i += (long long)gridDim.x * kVoxBlock)
    z[i] = vox_u32x4{0u, 0u, 0u, 0u};
}

// Eight or four consecutive points.  The loads are 16 bytes wide at any 4-byte address, which global loads allow.
template <int N>
struct __attribute__((packed, aligned(4))) VoxRun {
  float v[3 * N];
};
struct __attribute__((packed, aligned(4))) VoxIds {
  int v[4];
};

// Points per thread and trip, and entries of a workgroup's table.
constexpr int kVoxPts = 8;
constexpr int kVoxTrip = kVoxBlock * kVoxPts;   // 2048 points per workgroup and trip
constexpr int kVoxSlots = 1024;                  // 32 KiB of LDS: four workgroups per compute unit

// A workgroup adds `trips` * 2048 consecutive points of one object up in an LDS table before anything goes to memory.
// Bound by the atomics: the cubes are few (a few hundred per object), so every atomic in memory meets others at its
// address.  One set of them per run of equal cubes in a wave, found with a 64-lane scan, took 240 us for 64 objects of
// 100 000 points; with the table a workgroup issues one set per cube that its points touch (the whole call 253 -> 72 us).
// A thread takes 8 consecutive points, which in a spatially sorted cloud mostly share a cube, and goes to the table when
// the cube changes.  An entry belongs to the first cube that claims it (index modulo 1024: objects of up to 1024 cubes
// never collide); a cube that finds its entry taken adds to memory directly, so any number of cubes and any order of the
// points is served.  Integer sums: the result does not depend on the order in which they land.  The next trip's run, where there
// is one, is requested before this one is added up (6.4 M points, three trips: whole call 64.0 -> 62.6 us, the kernel 33 us for
// 77 MB; requested in the last trip too, 1 M points took 24.4 us instead of 22.9, 4 M 47.3 instead of 45.5).  Not the bound: the divisions
// and the conversions to fixed point (a product with 1 / s and a guard, shifts) and lanes that meet at one entry (sums of up to
// 16 lanes joined first) - with all three changed the kernel took 37 us.
__global__ __launch_bounds__(kVoxBlock) void k_vox_bin(VoxArgs a, VoxTable tab, int trips) {
  __shared__ unsigned long long s_sum[3][kVoxSlots];
  __shared__ unsigned s_cnt[kVoxSlots];
  __shared__ int s_key[kVoxSlots];                // cube within the object, -1: free
  const VoxObjDev ob = tab.o[blockIdx.y];
  const long long first = (long long)blockIdx.x * trips * kVoxTrip;
  if (first >= ob.n_pts) return;                  // uniform: whole workgroups leave
  for (int t = threadIdx.x; t < kVoxSlots; t += kVoxBlock) {
    s_sum[0][t] = s_sum[1][t] = s_sum[2][t] = 0ull;
    s_cnt[t] = 0u;
    s_key[t] = -1;
  }
  __syncthreads();
  VoxCell* __restrict__ cells = a.cells + ob.cell_begin;
  auto add = [&](int cube, const long long (&q)[3], int n) {
    const int slot = cube & (kVoxSlots - 1);
    int key = s_key[slot];
    if (key < 0) key = atomicCAS(&s_key[slot], -1, cube);
    if (key < 0 || key == cube) {
#pragma unroll
      for (int c = 0; c < 3; ++c) atomicAdd(&s_sum[c][slot], (unsigned long long)q[c]);
      atomicAdd(&s_cnt[slot], (unsigned)n);
    } else {
#pragma unroll
      for (int c = 0; c < 3; ++c) atomicAdd(reinterpret_cast<unsigned long long*>(&cells[cube].sum[c]), (unsigned long long)q[c]);
      atomicAdd(reinterpret_cast<unsigned long long*>(&cells[cube].cnt), (unsigned long long)n);
    }
  };
  auto fixed = [&](float x) { return __double2ll_rn(ldexp((double)x, a.shift)); };
  if (ob.n_pts < kVoxPts) {   // (uniform) a point per thread
    if ((int)threadIdx.x < ob.n_pts) {
      const float* __restrict__ p = a.xyz + 3 * (ob.pt_begin + threadIdx.x);
      const long long q[3] = {fixed(p[0]), fixed(p[1]), fixed(p[2])};
      add(vox_cell(ob, p) - ob.cell_begin, q, 1);
    }
    trips = 0;
  }
  // A thread's run of a trip, as six loads of 16 bytes at any 4-byte address.  The object's last run begins early enough to
  // end with the object (the points before the thread's own are left out), and threads and trips beyond it read it again.
  auto load = [&](int trip) {
    const long long l = min(first + (long long)trip * kVoxTrip + threadIdx.x * kVoxPts, (long long)ob.n_pts - kVoxPts);
    return *reinterpret_cast<const VoxRun<kVoxPts>*>(a.xyz + 3 * (ob.pt_begin + l));
  };
  VoxRun<kVoxPts> r, r_next;
  if (trips > 0) r_next = load(0);
  for (int trip = 0; trip < trips; ++trip) {
    const long long l0 = first + (long long)trip * kVoxTrip + threadIdx.x * kVoxPts;
    if (l0 >= ob.n_pts) break;
    r = r_next;
    if (trip + 1 < trips) r_next = load(trip + 1);   // (uniform) on its way while this trip is added up
    __builtin_amdgcn_sched_barrier(0);
    const long long l = min(l0, (long long)ob.n_pts - kVoxPts);
    long long q[3] = {0, 0, 0};
    int cube = -1, run = 0;
#pragma unroll
    for (int e = 0; e < kVoxPts; ++e) {
      if (l + e < l0) continue;
      const float x[3] = {r.v[3 * e], r.v[3 * e + 1], r.v[3 * e + 2]};
      const int now = vox_cell(ob, x) - ob.cell_begin;
      if (now != cube) {
        if (run > 0) add(cube, q, run);
        cube = now;
        run = 0;
        q[0] = q[1] = q[2] = 0;
      }
      ++run;
#pragma unroll
      for (int c = 0; c < 3; ++c) q[c] += fixed(x[c]);
    }
    add(cube, q, run);
  }
  __syncthreads();
  for (int t = threadIdx.x; t < kVoxSlots; t += kVoxBlock) {
    if (s_key[t] < 0) continue;
    VoxCell* cc = cells + s_key[t];
#pragma unroll
    for (int c = 0; c < 3; ++c) atomicAdd(reinterpret_cast<unsigned long long*>(&cc->sum[c]), s_sum[c][t]);
    atomicAdd(reinterpret_cast<unsigned long long*>(&cc->cnt), (unsigned long long)s_cnt[t]);
  }
}

// Number of occupied cubes among the thread's 8, and the workgroup's exclusive prefix of it.
__device__ __forceinline__ int vox_block_prefix(int mine, int* sh, int* total) {
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  int inc = mine;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int up = __shfl_up(inc, o, kWave);
    if (lane >= o) inc += up;
  }
  if (lane == kWave - 1) sh[wave] = inc;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kVoxBlock / kWave; ++w) {
    if (w < wave) before += sh[w];
    all += sh[w];
  }
  *total = all;
  return before + inc - mine;
}

__global__ __launch_bounds__(kVoxBlock) void k_vox_count(VoxArgs a) {
  __shared__ int sh[kVoxBlock / kWave];
  const long long c0 = (long long)blockIdx.x * kVoxCellsPerBlock + threadIdx.x * kVoxCellsPerThread;
  int mine = 0;
#pragma unroll
  for (int e = 0; e < kVoxCellsPerThread; ++e) mine += a.cells[c0 + e].cnt > 0 ? 1 : 0;
  int total;
  vox_block_prefix(mine, sh, &total);
  if (threadIdx.x == 0) a.block_cnt[blockIdx.x] = total;
}

// Every workgroup adds the counts of the blocks before its own up itself (one block per object of up to 2048 cubes, at most
// 8192), and the first one of an object, and the last one of all, write the object offsets; a scan of the counts by one workgroup
// was one more launch, and a serial one for many blocks (200 000 points on 3000 cubes 20.8 us with the scan, 19.8 so; 1 M points
// on 7 M cubes, 3500 blocks, 174 and 161; 64 objects on 100 000 cubes each 206 and 192).  (Counting a cube when the first points are added to it saves another launch, but
// the atomics then have to answer: 64 objects of 100 000 points 72 -> 108 us.)
__global__ __launch_bounds__(kVoxBlock) void k_vox_emit(VoxArgs a, VoxTable tab) {
  __shared__ int sh[kVoxBlock / kWave];
  int before = 0;
  for (int j = threadIdx.x; j < (int)blockIdx.x; j += kVoxBlock) before += a.block_cnt[j];
  int block_off;
  vox_block_prefix(before, sh, &block_off);   // (its total)
  const int first_cell = blockIdx.x * kVoxCellsPerBlock;
  for (int b = threadIdx.x; b < a.n_obj; b += kVoxBlock)
    if (tab.o[b].cell_begin == first_cell) a.out_offsets[b] = block_off;
  if (blockIdx.x + 1 == gridDim.x && threadIdx.x == 0) a.out_offsets[a.n_obj] = block_off + a.block_cnt[blockIdx.x];
  __syncthreads();   // sh is free again
  const long long c0 = (long long)blockIdx.x * kVoxCellsPerBlock + threadIdx.x * kVoxCellsPerThread;
  long long cnt[kVoxCellsPerThread];
  int mine = 0;
#pragma unroll
  for (int e = 0; e < kVoxCellsPerThread; ++e) {
    cnt[e] = a.cells[c0 + e].cnt;
    mine += cnt[e] > 0 ? 1 : 0;
  }
  int total;
  long long slot = block_off + vox_block_prefix(mine, sh, &total);
#pragma unroll
  for (int e = 0; e < kVoxCellsPerThread; ++e) {
    if (cnt[e] <= 0) {
      a.cell_slot[c0 + e] = -1;
      continue;
    }
    a.cell_slot[c0 + e] = (int)slot;
    if (slot < a.capacity) {
      const VoxCell cc = a.cells[c0 + e];
#pragma unroll
      for (int c = 0; c < 3; ++c) a.out_xyz[3 * slot + c] = (float)(ldexp((double)cc.sum[c], -a.shift) / (double)cc.cnt);
      if (a.out_count) a.out_count[slot] = (int)cc.cnt;
    }
    ++slot;
  }
}

// Four points per thread: loads and stores of 16 bytes.
__global__ __launch_bounds__(kVoxBlock) void k_vox_point(VoxArgs a, VoxTable tab) {
  const VoxObjDev ob = tab.o[blockIdx.y];
  const long long li = 4 * ((long long)blockIdx.x * kVoxBlock + threadIdx.x);
  if (li >= ob.n_pts) return;
  const float* __restrict__ p = a.xyz + 3 * (ob.pt_begin + li);
  int* __restrict__ out = a.voxel_of_point + ob.pt_begin + li;
  if (li + 4 <= ob.n_pts) {
    const VoxRun<4> r = *reinterpret_cast<const VoxRun<4>*>(p);
    VoxIds ids;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x[3] = {r.v[3 * e], r.v[3 * e + 1], r.v[3 * e + 2]};
      ids.v[e] = a.cell_slot[vox_cell(ob, x)];
    }
    *reinterpret_cast<VoxIds*>(out) = ids;
  } else {
    for (int e = 0; li + e < ob.n_pts; ++e) out[e] = a.cell_slot[vox_cell(ob, p + 3 * e)];
  }
}

// ---------------------------------------------------------------- host side

static size_t vox_align256(size_t x) { return (x + 255) & ~(size_t)255; }

// s_voxel and the cubes per axis of one box; false when the box is not a box or the grid is out of range.
bool voxel_grid(const float* lo, const float* hi, int n_target, float* s_out, int* dims) {
  float e[3], emax = 0.0f;
  for (int a = 0; a < 3; ++a) {
    e[a] = hi[a] - lo[a];
    if (!(e[a] >= 0.0f) || e[a] > 3.0e38f) return false;
    emax = e[a] > emax ? e[a] : emax;
  }
  float s = (float)cbrt((double)e[0] * (double)e[1] * (double)e[2] / (double)n_target);
  if (!(s > 0.0f)) s = (float)((double)emax / cbrt((double)n_target));   // flat box: the longest side stands in
  if (!(s > 0.0f)) s = 1.0f;                                             // a single point
  *s_out = s;
  for (int a = 0; a < 3; ++a) {
    const float q = floorf(e[a] / s);
    if (!(q < (float)kVoxelMaxCells)) return false;
    dims[a] = (int)q + 1;
  }
  return (long long)dims[0] * dims[1] * dims[2] <= kVoxelMaxCells;
}

static long long vox_padded(long long cells) { return (cells + kVoxCellsPerBlock - 1) / kVoxCellsPerBlock * kVoxCellsPerBlock; }

long long voxel_padded_cells(long long cells) { return vox_padded(cells); }

size_t voxel_workspace_bytes(long long padded_cells) {
  const size_t blocks = (size_t)(padded_cells / kVoxCellsPerBlock);
  return vox_align256((size_t)padded_cells * sizeof(VoxCell)) + vox_align256((size_t)padded_cells * sizeof(int)) +
         vox_align256(blocks * sizeof(int)) +
         vox_align256((blocks + 1) * sizeof(int));   // (the last part is not used: the size that the call asks for is kept)
}

hipError_t launch_voxel_downsample(const float* xyz, const VoxObj* objs, int B, float max_abs, long long n_points,
                                   float* out_xyz, int* out_count, long long capacity, int* out_offsets,
                                   int* voxel_of_point, void* workspace, hipStream_t stream) {
  VoxTable tab{};
  long long cells = 0;
  int max_pts = 0;
  for (int b = 0; b < B; ++b) {
    VoxObjDev& d = tab.o[b];
    d.pt_begin = objs[b].pt_begin; d.n_pts = objs[b].n_pts; d.s = objs[b].s;
    for (int a = 0; a < 3; ++a) { d.lo[a] = objs[b].lo[a]; d.dims[a] = objs[b].dims[a]; }
    d.cell_begin = (int)cells;
    cells += vox_padded((long long)d.dims[0] * d.dims[1] * d.dims[2]);
    max_pts = d.n_pts > max_pts ? d.n_pts : max_pts;
  }
  VoxArgs a{};
  a.xyz = xyz;
  a.n_blocks = (int)(cells / kVoxCellsPerBlock);
  char* ws = static_cast<char*>(workspace);
  size_t off = 0;
  a.cells = reinterpret_cast<VoxCell*>(ws + off);   off += vox_align256((size_t)cells * sizeof(VoxCell));
  a.cell_slot = reinterpret_cast<int*>(ws + off);   off += vox_align256((size_t)cells * sizeof(int));
  a.block_cnt = reinterpret_cast<int*>(ws + off);
  // fixed point: |x| 2^shift n_points < 2^62 for every coordinate up to max_abs
  int e = 0, nbits = 1;
  frexpf(max_abs, &e);
  if (!(max_abs > 0.0f)) e = 0;
  while (nbits < 40 && (1ll << nbits) <= n_points) ++nbits;
  a.shift = 62 - e - nbits;
  a.out_xyz = out_xyz; a.out_count = out_count; a.capacity = capacity; a.out_offsets = out_offsets;
  a.voxel_of_point = voxel_of_point; a.n_obj = B;

  const dim3 block(kVoxBlock);
  const int zero_groups = a.n_blocks * 4 < 2048 ? a.n_blocks * 4 : 2048;
  hipLaunchKernelGGL(k_vox_zero, dim3(zero_groups), block, 0, stream, a);
  if (max_pts > 0) {
    // longer workgroups issue fewer atomics per point, as long as about a thousand of them (four per compute unit) remain
    const long long want = n_points / (1024ll * kVoxTrip);
    const int trips = (int)(want < 1 ? 1 : (want > 8 ? 8 : want));
    const long long span = (long long)trips * kVoxTrip;
    hipLaunchKernelGGL(k_vox_bin, dim3((unsigned)((max_pts + span - 1) / span), B), block, 0, stream, a, tab, trips);
  }
  hipLaunchKernelGGL(k_vox_count, dim3(a.n_blocks), block, 0, stream, a);
  hipLaunchKernelGGL(k_vox_emit, dim3(a.n_blocks), block, 0, stream, a, tab);
  if (voxel_of_point && max_pts > 0)
    hipLaunchKernelGGL(k_vox_point, dim3((max_pts - 1) / (4 * kVoxBlock) + 1, B), block, 0, stream, a, tab);
  return hipGetLastError();
}

}  // namespace aura
