// What the matrix-core fusion kernels share: the operands of a k-step, reductions over half a wave, which tiles an XCD works on.
#pragma once

#include "aura_device.hpp"
#include "fuse_args.hpp"
#include "fuse_tile_groups.hpp"

namespace aura {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kHalf = 128;                     // channels of one half wave's row piece: 32 lanes x 4 channels
constexpr int kWinSide = 32;                   // side of the per-view cell map: one 32-bit word per row

static_assert(sizeof(TileStep) == 64 + 2048, "k-step layout");

template <int DT>
__device__ __forceinline__ void split_weight(float w, uint16_t& hi, uint16_t& lo) {
  if constexpr (DT == 1) {
    __bf16 h = (__bf16)w;
    __bf16 l = (__bf16)(w - (float)h);
    hi = __builtin_bit_cast(uint16_t, h);
    lo = __builtin_bit_cast(uint16_t, l);
  } else {
    _Float16 h = (_Float16)w;
    _Float16 l = (_Float16)(w - (float)h);
    hi = __builtin_bit_cast(uint16_t, h);
    lo = __builtin_bit_cast(uint16_t, l);
  }
}

// ---- half-wave reductions on the data-parallel-primitive lanes: after the call, lane 31 holds
// the result over lanes 0..31 and lane 63 the result over lanes 32..63.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ s16x2 dpp_pull(s16x2 identity, s16x2 v) {
  return __builtin_bit_cast(s16x2, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, identity), __builtin_bit_cast(int, v),
                                                                CTRL, ROW_MASK, 0xf, false));
}

template <bool IS_MIN>
__device__ __forceinline__ s16x2 half_wave_reduce(s16x2 v) {
  const s16x2 id = IS_MIN ? s16x2{0x7fff, 0x7fff} : s16x2{-0x8000, -0x8000};
#define AURA_RED_STEP(ctrl, mask)                                                                  \
  v = IS_MIN ? __builtin_elementwise_min(v, dpp_pull<ctrl, mask>(id, v)) : __builtin_elementwise_max(v, dpp_pull<ctrl, mask>(id, v))
  AURA_RED_STEP(0x111, 0xf);   // row_shr:1
  AURA_RED_STEP(0x112, 0xf);   // row_shr:2
  AURA_RED_STEP(0x114, 0xf);   // row_shr:4
  AURA_RED_STEP(0x118, 0xf);   // row_shr:8  -> lane 15 of every row of 16 holds the row's result
  AURA_RED_STEP(0x142, 0xa);   // row_bcast:15 into rows 1 and 3
#undef AURA_RED_STEP
  return v;
}

template <int CTRL>
__device__ __forceinline__ int row_shift_add(int v) {
  return v + __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false);
}

template <int CTRL>
__device__ __forceinline__ float lane_pull(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}

// One round of the sums below: of two values, lanes with `upper` keep the second, the others the first, each with the partner's
// share.
template <int CTRL>
__device__ __forceinline__ float keep_one(float a, float b, bool upper) {
  return (upper ? b : a) + lane_pull<CTRL>(upper ? a : b);
}

// Sums over each half of the wave of 16 (H = 1) or 32 (H = 2) values per lane, all together: in every round a lane passes on half
// of what it holds and adds what it gets, so the additions halve from round to round (five lane shifts for each of the
// values by itself were 80 or 160, and as many stores by two lanes: 200 000 points of 16 views and 768 channels 239 -> 232 us, 40
// objects of 50 000 points, single pass, 588 -> 575, 64 of 100 000 1440 -> 1416, 123 457 points of 11 views 173 -> 169).  Rounds:
// lanes 16 apart, 8, 2, 1 and 4; a value's additions are the same tree for both H.  Lane l (of 32) ends up with value
// lane_value<H>(l); with 16 values two lanes hold the same one.
template <int H>
__device__ __forceinline__ float half_wave_sums(float (&v)[16 * H], int lane) {
#pragma unroll
  for (int i = 0; i < 8 * H; ++i) {   // odd rows of 16 lanes of the first value against even rows of the second
    const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[2 * i]), __float_as_uint(v[2 * i + 1]), false, false);
    v[i] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
  }
#pragma unroll
  for (int i = 0; i < 4 * H; ++i) v[i] = keep_one<0x128>(v[2 * i], v[2 * i + 1], (lane & 8) != 0);   // row_ror:8
#pragma unroll
  for (int i = 0; i < 2 * H; ++i) v[i] = keep_one<0x4e>(v[2 * i], v[2 * i + 1], (lane & 2) != 0);   // quad_perm [2, 3, 0, 1]
#pragma unroll
  for (int i = 0; i < H; ++i) v[i] = keep_one<0xb1>(v[2 * i], v[2 * i + 1], (lane & 1) != 0);       // quad_perm [1, 0, 3, 2]
  // lanes 4 apart: eight lanes mirrored, then every four
  if constexpr (H == 1) return v[0] + lane_pull<0x1b>(lane_pull<0x141>(v[0]));
  const bool upper = (lane & 4) != 0;
  const float keep = upper ? v[H - 1] : v[0], send = upper ? v[0] : v[H - 1];
  return keep + lane_pull<0x1b>(lane_pull<0x141>(send));
}

template <int H>
__device__ __forceinline__ int lane_value(int l) {
  return ((l >> 4) & 1) | ((l >> 3) & 1) << 1 | ((l >> 1) & 1) << 2 | (l & 1) << 3 | (H == 2 ? ((l >> 2) & 1) << 4 : 0);
}

// What a point's sum of feature rows is multiplied by: one over the views that see it, and over the L2 norm of that mean or its lower
// bound.  0 where no view sees the point, whatever the bound (0 / 0 otherwise, where it is 0).  squares: of the sum.
__device__ __forceinline__ float point_factor(int seen_by, float squares, float norm_eps, bool mean_only) {
  const float inv = seen_by > 0 ? 1.0f / (float)seen_by : 0.0f;
  const float normed = inv / fmaxf(sqrtf(squares) * inv, norm_eps);
  return mean_only || seen_by == 0 ? inv : normed;
}

template <int DT>
__device__ __forceinline__ f32x16 mma(u32x4 a, u32x4 b, f32x16 c) {
  if constexpr (DT == 1)
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// Operands of one k-step in registers: the two weight operands, the lane's 8 cell offsets, and
// 8 cell rows.
struct StepA {
  u32x4 hi, lo;
};

struct StepC {
  u32x4 lo, hi;   // byte offsets of the lane's cells: 8 g .. 8 g + 3 and 8 g + 4 .. 8 g + 7
};

template <int H>
struct StepQ {
  u32x2 q[H][8];   // [128-channel piece of the wave's span][cell]: 4 channels each
};

// The matrix-core instructions of one k-step: operand t = 4 h + j holds channel 128 h + 4 m + j of
// the 8 cells.
template <int DT, int H>
__device__ __forceinline__ void mma_step(const StepA& w, const StepQ<H>& r, f32x16 (&acc)[4 * H]) {
#pragma unroll
  for (int t = 0; t < 4 * H; ++t) {
    u32x4 b;
#pragma unroll
    for (int e2 = 0; e2 < 4; ++e2) {
      // bytes 0..3 of the selector index the first cell's dword, 4..7 the second cell's
      const uint32_t lo = r.q[t >> 2][2 * e2][(t >> 1) & 1], hi = r.q[t >> 2][2 * e2 + 1][(t >> 1) & 1];
      b[e2] = __builtin_amdgcn_perm(hi, lo, (t & 1) ? 0x07060302u : 0x05040100u);
    }
    acc[t] = mma<DT>(w.hi, b, acc[t]);
    acc[t] = mma<DT>(w.lo, b, acc[t]);
  }
}

// Which of an object's tiles an XCD works on, in the order of its tickets.  The tiles go to the XCDs in chunks of
// consecutive tiles taken in turn (ticket t of XCD x is tile ((t / chunk) * 8 + x) * chunk + t % chunk): neighbouring
// tiles still meet in one L2, and every XCD gets a sample of the whole object instead of one contiguous eighth, whose
// k-steps per tile can differ (1 M points on six ellipsoids, 32 views: the eighths finished between 665 and 775 us).
// The tiles behind the last whole round of chunks are split into eight contiguous parts, so that the XCDs' shares
// differ by one tile at most and the first XCDs hold the larger ones (handed out as whole chunks, 6250 tiles gave two XCDs 832 and
// 810 tiles and the others 768).
struct XcdTiles {
  int sh, xcd_sh, full, rest_at, len;   // chunk = 2^sh; tickets below `full` are chunked, the others contiguous
  __device__ XcdTiles(int nblk, int xcd) {
    sh = 31 - __builtin_clz(max(1, min(64, nblk / (8 * kXcd))));   // chunk = 2^sh tiles: 64, fewer for small objects
    const int rounds = nblk >> (sh + 3);                            // kXcd = 8 chunks per round
    static_assert(kXcd == 8, "rounds of eight chunks");
    full = rounds << sh;
    const int base = rounds << (sh + 3), rest = nblk - base;
    // XCD x takes rest / 8 of them and one more while x < rest % 8: an object of fewer than eight tiles has workgroups on
    // its first XCDs only
    const int q = rest >> 3, extra = rest & 7;
    rest_at = base + xcd * q + min(xcd, extra) - full;
    len = full + q + (xcd < extra ? 1 : 0);
    xcd_sh = xcd << sh;
  }
  __device__ int at(int t) const {
    return t < full ? ((((t >> sh) * kXcd) << sh) + xcd_sh + (t & ((1 << sh) - 1))) : rest_at + t;
  }
};

// Orders the producer wave's LDS traffic for the compiler.  The LDS unit handles the instructions of one wave in
// program order, so a later read by any lane sees an earlier write by any other lane of the same wave: no wait and
// no barrier instruction is needed, only that the compiler keeps the order.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

}  // namespace aura
