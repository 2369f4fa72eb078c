// Device helpers of the tiled candidate sweeps.
#pragma once

#include <algorithm>
#include <cfloat>
#include <type_traits>

#include "block_sort.h"

namespace rkhsba {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kLanes = 64;
constexpr int kTile = 64;  // candidates fetched together, one per lane

__device__ inline int clamp_floor_d(double v, int lo, int hi) {
  v = floor(v);
  v = fmin(fmax(v, (double)lo), (double)hi);
  return (int)v;
}

__device__ inline float uniform_f(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// Cross-lane moves within rows of 16 lanes (DPP: no LDS round trip).
template <int CTRL>
__device__ inline float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
constexpr int kDppXor1 = 0xb1;         // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4e;         // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141;  // lane i <-> 7 - i within each half row
constexpr int kDppMirror = 0x140;      // lane i <-> 15 - i within each row
constexpr int kDppRor8 = 0x128;        // lane i <- lane (i + 8) mod 16 within each row, i.e. i ^ 8

// Minimum / maximum over the P consecutive lanes of each lane group (P = 8, 16 or 32): the quad, then the
// other quad of the half row, then the other half row, then the other row of the 32.
template <int P>
__device__ inline float group_min(float v) {
  static_assert(P == 8 || P == 16 || P == 32, "groups of 8, 16 or 32 lanes");
  v = fminf(v, dpp_f<kDppXor1>(v));
  v = fminf(v, dpp_f<kDppXor2>(v));
  v = fminf(v, dpp_f<kDppHalfMirror>(v));
  if constexpr (P >= 16) v = fminf(v, dpp_f<kDppMirror>(v));
  if constexpr (P == 32) v = fminf(v, __shfl_xor(v, 16, 64));
  return v;
}
template <int P>
__device__ inline float group_max(float v) {
  static_assert(P == 8 || P == 16 || P == 32, "groups of 8, 16 or 32 lanes");
  v = fmaxf(v, dpp_f<kDppXor1>(v));
  v = fmaxf(v, dpp_f<kDppXor2>(v));
  v = fmaxf(v, dpp_f<kDppHalfMirror>(v));
  if constexpr (P >= 16) v = fmaxf(v, dpp_f<kDppMirror>(v));
  if constexpr (P == 32) v = fmaxf(v, __shfl_xor(v, 16, 64));
  return v;
}

// The same over quads of consecutive lanes.
__device__ inline float quad_min(float v) {
  v = fminf(v, dpp_f<kDppXor1>(v));
  return fminf(v, dpp_f<kDppXor2>(v));
}
__device__ inline float quad_max(float v) {
  v = fmaxf(v, dpp_f<kDppXor1>(v));
  return fmaxf(v, dpp_f<kDppXor2>(v));
}

// A lane's value as a uniform one.
__device__ inline float lane_f(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// v + (v of lane ^ O), the same sum in both lanes (addition is commutative): a DPP row rotation for O = 8,
// a cross-lane read through the LDS crossbar for 16 and 32.
template <int O, typename T>
__device__ inline T xor_add(T v) {
  static_assert(O == 8 || O == 16 || O == 32, "lane distance");
  if constexpr (O == 8) {
    const uint32_t u = __builtin_bit_cast(uint32_t, v);
    return v + __builtin_bit_cast(T, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u, kDppRor8, 0xf, 0xf, false));
  } else {
    return v + __shfl_xor(v, O, 64);
  }
}

// Inclusive max-scan of unsigned values over the wavefront's 64 lanes: four
// row shifts within each row of 16 lanes, then the last lane of a row
// broadcast to the rows after it.  Lanes a shift leaves without a source read
// the identity 0.
__device__ inline uint32_t wave_inclusive_max(uint32_t v) {
  const int x = (int)v;
  int m = x;
  m = (int)max((uint32_t)m, (uint32_t)__builtin_amdgcn_update_dpp(0, m, 0x111, 0xf, 0xf, true));  // row_shr:1
  m = (int)max((uint32_t)m, (uint32_t)__builtin_amdgcn_update_dpp(0, m, 0x112, 0xf, 0xf, true));  // row_shr:2
  m = (int)max((uint32_t)m, (uint32_t)__builtin_amdgcn_update_dpp(0, m, 0x114, 0xf, 0xf, true));  // row_shr:4
  m = (int)max((uint32_t)m, (uint32_t)__builtin_amdgcn_update_dpp(0, m, 0x118, 0xf, 0xf, true));  // row_shr:8
  m = (int)max((uint32_t)m, (uint32_t)__builtin_amdgcn_update_dpp(0, m, 0x142, 0xa, 0xf, false));  // row_bcast:15
  m = (int)max((uint32_t)m, (uint32_t)__builtin_amdgcn_update_dpp(0, m, 0x143, 0xc, 0xf, false));  // row_bcast:31
  return (uint32_t)m;
}

// Squared distance of candidate z to the box [lo, hi], rounded like the membership rule: each axis term
// max(lo - z, z - hi, 0) and the fused sum in rule_s2's order.  Rounding is monotone, so for every point q of
// the box this is at most rule_s2(q, z): a candidate above rc2 here fails the rule for every source in the box.
__device__ inline float box_s2(float3 lo, float3 hi, float4 z) {
#pragma clang fp contract(off)
  const float bx = fmaxf(fmaxf(lo.x - z.x, z.x - hi.x), 0.f);
  const float by = fmaxf(fmaxf(lo.y - z.y, z.y - hi.y), 0.f);
  const float bz = fmaxf(fmaxf(lo.z - z.z, z.z - hi.z), 0.f);
  return fmaf(bz, bz, fmaf(by, by, bx * bx));
}

// The cell rows that the ball of the given reach around the box [lo, hi] can touch: z0 .. z0 + n / ny - 1 by
// y0 .. y0 + ny - 1 (n: 0 when there is none).
struct RowBox {
  int z0, y0, ny, n;
  double inv_ny;
  // r = oz * ny + oy, 0 <= r < n: the FP64 quotient is off by at most one (an integer division takes three times
  // the instructions, and every row of every pass needs one)
  __device__ void split(int r, int& oz, int& oy) const {
    oz = (int)((double)r * inv_ny);
    oy = r - oz * ny;
    if (oy < 0) { --oz; oy += ny; }
    else if (oy >= ny) { ++oz; oy -= ny; }
  }
};
__device__ inline RowBox row_box(const FrameInfo& F, const KConst& kc, float3 lo, float3 hi) {
  const double inv = kc.inv_cell, reach = kc.reach;
  RowBox B;
  B.z0 = max(clamp_floor_d(((double)lo.z - reach) * inv - F.org[2], -1, F.dim[2]), 0);
  const int z1 = min(clamp_floor_d(((double)hi.z + reach) * inv - F.org[2], -1, F.dim[2]), F.dim[2] - 1);
  B.y0 = max(clamp_floor_d(((double)lo.y - reach) * inv - F.org[1], -1, F.dim[1]), 0);
  const int y1 = min(clamp_floor_d(((double)hi.y + reach) * inv - F.org[1], -1, F.dim[1]), F.dim[1] - 1);
  B.ny = y1 - B.y0 + 1;
  B.inv_ny = 1.0 / (double)B.ny;  // (not used when there is no row)
  B.n = (z1 >= B.z0 && y1 >= B.y0) ? (z1 - B.z0 + 1) * B.ny : 0;
  return B;
}

// Of the 64 batches of `batch` consecutive rows from row rb of B on, those with a row within the reach of a valid
// source (the first P lanes hold the sources' q; invalid ones are not valid).
template <int P>
__device__ inline uint64_t near_batches(const FrameInfo& F, const KConst& kc, const RowBox& B, float3 q, bool valid,
                                        int rb, int batch) {
  const int lane = threadIdx.x & 63;
  const int r0 = rb + batch * lane, r1 = min(r0 + batch, B.n) - 1;
  const int za = r0 / B.ny, zb = r1 / B.ny;
  const int ya = za == zb ? r0 - za * B.ny : 0, yb = za == zb ? r1 - zb * B.ny : B.ny - 1;
  const double cell = kc.cell;
  const double z_lo = (double)(B.z0 + za + F.org[2]) * cell, z_hi = (double)(B.z0 + zb + F.org[2]) * cell + cell;
  const double y_lo = (double)(B.y0 + ya + F.org[1]) * cell, y_hi = (double)(B.y0 + yb + F.org[1]) * cell + cell;
  const uint64_t vm = __builtin_amdgcn_ballot_w64(valid);
  bool near = false;
  for (int s = 0; s < P; ++s) {
    if (!((vm >> s) & 1ull)) continue;  // uniform
    const double y = (double)lane_f(q.y, s), z = (double)lane_f(q.z, s);
    const double dz = fmax(0.0, fmax(z_lo - z, z - z_hi)), dy = fmax(0.0, fmax(y_lo - y, y - y_hi));
    near = near || dy * dy + dz * dz <= kc.reach2;
  }
  return __builtin_amdgcn_ballot_w64(near && r0 < B.n);
}

// Candidate range of row (kz, ky): its x-range trimmed to the ball around the box, as the frame's sorted points
// j0 .. j0 + count - 1.
__device__ inline void row_range(const FrameInfo& F, const KConst& kc, const int4* __restrict__ trows,
                                 const uint32_t* __restrict__ xtab, float3 lo, float3 hi, int kz, int ky,
                                 uint32_t& j0, uint32_t& count) {
  const double inv = kc.inv_cell, cell = kc.cell;
  j0 = count = 0u;
  const double cz = (double)(kz + F.org[2]) * cell;
  const double cy = (double)(ky + F.org[1]) * cell;
  const double bz = fmax(0.0, fmax(cz - (double)hi.z, (double)lo.z - (cz + cell)));
  const double by = fmax(0.0, fmax(cy - (double)hi.y, (double)lo.y - (cy + cell)));
  const double r2 = kc.reach2 - by * by - bz * bz;
  if (!(r2 >= 0.0)) return;
  const int4 R = trows[(int64_t)kz * F.dim[1] + ky];
  if (R.y < R.x) return;
  // half-width of the ball's chord in x: the hardware FP32 root (within an ulp) widened by 2^-16,
  // which exceeds the root's and the conversion's rounding, so no cell of the chord is lost
  const double h = (double)__builtin_amdgcn_sqrtf((float)r2) * (1.0 + 0x1p-16);
  const int xa = max(clamp_floor_d(((double)lo.x - h) * inv - F.org[0], -1, F.dim[0]), R.x);
  const int xb = min(clamp_floor_d(((double)hi.x + h) * inv - F.org[0], -1, F.dim[0]), R.y);
  if (xa > xb) return;
  const uint32_t* xt = xtab + F.xt_off + (uint32_t)R.z;
  j0 = xt[xa - R.x];
  count = xt[xb + 1 - R.x] - j0;
}

}  // namespace rkhsba
