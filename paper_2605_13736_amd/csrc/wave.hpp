#pragma once
// Wave-wide (64-lane) reductions on data-parallel-primitive (DPP) lane moves.
//
// A lane move through DPP is a VALU operand modifier: it costs one VALU
// instruction and no LDS round trip, where a __shfl_xor step is a
// ds_bpermute through the LDS crossbar with its full latency.  A reduction
// combines within quads (xor 1, xor 2), then rotates within each row of 16
// lanes by 4 and by 8, after which every lane of a row holds the row's
// result; readlane of lanes 0, 16, 32 and 48 then combines the four rows in
// the same order in every lane.  All 64 lanes must be active.
#include <hip/hip_runtime.h>

#include <climits>
#include <type_traits>

namespace mds {

// f(0), ..., f(n - 1) with compile-time indices
template <int N, int I = 0, typename F>
__device__ __attribute__((always_inline)) inline void static_for(F &&f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

namespace wave {

constexpr int kXor1 = 0xB1;  // quad_perm [1, 0, 3, 2]
constexpr int kXor2 = 0x4E;  // quad_perm [2, 3, 0, 1]
constexpr int kRor4 = 0x124; // row_ror:4
constexpr int kRor8 = 0x128; // row_ror:8

template <int C>
__device__ inline int dpp(int v) {
  return __builtin_amdgcn_update_dpp(v, v, C, 0xf, 0xf, false);
}
template <int C>
__device__ inline double dpp(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = dpp<C>((int)b), hi = dpp<C>((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ inline int lane_read(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ inline double lane_read(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// larger magnitude, then smaller position (a total order: every lane ends
// with the same pair whatever the combination order)
__device__ inline void amax2(double &v, int &i, double v2, int i2) {
  if (v2 > v || (v2 == v && i2 < i)) {
    v = v2;
    i = i2;
  }
}
__device__ inline void amax3(double &v, int &i, int &s, double v2, int i2, int s2) {
  if (v2 > v || (v2 == v && i2 < i)) {
    v = v2;
    i = i2;
    s = s2;
  }
}

// maximum over the wave (fmax: a NaN operand is ignored), every lane
__device__ inline double max(double v) {
  v = fmax(v, dpp<kXor1>(v));
  v = fmax(v, dpp<kXor2>(v));
  v = fmax(v, dpp<kRor4>(v));
  v = fmax(v, dpp<kRor8>(v));
  double r = fmax(lane_read(v, 0), lane_read(v, 16));
  return fmax(r, fmax(lane_read(v, 32), lane_read(v, 48)));
}

// minimum over the wave, every lane
__device__ inline int imin(int v) {
  v = min(v, dpp<kXor1>(v));
  v = min(v, dpp<kXor2>(v));
  v = min(v, dpp<kRor4>(v));
  v = min(v, dpp<kRor8>(v));
  return min(min(lane_read(v, 0), lane_read(v, 16)), min(lane_read(v, 32), lane_read(v, 48)));
}

// arg-max over the wave, result in every lane (wave-uniform): the maximum, then
// the least position that has it (a step of the pair together takes three
// times the instructions).  A NaN is never the maximum.
__device__ inline void amax(double &v, int &i) {
  const double m = max(v);
  i = imin(v == m ? i : INT_MAX);
  v = m;
}
// ... with a value s of the lane that holds it (positions differ)
__device__ inline void amax(double &v, int &i, int &s) {
  const double m = max(v);
  const int p = imin(v == m ? i : INT_MAX);
  const unsigned long long at = __ballot(v == m && i == p);
  s = lane_read(s, at ? __ffsll(at) - 1 : 0);
  v = m;
  i = p;
}

// sum over the 16 lanes of each row: every lane of the row
__device__ inline double row_sum(double v) {
  v = v + dpp<kXor1>(v);
  v = v + dpp<kXor2>(v);
  v = v + dpp<kRor4>(v);
  return v + dpp<kRor8>(v);
}

// sum over the wave, every lane (association: quads, rows, then rows 0..3)
__device__ inline double sum(double v) {
  v = v + dpp<kXor1>(v);
  v = v + dpp<kXor2>(v);
  v = v + dpp<kRor4>(v);
  v = v + dpp<kRor8>(v);
  return (lane_read(v, 0) + lane_read(v, 16)) + (lane_read(v, 32) + lane_read(v, 48));
}

// lane C of each row of 16 lanes, in every lane of the row (one 64-bit move)
template <int C>
__device__ inline double row_lane(double v) {
  static_assert(C >= 0 && C < 16, "row lane");
  return __longlong_as_double(
      __builtin_amdgcn_mov_dpp(__double_as_longlong(v), 0x150 + C, 0xf, 0xf, true));
}

// o[q] = x of lane (l & 15) + 16 q
__device__ inline void rows4(double x, double (&o)[4]) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  unsigned r[2][4];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const unsigned v = (unsigned)(b >> (32 * h));
    // [r0 r1 r0 r1], [r2 r3 r2 r3]; then one row of each pair everywhere
    const auto a = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    const auto lo = __builtin_amdgcn_permlane16_swap(a[0], a[0], false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(a[1], a[1], false, false);
    r[h][0] = lo[0];
    r[h][1] = lo[1];
    r[h][2] = hi[0];
    r[h][3] = hi[1];
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
    o[q] = __longlong_as_double((long long)(((unsigned long long)r[1][q] << 32) | r[0][q]));
}

__device__ inline double sel4(int q, double a, double b, double c, double d) {
  return (q < 2) ? (q == 0 ? a : b) : (q == 2 ? c : d);
}

}  // namespace wave
}  // namespace mds
