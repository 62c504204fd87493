// Exchanges between the lanes of a wave on the vector unit.  The general shuffles go through the LDS unit, about 50 ns
// each, one behind the other in a reduction; these take a few cycles.  Every reduction pairs the same lanes in the
// same order as the butterfly of exchanges by xor that it stands for, but both lanes of a pair may evaluate f with the same
// first argument: f must be commutative, and then the results are the same bits.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace pipesd {

typedef __attribute__((ext_vector_type(2))) unsigned lanes_u32x2;

// {x's of an even and an odd row of 16 lanes}, the same two for both: lanes l and l ^ 16
__device__ __forceinline__ lanes_u32x2 lanes_xor16(unsigned x) {
  return __builtin_bit_cast(lanes_u32x2, __builtin_amdgcn_permlane16_swap(x, x, false, false));
}
// {x of lane l % 32, x of lane l % 32 + 32}
__device__ __forceinline__ lanes_u32x2 lanes_xor32(unsigned x) {
  return __builtin_bit_cast(lanes_u32x2, __builtin_amdgcn_permlane32_swap(x, x, false, false));
}
// x of the lane N further down its row of 16, in a circle: of lane l ^ N where x repeats every 2 N lanes
template <int N>
__device__ __forceinline__ unsigned lanes_ror(unsigned x) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x120 + N, 0xf, 0xf, false);
}

template <class F>
__device__ __forceinline__ float fold16(float x, F f) {  // f(the even row's, the odd row's), in both of lanes l and l ^ 16
  const lanes_u32x2 p = lanes_xor16(__float_as_uint(x));
  return f(__uint_as_float(p.x), __uint_as_float(p.y));
}
template <class F>
__device__ __forceinline__ float fold32(float x, F f) {  // f(the lower half's, the upper half's), in both of lanes l and l ^ 32
  const lanes_u32x2 p = lanes_xor32(__float_as_uint(x));
  return f(__uint_as_float(p.x), __uint_as_float(p.y));
}
// the lanes {l, l ^ 16, l ^ 32, l ^ 48}: by 16, then by 32
template <class F>
__device__ __forceinline__ float fold_groups(float x, F f) {
  return fold32(fold16(x, f), f);
}
// all lanes: by 32, 16, 8, 4, 2, 1
template <class F>
__device__ __forceinline__ float fold_wave(float x, F f) {
  x = fold16(fold32(x, f), f);
  x = f(x, __uint_as_float(lanes_ror<8>(__float_as_uint(x))));
  x = f(x, __uint_as_float(lanes_ror<4>(__float_as_uint(x))));
  x = f(x, __uint_as_float(lanes_ror<2>(__float_as_uint(x))));
  return f(x, __uint_as_float(lanes_ror<1>(__float_as_uint(x))));
}
struct LaneAdd {
  __device__ __forceinline__ float operator()(float a, float b) const { return a + b; }
};
struct LaneMax {
  __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); }
};

// x of lane l + 16, for the lanes of even rows; of lane l + 32, for the lanes below 32
__device__ __forceinline__ float from16(float x) { return __uint_as_float(lanes_xor16(__float_as_uint(x)).y); }
__device__ __forceinline__ float from32(float x) { return __uint_as_float(lanes_xor32(__float_as_uint(x)).y); }

__device__ __forceinline__ unsigned long long lanes_u64(unsigned lo, unsigned hi) { return ((unsigned long long)hi << 32) | lo; }
// sum over all lanes (in 64 bits the order is no matter)
__device__ __forceinline__ unsigned long long sum_wave(unsigned long long v) {
  auto ror = [&](auto n) {
    constexpr int N = decltype(n)::value;
    v += lanes_u64(lanes_ror<N>((unsigned)v), lanes_ror<N>((unsigned)(v >> 32)));
  };
  lanes_u32x2 lo = lanes_xor32((unsigned)v), hi = lanes_xor32((unsigned)(v >> 32));
  v = lanes_u64(lo.x, hi.x) + lanes_u64(lo.y, hi.y);
  lo = lanes_xor16((unsigned)v), hi = lanes_xor16((unsigned)(v >> 32));
  v = lanes_u64(lo.x, hi.x) + lanes_u64(lo.y, hi.y);
  ror(std::integral_constant<int, 8>{});
  ror(std::integral_constant<int, 4>{});
  ror(std::integral_constant<int, 2>{});
  ror(std::integral_constant<int, 1>{});
  return v;
}
// sums of the lanes 0 .. own lane: inside the rows of 16, then the totals of the rows before (lane 15 of the row
// before into rows 1 and 3, lane 31 into rows 2 and 3)
__device__ __forceinline__ unsigned long long scan_wave(unsigned long long v) {
  auto add = [&](auto ctrl, auto rows) {
    constexpr int C = decltype(ctrl)::value, R = decltype(rows)::value;
    v += lanes_u64((unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)v, C, R, 0xf, true),
                   (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(v >> 32), C, R, 0xf, true));
  };
  typedef std::integral_constant<int, 0xf> all;
  add(std::integral_constant<int, 0x111>{}, all{});  // lane - 1 of the row, 0 beyond its start
  add(std::integral_constant<int, 0x112>{}, all{});
  add(std::integral_constant<int, 0x114>{}, all{});
  add(std::integral_constant<int, 0x118>{}, all{});
  add(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});
  add(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});
  return v;
}

}  // namespace pipesd
