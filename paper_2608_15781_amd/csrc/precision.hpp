// Storage precision of the populations. The arithmetic type R is double for FP64 storage and
// float otherwise. The *_DEV storages hold each population as its deviation from the lattice
// weight (scaled by 2^k for FP16 so that deviations of order 1e-6 stay out of the subnormal
// range); a uniform fluid at rest therefore stores exact zeros.
//
// Modes 0..3 address their arrays with 32-bit byte offsets from wave-uniform bases: the offset is
// one register and the base stays in scalar registers, where 64-bit per-lane addresses take a
// shift, a sign extension and a 64-bit add (or, for a selected plane, a 64-bit product at a quarter
// of the rate) on every gather. Modes 4..7 are the same storages with 64-bit offsets, for lattices
// whose arrays pass 4 GB (see offsets.hpp).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <hip/hip_bf16.h>

#include <cstdint>

namespace lbm {

template <int P>
struct Prec;

constexpr int kWideMode = 4;  // added to a storage's mode for 64-bit offsets

template <>
struct Prec<0> {
  using Off = uint32_t;
  static constexpr bool deviations = false;
  using S = double;
  using R = double;
  __device__ static inline R ld(S s, R, R) { return s; }
  __device__ static inline S st(R v, R, R) { return v; }
};

template <>
struct Prec<1> {
  using Off = uint32_t;
  static constexpr bool deviations = false;
  using S = float;
  using R = float;
  __device__ static inline R ld(S s, R, R) { return s; }
  __device__ static inline S st(R v, R, R) { return v; }
};

template <>
struct Prec<2> {
  using Off = uint32_t;
  static constexpr bool deviations = true;
  using S = __half;
  using R = float;
  __device__ static inline R ld(S s, R w, R inv_scale) { return w + __half2float(s) * inv_scale; }
  __device__ static inline S st(R v, R w, R scale) { return __float2half_rn((v - w) * scale); }
};

template <>
struct Prec<3> {
  using Off = uint32_t;
  static constexpr bool deviations = true;
  using S = __hip_bfloat16;
  using R = float;
  __device__ static inline R ld(S s, R w, R inv_scale) { return w + __bfloat162float(s) * inv_scale; }
  __device__ static inline S st(R v, R w, R scale) { return __float2bfloat16((v - w) * scale); }
};

template <int P>
struct Prec : Prec<P - kWideMode> {
  using Off = size_t;
};

}  // namespace lbm
