// Values that three bf16 parts cannot carry, and the plain fp32 kernels that take over for them.
//
// Three parts hold all 24 bits of an fp32 value from 2^-110 up to bf16's largest.  Infinities, NaN, larger and
// smaller values (the third part's lowest bit lies 2^23 below the value, and bf16's subnormals end at 2^-133)
// are noticed where an operand is split, sums past fp32's range where they are stored.  Either raises a word
// of the call, and the plain fp32 kernel that is launched behind the split one then computes the whole result
// again; without one its workgroups end at once.  A call on such values costs what the plain kernel (without
// offset splits) costs, whatever their number; any call the clearing of the words and a launch that ends at
// once, about 6 us.
#pragma once

#include "common.hpp"

namespace ssconv {

// The words of a call, cleared before its first kernel.
struct SplitFlags {
  int* w = nullptr;
  static constexpr size_t kBytes = 256;
  __host__ __device__ int* feats() const { return w; }         // rows of feats
  __host__ __device__ int* grad_out() const { return w + 1; }  // rows of grad_out
  __host__ __device__ int* kappa() const { return w + 2; }
  __host__ __device__ int* gathered() const { return w + 3; }  // sums of the gather
  __host__ __device__ int* kgrad() const { return w + 4; }     // sums of the kernel gradient
};

int clear_split_flags(const SplitFlags& f, hipStream_t st);

// Condition of a kernel launch: one of the words is set (a == nullptr: no condition).
struct OnlyIf {
  const int *a = nullptr, *b = nullptr, *c = nullptr;
};
__device__ __forceinline__ bool idle(const OnlyIf& o) { return o.a && (*o.a | *o.b | *o.c) == 0; }

__device__ __forceinline__ bool past_range(float v) { return !(fabsf(v) <= 3.4028234e38f); }

}  // namespace ssconv
