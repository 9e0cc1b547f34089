// Shared device helpers for the gfx950 kernels: vector types, bf16 packing,
// wave-level reductions.  Wavefronts are 64 lanes wide.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// Development switches (force a tile shape, a split count, a kernel choice): plain constants in the library
// build, so the choice logic they sit in folds away; the timing harnesses compile the sources with
// -DDS_DEV_SWITCHES and flip them at run time.  The kernels are the same in both builds; wall-clock stamps inside them
// need -DDS_DEV_STAMPS and give other code (the 256x160 GEMM loop: 279 vector instructions per k-tile, not 4).
#ifdef DS_DEV_SWITCHES
namespace ds {
struct SwitchReg {  // makes a switch settable by name through ds_dev_switch (development builds only)
  SwitchReg(const char* name, int* value);
};
}  // namespace ds
#define DS_SWITCH(name, value) \
  int name = value;            \
  static ::ds::SwitchReg switch_reg_##name(#name, &name)
#else
#define DS_SWITCH(name, value) static constexpr int name = value
#endif

namespace ds {

typedef __bf16 bf16_t;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;

constexpr int kWave = 64;

__device__ __forceinline__ float bf16_lo(uint32_t packed) { return __uint_as_float(packed << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t packed) { return __uint_as_float(packed & 0xffff0000u); }

// two floats -> packed bf16 pair (round to nearest even), lo in bits 0..15
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  bf16x2 v;
  v[0] = (__bf16)lo;
  v[1] = (__bf16)hi;
  return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  return v;
}

// 16-byte global load / store through plain vector accesses
__device__ __forceinline__ u32x4 ld16(const void* p) { return *reinterpret_cast<const u32x4*>(p); }
__device__ __forceinline__ void st16(void* p, u32x4 v) { *reinterpret_cast<u32x4*>(p) = v; }

// Workgroup barrier that closes this wave's LDS reads and leaves its direct-to-LDS loads in flight (behind
// __syncthreads() the compiler may wait for all of them).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace ds
