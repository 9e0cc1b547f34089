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

// op(v of this lane, v of lane ^ OFF).  Vector instructions only; by way of the LDS crossbar (ds_bpermute, which
// __shfl_xor is) every step waits for a round trip.  There is none that exchanges lanes 4 apart: kMirror4 meets the right
// value where each group of 4 lanes holds one (after the steps 1 and 2), kTurn4 where v repeats every 8 lanes (after 8).
// From shuffles to these, same bits: decode_attention_kernel<128> 102 -> 92 registers (4 -> 5 waves per SIMD), a decoding
// step of OPT-13B at 1 row 129.3 -> 128.2 us, at 64 rows 264.6 -> 262.3.
constexpr int kMirror4 = -1, kTurn4 = -2;
template <int OFF, class Op>
__device__ __forceinline__ float lane_op(float v, Op op) {
  const uint32_t u = __float_as_uint(v);
  if constexpr (OFF == 32) {
    const auto halves = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return op(__uint_as_float(halves[0]), __uint_as_float(halves[1]));
  } else if constexpr (OFF == 16) {
    const auto rows = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return op(__uint_as_float(rows[0]), __uint_as_float(rows[1]));
  } else {
    static_assert(OFF == 8 || OFF == kMirror4 || OFF == kTurn4 || OFF == 2 || OFF == 1);
    // row_ror:8, row_half_mirror, row_ror:4, quad_perm [2,3,0,1], quad_perm [1,0,3,2]
    constexpr int kCtrl = OFF == 8 ? 0x128 : (OFF == kMirror4 ? 0x141 : (OFF == kTurn4 ? 0x124 : (OFF == 2 ? 0x4e : 0xb1)));
    return op(v, __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)u, kCtrl, 0xf, 0xf, true)));
  }
}
struct AddOp {
  __device__ __forceinline__ float operator()(float a, float b) const { return a + b; }
};
struct MaxOp {
  __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); }
};
// Over all lanes that differ in the bits FROM .. 32 of their number, in every lane; FROM is 8 or more.
template <int FROM, class Op>
__device__ __forceinline__ float across_groups(float v, Op op) {
  if constexpr (FROM <= 8) v = lane_op<8>(v, op);
  if constexpr (FROM <= 16) v = lane_op<16>(v, op);
  return lane_op<32>(v, op);
}
// Over groups of 8 or 16 lanes.
template <int LANES, class Op>
__device__ __forceinline__ float within_group(float v, Op op) {
  static_assert(LANES == 8 || LANES == 16);
  v = lane_op<1>(v, op);
  v = lane_op<2>(v, op);
  v = lane_op<kMirror4>(v, op);
  if constexpr (LANES == 16) v = lane_op<8>(v, op);
  return v;
}
// Sum over the wave, in every lane.
__device__ __forceinline__ float wave_sum(float v) {
  v = lane_op<32>(v, AddOp());
  v = lane_op<16>(v, AddOp());
  v = lane_op<8>(v, AddOp());
  v = lane_op<kTurn4>(v, AddOp());
  v = lane_op<2>(v, AddOp());
  return lane_op<1>(v, AddOp());
}

// 16-byte global load / store through plain vector accesses
__device__ __forceinline__ u32x4 ld16(const void* p) { return *reinterpret_cast<const u32x4*>(p); }
__device__ __forceinline__ void st16(void* p, u32x4 v) { *reinterpret_cast<u32x4*>(p) = v; }

// The output segments (Q | K | V) of a product: buffers, row strides and first columns, as sums of what each of a lane's
// two comparisons adds.  Indexed by the lane's segment, or selected, the pointers would come from the argument block in
// memory (that is what the compiler makes of either): one load per store, and a store that waits for a load waits for
// the store before it too.
typedef __attribute__((address_space(1))) uint16_t gmem_u16;
struct OutSegments {
  uint64_t base, to_k, to_v;  // address of column 0 as Q has it; what K and then V add
  int ld, to_kv, c1, c2;
  __device__ __forceinline__ gmem_u16* at(int row, int n) const {
    const int kv = n >= c1 ? -1 : 0, v = n >= c2 ? -1 : 0;
    const uint64_t o = base + (to_k & (uint64_t)(int64_t)kv) + (to_v & (uint64_t)(int64_t)v);
    return (gmem_u16*)(o + 2 * ((uint64_t)row * (uint32_t)(ld + (to_kv & kv)) + n));
  }
};
template <class P>
__device__ __forceinline__ OutSegments out_segments(const P& p, int ld_first) {
  const int c1 = p.seg_cols, c2 = c1 + p.seg_cols_kv;
  const uint64_t q = (uint64_t)p.out[0], k = (uint64_t)p.out[1] - 2 * (uint64_t)c1, v = (uint64_t)p.out[2] - 2 * (uint64_t)c2;
  return OutSegments{q, k - q, v - k, ld_first, p.seg_cols_kv - ld_first, c1, c2};
}
__device__ __forceinline__ void st16(gmem_u16* p, u32x4 v) { *(__attribute__((address_space(1))) u32x4*)p = v; }
__device__ __forceinline__ void st8(gmem_u16* p, u32x2 v) { *(__attribute__((address_space(1))) u32x2*)p = v; }

// Workgroup barrier that closes this wave's LDS reads and leaves its direct-to-LDS loads in flight (behind
// __syncthreads() the compiler may wait for all of them).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace ds
