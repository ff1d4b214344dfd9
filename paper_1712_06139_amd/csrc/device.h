// What the kernel sources share: vector types, bf16 conversion, the MFMA
// kernels' LDS, DMA and transposition helpers, and launch support.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "../../include/rb.h"

namespace {

typedef uint16_t bf16_t;
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16_t;
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16_t f2bf(float f) {
  // round to nearest even on the 16 dropped bits; NaN stays a (quiet) NaN
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

__device__ __forceinline__ float bf2f(uint32_t h) { return __uint_as_float(h << 16); }

__device__ __forceinline__ uint32_t pack2(float a, float b) {
  return (uint32_t)f2bf(a) | ((uint32_t)f2bf(b) << 16);
}

template <int ACT>
__device__ __forceinline__ float act_fn(float z) {
  if (ACT == RB_ACT_RELU) return z > 0.f ? z : 0.f;
  if (ACT == RB_ACT_SIGMOID) return 1.f / (1.f + expf(-z));
  return z;
}

// Workgroups are handed to the 8 XCDs round-robin (block i runs on XCD i % 8)
// and each XCD has its own L2. Remap so that XCD x gets a contiguous range of
// tiles: with tiles ordered row-block-major, the tiles sharing an A row-block
// then run on the same XCD and re-read it from that XCD's L2.
__device__ __forceinline__ int xcd_tile(int bid, int nb) {
  const int nb8 = nb & ~7;
  return bid < nb8 ? (bid & 7) * (nb8 >> 3) + (bid >> 3) : bid;
}

__device__ __forceinline__ float wave_sum(float v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// value of v in lane l ^ 2 / l ^ 1 of the same quad (DPP quad permutations:
// plain VALU moves, no LDS traffic)
__device__ __forceinline__ float quad_xor2(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, false));  // [2,3,0,1]
}
__device__ __forceinline__ float quad_xor1(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, false));  // [1,0,3,2]
}

// 4 x 4 transpose across the four lanes of a quad: lane 4q + i holding x[k] =
// element (k, i) ends up holding x[j] = element (i, j), where element (k, c)
// is the value lane 4q + c held in x[k]. Two exchange rounds (lane xor 2, then
// lane xor 1), each sending two values and keeping two, with selects only.
__device__ __forceinline__ void quad_transpose4(float (&x)[4], int lane) {
  const bool b1 = lane & 2, b0 = lane & 1;
  float r0 = quad_xor2(b1 ? x[0] : x[2]), r1 = quad_xor2(b1 ? x[1] : x[3]);
  const float y0 = b1 ? r0 : x[0], y1 = b1 ? r1 : x[1], y2 = b1 ? x[2] : r0, y3 = b1 ? x[3] : r1;
  r0 = quad_xor1(b0 ? y0 : y1);
  r1 = quad_xor1(b0 ? y2 : y3);
  x[0] = b0 ? r0 : y0;
  x[1] = b0 ? y1 : r0;
  x[2] = b0 ? r1 : y2;
  x[3] = b0 ? y3 : r1;
}

// two floats rounded to bf16 (round to nearest even, v_cvt_pk_bf16_f32),
// the first in the low half
__device__ __forceinline__ uint32_t pack2_rne(float a, float b) {
  typedef __bf16 bf16x2_hw __attribute__((ext_vector_type(2)));
  typedef float float2_hw __attribute__((ext_vector_type(2)));
  const float2_hw f = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_hw));
}

// s_waitcnt vmcnt(N) lgkmcnt(0) (gfx9 encoding: vmcnt[3:0], expcnt[6:4],
// lgkmcnt[11:8], vmcnt[5:4] in bits 15:14): at most N vector memory
// operations of this wave in flight and every LDS read of it returned.
template <int N>
__device__ __forceinline__ void wait_vmcnt_lds() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
}

template <int I>
using ic = std::integral_constant<int, I>;

// f(ic<0>{}), f(ic<1>{}), ..., f(ic<N - 1>{}), unrolled at compile time
template <int... I, class F>
__device__ __forceinline__ void for_each_ic(std::integer_sequence<int, I...>, F&& f) {
  (f(ic<I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  for_each_ic(std::make_integer_sequence<int, N>{}, f);
}

// LDS byte address of a __shared__ object.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

__device__ __forceinline__ void lds_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Buffer resource (gfx9 layout: base address, stride 0, no range limit) for
// a wave-uniform base address.
__device__ __forceinline__ i32x4_t buffer_rsrc(const void* base) {
  const uint64_t p = (uint64_t)(uintptr_t)base;
  i32x4_t r;
  r.x = __builtin_amdgcn_readfirstlane((int)(uint32_t)p);
  r.y = __builtin_amdgcn_readfirstlane((int)((uint32_t)(p >> 32) & 0xffffu));
  r.z = -1;
  r.w = 0x00020000;
  return r;
}

// One 16-byte-per-lane buffer -> LDS load (buffer_load_dwordx4 ... lds) of the
// bytes at base + voff + soff: lane l's 16 bytes land at LDS byte lds + 16 l.
// Issued as inline assembly so that the compiler does not add its own
// conservative waits for it: the kernel waits with explicit vmcnt counts and
// a barrier before the data is read.
__device__ __forceinline__ void buffer_to_lds(i32x4_t rsrc, uint32_t voff, uint32_t soff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(rsrc),
               "s"(soff)
               : "memory", "m0");
}

// A narrow head applied in the epilogue instead of storing the layer's
// output (HEAD >= 0, the head's activation): the layer's bf16 outputs of
// the tile (all N = BN columns of its rows) go to LDS, and row r's head
// output act(w . y_r + b) is written to out[rows[r].out] when that is >= 0.
struct HeadArgs {
  const rb_k_row* rows;
  const bf16_t* w;  // BN bf16 weights, 16-byte aligned
  float b;
  float* out;
};

// fp32 outputs written through a row map instead of to Y (rows != nullptr):
// row r's first d_out columns go to out[rows[r].out ...] when that is >= 0
// (the merged run's split fused into its last layer); padding rows and
// columns past d_out are dropped.
struct OutMap {
  const rb_k_row* rows;
  float* out;
  int d_out;
};

inline rb_status launch_status() {
  return hipGetLastError() == hipSuccess ? RB_OK : RB_EDEVICE;
}

// compute units of the current device (cached per device)
inline unsigned device_cus() {
  static std::atomic<int> cus[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int c = cus[dev].load(std::memory_order_relaxed);
  if (c <= 0) {
    if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c <= 0) c = 256;
    cus[dev].store(c, std::memory_order_relaxed);
  }
  return (unsigned)c;
}

}  // namespace
