// Device helpers the convolution kernels share: direct-to-LDS wave loads,
// vmcnt waits, buffer descriptors, output stores; the launch with dispatch
// events.
#pragma once
#include <hip/hip_ext.h>

#include "common.hpp"

namespace dstack {

constexpr int BK = 64;          // depth per LDS stage (bf16 elements)
constexpr int ROW_BYTES = 128;  // one tile row = BK bf16
constexpr unsigned OOB = 0x80000000u;  // buffer offset past any tensor (< 2 GB): loads zeros
constexpr int CPOL_SC1 = 16;           // buffer cache-policy bit: device scope (past the per-XCD L2)

__device__ __forceinline__ void store_out4(void* y, bool f32, long idx, const float v[4]) {
  if (f32) {
    f32x4 o = {v[0], v[1], v[2], v[3]};
    *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(y) + idx) = o;
  } else {
    bf16x4 o = {(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]};
    *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(y) + idx) = o;
  }
}

// vmcnt wait with an immediate count (gfx9 encoding: vmcnt[3:0] | vmcnt[5:4] << 14,
// expcnt and lgkmcnt left at "no wait").
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt is 6 bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

typedef __attribute__((__vector_size__(4 * sizeof(int)))) int i32x4;

// Raw buffer descriptor: base, no stride, num_records = byte size (offsets at
// or past it read as zero), gfx9 data-format word.
__device__ __forceinline__ i32x4 make_rsrc(const void* base, unsigned bytes) {
  const unsigned long long p = (unsigned long long)base;
  i32x4 r;
  r[0] = (int)(unsigned)(p & 0xffffffffu);
  r[1] = (int)(unsigned)((p >> 32) & 0xffffu);
  r[2] = (int)bytes;
  r[3] = 0x00020000;
  return r;
}

// 32-bit LDS byte address of a pointer into a __shared__ array.
__device__ __forceinline__ unsigned lds_address(const void* p) {
  return (unsigned)(unsigned long long)(const __attribute__((address_space(3))) void*)p;
}

// NL wave-loads of 16 bytes per lane: load j moves buffer offsets off[j]
// into LDS at lds_base + 1024 * j + 16 * lane.  Issued as inline asm so that
// the compiler does not treat every later LDS read as dependent on it (it
// would wait for all loads in flight); the kernel's own vmcnt waits order
// these loads against the LDS reads.  M0 (the LDS destination) is saved once,
// stepped by 1 KB between loads (one wait state after each write), restored.
template <int NL>
__device__ __forceinline__ void load_group(i32x4 rsrc, const unsigned (&off)[NL], unsigned lds_base);

template <>
__device__ __forceinline__ void load_group<1>(i32x4 rsrc, const unsigned (&off)[1], unsigned lds_base) {
  unsigned saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %1\n\t"
      "s_nop 0\n\t"
      "buffer_load_dwordx4 %2, %3, 0 offen lds\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "s"(lds_base), "v"(off[0]), "s"(rsrc)
      : "memory");
}

template <>
__device__ __forceinline__ void load_group<2>(i32x4 rsrc, const unsigned (&off)[2], unsigned lds_base) {
  unsigned saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %1\n\t"
      "s_nop 0\n\t"
      "buffer_load_dwordx4 %2, %4, 0 offen lds\n\t"
      "s_add_u32 m0, m0, 0x400\n\t"
      "s_nop 0\n\t"
      "buffer_load_dwordx4 %3, %4, 0 offen lds\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "s"(lds_base), "v"(off[0]), "v"(off[1]), "s"(rsrc)
      : "memory", "scc");
}

template <>
__device__ __forceinline__ void load_group<4>(i32x4 rsrc, const unsigned (&off)[4], unsigned lds_base) {
  unsigned saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\t"
      "s_mov_b32 m0, %1\n\t"
      "s_nop 0\n\t"
      "buffer_load_dwordx4 %2, %6, 0 offen lds\n\t"
      "s_add_u32 m0, m0, 0x400\n\t"
      "s_nop 0\n\t"
      "buffer_load_dwordx4 %3, %6, 0 offen lds\n\t"
      "s_add_u32 m0, m0, 0x400\n\t"
      "s_nop 0\n\t"
      "buffer_load_dwordx4 %4, %6, 0 offen lds\n\t"
      "s_add_u32 m0, m0, 0x400\n\t"
      "s_nop 0\n\t"
      "buffer_load_dwordx4 %5, %6, 0 offen lds\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "s"(lds_base), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(rsrc)
      : "memory", "scc");
}

// A launch of `threads` threads per block; through hipExtLaunchKernelGGL when
// dispatch events are armed (and not while launch shapes are being recorded).
template <typename K, typename... Args>
inline void launch_k(K kernel, dim3 grid, int threads, hipStream_t st, hipEvent_t e0, hipEvent_t e1, Args... args) {
  if ((e0 || e1) && !shape_recorder())
    hipExtLaunchKernelGGL(kernel, grid, dim3(threads), 0, st, e0, e1, 0, args...);
  else
    launch(kernel, grid, dim3(threads), 0, st, args...);
}

// Estimated cost of a split-K plan: device-scope slice stores until
// acknowledged; per slice of 8192 fp32 values, the last block's read-back.
constexpr double CONV_SLICE_WRITE_US = 2.6, CONV_SLICE_READ_US = 0.75;

// Launch of the 3x3 stride-1 kernel: tile shape and pixel tiling of the first
// n_main images, depth slices, and (n_main < N) the tiling of the others;
// `cost` the estimated time in us.
struct HaloPlan {
  int tile, th, tw, splits, chunks_per_split, n_main;
  int rest_tile, rest_th, rest_tw;
  double cost;
};
// false: no tile shape takes it.  C % 64 == 0.
bool halo_plan(int N, int H, int W, int C, int K, int n_cu, bool can_split, size_t split_bytes, HaloPlan* out);
void halo_tile(const HaloPlan& p, int* bn, int* bm, int* stages);
// K % 8 == 0; a split plan needs the workspace and counters it was made for.
void launch_halo(const bf16* x, int N, int H, int W, int C, const bf16* w, int K, const float* scale,
                 const float* shift, const bf16* res, int act, bf16* y, const HaloPlan& p, float* splitk_ws,
                 unsigned* tile_counters, hipStream_t st);

}  // namespace dstack
