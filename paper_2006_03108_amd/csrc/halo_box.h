// Box tasks as a workgroup carries them out: element types, addresses, and the forward copy, which other launches may carry too.
#pragma once
#include "common.h"

namespace distdl {

constexpr int kThreads = 256;
constexpr int kUnroll = 4;

// ---- element helpers --------------------------------------------------------
__device__ inline float bf16_to_f32(uint32_t h) { return __uint_as_float(h << 16); }
__device__ inline uint32_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;  // quiet NaN
  u += 0x7fffu + ((u >> 16) & 1u);                                // round to nearest even
  return u >> 16;
}

struct F32x4 {
  using Store = float4;
  static constexpr int N = 4;
  __device__ static void unpack(const Store& s, float* a) { a[0] = s.x; a[1] = s.y; a[2] = s.z; a[3] = s.w; }
  __device__ static Store pack(const float* a) { return make_float4(a[0], a[1], a[2], a[3]); }
  __device__ static Store zero() { return make_float4(0.f, 0.f, 0.f, 0.f); }
};
struct F32x1 {
  using Store = float;
  static constexpr int N = 1;
  __device__ static void unpack(const Store& s, float* a) { a[0] = s; }
  __device__ static Store pack(const float* a) { return a[0]; }
  __device__ static Store zero() { return 0.f; }
};
struct BF16x8 {
  using Store = uint4;
  static constexpr int N = 8;
  __device__ static void unpack(const Store& s, float* a) {
    const uint32_t w[4] = {s.x, s.y, s.z, s.w};
    for (int i = 0; i < 4; ++i) {
      a[2 * i] = bf16_to_f32(w[i] & 0xffffu);
      a[2 * i + 1] = bf16_to_f32(w[i] >> 16);
    }
  }
  __device__ static Store pack(const float* a) {
    uint32_t w[4];
    for (int i = 0; i < 4; ++i) w[i] = f32_to_bf16(a[2 * i]) | (f32_to_bf16(a[2 * i + 1]) << 16);
    return make_uint4(w[0], w[1], w[2], w[3]);
  }
  __device__ static Store zero() { return make_uint4(0, 0, 0, 0); }
};
struct BF16x1 {
  using Store = uint16_t;
  static constexpr int N = 1;
  __device__ static void unpack(const Store& s, float* a) { a[0] = bf16_to_f32(s); }
  __device__ static Store pack(const float* a) { return (uint16_t)f32_to_bf16(a[0]); }
  __device__ static Store zero() { return 0; }
};

// Every halo, padding and band cell is touched once per call, so loads carry the
// non-temporal hint.  Stores: the ones that carry data (halo copies, band sums)
// are plain, the zero fills (padding cells, cleared halo cells) non-temporal.
// Measured on the 64-worker volumetric geometry, that mix runs the forward
// kernel at 6.3 TB/s and the adjoint at 6.0 TB/s; with every store non-temporal
// both stay at 4.9-5.0 TB/s, with every store plain at 5.4 / 4.7 TB/s, and the
// opposite mix is as fast only when a plan has padding to clear.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// The buffers are device allocations: the address-space cast makes these
// global_load / global_store instead of flat accesses.
#define DISTDL_GLOBAL __attribute__((address_space(1)))
template <class S>
__device__ inline S nt_load(const S* p) {
  if constexpr (sizeof(S) == 16) {
    u32x4 v = __builtin_nontemporal_load((const DISTDL_GLOBAL u32x4*)p);
    S out;
    __builtin_memcpy(&out, &v, 16);
    return out;
  } else {
    return __builtin_nontemporal_load((const DISTDL_GLOBAL S*)p);
  }
}
template <class S>
__device__ inline void plain_store(S* p, const S& val) {
  if constexpr (sizeof(S) == 16) {
    u32x4 v;
    __builtin_memcpy(&v, &val, 16);
    *(DISTDL_GLOBAL u32x4*)p = v;
  } else {
    *(DISTDL_GLOBAL S*)p = val;
  }
}
template <class S>
__device__ inline void nt_store(S* p, const S& val) {
  if constexpr (sizeof(S) == 16) {
    u32x4 v;
    __builtin_memcpy(&v, &val, 16);
    __builtin_nontemporal_store(v, (DISTDL_GLOBAL u32x4*)p);
  } else {
    __builtin_nontemporal_store(val, (DISTDL_GLOBAL S*)p);
  }
}

struct UnitPos {
  uint32_t n, c0, c1, col;
};
__device__ inline UnitPos decode(uint32_t u, const HaloTaskDev& t) {
  UnitPos p;
  uint32_t row = fd_div(u, t.div_row);
  p.col = u - row * t.div_row.d;
  uint32_t r1 = fd_div(row, t.div_e1);
  p.c1 = row - r1 * t.div_e1.d;
  p.n = fd_div(r1, t.div_e0);
  p.c0 = r1 - p.n * t.div_e0.d;
  return p;
}
__device__ inline size_t view_offset(const HaloView& v, const UnitPos& p) {
  return v.base + p.n * v.sn + (size_t)(p.c0 * v.s0 + p.c1 * v.s1 + p.col);
}

// Forward: copy boxes (nsrc == 1) and zero boxes (nsrc == 0).  A thread
// handles kUnroll units: all loads are issued before the first store.
template <class E>
__device__ __forceinline__ void halo_fwd_box(const BlockRef* __restrict__ blocks, const HaloTaskDev* __restrict__ tasks,
                                             void* const* __restrict__ bufs, int block) {
  using S = typename E::Store;
  const BlockRef br = blocks[block];
  const HaloTaskDev t = tasks[br.task];  // by value: the record is read once into scalar registers
  const uint32_t total = t.total;
  S* __restrict__ dst = (S*)bufs[t.dst.worker];
  if (t.nsrc == 0) {
#pragma unroll
    for (int i = 0; i < kUnroll; ++i) {
      uint32_t u = br.unit0 + threadIdx.x + i * kThreads;
      if (u < total) nt_store(dst + view_offset(t.dst, decode(u, t)), E::zero());
    }
    return;
  }
  const S* __restrict__ src = (const S*)bufs[t.src0.worker];
  S vals[kUnroll];
  size_t doff[kUnroll];
  bool live[kUnroll];
#pragma unroll
  for (int i = 0; i < kUnroll; ++i) {
    uint32_t u = br.unit0 + threadIdx.x + i * kThreads;
    live[i] = u < total;
    UnitPos p = decode(live[i] ? u : total - 1, t);  // clamped: loads need no branch
    doff[i] = view_offset(t.dst, p);
    vals[i] = nt_load(src + view_offset(t.src0, p));
  }
#pragma unroll
  for (int i = 0; i < kUnroll; ++i)
    if (live[i]) plain_store(dst + doff[i], vals[i]);
}

}  // namespace distdl
