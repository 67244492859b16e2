// Device helpers shared by the complex64 and complex-half kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "desc.h"

namespace matnc {

// Workspace addresses are plain integers; a pointer made from one carries no
// address space, and the compiler then emits FLAT accesses, which also count
// on the LDS wait counter (every LDS wait would drain the outstanding global
// loads as well).  Every access to the workspace goes through a global
// (address space 1) pointer instead.
template <typename T>
using gptr = __attribute__((address_space(1))) T*;

template <typename T>
__device__ __forceinline__ gptr<T> gmem(uint64_t a) {
  return (gptr<T>)a;
}

// Offset tables are written when a plan is bound and only read by the
// kernels.  A lookup at a wave-uniform index (a k step) through a constant
// (address space 4) pointer compiles to scalar loads, which count on the
// LDS/scalar wait counter: waiting for its result inside a k loop then does
// not also wait for the operand loads in flight, which complete in order on
// the vector-memory counter.
template <typename T>
using cptr = __attribute__((address_space(4))) T*;

template <typename T>
__device__ __forceinline__ cptr<T> cmem(uint64_t a) {
  return (cptr<T>)a;
}

typedef float floatx16 __attribute__((ext_vector_type(16)));  // MFMA accumulator

// element accessors (HIP's float2 / __half2 classes cannot be copied
// through an address-space-qualified reference; plain vectors can)
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float2 ldg_f2(uint64_t base, uint64_t i) {
  const f32x2 v = gmem<const f32x2>(base)[i];
  return make_float2(v.x, v.y);
}
__device__ __forceinline__ void stg_f2(uint64_t base, uint64_t i, float2 v) { gmem<f32x2>(base)[i] = f32x2{v.x, v.y}; }
__device__ __forceinline__ uint32_t ldg_u32(uint64_t base, uint64_t i) { return gmem<const uint32_t>(base)[i]; }
__device__ __forceinline__ void stg_u32(uint64_t base, uint64_t i, uint32_t v) { gmem<uint32_t>(base)[i] = v; }
__device__ __forceinline__ HalfScale ldg_scale(uint64_t base, int64_t i) {
  const u32x2 v = gmem<const u32x2>(base)[i];
  HalfScale h;
  h.e = (int32_t)v.x;
  h.mx = v.y;
  return h;
}
// exponent word of scale slot i, and an atomic max into its maximum word
__device__ __forceinline__ void stg_scale_e(uint64_t base, int64_t i, int32_t e) {
  gmem<int32_t>(base + (uint64_t)i * sizeof(HalfScale))[0] = e;
}
// The slot was cleared before the launch and only grows while it runs, so a
// value read from it is never above the final maximum: when it already holds
// at least mx_bits the atomic is skipped.  An instance spread over many tiles
// or blocks (a stem tensor) would otherwise send every one of them to the
// same address.
__device__ __forceinline__ void max_scale_mx(uint64_t base, int64_t i, uint32_t mx_bits) {
  uint32_t* p = (uint32_t*)(base + (uint64_t)i * sizeof(HalfScale) + offsetof(HalfScale, mx));
  if (__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < mx_bits) atomicMax(p, mx_bits);
}

// Workgroups are dispatched round-robin over the 8 XCDs, each with its own
// L2.  A grid-stride index vid (grid size a multiple of 8, or a single
// pass) maps to a logical tile so that XCD x works through the contiguous
// logical range [start(x), start(x) + count(x)): neighbouring tiles, which
// share operand data, then meet in the same L2.  A bijection on [0, total).
__device__ __forceinline__ uint32_t xcd_tile(uint32_t vid, uint32_t total) {
  const uint32_t q = total >> 3, r = total & 7;
  const uint32_t x = vid & 7, k = vid >> 3;
  return x * q + (x < r ? x : r) + k;
}

// Logical (unit, tile) of a logical tile index.  Units (output instances,
// or fan-table rows) are taken in blocks of R; inside a block the tile
// index is outermost, so that the R tiles at one position of the R units
// run next to each other on one XCD.  Units that read the same A instance
// are adjacent (fan tables are grouped by A instance, plain instances are
// in key order), so the later reads of each A tile hit the L2.  R = 1
// (plain steps) is the unit-major order; fan-out steps, whose A instances
// are shared by about two rows, take R = 2; a unit group sharing an A
// instance far larger than the caches takes R = its size, so that the
// instance streams from HBM once while the group's B instances are re-read
// from the caches.  A bijection on [0, units * tiles) for any R >= 1 (a
// short last block keeps the same order over its units).  All counts fit in
// 32 bits (a tile writes at least 64 elements of 4 bytes, so 2^31 of them
// would not fit the card's memory) and tiles = 2^tbits: 64-bit divisions here
// cost a few hundred cycles per tile, as much as two k steps.
__device__ __forceinline__ void unit_tile(uint32_t lt, uint32_t units, int tbits, uint32_t R, uint32_t& u,
                                          uint32_t& t) {
  if (R == 1) {
    u = lt >> tbits;
    t = lt & ((1u << tbits) - 1u);
    return;
  }
  const uint32_t blk = (lt >> tbits) / R;
  const uint32_t r = lt - ((blk * R) << tbits);
  const uint32_t rows = units - blk * R < R ? units - blk * R : R;  // units in this block
  t = r / rows;
  u = blk * R + (r - t * rows);
}

template <typename P>
__device__ __forceinline__ uint32_t tlook(P T, uint32_t x) {
  return T[x & 255u] + T[256 + ((x >> 8) & 255u)] + T[512 + ((x >> 16) & 255u)] + T[768 + (x >> 24)];
}

// offset of coordinate v (< 2^nbits) of class CLS, from the bit positions in
// the descriptor; positions of bits that v does not have are not used
template <int CLS>
__device__ __forceinline__ uint32_t dep(const NodeDesc& d, int nbits, uint32_t v) {
  uint32_t off = 0;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    if (4 * q < nbits) {
      uint32_t w;
      __builtin_memcpy(&w, &d.pos[CLS][4 * q], 4);
#pragma unroll
      for (int b = 0; b < 4; ++b) off |= ((v >> (4 * q + b)) & 1u) << ((w >> (8 * b)) & 31u);
    }
  }
  return off;
}

// ... of the coordinate whose bits 4q .. 4q + 3 are e and the rest zero
template <int CLS>
__device__ __forceinline__ uint32_t dep_nibble(const NodeDesc& d, int q, uint32_t e) {
  uint32_t w, off = 0;
  __builtin_memcpy(&w, &d.pos[CLS][4 * q], 4);
#pragma unroll
  for (int b = 0; b < 4; ++b) off |= ((e >> b) & 1u) << ((w >> (8 * b)) & 31u);
  return off;
}

template <int C>
struct Class {
  static constexpr int value = C;
};

template <typename P>
__device__ __forceinline__ int64_t operand_instance(const OpDesc& o, P gmap, int64_t j, int64_t s, int64_t sigma) {
  int64_t v = (int64_t)gmap[j] * o.nsv;
  for (int t = 0; t < o.nsb; ++t) v += ((sigma >> o.sbit[t]) & 1) << t;
  if (o.dep) v += s * (int64_t)o.w_child;
  return v;
}

__device__ __forceinline__ void cmac(float2& c, float2 a, float2 b) {
  c.x = fmaf(a.x, b.x, c.x);
  c.x = fmaf(-a.y, b.y, c.x);
  c.y = fmaf(a.x, b.y, c.y);
  c.y = fmaf(a.y, b.x, c.y);
}


// grid size for grid-stride loops
static inline unsigned grid_for(int64_t blocks) {
  const int64_t cap = 256 * 1024;
  return (unsigned)(blocks < 1 ? 1 : (blocks > cap ? cap : blocks));
}

}  // namespace matnc
