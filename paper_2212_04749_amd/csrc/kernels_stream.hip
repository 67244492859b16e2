// Streaming (VALU) kernels of one pairwise step C[m, n] = sum_k A[m, k] B[k, n],
// for both storage precisions.  These steps move more bytes than they
// compute (a big tensor times a gate-sized one, or a batched matrix-vector
// product), so the kernels are built for HBM bandwidth:
//
//  * k_wide<FL, KB, R>     small K (<= 16): every lane owns R values of m
//    spaced 256 apart (R x KB loads in flight) and up to 16 columns, whose B
//    is staged once per block in LDS.  A block covers 256*R consecutive m of
//    one instance, so instance decoding and B are block-uniform.
//  * k_narrow<FL, KB>      the same for instances smaller than 256 elements:
//    one lane per (instance, column group, m).
//  * k_kred<FL, NB>        large K: lanes own m (coalesced reads of A along
//    its low bits), groups of lanes split K, partial sums meet in LDS; B in LDS.
//  * k_kdir<FL, NB>        the same with B read where it lies.
//  * k_kdot<FL, NB>        large K, few outputs: one wave per instance.
//
// Bound: bytes, of small steps the launch.  Whole calls of a single contraction
// (m/n/k bits x instances) with an offset table read per access, uploaded for
// each call, one block per 256 m, and now: 22/2/2, 268 MB, 73 -> 53 us (5.07
// TB/s, a copy's rate); 10/1/11 x 33, 555 MB, 332 -> 108 us (it had 132 blocks, one
// chain of loads per lane); 4/12/5 x 9, 14 MB, 76 -> 16 us (it ran a lane per output
// with m, n as given; the wider side is M now); 5/3/2 x 7 40 -> 11 us.
//
// Offsets come from the bit positions in the descriptor (dep): no table is
// read, so that a first touch of one does not delay the operand loads, and a
// single contraction needs no table built before it.
//
// Precision policy P: C64 plans store float2 everywhere.  MIX (complex-half
// plans) stores each tensor as __half2 with a per-instance exponent e
// (value = half * 2^e) or as float2 (e = 0), as the plan decided; every
// stored instance also carries its measured maximum mx.  A FP16 output's
// exponent is chosen from the operands' maxima so that |Re|, |Im| of every
// output (bounded by 2^(kbits+1) mx_A mx_B 2^(e_A+e_B)) is stored below
// 2^15 (no FP16 overflow); the maximum of the stored output is measured
// (block reduction + unsigned atomicMax on the float bits, exact because
// all values are non-negative) for the next step.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "desc.h"
#include "device_common.h"
#include "kernels.h"

namespace matnc {

// Storage flags FL (compile-time): bit 3 = complex-half plan (scales
// tracked); bit 0 / 1 / 2 = A / B / C stored as FP16 (else FP32).
constexpr int kMixBit = 8;

// lanes that fill the chip, 256 CUs x 512; with twice as many a lane's A serves
// fewer columns (7/3/3 bits x 500 11.4 -> 8.2 us)
constexpr int64_t kNarrowLanes = 256 * 512;
// blocks that keep HBM busy in a long sum
constexpr int64_t kKredBlocks = 1024;
// persistent blocks of the long-sum kernels: 8 per CU, so that the offsets in
// LDS are set up once for several instances
constexpr int64_t kBlocks = 2048;
// one wave per instance fills the chip from four waves per CU up
constexpr int64_t kDotInstances = 1024;

template <int FL, int WHICH>
__device__ __forceinline__ float2 ldop(uint64_t base, uint32_t i) {
  if constexpr ((FL & kMixBit) && (FL & WHICH)) {
    const uint32_t u = ldg_u32(base, i);
    __half2 h;
    __builtin_memcpy(&h, &u, 4);
    return __half22float2(h);
  }
  return ldg_f2(base, i);
}

// Output scale of one instance; identity for complex64 plans.
struct OutScale {
  float f;       // multiply the FP32 result by f before storing
  int32_t e;     // exponent recorded for the output instance
};

template <int FL>
__device__ __forceinline__ OutScale out_scale(const NodeDesc& d, uint64_t ws, int64_t ai, int64_t bi) {
  OutScale o{1.f, 0};
  if constexpr ((FL & kMixBit) != 0) {
    const HalfScale sa = ldg_scale(ws + d.A.scale_off, ai);
    const HalfScale sb = ldg_scale(ws + d.B.scale_off, bi);
    if constexpr ((FL & 4) != 0) {
      const float bound = ldexpf(__uint_as_float(sa.mx) * __uint_as_float(sb.mx), d.kbits + 1);
      int ex = 0;
      if (bound > 0.f) frexpf(bound, &ex);  // bound < 2^ex
      o.e = sa.e + sb.e + ex - 15;
      o.f = ldexpf(1.f, 15 - ex);
    } else {
      o.e = 0;
      o.f = ldexpf(1.f, sa.e + sb.e);
    }
  }
  return o;
}

// store one output element; returns the largest stored |component|
template <int FL>
__device__ __forceinline__ float put(uint64_t base, uint32_t i, float2 c, const OutScale& s) {
  if constexpr ((FL & kMixBit) != 0) {
    const float2 v = make_float2(c.x * s.f, c.y * s.f);
    if constexpr ((FL & 4) != 0) {
      const __half2 h = __float22half2_rn(v);
      uint32_t u;
      __builtin_memcpy(&u, &h, 4);
      stg_u32(base, i, u);
      const float2 back = __half22float2(h);
      return fmaxf(fabsf(back.x), fabsf(back.y));
    }
    stg_f2(base, i, v);
    return fmaxf(fabsf(v.x), fabsf(v.y));
  } else {
    stg_f2(base, i, c);
    return 0.f;
  }
}

template <int FL>
__device__ __forceinline__ void record_scale(const NodeDesc& d, uint64_t ws, int64_t inst, const OutScale& s,
                                             float mx, bool writer) {
  if constexpr ((FL & kMixBit) != 0) {
    if (writer) stg_scale_e(ws + d.c_scale_off, inst, s.e);
    if (mx > 0.f) max_scale_mx(ws + d.c_scale_off, inst, __float_as_uint(mx));
  }
}

// max over the 64 lanes of a wave
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}

// max over lanes whose index agrees above bit log2(seg) (seg <= 64)
__device__ __forceinline__ float segment_max(float v, int seg) {
  for (int o = seg >> 1; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}

// record the output maximum: at most one atomic per wave, no block barrier;
// the exponent (the same for every block of the instance) is written by the
// first wave of the block that covers the instance's first elements
template <int FL>
__device__ __forceinline__ void block_record(const NodeDesc& d, uint64_t ws, int64_t inst, const OutScale& s, float mx,
                                             bool first_block) {
  if constexpr ((FL & kMixBit) != 0) {
    mx = wave_max(mx);
    if ((threadIdx.x & 63) == 0) record_scale<FL>(d, ws, inst, s, mx, first_block && threadIdx.x == 0);
  }
}

struct InstPtrs {
  int64_t inst, ai, bi;
  uint64_t pa, pb, pc;
};

__device__ __forceinline__ InstPtrs instance_ptrs(const NodeDesc& d, uint64_t ws, int64_t inst,
                                                  const int64_t* __restrict__ sig) {
  InstPtrs r;
  r.inst = inst;
  if (d.flat) {
    r.ai = r.bi = inst;
  } else {
    const int64_t s = d.dep ? inst / d.w : 0;
    const int64_t j = d.dep ? inst - s * d.w : inst;
    const int64_t sigma = sig[0] + s;
    const gptr<const int32_t> glA = gmem<const int32_t>(ws + d.A.gmap_off);
    const gptr<const int32_t> glB = gmem<const int32_t>(ws + d.B.gmap_off);
    r.ai = operand_instance(d.A, glA, j, s, sigma);
    r.bi = operand_instance(d.B, glB, j, s, sigma);
  }
  r.pa = ws + d.A.off + (uint64_t)r.ai * d.A.inst_bytes;
  r.pb = ws + d.B.off + (uint64_t)r.bi * d.B.inst_bytes;
  r.pc = ws + d.c_off + (uint64_t)inst * d.c_inst_bytes;
  return r;
}

// ---------------------------------------------------------------------------

// Columns are taken 16 at a time (a runtime bound below that); the blocks of
// one m range's column groups are neighbours, so A is read from HBM once.
template <int FL, int KB, int R>
__global__ __launch_bounds__(256) void k_wide(NodeDesc d, uint64_t ws, const int64_t* __restrict__ sig) {
  constexpr int LR = (R == 1) ? 0 : (R == 2) ? 1 : (R == 4) ? 2 : 3;
  __shared__ float2 Bs[KB * 16];
  __shared__ uint32_t cns[16];
  const int tid = threadIdx.x;
  const int nb = d.nbits < 4 ? d.nbits : 4;
  const int NB = 1 << nb;
  const int ng = d.nbits - nb;  // column groups = 2^ng
  const uint32_t oa_lo = dep<TAB_AM>(d, 8, tid), oc_lo = dep<TAB_CM>(d, 8, tid);
  uint32_t tak[KB];
#pragma unroll
  for (int k = 0; k < KB; ++k) tak[k] = dep<TAB_AK>(d, 4, k);
  // this lane's B element when staging (KB * NB <= 256)
  const uint32_t bk_mine = dep<TAB_BK>(d, 4, tid >> nb);
  const int sh = d.mbits - 8 - LR;
  const int64_t nblk = d.n_inst << (sh + ng);
  for (int64_t blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
    const InstPtrs ip = instance_ptrs(d, ws, blk >> (sh + ng), sig);
    const uint32_t n0 = ((uint32_t)blk & ((1u << ng) - 1u)) << nb;
    const uint32_t hi0 = ((uint32_t)(blk >> ng) & ((1u << sh) - 1u)) << LR;
    if (tid < KB * NB) Bs[tid] = ldop<FL, 2>(ip.pb, bk_mine + dep<TAB_BN>(d, d.nbits, n0 + (tid & (NB - 1))));
    if (tid < NB) cns[tid] = dep<TAB_CN>(d, d.nbits, n0 + tid);
    uint32_t oa[R], oc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      oa[r] = oa_lo + dep<TAB_AM>(d, d.mbits, (hi0 + r) << 8);
      oc[r] = oc_lo + dep<TAB_CM>(d, d.mbits, (hi0 + r) << 8);
    }
    float2 a[R][KB];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int k = 0; k < KB; ++k) a[r][k] = ldop<FL, 1>(ip.pa, oa[r] + tak[k]);
    const OutScale s = out_scale<FL>(d, ws, ip.ai, ip.bi);
    __syncthreads();
    float mx = 0.f;
    for (int n = 0; n < NB; ++n) {
      const uint32_t cn = cns[n];
      float2 b[KB];
#pragma unroll
      for (int k = 0; k < KB; ++k) b[k] = Bs[k * NB + n];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        float2 c = make_float2(0.f, 0.f);
#pragma unroll
        for (int k = 0; k < KB; ++k) cmac(c, a[r][k], b[k]);
        mx = fmaxf(mx, put<FL>(ip.pc, oc[r] + cn, c, s));
      }
    }
    block_record<FL>(d, ws, ip.inst, s, mx, hi0 == 0 && n0 == 0);
    __syncthreads();  // Bs is rewritten next iteration
  }
}

// npl: columns per lane (a power of two).  One where the step is so small
// that lanes are idle otherwise, all of them where that fills the chip (A is
// then read once per lane).
template <int FL, int KB>
__global__ __launch_bounds__(256) void k_narrow(NodeDesc d, uint64_t ws, const int64_t* __restrict__ sig, int nplbits) {
  const int NPL = 1 << nplbits;
  uint32_t tak[KB], tbk[KB];
#pragma unroll
  for (int k = 0; k < KB; ++k) {
    tak[k] = dep<TAB_AK>(d, 4, k);
    tbk[k] = dep<TAB_BK>(d, 4, k);
  }
  const int gb = d.mbits + d.nbits - nplbits;  // lanes per instance = 2^gb
  const int64_t total = d.n_inst << gb;
  const uint32_t mmask = (1u << d.mbits) - 1u, gmask = (1u << gb) - 1u;
  const int seg = gb >= 6 ? 64 : (1 << gb);
  // A lane keeps its m: its turns are a multiple of 256 apart, and where an
  // instance has more than 256 there is one turn only.  (With 16 k the two
  // offsets that are kept cost 7%.)
  constexpr bool kKept = KB < 16;
  const uint32_t m0 = (blockIdx.x * 256 + threadIdx.x) & mmask;
  const uint32_t oa0 = kKept ? dep<TAB_AM>(d, d.mbits, m0) : 0, oc0 = kKept ? dep<TAB_CM>(d, d.mbits, m0) : 0;
  for (int64_t base = (int64_t)blockIdx.x * 256; base < total; base += (int64_t)gridDim.x * 256) {
    const int64_t g = base + threadIdx.x;
    const bool live = g < total;
    float mx = 0.f;
    OutScale s{1.f, 0};
    int64_t inst = 0;
    if (live) {
      inst = g >> gb;
      const uint32_t m = (uint32_t)g & mmask;
      const uint32_t n0 = (((uint32_t)g & gmask) >> d.mbits) << nplbits;
      const InstPtrs ip = instance_ptrs(d, ws, inst, sig);
      const uint32_t oa = kKept ? oa0 : dep<TAB_AM>(d, d.mbits, m);
      const uint32_t oc = kKept ? oc0 : dep<TAB_CM>(d, d.mbits, m);
      float2 a[KB];
#pragma unroll
      for (int k = 0; k < KB; ++k) a[k] = ldop<FL, 1>(ip.pa, oa + tak[k]);
      s = out_scale<FL>(d, ws, ip.ai, ip.bi);
      auto column = [&](uint32_t n) {
        const uint32_t bn = dep<TAB_BN>(d, d.nbits, n);
        float2 c = make_float2(0.f, 0.f);
#pragma unroll
        for (int k = 0; k < KB; ++k) cmac(c, a[k], ldop<FL, 2>(ip.pb, bn + tbk[k]));
        mx = fmaxf(mx, put<FL>(ip.pc, oc + dep<TAB_CN>(d, d.nbits, n), c, s));
      };
      if (nplbits == d.nbits) {  // (all columns: their offsets are scalars)
        for (int n = 0; n < NPL; ++n) column(n);
      } else {
        for (int n = 0; n < NPL; ++n) column(n0 + n);
      }
    }
    if constexpr ((FL & kMixBit) != 0) {
      // lanes of one instance are contiguous; reduce within segments of a wave
      mx = segment_max(mx, seg);
      const int lane = threadIdx.x & 63;
      if (live && (lane & (seg - 1)) == 0) record_scale<FL>(d, ws, inst, s, mx, ((uint32_t)g & gmask) == 0);
    }
  }
}

// sum of part[g * stride + o] over g < groups (a power of two): in that order, or
// sixteen at a time in a tree, whose error does not grow with their number (1/0/11
// bits x 223: 3.1e-7 from 64 bits one by one, 1.2e-7).  Sixteen reads are in
// flight together (one at a time, 255 of them took 7 us)
__device__ __forceinline__ float2 add_groups(const float2* part, int o, int stride, int groups, bool in_order) {
  if (!in_order && groups >= 16) {
    float2 c = make_float2(0.f, 0.f);
    for (int g = 0; g < groups; g += 16) {
      float2 v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = part[(g + u) * stride + o];
#pragma unroll
      for (int h = 8; h > 0; h >>= 1)
#pragma unroll
        for (int u = 0; u < h; ++u) {
          v[u].x += v[u + h].x;
          v[u].y += v[u + h].y;
        }
      c.x += v[0].x;
      c.y += v[0].y;
    }
    return c;
  }
  float2 c = part[o];
  int g = 1;
  for (; g + 15 < groups; g += 16) {
    float2 v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = part[(g + u) * stride + o];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      c.x += v[u].x;
      c.y += v[u].y;
    }
  }
  for (; g < groups; ++g) {
    c.x += part[g * stride + o].x;
    c.y += part[g * stride + o].y;
  }
  return c;
}

// Large K: a block takes 2^mb values of m of one instance and NB of its
// columns; 2^ks_bits groups of lanes take every 2^ks_bits-th k each, and their
// partial sums are added up (add_groups).  B goes through LDS, 256 k at a time.
template <int FL, int NB>
__global__ __launch_bounds__(256) void k_kred(NodeDesc d, uint64_t ws, const int64_t* __restrict__ sig) {
  __shared__ uint32_t kofa[256], kofb[256];
  __shared__ float2 sb[256 * NB];  // B's chunk, then the partial sums
  const int tid = threadIdx.x;
  const int ksb = d.ks_bits;
  const int mb = d.mbits < 8 - ksb ? d.mbits : 8 - ksb;
  const int M = 1 << mb;
  const int KS = 1 << ksb;
  const int mloc = tid & (M - 1);
  const int grp = tid >> mb;           // >= KS: an idle lane
  const bool live = grp < KS;
  const int mch = d.mbits - mb;        // m chunks per instance = 2^mch
  const int nch = d.nbits - __builtin_ctz(NB);
  const int64_t nblk = d.n_inst << (mch + nch);
  const uint32_t kcount = 1u << d.kbits;
  const int klb = d.kbits < 8 ? d.kbits : 8;
  const uint32_t klo_n = 1u << klb;
  kofa[tid] = dep<TAB_AK>(d, klb, tid & (klo_n - 1));
  kofb[tid] = dep<TAB_BK>(d, klb, tid & (klo_n - 1));
  __syncthreads();
  for (int64_t blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
    const InstPtrs ip = instance_ptrs(d, ws, blk >> (mch + nch), sig);
    const uint32_t n0 = ((uint32_t)blk & ((1u << nch) - 1u)) * NB;
    const uint32_t chunk = (uint32_t)(blk >> nch) & ((1u << mch) - 1u);
    const uint32_t m = (chunk << mb) + mloc;
    const uint64_t pa = ip.pa, pb = ip.pb;
    const uint32_t om = dep<TAB_AM>(d, d.mbits, m);
    float2 acc[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[n] = make_float2(0.f, 0.f);
    for (uint32_t kh = 0; kh < kcount; kh += klo_n) {
      const uint32_t bb = dep<TAB_BK>(d, d.kbits, kh);
      __syncthreads();  // the last chunk (or the partial sums) has been read
      const uint32_t on = dep<TAB_BN>(d, d.nbits, n0 + tid % NB);
      for (uint32_t e = tid; e < klo_n * NB; e += 256) sb[e] = ldop<FL, 2>(pb, bb + kofb[e / NB] + on);
      __syncthreads();
      if (!live) continue;
      const uint32_t ba = om + dep<TAB_AK>(d, d.kbits, kh);
      uint32_t kl = grp;
      for (; kl + 7 * KS < klo_n; kl += 8 * KS) {
        float2 a[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] = ldop<FL, 1>(pa, ba + kofa[kl + u * KS]);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
#pragma unroll
          for (int n = 0; n < NB; ++n) cmac(acc[n], a[u], sb[(kl + u * KS) * NB + n]);
        }
      }
      for (; kl < klo_n; kl += KS) {
        const float2 a = ldop<FL, 1>(pa, ba + kofa[kl]);
#pragma unroll
        for (int n = 0; n < NB; ++n) cmac(acc[n], a, sb[kl * NB + n]);
      }
    }
    const OutScale s = out_scale<FL>(d, ws, ip.ai, ip.bi);
    float mx = 0.f;
    if (KS > 1) {
      __syncthreads();
      if (live) {
#pragma unroll
        for (int n = 0; n < NB; ++n) sb[tid * NB + n] = acc[n];
      }
      __syncthreads();
      const int out = M * NB;
      for (int o = tid; o < out; o += 256) {
        const float2 c = add_groups(sb, o, out, KS, d.keep_order != 0);
        const uint32_t mo = (chunk << mb) + o / NB, no = n0 + o % NB;
        mx = fmaxf(mx, put<FL>(ip.pc, dep<TAB_CM>(d, d.mbits, mo) + dep<TAB_CN>(d, d.nbits, no), c, s));
      }
    } else if (live) {
      const uint32_t oc = dep<TAB_CM>(d, d.mbits, m);
#pragma unroll
      for (int n = 0; n < NB; ++n) mx = fmaxf(mx, put<FL>(ip.pc, oc + dep<TAB_CN>(d, d.nbits, n0 + n), acc[n], s));
    }
    block_record<FL>(d, ws, ip.inst, s, mx, chunk == 0 && n0 == 0);
  }
}

// k of a lane in flight in k_kdir and k_kdot.  With more, the loads of a k's
// columns take so many registers that fewer waves hide them: eight instead of
// four or two cost 5-17%.
constexpr int k_in_flight(int columns) { return columns <= 2 ? 4 : 2; }

// How the offset of k changes where the bits from `shift` on are counted up by
// one and t of them carry: lane t holds it.  (A deposit of every k, though of
// scalars, took longer than its loads: 3/0/13 bits x 1 65 us instead of 25.)
template <int CLS>
__device__ __forceinline__ uint32_t k_carry(const NodeDesc& d, int shift) {
  const int t = threadIdx.x & 63;
  const uint32_t bits = t + shift < 31 ? ((2u << t) - 1u) << shift : 0u;
  return dep<CLS>(d, d.kbits, bits);
}

// The same sums (groups and order) with B read where it lies: a block takes 2^mb
// values of m of one instance, all of its NB columns.  Where the order is free, lanes of a
// wave that share an output meet in a tree of lane exchanges, and only the
// waves' sums go through LDS.
template <int FL, int NB>
__global__ __launch_bounds__(256) void k_kdir(NodeDesc d, uint64_t ws, const int64_t* __restrict__ sig) {
  constexpr int U = k_in_flight(NB), LU = U == 4 ? 2 : 1;
  __shared__ float2 sb[256 * NB];
  const int tid = threadIdx.x;
  const int ksb = d.ks_bits, KS = 1 << ksb;
  const int mb = d.mbits < 8 - ksb ? d.mbits : 8 - ksb;
  const int M = 1 << mb;
  const int mch = d.mbits - mb;  // m chunks per instance = 2^mch
  const uint32_t mloc = tid & (M - 1), grp = tid >> mb;  // grp >= KS: an idle lane
  const uint32_t kcount = 1u << d.kbits, runs = kcount >> (ksb + LU);
  const uint32_t oa = dep<TAB_AM>(d, 8, mloc) + dep<TAB_AK>(d, 12, grp & (KS - 1));
  const uint32_t ob = dep<TAB_BK>(d, 12, grp & (KS - 1));
  uint32_t tbn[NB], ta[U], tb[U];
#pragma unroll
  for (int n = 0; n < NB; ++n) tbn[n] = dep<TAB_BN>(d, 3, n);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    ta[u] = dep<TAB_AK>(d, d.kbits, (uint32_t)u << ksb);
    tb[u] = dep<TAB_BK>(d, d.kbits, (uint32_t)u << ksb);
  }
  const uint32_t da = k_carry<TAB_AK>(d, ksb + LU), db = k_carry<TAB_BK>(d, ksb + LU);
  const bool tree = d.keep_order == 0;
  const int64_t nblk = d.n_inst << mch;
  for (int64_t blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
    const InstPtrs ip = instance_ptrs(d, ws, blk >> mch, sig);
    const uint32_t m0 = ((uint32_t)blk & ((1u << mch) - 1u)) << mb;
    const uint32_t om = oa + dep<TAB_AM>(d, d.mbits, m0);
    float2 acc[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[n] = make_float2(0.f, 0.f);
    if (grp < (uint32_t)KS) {
      if (runs > 0) {
        uint32_t ha = 0, hb = 0;
        for (uint32_t r = 1;; ++r) {
          float2 a[U];
#pragma unroll
          for (int u = 0; u < U; ++u) a[u] = ldop<FL, 1>(ip.pa, om + (ha + ta[u]));
#pragma unroll
          for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int n = 0; n < NB; ++n) cmac(acc[n], a[u], ldop<FL, 2>(ip.pb, ob + (hb + tb[u] + tbn[n])));
          }
          if (r == runs) break;
          ha ^= __builtin_amdgcn_readlane(da, __builtin_ctz(r));
          hb ^= __builtin_amdgcn_readlane(db, __builtin_ctz(r));
        }
      } else {  // fewer to a lane, also in flight together
        float2 a[U / 2];
#pragma unroll
        for (int u = 0; u < U / 2; ++u)
          if (((uint32_t)u << ksb) < kcount) a[u] = ldop<FL, 1>(ip.pa, om + ta[u]);
#pragma unroll
        for (int u = 0; u < U / 2; ++u)
          if (((uint32_t)u << ksb) < kcount) {
#pragma unroll
            for (int n = 0; n < NB; ++n) cmac(acc[n], a[u], ldop<FL, 2>(ip.pb, ob + tb[u] + tbn[n]));
          }
      }
    }
    const OutScale s = out_scale<FL>(d, ws, ip.ai, ip.bi);
    float mx = 0.f;
    if (mb == 8) {
      const uint32_t oc = dep<TAB_CM>(d, d.mbits, m0 + mloc);
#pragma unroll
      for (int n = 0; n < NB; ++n) mx = fmaxf(mx, put<FL>(ip.pc, oc + dep<TAB_CN>(d, 3, n), acc[n], s));
      block_record<FL>(d, ws, ip.inst, s, mx, m0 == 0);
      continue;
    }
    int groups = KS;
    if (tree && M < 64) {
      for (int o = M; o < 64; o <<= 1) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
          acc[n].x += __shfl_xor(acc[n].x, o);
          acc[n].y += __shfl_xor(acc[n].y, o);
        }
      }
      groups = 4;
      const int lane = tid & 63;
      if (lane < M) {
#pragma unroll
        for (int n = 0; n < NB; ++n) sb[((tid >> 6) * M + lane) * NB + n] = acc[n];
      }
    } else {
#pragma unroll
      for (int n = 0; n < NB; ++n) sb[tid * NB + n] = acc[n];
    }
    __syncthreads();
    for (int o = tid; o < M * NB; o += 256) {
      const uint32_t oc = dep<TAB_CM>(d, d.mbits, m0 + (uint32_t)o / NB) + dep<TAB_CN>(d, 3, (uint32_t)o % NB);
      mx = fmaxf(mx, put<FL>(ip.pc, oc, add_groups(sb, o, M * NB, groups, !tree), s));
    }
    block_record<FL>(d, ws, ip.inst, s, mx, m0 == 0);
    __syncthreads();  // the partial sums are rewritten next iteration
  }
}

// Large K, few outputs (at most 64 m and 8 columns per instance): one wave per
// instance, whose lanes are 2^mbits values of m times 64 / 2^mbits groups that
// take every such k each; the groups' sums meet in a tree of lane exchanges.
// No LDS, no barrier, and four instances per block: a block per instance
// spent its time on its set-up and on adding 256 partial sums one by one.
// A few products at a time are summed on their own: a wave has fewer lanes than
// a block, and one chain of 64 products per lane (3/3/9 bits x 1024) was 2.1e-7
// from 64 bits, where a block's lanes with 16 each gave 1.5e-7.
template <int FL, int NB>
__global__ __launch_bounds__(256) void k_kdot(NodeDesc d, uint64_t ws, const int64_t* __restrict__ sig) {
  constexpr int U = k_in_flight(NB), LU = U == 4 ? 2 : 1;
  const int lane = threadIdx.x & 63;
  const int gb = 6 - d.mbits;
  const uint32_t m = lane & ((1 << d.mbits) - 1);
  const uint32_t grp = lane >> d.mbits;
  const uint32_t KS = 1u << gb, kcount = 1u << d.kbits;
  const uint32_t oa = dep<TAB_AM>(d, 6, m) + dep<TAB_AK>(d, 6, grp);
  const uint32_t ob = dep<TAB_BK>(d, 6, grp);
  uint32_t tbn[NB], ta[U], tb[U];
#pragma unroll
  for (int n = 0; n < NB; ++n) tbn[n] = dep<TAB_BN>(d, 3, n);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    ta[u] = dep<TAB_AK>(d, d.kbits, (uint32_t)u << gb);
    tb[u] = dep<TAB_BK>(d, d.kbits, (uint32_t)u << gb);
  }
  const uint32_t oc = dep<TAB_CM>(d, 6, m);
  const uint32_t da = k_carry<TAB_AK>(d, gb + LU), db = k_carry<TAB_BK>(d, gb + LU);
  const uint32_t runs = kcount >> (gb + LU);
  const int64_t stride = (int64_t)gridDim.x * 4;
  for (int64_t inst = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); inst < d.n_inst;
       inst += stride) {
    const InstPtrs ip = instance_ptrs(d, ws, inst, sig);
    float2 acc[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[n] = make_float2(0.f, 0.f);
    if (runs > 0) {
      uint32_t ha = 0, hb = 0;
      for (uint32_t r = 1;; ++r) {
        float2 a[U], part[NB];
#pragma unroll
        for (int n = 0; n < NB; ++n) part[n] = make_float2(0.f, 0.f);
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = ldop<FL, 1>(ip.pa, oa + (ha + ta[u]));
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
          for (int n = 0; n < NB; ++n) cmac(part[n], a[u], ldop<FL, 2>(ip.pb, ob + (hb + tb[u] + tbn[n])));
        }
#pragma unroll
        for (int n = 0; n < NB; ++n) {
          acc[n].x += part[n].x;
          acc[n].y += part[n].y;
        }
        if (r == runs) break;
        ha ^= __builtin_amdgcn_readlane(da, __builtin_ctz(r));
        hb ^= __builtin_amdgcn_readlane(db, __builtin_ctz(r));
      }
    } else if (grp < kcount) {  // (of fewer than 64 / 2^mbits k some lanes have none)
      float2 a[U / 2];
#pragma unroll
      for (int u = 0; u < U / 2; ++u)
        if (((uint32_t)u << gb) < kcount) a[u] = ldop<FL, 1>(ip.pa, oa + ta[u]);
#pragma unroll
      for (int u = 0; u < U / 2; ++u)
        if (((uint32_t)u << gb) < kcount) {
#pragma unroll
          for (int n = 0; n < NB; ++n) cmac(acc[n], a[u], ldop<FL, 2>(ip.pb, ob + (tb[u] + tbn[n])));
        }
    }
    for (int o = 1 << d.mbits; o < 64; o <<= 1) {
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        acc[n].x += __shfl_xor(acc[n].x, o);
        acc[n].y += __shfl_xor(acc[n].y, o);
      }
    }
    const OutScale s = out_scale<FL>(d, ws, ip.ai, ip.bi);
    float mx = 0.f;
    if (grp == 0) {
#pragma unroll
      for (int n = 0; n < NB; ++n) mx = fmaxf(mx, put<FL>(ip.pc, oc + dep<TAB_CN>(d, 3, n), acc[n], s));
    }
    if constexpr ((FL & kMixBit) != 0) {
      mx = wave_max(mx);
      if (lane == 0) record_scale<FL>(d, ws, inst, s, mx, true);
    }
  }
}

// ---------------------------------------------------------------------------
// dispatch

// Columns share their block's B and A in k_wide; with fewer than a block for
// every fourth CU, or 256 m whose few products do not pay for a barrier, lanes
// with a row or an output each are faster: 10/5/3 bits x 1 (2 blocks) 12.4 -> 5.0
// us, 12/6/0 x 1 (16) 11.6 -> 5.2, 8/0/0 x 5000 18.8 -> 15.7; from 64 blocks on it is
// the other way round (18/2/2 x 1, 14/2/2 x 9, 12/2/2 x 64: by 5% and more).
constexpr int64_t kWideBlocks = 64;

template <int FL, int KB>
static hipError_t launch_small(const NodeDesc& d, uint64_t ws, const int64_t* sig, hipStream_t st) {
  // R m-chunks per lane: as many as the instance allows, up to 4 (2 when
  // K is 16, to bound registers)
  constexpr int RMAX = KB >= 16 ? 1 : 2;
  // Thousands of small instances with few columns: kBlocks blocks take several
  // each, since a block's offsets cost as much as its outputs (8/0/0 bits x 5000
  // 15.9 -> 9.6 us, 8/1/1 19.3 -> 16.7, 10/0/0 21.0 -> 18.3; with offset tables 12.9,
  // 15.4, 18.6).  More work per block wants them all in flight (8/3/3 27.9 -> 31.4,
  // 8/0/4 28.0 -> 30.2, 10/0/1 21.7 -> 23.3).
  auto grid = [](int64_t blocks, bool turns) { return dim3(turns ? (unsigned)std::min(blocks, kBlocks) : grid_for(blocks)); };
  const bool turns = KB < 16 && d.nbits <= 2, turns_r = d.mbits + d.kbits + d.nbits <= 10;
  const int lr = std::min(RMAX, d.mbits - 8);
  const int ng = d.nbits < 4 ? 0 : d.nbits - 4;  // column groups of 16
  const int64_t wide = d.mbits >= 8 ? d.n_inst << (d.mbits - 8 - lr + ng) : 0;
  if (wide >= kWideBlocks && (d.mbits > 8 || d.kbits + 2 * d.nbits > 2)) {
    if (lr == 2)
      hipLaunchKernelGGL((k_wide<FL, KB, KB >= 16 ? 2 : 4>), grid(wide, turns_r), dim3(256), 0, st, d, ws, sig);
    else if (lr == 1)
      hipLaunchKernelGGL((k_wide<FL, KB, 2>), grid(wide, turns_r), dim3(256), 0, st, d, ws, sig);
    else
      hipLaunchKernelGGL((k_wide<FL, KB, 1>), grid(wide, turns), dim3(256), 0, st, d, ws, sig);
  } else {
    // as many columns per lane as still leave kNarrowLanes lanes
    int npl = d.nbits;
    while (npl > 0 && (d.n_inst << (d.mbits + d.nbits - npl)) < kNarrowLanes) --npl;
    const int64_t blocks = ((d.n_inst << (d.mbits + d.nbits - npl)) + 255) / 256;
    hipLaunchKernelGGL((k_narrow<FL, KB>), grid(blocks, turns), dim3(256), 0, st, d, ws, sig, npl);
  }
  return hipGetLastError();
}

// One wave per instance (and 64 m) pays where a lane's share of the sum is short:
// 3/0/10 bits x 1024, 128 k a lane, 36 us against 19 with a block per instance;
// 2/1/7 x 5000, 8 k, 10 against 20.  Few instances leave a wave nothing to
// overlap with, and the line moves by two bits.
constexpr int kDotBits = 12;
// B through LDS pays where a block has many values of m to share it and the sum
// several fills of it: 6/3/10 bits x 1 44 us against 160, 5/3/8 x 64 12 and 27;
// but 5/0/5 x 500 10.1 against 7.8, 3/0/13 x 1 65 against 25.  With many columns
// and a block for every CU it does for shorter sums too (8/3/6 x 1024 30 and 70).
inline bool stage_b(const NodeDesc& d) {
  const int m = d.mbits, n = d.nbits;
  const bool busy = d.n_ref >> 8 || (m > 8 && (d.n_ref << (m - 8)) >> 8);
  const int least = m < 6 ? 8 - (busy && n >= 2 ? m + n - 6 : 0) : n < 2 ? 8 : busy ? 5 : 7;
  return m >= 4 && m + n >= 6 && d.kbits >= least;
}

template <int FL>
static hipError_t launch_kred(const NodeDesc& d0, uint64_t ws, const int64_t* sig, hipStream_t st) {
  if (!d0.keep_order && d0.mbits <= 6 && d0.nbits <= 3 &&
      d0.kbits + d0.mbits + d0.nbits <= (d0.n_ref >= kDotInstances ? kDotBits : kDotBits - 2)) {
    const dim3 g((unsigned)std::min<int64_t>((d0.n_inst + 3) / 4, kBlocks)), b(256);
    switch (d0.nbits) {
      case 0: hipLaunchKernelGGL((k_kdot<FL, 1>), g, b, 0, st, d0, ws, sig); break;
      case 1: hipLaunchKernelGGL((k_kdot<FL, 2>), g, b, 0, st, d0, ws, sig); break;
      case 2: hipLaunchKernelGGL((k_kdot<FL, 4>), g, b, 0, st, d0, ws, sig); break;
      default: hipLaunchKernelGGL((k_kdot<FL, 8>), g, b, 0, st, d0, ws, sig); break;
    }
    return hipGetLastError();
  }
  NodeDesc d = d0;
  const int nb = d.nbits < 4 ? d.nbits : 4;
  const int mb = d.mbits < 8 ? d.mbits : 8;
  // The lanes of a block that m does not fill split the sum (where the order
  // of additions has to stay, sums of 16 columns run on one lane each).
  d.ks_bits = d.keep_order && nb == 4 ? 0 : 8 - mb;
  if (!d.keep_order) {
    // fewer m per block, down to one wave of them, until there are
    // kKredBlocks blocks: each lane's chain of loads gets shorter and more
    // of them are in flight
    while (8 - d.ks_bits > 6 && mb > 6 && (d.n_ref << (d.mbits - (8 - d.ks_bits) + d.nbits - nb)) < kKredBlocks)
      ++d.ks_bits;
  }
  if (d.ks_bits > d.kbits) d.ks_bits = d.kbits;
  const int m2 = d.mbits < 8 - d.ks_bits ? d.mbits : 8 - d.ks_bits;
  const int64_t blocks = d.n_inst << (d.mbits - m2 + d.nbits - nb);
  const dim3 g((unsigned)std::min<int64_t>(blocks, kBlocks)), b(256);
  if (d.nbits <= 3 && !stage_b(d)) {
    switch (nb) {
      case 0: hipLaunchKernelGGL((k_kdir<FL, 1>), g, b, 0, st, d, ws, sig); break;
      case 1: hipLaunchKernelGGL((k_kdir<FL, 2>), g, b, 0, st, d, ws, sig); break;
      case 2: hipLaunchKernelGGL((k_kdir<FL, 4>), g, b, 0, st, d, ws, sig); break;
      default: hipLaunchKernelGGL((k_kdir<FL, 8>), g, b, 0, st, d, ws, sig); break;
    }
    return hipGetLastError();
  }
  switch (nb) {
    case 0: hipLaunchKernelGGL((k_kred<FL, 1>), g, b, 0, st, d, ws, sig); break;
    case 1: hipLaunchKernelGGL((k_kred<FL, 2>), g, b, 0, st, d, ws, sig); break;
    case 2: hipLaunchKernelGGL((k_kred<FL, 4>), g, b, 0, st, d, ws, sig); break;
    case 3: hipLaunchKernelGGL((k_kred<FL, 8>), g, b, 0, st, d, ws, sig); break;
    default: hipLaunchKernelGGL((k_kred<FL, 16>), g, b, 0, st, d, ws, sig); break;
  }
  return hipGetLastError();
}

template <int FL>
static hipError_t launch_stream_fl(const NodeDesc& d, uint64_t ws, const int64_t* sig, hipStream_t st) {
  if (d.n_inst == 0) return hipSuccess;
  switch (d.kbits) {
    case 0: return launch_small<FL, 1>(d, ws, sig, st);
    case 1: return launch_small<FL, 2>(d, ws, sig, st);
    case 2: return launch_small<FL, 4>(d, ws, sig, st);
    case 3: return launch_small<FL, 8>(d, ws, sig, st);
    case 4: return launch_small<FL, 16>(d, ws, sig, st);
  }
  return launch_kred<FL>(d, ws, sig, st);
}

hipError_t launch_stream(const NodeDesc& d, uint64_t ws, const int64_t* sig, hipStream_t st) {
  return launch_stream_fl<0>(d, ws, sig, st);
}

// complex-half plans: the storage combinations a plan produces (an FP32
// output only comes from FP32 operands: the stem)
hipError_t launch_stream_h(const NodeDesc& d, uint64_t ws, const int64_t* sig, hipStream_t st) {
  const int fl = (d.A.half ? 1 : 0) | (d.B.half ? 2 : 0) | (d.c_half ? 4 : 0);
  switch (fl) {
    case 0: return launch_stream_fl<kMixBit | 0>(d, ws, sig, st);
    case 1: return launch_stream_fl<kMixBit | 1>(d, ws, sig, st);
    case 2: return launch_stream_fl<kMixBit | 2>(d, ws, sig, st);
    case 3: return launch_stream_fl<kMixBit | 3>(d, ws, sig, st);
    case 4: return launch_stream_fl<kMixBit | 4>(d, ws, sig, st);
    case 5: return launch_stream_fl<kMixBit | 5>(d, ws, sig, st);
    case 6: return launch_stream_fl<kMixBit | 6>(d, ws, sig, st);
    case 7: return launch_stream_fl<kMixBit | 7>(d, ws, sig, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace matnc
