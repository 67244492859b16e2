// Subtrees of small steps (gate absorption, narrow branch steps of a small
// circuit) as one launch: a workgroup contracts a whole subtree, its operands
// and intermediates in LDS, one barrier per level of the tree.
//
// Bound: launched one by one such a step is all latency -- 5 to 6 us of launch,
// descriptor and first-touch loads for a few thousand multiply-adds, and a
// circuit has 30 to 150 of them.  Here a level costs an LDS round trip and a
// barrier, whatever the number of its steps: their outputs are dealt to the
// waves 64 at a time.  Measured: the 75 small steps of the 20-qubit depth-12
// circuit 10.5 us instead of 400; a 12-qubit depth-8 circuit's 64 slices, one
// workgroup each, 13 us in one launch instead of 32 launch sequences of 30 us.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "desc.h"
#include "device_common.h"
#include "kernels.h"

namespace matnc {

// One component per workgroup and slice.  Its description (see TreeStep) is
// copied to LDS first, then its inputs, then the levels run.
__global__ __launch_bounds__(kTreeThreads) void k_tree(uint64_t ws, uint64_t table_off, int n_comp,
                                                       const int64_t* __restrict__ sig, int64_t sigma0) {
  __shared__ __attribute__((aligned(16))) uint32_t words[kTreeWords];
  __shared__ float2 data[kTreeElems];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int comp = blockIdx.x % n_comp, s = blockIdx.x / n_comp;
  const gptr<const uint32_t> table = gmem<const uint32_t>(ws + table_off);
  const uint32_t first = table[comp], count = table[comp + 1] - first;
  for (uint32_t i = tid; i < count; i += kTreeThreads) words[i] = table[first + i];
  const int64_t sigma = (sig ? sig[0] : sigma0) + s;
  __syncthreads();
  auto word = [&](uint32_t i) { return (uint32_t)__builtin_amdgcn_readfirstlane(words[i]); };
  TreeHeader h;
  h.n_levels = word(0);
  h.n_inputs = word(1);
  h.inputs = word(2);
  h.steps = word(3);
  h.levels = word(4);
  h.items = word(5);
  h.n_big = word(6);
  // inputs: the large ones by all waves together, of the others one to a wave
  // (a 32 KiB tensor is 64 loads of a wave, one after another: 10 us)
  auto copy = [&](uint32_t i, uint32_t first, uint32_t step) {
    const uint32_t at = h.inputs + i * (sizeof(TreeInput) / 4);
    const TreeInput in = *reinterpret_cast<const TreeInput*>(words + at);
    uint64_t sub = 0;
    for (uint32_t t = 0; t < word(at + 5); ++t)
      sub |= (uint64_t)((sigma >> ((words[at + 6 + (t >> 2)] >> (8 * (t & 3))) & 0xffu)) & 1) << t;
    const uint32_t emask = (1u << in.ebits) - 1u, n = in.keys << in.ebits;
    const uint64_t off = (uint64_t)in.off_lo | ((uint64_t)in.off_hi << 32);
    for (uint32_t e0 = first; e0 < n; e0 += 4 * step) {
      float2 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t e = e0 + u * step;
        // instance key * 2^nsb + sub of the leaf (nsb = 0: a tensor without sliced indices)
        const uint64_t inst = ((uint64_t)(e >> in.ebits) << in.nsb) + sub;
        if (e < n) v[u] = ldg_f2(ws + off, (inst << in.ebits) + (e & emask));
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (e0 + u * step < n) data[in.lds + e0 + u * step] = v[u];
    }
  };
  for (uint32_t i = 0; i < h.n_big; ++i) copy(i, tid, kTreeThreads);
  for (uint32_t i = h.n_big + wave; i < h.n_inputs; i += kTreeThreads / 64) copy(i, lane, 64);
  __syncthreads();
  for (uint32_t l = 0; l < h.n_levels; ++l) {
    const uint32_t i1 = word(h.levels + l + 1);
    for (uint32_t i = word(h.levels + l) + wave; i < i1; i += kTreeThreads / 64) {
      const uint32_t item = word(h.items + i);  // step << 16 | chunk of outputs
      const TreeStep t = *reinterpret_cast<const TreeStep*>(words + h.steps + (item >> 16) * (sizeof(TreeStep) / 4));
      const uint32_t cut = t.bits >> 25, ob = 6 - cut;  // 2^cut lanes share a sum
      const uint32_t o = ((item & 0xffffu) << ob) + (lane & ((1u << ob) - 1u));
      if (o >= t.outputs) continue;
      const uint32_t mb = t.bits & 0xffu, nb = (t.bits >> 8) & 0xffu, kb = (t.bits >> 16) & 0xffu;
      const uint32_t j = o >> (mb + nb);
      const uint32_t m = o & ((1u << mb) - 1u), n = (o >> mb) & ((1u << nb) - 1u);
      const uint32_t g = t.gmap ? words[t.gmap + j] : 0u;
      const uint32_t ga = g & 0xffffu, gb = g >> 16;
      const float2* a = data + t.a + (ga << (mb + kb)) + m;
      const float2* b = data + t.b + (gb << (nb + kb)) + n;
      float2 c = make_float2(0.f, 0.f);
      if (kb > 4) {
        // long sums: every 2^cut-th k to a lane, four of them at a time summed
        // on their own, the lanes' sums in a tree
        const uint32_t k1 = 1u << kb;
        for (uint32_t k = lane >> ob; k < k1; k += 4u << cut) {
          float2 av[4], bv[4], g4 = make_float2(0.f, 0.f);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            av[u] = a[(k + ((uint32_t)u << cut)) << mb];
            bv[u] = b[(k + ((uint32_t)u << cut)) << nb];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) cmac(g4, av[u], bv[u]);
          c.x += g4.x;
          c.y += g4.y;
        }
        for (uint32_t x = 32; x >> ob; x >>= 1) {
          c.x += __shfl_xor(c.x, (int)x);
          c.y += __shfl_xor(c.y, (int)x);
        }
      } else {
        uint32_t k = 0;
        for (; k + 4 <= (1u << kb); k += 4) {
          float2 av[4], bv[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            av[u] = a[(k + u) << mb];
            bv[u] = b[(k + u) << nb];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) cmac(c, av[u], bv[u]);
        }
        for (; k < (1u << kb); ++k) cmac(c, a[k << mb], b[k << nb]);
      }
      if (lane >> ob) continue;
      uint32_t oc = 0;
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) oc |= ((o >> (4 * q + e)) & (4 * q + e < (int)(mb + nb) ? 1u : 0u))
                                         << ((t.pos[q] >> (8 * e)) & 31u);
      const uint32_t inst = (j << (mb + nb)) + oc;
      if ((t.bits >> 24) & 1u) {  // a component's result goes to the arena
        const uint64_t off = (uint64_t)t.c_lo | ((uint64_t)t.c_hi << 32);
        stg_f2(ws + off, (((uint64_t)s * t.w) << (mb + nb)) + inst, c);
      } else {
        data[t.c_lo + inst] = c;
      }
    }
    __syncthreads();
  }
}

hipError_t launch_tree(uint64_t ws, uint64_t table_off, int n_comp, int nb, const int64_t* sig, int64_t sigma0,
                       hipStream_t st) {
  if (n_comp == 0 || nb == 0) return hipSuccess;
  hipLaunchKernelGGL(k_tree, dim3((unsigned)(n_comp * nb)), dim3(kTreeThreads), 0, st, ws, table_off, n_comp, sig, sigma0);
  return hipGetLastError();
}

}  // namespace matnc
