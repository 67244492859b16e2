// Matrix-core kernel of the FP32-stored steps (gfx950): C[m, n] = sum_k
// A[m, k] B[k, n] as a complex GEMM whose FP32 operands are split exactly into
// three bfloat16 parts each (8 + 8 + 8 of the 24 bits; bfloat16 has FP32's
// exponent range, so no scaling is involved).  Of the nine products of parts
// the six with index sum <= 2 are summed on v_mfma_f32_32x32x16_bf16 in FP32;
// the three left out are below 2^-25 of the product.  The FP32 instruction
// (v_mfma_f32_32x32x2f32, kernels_c64.hip) rounds the accumulator once per
// two real products; here it is rounded six times per sixteen, so the result
// is also nearer to the 64-bit one: relative error on normal operands
// 3.4e-8, 1.1e-7, 2.4e-7, 4.9e-7, 7.0e-7 at 3, 5, 7, 9, 10 k bits, against
// 7.4e-8, 1.4e-7, 2.9e-7, 5.7e-7, 8.1e-7.
//
// Bound: six bfloat16 products take 192 matrix-core cycles per 32 x 16 x 8
// complex block, the FP32 instruction 512.  At 20/8/9 bits of m/n/k the step
// runs 5.9 ms (186 TFLOP/s complex, 1118 TFLOP/s of bfloat16 -- what a large
// bfloat16 library product reaches on this card under its power limit)
// against 8.6 ms for the FP32 instruction's best tile.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "desc.h"
#include "device_common.h"
#include "kernels.h"

namespace matnc {

// Operands are scaled by 2^24 as they are split, so that the last part of the
// smallest FP32 number still is a bfloat16 number (gates hold cos(pi/2) =
// 6e-17 and products of two such entries, 4e-33, whose last parts would
// be lost otherwise).
constexpr float kScale = 16777216.f;             // 2^24
constexpr float kUnscale = 1.f / (kScale * kScale);

// Exact split of an FP32 pair into three packed (re, im) bfloat16 pairs:
// value = p[0] + p[1] + p[2], each part the rest rounded to nearest (8 + 8 + 8
// bits hold the 24 of an FP32 number).
struct Split3 {
  uint32_t p[3];
};

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ uint32_t pack_bf16(float x, float y) {
  const bf16x2 h = __builtin_convertvector(f32x2{x, y}, bf16x2);
  uint32_t u;
  __builtin_memcpy(&u, &h, 4);
  return u;
}

__device__ __forceinline__ float2 scaled(float2 v) { return make_float2(v.x * kScale, v.y * kScale); }

template <int NP>
__device__ __forceinline__ Split3 split3(float2 v) {
  Split3 s;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    s.p[p] = pack_bf16(v.x, v.y);
    v.x -= __uint_as_float(s.p[p] << 16);
    v.y -= __uint_as_float(s.p[p] & 0xffff0000u);
  }
  return s;
}

// Tile: TM = 32*RM*WM values of m, TN = 16*RN*WN complex n, 8 complex k.
// FAN: the tile's TN columns are TN >> nbits slots of 2^nbits columns, one
// per output instance of a fan-table row (see NodeDesc); the A tile is
// loaded once for all of them.
// REC (fan tiles only): also record each output instance's largest
// |component| into its scale slot (complex-half plans, whose FP32 branch
// tensors feed FP16 steps): half-wave reductions and one LDS atomic per
// slot column, one global atomic per slot and tile.
// HA, HB (complex-half plans only): A, B stored in FP16 with a per-instance
// exponent; the output is FP32 either way.
template <int RM, int RN, int WM, int WN, bool FAN, bool REC = false, bool HA = false, bool HB = false>
__global__ __launch_bounds__(64 * WM * WN, 2) void k_split(NodeDesc d, uint64_t ws, const int64_t* __restrict__ sig) {
  static_assert(!REC || FAN, "maxima are recorded by fan-out tiles only");
  constexpr int TK = 8;
  constexpr int NT = 64 * WM * WN;
  constexpr int TM = 32 * RM * WM;
  constexpr int TN = 16 * RN * WN;
  constexpr int QA = (TK / 4) * TM;  // quads of four consecutive k of the A tile
  constexpr int QB = (TK / 4) * TN;  // ... and of the B tile
  static_assert(QA % NT == 0 || NT % QA == 0, "A quads must split evenly over threads, or fit in fewer");
  static_assert(QB % NT == 0 || NT % QB == 0, "B quads must split evenly over threads, or fit in fewer");
  constexpr int EQA = QA >= NT ? QA / NT : 1;
  constexpr int EQB = QB >= NT ? QB / NT : 1;
  // parts of each operand (an FP16 value has 11 bits: two parts)
  constexpr int PA = HA ? 2 : 3;
  constexpr int PB = HB ? 2 : 3;
  // LDS tiles in the register layout of the MFMA operands, one plane per
  // part: As[k/4][m][k%4] holds A's (re, im) pairs; Bs[k/4][n][d][k%4] holds
  // B's rows of the real embedding, (re, -im) for d = 0 and (im, re) for d = 1
  constexpr int AQ = 4 * TM + 16;  // words per k quad (padded)
  __shared__ __attribute__((aligned(16))) uint32_t As[2][PA][(TK / 4) * AQ];
  __shared__ __attribute__((aligned(16))) uint32_t Bs[2][PB][(TK / 4) * TN * 8];
  // per-tile column data, shared by the waves instead of held per lane:
  // the C offset of each of the tile's TN columns, and for fan tiles the
  // B instance (byte offset) and output instance base of each slot
  __shared__ uint32_t s_cn[TN];
  __shared__ uint64_t s_bb[FAN ? TN : 1];
  __shared__ uint64_t s_cb[FAN ? TN : 1];
  __shared__ uint32_t s_mx[REC ? TN : 1];  // per-slot maxima (float bits)
  __shared__ float s_fb[(FAN && HB) ? TN : 1];  // per-slot factor 2^e of an FP16 B

  const gptr<const uint32_t> tab = gmem<const uint32_t>(ws + d.tab_off);
  const cptr<const uint32_t> ctab = cmem<const uint32_t>(ws + d.tab_off);  // k-step lookups
  const gptr<const int32_t> glA = gmem<const int32_t>(ws + d.A.gmap_off);
  const gptr<const int32_t> glB = gmem<const int32_t>(ws + d.B.gmap_off);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave % WM;
  const int wn = wave / WM;

  const int nt_bits = FAN ? 0 : d.nbits - __builtin_ctz(TN);
  const int tbits = d.mbits - __builtin_ctz(TM) + nt_bits;  // tiles per unit = 2^tbits
  const int ksteps = 1 << (d.kbits - __builtin_ctz(TK));
  const int64_t sigma0 = sig[0];
  // work units: output instances, or (slice, fan row) pairs
  const uint32_t units = (uint32_t)(FAN ? ((uint32_t)d.n_inst / (uint32_t)d.w) * (uint32_t)d.n_fan : d.n_inst);
  const uint32_t total = units << tbits;
  const gptr<const int32_t> fan = gmem<const int32_t>(ws + d.fan_off);
  const uint32_t nmask = (1u << d.nbits) - 1u;
  const int slots = FAN ? (TN >> d.nbits) : 1;
  const bool astage = QA >= NT || tid < QA;
  const bool bstage = QB >= NT || tid < QB;

  for (uint32_t blk = blockIdx.x; blk < total; blk += gridDim.x) {
    // logical tile order: n tiles innermost (they share the A tile), then m
    // tiles, then instances / fan rows (fan rows in blocks, see unit_tile);
    // each XCD takes a contiguous range
    const uint32_t lt = xcd_tile(blk, total);
    uint32_t u, t;
    unit_tile(lt, units, tbits, d.fan_rows > 0 ? (uint32_t)d.fan_rows : (FAN ? 2u : 1u), u, t);
    const uint32_t m0 = (t >> nt_bits) * TM;
    const uint32_t n0 = (t & ((1u << nt_bits) - 1u)) * TN;
    int64_t s, j;
    gptr<const int32_t> fj = nullptr;
    if (FAN) {
      s = d.dep ? u / (uint32_t)d.n_fan : 0u;
      fj = fan + (uint64_t)(u - (uint32_t)s * (uint32_t)d.n_fan) * slots;
      j = fj[0];
    } else {
      s = d.dep ? u / (uint32_t)d.w : 0u;
      j = (int64_t)u - s * d.w;
    }
    const int64_t inst = s * d.w + j;  // output instance (slot 0 for fan tiles)
    const int64_t sigma = sigma0 + s;
    const int64_t ai = operand_instance(d.A, glA, j, s, sigma);
    const int64_t bi = operand_instance(d.B, glB, j, s, sigma);
    const uint64_t pa = ws + d.A.off + ai * d.A.inst_bytes;
    const uint64_t pb = ws + d.B.off + bi * d.B.inst_bytes;
    const gptr<f32x2> pc = gmem<f32x2>(ws + d.c_off + inst * d.c_inst_bytes);
    const float ca = HA ? ldexpf(1.f, ldg_scale(ws + d.A.scale_off, ai).e) : 1.f;
    const float cb = HB ? ldexpf(1.f, ldg_scale(ws + d.B.scale_off, bi).e) : 1.f;
    if (tid < TN) s_cn[tid] = tlook(tab + TAB_CN * kTabSize, FAN ? (tid & nmask) : n0 + tid);
    if (FAN && tid < slots) {
      // an empty slot reads slot 0's B into columns that are never stored
      const int jg = fj[tid];
      const int64_t bg = operand_instance(d.B, glB, jg < 0 ? j : jg, s, sigma);
      s_bb[tid] = d.B.off + bg * d.B.inst_bytes;
      s_cb[tid] = jg < 0 ? 0 : d.c_off + (uint64_t)(s * d.w + jg) * d.c_inst_bytes;
      if (REC) s_mx[tid] = 0u;
      if (HB) s_fb[tid] = ldexpf(1.f, ldg_scale(ws + d.B.scale_off, bg).e);
    }
    __syncthreads();  // the column data above is read by every wave

    // quad coordinates (fixed across k steps): A quad e of this thread covers
    // m = amm[e], k = 4 akq[e] .. 4 akq[e] + 3 of the k step; likewise B over n
    uint32_t aoff[EQA][4], boff[EQB][4];
    int akq[EQA], bkq[EQB], amm[EQA], bnn[EQB];
#pragma unroll
    for (int e = 0; e < EQA; ++e) {
      const int flat = astage ? e * NT + tid : 0;
      amm[e] = flat % TM;
      akq[e] = flat / TM;
      const uint32_t om_ = tlook(tab + TAB_AM * kTabSize, m0 + amm[e]);
#pragma unroll
      for (int q = 0; q < 4; ++q) aoff[e][q] = om_ + tab[TAB_AK * kTabSize + 4 * akq[e] + q];
    }
    uint64_t pbe[EQB];  // B instance of each quad (fan tiles: its slot's)
    float cbe[EQB];     // and its factor (FP16 B)
#pragma unroll
    for (int e = 0; e < EQB; ++e) {
      const int flat = bstage ? e * NT + tid : 0;
      bnn[e] = flat % TN;
      bkq[e] = flat / TN;
      uint32_t on_;
      if (FAN) {
        pbe[e] = ws + s_bb[bnn[e] >> d.nbits];
        cbe[e] = HB ? s_fb[bnn[e] >> d.nbits] : 1.f;
        on_ = tlook(tab + TAB_BN * kTabSize, bnn[e] & nmask);
      } else {
        pbe[e] = pb;
        cbe[e] = cb;
        on_ = tlook(tab + TAB_BN * kTabSize, n0 + bnn[e]);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) boff[e][q] = on_ + tab[TAB_BK * kTabSize + 4 * bkq[e] + q];
    }
    typename FStage<HA>::type ra[EQA][4];
    typename FStage<HB>::type rb[EQB][4];
    auto gload = [&](uint32_t kba, uint32_t kbb) {
      if (astage) {
#pragma unroll
        for (int e = 0; e < EQA; ++e)
#pragma unroll
          for (int q = 0; q < 4; ++q) ra[e][q] = FStage<HA>::load(pa, aoff[e][q] + kba);
      }
      if (bstage) {
#pragma unroll
        for (int e = 0; e < EQB; ++e)
#pragma unroll
          for (int q = 0; q < 4; ++q) rb[e][q] = FStage<HB>::load(pbe[e], boff[e][q] + kbb);
      }
    };
    auto lstore = [&](int buf) {
      if (astage) {
#pragma unroll
        for (int e = 0; e < EQA; ++e) {
          Split3 v[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = split3<PA>(scaled(FStage<HA>::val(ra[e][q], ca)));
#pragma unroll
          for (int p = 0; p < PA; ++p)
            *reinterpret_cast<uint4*>(&As[buf][p][akq[e] * AQ + 4 * amm[e]]) =
                make_uint4(v[0].p[p], v[1].p[p], v[2].p[p], v[3].p[p]);
        }
      }
      if (bstage) {
#pragma unroll
        for (int e = 0; e < EQB; ++e) {
          Split3 v[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) v[q] = split3<PB>(scaled(FStage<HB>::val(rb[e][q], cbe[e])));
          const int base = ((bkq[e] * TN + bnn[e]) * 2) * 4;
#pragma unroll
          for (int p = 0; p < PB; ++p) {
            *reinterpret_cast<uint4*>(&Bs[buf][p][base]) =
                make_uint4(v[0].p[p] ^ 0x80000000u, v[1].p[p] ^ 0x80000000u, v[2].p[p] ^ 0x80000000u,
                           v[3].p[p] ^ 0x80000000u);
            *reinterpret_cast<uint4*>(&Bs[buf][p][base + 4]) =
                make_uint4(__builtin_amdgcn_alignbit(v[0].p[p], v[0].p[p], 16),
                           __builtin_amdgcn_alignbit(v[1].p[p], v[1].p[p], 16),
                           __builtin_amdgcn_alignbit(v[2].p[p], v[2].p[p], 16),
                           __builtin_amdgcn_alignbit(v[3].p[p], v[3].p[p], 16));
          }
        }
      }
    };

    floatx16 acc[RM][RN];
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
      for (int q = 0; q < RN; ++q)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][q][r] = 0.f;

    const int half = lane >> 5;  // this lane's k quad
    const int l32 = lane & 31;
    const int dsel = l32 & 1;    // row of the real embedding: 0 real part, 1 imaginary part
    const int ncol = l32 >> 1;

    // output offsets of this lane's m values, fetched before the k loop
    uint32_t om[RM];
#pragma unroll
    for (int i = 0; i < RM; ++i) om[i] = tlook(tab + TAB_CM * kTabSize, m0 + (wm * RM + i) * 32 + l32);

    // k offsets run one step ahead of the loads that use them, so that their
    // table reads are in flight during a whole step of MFMA work
    uint32_t kba = tlook(ctab + TAB_AK * kTabSize, 0u), kbb = tlook(ctab + TAB_BK * kTabSize, 0u);
    gload(kba, kbb);
    if (ksteps > 1) {
      kba = tlook(ctab + TAB_AK * kTabSize, (uint32_t)TK);
      kbb = tlook(ctab + TAB_BK * kTabSize, (uint32_t)TK);
    }
    lstore(0);
    __syncthreads();
    for (int ks = 0; ks < ksteps; ++ks) {
      const int buf = ks & 1;
      if (ks + 1 < ksteps) {
        gload(kba, kbb);
        if (ks + 2 < ksteps) {
          kba = tlook(ctab + TAB_AK * kTabSize, (uint32_t)(ks + 2) * TK);
          kbb = tlook(ctab + TAB_BK * kTabSize, (uint32_t)(ks + 2) * TK);
        }
      }
      auto afrag = [&](int p, int i) {
        return *reinterpret_cast<const bf16x8*>(&As[buf][p][half * AQ + 4 * ((wm * RM + i) * 32 + l32)]);
      };
      auto bfrag = [&](int p, int q) {
        return *reinterpret_cast<const bf16x8*>(&Bs[buf][p][((half * TN + (wn * RN + q) * 16 + ncol) * 2 + dsel) * 4]);
      };
      // products of parts pa, pb with pa + pb <= 2, the smallest first; the
      // fragments of the side with fewer tiles are held, the others read in turn
      if constexpr (RM <= RN) {
        bf16x8 yv[PA][RM];
#pragma unroll
        for (int p = 0; p < PA; ++p)
#pragma unroll
          for (int i = 0; i < RM; ++i) yv[p][i] = afrag(p, i);
#pragma unroll
        for (int q = 0; q < RN; ++q) {
          bf16x8 xv[PB];
#pragma unroll
          for (int p = 0; p < PB; ++p) xv[p] = bfrag(p, q);
#pragma unroll
          for (int g = 2; g >= 0; --g)
#pragma unroll
            for (int ap = 0; ap <= g; ++ap)
              if (ap < PA && g - ap < PB)
#pragma unroll
                for (int i = 0; i < RM; ++i)
                  acc[i][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xv[g - ap], yv[ap][i], acc[i][q], 0, 0, 0);
        }
      } else {
        bf16x8 xv[PB][RN];
#pragma unroll
        for (int p = 0; p < PB; ++p)
#pragma unroll
          for (int q = 0; q < RN; ++q) xv[p][q] = bfrag(p, q);
#pragma unroll
        for (int i = 0; i < RM; ++i) {
          bf16x8 yv[PA];
#pragma unroll
          for (int p = 0; p < PA; ++p) yv[p] = afrag(p, i);
#pragma unroll
          for (int g = 2; g >= 0; --g)
#pragma unroll
            for (int ap = 0; ap <= g; ++ap)
              if (ap < PA && g - ap < PB)
#pragma unroll
                for (int q = 0; q < RN; ++q)
                  acc[i][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xv[g - ap][q], yv[ap], acc[i][q], 0, 0, 0);
        }
      }
      if (ks + 1 < ksteps) lstore(buf ^ 1);
      __syncthreads();
    }

    // A sum with an infinite or NaN input, or one whose scaled value leaves
    // FP32's range (an operand above 2^104, a sum above 2^80), is not what
    // FP32 products give: a wave that holds a non-finite value computes its
    // part of the tile again with FP32 operations.
    float fin = 0.f;
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
      for (int q = 0; q < RN; ++q)
#pragma unroll
        for (int r = 0; r < 16; ++r) fin = fmaf(acc[i][q][r], 0.f, fin);
    if (__any(fin != 0.f)) {
      const uint32_t kcount = 1u << d.kbits;
      for (int e = lane; e < 32 * RM * 16 * RN; e += 64) {
        const int nl = wn * RN * 16 + e / (32 * RM);
        const uint32_t m = m0 + wm * RM * 32 + e % (32 * RM);
        const int g = FAN ? nl >> d.nbits : 0;
        if (FAN && s_cb[g] == 0) continue;
        const uint64_t pbg = FAN ? ws + s_bb[g] : pb;
        const float cbg = FAN ? (HB ? s_fb[g] : 1.f) : cb;
        const uint32_t oa = tlook(tab + TAB_AM * kTabSize, m);
        const uint32_t ob = tlook(tab + TAB_BN * kTabSize, FAN ? (nl & nmask) : n0 + nl);
        float2 c = make_float2(0.f, 0.f);
        for (uint32_t k = 0; k < kcount; ++k)
          cmac(c, FStage<HA>::val(FStage<HA>::load(pa, oa + tlook(tab + TAB_AK * kTabSize, k)), ca),
               FStage<HB>::val(FStage<HB>::load(pbg, ob + tlook(tab + TAB_BK * kTabSize, k)), cbg));
        const gptr<f32x2> dst = FAN ? gmem<f32x2>(ws + s_cb[g]) : pc;
        dst[tlook(tab + TAB_CM * kTabSize, m) + s_cn[nl]] = f32x2{c.x, c.y};
        if (REC) atomicMax(&s_mx[g], __float_as_uint(fmaxf(fmaxf(0.f, fabsf(c.x)), fabsf(c.y))));
      }
    } else {
      // epilogue: lane holds C[m][n] (re, im) in registers (r, r+1), r even
#pragma unroll
      for (int q = 0; q < RN; ++q) {
#pragma unroll
        for (int rr = 0; rr < 8; ++rr) {
          const int r = 2 * rr;
          const int row = 8 * (rr >> 1) + 4 * half + 2 * (rr & 1);
          const int nl = (wn * RN + q) * 16 + (row >> 1);  // column within the tile
          gptr<f32x2> dst = pc;
          bool live = true;
          if (FAN) {
            const uint64_t cbs = s_cb[nl >> d.nbits];  // uniform over the 32 lanes of a half-wave (one n)
            live = cbs != 0;
            dst = gmem<f32x2>(ws + cbs);
          }
          const uint32_t ocn = s_cn[nl];
          float v = 0.f;
#pragma unroll
          for (int i = 0; i < RM; ++i) {
            const float2 c = make_float2(acc[i][q][r] * kUnscale, acc[i][q][r + 1] * kUnscale);
            if (live) dst[om[i] + ocn] = f32x2{c.x, c.y};
            if (REC) v = fmaxf(v, fmaxf(fabsf(c.x), fabsf(c.y)));
          }
          if (REC) {
            // the half-wave's 32 lanes hold 32 values of m of one column
#pragma unroll
            for (int o = 16; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
            if (l32 == 0 && live) atomicMax(&s_mx[nl >> d.nbits], __float_as_uint(v));
          }
        }
      }
    }
    if (REC) {
      __syncthreads();
      if (tid < slots) {
        const int jg = fj[tid];
        if (jg >= 0 && s_mx[tid] > 0u) max_scale_mx(ws + d.c_scale_off, s * d.w + jg, s_mx[tid]);
      }
    }
    __syncthreads();  // the next tile rewrites the column data
  }
}

// ---------------------------------------------------------------------------
// launchers (the tile configurations are those of kernels_c64.hip)

template <bool FAN, bool REC, bool HA, bool HB>
static hipError_t launch_split_s(const NodeDesc& d, int cfg, unsigned grid, uint64_t ws, const int64_t* sig,
                                hipStream_t st) {
  switch (cfg) {
    case 0: hipLaunchKernelGGL((k_split<2, 1, 2, 2, FAN, REC, HA, HB>), dim3(grid), dim3(256), 0, st, d, ws, sig); break;
    case 1: hipLaunchKernelGGL((k_split<2, 2, 2, 2, FAN, REC, HA, HB>), dim3(grid), dim3(256), 0, st, d, ws, sig); break;
    case 2: hipLaunchKernelGGL((k_split<1, 1, 2, 2, FAN, REC, HA, HB>), dim3(grid), dim3(256), 0, st, d, ws, sig); break;
    case 3: hipLaunchKernelGGL((k_split<4, 1, 2, 2, FAN, REC, HA, HB>), dim3(grid), dim3(256), 0, st, d, ws, sig); break;
    case 4: hipLaunchKernelGGL((k_split<4, 2, 2, 2, FAN, REC, HA, HB>), dim3(grid), dim3(256), 0, st, d, ws, sig); break;
    case 5:
      if (FAN) return hipErrorInvalidValue;
      hipLaunchKernelGGL((k_split<2, 4, 2, 2, false, false, HA, HB>), dim3(grid), dim3(256), 0, st, d, ws, sig);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <bool FAN, bool REC = false>
static hipError_t launch_split_t(const NodeDesc& d, int cfg, uint64_t ws, const int64_t* sig, hipStream_t st) {
  if (d.n_inst == 0) return hipSuccess;
  const bool fits = FAN ? mfma_fan_config_fits(cfg, d.mbits, d.nbits, d.kbits, d.fan_tn)
                        : mfma_config_fits(cfg, d.mbits, d.nbits, d.kbits);
  if (!fits || (FAN && (d.w <= 0 || d.n_fan <= 0))) return hipErrorInvalidValue;
  const int64_t units = FAN ? (d.n_inst / d.w) * d.n_fan : d.n_inst;
  const int tbits = d.mbits - mfma_config_tm_bits(cfg) + (FAN ? 0 : d.nbits - mfma_config_tn_bits(cfg));
  const unsigned grid = grid_for(units << tbits);
  // FP16-stored operands occur only in complex-half plans
  if (d.A.half) {
    if (d.B.half) return launch_split_s<FAN, REC, true, true>(d, cfg, grid, ws, sig, st);
    return launch_split_s<FAN, REC, true, false>(d, cfg, grid, ws, sig, st);
  }
  if (d.B.half) return launch_split_s<FAN, REC, false, true>(d, cfg, grid, ws, sig, st);
  return launch_split_s<FAN, REC, false, false>(d, cfg, grid, ws, sig, st);
}

hipError_t launch_split(const NodeDesc& d, int cfg, uint64_t ws, const int64_t* sig, hipStream_t st) {
  return launch_split_t<false>(d, cfg, ws, sig, st);
}

hipError_t launch_split_fan(const NodeDesc& d, int cfg, uint64_t ws, const int64_t* sig, hipStream_t st) {
  return launch_split_t<true>(d, cfg, ws, sig, st);
}

hipError_t launch_split_fan_rec(const NodeDesc& d, int cfg, uint64_t ws, const int64_t* sig, hipStream_t st) {
  return launch_split_t<true, true>(d, cfg, ws, sig, st);
}

}  // namespace matnc
