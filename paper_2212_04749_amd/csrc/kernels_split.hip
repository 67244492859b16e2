// Matrix-core kernel of the FP32-stored steps (gfx950): C[m, n] = sum_k
// A[m, k] B[k, n] as a complex GEMM whose FP32 operands are split exactly into
// three bfloat16 parts each (8 + 8 + 8 of the 24 bits; bfloat16 has FP32's
// exponent range, so one constant factor serves every operand).  Of the nine
// products of parts the eight with index sum <= 3 are summed on
// v_mfma_f32_32x32x16_bf16; the ninth is below 2^-33 of the product.
//
// Accuracy.  The instruction drops what lies below the last bit of a nonzero
// accumulator at each addition (up to one unit of the last place, not half).
// The products of first parts, which are exact, have an accumulator of their
// own, so a sum of K products meets that once per eight complex k; the seven
// others add up in a second one 2^-8 as large, and the two are added once at the
// end.  The FP32 instruction (v_mfma_f32_32x32x2f32, kernels_c64.hip) rounds
// for every product.  Relative error against 64 bits at 3, 5, 7, 9, 10 k bits,
// that instruction and this kernel: normal operands 7.4e-8, 1.5e-7, 2.9e-7,
// 5.7e-7, 8.1e-7 and 3.2e-8, 4.9e-8, 8.9e-8, 1.9e-7, 2.7e-7; one product per
// sum, real, 2.5e-8 (at most 5.9e-8) in both; gate-like operands (zeros, +-i,
// cosines) 3.8e-8 .. 4.1e-7 and 2.5e-8 .. 2.1e-7; positive ones 4.7e-8 .. 4.9e-7
// and 2.8e-8 .. 2.5e-7.  (Six products in one accumulator, which this was
// before, left out 2^-24 of a product and rounded at full size six times per
// eight k: 3.5e-8, at most 1.4e-7, on single products, twice the instruction's
// error on sparse sums.)
//
// Bound: eight bfloat16 products take 256 matrix-core cycles per 32 x 16 x 8
// complex block, the FP32 instruction 512.  At 20/8/9 bits of m/n/k the step
// runs 6.97 ms (158 TFLOP/s complex, 1262 of bfloat16; a large bfloat16 library
// product reaches 1107 on this card under its power limit) against 8.60 ms for
// the FP32 instruction's best tile and 9.04 for the one that it chose.  At
// 22/6/6 bits 1.25 ms against 1.37.
//
// Fan-out tiles whose groups do not fill them multiply empty columns: at
// 10/3/11 bits (8 instances on average share an A) 0.70 of the 64-column
// tiles' columns hold an instance.  Leaving out the empty 16-column blocks by a
// condition in the k loop gave 4% there and cost 11% on 22/1/6 bits, whose
// tiles are full; with a loop of its own the kernel spills.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

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

// The least component of a result that is taken from a tile computed with
// operands scaled by 2^-24 instead: what such operands lose there is at most
// 2^-110 each, 2^18 of a product with the largest FP32 number.
constexpr float kLarge = 1152921504606846976.f;  // 2^60

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

__device__ __forceinline__ f32x2 load_f2(uint64_t base, uint32_t i) { return gmem<const f32x2>(base)[i]; }

// elements i (even) and i + 1
__device__ __forceinline__ void load_f2x2(uint64_t base, uint32_t i, f32x2 (&r)[2]) {
  const f32x4 v = *(gptr<const f32x4>)((gptr<const char>)base + 8 * i);
  r[0] = f32x2{v.x, v.y};
  r[1] = f32x2{v.z, v.w};
}

__device__ __forceinline__ float2 scaled(f32x2 v, float f) { return make_float2(v.x * f, v.y * f); }

__device__ __forceinline__ bool finite(float x) { return (__float_as_uint(x) & 0x7f800000u) != 0x7f800000u; }

__device__ __forceinline__ Split3 split3(float2 v) {
  Split3 s;
#pragma unroll
  for (int p = 0; p < 3; ++p) {
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
// LIN (every plan step): A[m + (k << mbits)], B[n + (k << nbits)] -- a thread
// loads two neighbouring m at once and every k row's address is a scalar step
// from the last; otherwise (a caller's own layout) an offset per element.
// S: k steps in flight.  One, except for few tiles of the smallest size, whose
// workgroups have a CU to themselves and wait for their loads (see kFewTiles);
// elsewhere a second stage costs a workgroup per CU (20/8/9 bits on the 128 x 64
// tile 6.4 ms with one, 6.9 ms with two).
template <int RM, int RN, int WM, int WN, bool FAN, bool LIN, int S = 1>
__global__ __launch_bounds__(64 * WM * WN, 2) void k_split(NodeDesc d, uint64_t ws, const int64_t* __restrict__ sig) {
  static_assert(LIN || !FAN, "fan-out tiles are a plan's");
  static_assert(RM * RN <= 4, "a lane's outputs have a bit each");
  constexpr int TK = 8;
  constexpr int NT = 64 * WM * WN;
  constexpr int TM = 32 * RM * WM;
  constexpr int TN = 16 * RN * WN;
  // m per block of A: two where every thread then still has a block; with half
  // of the threads idle tiles lose 7-15% to it
  constexpr int MA = LIN && TM == 256 && NT == 256 ? 2 : 1;
  constexpr int QA = (TK / 4) * TM / MA;  // blocks of four consecutive k of the A tile
  constexpr int QB = (TK / 4) * TN;  // ... and of the B tile
  static_assert(QA % NT == 0 || NT % QA == 0, "A quads must split evenly over threads, or fit in fewer");
  static_assert(QB % NT == 0 || NT % QB == 0, "B quads must split evenly over threads, or fit in fewer");
  constexpr int EQA = QA >= NT ? QA / NT : 1;
  constexpr int EQB = QB >= NT ? QB / NT : 1;
  // LDS tiles in the register layout of the MFMA operands, one plane per
  // part: As[k/4][m][k%4] holds A's (re, im) pairs; Bs[k/4][n][d][k%4] holds
  // B's rows of the real embedding, (re, -im) for d = 0 and (im, re) for d = 1
  constexpr int AQ = 4 * TM + 16;  // words per k quad (padded)
  __shared__ __attribute__((aligned(16))) uint32_t As[2][3][(TK / 4) * AQ];
  __shared__ __attribute__((aligned(16))) uint32_t Bs[2][3][(TK / 4) * TN * 8];
  // per-tile column data, shared by the waves instead of held per lane:
  // the C offset of each of the tile's TN columns, and for fan tiles the
  // B instance (byte offset) and output instance base of each slot
  __shared__ uint32_t s_cn[TN];
  __shared__ uint64_t s_bb[FAN ? TN : 1];
  __shared__ uint64_t s_cb[FAN ? TN : 1];
  // offsets of a tile's first row and column: [AM, CM, BN, CN][nibble][value];
  // of a k step's change of bits 3 .. t: [AK, BK][t]
  __shared__ uint32_t s_nib[4][8][16];
  __shared__ uint32_t s_kx[2][32];
  // tiles with a sum out of range, one bit for this workgroup's tiles 0, 1024, ..., and so on
  __shared__ uint32_t s_redo[33];  // [32]: there is one

  const gptr<const int32_t> glA = gmem<const int32_t>(ws + d.A.gmap_off);
  const gptr<const int32_t> glB = gmem<const int32_t>(ws + d.B.gmap_off);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave % WM;
  const int wn = wave / WM;

  const int nt_bits = FAN ? 0 : d.nbits - __builtin_ctz(TN);
  const int tbits = d.mbits - __builtin_ctz(TM) + nt_bits;  // tiles per unit = 2^tbits
  const int ksteps = 1 << (d.kbits - d.ksplit - __builtin_ctz(TK));  // of this part
  const int64_t sigma0 = d.flat ? 0 : sig[0] + d.s0;
  // work units: output instances, or (slice, fan row) pairs
  const uint32_t units = (uint32_t)(FAN ? ((uint32_t)d.n_inst / (uint32_t)d.w) * (uint32_t)d.n_fan : d.n_inst);
  const uint32_t upart = units << tbits;  // tiles of one part of the sum
  const uint32_t total = upart << d.ksplit;
  const gptr<const int32_t> fan = gmem<const int32_t>(ws + d.fan_off);
  const uint32_t nmask = (1u << d.nbits) - 1u;
  const int slots = FAN ? (TN >> d.nbits) : 1;
  const int half = lane >> 5;  // this lane's k quad
  const int l32 = lane & 31;
  const int dsel = l32 & 1;    // row of the real embedding: 0 real part, 1 imaginary part
  const int ncol = l32 >> 1;

  // Offsets inside a tile, the same for every tile of the launch (workgroups
  // are persistent): a bit-by-bit deposit for each element here, a lookup of
  // the tile's first row and column and of the k step's change in the loops.
  // (Deposits or table reads in the loops cost 20-40% at 22/6/6 bits.)
  if (lane < 16) {
    auto nibbles = [&](auto cls, uint32_t(&tab)[8][16]) {
      constexpr int C = decltype(cls)::value;
#pragma unroll
      for (int q = 0; q < 8; ++q) tab[q][lane] = dep_nibble<C>(d, q, lane);
    };
    if (wave == 0) nibbles(Class<TAB_AM>(), s_nib[0]);
    if (wave == 1) nibbles(Class<TAB_CM>(), s_nib[1]);
    if (wave == 2) nibbles(Class<TAB_BN>(), s_nib[2]);
    if (wave == 3) nibbles(Class<TAB_CN>(), s_nib[3]);
  } else if (lane < 48) {
    const uint32_t k = (2u << (lane - 16)) - 8u;
    if (wave == 0) s_kx[0][lane - 16] = dep<TAB_AK>(d, d.kbits, k);
    if (wave == 1) s_kx[1][lane - 16] = dep<TAB_BK>(d, d.kbits, k);
  }
  if (tid < 33) s_redo[tid] = 0;
  if (tid < TN) s_cn[tid] = dep<TAB_CN>(d, 8, FAN ? (tid & nmask) : tid);
  const bool astage = QA >= NT || tid < QA;
  // (B by other threads than A's where there are enough: 6/5/10 bits x 1 101 -> 78 us)
  const int btid = QA + QB <= NT ? (tid + NT - QA) % NT : tid;
  const bool bstage = QB >= NT || btid < QB;

  // A block e of this thread covers m = amm[e] .. amm[e] + MA - 1, k = 4 akq[e]
  // .. 4 akq[e] + 3 of the tile; likewise B blocks over n
  uint32_t aoff[LIN ? 1 : EQA][4], boff[LIN ? 1 : EQB][4];
  int akq[EQA], bkq[EQB], amm[EQA], bnn[EQB];
#pragma unroll
  for (int e = 0; e < EQA; ++e) {
    const int flat = astage ? e * NT + tid : 0;
    amm[e] = MA * (flat % (TM / MA));
    akq[e] = flat / (TM / MA);
    if constexpr (LIN) {
      if ((TM / MA) % 64 == 0) akq[e] = __builtin_amdgcn_readfirstlane(akq[e]);
    } else {
      const uint32_t om_ = dep<TAB_AM>(d, 8, amm[e]);
#pragma unroll
      for (int q = 0; q < 4; ++q) aoff[e][q] = om_ + dep<TAB_AK>(d, 4, 4 * akq[e] + q);
    }
  }
#pragma unroll
  for (int e = 0; e < EQB; ++e) {
    const int flat = bstage ? e * NT + btid : 0;
    bnn[e] = flat % TN;
    bkq[e] = flat / TN;
    if constexpr (!LIN) {
      const uint32_t on_ = dep<TAB_BN>(d, 8, bnn[e]);
#pragma unroll
      for (int q = 0; q < 4; ++q) boff[e][q] = on_ + dep<TAB_BK>(d, 4, 4 * bkq[e] + q);
    }
  }
  const uint64_t a_k = 8ull << d.mbits;  // LIN: bytes from one k to the next
  const uint64_t b_k = 8ull << d.nbits;
  uint32_t om[RM];  // output offsets of this lane's m values
#pragma unroll
  for (int i = 0; i < RM; ++i) om[i] = dep<TAB_CM>(d, 8, (wm * RM + i) * 32 + l32);
  __syncthreads();

  for (int pass = 0; pass < 2; ++pass) {
    if (pass) {  // the tiles that were out of range once more
      __syncthreads();
      if (!s_redo[32]) break;
    }
    const float sc = pass ? 1.f / kScale : kScale;
    uint32_t it = ~0u;
    for (uint32_t blk = blockIdx.x; blk < total; blk += gridDim.x) {
      ++it;
      if (pass && !((s_redo[(it >> 5) & 31] >> (it & 31)) & 1u)) continue;
      // logical tile order: n tiles innermost (they share the A tile), then m
      // tiles, then instances / fan rows (fan rows in blocks, see unit_tile);
      // each XCD takes a contiguous range
      uint32_t lt = xcd_tile(blk, total);
      uint32_t part = 0;
      if (d.ksplit) {  // tiles of one part are neighbours: they share A and B
        part = lt / upart;
        lt -= part * upart;
      }
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
      const int64_t ai = !FAN && d.flat ? inst : operand_instance(d.A, glA, j, s, sigma);
      const int64_t bi = !FAN && d.flat ? inst : operand_instance(d.B, glB, j, s, sigma);
      // offsets of (m0, n0): lane 8c + q looks up nibble q of class c
      uint32_t first = s_nib[(lane >> 3) & 3][lane & 7][((lane & 16 ? n0 : m0) >> (4 * (lane & 7))) & 15u];
#pragma unroll
      for (int o = 1; o < 8; o <<= 1) first |= __shfl_xor(first, o);
      const uint64_t oa0 = __builtin_amdgcn_readlane(first, 0), oc0 = (uint64_t)__builtin_amdgcn_readlane(first, 8) +
                                                                       (uint64_t)__builtin_amdgcn_readlane(first, 24);
      const uint64_t ob0 = __builtin_amdgcn_readlane(first, 16);
      const uint64_t pa = ws + d.A.off + ai * d.A.inst_bytes + oa0 * 8;
      const uint64_t pb = ws + d.B.off + bi * d.B.inst_bytes + ob0 * 8;
      const uint64_t c_off = d.ksplit ? d.part_off + (uint64_t)part * (uint64_t)d.n_inst * d.c_inst_bytes : d.c_off;
      const gptr<f32x2> pc = gmem<f32x2>(ws + c_off + inst * d.c_inst_bytes + oc0 * 8);
      if (FAN && tid < slots) {
        // an empty slot reads slot 0's B into columns that are never stored
        const int jg = fj[tid];
        const int64_t bg = operand_instance(d.B, glB, jg < 0 ? j : jg, s, sigma);
        s_bb[tid] = d.B.off + bg * d.B.inst_bytes;
        s_cb[tid] = jg < 0 ? 0 : c_off + (uint64_t)(s * d.w + jg) * d.c_inst_bytes + oc0 * 8;
      }
      if (FAN) __syncthreads();  // the column data above is read by every wave

      const uint32_t k0 = part * ((uint32_t)ksteps * TK);
      uint64_t pak[LIN ? EQA : 1], pbe[EQB];  // LIN: next k row of each block; else the instance's start
#pragma unroll
      for (int e = 0; e < EQB; ++e) {
        pbe[e] = FAN ? ws + s_bb[bnn[e] >> d.nbits] + (uint64_t)(bnn[e] & nmask) * 8
                     : pb + (LIN ? (uint64_t)bnn[e] * 8 : 0);
        if (LIN) pbe[e] += (uint64_t)(k0 + 4 * bkq[e]) * b_k;
      }
      if constexpr (LIN) {
#pragma unroll
        for (int e = 0; e < EQA; ++e) pak[e] = pa + (uint64_t)(k0 + 4 * akq[e]) * a_k;
      }
      uint32_t kba = 0, kbb = 0;  // offsets of the k step being loaded (not LIN)
      f32x2 ra[S][EQA][4][MA];
      f32x2 rb[S][EQB][4];
      // loads k step ks into stage st (where there are several, by every thread:
      // a load under a condition makes the compiler wait for all of them)
      auto gload = [&](int st, int ks) {
        if constexpr (!LIN) {
          if (ks > 0) {
            const int t = 3 + __builtin_ctz(ks);
            kba ^= __builtin_amdgcn_readfirstlane(s_kx[0][t]);
            kbb ^= __builtin_amdgcn_readfirstlane(s_kx[1][t]);
          }
        }
        if (S > 1 || astage) {
#pragma unroll
          for (int e = 0; e < EQA; ++e)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              if constexpr (LIN && MA == 2)
                load_f2x2(pak[e] + q * a_k, (uint32_t)amm[e], ra[st][e][q]);
              else if constexpr (LIN)
                ra[st][e][q][0] = load_f2(pak[e] + q * a_k, (uint32_t)amm[e]);
              else
                ra[st][e][q][0] = load_f2(pa, aoff[e][q] + kba);
            }
        }
        if (S > 1 || bstage) {
#pragma unroll
          for (int e = 0; e < EQB; ++e)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              if constexpr (LIN)
                rb[st][e][q] = load_f2(pbe[e] + q * b_k, 0);
              else
                rb[st][e][q] = load_f2(pbe[e], boff[e][q] + kbb);
            }
        }
        if constexpr (LIN) {
#pragma unroll
          for (int e = 0; e < EQA; ++e) pak[e] += TK * a_k;
#pragma unroll
          for (int e = 0; e < EQB; ++e) pbe[e] += TK * b_k;
        }
      };
      auto lstore = [&](int buf, int st) {
        if (astage) {
#pragma unroll
          for (int e = 0; e < EQA; ++e) {
#pragma unroll
            for (int i = 0; i < MA; ++i) {
              Split3 v[4];
#pragma unroll
              for (int q = 0; q < 4; ++q) v[q] = split3(scaled(ra[st][e][q][i], sc));
#pragma unroll
              for (int p = 0; p < 3; ++p)
                *reinterpret_cast<uint4*>(&As[buf][p][akq[e] * AQ + 4 * (amm[e] + i)]) =
                    make_uint4(v[0].p[p], v[1].p[p], v[2].p[p], v[3].p[p]);
            }
          }
        }
        if (bstage) {
#pragma unroll
          for (int e = 0; e < EQB; ++e) {
            Split3 v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = split3(scaled(rb[st][e][q], sc));
            const int base = ((bkq[e] * TN + bnn[e]) * 2) * 4;
#pragma unroll
            for (int p = 0; p < 3; ++p) {
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

      floatx16 acc[RM][RN], low[RM][RN];
#pragma unroll
      for (int i = 0; i < RM; ++i)
#pragma unroll
        for (int q = 0; q < RN; ++q)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][q][r] = low[i][q][r] = 0.f;

      auto kstep = [&](int buf) {
        auto afrag = [&](int p, int i) {
          return *reinterpret_cast<const bf16x8*>(&As[buf][p][half * AQ + 4 * ((wm * RM + i) * 32 + l32)]);
        };
        auto bfrag = [&](int p, int q) {
          return *reinterpret_cast<const bf16x8*>(&Bs[buf][p][((half * TN + (wn * RN + q) * 16 + ncol) * 2 + dsel) * 4]);
        };
        // products of parts pa, pb with pa + pb <= 3: those of the first parts into
        // acc, the others, smallest first, into low; the fragments of the side
        // with fewer tiles are held, the others read in turn
        auto tile = [&](floatx16& a, floatx16& lo, const bf16x8(&x)[3], const bf16x8(&y)[3]) {
#pragma unroll
          for (int g = 3; g >= 1; --g)
#pragma unroll
            for (int ap = g == 3 ? 1 : 0; ap <= (g == 3 ? 2 : g); ++ap)
              lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[g - ap], y[ap], lo, 0, 0, 0);
          a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], y[0], a, 0, 0, 0);
        };
        // In fan-out tiles the compiler moves the splitting of the next step's first
        // element, and with it the wait for its load, ahead of the products: 10/3/11
        // bits x 16372 20.9 -> 23.1 ms, 22/1/6 x 128 5.55 -> 6.04.  So not before the
        // last tiles' (elsewhere such a fence costs up to 2%).
        auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
        if constexpr (RM <= RN) {
          bf16x8 yv[RM][3];
#pragma unroll
          for (int i = 0; i < RM; ++i)
#pragma unroll
            for (int p = 0; p < 3; ++p) yv[i][p] = afrag(p, i);
#pragma unroll
          for (int q = 0; q < RN; ++q) {
            bf16x8 xv[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) xv[p] = bfrag(p, q);
            if (FAN && RN > 1 && q == RN - 1) fence();
#pragma unroll
            for (int i = 0; i < RM; ++i) tile(acc[i][q], low[i][q], xv, yv[i]);
          }
        } else {
          bf16x8 xv[RN][3];
#pragma unroll
          for (int q = 0; q < RN; ++q)
#pragma unroll
            for (int p = 0; p < 3; ++p) xv[q][p] = bfrag(p, q);
#pragma unroll
          for (int i = 0; i < RM; ++i) {
            bf16x8 yv[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) yv[p] = afrag(p, i);
            if (FAN && i == RM - 1) fence();
#pragma unroll
            for (int q = 0; q < RN; ++q) tile(acc[i][q], low[i][q], xv[q], yv);
          }
        }
      };

      // stages 0 .. S-1 hold k steps 0 .. S-1
      gload(0, 0);
#pragma unroll
      for (int u = 1; u < S; ++u)
        if (u < ksteps) gload(u, u);
      lstore(0, 0);
      __syncthreads();
      // Stage u held step k and was written to LDS at the end of step k - 1: it
      // now takes step k + S.  (The last S steps, which load nothing, have a copy
      // of their own; a single one without conditions, which cost 12% on the
      // 256 x 64 tile, 20/8/9 bits 6.97 -> 7.88 ms.)
      int ks = 0;
      for (; ks + S < ksteps; ks += S) {
#pragma unroll
        for (int u = 0; u < S; ++u) {
          gload(u, ks + u + S);
          kstep((ks + u) & 1);
          lstore((ks + u + 1) & 1, (u + 1) % S);
          __syncthreads();
        }
      }
      if constexpr (S == 1) {
        kstep(ks & 1);
        __syncthreads();
      } else {
#pragma unroll
        for (int u = 0; u < S; ++u) {
          const int k = ks + u;
          if (k < ksteps) {
            kstep(k & 1);
            if (k + 1 < ksteps) lstore((k + 1) & 1, (u + 1) % S);
            __syncthreads();
          }
        }
      }

      // A sum with an infinite or NaN input, or one whose scaled value leaves
      // FP32's range (an operand above 2^104, a sum above 2^80), is not what
      // FP32 products give.  Its tile is computed a second time after the
      // workgroup's others, with operands scaled down, for the outputs that are not
      // finite yet, and of these the ones that are still not right (see kLarge)
      // with FP32 operations: with operands of 1e13 everywhere, 12/6/9 bits x 64,
      // 1.09 ms against 0.50 in range (54 ms one output after another).
      float fin = 0.f;
#pragma unroll
      for (int i = 0; i < RM; ++i)
#pragma unroll
        for (int q = 0; q < RN; ++q)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            acc[i][q][r] += low[i][q][r];
            fin = fmaf(acc[i][q][r], 0.f, fin);
          }
      // (the epilogue: a lane holds C[m][n] (re, im) in registers (r, r+1), r even)
      if (pass == 0) {
        if (__any(fin != 0.f) && lane == 0) {
          atomicOr(&s_redo[(it >> 5) & 31], 1u << (it & 31));
          s_redo[32] = 1;
        }
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
#pragma unroll
            for (int i = 0; i < RM; ++i)
              if (live) dst[om[i] + ocn] = f32x2{acc[i][q][r] * kUnscale, acc[i][q][r + 1] * kUnscale};
          }
        }
      } else {
        uint32_t redo = 0;  // this lane's outputs that need FP32 operations
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
#pragma unroll
            for (int i = 0; i < RM; ++i) {
              if (!live) continue;
              const f32x2 was = dst[om[i] + ocn];
              if (finite(was.x) && finite(was.y)) continue;
              const f32x2 c = f32x2{acc[i][q][r] * (kScale * kScale), acc[i][q][r + 1] * (kScale * kScale)};
              if (finite(acc[i][q][r]) && finite(acc[i][q][r + 1]) && fabsf(c.x) >= kLarge && fabsf(c.y) >= kLarge)
                dst[om[i] + ocn] = c;
              else
                redo |= 1u << ((q * 8 + rr) * RM + i);
            }
          }
        }
        for (; redo; redo &= redo - 1) {
          const int bit = __builtin_ctz(redo), i = bit % RM, rr = bit / RM % 8, q = bit / RM / 8;
          const int nl = (wn * RN + q) * 16 + 4 * (rr >> 1) + 2 * half + (rr & 1);
          const uint32_t m = (wm * RM + i) * 32 + l32;
          const int g = FAN ? nl >> d.nbits : 0;
          const uint64_t pbg = FAN ? ws + s_bb[g] : pb;
          const uint32_t oa = dep<TAB_AM>(d, 8, m);
          const uint32_t ob = dep<TAB_BN>(d, 8, FAN ? (nl & nmask) : nl);
          float2 c = make_float2(0.f, 0.f);
          for (uint32_t k = k0; k < k0 + (uint32_t)ksteps * TK; ++k)
            cmac(c, ldg_f2(pa, oa + dep<TAB_AK>(d, d.kbits, k)), ldg_f2(pbg, ob + dep<TAB_BK>(d, d.kbits, k)));
          const gptr<f32x2> dst = FAN ? gmem<f32x2>(ws + s_cb[g]) : pc;
          dst[dep<TAB_CM>(d, 8, m) + s_cn[nl]] = f32x2{c.x, c.y};
        }
      }
      if (FAN) __syncthreads();  // the next tile rewrites the column data
    }
  }
}

// Adds the copies of a split sum in order.
__global__ __launch_bounds__(256) void k_split_add(NodeDesc d, uint64_t ws) {
  const int64_t total = d.n_inst << (d.mbits + d.nbits);
  const int parts = 1 << d.ksplit;
  const uint64_t src = ws + d.part_off, dst = ws + d.c_off;
  for (int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x; g < total; g += (int64_t)gridDim.x * 256) {
    float2 c = ldg_f2(src, g);
    for (int p = 1; p < parts; p += 1) {
      const float2 v = ldg_f2(src, (uint64_t)p * total + g);
      c.x += v.x;
      c.y += v.y;
    }
    stg_f2(dst, g, c);
  }
}

// ---------------------------------------------------------------------------
// launchers (the tile configurations are those of kernels_c64.hip; the two of
// 2^13 elements take eight waves, whose four tiles each leave room for both accumulators)

// Tiles of the smallest size up to which four k steps are in flight, for sums of
// at least 16: 6/6/10 bits x 40 (80 tiles) 85 -> 79 us, x 150 (300) 96 -> 84, but
// 6/5/8 x 600 (600) 36 -> 39 and 6/5/6 x 150 (150) 10.3 -> 10.4.
constexpr unsigned kFewTiles = 512;

template <bool FAN, bool LIN>
static hipError_t launch_split_s(const NodeDesc& d, int cfg, unsigned grid, uint64_t ws, const int64_t* sig,
                                hipStream_t st) {
  switch (cfg) {
    case 0: hipLaunchKernelGGL((k_split<2, 1, 2, 2, FAN, LIN>), dim3(grid), dim3(256), 0, st, d, ws, sig); break;
    case 1: hipLaunchKernelGGL((k_split<2, 2, 2, 2, FAN, LIN>), dim3(grid), dim3(256), 0, st, d, ws, sig); break;
    case 2:
      if (grid <= kFewTiles && d.kbits - d.ksplit >= 7)
        hipLaunchKernelGGL((k_split<1, 1, 2, 2, FAN, LIN, 4>), dim3(grid), dim3(256), 0, st, d, ws, sig);
      else
        hipLaunchKernelGGL((k_split<1, 1, 2, 2, FAN, LIN>), dim3(grid), dim3(256), 0, st, d, ws, sig);
      break;
    case 3: hipLaunchKernelGGL((k_split<4, 1, 2, 2, FAN, LIN>), dim3(grid), dim3(256), 0, st, d, ws, sig); break;
    case 4: hipLaunchKernelGGL((k_split<2, 2, 4, 2, FAN, LIN>), dim3(grid), dim3(512), 0, st, d, ws, sig); break;
    case 5:
      if (FAN) return hipErrorInvalidValue;
      hipLaunchKernelGGL((k_split<2, 2, 2, 4, false, LIN>), dim3(grid), dim3(512), 0, st, d, ws, sig);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <bool FAN>
static hipError_t launch_split_t(const NodeDesc& d, int cfg, uint64_t ws, const int64_t* sig, hipStream_t st) {
  if (d.n_inst == 0) return hipSuccess;
  const bool fits = FAN ? mfma_fan_config_fits(cfg, d.mbits, d.nbits, d.kbits, d.fan_tn)
                        : mfma_config_fits(cfg, d.mbits, d.nbits, d.kbits);
  if (!fits || (FAN && (d.w <= 0 || d.n_fan <= 0)) || d.A.half || d.B.half) return hipErrorInvalidValue;
  const int64_t units = FAN ? (d.n_inst / d.w) * d.n_fan : d.n_inst;
  const int tbits = d.mbits - mfma_config_tm_bits(cfg) + (FAN ? 0 : d.nbits - mfma_config_tn_bits(cfg));
  // persistent: see the in-tile offsets; 2048 workgroups as for the FP16 tiles
  const unsigned grid = (unsigned)std::min<int64_t>((units << tbits) << d.ksplit, 2048);
  hipError_t e;
  if (d.linear)
    e = launch_split_s<FAN, true>(d, cfg, grid, ws, sig, st);
  else if (FAN || d.ksplit)
    e = hipErrorInvalidValue;
  else  // a caller's own layout
    e = launch_split_s<false, false>(d, cfg, grid, ws, sig, st);
  if (e != hipSuccess || !d.ksplit) return e;
  const unsigned g2 = grid_for(((d.n_inst << (d.mbits + d.nbits)) + 255) / 256);
  hipLaunchKernelGGL(k_split_add, dim3(g2), dim3(256), 0, st, d, ws);
  return hipGetLastError();
}

int split_bits(int cfg, bool fan, int mbits, int nbits, int kbits, int64_t units) {
  const int tbits = mbits - mfma_config_tm_bits(cfg) + (fan ? 0 : nbits - mfma_config_tn_bits(cfg));
  const int64_t tiles = units << tbits;
  // two workgroups per CU need no split; below that, four per CU as long as a
  // part keeps 16 k steps
  int sb = 0;
  if (tiles < 512)
    while ((tiles << sb) < 1024 && kbits - sb > 7) ++sb;
  return sb;
}

hipError_t launch_split(const NodeDesc& d, int cfg, uint64_t ws, const int64_t* sig, hipStream_t st) {
  return launch_split_t<false>(d, cfg, ws, sig, st);
}

hipError_t launch_split_fan(const NodeDesc& d, int cfg, uint64_t ws, const int64_t* sig, hipStream_t st) {
  return launch_split_t<true>(d, cfg, ws, sig, st);
}

}  // namespace matnc
