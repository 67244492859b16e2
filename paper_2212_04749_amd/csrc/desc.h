// Device-visible descriptors of one contraction-tree node.
//
// Every index has dimension 2, so a tensor of rank r is 2^r elements and an
// element offset is a sum of independent bit contributions: the element at
// coordinates (m, n, k) of the pairwise step C[m, n] = sum_k A[m, k] B[k, n]
// sits at offset T_Am(m) + T_Ak(k) in A, T_Bk(k) + T_Bn(n) in B and
// T_Cm(m) + T_Cn(n) in C, which is how the index permutation of every operand
// is fused into its loads and stores.  Kernels form T_* from the storage bit of
// each coordinate bit (NodeDesc::pos, uint32 element offsets; ranks <= 32);
// k_mfma alone reads it from four 256-entry tables of 8 coordinate bits each.
#pragma once
#include <stdint.h>

namespace matnc {

constexpr int kMaxLeafSliced = 16;
constexpr int kTabLevels = 4;
constexpr int kTabEntries = 256;
constexpr int kTabSize = kTabLevels * kTabEntries;  // uint32 per class table

// table classes inside a node's table block
enum TabClass { TAB_AM = 0, TAB_CM = 1, TAB_BN = 2, TAB_CN = 3, TAB_AK = 4, TAB_BK = 5, TAB_COUNT = 6 };

// How one node reads one operand instance.  For output instance (s, j)
// (slice s of the batch, reuse-tree key j of the node):
//   inst = gmap[j] * nsv + sub(sigma) + (dep ? s * w_child : 0)
// where sub(sigma) gathers the sigma bits sbit[0..nsb) into an nsv-index
// (leaves holding sliced indices), and dep marks an intermediate operand
// whose instances are stored per slice.
struct OpDesc {
  uint64_t off;         // byte offset of instance 0 in the workspace
  uint64_t inst_bytes;  // bytes per instance
  uint64_t gmap_off;    // byte offset of the int32 gather map (one entry per j)
  uint64_t scale_off;   // complex-half: byte offset of the {int32 e, uint32 max} pair of instance 0
  int32_t w_child;      // instances per slice of the operand
  int32_t dep;          // 1: operand instances repeat per slice
  int32_t nsv;          // leaf: 2^nsb slice variants per key; else 1
  int32_t nsb;          // number of sliced indices on the leaf
  int32_t half;         // complex-half plans: 1 = stored as FP16 with scales, 0 = FP32
  int32_t pad0;
  int8_t sbit[kMaxLeafSliced];  // sigma bit of each sliced index
};

struct NodeDesc {
  OpDesc A, B;
  uint64_t c_off;        // byte offset of output instance 0
  uint64_t c_inst_bytes; // bytes per output instance
  uint64_t tab_off;      // steps on k_mfma: byte offset of the TAB_COUNT x kTabSize uint32 tables (no others have any)
  uint64_t c_scale_off;  // complex-half: byte offset of the output's {e, max} pairs
  int64_t n_inst;        // instances in this launch = w * (dep ? batch : 1)
  int32_t w;             // reuse-tree width w(v)
  int32_t dep;           // output instances repeat per slice
  int32_t mbits, nbits, kbits;
  int32_t c_half;        // complex-half plans: output stored as FP16 (1) or FP32 (0)
  // fan-out grouping (MFMA steps with few output columns whose A instance
  // is shared by several output instances): row g of the int32 table at
  // fan_off lists up to fan_tn >> nbits output instances j (-1 = empty
  // slot) that all read the same A instance; they are computed together as
  // one GEMM whose fan_tn columns are the slots' own B columns side by side
  // (fan_tn = the N width of the tile configuration)
  uint64_t fan_off;
  int64_t n_fan;         // rows of the fan table (per slice)
  int32_t fan_tn;
  // tile order: units (output instances, or fan-table rows) in blocks of
  // fan_rows with the units innermost (see unit_tile); 1 (plain) or 2 (fan
  // tables), or about the number of units that share one A instance when
  // that instance is too large for the caches
  int32_t fan_rows;
  int32_t flat;          // 1: output instance i reads instance i of A and of B (no gather map, no slices)
  int32_t s0;            // split sums: slices of the batch before this launch's first one
  // Instances that the choice of an order of additions goes by: a plan's keys
  // of the node, whatever the slice batch or key chunk of this launch, so that
  // results do not depend on how slices and keys are grouped
  int64_t n_ref;
  int32_t keep_order;    // 1: sums keep the order of additions fixed by the shape (plans with FP16 tensors)
  int32_t linear;        // 1: A[m + (k << mbits)] and B[n + (k << nbits)]
  int32_t ks_bits;       // long-sum kernel: 2^ks_bits lane groups share a sum
  // split sums (matrix-core steps of a plan with few tiles and a long sum): the
  // sum is cut into 2^ksplit parts, each a tile of its own writing to its own
  // copy of the output at part_off (c layout, n_inst instances per part); a
  // second kernel adds the copies in order.  The copies lie in the arena for as
  // long as the step runs; where they have room for fewer slices than the batch
  // has, the step runs in several launches (s0)
  int32_t ksplit;
  uint64_t part_off;
  // storage bit of coordinate bit t, per table class: offsets from these cost
  // a kernel two VALU operations per bit (none for wave-uniform coordinates)
  // and no table in memory
  int8_t pos[TAB_COUNT][32];
};

// Scaling of one stored instance in complex-half plans: true value = stored
// value * 2^e (e = 0 for FP32 storage); mx = largest |re| or |im| of the
// stored values (float bits, so that unsigned atomicMax orders it).
struct HalfScale {
  int32_t e;
  uint32_t mx;
};

// Fused subtrees of small steps (kernels_tree.hip): a table of n_comp + 1
// word offsets, then each component's words: TreeHeader, the inputs, the
// steps, level starts (n_levels + 1 positions in the item list), the items
// (step << 16 | chunk of 64 >> cut outputs) and the gather maps.  Offsets in the header
// and in TreeStep::gmap count words from the component's first.
constexpr int kTreeThreads = 1024;
constexpr int kTreeWords = 6 * 1024;    // 24 KiB of description
constexpr int kTreeElems = 16 * 1024;   // 128 KiB of tensors
constexpr int kTreeMaxBits = 12;        // output bits of one instance
constexpr int kTreeBig = 256;           // elements of an input that a wave loads at once

struct TreeHeader {
  uint32_t n_levels, n_inputs, inputs, steps, levels, items;
  uint32_t n_big;           // the first inputs: more than kTreeBig elements, copied by all waves
};

struct TreeInput {
  uint32_t off_lo, off_hi;  // byte offset of instance 0 in the workspace
  uint32_t lds;             // first element in LDS
  uint32_t ebits, keys;     // instances of 2^ebits elements
  uint32_t nsb;             // leaf: sliced indices; instance = key * 2^nsb + their bits of sigma
  uint32_t sbit[4];         // sigma bit of each, one byte per index
};

struct TreeStep {
  uint32_t bits;            // m | n << 8 | k << 16 | (result to the arena) << 24 | cut << 25: 2^cut lanes share a sum
  uint32_t outputs;         // w << (m + n)
  uint32_t a, b;            // operands' first elements in LDS: (k, m) and (k, n), k highest
  uint32_t c_lo, c_hi;      // LDS element, or byte offset in the workspace
  uint32_t w;               // instances per slice
  uint32_t gmap;            // B instance << 16 | A instance, per output instance; 0: instance 0 of both
  uint32_t pos[3];          // storage bit of output coordinate bit t (m bits, then n bits), one byte each
};

__host__ __device__ inline int64_t sub_index(const OpDesc& o, int64_t sigma) {
  int64_t v = 0;
  for (int t = 0; t < o.nsb; ++t) v |= ((sigma >> o.sbit[t]) & 1) << t;
  return v;
}

}  // namespace matnc
