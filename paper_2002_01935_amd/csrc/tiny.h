// Tables of the small-contraction kernel (tiny.hip): shared by the planner,
// which fills them, and the device code.  Not part of the public ABI.
//
// A circuit network has hundreds of contractions of a few dozen values each
// (gate merges) at the bottom of its tree.  The planner collects connected
// sets of them into groups (tiny_group.h); one workgroup runs a group: it
// loads the group's external operands into LDS at once, then works level by
// level (a level's contractions do not depend on each other) with every
// intermediate in LDS, and stores only the values that other ops read.
//
// A launch's tables form one blob, passed as a kernel argument: a directory
// (TinyDir per group), then per group, from 16-byte aligned offsets: levels
// and contractions (copied to LDS as one block), loads, and the loads'
// extended records.
#pragma once

#include "tn_internal.h"

namespace tn {

constexpr int kTinyClasses = 9;          // contractions on 2^10 .. 2^2 threads
constexpr int kTinyMaxThreadBits = 10;
constexpr int kTinyMinThreadBits = 2;
constexpr int kTinyAbsent = 15;          // nibble of a bit that an operand does not have

struct TinyDir {
  uint32_t tab_off;      // byte offset in the blob of the level table, the contractions right behind it
  uint32_t tab_units;    // 16-byte units of both
  uint32_t ops_off;      // byte offset of the contractions within that block
  uint32_t n_levels;
  uint32_t ld_off;       // byte offset in the blob of the loads (TinyLoad)
  uint32_t n_loads;
  uint32_t ext_off;      // byte offset in the blob of the extended records (TinyExt)
  uint32_t pad;
};

// One level: its contractions in falling order of their thread counts 2^10 ..
// 2^2, so that each starts at a multiple of its own count.  In units of four
// threads: class c (2^(10 - c) threads each) ends at end[c] and begins with
// contraction first[c]; end[kTinyClasses - 1] is the level's total.
struct TinyLevel {
  uint16_t end[kTinyClasses], first[kTinyClasses];
  uint16_t pad[6];
};

// 2^n_bits values copied to LDS: from pointer-table slot `src` (kind 0) or
// arena offset 256 * src (kind 1) in storage order, or (kind 2) through the
// extended record `src`.
struct TinyLoad {
  uint32_t src;
  uint16_t lds;          // element offset
  uint8_t kind, n_bits;
};

// A leaf whose values are not one run of memory (sliced axes): value bit i at
// position pos[i].
struct TinyExt {
  Ref ref;
  int8_t pos[16];
};

// C[o] = sum over k of opA(A[o, k]) opB(B[o, k]) over LDS operands; C's bits
// are enumerated in storage order.  Nibble i of oa / ob (ka / kb): position of
// output bit i (summed bit i) in A / B.  2^ks threads share an output, each
// summing 2^(n_k - ks) consecutive k.
struct TinyOp {
  uint32_t dst;          // external copy of C: arena offset / 256 (dst_kind 1) or pointer-table slot (2)
  uint16_t a, b, c;      // LDS element offsets
  uint8_t n_out, n_k, ks;
  uint8_t conj;          // bit 0: A, bit 1: B
  uint8_t dst_kind;      // 0: none
  uint8_t lds_c;         // C is read by a later contraction of the group
  uint64_t oa, ob, ka, kb;
};

// One leaf gradient of a scatter launch: the cotangent at arena offset
// 256 * src (2^n_bits values, compact) is added into pointer-table slot
// `slot`, bit i at position pos[i], in the block of each in-flight slice.
struct ScatterEntry {
  uint32_t src, slot;
  uint8_t n_bits, n_slice;
  uint8_t slice_bit[kMaxSliceTerms], slice_pos[kMaxSliceTerms];
  uint8_t pos[14];
};

static_assert(sizeof(ScatterEntry) == 40, "table layout");
static_assert(sizeof(TinyDir) == 32 && sizeof(TinyLevel) == 48 && sizeof(TinyLoad) == 8, "table layout");
static_assert(sizeof(TinyOp) == 48 && sizeof(TinyExt) % 8 == 0, "table layout");

// Blob sizes the kernel is instantiated for (bytes of kernel argument).
constexpr int kTinyBlobSmall = 4096, kTinyBlobMid = 12288, kTinyBlobLarge = 28672;

}  // namespace tn
