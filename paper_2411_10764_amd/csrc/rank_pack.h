// Rank form of an ensemble of perfect trees: the layout the rank walks read
// (rank_kernels) and the host code that builds it.  Plain C++17 (no HIP), so
// that it also builds on its own for the CPU tests.
//
// A split only asks whether x[f] < t, and an ensemble has finitely many
// thresholds per feature.  So each feature value is replaced by a code that
// keeps every such answer: with the feature's distinct thresholds t_0 < t_1 <
// ... < t_{N-1}, code(x) = the number of thresholds that x is not below
// (NaN: N), and x < t_j exactly when code(x) < j + 1.  A node takes four
// bytes: {offset of the feature's code in the tile, comparand}.
//
// Codes of a feature come in one of two ways:
//   grid    the thresholds are multiples of a power of two h <= 1 in a short
//           range (integer knobs): code = clamp(floor(x / h) + bias, 0, top),
//           no table.  Codes then count grid points, present or not.
//   search  a table of the thresholds, cut into segments where it is longer
//           than a staging slot; a segment's count of thresholds not above x
//           adds to the code.  A segment is a perfect binary search tree in
//           breadth-first order (entry 1 the root, 2^steps entries, padded
//           with +inf): the lanes of a step read one run of 2^l entries, so
//           the LDS banks spread them, where the probes of a sorted list lie
//           a power of two apart in one bank (16M x 128 performance walk, 64
//           features of about 2,000 thresholds: 15.6 -> 14.5 ms).  An x that
//           is not below the padding (+inf, NaN) counts some of it; any code
//           past the last threshold's means the same.
//
// Where a code lies in the tile (the mode):
//   byte    every feature has at most 255 codes above 0: a byte each.
//   half    a half-word each (more than 4095 codes).
//   packed  a field of w = 4, 8 or 12 bits; a half-word holds 12 + 4, 8 + 8,
//           8 + 4 + 4 or 4 + 4 + 4 + 4 bits.  A walk shifts the half-word
//           left by s, so that the field ends at bit 15 with other fields'
//           bits below it, and compares with the node's low half C, whose low
//           four bits are s (the 16-bit shift reads no others).  With T = t <<
//           (16 - w), t the split's code: C = T for s = 0, else T - 16 + s.
//           The shifted half-word of code t - 1 is at most T - 2^s and that
//           of code t at least T, so C orders them as the split does (s is 0,
//           4, 8 or 12, and 16 - s < 2^s from 4 on).  In the other modes C
//           is t.
#pragma once

#include <stdint.h>
#include <stdlib.h>

#include <memory>
#include <vector>

#include "pack.h"

namespace ml2 {

constexpr int kRankLine = 16;         // features ranked from one 64-byte half-line of a row
constexpr int kRankMaxDepth = 12;
constexpr int kRankMinDepth = 4;
constexpr uint32_t kRankRow = 256;    // bytes of one tile row (64 candidates x 4 bytes)

// Bytes of a tree of depth D, and dwords of its top part: with K = min(D, 5),
// the nodes of levels 0 .. K-1 lie in order (as a binary search tree) in
// dwords 1 .. 2^K - 1, level l >= K in dwords 2^l .. 2^(l+1) - 1, and the
// leaves (float32) in dwords 2^D .. 2^(D+1) - 1.  idx, the decisions of a
// walk so far (1: x < t), most significant first, names a node of level l:
//   l < K: dword idx * 2^(K-l) + 2^(K-1-l);   l >= K: dword 2^l + idx.
inline constexpr uint32_t rank_tree_bytes(int D) { return 8u << D; }
inline constexpr int rank_top(int D) { return D < 5 ? D : 5; }

// Where a feature's code goes: bits 15..0 the byte offset of its dword in a
// candidate's column of the tile, bits 20..16 the field's lowest bit there,
// bit 31 set where the dword has been written before (the code is added).
constexpr uint32_t kRankAdd = 0x80000000u;

enum RankMode { kRankByte, kRankHalf, kRankPacked };

struct RankGrid {     // per feature; top = 0: not a grid feature
  float scale, bias, top;
  uint32_t put;
};
struct RankSeg {      // one table segment
  uint32_t lane_reg;  // bits 7..0 the feature within its line, 31..8 its thresholds here
  uint32_t put;       // kRankNone: a repeat that fills the group
  uint32_t table_off; // bytes from the start of the slot
  uint32_t steps;
};
constexpr uint32_t kRankNone = 0xFFFFFFFFu;
struct RankGroup {    // four segments of one line in one slot, searched together:
  RankSeg seg[4];     // the same steps for all
};
struct RankChunk {    // trees of one slot
  int32_t slot, offset, trees, pad;
};

struct FreeBytes {
  void operator()(char *p) const { free(p); }
};
struct RankPack {
  RankMode mode = kRankByte;
  int lines = 0, slots = 0, group = 0;
  uint32_t rows = 0;                   // dword rows of the tile
  size_t bytes = 0;                    // slots * slot_bytes
  std::unique_ptr<char[], FreeBytes> data;
  std::vector<RankGrid> grid;          // lines * kRankLine
  std::vector<int32_t> line_group;     // lines + 1: first group of each line
  std::vector<int32_t> group_slot;
  std::vector<RankGroup> groups;
  std::vector<RankChunk> chunks;
};

// The codes of every split: per-feature distinct thresholds and, for every
// node, j + 1.
struct RankField {
  uint32_t off;    // byte offset in the column of the byte or half-word read
  uint8_t low;     // the field's lowest bit in it
  uint8_t width;   // 0: the ensemble has no split on the feature
};
struct RankCodes {
  RankMode mode = kRankByte;
  uint32_t rows = 0;
  std::vector<RankField> field;           // per feature
  std::vector<std::vector<float>> table;  // per feature; empty for grid features
  std::vector<RankGrid> grid;             // per feature
  std::unique_ptr<uint16_t[]> code;       // per node, trees in order
};
bool rank_codes(const std::vector<TreeView> &views, int num_features, RankCodes *out);

// Packs tables and trees of depth D into slots of slot_bytes; `group` trees
// are walked together, so every chunk holds a multiple of it (padded with
// trees of -0.0 leaves).  False where a group does not fit a slot.
bool rank_pack(const std::vector<TreeView> &views, const RankCodes &codes, int num_features,
               int D, int group, uint32_t slot_bytes, RankPack *out);

// Ragged trees (layout.h: default directions, any depth) over codes.  A
// missing value has a code of its own, the largest of its width, so the codes
// take a byte (up to 254 thresholds, missing 255) or 13 bits of a half-word,
// shifted left by three (missing 8191).  Slots keep their headers, roots and
// node order; a node becomes
//   split  word 0 {byte offset of the left child, C}, word 1 {S, code offset}
//   leaf   word 0 {byte offset of the next root, 0xFFFF}, word 1 the value
// (high half, low half).  With y the code in the upper bits of 16 (a byte
// shifted left by eight) and u its unit (256 or 8), a walk computes z = y + S
// modulo 2^16 and goes right exactly when z > C: S = 0 and C = u (t - 1) send
// a missing value right, S = u and C = u t wrap it to 0 and send it left.
// z never exceeds 0xFFFF, so a leaf always takes its one way on.
constexpr int kRankRaggedByte = 255, kRankRaggedHalf = 8191;  // the missing codes
bool rank_pack_ragged(const RaggedPack &ragged, const RankCodes &codes, int num_features,
                      RankPack *out);
// The codes' places for ragged trees; false where a feature has too many.
bool rank_ragged_fields(RankCodes *codes);

}  // namespace ml2
