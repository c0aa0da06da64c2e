// Launch shapes of the rank walks (rank_pack.h): waves, workgroups per CU,
// slots and LDS.  Plain C++17 (no HIP), so that it also builds on its own for
// the CPU tests.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "rank_pack.h"

namespace ml2 {

constexpr size_t kLdsBudget = 160 * 1024 - 256;  // LDS of a walk workgroup (static LDS headroom)

// Registers (16 bytes each) per thread that stage one slot of at most 64 KiB.
constexpr int rank_stage_regs(int waves) { return (64 + waves - 1) / waves; }
// The same for a 24 KiB slot of ragged trees and the smallest workgroup of a
// class: of 24 waves that share a CU twelve, of 16 eight, of 12 twelve, of 8
// and of 4 four.
constexpr int rank_ragged_stage_regs(int waves) {
  return waves == 24 || waves == 12 ? 2 : waves == 16 ? 3 : 6;
}

// Trees walked together by a lane, per depth.
constexpr int kRankGroup[kRankMaxDepth + 1] = {0, 0, 0, 0, 8, 8, 8, 8, 8, 4, 4, 2, 1};

// Waves of a workgroup, workgroups of a CU, trees per lane and slot size.
struct RankShape {
  int32_t waves, per_cu, group;
  uint32_t slot_bytes;
};
// For tiles of `tile` bytes per wave and perfect trees of depth D, or ragged
// trees; false where no workgroup fits.
bool rank_shape(uint32_t tile, int D, RankShape *out);
bool rank_ragged_shape(uint32_t tile, RankShape *out);

// One launch over `units` units of 64 rows.
struct RankLaunch {
  int32_t waves, per_cu, grid;
  int32_t cls;  // register class: the most waves that share a CU
  size_t lds;
};
RankLaunch rank_launch(const RankShape &shape, uint32_t tile, bool ragged, int64_t units,
                       int cu_count, bool perf);
// Whether a launch's staging registers hold a slot and its LDS fits (else the
// slot's end would stay unwritten).
bool rank_stages_slot(const RankShape &shape, bool ragged, const RankLaunch &l);

// What the walks of an ensemble do, for the two estimates below.
struct WalkWork {
  int32_t ragged, features, depth;
  int32_t records;         // staged by the float walk: trees (padded) or ragged slots
  int32_t trees, slots;    // of the ensemble; of the rank form, tables included
  int32_t steps, grids;    // search steps and grid features of ranking a row
  double path;             // ragged: nodes on a row's walks, leaves included
};
// The shape of a float walk: lanes per candidate, waves, trees per lane,
// records per chunk, workgroups; copied: chunks are copied while the waves wait
// (else fetched ahead).
struct FloatShape {
  int32_t split, waves, group, chunk, grid, copied;
};
// How rows lie: loaded as whole 16-byte vectors and a round ahead, as vectors,
// or a float at a time.
enum RowKind { kRowsAhead, kRowsVector, kRowsSingle };
RowKind row_kind(bool aligned, int32_t features);

// Estimated time in microseconds of a walk over `rows` rows.
double float_walk_us(const WalkWork &w, const FloatShape &s, RowKind kind, double rows, int cus);
double rank_walk_us(const WalkWork &w, const RankShape &s, RowKind kind, double rows, int cus);
// Whether the rank walk takes such a call: where its estimate is the lower one, or
// no more than a tenth above.  The estimates err by about that much, and of
// 14,800 timed walks a tenth more or less left the mean where it was.
inline bool rank_walk_wins(const WalkWork &w, const FloatShape &f, const RankShape &r,
                           RowKind kind, double rows, int cus) {
  return rank_walk_us(w, r, kind, rows, cus) < 1.1 * float_walk_us(w, f, kind, rows, cus);
}
// Rows of n at which a walk over the rows that a mask accepts is priced.
inline double masked_rows(double n) { return 0.2 * n; }

// Ragged trees: the bits of a code's offset in the tile.
uint32_t rank_ragged_mask(uint32_t tile, RankMode mode);

}  // namespace ml2
