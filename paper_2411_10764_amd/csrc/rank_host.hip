// Loading, planning and launching of the rank form (rank_pack.h).
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <new>

#include "rank_walk.h"

namespace ml2 {
namespace {

template <typename T>
size_t place(size_t *at, const std::vector<T> &v) {
  const size_t o = *at;
  *at = (o + v.size() * sizeof(T) + 255) & ~(size_t)255;
  return o;
}

FloatShape float_shape(const WalkPlan &p) {
  return FloatShape{p.split, p.waves, p.group, p.chunk_trees, p.grid, p.copied};
}

WalkWork work_of(const std::vector<TreeView> &views, const RankCodes &codes, const Forest &f,
                 const RankShape &shape, double path) {
  WalkWork w{};
  w.ragged = f.ragged;
  w.features = f.num_features;
  w.depth = f.depth;
  w.records = f.records;
  w.trees = (int32_t)views.size();
  w.path = path;
  size_t tables = 0;
  for (int32_t c = 0; c < f.num_features; ++c) {
    int32_t steps = 0;
    for (size_t n = codes.table[(size_t)c].size(); n; n >>= 1) ++steps;
    w.steps += steps;
    tables += steps ? (size_t)4 << steps : 0;
    w.grids += codes.grid[(size_t)c].top != 0.0f;
  }
  const size_t trees = f.ragged ? (size_t)f.records * shape.slot_bytes
                                : views.size() * rank_tree_bytes(f.depth);
  w.slots = (int32_t)((tables + trees + shape.slot_bytes - 1) / shape.slot_bytes);
  return w;
}

// Ensembles that are small beside the searches of a row keep the float form
// alone, whatever the estimates say: of 970 timed walks of such ensembles over
// aligned rows ranking won by a tenth in 12 %, by 35 us (412,590 x 136, 42 trees
// of depth 4: 53 us against 109; 427,763 x 96, 190 of depth 6: 149 against 155;
// 16M x 128, 300 of depth 6, not small: 7.84 ms against 7.0), and loading a
// second form takes longer than that.  (Rows loaded a float at a time are
// another matter: ranking won 80 % of 877 such walks, by 110 us in the median.)
// In node visits per row, a visit saves 0.28 (0.56 where the float walk cannot
// prefetch its rows), a ragged tree 9, and ranking costs 0.8 per search step and
// 1 per grid feature.  Trees of depth 9 and above leave the float walk few trees
// per lane or few waves, and are never small (500,000 x 256, 100 of depth 12:
// 47.3 ms against 1.3).
bool small(const WalkWork &w) {
  if (!w.ragged && w.depth >= 9) return false;
  const bool prefetched = row_kind(true, w.features) == kRowsAhead;
  const int64_t saves = w.ragged ? 450 * (int64_t)w.trees
                                 : (prefetched ? 14 : 28) * (int64_t)w.trees * w.depth;
  return saves < 40 * (int64_t)w.steps + 50 * (int64_t)w.grids;
}

// Whether the estimates ever choose the form: of 16 million rows, aligned or
// not.  Few deep trees over many features and ragged trees of one or two
// splits do not (1 million rows, 10 trees of depth 9 over 128 features 152 us
// against 209; 20 ragged stumps 168 against 390 at 1.5 million).
bool ever_pays(const Forest &f, const RankForm &r, int cu_count) {
  const double n = 1 << 24;
  WalkPlan p;
  const char *why = nullptr;
  if (!plan_walk(f, (int64_t)n, cu_count, &p, &why, false, false)) return false;
  for (bool aligned : {true, false}) {
    const RowKind kind = row_kind(aligned, f.num_features);
    if (rank_walk_wins(r.work, float_shape(p), r.shape, kind, n, cu_count)) return true;
  }
  return false;
}

}  // namespace

void rank_load(const std::vector<TreeView> &views, const RaggedPack *ragged, double path,
               int cu_count, Forest *f) {
  RankForm r{};
  f->rank = r;
  const int D = f->depth;
  if (!ragged && (D < kRankMinDepth || D > kRankMaxDepth)) return;
  try {
    RankCodes codes;
    if (!rank_codes(views, f->num_features, &codes)) return;
    if (ragged && !rank_ragged_fields(&codes)) return;
    r.tile_bytes = codes.rows * kRankRow;
    if (!(ragged ? rank_ragged_shape(r.tile_bytes, &r.shape)
                 : rank_shape(r.tile_bytes, D, &r.shape)))
      return;
    r.work = work_of(views, codes, *f, r.shape, path);
    if (small(r.work) || !ever_pays(*f, r, cu_count)) return;
    RankPack p;
    if (!(ragged ? rank_pack_ragged(*ragged, codes, f->num_features, &p)
                 : rank_pack(views, codes, f->num_features, D, r.shape.group, r.shape.slot_bytes, &p)))
      return;
    size_t bytes = p.bytes + kTreeSlack;  // staging reads whole register sets past a slot
    const size_t o_slots = 0, o_grid = place(&bytes, p.grid),
                 o_lg = place(&bytes, p.line_group), o_gs = place(&bytes, p.group_slot),
                 o_gr = place(&bytes, p.groups), o_ch = place(&bytes, p.chunks);
    const size_t tail = p.bytes;  // zeros and the small tables
    std::vector<char> host(bytes - tail, 0);
    auto put = [&](size_t o, const auto &v) {
      if (!v.empty()) memcpy(host.data() + (o - tail), v.data(), v.size() * sizeof(v[0]));
    };
    put(o_grid, p.grid);
    put(o_lg, p.line_group);
    put(o_gs, p.group_slot);
    put(o_gr, p.groups);
    put(o_ch, p.chunks);
    if (hipMalloc(&r.block, bytes) != hipSuccess) {
      (void)hipGetLastError();  // the float walks need none of it
      return;
    }
    if (hipMemcpy(r.block, p.data.get(), tail, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(static_cast<char *>(r.block) + tail, host.data(), host.size(),
                  hipMemcpyHostToDevice) != hipSuccess) {
      (void)hipGetLastError();
      (void)hipFree(r.block);
      return;
    }
    char *b = static_cast<char *>(r.block);
    r.slots = b + o_slots;
    r.grid = b + o_grid;
    r.line_group = b + o_lg;
    r.group_slot = b + o_gs;
    r.groups = b + o_gr;
    r.chunks = b + o_ch;
    r.depth = D;
    r.nslots = p.slots;
    r.nchunks = (int32_t)p.chunks.size();
    r.nlines = p.lines;
    r.mode = p.mode;
    r.ok = 1;
    f->rank = r;
  } catch (const std::bad_alloc &) {
  }
}

void rank_free(Forest *f) {
  if (f->rank.block) (void)hipFree(f->rank.block);
  f->rank = RankForm{};
}

// A walk ranks where the estimates choose it, from three
// quarters of a round of every CU on (196,608 rows with 16 waves a CU): below,
// a walk takes as long as its longest lane, and the float walk's two lanes per
// candidate and shorter start win (validity, 300 trees of depth 6 over 128
// features, 65,536 rows 38 us against 84; performance, 177 trees of depth 7
// over 76, 4,320 rows 28 us against 58).  Not so where the float walk's plan
// holds at most eight walks per lane column (waves times trees per lane) and
// the pool has some rows per CU: 644 trees of depth 10 over 112 features,
// 167,534 rows 1,040 us against 400; 499 over 159, 54,335 rows 984 against
// 313; but 681 over 112 and 2,173 rows 362 against 394.
//
// How many rows a mask accepts is known on the device only, and a walk over
// few is the float walk's (300 trees of depth 6 over 128 features, 1 million
// rows: 30,000 accepted 40 us against 87, 300,000 213 and 212, 600,000 368 and
// 326).  Such a walk is priced at a fifth of its rows.  Of 7,500 timed ones, the
// walk taken is more than 5 % slower than the float walk for 12 % of those with
// 5 to 15 % accepted (priced at every row: 18 %), 3 % up to 35 % (4 %) and 1 %
// above; a seventh instead gives away more above (5 instead of 3 % of the time).
bool rank_takes(const Forest &f, const float *X, int64_t n, int64_t ld, const WalkPlan &plan,
                bool perf, bool masked) {
  const RankForm &r = f.rank;
  if (!r.ok) return false;
  for (int t : {kTuneSplit, kTuneGroup, kTuneWaves, kTuneNbuf, kTuneChunk})
    if (get_tune(t) != 0) return false;  // the overrides shape the float walks
  const bool round = n >= (int64_t)48 * r.shape.waves * r.shape.per_cu * plan.cus;
  const bool few_walks =
      perf && !f.ragged && plan.waves * plan.group <= 8 && n >= (int64_t)64 * plan.cus;
  if (!round && !few_walks) return false;
  const bool aligned = (reinterpret_cast<uintptr_t>(X) & 15u) == 0 && (ld & 3) == 0;
  const RowKind kind = row_kind(aligned, f.num_features);
  const double rows = masked ? masked_rows((double)n) : (double)n;
  return rank_walk_wins(r.work, float_shape(plan), r.shape, kind, rows, plan.cus);
}

// The arguments of a launch over n rows.
static RankArgs args_for(const Forest &f, const float *X, int64_t n, int64_t ld, int cu_count,
                         bool perf, RankLaunch *l) {
  const RankForm &r = f.rank;
  *l = rank_launch(r.shape, r.tile_bytes, f.ragged != 0, (n + rank::kLanes - 1) / rank::kLanes,
                   cu_count, perf);
  RankArgs a{};
  a.X = X;
  a.n = n;
  a.ld = ld;
  a.slots = static_cast<const char *>(r.slots);
  a.grid = static_cast<const RankGrid *>(r.grid);
  a.line_group = static_cast<const int32_t *>(r.line_group);
  a.groups = static_cast<const RankGroup *>(r.groups);
  a.group_slot = static_cast<const int32_t *>(r.group_slot);
  a.chunks = static_cast<const RankChunk *>(r.chunks);
  a.nslots = r.nslots;
  a.nchunks = r.nchunks;
  a.nlines = r.nlines;
  a.F = f.num_features;
  a.slot_bytes = r.shape.slot_bytes;
  a.tile_bytes = r.tile_bytes;
  a.nthreads = l->waves * rank::kLanes;
  a.vec4 = ((reinterpret_cast<uintptr_t>(X) & 15u) == 0 && (ld & 3) == 0 &&
            (f.num_features & 3) == 0)
               ? 1
               : 0;
  a.base = f.base;
  a.missing = r.mode == kRankByte ? kRankRaggedByte : kRankRaggedHalf;
  a.off_mask = rank_ragged_mask(r.tile_bytes, (RankMode)r.mode);
  return a;
}

hipError_t launch_rank_validity(const Forest &f, const float *X, int64_t n, int64_t ld,
                                uint8_t *valid_out, float *margin_out, int cu_count,
                                hipStream_t s) {
  RankLaunch l{};
  RankArgs a = args_for(f, X, n, ld, cu_count, false, &l);
  if (!rank_stages_slot(f.rank.shape, f.ragged != 0, l)) return hipErrorInvalidValue;
  a.valid_out = valid_out;
  a.margin_out = margin_out;
  if (f.ragged)
    return launch_rank_ragged_kernel(false, (RankMode)f.rank.mode, l.cls, a, l.grid, l.lds, s);
  return launch_rank_validity_kernel(f.rank.depth, (RankMode)f.rank.mode, l.cls, a, l.grid, l.lds, s);
}

hipError_t launch_rank_perf(const Forest &f, const float *X, int64_t n, int64_t ld,
                            const uint8_t *valid, float *score_out, int cu_count,
                            hipStream_t s) {
  RankLaunch l{};
  RankArgs a = args_for(f, X, n, ld, cu_count, true, &l);
  if (!rank_stages_slot(f.rank.shape, f.ragged != 0, l)) return hipErrorInvalidValue;
  a.valid_in = valid;
  a.score_out = score_out;
  if (f.ragged)
    return launch_rank_ragged_kernel(true, (RankMode)f.rank.mode, l.cls, a, l.grid, l.lds, s);
  return launch_rank_perf_kernel(f.rank.depth, (RankMode)f.rank.mode, l.cls, a, l.grid, l.lds, s);
}

}  // namespace ml2
