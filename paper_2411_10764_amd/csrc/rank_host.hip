// Loading, planning and launching of the rank form (rank_pack.h).
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <new>

#include "rank_walk.h"

namespace ml2 {
namespace {

constexpr uint32_t kMaxSlot = 64 * 1024;

// The register class of a kernel that shares a CU with `total` waves in all.
int wave_class(int total) { return total > 16 ? 24 : total > 12 ? 16 : total > 8 ? 12 : total > 4 ? 8 : 4; }

// Bytes that the staging registers of `waves` waves of a class hold.
size_t stage_bytes(int cls, int waves) {
  return (size_t)rank_stage_regs(cls) * 16 * rank::kLanes * waves;
}

size_t queue_bytes(int waves) { return (size_t)waves * 2 * rank::kLanes * sizeof(int32_t); }

// Waves per workgroup, workgroups per CU, trees per lane and slot size for
// tiles of `tile` bytes per wave and trees of depth D.  Two workgroups of
// eight waves first: one walks while the other waits at a barrier or for its
// rows (16M x 128 validity 7.20 -> 6.76 ms against one of sixteen).  They need
// room for a slot of two groups of trees each, or of 32 KiB (a shorter one
// spends the gain on restaging: 4M x 96, depth 8, 24 KiB slots: 3.83 ms, one
// workgroup of sixteen waves with 55 KiB: 3.64); else one workgroup of as many
// waves as leave that room, by fours, as each SIMD takes a fourth (16M x 128
// performance: twelve waves and a 58 KiB slot 14.5 ms, sixteen and 23 KiB
// 16.7, ten 16.4, eight 16.6).  Last, whatever holds one group.  False where
// no workgroup does.
bool shape(uint32_t tile, int D, RankForm *r) {
  struct Shape {
    int waves, per_cu;
  };
  const Shape shapes[] = {{8, 2}, {16, 1}, {12, 1}, {8, 1}, {7, 1}, {6, 1},
                          {5, 1}, {4, 1},  {3, 1},  {2, 1}, {1, 1}};
  const uint32_t RB = rank_tree_bytes(D);
  for (const bool roomy : {true, false}) {
    for (const auto &groups : rank::kGroups) {
      const uint32_t one = (uint32_t)groups[D] * RB;
      if (one == 0) continue;
      const uint32_t need = roomy ? std::min<uint32_t>(2 * one, 32 * 1024) : 8 * 1024;
      for (const Shape &sh : shapes) {
        const size_t fixed = (size_t)sh.waves * tile + queue_bytes(sh.waves);
        const size_t lds = kLdsBudget / sh.per_cu;
        if (fixed >= lds) continue;
        const uint32_t slot =
            (uint32_t)std::min({lds - fixed, (size_t)kMaxSlot,
                                stage_bytes(wave_class(sh.waves * sh.per_cu), sh.waves)}) & ~255u;
        if (slot < std::max(one, need)) continue;
        r->waves = sh.waves;
        r->per_cu = sh.per_cu;
        r->group = groups[D];
        r->slot_bytes = slot;
        return true;
      }
    }
  }
  return false;
}

// The same for ragged trees, whose slot is fixed.  The walk is bound by the
// latency of its chain of reads, so as many waves as fit, two workgroups of
// twelve first (16M x 128 round, 300 trees of depth up to 14 over 64
// features: 8 waves per CU 9.2 ms, 12 6.6, 16 5.4, 24 4.6).
size_t ragged_lds(uint32_t tile, int waves) {
  // a leaf reads a code within ragged_mask of its lane's column
  size_t past = kRankRow;
  while (past < tile) past *= 2;
  const size_t fixed = kRaggedChunkBytes + (size_t)waves * tile;
  return std::max(fixed + queue_bytes(waves) + waves * sizeof(int), fixed - tile + kRankRow + past);
}

uint32_t ragged_mask(uint32_t tile, RankMode mode) {
  uint32_t past = kRankRow;
  while (past < tile) past *= 2;
  return (past - 1) & (mode == kRankByte ? ~0xFCu : ~0xFDu);
}

bool ragged_shape(uint32_t tile, RankForm *r) {
  struct Shape {
    int waves, per_cu;
  };
  const Shape shapes[] = {{12, 2}, {16, 1}, {12, 1}, {8, 1}, {4, 1}};  // (four hold any tile)
  for (const Shape &sh : shapes) {
    if (ragged_lds(tile, sh.waves) * sh.per_cu > kLdsBudget) continue;
    r->waves = sh.waves;
    r->per_cu = sh.per_cu;
    r->group = 1;
    r->slot_bytes = kRaggedChunkBytes;
    return true;
  }
  return false;
}

template <typename T>
size_t place(size_t *at, const std::vector<T> &v) {
  const size_t o = *at;
  *at = (o + v.size() * sizeof(T) + 255) & ~(size_t)255;
  return o;
}

}  // namespace

void rank_load(const std::vector<TreeView> &views, const RaggedPack *ragged, Forest *f) {
  RankForm r{};
  f->rank = r;
  const int D = f->depth;
  if (!ragged && (D < kRankMinDepth || D > kRankMaxDepth)) return;
  try {
    RankCodes codes;
    if (!rank_codes(views, f->num_features, &codes)) return;
    if (ragged && !rank_ragged_fields(&codes)) return;
    r.tile_bytes = codes.rows * kRankRow;
    if (!(ragged ? ragged_shape(r.tile_bytes, &r) : shape(r.tile_bytes, D, &r))) return;
    // Ranking a row costs about 0.8 of a node visit per search step and one
    // per grid feature; a visit of the rank walk takes about 0.28 of a visit
    // less than one of the float walk, 0.56 where that cannot prefetch its
    // rows, and a ragged tree about nine visits less.  So small ensembles over
    // many features keep the float walks (412,590 x 136, 42 trees of depth 4:
    // 53 us against 109; 427,763 x 96, 190 of depth 6: 149 against 155; 16M x
    // 128, 300 of depth 6: 7.84 ms against 7.0).  Trees of depth 9 and above
    // leave those few trees per lane or few waves, and always rank (262,144 x
    // 96, 100 trees of depth 10: 193 us against 101; 500,000 x 256, 100 of
    // depth 12: 47.3 ms against 1.3).
    int64_t steps = 0, grids = 0;  // of ranking one row
    for (int32_t c = 0; c < f->num_features; ++c) {
      for (size_t n = codes.table[(size_t)c].size(); n; n >>= 1) ++steps;
      grids += codes.grid[(size_t)c].top != 0.0f;
    }
    const bool prefetched = f->num_features <= 128 && f->num_features % 4 == 0;
    const int64_t saves = ragged ? 450 * (int64_t)f->num_trees
                                 : (prefetched ? 14 : 28) * (int64_t)f->num_trees * D;
    if ((ragged || D < 9) && saves < 40 * steps + 50 * grids) return;
    RankPack p;
    if (!(ragged ? rank_pack_ragged(*ragged, codes, f->num_features, &p)
                 : rank_pack(views, codes, f->num_features, D, r.group, r.slot_bytes, &p)))
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

// From three quarters of a round of every CU on (196,608 rows with 16 waves a
// CU) a walk ranks where that pays.  Below, a walk takes as long as its
// longest lane, and the float walk's two lanes per candidate and shorter
// start win: validity, 300 trees of depth 6 over 128 features, 65,536 rows 38
// us against 84, 262,144 rows 129 against 132, 16M rows 7.84 ms against 7.0;
// performance, 177 trees of depth 7 over 76, 4,320 rows 28 us against 58.
// Not so where the float walk's plan holds at most eight walks per lane column
// (waves times trees per lane) and the pool has some rows per CU: 644 trees of
// depth 10 over 112 features, 167,534 rows 1,040 us against 400; 499 over 159,
// 54,335 rows 984 against 313; but 681 over 112 and 2,173 rows 362 against
// 394.
bool rank_takes(const Forest &f, int64_t n_work, const WalkPlan &plan, bool perf) {
  const RankForm &r = f.rank;
  if (!r.ok) return false;
  for (int t : {kTuneSplit, kTuneGroup, kTuneWaves, kTuneNbuf, kTuneChunk})
    if (get_tune(t) != 0) return false;  // the overrides shape the float walks
  if (n_work >= (int64_t)48 * r.waves * r.per_cu * plan.cus) return true;
  return perf && !f.ragged && plan.waves * plan.group <= 8 && n_work >= (int64_t)64 * plan.cus;
}

namespace {

struct Launch {
  int grid, cls;
  size_t lds;
};

// The launch shape for n rows: as many workgroups as the chip holds or the
// pool has units of 64 rows, of no more waves than a workgroup has units.
RankArgs args_for(const Forest &f, const float *X, int64_t n, int64_t ld, int cu_count,
                  bool perf, Launch *l) {
  const RankForm &r = f.rank;
  const int64_t units = (n + rank::kLanes - 1) / rank::kLanes;
  int w = r.waves, per_cu = r.per_cu;
  if (units <= (int64_t)cu_count * 8) per_cu = 1;
  for (int less : {12, 8, 4})
    if (less < w && units <= (int64_t)cu_count * per_cu * less) w = less;
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
  a.slot_bytes = r.slot_bytes;
  a.tile_bytes = r.tile_bytes;
  a.nthreads = w * rank::kLanes;
  a.vec4 = ((reinterpret_cast<uintptr_t>(X) & 15u) == 0 && (ld & 3) == 0 &&
            (f.num_features & 3) == 0)
               ? 1
               : 0;
  a.base = f.base;
  a.missing = r.mode == kRankByte ? kRankRaggedByte : kRankRaggedHalf;
  a.off_mask = ragged_mask(r.tile_bytes, (RankMode)r.mode);
  l->lds = f.ragged ? ragged_lds(r.tile_bytes, w)
                    : (size_t)w * r.tile_bytes + r.slot_bytes + (perf ? queue_bytes(w) : 0);
  l->cls = wave_class(w * per_cu);
  l->grid = (int)std::max<int64_t>(1, std::min<int64_t>(units, (int64_t)cu_count * per_cu));
  return a;
}

}  // namespace

// A slot must fit the staging registers of the launch, or its end would stay
// unwritten.
static bool stages_slot(const Forest &f, const RankArgs &a, const Launch &l) {
  const int regs = f.ragged ? rank_ragged_stage_regs(l.cls) : rank_stage_regs(l.cls);
  return (size_t)regs * 16 * a.nthreads >= a.slot_bytes && l.lds <= kLdsBudget;
}

hipError_t launch_rank_validity(const Forest &f, const float *X, int64_t n, int64_t ld,
                                uint8_t *valid_out, float *margin_out, int cu_count,
                                hipStream_t s) {
  Launch l{};
  RankArgs a = args_for(f, X, n, ld, cu_count, false, &l);
  if (!stages_slot(f, a, l)) return hipErrorInvalidValue;
  a.valid_out = valid_out;
  a.margin_out = margin_out;
  if (f.ragged)
    return launch_rank_ragged_kernel(false, (RankMode)f.rank.mode, l.cls, a, l.grid, l.lds, s);
  return launch_rank_validity_kernel(f.rank.depth, (RankMode)f.rank.mode, f.rank.group,
                                     l.cls, a, l.grid, l.lds, s);
}

hipError_t launch_rank_perf(const Forest &f, const float *X, int64_t n, int64_t ld,
                            const uint8_t *valid, float *score_out, int cu_count,
                            hipStream_t s) {
  Launch l{};
  RankArgs a = args_for(f, X, n, ld, cu_count, true, &l);
  if (!stages_slot(f, a, l)) return hipErrorInvalidValue;
  a.valid_in = valid;
  a.score_out = score_out;
  if (f.ragged)
    return launch_rank_ragged_kernel(true, (RankMode)f.rank.mode, l.cls, a, l.grid, l.lds, s);
  return launch_rank_perf_kernel(f.rank.depth, (RankMode)f.rank.mode, f.rank.group,
                                 l.cls, a, l.grid, l.lds, s);
}

}  // namespace ml2
