// Host side of the rank form (rank_pack.h).
#include "rank_pack.h"

#include "host_parallel.h"

#include <math.h>
#include <string.h>

#include <algorithm>
#include <memory>
#include <new>

namespace ml2 {
namespace {

uint32_t bits_of(float v) {
  uint32_t b;
  memcpy(&b, &v, 4);
  return b;
}

float float_of(uint32_t b) {
  float v;
  memcpy(&v, &b, 4);
  return v;
}

// Order-preserving key of a threshold; -0.0 and +0.0 are the same threshold.
uint32_t key_of(float t) {
  const uint32_t b = bits_of(t == 0.0f ? 0.0f : t);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

float value_of(uint32_t key) {
  return float_of((key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key);
}

struct Entry {
  uint32_t key, node;
};

// Thresholds of one feature: a code, the padding of its last segment
// included, fits 16 bits.
constexpr size_t kMostThresholds = 65535 - 8192;

// Stable LSD radix sort by key in `passes` digits of B bits; the result is in
// e (passes even) or tmp.
template <int B>
void radix_passes(Entry *e, Entry *tmp, size_t n, int passes) {
  constexpr int kMost = 4;
  constexpr uint32_t mask = (1u << B) - 1;
  uint32_t count[kMost][1 << B] = {{0}};
  for (size_t i = 0; i < n; ++i)
    for (int pass = 0; pass < passes; ++pass) ++count[pass][(e[i].key >> (pass * B)) & mask];
  for (int pass = 0; pass < passes; ++pass) {
    uint32_t at = 0;
    for (uint32_t &c : count[pass]) {
      const uint32_t k = c;
      c = at;
      at += k;
    }
    for (size_t i = 0; i < n; ++i)
      tmp[count[pass][(e[i].key >> (pass * B)) & mask]++] = e[i];
    std::swap(e, tmp);
  }
}

// By key, ascending: comparisons for a few entries, else radix digits small
// enough for their counters not to cost more than the entries (1,000 entries:
// 40 us by comparisons, 8 us by bytes).
void sort_entries(Entry *e, Entry *tmp, size_t n) {
  if (n < 64) {
    std::sort(e, e + n, [](const Entry &a, const Entry &b) { return a.key < b.key; });
  } else if (n < 8192) {
    radix_passes<8>(e, tmp, n, 4);
  } else {
    radix_passes<11>(e, tmp, n, 3);
    memcpy(e, tmp, n * sizeof(Entry));
  }
}

// The exponent of the lowest set bit of v (not 0): v is a multiple of 2^that.
int low_bit(float v) {
  const uint32_t b = bits_of(v), e = (b >> 23) & 0xFFu;
  const uint32_t m = (b & 0x7FFFFFu) | (e ? 0x800000u : 0u);
  return (int)(e ? e : 1u) - 150 + __builtin_ctz(m);
}

// The grid of a sorted list of distinct thresholds: multiples of a power of
// two h <= 1 whose range holds at most `most` points.  h is not above 1, so
// x / h never rounds towards zero (no underflow) and floor(x / h) < t / h
// exactly when x < t; overflow to infinity keeps the order.  Most lists that
// have none are known by their first few thresholds.
bool find_grid(const std::vector<float> &t, int most, RankGrid *g) {
  if (!std::isfinite(t.front()) || !std::isfinite(t.back())) return false;
  const double range = (double)t.back() - (double)t.front();
  int e = 0;  // h = 2^e
  for (float v : t) {
    if (v == 0.0f || low_bit(v) >= e) continue;
    e = low_bit(v);
    if (e < -100 || ldexp(range, -e) + 1.0 > (double)most) return false;
  }
  const double lo = ldexp((double)t.front(), -e), hi = ldexp((double)t.back(), -e);
  if (fabs(lo) > 4194304.0 || fabs(hi) > 4194304.0 || hi - lo + 1.0 > (double)most) return false;
  g->scale = (float)ldexp(1.0, -e);
  g->bias = (float)(1.0 - lo);
  g->top = (float)(hi - lo + 1.0);
  return true;
}

// Keys of n entries that have at most kFewKeys distinct ones: those, ascending,
// and place[i] the one of entry i; 0 where there are more.  (The splits on a
// knob of nine values have nine thresholds: 4 ns an entry, 25 by sorting.)
constexpr int kFewKeys = 24;
int few_keys(const Entry *e, size_t n, uint32_t (&keys)[kFewKeys], uint8_t *place) {
  constexpr int kBuckets = 64;
  uint32_t seen[kFewKeys];
  int8_t bucket[kBuckets];  // an index into seen, -1: none
  memset(bucket, -1, sizeof bucket);
  int m = 0;
  for (size_t i = 0; i < n; ++i) {
    const uint32_t key = e[i].key;
    uint32_t h = (key * 0x9E3779B1u) >> 26;
    while (bucket[h] >= 0 && seen[bucket[h]] != key) h = (h + 1) % kBuckets;
    if (bucket[h] < 0) {
      if (m == kFewKeys) return 0;
      bucket[h] = (int8_t)m;
      seen[m++] = key;
    }
    place[i] = (uint8_t)bucket[h];
  }
  std::copy(seen, seen + m, keys);
  std::sort(keys, keys + m);
  uint8_t at[kFewKeys];
  for (int j = 0; j < m; ++j) at[j] = (uint8_t)(std::lower_bound(keys, keys + m, seen[j]) - keys);
  for (size_t i = 0; i < n; ++i) place[i] = at[place[i]];
  return m;
}

// The node of a split: its feature's half-word and the comparand of code t.
uint32_t node_word(const RankCodes &c, int feat, uint32_t t) {
  const RankField &fd = c.field[(size_t)feat];
  if (c.mode != kRankPacked) return (fd.off << 16) | t;
  const uint32_t s = 16u - fd.low - fd.width, T = t << (16 - fd.width);
  return (fd.off << 16) | (s ? T - 16u + s : T);
}

// Rows of a tile of one byte per feature up to which sixteen waves' tiles
// leave room for a slot of trees (64 features).
constexpr uint32_t kMostByteRows = 16;

// The mode of a tile whose features have codes[f] codes above 0, and the
// features' places in it.
void place_fields(const std::vector<size_t> &codes, RankCodes *out) {
  size_t most = 0;
  uint32_t used = 0;
  for (size_t c : codes) {
    most = std::max(most, c);
    used += c != 0;
  }
  out->mode = most > 4095 ? kRankHalf
              : most <= 255 && used <= 4 * kMostByteRows ? kRankByte
                                                         : kRankPacked;
  std::vector<int> by_width[3];  // 4, 8, 12 bits
  uint32_t half = 0;             // half-words used
  auto at = [&](uint32_t h) { return (h >> 1) * kRankRow + (h & 1) * 2u; };
  uint32_t n = 0;
  for (size_t f = 0; f < codes.size(); ++f) {
    out->field[f] = RankField{0, 0, 0};
    if (codes[f] == 0) continue;
    if (out->mode == kRankByte) {
      out->field[f] = RankField{(n >> 2) * kRankRow + (n & 3), 0, 8};
      ++n;
      half = (n + 1) / 2;
    } else if (out->mode == kRankHalf) {
      out->field[f] = RankField{at(half++), 0, 16};
    } else {
      by_width[codes[f] <= 15 ? 0 : codes[f] <= 255 ? 1 : 2].push_back((int)f);
    }
  }
  size_t n4 = 0;  // 4-bit features placed
  auto put = [&](int f, int low, int width) {
    out->field[(size_t)f] = RankField{at(half), (uint8_t)low, (uint8_t)width};
  };
  auto put4 = [&](int low) {
    if (n4 < by_width[0].size()) put(by_width[0][n4++], low, 4);
  };
  for (int f : by_width[2]) {
    put(f, 4, 12);
    put4(0);
    ++half;
  }
  for (size_t i = 0; i < by_width[1].size(); ++half) {
    put(by_width[1][i++], 8, 8);
    if (i < by_width[1].size()) {
      put(by_width[1][i++], 0, 8);
    } else {
      put4(4);
      put4(0);
    }
  }
  for (; n4 < by_width[0].size(); ++half)
    for (int low : {12, 8, 4, 0}) put4(low);
  out->rows = std::max<uint32_t>(1, (half + 1) / 2);
}

// Levels of the smallest perfect search tree of n thresholds.
int steps_of(size_t n) {
  int s = 1;
  while (n >> s) ++s;
  return s;
}

// n sorted thresholds as a search tree of s levels, breadth-first from entry
// 1, padded with +inf.
void put_search_tree(const float *t, size_t n, int s, char *dst) {
  memset(dst, 0, 4);
  for (int l = 0; l < s; ++l) {
    for (size_t i = 0; i < (size_t)1 << l; ++i) {  // entries of level l, left to right
      const size_t in_order = ((2 * i + 1) << (s - 1 - l)) - 1;
      const float v = in_order < n ? t[in_order] : INFINITY;
      memcpy(dst + 4 * (((size_t)1 << l) + i), &v, 4);
    }
  }
}

// One tree of the rank form; leaves above depth D are replicated.
void put_tree(const TreeView &tv, const RankCodes &codes, const uint16_t *code, int D,
              char *dst) {
  const int K = rank_top(D);
  memset(dst, 0, 4);
  std::vector<int32_t> level(1, 0), below;  // node ids of a level, by idx
  for (int l = 0; l < D; ++l) {
    below.resize((size_t)2 << l);
    for (uint32_t idx = 0; idx < 1u << l; ++idx) {
      const int32_t node = level[idx];
      const bool leaf = tv.left[node] == -1 && tv.right[node] == -1;
      const uint32_t at =
          l < K ? (idx << (K - l)) + (1u << (K - 1 - l)) : (1u << l) + idx;
      // a replicated leaf: nothing is below 0, and both sides hold it
      const uint32_t w = leaf ? 0u : node_word(codes, tv.feat[node], code[node]);
      memcpy(dst + 4 * (size_t)at, &w, 4);
      below[2 * idx + 1] = leaf ? node : tv.left[node];  // x < t
      below[2 * idx] = leaf ? node : tv.right[node];
    }
    level.swap(below);
  }
  for (uint32_t idx = 0; idx < 1u << D; ++idx)
    memcpy(dst + 4 * ((size_t)(1u << D) + idx), &tv.val[level[idx]], 4);
}

struct Table {  // a search tree to write once the slots are laid out
  const float *t;
  size_t n;
  int steps, slot;
  uint32_t offset;
};

// Grids, table segments and their groups in slots of slot_bytes, from slot 0
// on, each from byte `base` on; *fill: the bytes used of the last slot.
void lay_out_tables(const RankCodes &codes, int num_features, uint32_t slot_bytes, uint32_t base,
                    RankPack *out, std::vector<Table> *tables, uint32_t *fill) {
  auto new_slot = [&]() {
    ++out->slots;
    *fill = base;
  };
  new_slot();
  out->mode = codes.mode;
  out->rows = codes.rows;
  out->lines = (num_features + kRankLine - 1) / kRankLine;
  out->grid.assign((size_t)out->lines * kRankLine, RankGrid{0.0f, 0.0f, 0.0f, 0u});
  // the order in which the kernels write codes, and so which of a dword's
  // fields comes first: per line the grid features, then the groups
  std::vector<uint8_t> written(codes.rows, 0);
  auto put_of = [&](int f, bool again) {
    const RankField &fd = codes.field[(size_t)f];
    const uint32_t dword = fd.off & ~3u, bit = (fd.off & 3u) * 8u + fd.low;
    uint8_t &w = written[dword / kRankRow];
    const uint32_t put = dword | (bit << 16) | ((w || again) ? kRankAdd : 0u);
    w = 1;
    return put;
  };
  for (int l = 0; l < out->lines; ++l) {
    out->line_group.push_back((int32_t)out->groups.size());
    std::vector<int> search;
    for (int f = l * kRankLine; f < std::min(num_features, (l + 1) * kRankLine); ++f) {
      if (codes.grid[(size_t)f].top != 0.0f) {
        out->grid[(size_t)f] = codes.grid[(size_t)f];
        out->grid[(size_t)f].put = put_of(f, false);
      } else if (!codes.table[(size_t)f].empty()) {
        search.push_back(f);
      }
    }
    // tables of like sizes next to one another, so that they share groups
    std::stable_sort(search.begin(), search.end(), [&](int a, int b) {
      return codes.table[(size_t)a].size() < codes.table[(size_t)b].size();
    });
    int in_group = 4, group_steps = 0;  // segments of the open group (4: none open)
    for (int f : search) {
      const std::vector<float> &t = codes.table[(size_t)f];
      for (size_t done = 0; done < t.size();) {
        size_t n = t.size() - done;
        int steps = steps_of(n);
        if (*fill + (4u << steps) > slot_bytes) {
          if (*fill != base) {
            new_slot();
            in_group = 4;
          }
          while ((4u << steps) > slot_bytes || steps > 13) --steps;
          n = std::min(n, ((size_t)1 << steps) - 1);
        }
        if (in_group == 4 || group_steps != steps) {
          out->groups.push_back(RankGroup{});
          out->group_slot.push_back(out->slots - 1);
          in_group = 0;
          group_steps = steps;
        }
        RankSeg &s = out->groups.back().seg[in_group];
        s.lane_reg = (uint32_t)(f % kRankLine) | ((uint32_t)n << 8);
        s.put = put_of(f, done != 0);
        s.table_off = *fill;
        s.steps = (uint32_t)steps;
        for (int i = in_group + 1; i < 4; ++i) {  // repeats until another segment takes the place
          out->groups.back().seg[i] = s;
          out->groups.back().seg[i].put = kRankNone;
        }
        ++in_group;
        tables->push_back({t.data() + done, n, steps, out->slots - 1, *fill});
        *fill += 4u << steps;
        done += n;
        if (done < t.size()) {  // the rest in a slot and a group of its own
          new_slot();
          in_group = 4;
        }
      }
    }
  }
  out->line_group.push_back((int32_t)out->groups.size());
}

// Room for the slots, and the tables in them.
void put_tables(const std::vector<Table> &tables, uint32_t slot_bytes, RankPack *out) {
  out->bytes = (size_t)out->slots * slot_bytes;
  // (bytes between tables and trees stay zero)
  out->data.reset(static_cast<char *>(calloc(out->bytes, 1)));
  if (!out->data) throw std::bad_alloc();
  parallel_for((int64_t)tables.size(), (int64_t)tables.size() * 512, [&](int64_t i) {
    const Table &t = tables[(size_t)i];
    put_search_tree(t.t, t.n, t.steps,
                    out->data.get() + (size_t)t.slot * slot_bytes + t.offset);
  });
}

}  // namespace

bool rank_codes(const std::vector<TreeView> &views, int num_features, RankCodes *out) {
  const size_t F = (size_t)num_features, T = views.size();
  std::vector<size_t> node0(T + 1, 0);  // first node of each tree
  for (size_t t = 0; t < T; ++t) node0[t + 1] = node0[t] + (size_t)views[t].size;
  const size_t nodes = node0[T];
  if (nodes > 0xFFFFFFFFull) return false;
  // splits grouped by feature, in node order: counted and then placed by
  // blocks of trees
  const size_t blocks = std::min<size_t>(T, 16);
  auto tree_of = [&](size_t b) { return T * b / blocks; };
  std::vector<std::vector<size_t>> at(blocks, std::vector<size_t>(F, 0));
  parallel_for((int64_t)blocks, (int64_t)nodes, [&](int64_t b) {
    std::vector<size_t> &c = at[(size_t)b];
    for (size_t t = tree_of((size_t)b); t < tree_of((size_t)b + 1); ++t)
      for (int64_t i = 0; i < views[t].size; ++i)
        if (views[t].left[i] != -1) ++c[(size_t)views[t].feat[i]];
  });
  std::vector<size_t> first(F + 1, 0);
  for (size_t f = 0, sum = 0; f < F; ++f) {
    first[f] = sum;
    for (size_t b = 0; b < blocks; ++b) {
      const size_t n = at[b][f];
      at[b][f] = sum;
      sum += n;
    }
    first[f + 1] = sum;
  }
  const size_t splits = first[F];
  std::unique_ptr<Entry[]> all(new Entry[splits]), tmp(new Entry[splits]);
  parallel_for((int64_t)blocks, (int64_t)nodes, [&](int64_t b) {
    std::vector<size_t> &c = at[(size_t)b];
    for (size_t t = tree_of((size_t)b); t < tree_of((size_t)b + 1); ++t) {
      const TreeView &tv = views[t];
      for (int64_t i = 0; i < tv.size; ++i)
        if (tv.left[i] != -1)
          all[c[(size_t)tv.feat[i]]++] = {key_of(tv.thr[i]), (uint32_t)(node0[t] + (size_t)i)};
    }
  });
  out->code.reset(new uint16_t[nodes]);  // leaves' stay unset
  out->table.assign(F, {});
  out->grid.assign(F, RankGrid{0.0f, 0.0f, 0.0f, 0u});
  out->field.assign(F, RankField{0, 0, 0});
  std::vector<size_t> codes(F, 0);
  std::vector<uint8_t> too_many(F, 0);
  parallel_for((int64_t)F, (int64_t)nodes, [&](int64_t fi) {
    const size_t f = (size_t)fi, n = first[f + 1] - first[f];
    if (n == 0) return;
    Entry *e = all.get() + first[f];
    std::vector<float> &t = out->table[f];
    uint32_t keys[kFewKeys];
    uint8_t *place = reinterpret_cast<uint8_t *>(tmp.get() + first[f]);
    const int few = few_keys(e, n, keys, place);
    if (few) {
      for (int j = 0; j < few; ++j) t.push_back(value_of(keys[j]));
    } else {
      sort_entries(e, tmp.get() + first[f], n);
      for (size_t i = 0; i < n; ++i)
        if (i == 0 || e[i].key != e[i - 1].key) t.push_back(value_of(e[i].key));
    }
    const size_t n_t = t.size();
    if (n_t > kMostThresholds) {
      too_many[f] = 1;
      return;
    }
    // a grid whose codes take no wider a field than the table's would, or
    // that a byte holds (a table costs a search)
    RankGrid g{};
    const bool grid = find_grid(t, n_t <= 255 ? 255 : n_t <= 4095 ? 4095 : 65535, &g);
    auto code_of = [&](size_t j) {  // of threshold j
      return (uint16_t)(grid ? (uint32_t)((double)t[j] * g.scale + g.bias) : (uint32_t)j + 1);
    };
    if (few) {
      for (size_t i = 0; i < n; ++i) out->code[e[i].node] = code_of(place[i]);
    } else {
      uint16_t c = 0;
      for (size_t i = 0, j = 0; i < n; ++i) {
        if (i == 0 || e[i].key != e[i - 1].key) c = code_of(j++);
        out->code[e[i].node] = c;
      }
    }
    codes[f] = grid ? (size_t)g.top : n_t;
    if (grid) {
      out->grid[f] = g;
      t.clear();
    }
  });
  for (uint8_t m : too_many)
    if (m) return false;
  place_fields(codes, out);
  return true;
}

bool rank_pack(const std::vector<TreeView> &views, const RankCodes &codes, int num_features,
               int D, int group, uint32_t slot_bytes, RankPack *out) {
  const uint32_t RB = rank_tree_bytes(D);
  if (slot_bytes % 16 || (uint64_t)group * RB > slot_bytes) return false;
  out->group = group;
  uint32_t fill = 0;  // bytes used of the last slot
  std::vector<Table> tables;
  lay_out_tables(codes, num_features, slot_bytes, 0, out, &tables, &fill);
  fill = (fill + 127u) & ~127u;  // trees start on a bank row
  const size_t total = (views.size() + group - 1) / group * group;
  for (size_t t = 0; t < total;) {
    uint32_t fit = fill < slot_bytes ? (slot_bytes - fill) / RB / group * group : 0;
    if (fit == 0) {
      ++out->slots;
      fill = 0;
      fit = slot_bytes / RB / group * group;
    }
    const size_t n = std::min<size_t>(fit, total - t);
    out->chunks.push_back({out->slots - 1, (int32_t)fill, (int32_t)n, 0});
    fill += (uint32_t)n * RB;
    t += n;
  }
  put_tables(tables, slot_bytes, out);
  auto slot = [&](int s) { return out->data.get() + (size_t)s * slot_bytes; };
  std::vector<size_t> node0(views.size() + 1, 0), first(out->chunks.size() + 1, 0);
  for (size_t t = 0; t < views.size(); ++t) node0[t + 1] = node0[t] + (size_t)views[t].size;
  for (size_t c = 0; c < out->chunks.size(); ++c)
    first[c + 1] = first[c] + (size_t)out->chunks[c].trees;
  parallel_for((int64_t)out->chunks.size(), (int64_t)node0.back(), [&](int64_t c) {
    const RankChunk &ch = out->chunks[(size_t)c];
    char *dst = slot(ch.slot) + ch.offset;
    for (size_t t = first[(size_t)c]; t < first[(size_t)c + 1]; ++t, dst += RB) {
      if (t < views.size()) {
        put_tree(views[t], codes, codes.code.get() + node0[t], D, dst);
      } else {  // padding: every leaf -0.0 (x + (-0.0) == x)
        const uint32_t z = 0x80000000u;
        memset(dst, 0, (size_t)4 << D);
        for (uint32_t j = 1u << D; j < 2u << D; ++j) memcpy(dst + 4 * (size_t)j, &z, 4);
      }
    }
  });
  return true;
}

bool rank_ragged_fields(RankCodes *codes) {
  std::vector<size_t> n(codes->field.size(), 0);
  size_t most = 0;
  for (size_t f = 0; f < n.size(); ++f) {
    n[f] = codes->grid[f].top != 0.0f ? (size_t)codes->grid[f].top : codes->table[f].size();
    most = std::max(most, n[f]);
  }
  if (most > 4095) return false;  // (a table then fits a slot)
  codes->mode = most < (size_t)kRankRaggedByte ? kRankByte : kRankHalf;
  uint32_t used = 0;
  const uint32_t per = codes->mode == kRankByte ? 4 : 2;  // codes per dword
  for (size_t f = 0; f < n.size(); ++f) {
    codes->field[f] = RankField{0, 0, 0};
    if (n[f] == 0) continue;
    codes->field[f] = codes->mode == kRankByte
                          ? RankField{used / 4 * kRankRow + used % 4, 0, 8}
                          : RankField{used / 2 * kRankRow + used % 2 * 2, 3, 13};
    ++used;
  }
  codes->rows = std::max<uint32_t>(1, (used + per - 1) / per);
  return true;
}

bool rank_pack_ragged(const RaggedPack &ragged, const RankCodes &codes, int num_features,
                      RankPack *out) {
  constexpr uint32_t SB = kRaggedChunkBytes;
  uint32_t fill = 0;
  std::vector<Table> tables;
  // (the slot lies at LDS address 0, and a search subtracts 4 from its table's)
  lay_out_tables(codes, num_features, SB, 16, out, &tables, &fill);
  const int slot0 = fill != 16 ? out->slots : 0;  // the first slot of trees
  out->slots = slot0 + ragged.slots;
  put_tables(tables, SB, out);
  char *dst0 = out->data.get() + (size_t)slot0 * SB;
  memcpy(dst0, ragged.bytes.data(), (size_t)ragged.slots * SB);
  const uint32_t unit = codes.mode == kRankByte ? 256u : 8u;
  const uint32_t *origin = ragged.origin.data();
  for (int s = 0; s < ragged.slots; ++s) {
    char *slot = dst0 + (size_t)s * SB;
    uint32_t head[4];  // trees, deepest path, the sentinel's node, first tree
    memcpy(head, slot, sizeof head);
    out->chunks.push_back({slot0 + s, 0, (int32_t)head[0], 0});
    uint32_t node;
    memcpy(&node, slot + 16, 4);  // the first root: the first node
    for (; node <= head[2]; ++node, ++origin) {
      uint32_t w[2];
      memcpy(w, slot + 8 * (size_t)node, 8);
      if ((w[0] >> 16) == 0x7FFFu) {
        w[0] = (w[0] << 16) | 0xFFFFu;
      } else {
        const uint32_t left = node + ((w[0] >> 16) & 0x7FFFu), f = (w[0] >> 8) & 0xFFu;
        const uint32_t code = codes.code[*origin];  // x < t exactly when code(x) < code
        const bool default_left = (w[0] >> 31) != 0;
        w[0] = (8u * left << 16) | (unit * (default_left ? code : code - 1));
        w[1] = ((default_left ? unit : 0u) << 16) | codes.field[f].off;
      }
      memcpy(slot + 8 * (size_t)node, w, 8);
    }
  }
  return true;
}

}  // namespace ml2
