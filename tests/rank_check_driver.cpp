// Rank form checked on the host: packs random ensembles, then ranks and walks
// rows with the kernels' arithmetic (grid formula, segment search, float
// address steps) and compares every leaf with the unpacked tree's, bit for
// bit.  Every table, tree and tile access is checked against its slot or
// tile.  Prints one "ok ..." line per ensemble.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <limits>
#include <random>
#include <vector>

#include "rank_pack.h"

using namespace ml2;

#define CHECK(c)                                                   \
  do {                                                             \
    if (!(c)) {                                                    \
      fprintf(stderr, "%s:%d: %s\n", __FILE__, __LINE__, #c);      \
      exit(1);                                                     \
    }                                                              \
  } while (0)

struct Tree {
  std::vector<int32_t> left, right, feat;
  std::vector<float> thr, val;
  TreeView view() const {
    return {left.data(), right.data(), feat.data(), thr.data(), val.data(), nullptr,
            (int64_t)left.size()};
  }
};

static std::mt19937 rng(7);
static int below(int n) { return (int)(rng() % (uint32_t)n); }
static float normal() { return std::normal_distribution<float>(0, 1)(rng); }

// Threshold kinds: 0 small integers, 1 lognormal, 2 few values, 3 eighths,
// 4 specials (infinities, signed zeros, subnormals), 5 wide integers.
static float draw_threshold(int kind) {
  const float inf = std::numeric_limits<float>::infinity();
  switch (kind) {
    case 0: return (float)below(9);
    case 1: return expf(normal());
    case 2: return (float)(below(3) - 1) * 0.3f;
    case 3: return (float)(below(200) - 100) * 0.125f;
    case 4: {
      const float v[] = {inf, -inf, 0.0f, -0.0f, 1e-45f, -1e-45f, 3.0f, 3.4e38f, -3.4e38f};
      return v[below(9)];
    }
    default: return (float)(below(3000) - 1500);
  }
}

static Tree grow(int D, bool full, int F, const std::vector<int> &kinds, int leaf_percent = 25) {
  Tree t;
  struct Item { int node, level; };
  std::vector<Item> todo{{0, 0}};
  auto add = [&]() {
    t.left.push_back(-1);
    t.right.push_back(-1);
    t.feat.push_back(-1);
    t.thr.push_back(0);
    t.val.push_back(normal());
    return (int)t.left.size() - 1;
  };
  add();
  while (!todo.empty()) {
    const Item it = todo.back();
    todo.pop_back();
    if (it.level == D || (!full && it.level > 0 && below(100) < leaf_percent))
      continue;
    const int f = below(F);
    t.feat[(size_t)it.node] = f;
    t.thr[(size_t)it.node] = draw_threshold(kinds[(size_t)f]);
    const int l = add(), r = add();
    t.left[(size_t)it.node] = l;
    t.right[(size_t)it.node] = r;
    todo.push_back({l, it.level + 1});
    todo.push_back({r, it.level + 1});
  }
  return t;
}

static float leaf_of(const Tree &t, const std::vector<float> &x) {
  int n = 0;
  while (t.left[(size_t)n] != -1)
    n = x[(size_t)t.feat[(size_t)n]] < t.thr[(size_t)n] ? t.left[(size_t)n] : t.right[(size_t)n];
  return t.val[(size_t)n];
}

static float as_float(uint32_t b) {
  float v;
  memcpy(&v, &b, 4);
  return v;
}
static uint32_t as_bits(float v) {
  uint32_t b;
  memcpy(&b, &v, 4);
  return b;
}

// One row ranked into a lane's column with the kernels' arithmetic.
struct Column {
  const RankPack &p;
  uint32_t slot_bytes, buf;
  int missing;  // the missing code of ragged trees, or -1
  std::vector<uint32_t> col;
  int at_slot = 0;

  Column(const RankPack &p_, uint32_t sb, uint32_t buf_, int missing_)
      : p(p_), slot_bytes(sb), buf(buf_), missing(missing_), col(p_.rows, 0xABABABABu) {}
  void put(uint32_t where, uint32_t code) {
    const uint32_t at = where & 0xFFFFu, bit = (where >> 16) & 31u;
    CHECK(at % kRankRow == 0 && at / kRankRow < p.rows);
    CHECK(code <= 65535u && (((uint64_t)code << bit) >> 32) == 0);
    uint32_t &w = col[at / kRankRow];
    w = (code << bit) + ((where & kRankAdd) ? w : 0u);
  }
  uint32_t get(uint32_t at) const {
    CHECK(at % kRankRow < 4 && at / kRankRow < p.rows && (p.mode == kRankByte || at % 2 == 0));
    return (col[at / kRankRow] >> (at % kRankRow * 8)) & (p.mode == kRankByte ? 0xFFu : 0xFFFFu);
  }
  void need(int s) {  // slots are needed in order, one after the other
    CHECK(s == at_slot || s == at_slot + 1);
    CHECK(s < p.slots);
    at_slot = s;
  }
  void rank(const std::vector<float> &x) {
    for (int l = 0; l < p.lines; ++l) {
      for (int k = 0; k < kRankLine; ++k) {
        const RankGrid &g = p.grid[(size_t)(l * kRankLine + k)];
        if (g.top == 0.0f) continue;
        const float v = x[(size_t)(l * kRankLine + k)];
        const float c = fmaxf(fminf(floorf(v * g.scale) + g.bias, g.top), 0.0f);
        put(g.put, missing >= 0 && std::isnan(v) ? (uint32_t)missing : (uint32_t)c);
      }
      for (int g = p.line_group[(size_t)l]; g < p.line_group[(size_t)l + 1]; ++g) {
        need(p.group_slot[(size_t)g]);
        for (const RankSeg &s : p.groups[(size_t)g].seg) {
          const uint32_t steps = p.groups[(size_t)g].seg[0].steps;
          CHECK(s.steps == steps && steps > 0 && s.table_off % 4 == 0);
          CHECK(s.table_off + (4u << steps) <= slot_bytes);
          const char *tab = p.data.get() + (size_t)at_slot * slot_bytes + s.table_off;
          const float v = x[(size_t)(l * kRankLine + (int)(s.lane_reg & 255u))];
          const uint32_t first = buf + s.table_off;
          float a = as_float(first + 4);
          for (uint32_t step = 0; step < steps; ++step) {
            const uint32_t at = as_bits(a) - first;
            CHECK(at >= 4 && at < (4u << steps) && at % 4 == 0);
            float t;
            memcpy(&t, tab + at, 4);
            a = fmaf(a, 2.0f, as_float((!(v < t) ? first - 4 : first) | 0x80000000u));
          }
          uint32_t pos = ((as_bits(a) - first) >> 2) - (1u << steps);
          if (missing >= 0) {
            pos = std::min(pos, s.lane_reg >> 8);
            if (std::isnan(v)) pos = (uint32_t)missing;
          }
          if (s.put != kRankNone) put(s.put, pos);
        }
      }
    }
  }
};

static void draw_row(std::vector<float> &x, const std::vector<int> &kinds) {
  const float special[] = {NAN, INFINITY, -INFINITY, 0.0f, -0.0f, 1e-45f, -1e-45f, 3.4e38f,
                           -3.4e38f};
  for (size_t f = 0; f < x.size(); ++f) {
    float v = draw_threshold(kinds[f]);
    const int how = below(6);
    if (how == 0) v = nextafterf(v, INFINITY);
    if (how == 1) v = nextafterf(v, -INFINITY);
    if (how == 2) v = normal() * 3;
    if (how == 3 && below(3) == 0) v = special[below(9)];
    if (how == 4 && below(3) == 0) v = NAN;
    x[f] = v;
  }
}

static void check(int D, int F, int trees, int group, uint32_t slot_bytes, bool full,
                  const std::vector<int> &kinds, int rows) {
  std::vector<Tree> forest;
  for (int t = 0; t < trees; ++t) forest.push_back(grow(D, full, F, kinds));
  std::vector<TreeView> views;
  for (const Tree &t : forest) views.push_back(t.view());
  RankCodes codes;
  CHECK(rank_codes(views, F, &codes));
  RankPack p;
  CHECK(rank_pack(views, codes, F, D, group, slot_bytes, &p));
  const uint32_t RB = rank_tree_bytes(D);
  const int K = rank_top(D);
  CHECK(p.bytes == (size_t)p.slots * slot_bytes);
  CHECK((int)p.line_group.size() == p.lines + 1 && p.grid.size() == (size_t)p.lines * kRankLine);
  const uint32_t buf = p.rows * kRankRow + 1024;  // LDS address of the slot, beyond the tile
  std::vector<float> x((size_t)F);
  for (int i = 0; i < rows; ++i) {
    draw_row(x, kinds);
    Column c(p, slot_bytes, buf, -1);
    c.rank(x);
    size_t t = 0;
    for (const RankChunk &ch : p.chunks) {
      c.need(ch.slot);
      CHECK(ch.trees % group == 0 && ch.offset % 128 == 0);
      CHECK((uint32_t)ch.offset + (uint32_t)ch.trees * RB <= slot_bytes);
      for (int j = 0; j < ch.trees; ++j, ++t) {
        const uint32_t rec = buf + (uint32_t)ch.offset + (uint32_t)j * RB;
        auto word = [&](uint32_t at) {
          CHECK(at >= rec + 4 && at + 4 <= rec + RB && at % 4 == 0);
          uint32_t w;
          memcpy(&w, p.data.get() + (size_t)c.at_slot * slot_bytes + (at - buf), 4);
          return w;
        };
        float a = as_float(rec);
        const float minus_rec = as_float(rec | 0x80000000u);
        for (int l = 0; l < D; ++l) {
          const uint32_t w = word(as_bits(a) + (l < K ? 4u << (K - 1 - l) : 4u << l));
          const uint32_t cmp = w & 0xFFFFu;
          uint32_t code = c.get(w >> 16);
          if (p.mode == kRankPacked) code = (code << (cmp & 15u)) & 0xFFFFu;
          const float bit = as_float(std::min(cmp > code ? cmp - code : 0u, 1u));
          if (l < K)
            a = fmaf(bit, (float)(4u << (K - 1 - l)), a);
          else
            a = fmaf(a, 2.0f, fmaf(bit, 4.0f, minus_rec));
        }
        const uint32_t leaf = word(as_bits(a) + (4u << D));
        const float want = t < forest.size() ? leaf_of(forest[t], x) : -0.0f;
        CHECK(leaf == as_bits(want));
      }
    }
    CHECK(t == (size_t)((trees + group - 1) / group * group));
  }
  const char *name[] = {"byte", "half", "packed"};
  printf("ok %d rows, %s, tile %u, %zu groups, %d slots\n", rows, name[p.mode], p.rows,
         p.groups.size(), p.slots);
}

// Ragged trees with default directions over codes.
static float ragged_leaf_of(const Tree &t, const std::vector<uint8_t> &dl,
                            const std::vector<float> &x) {
  int n = 0;
  while (t.left[(size_t)n] != -1) {
    const float v = x[(size_t)t.feat[(size_t)n]];
    const bool left = std::isnan(v) ? dl[(size_t)n] != 0 : v < t.thr[(size_t)n];
    n = left ? t.left[(size_t)n] : t.right[(size_t)n];
  }
  return t.val[(size_t)n];
}

static void check_ragged(int D, int F, int trees, const std::vector<int> &kinds, int rows) {
  std::vector<Tree> forest;
  std::vector<std::vector<uint8_t>> dl;
  std::vector<TreeView> views;
  std::vector<int> depths;
  for (int t = 0; t < trees; ++t) {
    Tree tr;
    do tr = grow(D, false, F, kinds, D > 12 ? 45 : 25);
    while (tr.left.size() > 3000);
    std::vector<uint8_t> d(tr.left.size());
    for (uint8_t &b : d) b = (uint8_t)below(2);
    forest.push_back(std::move(tr));
    dl.push_back(std::move(d));
    depths.push_back(D);
  }
  for (int t = 0; t < trees; ++t) {
    TreeView v = forest[(size_t)t].view();
    v.dl = dl[(size_t)t].data();
    views.push_back(v);
  }
  RaggedPack ragged;
  pack_ragged(views, depths, &ragged);
  RankCodes codes;
  CHECK(rank_codes(views, F, &codes));
  CHECK(rank_ragged_fields(&codes));
  RankPack p;
  CHECK(rank_pack_ragged(ragged, codes, F, &p));
  const bool byte = p.mode == kRankByte;
  const uint32_t unit = byte ? 256 : 8;
  std::vector<float> x((size_t)F);
  for (int i = 0; i < rows; ++i) {
    draw_row(x, kinds);
    Column c(p, kRaggedChunkBytes, 0, byte ? kRankRaggedByte : kRankRaggedHalf);
    c.rank(x);
    size_t t = 0;
    for (const RankChunk &ch : p.chunks) {
      c.need(ch.slot);
      const char *slot = p.data.get() + (size_t)ch.slot * kRaggedChunkBytes;
      uint32_t head[4], at, w[2];
      memcpy(head, slot, 16);
      memcpy(&at, slot + 16, 4);
      at *= 8;
      const uint32_t end = 8 * head[2];
      for (int steps = 0; at != end; ++steps) {
        CHECK(steps < (int)head[0] * ((int)head[1] + 2));
        CHECK(at % 8 == 0 && at >= 16 && at + 8 <= kRaggedChunkBytes);
        memcpy(w, slot + at, 8);
        if ((w[0] & 0xFFFFu) == 0xFFFFu) {  // a leaf: on to the next root
          if (w[1] != 0x80000000u) {  // (a padding tree's leaf is -0.0)
            CHECK(t < forest.size() && w[1] == as_bits(ragged_leaf_of(forest[t], dl[t], x)));
            ++t;
          }
          at = w[0] >> 16;
          continue;
        }
        const uint32_t y = byte ? c.get(w[1] & 0xFFFFu) << 8 : c.get(w[1] & 0xFFFFu);
        const uint32_t z = (y + (w[1] >> 16)) & 0xFFFFu, cmp = w[0] & 0xFFFFu;
        CHECK(z % unit == 0 && cmp % unit == 0);
        at = (w[0] >> 16) + std::min(z > cmp ? z - cmp : 0u, 8u);
      }
      memcpy(w, slot + end, 8);  // the sentinel: onto itself, -0.0
      CHECK(w[0] == ((end << 16) | 0xFFFFu) && w[1] == 0x80000000u);
    }
    CHECK(t == forest.size());
  }
  printf("ok %d rows, ragged %s, tile %u, %zu groups, %d slots\n", rows, byte ? "byte" : "half",
         p.rows, p.groups.size(), p.slots);
}

int main() {
  check_ragged(14, 64, 60, std::vector<int>(64, 0), 60);   // grids
  check_ragged(10, 20, 200, std::vector<int>(20, 1), 40);  // half: long tables
  check_ragged(9, 96, 40, std::vector<int>(96, 1), 40);    // byte: tables
  check_ragged(32, 7, 30, std::vector<int>(7, 4), 200);    // specials
  check_ragged(1, 1, 1, std::vector<int>(1, 2), 100);
  check_ragged(6, 256, 90, std::vector<int>(256, 3), 30);

  for (int D = kRankMinDepth; D <= kRankMaxDepth; ++D) {
    const int group = D <= 8 ? 8 : D <= 10 ? 4 : D == 11 ? 2 : 1;
    const int F = 1 + below(70);
    std::vector<int> kinds;
    for (int f = 0; f < F; ++f) kinds.push_back(below(6));
    check(D, F, D <= 9 ? 21 : 5, group, 64 * 1024, D % 2 == 0, kinds, 40);
  }
  check(6, 64, 40, 8, 16 * 1024, true, std::vector<int>(64, 0), 60);    // grids only: no table
  check(6, 128, 100, 8, 24064, true, std::vector<int>(128, 1), 40);     // one byte, tables
  check(8, 128, 260, 8, 28416, true, std::vector<int>(128, 1), 20);     // two bytes
  check(10, 3, 24, 4, 32 * 1024, true, std::vector<int>(3, 1), 20);     // tables longer than a slot
  check(5, 256, 33, 8, 32 * 1024, false, std::vector<int>(256, 4), 60); // specials, widest row
  check(7, 33, 30, 8, 30464, true, std::vector<int>(33, 5), 60);        // wide grids
  check(8, 24, 700, 8, 60 * 1024, true, std::vector<int>(24, 1), 20);   // wide: codes beyond 4095
  check(4, 1, 1, 8, 8192, true, std::vector<int>(1, 3), 200);
  return 0;
}
