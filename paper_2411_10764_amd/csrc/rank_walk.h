// Walks over an ensemble's rank form (rank_pack.h): the validity filter and
// the performance prediction of ML2Tuner's explorer (Section 2, "ML Model V"
// / "ML Model P") for pools large enough to pay for ranking each row.
//
// One workgroup = W waves, persistent over the pool; a wave owns a tile of 64
// candidates, one per lane, whose feature codes sit in LDS as 256-byte rows
// (a lane owns one bank column).  A round of a wave:
//   1. ranks its rows: a half-line of 16 features at a time in registers, each
//      value to its code by the feature's grid or by a binary search of the
//      feature's staged table;
//   2. walks every tree of the ensemble over the codes, G trees per lane in
//      two halves offset by half a level, and folds the leaves in tree order.
// Tables and trees stream through one LDS slot in the same fixed sequence
// every round (the next slot is fetched into registers while the current one
// is in use); where one slot holds both, nothing is restaged.
//
// Why codes: a float tile of 128 features lets eight waves hold 32 candidates
// each, a packed tile sixteen waves of 64, so the ensemble is staged for four
// times the candidates, in nodes of four bytes instead of eight.  And a node
// visit takes its place in the two units that bound it:
//   LDS    4-byte node reads and column-owned code reads: about 2.9 clocks
//          per 64-lane read (8-byte nodes at random: 10.7);
//   VALU   address, shift (packed codes), subtract, minimum and multiply-add
//          (two from the sixth level on) in place of address, compare,
//          add-with-carry and address: 15 to 18 instead of 19 clocks of a SIMD
//          per visit.  v_cmp, v_addc and v_lshl_add issue at half the rate of
//          v_sub_u16, v_min_u16 and v_fmac_f32 (measured: 4.7 and 2.7 clocks
//          per 64-lane instruction).
#pragma once

#include <math.h>

#include "ml2_internal.h"
#include "rank_pack.h"

namespace ml2 {

// Kernel arguments (device pointers unless noted).
struct RankArgs {
  const float *X;
  int64_t n, ld;
  const char *slots;
  const RankGrid *grid;
  const int32_t *line_group;
  const RankGroup *groups;
  const int32_t *group_slot;
  const RankChunk *chunks;
  int32_t nslots, nchunks, nlines, F;
  uint32_t slot_bytes, tile_bytes;
  int32_t nthreads;
  uint32_t missing;  // ragged trees: a missing value's code, and
  uint32_t off_mask;  // the bits of a code's offset in the tile
  int32_t vec4;  // rows load as 16-byte vectors (X aligned, ld % 4 == 0, F % 4 == 0)
  float base;
  uint8_t *valid_out;        // validity
  float *margin_out;
  const uint8_t *valid_in;   // perf
  float *score_out;
};

namespace rank {

constexpr int kLanes = 64;
constexpr int kMaxWaves = 16;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// LDS by byte address (32 bits), so that addresses are plain integers.
template <typename T>
__device__ __forceinline__ T lds_read(uint32_t at) {
  return *(const __attribute__((address_space(3))) T *)(uintptr_t)at;
}
template <typename T>
__device__ __forceinline__ void lds_write(uint32_t at, T v) {
  *(__attribute__((address_space(3))) T *)(uintptr_t)at = v;
}
__device__ __forceinline__ uint32_t lds_address(const void *p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)p;
}
// Tables the kernels only read, through the scalar cache.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T *constant(const T *p) {
  return (const __attribute__((address_space(4))) T *)(uintptr_t)p;
}

// A wave's own tile, written by its lanes and then read by them: the LDS
// performs one wave's operations in issue order, so only the compiler must
// keep the accesses on their side of this point.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// H walks of one half.  `a` holds the byte address of the current node less
// the level's constant, as the bits of a (denormal) float: address steps are
// float multiply-adds of small integers, which are exact and issue at twice
// the rate of the shift-adds they replace.  Denormals are on in every kernel
// of this library.
template <int D, int H, RankMode M>
struct Walks {
  static constexpr uint32_t RB = rank_tree_bytes(D);
  static constexpr int K = rank_top(D);
  float a[H];
  uint32_t nd[H];
  uint32_t x[H];
  float leaf[H];

  __device__ __forceinline__ void start(uint32_t rec) {
#pragma unroll
    for (int g = 0; g < H; ++g) a[g] = __uint_as_float(rec);
  }
  template <int l>
  __device__ __forceinline__ void read_nodes() {
    constexpr uint32_t at = l < K ? 4u << (K - 1 - l) : 4u << l;
#pragma unroll
    for (int g = 0; g < H; ++g) nd[g] = lds_read<uint32_t>(__float_as_uint(a[g]) + (g * RB + at));
  }
  __device__ __forceinline__ void read_codes(uint32_t tile_lane) {
#pragma unroll
    for (int g = 0; g < H; ++g) {
      const uint32_t at = tile_lane + (nd[g] >> 16);
      x[g] = M == kRankByte ? lds_read<uint8_t>(at) : lds_read<uint16_t>(at);
    }
  }
  // bit = [x < t] as min(C - x with unsigned saturation, 1).  Above level K
  // the decision adds its weight; below, a <- 2a - rec + 4 bit.
  template <int l>
  __device__ __forceinline__ void descend(float minus_rec) {
    uint32_t b[H];  // a 16-bit instruction clears the upper half
    if constexpr (M == kRankPacked) {  // the field to the top: by the comparand's low four bits
#pragma unroll
      for (int g = 0; g < H; ++g)
        asm("v_lshlrev_b16_e32 %0, %1, %0" : "+v"(x[g]) : "v"(nd[g]));
    }
#pragma unroll
    for (int g = 0; g < H; ++g)  // (in C++ the compiler makes a compare and a select of these)
      asm("v_sub_u16_e64 %0, %1, %2 clamp" : "=v"(b[g]) : "v"(nd[g]), "v"(x[g]));
#pragma unroll
    for (int g = 0; g < H; ++g) asm("v_min_u16_e32 %0, 1, %0" : "+v"(b[g]));
#pragma unroll
    for (int g = 0; g < H; ++g) {
      const float bit = __uint_as_float(b[g]);
      if constexpr (l < K) {
        a[g] = __builtin_fmaf(bit, (float)(4u << (K - 1 - l)), a[g]);
      } else {
        a[g] = __builtin_fmaf(a[g], 2.0f, __builtin_fmaf(bit, 4.0f, minus_rec));
      }
    }
  }
  __device__ __forceinline__ void read_leaves() {
#pragma unroll
    for (int g = 0; g < H; ++g)
      leaf[g] = lds_read<float>(__float_as_uint(a[g]) + (g * RB + (4u << D)));
  }
  __device__ __forceinline__ float fold(float m) const {
#pragma unroll
    for (int g = 0; g < H; ++g) m = m + leaf[g];
    return m;
  }
};

template <int l, int D, int H, RankMode M>
__device__ __forceinline__ void walk_levels(Walks<D, H, M> &A, Walks<D, H, M> &B,
                                            uint32_t tile_lane, float mA, float mB) {
  if constexpr (l < D) {
    A.read_codes(tile_lane);
    __builtin_amdgcn_sched_barrier(0);
    B.read_codes(tile_lane);
    __builtin_amdgcn_sched_barrier(0);
    A.template descend<l>(mA);
    if constexpr (l + 1 < D) A.template read_nodes<l + 1>(); else A.read_leaves();
    __builtin_amdgcn_sched_barrier(0);
    B.template descend<l>(mB);
    if constexpr (l + 1 < D) B.template read_nodes<l + 1>(); else B.read_leaves();
    __builtin_amdgcn_sched_barrier(0);
    walk_levels<l + 1, D, H, M>(A, B, tile_lane, mA, mB);
  }
}

template <int l, int D, RankMode M>
__device__ __forceinline__ void walk_single(Walks<D, 1, M> &A, uint32_t tile_lane, float mA) {
  if constexpr (l < D) {
    A.read_codes(tile_lane);
    A.template descend<l>(mA);
    if constexpr (l + 1 < D) A.template read_nodes<l + 1>(); else A.read_leaves();
    walk_single<l + 1, D, M>(A, tile_lane, mA);
  }
}

// ntr trees (a multiple of G) at LDS address `rec`, folded into m in order.
template <int D, int G, RankMode M>
__device__ __forceinline__ float walk_trees(uint32_t rec, int ntr, uint32_t tile_lane, float m) {
  constexpr uint32_t RB = rank_tree_bytes(D);
  for (int t0 = 0; t0 < ntr; t0 += G, rec += G * RB) {
    float mA = __uint_as_float(rec | 0x80000000u);
    asm("" : "+v"(mA));  // a vector register: a scalar operand halves the rate of the multiply-add
    if constexpr (G == 1) {
      Walks<D, 1, M> A;
      A.start(rec);
      A.template read_nodes<0>();
      walk_single<0, D, M>(A, tile_lane, mA);
      m = A.fold(m);
    } else {
      constexpr int H = G / 2;
      const uint32_t recB = rec + H * RB;
      Walks<D, H, M> A, B;
      A.start(rec);
      B.start(recB);
      A.template read_nodes<0>();
      B.template read_nodes<0>();
      __builtin_amdgcn_sched_barrier(0);
      float mB = __uint_as_float(recB | 0x80000000u);
      asm("" : "+v"(mB));
      walk_levels<0, D, H, M>(A, B, tile_lane, mA, mB);
      m = B.fold(A.fold(m));
    }
  }
  return m;
}

// The rows of lanes q, q + 16, q + 32 and q + 48, which those four lanes load
// together (-1: none; lanes without a row read row 0, features past the last
// repeat it, and neither is used).
struct Rows {
  int32_t r[4];
  __device__ __forceinline__ int32_t own() const {
    const int p = (threadIdx.x >> 4) & 3;
    const int32_t a = (p & 1) ? r[1] : r[0], b = (p & 1) ? r[3] : r[2];
    return (p & 2) ? b : a;
  }
};

// A half-line (16 features) of each lane's row in registers.  A lane's own
// half-line takes four 16-byte loads, and a wave instruction in which every
// lane reads its own row touches 64 lines; so lane 16 p + q loads the p-th
// quarter of the half-lines of the four rows of lanes q, q + 16, .., and two
// stages of lane swaps hand each lane its row.  An instruction then touches
// 16 half-lines once each (16M x 128 pool, rows alone: 2.5 -> 1.85 ms).
struct Line {
  f32x16 v;
  // element 4 i + c: feature 4 p + c of row i until arrange(), then feature
  // 4 i + c of the lane's own row
  __device__ __forceinline__ void load(const RankArgs &a, const Rows &rows, int line) {
    const int p = (threadIdx.x >> 4) & 3;
    if (a.vec4) {
      const int q = min(line * 4 + p, a.F / 4 - 1);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f32x4 w =
            reinterpret_cast<const f32x4 *>(a.X + (int64_t)max(rows.r[i], 0) * a.ld)[q];
#pragma unroll
        for (int c = 0; c < 4; ++c) v[4 * i + c] = w[c];
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float *src = a.X + (int64_t)max(rows.r[i], 0) * a.ld;
#pragma unroll
        for (int c = 0; c < 4; ++c)
          v[4 * i + c] = src[min(line * kRankLine + 4 * p + c, a.F - 1)];
      }
    }
  }
  __device__ __forceinline__ void arrange() {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      uint32_t w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = __float_as_uint(v[4 * i + c]);
#pragma unroll
      for (int i = 0; i < 2; ++i) {  // upper half of row i with lower half of row i + 2
        const auto t = __builtin_amdgcn_permlane32_swap(w[i], w[i + 2], false, false);
        w[i] = t[0];
        w[i + 2] = t[1];
      }
#pragma unroll
      for (int i = 0; i < 4; i += 2) {  // odd 16-lane rows of the first with even ones
        const auto t = __builtin_amdgcn_permlane16_swap(w[i], w[i + 1], false, false);
        w[i] = t[0];
        w[i + 1] = t[1];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) v[4 * i + c] = __uint_as_float(w[i]);
    }
  }
};

// A code into its field: the first write of a dword clears the others.
__device__ __forceinline__ void put_code(uint32_t tile_lane, uint32_t put, uint32_t code) {
  const uint32_t at = tile_lane + (put & 0xFFFFu);
  const uint32_t v = code << ((put >> 16) & 31u);
  if (put & kRankAdd)
    __hip_atomic_fetch_add((__attribute__((address_space(3))) uint32_t *)(uintptr_t)at, v,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  else
    lds_write<uint32_t>(at, v);
}

// The slots in LDS: `cur` is resident at `buf`; slot cur + 1 (cyclic) is in
// flight to the registers.  Every wave of the workgroup takes the same
// sequence of slots.
template <int R>
struct Slots {
  u32x4 r[R];
  int cur;
  char *buf;

  __device__ __forceinline__ void fetch(const RankArgs &a, int s) {
    const u32x4 *src = reinterpret_cast<const u32x4 *>(a.slots + (size_t)s * a.slot_bytes);
#pragma unroll
    for (int k = 0; k < R; ++k) {
      if ((uint32_t)k * a.nthreads * 16u >= a.slot_bytes) break;
      r[k] = src[threadIdx.x + (uint32_t)k * a.nthreads];
    }
  }
  __device__ __forceinline__ void commit(const RankArgs &a) {
    const uint32_t nv = a.slot_bytes / 16u;
    u32x4 *d = reinterpret_cast<u32x4 *>(buf);
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t i = threadIdx.x + (uint32_t)k * a.nthreads;
      if (i < nv) d[i] = r[k];
    }
  }
  __device__ __forceinline__ void prime(const RankArgs &a) {
    cur = 0;
    fetch(a, 0);
    commit(a);
    if (a.nslots > 1) fetch(a, 1);
    __syncthreads();
  }
  __device__ __forceinline__ void need(const RankArgs &a, int s) {
    if (s == cur) return;
    __syncthreads();  // every wave is done with the slot
    commit(a);
    cur = s;
    fetch(a, s + 1 < a.nslots ? s + 1 : 0);
    __syncthreads();
  }
};

// Counts of thresholds not above x (NaN: all) in four search trees of
// `steps` levels, side by side.  `a` is the byte address of the current entry
// as in Walks: a <- 2a - first + 4 [x not below the entry].
__device__ __forceinline__ void search4(const float (&x)[4], const uint32_t (&first)[4],
                                        uint32_t steps, uint32_t (&count)[4]) {
  float a[4], go_left[4], go_right[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    a[i] = __uint_as_float(first[i] + 4u);
    go_left[i] = __uint_as_float(first[i] | 0x80000000u);
    go_right[i] = __uint_as_float((first[i] - 4u) | 0x80000000u);
    asm("" : "+v"(go_left[i]), "+v"(go_right[i]));
  }
  for (uint32_t s = 0; s < steps; ++s) {
    float t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = lds_read<float>(__float_as_uint(a[i]));
#pragma unroll
    for (int i = 0; i < 4; ++i)
      a[i] = __builtin_fmaf(a[i], 2.0f, !(x[i] < t[i]) ? go_right[i] : go_left[i]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
    count[i] = ((__float_as_uint(a[i]) - first[i]) >> 2) - (1u << steps);
}

// Ranks the wave's rows into its tile; line[0] and line[1] hold their first
// half-lines, and two stay in flight.  A wave without a row (not busy) only
// keeps step with the slots.  MISSING (ragged trees): a missing value takes a
// code of its own.
template <bool MISSING, int R>
__device__ __forceinline__ void rank_rows(const RankArgs &a, const Rows &rows, Line (&line)[2],
                                          bool busy,
                                          uint32_t tile_lane, uint32_t buf, Slots<R> &st) {
  const auto *grid = constant(a.grid);
  const auto *line_group = constant(a.line_group);
  const auto *group_slot = constant(a.group_slot);
  const auto *groups = constant(a.groups);
  for (int l = 0; l < a.nlines; ++l) {
    Line cur = line[0];
    line[0] = line[1];
    if (l + 2 < a.nlines) line[1].load(a, rows, l + 2);
    cur.arrange();
#pragma unroll
    for (int k = 0; k < kRankLine; ++k) {
      const float top = grid[l * kRankLine + k].top;
      if (top != 0.0f) {
        const float s = grid[l * kRankLine + k].scale, b = grid[l * kRankLine + k].bias;
        const float c = __builtin_fmaxf(
            __builtin_fminf(__builtin_floorf(cur.v[k] * s) + b, top), 0.0f);
        uint32_t code = (uint32_t)c;
        if (MISSING) code = __builtin_isnan(cur.v[k]) ? a.missing : code;
        put_code(tile_lane, grid[l * kRankLine + k].put, code);
      }
    }
    const int g1 = line_group[l + 1];
    for (int g = line_group[l]; g < g1; ++g) {
      st.need(a, group_slot[g]);
      if (!busy) continue;
      float x[4];
      uint32_t first[4], count[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        x[i] = cur.v[groups[g].seg[i].lane_reg & (kRankLine - 1)];
        first[i] = buf + groups[g].seg[i].table_off;
      }
      search4(x, first, groups[g].seg[0].steps, count);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t put = groups[g].seg[i].put;
        if (MISSING) {
          count[i] = min(count[i], groups[g].seg[i].lane_reg >> 8);  // (not the padding)
          count[i] = __builtin_isnan(x[i]) ? a.missing : count[i];
        }
        if (put != kRankNone) put_code(tile_lane, put, count[i]);
      }
    }
  }
}

template <int D, int G, RankMode M, int R>
__device__ __forceinline__ float walk_all(const RankArgs &a, bool busy, uint32_t tile_lane,
                                          uint32_t buf, Slots<R> &st) {
  const auto *chunks = constant(a.chunks);
  float m = a.base;
  for (int c = 0; c < a.nchunks; ++c) {
    st.need(a, chunks[c].slot);
    if (busy) m = walk_trees<D, G, M>(buf + (uint32_t)chunks[c].offset, chunks[c].trees, tile_lane, m);
  }
  return m;
}

// The performance walks' rows: the accepted rows of the pool, compacted into a
// queue of 2 NT entries in LDS (NT: threads of the workgroup), NT at a time.
struct Survivors {
  int32_t *queue;
  int *wave_count;
  int64_t round, step, mine;  // the mask in units of 64 rows per wave, as in the validity walk
  int qn, took;  // queued rows, and those the last next() took (the same in every thread)

  __device__ __forceinline__ Survivors(const RankArgs &a, int32_t *q, int *counts)
      : queue(q), wave_count(counts) {
    const int lane = threadIdx.x & (kLanes - 1), wave = threadIdx.x / kLanes;
    round = (int64_t)blockIdx.x * kLanes;
    step = (int64_t)gridDim.x * a.nthreads;
    mine = (int64_t)wave * gridDim.x * kLanes + lane;
    qn = took = 0;
  }
  // Scans the mask NT entries at a time until NT rows are queued (or the pool
  // is exhausted), then takes up to NT rows off the queue, which never holds
  // more than 2 NT - 1.  Rejected rows get -inf.
  __device__ __forceinline__ Rows next(const RankArgs &a) {
    const int lane = threadIdx.x & (kLanes - 1), wave = threadIdx.x / kLanes;
    const int NT = a.nthreads, nw = NT / kLanes;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    while (qn < NT && round < a.n) {
      const int64_t i = round + mine;
      const bool in = i < a.n;
      const bool v = in && (a.valid_in == nullptr || a.valid_in[i] != 0);
      if (in && !v) __builtin_nontemporal_store(-INFINITY, a.score_out + i);
      const uint64_t bal = __ballot(v);
      if (lane == 0) wave_count[wave] = __popcll(bal);
      __syncthreads();
      int off = 0, tot = 0;
      for (int w = 0; w < nw; ++w) {
        const int c = wave_count[w];
        off += (w < wave) ? c : 0;
        tot += c;
      }
      if (v) queue[qn + off + __popcll(bal & below)] = (int32_t)i;
      qn = __builtin_amdgcn_readfirstlane(qn + tot);
      round += step;
      __syncthreads();
    }
    const int take = min(qn, NT);
    took = take;
    Rows r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = (int)(threadIdx.x & ~63u) + (lane & 15) + 16 * i;
      r.r[i] = e < take ? queue[e] : -1;
    }
    const int rem = qn - take;  // < NT
    const int32_t carry = ((int)threadIdx.x < rem) ? queue[take + threadIdx.x] : 0;
    __syncthreads();
    if ((int)threadIdx.x < rem) queue[threadIdx.x] = carry;
    qn = rem;
    __syncthreads();
    return r;
  }
};

// The round loops of a walk: `walk(busy)` folds every tree over the tile.
template <bool PERF, bool MISSING, int R, typename Walk>
__device__ __forceinline__ void rounds(const RankArgs &a, uint32_t tile_lane, uint32_t buf,
                                       Slots<R> &st, int32_t *queue, int *wave_count,
                                       Walk walk) {
  const int lane = threadIdx.x & (kLanes - 1);
  Line line[2];
  if constexpr (!PERF) {
    // A round's rows of wave w of workgroup b: unit (round * nw + w) * grid +
    // b of 64 rows, so that the units spread evenly over the workgroups and a
    // short round leaves whole waves idle.
    const int64_t step = (int64_t)gridDim.x * a.nthreads;
    int64_t round = (int64_t)blockIdx.x * kLanes;  // wave 0's first row
    const int64_t mine = (int64_t)(threadIdx.x / kLanes) * gridDim.x * kLanes;
    auto rows_at = [&](int64_t first) {
      Rows w;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t r = first + (lane & 15) + 16 * i;
        w.r[i] = r < a.n ? (int32_t)r : -1;
      }
      return w;
    };
    Rows rows = rows_at(round + mine);
    line[0].load(a, rows, 0);
    line[1].load(a, rows, 1);
    for (; round < a.n; round += step) {
      const int64_t first = round + mine;
      const bool busy = first < a.n;  // the same in every lane
      rank_rows<MISSING>(a, rows, line, busy, tile_lane, buf, st);
      rows = rows_at(first + step);
      line[0].load(a, rows, 0);  // the next round's, in flight during the walk
      line[1].load(a, rows, 1);
      wave_sync();
      const float m = walk(busy);
      wave_sync();
      const int64_t row = first + lane;
      if (row < a.n) {
        __builtin_nontemporal_store((uint8_t)((m > 0.0f) ? 1 : 0), a.valid_out + row);
        if (a.margin_out) __builtin_nontemporal_store(m, a.margin_out + row);
      }
    }
  } else {
    Survivors sv(a, queue, wave_count);
    Rows rows = sv.next(a);
    int cur = sv.took;  // rows of this round: the loop ends where there are none
    line[0].load(a, rows, 0);
    line[1].load(a, rows, 1);
    while (cur != 0) {
      const bool busy = (int)(threadIdx.x & ~63u) < cur;  // the same in every lane
      rank_rows<MISSING>(a, rows, line, busy, tile_lane, buf, st);
      const int32_t row = rows.own();
      rows = sv.next(a);
      line[0].load(a, rows, 0);
      line[1].load(a, rows, 1);
      wave_sync();
      const float m = walk(busy);
      wave_sync();
      if (row >= 0) __builtin_nontemporal_store(m, a.score_out + row);
      cur = sv.took;
    }
  }
}

// W: the most waves that share a CU (16, 12, 8 or 4), which sets the registers.
template <int D, int G, RankMode M, int W, bool PERF>
__global__ void __launch_bounds__(kLanes *W) __attribute__((amdgpu_waves_per_eu(W / 4, W / 4)))
rank_kernel(RankArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ int wave_count[kMaxWaves];
  const int lane = threadIdx.x & (kLanes - 1);
  const int wave = threadIdx.x / kLanes;
  Slots<rank_stage_regs(W)> st;
  st.buf = smem + (size_t)(a.nthreads / kLanes) * a.tile_bytes;
  const uint32_t buf = lds_address(st.buf);
  const uint32_t tile_lane = lds_address(smem) + (uint32_t)wave * a.tile_bytes + 4u * lane;
  st.prime(a);
  rounds<PERF, false>(a, tile_lane, buf, st, reinterpret_cast<int32_t *>(st.buf + a.slot_bytes),
                      wave_count, [&](bool busy) {
                        return walk_all<D, G, M>(a, busy, tile_lane, buf, st);
                      });
}

template <int D, int G, RankMode M, int W, bool PERF>
hipError_t launch_one(const RankArgs &a, int grid, size_t lds, hipStream_t s) {
  const void *fn = reinterpret_cast<const void *>(&rank_kernel<D, G, M, W, PERF>);
  hipError_t e = ensure_dynamic_lds(fn, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((rank_kernel<D, G, M, W, PERF>), dim3(grid), dim3(a.nthreads), lds, s, a);
  return hipGetLastError();
}

template <int D, int G, RankMode M, bool PERF>
hipError_t launch_waves(int waves, const RankArgs &a, int grid, size_t lds, hipStream_t s) {
  if (waves > 12) return launch_one<D, G, M, 16, PERF>(a, grid, lds, s);
  if (waves > 8) return launch_one<D, G, M, 12, PERF>(a, grid, lds, s);
  if (waves > 4) return launch_one<D, G, M, 8, PERF>(a, grid, lds, s);
  return launch_one<D, G, M, 4, PERF>(a, grid, lds, s);
}

template <int D, bool PERF>
hipError_t launch_depth(RankMode mode, int waves, const RankArgs &a, int grid, size_t lds,
                        hipStream_t s) {
  constexpr int G = kRankGroup[D];
  switch (mode) {
    case kRankByte: return launch_waves<D, G, kRankByte, PERF>(waves, a, grid, lds, s);
    case kRankHalf: return launch_waves<D, G, kRankHalf, PERF>(waves, a, grid, lds, s);
    default: return launch_waves<D, G, kRankPacked, PERF>(waves, a, grid, lds, s);
  }
}

template <bool PERF>
hipError_t launch(int depth, RankMode mode, int waves, const RankArgs &a, int grid, size_t lds,
                  hipStream_t s) {
  switch (depth) {
    case 4: return launch_depth<4, PERF>(mode, waves, a, grid, lds, s);
    case 5: return launch_depth<5, PERF>(mode, waves, a, grid, lds, s);
    case 6: return launch_depth<6, PERF>(mode, waves, a, grid, lds, s);
    case 7: return launch_depth<7, PERF>(mode, waves, a, grid, lds, s);
    case 8: return launch_depth<8, PERF>(mode, waves, a, grid, lds, s);
    case 9: return launch_depth<9, PERF>(mode, waves, a, grid, lds, s);
    case 10: return launch_depth<10, PERF>(mode, waves, a, grid, lds, s);
    case 11: return launch_depth<11, PERF>(mode, waves, a, grid, lds, s);
    case 12: return launch_depth<12, PERF>(mode, waves, a, grid, lds, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace rank

hipError_t launch_rank_ragged_kernel(bool perf, RankMode mode, int waves, const RankArgs &a,
                                     int grid, size_t lds, hipStream_t s);
hipError_t launch_rank_validity_kernel(int depth, RankMode mode, int waves, const RankArgs &a,
                                       int grid, size_t lds, hipStream_t s);
hipError_t launch_rank_perf_kernel(int depth, RankMode mode, int waves, const RankArgs &a,
                                   int grid, size_t lds, hipStream_t s);

}  // namespace ml2
