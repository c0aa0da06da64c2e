// Selection of the k best accepted candidates (ML2Tuner Section 2: the
// explorer keeps the highest predicted performance among the configurations
// model V accepts, until (alpha+1)*N are held).
//
// Every included candidate i (mask set, score not NaN) gets a unique 64-bit
// key   (ord(score) << 32) | (0xFFFFFFFF - i)
// where ord maps float32 to uint32 monotonically (-0.0 first canonicalised to
// +0.0).  Larger keys are better: higher score, then lower index.  The k-th
// largest key is found by a most-significant-digit radix select over 12-bit
// digits.  A pool of at most kSmallN candidates is selected in one launch of
// one workgroup (topk_small: the included keys are gathered into LDS and the
// same digit passes run there).  Larger pools take three launches:
//   topk_init    clears the state and the digit histograms;
//   topk_select  one workgroup per CU at most, persistent over the pool: each
//                pass histograms (in LDS, then into a global histogram) the
//                digit below the decided prefix of the keys that match it;
//                after a grid-wide barrier every workgroup reads the
//                histogram and picks the same digit.  The passes stop once
//                the bin holding the k-th key is small (at most kInCap keys)
//                or holds exactly the keys still needed; one last pass over
//                the pool appends the keys above that bin (all selected) to
//                one list and the keys in it to another;
//   topk_finish  a workgroup per 64 keys of the two lists: each key's place is
//                the number of its list's keys above it; the selected ones
//                are written there.
// The grid barrier waits a bounded time (every workgroup of the launch can
// be resident at once: the grid is at most one workgroup of 512 threads and
// 16 KiB of LDS per CU); a wait
// that runs out marks the selection failed (num_selected = -1) and every
// workgroup exits.
#include <math.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "ml2_internal.h"

namespace ml2 {
namespace {

constexpr int kDigitBits = 12;
constexpr int kBins = 1 << kDigitBits;
constexpr int kMaxPasses = 6;    // 5 x 12 + 4 bits
constexpr int kSelThreads = 512;
constexpr int kSortThreads = 1024;
constexpr int kInCap = 8192;     // keys of the threshold bin that topk_finish places
constexpr int kSmallN = 8192;    // pools selected in one launch of one workgroup
constexpr int kTile = 1024;      // candidates a wave reads per step (16 per lane)
constexpr size_t kStateBytes = 256;
constexpr size_t kHistBytes = 3 * kBins * sizeof(uint32_t);
constexpr double kBarrierSeconds = 2.0;

// How the final pass classifies keys.
constexpr int kTakeAll = 1;  // every included key is selected (#included <= k)
constexpr int kExact = 2;    // keys whose decided bits are >= prefix: exactly the k
constexpr int kInBin = 3;    // above prefix: selected; equal: the bin, need_in of them

struct TopkState {
  uint32_t arrive;   // grid-barrier arrivals in this call
  uint32_t failed;   // a barrier wait ran out
  uint32_t n_take;   // keys appended to the selected list
  uint32_t n_in;     // keys appended to the bin list
  int32_t k;
  int32_t total;     // included candidates
  int32_t mode;
  int32_t nbits;     // decided high bits
  int32_t need_in;   // keys of the bin to select
  int32_t pad;
  unsigned long long prefix;
};

__device__ __forceinline__ unsigned long long make_key(float s, int64_t i) {
  uint32_t b = __float_as_uint(s);
  if (b == 0x80000000u) b = 0u;
  const uint32_t ord = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
  return ((unsigned long long)ord << 32) | (unsigned long long)(0xFFFFFFFFu - (uint32_t)i);
}

__device__ __forceinline__ int digit_width(int nbits) { return min(kDigitBits, 64 - nbits); }

// f(included, key) for every candidate of this wave's share of the pool,
// called the same number of times by every lane of a wave (out-of-range
// candidates come as not included), so f may use wave ballots.  A wave reads
// kTile candidates per step: with 16-byte aligned scores (and a 4-byte
// aligned mask) four 16-byte score loads and four 4-byte mask loads per
// lane, each instruction covering 256 consecutive candidates, issued one
// step ahead of the step being processed; otherwise sixteen single loads
// per lane.
struct Tile {
  float4 s[4];
  uint32_t m[4];
};

__device__ __forceinline__ void load_tile(const uint8_t *valid, const float *scores, int64_t base,
                                          int lane, Tile &t) {
#pragma unroll
  for (int j = 0; j < 4; ++j)
    t.s[j] = reinterpret_cast<const float4 *>(scores + base)[j * 64 + lane];
#pragma unroll
  for (int j = 0; j < 4; ++j)
    t.m[j] = valid ? reinterpret_cast<const uint32_t *>(valid + base)[j * 64 + lane] : 0x01010101u;
}

// f(inc[16], key[16]) for every group of 16 candidates of this wave's share
// of the pool (each lane's 16 of a tile of kTile), called the same number of
// times by every lane of a wave (out-of-range candidates come as not
// included), so f may use wave ballots.
template <typename F>
__device__ __forceinline__ void for_each_tile(const uint8_t *valid, const float *scores, int64_t n,
                                              int vec, F f) {
  const int lane = threadIdx.x & 63;
  const int64_t wave = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const int64_t waves = (int64_t)gridDim.x * (blockDim.x >> 6);
  const int64_t full = vec ? n / kTile : 0;  // whole tiles read with vector loads
  int64_t t = wave;
  bool inc[16];
  unsigned long long key[16];
  for (; t < full; t += waves) {
    Tile cur;
    load_tile(valid, scores, t * kTile, lane, cur);
    const int64_t base = t * kTile;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t i0 = base + 4 * (j * 64 + lane);
      const float c[4] = {cur.s[j].x, cur.s[j].y, cur.s[j].z, cur.s[j].w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        inc[4 * j + q] = ((cur.m[j] >> (8 * q)) & 0xFFu) != 0 && !isnan(c[q]);
        key[4 * j + q] = make_key(c[q], i0 + q);
      }
    }
    f(inc, key);
  }
  // the rest (a partial tile, or every tile without vector loads)
  for (; t * kTile < n; t += waves) {
    const int64_t base = t * kTile;
#pragma unroll
    for (int j = 0; j < kTile / 64; ++j) {
      const int64_t i = base + j * 64 + lane;
      bool in = false;
      float sc = 0.0f;
      if (i < n) {
        sc = scores[i];
        in = (!valid || valid[i] != 0) && !isnan(sc);
      }
      inc[j] = in;
      key[j] = make_key(sc, i);
    }
    f(inc, key);
  }
}

// The digit holding the need-th largest key (1 <= need <= total) from a
// histogram h[nb] in LDS: bin, keys in higher bins, keys in the bin, and the
// histogram's total.  Every thread of the workgroup calls it; thread t
// covers bins from the top down.
struct Pick {
  int bin;
  uint32_t above, cnt, total;
};

__device__ __forceinline__ Pick block_pick(const uint32_t *h, int nb, uint32_t need, uint32_t *wave_sum,
                           Pick *out) {
  const int T = blockDim.x, t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int per = nb / T > 0 ? nb / T : 1;
  const int hi = nb - t * per;  // bins [hi - per, hi)
  uint32_t sum = 0;
  for (int j = 1; j <= per; ++j)
    if (hi - j >= 0) sum += h[hi - j];
  uint32_t incl = sum;
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t v = __shfl_up(incl, d);
    if (lane >= d) incl += v;
  }
  if (lane == 63) wave_sum[wave] = incl;
  __syncthreads();
  if (t == 0) {
    uint32_t acc = 0;
    for (int w = 0; w < (T >> 6); ++w) {
      const uint32_t v = wave_sum[w];
      wave_sum[w] = acc;
      acc += v;
    }
    wave_sum[T >> 6] = acc;
  }
  __syncthreads();
  incl += wave_sum[wave];
  const uint32_t excl = incl - sum;
  const uint32_t total = wave_sum[T >> 6];
  if (excl < need && need <= incl) {  // exactly one thread
    uint32_t c = excl;
    for (int j = 1; j <= per; ++j) {
      const int b = hi - j;
      if (c + h[b] >= need) {
        *out = Pick{b, c, h[b], total};
        break;
      }
      c += h[b];
    }
  }
  if (need > total && t == 0) *out = Pick{-1, 0, 0, total};
  __syncthreads();
  const Pick r = *out;
  __syncthreads();
  return r;
}

// Sort keys[0, size) descending in one workgroup of kSortThreads threads
// (bitonic network; size a power of two from 64 to 16 * kSortThreads; keys
// beyond the entries to sort are 0 and end up last).  Thread t holds the
// entries q * kSortThreads + t (t < size) in registers: a compare-exchange at
// distance 1024 or more stays in a thread, one below 64 goes through wave
// shuffles, and only the distances 64 .. 512 go through LDS (two barriers
// each); a size of 64 is sorted by the first wave alone, without barriers.
template <int Q>
__device__ __forceinline__ void block_sort_regs(unsigned long long *keys, int size) {
  const int t = threadIdx.x;
  const bool active = t < size;  // size < kSortThreads: whole waves idle
  unsigned long long r[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) r[q] = active ? keys[q * kSortThreads + t] : 0ull;
  for (int len = 2; len <= size; len <<= 1) {
    for (int stride = len >> 1; stride > 0; stride >>= 1) {
      if (stride >= kSortThreads) {
        const int qs = stride / kSortThreads;
#pragma unroll
        for (int c = 1; c < Q; c <<= 1) {  // c: the distance in registers, a constant
          if (qs == c) {
#pragma unroll
            for (int q = 0; q < Q; ++q) {
              if ((q & c) == 0) {
                const int j = q * kSortThreads + t;
                const bool desc = (j & len) == 0;
                const unsigned long long a = r[q], b = r[q | c];
                if (desc ? (a < b) : (a > b)) {
                  r[q] = b;
                  r[q | c] = a;
                }
              }
            }
          }
        }
      } else if (stride >= 64) {
        __syncthreads();
        if (active) {
#pragma unroll
          for (int q = 0; q < Q; ++q) keys[q * kSortThreads + t] = r[q];
        }
        __syncthreads();
        if (active) {
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            const int j = q * kSortThreads + t;
            const unsigned long long o = keys[j ^ stride];
            const bool lower = (j & stride) == 0;
            const bool desc = (j & len) == 0;
            const bool keep_max = lower == desc;
            r[q] = keep_max ? (r[q] > o ? r[q] : o) : (r[q] < o ? r[q] : o);
          }
        }
      } else if (active) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const int j = q * kSortThreads + t;
          const uint32_t lo = __shfl_xor((uint32_t)r[q], stride);
          const uint32_t hi = __shfl_xor((uint32_t)(r[q] >> 32), stride);
          const unsigned long long o = ((unsigned long long)hi << 32) | lo;
          const bool lower = (j & stride) == 0;
          const bool desc = (j & len) == 0;
          const bool keep_max = lower == desc;
          r[q] = keep_max ? (r[q] > o ? r[q] : o) : (r[q] < o ? r[q] : o);
        }
      }
    }
  }
  __syncthreads();
  if (active) {
#pragma unroll
    for (int q = 0; q < Q; ++q) keys[q * kSortThreads + t] = r[q];
  }
  __syncthreads();
}

// keys[0, size) in LDS with size a power of two >= 64.
__device__ __forceinline__ void block_sort_desc(unsigned long long *keys, int size) {
  switch (size <= kSortThreads ? 1 : size / kSortThreads) {
    case 1: block_sort_regs<1>(keys, size); break;
    case 2: block_sort_regs<2>(keys, size); break;
    case 4: block_sort_regs<4>(keys, size); break;
    case 8: block_sort_regs<8>(keys, size); break;
    default: block_sort_regs<16>(keys, size); break;
  }
}

// Sort size of cnt keys: the next power of two, at least one wave.
__host__ __device__ constexpr int sort_size(int cnt) {
  int size = 64;
  while (size < cnt) size <<= 1;
  return size;
}

// Grid-wide barrier number `round` (1, 2, ...) of this call; false if the
// wait ran out (or another workgroup's did): the selection has failed.
__device__ __forceinline__ bool grid_sync(TopkState *st, uint32_t round, long long timeout_ticks, int *ok_s) {
  __syncthreads();
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_add(&st->arrive, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t target = round * gridDim.x;
    const long long t0 = wall_clock64();
    int ok = 1;
    while (__hip_atomic_load(&st->arrive, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) < target) {
      if (__hip_atomic_load(&st->failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u ||
          wall_clock64() - t0 > timeout_ticks) {
        ok = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(4);
    }
    if (!ok) __hip_atomic_store(&st->failed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *ok_s = ok;
  }
  // Only the waiting thread takes the acquire: what the workgroups read of
  // one another's writes (the digit histogram) is read with device-scope
  // atomic loads, and an acquire on every wave would invalidate the L2 once
  // per wave.
  __syncthreads();
  return *ok_s != 0;
}

// In one workgroup: of m keys (get(j), j < m) that share their top `nbits`
// bits (= prefix), the `need` largest (1 <= need <= m) are those whose top
// bits, on return, are >= prefix.  Digit passes over the keys with an LDS
// histogram, until the bin of the need-th key holds exactly the keys still
// needed (at the latest at 64 bits: keys are unique).
template <typename Get>
__device__ __forceinline__ void select_in_block(Get get, int m, uint32_t need, int &nbits,
                                unsigned long long &prefix, uint32_t *h, uint32_t *wave_sum,
                                Pick *pick_s) {
  const int T = blockDim.x;
  for (;;) {
    const int w = digit_width(nbits);
    const int shift = 64 - nbits - w;
    const unsigned long long dmask = (1ull << w) - 1ull;
    for (int b = threadIdx.x; b < kBins; b += T) h[b] = 0;
    __syncthreads();
    for (int j = threadIdx.x; j < m; j += T) {
      const unsigned long long key = get(j);
      if (nbits == 0 || (key >> (64 - nbits)) == prefix) atomicAdd(&h[(key >> shift) & dmask], 1u);
    }
    __syncthreads();
    const Pick p = block_pick(h, 1 << w, need, wave_sum, pick_s);
    need -= p.above;
    prefix = (nbits > 0 ? (prefix << w) : 0ull) | (unsigned long long)p.bin;
    nbits += w;
    if (p.cnt == need || nbits >= 64) return;
  }
}

__global__ void __launch_bounds__(256) topk_init(TopkState *st, uint32_t *hist, int32_t k) {
  for (int b = threadIdx.x; b < 3 * kBins; b += blockDim.x) hist[b] = 0;
  if (threadIdx.x == 0) {
    st->arrive = 0;
    st->failed = 0;
    st->n_take = 0;
    st->n_in = 0;
    st->k = k;
    st->total = 0;
    st->mode = 0;
    st->nbits = 0;
    st->need_in = 0;
    st->prefix = 0;
  }
}

__global__ void __launch_bounds__(kSelThreads) topk_select(
    const uint8_t *valid, const float *scores, int64_t n, int32_t k, int vec,
    long long timeout_ticks, TopkState *st, uint32_t *hist, unsigned long long *take,
    unsigned long long *inbin) {
  __shared__ __align__(8) uint32_t h[kBins];
  __shared__ uint32_t wave_sum[kSelThreads / 64 + 1];
  __shared__ Pick pick_s;
  __shared__ int ok_s;
  const int T = blockDim.x;
  const int lane = threadIdx.x & 63;
  const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  unsigned long long prefix = 0ull;
  int nbits = 0;
  uint32_t need = (uint32_t)k;
  int mode = 0;
  for (int pass = 0; pass < kMaxPasses && mode == 0; ++pass) {
    const int w = digit_width(nbits);
    const int shift = 64 - nbits - w;
    const unsigned long long dmask = (1ull << w) - 1ull;
    for (int b = threadIdx.x; b < kBins; b += T) h[b] = 0;
    __syncthreads();
    for_each_tile(valid, scores, n, vec, [&](const bool *inc, const unsigned long long *key) {
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (inc[e] && (nbits == 0 || (key[e] >> (64 - nbits)) == prefix))
          atomicAdd(&h[(key[e] >> shift) & dmask], 1u);
    });
    __syncthreads();
    uint32_t *H = hist + (pass % 3) * kBins;
    for (int b = threadIdx.x; b < (1 << w); b += T)
      if (h[b]) atomicAdd(&H[b], h[b]);
    if (!grid_sync(st, (uint32_t)pass + 1, timeout_ticks, &ok_s)) return;
    for (int b = threadIdx.x; b < (1 << w); b += T)
      h[b] = __hip_atomic_load(&H[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // the buffer two passes ahead was last read before this barrier
    if (blockIdx.x == 0)
      for (int b = threadIdx.x; b < kBins; b += T) hist[((pass + 2) % 3) * kBins + b] = 0;
    __syncthreads();
    const Pick p = block_pick(h, 1 << w, need, wave_sum, &pick_s);
    if (pass == 0) {  // every workgroup sums the same histogram
      if (blockIdx.x == 0 && threadIdx.x == 0) st->total = (int32_t)p.total;
      if (p.total <= need) {
        mode = kTakeAll;
        break;
      }
    }
    need -= p.above;
    prefix = (nbits > 0 ? (prefix << w) : 0ull) | (unsigned long long)p.bin;
    nbits += w;
    if (p.cnt == need)
      mode = kExact;
    else if (p.cnt <= (uint32_t)kInCap)
      mode = kInBin;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->mode = mode;
    st->nbits = nbits;
    st->prefix = prefix;
    st->need_in = (int32_t)need;
  }
  // The final pass: selected keys and the bin's keys.  A workgroup gathers
  // them in LDS (the histogram's space) and appends them to the lists at its
  // end, with one device-wide addition each: an addition per wave and group of
  // 16 candidates that holds one queued up at the two counters (k = 2048 of
  // 16M: 112 -> 71 us).  Keys past a full gather are appended directly.  A
  // group of which no lane selects any costs one ballot.
  constexpr int kGather = kBins * (int)sizeof(uint32_t) / 2 / (int)sizeof(unsigned long long);
  unsigned long long *gather = reinterpret_cast<unsigned long long *>(h);  // selected, bin
  __shared__ uint32_t gathered[2], base_s[2];
  if (threadIdx.x < 2) gathered[threadIdx.x] = 0;
  __syncthreads();
  auto append = [&](int list, bool mine, unsigned long long key) {
    const uint64_t b = __ballot(mine);
    if (b == 0) return;
    uint32_t p0 = 0;
    if (lane == 0) p0 = atomicAdd(&gathered[list], (uint32_t)__popcll(b));
    p0 = __shfl(p0, 0);
    const uint32_t pos = p0 + (uint32_t)__popcll(b & below);
    if (mine && pos < (uint32_t)kGather) gather[list * kGather + pos] = key;
    const uint64_t rest = __ballot(mine && pos >= (uint32_t)kGather);
    if (rest == 0) return;
    uint32_t g0 = 0;
    if (lane == 0)
      g0 = atomicAdd(list == 0 ? &st->n_take : &st->n_in, (uint32_t)__popcll(rest));
    g0 = __shfl(g0, 0);
    const uint32_t at = g0 + (uint32_t)__popcll(rest & below);
    if (mine && pos >= (uint32_t)kGather) {
      if (list == 0 && at < (uint32_t)k) take[at] = key;
      if (list == 1 && at < (uint32_t)kInCap) inbin[at] = key;
    }
  };
  for_each_tile(valid, scores, n, vec, [&](const bool *inc, const unsigned long long *key) {
    int cls[16];  // 1 selected, 2 in the bin
    bool any = false;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      cls[e] = 0;
      if (inc[e]) {
        if (mode == kTakeAll) {
          cls[e] = 1;
        } else {
          const unsigned long long top = key[e] >> (64 - nbits);
          cls[e] = top > prefix ? 1 : top == prefix ? (mode == kExact ? 1 : 2) : 0;
        }
      }
      any = any || cls[e] != 0;
    }
    if (__ballot(any) == 0) return;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      append(0, cls[e] == 1, key[e]);
      append(1, cls[e] == 2, key[e]);
    }
  });
  __syncthreads();
  if (threadIdx.x < 2) {
    const uint32_t c = min(gathered[threadIdx.x], (uint32_t)kGather);
    gathered[threadIdx.x] = c;
    base_s[threadIdx.x] =
        c ? atomicAdd(threadIdx.x == 0 ? &st->n_take : &st->n_in, c) : 0u;
  }
  __syncthreads();
  for (uint32_t j = threadIdx.x; j < gathered[0]; j += T)
    if (base_s[0] + j < (uint32_t)k) take[base_s[0] + j] = gather[j];
  for (uint32_t j = threadIdx.x; j < gathered[1]; j += T)
    if (base_s[1] + j < (uint32_t)kInCap) inbin[base_s[1] + j] = gather[kGather + j];
}

// The place of a key in its list, counted by a workgroup: sixteen threads per
// key, each over a sixteenth of the list, which passes through LDS kRankTile
// keys at a time.  Thread t has key x of entry (t & 63) of the workgroup;
// returns the keys of list[0, m) above x, and with POS those equal to it at
// earlier positions than `pos` (to all sixteen threads of the key; every thread
// of the workgroup calls it).
//
// Why counting and not a sort: the sort of k keys is a chain of compare
// exchanges in one workgroup, while the k * m comparisons spread over m / 64
// workgroups and have no chain (selection of a 16M pool, k = 1024: 84 -> 75 us;
// second level's 1,024 rows: 14 -> 5 us).
constexpr int kRankThreads = 1024;
constexpr int kRankKeys = 64;  // keys ranked by a workgroup
constexpr int kRankParts = kRankThreads / kRankKeys;
constexpr int kRankTile = 1024;
template <bool POS, typename Get>
__device__ __forceinline__ int count_above(Get get, int m, unsigned long long x, int pos,
                                           unsigned long long *tile, int *sum) {
  const int part = threadIdx.x >> 6, key = threadIdx.x & 63;
  int above = 0;
  for (int base = 0; base < m; base += kRankTile) {
    const int left = m - base < kRankTile ? m - base : kRankTile;
    static_assert(kRankTile == kRankThreads, "a thread stages one key of a tile");
    const int j0 = (int)threadIdx.x;
    const unsigned long long staged = j0 < left ? get(base + j0) : 0ull;  // no key is below 0
    __syncthreads();
    tile[j0] = staged;
    __syncthreads();
    const int per = (left + kRankParts - 1) / kRankParts;
    const int lo = part * per, hi = lo + per < kRankTile ? lo + per : kRankTile;
#pragma unroll 8
    for (int j = lo; j < hi; ++j) {
      // at an earlier position an equal key counts too
      const unsigned long long y = (POS && base + j < pos) ? x - 1ull : x;
      above += tile[j] > y ? 1 : 0;
    }
  }
  __syncthreads();
  sum[threadIdx.x] = above;
  __syncthreads();
  int all = 0;
#pragma unroll
  for (int p = 0; p < kRankParts; ++p) all += sum[p * kRankKeys + key];
  return all;
}

// The outputs.  Workgroup w ranks keys [64 w, 64 w + 64) of the selected list
// followed by the threshold bin's: a selected key's place is the number of
// selected keys above it, a bin's key comes after all of them, at the number
// of the bin's above it, and is selected if that is below need_in.
__global__ void __launch_bounds__(kRankThreads) topk_finish(const float *scores, int64_t n,
                                                            const TopkState *st,
                                                            const unsigned long long *take,
                                                            const unsigned long long *inbin,
                                                            int32_t *idx, float *out,
                                                            int32_t *num) {
  __shared__ unsigned long long tile[kRankTile];
  __shared__ int sum[kRankThreads];
  const int k = st->k;
  const int mode = st->failed ? 0 : st->mode;
  const int cnt = mode == 0 ? 0 : min(k, st->total);
  const int nt = mode == 0 ? 0 : (int)min(st->n_take, (uint32_t)k);
  const int m = mode == kInBin ? (int)min(st->n_in, (uint32_t)kInCap) : 0;
  for (int j = cnt + (int)(blockIdx.x * kRankThreads + threadIdx.x); j < k;
       j += (int)gridDim.x * kRankThreads) {
    idx[j] = -1;
    out[j] = -INFINITY;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) *num = st->failed ? -1 : cnt;
  // the workgroup's keys lie in one list: the bin's start at a multiple of 64
  const int first = (int)blockIdx.x * kRankKeys, bin0 = (nt + kRankKeys - 1) / kRankKeys * kRankKeys;
  const bool in_bin = first >= bin0;
  const int e = first + (int)(threadIdx.x & 63) - (in_bin ? bin0 : 0);
  const int len = in_bin ? m : nt;
  if (first - (in_bin ? bin0 : 0) >= len) return;  // the same in every thread
  const unsigned long long *list = in_bin ? inbin : take;
  const unsigned long long x = e < len ? list[e] : 0ull;
  const int above =
      count_above<false>([&](int j) { return list[j]; }, len, x, 0, tile, sum);
  const int place = (in_bin ? nt : 0) + above;
  const int limit = in_bin ? min(cnt, nt + st->need_in) : cnt;
  const int64_t i = (int64_t)(0xFFFFFFFFu - (uint32_t)(x & 0xFFFFFFFFull));
  if (threadIdx.x < kRankKeys && e < len && place < limit && i < n) {
    idx[place] = (int32_t)i;
    out[place] = scores[i];
  }
}

// Pools of at most kSmallN candidates, in one launch of one workgroup: the
// included keys are gathered into LDS, the k largest selected there (digit
// passes) and sorted.  LDS: the sort area (sort_size(min(k, n)) keys), then
// the gathered keys (n).
__global__ void __launch_bounds__(kSortThreads) topk_small(const uint8_t *valid,
                                                           const float *scores, int64_t n,
                                                           int32_t k, int32_t *idx, float *out,
                                                           int32_t *num) {
  extern __shared__ unsigned long long lds_keys[];
  __shared__ uint32_t h[kBins];
  __shared__ uint32_t wave_sum[kSortThreads / 64 + 1];
  __shared__ Pick pick_s;
  __shared__ uint32_t cnt_s, fill_s;
  const int T = blockDim.x;
  const int lane = threadIdx.x & 63;
  const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  const int nn = (int)n;
  const int size = sort_size(min(k, nn));
  unsigned long long *B = lds_keys;
  unsigned long long *A = lds_keys + size;
  if (threadIdx.x == 0) {
    cnt_s = 0;
    fill_s = 0;
  }
  for (int j = threadIdx.x; j < size; j += T) B[j] = 0ull;
  __syncthreads();
  for (int base = 0; base < nn; base += T) {  // uniform trip count: ballots below
    const int i = base + threadIdx.x;
    bool inc = false;
    float sc = 0.0f;
    if (i < nn) {
      sc = scores[i];
      inc = (!valid || valid[i] != 0) && !isnan(sc);
    }
    const uint64_t bal = __ballot(inc);
    if (bal) {
      uint32_t p0 = 0;
      if (lane == 0) p0 = atomicAdd(&cnt_s, (uint32_t)__popcll(bal));
      p0 = __shfl(p0, 0);
      if (inc) A[p0 + __popcll(bal & below)] = make_key(sc, i);
    }
  }
  __syncthreads();
  const int m = (int)cnt_s;
  const int cnt = min(k, m);
  if (m <= k) {
    for (int j = threadIdx.x; j < m; j += T) B[j] = A[j];
  } else if (cnt > 0) {
    int nbits = 0;
    unsigned long long prefix = 0ull;
    select_in_block([&](int j) { return A[j]; }, m, (uint32_t)k, nbits, prefix, h, wave_sum,
                    &pick_s);
    for (int j = threadIdx.x; j < m; j += T) {
      const unsigned long long key = A[j];
      if ((key >> (64 - nbits)) >= prefix) {
        const uint32_t pos = atomicAdd(&fill_s, 1u);
        if ((int)pos < size) B[pos] = key;
      }
    }
  }
  __syncthreads();
  block_sort_desc(B, size);
  for (int j = threadIdx.x; j < k; j += T) {
    const int64_t i = (int64_t)(0xFFFFFFFFu - (uint32_t)(B[j] & 0xFFFFFFFFull));
    if (j < cnt && B[j] != 0ull && i < n) {
      idx[j] = (int32_t)i;
      out[j] = scores[i];
    } else {
      idx[j] = -1;
      out[j] = -INFINITY;
    }
  }
  if (threadIdx.x == 0) *num = cnt;
}

// Float32 of an order-preserving key's high word (inverse of make_key's map;
// a zero comes back as +0.0).
__device__ __forceinline__ float key_score(unsigned long long key) {
  const uint32_t ord = (uint32_t)(key >> 32);
  const uint32_t b = (ord & 0x80000000u) ? (ord & 0x7FFFFFFFu) : ~ord;
  return __uint_as_float(b);
}

// Key of a listed row for the second-level selection: the high word orders
// by score (-0.0 and +0.0 equal), the low word by pool row ascending
// (0x7FFFFFFF - row, row < 2^31, in bits 31..1) and keeps, in bit 0, the
// sign of a zero score, so that the chosen entry's score comes back bit for
// bit.  Two entries of one row carry the same score (the same row walked by
// the same model), so bit 0 never reorders distinct scores.
__device__ __forceinline__ unsigned long long row_key(float s, int32_t row) {
  const uint32_t neg_zero = (__float_as_uint(s) == 0x80000000u) ? 1u : 0u;
  const uint32_t lo = ((0x7FFFFFFFu - (uint32_t)row) << 1) | neg_zero;
  return (make_key(s, 0) & 0xFFFFFFFF00000000ull) | (unsigned long long)lo;
}
__device__ __forceinline__ int32_t row_key_row(unsigned long long key) {
  return (int32_t)(0x7FFFFFFFu - ((uint32_t)key >> 1));
}
__device__ __forceinline__ float row_key_score(unsigned long long key) {
  return (key & 1ull) ? -0.0f : key_score(key);
}

// Second-level selection (model A): workgroup w ranks list entries [64 w, 64 w
// + 64) by their keys (row_key; equal keys, a row listed twice, in list
// order) and writes those of the best `keep`.  Rows outside [0, n) and NaN
// scores are left out (key 0, below every included key: a zero high word is
// the ord of a negative NaN).
__global__ void __launch_bounds__(kRankThreads) rerank_select(const int32_t *rows,
                                                              const float *scores, int32_t m,
                                                              int64_t n, int32_t keep,
                                                              int32_t *idx, float *out,
                                                              int32_t *num) {
  __shared__ unsigned long long tile[kRankTile];
  __shared__ int sum[kRankThreads];
  __shared__ int included_s;
  int mine = 0;  // included entries this thread has fetched
  auto key_of = [&](int j) -> unsigned long long {
    const int32_t r = rows[j];
    const float sc = scores[j];
    return (r >= 0 && r < n && !isnan(sc)) ? row_key(sc, r) : 0ull;
  };
  if (threadIdx.x == 0) included_s = 0;
  const int e = (int)blockIdx.x * kRankKeys + (int)(threadIdx.x & 63);
  const unsigned long long x = e < m ? key_of(e) : 0ull;
  const int place = count_above<true>(
      [&](int j) {
        const unsigned long long key = key_of(j);
        mine += key != 0ull ? 1 : 0;
        return key;
      },
      m, x, e, tile, sum);
  if (mine) atomicAdd(&included_s, mine);
  __syncthreads();
  const int cnt = min(included_s, keep);
  if (threadIdx.x < kRankKeys && x != 0ull && place < cnt) {
    idx[place] = row_key_row(x);
    out[place] = row_key_score(x);
  }
  for (int j = cnt + (int)(blockIdx.x * kRankThreads + threadIdx.x); j < keep;
       j += (int)gridDim.x * kRankThreads) {
    idx[j] = -1;
    out[j] = -INFINITY;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) *num = cnt;
}

// The same in one workgroup that has read every entry before it writes one
// (a bitonic sort in LDS): for outputs that share memory with the list.
__global__ void __launch_bounds__(kSortThreads) rerank_select_one(const int32_t *rows,
                                                                  const float *scores, int32_t m,
                                                                  int64_t n, int32_t keep,
                                                                  int32_t *idx, float *out,
                                                                  int32_t *num) {
  extern __shared__ unsigned long long keys[];
  __shared__ int included_s;
  if (threadIdx.x == 0) included_s = 0;
  const int size = sort_size(m);
  __syncthreads();
  int mine = 0;
  for (int j = threadIdx.x; j < size; j += blockDim.x) {
    unsigned long long key = 0ull;
    if (j < m) {
      const int32_t r = rows[j];
      const float sc = scores[j];
      if (r >= 0 && r < n && !isnan(sc)) {
        key = row_key(sc, r);
        ++mine;
      }
    }
    keys[j] = key;
  }
  if (mine) atomicAdd(&included_s, mine);
  __syncthreads();
  block_sort_desc(keys, size);
  const int cnt = min(included_s, keep);
  for (int j = threadIdx.x; j < keep; j += blockDim.x) {
    if (j < cnt) {
      idx[j] = row_key_row(keys[j]);
      out[j] = row_key_score(keys[j]);
    } else {
      idx[j] = -1;
      out[j] = -INFINITY;
    }
  }
  if (threadIdx.x == 0) *num = cnt;
}

// Rows already proposed leave the pool: mask[rows[j]] = 0 for the listed rows
// inside [0, n) (the -1 padding of short rounds is skipped).
__global__ void __launch_bounds__(256) exclude_rows(uint8_t *mask, int64_t n,
                                                    const int32_t *rows, int32_t m) {
  const int32_t j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= m) return;
  const int32_t r = rows[j];
  if (r >= 0 && r < n) mask[r] = 0;
}

// A chunk of pool rows row0 .. row0+m-1 (streamed explorer): rows proposed in
// earlier rounds leave the chunk's mask, mask[r - row0] = 0 for every listed
// row r inside the chunk (the -1 padding of short rounds never is).
__global__ void __launch_bounds__(256) exclude_range(uint8_t *mask, int64_t row0, int64_t m,
                                                     const int32_t *rows, int32_t count) {
  const int32_t j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= count) return;
  const int64_t r = rows[j];
  if (r >= row0 && r < row0 + m) mask[r - row0] = 0;
}

// An empty held set: no rows, every slot -1 / -inf.
__global__ void __launch_bounds__(256) held_reset(int32_t *held_id, float *held_p,
                                                  float *held_a, int32_t *held_n, int32_t k) {
  for (int32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < k; j += gridDim.x * blockDim.x) {
    held_id[j] = -1;
    held_p[j] = -INFINITY;
    held_a[j] = -INFINITY;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) *held_n = 0;
}

// The held set of the streamed explorer after one more chunk: the k best of
// the rows held so far (h_*, *h_n of them) and the chunk's selection (c_*,
// *c_n of them, chunk-local indices; pool row = row0 + index) by (P score
// desc, pool row asc), a row present in both counted once.  Each entry
// carries its P score and its second-level score (model A's, or P's again
// when c_a is NULL), copied bit for bit.  One workgroup: both lists are sorted
// by their keys (ord(P) << 32) | (0xFFFFFFFF - row) and have no key twice, so
// an entry's place is its position in its own list plus the other list's keys
// above it (a binary search in LDS), less the chunk's entries above it that
// are held already (a prefix count); equal keys are the same row with the
// same score, and the chunk's is dropped.
__device__ __forceinline__ int keys_above(const unsigned long long *list, int n,
                                          unsigned long long x) {
  int lo = 0, len = n;
  while (len > 0) {
    const int half = (len + 1) >> 1;
    lo = list[lo + half - 1] > x ? lo + half : lo;
    len -= half;
  }
  return lo;
}

__global__ void __launch_bounds__(kSortThreads) merge_held(
    const int32_t *h_id, const float *h_p, const float *h_a, const int32_t *h_n,
    const int32_t *c_idx, const float *c_p, const float *c_a, const int32_t *c_n, int64_t row0,
    int32_t k, int32_t *o_id, float *o_p, float *o_a, int32_t *o_n) {
  extern __shared__ unsigned long long keys[];  // held [k], chunk [k], then twins [k + 1]
  __shared__ int warp_sum[kSortThreads / 64 + 1];
  unsigned long long *held = keys, *chunk = keys + k;
  int32_t *twins = reinterpret_cast<int32_t *>(keys + 2 * k);  // chunk entries held, before j
  const int hn = max(min(*h_n, k), 0), cn = max(min(*c_n, k), 0);
  for (int j = threadIdx.x; j < hn; j += blockDim.x) held[j] = make_key(h_p[j], h_id[j]);
  for (int j = threadIdx.x; j < cn; j += blockDim.x)
    chunk[j] = make_key(c_p[j], row0 + c_idx[j]);
  __syncthreads();
  // twins[j], by threads of four consecutive entries (k <= 4 * kSortThreads)
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lo = 4 * (int)threadIdx.x;
  int twin[4], mine = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int j = lo + q;
    twin[q] = 0;
    if (j < cn) {
      const int at = keys_above(held, hn, chunk[j]);
      twin[q] = (at < hn && held[at] == chunk[j]) ? 1 : 0;
    }
    mine += twin[q];
  }
  int incl = mine;
  for (int d = 1; d < 64; d <<= 1) {
    const int v = __shfl_up(incl, d);
    if (lane >= d) incl += v;
  }
  if (lane == 63) warp_sum[wave] = incl;
  __syncthreads();
  if (threadIdx.x == 0) {
    int acc = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
      const int t = warp_sum[w];
      warp_sum[w] = acc;
      acc += t;
    }
    warp_sum[blockDim.x >> 6] = acc;
  }
  __syncthreads();
  int before = warp_sum[wave] + incl - mine;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (lo + q < k) twins[lo + q] = before;
    before += twin[q];
  }
  const int all_twins = warp_sum[blockDim.x >> 6];
  if (threadIdx.x == 0) twins[k] = all_twins;
  __syncthreads();
  for (int j = threadIdx.x; j < hn; j += blockDim.x) {
    const int above = keys_above(chunk, cn, held[j]);
    const int r = j + above - (above < cn ? twins[above] : all_twins);
    if (r < k) {
      o_id[r] = h_id[j];
      o_p[r] = h_p[j];
      o_a[r] = h_a[j];
    }
  }
  for (int j = threadIdx.x; j < cn; j += blockDim.x) {
    const int above = keys_above(held, hn, chunk[j]);
    if (above < hn && held[above] == chunk[j]) continue;  // held already
    const int r = j - twins[j] + above;
    if (r < k) {
      o_id[r] = (int32_t)(row0 + c_idx[j]);
      o_p[r] = c_p[j];
      o_a[r] = c_a ? c_a[j] : c_p[j];
    }
  }
  const int total = min(hn + cn - all_twins, k);
  for (int r = total + (int)threadIdx.x; r < k; r += blockDim.x) {
    o_id[r] = -1;
    o_p[r] = -INFINITY;
    o_a[r] = -INFINITY;
  }
  if (threadIdx.x == 0) *o_n = total;
}

}  // namespace

// Workspace: state, three digit histograms, the selected list (k keys) and
// the threshold bin's list (kInCap keys).  Independent of n.
size_t topk_workspace_bytes(int64_t n, int32_t k) {
  (void)n;
  const size_t take = (size_t)(k > 0 ? k : 1) * sizeof(unsigned long long);
  const size_t inbin = (size_t)kInCap * sizeof(unsigned long long);
  return (kStateBytes + kHistBytes + take + inbin + 255) & ~(size_t)255;
}

// The selection's workspace for callers that cannot allocate
// (ml2_filter_topk_noalloc): one file-scope array per device, sized for the
// largest k, shared by every such call on that device.  Host code never
// passes `scratch` itself to a kernel (on the host it only names the
// symbol); it uses the device address hipGetSymbolAddress returns, taken
// once per device with that device current.
constexpr size_t kStaticScratchBytes =
    (kStateBytes + kHistBytes + (size_t)(ML2_MAX_TOPK + kInCap) * sizeof(unsigned long long) +
     255) &
    ~(size_t)255;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

size_t static_scratch_bytes() { return kStaticScratchBytes; }

hipError_t static_scratch(int device, void **ptr) {
  static std::mutex mu;
  static std::vector<void *> addr;
  std::lock_guard<std::mutex> lock(mu);
  if ((int)addr.size() <= device) addr.resize((size_t)device + 1, nullptr);
  if (!addr[(size_t)device]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p || (reinterpret_cast<uintptr_t>(p) & 255u)) return hipErrorInvalidSymbol;
    addr[(size_t)device] = p;
  }
  *ptr = addr[(size_t)device];
  return hipSuccess;
}

namespace {

// Wall-clock ticks of the grid barrier's longest wait, per device.
hipError_t barrier_ticks(long long *ticks) {
  static std::mutex mu;
  static std::vector<long long> cache;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(mu);
  if ((int)cache.size() <= dev) cache.resize((size_t)dev + 1, 0);
  if (cache[(size_t)dev] == 0) {
    int khz = 0;
    e = hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev);
    if (e != hipSuccess) return e;
    if (khz <= 0) khz = 100000;  // the 100 MHz constant clock
    cache[(size_t)dev] = (long long)(kBarrierSeconds * 1000.0 * khz);
  }
  *ticks = cache[(size_t)dev];
  return hipSuccess;
}


}  // namespace

hipError_t launch_topk(const uint8_t *valid, const float *scores, int64_t n, int32_t k,
                       int32_t *idx, float *score, int32_t *num, void *ws, int cu_count,
                       hipStream_t s) {
  char *w = static_cast<char *>(ws);
  TopkState *st = reinterpret_cast<TopkState *>(w);
  uint32_t *hist = reinterpret_cast<uint32_t *>(w + kStateBytes);
  unsigned long long *take =
      reinterpret_cast<unsigned long long *>(w + kStateBytes + kHistBytes);
  unsigned long long *inbin = take + (k > 0 ? k : 1);
  if (n <= kSmallN) {
    const size_t lds =
        ((size_t)sort_size(min((int64_t)k, n)) + (size_t)(n > 0 ? n : 1)) * sizeof(unsigned long long);
    const size_t most = ((size_t)sort_size(kSmallN) + kSmallN) * sizeof(unsigned long long);
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(&topk_small), most);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(topk_small, dim3(1), dim3(kSortThreads), lds, s, valid, scores, n, k, idx,
                       score, num);
    return hipGetLastError();
  }
  long long ticks = 0;
  hipError_t e = barrier_ticks(&ticks);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(topk_init, dim3(1), dim3(256), 0, s, st, hist, k);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (n > 0 && k > 0) {
    const int vec = ((reinterpret_cast<uintptr_t>(scores) & 15u) == 0 &&
                     (reinterpret_cast<uintptr_t>(valid) & 3u) == 0)
                        ? 1
                        : 0;
    const int64_t per_wg = (int64_t)kTile * (kSelThreads / 64);
    int64_t grid = (n + per_wg - 1) / per_wg;
    if (grid > cu_count) grid = cu_count;
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(topk_select, dim3((unsigned)grid), dim3(kSelThreads), 0, s, valid, scores,
                       n, k, vec, ticks, st, hist, take, inbin);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  // a workgroup per 64 selected keys (at most k) and per 64 of the bin's
  const unsigned finish = (unsigned)((k + kRankKeys - 1) / kRankKeys + kInCap / kRankKeys);
  hipLaunchKernelGGL(topk_finish, dim3(finish), dim3(kRankThreads), 0, s, scores, n, st, take,
                     inbin, idx, score, num);
  return hipGetLastError();
}

hipError_t launch_rerank_select(const int32_t *rows, const float *scores, int32_t m, int64_t n,
                                int32_t keep, int32_t *idx, float *score, int32_t *num,
                                hipStream_t s) {
  auto overlap = [](const void *a, size_t na, const void *b, size_t nb) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y + nb && y < x + na;
  };
  const size_t in = 4 * (size_t)m, outs = 4 * (size_t)keep;
  bool shared = false;
  for (const void *list : {static_cast<const void *>(rows), static_cast<const void *>(scores)})
    shared = shared || overlap(list, in, idx, outs) || overlap(list, in, score, outs) ||
             overlap(list, in, num, 4);
  if (shared) {
    const size_t lds = (size_t)sort_size(m) * sizeof(unsigned long long);
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(&rerank_select_one), lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(rerank_select_one, dim3(1), dim3(kSortThreads), lds, s, rows, scores, m, n,
                       keep, idx, score, num);
    return hipGetLastError();
  }
  const unsigned grid = (unsigned)std::max(1, (m + kRankKeys - 1) / kRankKeys);
  hipLaunchKernelGGL(rerank_select, dim3(grid), dim3(kRankThreads), 0, s, rows, scores, m, n,
                     keep, idx, score, num);
  return hipGetLastError();
}

hipError_t launch_exclude(uint8_t *mask, int64_t n, const int32_t *rows, int32_t m,
                          hipStream_t s) {
  if (m <= 0) return hipSuccess;
  hipLaunchKernelGGL(exclude_rows, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, s, mask, n,
                     rows, m);
  return hipGetLastError();
}

hipError_t launch_exclude_range(uint8_t *mask, int64_t row0, int64_t m, const int32_t *rows,
                                int32_t count, hipStream_t s) {
  if (count <= 0 || m <= 0) return hipSuccess;
  hipLaunchKernelGGL(exclude_range, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, mask,
                     row0, m, rows, count);
  return hipGetLastError();
}

hipError_t launch_held_reset(int32_t *held_id, float *held_p, float *held_a, int32_t *held_n,
                             int32_t k, hipStream_t s) {
  hipLaunchKernelGGL(held_reset, dim3((unsigned)((k + 255) / 256)), dim3(256), 0, s, held_id,
                     held_p, held_a, held_n, k);
  return hipGetLastError();
}

size_t merge_held_lds(int32_t k) {
  return (size_t)k * (2 * sizeof(unsigned long long) + sizeof(int32_t)) + sizeof(int64_t);
}

hipError_t launch_merge_held(const int32_t *h_id, const float *h_p, const float *h_a,
                             const int32_t *h_n, const int32_t *c_idx, const float *c_p,
                             const float *c_a, const int32_t *c_n, int64_t row0, int32_t k,
                             int32_t *o_id, float *o_p, float *o_a, int32_t *o_n, hipStream_t s) {
  const size_t lds = merge_held_lds(k);
  hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(&merge_held), lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(merge_held, dim3(1), dim3(kSortThreads), lds, s, h_id, h_p, h_a, h_n, c_idx,
                     c_p, c_a, c_n, row0, k, o_id, o_p, o_a, o_n);
  return hipGetLastError();
}

}  // namespace ml2
