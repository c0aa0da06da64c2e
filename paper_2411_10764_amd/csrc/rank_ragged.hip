// Walks over the rank form of ragged trees (rank_pack.h).
//
// Each lane walks one tree at a time at its own pace, as the float walk over
// ragged slots does (walk_slot_single): a leaf's value is added and the walk
// moves to the next tree's root in the same step, and past the last tree a
// lane adds -0.0 on the slot's sentinel.  A step is a chain: the node's read,
// the code's read, and the instructions that pick the next node between them.
// Codes shorten both sides of it.  A byte per feature lets 24 waves share a CU
// where float tiles of 64 features let eight, and the step takes ten
// vector instructions instead of nineteen: the direction is one saturated
// subtraction and a minimum, 0 or 8, added to the child's offset, with the
// missing value's way folded into the code by an addition modulo 2^16.
// 16M x 128 pool, half accepted, P 300 trees of depth up to 14 over 64 visible
// features: 10.3 -> 4.6 ms; 3M x 96, P over all features with missing values:
// 3.3 -> 1.0 ms.
#include "rank_walk.h"

namespace ml2 {
namespace rank {
namespace {

// The trees of the slot at LDS address 0.  Every lane is done after at most
// (trees) x (depth + 1) steps; the loop stops a little past that at the
// latest.
template <bool BYTE>
__device__ __forceinline__ float walk_slot(uint32_t mask, uint32_t tile_lane, float m) {
  const u32x4 head = lds_read<u32x4>(0);  // trees, deepest path, the sentinel's node
  uint32_t at = 8u * lds_read<uint32_t>(16);
  const uint32_t end = 8u * head.z;
  const uint32_t cap = (uint32_t)__builtin_amdgcn_readfirstlane((int)(head.x * (head.y + 2u))) + 8u;
  uint64_t nd = lds_read<uint64_t>(at);
  uint32_t it = 0;
  bool go = true;
  while (go) {
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint32_t w0 = (uint32_t)nd, w1 = (uint32_t)(nd >> 32);
      // a leaf reads some code of the tile too, and ignores it
      const uint32_t where = tile_lane + (w1 & mask);
      uint32_t x = BYTE ? lds_read<uint8_t>(where) : lds_read<uint16_t>(where);
      __builtin_amdgcn_sched_barrier(0);
      const float add = (w0 & 0xFFFFu) == 0xFFFFu ? __uint_as_float(w1) : -0.0f;
      m = m + add;
      if (BYTE) x <<= 8;
      const uint32_t z = x + (w1 >> 16);  // (its low half)
      uint32_t d;
      asm("v_sub_u16_e64 %0, %1, %2 clamp" : "=v"(d) : "v"(z), "v"(w0));
      asm("v_min_u16_e32 %0, 8, %0" : "+v"(d));
      at = (w0 >> 16) + d;
      nd = lds_read<uint64_t>(at);
      __builtin_amdgcn_sched_barrier(0);
    }
    it += 8;
    go = !__all(at == end) && it < cap;
  }
  return m;
}

// LDS: the slot at address 0 (nodes hold LDS addresses, so the kernel has no
// static LDS), the tiles, the queue, the waves' counts.
template <bool BYTE, int W, bool PERF>
__global__ void __launch_bounds__(kLanes *(W == 24 ? 12 : W))
__attribute__((amdgpu_waves_per_eu(W / 4, W / 4))) ragged_kernel(RankArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int lane = threadIdx.x & (kLanes - 1);
  const int wave = threadIdx.x / kLanes;
  const int nw = a.nthreads / kLanes;
  Slots<rank_ragged_stage_regs(W)> st;
  st.buf = smem;
  const uint32_t tile_lane = a.slot_bytes + (uint32_t)wave * a.tile_bytes + 4u * lane;
  char *queue = smem + a.slot_bytes + (size_t)nw * a.tile_bytes;
  int *wave_count = reinterpret_cast<int *>(queue + (size_t)nw * 2 * kLanes * sizeof(int32_t));
  st.prime(a);
  const auto *chunks = constant(a.chunks);
  uint32_t mask = a.off_mask;
  asm("" : "+v"(mask));
  rounds<PERF, true>(a, tile_lane, 0u, st, reinterpret_cast<int32_t *>(queue), wave_count,
                     [&](bool busy) {
                       float m = a.base;
                       for (int c = 0; c < a.nchunks; ++c) {
                         st.need(a, chunks[c].slot);
                         if (busy) m = walk_slot<BYTE>(mask, tile_lane, m);
                       }
                       return m;
                     });
}

template <bool BYTE, int W, bool PERF>
hipError_t launch_ragged_one(const RankArgs &a, int grid, size_t lds, hipStream_t s) {
  const void *fn = reinterpret_cast<const void *>(&ragged_kernel<BYTE, W, PERF>);
  hipError_t e = ensure_dynamic_lds(fn, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((ragged_kernel<BYTE, W, PERF>), dim3(grid), dim3(a.nthreads), lds, s, a);
  return hipGetLastError();
}

template <bool BYTE, bool PERF>
hipError_t launch_ragged(int waves, const RankArgs &a, int grid, size_t lds, hipStream_t s) {
  if (waves > 16) return launch_ragged_one<BYTE, 24, PERF>(a, grid, lds, s);
  if (waves > 12) return launch_ragged_one<BYTE, 16, PERF>(a, grid, lds, s);
  if (waves > 8) return launch_ragged_one<BYTE, 12, PERF>(a, grid, lds, s);
  if (waves > 4) return launch_ragged_one<BYTE, 8, PERF>(a, grid, lds, s);
  return launch_ragged_one<BYTE, 4, PERF>(a, grid, lds, s);
}

}  // namespace
}  // namespace rank

hipError_t launch_rank_ragged_kernel(bool perf, RankMode mode, int waves, const RankArgs &a,
                                     int grid, size_t lds, hipStream_t s) {
  if (mode == kRankByte)
    return perf ? rank::launch_ragged<true, true>(waves, a, grid, lds, s)
                : rank::launch_ragged<true, false>(waves, a, grid, lds, s);
  return perf ? rank::launch_ragged<false, true>(waves, a, grid, lds, s)
              : rank::launch_ragged<false, false>(waves, a, grid, lds, s);
}

}  // namespace ml2
