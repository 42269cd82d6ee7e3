// A one-pass exclusive prefix sum fused with the kernel that makes its inputs
// and the one that uses its results (device code of level_pass.hip).
//
// A level of a build needs the prefix sums of a handful of flags and counts per
// block (runs, unmarked ranks, children, windows).  As separate launches, each
// wrote an array, scanned it in one to five launches and read it again in the
// next kernel; at a few thousand blocks a launch costs more than its work.  Here
// f.value(i, v) makes element i's NV values in registers, the tile's sums pass
// along by decoupled look-back (Section 2.2's all-prefix operation, one status
// word per tile and value), and f.apply(i, ex, v) writes what the sums are for.
//
// A status word packs a 40-bit sum, two state bits and the 22-bit epoch of the
// scan, so one buffer, cleared when it is allocated, serves all scans of a build
// in turn; tiles are handed out by a ticket counter that only grows, so a tile
// waits only on tiles that running workgroups hold.
#pragma once
#include "common.hpp"
#include "internal.hpp"

namespace bt {

// A wave takes ROWS rows of 64 consecutive elements, one after another, each a
// chain of dependent loads: one row up to 2^18 elements, so that a small level is
// spread over the chip (marks of levels of 2 to 65536 blocks: 15.5 -> 7.1 us each,
// against eight rows), two up to 2^21, eight beyond, where the chip is full anyway
// and fewer tiles mean a shorter look-back.
constexpr int kPassWaves = kPassThreads / 64;
static_assert(kPassThreads == 256, "four waves");
constexpr uint64_t kPassSum = (1ull << 40) - 1;

// Sum of the tiles before `tile`; publishes this tile's own (whole wave calls it).
__device__ __forceinline__ uint64_t pass_look_back(uint64_t* status, uint64_t epoch, uint64_t tile,
                                                   uint64_t agg) {
  const uint64_t tag = epoch << 42, has_agg = 1ull << 40, has_all = 2ull << 40;
  const int lane = lane_id();
  if (tile == 0) {
    if (lane == 0) st_relaxed(&status[0], tag | has_all | agg);
    return 0;
  }
  if (lane == 0) st_relaxed(&status[tile], tag | has_agg | agg);
  uint64_t excl = 0;
  int64_t look = (int64_t)tile - 1;
  while (true) {
    const int64_t pred = look - lane;
    uint64_t w = 0;
    if (pred >= 0) {
      do { w = ld_relaxed(&status[pred]); } while ((w >> 42) != epoch || !((w >> 40) & 3));
    }
    const uint64_t all = __ballot(pred >= 0 && (w & has_all));
    const int stop = all ? __ffsll((unsigned long long)all) - 1 : 64;
    uint64_t term = (lane <= stop && pred >= 0) ? (w & kPassSum) : 0;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) term += __shfl_xor(term, d);
    excl += term;
    if (all) break;
    look -= 64;
  }
  if (lane == 0) st_relaxed(&status[tile], tag | has_all | (excl + agg));
  return excl;
}

// The whole grid (one workgroup of kPassThreads per tile of kPassThreads * ROWS)
// scans n elements.
// Values whose bit is set in FLAGS are 0 or 1.  f.total(sums) runs once.
template <int NV, uint32_t FLAGS, int ROWS, class F>
__device__ __forceinline__ void scan_pass(uint64_t n, const ScanDev& sd, F&& f) {
  __shared__ uint64_t s_w[NV][kPassWaves];
  __shared__ uint64_t s_ex[NV];
  __shared__ uint64_t s_tile;
  const int lane = lane_id(), wv = threadIdx.x >> 6;
  uint64_t tile = 0;
  if (gridDim.x > 1) {  // (a lone tile takes no ticket and looks at no other)
    if (threadIdx.x == 0) s_tile = atomicAdd((unsigned long long*)sd.ticket, 1ull) - sd.base;
    __syncthreads();
    tile = s_tile;
  }
  const uint64_t wbase = (tile * kPassWaves + wv) * (64 * ROWS);
  uint64_t v[ROWS][NV], ex[ROWS][NV], run[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) run[q] = 0;
#pragma unroll
  for (int k = 0; k < ROWS; ++k) {
    const uint64_t i = wbase + 64ull * k + lane;
#pragma unroll
    for (int q = 0; q < NV; ++q) v[k][q] = 0;
    if (i < n) f.value(i, v[k]);
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      if ((FLAGS >> q) & 1) {
        const uint64_t bal = __ballot(v[k][q] != 0);
        ex[k][q] = run[q] + __popcll(bal & ((1ull << lane) - 1));
        run[q] += __popcll(bal);
      } else {
        uint64_t x = v[k][q];
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const uint64_t o = __shfl_up(x, d);
          if (lane >= d) x += o;
        }
        ex[k][q] = run[q] + x - v[k][q];
        run[q] += shfl64(x, 63);
      }
    }
  }
  if (lane == 0) {
#pragma unroll
    for (int q = 0; q < NV; ++q) s_w[q][wv] = run[q];
  }
  __syncthreads();
  uint64_t before[NV], agg[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    before[q] = agg[q] = 0;
#pragma unroll
    for (int w = 0; w < kPassWaves; ++w) {
      if (w < wv) before[q] += s_w[q][w];
      agg[q] += s_w[q][w];
    }
  }
  if (gridDim.x > 1) {
    if (wv == 0) {
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        const uint64_t e = pass_look_back(sd.status + q * sd.stride, sd.epoch, tile, agg[q]);
        if (lane == 0) s_ex[q] = e;
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      before[q] += s_ex[q];
      agg[q] += s_ex[q];
    }
  }
#pragma unroll
  for (int k = 0; k < ROWS; ++k) {
    const uint64_t i = wbase + 64ull * k + lane;
#pragma unroll
    for (int q = 0; q < NV; ++q) ex[k][q] += before[q];
    if (i < n) f.apply(i, ex[k], v[k]);
  }
  if (tile + 1 == gridDim.x && threadIdx.x == 0) f.total(agg);
}

}  // namespace bt
