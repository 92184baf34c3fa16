// agg_walk.h -- how a workgroup of four wavefronts walks the rows of a compressed matrix, one
// row per wavefront and turn (included by the aggregations over 16-byte rows).
//
// A wavefront holds SL = 64 / LANES slices of LANES lanes and takes one row's piece at a time,
// in chunks of up to 64 entries cut into SL runs; lane i of a slice requests the i-th entry of
// its run, so that step u takes the entry of lane u of each slice.  A piece of more than kHub
// entries is shared: each of the four wavefronts takes a quarter, and the quarters meet in LDS.
// Which pieces are shared depends on the piece alone, so results do not depend on which rows
// share a workgroup.
#pragma once

#include "agg_device.h"

namespace gcn {
namespace {

constexpr int kWalkThreads = 256;
constexpr int kWalkWaves = kWalkThreads / 64;
constexpr int kMaxRounds = 64 / kWalkWaves / kWalkWaves;  // one lane per item at most
constexpr int kHub = 512;  // eight chunks: about 10 us for one wavefront

// Entries of one row (row < 0: none).
struct __attribute__((aligned(16))) Piece {
  int64_t beg;
  int32_t len, row;
};

// Value of lane U of each slice: one LDS-crossbar swizzle with a constant pattern, no index
// arithmetic per gather.
template <int LANES, int U>
__device__ __forceinline__ uint32_t from_lane(uint32_t v) {
  constexpr int pattern = (U << 5) | (0x1f & ~(LANES - 1));  // and-mask keeps the slice, or-mask names lane U
  return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, pattern);
}

template <int LANES>
__device__ __forceinline__ Lanes walk_lanes() {
  Lanes L;
  L.gw = 64;
  L.lig = threadIdx.x & 63;
  L.slot = L.lig / LANES;
  L.lane = L.lig & (LANES - 1);
  L.c0 = ((int)blockIdx.y * LANES + L.lane) * 4;
  return L;
}

// The rows of a workgroup: workgroup ids are dealt to the eight XCDs in turn, and where row lengths
// go with the low bits of the row (RMAT ids as they are drawn: 44 % of all entries lie in every
// eighth group of four rows) one XCD would get most of the work.  So each eight consecutive
// workgroups take their places turned by a hash of which eight they are.  (2^20 rows of 31, RMAT
// ids not permuted: width 40 2,494 -> 1,106 us, 256 6,294 -> 4,919, max aggregation of width 256
// 14,431 -> 6,612, its gradient 27,894 -> 9,880; 4,096 rows of 33, width 256 31 -> 23.  Permuted ids
// lose up to 0.3 us a launch, which the smallest graphs would feel: 2,708 rows, an epoch of 65 us 0.9.)
__device__ __forceinline__ uint32_t walk_group(uint32_t b, uint32_t groups) {
  const uint32_t eight = b >> 3;
  if (groups < 1024 || 8 * eight + 8 > groups) return b;
  return (b & ~7u) | ((b + ((eight * 0x9E3779B1u) >> 29)) & 7u);
}
// The row of lane 4 r + q: round r, wavefront q of workgroup `group` of `groups`.
__device__ __forceinline__ uint32_t walk_row(uint32_t group, uint32_t groups, int lig) {
  return group * kWalkWaves + (uint32_t)lig % kWalkWaves + (uint32_t)lig / kWalkWaves * groups * kWalkWaves;
}

// What a wavefront does, item t in lane t: its own piece of a round, or its quarter of a shared
// one (kind: the wavefront that finishes it, or -1).  Every wavefront has the shared items in
// the same order, with one barrier each.
struct Items {
  int n;
  int row, len, kind;
  int64_t beg;
};

// h: lane 4 r + q holds the piece of round r, wavefront q.
__device__ __forceinline__ Items make_items(const Piece& h, int rounds, int wave, int lig, bool share) {
  Items it;
  const uint64_t hubs = share ? __ballot(h.len > kHub) : 0;
  int src = kWalkWaves * lig + wave;
  it.n = rounds;
  it.kind = -1;
  if (hubs) {
    it.n = 0;
    src = 0;
    for (int r = 0; r < rounds; ++r) {
      const uint32_t shared = (uint32_t)(hubs >> (kWalkWaves * r)) & ((1u << kWalkWaves) - 1);
      for (int q = 0; q < kWalkWaves; ++q) {
        if (!((shared >> q) & 1) && q != wave) continue;
        if (lig == it.n) {
          src = kWalkWaves * r + q;
          it.kind = (shared >> q) & 1 ? q : -1;
        }
        ++it.n;
      }
    }
  }
  it.row = __shfl(h.row, src, 64);
  it.len = __shfl(h.len, src, 64);
  it.beg = __shfl(h.beg, src, 64);
  if (it.kind >= 0) {
    const int part = (it.len + kWalkWaves - 1) / kWalkWaves;
    const int lo = part * wave < it.len ? part * wave : it.len;
    it.beg += lo;
    it.len = it.len - lo < part ? it.len - lo : part;
  }
  return it;
}

// The chunks of all items, one after the other; every item has at least one (empty) chunk.
template <int LANES>
struct Cursor {
  int item = 0, done = 0;
  // Whether this lane has an entry in the next chunk, and which.
  __device__ __forceinline__ bool next(const Items& it, const Lanes& L, int64_t* at) {
    constexpr int SL = 64 / LANES;
    if (item >= it.n) return false;
    const int len = __builtin_amdgcn_readlane(it.len, item);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)it.beg, item);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)it.beg >> 32), item);
    const int64_t base = (int64_t)(((uint64_t)hi << 32) | lo) + done;
    const int cnt = len - done < 64 ? len - done : 64;
    const int run = (cnt + SL - 1) / SL;
    const int e = L.slot * run + L.lane;
    *at = base + e;
    done += 64;
    if (done >= len) {
      ++item;
      done = 0;
    }
    return L.lane < run && e < cnt;
  }
};

// Entries of this slice in a chunk of cnt: have; run in the fullest slice, least in the emptiest.
struct Runs {
  int run, have, least;
};
template <int LANES>
__device__ __forceinline__ Runs runs_of(int cnt, int slot) {
  constexpr int SL = 64 / LANES;
  Runs r;
  r.run = (cnt + SL - 1) / SL;
  const int left = cnt - slot * r.run, tail = cnt - (SL - 1) * r.run;
  r.have = left < r.run ? left : r.run;
  r.least = tail < 0 ? 0 : tail;
  return r;
}

}  // namespace
}  // namespace gcn
