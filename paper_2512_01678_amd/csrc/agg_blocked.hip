// agg_blocked.hip -- the aggregation with 16-byte rows.
//
// Z[u,:] = sum_{e in row u} val[e] * M[col[e], :]  (+ bias, epilogue), as in aggregate.hip, for
// matrices M below 4 GB: a wavefront sums one row at a time over a panel of 4 LANES columns.
//
// What bounds it: every gather that misses the XCD's 4 MB L2 is served by the fabric behind it
// at about 55-70 G random 128-byte lines/s (7-9 TB/s), and every 1 KB gather instruction takes
// 16 cycles of the CU's address unit (measured busy 83 % of the time where the gathers hit).
// So beside the gathers themselves the kernel issues little: entries are loaded contiguously
// (one index and one value load per 64 entries, two chunks ahead), handed to the lanes by a
// constant-pattern LDS swizzle, and rows are addressed by 32-bit offsets; a panel covers whole
// lines, so that no line is fetched for two panels.
//
// Long rows: a piece of more than kHub entries is cut over the four wavefronts of its
// workgroup; rows beyond GCN_SPLIT_MIN with a split plan (beyond that many per block where sums are
// blocked) are summed chunk by chunk by wavefronts that start ahead of the others in the same launch.  (On graphs of few rows the
// longest one bounds the call: 2,500 entries walked by one lane group took 110 us.)
//
// Dense graphs are blocked by source rows.  Gathered in row order, M is read from behind the L2
// once per entry (4 nnz w bytes).  Where a row has enough entries in each block of M's rows
// (agg_blocked_plan), one launch per block adds the block's share to every row, panel after
// panel, so that a line is fetched into each L2 once and most further gathers of it hit there.
// The entries of a row that fall into a block are a contiguous piece of it, found by binary
// search at the start of the call.  Between the launches a row's partial sum rests in Z; the
// last launch applies the epilogue.  The others leave a row alone that they have no entry of
// (with local ids a row's entries lie in one block or two: 232,965 rows joined to the 490 around
// them, width 256, 6,452 -> 5,197 us).  Every sum has a fixed order: deterministic.
//
// Measured (us, lane groups -> now): 232,965 rows of 484 entries, width 256 13,700 -> 7,390, width
// 41 3,050 -> 1,930; 169,343 rows of 15, width 256 335 -> 306, 128 169 -> 158, 64 108 -> 83; RMAT 2^21
// rows of 31, width 128 4,000 -> 3,610; 2,449,029 rows of 51, width 256 17,900 -> 17,600 (bound by the
// fabric); 100,000 rows of 32, width 128 272 -> 171.  Slower than the lane groups where ids are local,
// whose gathers hit the L2 either way: 232,965 rows joined to the 490 around them, width 256 4,446 ->
// 5,164, to the 16 around them 284 -> 314; 2,000,000 joined to 50 4,373 -> 4,842.
#include "agg_walk.h"

namespace gcn {
namespace {

// Gathers of steps U .. U + N - 1.  FULL: every slice has an entry in each; else step u is this
// slice's only if u < mine (a skipped entry must not be multiplied by zero instead: the row
// could hold an infinity).
template <int LANES, int U, int N, bool FULL>
__device__ __forceinline__ void gather_load(const char* Mc, uint32_t off, uint32_t lane_off, int mine, float4* x) {
  auto load = [&](auto ic) __attribute__((always_inline)) {
    constexpr int I = decltype(ic)::value;
    const uint32_t o = from_lane<LANES, U + I>(off) + lane_off;
    if constexpr (FULL) {
      x[I] = *reinterpret_cast<const float4*>(Mc + o);
    } else {
      x[I] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (U + I < mine) x[I] = *reinterpret_cast<const float4*>(Mc + o);
    }
  };
  [&]<int... I>(std::integer_sequence<int, I...>) { (load(std::integral_constant<int, I>{}), ...); }
  (std::make_integer_sequence<int, N>{});
}

template <int LANES, int U, int N>
__device__ __forceinline__ void gather_add(float w, const float4* x, float4& acc) {
  auto add = [&](auto ic) __attribute__((always_inline)) {
    constexpr int I = decltype(ic)::value;
    Vec<4>::fma(acc, __uint_as_float(from_lane<LANES, U + I>(__float_as_uint(w))), x[I]);
  };
  [&]<int... I>(std::integer_sequence<int, I...>) { (add(std::integral_constant<int, I>{}), ...); }
  (std::make_integer_sequence<int, N>{});
}

// Steps U .. U + 7 of a chunk, half of them at a time where the chunk ends among them (slices of
// 4 lanes have four steps in all); `between` runs after the loads are issued.
template <int LANES, int U, class Between>
__device__ __forceinline__ void gather_eight(const char* Mc, uint32_t off, float w, uint32_t lane_off, const Runs& rn,
                                             float4& acc, Between between) {
  float4 x[8];
  if constexpr (LANES >= 8) {
    if (rn.least >= U + 8) {
      gather_load<LANES, U, 8, true>(Mc, off, lane_off, rn.have, x);
      between();
      gather_add<LANES, U, 8>(w, x, acc);
      return;
    }
    if (rn.run > U + 4) {
      if (rn.least >= U + 4) gather_load<LANES, U, 4, true>(Mc, off, lane_off, rn.have, x);
      else gather_load<LANES, U, 4, false>(Mc, off, lane_off, rn.have, x);
      gather_load<LANES, U + 4, 4, false>(Mc, off, lane_off, rn.have, x + 4);
      between();
      gather_add<LANES, U, 8>(w, x, acc);
      return;
    }
  }
  gather_load<LANES, U, 4, false>(Mc, off, lane_off, rn.have, x);
  between();
  gather_add<LANES, U, 4>(w, x, acc);
}

// Rows of more than `over` entries: `groups` workgroups ahead of the others (in the first of several
// launches) sum one chunk of such a row per wavefront into part (pitch pw); k_finish_long adds a
// row's chunks.  over is GCN_SPLIT_MIN, or GCN_SPLIT_MIN per block: a chunk of such a row spans
// about a block anyway, while its pieces, a workgroup each, would be the length of every launch
// (200,000 rows of 128 and eight hubs of 190,000, width 64, 2,834 us in pieces, 855 so, 932
// with lane groups).
struct LongRows {
  gcn_split sp;
  float* part;
  int64_t pw;
  int32_t groups;
  int64_t over;
};

// A row's partial sum, this lane's `left` columns of it: what lies beyond the width is the caller's.
__device__ __forceinline__ void store_sum(float* z, const float4& v, int left) {
  if (left >= 4) {
    *reinterpret_cast<float4*>(z) = v;
  } else {
    z[0] = v.x;
    if (left > 1) z[1] = v.y;
    if (left > 2) z[2] = v.z;
  }
}

// The finished columns of one row (every slice holds them; slice 0 writes): ReLU with its
// bitmask, or the mask (mk, this lane's columns of it).
template <int LANES, int EPI>
__device__ __forceinline__ void store_row(const AggParams& p, int64_t row, float4 v, const float4& mk, const Lanes& L,
                                          bool cok) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const int c0 = L.c0;
  if constexpr (EPI == AGG_RELU) {
    if (p.relu_bits) {
      // 1[v > 0] of this lane's columns, OR-ed over the eight lanes of a 32-column word
      uint32_t bits = 0;
      if (cok) {
        bits |= v.x > 0.f ? 1u : 0u;
        bits |= c0 + 1 < p.w && v.y > 0.f ? 2u : 0u;
        bits |= c0 + 2 < p.w && v.z > 0.f ? 4u : 0u;
        bits |= c0 + 3 < p.w && v.w > 0.f ? 8u : 0u;
      }
      bits = group_or<(LANES < 8 ? LANES : 8)>(bits << (c0 % 32));
      if (L.slot == 0 && cok && L.lane % 8 == 0) p.relu_bits[row * p.ld_relu_bits + c0 / 32] = bits;
    }
    v = make_float4(fmaxf(v.x, 0.f), fmaxf(v.y, 0.f), fmaxf(v.z, 0.f), fmaxf(v.w, 0.f));
  }
  if constexpr (EPI == AGG_MASK) {
    v.x = mk.x > 0.f ? v.x : 0.f;
    v.y = mk.y > 0.f ? v.y : 0.f;
    v.z = mk.z > 0.f ? v.z : 0.f;
    v.w = mk.w > 0.f ? v.w : 0.f;
  }
  if (!cok || L.slot != 0) return;
  float* out = p.Z + row * p.ldz + c0;
  if (c0 + 4 <= p.w) {
    // written once and not read by this kernel: L2 is left to the gathered rows
    const f32x4 o = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(o, reinterpret_cast<f32x4*>(out));
  } else {
    out[0] = v.x;
    if (c0 + 1 < p.w) out[1] = v.y;
    if (c0 + 2 < p.w) out[2] = v.z;
  }
}

// In a blocked launch a piece's row carries whether earlier blocks left a partial sum of the row
// (rows stay below 2^26: M is below 4 GB and more than 16 columns wide).
constexpr int32_t kGoesOn = 1 << 30;

// Workgroup b's wavefront w sums the pieces of rows 4 b + w, 4 b + w + nwaves, ... (`rounds` of
// them; in processing order when blocked, so that rows of like length run together).
template <int LANES, int EPI, bool BLOCKED>
__global__ void __launch_bounds__(kWalkThreads) k_agg_blocked(AggParams p, const Piece* pieces, int32_t block,
                                                               int32_t nblock, int32_t rounds, LongRows lr) {
  constexpr int SL = 64 / LANES;
  __shared__ __attribute__((aligned(16))) float s_part[2][kWalkWaves][4 * LANES];
  const Lanes L = walk_lanes<LANES>();
  const bool cok = L.c0 < p.w;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const char* Mc = reinterpret_cast<const char*>(p.M);
  const uint32_t lane_off = cok ? 4u * (uint32_t)L.c0 : 0u;  // lanes past the width re-read column 0 (not used)
  const uint32_t pitch = 4u * (uint32_t)p.ldm;
  const bool last = !BLOCKED || block == nblock - 1;

  // Lane 4 r + q holds the piece of round r, wavefront q: every wavefront knows all of them.
  const bool chunks = (int)blockIdx.x < lr.groups;
  const uint32_t groups = gridDim.x - (uint32_t)lr.groups;
  const uint32_t group = chunks ? blockIdx.x : walk_group(blockIdx.x - (uint32_t)lr.groups, groups);
  const uint32_t hi = walk_row(group, groups, L.lig);
  Piece h{0, 0, -1};
  if (chunks) {
    rounds = 1;
    if (L.lig < kWalkWaves && hi < lr.sp.n_chunk) {
      const int64_t ch = lr.sp.order ? lr.sp.order[hi] : hi;
      const int32_t o = lr.sp.owner[ch], row = lr.sp.rows[o];
      h.beg = p.row_ptr[row] + (ch - lr.sp.first[o]) * (int64_t)GCN_SPLIT_CHUNK;
      const int64_t end = p.row_ptr[row + 1], left = end - h.beg;
      if (!BLOCKED || end - p.row_ptr[row] > lr.over) {
        h.len = (int)(left < GCN_SPLIT_CHUNK ? left : GCN_SPLIT_CHUNK);
        h.row = (int)ch;
      }
    }
  } else if (L.lig < kWalkWaves * rounds && hi < (uint32_t)p.n) {
    if (BLOCKED) {
      h = pieces[(int64_t)block * p.n + hi];
    } else {
      const int64_t beg = p.row_ptr[hi], end = p.row_ptr[hi + 1];
      if (lr.groups == 0 || end - beg <= lr.over) h = Piece{beg, (int32_t)(end - beg), (int32_t)hi};
    }
  }
  const Items items = make_items(h, rounds, wave, L.lig, !chunks);

  // Epilogue inputs that need no waiting for at a row's end: the bias of this lane's columns,
  // the mean's factor of the item's row.
  float4 bias = make_float4(0.f, 0.f, 0.f, 0.f);
  if (EPI != AGG_SOFTMAX && last && p.bias && cok) {
    bias.x = p.bias[L.c0];
    if (L.c0 + 1 < p.w) bias.y = p.bias[L.c0 + 1];
    if (L.c0 + 2 < p.w) bias.z = p.bias[L.c0 + 2];
    if (L.c0 + 3 < p.w) bias.w = p.bias[L.c0 + 3];
  }
  const float h_scale = EPI != AGG_SOFTMAX && last && !chunks && items.row >= 0 ? row_scale(p, BLOCKED ? items.row & ~kGoesOn : items.row) : 1.f;

  // The entries are requested two chunks ahead of the gathers: a chunk's indices come from
  // behind the L2, its gathers mostly from it.
  Cursor<LANES> cursor;
  auto fetch = [&](int& j, float& w) __attribute__((always_inline)) {
    j = 0;
    w = 0.f;
    int64_t at;
    if (cursor.next(items, L, &at)) {
      j = p.col[at];
      if (p.kind == AGG_W_VAL) w = p.val[at];
    }
  };
  int j0, j1;
  float w0, w1;
  fetch(j0, w0);
  fetch(j1, w1);
  // The loss epilogue (row maximum, exponentials, three slice reductions, loss and gradient row)
  // costs every slice the same instructions: slice s keeps the sums of one row, and SL rows are
  // finished at once (rows in one panel only; wider ones by k_finish_softmax).
  float4 keep = make_float4(0.f, 0.f, 0.f, 0.f);
  int keep_row = -1, kept = 0;
  auto finish_kept = [&]() {
    finish_row<LANES, 4, EPI, true>(p, keep_row, keep, L, cok, keep_row >= 0);
    keep_row = -1;
    kept = 0;
  };
  int parity = 0;
  for (int t = 0; t < items.n; ++t) {
    const int tagged = __builtin_amdgcn_readlane(items.row, t);
    const int len = __builtin_amdgcn_readlane(items.len, t);
    const int fin = __builtin_amdgcn_readlane(items.kind, t);
    const int row = BLOCKED && tagged >= 0 ? tagged & ~kGoesOn : tagged;
    const bool mine = row >= 0 && (fin < 0 || fin == wave);
    float* z = (chunks ? lr.part + row * lr.pw : p.Z + (int64_t)(row < 0 ? 0 : row) * p.ldz) + L.c0;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float4 part = acc, mk = acc;
    // (the loss epilogue keeps a row's sum in any slice, the others in slice 0)
    if (BLOCKED && (tagged & kGoesOn) && cok && (EPI == AGG_SOFTMAX || L.slot == 0) && mine) part = *reinterpret_cast<const float4*>(z);
    if (EPI == AGG_MASK && last && !chunks && cok && L.slot == 0 && mine)
      mk = *reinterpret_cast<const float4*>(p.mask + (int64_t)row * p.ldmask + L.c0);
    int done = 0;
    do {
      const int cnt = len - done < 64 ? len - done : 64;
      const Runs rn = runs_of<LANES>(cnt, L.slot);
      const uint32_t off = (uint32_t)j0 * pitch;
      float w = w0;
      if (p.kind != AGG_W_VAL)
        w = L.lane < rn.have ? (p.kind == AGG_W_COLMEAN ? 1.f / (float)p.deg[j0] : 1.f) : 0.f;
      j0 = j1;
      w0 = w1;
      auto more = [&]() __attribute__((always_inline)) { fetch(j1, w1); };
      gather_eight<LANES, 0>(Mc, off, w, lane_off, rn, acc, more);
      if constexpr (LANES > 8)
        if (rn.run > 8) gather_eight<LANES, 8>(Mc, off, w, lane_off, rn, acc, [] {});
      if constexpr (LANES > 16) {
        if (rn.run > 16) gather_eight<LANES, 16>(Mc, off, w, lane_off, rn, acc, [] {});
        if (rn.run > 24) gather_eight<LANES, 24>(Mc, off, w, lane_off, rn, acc, [] {});
      }
      done += 64;
    } while (done < len);
    for (int o = LANES; o < 64; o <<= 1) Vec<4>::add_xor(acc, o, 64);
    if (fin >= 0) {
      float* sp = s_part[parity][0] + 4 * L.lane;
      parity ^= 1;
      if (L.slot == 0) *reinterpret_cast<float4*>(sp + wave * 4 * LANES) = acc;
      __syncthreads();  // every wavefront has the same shared items
      if (!mine) continue;
      acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int q = 0; q < kWalkWaves; ++q) Vec<4>::add(acc, *reinterpret_cast<const float4*>(sp + q * 4 * LANES));
    }
    if (!mine) continue;
    Vec<4>::add(acc, part);
    if (!last || chunks || (EPI == AGG_SOFTMAX && gridDim.y > 1)) {
      if (cok && L.slot == 0) store_sum(z, acc, chunks ? 4 : p.w - L.c0);
      continue;
    }
    if constexpr (EPI == AGG_SOFTMAX) {
      if (L.slot == kept) {
        keep = acc;
        keep_row = row;
      }
      if (++kept == SL) finish_kept();
      continue;
    }
    const float sc = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(h_scale), t));
    float4 v = make_float4(sc * acc.x + bias.x, sc * acc.y + bias.y, sc * acc.z + bias.z, sc * acc.w + bias.w);
    store_row<LANES, EPI>(p, row, v, mk, L, cok);
  }
  if constexpr (EPI == AGG_SOFTMAX)
    if (kept > 0) finish_kept();
}

// One slice per long row: its chunk sums in chunk order, then the epilogue.
template <int LANES, int EPI>
__global__ void __launch_bounds__(kWalkThreads) k_finish_long(AggParams p, LongRows lr) {
  Lanes L;
  L.gw = LANES;
  L.lig = threadIdx.x & (LANES - 1);
  L.slot = 0;
  L.lane = L.lig;
  L.c0 = ((int)blockIdx.y * LANES + L.lane) * 4;
  const int64_t o = ((int64_t)blockIdx.x * kWalkThreads + threadIdx.x) / LANES;
  if (o >= lr.sp.n_long) return;
  const int64_t row = lr.sp.rows[o];
  if (p.row_ptr[row + 1] - p.row_ptr[row] <= lr.over) return;  // summed piece by piece
  const bool cok = L.c0 < p.w;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  if (cok)
    for (int64_t ch = lr.sp.first[o]; ch < lr.sp.first[o + 1]; ++ch)
      Vec<4>::add(acc, *reinterpret_cast<const float4*>(lr.part + ch * lr.pw + L.c0));
  if (EPI == AGG_SOFTMAX && gridDim.y > 1) {
    if (cok) store_sum(p.Z + row * p.ldz + L.c0, acc, p.w - L.c0);
  } else {
    finish_row<LANES, 4, EPI>(p, row, acc, L, cok);
  }
}

// pieces[b * n + i]: the entries of the i-th row in processing order whose source rows lie in
// block b.  A group of G lanes per row, a lane per block: each finds the end of its block by binary
// search, and the running maximum over the lanes makes the pieces make up the row whatever the
// order of its columns; ascending ones (gcn_build_csr) make each block's gathers stay in it.
// (Bound by the latency of the searches: one thread per row, block after block, took 202 us for
// 232,965 permuted rows of 490 and ten blocks, 134 now, 70 where ids are local.)
template <int G>
__global__ void __launch_bounds__(256) k_block_pieces(int32_t n, const int64_t* row_ptr, const int32_t* col,
                                                      const int32_t* order, int32_t rows, int32_t nblock,
                                                      int64_t over, Piece* pieces) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / G;
  const int lane = threadIdx.x % G;
  if (i >= n) return;  // whole groups leave together
  const int32_t row = order ? order[i] : (int32_t)i;
  const int64_t beg = row_ptr[row];
  const int32_t len = (int32_t)(row_ptr[row + 1] - beg);
  const int32_t* const c = col + beg;
  int32_t from = 0;  // where the blocks of this turn start
  for (int32_t b0 = 0; b0 < nblock; b0 += G) {
    const int32_t b = b0 + lane;
    int32_t at = len;
    if (b + 1 < nblock) {
      const int64_t bound = (int64_t)(b + 1) * rows;
      int32_t lo = from;
      while (lo < at) {
        const int32_t mid = lo + (at - lo) / 2;
        if (c[mid] < bound) lo = mid + 1;
        else at = mid;
      }
    }
    for (int o = 1; o < G; o <<= 1) {
      const int32_t before = __shfl_up(at, o, G);
      if (lane >= o && before > at) at = before;
    }
    int32_t start = __shfl_up(at, 1, G);
    if (lane == 0) start = from;
    if (b < nblock) {
      // no entry here: nothing to do before the end; a long row: its chunks are summed elsewhere
      const bool idle = (at == start && b + 1 < nblock) || len > over;
      pieces[(int64_t)b * n + i] = Piece{beg + start, idle ? 0 : at - start, idle ? -1 : row | (start > 0 ? kGoesOn : 0)};
    }
    from = __shfl(at, G - 1, G);
  }
}

// The loss epilogue over the finished sums in Z (a whole row per slice), where a row takes
// several panels.
template <int LANES>
__global__ void __launch_bounds__(kWalkThreads) k_finish_softmax(AggParams p) {
  Lanes L;
  L.gw = LANES;
  L.lig = threadIdx.x & (LANES - 1);
  L.slot = 0;
  L.lane = L.lig;
  L.c0 = 4 * L.lane;
  const int64_t row = ((int64_t)blockIdx.x * kWalkThreads + threadIdx.x) / LANES;
  if (row >= p.n) return;
  const bool cok = L.c0 < p.w;
  const float4 acc = cok ? *reinterpret_cast<const float4*>(p.Z + row * p.ldz + L.c0) : make_float4(0.f, 0.f, 0.f, 0.f);
  finish_row<LANES, 4, AGG_SOFTMAX>(p, row, acc, L, cok);
}

template <int LANES, int EPI>
gcn_status run_blocks(const AggParams& p, const BlockedPlan& b, const Piece* pieces, const LongRows& lr, hipStream_t s) {
  const int64_t panels = ceil_div(p.w, 4 * LANES);
  // rows per wavefront: more hide the start of each (offsets, first entries), fewer fill the
  // chip on small graphs and keep its end short (2 against 1 and 4: within 2 % on large ones)
  const int most = b.nblock > 1 || EPI == AGG_SOFTMAX ? kMaxRounds : 2;
  const int rounds = (int)std::max<int64_t>(1, std::min<int64_t>(most, (int64_t)p.n * panels / 32768));
  for (int32_t c = 0; c < b.nblock; ++c) {
    LongRows mine = lr;
    if (c > 0) mine.groups = 0;
    const dim3 grid((unsigned)(mine.groups + ceil_div(p.n, (int64_t)rounds * kWalkWaves)), (unsigned)panels);
    if (b.nblock == 1)
      hipLaunchKernelGGL((k_agg_blocked<LANES, EPI, false>), grid, dim3(kWalkThreads), 0, s, p, pieces, c, 1, rounds, mine);
    else if (c == b.nblock - 1)
      hipLaunchKernelGGL((k_agg_blocked<LANES, EPI, true>), grid, dim3(kWalkThreads), 0, s, p, pieces, c, b.nblock, rounds, mine);
    else
      hipLaunchKernelGGL((k_agg_blocked<LANES, AGG_NONE, true>), grid, dim3(kWalkThreads), 0, s, p, pieces, c, b.nblock, rounds, mine);
    GCN_TRY(check_launch("blocked aggregation"));
  }
  if (lr.groups > 0) {
    hipLaunchKernelGGL((k_finish_long<LANES, EPI>), dim3((unsigned)ceil_div((int64_t)lr.sp.n_long * LANES, kWalkThreads), (unsigned)panels),
                       dim3(kWalkThreads), 0, s, p, lr);
    GCN_TRY(check_launch("long rows"));
  }
  return GCN_OK;
}

template <int LANES>
gcn_status run_lanes(const AggParams& p, const BlockedPlan& b, const Piece* pieces, const LongRows& lr, hipStream_t s) {
  switch (p.epi) {
    case AGG_NONE: return run_blocks<LANES, AGG_NONE>(p, b, pieces, lr, s);
    case AGG_RELU: return run_blocks<LANES, AGG_RELU>(p, b, pieces, lr, s);
    case AGG_MASK: return run_blocks<LANES, AGG_MASK>(p, b, pieces, lr, s);
    default: break;
  }
  GCN_TRY((run_blocks<LANES, AGG_SOFTMAX>(p, b, pieces, lr, s)));
  const int64_t need = ceil_div(p.w, 4);
  if (need <= LANES) return GCN_OK;
  auto finish = [&](auto ln) {
    constexpr int LN = decltype(ln)::value;
    hipLaunchKernelGGL(k_finish_softmax<LN>, dim3((unsigned)ceil_div((int64_t)p.n * LN, kWalkThreads)),
                       dim3(kWalkThreads), 0, s, p);
    return check_launch("softmax epilogue");
  };
  if (need <= 32) return finish(std::integral_constant<int, 32>{});
  return finish(std::integral_constant<int, 64>{});
}

}  // namespace

// Panel and block of an aggregation of n rows with nnz entries from src_rows rows of M (pitch
// ldm), w columns.  All lines measured with Chung-Lu and uniform graphs of 2,000 to 2,300,000 rows
// and 3 to 490 entries per row, and with matrices of uniform rows; times in us, the lane groups of
// aggregate.hip first.
//
// Many rows of few entries leave most of a wavefront idle, and narrow ones gather little: they
// stay with the lane groups, several rows to a wavefront.  Up to 8 columns, where those share long
// rows, below 32 entries per row (8 columns, uniform and Chung-Lu, 100,000 rows of 6: 10 and 14
// against 27 and 29; 200,000 of 24: 46 and 61 against 56 and 64; of 48: 88 and 128 against 85 and 92);
// on up to 32,768 rows the longest one decides (20,000 of 6, width 4, Chung-Lu: 14 against 10); of a
// matrix, whose M is in the L2, below 64 (1,048,576 of 41 from 4,096: 330 against 353).  Up
// to 16 columns a group walks a long row by itself (100,000 rows of 3: 11 and 26 against 28 and 28;
// of 6: 12 and 40 against 28 and 30; 400,000 of 12: 92 and 117 against 106 and 109); the rows of a
// matrix are more alike than a graph's (100,000 of 12: 19 against 26; of 40: 46 against 32).  Up to
// 32 columns 328,000 rows of 7: 85 against 106, of 10: 135 against 111; up to 64 columns of 3: 68
// against 98, of 5: 125 against 104.  Rows of many 64-byte gathers from beyond the L2s gain from the
// row order, which only the lane groups take (width 16, 150,000 rows of 400: 531 against 563; 284,480
// of 306: 1,005 against 1,060; 400,000 of 200: 1,031 against 1,072, of 127: 686 against 680; 80,000
// of 480: 297 against 302).  Built without an order they lose as much; the choice does not depend
// on it, since results are the same with it and without.
//
// Panel: one slice per row where the row fits (4 lanes up to 16 columns, 8 up to 32, 16 up to 64,
// 32 above); wider rows that start at line boundaries take 64-column panels of two lines
// instead (width 256, 169,343 rows of 15: 306 against 340 with 32 lanes; RMAT 2^21 rows of 31
// 7,170 against 7,718), since half of the panel fits the L2 twice, unless a row has too few
// entries to pay for a second walk (1,000,000 rows of 3, width 128: 715; width 100 in one panel
// 405; lane groups 476 and 461).  (Where the gathers hit the L2, as with local ids, one panel would
// be the better: 233,000 rows joined to the 16 around them, width 256, 312 against 214.)  Where rows
// are not line-aligned a narrower panel would fetch its edge lines twice (width 100, 2,449,029 rows:
// 8,790 in one panel, 12,900 in two).  32-column panels pay where rows are gathered often and M is
// between the L2's size and a few times that (100,000 rows of 64: 564 against 671; 50,000 of 60,
// width 128: 120 against 140; of 8: 106 against 63).
//
// Blocks: 6 MB panels of M (R1) where a row has 24 entries per block, else 12 MB ones (R2) where
// it has 24 (100,000 rows of 128 entries, width 256: 957 with R1, 1,047 unblocked; 200,000 of
// 128: 2,429 with R2, 2,713 unblocked; of 64: 1,594 against 1,416).  With 32 lanes the entries
// are twice the bytes and from 131,072 rows on 12 suffice for R2 (200,000 of 128, width 100: 1,205
// against 1,612; but 50,000 of 60: 222 against 161).  Each launch costs its start and its end, so few
// entries in all don't pay: below 8 M with 16 lanes (Chung-Lu, width 64, 30,000 rows of 60: 81 against
// 39; of 236: 112 against 117; 60,000 of 119: 163 against 163; 45,000 of 236: 149 against 215; uniform
// 30,000 of 240: 117 against 132), below 3.5 M with 32 (width 100 and 200, Chung-Lu, 20,000 of 118: 106
// against 82 and 173 against 186; of 235: 126 against 150 and 253 against 371; 45,000 of 60: 182 against
// 143 and 303 against 300).  Rows of one line (8 lanes) gain from larger blocks alone, and from 2^17 rows
// on (200,000 of 128, width 24: 406 against 464; 100,000 of 128: 203 against 176).
BlockedPlan agg_blocked_plan(int64_t n, int64_t src_rows, int64_t nnz, int32_t w, int64_t ldm, RowKind kind,
                             bool may_block) {
  BlockedPlan b{};
  if (w <= 0 || n <= 0 || nnz < 0 || src_rows <= 0 || 4 * src_rows * ldm > (int64_t)UINT32_MAX) return b;
  const double avg = (double)nnz / (double)n;
  const bool matrix = kind == ROWS_MATRIX;
  if (matrix && nnz > INT32_MAX) return b;  // a row may repeat columns and be longer than a piece counts
  if (w <= 8) {
    if (n > 32768 && avg < (matrix ? 64 : 32)) return b;
  } else if (w <= 16) {
    if ((n > 65536 && avg < 5) || (n > 131072 && avg < 12) || (n > 400000 && avg < 16)) return b;
    if (matrix && n > 32768 && avg < 16) return b;
    if (kind == ROWS_GRAPH && n > 131072 && avg >= 160) return b;
  } else if (n > 65536 && (w <= 32 ? avg < 8 : w <= 64 && avg < 4)) {
    return b;
  }
  if (w <= 16) {
    b.lanes = 4;
    b.nblock = 1;
    return b;
  }
  const bool lines = ldm % 32 == 0;
  const bool halves = lines && ((n <= 400000 && avg >= 12) || avg >= 24);  // 64 of more than 64 columns
  b.lanes = w <= 32 ? 8 : (w <= 64 || halves ? 16 : 32);
  b.nblock = 1;
  auto entries = [&](int64_t rows) { return (double)nnz / ((double)n * (double)ceil_div(src_rows, rows)); };
  if (may_block && src_rows <= INT32_MAX) {
    const int64_t r1 = 24576 * 16 / b.lanes, r2 = 2 * r1;
    int64_t rows = 0;
    if (b.lanes == 8) {
      if (src_rows >= (1 << 17) && entries(r1) >= 24) rows = r1;
    } else if (nnz >= (b.lanes == 16 ? 8000000 : 3500000)) {
      if (entries(r1) >= 24) rows = r1;
      else if (entries(r2) >= (b.lanes == 32 && src_rows >= 131072 ? 12 : 24)) rows = r2;
    }
    if (rows > 0 && src_rows > rows) {
      b.rows = (int32_t)rows;
      b.nblock = (int32_t)ceil_div(src_rows, rows);
      return b;
    }
  }
  // Two panels of rows that share lines, unblocked: the lane groups with the row order (width 200,
  // 169,343 rows of 15: 330 against 366; 400,000 of 200: 9,865 against 11,204; RMAT 2^19 rows of 33,
  // width 246: 1,877 against 2,198; but 100,000 of 15, width 200: 204 against 203, 200,000 of 6: 212
  // against 189).
  if (kind == ROWS_GRAPH && w > 128 && !lines && (n > 400000 || (n > 131072 && avg >= 12))) return BlockedPlan{};
  // M in the L2s as it is (the weight of a sparse first layer): fewer passes over the entries (1,048,576
  // rows of 41 from 4,096, width 256: 1,891 against 2,241 in two panels, lane groups 2,065; 20,000 of 18
  // from 1,433: 19 against 25 and 23)
  if (w > 64 && n >= (matrix ? 8192 : 32768) && 4 * src_rows * ldm <= (matrix ? 8 << 20 : 3 << 20)) b.lanes = 32;
  if (lines && w > 64 && avg >= 32 && src_rows >= 32768 && src_rows <= 400000) b.lanes = 8;
  return b;
}

// The row pieces of a blocked aggregation; the chunk sums of long rows come after them.
size_t agg_blocked_workspace(const BlockedPlan& b, int64_t n) {
  return b.nblock > 1 ? sizeof(Piece) * (size_t)n * (size_t)b.nblock : 0;
}

gcn_status launch_agg_blocked(const AggParams& p, const BlockedPlan& b, const gcn_split* split, void* ws, hipStream_t s) {
  Piece* pieces = nullptr;
  LongRows lr{};
  lr.over = INT64_MAX;
  if (has_split(split)) {
    lr.sp = *split;
    lr.part = reinterpret_cast<float*>(static_cast<char*>(ws) + agg_blocked_workspace(b, p.n));
    lr.pw = round_up(p.w, 4);
    lr.groups = (int32_t)ceil_div(split->n_chunk, kWalkWaves);
    lr.over = (int64_t)GCN_SPLIT_MIN * b.nblock;
  }
  if (b.nblock > 1) {
    pieces = static_cast<Piece*>(ws);
    auto find = [&](auto lanes) {
      constexpr int G = decltype(lanes)::value;
      hipLaunchKernelGGL(k_block_pieces<G>, dim3((unsigned)ceil_div((int64_t)p.n * G, 256)), dim3(256), 0, s, p.n,
                         p.row_ptr, p.col, p.order, b.rows, b.nblock, lr.over, pieces);
    };
    if (b.nblock <= 4) find(std::integral_constant<int, 4>{});
    else if (b.nblock <= 8) find(std::integral_constant<int, 8>{});
    else find(std::integral_constant<int, 16>{});
    GCN_TRY(check_launch("row pieces"));
  }
  switch (b.lanes) {
    case 4: return run_lanes<4>(p, b, pieces, lr, s);
    case 8: return run_lanes<8>(p, b, pieces, lr, s);
    case 16: return run_lanes<16>(p, b, pieces, lr, s);
    default: return run_lanes<32>(p, b, pieces, lr, s);
  }
}

}  // namespace gcn
