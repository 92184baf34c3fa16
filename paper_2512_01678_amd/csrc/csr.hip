// csr.hip -- A + I in CSR form from an edge list, on the device.
//
// Section III-A's GCN operator needs, for every node, the set of its distinct
// neighbours plus itself, in a fixed (ascending) order so that the result is
// canonical and bit-exact against any other correct construction.
//
//  1. partition: both directions of every non-self pair go to the bucket of their row (2^s1
//     rows each), then, bucket by bucket, to the sub-bucket (2^s2 rows, about 6,000 entries):
//     counts in LDS, one scan, and a scatter whose open lines (one per bucket and workgroup)
//     stay in the L2 until they are full.  No atomic leaves a CU.
//  2. rows: one workgroup per sub-bucket counts its rows, adds each row's self entry and puts
//     the columns into their rows in LDS (in memory where they do not fit); a wavefront sorts
//     and deduplicates each row of up to 512 entries in registers (bitonic over lanes) and
//     writes it to the row's raw place.  The order in which entries arrive depends on
//     scheduling; the sort removes that dependence.
//  3. longer rows in place:
//       <= 4096 entries  one workgroup, bitonic sort in LDS;
//       larger           one workgroup, a bitmap of 2^19 columns at a time in LDS, read
//                        back in column order.
//  4. scan the unique counts (the degrees) into row_ptr; dinv = (float)(1 / sqrt((double)deg)).
//  5. compact into col_idx and write the entries of A_hat beside, val[e] = dinv[row] *
//     dinv[col[e]] (fp32).
//  6. (optional) the row order of the aggregations: rows by decreasing length class,
//     longest first, so that the long rows start early and the short ones fill the end
//     of a launch (a longest-job-first schedule; the results do not depend on it).  A
//     stable counting sort over 64 classes of the degree: per-block class counts, one
//     scan in class-major order, then each block places its rows (ties in row order).
//
// Bound: memory.  2,449,029 nodes, 61,859,140 pairs: the pairs, two passes of 8-byte (row,
// column) entries, the raw rows and the result are about 8 GB.  Whole call 22.2 -> 5.85 ms:
// partition 2.4 and rows 1.0 (before: an atomic per entry for the counts and one for the places,
// both to memory, scattered 4-byte writes, 11.6; a rank by comparison per row, 4.1), longer
// rows 0.7 (3.1), compaction with the gather of dinv 1.4 (2.1).  A bucket and a sub-bucket are one
// workgroup's, so ids that gather the entries in few buckets lengthen the call (RMAT 2^21 rows, 33.6 M
// pairs, ids as drawn 12.8 ms, permuted 5.4; with an atomic per entry 33.6 and 19.4; a star of 20 M
// rows 362 and 759).
#include "internal.h"

namespace gcn {
namespace {

constexpr int kSmall = 512;   // longest row that a wavefront sorts in registers
constexpr int kMedium = 4096;
constexpr int kLargeBlocks = 512;
constexpr int kMaxBuckets = 1024;  // buckets of a partition pass (LDS counters)
constexpr int kPartThreads = 1024;
constexpr int kMaxSubRows = 1024;
constexpr int kRowsThreads = 512;
constexpr int kRowsCap = 10240;    // entries of a sub-bucket that are sorted from LDS

// Rows 2^s1 per bucket and 2^s2 per sub-bucket; nw workgroups share the input pairs.
struct Parts {
  int s1, s2;
  int64_t buckets, subs, nw;
};

constexpr Parts make_parts(int32_t n, int64_t n_edges) {
  Parts q{};
  const double avg = n > 0 ? 2.0 * (double)n_edges / n + 1.0 : 1.0;
  q.s2 = 0;
  while (q.s2 < 10 && avg * (double)(int64_t(2) << q.s2) <= 7000.0) ++q.s2;
  // as many buckets as one pass takes (their open lines stay in the L2), so few or no
  // sub-buckets: 598 of 32 each for 2,449,029 rows of 51
  q.s1 = q.s2;
  while (ceil_div(n > 0 ? n : 1, int64_t(1) << q.s1) > kMaxBuckets) ++q.s1;
  if (q.s1 - q.s2 > 10) q.s2 = q.s1 - 10;
  q.buckets = ceil_div(n > 0 ? n : 1, int64_t(1) << q.s1);
  q.subs = q.buckets << (q.s1 - q.s2);
  q.nw = std::max<int64_t>(1, std::min<int64_t>(512, ceil_div(n_edges, 4096)));
  return q;
}
// What the kernels hold in LDS: counters of one bucket's sub-buckets, of one sub-bucket's rows.
constexpr bool parts_fit(int32_t n, int64_t n_edges) {
  const Parts q = make_parts(n, n_edges);
  return q.buckets <= kMaxBuckets && (1 << (q.s1 - q.s2)) <= kMaxBuckets && (1 << q.s2) <= kMaxSubRows;
}
static_assert(parts_fit(kMaxGraphRows, 0) && parts_fit(kMaxGraphRows, (1 << 30) - 1) && parts_fit(1 << 20, (1 << 30) - 1) &&
                  parts_fit((1 << 20) + 1, 0) && parts_fit(1, 0) && parts_fit(0, 0),
              "a bucket or sub-bucket outgrows its counters");

struct Pair {
  int32_t row, col;
};

struct CsrWs {
  Parts parts;
  int32_t* part_cnt;  // buckets * nw
  int64_t* part_off;  // buckets * nw + 1
  int64_t* sub_off;   // subs + 1
  Pair* pa;           // 2 E: entries by bucket
  Pair* pb;           // 2 E: entries by sub-bucket (where buckets are split)
  int32_t* raw;       // 2 E + n columns: the raw rows, in the place of pa (of pb if unsplit)
  int32_t* alt;       // likewise in the other one: the sorted rows of k_sort_large
  int32_t* cnt;       // n: raw entries per row
  int64_t* raw_off;   // n
  int32_t* lists;     // 2 n: medium / large row lists
  int32_t* flags;     // [0] range error, [1..2] list sizes
  void* scan;
  void* split;        // hub split plan scratch
  int32_t* ord_cnt;   // kClasses * blocks of 256 rows: rows per (class, block)
  int64_t* ord_off;   // kClasses * blocks + 1: their exclusive scan
};

constexpr int kClasses = 64;
constexpr int kOrderBlock = 256;
inline int64_t order_blocks(int32_t n) { return ceil_div(n > 0 ? n : 1, kOrderBlock); }

CsrWs carve(Arena& a, int32_t n, int64_t n_edges) {
  CsrWs w;
  w.parts = make_parts(n, n_edges);
  const int64_t pcount = w.parts.buckets * w.parts.nw;
  w.part_cnt = a.take<int32_t>(pcount);
  w.part_off = a.take<int64_t>(pcount + 1);
  w.sub_off = a.take<int64_t>(w.parts.subs + 1);
  const int64_t room = std::max<int64_t>(2 * n_edges, ceil_div(2 * n_edges + n, 2));
  w.pa = a.take<Pair>(room);
  w.pb = a.take<Pair>(room);
  const bool split = w.parts.s1 > w.parts.s2;
  w.raw = reinterpret_cast<int32_t*>(split ? w.pa : w.pb);
  w.alt = reinterpret_cast<int32_t*>(split ? w.pb : w.pa);
  w.cnt = a.take<int32_t>(n);
  w.raw_off = a.take<int64_t>(n);
  w.lists = a.take<int32_t>(2 * (int64_t)n);
  w.flags = a.take<int32_t>(8);
  const int64_t ocount = kClasses * order_blocks(n);
  w.scan = a.take<char>((int64_t)scan_workspace(std::max<int64_t>(std::max<int64_t>((int64_t)n + 1, ocount + 1), pcount + 1)));
  w.split = a.take<char>((int64_t)split_workspace(n));
  w.ord_cnt = a.take<int32_t>(ocount);
  w.ord_off = a.take<int64_t>(ocount + 1);
  return w;
}

// Calls f(u, v) for the pairs of this workgroup's share; out-of-range endpoints set flags[0].
template <class F>
__device__ __forceinline__ void for_pairs(int32_t n, int64_t ne, const int32_t* src, const int32_t* dst,
                                          int32_t* flags, F f) {
  constexpr int U = 4;
  const int64_t per = (ne + gridDim.x - 1) / gridDim.x;
  const int64_t e0 = (int64_t)blockIdx.x * per, e1 = e0 + per < ne ? e0 + per : ne;
  for (int64_t e = e0 + threadIdx.x; e < e1; e += U * kPartThreads) {
    int32_t u[U], v[U];
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int64_t ei = e + (int64_t)i * kPartThreads;
      u[i] = v[i] = 0;  // a self pair: dropped
      if (ei < e1) {
        u[i] = src[ei];
        v[i] = dst[ei];
      }
    }
#pragma unroll
    for (int i = 0; i < U; ++i) {
      if (u[i] < 0 || u[i] >= n || v[i] < 0 || v[i] >= n) {
        if (flags) atomicOr(&flags[0], 1);
        continue;
      }
      if (u[i] != v[i]) f(u[i], v[i]);
    }
  }
}

__global__ void k_init(int32_t* flags) {
  if (threadIdx.x < 8) flags[threadIdx.x] = 0;
}

// Entries per (bucket, workgroup).
__global__ void __launch_bounds__(kPartThreads) k_bucket_count(int32_t n, int64_t ne, const int32_t* src,
                                                               const int32_t* dst, int s1, int32_t nb, int32_t* cnt,
                                                               int32_t* flags) {
  __shared__ int32_t c[kMaxBuckets];
  for (int b = threadIdx.x; b < nb; b += kPartThreads) c[b] = 0;
  __syncthreads();
  for_pairs(n, ne, src, dst, flags, [&](int32_t u, int32_t v) {
    atomicAdd(&c[u >> s1], 1);
    atomicAdd(&c[v >> s1], 1);
  });
  __syncthreads();
  for (int b = threadIdx.x; b < nb; b += kPartThreads) cnt[(int64_t)b * gridDim.x + blockIdx.x] = c[b];
}

// Every entry to its bucket (positions are below 2 E < 2^31).
__global__ void __launch_bounds__(kPartThreads) k_bucket_scatter(int32_t n, int64_t ne, const int32_t* src,
                                                                 const int32_t* dst, int s1, int32_t nb,
                                                                 const int64_t* off, Pair* out) {
  __shared__ int32_t cur[kMaxBuckets];
  for (int b = threadIdx.x; b < nb; b += kPartThreads) cur[b] = (int32_t)off[(int64_t)b * gridDim.x + blockIdx.x];
  __syncthreads();
  for_pairs(n, ne, src, dst, nullptr, [&](int32_t u, int32_t v) {
    out[atomicAdd(&cur[u >> s1], 1)] = Pair{u, v};
    out[atomicAdd(&cur[v >> s1], 1)] = Pair{v, u};
  });
}

// One workgroup per bucket: its entries to their sub-buckets.
__global__ void __launch_bounds__(kPartThreads) k_sub_split(int s1, int s2, int64_t nw, const int64_t* part_off,
                                                            const Pair* in, Pair* out, int64_t* sub_off) {
  constexpr int U = 4;
  __shared__ int32_t cur[kMaxBuckets];
  const int f = 1 << (s1 - s2);  // <= kMaxBuckets
  const int64_t b = blockIdx.x;
  const int32_t lo = (int32_t)part_off[b * nw], hi = (int32_t)part_off[(b + 1) * nw];
  for (int q = threadIdx.x; q < f; q += kPartThreads) cur[q] = 0;
  __syncthreads();
  auto each = [&](auto g) {
    for (int64_t e = lo + (int64_t)threadIdx.x; e < hi; e += U * kPartThreads) {
      Pair p[U];
#pragma unroll
      for (int i = 0; i < U; ++i) p[i] = e + i * kPartThreads < hi ? in[e + i * kPartThreads] : Pair{-1, -1};
#pragma unroll
      for (int i = 0; i < U; ++i)
        if (p[i].row >= 0) g(p[i]);
    }
  };
  auto sub = [&](const Pair& p) { return (p.row >> s2) & (f - 1); };
  each([&](const Pair& p) { atomicAdd(&cur[sub(p)], 1); });
  __syncthreads();
  if (threadIdx.x < 64) {  // exclusive scan over the sub-buckets by one wavefront
    int32_t run = lo;
    for (int q0 = 0; q0 < f; q0 += 64) {
      const int q = q0 + (int)threadIdx.x;
      const int32_t c = q < f ? cur[q] : 0;
      int32_t incl = c;
      for (int o = 1; o < 64; o <<= 1) {
        const int32_t up = __shfl_up(incl, o, 64);
        if ((int)threadIdx.x >= o) incl += up;
      }
      if (q < f) {
        cur[q] = run + incl - c;
        sub_off[b * f + q] = run + incl - c;
      }
      run += __shfl(incl, 63, 64);
    }
    if (threadIdx.x == 0 && b == (int64_t)gridDim.x - 1) sub_off[(b + 1) * f] = hi;
  }
  __syncthreads();
  each([&](const Pair& p) { out[atomicAdd(&cur[sub(p)], 1)] = p; });
}

// Lane exchange with lane ^ J.
template <int J>
__device__ __forceinline__ int32_t xor_lane(int32_t v) {
  if constexpr (J == 1) return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);
  else if constexpr (J == 2) return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);
  else if constexpr (J < 32) return __builtin_amdgcn_ds_swizzle(v, (J << 10) | 0x1f);
  else return __shfl_xor(v, J, 64);
}

// One step of the bitonic network over 64 K values (value r * 64 + lane in register r).
template <int K, int KK, int J>
__device__ __forceinline__ void bitonic_step(int32_t (&x)[K], int lane) {
  if constexpr (J >= 64) {
#pragma unroll
    for (int r = 0; r < K; ++r)
      if (!(r & (J / 64))) {
        const int32_t a = x[r], b = x[r | (J / 64)];
        const bool up = ((r * 64) & KK) == 0;
        x[r] = up ? min(a, b) : max(a, b);
        x[r | (J / 64)] = up ? max(a, b) : min(a, b);
      }
  } else {
#pragma unroll
    for (int r = 0; r < K; ++r) {
      const int32_t o = xor_lane<J>(x[r]);
      const bool up = ((r * 64 + lane) & KK) == 0, low = (lane & J) == 0;
      x[r] = up == low ? min(x[r], o) : max(x[r], o);
    }
  }
  if constexpr (J > 1) bitonic_step<K, KK, J / 2>(x, lane);
}
template <int K, int KK = 2>
__device__ __forceinline__ void bitonic_sort(int32_t (&x)[K], int lane) {
  bitonic_step<K, KK, KK / 2>(x, lane);
  if constexpr (KK < 64 * K) bitonic_sort<K, 2 * KK>(x, lane);
}

// Sort and deduplicate the len <= 64 K columns at `from` into `to`; returns the unique count.
template <int K>
__device__ __forceinline__ int32_t sort_row(const int32_t* from, int32_t* to, int32_t len, int lane) {
  int32_t x[K];
#pragma unroll
  for (int r = 0; r < K; ++r) x[r] = r * 64 + lane < len ? from[r * 64 + lane] : INT32_MAX;
  bitonic_sort<K>(x, lane);
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  int32_t out = 0, before = -1;  // columns are >= 0
#pragma unroll
  for (int r = 0; r < K; ++r) {
    const int32_t up = __shfl_up(x[r], 1, 64);
    const bool keep = x[r] != INT32_MAX && x[r] != (lane == 0 ? before : up);
    const uint64_t bal = __ballot(keep);
    if (keep) to[out + (int32_t)__popcll(bal & below)] = x[r];
    out += (int32_t)__popcll(bal);
    before = __shfl(x[r], 63, 64);
  }
  return out;
}

// One workgroup per sub-bucket of 2^s2 rows.
__global__ void __launch_bounds__(kRowsThreads) k_rows(int32_t n, int s2, const int64_t* sub_off, int64_t stride, const Pair* in,
                                                       int32_t* raw, int64_t* raw_off, int32_t* cnt, int32_t* deg,
                                                       int32_t* lists, int32_t* flags) {
  constexpr int U = 4;
  __shared__ int32_t len[kMaxSubRows];
  __shared__ uint32_t cur[kMaxSubRows];  // up to 2 E + rows, just beyond 2^31 at the most
  __shared__ int32_t buf[kRowsCap];
  const int32_t r0 = (int32_t)((int64_t)blockIdx.x << s2);
  const int32_t rows = n - r0 < (1 << s2) ? n - r0 : 1 << s2;
  const int32_t lo = (int32_t)sub_off[blockIdx.x * stride], hi = (int32_t)sub_off[(blockIdx.x + 1) * stride];
  const int64_t base = (int64_t)lo + r0;  // every row before has its self entry
  const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
  const bool fits = (int64_t)hi - lo + rows <= kRowsCap;
  for (int r = threadIdx.x; r < rows; r += kRowsThreads) len[r] = 1;
  __syncthreads();
  auto each = [&](auto g) {
    for (int64_t e = lo + (int64_t)threadIdx.x; e < hi; e += U * kRowsThreads) {
      Pair p[U];
#pragma unroll
      for (int i = 0; i < U; ++i) p[i] = e + i * kRowsThreads < hi ? in[e + i * kRowsThreads] : Pair{-1, -1};
#pragma unroll
      for (int i = 0; i < U; ++i)
        if (p[i].row >= 0) g(p[i]);
    }
  };
  each([&](const Pair& p) { atomicAdd(&len[p.row - r0], 1); });
  __syncthreads();
  if (wave == 0) {  // exclusive scan of the rows' lengths
    uint32_t run = 0;
    for (int q0 = 0; q0 < rows; q0 += 64) {
      const int q = q0 + lane;
      const uint32_t c = q < rows ? (uint32_t)len[q] : 0u;
      uint32_t incl = c;
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t up = __shfl_up(incl, o, 64);
        if (lane >= o) incl += up;
      }
      if (q < rows) cur[q] = run + incl - c;
      run += __shfl(incl, 63, 64);
    }
  }
  __syncthreads();
  int32_t* const seg = raw + base;
  // each row's self entry first, then its columns as they come; afterwards cur[r] is its end
  for (int r = threadIdx.x; r < rows; r += kRowsThreads) {
    const uint32_t at = cur[r];
    cnt[r0 + r] = len[r];
    raw_off[r0 + r] = base + at;
    if (fits) buf[at] = r0 + r;
    else seg[at] = r0 + r;
    cur[r] = at + 1;
  }
  __syncthreads();
  if (fits) each([&](const Pair& p) { buf[atomicAdd(&cur[p.row - r0], 1u)] = p.col; });
  else each([&](const Pair& p) { seg[atomicAdd(&cur[p.row - r0], 1u)] = p.col; });
  __syncthreads();
  for (int r = wave; r < rows; r += kRowsThreads / 64) {
    const int32_t l = len[r];
    const uint32_t at = cur[r] - (uint32_t)l;
    const int32_t* from = fits ? buf + at : seg + at;
    if (l <= kSmall) {
      const int32_t d = l <= 64    ? sort_row<1>(from, seg + at, l, lane)
                      : l <= 128 ? sort_row<2>(from, seg + at, l, lane)
                      : l <= 256 ? sort_row<4>(from, seg + at, l, lane) : sort_row<8>(from, seg + at, l, lane);
      if (lane == 0) deg[r0 + r] = d;
    } else {
      if (fits)
        for (int32_t i = lane; i < l; i += 64) seg[at + i] = from[i];
      if (lane == 0) {
        const int c = l <= kMedium ? 0 : 1;
        lists[(int64_t)c * n + atomicAdd(&flags[1 + c], 1)] = r0 + r;
      }
    }
  }
}

// one workgroup per row of 513..4096 entries: bitonic sort in LDS, then compact
__global__ void __launch_bounds__(256) k_sort_medium(const int32_t* pcount, const int32_t* list,
                                                     const int64_t* off, const int32_t* cnt,
                                                     int32_t* raw, int32_t* deg) {
  __shared__ int32_t a[kMedium];
  __shared__ int32_t part[256];
  const int tid = threadIdx.x;
  const int32_t count = *pcount;
  for (int64_t item = blockIdx.x; item < count; item += gridDim.x) {
    const int32_t row = list[item];
    const int32_t len = cnt[row];
    int32_t* seg = raw + off[row];
    int P = 256;
    while (P < len) P <<= 1;
    for (int i = tid; i < P; i += 256) a[i] = i < len ? seg[i] : INT32_MAX;
    __syncthreads();
    for (int k = 2; k <= P; k <<= 1) {
      for (int j = k >> 1; j > 0; j >>= 1) {
        for (int i = tid; i < P; i += 256) {
          const int ij = i ^ j;
          if (ij > i) {
            const int32_t x = a[i], y = a[ij];
            const bool up = (i & k) == 0;
            if ((x > y) == up) {
              a[i] = y;
              a[ij] = x;
            }
          }
        }
        __syncthreads();
      }
    }
    // each thread owns P/256 consecutive slots
    const int per = P / 256;
    const int b0 = tid * per;
    int c = 0;
    for (int i = b0; i < b0 + per; ++i)
      if (i < len && (i == 0 || a[i] != a[i - 1])) ++c;
    part[tid] = c;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
      const int add = tid >= o ? part[tid - o] : 0;
      __syncthreads();
      part[tid] += add;
      __syncthreads();
    }
    int pos = part[tid] - c;
    for (int i = b0; i < b0 + per; ++i)
      if (i < len && (i == 0 || a[i] != a[i - 1])) seg[pos++] = a[i];
    if (tid == 255) deg[row] = part[255];
    __syncthreads();
  }
}

// One workgroup per row of > 4096 entries: for each window of kWindow columns, a bitmap of the
// row's columns in LDS, read back in order.  The result goes to `alt` (the row is read once per
// window) and raw_off follows it.
constexpr int kWindow = 1 << 19;
constexpr int kLargeThreads = 512;
__global__ void __launch_bounds__(kLargeThreads) k_sort_large(const int32_t* pcount, const int32_t* list, int32_t n,
                                                              int64_t* raw_off, const int32_t* cnt, const int32_t* raw,
                                                              int32_t* alt, int32_t* deg) {
  constexpr int U = 16, kWords = kWindow / 32, kPer = kWords / kLargeThreads;
  __shared__ uint32_t bm[kWords];
  __shared__ int32_t wsum[kLargeThreads / 64];
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
  const int32_t count = *pcount;
  for (int64_t item = blockIdx.x; item < count; item += gridDim.x) {
    const int32_t row = list[item], len = cnt[row];
    const int64_t off = raw_off[row];
    const int32_t* in = raw + off;
    int32_t* out = alt + off;
    int32_t run = 0;
    for (int64_t w0 = 0; w0 < n; w0 += kWindow) {
      for (int i = tid; i < kWords; i += kLargeThreads) bm[i] = 0;
      __syncthreads();
      for (int64_t j = tid; j < len; j += U * kLargeThreads) {
        int32_t c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = j + u * kLargeThreads < len ? in[j + u * kLargeThreads] : -1;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int64_t x = c[u] - w0;
          if (c[u] >= 0 && x >= 0 && x < kWindow) atomicOr(&bm[x >> 5], 1u << (x & 31));
        }
      }
      __syncthreads();
      // thread t reads words t * kPer ..; a scan over the workgroup gives its place
      int32_t c = 0;
      for (int i = 0; i < kPer; ++i) c += __popc(bm[tid * kPer + i]);
      int32_t incl = c;
      for (int o = 1; o < 64; o <<= 1) {
        const int32_t up = __shfl_up(incl, o, 64);
        if (lane >= o) incl += up;
      }
      if (lane == 63) wsum[wave] = incl;
      __syncthreads();
      int32_t pos = run + incl - c;
      for (int q = 0; q < kLargeThreads / 64; ++q) {
        if (q < wave) pos += wsum[q];
        run += wsum[q];
      }
      for (int i = 0; i < kPer; ++i) {
        uint32_t bits = bm[tid * kPer + i];
        const int64_t first = w0 + (int64_t)(tid * kPer + i) * 32;
        while (bits) {
          out[pos++] = (int32_t)(first + __ffs(bits) - 1);
          bits &= bits - 1;
        }
      }
      __syncthreads();
    }
    if (tid == 0) {
      deg[row] = run;
      raw_off[row] = off + (alt - raw);
    }
    __syncthreads();
  }
}

__global__ void __launch_bounds__(256) k_dinv(int32_t n, const int32_t* deg, float* dinv) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) dinv[i] = (float)(1.0 / sqrt((double)deg[i]));
}

// A group of G lanes per row: its unique columns to their place, the entries of A_hat beside.
template <int G>
__global__ void __launch_bounds__(256) k_compact(int32_t n, const int64_t* raw_off, const int32_t* raw,
                                                 const int64_t* row_ptr, const int32_t* deg, const float* dinv,
                                                 int32_t* col_idx, float* val) {
  const int64_t row = ((int64_t)blockIdx.x * 256 + threadIdx.x) / G;
  const int lane = threadIdx.x % G;
  if (row >= n) return;
  const int32_t d = deg[row];
  const int32_t* s = raw + raw_off[row];
  const int64_t o = row_ptr[row];
  const float di = dinv[row];
  int32_t j = lane;
  for (; j + 3 * G < d; j += 4 * G) {  // a long row: four gathers in flight
    int32_t c[4];
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) c[u] = s[j + u * G];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = dinv[c[u]];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      col_idx[o + j + u * G] = c[u];
      val[o + j + u * G] = di * v[u];
    }
  }
  for (; j < d; j += G) {
    const int32_t c = s[j];
    col_idx[o + j] = c;
    val[o + j] = di * dinv[c];
  }
}

// Length class of a row: 4 classes per power of two of the degree (its two bits below
// the leading one), class 0 for the longest rows (degree >= 2^15.75).
__device__ __forceinline__ int length_class(int32_t d) {
  if (d < 4) return kClasses - 1 - d;
  const int lg = 31 - __clz(d);
  const int key = 4 * lg + ((d >> (lg - 2)) & 3);
  return kClasses - 1 - (key < kClasses - 1 ? key : kClasses - 1);
}

__global__ void __launch_bounds__(kOrderBlock) k_order_count(int32_t n, const int32_t* deg, int32_t* cnt,
                                                             int64_t nblk) {
  __shared__ int32_t h[kClasses];
  if (threadIdx.x < kClasses) h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t row = (int64_t)blockIdx.x * kOrderBlock + threadIdx.x;
  if (row < n) atomicAdd(&h[length_class(deg[row])], 1);  // LDS integer counts
  __syncthreads();
  if (threadIdx.x < kClasses) cnt[(int64_t)threadIdx.x * nblk + blockIdx.x] = h[threadIdx.x];
}

__global__ void __launch_bounds__(kOrderBlock) k_order_place(int32_t n, const int32_t* deg, const int64_t* off,
                                                             int64_t nblk, int32_t* order) {
  __shared__ int32_t cls[kOrderBlock];
  const int64_t row = (int64_t)blockIdx.x * kOrderBlock + threadIdx.x;
  const int c = row < n ? length_class(deg[row]) : -1;
  cls[threadIdx.x] = c;
  __syncthreads();
  if (row >= n) return;
  int rank = 0;  // rows of the same class before this one in the block
  for (int t = 0; t < (int)threadIdx.x; ++t) rank += cls[t] == c ? 1 : 0;
  order[off[(int64_t)c * nblk + blockIdx.x] + rank] = (int32_t)row;
}

}  // namespace

size_t build_csr_workspace(int32_t n, int64_t n_edges) {
  Arena a;
  carve(a, n, n_edges);
  return a.used;
}

gcn_status run_build_csr(int32_t n, int64_t n_edges, const int32_t* src, const int32_t* dst,
                         gcn_graph* g, void* ws, hipStream_t s) {
  Arena a;
  a.base = static_cast<char*>(ws);
  CsrWs w = carve(a, n, n_edges);
  const Parts& q = w.parts;
  hipLaunchKernelGGL(k_init, dim3(1), dim3(64), 0, s, w.flags);
  GCN_TRY(check_launch("csr init"));
  hipLaunchKernelGGL(k_bucket_count, dim3((unsigned)q.nw), dim3(kPartThreads), 0, s, n, n_edges, src, dst, q.s1,
                     (int32_t)q.buckets, w.part_cnt, w.flags);
  GCN_TRY(check_launch("csr bucket count"));
  GCN_TRY(launch_scan_i32(w.part_cnt, q.buckets * q.nw, w.part_off, w.scan, s));
  hipLaunchKernelGGL(k_bucket_scatter, dim3((unsigned)q.nw), dim3(kPartThreads), 0, s, n, n_edges, src, dst, q.s1,
                     (int32_t)q.buckets, w.part_off, w.pa);
  GCN_TRY(check_launch("csr bucket scatter"));
  const bool split = q.s1 > q.s2;
  if (split) {
    hipLaunchKernelGGL(k_sub_split, dim3((unsigned)q.buckets), dim3(kPartThreads), 0, s, q.s1, q.s2, q.nw, w.part_off,
                       w.pa, w.pb, w.sub_off);
    GCN_TRY(check_launch("csr sub-buckets"));
  }
  if (n > 0) {
    hipLaunchKernelGGL(k_rows, dim3((unsigned)ceil_div(n, int64_t(1) << q.s2)), dim3(kRowsThreads), 0, s, n, q.s2,
                       split ? w.sub_off : w.part_off, split ? (int64_t)1 : q.nw, split ? w.pb : w.pa, w.raw, w.raw_off,
                       w.cnt, g->deg, w.lists, w.flags);
    GCN_TRY(check_launch("csr rows"));
    // the lists' sizes stay on the device; a row of more than kSmall raw entries takes as many
    // pairs, which bounds how many there can be
    const int64_t most = std::min<int64_t>(n, 2 * n_edges / kSmall);
    if (most > 0) {
      hipLaunchKernelGGL(k_sort_medium, dim3((unsigned)std::min<int64_t>(most, 8192)), dim3(256), 0, s, w.flags + 1,
                         w.lists, w.raw_off, w.cnt, w.raw, g->deg);
      GCN_TRY(check_launch("csr sort medium"));
    }
    const int64_t most_large = std::min<int64_t>(n, 2 * n_edges / kMedium);
    if (most_large > 0) {
      hipLaunchKernelGGL(k_sort_large, dim3((unsigned)std::min<int64_t>(most_large, kLargeBlocks)),
                         dim3(kLargeThreads), 0, s, w.flags + 2, w.lists + n, n, w.raw_off, w.cnt, w.raw, w.alt, g->deg);
      GCN_TRY(check_launch("csr sort large"));
    }
  }
  GCN_TRY(launch_scan_i32(g->deg, n, g->row_ptr, w.scan, s));
  int64_t nnz = 0;
  int32_t flags[4];
  GCN_HIP(hipMemcpyAsync(flags, w.flags, sizeof flags, hipMemcpyDeviceToHost, s), "csr flags");
  GCN_HIP(hipMemcpyAsync(&nnz, g->row_ptr + n, sizeof nnz, hipMemcpyDeviceToHost, s), "csr nnz");
  GCN_HIP(hipStreamSynchronize(s), "csr sync");
  if (flags[0]) return fail(GCN_E_RANGE, "gcn_build_csr: an edge endpoint is outside [0, n)");
  g->nnz = nnz;
  if (nnz > g->nnz_cap)
    return fail(GCN_E_CAPACITY, "gcn_build_csr: nnz " + std::to_string(nnz) + " exceeds nnz_cap " +
                                    std::to_string(g->nnz_cap));
  if (n > 0) {
    hipLaunchKernelGGL(k_dinv, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, s, n, g->deg, g->dinv);
    GCN_TRY(check_launch("csr dinv"));
    if (nnz < 20 * (int64_t)n)
      hipLaunchKernelGGL(k_compact<16>, dim3((unsigned)ceil_div(n, 16)), dim3(256), 0, s, n, w.raw_off, w.raw, g->row_ptr,
                         g->deg, g->dinv, g->col_idx, g->val);
    else
      hipLaunchKernelGGL(k_compact<64>, dim3((unsigned)ceil_div(n, 4)), dim3(256), 0, s, n, w.raw_off, w.raw, g->row_ptr,
                         g->deg, g->dinv, g->col_idx, g->val);
    GCN_TRY(check_launch("csr compact"));
  }
  if (g->order && n > 0) {
    const int64_t nblk = order_blocks(n);
    hipLaunchKernelGGL(k_order_count, dim3((unsigned)nblk), dim3(kOrderBlock), 0, s, n, g->deg, w.ord_cnt, nblk);
    GCN_TRY(check_launch("csr order count"));
    GCN_TRY(launch_scan_i32(w.ord_cnt, kClasses * nblk, w.ord_off, w.scan, s));
    hipLaunchKernelGGL(k_order_place, dim3((unsigned)nblk), dim3(kOrderBlock), 0, s, n, g->deg, w.ord_off, nblk,
                       g->order);
    GCN_TRY(check_launch("csr order place"));
  }
  g->split.order = nullptr;
  if (g->split.rows) GCN_TRY(build_split(g->row_ptr, n, &g->split, false, w.split, s));
  GCN_HIP(hipStreamSynchronize(s), "csr sync");
  return GCN_OK;
}

}  // namespace gcn
