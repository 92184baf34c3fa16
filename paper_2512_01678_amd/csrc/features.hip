// features.hip -- density probe and compressed views of the input features.
//
// Section IV-B / Algorithm 1 (Initialize): s = 1 - nnz(X)/(N F) is measured
// once at load time; the sparse path is taken iff s >= tau, and then X is
// converted to CSR (forward) and CSC (backward).  Everything here is integer
// work (counts, offsets, index lists) plus bit-exact copies of the values, so
// the results are identical to any other correct construction.
//
// Every call reads X once to count (16-byte loads, a wavefront per row, or several narrow rows to
// one), leaving one bit per element in the workspace when the views are wanted (a program that
// counts first, to size the views, has X read by both calls):
//  * DenseToCSR: a lane takes 32 columns' bits, a scan over the row's lanes gives its place, and
//    only the nonzeros are read again; from one nonzero in 20 on, the row is read again whole
//    and each nonzero placed by the popcount of the wavefront's ballot below its lane (columns
//    stay ascending either way);
//  * DenseToCSC from the CSR view, a counting sort by column that keeps the rows in order: rows
//    are cut into chunks; per (chunk, column) counts in LDS, a per-column scan over chunks,
//    then one wavefront per chunk walks its rows in order and takes each entry's place from a
//    running count per column in LDS (the columns of a row are distinct, and a wavefront's LDS
//    operations complete in order, so the rows of a column stay ascending).
// Bound: the reads of X.  1,048,576 x 1,024 at 1 % (4.3 GB): the count takes 800 us (5.4 TB/s;
// 1,210 with 4-byte loads and one short-lived wavefront per row), CSR 270 us (1,310 with a
// second walk over X), CSC 630 us (4,710 with two more walks).
#include "internal.h"
#include "lanes.h"

namespace gcn {
namespace {

constexpr int kColBlock = 4096;  // columns that a counting workgroup holds in LDS (16 KB)

// Rows of a CSC chunk: 64 at least, and no more chunks than keep the (chunk, column) counts at
// about 32 MB (2,048 chunks of 4,096 columns).
int64_t chunk_rows(int32_t n, int32_t f) {
  const int64_t most = std::max<int64_t>(64, (int64_t)(8 << 20) / std::max(f, 1));
  return round_up(std::max<int64_t>(64, ceil_div(n, most)), 64);
}

struct FeatWs {
  int32_t* row_cnt;    // n
  int64_t* row_off;    // n + 1 (used when the caller supplies no CSR buffer)
  void* scan;
  int32_t* chunk_cnt;  // nchunks * f
  int32_t* chunk_off;  // nchunks * f
  int32_t* col_tot;    // f
  int64_t nchunks;
  void* split;         // split plan scratch for long CSC columns
  uint32_t* bits;      // n * words: 1[x != 0], 32 columns per word (last: a workspace may end before it)
  int64_t words;
};

FeatWs carve(Arena& a, int32_t n, int32_t f, bool bits, bool csc) {
  FeatWs w;
  w.row_cnt = a.take<int32_t>(n);
  w.row_off = a.take<int64_t>((int64_t)n + 1);
  w.scan = a.take<char>((int64_t)scan_workspace(std::max<int64_t>(n, f) + 1));
  w.nchunks = ceil_div(n, chunk_rows(n, f));
  w.chunk_cnt = a.take<int32_t>(csc ? w.nchunks * f : 0);
  w.chunk_off = a.take<int32_t>(csc ? w.nchunks * f : 0);
  w.col_tot = a.take<int32_t>(csc ? f : 0);
  w.split = a.take<char>(csc ? (int64_t)split_workspace(f) : 0);
  w.words = ceil_div(f, 32);
  w.bits = bits ? a.take<uint32_t>(n * w.words) : nullptr;
  return w;
}

// Nonzeros of each row (and its bits), a wavefront per row.  VEC: 16-byte rows.
template <bool VEC>
__global__ void __launch_bounds__(256) k_row_counts(const float* X, int32_t n, int32_t f, int64_t ldx,
                                                    int32_t* cnt, int64_t* cnt64, uint32_t* bits, int64_t words) {
  const int lane = threadIdx.x % 64;
  const int64_t nwaves = (int64_t)gridDim.x * 4;
  for (int64_t row = (int64_t)blockIdx.x * 4 + threadIdx.x / 64; row < n; row += nwaves) {
    const float* x = X + row * ldx;
    int c = 0;
    if constexpr (VEC) {
      for (int j0 = 0; j0 < f; j0 += 1024) {
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int j = j0 + 256 * u + 4 * lane;
          v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
          if (j < f) v[u] = *reinterpret_cast<const float4*>(x + j);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int j = j0 + 256 * u + 4 * lane;
          uint32_t m = (v[u].x != 0.f ? 1u : 0u) | (v[u].y != 0.f ? 2u : 0u) | (v[u].z != 0.f ? 4u : 0u) |
                       (v[u].w != 0.f ? 8u : 0u);
          if (j + 4 > f) m &= j < f ? (1u << (f - j)) - 1u : 0u;  // columns past f are padding
          c += __popc(m);
          if (bits) {
            const uint32_t word = group_or<8>(m << (4 * (lane % 8)));
            if (lane % 8 == 0 && j < f) bits[row * words + j / 32] = word;
          }
        }
      }
    } else {
      for (int j0 = 0; j0 < f; j0 += 512) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int j = j0 + 64 * u + lane;
          v[u] = j < f ? x[j] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          c += v[u] != 0.f ? 1 : 0;
          if (bits) {
            const uint64_t bal = __ballot(v[u] != 0.f);
            const int j = j0 + 64 * u + 32 * lane;  // lanes 0 and 1 store a half each
            if (lane < 2 && j < f) bits[row * words + j / 32] = (uint32_t)(bal >> (32 * lane));
          }
        }
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
    if (lane == 0) {
      cnt[row] = c;
      if (cnt64) cnt64[row] = c;
    }
  }
}

// The same for 16-byte rows of at most 4 G columns: G lanes per row, four rows in flight each.  (A
// wavefront per row leaves most lanes idle: 1,048,576 x 64, whole count call, 215 -> 90 us;
// 4,000,000 x 16 683 -> 140.)
template <int G>
__global__ void __launch_bounds__(256) k_row_counts_narrow(const float* X, int32_t n, int32_t f, int64_t ldx,
                                                           int32_t* cnt, int64_t* cnt64, uint32_t* bits, int64_t words) {
  constexpr int U = 4;
  const int lane = threadIdx.x % G, j = 4 * lane;
  const int64_t groups = (int64_t)gridDim.x * (256 / G);
  for (int64_t r0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) / G; r0 < n; r0 += U * groups) {
    float4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t row = r0 + u * groups;
      v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (row < n && j < f) v[u] = *reinterpret_cast<const float4*>(X + row * ldx + j);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t row = r0 + u * groups;
      if (row >= n) break;  // whole groups
      uint32_t m = (v[u].x != 0.f ? 1u : 0u) | (v[u].y != 0.f ? 2u : 0u) | (v[u].z != 0.f ? 4u : 0u) |
                   (v[u].w != 0.f ? 8u : 0u);
      if (j + 4 > f) m &= j < f ? (1u << (f - j)) - 1u : 0u;  // columns past f are padding
      int c = __popc(m);
#pragma unroll
      for (int o = G / 2; o > 0; o >>= 1) c += __shfl_xor(c, o, G);
      if (bits) {
        const uint32_t word = group_or<8>(m << (4 * (lane % 8)));
        if (lane % 8 == 0 && j < f) bits[row * words + j / 32] = word;
      }
      if (lane == 0) {
        cnt[row] = c;
        if (cnt64) cnt64[row] = c;
      }
    }
  }
}

// X_csr from the bits: `G` lanes per row (a power of two), 32 columns per lane and turn.
template <int G>
__global__ void __launch_bounds__(256) k_bits_to_csr(const float* X, int32_t n, int64_t ldx, const uint32_t* bits,
                                                     int64_t words, const int64_t* row_ptr, int32_t* col,
                                                     float* val) {
  const int64_t row = ((int64_t)blockIdx.x * 256 + threadIdx.x) / G;
  const int lane = threadIdx.x % G;
  if (row >= n) return;  // whole groups leave together
  const float* x = X + row * ldx;
  int64_t base = row_ptr[row];
  for (int64_t w0 = 0; w0 < words; w0 += G) {
    uint32_t m = w0 + lane < words ? bits[row * words + w0 + lane] : 0u;
    const int c = __popc(m);
    int incl = c;
#pragma unroll
    for (int o = 1; o < G; o <<= 1) {
      const int up = __shfl_up(incl, o, G);
      if (lane >= o) incl += up;
    }
    int64_t pos = base + incl - c;
    while (m) {
      const int j = (int)(w0 + lane) * 32 + __ffs(m) - 1;
      m &= m - 1;
      col[pos] = j;
      val[pos] = x[j];
      ++pos;
    }
    base += __shfl(incl, G - 1, G);
  }
}

// X_csr from a second walk over X, for dense rows.
__global__ void __launch_bounds__(256) k_to_csr(const float* X, int32_t n, int32_t f, int64_t ldx,
                                                const int64_t* row_ptr, int32_t* col, float* val) {
  const int64_t row = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 64;
  const int lane = threadIdx.x % 64;
  if (row >= n) return;
  const float* x = X + row * ldx;
  int64_t pos = row_ptr[row];
  const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  for (int j0 = 0; j0 < f; j0 += 512) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int j = j0 + 64 * u + lane;
      v[u] = j < f ? x[j] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const bool nz = v[u] != 0.0f;
      const uint64_t bal = __ballot(nz);
      if (nz) {
        const int64_t p = pos + __popcll(bal & below);
        col[p] = j0 + 64 * u + lane;
        val[p] = v[u];
      }
      pos += __popcll(bal);
    }
  }
}

// Entries of X_csr per (row chunk, column); blockIdx.y: block of kColBlock columns.
__global__ void __launch_bounds__(256) k_chunk_counts(const int64_t* row_ptr, const int32_t* col, int32_t n,
                                                      int32_t f, int64_t rows, int32_t* chunk_cnt) {
  __shared__ int32_t cnt[kColBlock];
  const int32_t c0 = (int32_t)blockIdx.y * kColBlock;
  const int32_t nc = f - c0 < kColBlock ? f - c0 : kColBlock;
  for (int j = threadIdx.x; j < nc; j += 256) cnt[j] = 0;
  __syncthreads();
  const int64_t r0 = (int64_t)blockIdx.x * rows, r1 = r0 + rows < n ? r0 + rows : n;
  const int64_t end = row_ptr[r1];
  for (int64_t e = row_ptr[r0] + threadIdx.x; e < end; e += 256) {
    const int32_t j = col[e] - c0;
    if (j >= 0 && j < nc) atomicAdd(&cnt[j], 1);
  }
  __syncthreads();
  for (int j = threadIdx.x; j < nc; j += 256) chunk_cnt[(int64_t)blockIdx.x * f + c0 + j] = cnt[j];
}

// Per column: exclusive offsets of each chunk within the column, and the column total.  A
// workgroup takes 64 columns; its 16 wavefronts sum a sixteenth of the chunks each, exchange
// their sums, and write their offsets.
__global__ void __launch_bounds__(1024) k_chunk_scan(int64_t nchunks, int32_t f, const int32_t* chunk_cnt,
                                                     int32_t* chunk_off, int32_t* col_tot) {
  __shared__ int32_t sums[16][64];
  const int c = threadIdx.x % 64, seg = threadIdx.x / 64;
  const int64_t j = (int64_t)blockIdx.x * 64 + c;
  const int64_t per = (nchunks + 15) / 16;
  const int64_t k0 = seg * per < nchunks ? seg * per : nchunks;
  const int64_t k1 = k0 + per < nchunks ? k0 + per : nchunks;
  int32_t sum = 0;
  if (j < f) {
#pragma unroll 8
    for (int64_t k = k0; k < k1; ++k) sum += chunk_cnt[k * f + j];
  }
  sums[seg][c] = sum;
  __syncthreads();
  if (j >= f) return;
  int32_t run = 0;
  for (int q = 0; q < seg; ++q) run += sums[q][c];
  int64_t k = k0;
  for (; k + 8 <= k1; k += 8) {
    int32_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = chunk_cnt[(k + u) * f + j];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      chunk_off[(k + u) * f + j] = run;
      run += v[u];
    }
  }
  for (; k < k1; ++k) {
    chunk_off[k * f + j] = run;
    run += chunk_cnt[k * f + j];
  }
  if (seg == 15) col_tot[j] = run;
}

// One wavefront per row chunk (and block of columns): its entries, row after row, to their
// places in the columns.  Eight rows' entries are requested while the eight before are placed.
__global__ void __launch_bounds__(64) k_to_csc(const int64_t* row_ptr, const int32_t* col, const float* val, int32_t n,
                                               int32_t f, int64_t rows, const int64_t* col_ptr,
                                               const int32_t* chunk_off, int32_t* rowi, float* cval) {
  constexpr int U = 8;
  __shared__ int32_t off[kColBlock];  // running count of each column (from the chunk's offset)
  const int lane = threadIdx.x;
  const int32_t c0 = (int32_t)blockIdx.y * kColBlock;
  const int32_t nc = f - c0 < kColBlock ? f - c0 : kColBlock;
  for (int j = lane; j < nc; j += 64) off[j] = chunk_off[(int64_t)blockIdx.x * f + c0 + j];
  __syncthreads();
  const int64_t r0 = (int64_t)blockIdx.x * rows, r1 = r0 + rows < n ? r0 + rows : n;
  auto place = [&](int64_t row, int32_t j, float v, bool ok) {
    const int32_t jc = j - c0;
    if (!ok || jc < 0 || jc >= nc) return;
    const int64_t pos = col_ptr[j] + atomicAdd(&off[jc], 1);
    rowi[pos] = (int32_t)row;
    cval[pos] = v;
  };
  for (int64_t rb = r0; rb < r1; rb += 64) {
    // lane l holds the offsets of row rb + l
    const int64_t lr = rb + lane < r1 ? rb + lane : r1;
    const int64_t my_beg = row_ptr[lr], my_end = row_ptr[lr < r1 ? lr + 1 : r1];
    int32_t j[2][U];
    float v[2][U];
    auto load = [&](int g, int32_t (&jj)[U], float (&vv)[U]) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t beg = __shfl(my_beg, g + u, 64), end = __shfl(my_end, g + u, 64);
        jj[u] = 0;
        vv[u] = 0.f;
        if (beg + lane < end) {
          jj[u] = col[beg + lane];
          vv[u] = val[beg + lane];
        }
      }
    };
    auto put = [&](int g, const int32_t (&jj)[U], const float (&vv)[U]) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t beg = __shfl(my_beg, g + u, 64), end = __shfl(my_end, g + u, 64);
        place(rb + g + u, jj[u], vv[u], beg + lane < end);
        for (int64_t e = beg + 64; e < end; e += 256) {  // wave-uniform: the rest of a long row
          int32_t jl[4];
          float vl[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int64_t at = e + 64 * q + lane;
            jl[q] = at < end ? col[at] : 0;
            vl[q] = at < end ? val[at] : 0.f;
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) place(rb + g + u, jl[q], vl[q], e + 64 * q + lane < end);
        }
      }
    };
    load(0, j[0], v[0]);
#pragma unroll
    for (int g = 0; g < 64; g += 2 * U) {
      load(g + U, j[1], v[1]);
      put(g, j[0], v[0]);
      if (g + 2 * U < 64) load(g + 2 * U, j[0], v[0]);
      put(g + U, j[1], v[1]);
    }
  }
}

}  // namespace

size_t feature_stats_workspace(int32_t n, int32_t f, bool bits, bool want_csc) {
  Arena a;
  carve(a, n, f, bits, want_csc);
  return a.used;
}

gcn_status run_feature_stats(const float* X, int32_t n, int32_t f, int64_t ldx, int32_t tau_num,
                             int32_t tau_den, int32_t force_mode, int64_t* row_nnz, gcn_feature_info* info,
                             gcn_sparse_x* x, bool have_bits, void* ws, hipStream_t s) {
  const bool want_csc = x && x->col_ptr;
  Arena a;
  a.base = static_cast<char*>(ws);
  FeatWs w = carve(a, n, f, have_bits, want_csc);
  uint32_t* const bits = w.bits;
  if (n > 0) {
    // a grid that fills the chip twice over: a wavefront walks many rows
    const unsigned gw = (unsigned)std::min<int64_t>(ceil_div(n, 4), 4096);
    const bool vec = ldx % 4 == 0 && aligned16(X);
    auto narrow = [&](auto lanes) {
      constexpr int G = decltype(lanes)::value;
      const unsigned gn = (unsigned)std::min<int64_t>(ceil_div((int64_t)n * G, 256), 4096);
      hipLaunchKernelGGL(k_row_counts_narrow<G>, dim3(gn), dim3(256), 0, s, X, n, f, ldx, w.row_cnt, row_nnz, bits, w.words);
    };
    if (vec && f <= 32) narrow(std::integral_constant<int, 8>{});
    else if (vec && f <= 64) narrow(std::integral_constant<int, 16>{});
    else if (vec && f <= 128) narrow(std::integral_constant<int, 32>{});
    else if (vec)
      hipLaunchKernelGGL(k_row_counts<true>, dim3(gw), dim3(256), 0, s, X, n, f, ldx, w.row_cnt, row_nnz, bits, w.words);
    else
      hipLaunchKernelGGL(k_row_counts<false>, dim3(gw), dim3(256), 0, s, X, n, f, ldx, w.row_cnt, row_nnz, bits, w.words);
    GCN_TRY(check_launch("feature row counts"));
  }
  int64_t* rp = (x && x->row_ptr) ? x->row_ptr : w.row_off;
  GCN_TRY(launch_scan_i32(w.row_cnt, n, rp, w.scan, s));
  int64_t nnz = 0;
  GCN_HIP(hipMemcpyAsync(&nnz, rp + n, sizeof nnz, hipMemcpyDeviceToHost, s), "feature nnz");
  GCN_HIP(hipStreamSynchronize(s), "feature sync");
  const __int128 nf = (__int128)n * f;
  info->nnz = nnz;
  info->sparsity = nf > 0 ? 1.0 - (double)nnz / (double)nf : 0.0;
  const bool sparse = (__int128)tau_den * (nf - nnz) >= (__int128)tau_num * nf;
  info->mode = force_mode >= 0 ? force_mode : (sparse ? GCN_SPARSE : GCN_DENSE);
  if (!x) return GCN_OK;

  if (nnz > x->nnz)
    return fail(GCN_E_CAPACITY, "gcn_feature_stats: nnz(X) = " + std::to_string(nnz) +
                                    " exceeds the sparse capacity " + std::to_string(x->nnz));
  x->nnz = nnz;
  x->n = n;
  x->f = f;
  if (n > 0 && f > 0) {
    // From one nonzero in 20 on, most lines of X hold one: read it again in order (262,144 x
    // 1,024, whole call: 3 % 629 us from the bits, 685 by the walk; 6 % 723 and 706; 50 % 4,234
    // and 903).
    if (!bits || (__int128)nnz * 20 >= nf) {
      hipLaunchKernelGGL(k_to_csr, dim3((unsigned)ceil_div(n, 4)), dim3(256), 0, s, X, n, f, ldx, x->row_ptr, x->col,
                         x->val);
    } else {
      auto go = [&](auto lanes) {
        constexpr int G = decltype(lanes)::value;
        hipLaunchKernelGGL(k_bits_to_csr<G>, dim3((unsigned)ceil_div((int64_t)n * G, 256)), dim3(256), 0, s, X, n, ldx,
                           w.bits, w.words, x->row_ptr, x->col, x->val);
      };
      if (w.words <= 4) go(std::integral_constant<int, 4>{});
      else if (w.words <= 8) go(std::integral_constant<int, 8>{});
      else if (w.words <= 16) go(std::integral_constant<int, 16>{});
      else if (w.words <= 32) go(std::integral_constant<int, 32>{});
      else go(std::integral_constant<int, 64>{});
    }
    GCN_TRY(check_launch("dense to csr"));
  }
  if (want_csc) {
    const int64_t rows = chunk_rows(n, f);
    const dim3 grid((unsigned)w.nchunks, (unsigned)ceil_div(f, kColBlock));
    if (w.nchunks > 0 && f > 0) {
      hipLaunchKernelGGL(k_chunk_counts, grid, dim3(256), 0, s, x->row_ptr, x->col, n, f, rows, w.chunk_cnt);
      GCN_TRY(check_launch("csc chunk counts"));
    }
    hipLaunchKernelGGL(k_chunk_scan, dim3((unsigned)std::max<int64_t>(1, ceil_div(f, 64))), dim3(1024), 0, s, w.nchunks,
                       f, w.chunk_cnt, w.chunk_off, w.col_tot);
    GCN_TRY(check_launch("csc chunk scan"));
    GCN_TRY(launch_scan_i32(w.col_tot, f, x->col_ptr, w.scan, s));
    if (w.nchunks > 0 && f > 0) {
      hipLaunchKernelGGL(k_to_csc, grid, dim3(64), 0, s, x->row_ptr, x->col, x->val, n, f, rows, x->col_ptr,
                         w.chunk_off, x->row, x->cval);
      GCN_TRY(check_launch("dense to csc"));
    }
    if (x->csc_split.rows) GCN_TRY(build_split(x->col_ptr, f, &x->csc_split, true, w.split, s));
  }
  GCN_HIP(hipStreamSynchronize(s), "feature sync");
  return GCN_OK;
}

}  // namespace gcn
