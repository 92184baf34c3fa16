// aggmax.hip -- max aggregation over the rows of A + I and its gradient.
//
// Section III-A names mean, max and sum aggregators; Listing 1 trains GraphSAGE
// with "Max".  Forward, per row u and column c:
//   P[u,c] = max over v in row u of M[v,c],  arg[u,c] = the first such v
// (columns ascending), the same lane-slice mapping as the linear aggregation:
// each slice keeps (value, column) of its entries in order, and slices combine by
// "larger value, then smaller column", so the result does not depend on how the
// row was cut.  Backward is the gradient's gather form over the symmetric rows:
//   dM[u,c] = sum over v in row u of dP[v,c] * [arg[v,c] == u]
// (optionally times 1[mask > 0]); no atomics, fixed order.
//
// Rows of 16-byte pieces wider than 16 columns are walked one row per wavefront (agg_walk.h;
// k_walk_max, k_walk_max_bwd); narrower and unaligned ones by lane groups, a long row by one of
// them.  Both directions are bound as the linear aggregation is, by the gathers from behind the
// L2; the gradient gathers two rows per entry (dP and the maximisers).  169,343 rows of 15, width
// 128 (lane groups -> wavefronts): forward 274 -> 202 us, gradient 404 -> 346.  (With local ids, where
// the gathers hit the L2, two panels cost more than one: 232,965 rows joined to the 16 around them,
// width 256, forward 353 -> 475, gradient 411 -> 451.)
#include "agg_walk.h"

namespace gcn {
namespace {

constexpr int kBlock = 256;

struct MaxArgs {
  AggParams a;          // rows / graph and M (forward) or dP (backward) in a.M, a.ldm
  int32_t* arg;         // forward output
  const int32_t* carg;  // backward input
  int64_t ldarg;
  float* out;           // P (forward) or dM (backward)
  int64_t ldo;
  const float* mask;    // backward: 1[mask > 0] applied when non-NULL
  int64_t ldmask;
};

template <int VEC>
struct Lane {
  float v[VEC];
  int j[VEC];
};

template <int LANES, int VEC>
__global__ void __launch_bounds__(kBlock) k_agg_max(MaxArgs m, int slots) {
  using V = Vec<VEC>;
  constexpr int UNR = LANES >= 4 ? 8 : 4;
  const AggParams& p = m.a;
  const Lanes L = lanes_of<LANES, VEC>(slots);
  const int64_t row = (int64_t)blockIdx.x * (kBlock / L.gw) + threadIdx.x / L.gw;
  if (row >= p.n) return;  // whole groups leave together
  const int64_t beg = p.row_ptr[row], end = p.row_ptr[row + 1];
  const bool cok = L.c0 < p.w;
  Lane<VEC> best;
#pragma unroll
  for (int i = 0; i < VEC; ++i) {
    best.v[i] = -INFINITY;
    best.j[i] = INT32_MAX;
  }
  const float* Mc = p.M + L.c0;
  for (int64_t base = beg; base < end; base += L.gw) {
    const int cnt = (int)((end - base) < L.gw ? (end - base) : L.gw);
    const int my_j = L.lig < cnt ? p.col[base + L.lig] : 0;
    for (int t = 0; t < cnt; t += slots * UNR) {
      int jj[UNR];
      bool ok[UNR];
      typename V::T xs[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int e = t + u * slots + L.slot;
        ok[u] = e < cnt;
        jj[u] = __shfl(my_j, ok[u] ? e : 0, L.gw);
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u) xs[u] = (ok[u] && cok) ? V::load(Mc + (int64_t)jj[u] * p.ldm) : V::zero();
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        if (!ok[u]) continue;
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
          const float x = V::get(xs[u], i);
          // entries of a slice come in increasing column order: strict > keeps the first
          if (x > best.v[i] || best.j[i] == INT32_MAX) {
            best.v[i] = x;
            best.j[i] = jj[u];
          }
        }
      }
    }
  }
  // combine the slices: larger value, then smaller column
  for (int o = LANES; o < L.gw; o <<= 1) {
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      const float ov = __shfl_xor(best.v[i], o, L.gw);
      const int oj = __shfl_xor(best.j[i], o, L.gw);
      if (ov > best.v[i] || (ov == best.v[i] && oj < best.j[i]) || best.j[i] == INT32_MAX) {
        if (oj != INT32_MAX) {
          best.v[i] = ov;
          best.j[i] = oj;
        }
      }
    }
  }
  if (!cok || L.slot != 0) return;
  float* po = m.out + row * m.ldo + L.c0;
  int32_t* ao = m.arg + row * m.ldarg + L.c0;
#pragma unroll
  for (int i = 0; i < VEC; ++i)
    if (L.c0 + i < p.w) {
      po[i] = best.v[i];
      ao[i] = best.j[i];
    }
}

template <int LANES, int VEC, bool MASK>
__global__ void __launch_bounds__(kBlock) k_agg_max_bwd(MaxArgs m, int slots) {
  using V = Vec<VEC>;
  constexpr int UNR = LANES >= 4 ? 8 : 4;
  const AggParams& p = m.a;
  const Lanes L = lanes_of<LANES, VEC>(slots);
  const int64_t row = (int64_t)blockIdx.x * (kBlock / L.gw) + threadIdx.x / L.gw;
  if (row >= p.n) return;
  const int64_t beg = p.row_ptr[row], end = p.row_ptr[row + 1];
  const bool cok = L.c0 < p.w;
  float acc[VEC];
#pragma unroll
  for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
  const float* Dc = p.M + L.c0;
  const int32_t* Ac = m.carg + L.c0;
  const int me = (int)row;
  for (int64_t base = beg; base < end; base += L.gw) {
    const int cnt = (int)((end - base) < L.gw ? (end - base) : L.gw);
    const int my_j = L.lig < cnt ? p.col[base + L.lig] : 0;
    for (int t = 0; t < cnt; t += slots * UNR) {
      int jj[UNR];
      bool ok[UNR];
      typename V::T xs[UNR];
      int as[UNR][VEC];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int e = t + u * slots + L.slot;
        ok[u] = e < cnt;
        jj[u] = __shfl(my_j, ok[u] ? e : 0, L.gw);
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        xs[u] = V::zero();
#pragma unroll
        for (int i = 0; i < VEC; ++i) as[u][i] = -1;
        if (ok[u] && cok) {
          xs[u] = V::load(Dc + (int64_t)jj[u] * p.ldm);
          const int32_t* ap = Ac + (int64_t)jj[u] * m.ldarg;
          if constexpr (VEC == 4) {
            const int4 a4 = *reinterpret_cast<const int4*>(ap);
            as[u][0] = a4.x;
            as[u][VEC > 1 ? 1 : 0] = a4.y;
            as[u][VEC > 2 ? 2 : 0] = a4.z;
            as[u][VEC > 3 ? 3 : 0] = a4.w;
          } else {
            as[u][0] = ap[0];
          }
        }
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u)
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[i] += as[u][i] == me ? V::get(xs[u], i) : 0.f;
    }
  }
  for (int o = LANES; o < L.gw; o <<= 1)
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] += __shfl_xor(acc[i], o, L.gw);
  if (!cok || L.slot != 0) return;
  float* out = m.out + row * m.ldo + L.c0;
#pragma unroll
  for (int i = 0; i < VEC; ++i) {
    if (L.c0 + i >= p.w) continue;
    float v = acc[i];
    if constexpr (MASK) v = m.mask[row * m.ldmask + L.c0 + i] > 0.f ? v : 0.f;
    out[i] = v;
  }
}

// Larger value, then smaller column; an entry replaces "none" (INT32_MAX).
__device__ __forceinline__ void take_max(float& v, int& j, float ov, int oj) {
  if (oj != INT32_MAX && (ov > v || (ov == v && oj < j) || j == INT32_MAX)) {
    v = ov;
    j = oj;
  }
}

template <int LANES>
__global__ void __launch_bounds__(kWalkThreads) k_walk_max(MaxArgs m, int32_t rounds) {
  __shared__ __attribute__((aligned(16))) float s_v[2][kWalkWaves][4 * LANES];
  __shared__ __attribute__((aligned(16))) int s_j[2][kWalkWaves][4 * LANES];
  const AggParams& p = m.a;
  const Lanes L = walk_lanes<LANES>();
  const bool cok = L.c0 < p.w;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const char* Mc = reinterpret_cast<const char*>(p.M);
  const uint32_t lane_off = cok ? 4u * (uint32_t)L.c0 : 0u;
  const uint32_t pitch = 4u * (uint32_t)p.ldm;
  const uint32_t hi = walk_row(walk_group(blockIdx.x, gridDim.x), gridDim.x, L.lig);
  Piece h{0, 0, -1};
  if (L.lig < kWalkWaves * rounds && hi < (uint32_t)p.n)
    h = Piece{p.row_ptr[hi], (int32_t)(p.row_ptr[hi + 1] - p.row_ptr[hi]), (int32_t)hi};
  const Items items = make_items(h, rounds, wave, L.lig, true);
  Cursor<LANES> cursor;
  auto fetch = [&]() __attribute__((always_inline)) {
    int64_t at;
    return cursor.next(items, L, &at) ? p.col[at] : 0;
  };
  int j0 = fetch(), j1 = fetch();
  int parity = 0;
  for (int t = 0; t < items.n; ++t) {
    const int row = __builtin_amdgcn_readlane(items.row, t);
    const int len = __builtin_amdgcn_readlane(items.len, t);
    const int fin = __builtin_amdgcn_readlane(items.kind, t);
    const bool mine = row >= 0 && (fin < 0 || fin == wave);
    float bv[4];
    int bj[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      bv[i] = -INFINITY;
      bj[i] = INT32_MAX;
    }
    int done = 0;
    do {
      const int cnt = len - done < 64 ? len - done : 64;
      const Runs rn = runs_of<LANES>(cnt, L.slot);
      const int j = j0;
      const uint32_t off = (uint32_t)j0 * pitch;
      j0 = j1;
      // four steps at a time: a slice's entries come in increasing column order, so a strictly
      // larger value keeps the first maximiser
      auto steps = [&](auto uc, auto between) __attribute__((always_inline)) {
        constexpr int U = decltype(uc)::value;
        float4 x[4];
        int jj[4];
        auto load = [&](auto ic) __attribute__((always_inline)) {
          constexpr int I = decltype(ic)::value;
          const uint32_t o = from_lane<LANES, U + I>(off) + lane_off;
          jj[I] = (int)from_lane<LANES, U + I>((uint32_t)j);
          x[I] = make_float4(0.f, 0.f, 0.f, 0.f);
          if (U + I < rn.have) x[I] = *reinterpret_cast<const float4*>(Mc + o);
        };
        load(std::integral_constant<int, 0>{});
        load(std::integral_constant<int, 1>{});
        load(std::integral_constant<int, 2>{});
        load(std::integral_constant<int, 3>{});
        between();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (U + q >= rn.have) continue;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float v = Vec<4>::get(x[q], i);
            if (v > bv[i] || bj[i] == INT32_MAX) {
              bv[i] = v;
              bj[i] = jj[q];
            }
          }
        }
      };
      steps(std::integral_constant<int, 0>{}, [&]() __attribute__((always_inline)) { j1 = fetch(); });
      if (rn.run > 4) steps(std::integral_constant<int, 4>{}, [] {});
      if constexpr (LANES > 8) {
        if (rn.run > 8) steps(std::integral_constant<int, 8>{}, [] {});
        if (rn.run > 12) steps(std::integral_constant<int, 12>{}, [] {});
      }
      if constexpr (LANES > 16) {
        if (rn.run > 16) steps(std::integral_constant<int, 16>{}, [] {});
        if (rn.run > 20) steps(std::integral_constant<int, 20>{}, [] {});
        if (rn.run > 24) steps(std::integral_constant<int, 24>{}, [] {});
        if (rn.run > 28) steps(std::integral_constant<int, 28>{}, [] {});
      }
      done += 64;
    } while (done < len);
    for (int o = LANES; o < 64; o <<= 1)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float ov = __shfl_xor(bv[i], o, 64);
        const int oj = __shfl_xor(bj[i], o, 64);
        take_max(bv[i], bj[i], ov, oj);
      }
    if (fin >= 0) {
      const int at = parity;
      parity ^= 1;
      if (L.slot == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          s_v[at][wave][4 * L.lane + i] = bv[i];
          s_j[at][wave][4 * L.lane + i] = bj[i];
        }
      }
      __syncthreads();  // every wavefront has the same shared items
      if (!mine) continue;
#pragma unroll
      for (int q = 0; q < kWalkWaves; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) take_max(bv[i], bj[i], s_v[at][q][4 * L.lane + i], s_j[at][q][4 * L.lane + i]);
    }
    if (!mine || !cok || L.slot != 0) continue;
    float* po = m.out + (int64_t)row * m.ldo + L.c0;
    int32_t* ao = m.arg + (int64_t)row * m.ldarg + L.c0;
    if (L.c0 + 4 <= p.w) {
      *reinterpret_cast<float4*>(po) = make_float4(bv[0], bv[1], bv[2], bv[3]);
      *reinterpret_cast<int4*>(ao) = make_int4(bj[0], bj[1], bj[2], bj[3]);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (L.c0 + i < p.w) {
          po[i] = bv[i];
          ao[i] = bj[i];
        }
    }
  }
}

template <int LANES, bool MASK>
__global__ void __launch_bounds__(kWalkThreads) k_walk_max_bwd(MaxArgs m, int32_t rounds) {
  __shared__ __attribute__((aligned(16))) float s_part[2][kWalkWaves][4 * LANES];
  const AggParams& p = m.a;
  const Lanes L = walk_lanes<LANES>();
  const bool cok = L.c0 < p.w;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  const char* Dc = reinterpret_cast<const char*>(p.M);
  const char* Ac = reinterpret_cast<const char*>(m.carg);
  const uint32_t lane_off = cok ? 4u * (uint32_t)L.c0 : 0u;
  const uint32_t dpitch = 4u * (uint32_t)p.ldm, apitch = 4u * (uint32_t)m.ldarg;
  const uint32_t hi = walk_row(walk_group(blockIdx.x, gridDim.x), gridDim.x, L.lig);
  Piece h{0, 0, -1};
  if (L.lig < kWalkWaves * rounds && hi < (uint32_t)p.n)
    h = Piece{p.row_ptr[hi], (int32_t)(p.row_ptr[hi + 1] - p.row_ptr[hi]), (int32_t)hi};
  const Items items = make_items(h, rounds, wave, L.lig, true);
  Cursor<LANES> cursor;
  auto fetch = [&]() __attribute__((always_inline)) {
    int64_t at;
    return cursor.next(items, L, &at) ? p.col[at] : 0;
  };
  int j0 = fetch(), j1 = fetch();
  int parity = 0;
  for (int t = 0; t < items.n; ++t) {
    const int row = __builtin_amdgcn_readlane(items.row, t);
    const int len = __builtin_amdgcn_readlane(items.len, t);
    const int fin = __builtin_amdgcn_readlane(items.kind, t);
    const bool mine = row >= 0 && (fin < 0 || fin == wave);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f), mk = acc;
    if (MASK && mine && cok && L.slot == 0) mk = *reinterpret_cast<const float4*>(m.mask + (int64_t)row * m.ldmask + L.c0);
    int done = 0;
    do {
      const int cnt = len - done < 64 ? len - done : 64;
      const Runs rn = runs_of<LANES>(cnt, L.slot);
      const uint32_t doff = (uint32_t)j0 * dpitch, aoff = (uint32_t)j0 * apitch;
      j0 = j1;
      auto steps = [&](auto uc, auto between) __attribute__((always_inline)) {
        constexpr int U = decltype(uc)::value;
        float4 x[4];
        int4 a[4];
        auto load = [&](auto ic) __attribute__((always_inline)) {
          constexpr int I = decltype(ic)::value;
          const uint32_t od = from_lane<LANES, U + I>(doff) + lane_off, oa = from_lane<LANES, U + I>(aoff) + lane_off;
          x[I] = make_float4(0.f, 0.f, 0.f, 0.f);
          a[I] = make_int4(-1, -1, -1, -1);
          if (U + I < rn.have) {
            x[I] = *reinterpret_cast<const float4*>(Dc + od);
            a[I] = *reinterpret_cast<const int4*>(Ac + oa);
          }
        };
        load(std::integral_constant<int, 0>{});
        load(std::integral_constant<int, 1>{});
        load(std::integral_constant<int, 2>{});
        load(std::integral_constant<int, 3>{});
        between();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          acc.x += a[q].x == row ? x[q].x : 0.f;
          acc.y += a[q].y == row ? x[q].y : 0.f;
          acc.z += a[q].z == row ? x[q].z : 0.f;
          acc.w += a[q].w == row ? x[q].w : 0.f;
        }
      };
      steps(std::integral_constant<int, 0>{}, [&]() __attribute__((always_inline)) { j1 = fetch(); });
      if (rn.run > 4) steps(std::integral_constant<int, 4>{}, [] {});
      if constexpr (LANES > 8) {
        if (rn.run > 8) steps(std::integral_constant<int, 8>{}, [] {});
        if (rn.run > 12) steps(std::integral_constant<int, 12>{}, [] {});
      }
      if constexpr (LANES > 16) {
        if (rn.run > 16) steps(std::integral_constant<int, 16>{}, [] {});
        if (rn.run > 20) steps(std::integral_constant<int, 20>{}, [] {});
        if (rn.run > 24) steps(std::integral_constant<int, 24>{}, [] {});
        if (rn.run > 28) steps(std::integral_constant<int, 28>{}, [] {});
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
    if (!mine || !cok || L.slot != 0) continue;
    if (MASK) {
      acc.x = mk.x > 0.f ? acc.x : 0.f;
      acc.y = mk.y > 0.f ? acc.y : 0.f;
      acc.z = mk.z > 0.f ? acc.z : 0.f;
      acc.w = mk.w > 0.f ? acc.w : 0.f;
    }
    float* out = m.out + (int64_t)row * m.ldo + L.c0;
    if (L.c0 + 4 <= p.w) {
      *reinterpret_cast<float4*>(out) = acc;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (L.c0 + i < p.w) out[i] = Vec<4>::get(acc, i);
    }
  }
}

template <int VEC, class F>
gcn_status dispatch_lanes(int lanes, F&& f) {
  switch (lanes) {
    case 1: return f(std::integral_constant<int, 1>{});
    case 2: return f(std::integral_constant<int, 2>{});
    case 4: return f(std::integral_constant<int, 4>{});
    case 8: return f(std::integral_constant<int, 8>{});
    case 16: return f(std::integral_constant<int, 16>{});
    case 32: return f(std::integral_constant<int, 32>{});
    default: return f(std::integral_constant<int, 64>{});
  }
}

}  // namespace

// vec4 needs 16-byte rows for every operand the kernel touches
static bool max_vec4(const MaxArgs& m, bool fwd) {
  const AggParams& p = m.a;
  bool ok = p.ldm % 4 == 0 && aligned16(p.M) && m.ldo % 4 == 0 && aligned16(m.out) && m.ldarg % 4 == 0;
  ok = ok && aligned16(fwd ? (const void*)m.arg : (const void*)m.carg);
  if (!fwd && m.mask) ok = ok && m.ldmask % 4 == 0 && aligned16(m.mask);
  return ok;
}

static gcn_status launch_max(const MaxArgs& m, int64_t nnz, bool fwd, hipStream_t s) {
  const AggParams& p = m.a;
  if (p.n == 0 || p.w == 0) return GCN_OK;
  const bool vec4 = max_vec4(m, fwd);
  const int vec = vec4 ? 4 : 1;
  char name[64];
  snprintf(name, sizeof name, "%s_w%d", fwd ? "aggmax" : "aggmax_bwd", p.w);
  // The panel of the linear aggregation (its own measurements); rows of dP and of the
  // maximisers are addressed by 32-bit offsets.
  if (vec4 && p.w > 16 && (fwd || 4 * p.src_rows * m.ldarg <= (int64_t)UINT32_MAX)) {
    const BlockedPlan b = agg_blocked_plan(p.n, p.src_rows, nnz, p.w, p.ldm, ROWS_GRAPH_MAX, false);
    if (b.nblock > 0) {
      ProfScope prof(name, p.w, p.n, nnz, s);
      const int64_t panels = ceil_div(p.w, 4 * b.lanes);
      const int rounds = (int)std::max<int64_t>(1, std::min<int64_t>(2, (int64_t)p.n * panels / 32768));
      const dim3 grid((unsigned)ceil_div(p.n, (int64_t)rounds * kWalkWaves), (unsigned)panels);
      auto go = [&](auto lt) -> gcn_status {
        constexpr int LN = decltype(lt)::value;
        if (fwd) hipLaunchKernelGGL((k_walk_max<LN>), grid, dim3(kWalkThreads), 0, s, m, rounds);
        else if (m.mask) hipLaunchKernelGGL((k_walk_max_bwd<LN, true>), grid, dim3(kWalkThreads), 0, s, m, rounds);
        else hipLaunchKernelGGL((k_walk_max_bwd<LN, false>), grid, dim3(kWalkThreads), 0, s, m, rounds);
        return check_launch(fwd ? "max aggregation" : "max aggregation gradient");
      };
      if (b.lanes == 8) return go(std::integral_constant<int, 8>{});
      if (b.lanes == 16) return go(std::integral_constant<int, 16>{});
      return go(std::integral_constant<int, 32>{});
    }
  }
  int lanes = 1;
  while (lanes < ceil_div(p.w, vec) && lanes < 64) lanes <<= 1;
  if ((int64_t)lanes * vec < p.w) return fail(GCN_E_UNSUPPORTED, "max aggregation: width above 256 (vector) or 64");
  const int slots = agg_slots(lanes, nnz, p.n);
  const int gw = lanes * slots;
  const dim3 grid((unsigned)ceil_div(p.n, kBlock / gw));
  ProfScope prof(name, p.w, p.n, nnz, s);
  auto go = [&](auto lt) -> gcn_status {
    constexpr int LN = decltype(lt)::value;
    if (vec4) {
      if (fwd) hipLaunchKernelGGL((k_agg_max<LN, 4>), grid, dim3(kBlock), 0, s, m, slots);
      else if (m.mask) hipLaunchKernelGGL((k_agg_max_bwd<LN, 4, true>), grid, dim3(kBlock), 0, s, m, slots);
      else hipLaunchKernelGGL((k_agg_max_bwd<LN, 4, false>), grid, dim3(kBlock), 0, s, m, slots);
    } else {
      if (fwd) hipLaunchKernelGGL((k_agg_max<LN, 1>), grid, dim3(kBlock), 0, s, m, slots);
      else if (m.mask) hipLaunchKernelGGL((k_agg_max_bwd<LN, 1, true>), grid, dim3(kBlock), 0, s, m, slots);
      else hipLaunchKernelGGL((k_agg_max_bwd<LN, 1, false>), grid, dim3(kBlock), 0, s, m, slots);
    }
    return check_launch(fwd ? "max aggregation" : "max aggregation gradient");
  };
  return vec4 ? dispatch_lanes<4>(lanes, go) : dispatch_lanes<1>(lanes, go);
}

gcn_status launch_aggregate_max(const AggParams& p, int64_t nnz, float* P, int64_t ldp, int32_t* arg,
                                int64_t ldarg, hipStream_t s) {
  MaxArgs m{};
  m.a = p;
  m.arg = arg;
  m.ldarg = ldarg;
  m.out = P;
  m.ldo = ldp;
  return launch_max(m, nnz, true, s);
}

gcn_status launch_aggregate_max_bwd(const AggParams& p, int64_t nnz, const int32_t* arg, int64_t ldarg,
                                    const float* mask, int64_t ldmask, float* dM, int64_t ldo, hipStream_t s) {
  MaxArgs m{};
  m.a = p;
  m.carg = arg;
  m.ldarg = ldarg;
  m.out = dM;
  m.ldo = ldo;
  m.mask = mask;
  m.ldmask = ldmask;
  return launch_max(m, nnz, false, s);
}

}  // namespace gcn
