// agg_device.h -- device-side building blocks of the row-parallel sparse products
// (included by the aggregation kernels).
//
// A slice of LANES lanes covers a row's columns, VEC consecutive columns per lane;
// `slots` slices share a row and take every slots-th entry; UNR neighbour-row loads
// are kept in flight per lane; the slices are summed with cross-lane adds, so every
// slice ends with the row's total.  No atomics: results are deterministic.
#pragma once

#include "internal.h"
#include "lanes.h"

#ifndef GCN_AGG_UNR
#define GCN_AGG_UNR 16  // neighbour-row loads kept in flight per lane, full-wavefront rows
#endif

namespace gcn {
namespace {

template <int VEC>
struct Vec;
template <>
struct Vec<4> {
  using T = float4;
  static __device__ __forceinline__ T load(const float* p) { return *reinterpret_cast<const float4*>(p); }
  static __device__ __forceinline__ void store(float* p, const T& v) { *reinterpret_cast<float4*>(p) = v; }
  static __device__ __forceinline__ T zero() { return make_float4(0.f, 0.f, 0.f, 0.f); }
  static __device__ __forceinline__ void fma(T& acc, float w, const T& x) {
    acc.x = fmaf(w, x.x, acc.x);
    acc.y = fmaf(w, x.y, acc.y);
    acc.z = fmaf(w, x.z, acc.z);
    acc.w = fmaf(w, x.w, acc.w);
  }
  static __device__ __forceinline__ void add(T& acc, const T& x) {
    acc.x += x.x;
    acc.y += x.y;
    acc.z += x.z;
    acc.w += x.w;
  }
  static __device__ __forceinline__ float get(const T& v, int i) {
    return i == 0 ? v.x : (i == 1 ? v.y : (i == 2 ? v.z : v.w));
  }
  static __device__ __forceinline__ void add_xor(T& v, int o, int width) {
    v.x += __shfl_xor(v.x, o, width);
    v.y += __shfl_xor(v.y, o, width);
    v.z += __shfl_xor(v.z, o, width);
    v.w += __shfl_xor(v.w, o, width);
  }
};
template <>
struct Vec<1> {
  using T = float;
  static __device__ __forceinline__ T load(const float* p) { return *p; }
  static __device__ __forceinline__ void store(float* p, const T& v) { *p = v; }
  static __device__ __forceinline__ T zero() { return 0.f; }
  static __device__ __forceinline__ void fma(T& acc, float w, const T& x) { acc = fmaf(w, x, acc); }
  static __device__ __forceinline__ void add(T& acc, const T& x) { acc += x; }
  static __device__ __forceinline__ float get(const T& v, int) { return v; }
  static __device__ __forceinline__ void add_xor(T& v, int o, int width) { v += __shfl_xor(v, o, width); }
};

template <int LANES>
__device__ __forceinline__ float group_max(float v) {
  return group_reduce<LANES>(v, [](float a, float b) { return fmaxf(a, b); });
}
template <int LANES>
__device__ __forceinline__ float group_sum(float v) {
  return group_reduce<LANES>(v, [](float a, float b) { return a + b; });
}

// Lane geometry of a group of LANES * slots lanes owning one (virtual) row.
struct Lanes {
  int gw, lig, slot, lane, c0;
};

template <int LANES, int VEC>
__device__ __forceinline__ Lanes lanes_of(int slots) {
  Lanes L;
  L.gw = LANES * slots;
  L.lig = threadIdx.x & (L.gw - 1);
  L.slot = L.lig / LANES;
  L.lane = L.lig & (LANES - 1);
  L.c0 = (blockIdx.y * LANES + L.lane) * VEC;
  return L;
}

// Column index and value of entry beg + lig (lane lig of the group), the first chunk
// of a row; zero past the row's end.
struct First {
  int j;
  float w;
};

// Weight of entry e (column j) by the aggregation kind (wave-uniform branch).
__device__ __forceinline__ float entry_weight(const AggParams& p, int64_t e, int j) {
  if (p.kind == AGG_W_VAL) return p.val[e];
  if (p.kind == AGG_W_COLMEAN) return 1.f / (float)p.deg[j];
  return 1.f;
}

// Factor applied to a row's sum: 1 / deg[row] for the mean, else 1.
__device__ __forceinline__ float row_scale(const AggParams& p, int64_t row) {
  return p.kind == AGG_W_ROWMEAN ? 1.f / (float)p.deg[row] : 1.f;
}

template <int LANES>
__device__ __forceinline__ First load_first(const AggParams& p, int64_t beg, int64_t end, const Lanes& L) {
  First f{0, 0.f};
  if (beg + L.lig < end) {
    f.j = p.col[beg + L.lig];
    f.w = entry_weight(p, beg + L.lig, f.j);
  }
  return f;
}

// sum_{e in [beg, end)} w_e M[col[e], c0 .. c0+VEC), every slice of the group holding the
// total.  first: the group's first chunk of entries (load_first), already requested by
// the caller.
// UNR: loads kept in flight per lane.
template <int LANES>
constexpr int agg_unroll() { return LANES == 64 ? GCN_AGG_UNR : (LANES >= 4 ? 8 : 4); }
template <int LANES, int VEC, int UNR = agg_unroll<LANES>()>
__device__ __forceinline__ typename Vec<VEC>::T accumulate(const AggParams& p, int64_t beg, int64_t end,
                                                           const Lanes& L, int slots, bool cok, First first) {
  using V = Vec<VEC>;
  typename V::T acc = V::zero();
  const float* Mc = p.M + L.c0;
  for (int64_t base = beg; base < end; base += L.gw) {
    const int cnt = (int)((end - base) < L.gw ? (end - base) : L.gw);
    int my_j = first.j;
    float my_w = first.w;
    if (base != beg) {
      my_j = L.lig < cnt ? p.col[base + L.lig] : 0;
      my_w = L.lig < cnt ? entry_weight(p, base + L.lig, my_j) : 0.f;
    }
    for (int t = 0; t < cnt; t += slots * UNR) {
      int jj[UNR];
      float ww[UNR];
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
      for (int u = 0; u < UNR; ++u) ww[u] = __shfl(my_w, ok[u] ? t + u * slots + L.slot : 0, L.gw);
#pragma unroll
      for (int u = 0; u < UNR; ++u) V::fma(acc, ok[u] ? ww[u] : 0.f, xs[u]);
    }
  }
  for (int o = LANES; o < L.gw; o <<= 1) V::add_xor(acc, o, L.gw);
  return acc;
}

// Bias and epilogue of one row.  Every slice of the group holds the row's total and
// slice 0 writes; with OWN, each slice holds a row of its own (own: that row exists and
// is finished here) and writes it.
template <int LANES, int VEC, int EPI, bool OWN = false>
__device__ __forceinline__ void finish_row(const AggParams& p, int64_t row, const typename Vec<VEC>::T& acc,
                                           const Lanes& L, bool cok, bool own = true) {
  using V = Vec<VEC>;
  const int c0 = L.c0;
  const bool writer = OWN ? own : L.slot == 0;
  const float sc = own ? row_scale(p, row) : 1.f;
  float z[VEC];
#pragma unroll
  for (int i = 0; i < VEC; ++i) {
    const int c = c0 + i;
    z[i] = sc * V::get(acc, i);
    if (p.bias && c < p.w) z[i] += p.bias[c];
  }
  if constexpr (EPI == AGG_SOFTMAX) {
    // whole logits row is held by each slice (w <= LANES * VEC); slice 0 writes
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < VEC; ++i)
      if (c0 + i < p.w) mx = fmaxf(mx, z[i]);
    mx = group_max<LANES>(mx);
    float e[VEC];
    float se = 0.f;
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      e[i] = (c0 + i < p.w) ? expf(z[i] - mx) : 0.f;
      se += e[i];
    }
    se = group_sum<LANES>(se);
    const int y = own ? p.labels[row] : -1;
    float zy = 0.f;
#pragma unroll
    for (int i = 0; i < VEC; ++i)
      if (c0 + i == y) zy = z[i];
    zy = group_sum<LANES>(zy);
    if (!writer) return;
    if (L.lane == 0) p.row_loss[row] = (logf(se) + mx) - zy;
    if (!cok) return;
    const float inv_se = 1.f / se;
    float gv[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) gv[i] = (e[i] * inv_se - (c0 + i == y ? 1.f : 0.f)) * p.inv_n;
    float* out = p.Z + row * p.ldz + c0;
    float* lg = p.logits ? p.logits + row * p.ldl + c0 : nullptr;
    if (VEC == 4 && c0 + 4 <= p.w) {
      *reinterpret_cast<float4*>(out) = make_float4(gv[0], gv[VEC > 1 ? 1 : 0], gv[VEC > 2 ? 2 : 0],
                                                    gv[VEC > 3 ? 3 : 0]);
    } else {
#pragma unroll
      for (int i = 0; i < VEC; ++i)
        if (c0 + i < p.w) out[i] = gv[i];
    }
    if (lg) {
#pragma unroll
      for (int i = 0; i < VEC; ++i)
        if (c0 + i < p.w) lg[i] = z[i];
    }
  } else {
    if constexpr (EPI == AGG_RELU) {
      if (p.relu_bits) {
        // 1[z > 0] of this lane's columns, OR-ed over the lanes of one 32-column word
        // (every lane of the group takes part before any leaves)
        constexpr int kWordLanes = LANES < 32 / VEC ? LANES : 32 / VEC;
        uint32_t bits = 0;
#pragma unroll
        for (int i = 0; i < VEC; ++i)
          if (c0 + i < p.w && z[i] > 0.f) bits |= 1u << ((c0 + i) % 32);
        bits = group_or<kWordLanes>(bits);
        if (writer && c0 < p.w && L.lane % kWordLanes == 0) p.relu_bits[row * p.ld_relu_bits + c0 / 32] = bits;
      }
    }
    if (!cok || !writer) return;
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
      if constexpr (EPI == AGG_RELU) z[i] = fmaxf(z[i], 0.f);
      if constexpr (EPI == AGG_MASK) {
        const int c = c0 + i;
        if (c < p.w) z[i] = p.mask[row * p.ldmask + c] > 0.f ? z[i] : 0.f;
      }
    }
    float* out = p.Z + row * p.ldz + c0;
    if (VEC == 4 && c0 + 4 <= p.w) {
      // written once and not read by this kernel: a non-temporal store leaves L2 to the
      // gathered rows
      typedef float f32x4 __attribute__((ext_vector_type(4)));
      const f32x4 o = {z[0], z[VEC > 1 ? 1 : 0], z[VEC > 2 ? 2 : 0], z[VEC > 3 ? 3 : 0]};
      __builtin_nontemporal_store(o, reinterpret_cast<f32x4*>(out));
    } else {
#pragma unroll
      for (int i = 0; i < VEC; ++i)
        if (c0 + i < p.w) out[i] = z[i];
    }
  }
}

}  // namespace
}  // namespace gcn
