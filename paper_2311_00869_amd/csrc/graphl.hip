// graphL (Section "graphL: optimization formulation"): the relaxed loss of
// Eq. eq-loss_imbalance_new, its gradient, the descent update of
// Alg. alg-gradient and the final rounding plus exact count, for R restarts
// stored as the columns of Gamma[n][R].
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "fi_internal.h"
#include "fi_prims.h"

// No multiply-add contraction in this file: every kernel that computes an
// update rounds the same operations the same way, so the fused small-graph
// descent, the per-step kernels and their vector variants agree bit for bit.
#pragma clang fp contract(off)

namespace fi {

namespace {

constexpr int kGLBlock = 256;

// lanes per edge / row: the smallest power of two >= R (R <= 64)
__host__ __device__ __forceinline__ int lanes_for(int R) {
  int p = 1;
  while (p < R) p <<= 1;
  return p;
}

// V consecutive restarts of a lane (4 as one 16-byte access, or 1).
template <int V>
struct Lane {
  float x[V];
};
template <int V>
__device__ __forceinline__ Lane<V> load_lane(const float* p) {
  Lane<V> r;
  if constexpr (V == 4) {
    const float4 q = *reinterpret_cast<const float4*>(p);
    r.x[0] = q.x;
    r.x[1] = q.y;
    r.x[2] = q.z;
    r.x[3] = q.w;
  } else {
    r.x[0] = *p;
  }
  return r;
}
template <int V>
__device__ __forceinline__ void store_lane(float* p, const Lane<V>& v) {
  if constexpr (V == 4) *reinterpret_cast<float4*>(p) = make_float4(v.x[0], v.x[1], v.x[2], v.x[3]);
  else *p = v.x[0];
}

// Loss partials: block b, restart r -> part[b * 64 + r].  Edge terms
// (1 - e G_u G_v) / 2 are formed in float32 and accumulated in float64; the
// assignment of edges to threads and the reduction tree are fixed, so the
// result is bit-reproducible.  Each lane owns V restarts and P lanes share an
// edge, kFwdEdges edges per lane in flight.  The counting edge list has every
// edge once, in the row of its endpoint of lower rank: that endpoint's row of
// Gamma is read in order, and the gathered one is the endpoint of higher
// degree, which the caches hold.  1M vertices, 4M edges, R = 32:
// 69 us (one restart per lane, one edge in flight, in the order of the smaller
// id: 327); 4M / 16M 327 us (1.55 ms).
constexpr int kFwdEdges = 4;
template <int P, int V>
__global__ void __launch_bounds__(kGLBlock) k_gl_forward(const uint2* edges, int64_t m,
                                                         const float* gamma, int R, double* part) {
  constexpr int kGroups = kGLBlock / P;
  __shared__ double s_acc[kGLBlock * V];
  const int sub = threadIdx.x % P, grp = threadIdx.x / P;
  const bool active = V * sub < R;
  double acc[V];
#pragma unroll
  for (int q = 0; q < V; ++q) acc[q] = 0.0;
  for (int64_t b = (int64_t)blockIdx.x * kGroups * kFwdEdges; b < m;
       b += (int64_t)gridDim.x * kGroups * kFwdEdges) {
    uint2 uv[kFwdEdges];
    Lane<V> gu[kFwdEdges], gv[kFwdEdges];
#pragma unroll
    for (int k = 0; k < kFwdEdges; ++k) uv[k] = edges[min(b + k * kGroups + grp, m - 1)];
#pragma unroll
    for (int k = 0; k < kFwdEdges; ++k) {
      gu[k] = gv[k] = Lane<V>{};
      if (active && b + k * kGroups + grp < m) {
        gu[k] = load_lane<V>(gamma + (size_t)uv[k].x * R + V * sub);
        gv[k] = load_lane<V>(gamma + (size_t)(uv[k].y & kVertexMask) * R + V * sub);
      }
    }
#pragma unroll
    for (int k = 0; k < kFwdEdges; ++k) {
      const float sg = (uv[k].y >> 31) ? -1.0f : 1.0f;
      if (b + k * kGroups + grp < m)
#pragma unroll
        for (int q = 0; q < V; ++q)
          acc[q] += (double)((1.0f - sg * gu[k].x[q] * gv[k].x[q]) * 0.5f);
    }
  }
#pragma unroll
  for (int q = 0; q < V; ++q) s_acc[threadIdx.x * V + q] = acc[q];
  __syncthreads();
  // fold the edge slots of each restart: fixed pairwise tree over the groups
  for (int h = kGroups / 2; h > 0; h >>= 1) {
    for (int i = threadIdx.x; i < h * P * V; i += kGLBlock) s_acc[i] += s_acc[i + h * P * V];
    __syncthreads();
  }
  if ((int)threadIdx.x < R) part[(size_t)blockIdx.x * kGraphLMaxR + threadIdx.x] = s_acc[threadIdx.x];
}

// loss[r] = the sum of restart r's partials: one block per restart, each
// thread a fixed stride of them, then a fixed tree.  (One thread per restart
// adding all 1,024 in a chain took 243 us.)
__global__ void __launch_bounds__(kGLBlock) k_gl_forward_final(const double* part, int nblocks,
                                                               double* loss) {
  __shared__ double s_acc[kGLBlock];
  double s = 0.0;
  for (int b = threadIdx.x; b < nblocks; b += kGLBlock)
    s += part[(size_t)b * kGraphLMaxR + blockIdx.x];
  s_acc[threadIdx.x] = s;
  __syncthreads();
  for (int h = kGLBlock / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) s_acc[threadIdx.x] += s_acc[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss[blockIdx.x] = s_acc[0];
}

// Row gathers: g[i][r] = -1/2 * w_r * sum over the row of e_ij G[j][r].
// With `update` the kernels write the descent update G - alpha * g instead.
// Every row's summation order is fixed, so the result is bit-reproducible.
//
// Overflow policy of the descent (graphs whose hubs make the update grow by
// up to (1 + alpha * lambda_max / 2) per step).  The update never mixes
// connected components, and components grow at very different rates (a hub
// component by many orders of magnitude more than a two-vertex one), so
// each (component, restart) pair keeps its own power-of-two scale: when the
// pair's largest |G| reached 2^shift after the previous step, this step
// reads the pair's entries scaled by 2^-shift and adds shift to its log2
// scale.  Scaling by a power of two is exact in floating point, so each
// component's stored iterates are the plain descent's times 2^-scale, bit
// for bit, unless an entry falls 2^-149 below its own component's largest.
// Vertices without edges never change and keep scale 0.
struct RowArgs {
  const double* w;          // gradient weights per restart, or null (1)
  float alpha;
  int update;
  // descent with scaling (all null for a plain step or gradient)
  const int32_t* comp;      // anchor of each vertex's component
  const int32_t* aslot;     // component slot of each anchor
  const int32_t* anchors;   // anchor of each component slot
  const uint32_t* max_in;   // [C][R] float bits of max |G_in| (exact from the threshold on)
  uint32_t* max_out;        // [C][R] max |G_out| (atomic max)
  uint32_t* max_clear;      // [C][R] the buffer the step after next fills
  int32_t* exps;            // [C][R] log2 scales
  int64_t ncr;              // C * R
  int32_t main_slot;        // the largest component: its maxima are combined per block
  int shift;                // rescale threshold and step, log2
};

__device__ __forceinline__ uint32_t scale_threshold(const RowArgs& A) {
  return (uint32_t)(127 + A.shift) << 23;  // 2^shift
}
__device__ __forceinline__ float pair_scale(const RowArgs& A, int32_t c, int R, int sub) {
  if (c < 0) return 1.0f;
  return A.max_in[(size_t)c * R + sub] >= scale_threshold(A)
             ? __uint_as_float((uint32_t)(127 - A.shift) << 23)
             : 1.0f;
}

// After a row's output v of restart `sub`: its component's maximum and, on
// the component's anchor row, the scale.  NAN_COUNTS: a NaN is above every
// threshold in the main component too.
template <bool NAN_COUNTS>
__device__ __forceinline__ void note_row(const RowArgs& A, int64_t i, int32_t c, int R, int sub,
                                         float sc, float v, float& mx_main) {
  if (c < 0) return;
  const float a = fabsf(v);
  if (c == A.main_slot) mx_main = fmaxf(mx_main, a);
  // only whether the threshold is reached matters (20 rings of 1,000 at R = 64
  // spent 120 of a step's 128 us on the maxima of values below it)
  if ((c != A.main_slot || (NAN_COUNTS && a != a)) && __float_as_uint(a) >= scale_threshold(A))
    atomicMax((unsigned int*)&A.max_out[(size_t)c * R + sub], __float_as_uint(a));
  if (A.comp[i] == i && sc != 1.0f) A.exps[(size_t)c * R + sub] += A.shift;
}

// max_out = max(max_out, m) for the main component, whose maximum every
// workgroup updates: only a workgroup above the value it reads does (the value
// never falls within a launch, so a stale read costs an atomic and loses
// nothing).  65,536 workgroups of 32 atomics each on one line took 2.1 ms of a
// 3.1 ms step on 4M vertices.
__device__ __forceinline__ void raise_max(uint32_t* max_out, float m) {
  const uint32_t b = __float_as_uint(m);
  if (m > 0.0f && b > __hip_atomic_load(max_out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMax((unsigned int*)max_out, b);
}

// The component slot of row i (-1: no edges): most rows lie in the main
// component (anchor main_label), which needs no second load.
__device__ __forceinline__ int32_t row_slot(const RowArgs& A, int64_t i, int64_t e0, int64_t e1,
                                            int32_t main_label) {
  if (e1 <= e0) return -1;
  const int32_t label = A.comp[i];
  return label == main_label ? A.main_slot : A.aslot[label];
}

// The rows that are not one group's, as listed at upload.
struct GLPlan {
  const int32_t* heavy;  // rows of more than kGLHeavy entries, cut into items
  const int2* items;     // (place in heavy, chunk)
  float* part;           // [nitems][kGraphLMaxR]
  const int32_t* mid;    // rows of mid_len + 1 .. kGLHeavy entries
  uint32_t nitems, nmid;
  int32_t mid_len;
  uint32_t mid_at, short_at;  // the first block of the mid rows and of the short ones
};

constexpr int kGLBatch = 8;  // gathers of a row in flight per lane

// Entries a[k] = e0 + k step (k < 8) that lie below e1, and y[k] = G[j] for the
// lane's restarts, zero past e1.  All entries are loaded before the gathers
// and all gathers are in flight together, those of the last few entries of a
// row too.  Of fewer than eight, with P >= 8 lanes to a row, each lane loads
// one and they are exchanged.
template <int P, int V>
__device__ __forceinline__ void gather8(const uint32_t* adj, int32_t e0, int32_t e1, int32_t step,
                                        const float* gamma, int R, int sub, bool active,
                                        uint32_t* a, Lane<V>* y) {
  if (e1 - e0 > (kGLBatch - 1) * step) {  // eight: nothing to mask
    const int r0 = active ? V * sub : 0;
#pragma unroll
    for (int k = 0; k < kGLBatch; ++k) a[k] = adj[e0 + k * step];
#pragma unroll
    for (int k = 0; k < kGLBatch; ++k) y[k] = load_lane<V>(gamma + (size_t)(a[k] & kVertexMask) * R + r0);
    return;
  }
  if constexpr (P >= kGLBatch) {
    const int base = lane_id() & ~(P - 1);
    const uint32_t mine = adj[e0 + min((sub & (kGLBatch - 1)) * step, e1 - e0 - 1)];
#pragma unroll
    for (int k = 0; k < kGLBatch; ++k) a[k] = (uint32_t)__shfl((int)mine, base + k);
  } else {
#pragma unroll
    for (int k = 0; k < kGLBatch; ++k) a[k] = adj[e0 + min(k * step, e1 - e0 - 1)];
  }
#pragma unroll
  for (int k = 0; k < kGLBatch; ++k) {
    y[k] = Lane<V>{};
    if (active && k * step < e1 - e0)
      y[k] = load_lane<V>(gamma + (size_t)(a[k] & kVertexMask) * R + V * sub);
  }
}

// y[k] = e_ij * G[j] * sc.
template <int V>
__device__ __forceinline__ void sign_scale(const uint32_t* a, const Lane<V>& sc, Lane<V>* y) {
#pragma unroll
  for (int k = 0; k < kGLBatch; ++k) {
    const bool ng = (a[k] >> 31) != 0;
#pragma unroll
    for (int q = 0; q < V; ++q) {
      const float x = y[k].x[q] * sc.x[q];
      y[k].x[q] = ng ? -x : x;
    }
  }
}

// Sum over entries e0, e0 + step, ... < e1, added in that order (the zeros past
// e1 change no sum).  The scale is asked for once the first gathers are in
// flight, so that its own loads do not go before them.
template <int P, int V, class Scale>
__device__ __forceinline__ Lane<V> row_sum(const uint32_t* adj, int32_t e0, int32_t e1, int32_t step,
                                           const float* gamma, int R, int sub, bool active,
                                           Scale scale) {
  Lane<V> acc{};
  Lane<V> sc{};
  for (int32_t left = e1 - e0; left > 0; left -= kGLBatch * step) {
    const int32_t e = e1 - left;
    uint32_t a[kGLBatch];
    Lane<V> y[kGLBatch];
    gather8<P, V>(adj, e, e1, step, gamma, R, sub, active, a, y);
    if (left == e1 - e0) sc = scale();
    sign_scale<V>(a, sc, y);
#pragma unroll
    for (int k = 0; k < kGLBatch; ++k)
#pragma unroll
      for (int q = 0; q < V; ++q) acc.x[q] += y[k].x[q];
  }
  return acc;
}

// One pass over the rows: g[i][r] = -1/2 * w_r * sum over the row, or the
// update.  Each lane owns V restarts and P lanes (a power of two with V P >= R)
// share a row; a wave holds 64 / P such groups.
//   long rows (more than kGLHeavy entries): items of up to kGLChunk entries,
//     one per workgroup, its groups striding over the item and their sums added
//     in group order into part[item][r]; k_gl_combine adds a row's items in order
//   rows of mid_len + 1 .. kGLHeavy entries: one wave each, eight entries per
//     group at a time, their sum carried from group to group in the row's order
//   shorter rows: one group each
// Longest first, each kind from the block after the last one's, so that no long
// chain starts last and a small graph's blocks have one each.  Every row but the long
// ones is summed in its own order whatever P and V are, so the variants agree
// bit for bit.  Bound by the rate of random line fetches (52 to 59 G/s of 128
// bytes here; R = 32 gathers one line per entry), as long as a row's gathers
// are in flight together: with a row's last few entries gathered one by one
// and long rows in a launch of their own, 4M vertices and 16M edges at R = 32
// took 3.28 ms per step (2.1 of it the maxima, raise_max), now 0.96 (0.73 for
// a gradient); a gradient of 100,000 / 500,000 took 82 us with rows up to 256
// entries on one group each, now 22, of 5,000 / 20,000 29 us, now 15.  SCALED keeps
// the registers of the overflow policy out of gradients, four and five waves per
// SIMD (200,000 / 2M at R = 64: 100 us; one kernel of 134 registers, three: 128).
template <int P, int V, bool SCALED, bool NAN_COUNTS>
__global__ void __launch_bounds__(kGLBlock, P * V < 16 ? 1 : SCALED ? 4 : 5) k_gl_pass(const int32_t* rp, const uint32_t* adj,
                                                      int32_t n, GLPlan L, const float* gamma, int R,
                                                      RowArgs A, float* out) {
  constexpr int kGroups = kGLBlock / P, kWaveGroups = 64 / P, NW = kGLBlock / 64;
  constexpr int kStage = kWaveGroups * kGLBatch;  // entries a wave takes at a time
  __shared__ float s_mx[kGLBlock * V];
  const int sub = threadIdx.x % P, grp = threadIdx.x / P;
  const int wave = threadIdx.x >> 6, wgrp = grp % kWaveGroups;
  const int r0 = V * sub;
  const bool active = r0 < R;
  const int32_t main_label = SCALED && A.main_slot >= 0 ? A.anchors[A.main_slot] : -1;
  Lane<V> wr, scm, mx;
#pragma unroll
  for (int k = 0; k < V; ++k) {
    wr.x[k] = (A.w && active) ? (float)A.w[r0 + k] : 1.0f;
    scm.x[k] = SCALED && active ? pair_scale(A, A.main_slot, R, r0 + k) : 1.0f;
    mx.x[k] = 0.0f;
  }
  if constexpr (SCALED)
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < A.ncr;
         k += (int64_t)gridDim.x * blockDim.x)
      A.max_clear[k] = 0;
  auto slot_of = [&](int32_t label) {
    return !SCALED ? -1 : label == main_label ? A.main_slot : A.aslot[label];
  };
  auto scale_of = [&](int32_t c) {
    Lane<V> sc;
#pragma unroll
    for (int k = 0; k < V; ++k)
      sc.x[k] = !SCALED || !active || c < 0 ? 1.0f
                : c == A.main_slot          ? scm.x[k]
                                            : pair_scale(A, c, R, r0 + k);
    return sc;
  };
  // (read before the row's gathers, so that it is in flight with them)
  auto load_self = [&](int64_t i) {
    return A.update && active ? load_lane<V>(gamma + (size_t)i * R + r0) : Lane<V>{};
  };
  auto finish = [&](int64_t i, int32_t c, const Lane<V>& sc, const Lane<V>& self, const Lane<V>& acc) {
    const size_t o = (size_t)i * R + r0;
    Lane<V> v;
#pragma unroll
    for (int k = 0; k < V; ++k) {
      const float g = -0.5f * acc.x[k] * wr.x[k];
      v.x[k] = A.update ? self.x[k] * sc.x[k] - A.alpha * g : g;
    }
    store_lane<V>(out + o, v);
    if constexpr (SCALED)
#pragma unroll
      for (int k = 0; k < V; ++k) note_row<NAN_COUNTS>(A, i, c, R, r0 + k, sc.x[k], v.x[k], mx.x[k]);
  };

  // long rows' items
  for (uint32_t it = blockIdx.x; it < L.nitems; it += gridDim.x) {
    const int2 hc = L.items[it];
    const int64_t i = L.heavy[hc.x];
    const int32_t b0 = rp[i], b1 = rp[i + 1];
    const int32_t e0 = b0 + hc.y * kGLChunk;
    const int32_t e1 = e0 + min(b1 - e0, kGLChunk);
    const Lane<V> acc = row_sum<P, V>(adj, e0 + grp, e1, kGroups, gamma, R, sub, active, [&] {
      return scale_of(SCALED ? row_slot(A, i, b0, b1, main_label) : -1);
    });
#pragma unroll
    for (int k = 0; k < V; ++k) s_mx[threadIdx.x * V + k] = acc.x[k];
    __syncthreads();
    if ((int)threadIdx.x < R) {
      float tot = 0.0f;
      for (int g = 0; g < kGroups; ++g) tot += s_mx[g * P * V + threadIdx.x];
      L.part[(size_t)it * kGraphLMaxR + threadIdx.x] = tot;
    }
    __syncthreads();
  }

  // rows of one wave each
  auto block_from = [&](uint32_t at) {
    return (int64_t)(blockIdx.x >= at ? blockIdx.x - at : blockIdx.x + gridDim.x - at);
  };
  const int64_t nwaves = (int64_t)gridDim.x * NW;
  for (int64_t m = block_from(L.mid_at) * NW + wave; m < (int64_t)L.nmid; m += nwaves) {
    const int64_t i = L.mid[m];
    const int32_t b0 = rp[i], b1 = rp[i + 1];
    const int32_t label = SCALED ? A.comp[i] : -1;
    const Lane<V> self = load_self(i);
    int32_t c = -1;
    Lane<V> acc{}, sc{};
    for (int32_t left = b1 - b0; left > 0; left -= kStage) {
      const int32_t mine = left - wgrp * kGLBatch;  // entries from the group's first on
      uint32_t a[kGLBatch];
      Lane<V> y[kGLBatch] = {};
      if (mine > 0) gather8<P, V>(adj, b1 - mine, b1, 1, gamma, R, sub, active, a, y);
      if (left == b1 - b0) {
        c = slot_of(label);
        sc = scale_of(c);
      }
      if (mine > 0) sign_scale<V>(a, sc, y);
#pragma unroll
      for (int w = 0; w < kWaveGroups; ++w) {
        // (past the row's end y is zero)
        Lane<V> t = acc;
#pragma unroll
        for (int k = 0; k < kGLBatch; ++k)
#pragma unroll
          for (int q = 0; q < V; ++q) t.x[q] += y[k].x[q];
#pragma unroll
        for (int q = 0; q < V; ++q) acc.x[q] = __shfl(t.x[q], w * P + sub);
      }
    }
    if (wgrp == 0 && active) finish(i, c, sc, self, acc);
  }

  // short rows
  for (int64_t i = block_from(L.short_at) * kGroups + grp; i < n; i += (int64_t)gridDim.x * kGroups) {
    const int32_t e0 = rp[i], e1 = rp[i + 1];
    if (e1 - e0 > L.mid_len) continue;
    const int32_t label = SCALED ? A.comp[i] : -1;
    const Lane<V> self = load_self(i);
    int32_t c = -1;
    Lane<V> sc = scale_of(-1);  // (of a row without entries)
    const Lane<V> acc = row_sum<P, V>(adj, e0, e1, 1, gamma, R, sub, active, [&] {
      c = slot_of(label);
      sc = scale_of(c);
      return sc;
    });
    if (active) finish(i, c, sc, self, acc);
  }

  if constexpr (SCALED) {
#pragma unroll
    for (int k = 0; k < V; ++k) s_mx[threadIdx.x * V + k] = mx.x[k];
    __syncthreads();
    if ((int)threadIdx.x < R && A.main_slot >= 0) {
      float m = 0.0f;
      for (int g = 0; g < kGroups; ++g) m = fmaxf(m, s_mx[g * P * V + threadIdx.x]);
      raise_max(&A.max_out[(size_t)A.main_slot * R + threadIdx.x], m);
    }
  }
}

// One group of lanes per heavy row: its items in order, then the update.
__global__ void __launch_bounds__(kGLBlock) k_gl_combine(const int32_t* rp, const int32_t* list,
                                                         const int32_t* first, uint32_t cnt,
                                                         const float* part, const float* gamma,
                                                         int R, RowArgs A, float* out) {
  __shared__ float s_mx[kGLBlock];
  const int P = lanes_for(R);
  const int sub = threadIdx.x % P;
  const int grp = threadIdx.x / P;
  const int gpb = kGLBlock / P;
  const bool active = sub < R;
  const bool scaled = A.max_in != nullptr;
  const float wr = (A.w && active) ? (float)A.w[sub] : 1.0f;
  const int32_t main_label = scaled && A.main_slot >= 0 ? A.anchors[A.main_slot] : -1;
  float mx_main = 0.0f;
  if (active) {
    for (int64_t h = (int64_t)blockIdx.x * gpb + grp; h < cnt; h += (int64_t)gridDim.x * gpb) {
      const int64_t i = list[h];
      const int32_t c = scaled ? row_slot(A, i, rp[i], rp[i + 1], main_label) : -1;
      const float sc = scaled ? pair_scale(A, c, R, sub) : 1.0f;
      float tot = 0.0f;
      const int32_t i1 = first[h + 1];
      for (int32_t it = first[h]; it < i1; it += 8) {  // eight loads in flight, added in order
        float x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
          x[k] = it + k < i1 ? part[(size_t)(it + k) * kGraphLMaxR + sub] : 0.0f;
#pragma unroll
        for (int k = 0; k < 8; ++k)
          if (it + k < i1) tot += x[k];
      }
      const float g = -0.5f * tot * wr;
      const size_t o = (size_t)i * R + sub;
      const float v = A.update ? gamma[o] * sc - A.alpha * g : g;
      out[o] = v;
      if (scaled) note_row<false>(A, i, c, R, sub, sc, v, mx_main);
    }
  }
  if (scaled) {
    s_mx[threadIdx.x] = mx_main;
    __syncthreads();
    if (grp == 0 && active && A.main_slot >= 0) {
      float m = 0.0f;
      for (int g = 0; g < gpb; ++g) m = fmaxf(m, s_mx[g * P + sub]);
      raise_max(&A.max_out[(size_t)A.main_slot * R + sub], m);
    }
  }
}

// Items of the heavy rows (one workgroup): first[h] = the first item of
// heavy row h, first[count] = ctl[1] = the number of items.
__global__ void __launch_bounds__(1024) k_gl_plan(const int32_t* rp, const int32_t* list,
                                                  uint32_t* ctl, int32_t* first, int2* items) {
  __shared__ int s_scan[1024 / 64 + 1];
  const int64_t cnt = ctl[0];
  const int64_t per = (cnt + 1023) / 1024;
  const int64_t h0 = (int64_t)threadIdx.x * per, h1 = min(cnt, h0 + per);
  int mine = 0;
  for (int64_t h = h0; h < h1; ++h) {
    const int64_t i = list[h];
    mine += (int)((rp[i + 1] - rp[i] + kGLChunk - 1) / kGLChunk);
  }
  int total = 0;
  int at = block_exclusive_scan<1024>(mine, total, s_scan);
  for (int64_t h = h0; h < h1; ++h) {
    const int64_t i = list[h];
    const int nch = (int)((rp[i + 1] - rp[i] + kGLChunk - 1) / kGLChunk);
    first[h] = at;
    for (int c = 0; c < nch; ++c) items[at + c] = make_int2((int)h, c);
    at += nch;
  }
  if (threadIdx.x == 0) {
    first[cnt] = total;
    ctl[1] = (uint32_t)total;
  }
}

// The whole descent on a small graph: one workgroup per
// restart, Gamma's column in LDS (ping-pong), and the per-component overflow
// flags and scales in LDS too, so the steps run with no launch between them.
// Same rows, same order, same operations as the per-step kernels; a row of more
// than kGLHeavy entries by a wave, whose lanes are the `groups` of k_gl_pass.
//
// A step is bound by the CU's LDS gathers and by the instructions around them
// (a wave's instruction counts its longest row), so each value is kept beside
// its negation and an entry is the LDS offset of the one it adds: a gather and
// a multiply-add.  The leading entries of a row sit in registers, missing ones
// point at a zero, and rows are dealt by length so that a wave's are alike.
// The overflow policy compares a component's maximum with one threshold, so a
// value that reaches it sets a flag.  500 steps at R = 32, us: 1,000 vertices,
// 5,000 edges 457 (with long rows' code in the same kernel 475; the row's entries
// decoded in every step, the CSR in LDS: 755), 300 / 1,200 262 (485), 4,096 /
// 12,000 1,180 (2,425); with hubs, 1,000 / 5,000 3,420 (a launch per step: 6,930).
constexpr int kSmallDescentN = 4096;
constexpr size_t kSmallDescentLds = 152 * 1024;
// Beyond, a restart's one CU takes longer than a launch per step (500 steps, us:
// 4,000 / 60,000 4,770 and 6,300, 1,000 / 60,000 5,990 and 5,380, 1,000 / 200,000
// 28,600 and 6,000); with long rows from half as many (4,000 / 30,000 6,120 and
// 8,090, 4,000 / 60,000 9,900 and 8,100).
constexpr int64_t kSmallEntries = 1 << 17;
constexpr int kSmallLens = 64;  // row lengths told apart (the last: over kGLHeavy)
struct SmallHeavy {  // a long row
  int32_t row, begin, end, slot;
};

// leading entries of a row in registers, for so many rows per thread
constexpr int held_entries(int q) { return q == 1 ? 32 : q == 2 ? 24 : 16; }
// rows per thread
constexpr int small_rows(int32_t n) { return n <= 1024 ? 1 : n <= 2048 ? 2 : 4; }
// LDS bytes of the two columns: n pairs (value, negation), then a zero
constexpr size_t small_column(int q) { return 8 * ((size_t)1024 * q + 1); }

// LONG: with rows of more than H entries, and of more than kGLHeavy if there are
// any (without that code in the same kernel those of H to kGLHeavy take longer: 500
// steps of 1,413 vertices, 3,500 entries and rows of up to 148 2,346 us, here 1,815).
template <int Q, bool LONG>
__global__ void __launch_bounds__(1024) k_gl_descend_small(const int32_t* rp, const uint32_t* adj,
                                                           const int32_t* comp,
                                                           const int32_t* aslot, int32_t n,
                                                           int32_t ncomp, int32_t nheavy, int groups, int R,
                                                           float alpha, int64_t steps, int shift,
                                                           int32_t main_slot, const float* start,
                                                           float* gamma, int32_t* exps) {
  constexpr int H = held_entries(Q), kBatch = Q == 4 ? 4 : 8, kTail = 8;
  constexpr uint32_t kCol = (uint32_t)small_column(Q), kZero = 8 * 1024 * Q;
  extern __shared__ uint32_t sm[];
  __shared__ uint32_t lens[kSmallLens];
  char* const lds = (char*)sm;
  uint32_t* mx = (uint32_t*)(lds + 2 * kCol);  // [3][ncomp]
  int32_t* ex = (int32_t*)(mx + 3 * ncomp);
  SmallHeavy* heavy = (SmallHeavy*)(ex + ncomp);
  uint32_t* perm = (uint32_t*)(lds + kCol);  // (until the first step)
  const int tid = threadIdx.x, r = blockIdx.x;
  const uint32_t thresh = (uint32_t)(127 + shift) << 23;
  const float down = __uint_as_float((uint32_t)(127 - shift) << 23);
  auto offset = [](uint32_t a) { return 8 * (a & kVertexMask) + (a >> 31) * 4; };
  auto len_of = [&](int32_t i) {
    const int32_t d = rp[i + 1] - rp[i];
    return d > kGLHeavy ? kSmallLens - 1 : min(d, kSmallLens - 2);
  };
  // the offsets of entries e .. e + kTail - 1, as far as below end (those behind a
  // row are read with it: the edge list lies behind the last one)
  auto entries = [&](int32_t e, int32_t end, uint32_t* o) {
#pragma unroll
    for (int t = 0; t < kTail; ++t) o[t] = adj[e + t];
#pragma unroll
    for (int t = 0; t < kTail; ++t) o[t] = e + t < end ? offset(o[t]) : kZero;
  };

  if (tid < kSmallLens) lens[tid] = 0;
  for (int32_t c = tid; c < 3 * ncomp; c += 1024) mx[c] = 0;
  for (int32_t c = tid; c < ncomp; c += 1024) ex[c] = 0;
  if (tid < 2) *(float2*)(lds + tid * kCol + kZero) = make_float2(0.0f, 0.0f);
  for (int32_t i = tid; i < n; i += 1024) {
    const float v = start[(size_t)i * R + r];
    *(float2*)(lds + 8 * i) = make_float2(v, -v);
  }
  __syncthreads();
  // rows by length, longest first
  for (int32_t i = tid; i < n; i += 1024) atomicAdd(&lens[len_of(i)], 1u);
  __syncthreads();
  if (tid < 64) {
    uint32_t mine = lens[63 - tid], upto = mine;
    for (int d = 1; d < 64; d *= 2) {
      const uint32_t below = __shfl_up(upto, d);
      if (tid >= d) upto += below;
    }
    lens[63 - tid] = upto - mine;
  }
  __syncthreads();
  for (int32_t i = tid; i < n; i += 1024) perm[atomicAdd(&lens[len_of(i)], 1u)] = (uint32_t)i;
  __syncthreads();

  // each thread's rows: their vertex, end, component slot, anchor flag, value
  // and leading entries in registers, and the wave's longest (in an SGPR)
  int32_t row[Q], rb[Q], re[Q], rc[Q], longest[Q];
  bool ra[Q];
  float own[Q];
  uint32_t held[Q][H];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    // (every other thousand runs backwards, so that waves share the long ones)
    const int32_t p = q * 1024 + (q & 1 ? 1023 - tid : tid);
    row[q] = p < n && p >= nheavy ? (int32_t)perm[p] : -1;
    const int32_t i = max(row[q], 0);
    rb[q] = row[q] >= 0 ? rp[i] : 0;
    re[q] = row[q] >= 0 ? rp[i + 1] : 0;
    rc[q] = re[q] > rb[q] ? aslot[comp[i]] : -1;
    ra[q] = row[q] >= 0 && comp[i] == i;
    own[q] = row[q] >= 0 ? *(float*)(lds + 8 * i) : 0.0f;
    longest[q] = (int32_t)__builtin_amdgcn_readfirstlane((int)wave_max_u32((uint32_t)(re[q] - rb[q])));
#pragma unroll
    for (int t = 0; t < H; ++t) held[q][t] = rb[q] + t < re[q] ? offset(adj[rb[q] + t]) : kZero;
  }
  for (int32_t h = tid; h < nheavy; h += 1024) {
    const int32_t i = (int32_t)perm[h];
    heavy[h] = SmallHeavy{i, rp[i], rp[i + 1], aslot[comp[i]]};
  }
  __syncthreads();

  int k3 = 0;  // step mod 3: which flags are read, written, cleared
  // one step from the column at `from` into the one at `to`
  auto step = [&](auto from, auto to) {
    const uint32_t* min_ = mx + k3 * ncomp;
    uint32_t* mout = mx + (k3 == 2 ? 0 : k3 + 1) * ncomp;
    uint32_t* mclr = mx + (k3 == 0 ? 2 : k3 - 1) * ncomp;
    const char* gin = lds + decltype(from)::value;
    char* gout = lds + decltype(to)::value;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (q * 1024 >= n) break;
      const int32_t c = rc[q];
      const uint32_t over = c >= 0 ? min_[c] : 0u;
      float acc = 0.0f;
      const float sc = over ? down : 1.0f;
#pragma unroll
      for (int t0 = 0; t0 < H; t0 += kBatch) {
        if (longest[q] <= t0) break;
        float x[kBatch];
#pragma unroll
        for (int t = 0; t < kBatch; ++t) x[t] = *(const float*)(gin + held[q][t0 + t]);
#pragma unroll
        for (int t = 0; t < kBatch; ++t) acc += x[t] * sc;
      }
      if (longest[q] > H) {
        // (a lane past its row's end stays there)
        uint32_t a[kTail];
        entries(min(rb[q] + H, re[q]), re[q], a);
        for (int32_t t0 = H; t0 < longest[q]; t0 += kTail) {
          float x[kTail];
#pragma unroll
          for (int t = 0; t < kTail; ++t) x[t] = *(const float*)(gin + a[t]);
          entries(min(rb[q] + t0 + kTail, re[q]), re[q], a);
#pragma unroll
          for (int t = 0; t < kTail; ++t) acc += x[t] * sc;
        }
      }
      if (row[q] >= 0) {
        const float g = -0.5f * acc * 1.0f;
        const float v = own[q] * sc - alpha * g;
        own[q] = v;
        *(float2*)(gout + 8 * row[q]) = make_float2(v, -v);
        if (sc != 1.0f && ra[q]) ex[c] += shift;
        if (c >= 0 && __float_as_uint(fabsf(v)) >= thresh && (!LONG || c != main_slot || v == v)) mout[c] = 1u;
      }
    }
    for (int32_t h = tid >> 6; LONG && h < nheavy; h += 16) {
      const SmallHeavy w = heavy[h];
      const float sc = min_[w.slot] ? down : 1.0f;
      float acc = 0.0f;
      for (int32_t e0 = w.begin; e0 < w.end; e0 += kGLChunk) {
        const int32_t len = min(kGLChunk, w.end - e0);
        float item = 0.0f;
        for (int g0 = 0; g0 < groups; g0 += 64) {
          const int grp = g0 + (tid & 63);
          float sum = 0.0f;
          for (int32_t at = grp < groups ? grp : len; at < len; at += groups * kBatch) {
            uint32_t a[kBatch];
            float x[kBatch];
#pragma unroll
            for (int t = 0; t < kBatch; ++t) a[t] = adj[e0 + min(at + groups * t, len - 1)];
#pragma unroll
            for (int t = 0; t < kBatch; ++t)
              x[t] = *(const float*)(gin + (at + groups * t < len ? offset(a[t]) : kZero));
#pragma unroll
            for (int t = 0; t < kBatch; ++t) sum += x[t] * sc;
          }
          for (int k = 0; k < min(64, groups - g0); ++k)
            item += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sum), k));
        }
        acc += item;
      }
      if ((tid & 63) == 0) {
        const float g = -0.5f * acc * 1.0f;
        const float v = *(const float*)(gin + 8 * w.row) * sc - alpha * g;
        *(float2*)(gout + 8 * w.row) = make_float2(v, -v);
        if (sc != 1.0f && comp[w.row] == w.row) ex[w.slot] += shift;
        if (__float_as_uint(fabsf(v)) >= thresh && (w.slot != main_slot || v == v)) mout[w.slot] = 1u;
      }
    }
    k3 = k3 == 2 ? 0 : k3 + 1;
    for (int32_t c = tid; c < ncomp; c += 1024) mclr[c] = 0;
    __syncthreads();
  };
  using Col0 = std::integral_constant<uint32_t, 0>;
  using Col1 = std::integral_constant<uint32_t, kCol>;
  for (int64_t k = 0; k + 1 < steps; k += 2) {
    step(Col0{}, Col1{});
    step(Col1{}, Col0{});
  }
  if (steps & 1) step(Col0{}, Col1{});
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (row[q] >= 0) gamma[(size_t)row[q] * R + r] = own[q];
  for (int32_t h = tid; h < nheavy; h += 1024)
    gamma[(size_t)heavy[h].row * R + r] = *(const float*)(lds + (steps & 1) * kCol + 8 * heavy[h].row);
  for (int32_t c = tid; c < ncomp; c += 1024) exps[(size_t)c * R + r] = ex[c];
}

// Per-vertex log2 scales of a descent: out[i][r] = the scale of (component
// of i, r), 0 for vertices without edges.
__global__ void k_gl_scales(const int32_t* rp, const int32_t* comp, const int32_t* aslot,
                            int32_t n, const int32_t* exps, int R, int32_t* out) {
  const int64_t total = (int64_t)n * R;
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < total;
       k += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = k / R;
    const int r = (int)(k - i * R);
    out[k] = rp[i + 1] > rp[i] ? exps[(size_t)aslot[comp[i]] * R + r] : 0;
  }
}

// Rows longer than kGLHeavy and rows longer than mid_len, in any order (each is
// summed on its own), and whether any is longer than `held`.
__global__ void k_gl_heavy_list(const int32_t* rp, int32_t n, int32_t mid_len, int32_t held, int32_t* list,
                                int32_t* mid, uint32_t* ctl) {
  for (int64_t b = (int64_t)blockIdx.x * blockDim.x; b < n; b += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = b + threadIdx.x;
    const int32_t d = i < n ? rp[i + 1] - rp[i] : 0;
    wave_append(d > kGLHeavy, (int32_t)i, list, ctl);
    wave_append(d > mid_len && d <= kGLHeavy, (int32_t)i, mid, ctl + 2);
    if (d > held) ctl[3] = 1;
  }
}

__global__ void k_fill_u32(uint32_t* p, int64_t len, uint32_t v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < len;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// theta = +1 where Gamma >= 0, else -1 (NaN: -1), as one word per vertex:
// bit r of st[v] is set when restart r rounds v to -1 (T: uint32_t for up to
// 32 restarts, else uint64_t).  When R divides 64 a wave reads 64
// consecutive floats of Gamma (64 / R whole vertices) and one ballot gives
// all their words, so Gamma streams through once, coalesced; otherwise each
// thread reads its own vertex's R floats.  Also sets the R counts to zero.
template <typename T>
__global__ void k_gl_round(const float* gamma, int32_t n, int R, T* st, uint64_t* counts) {
  if (blockIdx.x == 0 && (int)threadIdx.x < R) counts[threadIdx.x] = 0;
  const int lane = lane_id();
  const int64_t tid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t nthr = (int64_t)gridDim.x * blockDim.x;
  if (64 % R == 0) {
    const int64_t total = (int64_t)n * R;
    const int per = 64 / R;
    const uint64_t rmask = R == 64 ? ~0ull : ((1ull << R) - 1);
    // wave-uniform chunks of 64 elements (vertex-major, restart-minor)
    for (int64_t e0 = (tid >> 6) << 6; e0 < total; e0 += (nthr >> 6) << 6) {
      const int64_t e = e0 + lane;
      const bool neg = e < total && !(gamma[e] >= 0.0f);
      const uint64_t W = __ballot(neg);
      const int64_t v = e0 / R + lane;
      if (lane < per && v < n) st[v] = (T)((W >> (lane * R)) & rmask);
    }
  } else {
    for (int64_t v = tid; v < n; v += nthr) {
      uint64_t w = 0;
      for (int r = 0; r < R; ++r) w |= (uint64_t)!(gamma[(size_t)v * R + r] >= 0.0f) << r;
      st[v] = (T)w;
    }
  }
}

// Bit i of the low 16 bits of x moved to bit 4 i.
__device__ __forceinline__ uint64_t spread4(uint64_t x) {
  x &= 0xFFFFull;
  x = (x | (x << 24)) & 0x000000FF000000FFull;
  x = (x | (x << 12)) & 0x000F000F000F000Full;
  x = (x | (x << 6)) & 0x0303030303030303ull;
  x = (x | (x << 3)) & 0x1111111111111111ull;
  return x;
}

// The same rounding for R a multiple of 4 that divides 64, Gamma 16-byte
// aligned: lane l of a wave reads floats 4 l .. 4 l + 3 of a 256-float chunk
// (256 / R whole vertices, R / 4 lanes each), one ballot per float of the
// four gives (vertex, restart) bits, and lane j < 256 / R interleaves vertex
// j's bits from them into its word.  Each wave takes two chunks per step, so
// two 16-byte loads per lane are in flight.
template <typename T>
__global__ void k_gl_round4(const float4* gamma4, int32_t n, int R, T* st, uint64_t* counts) {
  if (blockIdx.x == 0 && (int)threadIdx.x < R) counts[threadIdx.x] = 0;
  const int lane = lane_id();
  const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  const int64_t total4 = (int64_t)n * R / 4;
  const int q = R / 4;       // lanes per vertex
  const int per = 64 / q;    // vertices per chunk
  const uint64_t qmask = q == 16 ? 0xFFFFull : ((1ull << q) - 1);
  for (int64_t c0 = wave * 128; c0 < total4; c0 += nwaves * 128) {
    float4 x[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t i = c0 + 64 * h + lane;
      x[h] = i < total4 ? gamma4[i] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint64_t b0 = __ballot(!(x[h].x >= 0.0f)), b1 = __ballot(!(x[h].y >= 0.0f));
      const uint64_t b2 = __ballot(!(x[h].z >= 0.0f)), b3 = __ballot(!(x[h].w >= 0.0f));
      const int64_t v = (c0 + 64 * h) / q + lane;
      if (lane < per && v < n) {
        const int sh = lane * q;
        const uint64_t w = spread4((b0 >> sh) & qmask) | (spread4((b1 >> sh) & qmask) << 1) |
                           (spread4((b2 >> sh) & qmask) << 2) | (spread4((b3 >> sh) & qmask) << 3);
        st[v] = (T)w;
      }
    }
  }
}

// The rounded states as bitmaps, restart by restart: bits[r * nwords + i],
// vertex v is bit v % 64 of word v / 64 (set = -1).  One wave per word: each
// lane reads its vertex's word once, R ballots transpose the 64 x R bits.
template <typename T>
__global__ void k_gl_unpack(const T* st, int32_t n, int32_t nwords, int R, uint64_t* bits) {
  const int lane = lane_id();
  const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t i = wave; i < nwords; i += nwaves) {
    const int64_t v = i * 64 + lane;
    const uint64_t x = v < n ? (uint64_t)st[v] : 0ull;
    uint64_t mine = 0;
    for (int r = 0; r < R; ++r) {
      const uint64_t W = __ballot((x >> r) & 1);
      if (lane == r) mine = W;
    }
    if (lane < R) bits[(size_t)lane * nwords + i] = mine;
  }
}

int grid_for_gl(int64_t work, int block) {
  return (int)std::max<int64_t>(1, std::min<int64_t>((work + block - 1) / block, 65536));
}

// Rows longer than this take a wave each: those that would hold up the other
// rows of a wave, so it follows the mean length (us per gradient, R = 32: 1M /
// 4M 172 with 48 or 256 and 160 with 64; 200,000 / 3M, 85 with 48, 94 with 256,
// 82 with 90; 200,000 / 6M without skew 227 with 48, 196 with 180), unless there
// are too few rows to fill the chip (4,000 / 100,000: 8.7 with 48, 10.4 with 150).
int32_t mid_len(const fi_graph* g) {
  const int64_t mean = g->dg.nnz / std::max<int32_t>(g->dg.n, 1);
  return g->dg.n <= 8192 ? kGLMid : (int32_t)std::max<int64_t>(64, std::min<int64_t>(3 * mean, kGLHeavy));
}

// Workgroups of a pass's short rows, P lanes to a row: a few rounds each, so
// that a workgroup's start and its share of the maxima cost little.
constexpr int64_t kGLPassBlocks = 4096;
int pass_grid(int32_t n, int P) {
  const int gpb = kGLBlock / P;
  return (int)std::max<int64_t>(1, std::min<int64_t>(((int64_t)n + gpb - 1) / gpb, kGLPassBlocks));
}

// graphL control words in the workspace: heavy rows, their items, mid rows
uint32_t* gl_ctl(fi_graph* g) { return (uint32_t*)(g->ws + g->L.glctl); }

// Descent scales in the caller's buffer: exponents, then three max buffers,
// each [C][R] 32-bit words (C = components with an edge, at least 1).
size_t aux_part(const fi_graph* g, int R) {
  const size_t c = (size_t)std::max<int32_t>(g->nanch, 1);
  return (4 * c * (size_t)R + 255) / 256 * 256;
}

// f(P, V) with the lanes per row and the restarts per lane as constants: four
// restarts per lane when each vertex's R floats are whole aligned float4s.
template <class F>
void with_lanes(int R, bool aligned, F f) {
  using std::integral_constant;
  if (R % 4 == 0 && aligned) {
    integral_constant<int, 4> four;
    switch (lanes_for(R / 4)) {
      case 1: f(integral_constant<int, 1>(), four); break;
      case 2: f(integral_constant<int, 2>(), four); break;
      case 4: f(integral_constant<int, 4>(), four); break;
      case 8: f(integral_constant<int, 8>(), four); break;
      default: f(integral_constant<int, 16>(), four); break;
    }
  } else {
    integral_constant<int, 1> one;
    switch (lanes_for(R)) {
      case 1: f(integral_constant<int, 1>(), one); break;
      case 2: f(integral_constant<int, 2>(), one); break;
      case 4: f(integral_constant<int, 4>(), one); break;
      case 8: f(integral_constant<int, 8>(), one); break;
      case 16: f(integral_constant<int, 16>(), one); break;
      case 32: f(integral_constant<int, 32>(), one); break;
      default: f(integral_constant<int, 64>(), one); break;
    }
  }
}

// A NaN counts for the scales in every component.
bool nan_counts_all(const fi_graph* g) { return g->dg.n <= kSmallDescentN && g->gl_nheavy == 0; }

hipError_t launch_rows(fi_graph* g, const float* gin, int R, const RowArgs& A, float* out,
                       hipStream_t s) {
  const Layout& L = g->L;
  const int32_t* first = (const int32_t*)(g->ws + L.glfirst);
  GLPlan plan;
  plan.heavy = (const int32_t*)(g->ws + L.glheavy);
  plan.items = (const int2*)(g->ws + L.glitems);
  plan.part = (float*)(g->ws + L.glpart);
  plan.mid = (const int32_t*)(g->ws + L.glmid);
  plan.nitems = (uint32_t)g->gl_nitems;
  plan.nmid = (uint32_t)g->gl_nmid;
  plan.mid_len = mid_len(g);
  constexpr int NW = kGLBlock / 64;
  with_lanes(R, (uintptr_t)gin % 16 == 0 && (uintptr_t)out % 16 == 0, [&](auto p, auto v) {
    constexpr int P = decltype(p)::value, V = decltype(v)::value;
    // (so that the blocks of a small graph have one kind of row each)
    const int64_t mid = (plan.nmid + NW - 1) / NW;
    const int grid = (int)std::min<int64_t>(plan.nitems + mid + pass_grid(g->dg.n, P), kGLPassBlocks);
    plan.mid_at = plan.nitems % grid;
    plan.short_at = (plan.nitems + mid) % grid;
    const auto pass = !A.max_in           ? k_gl_pass<P, V, false, false>
                      : nan_counts_all(g) ? k_gl_pass<P, V, true, true>
                                          : k_gl_pass<P, V, true, false>;
    hipLaunchKernelGGL(pass, dim3(grid), dim3(kGLBlock), 0, s, g->dg.row_ptr, g->dg.adj, g->dg.n, plan, gin,
                       R, A, out);
  });
  if (g->gl_nheavy == 0) return hipGetLastError();
  const uint32_t nheavy = (uint32_t)g->gl_nheavy, rows_per_block = kGLBlock / lanes_for(R);
  const int hgrid = (int)std::min<uint32_t>((nheavy + rows_per_block - 1) / rows_per_block, 4096);
  hipLaunchKernelGGL(k_gl_combine, dim3(hgrid), dim3(kGLBlock), 0, s, g->dg.row_ptr, plan.heavy, first,
                     nheavy, plan.part, gin, R, A, out);
  return hipGetLastError();
}

}  // namespace

// At graph upload: the rows longer than kGLHeavy and their items (blocks).
hipError_t graphl_setup(fi_graph* g, hipStream_t s) {
  const Layout& L = g->L;
  int32_t* list = (int32_t*)(g->ws + L.glheavy);
  int32_t* first = (int32_t*)(g->ws + L.glfirst);
  int2* items = (int2*)(g->ws + L.glitems);
  uint32_t* ctl = gl_ctl(g);
  hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(64), 0, s, ctl, (int64_t)4, 0u);
  if (g->dg.n > 0) {
    const int grid =
        (int)std::max<int64_t>(1, std::min<int64_t>(((int64_t)g->dg.n + 255) / 256, 16384));
    hipLaunchKernelGGL(k_gl_heavy_list, dim3(grid), dim3(256), 0, s, g->dg.row_ptr, g->dg.n, mid_len(g),
                       held_entries(small_rows(g->dg.n)), list, (int32_t*)(g->ws + L.glmid), ctl);
    hipLaunchKernelGGL(k_gl_plan, dim3(1), dim3(1024), 0, s, g->dg.row_ptr, list, ctl, first, items);
  }
  uint32_t cnt[4] = {0, 0, 0, 0};
  hipError_t e = hipMemcpyAsync(cnt, ctl, sizeof(cnt), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  g->gl_nheavy = (int32_t)cnt[0];
  g->gl_nitems = (int32_t)cnt[1];
  g->gl_nmid = (int32_t)cnt[2];
  g->gl_longer = cnt[3] != 0;
  return e == hipSuccess ? hipGetLastError() : e;
}

}  // namespace fi

using namespace fi;

#define FI_HIP(call)                              \
  do {                                            \
    if ((call) != hipSuccess) return FI_EDEVICE;  \
  } while (0)

extern "C" {

int fi_graphl_forward(fi_graph* g, const float* d_gamma, int32_t R, double* d_loss, void* stream) {
  if (!g || g->is_batch || R < 1 || R > kGraphLMaxR || !d_loss || (g->dg.n > 0 && !d_gamma))
    return FI_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  double* part = (double*)(g->ws + g->L.gl);
  int blocks = 0;
  with_lanes(R, (uintptr_t)d_gamma % 16 == 0, [&](auto p, auto v) {
    constexpr int P = decltype(p)::value, V = decltype(v)::value;
    constexpr int64_t per = (int64_t)(kGLBlock / P) * kFwdEdges;
    blocks = (int)std::min<int64_t>((g->dg.m + per - 1) / per, kGraphLBlocks);
    if (blocks > 0)
      hipLaunchKernelGGL((k_gl_forward<P, V>), dim3(blocks), dim3(kGLBlock), 0, s, g->dg.cedges,
                         g->dg.m, d_gamma, (int)R, part);
  });
  hipLaunchKernelGGL(k_gl_forward_final, dim3(R), dim3(kGLBlock), 0, s, part, blocks, d_loss);
  return hipGetLastError() == hipSuccess ? FI_OK : FI_EDEVICE;
}

int fi_graphl_backward(fi_graph* g, const float* d_gamma, int32_t R, const double* d_grad_loss,
                       float* d_grad_gamma, void* stream) {
  if (!g || g->is_batch || R < 1 || R > kGraphLMaxR) return FI_EINVAL;
  if (g->dg.n == 0) return FI_OK;
  if (!d_gamma || !d_grad_gamma) return FI_EINVAL;
  RowArgs A{};
  A.w = d_grad_loss;
  A.update = 0;
  return launch_rows(g, d_gamma, R, A, d_grad_gamma, (hipStream_t)stream) == hipSuccess ? FI_OK
                                                                                        : FI_EDEVICE;
}

int fi_graphl_step(fi_graph* g, const float* d_gamma_in, int32_t R, float alpha,
                   float* d_gamma_out, void* stream) {
  if (!g || g->is_batch || R < 1 || R > kGraphLMaxR) return FI_EINVAL;
  if (g->dg.n == 0) return FI_OK;
  if (!d_gamma_in || !d_gamma_out || d_gamma_in == d_gamma_out) return FI_EINVAL;
  RowArgs A{};
  A.alpha = alpha;
  A.update = 1;
  return launch_rows(g, d_gamma_in, R, A, d_gamma_out, (hipStream_t)stream) == hipSuccess
             ? FI_OK
             : FI_EDEVICE;
}

int fi_graphl_aux_size(fi_graph* g, int32_t R, size_t* out_bytes) {
  if (!g || g->is_batch || R < 1 || R > kGraphLMaxR || !out_bytes) return FI_EINVAL;
  *out_bytes = 4 * aux_part(g, R);
  return FI_OK;
}

}  // extern "C"

namespace {

template <int Q>
size_t small_lds(const fi_graph* g, int32_t ncomp) {
  return 2 * small_column(Q) + 16 * ((size_t)ncomp + (size_t)g->gl_nheavy);
}

// Whether a step of the fused descent, whose waves add the long rows' items one
// after the other, would take longer than launches of its own: per item 10.2 us
// in 256 groups, 5.8 in 128, 3.6 in 64 and 32, 4.7 in 16, against about 11 us a
// step (50 steps of stars, us: 2,360 vertices, R = 1 1,582 and 585, R = 8 880 and
// 483, R = 32 505 and 551; 1,200, R = 2 521 and 473, R = 3 310 and 433; 4,000, R = 16
// 724 and 497, R = 64 964 and 888).
bool long_rows_wait(const fi_graph* g, int32_t R, int groups) {
  if (g->gl_nheavy == 0) return false;
  const double items = (double)g->gl_nitems / std::min(16, g->gl_nheavy);
  return items * (0.04 * groups + 64.0 / groups) > 10.6 + 2.5e-5 * (double)R * g->dg.n;
}

// The fused descent, Q rows per thread (n <= 1024 Q).
template <int Q>
hipError_t descend_small(fi_graph* g, int32_t ncomp, int groups, int32_t R, float alpha, int64_t steps,
                         int32_t shift, const float* start, float* gamma, int32_t* exps, hipStream_t s) {
  const size_t lds = small_lds<Q>(g, ncomp);
  const auto f = g->gl_longer ? k_gl_descend_small<Q, true> : k_gl_descend_small<Q, false>;
  const hipError_t e = hipFuncSetAttribute((const void*)f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(f, dim3(R), dim3(1024), lds, s, g->dg.row_ptr, g->dg.adj, g->dg.comp,
                     (const int32_t*)(g->ws + g->L.aslot), g->dg.n, ncomp, g->gl_nheavy, groups, (int)R, alpha,
                     steps, (int)shift, g->gl_nheavy ? g->gl_main_slot : -1, start, gamma, exps);
  return hipGetLastError();
}

// The descent from `start` (d_gamma itself, or another buffer, which is only
// read) into d_gamma, with d_work as the other buffer.
int descend(fi_graph* g, const float* start, float* d_gamma, float* d_work, int32_t R, float alpha,
            int64_t steps, int32_t rescale_log2, void* d_aux, size_t aux_bytes, void* stream) {
  if (!g || g->is_batch || R < 1 || R > kGraphLMaxR || steps < 0) return FI_EINVAL;
  if (rescale_log2 == 0) rescale_log2 = 64;
  if (rescale_log2 < 1 || rescale_log2 > 100) return FI_EINVAL;
  const size_t part = aux_part(g, R);
  if (!d_aux || aux_bytes < 4 * part || ((uintptr_t)d_aux % 256)) return FI_EWORKSPACE;
  if (g->dg.n > 0 && (!start || !d_gamma || !d_work || d_gamma == d_work || start == d_work))
    return FI_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  char* aux = (char*)d_aux;
  // exponents and all three max buffers start at zero
  hipLaunchKernelGGL(k_fill_u32, dim3(256), dim3(256), 0, s, (uint32_t*)aux,
                     (int64_t)(part), 0u);
  const size_t bytes = sizeof(float) * (size_t)g->dg.n * R;
  if (g->dg.n > 0 && steps == 0 && start != d_gamma)
    FI_HIP(hipMemcpyAsync(d_gamma, start, bytes, hipMemcpyDeviceToDevice, s));
  if (g->dg.n == 0 || steps == 0) return hipGetLastError() == hipSuccess ? FI_OK : FI_EDEVICE;
  const int32_t ncomp = std::max<int32_t>(g->nanch, 1);
  int groups = 0;
  with_lanes(R, ((uintptr_t)start | (uintptr_t)d_gamma | (uintptr_t)d_work) % 16 == 0,
             [&](auto p, auto) { groups = kGLBlock / decltype(p)::value; });
  if (g->dg.n <= kSmallDescentN && g->dg.nnz <= (g->gl_nheavy ? kSmallEntries / 2 : kSmallEntries) &&
      small_lds<4>(g, ncomp) <= kSmallDescentLds && !long_rows_wait(g, R, groups)) {
    const int q = small_rows(g->dg.n);
    const auto f = q == 1 ? descend_small<1> : q == 2 ? descend_small<2> : descend_small<4>;
    return f(g, ncomp, groups, R, alpha, steps, rescale_log2, start, d_gamma, (int32_t*)aux, s) == hipSuccess
               ? FI_OK
               : FI_EDEVICE;
  }
  // steps alternate between the buffers; from another start the last one ends
  // in d_gamma, from d_gamma an odd number of steps ends in d_work
  const bool own = start == d_gamma;
  const float* in = start;
  for (int64_t k = 0; k < steps; ++k) {
    float* outb = own ? (k & 1 ? d_gamma : d_work) : ((steps - 1 - k) & 1 ? d_work : d_gamma);
    RowArgs A{};
    A.alpha = alpha;
    A.update = 1;
    A.comp = g->dg.comp;
    A.aslot = (const int32_t*)(g->ws + g->L.aslot);
    A.anchors = g->dg.anchors;
    A.exps = (int32_t*)aux;
    A.max_in = (const uint32_t*)(aux + (1 + k % 3) * part);
    A.max_out = (uint32_t*)(aux + (1 + (k + 1) % 3) * part);
    A.max_clear = (uint32_t*)(aux + (1 + (k + 2) % 3) * part);
    A.ncr = (int64_t)std::max<int32_t>(g->nanch, 1) * R;
    A.main_slot = g->gl_main_slot;
    A.shift = rescale_log2;
    if (launch_rows(g, in, R, A, outb, s) != hipSuccess) return FI_EDEVICE;
    in = outb;
  }
  if (in != d_gamma) FI_HIP(hipMemcpyAsync(d_gamma, in, bytes, hipMemcpyDeviceToDevice, s));
  return FI_OK;
}

}  // namespace

extern "C" {

int fi_graphl_descend(fi_graph* g, float* d_gamma, float* d_work, int32_t R, float alpha,
                      int64_t steps, int32_t rescale_log2, void* d_aux, size_t aux_bytes,
                      void* stream) {
  return descend(g, d_gamma, d_gamma, d_work, R, alpha, steps, rescale_log2, d_aux, aux_bytes, stream);
}

int fi_graphl_descend_from(fi_graph* g, const float* d_gamma0, float* d_gamma, float* d_work,
                           int32_t R, float alpha, int64_t steps, int32_t rescale_log2, void* d_aux,
                           size_t aux_bytes, void* stream) {
  if (d_gamma0 && d_gamma0 == d_gamma) return FI_EINVAL;
  return descend(g, d_gamma0, d_gamma, d_work, R, alpha, steps, rescale_log2, d_aux, aux_bytes, stream);
}

int fi_graphl_scales(fi_graph* g, const void* d_aux, int32_t R, int32_t* d_out, void* stream) {
  if (!g || g->is_batch || R < 1 || R > kGraphLMaxR || !d_aux || (g->dg.n > 0 && !d_out))
    return FI_EINVAL;
  if (g->dg.n == 0) return FI_OK;
  const int64_t total = (int64_t)g->dg.n * R;
  const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((total + 255) / 256, 65536));
  hipLaunchKernelGGL(k_gl_scales, dim3(grid), dim3(256), 0, (hipStream_t)stream, g->dg.row_ptr,
                     g->dg.comp, (const int32_t*)(g->ws + g->L.aslot), g->dg.n,
                     (const int32_t*)d_aux, (int)R, d_out);
  return hipGetLastError() == hipSuccess ? FI_OK : FI_EDEVICE;
}

int fi_round_count(fi_graph* g, const float* d_gamma, int32_t R, uint64_t* d_counts,
                   uint64_t* d_bits_out, void* stream) {
  if (!g || g->is_batch || R < 1 || R > kGraphLMaxR || !d_counts) return FI_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  if (g->dg.n == 0) {
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(128), 0, s, (uint32_t*)d_counts, (int64_t)2 * R, 0u);
    return hipGetLastError() == hipSuccess ? FI_OK : FI_EDEVICE;
  }
  if (!d_gamma) return FI_EINVAL;
  void* tok = nullptr;
  if (prof_begin(g, s, &tok)) return FI_EDEVICE;
  // rounded states, one word per vertex (4 bytes for up to 32 restarts, else
  // 8), in the scratch region (8 (n + 64) bytes)
  void* st = g->ws + g->L.scratch;
  const int64_t work = 64 % R == 0 ? (int64_t)g->dg.n * R : (int64_t)g->dg.n;
  const int ugrid = (int)std::max<int64_t>(1, std::min<int64_t>((g->dg.nwords + 3) / 4, 65536));
  // 16-byte reads when each vertex's R floats fill whole float4s
  const bool wide = R % 4 == 0 && 64 % R == 0 && ((uintptr_t)d_gamma & 15) == 0;
  const int wgrid = grid_for_gl(((int64_t)g->dg.n * R / 4 + 127) / 128 * 64, 256);
  if (R <= 32) {
    if (wide)
      hipLaunchKernelGGL(k_gl_round4<uint32_t>, dim3(wgrid), dim3(256), 0, s, (const float4*)d_gamma,
                         g->dg.n, (int)R, (uint32_t*)st, d_counts);
    else
      hipLaunchKernelGGL(k_gl_round<uint32_t>, dim3(grid_for_gl(work, 256)), dim3(256), 0, s, d_gamma,
                         g->dg.n, (int)R, (uint32_t*)st, d_counts);
    if (d_bits_out)
      hipLaunchKernelGGL(k_gl_unpack<uint32_t>, dim3(ugrid), dim3(256), 0, s, (const uint32_t*)st,
                         g->dg.n, g->dg.nwords, (int)R, d_bits_out);
  } else {
    if (wide)
      hipLaunchKernelGGL(k_gl_round4<uint64_t>, dim3(wgrid), dim3(256), 0, s, (const float4*)d_gamma,
                         g->dg.n, (int)R, (uint64_t*)st, d_counts);
    else
      hipLaunchKernelGGL(k_gl_round<uint64_t>, dim3(grid_for_gl(work, 256)), dim3(256), 0, s, d_gamma,
                         g->dg.n, (int)R, (uint64_t*)st, d_counts);
    if (d_bits_out)
      hipLaunchKernelGGL(k_gl_unpack<uint64_t>, dim3(ugrid), dim3(256), 0, s, (const uint64_t*)st,
                         g->dg.n, g->dg.nwords, (int)R, d_bits_out);
  }
  hipError_t e = launch_count(g->dg, st, R, (uint64_t*)(g->ws + g->L.cntpart), d_counts, s);
  prof_end(g, s, tok, 1);
  return e == hipSuccess ? FI_OK : FI_EDEVICE;
}

}  // extern "C"
