// Trees in LDS over a graph's edges: shared by the single-graph sweep
// (sweep_edges.hip) and the batched sweep of many graphs (batch.hip).
//
// A level of such a tree has little work and a long chain of dependent steps
// (queue entry, row bounds, a search for the row of each entry, the entry, its
// tree word), so the chain is cut instead of the work: every thread holds its
// share of the edge list in registers, two vertices and the sign to a word, and
// a level reads both ends' levels from LDS for each of them.  An edge counts in
// the one level where one end was reached last and the other is not, and the
// search ends with the last vertex reached.  1,000 trees of n = 1,000,
// m = 5,000: 47 us (through a queue of each level's vertices: 82), 100 of them 16
// (30); 760 of 4,709 / 16,129 105 (216), 300 of 10,000 / 80,000 238 (451).  110
// registers: with 24 edges held 96 and the same times, with 16 80 and 5 to 15% more.
// On a deep graph few edges lie in a level and all are looked at in each, so once
// the vertices left are more than kEFew levels like the last, a tree goes on
// through a queue, lanes spread over the frontier's rows (deep_levels).  100 trees
// of a 100 by 100 grid 195 us (over the edges to the end 496, through a queue alone
// 409), of a ring of 10,000 with 10 neighbours on either side 539 (7,760, 1,039).
// Edges past those in registers are read from memory at every level, so there the
// queue takes over as soon as the levels shrink and its rows, by the mean degree,
// are half of what the levels to come look at: 64 trees of 5,400 vertices of degree
// 40 beside a ring of 167 177 us (at the seventh level 495, through a queue alone 319).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fi_internal.h"
#include "fi_prims.h"
#include "fi_wg.h"

namespace fi {
namespace wg {

constexpr int kEHeld = 32;   // edges per thread in registers; the rest are read per level
constexpr int kEBatch = 8;   // edges in flight
constexpr uint32_t kEMask = 0x7FFF;   // a vertex as its byte offset in the 16-bit levels
constexpr int32_t kEMaxN = 1 << 14;
constexpr uint32_t kELast = 0xFFFF;   // level of a vertex not yet reached
// levels that go over the edges in any case (a random graph's largest level comes
// by then; the first 16 of the ring above take 140 us more than the first 6)
constexpr uint32_t kEDeep = 6;
constexpr int32_t kEFew = 16;

template <int NT>
struct EShared {
  uint64_t red[3][NT / 64];
  uint32_t found[3];  // vertices reached, by level modulo 3
};

__device__ __forceinline__ uint32_t pack_edge(uint2 e) {
  return 2 * e.x | (2 * (e.y & kVertexMask)) << 15 | (e.y & 0x80000000u);
}

// The levels after level L of a tree with `left` vertices to reach, through a
// queue in the place of the levels (16 bits a vertex too).  A word gets the
// number of the level in front of its parent key, those of vertices reached
// before 0, so that no later level changes it.  Each row of the frontier is
// read by as many lanes, a power of two up to 64, as the threads give it.
template <int NT>
__device__ __forceinline__ void deep_levels(const DevGraph& G, const KeyMix& km, uint32_t L, int32_t left,
                                            EShared<NT>& sh, uint64_t* pw, uint16_t* lev) {
  const int tid = threadIdx.x;
  for (int32_t v = tid; v < G.n; v += NT) {
    const uint64_t w = pw[v];
    if (w != ~0ull) pw[v] = (w & 1) | (uint64_t)(lev[v] == L) << 33;
  }
  __syncthreads();
  if (tid < 3) sh.found[tid] = 0;
  __syncthreads();
  uint16_t* q = lev;
  for (int32_t v = tid; v < G.n; v += NT)
    if (pw[v] >> 33 == 1) q[atomicAdd(&sh.found[0], 1u)] = (uint16_t)v;
  __syncthreads();
  uint32_t lo = 0, hi = sh.found[0];
  for (uint32_t k = 2; left > 0 && lo < hi; ++k) {
    uint32_t* found = &sh.found[(k - 1) % 3];
    int lg = 0;
    while (lg < 6 && (hi - lo) << (lg + 1) <= (uint32_t)NT) ++lg;
    const int32_t lane = tid & ((1 << lg) - 1);
    for (uint32_t i = lo + ((uint32_t)tid >> lg); i < hi; i += (uint32_t)NT >> lg) {
      const int32_t u = q[i];
      const int32_t e1 = G.row_ptr[u + 1];
      const uint64_t w0 = (uint64_t)k << 33 | (uint64_t)vkey(km, (uint32_t)u) << 1 | (pw[u] & 1);
      for (int32_t e = G.row_ptr[u] + lane; e < e1; e += 1 << lg) {
        const uint32_t a = G.adj[e], v = a & kVertexMask;
        const uint64_t w = w0 ^ (uint64_t)(a >> 31);
        if (pw[v] > w && amin64(pw + v, w) == ~0ull) q[hi + atomicAdd(found, 1u)] = (uint16_t)v;
      }
    }
    __syncthreads();
    const uint32_t f = *found;
    if (tid == 0) sh.found[(k + 1) % 3] = 0;
    lo = hi;
    hi += f;
    left -= (int32_t)f;
  }
}

// Trees t0, t0 + step, ... below t1 of G; `later`: its vertices that are not a
// root and have an edge; dyn: 10 n bytes.
template <int NT>
__device__ __forceinline__ void edges_trees(const DevGraph& G, const SweepArgs& A, uint64_t t0, uint64_t t1,
                                            uint64_t step, int32_t later, EShared<NT>& sh, uint64_t* dyn) {
  const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  const int32_t n = G.n, m = (int32_t)G.m;
  // a vertex's parent key << 1 | its state
  uint64_t* pw = dyn;
  uint16_t* lev = (uint16_t*)(dyn + n);
  auto level = [&](uint32_t at) { return (uint32_t) * (const uint16_t*)((const char*)lev + at); };

  uint32_t held[kEHeld];
#pragma unroll
  for (int k = 0; k < kEHeld; ++k) {
    const int32_t e = k * NT + tid;
    // (an edge from a vertex to itself counts nowhere)
    held[k] = e < m ? pack_edge(G.edges[e]) : 0u;
  }
  // f over the edges, kEBatch at a time
  auto edges = [&](auto f) {
#pragma unroll
    for (int k = 0; k < kEHeld; k += kEBatch) {
      if (k * NT >= m) break;
      uint32_t x[kEBatch];
#pragma unroll
      for (int j = 0; j < kEBatch; ++j) {
        x[j] = held[k + j];
        asm volatile("" : "+v"(x[j]));  // or the offsets in it are kept for every level
      }
      f(x);
    }
    for (int32_t e0 = kEHeld * NT; e0 < m; e0 += kEBatch * NT) {
      uint32_t x[kEBatch];
#pragma unroll
      for (int j = 0; j < kEBatch; ++j) {
        const int32_t e = e0 + j * NT + tid;
        x[j] = e < m ? pack_edge(G.edges[e]) : 0u;
      }
      f(x);
    }
  };

  for (uint64_t t = t0; t < t1; t += step) {
    const uint64_t salt = tree_salt(A.seed, t);
    // (the hybrid's other trees are randomized DFS)
    if (A.sampler == kSamplerHybrid && hybrid_coin(salt)) continue;
    const KeyMix km = key_mix(salt);
    // every vertex unreached, those without edges of state 0
    for (int32_t v = tid; v < n; v += NT) {
      lev[v] = (uint16_t)kELast;
      pw[v] = G.row_ptr[v + 1] > G.row_ptr[v] ? ~0ull : 0ull;
    }
    if (tid < 3) sh.found[tid] = 0;
    __syncthreads();
    // component roots: the minimum key, gathered in the anchor's word, one
    // atomic per wave where its vertices share a component
    for (int32_t v0 = 0; v0 < n; v0 += NT) {
      const int32_t v = v0 + tid;
      const bool in = v < n && G.row_ptr[min(v, n - 1) + 1] > G.row_ptr[min(v, n - 1)];
      const int32_t c = in ? G.comp[v] : -1;
      const uint32_t key = in ? vkey(km, (uint32_t)v) : ~0u;
      const uint64_t m_in = __ballot(in);
      if (m_in == 0) continue;
      const int32_t c0 = __builtin_amdgcn_readlane(c, __builtin_ctzll(m_in));
      if (__ballot(in && c != c0) == 0) {
        const uint32_t least = wave_reduce<false>(key, [](uint32_t a, uint32_t b) { return a < b ? a : b; });
        if (in && key == least) amin64(pw + c, (uint64_t)key << 32 | (uint32_t)v);
      } else if (in) {
        amin64(pw + c, (uint64_t)key << 32 | (uint32_t)v);
      }
    }
    __syncthreads();
    for (int32_t v = tid; v < n; v += NT) {
      if (G.comp[v] == v && G.row_ptr[v + 1] > G.row_ptr[v]) {
        const uint32_t r = (uint32_t)pw[v];
        pw[v] = ~0ull;
        pw[r] = 0;
        lev[r] = 0;
      }
    }
    __syncthreads();
    int32_t left = later, go = left;  // go: vertices left, or -1 of a deep tree
    int32_t last = 0;                 // vertices that the level before reached
    uint32_t L = 0;
    for (; go > 0; ++L) {
      uint32_t mine = 0;
      edges([&](const uint32_t* x) {
        uint32_t lu[kEBatch], lv[kEBatch];
#pragma unroll
        for (int j = 0; j < kEBatch; ++j) {
          lu[j] = level(x[j] & kEMask);
          lv[j] = level((x[j] >> 15) & kEMask);
        }
#pragma unroll
        for (int j = 0; j < kEBatch; ++j) {
          if (lu[j] != lv[j] && min(lu[j], lv[j]) == L) {
            const uint32_t a = x[j] & kEMask, b = (x[j] >> 15) & kEMask;
            const uint32_t from = lu[j] == L ? a : b, to = a ^ b ^ from;
            const uint32_t bit = (*(const uint32_t*)((const char*)pw + 4 * from) ^ (x[j] >> 31)) & 1u;
            const uint64_t w = (uint64_t)vkey(km, from >> 1) << 1 | bit;
            *(uint16_t*)((char*)lev + to) = (uint16_t)(L + 1);
            mine += amin64((uint64_t*)((char*)pw + 4 * to), w) == ~0ull;
          }
        }
      });
      const uint32_t found = wave_reduce<false>(mine, [](uint32_t a, uint32_t b) { return a + b; });
      if (lane == 0 && found) atomicAdd(&sh.found[L % 3], found);
      __syncthreads();
      const uint32_t f = sh.found[L % 3];
      if (tid == 0) sh.found[(L + 2) % 3] = 0;
      left -= (int32_t)f;
      const bool few = m > kEHeld * NT && (int32_t)f < last &&
                       4 * (int32_t)f * ((int32_t)f + left) < n * max((int32_t)f, left);
      go = left > 0 && (few || (L + 1 >= kEDeep && left > kEFew * (int32_t)f)) ? -1 : left;
      last = (int32_t)f;
    }
    if (go < 0) deep_levels<NT>(G, km, L, left, sh, pw, lev);

    // the states in place of the levels
    for (int32_t v = tid; v < n; v += NT) lev[v] = (uint16_t)(pw[v] & 1);
    __syncthreads();
    uint64_t khi = 0, klo = 0;
    uint32_t frustrated = 0;
    for (int32_t i = wave; i < G.nwords; i += NT / 64) {
      const int32_t v = i * 64 + lane;
      const uint64_t W = __ballot(v < n && (lev[min(v, n - 1)] ^ lev[G.comp[min(v, n - 1)]]));
      if (lane == 0) {
        key_terms((uint64_t)i, W, khi, klo);
        if (A.bits_out) A.bits_out[i] = W;
      }
    }
    edges([&](const uint32_t* x) {
#pragma unroll
      for (int j = 0; j < kEBatch; ++j)
        frustrated += (x[j] >> 31) ^ level(x[j] & kEMask) ^ level((x[j] >> 15) & kEMask);
    });
    const uint64_t S = wave_sum_u64(frustrated);
    khi = wave_sum_u64(khi);
    klo = wave_sum_u64(klo);
    if (lane == 0) {
      sh.red[0][wave] = khi;
      sh.red[1][wave] = klo;
      sh.red[2][wave] = S;
    }
    __syncthreads();
    if (tid == 0) {
      uint64_t sum[3] = {0, 0, 0};
      for (int i = 0; i < NT / 64; ++i)
        for (int k = 0; k < 3; ++k) sum[k] += sh.red[k][i];
      if (A.insert) cloud_insert(G, sum[0], sum[1], sum[2], t);
      if (A.tree_switches) A.tree_switches[t - A.t0] = sum[2];
    }
  }
}

}  // namespace wg
}  // namespace fi
