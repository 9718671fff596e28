// The tree samplers other than BFS (Section "Tree-Sampling techniques for
// graphBpp" and Alg. alg-hybrid), with all randomness from the tree's salt as
// for BFS: randomized DFS, one wave per tree, and Kruskal on random weights,
// one workgroup per tree.  Each builds a spanning forest and its vertex states,
// then counts, keys and inserts the tree as the BFS sweep does.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "fi_edges.h"
#include "fi_internal.h"
#include "fi_prims.h"
#include "fi_wg.h"

namespace fi {

namespace {

using wg::amin64;

// ------------------------------------------------------------ randomized DFS
// From the current vertex, move to the unvisited neighbour of smallest key
// (the shuffled adjacency order), back up when there is none; one search per
// component from its minimum-key vertex, until the component is visited.
//
// A search is one chain of dependent steps (row bounds, row, visited bits,
// minimum), so its time is the latency of a step, in loads and in instructions,
// and the trees run beside one another: a wave per tree, its marks in LDS, and
// the stack and the CSR there too while they fit; with the CSR in global memory
// a neighbour's row bounds come with its entry (links).  A hub is scanned again
// at every return to it, with four loads per lane in flight, eight in rows of more
// entries than those (a star of 99 leaves 124 us, with eight everywhere 144; of 999
// 2,000, with four 2,080; 20,000 / 100,000 with hubs, 64 trees 14.9 ms and 15.3 with
// eight).  Backing up looks
// at four stack entries at a time, and the search ends with the last vertex
// instead of unwinding.  Components are chains of their own, so while a CU has
// few trees, a tree's components go to several waves.  1,000 trees of n = 1,000,
// m = 5,000: 0.45 ms, that is 0.45 us a vertex (a workgroup per tree, its waves
// but one idle: 0.97); 4,000 / 16,000: 2.2 ms (7.6); 500 trees of 20,000 /
// 100,000: 15.7 (36.7).
struct RdfsArgs {
  const int32_t* cptr;    // [components + 1] ranges of cverts
  const int32_t* cverts;  // vertices by component
  const uint2* links;     // [nnz] entries with their neighbour's row, or null
  char* slots;            // per resident wave, what does not fit LDS
  size_t slot_stride;
  int share;              // waves to a tree, a power of two
  uint32_t cus;
  // with the hybrid's BFS trees in the same launch:
  int ntree;              // randomized DFS trees of a workgroup at a time
  uint32_t dfs;           // workgroups of them, the first ones; 0: each has one tree of either kind
  int32_t later;          // BFS in LDS: vertices that are not a root and have an edge
  char* bfs_slots;        // else per workgroup, words and queue
  size_t bfs_stride;
};

// 32-bit words of a wave's marks: two bits per vertex, visited and state.
__host__ __device__ constexpr int32_t mark_words(int32_t n) { return (n + 15) / 16; }
// and of its stack in LDS, of 16-bit vertices (so up to kStackMaxN of them)
__host__ __device__ constexpr int32_t stack_words(int32_t n) { return (n + 1) / 2; }
constexpr int32_t kStackMaxN = 1 << 16;
constexpr size_t kRdfsStatic = 64;  // LDS bytes beside the trees'
constexpr int kRdfsBatch = 4;  // loads of a long row in flight per lane
constexpr int kRdfsMore = 8;   // of a longer one than those
constexpr int kRdfsCount = 8;  // and of edges counted

// An adjacency entry together with its neighbour's row: x = vertex | its
// degree (kLinkLong for a longer row) << kLinkShift | negative << 31, y = first entry.
constexpr int kLinkShift = 20;
constexpr uint32_t kLinkLong = 0x7FF, kLinkVertex = (1u << kLinkShift) - 1;
constexpr int32_t kLinkMaxN = 1 << kLinkShift;

__global__ void k_rdfs_links(const int32_t* rp, const uint32_t* adj, int64_t nnz, uint2* links) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nnz;
       e += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t a = adj[e], v = a & kVertexMask;
    const int32_t r0 = rp[v];
    const uint32_t d = min((uint32_t)(rp[v + 1] - r0), kLinkLong);
    links[e] = make_uint2(v | d << kLinkShift | (a & 0x80000000u), (uint32_t)r0);
  }
}

// The least x over the wave, in every lane; with few, only lanes 0 .. 15 count.
__device__ __forceinline__ uint32_t least_key(uint32_t x, bool few) {
  auto least = [](uint32_t a, uint32_t b) { return a < b ? a : b; };
  if (!few) return wave_reduce<false>(x, least);
  x = least(x, dpp32<0xB1, 0xF>(x, x));
  x = least(x, dpp32<0x4E, 0xF>(x, x));
  x = least(x, dpp32<0x141, 0xF>(x, x));
  x = least(x, dpp32<0x140, 0xF>(x, x));
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

// CSR: the graph's row offsets and adjacency in LDS, once per workgroup; LINKS
// (without CSR): entries read with their neighbour's row; STK: the tree's stack
// in LDS; MARKS: its marks in LDS; SHARED (with MARKS): R.share waves to a tree.
// BFS: the workgroups past R.dfs, or with no such line those of a BFS tree, take the
// hybrid's other trees (all are of kBothThreads threads), so that neither kind waits for the other (a path of 13,000, 100 trees
// 32.7 ms in two launches, 27.3 here; of 2,000 2,020 us and 1,230; 50 / 100, 500 trees
// 69 and 53).
constexpr int kBothThreads = 256;
enum : int { kNoBfs = 0, kBfsLds = 1, kBfsSlots = 2 };

template <bool CSR, bool LINKS, bool STK, bool MARKS, bool SHARED, int BFS>
__global__ void __launch_bounds__(BFS ? kBothThreads : 1024) k_sweep_rdfs(DevGraph G, SweepArgs A, RdfsArgs R) {
  extern __shared__ __align__(16) uint32_t sm[];
  if constexpr (BFS != kNoBfs) {
    const bool own = R.dfs == 0;  // a tree per workgroup, of either kind
    if (own ? A.t0 + blockIdx.x < A.t1 && !wg::hybrid_coin(tree_salt(A.seed, A.t0 + blockIdx.x))
            : blockIdx.x >= R.dfs) {
      const uint32_t b = blockIdx.x - R.dfs, step = gridDim.x - R.dfs;
      if constexpr (BFS == kBfsLds) {
        __shared__ wg::EShared<kBothThreads> sh;
        wg::edges_trees<kBothThreads>(G, A, A.t0 + b, A.t1, step, R.later, sh, (uint64_t*)sm);
      } else {
        __shared__ wg::WgShared<kBothThreads> sh;
        uint64_t* pw = (uint64_t*)(R.bfs_slots + (size_t)b * R.bfs_stride);
        for (uint64_t t = A.t0 + b; t < A.t1; t += step)
          if (!wg::hybrid_coin(tree_salt(A.seed, t)))
            wg::wg_tree<kBothThreads>(G, A, t, pw, (int32_t*)(pw + G.n), sh);
      }
      return;
    }
  }
  const uint32_t blocks = BFS && R.dfs ? R.dfs : gridDim.x;
  __shared__ uint32_t s_next[kRdfsStatic / 4];  // per tree of the workgroup: components handed out
  // the wave's tree among the workgroup's `ntree`, and which of the tree's waves
  // it is: the first takes the first component, mostly the longest, so those of
  // the trees on a CU lie on different SIMDs
  const int lane = lane_id(), wave = threadIdx.x >> 6, nwv = blockDim.x >> 6;
  const int share = SHARED ? R.share : 1, ntree = SHARED ? nwv / share : BFS ? R.ntree : nwv;
  const int tree = SHARED ? wave % ntree : wave;
  const int part = SHARED ? (int)(wave / ntree + blockIdx.x / R.cus) % share : 0;
  const int32_t n = G.n, mw = mark_words(n);
  const int32_t* rp = G.row_ptr;
  const uint32_t* adj = G.adj;
  uint32_t* at = sm;
  if constexpr (CSR) {
    for (int32_t i = threadIdx.x; i <= n; i += blockDim.x) at[i] = (uint32_t)G.row_ptr[i];
    for (int64_t e = threadIdx.x; e < G.nnz; e += blockDim.x) at[n + 1 + e] = G.adj[e];
    rp = (const int32_t*)at;
    adj = at + n + 1;
    at += n + 1 + G.nnz;
    __syncthreads();
  }
  if (BFS && !SHARED && wave >= ntree) return;
  char* slot = R.slots + ((size_t)blockIdx.x * ntree + tree) * R.slot_stride;
  uint32_t* mark;
  std::conditional_t<STK, uint16_t, int32_t>* stk;
  {
    uint32_t* mine = at + (size_t)tree * ((MARKS ? mw : 0) + (STK ? stack_words(n) : 0));
    if constexpr (MARKS) mark = mine;
    else mark = (uint32_t*)slot;
    if constexpr (STK) stk = (uint16_t*)(mine + (MARKS ? mw : 0));
    else stk = (int32_t*)(slot + (MARKS ? 0 : 4 * (size_t)mw));
  }
  // the wave's own writes, before its next reads of them: a wave's LDS
  // operations stay in order, its global ones are waited for
  auto order = [](bool in_lds) {
    if (in_lds) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    else __threadfence_block();
  };
  auto visited = [&](int32_t v) { return (mark[v >> 4] >> (2 * (v & 15))) & 1u; };
  auto state = [&](int32_t v) { return (mark[v >> 4] >> (2 * (v & 15) + 1)) & 1u; };
  auto visit = [&](int32_t v, uint32_t b) {  // by one lane; no other writer
    const uint32_t m = (1u | b << 1) << (2 * (v & 15));
    if constexpr (MARKS) atomicOr(&mark[v >> 4], m);
    else mark[v >> 4] |= m;
  };
  const int32_t ncomp = (int32_t)G.ctl[C_NANCH];

  // between the waves of a tree (the trees of a workgroup go in step then)
  auto together = [&] {
    if constexpr (SHARED) __syncthreads();
    else order(MARKS);
  };
  const uint64_t first = A.t0 + (SHARED ? 0ull : (uint64_t)wave * blocks) + blockIdx.x;
  for (uint64_t t0 = first; t0 < A.t1; t0 += (uint64_t)ntree * blocks) {
    const uint64_t t = t0 + (SHARED ? (uint64_t)tree * blocks : 0ull);
    const uint64_t salt = tree_salt(A.seed, t);
    const bool bfs = A.sampler == kSamplerHybrid && !wg::hybrid_coin(salt);  // not this kind
    if (!SHARED && bfs) continue;
    const bool live = !SHARED || (t < A.t1 && !bfs);
    const KeyMix km = key_mix(salt);
    for (int32_t i = part * 64 + lane; i < mw; i += 64 * share) mark[i] = 0;
    if (SHARED && part == 0 && lane == 0) s_next[tree] = (uint32_t)share;
    together();
    auto draw = [&] {  // the wave's next component
      uint32_t x = 0;
      if (lane == 0) x = atomicAdd(&s_next[tree], 1u);
      return __builtin_amdgcn_readfirstlane((int)x);
    };
    for (int32_t k = SHARED ? (live ? __builtin_amdgcn_readfirstlane(part) : ncomp) : 0; k < ncomp;
         k = SHARED ? draw() : k + 1) {
      const int32_t b = R.cptr[k], e = R.cptr[k + 1];
      auto* stack = SHARED ? stk + b : stk;  // a component's part of it
      // the component's minimum-key vertex
      uint32_t bk = ~0u;
      int32_t bv = -1;
      for (int32_t i = b + lane; i < e; i += 64) {
        const int32_t v = R.cverts[i];
        const uint32_t key = vkey(km, (uint32_t)v);
        if (bv < 0 || key < bk) {
          bk = key;
          bv = v;
        }
      }
      uint32_t kmin = least_key(bk, false);
      int32_t u = __builtin_amdgcn_readlane(bv, __builtin_ctzll(__ballot(bv >= 0 && bk == kmin)));
      // the current vertex's row, its state, its place on the stack
      int32_t e0 = __builtin_amdgcn_readfirstlane(rp[u]);
      int32_t d = __builtin_amdgcn_readfirstlane(rp[u + 1]) - e0;
      uint32_t bu = 0;
      int32_t top = 0, left = e - b - 1;
      if (lane == 0) {
        visit(u, 0);
        stack[0] = (std::remove_reference_t<decltype(*stk)>)u;
      }
      order(MARKS);
      while (left > 0) {
        bool found = false;
        uint32_t neg = 0;
        // (the hint: without it 1,000 trees of n = 1,000 take 499 us, with it 473)
        if (__builtin_expect(d <= 64, 1)) {
          // (lanes past the row repeat its last entry)
          const int32_t at_e = e0 + min(lane, d - 1);
          uint32_t a, next = 0;
          if constexpr (LINKS) {
            const uint2 l = R.links[at_e];
            a = l.x;
            next = l.y;
          } else {
            a = adj[at_e];
          }
          const int32_t v = (int32_t)(a & (LINKS ? kLinkVertex : kVertexMask));
          const uint32_t key = vkey(km, (uint32_t)v);
          const bool open = !visited(v);
          const uint64_t m = __ballot(open);
          if (m) {
            // the keys of one row's neighbours are distinct
            kmin = least_key(open ? key : ~0u, d <= 16);
            const int wl = __builtin_ctzll(__ballot(key == kmin) & m);
            const uint32_t aw = (uint32_t)__builtin_amdgcn_readlane((int)a, wl);
            found = true;
            neg = aw >> 31;
            u = (int32_t)(aw & (LINKS ? kLinkVertex : kVertexMask));
            if constexpr (LINKS) {
              e0 = __builtin_amdgcn_readlane((int)next, wl);
              d = (int32_t)((aw >> kLinkShift) & kLinkLong);
              if (d == (int32_t)kLinkLong) d = __builtin_amdgcn_readfirstlane(rp[u + 1]) - e0;
            }
          }
        } else {
          uint32_t ck = ~0u, ca = 0;
          bool has = false;
          if (d <= 64 * kRdfsBatch) {
            for (int32_t c = lane; c - lane < d; c += 64 * kRdfsBatch) {
              uint32_t a[kRdfsBatch], w[kRdfsBatch];
#pragma unroll
              for (int q = 0; q < kRdfsBatch; ++q) a[q] = adj[e0 + min(c + 64 * q, d - 1)];
#pragma unroll
              for (int q = 0; q < kRdfsBatch; ++q) w[q] = visited((int32_t)(a[q] & kVertexMask));
#pragma unroll
              for (int q = 0; q < kRdfsBatch; ++q) {
                const uint32_t key = vkey(km, a[q] & kVertexMask);
                if (!w[q] && (!has || key < ck)) {
                  ck = key;
                  ca = a[q];
                  has = true;
                }
              }
            }
          } else {
            for (int32_t c = lane; c - lane < d; c += 64 * kRdfsMore) {
              uint32_t a[kRdfsMore], w[kRdfsMore];
#pragma unroll
              for (int q = 0; q < kRdfsMore; ++q) a[q] = adj[e0 + min(c + 64 * q, d - 1)];
#pragma unroll
              for (int q = 0; q < kRdfsMore; ++q) w[q] = visited((int32_t)(a[q] & kVertexMask));
#pragma unroll
              for (int q = 0; q < kRdfsMore; ++q) {
                const uint32_t key = vkey(km, a[q] & kVertexMask);
                if (!w[q] && (!has || key < ck)) {
                  ck = key;
                  ca = a[q];
                  has = true;
                }
              }
            }
          }
          const uint64_t m = __ballot(has);
          if (m) {
            kmin = least_key(ck, false);
            const uint32_t aw =
                (uint32_t)__builtin_amdgcn_readlane((int)ca, __builtin_ctzll(__ballot(ck == kmin) & m));
            found = true;
            neg = aw >> 31;
            u = (int32_t)(aw & kVertexMask);
            if constexpr (LINKS) {
              e0 = __builtin_amdgcn_readfirstlane(rp[u]);
              d = __builtin_amdgcn_readfirstlane(rp[u + 1]) - e0;
            }
          }
        }
        if (found) {
          if constexpr (!LINKS) {
            e0 = __builtin_amdgcn_readfirstlane(rp[u]);
            d = __builtin_amdgcn_readfirstlane(rp[u + 1]) - e0;
          }
          bu ^= neg;
          ++top;
          --left;
          if (lane == 0) {
            visit(u, bu);
            stack[top] = (std::remove_reference_t<decltype(*stk)>)u;
          }
          order(MARKS);
          continue;
        }
        // back up to the nearest of the entries below that may have an
        // unvisited neighbour: four at a time, 16 lanes each (a longer row
        // counts as one that may)
        order(STK);
        const int grp = lane >> 4, sub = lane & 15;
        while (true) {
          const int32_t i = top - 1 - grp;
          const int32_t w = i >= 0 ? (int32_t)stack[i] : 0;
          const int32_t f0 = rp[w], dw = rp[w + 1] - f0;
          bool may = false;
          if (i >= 0) {
            may = dw > 16 || (sub < dw && !visited((int32_t)(adj[f0 + min(sub, dw - 1)] & kVertexMask)));
          }
          const uint64_t m = __ballot(may);
          if (m) {
            const int g0 = __builtin_ctzll(m) >> 4;
            top -= 1 + g0;
            u = __builtin_amdgcn_readlane(w, 16 * g0);
            e0 = __builtin_amdgcn_readlane(f0, 16 * g0);
            d = __builtin_amdgcn_readlane(dw, 16 * g0);
            break;
          }
          top -= 4;
          if (top <= 0) {  // (a connected component never runs out)
            left = 0;
            break;
          }
        }
        bu = (uint32_t)__builtin_amdgcn_readfirstlane((int)state(u));
      }
    }

    together();

    // ---- canonical words, key terms and the exact count (its first wave)
    if (part == 0 && live) {
      uint64_t khi = 0, klo = 0, S = 0, mine = 0;
      for (int32_t i = 0; i < G.nwords; ++i) {
        const int32_t v = i * 64 + lane;
        const uint64_t W = __ballot(v < n && (state(min(v, n - 1)) ^ state(G.comp[min(v, n - 1)])));
        if (lane == (i & 63)) mine = W;
        if (lane == 0 && A.bits_out) A.bits_out[i] = W;
        if ((i & 63) == 63 || i + 1 == G.nwords) {  // a word per lane
          const int32_t i0 = i & ~63;
          if (i0 + lane <= i) key_terms((uint64_t)(i0 + lane), mine, khi, klo);
        }
      }
      for (int64_t b0 = 0; b0 < G.m; b0 += 64 * kRdfsCount) {
        uint2 uv[kRdfsCount];
#pragma unroll
        for (int q = 0; q < kRdfsCount; ++q) {
          const int64_t e = b0 + 64 * q + lane;
          uv[q] = e < G.m ? G.edges[e] : make_uint2(0u, 0u);  // (0, 0) is never frustrated
        }
#pragma unroll
        for (int q = 0; q < kRdfsCount; ++q)
          S += (uv[q].y >> 31) ^ state((int32_t)uv[q].x) ^ state((int32_t)(uv[q].y & kVertexMask));
      }
      S = wave_sum_u64(S);
      khi = wave_sum_u64(khi);
      klo = wave_sum_u64(klo);
      if (lane == 0) {
        if (A.insert) cloud_insert(G, khi, klo, S, t);
        if (A.tree_switches) A.tree_switches[t - A.t0] = S;
      }
    }
    together();
  }
}

template <bool CSR, bool LINKS, bool STK, bool MARKS, bool SHARED>
hipError_t rdfs_run(fi_graph* g, const SweepArgs& a, const RdfsArgs& r, int trees_per_wg, size_t lds,
                       size_t slots, hipStream_t s) {
  const int waves = trees_per_wg * r.share;
  const void* f = (const void*)k_sweep_rdfs<CSR, LINKS, STK, MARKS, SHARED, kNoBfs>;
  hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_sweep_rdfs<CSR, LINKS, STK, MARKS, SHARED, kNoBfs>,
                                                   64 * waves, lds);
  if (e != hipSuccess) return e;
  int64_t grid = (int64_t)std::max(1, per_cu) * g->cu_count;
  if (g->sched.grid > 0) grid = std::min<int64_t>(grid, g->sched.grid);
  if (!(STK && MARKS)) grid = std::min<int64_t>(grid, (int64_t)slots / trees_per_wg);
  const uint64_t trees = a.t1 - a.t0;
  grid = std::min<int64_t>(grid, (int64_t)((trees + trees_per_wg - 1) / trees_per_wg));
  hipLaunchKernelGGL((k_sweep_rdfs<CSR, LINKS, STK, MARKS, SHARED, kNoBfs>),
                     dim3((unsigned)std::max<int64_t>(grid, 1)), dim3(64 * waves), lds, s, g->dg, a, r);
  return hipGetLastError();
}

// Both kinds of the hybrid's trees in one launch, while its workgroups are resident
// at once (half of the BFS trees' find none); *both: whether it was made.
template <bool CSR, bool LINKS, bool STK, bool MARKS, bool SHARED, int BFS>
hipError_t both_run(fi_graph* g, const SweepArgs& a, RdfsArgs r, size_t lds, size_t region, bool* both,
                    hipStream_t s) {
  const auto f = k_sweep_rdfs<CSR, LINKS, STK, MARKS, SHARED, BFS>;
  const size_t fixed =
      kRdfsStatic + (BFS == kBfsLds ? sizeof(wg::EShared<kBothThreads>) : sizeof(wg::WgShared<kBothThreads>));
  if (BFS == kBfsLds) lds = std::max(lds, 10 * (size_t)g->dg.n);
  if (lds + fixed + 64 > (size_t)g->max_shared) return hipSuccess;
  hipError_t e = hipFuncSetAttribute((const void*)f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, kBothThreads, lds);
  if (e != hipSuccess) return e;
  const uint64_t trees = a.t1 - a.t0, dfs = (trees + r.ntree - 1) / r.ntree;
  const bool own = r.ntree == 1;
  if (own ? trees > (uint64_t)per_cu * g->cu_count : 2 * dfs + trees > 2 * (uint64_t)per_cu * g->cu_count)
    return hipSuccess;
  const size_t used = STK && MARKS ? 0 : dfs * r.ntree * r.slot_stride;
  if (BFS == kBfsSlots) {
    if (used > region || (region - used) / g->L.slot_stride < trees) return hipSuccess;
    r.bfs_slots = r.slots + used;
    r.bfs_stride = g->L.slot_stride;
  } else if (used) {
    return hipSuccess;
  }
  r.dfs = own ? 0 : (uint32_t)dfs;
  r.later = g->dg.n - g->nisolated - g->nanch;
  hipLaunchKernelGGL(f, dim3((unsigned)(r.dfs + trees)), dim3(kBothThreads), lds, s, g->dg, a, r);
  *both = true;
  return hipGetLastError();
}

// both: null, or where to say that the hybrid's BFS trees were launched with them
template <bool CSR, bool LINKS, bool STK, bool MARKS>
hipError_t rdfs_launch(fi_graph* g, const SweepArgs& a, const RdfsArgs& r, int path, int trees_per_wg, size_t lds,
                       size_t region, bool* both, hipStream_t s) {
  if constexpr (CSR || LINKS) {
    if (both) {
      constexpr int kWaves = kBothThreads / 64;
      RdfsArgs b = r;
      b.ntree = r.share > 1 ? kWaves / r.share : CSR ? std::min(kWaves, trees_per_wg) : 1;
      const size_t tree = 4 * ((MARKS ? (size_t)mark_words(g->dg.n) : 0) + (STK ? (size_t)stack_words(g->dg.n) : 0));
      const size_t blds = lds - tree * trees_per_wg + tree * b.ntree;
      auto run = [&](auto kind) -> hipError_t {
        constexpr int BFS = decltype(kind)::value;
        if constexpr (MARKS)
          if (r.share > 1) return both_run<CSR, LINKS, STK, MARKS, true, BFS>(g, a, b, blds, region, both, s);
        return both_run<CSR, LINKS, STK, MARKS, false, BFS>(g, a, b, blds, region, both, s);
      };
      hipError_t e = hipSuccess;
      if (path == 2) e = run(std::integral_constant<int, kBfsSlots>{});
      else if constexpr (STK && MARKS) e = run(std::integral_constant<int, kBfsLds>{});
      if (e != hipSuccess || *both) return e;
    }
  }
  const size_t slots = r.slot_stride ? region / r.slot_stride : 0;
  if constexpr (MARKS)
    if (r.share > 1) return rdfs_run<CSR, LINKS, STK, MARKS, true>(g, a, r, trees_per_wg, lds, slots, s);
  return rdfs_run<CSR, LINKS, STK, MARKS, false>(g, a, r, trees_per_wg, lds, slots, s);
}

// ------------------------------------------------------------ Kruskal
// Kruskal on random edge weights, as Boruvka rounds: each tree of the forest
// takes its lightest outgoing edge (weight, then position in the edge list:
// a strict order, so the result is the unique minimum spanning forest, the
// one Kruskal's algorithm builds) and hooks onto the tree across it; when
// two trees take the same edge, the larger root hooks.  q[v] = parent | parity
// << 31 (a union-find whose parity is v's state relative to its parent),
// flattened after every round so that every vertex points at its root.
//
// Rounds over all the edges are rounds over mostly useless ones, so the
// lightest come first: the edges below a weight that about n of them lie
// below are listed, and rounds over that list build the forest Kruskal's
// algorithm has when it reaches that weight; of the others only those that
// then join two trees are listed for the rest.  An edge's weight is formed
// when the lists are and in the rounds that still hold it, q lies in LDS while
// it fits, and a round touches the roots left, not all vertices.
// 500 trees of 20,000 vertices, 100,000 edges: 2.0 ms (rounds over all edges
// in 256 threads: 4.95); 512 of 100,000 / 500,000: 22.3 (37.4).
struct KruskalArgs {
  char* slots;         // per workgroup: what does not lie in LDS
  size_t slot_stride;
  uint32_t cap;        // entries of a list
  uint32_t tau;        // weight that parts the two lists (0: all edges at once)
};

__device__ __forceinline__ uint32_t kruskal_weight(uint64_t salt, uint32_t u, uint32_t v) {
  return (uint32_t)(mix64(salt ^ ((uint64_t)u << 32 | v)) >> 32);
}

template <int NT>
struct KShared {
  uint64_t red[NT / 64];
  uint32_t count, next, hooked;
};

// edges per thread in flight (with the trees in LDS, 1,000 of 8,000 / 40,000 476 us
// with four, 510 with two; else 500 of 20,000 / 100,000 1,996 and 1,933)
constexpr int k_batch(int mode) { return mode == 0 ? 4 : 2; }

// MODE 0: lightest edges and forest in LDS, a round touches every vertex; 1:
// the forest in LDS; 2: none.
template <int NT, int MODE>
__global__ void __launch_bounds__(NT) k_sweep_kruskal(DevGraph G, SweepArgs A, KruskalArgs K) {
  constexpr uint32_t kPar = 0x80000000u, kPtr = 0x7FFFFFFFu;
  constexpr int kKBatch = k_batch(MODE);
  __shared__ KShared<NT> sh;
  extern __shared__ uint64_t dyn[];
  const int tid = threadIdx.x;
  const int32_t n = G.n;
  // [n] a root's lightest outgoing edge (weight << 32 | edge); once it is
  // found, what the root decides in place of the weight
  uint64_t* pw;
  uint32_t* q;               // [n] the forest
  int32_t* root = nullptr;   // [n] the roots left (MODE 0: all vertices)
  int32_t* left = nullptr;   // [n] those that stay
  uint32_t* list = nullptr;  // [cap]
  if constexpr (MODE == 0) {
    pw = dyn;
    q = (uint32_t*)(dyn + n);
  } else {
    pw = (uint64_t*)(K.slots + (size_t)blockIdx.x * K.slot_stride);
    root = (int32_t*)(pw + n);
    left = root + n;
    list = (uint32_t*)(left + n);
    if constexpr (MODE == 1) q = (uint32_t*)dyn;
    else q = list + K.cap;
  }
  auto root_at = [&](uint32_t i) { return MODE == 0 ? i : (uint32_t)root[i]; };
  auto edge_of = [&](uint32_t r) { return ((uint32_t*)pw)[2 * (size_t)r]; };
  auto decided = [&](uint32_t r) -> uint32_t& { return ((uint32_t*)pw)[2 * (size_t)r + 1]; };

  for (uint64_t t = A.t0 + blockIdx.x; t < A.t1; t += gridDim.x) {
    const uint64_t salt = tree_salt(A.seed, t);
    if (tid == 0) sh.count = 0;
    __syncthreads();
    for (int32_t v0 = 0; v0 < n; v0 += NT) {
      const int32_t v = v0 + tid;
      if (v < n) q[v] = (uint32_t)v;
      if constexpr (MODE != 0)
        wave_append(v < n && G.row_ptr[min(v, n - 1) + 1] > G.row_ptr[min(v, n - 1)], v, root, &sh.count);
    }
    __syncthreads();
    uint32_t nroot = MODE == 0 ? (uint32_t)n : sh.count;
    __syncthreads();  // make_list counts in the same word

    // f(k, e, uv) for the kKBatch edges of each thread at a time: list entries
    // or, without a list, all the edges (a thread past the end has e < 0)
    auto batches = [&](const uint32_t* from, int64_t len, auto f) {
      for (int64_t b = 0; b < len; b += (int64_t)kKBatch * NT) {
        int64_t e[kKBatch];
        uint2 uv[kKBatch];
#pragma unroll
        for (int k = 0; k < kKBatch; ++k) {
          const int64_t i = b + (int64_t)k * NT + tid;
          e[k] = i < len ? (from ? (int64_t)from[i] : i) : -1;
        }
#pragma unroll
        for (int k = 0; k < kKBatch; ++k) uv[k] = G.edges[e[k] < 0 ? 0 : e[k]];
        f(e, uv);
      }
    };
    // Boruvka rounds over the edges until no tree finds one that leaves it
    auto rounds = [&](const uint32_t* from, int64_t len) {
      while (true) {
        for (uint32_t i = tid; i < nroot; i += NT) pw[root_at(i)] = ~0ull;
        if (tid == 0) {
          sh.next = 0;
          sh.hooked = 0;
        }
        __syncthreads();
        batches(from, len, [&](const int64_t* e, const uint2* uv) {
          uint32_t ru[kKBatch], rv[kKBatch];
          uint64_t key[kKBatch], pu[kKBatch], pv[kKBatch];
#pragma unroll
          for (int k = 0; k < kKBatch; ++k) {
            ru[k] = q[uv[k].x] & kPtr;
            rv[k] = q[uv[k].y & kVertexMask] & kPtr;
          }
          // (in the last rounds most edges lie inside a tree)
          bool any = false;
#pragma unroll
          for (int k = 0; k < kKBatch; ++k) any |= e[k] >= 0 && ru[k] != rv[k];
          if (!__ballot(any)) return;
#pragma unroll
          for (int k = 0; k < kKBatch; ++k) {
            const bool out = e[k] >= 0 && ru[k] != rv[k];
            key[k] = (uint64_t)kruskal_weight(salt, uv[k].x, uv[k].y & kVertexMask) << 32 | (uint64_t)e[k];
            pu[k] = out ? pw[ru[k]] : 0ull;
            pv[k] = out ? pw[rv[k]] : 0ull;
          }
#pragma unroll
          for (int k = 0; k < kKBatch; ++k) {
            if (pu[k] > key[k]) amin64(pw + ru[k], key[k]);
            if (pv[k] > key[k]) amin64(pw + rv[k], key[k]);
          }
        });
        __syncthreads();
        // decide every hook before any is made (q and pw's edges stay unchanged
        // here); the roots that stay go into the other list
        for (uint32_t i0 = 0; i0 < nroot; i0 += kKBatch * NT) {
          uint32_t r[kKBatch], e[kKBatch], other[kKBatch], h[kKBatch], eo[kKBatch];
          uint2 uv[kKBatch];
#pragma unroll
          for (int k = 0; k < kKBatch; ++k) {
            const uint32_t i = i0 + k * NT + tid;
            r[k] = i < nroot ? root_at(i) : 0u;
          }
#pragma unroll
          for (int k = 0; k < kKBatch; ++k) e[k] = i0 + k * NT + tid < nroot ? edge_of(r[k]) : ~0u;
          if constexpr (MODE == 0) {  // (and most vertices are no roots)
            bool any = false;
#pragma unroll
            for (int k = 0; k < kKBatch; ++k) any |= e[k] != ~0u;
            if (!__ballot(any)) {
#pragma unroll
              for (int k = 0; k < kKBatch; ++k)
                if (i0 + k * NT + tid < nroot) decided(r[k]) = ~0u;
              continue;
            }
          }
#pragma unroll
          for (int k = 0; k < kKBatch; ++k)
            uv[k] = e[k] != ~0u ? G.edges[e[k]] : make_uint2(0u, 0u);
#pragma unroll
          for (int k = 0; k < kKBatch; ++k) {
            const uint32_t qu = q[uv[k].x], qv = q[uv[k].y & kVertexMask];
            other[k] = (qu & kPtr) == r[k] ? (qv & kPtr) : (qu & kPtr);
            // parity(r -> other) = parity(u) ^ parity(v) ^ [edge negative]
            h[k] = other[k] | ((qu ^ qv ^ uv[k].y) & kPar);
          }
#pragma unroll
          for (int k = 0; k < kKBatch; ++k) eo[k] = e[k] != ~0u ? edge_of(other[k]) : ~0u;
#pragma unroll
          for (int k = 0; k < kKBatch; ++k) {
            const uint32_t i = i0 + k * NT + tid;
            const bool hooks = e[k] != ~0u && (eo[k] != e[k] || r[k] > other[k]);
            if (i < nroot) decided(r[k]) = hooks ? h[k] : ~0u;
            if (hooks) sh.hooked = 1;
            if constexpr (MODE != 0) wave_append(i < nroot && !hooks, (int32_t)r[k], left, &sh.next);
          }
        }
        __syncthreads();
        const bool any = sh.hooked != 0;
        const uint32_t stay = sh.next;
        for (uint32_t i = tid; i < nroot; i += NT) {
          const uint32_t r = root_at(i), h = decided(r);
          if (h != ~0u) q[r] = h;
        }
        if constexpr (MODE != 0) {
          nroot = stay;
          int32_t* swap = root;
          root = left;
          left = swap;
        }
        __syncthreads();
        if (!any) break;
        // every vertex follows its chain to the root; a word read along the
        // way is its vertex's old parent or already its root, with the parity
        // that goes with it
        for (int32_t v = tid; v < n; v += NT) {
          uint32_t x = q[v];
          while (true) {
            const uint32_t y = q[x & kPtr];
            if ((y & kPtr) == (x & kPtr)) break;
            x = (y & kPtr) | ((x ^ y) & kPar);
          }
          q[v] = x;
        }
        __syncthreads();
      }
    };
    // the edges of weight < tau (heavy: of weight >= tau that join two trees);
    // false if they do not fit the list
    uint32_t listed = 0;
    auto make_list = [&](bool heavy) {
      if (tid == 0) sh.count = 0;
      __syncthreads();
      batches(nullptr, G.m, [&](const int64_t* e, const uint2* uv) {
#pragma unroll
        for (int k = 0; k < kKBatch; ++k) {
          const uint32_t u = uv[k].x, v = uv[k].y & kVertexMask;
          bool in = e[k] >= 0 && (kruskal_weight(salt, u, v) < K.tau) != heavy;
          if (heavy && in) in = (q[u] & kPtr) != (q[v] & kPtr);
          const uint64_t m = __ballot(in);
          if (m) {
            uint32_t base = 0;
            if (lane_id() == 0) base = atomicAdd(&sh.count, (uint32_t)__popcll(m));
            base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base) + lanes_below(m);
            if (in && base < K.cap) list[base] = (uint32_t)e[k];
          }
        }
      });
      __syncthreads();
      listed = sh.count;
      __syncthreads();
      return listed <= K.cap;
    };
    if (MODE != 0 && K.tau != 0 && make_list(false)) {
      rounds(list, listed);
      if (make_list(true)) rounds(list, listed);
      else rounds(nullptr, G.m);
    } else {
      rounds(nullptr, G.m);
    }
    wg::wg_finish<NT>(G, A, t, [&](uint32_t v) { return q[v] >> 31; }, sh.red);
  }
}

template <int NT, int MODE>
hipError_t kruskal_launch(fi_graph* g, const SweepArgs& a, KruskalArgs k, hipStream_t s) {
  const size_t n = (size_t)g->dg.n;
  const size_t lds = MODE == 0 ? 12 * n : MODE == 1 ? 4 * n : 0;
  const void* f = (const void*)k_sweep_kruskal<NT, MODE>;
  hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_sweep_kruskal<NT, MODE>, NT, lds);
  if (e != hipSuccess) return e;
  // (six resident workgroups per CU: with eight a 1,000-vertex graph ran slower)
  int64_t grid = (int64_t)std::max(1, std::min(per_cu, 6)) * g->cu_count;
  if (g->sched.grid > 0) grid = std::min<int64_t>(grid, g->sched.grid);
  if (MODE != 0) {
    // lists of 3 n edges (with 1.5 n, 60,000 / 400,000 overflows the second and
    // 400 trees take 16.3 ms for 12.9), and what does not lie in LDS
    k.cap = (uint32_t)(3 * n + 64);
    k.slot_stride = ((MODE == 1 ? 16 : 20) * n + 4 * (size_t)k.cap + 255) & ~(size_t)255;
    const size_t slots = g->L.slot_stride * g->L.nslots / k.slot_stride;
    if (slots == 0) return hipErrorInvalidValue;
    grid = std::min<int64_t>(grid, (int64_t)slots);
  }
  grid = (int64_t)std::min<uint64_t>((uint64_t)grid, a.t1 - a.t0);
  hipLaunchKernelGGL((k_sweep_kruskal<NT, MODE>), dim3((unsigned)grid), dim3(NT), lds, s, g->dg, a, k);
  return hipGetLastError();
}

template <int NT>
hipError_t kruskal_block(fi_graph* g, const SweepArgs& a, const KruskalArgs& k, int mode, hipStream_t s) {
  return mode == 0 ? kruskal_launch<NT, 0>(g, a, k, s)
         : mode == 1 ? kruskal_launch<NT, 1>(g, a, k, s)
                     : kruskal_launch<NT, 2>(g, a, k, s);
}

}  // namespace

bool kruskal_forest_fits(const fi_graph* g) {
  return 4 * (size_t)g->dg.n + 16384 <= (size_t)g->max_shared;
}

// path 1: tree state in LDS; 2: in workspace slots (with what still fits LDS)
hipError_t launch_kruskal(fi_graph* g, const SweepArgs& a, int path, int nt, hipStream_t s) {
  const int64_t n = g->dg.n, m = g->dg.m;
  KruskalArgs k{};
  k.slots = g->ws + g->L.slots;
  // about n edges in the first list; a graph of little more than that has one pass
  const int mode = path == 1 ? 0 : kruskal_forest_fits(g) ? 1 : 2;
  // in LDS a round over all the edges costs less than the lists (7,000 vertices,
  // 40,000 edges, 1,000 trees: 539 us and 680)
  k.tau = mode == 0 || m <= n + n / 4 ? 0u : (uint32_t)(4294967296.0 * (double)n / (double)m);
  return nt == 1024 ? kruskal_block<1024>(g, a, k, mode, s)
         : nt == 512 ? kruskal_block<512>(g, a, k, mode, s)
                     : kruskal_block<256>(g, a, k, mode, s);
}

// path 1: the trees in LDS; 2: what does not fit there, for as many waves as
// the trees need, in workspace slots.  both: null, or where to say whether the
// hybrid's BFS trees were launched with them.
hipError_t launch_rdfs(fi_graph* g, const SweepArgs& a, int path, bool* both, hipStream_t s) {
  const size_t n = (size_t)g->dg.n, marks = 4 * (size_t)mark_words(g->dg.n);
  const size_t stack = 4 * (size_t)stack_words(g->dg.n);
  const size_t csr = 4 * (n + 1) + 4 * (size_t)g->dg.nnz;
  const size_t most = (size_t)g->max_shared - kRdfsStatic;
  RdfsArgs r{};
  r.cptr = (const int32_t*)(g->ws + g->L.cptr);
  r.cverts = (const int32_t*)(g->ws + g->L.cverts);
  r.slots = g->ws + g->L.slots;
  // waves that the trees of a CU want
  const uint64_t trees = a.t1 - a.t0, cus = (uint64_t)g->cu_count;
  const size_t want = (size_t)std::max<uint64_t>(1, std::min<uint64_t>(16, (trees + cus - 1) / cus));
  const bool marks_lds = marks * want <= most;
  // waves to a tree, while a CU has few trees and the components beside the main
  // one take more than an eighth of its time (starting one costs about four steps)
  const int64_t main = g->main_end - g->main_begin;
  const int64_t beside = (int64_t)g->dg.n - g->nisolated - main + 4 * (int64_t)(g->nanch - 1);
  r.share = 8 * beside <= main || !marks_lds ? 1 : want <= 4 ? 4 : want <= 8 ? 2 : 1;
  r.cus = (uint32_t)cus;
  // the CSR in LDS while it leaves room for them
  if (csr + want * (marks + stack) <= most)
    return rdfs_launch<true, false, true, true>(g, a, r, path, (int)want, csr + want * (marks + stack),
                                                g->L.slot_stride * g->L.nslots, both, s);
  // else one tree per workgroup, with links: on path 1, whose sweeps may overlap
  // others of the handle, in a region of their own (every launch writes the same
  // bytes there); on path 2 in the slots' region, in front of the slots, where
  // they leave room for four waves per CU
  size_t region = g->L.slot_stride * g->L.nslots;
  const bool stk_lds = path == 1 || (g->dg.n <= kStackMaxN && (marks + stack) * want <= most);
  r.slot_stride = ((stk_lds ? 0 : 4 * n) + (stk_lds || marks_lds ? 0 : marks) + 255) & ~(size_t)255;
  const size_t links = (8 * (size_t)g->dg.nnz + 255) & ~(size_t)255;
  uint2* at = nullptr;
  if (path == 1) {
    if (g->L.nlinks == (size_t)g->dg.nnz) at = (uint2*)(g->ws + g->L.links);
  } else if (g->dg.n <= kLinkMaxN && links + r.slot_stride * std::min<uint64_t>(trees, 4 * cus) <= region) {
    at = (uint2*)r.slots;
    r.slots += links;
    region -= links;
  }
  if (at) {
    const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((g->dg.nnz + 255) / 256, 16384));
    hipLaunchKernelGGL(k_rdfs_links, dim3(grid), dim3(256), 0, s, g->dg.row_ptr, g->dg.adj, g->dg.nnz, at);
    r.links = at;
  }
  const size_t lds = (stk_lds ? stack : 0) + (stk_lds || marks_lds ? marks : 0);
  if (r.links)
    return stk_lds    ? rdfs_launch<false, true, true, true>(g, a, r, path, 1, lds, region, both, s)
           : marks_lds ? rdfs_launch<false, true, false, true>(g, a, r, path, 1, lds, region, both, s)
                      : rdfs_launch<false, true, false, false>(g, a, r, path, 1, lds, region, both, s);
  return stk_lds    ? rdfs_launch<false, false, true, true>(g, a, r, path, 1, lds, region, both, s)
         : marks_lds ? rdfs_launch<false, false, false, true>(g, a, r, path, 1, lds, region, both, s)
                    : rdfs_launch<false, false, false, false>(g, a, r, path, 1, lds, region, both, s);
}

}  // namespace fi
