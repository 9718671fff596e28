// The graphBpp sweep (Alg. alg-index): per tree, a level-synchronous BFS with
// the min-key parent rule and fused state propagation, the exact frustration
// count, the canonical-state key, and the cloud insert.
//
// Four kernel families compute identical results:
//   k_sweep_edges - sweep_edges.hip: one workgroup per tree, the tree in LDS.
//   k_sweep_wg   - here: one workgroup per tree; the tree words and the BFS
//                  queue live in a per-workgroup slice of the workspace.
//                  Trees are spread over workgroups, so one launch runs
//                  thousands of trees with no grid barrier.
//   k_sweep_grid - sweep_grid.hip: the whole grid works on a few trees at a
//                  time (persistent cooperative kernel), for graphs far
//                  beyond one workgroup.
//   k_sweep_multi - sweep_multi.hip: the whole grid sweeps 64 or 128 trees
//                  at once with one bit per tree in the fields of each
//                  vertex's record.
// The samplers other than BFS are in sampler.hip.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fi_internal.h"
#include "fi_prims.h"

#include "fi_wg.h"

namespace fi {

namespace {

using wg::WgShared;

// HYBRID: only the hybrid sampler's BFS trees.  (Asking in every kernel cost the
// BFS sweep's levels 5 %: 100 trees of 9,000 levels 18.6 and 20.0 ms.)
template <int NT, bool HYBRID>
__global__ void __launch_bounds__(NT) k_sweep_wg(DevGraph G, SweepArgs A) {
  __shared__ WgShared<NT> sh;
  char* slot = (char*)A.pw + (size_t)blockIdx.x * A.slot_stride;
  uint64_t* pw = (uint64_t*)slot;
  int32_t* q = (int32_t*)(slot + 8 * (size_t)G.n);
  for (uint64_t t = A.t0 + blockIdx.x; t < A.t1; t += gridDim.x) {
    // (the hybrid's other trees are randomized DFS)
    if (HYBRID && wg::hybrid_coin(tree_salt(A.seed, t))) continue;
    wg::wg_tree<NT>(G, A, t, pw, q, sh);
  }
}

// bound of a tree's LDS: tree words and levels; Kruskal also keeps its roots
size_t wg_lds_bytes(int32_t n, int sampler = kSamplerBfs) {
  return (sampler == kSamplerKruskal ? 16 : 12) * (size_t)n;
}

template <int NT>
hipError_t launch_wg(fi_graph* g, const SweepArgs& a, hipStream_t s) {
  SweepArgs b = a;
  b.pw = (uint64_t*)(g->ws + g->L.slots);
  b.slot_stride = g->L.slot_stride;
  int grid = g->sched.grid;
  if (grid <= 0) grid = 8 * g->cu_count;
  grid = (int)std::min<uint64_t>(std::min<uint64_t>((uint64_t)grid, a.t1 - a.t0), g->L.nslots);
  if (a.sampler == kSamplerHybrid)
    hipLaunchKernelGGL((k_sweep_wg<NT, true>), dim3(grid), dim3(NT), 0, s, g->dg, b);
  else
    hipLaunchKernelGGL((k_sweep_wg<NT, false>), dim3(grid), dim3(NT), 0, s, g->dg, b);
  return hipGetLastError();
}

// Edges, and edges times trees, from which a small graph's sweep goes to the
// multi-tree path.
constexpr int64_t kMultiMinEdges = 65536;
constexpr uint64_t kMultiMinTreeEdges = 80000000;

bool tree_fits_lds(const fi_graph* g) {
  return wg_lds_bytes(g->dg.n, g->sampler) + 32768 <= (size_t)g->max_shared;
}

bool capturing(hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) != hipSuccess) {
    (void)hipGetLastError();  // (the null stream beside another stream's capture)
    return true;
  }
  return st != hipStreamCaptureStatusNone;
}

// path 0: what the graph and the trees ask for; a sweep that is being captured
// keeps to one tree per workgroup, in ordinary launches, where a tree fits LDS
// and up to kDeepWork beyond.
int pick_path(fi_graph* g, uint64_t trees, hipStream_t s) {
  const int32_t n = g->dg.n;
  const bool fits = tree_fits_lds(g);
  if (g->sampler != kSamplerBfs) {
    // the other samplers run one tree per workgroup only
    if (g->sched.path == 1 && fits) return 1;
    if (g->sched.path == 2 && g->L.nslots > 0) return 2;
    if (fits) return 1;
    return g->L.nslots > 0 ? 2 : 0;
  }
  if (g->sched.path != 0) return g->sched.path;
  const int64_t work = (int64_t)n + g->dg.m / 2;
  // A tree in LDS is swept alone in 20 to 130 us, as many at once as the CUs
  // hold, in proportion to its edges; the multi-tree pass needs 300 us and up
  // whatever its trees (us: n = 6,000, m = 50,000: 1,000 trees 289 and 363 on it,
  // 4,000 1,090 and 1,281; 10,000 / 80,000: 1,000 446 and 442; 3,000 / 300,000: 100
  // 222 and 224, 300 512 and 338), but on a deep graph it pays its barriers at
  // every level.
  const bool many = g->dg.m >= kMultiMinEdges && trees * (uint64_t)g->dg.m >= kMultiMinTreeEdges;
  const bool plain = g->levels > deep_line(g, trees) || ((fits ? many : work <= kDeepWork) && capturing(s));
  if (fits && (!many || plain)) return 1;
  // One tree per workgroup in workspace memory costs about m per tree (30,000
  // / 150,000: 1.5 ms for 100 trees, 7.3 ms for 1,000; the multi-tree path 0.4
  // and 0.77), but a level of it needs no grid barrier.
  if (plain && work <= kDeepWork && g->L.nslots > 0) return 2;
  return multi_words(g, trees) == 1 ? 4 : 5;
}

// threads per workgroup of the automatic schedule's one-tree-per-workgroup
// paths (measured up to 3 times apart).  Path 2: 256 for sparse graphs
// (average degree up to 10), else 1,024.  Path 1: the tree's LDS bounds the
// workgroups a CU holds, so the fewer fit, the wider each one; while the trees
// are few, a tree's own time counts, so up to one tree per CU takes 1,024
// threads (n = 1,000: 43 us for 100 trees, 70 with 256; n = 4,000: 90 and
// 213) and up to three per CU 512 (n = 1,000, 300 trees: 60 us, 78 with 256,
// 74 with 1,024).  (BFS and Kruskal; the randomized DFS has its own rule and
// the hybrid's BFS trees take 256.)
int auto_block(fi_graph* g, int path, uint64_t trees) {
  // (Kruskal on 20,000 vertices, 100,000 edges: 100 trees 889 us with 1,024
  // threads, 1,007 with 512; 500 trees 2,330 and 1,932.  With the forest in
  // memory, 100,000 / 500,000: 512 trees 21.4 ms and 23.3)
  if (path == 2 && g->sampler == kSamplerKruskal)
    return trees <= (uint64_t)g->cu_count || !kruskal_forest_fits(g) ? 1024 : 512;
  if (path == 2) return g->dg.m <= 5 * (int64_t)g->dg.n ? 256 : 1024;
  if (path != 1 || g->sampler == kSamplerRdfs || g->sampler == kSamplerHybrid) return 256;
  // (Kruskal's rounds on a few hundred edges are barriers: 64 trees of 50 vertices
  // 15.1 us with 256 threads, 16.8 with 1,024; of 300 25.8 and 23.5)
  if (g->sampler == kSamplerKruskal && g->dg.n <= 256) return 256;
  // (BFS in less than the time of its barriers: one vertex 18.8 us with 256 threads,
  // 19.6 with 1,024; 100 22.2 and 22.8, 200 23.3 and 23.3)
  if (g->dg.n <= 128) return 256;
  const size_t lds = wg_lds_bytes(g->dg.n, g->sampler);
  if (lds > 65536 || trees <= (uint64_t)g->cu_count) return 1024;
  return lds <= 24576 && trees > 3 * (uint64_t)g->cu_count ? 256 : 512;
}

}  // namespace

hipError_t launch_sweep(fi_graph* g, const SweepArgs& a, hipStream_t s) {
  if (a.t1 <= a.t0) return hipSuccess;
  int path = pick_path(g, a.t1 - a.t0, s);
  if (path == 0) return hipErrorInvalidValue;  // a sampler other than BFS above 1M vertices
  // the multi-tree path keeps no per-tree state words to hand out; it alone
  // gathers the cloud statistics
  if ((path == 4 || path == 5) && a.bits_out) path = 3;
  if (a.vminus || a.eswitch) path = path == 5 ? 5 : 4;  // (BFS only: checked by the caller)
  const int nt = g->sched.path == 0 ? auto_block(g, path, a.t1 - a.t0) : g->sched.block;
  void* tok = nullptr;
  if (prof_begin(g, s, &tok)) return hipErrorUnknown;
  hipError_t e;
  if ((path == 4 || path == 5) && g->sched.path == 0 && tree_fits_lds(g) && !capturing(s)) {
    // Sweeps in LDS share no scratch memory that they do not all fill alike
    // (launch_rdfs), so those of one handle may overlap on several streams; here
    // they take turns with it.  (Not a captured one, statistics: its event would
    // be the graph's, and the next sweep would not wait for the last one.)
    std::lock_guard<std::mutex> lock(g->ms_lock);
    e = hipSuccess;
    if (!g->ms_done) e = hipEventCreateWithFlags(&g->ms_done, hipEventDisableTiming);
    else e = hipStreamWaitEvent(s, g->ms_done, 0);
    if (e == hipSuccess) e = launch_multi(g, a, path == 5 ? 2 : 1, s);
    if (e == hipSuccess) e = hipEventRecord(g->ms_done, s);
  } else if (path == 4 || path == 5) {
    e = launch_multi(g, a, path == 5 ? 2 : 1, s);
  } else if (path == 3) {
    e = launch_grid(g, a, s);
  } else if (a.sampler == kSamplerKruskal) {
    e = launch_kruskal(g, a, path, nt, s);
  } else if (a.sampler == kSamplerRdfs) {
    e = launch_rdfs(g, a, path, nullptr, s);
  } else {
    e = hipSuccess;
    bool both = false;
    if (a.sampler == kSamplerHybrid) {
      const bool may = g->sched.grid == 0 && (g->sched.path == 0 || nt == 256);
      e = launch_rdfs(g, a, path, may ? &both : nullptr, s);
    }
    if (e == hipSuccess && !both)
      e = path == 1   ? launch_edges(g, a, nt, s)
          : nt == 1024 ? launch_wg<1024>(g, a, s)
          : nt == 512  ? launch_wg<512>(g, a, s)
                       : launch_wg<256>(g, a, s);
  }
  prof_end(g, s, tok, 0);
  return e;
}

}  // namespace fi

using namespace fi;

namespace {
SweepArgs base_args(fi_graph* g, uint64_t seed) {
  SweepArgs a{};
  a.seed = seed;
  a.sampler = g->sampler;
  return a;
}
}  // namespace

extern "C" {

int fi_sweep_range(fi_graph* g, int64_t t0, int64_t t1, uint64_t seed, uint64_t* d_tree_switches,
                   void* stream) {
  if (!g || g->is_batch || t0 < 0 || t1 < t0) return FI_EINVAL;
  if (t1 > ((int64_t)1 << 32)) return FI_ERANGE;
  if (t1 == t0) return FI_OK;
  SweepArgs a = base_args(g, seed);
  a.t0 = (uint64_t)t0;
  a.t1 = (uint64_t)t1;
  a.tree_switches = d_tree_switches;
  a.bits_out = nullptr;
  a.insert = 1;
  return launch_sweep(g, a, (hipStream_t)stream) == hipSuccess ? FI_OK : FI_EDEVICE;
}

int fi_sweep_stats(fi_graph* g, int64_t t0, int64_t t1, uint64_t seed, uint64_t* d_vertex_minus,
                   uint64_t* d_edge_switched, void* stream) {
  if (!g || g->is_batch || t0 < 0 || t1 < t0 || (!d_vertex_minus && !d_edge_switched) ||
      g->sampler != kSamplerBfs)
    return FI_EINVAL;
  if (t1 > ((int64_t)1 << 32)) return FI_ERANGE;
  if (t1 == t0) return FI_OK;
  SweepArgs a = base_args(g, seed);
  a.t0 = (uint64_t)t0;
  a.t1 = (uint64_t)t1;
  a.insert = 1;
  a.vminus = d_vertex_minus;
  a.eswitch = d_edge_switched;
  return launch_sweep(g, a, (hipStream_t)stream) == hipSuccess ? FI_OK : FI_EDEVICE;
}

int fi_set_sampler(fi_graph* g, int32_t sampler) {
  if (!g || g->is_batch || sampler < kSamplerBfs || sampler > kSamplerKruskal) return FI_EINVAL;
  if (sampler != kSamplerBfs && g->L.nslots == 0) {
    // one tree per workgroup needs the tree in LDS or in a workspace slot
    const size_t lds = (sampler == kSamplerKruskal ? 16 : 12) * (size_t)g->dg.n;
    if (lds + 32768 > (size_t)g->max_shared) return FI_ERANGE;
  }
  g->sampler = sampler;
  return FI_OK;
}

int fi_get_sampler(fi_graph* g, int32_t* out) {
  if (!g || g->is_batch || !out) return FI_EINVAL;
  *out = g->sampler;
  return FI_OK;
}

int fi_sweep(fi_graph* g, int64_t K, uint64_t seed, void* stream) {
  return fi_sweep_range(g, 0, K, seed, nullptr, stream);
}

int fi_tree_state(fi_graph* g, uint64_t seed, int64_t t, uint64_t* d_bits_out,
                  uint64_t* d_switches_out, void* stream) {
  if (!g || g->is_batch || t < 0 || !d_bits_out) return FI_EINVAL;
  if (t >= ((int64_t)1 << 32)) return FI_ERANGE;
  SweepArgs a = base_args(g, seed);
  a.t0 = (uint64_t)t;
  a.t1 = (uint64_t)t + 1;
  a.tree_switches = d_switches_out;
  a.bits_out = d_bits_out;
  a.insert = 0;
  return launch_sweep(g, a, (hipStream_t)stream) == hipSuccess ? FI_OK : FI_EDEVICE;
}

}  // extern "C"
