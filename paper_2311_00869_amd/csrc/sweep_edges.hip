// One tree per workgroup, level by level over the edges (fi_edges.h): the BFS
// sweep of a graph whose trees fit LDS.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fi_edges.h"
#include "fi_internal.h"

namespace fi {

namespace {

template <int NT>
__global__ void __launch_bounds__(NT) k_sweep_edges(DevGraph G, SweepArgs A, int32_t later) {
  __shared__ wg::EShared<NT> sh;
  extern __shared__ uint64_t dyn[];
  wg::edges_trees<NT>(G, A, A.t0 + blockIdx.x, A.t1, gridDim.x, later, sh, dyn);
}

template <int NT>
hipError_t edges_launch(fi_graph* g, const SweepArgs& a, hipStream_t s) {
  if (g->dg.n > wg::kEMaxN) return hipErrorInvalidValue;
  const size_t lds = 10 * (size_t)g->dg.n;
  hipError_t e = hipFuncSetAttribute((const void*)k_sweep_edges<NT>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  int per_cu = 0;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_sweep_edges<NT>, NT, lds);
  if (e != hipSuccess) return e;
  int64_t grid = (int64_t)std::max(1, per_cu) * g->cu_count;
  if (g->sched.grid > 0) grid = g->sched.grid;
  grid = (int64_t)std::min<uint64_t>((uint64_t)grid, a.t1 - a.t0);
  hipLaunchKernelGGL(k_sweep_edges<NT>, dim3((unsigned)grid), dim3(NT), lds, s, g->dg, a,
                     g->dg.n - g->nisolated - g->nanch);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_edges(fi_graph* g, const SweepArgs& a, int nt, hipStream_t s) {
  return nt == 1024 ? edges_launch<1024>(g, a, s)
         : nt == 512 ? edges_launch<512>(g, a, s)
                     : edges_launch<256>(g, a, s);
}

}  // namespace fi
