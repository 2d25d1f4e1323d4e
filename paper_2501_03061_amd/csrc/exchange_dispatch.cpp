// Size dispatch of the pair pipeline: the grids with compiled plans.
#include "px_internal.hpp"

namespace px {

template <int N0, int N1, int N2>
hipError_t launch_chunk_t(bool fp32, const ChunkArgs& a, const ChunkDims& d, bool ex, int cfg,
                          hipStream_t s, hipEvent_t* ev, const ChunkArgs* tasks);

#define PX_CUBE(X, N) X(N, N, N)
#define PX_GRIDS(X)                                                                             \
  PX_CUBE(X, 16) PX_CUBE(X, 24) PX_CUBE(X, 32) PX_CUBE(X, 40) PX_CUBE(X, 48) PX_CUBE(X, 60)     \
  PX_CUBE(X, 64) PX_CUBE(X, 72) PX_CUBE(X, 80) PX_CUBE(X, 96) X(60, 60, 90) X(60, 90, 120)

bool grid_supported(int n0, int n1, int n2) {
#define PX_CASE(A, B, C) if (n0 == A && n1 == B && n2 == C) return true;
  PX_GRIDS(PX_CASE)
#undef PX_CASE
  return false;
}

static hipError_t dispatch(bool fp32, const int* n, const ChunkArgs& a, const ChunkDims& d, bool ex,
                           int cfg, hipStream_t s, hipEvent_t* ev, const ChunkArgs* tasks) {
#define PX_CASE(A, B, C)                         \
  if (n[0] == A && n[1] == B && n[2] == C)       \
    return launch_chunk_t<A, B, C>(fp32, a, d, ex, cfg, s, ev, tasks);
  PX_GRIDS(PX_CASE)
#undef PX_CASE
  return hipErrorInvalidValue;
}

hipError_t launch_chunk(bool fp32, const int* n, const ChunkArgs& a, bool ex, int cfg, hipStream_t s,
                        hipEvent_t* ev) {
  const ChunkDims d{1, a.ic, a.jc, chunk_pairs(a), a.store_v};
  return dispatch(fp32, n, a, d, ex, cfg, s, ev, nullptr);
}

hipError_t launch_chunk_tasks(bool fp32, const int* n, const ChunkArgs* tasks, const ChunkDims& d, bool ex,
                              int cfg, hipStream_t s) {
  return dispatch(fp32, n, ChunkArgs{}, d, ex, cfg, s, nullptr, tasks);
}

}  // namespace px
