// Pass 4 of the Hermitian-pair mode: pass 3 has left, for every row i of a
// chunk and every group of gj density orbitals, the sum over the group's pairs
//     sum_j f_j / N_g * psi_j(r) * N_g v_ij(r)
// in the pair slab of the row's first pair of the group; this pass subtracts a
// row's sums from the output orbital i in a fixed order (no atomics).  Pure
// streaming: one read of jc/gj slabs per row and one read-modify-write of the
// output.
#include "fft_core.hpp"
#include "px_internal.hpp"

namespace px {

// One thread's 16 bytes: two complex64 (FP32 form) or one complex128.
// Address-space-1 accesses: global instructions rather than flat ones (the
// pointers come from a struct, so the compiler cannot infer it).
#define PX_GLOBAL __attribute__((address_space(1)))
template <typename T> struct Lane;
template <> struct Lane<float> {
  static constexpr int EV = 2;
  typedef float v __attribute__((ext_vector_type(4)));
};
template <> struct Lane<double> {
  static constexpr int EV = 1;
  typedef double v __attribute__((ext_vector_type(2)));
};

// grid (ceil(N_g / (256 EV)), ic).  N_g is even for every supported grid.
template <typename T>
__global__ __launch_bounds__(256) void pass4_rows(ChunkArgs a0, const ChunkArgs* tasks, size_t ng, int gj) {
  using V = typename Lane<T>::v;
  const ChunkArgs a = chunk_args(a0, tasks);
  const size_t e = (size_t(blockIdx.x) * 256 + threadIdx.x) * Lane<T>::EV;
  const int ii = blockIdx.y;
  if (ii >= a.ic || e >= ng) return;
  const int jend = a.tri ? ii + 1 : a.jc;  // a triangular block holds jj <= ii
  const T* t = reinterpret_cast<const T*>(a.t) + 2 * (size_t(ii) * a.jc * ng + e);
  T* const o = reinterpret_cast<T*>(a.out) + 2 * (size_t(a.i0 + ii) * ng + e);
  // a triangular block's output was written by its pass 3 already
  V prev = V{};
  if (!a.first || a.tri) prev = *(const PX_GLOBAL V*)o;
  // the chunk's sum first: one rounding at the output's magnitude per chunk
  V acc = V{};
#pragma unroll 8
  for (int j = 0; j < jend; j += gj) acc += __builtin_nontemporal_load((const PX_GLOBAL V*)(t + 2 * size_t(j) * ng));
  *(PX_GLOBAL V*)o = prev - acc;
}

hipError_t launch_pass4(bool fp32, const ChunkArgs& a, const ChunkDims& d, int gj, size_t ng,
                        const ChunkArgs* tasks, hipStream_t s) {
  if (ng % 2 || gj < 1) return hipErrorInvalidValue;
  const size_t per = 256 * size_t(fp32 ? Lane<float>::EV : Lane<double>::EV);
  const dim3 g(unsigned((ng + per - 1) / per), d.max_ic, d.ntasks);
  if (fp32) hipLaunchKernelGGL(pass4_rows<float>, g, dim3(256), 0, s, a, tasks, ng, gj);
  else hipLaunchKernelGGL(pass4_rows<double>, g, dim3(256), 0, s, a, tasks, ng, gj);
  return hipGetLastError();
}

}  // namespace px
