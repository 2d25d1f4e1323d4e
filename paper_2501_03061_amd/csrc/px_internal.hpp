// Internal interfaces between the host orchestration (px_api.cpp) and the
// kernel translation units.  Not part of the public ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace px {

// FP64 sums of one pair product over a z tile (FP32 form): sum of rho, and sum
// of |rho|^2 of the values handed to the transform.
struct G0Part {
  double re, im, en, pad;
};

// One chunk of orbital pairs: i in [i0, i0+ic) (output orbitals phi_i) times
// j in [j0, j0+jc) (density orbitals psi_j).  Pair p = (i-i0)*jc + (j-j0)
// owns slab p of the pair buffer t ([pairs][n2][n1][n0]).
struct ChunkArgs {
  const void* psi;      // [n_psi][N_g] complex (precision of the call)
  const void* phi;      // [n_phi][N_g]
  void* t;              // pair buffer, >= ic*jc*N_g complex
  void* out;            // [n_phi][N_g]
  const double* occ;    // [n_psi]
  const double* kern;   // [N_g] FP64, FFT order
  const void* kt;       // [n2][n0][n1] the table of the form: FP64, or rounded to FP32 (FP32
                        // form; K(0) is read from kern)
  G0Part* g0;           // [ic*jc][tiles] FP64 tile sums (FP32 form)
  double* expart;       // FP64 energy partials per (pair, kz): sum K|rho(G)|^2 (FP64 form),
                        // or {sum_{G!=0} K|rho|^2, sum_{G!=0} |rho|^2, G=0 term} (FP32 form)
  int i0, ic, j0, jc;
  int first;            // the chunk's first pass to write the output block i0 overwrites it
                        // instead of accumulating
  double* S;            // pair-energy matrix of the instance (task-table mode)
  int s_ld;             // its row stride
  int store_v;          // Hermitian-pair mode: pass 3 also sums the transposed pairs, pass 4 runs
  double inv_ng;
  int tri;              // diagonal block of the symmetric mode (i0 == j0, ic == jc) solved as
                        // its lower triangle jj <= ii: passes 1 and 3 run jj = 0..ii, pass 2
                        // takes the ic (ic + 1) / 2 pairs of the triangle (slots keep the
                        // square layout p = ii jc + jj), the transposed sums take jj < ii
};

#if defined(__HIPCC__)
// Pairs of a chunk, and the pair slot of the q-th of them (row-major over the
// triangle jj <= ii when tri is set).
__host__ __device__ inline int chunk_pairs(const ChunkArgs& a) {
  return a.tri ? a.ic * (a.ic + 1) / 2 : a.ic * a.jc;
}
__device__ __forceinline__ int pair_slot(const ChunkArgs& a, int q) {
  if (!a.tri) return q;
  int ii = int((sqrt(8.0 * double(q) + 1.0) - 1.0) * 0.5);
  if ((ii + 1) * (ii + 2) / 2 <= q) ++ii;  // rounding of the square root
  if (ii * (ii + 1) / 2 > q) --ii;
  return ii * a.jc + (q - ii * (ii + 1) / 2);
}
#endif

// The chunk of a kernel launch: the launch argument, or entry blockIdx.z of a
// task table in device memory.  A table entry is read through the constant
// address space (scalar loads), so that its fields are known to be uniform:
// the compiler then keeps the base pointers in scalar registers and forms
// addresses from 32-bit per-lane offsets.
#if defined(__HIPCC__)
__device__ __forceinline__ ChunkArgs chunk_args(const ChunkArgs& a0, const ChunkArgs* tasks) {
#if defined(__HIP_DEVICE_COMPILE__)
  if (tasks) {
    typedef const __attribute__((address_space(4))) ChunkArgs CChunk;
    CChunk* c = (CChunk*)(tasks + blockIdx.z);
    ChunkArgs a;
    a.psi = c->psi;
    a.phi = c->phi;
    a.t = c->t;
    a.out = c->out;
    a.occ = c->occ;
    a.kern = c->kern;
    a.kt = c->kt;
    a.g0 = c->g0;
    a.expart = c->expart;
    a.i0 = c->i0;
    a.ic = c->ic;
    a.j0 = c->j0;
    a.jc = c->jc;
    a.first = c->first;
    a.S = c->S;
    a.s_ld = c->s_ld;
    a.store_v = c->store_v;
    a.inv_ng = c->inv_ng;
    a.tri = c->tri;
    return a;
  }
  return a0;
#else
  return tasks ? tasks[blockIdx.z] : a0;
#endif
}
#endif

// Grids with compiled pipelines: the cubic sizes and the non-cubic shapes.
bool grid_supported(int n0, int n1, int n2);

// Points of the plane in a z tile (see exchange_kernels.hpp): rows of 256 bytes
// (configuration 0) or 512 (1, which the autotuner times as well).
constexpr int ztile_width(bool fp32, int cfg) { return (cfg == 0 ? 256 : 512) / (fp32 ? 8 : 16); }
constexpr int kTileConfigs = 2;
// z tiles of a pair on grid n[3]: the slots of a pair's G = 0 tile sums.
inline int ztile_count(bool fp32, const int* n, int cfg) {
  const int w = ztile_width(fp32, cfg);
  return (n[0] * n[1] + w - 1) / w;
}
// Density orbitals j whose sums pass 3 keeps in registers (Hermitian-pair mode)
// when a thread holds rs points of a tile: GJ rs complex sums, as many as leave
// two waves per SIMD without spills (checked with -Rpass-analysis on every
// grid; spills inside the loop cost more than the columns save).  More columns cost pass 3
// registers and save pass 4 2/GJ of a slab (72^3 FP32, rs = 9, passes 3 and 4:
// GJ = 2 2.1 us a pair, 3 1.36, 4 1.24, 5 1.23).
constexpr int col_group(bool fp32, int rs) {
  return fp32 ? (rs <= 5 ? 8 : rs <= 8 ? 6 : rs >= 10 ? 3 : 4) : (rs <= 5 ? 4 : rs >= 10 ? 2 : 3);
}
// Waves per SIMD that the register allocation of pass 3 aims at.
constexpr int pass3_waves(bool fp32, bool sym, int nt) { return sym ? (fp32 && nt > 512 ? 3 : 2) : 1; }
// Largest sizes of the chunks of one launch.
struct ChunkDims {
  int ntasks;     // chunks
  int max_ic, max_jc;
  int max_pairs;  // solved pairs (chunk_pairs)
  int store_v;    // of every chunk
};
// Whether pass 3 has too few workgroups with groups of gj columns to fill the
// chip (256 CUs): then one column per workgroup.  Passes 3 and 4 of builds, ms per
// 1000 pairs, with groups always / below 384 workgroups / below 1536: 24^3 FP32 8
// orbitals 1.36 / 0.65 / 0.65, 40 orbitals 0.37 / 0.12 / 0.12; 48^3 FP32 16 orbitals 0.90 /
// 0.92 / 0.93, 40 orbitals 0.44 / 0.44 / 0.61, 128 orbitals 0.36 / 0.36 / 0.55.
inline bool small_group(int ntile, int max_jc, int gj, int ntasks) {
  return size_t(ntile) * ((max_jc + gj - 1) / gj) * ntasks < 384;
}
// Pairs that a pass-2 workgroup takes one after the other (its twiddle tables are
// made once for them), with at least 4096 workgroups left.  Pass 2, ms per 1000
// pairs, with at least 1024 / 4096 / 16384 left: 48^3 x 16 FP32 0.54 / 0.40 / 0.41, FP64 0.98 /
// 0.72 / 0.72; 24^3 x 16 FP32 0.153 / 0.127 / 0.126; 65536 at 72^3 x 96: FP32 1.58 -> 1.77.
constexpr int kSlabPairs = 8;  // at most
inline int pairs_per_slab_wg(int n2, int max_pairs, int ntasks) {
  const size_t wgs = size_t(n2) * max_pairs * ntasks;
  const size_t q = wgs / 4096;
  return q < 1 ? 1 : q > kSlabPairs ? kSlabPairs : int(q);
}

// Launches passes 1 to 3 (and 4 with store_v) of one chunk on grid n[3] in tile
// configuration cfg; ev (nullable) = 5 events recorded before pass 1, between
// the passes and after the last.
hipError_t launch_chunk(bool fp32, const int* n, const ChunkArgs& a, bool ex, int cfg, hipStream_t s,
                        hipEvent_t* ev);
// The same passes over a task table in device memory (chunks of one grid
// within the sizes of d), one launch each.
hipError_t launch_chunk_tasks(bool fp32, const int* n, const ChunkArgs* tasks, const ChunkDims& d, bool ex,
                              int cfg, hipStream_t s);
// Pass 4 (Hermitian-pair mode): out[i] -= the sums over groups of gj pairs that
// pass 3 left in the pair buffer, for one chunk or a task table.
hipError_t launch_pass4(bool fp32, const ChunkArgs& a, const ChunkDims& d, int gj, size_t ng,
                        const ChunkArgs* tasks, hipStream_t s);
// Energy partials -> S for every task of a table (see launch_expart_reduce).
// max_slots: the largest ic * jc of the table.
hipError_t launch_expart_reduce_tasks(bool fp32, const ChunkArgs* tasks, int ntasks, int max_slots,
                                      int n2, int ntile, double ng, hipStream_t s);

// misc_kernels.hip
hipError_t launch_kernel_hse(int n0, int n1, int n2, double L0, double L1, double L2, double mu,
                             double* kern, hipStream_t s);
hipError_t launch_convert_c128_c64(size_t n, const void* src, void* dst, hipStream_t s);
// The kernel table [n2][n1][n0] transposed to [n2][n0][n1], FP64 or rounded to FP32
hipError_t launch_kernel_transpose(bool fp32, int n0, int n1, int n2, const double* kern, void* kt,
                                   hipStream_t s);
// n real FP64 values -> FP32 (round to nearest even)
hipError_t launch_convert_f64_f32(size_t n, const double* src, float* dst, hipStream_t s);
hipError_t launch_stream_copy(size_t bytes, const void* src, void* dst, hipStream_t s);
// S[i][j] (row stride lds) from the chunk's energy partials (see ChunkArgs);
// FP32 form (g0 non-null): the G != 0 part is rescaled so that its energy
// matches Parseval's identity with the FP64 energy of the transform input.
hipError_t launch_expart_reduce(const double* expart, const G0Part* g0, int n2, int ntile, double ng,
                                int i0, int ic, int j0, int jc, double* S, int lds, bool mirror,
                                bool tri, hipStream_t s);
// e_x = scale * sum_i sum_j f_i f_j S[i][j]
hipError_t launch_energy(const double* S, const double* occ, int n, double scale, double* e_x,
                         hipStream_t s);

// mid = (a + b)/2 over n complex128 values
hipError_t launch_midpoint(size_t n, const double* a, const double* b, double* mid, hipStream_t s);

// rho[r] = sum_i w[i] |phi_i(r)|^2 (FP64), phi [n][ng] complex in the form's precision
hipError_t launch_density(bool fp32, size_t ng, int n, const void* phi, const double* w,
                          double* rho, hipStream_t s);

// eig_kernels.hip: sigma = Q diag(d) Q^H (FP64, complex128 n x n row-major), d ascending;
// status[0] = 0 when converged within max_sweeps Jacobi sweeps, else the sweeps made.
// work: eig_work_bytes(n).
size_t eig_work_bytes(int n);
hipError_t launch_eig_hermitian(const double* sigma, int n, double* Q, double* d, int32_t* status,
                                void* work, int max_sweeps, hipStream_t s);

// gemm_kernels.hip: complex GEMMs on MFMA
// M[a][b] (a < na, b < nb, row-major ldm) = scale * sum_r conj(X[a][r]) Y[b][r]
//   X: [na][ng], Y: [nb][ng]; FP64 result.  part: workspace of nsplit*na*nb complex128,
//   where nsplit (the splits available) may be below gemm_xhy_part_elems' count: the
//   sum over r then runs in fewer, longer splits.
//   M32 (nullable): the result rounded to complex64 as well, same layout.
hipError_t launch_gemm_xhy(bool fp32, int na, int nb, size_t ng, const void* X, const void* Y,
                           double scale, double* M, int ldm, double* part, int nsplit,
                           float* M32, hipStream_t s);
// The same for a result known to be Hermitian (n x n, ldm = n, e.g. M = dV
// Psi^H W of the ACE construction): only the 64 x 64 tiles on and above the
// diagonal are contracted (about half the flops); each tile below the diagonal
// is the conjugate transpose of its mirror.  The diagonal tiles are computed in
// full, so they keep their (rounding-level) non-Hermitian part.
hipError_t launch_gemm_xhy_herm(bool fp32, int n, size_t ng, const void* X, const void* Y,
                                double scale, double* M, double* part, int nsplit,
                                hipStream_t s);
// (max_split > 0: at most so many splits)
size_t gemm_xhy_part_elems(int na, int nb, size_t ng, int* nsplit, bool herm = false, int max_split = 0);
// Splits launch_gemm_xhy uses when at most max_split are available (fewer,
// longer splits than the default when max_split is below it).
int gemm_xhy_splits(int na, int nb, size_t ng, int max_split);
// One update of the implicit-midpoint fixed point with the product Z[b][r] =
// -sum_a X[a][r] C[a][b] as its last term (gemm_xc with alpha = -1; the product
// rounded to the form's type, then added to y in FP64):
//   nxt = phi_n - i c (y + Z) (y nullable), mid = (phi_n + nxt)/2 (nullable; the
//   next iteration's midpoint), res = ||nxt - cur|| / ||nxt|| summed in FP64.
// Blocks [nb][ng]; nxt and mid may not overlap X (other workgroups read it).
// partial: ptim_xc_partials(nb, ng) doubles.
struct PtimUpdate {
  const void* phi_n;
  const void* y;
  const void* cur;
  void* nxt;
  void* mid;
  double c;
  double* partial;
  double* res;
};
size_t ptim_xc_partials(int nb, size_t ng);
hipError_t launch_ptim_xc(bool fp32, int na, int nb, size_t ng, const void* X, const void* C, int ldc,
                          const PtimUpdate& p, hipStream_t s);
// Z[b][r] = alpha * sum_a X[a][r] C[a][b]
//   X: [na][ng], C: [na][ldc] row-major in the precision of the form (complex128, or
//   complex64 rounded from the FP64 matrix), Z: [nb][ng]; upper: C upper triangular
hipError_t launch_gemm_xc(bool fp32, int na, int nb, size_t ng, const void* X, const void* C,
                          int ldc, double alpha, void* Z, bool upper, hipStream_t s);
// The same with alpha = 1 for a C whose imaginary parts are zero (they are not
// multiplied).
hipError_t launch_gemm_xc_real(bool fp32, int na, int nb, size_t ng, const void* X, const void* C, int ldc,
                               void* Z, hipStream_t s);

// chol_kernels.hip: FP64 Hermitian tools on an n x n complex128 matrix (row-major)
hipError_t launch_hermitize(double* M, int n, hipStream_t s);
// U = L^{-H} where -M = L L^H; status[0] = 0 on success or the 1-based failing column
// dinv: workspace of chol_dinv_bytes(n) (inverses of the 32 x 32 diagonal blocks)
size_t chol_dinv_bytes(int n);
hipError_t launch_chol_inv(const double* M, int n, double* L, double* U, int32_t* status,
                           double* dinv, hipStream_t s);
// One factorisation of a group: its matrices and status word (M is hermitized in place).
struct CholJob {
  double* M;
  double* L;
  double* U;
  double* dinv;
  int32_t* status;
  int n;
  int pad;
};
// hermitize + launch_chol_inv for every job of a device-resident table, one
// launch per step for the whole group (blockIdx.z = job); max_n >= every n.
hipError_t launch_chol_inv_group(const CholJob* jobs, int njobs, int max_n, hipStream_t s);
// C = op(A) B, n x n complex128 row-major, op(A) = A^H when ah
hipError_t launch_zgemm(bool ah, int n, const double* A, const double* B, double* C, hipStream_t s);
// C = alpha op(A) B: op(A) m x k (A^H of a k x m A when ah), B k x n, C m x n,
// complex128 row-major with leading dimensions lda, ldb, ldc (elements)
hipError_t launch_zgemm_gen(bool ah, int m, int n, int k, const double* A, int lda, const double* B,
                            int ldb, double* C, int ldc, double alpha, hipStream_t s);
// dst = alpha * src, n real FP64 values
hipError_t launch_scale(size_t n, const double* src, double alpha, double* dst, hipStream_t s);
// nxt = sigma_n - i c (A1 - A2) (n x n complex128); *res = ||nxt - cur|| / ||nxt|| (FP64)
hipError_t launch_sigma_update(int n, const double* sigma_n, const double* A1, const double* A2,
                               const double* cur, double* nxt, double c, double* res, hipStream_t s);
// out[0] = first non-zero of st[0 .. k), else 0
hipError_t launch_status_first(const int32_t* st, int k, int32_t* out, hipStream_t s);

}  // namespace px
