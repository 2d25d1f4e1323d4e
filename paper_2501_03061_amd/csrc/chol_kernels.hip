// FP64 dense kernels on the small n x n complex128 matrix of the ACE
// construction (row-major, interleaved re/im):
//
//   hermitize : M <- (M + M^H)/2
//   cholesky  : -M = L L^H, L lower triangular with real positive diagonal
//               (the unique factor), blocked in 32-column panels; on
//               breakdown the 1-based column goes to the status word
//   inverse   : U = L^{-H} (upper triangular), the right factor of xi = W U
//
// These steps stay in FP64 in both precision forms.
#include "px_internal.hpp"

namespace px {

// The factorisation of a launch: the argument, or entry blockIdx.z of a job
// table in device memory (a group shares one launch per step).
__device__ __forceinline__ CholJob chol_job(const CholJob& j0, const CholJob* jobs) {
  return jobs ? jobs[blockIdx.z] : j0;
}

__global__ void hermitize_k(CholJob j0, const CholJob* jobs) {
  const CholJob j = chol_job(j0, jobs);
  double* const M = j.M;
  const int n = j.n;
  const size_t total = size_t(n) * n;
  for (size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total;
       e += size_t(gridDim.x) * blockDim.x) {
    const int i = int(e / n), c = int(e % n);
    if (c < i) continue;
    double* a = M + (size_t(i) * n + c) * 2;
    double* b = M + (size_t(c) * n + i) * 2;
    const double re = 0.5 * (a[0] + b[0]);
    const double im = 0.5 * (a[1] - b[1]);
    a[0] = re;
    a[1] = im;
    b[0] = re;
    b[1] = -im;
  }
}

namespace {
int elementwise_blocks(int n) {
  const size_t total = size_t(n) * n;
  return int((total + 255) / 256 < 4096 ? (total + 255) / 256 : 4096);
}
}  // namespace

hipError_t launch_hermitize(double* M, int n, hipStream_t s) {
  CholJob j{};
  j.M = M;
  j.n = n;
  hipLaunchKernelGGL(hermitize_k, dim3(elementwise_blocks(n)), dim3(256), 0, s, j,
                     static_cast<const CholJob*>(nullptr));
  return hipGetLastError();
}

// Blocked right-looking Cholesky of A = -M, block width KB = 32:
//   for each diagonal block k: factor A_kk = L_kk L_kk^H in LDS (one
//   workgroup) and keep inv(L_kk); panel L_ik = A_ik L_kk^{-H} (one thread per
//   row); trailing update A_ij -= L_ik L_jk^H for i >= j (32 x 32 tiles).
// The working matrix L starts as -M and ends as the lower factor with a
// zeroed strict upper triangle.  A non-positive pivot stops the factorisation:
// status = 1-based global column, and every later kernel returns at once.
// In a group every job runs the steps of the largest n; a step past a job's
// own size returns at once.
constexpr int KB = 32;

__global__ void chol_init_k(CholJob j0, const CholJob* jobs) {
  const CholJob j = chol_job(j0, jobs);
  const size_t total = size_t(j.n) * j.n;
  for (size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total;
       e += size_t(gridDim.x) * blockDim.x) {
    j.L[2 * e] = -j.M[2 * e];
    j.L[2 * e + 1] = -j.M[2 * e + 1];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) j.status[0] = 0;
}

// Factor the diagonal block at k0 (size kb <= KB); write L_kk back and
// inv(L_kk) into the job's dinv (KB x KB per block, row-major complex).
//
// Elimination on [A | I] without roots (A = L1 D L1^H): step k subtracts
// m = a[r][k] / d_k times row k from the rows r > k, of A for the columns
// c > k and of the inverse for c <= k, so that one value per (r, c) is live, in
// a register: a[r][c] up to step c, (L1^{-1})[r][c] from then on.  LDS carries
// column k of A and row k of the inverse only, one barrier a step.  Bound by the
// latency of the kb dependent steps: 46 us a block with three barriers a step
// and the inverse by one thread per column, now 29 (one formula for all entries
// instead of the branches, and a shorter reciprocal: no change).
__global__ __launch_bounds__(256) void chol_diag_k(CholJob j0, const CholJob* jobs, int k0) {
  __shared__ double2 col[2][KB], row[2][KB];
  __shared__ double dd[KB];
  const CholJob j = chol_job(j0, jobs);
  const int n = j.n;
  if (k0 >= n || j.status[0] != 0) return;
  double2* const L = reinterpret_cast<double2*>(j.L);
  double2* const Dinv = reinterpret_cast<double2*>(j.dinv) + size_t(k0 / KB) * KB * KB;
  const int kb = (n - k0) < KB ? (n - k0) : KB;
  const int t = threadIdx.x, c = t % KB, r0 = t / KB;  // entries (r0 + 8 i, c)
  double2 v[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = r0 + 8 * i;
    const bool in = r < kb && c <= r;
    v[i] = in ? L[size_t(k0 + r) * n + k0 + c] : make_double2(0.0, 0.0);
    l[i] = make_double2(0.0, 0.0);
    if (c == 0) col[0][r] = v[i];
  }
  __syncthreads();
  for (int k = 0; k < kb; ++k) {
    const double2* const cl = col[k & 1];
    const double d = cl[k].x;
    if (!(d > 0.0)) {  // (the same for every thread)
      if (t == 0) j.status[0] = k0 + k + 1;
      return;
    }
    const double inv = 1.0 / d;
    const double2 cc = cl[c], rw = row[k & 1][c];
    if (t == 0) dd[k] = d;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = r0 + 8 * i;
      if (r > k) {
        const double2 a = cl[r], m = make_double2(a.x * inv, a.y * inv);
        if (c > k) {  // a[r][c] -= m conj(a[c][k])
          if (c <= r) {
            v[i].x -= m.x * cc.x + m.y * cc.y;
            v[i].y -= m.y * cc.x - m.x * cc.y;
          }
        } else if (c == k) {
          l[i] = v[i];
          v[i] = make_double2(-m.x, -m.y);
        } else {
          v[i].x -= m.x * rw.x - m.y * rw.y;
          v[i].y -= m.x * rw.y + m.y * rw.x;
        }
      } else if (r == k && c == k) {
        v[i] = make_double2(1.0, 0.0);
      }
      if (c == k + 1 && r > k) col[(k + 1) & 1][r] = v[i];
      if (r == k + 1 && c <= k) row[(k + 1) & 1][c] = v[i];
    }
    __syncthreads();
  }
  const double sc = c < kb ? sqrt(dd[c]) : 1.0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = r0 + 8 * i;
    const bool low = r < kb && c <= r;
    const double sr = low ? sqrt(dd[r]) : 1.0;
    Dinv[r * KB + c] = low ? make_double2(v[i].x / sr, v[i].y / sr) : make_double2(0.0, 0.0);
    if (r < kb && c < kb)
      L[size_t(k0 + r) * n + k0 + c] = !low ? make_double2(0.0, 0.0) : r == c ? make_double2(sc, 0.0)
                                                                            : make_double2(l[i].x / sc, l[i].y / sc);
  }
}

// Panel: for rows i >= k0 + kb, L[i][k0:k0+kb] = A[i][k0:k0+kb] * inv(L_kk)^H,
// and zero the block above the diagonal (L[k0..][i] for the same columns).
// A workgroup takes 32 rows; both factors in LDS, one wave per 16 x 16 quarter
// of the product on v_mfma_f64_16x16x4f64 (lane l: left row and right column
// l % 16, k = l / 16; result rows l / 16 + 4 t, column l % 16).  One thread per
// row with its row in (spilled) registers took 56 us a panel, this 4.7.
typedef double d4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void chol_panel_k(CholJob j0, const CholJob* jobs, int k0) {
  __shared__ double2 a[KB][KB + 1], x[KB][KB + 1];
  const CholJob j = chol_job(j0, jobs);
  const int n = j.n;
  if (k0 >= n || j.status[0] != 0) return;
  const int kb = (n - k0) < KB ? (n - k0) : KB;
  const int base = k0 + kb + int(blockIdx.x) * KB;
  if (base >= n) return;  // no row of this job in the workgroup
  const double2* const Dinv = reinterpret_cast<const double2*>(j.dinv) + size_t(k0 / KB) * KB * KB;
  double2* const L = reinterpret_cast<double2*>(j.L);
  const int t = threadIdx.x;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = t / KB + 8 * i, c = t % KB;
    a[r][c] = base + r < n && c < kb ? L[size_t(base + r) * n + k0 + c] : make_double2(0.0, 0.0);
    x[r][c] = Dinv[r * KB + c];
  }
  __syncthreads();
  const int i0 = ((t >> 6) & 1) * 16, c0 = (t >> 7) * 16, m = t & 15, q = (t >> 4) & 3;
  d4 re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
#pragma unroll
  for (int k = 0; k < KB; k += 4) {  // sum_p a[i][p] conj(x[c][p])
    const double2 u = a[i0 + m][k + q], w = x[c0 + m][k + q];
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(u.x, w.x, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(u.y, w.x, im, 0, 0, 0);
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(u.y, w.y, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(-u.x, w.y, im, 0, 0, 0);
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int i = base + i0 + q + 4 * s, c = c0 + m;
    if (i < n && c < kb) L[size_t(i) * n + k0 + c] = make_double2(re[s], im[s]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {  // strict upper triangle of the final factor
    const int c = t / KB + 8 * i, r = base + t % KB;
    if (c < kb && r < n) L[size_t(k0 + c) * n + r] = make_double2(0.0, 0.0);
  }
}

// Trailing update of the lower triangle: tile (bi, bj) of 32 x 32 with
// bi >= bj over rows/columns >= k0 + kb.
__global__ __launch_bounds__(256) void chol_update_k(CholJob j0, const CholJob* jobs, int k0) {
  __shared__ double pi_[KB][KB + 1][2];
  __shared__ double pj_[KB][KB + 1][2];
  const CholJob j = chol_job(j0, jobs);
  const int n = j.n;
  if (k0 >= n || j.status[0] != 0) return;
  const int kb = (n - k0) < KB ? (n - k0) : KB;
  const int base = k0 + kb;
  const int bi = blockIdx.x, bj = blockIdx.y;
  if (bj > bi) return;
  const int r0 = base + bi * KB, c0 = base + bj * KB;
  if (r0 >= n) return;
  double* const L = j.L;
  const int t = threadIdx.x;
  for (int e = t; e < KB * KB; e += 256) {
    const int r = e / KB, p = e % KB;
    const bool vi = r0 + r < n && p < kb, vj = c0 + r < n && p < kb;
    pi_[r][p][0] = vi ? L[(size_t(r0 + r) * n + k0 + p) * 2] : 0.0;
    pi_[r][p][1] = vi ? L[(size_t(r0 + r) * n + k0 + p) * 2 + 1] : 0.0;
    pj_[r][p][0] = vj ? L[(size_t(c0 + r) * n + k0 + p) * 2] : 0.0;
    pj_[r][p][1] = vj ? L[(size_t(c0 + r) * n + k0 + p) * 2 + 1] : 0.0;
  }
  __syncthreads();
  for (int e = t; e < KB * KB; e += 256) {
    const int r = e / KB, c = e % KB;
    const int gi = r0 + r, gj = c0 + c;
    if (gi >= n || gj >= n || gj > gi) continue;
    double sr = 0.0, si = 0.0;
#pragma unroll 8
    for (int p = 0; p < KB; ++p) {
      const double ar = pi_[r][p][0], ai = pi_[r][p][1], br = pj_[c][p][0], bi2 = pj_[c][p][1];
      sr += ar * br + ai * bi2;
      si += ai * br - ar * bi2;
    }
    L[(size_t(gi) * n + gj) * 2] -= sr;
    L[(size_t(gi) * n + gj) * 2 + 1] -= si;
  }
}

// U = L^{-H} from the blocked inverse X = L^{-1}, by block wavefronts.  The
// factorisation leaves inv(L_kk) of every diagonal block in dinv
// (nb x KB x KB).  Wavefront d = 0 sets X_cc = inv(L_cc); wavefront d >= 1
// computes, for every block column c with r = c + d < nb,
//   X_rc = -inv(L_rr) * sum_{p=c}^{r-1} L_rp X_pc,
// one workgroup per block.  X is never stored itself: block (r, c) of X goes
// to U as U[c0 + j][r0 + i] = conj(X_rc[i][j]), and later wavefronts read X_pc
// back from there (a launch boundary orders the store before the load).
// The strict lower triangle of U is zeroed first; after a breakdown U stays 0.
__global__ void tri_zero_k(CholJob j0, const CholJob* jobs) {
  const CholJob j = chol_job(j0, jobs);
  const size_t total = size_t(j.n) * j.n * 2;
  for (size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total;
       e += size_t(gridDim.x) * blockDim.x)
    j.U[e] = 0.0;
}

//
// The products run on v_mfma_f64_16x16x4f64, one wave per 16 x 16 quarter (lane
// layout as in the panel), the next block pair in flight meanwhile; 200 columns: 10.8 us a
// wavefront, with the products on the vector units from LDS 20.
__global__ __launch_bounds__(256) void tri_wave_k(CholJob j0, const CholJob* jobs, int d) {
  __shared__ double2 ls[KB][KB + 1], xs[KB][KB + 1];
  const CholJob jb = chol_job(j0, jobs);
  if (jb.status[0] != 0) return;
  const int n = jb.n;
  const double2* const L = reinterpret_cast<const double2*>(jb.L);
  const double2* const Dinv = reinterpret_cast<const double2*>(jb.dinv);
  double2* const U = reinterpret_cast<double2*>(jb.U);
  const int nb = (n + KB - 1) / KB;
  const int c = blockIdx.x, r = c + d;
  if (r >= nb) return;
  const int c0 = c * KB, r0 = r * KB;
  const int rb = (n - r0) < KB ? (n - r0) : KB;   // only the last block row can be short
  const int t = threadIdx.x, hi = t / KB, lo = t % KB;
  const double2* const dr = Dinv + size_t(r) * KB * KB;
  if (d == 0) {
    for (int i = 0; i < 4; ++i) {
      const int jj = hi + 8 * i;
      const double2 x = dr[lo * KB + jj];
      if (lo < rb && c0 + jj < n) U[size_t(c0 + jj) * n + r0 + lo] = make_double2(x.x, -x.y);
    }
    return;
  }
  double2 lv[4], xv[4];
  auto load = [&](int p) {  // L_rp by rows, X_pc by rows of U (or of the diagonal inverse)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = hi + 8 * i;
      lv[i] = k < rb ? L[size_t(r0 + k) * n + p * KB + lo] : make_double2(0.0, 0.0);
      if (p == c) {
        xv[i] = Dinv[size_t(p) * KB * KB + lo * KB + k];
      } else {
        const double2 u = U[size_t(c0 + k) * n + p * KB + lo];
        xv[i] = make_double2(u.x, -u.y);
      }
    }
  };
  const int i0 = ((t >> 6) & 1) * 16, c1 = (t >> 7) * 16, m = t & 15, q = (t >> 4) & 3;
  // T = sum_p L_rp X_pc
  d4 re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
  load(c);
  for (int p = c; p < r; ++p) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      ls[hi + 8 * i][lo] = lv[i];
      xs[lo][hi + 8 * i] = xv[i];
    }
    __syncthreads();
    if (p + 1 < r) load(p + 1);
#pragma unroll
    for (int k = 0; k < KB; k += 4) {
      const double2 a = ls[i0 + m][k + q], b = xs[k + q][c1 + m];
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, im, 0, 0, 0);
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, im, 0, 0, 0);
    }
    __syncthreads();
  }
  // X_rc = -inv(L_rr) T, as its transpose T^T inv(L_rr)^T: rows of U
#pragma unroll
  for (int s = 0; s < 4; ++s) xs[i0 + q + 4 * s][c1 + m] = make_double2(re[s], im[s]);
#pragma unroll
  for (int i = 0; i < 4; ++i) ls[hi + 8 * i][lo] = dr[(hi + 8 * i) * KB + lo];
  __syncthreads();
  re = d4{0, 0, 0, 0};
  im = d4{0, 0, 0, 0};
#pragma unroll
  for (int k = 0; k < KB; k += 4) {
    const double2 a = xs[k + q][c1 + m], b = ls[i0 + m][k + q];
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, im, 0, 0, 0);
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, im, 0, 0, 0);
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int jc = c1 + q + 4 * s, i = i0 + m;
    if (i < rb && c0 + jc < n) U[size_t(c0 + jc) * n + r0 + i] = make_double2(-re[s], im[s]);
  }
}

namespace {
// Every step of the factorisation and the inverse for one job (jobs ==
// nullptr) or a table of njobs (steps and grids of the largest size n).
hipError_t chol_steps(const CholJob& j0, const CholJob* jobs, int njobs, int n, hipStream_t s) {
  const int blocks = elementwise_blocks(n);
  hipLaunchKernelGGL(chol_init_k, dim3(blocks, 1, njobs), dim3(256), 0, s, j0, jobs);
  for (int k0 = 0; k0 < n; k0 += KB) {
    hipLaunchKernelGGL(chol_diag_k, dim3(1, 1, njobs), dim3(256), 0, s, j0, jobs, k0);
    const int kb = (n - k0) < KB ? (n - k0) : KB;
    const int rest = n - k0 - kb;
    if (rest > 0) {
      hipLaunchKernelGGL(chol_panel_k, dim3((rest + KB - 1) / KB, 1, njobs), dim3(256), 0, s, j0,
                         jobs, k0);
      const int nt = (rest + KB - 1) / KB;
      hipLaunchKernelGGL(chol_update_k, dim3(nt, nt, njobs), dim3(256), 0, s, j0, jobs, k0);
    }
  }
  hipLaunchKernelGGL(tri_zero_k, dim3(blocks, 1, njobs), dim3(256), 0, s, j0, jobs);
  const int nb = (n + KB - 1) / KB;
  for (int d = 0; d < nb; ++d)
    hipLaunchKernelGGL(tri_wave_k, dim3(nb - d, 1, njobs), dim3(256), 0, s, j0, jobs, d);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_chol_inv(const double* M, int n, double* L, double* U, int32_t* status,
                           double* dinv, hipStream_t s) {
  CholJob j{};
  j.M = const_cast<double*>(M);  // read only by these kernels
  j.L = L;
  j.U = U;
  j.dinv = dinv;
  j.status = status;
  j.n = n;
  return chol_steps(j, nullptr, 1, n, s);
}

hipError_t launch_chol_inv_group(const CholJob* jobs, int njobs, int max_n, hipStream_t s) {
  const CholJob none{};
  hipLaunchKernelGGL(hermitize_k, dim3(elementwise_blocks(max_n), 1, njobs), dim3(256), 0, s, none,
                     jobs);
  return chol_steps(none, jobs, njobs, max_n, s);
}

size_t chol_dinv_bytes(int n) { return size_t((n + KB - 1) / KB) * KB * KB * 16; }


}  // namespace px

// ---------------------------------------------------------------- small FP64 products
namespace px {

// C = alpha op(A) B for complex128 row-major matrices: op(A) is m x k (A
// itself, or A^H with A stored k x m), B is k x n, C is m x n, with leading
// dimensions lda, ldb, ldc in elements.  16 x 16 tiles of C per workgroup,
// 16 x 16 tiles of op(A) and B staged in LDS, one entry of C per thread.
// Used for the small matrix algebra of the PT-IM step (N_phi x N_phi, and
// N_phi x N_phi products over the rank of xi), where the FP64 vector rate is
// ample.
template <bool AH>
__global__ __launch_bounds__(256) void zgemm_k(int m, int n, int kd, const double* A, int lda,
                                               const double* B, int ldb, double* C, int ldc,
                                               double alpha) {
  __shared__ double2 sa[16][17], sb[16][17];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int row = blockIdx.y * 16 + ty, col = blockIdx.x * 16 + tx;
  double cr = 0.0, ci = 0.0;
  for (int k0 = 0; k0 < kd; k0 += 16) {
    // op(A)[row][k0 + tx]: A[row][k] or conj(A[k][row])
    {
      const int k = k0 + tx;
      double2 v = make_double2(0.0, 0.0);
      if (row < m && k < kd) {
        if (AH) {
          const double* p = A + (size_t(k) * lda + row) * 2;
          v = make_double2(p[0], -p[1]);
        } else {
          const double* p = A + (size_t(row) * lda + k) * 2;
          v = make_double2(p[0], p[1]);
        }
      }
      sa[ty][tx] = v;
    }
    {
      const int k = k0 + ty;
      double2 v = make_double2(0.0, 0.0);
      if (k < kd && col < n) {
        const double* p = B + (size_t(k) * ldb + col) * 2;
        v = make_double2(p[0], p[1]);
      }
      sb[ty][tx] = v;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const double2 a = sa[ty][k], b = sb[k][tx];
      cr += a.x * b.x - a.y * b.y;
      ci += a.x * b.y + a.y * b.x;
    }
    __syncthreads();
  }
  if (row < m && col < n) {
    C[(size_t(row) * ldc + col) * 2] = alpha * cr;
    C[(size_t(row) * ldc + col) * 2 + 1] = alpha * ci;
  }
}

hipError_t launch_zgemm_gen(bool ah, int m, int n, int k, const double* A, int lda, const double* B,
                            int ldb, double* C, int ldc, double alpha, hipStream_t s) {
  if (m <= 0 || n <= 0 || k <= 0) return hipErrorInvalidValue;
  const dim3 g((n + 15) / 16, (m + 15) / 16);
  if (ah)
    hipLaunchKernelGGL(zgemm_k<true>, g, dim3(256), 0, s, m, n, k, A, lda, B, ldb, C, ldc, alpha);
  else
    hipLaunchKernelGGL(zgemm_k<false>, g, dim3(256), 0, s, m, n, k, A, lda, B, ldb, C, ldc, alpha);
  return hipGetLastError();
}

hipError_t launch_zgemm(bool ah, int n, const double* A, const double* B, double* C, hipStream_t s) {
  return launch_zgemm_gen(ah, n, n, n, A, n, B, n, C, n, 1.0, s);
}

// dst = alpha * src over n real values
__global__ void scale_k(size_t n, const double* src, double alpha, double* dst) {
  for (size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x; e < n;
       e += size_t(gridDim.x) * blockDim.x)
    dst[e] = alpha * src[e];
}

hipError_t launch_scale(size_t n, const double* src, double alpha, double* dst, hipStream_t s) {
  const int blocks = int((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
  hipLaunchKernelGGL(scale_k, dim3(blocks > 0 ? blocks : 1), dim3(256), 0, s, n, src, alpha, dst);
  return hipGetLastError();
}

// sigma_nxt = sigma_n - i c (A1 - A2) over n x n complex values, and
// res = ||sigma_nxt - sigma_cur||_F / ||sigma_nxt||_F (one workgroup, fixed
// summation order).
__global__ __launch_bounds__(1024) void sigma_update_k(size_t nel, const double* sigma_n,
                                                       const double* A1, const double* A2,
                                                       const double* cur, double* nxt, double c,
                                                       double* res) {
  __shared__ double rd[1024], rn[1024];
  double dd = 0.0, nn = 0.0;
  for (size_t e = threadIdx.x; e < nel; e += blockDim.x) {
    const double gr = A1[2 * e] - A2[2 * e], gi = A1[2 * e + 1] - A2[2 * e + 1];
    // -i c (gr + i gi) = c gi - i c gr
    const double xr = sigma_n[2 * e] + c * gi, xi = sigma_n[2 * e + 1] - c * gr;
    nxt[2 * e] = xr;
    nxt[2 * e + 1] = xi;
    const double dr = xr - cur[2 * e], di = xi - cur[2 * e + 1];
    dd += dr * dr + di * di;
    nn += xr * xr + xi * xi;
  }
  rd[threadIdx.x] = dd;
  rn[threadIdx.x] = nn;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (int(threadIdx.x) < w) {
      rd[threadIdx.x] += rd[threadIdx.x + w];
      rn[threadIdx.x] += rn[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) *res = rn[0] > 0.0 ? sqrt(rd[0] / rn[0]) : 0.0;
}

hipError_t launch_sigma_update(int n, const double* sigma_n, const double* A1, const double* A2,
                               const double* cur, double* nxt, double c, double* res, hipStream_t s) {
  hipLaunchKernelGGL(sigma_update_k, dim3(1), dim3(1024), 0, s, size_t(n) * n, sigma_n, A1, A2, cur,
                     nxt, c, res);
  return hipGetLastError();
}

// out[0] = the first non-zero of st[0 .. k), else 0
__global__ void status_first_k(const int32_t* st, int k, int32_t* out) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  int32_t v = 0;
  for (int i = 0; i < k && v == 0; ++i) v = st[i];
  out[0] = v;
}

hipError_t launch_status_first(const int32_t* st, int k, int32_t* out, hipStream_t s) {
  hipLaunchKernelGGL(status_first_k, dim3(1), dim3(64), 0, s, st, k, out);
  return hipGetLastError();
}

}  // namespace px
