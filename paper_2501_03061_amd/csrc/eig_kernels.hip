// FP64 Hermitian eigendecomposition of the occupation matrix, sigma = Q D Q^H
// (Sec. IV-A-1, Eq. 11), by the cyclic Jacobi method in a blocked parallel
// ordering.
//
// The indices are cut into blocks of BJ = 16 (nb blocks, rounded up to even;
// indices past n are absent).  A sweep visits every pair of blocks once, in
// nb - 1 rounds of nb/2 disjoint block pairs (the circle method: block nb - 1
// stays put, the others rotate).  In a round, one workgroup per block pair
// takes the 32 x 32 Hermitian submatrix of its 32 indices into LDS and runs
// one sweep of scalar cyclic Jacobi on it (31 rounds of 16 disjoint index
// pairs in the same circle ordering; each pair gets the unitary G = P J that
// zeroes its off-diagonal entry: with A_pq = |A_pq| e^{i theta},
// P = diag(1, e^{-i theta}) makes the 2 x 2 block real symmetric and J is its
// real Jacobi rotation, tangent t = sgn(tau)/(|tau| + sqrt(1 + tau^2)),
// tau = (A_qq - A_pp)/(2 |A_pq|), the smaller angle), accumulating the 32 x 32
// unitary U of the pair.  The U of a round act on disjoint index sets, so
// A <- G^H A G splits into 32 x 32 tiles A_PS <- U_P^H A_PS U_S and V <- V G
// into 32-row tiles V_rS <- V_rS U_S, one workgroup per tile.  Compared with
// rotating single index pairs, a sweep reads and writes A and V nb - 1 times
// instead of n - 1 times, which is what bounds the method at these sizes.
// After each sweep the off-diagonal Frobenius norm is formed (partial sums,
// then a fixed-order total); below
// 64 eps sqrt(n) ||A||_F a device flag makes the remaining launches return at
// once, so the host enqueues a fixed number of sweeps without waiting for the
// device.  Finally d = diag(A) in ascending order, Q the matching columns of V.
#include <float.h>

#include "px_internal.hpp"

namespace px {

namespace {

// A rotation G of an index pair: g00 = c, g01 = s, g10 = -s e, g11 = c e with
// e = e^{-i theta} = er + i ei; s = 0 and e = 1 for the identity.
struct Rot {
  double c, s, er, ei;
};

// Pair `slot` of round k (0 <= k < np - 1) of the circle ordering of np
// (even) indices; p < q.
__device__ __forceinline__ void round_pair(int np, int k, int slot, int& p, int& q) {
  const int m = np - 1;
  int a, b;
  if (slot == 0) {
    a = k % m;
    b = m;
  } else {
    a = (k + slot) % m;
    b = (k - slot + m) % m;
  }
  p = a < b ? a : b;
  q = a < b ? b : a;
}

// (x0, x1) <- (x0, x1) G
__device__ __forceinline__ void rotate_cols(const Rot& g, double2& x0, double2& x1) {
  const double2 t = make_double2(x1.x * g.er - x1.y * g.ei, x1.x * g.ei + x1.y * g.er);
  const double2 y0 = make_double2(g.c * x0.x - g.s * t.x, g.c * x0.y - g.s * t.y);
  x1 = make_double2(g.s * x0.x + g.c * t.x, g.s * x0.y + g.c * t.y);
  x0 = y0;
}
// (x0, x1)^T <- G^H (x0, x1)^T
__device__ __forceinline__ void rotate_rows(const Rot& g, double2& x0, double2& x1) {
  const double2 t = make_double2(x1.x * g.er + x1.y * g.ei, x1.y * g.er - x1.x * g.ei);
  const double2 y0 = make_double2(g.c * x0.x - g.s * t.x, g.c * x0.y - g.s * t.y);
  x1 = make_double2(g.s * x0.x + g.c * t.x, g.s * x0.y + g.c * t.y);
  x0 = y0;
}

__device__ __forceinline__ double2 ld2(const double* A, int n, int r, int c) {
  return *reinterpret_cast<const double2*>(A + (size_t(r) * n + c) * 2);
}
__device__ __forceinline__ void st2(double* A, int n, int r, int c, double2 v) {
  *reinterpret_cast<double2*>(A + (size_t(r) * n + c) * 2) = v;
}

// A = (sigma + sigma^H)/2, V = I, flags cleared.
__global__ void eig_init_k(const double* sigma, int n, double* A, double* V, int* flags) {
  const size_t total = size_t(n) * n;
  for (size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total;
       e += size_t(gridDim.x) * blockDim.x) {
    const int i = int(e / n), j = int(e % n);
    const double2 a = ld2(sigma, n, i, j), b = ld2(sigma, n, j, i);
    st2(A, n, i, j, make_double2(0.5 * (a.x + b.x), 0.5 * (a.y - b.y)));
    st2(V, n, i, j, make_double2(i == j ? 1.0 : 0.0, 0.0));
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    flags[0] = 0;  // converged
    flags[1] = 0;  // sweeps completed
  }
}

constexpr int BJ = 16;        // indices per block
constexpr int BJ2 = 2 * BJ;   // size of a block pair's subproblem

// Index t (0 <= t < 32) of block pair `slot` in block round k: block I's 16
// indices, then block J's.
__device__ __forceinline__ int bj_index(int nb, int k, int slot, int t) {
  int I, J;
  round_pair(nb, k, slot, I, J);
  return t < BJ ? I * BJ + t : J * BJ + (t - BJ);
}

// 1/sqrt(x) of a normal x: the hardware's approximation (5e-8) with one Newton
// step (4e-15 at most, 3e-16 rms over 1 M values).
__device__ __forceinline__ double rsq1(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}
// 1/sqrt(x) and 1/x with one step of third order (rounded): one dependent
// operation more than a Newton step, two (one) fewer than a second one.
__device__ __forceinline__ double rsq3(double x) {
  const double y = __builtin_amdgcn_rsq(x), e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}
__device__ __forceinline__ double rcp3(double x) {
  const double y = __builtin_amdgcn_rcp(x), e = fma(-x, y, 1.0);
  return fma(y, fma(e, e, e), y);
}

// Rotation of the 2 x 2 diagonal block (app, aqq real, apq).  With m = |apq|,
// d = aqq - app and h = 2 m the tangent is h / (|d| + sqrt(d^2 + h^2)), its roots and
// reciprocals rounded: what a rotation leaves of the entry is rounding, also where
// it is the last one.  c^2 + s^2 = 1 and |e| = 1, which thousands of rotations
// accumulate in V, are restored to the rounding of the four numbers by one
// correction each (so c takes one step).
// Outside the normal range of the squares: hypot and exact division.
__device__ __forceinline__ Rot make_rot(double app, double aqq, double2 apq, double skip2) {
  Rot r = {1.0, 0.0, 1.0, 0.0};
  const double m2 = apq.x * apq.x + apq.y * apq.y, d = aqq - app;
  if (m2 <= skip2 || (apq.x == 0.0 && apq.y == 0.0)) return r;
  double im, t;
  if (m2 > 1e-280 && m2 < 1e280 && fabs(d) < 1e140) {
    im = rsq3(m2);
    const double x = fma(d, d, 4.0 * m2);
    t = (d >= 0.0 ? 2.0 : -2.0) * (m2 * im) * rcp3(fma(x, rsq3(x), fabs(d)));
  } else {
    const double m = hypot(apq.x, apq.y);
    im = 1.0 / m;
    t = (d >= 0.0 ? 2.0 : -2.0) * m / (fabs(d) + hypot(d, 2.0 * m));
  }
  r.c = rsq1(fma(t, t, 1.0));
  r.s = t * r.c;
  r.er = apq.x * im;  // e^{-i theta} = conj(A_pq)/|A_pq|
  r.ei = -apq.y * im;
  const double fc = 0.5 * fma(-r.c, r.c, fma(-r.s, r.s, 1.0)), fe = 0.5 * fma(-r.er, r.er, fma(-r.ei, r.ei, 1.0));
  r.c = fma(r.c, fc, r.c);
  r.s = fma(r.s, fc, r.s);
  r.er = fma(r.er, fe, r.er);
  r.ei = fma(r.ei, fe, r.ei);
  return r;
}

// ||A||_F^2, kept behind the flags.
__device__ __forceinline__ double norm2(const int* flags) { return reinterpret_cast<const double*>(flags)[1]; }
// Entries with |A_pq| <= 8 eps ||A||_F / sqrt(n), the level of their rounding
// errors, are not rotated away: where eigenvalues coincide (occupations at 0 and
// 1) both A_pq and A_qq - A_pp are rounding noise, the rotation angle is
// arbitrary, and every sweep mixed the noise anew (256 and 500 indices with
// Fermi-Dirac eigenvalues or a projector: not converged after 40 sweeps before,
// now in 15 to 20).  All entries at that level leave an off-diagonal norm of
// 8 eps sqrt(n) ||A||_F, an eighth of the convergence bound.  From the second sweep
// on only: an input's own entries at that level (the identity plus 1e-15) are
// rotated once, as all others (with the skip from the first on, the eigenvalues of
// such matrices were off by twice as much, 2 x 2 by five times).
__device__ __forceinline__ double skip_factor(int n) { return 64.0 * DBL_EPSILON * DBL_EPSILON / double(n); }

// One inner sweep on the 32 x 32 subproblem of each block pair of round k
// (one workgroup per pair): U_P (32 x 32, row-major) into Ug[P].  Bound by the
// chain rotation -> S -> rotation of the inner rounds (few workgroups, no
// bandwidth): per round one phase of S on all four waves, and one in which wave
// 0 forms the next rotations while the others apply the current ones to U.  A
// launch took 66 us with both updates after the rotations and 2 x 2 complex
// matrix products, now 30 (twelve waves, U beside S: 31; what is left is mostly
// the LDS traffic of the rotations, S and U).
__global__ __launch_bounds__(256) void bj_solve_k(const double* A, int n, int nb, int k, double* Ug,
                                                  const int* flags, int first) {
  if (flags[0]) return;
  __shared__ double2 S[BJ2][BJ2 + 1];
  __shared__ double2 U[BJ2][BJ2 + 1];
  __shared__ Rot rot[2][BJ];
  __shared__ int gi[BJ2];
  const int P = blockIdx.x, tid = threadIdx.x;
  if (tid < BJ2) gi[tid] = bj_index(nb, k, P, tid);
  __syncthreads();
  for (int e = tid; e < BJ2 * BJ2; e += 256) {
    const int i = e / BJ2, j = e % BJ2;
    S[i][j] = (gi[i] < n && gi[j] < n) ? ld2(A, n, gi[i], gi[j]) : make_double2(0.0, 0.0);
    U[i][j] = make_double2(i == j ? 1.0 : 0.0, 0.0);
  }
  __syncthreads();
  const double skip2 = first ? -1.0 : skip_factor(n) * norm2(flags);
  auto next_rot = [&](int kk) {
    int p, q;
    round_pair(BJ2, kk, tid, p, q);
    rot[kk & 1][tid] = make_rot(S[p][p].x, S[q][q].x, S[p][q], skip2);
  };
  if (tid < BJ) next_rot(0);
  __syncthreads();
  for (int kk = 0; kk < BJ2 - 1; ++kk) {
    {  // S <- G^H S G on the 2 x 2 blocks (pair x, pair y): 16 x 16 = 256 blocks
      const int x = tid / BJ, y = tid % BJ;
      const Rot gx = rot[kk & 1][x], gy = rot[kk & 1][y];
      int p, q, u, v;
      round_pair(BJ2, kk, x, p, q);
      round_pair(BJ2, kk, y, u, v);
      double2 a = S[p][u], b = S[p][v], c = S[q][u], d = S[q][v];
      rotate_cols(gy, a, b);
      rotate_cols(gy, c, d);
      rotate_rows(gx, a, c);
      rotate_rows(gx, b, d);
      S[p][u] = a;
      S[p][v] = b;
      S[q][u] = c;
      S[q][v] = d;
    }
    __syncthreads();
    if (tid < 64) {
      if (tid < BJ && kk + 1 < BJ2 - 1) next_rot(kk + 1);
    } else {
      for (int e = tid - 64; e < BJ2 * BJ; e += 192) {  // U <- U G: (row, pair) pieces
        const int r = e / BJ, y = e % BJ;
        int p, q;
        round_pair(BJ2, kk, y, p, q);
        double2 x0 = U[r][p], x1 = U[r][q];
        rotate_cols(rot[kk & 1][y], x0, x1);
        U[r][p] = x0;
        U[r][q] = x1;
      }
    }
    __syncthreads();
  }
  double2* out = reinterpret_cast<double2*>(Ug) + size_t(P) * BJ2 * BJ2;
  for (int e = tid; e < BJ2 * BJ2; e += 256) out[e] = U[e / BJ2][e % BJ2];
}

typedef double d4 __attribute__((ext_vector_type(4)));

// D (16 x 16 tile at (i0, j0)) = op(L) R of 32 x 32 complex matrices in LDS, one
// wave per tile on v_mfma_f64_16x16x4f64 (lane l: left row and right column
// l % 16, k = l / 16; result rows l / 16 + 4 t, column l % 16).  op: the matrix
// itself, or its conjugate transpose.
template <bool CT>
__device__ __forceinline__ void tile_product(const double2 (*L)[BJ2 + 1], const double2 (*R)[BJ2 + 1], int i0, int j0,
                                             d4& re, d4& im) {
  const int m = threadIdx.x & 15, q = (threadIdx.x >> 4) & 3;
  re = d4{0, 0, 0, 0};
  im = d4{0, 0, 0, 0};
#pragma unroll
  for (int k = 0; k < BJ2; k += 4) {
    double2 a = CT ? L[k + q][i0 + m] : L[i0 + m][k + q];
    if (CT) a.y = -a.y;
    const double2 b = R[k + q][j0 + m];
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, im, 0, 0, 0);
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, im, 0, 0, 0);
  }
}

// The block rotations of round k: A_PS <- U_P^H A_PS U_S for every pair of
// block pairs (blockIdx.y = 0, blockIdx.x = P * m + S), V_rS <- V_rS U_S for
// every 32-row tile r and block pair S (blockIdx.y = 1, blockIdx.x = r * m + S).
// Each tile is read and written by its own workgroup only.  One wave per 16 x 16
// quarter of the tile; bound by the latency of its loads (all three matrices
// are requested together) and of the two dependent products: 6.6 us a launch,
// against 16 with the products on the vector units from LDS and U_P requested
// after the first.
__global__ __launch_bounds__(256) void bj_apply_k(double* A, double* V, int n, int nb, int k,
                                                  const double* Ug, const int* flags) {
  if (flags[0]) return;
  const int m = nb / 2, tid = threadIdx.x;
  const int rows = (n + BJ2 - 1) / BJ2;
  const bool is_a = blockIdx.y == 0;
  if (blockIdx.x >= unsigned(is_a ? m * m : rows * m)) return;
  __shared__ double2 X[BJ2][BJ2 + 1];
  __shared__ double2 W[BJ2][BJ2 + 1];
  __shared__ double2 L[BJ2][BJ2 + 1];
  const int P = blockIdx.x / m, Sx = blockIdx.x % m;
  auto row_of = [&](int t) { return is_a ? bj_index(nb, k, P, t) : P * BJ2 + t; };
  double* M = is_a ? A : V;
  const double2* us = reinterpret_cast<const double2*>(Ug) + size_t(Sx) * BJ2 * BJ2;
  const double2* up = reinterpret_cast<const double2*>(Ug) + size_t(is_a ? P : Sx) * BJ2 * BJ2;
  {
    const int j = tid % BJ2, c = bj_index(nb, k, Sx, j);
    double2 x[4], u[4], l[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = tid / BJ2 + 8 * q, r = row_of(i);
      const bool in = r < n && c < n;
      x[q] = ld2(M, n, in ? r : 0, in ? c : 0);
      if (!in) x[q] = make_double2(0.0, 0.0);
      u[q] = us[i * BJ2 + j];
      l[q] = up[i * BJ2 + j];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = tid / BJ2 + 8 * q;
      X[i][j] = x[q];
      W[i][j] = u[q];
      L[i][j] = l[q];
    }
  }
  __syncthreads();
  const int i0 = ((tid >> 6) & 1) * 16, j0 = (tid >> 7) * 16;
  const int mm = tid & 15, qq = (tid >> 4) & 3;
  d4 re, im;
  tile_product<false>(X, W, i0, j0, re, im);  // T = X U_S
  if (is_a) {
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 4; ++t) X[i0 + qq + 4 * t][j0 + mm] = make_double2(re[t], im[t]);
    __syncthreads();
    tile_product<true>(L, X, i0, j0, re, im);  // U_P^H T
  }
  const int c = bj_index(nb, k, Sx, j0 + mm);
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int r = row_of(i0 + qq + 4 * t);
    if (r < n && c < n) st2(M, n, r, c, make_double2(re[t], im[t]));
  }
}

// End of a sweep: off-diagonal and total squared Frobenius norms, first as
// partial sums of kConvBlocks workgroups (a strided share of the entries
// each), then summed in fixed order by one workgroup, which sets the
// convergence flag.
constexpr int kConvBlocks = 256;

__global__ __launch_bounds__(256) void eig_norm_part_k(const double* A, int n, double* part, const int* flags) {
  __shared__ double so[256], st[256];
  if (flags[0]) return;
  double off = 0.0, tot = 0.0;
  const size_t total = size_t(n) * n;
  for (size_t e = size_t(blockIdx.x) * 256 + threadIdx.x; e < total; e += size_t(kConvBlocks) * 256) {
    const int i = int(e / n), j = int(e % n);
    const double2 a = ld2(A, n, i, j);
    const double m2 = a.x * a.x + a.y * a.y;
    tot += m2;
    if (i != j) off += m2;
  }
  so[threadIdx.x] = off;
  st[threadIdx.x] = tot;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (int(threadIdx.x) < w) {
      so[threadIdx.x] += so[threadIdx.x + w];
      st[threadIdx.x] += st[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = so[0];
    part[2 * blockIdx.x + 1] = st[0];
  }
}

__global__ __launch_bounds__(kConvBlocks) void eig_conv_k(const double* part, int n, int* flags, int first) {
  __shared__ double so[kConvBlocks], st[kConvBlocks];
  if (flags[0]) return;
  so[threadIdx.x] = part[2 * threadIdx.x];
  st[threadIdx.x] = part[2 * threadIdx.x + 1];
  __syncthreads();
  for (int w = kConvBlocks / 2; w > 0; w >>= 1) {
    if (int(threadIdx.x) < w) {
      so[threadIdx.x] += so[threadIdx.x + w];
      st[threadIdx.x] += st[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0 && first) {
    reinterpret_cast<double*>(flags)[1] = st[0];
  } else if (threadIdx.x == 0) {
    const double tol = 64.0 * DBL_EPSILON * sqrt(double(n > 1 ? n : 1));
    flags[1] += 1;
    if (so[0] <= tol * tol * st[0]) flags[0] = 1;
  }
}

// Ascending order of the eigenvalues (ties by index): rank of each, d in
// order, and the status word (0 converged, else the sweeps made).
__global__ void eig_rank_k(const double* A, int n, int* rank, double* d, const int* flags,
                           int32_t* status) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) status[0] = flags[0] ? 0 : (flags[1] > 0 ? flags[1] : 1);
  if (i >= n) return;
  const double di = ld2(A, n, i, i).x;
  int r = 0;
  for (int j = 0; j < n; ++j) {
    const double dj = ld2(A, n, j, j).x;
    r += (dj < di || (dj == di && j < i)) ? 1 : 0;
  }
  rank[i] = r;
  d[r] = di;
}

// Q[:, rank[i]] = V[:, i]
__global__ void eig_permute_k(const double* V, int n, const int* rank, double* Q) {
  const size_t total = size_t(n) * n;
  for (size_t e = size_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total;
       e += size_t(gridDim.x) * blockDim.x) {
    const int r = int(e / n), i = int(e % n);
    st2(Q, n, r, rank[i], ld2(V, n, r, i));
  }
}

int grid_for(size_t total) {
  const size_t b = (total + 255) / 256;
  return int(b < 4096 ? (b > 0 ? b : 1) : 4096);
}

}  // namespace

int eig_blocks(int n) {
  const int nb = (n + BJ - 1) / BJ;
  return nb + (nb & 1) < 2 ? 2 : nb + (nb & 1);
}

size_t eig_work_bytes(int n) {
  const size_t mat = size_t(n) * n * 16;
  const size_t ug = size_t(eig_blocks(n) / 2) * BJ2 * BJ2 * 16;
  return 2 * mat + ug + size_t(2 * kConvBlocks) * sizeof(double) + size_t(n) * sizeof(int) + 4 * sizeof(int) +
         5 * 256;
}

hipError_t launch_eig_hermitian(const double* sigma, int n, double* Q, double* d, int32_t* status,
                                void* work, int max_sweeps, hipStream_t s) {
  const int nb = eig_blocks(n), m = nb / 2;
  char* w = static_cast<char*>(work);
  auto carve = [&w](size_t bytes) {
    char* p = w;
    w += (bytes + 255) / 256 * 256;
    return p;
  };
  double* A = reinterpret_cast<double*>(carve(size_t(n) * n * 16));
  double* V = reinterpret_cast<double*>(carve(size_t(n) * n * 16));
  double* Ug = reinterpret_cast<double*>(carve(size_t(m) * BJ2 * BJ2 * 16));
  double* part = reinterpret_cast<double*>(carve(size_t(2 * kConvBlocks) * sizeof(double)));
  int* rank = reinterpret_cast<int*>(carve(size_t(n) * sizeof(int)));
  int* flags = reinterpret_cast<int*>(carve(4 * sizeof(int)));
  const size_t total = size_t(n) * n;
  hipLaunchKernelGGL(eig_init_k, dim3(grid_for(total)), dim3(256), 0, s, sigma, n, A, V, flags);
  if (n > 1) {
    hipLaunchKernelGGL(eig_norm_part_k, dim3(kConvBlocks), dim3(256), 0, s, A, n, part, flags);
    hipLaunchKernelGGL(eig_conv_k, dim3(1), dim3(kConvBlocks), 0, s, part, n, flags, 1);
    const int rows = (n + BJ2 - 1) / BJ2;
    const int tiles = m * m > rows * m ? m * m : rows * m;
    for (int sweep = 0; sweep < max_sweeps; ++sweep) {
      for (int k = 0; k < nb - 1; ++k) {
        hipLaunchKernelGGL(bj_solve_k, dim3(m), dim3(256), 0, s, A, n, nb, k, Ug, flags, int(sweep == 0));
        hipLaunchKernelGGL(bj_apply_k, dim3(tiles, 2), dim3(256), 0, s, A, V, n, nb, k, Ug, flags);
      }
      hipLaunchKernelGGL(eig_norm_part_k, dim3(kConvBlocks), dim3(256), 0, s, A, n, part, flags);
      hipLaunchKernelGGL(eig_conv_k, dim3(1), dim3(kConvBlocks), 0, s, part, n, flags, 0);
    }
  } else {
    hipLaunchKernelGGL(eig_norm_part_k, dim3(kConvBlocks), dim3(256), 0, s, A, n, part, flags);
    hipLaunchKernelGGL(eig_conv_k, dim3(1), dim3(kConvBlocks), 0, s, part, n, flags, 0);
  }
  hipLaunchKernelGGL(eig_rank_k, dim3((n + 255) / 256), dim3(256), 0, s, A, n, rank, d, flags, status);
  hipLaunchKernelGGL(eig_permute_k, dim3(grid_for(total)), dim3(256), 0, s, V, n, rank, Q);
  return hipGetLastError();
}

}  // namespace px
