// Complex contractions of the ACE construction and application on MFMA
// (gfx950 matrix cores):
//
//   xhy:  M[a][b] = scale * sum_r conj(X[a][r]) Y[b][r]     (M = dV Psi^H W,
//                                                           C = dV xi^H Phi)
//   xc :  Z[b][r] = alpha * sum_a X[a][r] C[a][b]           (xi = W U,
//                                                           Y = -xi C)
//
// X, Y, Z are orbital blocks [orb][N_g] (complex128 or complex64), C and M are
// small complex128 matrices.  A complex product takes three real MFMAs
// (Gauss): for (a + ib)(c + id), k1 = (a + b) c, k2 = a (d - c),
// k3 = b (c + d), re = k1 - k3, im = k1 + k2, with b = -Im x for the
// conjugated left operand of xhy.  The operand sums are formed in registers
// from the loaded values; against four MFMAs per product this is 9 % faster
// for the ACE application in both forms (512 x 512 x 72^3), at a few more
// accumulator registers.  MFMA: v_mfma_f64_16x16x4f64 (FP64 form) or
// v_mfma_f32_16x16x4f32 (FP32 form).  Operand layout of both 16x16x4 instructions: lane l supplies
// A[l%16][l/16] and B[l/16][l%16].  The result layouts differ: item t of lane
// l holds D[4*(l/16)+t][l%16] for f32 but D[l/16+4*t][l%16] for f64 (checked
// on gfx950 with a one-hot B operand).
//
// xhy splits the long r sum across workgroups; each writes FP64 partials that
// a second kernel adds in a fixed order (deterministic).  In the FP32 form
// the MFMA accumulators cover at most 1024 consecutive r before they are
// added into FP64 registers, which keeps the contraction error near 1e-8.
#include "fft_core.hpp"
#include "px_internal.hpp"

namespace px {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef double vd2g __attribute__((ext_vector_type(2)));
typedef float vf2g __attribute__((ext_vector_type(2)));

template <typename T> struct Acc;
template <> struct Acc<double> { using t = d4; };
template <> struct Acc<float> { using t = f4; };

__device__ __forceinline__ d4 mfma(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <typename T> __device__ __forceinline__ cpx<T> load_c(const cpx<T>* p) {
  if constexpr (sizeof(T) == 8) {
    vd2g v = *reinterpret_cast<const vd2g*>(p);
    return {v.x, v.y};
  } else {
    vf2g v = *reinterpret_cast<const vf2g*>(p);
    return {v.x, v.y};
  }
}

typedef float vf4g __attribute__((ext_vector_type(4)));

// Row of the 16x16 result held in item t of a lane with l/16 = q.
template <typename T> __device__ __forceinline__ int drow(int q, int t) {
  return sizeof(T) == 8 ? q + 4 * t : 4 * q + t;
}

constexpr int XHY_SUB = 1024;  // FP32 form: r-span of one FP32 accumulation

// 16 bytes per lane from global memory into LDS (lane l of the wave to the
// l-th 16 bytes of the wave-uniform destination).
__device__ __forceinline__ void dma16(const void* g, void* l) {
  __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)g,
                                   (void __attribute__((address_space(3)))*)l, 16, 0, 0);
}

// f(integral_constant NI, integral_constant NJ) with a wave's valid 16-wide
// tiles in each direction (0 to 2): sub-tiles past the matrix are not computed.
template <class F> __device__ __forceinline__ void by_tiles(int ni, int nj, F&& f) {
  using std::integral_constant;
  if (ni >= 2 && nj >= 2) f(integral_constant<int, 2>{}, integral_constant<int, 2>{});
  else if (ni >= 2 && nj == 1) f(integral_constant<int, 2>{}, integral_constant<int, 1>{});
  else if (ni == 1 && nj >= 2) f(integral_constant<int, 1>{}, integral_constant<int, 2>{});
  else if (ni == 1 && nj == 1) f(integral_constant<int, 1>{}, integral_constant<int, 1>{});
  else f(integral_constant<int, 0>{}, integral_constant<int, 0>{});
}

// ---------------------------------------------------------------- xhy
// grid (ceil(na/64), ceil(nb/64), nsplit), 256 threads; wave w covers the
// 32x32 sub-block (w&1, w>>1) as 2x2 MFMA tiles.  tri > 0 (a Hermitian result,
// na = nb): only the tiles (ta, tb) with ta <= tb of the tri x tri tile grid are
// computed, blockIdx.x enumerating them row by row; the reduction mirrors the
// others.
//
// Stages of 256 bytes of each row (32 complex64, 16 complex128) of the 64 + 64
// rows go through LDS by global -> LDS transfers, the next stage moving while
// one is multiplied.  The two stages are arrays of their own: LDS reads that
// may alias a transfer in flight would wait for it.  16-byte piece c of row i
// sits at slot c ^ (i & 7), so that eight rows' same pieces lie in eight
// different 16-byte columns (no bank conflicts), which the transfer's free
// choice of source addresses gives at no cost.  Rows past the matrix repeat
// its last row, pieces past the chunk its last piece (masked in the last stage,
// which has a copy of the loop body of its own: a masked path inside the loop
// cost 80 registers).
//
// Bound by the matrix cores: 6 na nb N_g real operations at 157 TFLOP/s (FP32)
// or 79 (FP64).  512 x 512 x 72^3 FP32 (with xc, the ACE application) 12.25 ->
// 9.75 ms, 120 TFLOP/s, against operands loaded by every wave from global memory into
// registers with masks; 200 x 200 x 48^3 FP64 1.82 -> 1.34 ms, of which the
// 16-wide tiles past 200 that are no longer computed are a third.
struct XhyStage { static constexpr int ROW = 256, BYTES = 128 * ROW; };  // X rows, then Y rows
// WIDE: lane offsets of 64 bits, formed at every transfer.  The 32-bit offsets
// (kept in registers, added to a scalar base by the transfer itself) reach three
// rows of N_g and a chunk with its last stage rounded up: N_g below about 89.5
// million in FP64, 179 million in FP32.
constexpr bool xhy_wide(size_t ng, size_t kchunk, size_t sz) {
  return 3 * ng * sz + kchunk * sz + 2 * XhyStage::ROW > (size_t(1) << 32);
}
static_assert(!xhy_wide(size_t(447) * 447 * 447, 1 << 18, 16) && xhy_wide(size_t(448) * 448 * 448, 0, 16), "FP64 edge");
static_assert(!xhy_wide(size_t(562) * 562 * 562, 1 << 19, 8) && xhy_wide(size_t(564) * 564 * 564, 0, 8), "FP32 edge");
static_assert(xhy_wide(size_t(67200000), 67200000, 16), "the whole sum in one chunk");
template <typename T, bool WIDE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void gemm_xhy_k(int na, int nb, size_t ng, const cpx<T>* X,
                                                  const cpx<T>* Y, double* part, size_t kchunk,
                                                  int tri) {
  using A = typename Acc<T>::t;
  constexpr int SZ = int(sizeof(cpx<T>)), KT = XhyStage::ROW / SZ;  // r of a stage
  __shared__ __attribute__((aligned(16))) char st0[XhyStage::BYTES], st1[XhyStage::BYTES];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int ta = blockIdx.x, tb = blockIdx.y;
  if (tri > 0) {  // wave-uniform decode of the upper-triangle tile index
    int k = blockIdx.x;
    ta = 0;
    while (k >= tri - ta) {
      k -= tri - ta;
      ++ta;
    }
    tb = ta + k;
  }
  const int a_base = ta * 64 + (w & 1) * 32;
  const int b_base = tb * 64 + (w >> 1) * 32;
  const size_t r_begin = size_t(blockIdx.z) * kchunk;
  const size_t r_end = (r_begin + kchunk < ng) ? r_begin + kchunk : ng;
  const int q = lane >> 4, m = lane & 15;

  // transfers: waves 0 and 1 move X's rows, 2 and 3 Y's, four rows each time
  // (a wave-uniform row and a lane offset of up to three rows more)
  using Off = typename std::conditional<WIDE, size_t, unsigned>::type;
  const bool isx = w < 2;
  const int row0 = (isx ? ta : tb) * 64 + (w & 1) * 32, rlim = (isx ? na : nb) - 1;
  const char* const src = reinterpret_cast<const char*>(isx ? X : Y) + r_begin * SZ;
  auto row_off = [&](int i, int ql) {
    const int r = row0 + 4 * i < rlim ? row0 + 4 * i : rlim;
    return Off(r + ql < rlim ? ql : rlim - r) * Off(ng * SZ);
  };
  unsigned off[WIDE ? 1 : 8];
  if constexpr (!WIDE) {
#pragma unroll
    for (int i = 0; i < 8; ++i) off[i] = row_off(i, q);
  }
  const Off last = Off((r_end - r_begin) * SZ) - 16;  // the chunk's last piece
  auto stage_in = [&](int k, char* st) {
    char* const dst = st + w * 32 * XhyStage::ROW;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = row0 + 4 * i < rlim ? row0 + 4 * i : rlim;
      const Off c = Off(k) * XhyStage::ROW + Off((m ^ ((4 * i + q) & 7)) * 16);
      int ql = q;
      if constexpr (WIDE) __asm__("" : "+v"(ql));  // (not kept over the loop: spills)
      const Off o = WIDE ? row_off(i, ql) : Off(off[WIDE ? 0 : i]);
      dma16(src + size_t(r) * ng * SZ + (o + (c < last ? c : last)), dst + i * 4 * XhyStage::ROW);
    }
  };

  // Gauss's three products: with x = a + ib (a = xr, b = -xi) and y = c + id,
  // k1 = (a + b) c, k2 = a (d - c), k3 = b (c + d); re = k1 - k3, im = k1 + k2
  A k1[2][2], k2[2][2], k3[2][2];
  double dre[2][2][4], dim[2][2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      k1[i][j] = k2[i][j] = k3[i][j] = A{0, 0, 0, 0};
#pragma unroll
      for (int t = 0; t < 4; ++t) dre[i][j][t] = dim[i][j][t] = 0.0;
    }
  const int nst = int((r_end - r_begin + KT - 1) / KT);
  const int rem = int((r_end - r_begin) - size_t(nst - 1) * KT);  // r of the last stage

  const int ni = a_base >= na ? 0 : a_base + 16 >= na ? 1 : 2;
  const int nj = b_base >= nb ? 0 : b_base + 16 >= nb ? 1 : 2;
  by_tiles(ni, nj, [&](auto nic, auto njc) {
    constexpr int NI = decltype(nic)::value, NJ = decltype(njc)::value;
    // a stage: four k-steps of 4 r per 16 r; lane q holds r = 4 q + s of them
    constexpr int PS = 16 / SZ;  // values of r in a piece
    auto multiply = [&](const char* st, auto tail) {
      if constexpr (NI > 0) {
        const char* const xr = st + ((w & 1) * 32 + m) * XhyStage::ROW;
        const char* const yr = st + (64 + (w >> 1) * 32 + m) * XhyStage::ROW;
#pragma unroll
        for (int h = 0; h < KT / (4 * PS); ++h) {
          // piece of this lane: PS values of r, the same k-steps for all rows
          const int r0 = SZ == 8 ? 16 * (h / 2) + 4 * q + 2 * (h % 2) : 4 * q + h;
          const int slot = ((r0 / PS) ^ (m & 7)) * 16;
          cpx<T> xa[NI][PS], yb[NJ][PS];
          auto get = [&](const char* row, cpx<T>(&v)[PS]) {
            if constexpr (SZ == 8) {
              const vf4g x = *reinterpret_cast<const vf4g*>(row + slot);
              v[0] = {x.x, x.y};
              v[1] = {x.z, x.w};
            } else {
              v[0] = load_c(reinterpret_cast<const cpx<T>*>(row + slot));
            }
            if constexpr (decltype(tail)::value) {
#pragma unroll
              for (int s = 0; s < PS; ++s)
                if (r0 + s >= rem) v[s] = {T(0), T(0)};
            }
          };
#pragma unroll
          for (int i = 0; i < NI; ++i) get(xr + i * 16 * XhyStage::ROW, xa[i]);
#pragma unroll
          for (int j = 0; j < NJ; ++j) get(yr + j * 16 * XhyStage::ROW, yb[j]);
#pragma unroll
          for (int s = 0; s < PS; ++s) {
            T xs[NI], yd[NJ], ys[NJ];
#pragma unroll
            for (int i = 0; i < NI; ++i) xs[i] = xa[i][s].x - xa[i][s].y;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
              yd[j] = yb[j][s].y - yb[j][s].x;
              ys[j] = yb[j][s].x + yb[j][s].y;
            }
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
              for (int j = 0; j < NJ; ++j) {
                k1[i][j] = mfma(xs[i], yb[j][s].x, k1[i][j]);
                k2[i][j] = mfma(xa[i][s].x, yd[j], k2[i][j]);
                k3[i][j] = mfma(-xa[i][s].y, ys[j], k3[i][j]);
              }
          }
        }
      }
    };
    auto flush = [&] {  // FP32 accumulators to FP64
      if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              dre[i][j][t] += double(k1[i][j][t]) - double(k3[i][j][t]);
              dim[i][j][t] += double(k1[i][j][t]) + double(k2[i][j][t]);
            }
            k1[i][j] = k2[i][j] = k3[i][j] = A{0, 0, 0, 0};
          }
      }
    };
    auto step = [&](int k, const char* cur, char* nxt) {
      stage_in(k + 1, nxt);
      multiply(cur, std::false_type{});
      dma_sync();
    };
    stage_in(0, st0);
    dma_sync();
    int k = 0;
    for (; k + 2 < nst; k += 2) {
      step(k, st0, st1);
      step(k + 1, st1, st0);
      // FP32 accumulators span at most XHY_SUB values of r
      if ((k + 2) % (XHY_SUB / KT) == 0) flush();
    }
    if (k + 1 < nst) step(k++, st0, st1);
    multiply(k % 2 ? st1 : st0, std::true_type{});  // the last stage, masked
    flush();
  });
  double* out = part + size_t(blockIdx.z) * na * nb * 2;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int a = a_base + 16 * i + drow<T>(q, t), b = b_base + 16 * j + m;
        if (a < na && b < nb) {
          double re, im;
          if constexpr (sizeof(T) == 4) {
            re = dre[i][j][t];
            im = dim[i][j][t];
          } else {
            re = k1[i][j][t] - k3[i][j][t];
            im = k1[i][j][t] + k2[i][j][t];
          }
          out[(size_t(a) * nb + b) * 2] = re;
          out[(size_t(a) * nb + b) * 2 + 1] = im;
        }
      }
}

// Sum of the splits' partials of each entry: R threads of a workgroup take every
// R-th split of 256 / R neighbouring entries, and the first of them adds the R
// sums in order.  R > 1 where the splits are many (small matrices): with one
// thread per entry, 108 splits of a 16 x 16 matrix were one workgroup's serial
// loop.  ACE application, us, R = 1 -> R = 16: 24^3 x 16 FP32 (108 splits) 36.7 -> 25.8, 48^3 x
// 64 (494) 189 -> 78, 60^3 x 128 (128) 423 -> 397; at 32 splits 16^3 x 16 23.9 -> 25.9, but
// the time step at 48^3 x 200 8,780 -> 8,740; below that equal.
template <int R>
__global__ __launch_bounds__(256) void xhy_reduce_k(int na, int nb, const double* part, int nsplit, double scale,
                             double* M, int ldm, float* M32, int herm) {
  constexpr int E = 256 / R;
  __shared__ double2 sum[R > 1 ? R : 1][R > 1 ? E : 1];
  const size_t n = size_t(na) * nb;
  const int le = threadIdx.x % E, row = threadIdx.x / E;
  for (size_t e0 = size_t(blockIdx.x) * E; e0 < n; e0 += size_t(gridDim.x) * E) {
    const size_t e = e0 + le;
    const bool in = e < n;
    const size_t a = in ? e / nb : 0, b = in ? e % nb : 0;
    // a Hermitian result keeps only the tiles on and above the diagonal:
    // entries below it are the conjugates of their mirror images
    const bool mirror = herm && (a / 64) > (b / 64);
    const size_t src = mirror ? b * nb + a : a * nb + b;
    double re = 0.0, im = 0.0;
    for (int s = row; s < nsplit; s += R) {
      const double2 v = *reinterpret_cast<const double2*>(part + (size_t(s) * n + src) * 2);
      re += v.x;
      im += v.y;
    }
    if constexpr (R > 1) {
      __syncthreads();  // the previous entries have been added
      sum[row][le] = make_double2(re, im);
      __syncthreads();
      if (row > 0) continue;
#pragma unroll
      for (int k = 1; k < R; ++k) {
        re += sum[k][le].x;
        im += sum[k][le].y;
      }
    }
    if (!in) continue;
    if (mirror) im = -im;
    M[(a * ldm + b) * 2] = scale * re;
    M[(a * ldm + b) * 2 + 1] = scale * im;
    if (M32) {  // the same, rounded to FP32 (operand of an FP32 contraction)
      M32[(a * ldm + b) * 2] = float(scale * re);
      M32[(a * ldm + b) * 2 + 1] = float(scale * im);
    }
  }
}

// r-span of one split: aim at one round of resident workgroups (two per CU on
// 256 CUs), at least 128 values of r, and at most max_split splits (the partials
// need max_split * na * nb complex128 values of scratch).  Among 1 to 2 times
// the aimed split count the one whose workgroups best fill whole rounds is
// taken: the workgroups of a launch all run about equally long, so a last round
// half full idles half the chip for one workgroup's time (ACE application at
// 96^3 x 1536: 4 -> 8 splits, about -2 %).  herm counts the tiles on and above
// the diagonal that the Hermitian form launches.  Against four rounds of at
// least 1024 values (the contraction with its reduction, us): 16 x 16 x 24^3
// FP32 31 -> 11, 64 x 64 x 48^3 FP32 106 -> 47, 200 x 200 x 48^3 FP64 871 ->
// 828, 300 x 300 x 60 x 60 x 90 FP32 1883 -> 1870; at least 64 values: 48^3
// a fifth slower again (more partials to add).
constexpr size_t kMinChunk = 128;
static size_t xhy_kchunk(int na, int nb, size_t ng, int max_split, bool herm, int* nsplit) {
  constexpr size_t kResident = 2 * 256;
  const size_t ta = size_t(na + 63) / 64, tb = size_t(nb + 63) / 64;
  const size_t tiles = herm ? ta * (ta + 1) / 2 : ta * tb;
  const size_t want0 = (kResident + tiles - 1) / tiles;
  size_t want = want0;
  double best = 0.0;
  for (size_t s = want0; s <= 2 * want0; ++s) {
    const size_t wg = tiles * s, rounds = (wg + kResident - 1) / kResident;
    const double fill = double(wg) / double(rounds * kResident);
    if (fill > best + 1e-9) {
      best = fill;
      want = s;
    }
  }
  size_t kchunk = (ng + want - 1) / want;
  if (kchunk < kMinChunk) kchunk = kMinChunk;
  if (max_split > 0 && (ng + kchunk - 1) / kchunk > size_t(max_split))
    kchunk = (ng + size_t(max_split) - 1) / size_t(max_split);
  kchunk = (kchunk + 15) / 16 * 16;
  *nsplit = int((ng + kchunk - 1) / kchunk);
  return kchunk;
}

size_t gemm_xhy_part_elems(int na, int nb, size_t ng, int* nsplit, bool herm, int max_split) {
  xhy_kchunk(na, nb, ng, max_split, herm, nsplit);
  return size_t(*nsplit) * na * nb;
}

int gemm_xhy_splits(int na, int nb, size_t ng, int max_split) {
  int nsplit = 0;
  xhy_kchunk(na, nb, ng, max_split, false, &nsplit);
  return nsplit;
}

static hipError_t xhy_launch(bool fp32, int na, int nb, size_t ng, const void* X, const void* Y,
                             double scale, double* M, int ldm, double* part, int nsplit_avail,
                             float* M32, bool herm, hipStream_t s) {
  int nsplit;
  const size_t kchunk = xhy_kchunk(na, nb, ng, nsplit_avail, herm, &nsplit);
  if (nsplit > nsplit_avail || (herm && na != nb)) return hipErrorInvalidValue;
  const int ta = (na + 63) / 64, tb = (nb + 63) / 64;
  const int tri = herm ? ta : 0;
  dim3 grid(herm ? ta * (ta + 1) / 2 : ta, herm ? 1 : tb, nsplit);
  auto run = [&](auto t, auto wide) {
    using T = decltype(t);
    hipLaunchKernelGGL((gemm_xhy_k<T, decltype(wide)::value>), grid, dim3(256), 0, s, na, nb, ng,
                       static_cast<const cpx<T>*>(X), static_cast<const cpx<T>*>(Y), part, kchunk, tri);
  };
  const bool wide = xhy_wide(ng, kchunk, fp32 ? 8 : 16);
  if (fp32 && wide) run(float{}, std::true_type{});
  else if (fp32) run(float{}, std::false_type{});
  else if (wide) run(double{}, std::true_type{});
  else run(double{}, std::false_type{});
  const size_t n = size_t(na) * nb;
  const bool many = nsplit >= 32;
  const size_t blocks = many ? (n + 15) / 16 : (n + 255) / 256;
  const dim3 rg(unsigned(blocks < 4096 ? blocks : 4096));
  if (many)
    hipLaunchKernelGGL(xhy_reduce_k<16>, rg, dim3(256), 0, s, na, nb, part, nsplit, scale, M, ldm, M32, int(herm));
  else
    hipLaunchKernelGGL(xhy_reduce_k<1>, rg, dim3(256), 0, s, na, nb, part, nsplit, scale, M, ldm, M32, int(herm));
  return hipGetLastError();
}

hipError_t launch_gemm_xhy(bool fp32, int na, int nb, size_t ng, const void* X, const void* Y,
                           double scale, double* M, int ldm, double* part, int nsplit_avail,
                           float* M32, hipStream_t s) {
  return xhy_launch(fp32, na, nb, ng, X, Y, scale, M, ldm, part, nsplit_avail, M32, false, s);
}

hipError_t launch_gemm_xhy_herm(bool fp32, int n, size_t ng, const void* X, const void* Y,
                                double scale, double* M, double* part, int nsplit_avail,
                                hipStream_t s) {
  return xhy_launch(fp32, n, n, ng, X, Y, scale, M, n, part, nsplit_avail, nullptr, true, s);
}

// ---------------------------------------------------------------- xc
// grid ceil(ng/64) * ceil(nb/64) in one dimension.  Dense C: the b tile
// varies fastest, so the workgroups that share an r tile of X run together
// and read it through the caches once, and each XCD (every eighth workgroup)
// keeps a few b column blocks of C in its L2 (ACE application at 96^3 x 1536
// -2 %, at 72^3 x 512 -6 %, against r tiles fastest).  Upper-triangular C
// (upper): the r tile varies fastest, so the workgroups in flight share one b
// tile and the same sum length (b-fastest mixes lengths 1 to nb/64 and was
// 21 % slower for xi = W U at 96^3 x 1536).  256 threads; wave w covers
// r-block (w&1) and b-block (w>>1) of 32 each, as 2x2 MFMA tiles (i: r,
// j: b).  Occupancy
// targets (no spills): three waves per SIMD in the FP32 form, two in FP64
// (one by default; ACE application in FP64 -15 %).
//
// Stages of KT rows a: 64 values of r of X by global -> LDS transfers (the
// next stage moving while one is multiplied), 64 columns b of C through
// registers (its rows need not be 16-byte aligned).  FP32: 16-byte piece c of
// row a sits at slot c ^ 8 (a & 3), so that the four rows that one read covers
// lie in different banks.  A is C^T and B is X: a lane's results then have one r and
// the stores of 16 lanes are contiguous.
template <typename T> struct XcStage {
  static constexpr int SZ = int(sizeof(cpx<T>)), KT = 128 / SZ, ROW = 64 * SZ, BYTES = KT * ROW;
  static constexpr int NC = KT * 64 / 256;  // entries of C per thread
  static __device__ __forceinline__ int at(int a, int c) {  // byte offset of entry (a, c)
    const int b = c * SZ;
    return a * ROW + (SZ == 8 ? b ^ ((a & 3) << 7) : b);
  }
};
//
// UPD: the fixed point's update in place of the store of Z (see launch_ptim_xc).
// The product is rounded to T first, so the results are those of a pass of its
// own over Z, which cost (with the midpoint pass) five block passes more:
// 300 x 60 x 60 x 90 FP32, an iteration 4.4 -> 3.9 ms.
template <typename T> struct Update {
  const cpx<T>* phi_n;
  const cpx<T>* y;    // nullable
  const cpx<T>* cur;
  cpx<T>* nxt;
  cpx<T>* mid;        // nullable
  double c;
  double* partial;    // two per workgroup
};
// REAL: C has no imaginary part, two products instead of Gauss's three (the z
// interpolation of the fine density, 16 orbitals, 72^3 FP64: 344 -> 262 us).
// WIDE: the lane offset of X in 64 bits (FP32, where a transfer spans two rows,
// from about 537 million N_g; an FP64 transfer stays within one).
template <typename T> constexpr bool xc_wide(size_t ng) {
  return sizeof(T) == 4 && (ng + 128) * sizeof(cpx<T>) > (size_t(1) << 32);
}
static_assert(!xc_wide<float>(size_t(812) * 812 * 812) && xc_wide<float>(size_t(1) << 29), "FP32 edge");
template <typename T, bool UPD, bool REAL, bool WIDE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 3 : 2))) void gemm_xc_k(int na, int nb, size_t ng, const cpx<T>* X,
                                                 const T* C, int ldc, double alpha,
                                                 cpx<T>* Z, int upper, Update<T> u) {
  using A = typename Acc<T>::t;
  using S = XcStage<T>;
  constexpr int KT = S::KT, SZ = S::SZ;
  __shared__ __attribute__((aligned(16))) char xs0[S::BYTES], xs1[S::BYTES], cs0[S::BYTES], cs1[S::BYTES];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const unsigned nbt = unsigned(nb + 63) / 64, nrt = unsigned((ng + 63) / 64);
  const int bt = int(upper ? blockIdx.x / nrt : blockIdx.x % nbt);
  const size_t rt = upper ? blockIdx.x % nrt : blockIdx.x / nbt;
  const size_t r_base = rt * 64 + (w & 1) * 32;
  const int b_base = bt * 64 + (w >> 1) * 32;
  const int q = lane >> 4, m = lane & 15;
  int a_end = na;
  if (upper) {
    const int lim = bt * 64 + 64;
    a_end = lim < na ? lim : na;
  }
  // Gauss's three products (x = a + ib, C entry c + id): k1 = (a + b) c,
  // k2 = a (d - c), k3 = b (c + d); re = k1 - k3, im = k1 + k2.  [j][i]: b, r
  A k1[2][2], k2[2][2], k3[2][2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < 2; ++i) k1[j][i] = k2[j][i] = k3[j][i] = A{0, 0, 0, 0};
  const int nst = (a_end + KT - 1) / KT;

  // X: each transfer of a wave moves 1 KiB (two rows of complex64, one of
  // complex128); rows past a_end repeat the last, values past N_g the last piece
  constexpr int LPR = S::ROW / 16, RPT = 64 / LPR, NX = S::BYTES / 4096;
  // (a wave-uniform row and a lane offset of at most one row more)
  using Off = typename std::conditional<WIDE, size_t, unsigned>::type;
  const int xrow = lane / LPR;
  const unsigned rmax = unsigned(ng - rt * 64 < 64 ? ng - rt * 64 : 64) - 16 / SZ;
  const cpx<T>* const xt = X + rt * 64;
  auto x_in = [&](int k, char* st) {
#pragma unroll
    for (int i = 0; i < NX; ++i) {
      const int al = (w * NX + i) * RPT;  // first row within the stage
      const int a = k * KT + al < a_end ? k * KT + al : a_end - 1;
      const int ar = a + xrow < a_end ? xrow : 0;
      // the entry that belongs at this lane's slot (its piece's first)
      const unsigned c = unsigned(SZ == 8 ? (((lane % LPR) * 16) ^ (((al + xrow) & 3) << 7)) / SZ : lane % LPR);
      dma16(reinterpret_cast<const char*>(xt + size_t(a) * ng) + (Off(ar) * Off(ng) + (c < rmax ? c : rmax)) * Off(SZ),
            st + (w * NX + i) * 1024);
    }
  };
  // C: entry e = tid + 256 i of the stage (zero past the matrix)
  cpx<T> cr[S::NC];
  const int cb = bt * 64 + lane;
  auto c_get = [&](int k) {
#pragma unroll
    for (int i = 0; i < S::NC; ++i) {
      const int a = k * KT + w + 4 * i;  // wave-uniform
      const cpx<T> c = load_c(reinterpret_cast<const cpx<T>*>(C) + size_t(a < a_end ? a : 0) * ldc + unsigned(cb < nb ? cb : 0));
      cr[i] = a < a_end && cb < nb ? c : cpx<T>{T(0), T(0)};
    }
  };
  auto c_put = [&](char* st) {
#pragma unroll
    for (int i = 0; i < S::NC; ++i)
      *reinterpret_cast<cpx<T>*>(st + S::at(w + 4 * i, lane)) = cr[i];
  };

  const int nj = b_base >= nb ? 0 : b_base + 16 >= nb ? 1 : 2;
  const int ni = r_base >= ng ? 0 : r_base + 16 >= ng ? 1 : 2;
  by_tiles(ni, nj, [&](auto nic, auto njc) {
    constexpr int NI = decltype(nic)::value, NJ = decltype(njc)::value;
    auto multiply = [&](const char* xs, const char* cs, int left, auto tail) {
      if constexpr (NI > 0) {
#pragma unroll
        for (int s = 0; s < KT / 4; ++s) {
          const int a = 4 * s + q;
          cpx<T> x[NI], c[NJ];
#pragma unroll
          for (int i = 0; i < NI; ++i) {
            x[i] = load_c(reinterpret_cast<const cpx<T>*>(xs + S::at(a, (w & 1) * 32 + 16 * i + m)));
            if (decltype(tail)::value && a >= left) x[i] = {T(0), T(0)};
          }
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            c[j] = load_c(reinterpret_cast<const cpx<T>*>(cs + S::at(a, (w >> 1) * 32 + 16 * j + m)));
          T xq[NI], cd[NJ], cq[NJ];
#pragma unroll
          for (int i = 0; i < NI; ++i) xq[i] = x[i].x + x[i].y;
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            cd[j] = c[j].y - c[j].x;
            cq[j] = c[j].x + c[j].y;
          }
#pragma unroll
          for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int i = 0; i < NI; ++i) {
              if constexpr (REAL) {  // re = k1, im = k2
                k1[j][i] = mfma(c[j].x, x[i].x, k1[j][i]);
                k2[j][i] = mfma(c[j].x, x[i].y, k2[j][i]);
              } else {
                k1[j][i] = mfma(c[j].x, xq[i], k1[j][i]);
                k2[j][i] = mfma(cd[j], x[i].x, k2[j][i]);
                k3[j][i] = mfma(cq[j], x[i].y, k3[j][i]);
              }
            }
          if (s % 2 == 1) __builtin_amdgcn_sched_barrier(0);  // two steps' operands at a time
        }
      }
    };
    auto step = [&](int k, const char* xs, const char* cs, char* xn, char* cn) {
      c_put(cn);  // stage k + 1
      x_in(k + 1, xn);
      c_get(k + 2);
      multiply(xs, cs, KT, std::false_type{});
      dma_sync();
    };
    x_in(0, xs0);
    c_get(0);
    c_put(cs0);
    c_get(1);
    dma_sync();
    int k = 0;
    for (; k + 2 < nst; k += 2) {
      step(k, xs0, cs0, xs1, cs1);
      step(k + 1, xs1, cs1, xs0, cs0);
    }
    if (k + 1 < nst) step(k++, xs0, cs0, xs1, cs1);
    multiply(k % 2 ? xs1 : xs0, k % 2 ? cs1 : cs0, a_end - k * KT, std::true_type{});  // the last stage, masked
  });
  const T al = T(alpha);
  [[maybe_unused]] double dd = 0.0, nn = 0.0;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int b = b_base + 16 * j + drow<T>(q, t);
      if (b >= nb) continue;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const size_t r = r_base + 16 * i + m;
        if (r >= ng) continue;
        const size_t e = size_t(b) * ng + r;
        const cpx<T> z = REAL ? cpx<T>{al * k1[j][i][t], al * k2[j][i][t]}
                              : cpx<T>{al * (k1[j][i][t] - k3[j][i][t]), al * (k1[j][i][t] + k2[j][i][t])};
        if constexpr (UPD) {
          double vr = double(z.x), vi = double(z.y);
          if (u.y) {  // the two terms are added in FP64
            const cpx<T> y = load_c(u.y + e);
            vr = double(y.x) + vr;
            vi = double(y.y) + vi;
          }
          const cpx<T> p = load_c(u.phi_n + e), o0 = load_c(u.cur + e);
          // -i c (vr + i vi) = c vi - i c vr
          const cpx<T> o = {T(double(p.x) + u.c * vi), T(double(p.y) - u.c * vr)};
          u.nxt[e] = o;
          if (u.mid) u.mid[e] = {T(0.5) * (p.x + o.x), T(0.5) * (p.y + o.y)};
          const double dr = double(o.x) - double(o0.x), di = double(o.y) - double(o0.y);
          dd += dr * dr + di * di;
          nn += double(o.x) * double(o.x) + double(o.y) * double(o.y);
        } else {
          Z[e] = z;
        }
      }
    }
  if constexpr (UPD) {
    double* const red = reinterpret_cast<double*>(xs0);  // [2][256]
    __syncthreads();
    red[tid] = dd;
    red[256 + tid] = nn;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
      if (tid < off) {
        red[tid] += red[tid + off];
        red[256 + tid] += red[256 + tid + off];
      }
      __syncthreads();
    }
    if (tid < 2) u.partial[2 * size_t(blockIdx.x) + tid] = red[256 * tid];
  }
}

static dim3 xc_grid(int nb, size_t ng) { return dim3(unsigned((ng + 63) / 64) * unsigned((nb + 63) / 64)); }

template <typename T, bool REAL>
static void xc_run(int na, int nb, size_t ng, const void* X, const void* C, int ldc, double alpha, void* Z, bool upper,
                   hipStream_t s) {
  auto run = [&](auto wide) {
    hipLaunchKernelGGL((gemm_xc_k<T, false, REAL, decltype(wide)::value>), xc_grid(nb, ng), dim3(256), 0, s, na, nb, ng,
                       static_cast<const cpx<T>*>(X), static_cast<const T*>(C), ldc, alpha,
                       static_cast<cpx<T>*>(Z), int(upper), Update<T>{});
  };
  if constexpr (sizeof(T) == 4 && !REAL) {
    if (xc_wide<T>(ng)) return run(std::true_type{});
  }
  run(std::false_type{});
}

hipError_t launch_gemm_xc(bool fp32, int na, int nb, size_t ng, const void* X, const void* C,
                          int ldc, double alpha, void* Z, bool upper, hipStream_t s) {
  if (fp32) xc_run<float, false>(na, nb, ng, X, C, ldc, alpha, Z, upper, s);
  else xc_run<double, false>(na, nb, ng, X, C, ldc, alpha, Z, upper, s);
  return hipGetLastError();
}

hipError_t launch_gemm_xc_real(bool fp32, int na, int nb, size_t ng, const void* X, const void* C, int ldc,
                               void* Z, hipStream_t s) {
  if (fp32 && xc_wide<float>(ng)) return hipErrorInvalidValue;
  if (fp32) xc_run<float, true>(na, nb, ng, X, C, ldc, 1.0, Z, false, s);
  else xc_run<double, true>(na, nb, ng, X, C, ldc, 1.0, Z, false, s);
  return hipGetLastError();
}

// res = sqrt(sum dd / sum nn) over n pairs of partials, fixed order.
__global__ __launch_bounds__(1024) void residual_k(const double* partial, size_t n, double* res) {
  __shared__ double rd[1024], rn[1024];
  double a = 0.0, b = 0.0;
  for (size_t k = threadIdx.x; k < n; k += 1024) {
    a += partial[2 * k];
    b += partial[2 * k + 1];
  }
  rd[threadIdx.x] = a;
  rn[threadIdx.x] = b;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if (int(threadIdx.x) < w) {
      rd[threadIdx.x] += rd[threadIdx.x + w];
      rn[threadIdx.x] += rn[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) *res = sqrt(rd[0] / rn[0]);
}

size_t ptim_xc_partials(int nb, size_t ng) { return size_t(xc_grid(nb, ng).x) * 2; }

template <typename T>
static void ptim_xc(int na, int nb, size_t ng, const void* X, const void* C, int ldc, const PtimUpdate& p,
                    hipStream_t s) {
  const Update<T> u = {static_cast<const cpx<T>*>(p.phi_n), static_cast<const cpx<T>*>(p.y),
                       static_cast<const cpx<T>*>(p.cur), static_cast<cpx<T>*>(p.nxt),
                       static_cast<cpx<T>*>(p.mid), p.c, p.partial};
  auto run = [&](auto wide) {
    hipLaunchKernelGGL((gemm_xc_k<T, true, false, decltype(wide)::value>), xc_grid(nb, ng), dim3(256), 0, s, na, nb, ng,
                       static_cast<const cpx<T>*>(X), static_cast<const T*>(C), ldc, -1.0,
                       static_cast<cpx<T>*>(nullptr), 0, u);
  };
  if constexpr (sizeof(T) == 4) {
    if (xc_wide<T>(ng)) return run(std::true_type{});
  }
  run(std::false_type{});
}

hipError_t launch_ptim_xc(bool fp32, int na, int nb, size_t ng, const void* X, const void* C, int ldc,
                          const PtimUpdate& p, hipStream_t s) {
  if (fp32) ptim_xc<float>(na, nb, ng, X, C, ldc, p, s);
  else ptim_xc<double>(na, nb, ng, X, C, ldc, p, s);
  hipLaunchKernelGGL(residual_k, dim3(1), dim3(1024), 0, s, p.partial, size_t(xc_grid(nb, ng).x), p.res);
  return hipGetLastError();
}

}  // namespace px
