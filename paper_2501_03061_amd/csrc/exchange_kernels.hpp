// The fused pair pipeline of the exchange operator (Eq. 13 with occupations f_j):
//
//   (Vx phi_i)(r) = -sum_j f_j psi_j(r) * IFFT[ K(G) * FFT(conj(psi_j) * phi_i) ](r)
//
// over a chunk of orbital pairs (i, j) in passes that each keep a piece of a
// pair's grid in LDS:
//
//   pass 1  (z tile, i) : pair product conj(psi_j)*phi_i, forward z transform,
//                         written to the pair buffer T.
//   pass 2  (xy slab, pair): forward y and x transforms, multiply by K(G) (and,
//                         in FP32 form, the G = 0 coefficient taken from FP64
//                         tile sums), FP64 partial of sum_G K |rho(G)|^2 for
//                         the exchange energy, inverse x and y transforms; in
//                         place.
//   pass 3  (z tile)    : inverse z transform, then the weighted sums over the
//                         chunk's pairs, kept in registers: per output orbital
//                         i, sum_j f_j/N_g psi_j v_ij, and in the Hermitian-pair
//                         mode for the transposed pairs (v_ji = conj v_ij) also
//                         sum_i f_i/N_g psi_i conj(v_ij) for every j.
//   pass 4  (Hermitian-pair mode): adds the sums over groups of j that pass 3
//                         left in the pair buffer to the output orbitals i.
//
// A z tile is W consecutive points of the xy plane times all z: small enough
// that the sums of several orbitals fit the registers of one workgroup, which
// is why z is the axis of the first and the last transform.  The pair slab
// makes four trips to memory (written by pass 1, read and written by pass 2,
// read by pass 3), and v_ij itself is never stored: pass 3 writes one sum per
// group of GJ pairs of a row, which pass 4 reads back (2/GJ of a slab per pair
// instead of two).
//
// Layout of every grid array: [n2][n1][n0] with x = n0 fastest; orbital blocks
// are orbital-major.  T is float (complex64 data) or double (complex128).
#pragma once
#include "fft_core.hpp"
#include "px_internal.hpp"

namespace px {

// Global-memory access through address-space-1 pointers.  The chunk
// arguments arrive in a struct (or a task table), so the compiler cannot
// prove that their pointers are global and would otherwise emit flat
// instructions, which count against the LDS wait counter as well: every
// wait for an LDS access would then also wait for the prefetched slabs.
#define PX_GLOBAL __attribute__((address_space(1)))
template <typename V> __device__ __forceinline__ V gld(const V* p) {
  return *(const PX_GLOBAL V*)p;
}
template <typename V> __device__ __forceinline__ void gst(V* p, V v) {
  *(PX_GLOBAL V*)p = v;
}

// Element at lane byte offset `off` plus the constant `step` elements from a
// wave-uniform base, as a raw buffer access: base, size and step are scalar
// operands and the lane offset has 32 bits, so that a load or store needs no
// vector address arithmetic (global accesses with such a base took two 64-bit
// vector additions each, once the compiler had moved the offset's extension
// out of the loop).
template <typename T> struct Raw;
template <> struct Raw<float> { typedef unsigned v __attribute__((ext_vector_type(2))); };
template <> struct Raw<double> { typedef unsigned v __attribute__((ext_vector_type(4))); };
template <typename T> __device__ __forceinline__ __amdgpu_buffer_rsrc_t view(const cpx<T>* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<cpx<T>*>(base), 0, -1, 0x00020000);
}
template <typename T, int AUX>
__device__ __forceinline__ cpx<T> ld_raw(__amdgpu_buffer_rsrc_t b, unsigned off, int step) {
  const int so = step * int(sizeof(cpx<T>));
  if constexpr (sizeof(T) == 4) return __builtin_bit_cast(cpx<T>, __builtin_amdgcn_raw_buffer_load_b64(b, off, so, AUX));
  else return __builtin_bit_cast(cpx<T>, __builtin_amdgcn_raw_buffer_load_b128(b, off, so, AUX));
}
template <typename T, int AUX>
__device__ __forceinline__ void st_raw(__amdgpu_buffer_rsrc_t b, unsigned off, int step, cpx<T> x) {
  const int so = step * int(sizeof(cpx<T>));
  using R = typename Raw<T>::v;
  if constexpr (sizeof(T) == 4) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(R, x), b, off, so, AUX);
  else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(R, x), b, off, so, AUX);
}
// Cached, and with the streaming (non-temporal) policy: a pair slab is read
// once by the next pass, so it should not displace the orbital tiles that the
// current pass re-reads from the caches.
template <typename T> __device__ __forceinline__ cpx<T> ldc(__amdgpu_buffer_rsrc_t b, unsigned off, int step) { return ld_raw<T, 0>(b, off, step); }
template <typename T> __device__ __forceinline__ cpx<T> ldg(__amdgpu_buffer_rsrc_t b, unsigned off, int step) { return ld_raw<T, 2>(b, off, step); }
template <typename T> __device__ __forceinline__ void stg(__amdgpu_buffer_rsrc_t b, unsigned off, int step, cpx<T> x) { st_raw<T, 0>(b, off, step, x); }
template <typename T> __device__ __forceinline__ void stn(__amdgpu_buffer_rsrc_t b, unsigned off, int step, cpx<T> x) { st_raw<T, 2>(b, off, step, x); }

// Twiddle table of a second stage of span NS: t[r NS + k] = exp(-2 pi i r k / N)
// from the compile-time roots (FP64, about one ulp) rounded to T; written into
// LDS by each workgroup.
template <typename T, int N, int NS, int NT> __device__ __forceinline__ void fill_stage_table(cpx<T>* t) {
  constexpr const RootTable<N>& tab = kRoots<N>;
  for (int m = threadIdx.x; m < N; m += NT) {
    const int e = (m / NS) * (m % NS);  // < N
    t[m] = {T(tab.c[e]), T(-tab.s[e])};
  }
}

// One DPP step on an FP64 value (both 32-bit halves moved with the same
// control).  With ROW_MASK = 0xF every lane is written; otherwise lanes of the
// rows outside the mask receive 0.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_f64(double v) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  int lo, hi;
  if constexpr (ROW_MASK == 0xF) {
    lo = __builtin_amdgcn_mov_dpp(int(unsigned(u)), CTRL, 0xF, 0xF, false);
    hi = __builtin_amdgcn_mov_dpp(int(unsigned(u >> 32)), CTRL, 0xF, 0xF, false);
  } else {
    lo = __builtin_amdgcn_update_dpp(0, int(unsigned(u)), CTRL, ROW_MASK, 0xF, false);
    hi = __builtin_amdgcn_update_dpp(0, int(unsigned(u >> 32)), CTRL, ROW_MASK, 0xF, false);
  }
  return __builtin_bit_cast(double, (static_cast<unsigned long long>(unsigned(hi)) << 32) | unsigned(lo));
}

// FP64 sum over the 64 lanes of a wave, returned wave-uniform.  Data-parallel
// moves only: pair and quad swaps, half-row and row mirrors (every lane of a
// 16-lane row then holds the row sum), then the GFX9 row broadcasts of lanes
// 15 and 31, after which lane 63 holds the total.
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_f64<0xB1, 0xF>(v);   // quad_perm [1,0,3,2]
  v += dpp_f64<0x4E, 0xF>(v);   // quad_perm [2,3,0,1]
  v += dpp_f64<0x141, 0xF>(v);  // row_half_mirror
  v += dpp_f64<0x140, 0xF>(v);  // row_mirror
  v += dpp_f64<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
  v += dpp_f64<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = __builtin_amdgcn_readlane(int(unsigned(u)), 63);
  const unsigned hi = __builtin_amdgcn_readlane(int(unsigned(u >> 32)), 63);
  return __builtin_bit_cast(double, (static_cast<unsigned long long>(hi) << 32) | lo);
}


// Occupancy target of a kernel: the waves per SIMD of a CU that holds as many
// workgroups of nt threads and lds_bytes of LDS as fit, at most cap, so that
// the register allocation does not become the tighter limit.  A workgroup
// takes ceil(waves / 4) wave slots on every SIMD (counters: six-wave
// workgroups with registers for five waves per SIMD ran two per CU, not three).
constexpr int lds_waves_per_simd(int lds_bytes, int nt, int cap) {
  const int per = (nt + 255) / 256;
  int wgs = (160 * 1024) / lds_bytes;
  while (wgs > 1 && wgs * per > cap) --wgs;
  const int w = wgs * per;
  return w > 8 ? 8 : w;
}
constexpr int round64(int n) { return (n + 63) / 64 * 64; }
// Workgroup size for the register allocation: whole waves on every SIMD.
constexpr int round256(int n) { return (n + 255) / 256 * 256; }

// ============================================================== z tiles
// Geometry of the z-tile passes on an N0 x N1 x N2 grid: W points of the plane
// (the last tile is short when W does not divide N0 N1: its lanes past the
// plane load a valid point and store nothing).  A thread holds RS points of a
// tile, one butterfly of the stage of that radix: the first of the forward and
// the last of the inverse transform, where the product (pass 1) and the sums
// (pass 3) happen.  The other stage has RB = N2 / RS.
template <int N2> constexpr int ztile_radix() {
  return Plan<N2>::rad[0] == 8 ? Plan<N2>::rad[1] : Plan<N2>::rad[0];
}
// Pass 3 in FP64 takes the plan's smaller radix: its GJ + 1 sums of RS points
// then fit the registers with more columns (96^3: 8 points with GJ = 3 6.4 us a
// pair in passes 3 and 4, 12 with GJ = 2 8.9).
template <typename T, int N2> constexpr int ztile_radix3() {
  constexpr int a = Plan<N2>::rad[0], b = Plan<N2>::rad[1];
  return sizeof(T) == 4 ? ztile_radix<N2>() : a < b ? a : b;
}
template <typename T, int N0, int N1, int N2, int W, int RS_ = ztile_radix<N2>()> struct ZTile {
  static constexpr int PL = N0 * N1;
  static constexpr int NTILE = (PL + W - 1) / W;
  static constexpr bool RAG = PL % W != 0;
  static constexpr int RS = RS_, RB = N2 / RS;
  static constexpr bool FWD = Plan<N2>::rad[0] == RS;  // radix order of the forward transform
  using F0 = StageOf<N2, 0, !FWD>;
  using FL = StageOf<N2, 1, !FWD>;
  using I0 = StageOf<N2, 0, FWD>;
  using IL = StageOf<N2, 1, FWD>;
  static_assert(F0::R == RS && FL::R == RB && I0::R == RB && IL::R == RS, "stage order");
  static constexpr int NBS = W * RB;             // butterflies of the radix-RS stage
  static constexpr int NBB = W * RS;             // and of the radix-RB stage
  static constexpr int NT = round64(NBS);
  static constexpr int SB = (NBB + NT - 1) / NT; // slots of a thread in the radix-RB stage
};

// Tile and row of a workgroup in a grid of tile_grid(NTILE) x rows.  Workgroups
// go to the 8 XCDs in turn by linear id; XCD x takes the x-th eighth of the
// tiles, each with its rows one after the other, so that the rows' workgroups,
// which read the same tiles of the density orbitals, share one L2.  Against
// workgroups in launch order: pass 1 at 96^3 FP64 5.6 -> 3.2 us a pair, at 72^3
// FP32 0.87 -> 0.68 (every eighth tile instead of a run of tiles per XCD: up to
// 10% slower in pass 3).
constexpr int tile_grid(int ntile) { return (ntile + 7) / 8 * 8; }
__device__ __forceinline__ void tile_order(int& tile, int& row) {
  const int nt = int(gridDim.x), nr = int(gridDim.y);
  const int id = int(blockIdx.x) + int(blockIdx.y) * nt, k = id >> 3;
  tile = (id & 7) * (nt / 8) + k / nr;
  row = k % nr;
}

// ============================================================== pass 1
// Workgroup = (tile, output orbital i), looping over the chunk's j; the next
// density orbital's tile is in flight while the current one is transformed.
// Four waves per SIMD in FP32 (five gave the same, with spills; 120 planes spill
// with four), FP64 as the registers come out (two).
template <typename T, int N0, int N1, int N2, int W, bool G0>
__global__ __launch_bounds__((round256(ZTile<T, N0, N1, N2, W>::NT))) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 1 : N2 > 96 ? 3 : 4)))
void pass1_z(ChunkArgs a0, const ChunkArgs* tasks) {
  using Z = ZTile<T, N0, N1, N2, W>;
  using FL = typename Z::FL;
  constexpr int NT = Z::NT, RS = Z::RS, RB = Z::RB, PL = Z::PL, NW = NT / 64;
  const ChunkArgs a = chunk_args(a0, tasks);
  int tile, ii;
  tile_order(tile, ii);
  if (tile >= Z::NTILE || ii >= a.ic) return;
  __shared__ cpx<T> lds[N2 * W];
  __shared__ cpx<T> tw[N2];
  // G = 0 sums: every thread leaves its FP32 partials in LDS and one wave per
  // sum adds them in FP64 after the barrier that follows the first stage
  __shared__ T gpart[G0 ? 3 * NT : 1];
  fill_stage_table<T, N2, FL::NS, NT>(tw);
  const int tid = threadIdx.x;
  // the last SW waves add the three G = 0 sums, GPW each
  constexpr int SW = NW >= 4 ? 3 : 1, GPW = SW == 3 ? 1 : 3;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t0 = tile * W;
  const int jend = a.tri ? ii + 1 : a.jc;  // pairs jj < jend of row ii
  const size_t ng = size_t(PL) * N2;
  const cpx<T>* phi = reinterpret_cast<const cpx<T>*>(a.phi) + size_t(a.i0 + ii) * ng;
  const cpx<T>* psi0 = reinterpret_cast<const cpx<T>*>(a.psi) + size_t(a.j0) * ng;

  const bool live0 = Z::NBS % NT == 0 || tid < Z::NBS;
  const int b0 = live0 ? tid : Z::NBS - 1;  // (threads past the last butterfly repeat it)
  const int l0 = b0 % W, j0 = b0 / W;
  const bool in0 = !Z::RAG || t0 + l0 < PL;
  const unsigned off0 = unsigned(j0 * PL + (in0 ? t0 + l0 : PL - 1)) * unsigned(sizeof(cpx<T>));
  cpx<T> ph[RS], nx[RS];
#pragma unroll
  for (int r = 0; r < RS; ++r) ph[r] = ldc<T>(view(phi), off0, r * RB * PL);
#pragma unroll
  for (int r = 0; r < RS; ++r) nx[r] = ldc<T>(view(psi0), off0, r * RB * PL);
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): nothing outstanding when a loop starts
  __syncthreads();

  // The waves take one of two loops, so that within each every pair issues the
  // same memory operations: the compiler's wait for the prefetched tile then
  // counts the stores issued after it instead of waiting for them too.  The
  // last waves (the fewest butterflies of the last stage) add the G = 0
  // partials in FP64; lanes past the last butterfly repeat it (the same values
  // to the same addresses).
  auto loop = [&](auto slots_c, auto sums_c) {
    constexpr int SLOTS = decltype(slots_c)::value;
    constexpr bool SUMS = decltype(sums_c)::value;
    for (int jj = 0; jj < jend; ++jj) {
      const int p = ii * a.jc + jj;
      cpx<T> v[RS];
      T fen = T(0);
      // product and first butterfly.  G = 0 (FP32 form): the thread's few
      // products are summed in FP32 (the butterfly's DC output is that sum), the
      // partials in FP64.  These are the transform's own inputs; with random
      // rounding the partial sums add about 1e-10 relative to the coefficient of
      // a diagonal pair, far below the FP32 transform's error.
#pragma unroll
      for (int r = 0; r < RS; ++r) {
        v[r] = cmulc(nx[r], ph[r]);
        if (G0) fen += v[r].x * v[r].x + v[r].y * v[r].y;
      }
      // the next density orbital's tile (the last pair requests its own again)
      const auto pn = view(psi0 + size_t(jj + 1 < jend ? jj + 1 : jj) * ng);
#pragma unroll
      for (int r = 0; r < RS; ++r) nx[r] = ldc<T>(pn, off0, r * RB * PL);
      dft<T, RS, false>(v);
      if constexpr (G0) {
        const bool cnt = live0 && in0;
        gpart[tid] = cnt ? v[0].x : T(0);
        gpart[NT + tid] = cnt ? v[0].y : T(0);
        gpart[2 * NT + tid] = cnt ? fen : T(0);
      }
#pragma unroll
      for (int r = 0; r < RS; ++r) lds[out_pos<RS, 1>(j0, r) * W + l0] = v[r];
      lds_sync();
      if constexpr (G0 && SUMS) {
        double* g = reinterpret_cast<double*>(a.g0 + size_t(p) * Z::NTILE + tile);
#pragma unroll
        for (int k = 0; k < GPW; ++k) {
          int c = (wave - (NW - SW)) * GPW + k;
          c = c < 2 ? c : 2;
          double sc = 0.0;
#pragma unroll
          for (int q = 0; q < NW; ++q) sc += double(gpart[c * NT + q * 64 + (tid & 63)]);
          gst(g + c, wave_sum(sc));  // (every lane, one address)
        }
      }
      const auto out = view(reinterpret_cast<cpx<T>*>(a.t) + size_t(p) * ng);
#pragma unroll
      for (int k = 0; k < SLOTS; ++k) {
        int b = tid + k * NT;
        if (Z::NBB % NT != 0) b = b < Z::NBB ? b : Z::NBB - 1;
        const int l1 = b % W, j1 = b / W;
        cpx<T> u[RB];
#pragma unroll
        for (int r = 0; r < RB; ++r) u[r] = lds[(j1 + r * RS) * W + l1];
        twiddle<T, N2, RB, FL::NS, false>(u, j1, tw);
        dft<T, RB, false>(u);
        if (!Z::RAG || t0 + l1 < PL) {
          const unsigned off1 = unsigned(j1 * PL + t0 + l1) * unsigned(sizeof(cpx<T>));
#pragma unroll
          for (int r = 0; r < RB; ++r) stn<T>(out, off1, r * RS * PL, u[r]);
        }
      }
      lds_sync();
    }
  };
  using std::integral_constant;
  // slots of the waves before and from NW - SW on
  constexpr int S0 = Z::SB, S1 = NW > SW ? (Z::NBB - (NW - SW) * 64 + NT - 1) / NT : Z::SB;
  constexpr int S1C = S1 < 0 ? 0 : S1;
  if (NW > SW && wave < NW - SW) loop(integral_constant<int, S0>{}, integral_constant<bool, false>{});
  else loop(integral_constant<int, S1C>{}, integral_constant<bool, true>{});
}

template <typename T, int CFG> constexpr int tile_width() { return ztile_width(sizeof(T) == 4, CFG); }

// ============================================================== pass 2
// Workgroup = the xy slab at kz = blockIdx.x of pq consecutive pairs; the
// kernel values of the slab are loaded once.  y first and last: a row of the
// slab is then one contiguous run of lanes for the global loads and stores,
// and the x lines are read with the line index across lanes (odd row pitch: no
// bank conflicts in either direction).  The kernel table is [z][x][y] for the
// same reason.  The inverse x transform starts with the forward's last radix,
// so the two meet in registers around the kernel multiply.
template <typename T, int N0, int N1> struct Slab {
  static constexpr int P0 = N0 + 1;
  using GX = Lines<N0, N1, P0, 1, true>;
  using GY = Lines<N1, N0, 1, P0, true>;
};
template <typename T, int N0, int N1, int NT> constexpr int slab_lds_bytes() {
  return (N1 * (N0 + 1) + 2 * N0 + (N0 == N1 ? 2 : 2 * N1)) * int(sizeof(cpx<T>)) + (NT / 64) * 16 + 64;
}

// NA: threads that take butterflies (see slab_threads).
template <bool FIRST, class A, class B> __device__ __forceinline__ auto& pick(A& a, B& b) {
  if constexpr (FIRST) return a;
  else return b;
}
template <typename T, int N0, int N1, int N2, int NTILE, int NA, bool G0, bool EX, bool PF>
__global__ __launch_bounds__(round256(NA)) __attribute__((amdgpu_waves_per_eu(
    lds_waves_per_simd(slab_lds_bytes<T, N0, N1, round64(NA)>(), NA, 4))))
void pass2_xy(ChunkArgs a0, const ChunkArgs* tasks, int pq) {
  using S = Slab<T, N0, N1>;
  using GX = typename S::GX;
  using GY = typename S::GY;
  constexpr int P0 = S::P0, NT = round64(NA), NW = NT / 64, PL = N0 * N1;
  const ChunkArgs a = chunk_args(a0, tasks);
  const int np = chunk_pairs(a);
  const int z = blockIdx.x, qbeg = int(blockIdx.y) * pq;
  if (qbeg >= np) return;
  const int qend = qbeg + pq < np ? qbeg + pq : np;
  __shared__ cpx<T> lds[N1 * P0];
  // twiddles of the second stages: forward and inverse x, forward and inverse y
  constexpr bool SQ = N0 == N1;
  __shared__ cpx<T> tfx[N0], tix[N0], tfy_[SQ ? 1 : N1], tiy_[SQ ? 1 : N1];
  __shared__ double red[2][NW];
  __shared__ double gsum[2], red0;
  __shared__ double esum[EX ? kSlabPairs : 1][3];
  // forward y in the order whose first stage, which loads, has the fuller slots
  constexpr int YA = StageOf<N1, 0, false>::R, YB = StageOf<N1, 1, false>::R;
  constexpr bool YREV = slots<GY, YB, NA>() * YB < slots<GY, YA, NA>() * YA;
  using Y0 = StageOf<N1, 0, YREV>;
  using Y1 = StageOf<N1, 1, YREV>;
  using X0 = StageOf<N0, 0, false>;
  using X1 = StageOf<N0, 1, false>;
  using J0 = StageOf<N0, 0, true>;   // inverse x
  using J1 = StageOf<N0, 1, true>;
  using V0 = StageOf<N1, 0, !YREV>;  // inverse y
  using V1 = StageOf<N1, 1, !YREV>;
  // (equal axes: a table depends on the length and the span only)
  cpx<T>* const tfy = !SQ ? tfy_ : Y1::NS == X1::NS ? tfx : tix;
  cpx<T>* const tiy = !SQ ? tiy_ : V1::NS == J1::NS ? tix : tfx;
  static_assert(J0::R == X1::R, "inverse must start with the forward's last radix");
  using KT = typename std::conditional<G0, float, double>::type;
  const int tid = threadIdx.x;
  cpx<T>* const tz = reinterpret_cast<cpx<T>*>(a.t) + size_t(z) * PL;
  const size_t ng = size_t(PL) * N2;

  fill_stage_table<T, N0, X1::NS, NT>(tfx);
  fill_stage_table<T, N0, J1::NS, NT>(tix);
  if constexpr (!SQ) {
    fill_stage_table<T, N1, Y1::NS, NT>(tfy);
    fill_stage_table<T, N1, V1::NS, NT>(tiy);
  }
  // Twiddles of the second stages (x and y, forward and inverse).  Where a thread
  // has one butterfly in each stage, and LDS leaves the registers (one workgroup per
  // CU), its twiddles do not change from pair to pair and are kept: 72^3 FP64, pass 2
  // 2.90 -> 2.83 ms per 1000 pairs (98 -> 158 registers).
  constexpr bool KEEP = sizeof(T) == 8 && SQ && slots<GY, Y1::R, NA>() == 1 && slots<GY, V1::R, NA>() == 1 &&
                        Y1::R == X1::R && V1::R == J1::R && 2 * slab_lds_bytes<T, N0, N1, NT>() > 160 * 1024;
  cpx<T> wf[KEEP ? Y1::R - 1 : 1], wi[KEEP ? V1::R - 1 : 1];
  if constexpr (KEEP) {
    lds_sync();
    auto powers = [](auto& w, cpx<T> w1) {
      w[0] = w1;
#pragma unroll
      for (int r = 1; r < int(sizeof(w) / sizeof(w[0])); ++r) w[r] = cmul(w[r - 1], w1);
    };
    int line, j;
    slot<GY, Y1::R, NA>(tid, 0, line, j);
    powers(wf, tfy[Y1::NS + j % Y1::NS]);
    slot<GY, V1::R, NA>(tid, 0, line, j);
    const cpx<T> c = tiy[V1::NS + j % V1::NS];
    powers(wi, cpx<T>{c.x, -c.y});
  }
  auto kept = [](auto& w, cpx<T>* v) {
#pragma unroll
    for (int r = 0; r < int(sizeof(w) / sizeof(w[0])); ++r) v[r + 1] = cmul(v[r + 1], w[r]);
  };
  auto tw_y1 = [&](cpx<T>* v, int j) {
    if constexpr (KEEP) kept(wf, v);
    else twiddle<T, N1, Y1::R, Y1::NS, false>(v, j, tfy);
  };
  auto tw_x1 = [&](cpx<T>* v, int j) {
    if constexpr (KEEP) kept(wf, v);
    else twiddle<T, N0, X1::R, X1::NS, false>(v, j, tfx);
  };
  auto tw_j1 = [&](cpx<T>* v, int j) {
    if constexpr (KEEP) kept(wi, v);
    else twiddle<T, N0, J1::R, J1::NS, true>(v, j, tix);
  };
  auto tw_v1 = [&](cpx<T>* v, int j) {
    if constexpr (KEEP) kept(wi, v);
    else twiddle<T, N1, V1::R, V1::NS, true>(v, j, tiy);
  };
  auto no_tw = [](cpx<T>*, int) {};
  const auto ktab = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<KT*>(reinterpret_cast<const KT*>(a.kt) + size_t(z) * PL), 0, -1, 0x00020000);
  auto ld_real = [](__amdgpu_buffer_rsrc_t b, unsigned off, int step) {
    const int so = step * int(sizeof(KT));
    if constexpr (sizeof(KT) == 4) return __builtin_bit_cast(KT, __builtin_amdgcn_raw_buffer_load_b32(b, off, so, 0));
    else return __builtin_bit_cast(KT, __builtin_amdgcn_raw_buffer_load_b64(b, off, so, 0));
  };
  // PF: the slab of the next pair is requested after the kernel multiply (its
  // registers are free then and the kernel loads done) and arrives during the
  // inverse transforms.  (Requested right after its predecessor's first stage, with
  // the kernel values kept in registers: 72^3 FP64 2.95 ms per 1000 pairs against 2.88.)
  constexpr int S0 = slots<GY, Y0::R, NA>();
  static_assert(!PF || (N1 / Y0::R) % (NA / N0) == 0, "prefetch needs full slots");
  auto request = [&](__amdgpu_buffer_rsrc_t b, auto& v, int t, auto sc) {
#pragma unroll
    for (int k = 0; k < decltype(sc)::value; ++k) {
      int line, j;
      slot<GY, Y0::R, NA>(t, k, line, j);
#pragma unroll
      for (int r = 0; r < Y0::R; ++r)
        v[k][r] = ldg<T>(b, unsigned(j * N0 + line) * unsigned(sizeof(cpx<T>)), r * (N1 / Y0::R) * N0);
    }
  };
  cpx<T> nx[PF ? S0 : 1][Y0::R];
  if constexpr (PF) {
    request(view(tz + size_t(pair_slot(a, qbeg)) * ng), nx, tid, std::integral_constant<int, S0>{});
    __builtin_amdgcn_s_waitcnt(0x0f70);
  }
  for (int q = qbeg; q < qend; ++q) {
    const int p = pair_slot(a, q);
    const auto buf = view(tz + size_t(p) * ng);
    // the thread index, opaque to the compiler in every iteration: it would
    // otherwise keep the addresses of all stages in registers across the loop
    // (and spill them) instead of forming them where they are used
    int t = tid;
    __asm__("" : "+v"(t));
    if (G0 && z == 0 && tid >= NT - 64) {
      // G = 0 from the FP64 tile sums of pass 1, one wave, fixed order
      double s0 = 0.0, s1 = 0.0;
      const G0Part* g = a.g0 + size_t(p) * NTILE;
      for (int i = t & 63; i < NTILE; i += 64) {  // (t: with tid the addresses were kept, and spilled at 96^3)
        s0 += gld(&g[i].re);
        s1 += gld(&g[i].im);
      }
      s0 = wave_sum(s0);
      s1 = wave_sum(s1);
      if ((tid & 63) == 0) {
        gsum[0] = s0;
        gsum[1] = s1;
      }
    }
    // first forward y stage from global
    by_slots<GY, Y0::R, NA>([&](auto sc) {
      constexpr int SL = decltype(sc)::value;
      cpx<T> u[PF ? 1 : SL > 0 ? SL : 1][Y0::R];
      auto& v = pick<PF>(nx, u);
      if constexpr (!PF) request(buf, v, t, sc);
      lds_sync();  // twiddles written; the previous pair's last stage has read LDS
#pragma unroll
      for (int k = 0; k < SL; ++k) {
        int line, j;
        slot<GY, Y0::R, NA>(t, k, line, j);
        dft<T, Y0::R, false>(v[k]);
#pragma unroll
        for (int r = 0; r < Y0::R; ++r) lds[out_pos<Y0::R, 1>(j, r) * P0 + line] = v[k][r];
        __builtin_amdgcn_sched_barrier(0);
      }
      lds_sync();
    });
    stage_lds<T, GY, Y1::R, Y1::NS, false, NA>(lds, t, tw_y1);
    stage_lds<T, GX, X0::R, X0::NS, false, NA>(lds, t, no_tw);
    // last forward x stage into registers, kernel multiply, first inverse stage
    by_slots<GX, X1::R, NA>([&](auto sc) {
      constexpr int SL = decltype(sc)::value;
      cpx<T> v[SL > 0 ? SL : 1][X1::R];
      double ex = 0.0, en = 0.0, ex0 = 0.0;  // FP32 form: sum_{G!=0} K|rho|^2, sum_{G!=0} |rho|^2, G = 0 term
#pragma unroll
      for (int k = 0; k < SL; ++k) {
        int line, j;
        slot<GX, X1::R, NA>(t, k, line, j);
#pragma unroll
        for (int r = 0; r < X1::R; ++r) v[k][r] = lds[line * P0 + j + r * (N0 / X1::R)];
      }
      lds_sync();  // every thread has read its lines before they are overwritten
#pragma unroll
      for (int k = 0; k < SL; ++k) {
        int line, j;
        slot<GX, X1::R, NA>(t, k, line, j);
        KT kv[X1::R];
        const unsigned off = unsigned(j * N1 + line) * unsigned(sizeof(KT));
#pragma unroll
        for (int r = 0; r < X1::R; ++r) kv[r] = ld_real(ktab, off, r * (N0 / X1::R) * N1);
        tw_x1(v[k], j);
        dft<T, X1::R, false>(v[k]);
        T fex = T(0), fen = T(0);  // the butterfly's partial energy sums
#pragma unroll
        for (int r = 0; r < X1::R; ++r) {
          const cpx<T> c = v[k][r];
          const KT kg = kv[r];
          if (G0 && r == 0 && k == 0 && z == 0 && tid == 0) {
            // G = 0: butterfly 0 of line 0
            const double k0 = gld(a.kern);
            const double s0 = gsum[0], s1 = gsum[1];
            if (EX) ex0 = k0 * (s0 * s0 + s1 * s1);
            v[k][r] = {T(k0 * s0), T(k0 * s1)};
          } else {
            // FP32 form: K(G) rounded to FP32; the energy terms of the
            // thread's few values are summed in FP32, the partials in FP64
            // (random rounding: about 1e-10 relative on a pair's energy)
            if (EX) {
              const T c2 = c.x * c.x + c.y * c.y;
              fex += kg * c2;
              if (G0) fen += c2;
            }
            v[k][r] = {kg * c.x, kg * c.y};
          }
        }
        if constexpr (EX) {
          // lanes that repeat a butterfly do not count
          constexpr int STEP = NA / N1, NJ = N0 / X1::R;
          const bool own = (NA % 64 == 0 || tid < NA) && (NJ % STEP == 0 || tid / N1 + k * STEP < NJ);
          ex += own ? double(fex) : 0.0;
          if (G0) en += own ? double(fen) : 0.0;
        }
        dft<T, J0::R, true>(v[k]);
#pragma unroll
        for (int r = 0; r < J0::R; ++r) lds[line * P0 + out_pos<J0::R, 1>(j, r)] = v[k][r];
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (EX) {
        ex = wave_sum(ex);
        if (G0) en = wave_sum(en);
        if ((tid & 63) == 0) {
          red[0][tid >> 6] = ex;
          if (G0) red[1][tid >> 6] = en;
        }
        if (G0 && tid == 0) red0 = ex0;
      }
      lds_sync();
    });
    if constexpr (EX) {
      if (tid == 0) {
        double s2 = 0.0, s3 = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
          s2 += red[0][w];
          if (G0) s3 += red[1][w];
        }
        esum[q - qbeg][0] = s2;
        if constexpr (G0) {
          esum[q - qbeg][1] = s3;
          esum[q - qbeg][2] = red0;
        }
      }
    }
    if constexpr (PF)  // the next pair's slab (the last pair requests its own again)
      request(view(tz + size_t(pair_slot(a, q + 1 < qend ? q + 1 : q)) * ng), nx, t, std::integral_constant<int, S0>{});
    stage_lds<T, GX, J1::R, J1::NS, true, NA>(lds, t, tw_j1);
    stage_lds<T, GY, V0::R, V0::NS, true, NA>(lds, t, no_tw);
    // last inverse y stage back to global, in place
    by_slots<GY, V1::R, NA>([&](auto sc) {
      constexpr int SL = decltype(sc)::value;
#pragma unroll
      for (int k = 0; k < SL; ++k) {
        int line, j;
        slot<GY, V1::R, NA>(t, k, line, j);
        cpx<T> w[V1::R];
#pragma unroll
        for (int r = 0; r < V1::R; ++r) w[r] = lds[(j + r * (N1 / V1::R)) * P0 + line];
        tw_v1(w, j);
        dft<T, V1::R, true>(w);
#pragma unroll
        for (int r = 0; r < V1::R; ++r)
          stn<T>(buf, unsigned(j * N0 + line) * unsigned(sizeof(cpx<T>)), r * (N1 / V1::R) * N0, w[r]);
        __builtin_amdgcn_sched_barrier(0);
      }
    });
  }
  if constexpr (EX) {
    constexpr int NE = G0 ? 3 : 1;
    lds_sync();
    if (tid < (qend - qbeg) * NE)
      gst(a.expart + (size_t(pair_slot(a, qbeg + tid / NE)) * N2 + z) * NE + tid % NE, esum[tid / NE][tid % NE]);
  }
}

// ============================================================== pass 3
// Moves a z tile (N2 rows of W points, rows PL points apart) into LDS with
// 16-byte global -> LDS transfers: a wave moves 1 KiB pieces of consecutive
// rows, lane l the l-th 16 bytes (the LDS destination of a transfer is
// wave-uniform, its lanes fill consecutive 16-byte slots).  lim: bytes of the
// row that lie inside the plane (ragged last tile; lanes past it re-read its
// last 16 bytes).  Streaming policy: each slab is read once.
template <typename T, int N2, int W, int PL, int NT, bool RAG>
__device__ __forceinline__ void dma_tile(const cpx<T>* src, cpx<T>* dst, int lim) {
  constexpr int RBYTES = W * int(sizeof(cpx<T>)), LR = RBYTES / 16, RPI = 64 / LR;
  static_assert(RBYTES % 16 == 0 && 64 % LR == 0, "whole rows per transfer");
  constexpr int NW = NT / 64, NCH = (N2 + RPI - 1) / RPI;
  const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const int lane = int(threadIdx.x) & 63;
  int col = (lane % LR) * 16;
  if (RAG) col = col < lim ? col : lim - 16;
  const char PX_GLOBAL* g = (const char PX_GLOBAL*)(src);
  char __attribute__((address_space(3)))* l = (char __attribute__((address_space(3)))*)(dst);
#pragma unroll
  for (int q0 = 0; q0 < NCH; q0 += NW) {
    // every wave issues the same transfers: pieces (and rows) past the tile
    // repeat its last (the compiler's waits then count them)
    int q = q0 + w;
    if (NCH % NW != 0) q = q < NCH ? q : NCH - 1;
    int row = q * RPI + lane / LR;
    if (N2 % RPI != 0) row = row < N2 ? row : N2 - 1;
    __builtin_amdgcn_global_load_lds(
        (const void PX_GLOBAL*)(g + (unsigned(row) * unsigned(PL * sizeof(cpx<T>)) + unsigned(col))),
        (void __attribute__((address_space(3)))*)(l + q * 1024), 16, 0, 2);
  }
}

constexpr int kRowSum = 16;  // pairs of one FP32 sum in the general form
// Workgroup = (tile, i) looping over j (SYM = false), or (tile, group of GJ
// density orbitals j) looping over the rows i and within a row over the
// group's j (SYM).  One staging tile, filled by global -> LDS transfers while
// the previous pair is transformed, and one working tile.
// SYM: the sums over i of the group's GJ columns stay in registers for the
// whole chunk and end in one read-modify-write of the columns' output tiles;
// the sum over the group's j of a row goes to the tile of the row's first pair
// slab of the group (which this workgroup alone has just consumed), for pass 4.
template <typename T, int N0, int N1, int N2, int W, bool SYM, int GJ>
__global__ __launch_bounds__((round256(ZTile<T, N0, N1, N2, W, ztile_radix3<T, N2>()>::NT))) __attribute__((amdgpu_waves_per_eu(
    pass3_waves(sizeof(T) == 4, SYM, ZTile<T, N0, N1, N2, W, ztile_radix3<T, N2>()>::NT))))
void pass3_z(ChunkArgs a0, const ChunkArgs* tasks) {
  using Z = ZTile<T, N0, N1, N2, W, ztile_radix3<T, N2>()>;
  using IL = typename Z::IL;
  constexpr int NT = Z::NT, RS = Z::RS, RB = Z::RB, PL = Z::PL;
  const ChunkArgs a = chunk_args(a0, tasks);
  int tile, by;
  tile_order(tile, by);
  if (tile >= Z::NTILE || by * (SYM ? GJ : 1) >= (SYM ? a.jc : a.ic)) return;
  // staging: whole 1 KiB pieces (see dma_tile)
  constexpr int PIECE = 1024 / int(sizeof(cpx<T>));
  __shared__ __attribute__((aligned(16))) cpx<T> sbuf[(N2 * W + PIECE - 1) / PIECE * PIECE];
  __shared__ cpx<T> lds[N2 * W];
  __shared__ cpx<T> tw[N2];
  fill_stage_table<T, N2, IL::NS, NT>(tw);
  const int tid = threadIdx.x;
  const int t0 = tile * W;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const size_t ng = size_t(PL) * N2;
  const cpx<T>* tb = reinterpret_cast<const cpx<T>*>(a.t) + t0;
  const int lim = (PL - t0 < W ? PL - t0 : W) * int(sizeof(cpx<T>));
  // last inverse stage and sums: butterfly (j1, l1)
  const bool live1 = Z::NBS % NT == 0 || tid < Z::NBS;
  const int b1 = live1 ? tid : Z::NBS - 1;
  const int l1 = b1 % W, j1 = b1 / W;
  const bool in1 = live1 && (!Z::RAG || t0 + l1 < PL);
  const unsigned o1 = unsigned(j1 * PL + (!Z::RAG || t0 + l1 < PL ? t0 + l1 : PL - 1)) * unsigned(sizeof(cpx<T>));
  constexpr int RSTEP = RB * PL;  // between a thread's points
  const cpx<T>* psi = reinterpret_cast<const cpx<T>*>(a.psi);
  cpx<T>* const out = reinterpret_cast<cpx<T>*>(a.out);
  auto weight = [&](int orb) {
    // uniform: a scalar load (counted with the LDS operations, so that waiting
    // for it never waits for the tile transfer)
    return T(*(const __attribute__((address_space(4))) double*)(a.occ + orb) * a.inv_ng);
  };
  // Inverse z transform of the staged tile.  Once every thread has read it, the
  // next pair's tile starts to move into its place.  The psi_j tile is
  // requested before: memory requests complete in order, so the wait for it
  // never waits for the transfer.  (Staging and working tile are two arrays:
  // an LDS read that might alias a transfer's destination is made to wait for
  // the transfer, as it was with two exchanged buffers.)
  auto transform = [&](cpx<T>(&v)[RS], cpx<T>(&pc)[RS], const cpx<T>* pj, const cpx<T>* next) {
    const auto pjv = view(pj);
#pragma unroll
    for (int r = 0; r < RS; ++r) pc[r] = ldc<T>(pjv, o1, r * RSTEP);
    // first stage, the waves with a butterfly less by a path of their own
    // (branch-free slots, as in pass 2)
    auto first = [&](auto sc) {
      constexpr int SL = decltype(sc)::value;
      cpx<T> u[SL > 0 ? SL : 1][RB];
      auto pos = [&](int k, int& l, int& j) {
        int b = tid + k * NT;
        if (Z::NBB % NT != 0) b = b < Z::NBB ? b : Z::NBB - 1;
        l = b % W;
        j = b / W;
      };
#pragma unroll
      for (int k = 0; k < SL; ++k) {
        int l, j;
        pos(k, l, j);
#pragma unroll
        for (int r = 0; r < RB; ++r) u[k][r] = sbuf[(j + r * RS) * W + l];
      }
#pragma unroll
      for (int k = 0; k < SL; ++k) {
        int l, j;
        pos(k, l, j);
        dft<T, RB, true>(u[k]);
#pragma unroll
        for (int r = 0; r < RB; ++r) lds[out_pos<RB, 1>(j, r) * W + l] = u[k][r];
      }
    };
    if (Z::NBB % NT == 0 || wave * 64 + (Z::SB - 1) * NT < Z::NBB) first(std::integral_constant<int, Z::SB>{});
    else first(std::integral_constant<int, Z::SB - 1>{});
    lds_sync();
    // (outside of the two paths: on a path that does not issue it the compiler
    // would wait for everything)
    dma_tile<T, N2, W, PL, NT, Z::RAG>(next, sbuf, lim);
#pragma unroll
    for (int r = 0; r < RS; ++r) v[r] = lds[(j1 + r * RB) * W + l1];
    twiddle<T, N2, RS, IL::NS, true>(v, j1, tw);
    dft<T, RS, true>(v);
  };
  cpx<T> row[RS];
#pragma unroll
  for (int r = 0; r < RS; ++r) row[r] = {T(0), T(0)};

  if constexpr (!SYM) {
    const int ii = by;
    const cpx<T>* t = tb + size_t(ii) * a.jc * ng;
    dma_tile<T, N2, W, PL, NT, Z::RAG>(t, sbuf, lim);
    dma_sync();
    // FP32: sums of kRowSum pairs, added to a sum of sums.  (One running sum over a
    // chunk of 64 pairs against sums of 16: error of Vx at 24^3 x 100 1.76e-7
    // against 1.20e-7, at 48^3 x 130 1.65e-7 against 1.43e-7.)
    constexpr bool TWO = sizeof(T) == 4;
    cpx<T> sums[TWO ? RS : 1];
    if constexpr (TWO) {
#pragma unroll
      for (int r = 0; r < RS; ++r) sums[r] = {T(0), T(0)};
    }
    for (int jj = 0; jj < a.jc; ++jj) {
      const T wj = weight(a.j0 + jj);
      const cpx<T>* pj = psi + size_t(a.j0 + jj) * ng;
      cpx<T> pc[RS], v[RS];
      // (the last pair moves its own tile again: the same transfers on every pair)
      transform(v, pc, pj, t + size_t(jj + 1 < a.jc ? jj + 1 : jj) * ng);
#pragma unroll
      for (int r = 0; r < RS; ++r) {
        const cpx<T> c = cmul(pc[r], v[r]);
        row[r].x += wj * c.x;
        row[r].y += wj * c.y;
      }
      if constexpr (TWO) {
        if (jj % kRowSum == kRowSum - 1 || jj + 1 == a.jc) {
#pragma unroll
          for (int r = 0; r < RS; ++r) {
            sums[r] = cadd(sums[r], row[r]);
            row[r] = {T(0), T(0)};
          }
        }
      }
      dma_sync();
    }
    if constexpr (TWO) {
#pragma unroll
      for (int r = 0; r < RS; ++r) row[r] = sums[r];
    }
    cpx<T>* o = out + size_t(a.i0 + ii) * ng;
    cpx<T> prev[RS];
    if (!a.first) {
#pragma unroll
      for (int r = 0; r < RS; ++r) prev[r] = ldc<T>(view(o), o1, r * RSTEP);
    }
    if (in1) {
#pragma unroll
      for (int r = 0; r < RS; ++r) stg<T>(view(o), o1, r * RSTEP, csub(a.first ? cpx<T>{T(0), T(0)} : prev[r], row[r]));
    }
  } else {
    // psi_i's tile is kept for the group's pairs where the registers hold it
    // with the sums, and read again for each pair where the kernel would spill
    // (80^3, 96^3 and the non-cubic grids in FP64, ten-wave workgroups).  FP64,
    // 60 x 90 x 120, GJ = 2: 3.7 us a pair against 4.4 with 26 registers
    // spilled, or 4.6 and another 1.0 in pass 4 with GJ = 1; 72^3, where it
    // fits: 1.9 against 2.0 read again.
    constexpr bool AGAIN = (sizeof(T) == 8 && RS + RB >= 18) || NT > 512;
    const int jg = by * GJ;                  // first j of the group
    const int gn = a.jc - jg < GJ ? a.jc - jg : GJ;       // its j's
    const int ibeg = a.tri ? jg : 0;                      // triangular block: pairs jj <= ii
    cpx<T> col[GJ][RS];
#pragma unroll
    for (int u = 0; u < GJ; ++u)
#pragma unroll
      for (int r = 0; r < RS; ++r) col[u][r] = {T(0), T(0)};
    const cpx<T>* t = tb + (size_t(ibeg) * a.jc + jg) * ng;
    dma_tile<T, N2, W, PL, NT, Z::RAG>(t, sbuf, lim);
    dma_sync();
    for (int ii = ibeg; ii < a.ic; ++ii) {
      const int un = a.tri && ii - jg + 1 < gn ? ii - jg + 1 : gn;  // live pairs of the row
      const cpx<T>* ti = tb + (size_t(ii) * a.jc + jg) * ng;
      const T wi = weight(a.i0 + ii);
      cpx<T> pi[RS];
      const auto piv = view(psi + size_t(a.i0 + ii) * ng);
      if constexpr (!AGAIN) {
#pragma unroll
        for (int r = 0; r < RS; ++r) pi[r] = ldc<T>(piv, o1, r * RSTEP);
      }
#pragma unroll
      for (int u = 0; u < GJ; ++u) {
        if (u < un) {
          const T wj = weight(a.j0 + jg + u);
          const cpx<T>* pj = psi + size_t(a.j0 + jg + u) * ng;
          cpx<T> pc[RS], v[RS];
          const cpx<T>* next = u + 1 < un ? ti + size_t(u + 1) * ng
                             : ii + 1 < a.ic ? ti + size_t(a.jc) * ng : ti + size_t(u) * ng;
          transform(v, pc, pj, next);
          const bool diag = a.tri && jg + u == ii;  // the pair (i, i) counts once
          const T wc = diag ? T(0) : wi;
#pragma unroll
          for (int r = 0; r < RS; ++r) {
            const cpx<T> c = cmul(pc[r], v[r]);
            row[r].x += wj * c.x;
            row[r].y += wj * c.y;
          }
          if constexpr (AGAIN) {
            __builtin_amdgcn_sched_barrier(0);  // psi_j's registers are free now
#pragma unroll
            for (int r = 0; r < RS; ++r) pi[r] = ldc<T>(piv, o1, r * RSTEP);
          }
#pragma unroll
          for (int r = 0; r < RS; ++r) {
            // f_i/N_g psi_i conj(v)
            const cpx<T> d = cmulc(v[r], pi[r]);
            col[u][r].x += wc * d.x;
            col[u][r].y += wc * d.y;
          }
          dma_sync();
        }
      }
      if (in1) {
        cpx<T>* o = const_cast<cpx<T>*>(ti) - t0;
#pragma unroll
        for (int r = 0; r < RS; ++r) stn<T>(view(o), o1, r * RSTEP, row[r]);
      }
#pragma unroll
      for (int r = 0; r < RS; ++r) row[r] = {T(0), T(0)};
    }
    const bool init = a.first && a.tri;  // the block's first writer (a.first: pass 4 otherwise)
#pragma unroll
    for (int u = 0; u < GJ; ++u) {
      if (u < gn) {
        cpx<T>* o = out + size_t(a.j0 + jg + u) * ng;
        cpx<T> prev[RS];
        if (!init) {
#pragma unroll
          for (int r = 0; r < RS; ++r) prev[r] = ldc<T>(view(o), o1, r * RSTEP);
        }
        if (in1) {
#pragma unroll
          for (int r = 0; r < RS; ++r) stg<T>(view(o), o1, r * RSTEP, csub(init ? cpx<T>{T(0), T(0)} : prev[r], col[u][r]));
        }
      }
    }
  }
}

// ============================================================== host launcher
// Threads of a pass-2 workgroup that take butterflies (the workgroup has whole
// waves): a multiple of the line counts, so that a thread keeps its line, with
// one to four butterflies in each stage.  More threads hide less of the LDS round
// trips by independent butterflies and fill ragged slots worse, fewer run out of
// registers.  Pass 2 with the energy, ms per 1000 pairs, here against others:
//   FP32  24^3 192: 0.065, 96: 0.061 (with 16 orbitals 0.127, 0.119); 48^3 192: 0.37, 288: 0.45,
//         384: 0.42; 60^3 180: 0.85, 360: 0.97; 72^3 216: 1.58, 360: 1.66, 432: 1.66, 648: 2.09;
//         80^3 320: 2.28, 640: 2.88; 96^3 384: 3.50, 576: 4.84, 768: 4.36; 60 x 90 180: 2.85, 360: 3.20,
//         540: 4.19
//   FP64  24^3 192: 0.097, 96: 0.094; 48^3 192: 0.70, 288: 0.90, 384: 0.72; 60^3 360: 1.60, 180: 1.72;
//         72^3 648: 3.0, 360: 3.8; 80^3 640: 4.05, 320: 5.2; 96^3 768: 6.5, 384: 7.1; 60 x 90 540: 5.76,
//         360: 6.6, 180: 7.5
template <typename T, int N0, int N1> constexpr int slab_threads() {
  constexpr bool f = sizeof(T) == 4;
  if (N0 != N1) return f ? 180 : 540;  // 60 x 90
  return N0 == 16 ? 64 : N0 == 24 ? 192 : N0 == 32 ? 128 : N0 == 40 ? 320 : N0 == 48 ? 192
       : N0 == 60 ? (f ? 180 : 360) : N0 == 64 ? (f ? 256 : 512) : N0 == 72 ? (f ? 216 : 648)
       : N0 == 80 ? (f ? 320 : 640) : f ? 384 : 768;
}
// Whether pass 2 requests the next pair's slab ahead (see PF): from 64^3 in FP32
// and 60 points in FP64, where few workgroups fit a CU (FP64: one from 72^3 on).
// Pass 2 with the energy, ms per 1000 pairs, without -> with: FP32 64^3 0.864 -> 0.850,
// 72^3 1.573 -> 1.583 (without the energy 1.515 -> 1.474), 80^3 2.33 -> 2.28, 96^3 3.56 -> 3.50;
// FP64 60^3 1.68 -> 1.63, 64^3 1.52 -> 1.47, 72^3 3.40 -> 3.00, 80^3 4.50 -> 4.05, 96^3 6.97 ->
// 6.51, 60 x 90 x 120 6.29 -> 5.76.  FP32 at 60^3 would spill, 60 x 90 has no full slots; below
// 60 points the threads' slots are not full either, and many workgroups fit.
template <typename T, int N0, int N1> constexpr bool slab_prefetch() {
  return sizeof(T) == 8 ? N0 >= 60 : N0 == N1 && N0 >= 64;
}

template <int N0, int N1, int N2, int CFG>
hipError_t launch_chunk_cfg(bool fp32, const ChunkArgs& a, const ChunkDims& d, bool ex, hipStream_t s,
                            hipEvent_t* ev, const ChunkArgs* tasks) {
  constexpr int WF = tile_width<float, CFG>(), WD = tile_width<double, CFG>();
  using ZF = ZTile<float, N0, N1, N2, WF>;
  using ZD = ZTile<double, N0, N1, N2, WD>;
  // pass 3
  using YF = ZTile<float, N0, N1, N2, WF, ztile_radix3<float, N2>()>;
  using YD = ZTile<double, N0, N1, N2, WD, ztile_radix3<double, N2>()>;
  const int ntile = fp32 ? ZF::NTILE : ZD::NTILE;
  if (ev) (void)hipEventRecord(ev[0], s);
  const dim3 g1(tile_grid(ntile), d.max_ic, d.ntasks);
  if (fp32) hipLaunchKernelGGL((pass1_z<float, N0, N1, N2, WF, true>), g1, dim3(ZF::NT), 0, s, a, tasks);
  else hipLaunchKernelGGL((pass1_z<double, N0, N1, N2, WD, false>), g1, dim3(ZD::NT), 0, s, a, tasks);
  if (ev) (void)hipEventRecord(ev[1], s);
  const int pq = pairs_per_slab_wg(N2, d.max_pairs, d.ntasks);
  const dim3 g2(N2, (d.max_pairs + pq - 1) / pq, d.ntasks);
  constexpr int NF = slab_threads<float, N0, N1>(), ND = slab_threads<double, N0, N1>();
  constexpr bool PFF = slab_prefetch<float, N0, N1>(), PFD = slab_prefetch<double, N0, N1>();
  if (fp32 && ex) hipLaunchKernelGGL((pass2_xy<float, N0, N1, N2, ZF::NTILE, NF, true, true, PFF>), g2, dim3(round64(NF)), 0, s, a, tasks, pq);
  else if (fp32) hipLaunchKernelGGL((pass2_xy<float, N0, N1, N2, ZF::NTILE, NF, true, false, PFF>), g2, dim3(round64(NF)), 0, s, a, tasks, pq);
  else if (ex) hipLaunchKernelGGL((pass2_xy<double, N0, N1, N2, ZD::NTILE, ND, false, true, PFD>), g2, dim3(round64(ND)), 0, s, a, tasks, pq);
  else hipLaunchKernelGGL((pass2_xy<double, N0, N1, N2, ZD::NTILE, ND, false, false, PFD>), g2, dim3(round64(ND)), 0, s, a, tasks, pq);
  if (ev) (void)hipEventRecord(ev[2], s);
  int gj = 0;
  if (!d.store_v) {
    if (fp32) hipLaunchKernelGGL((pass3_z<float, N0, N1, N2, WF, false, 1>), dim3(tile_grid(ntile), d.max_ic, d.ntasks), dim3(YF::NT), 0, s, a, tasks);
    else hipLaunchKernelGGL((pass3_z<double, N0, N1, N2, WD, false, 1>), dim3(tile_grid(ntile), d.max_ic, d.ntasks), dim3(YD::NT), 0, s, a, tasks);
  } else {
    constexpr int GF = col_group(true, YF::RS), GD = col_group(false, YD::RS);
    gj = fp32 ? GF : GD;
    if (small_group(ntile, d.max_jc, gj, d.ntasks)) gj = 1;
    const dim3 g3(tile_grid(ntile), (d.max_jc + gj - 1) / gj, d.ntasks);
    if (fp32 && gj > 1) hipLaunchKernelGGL((pass3_z<float, N0, N1, N2, WF, true, GF>), g3, dim3(YF::NT), 0, s, a, tasks);
    else if (fp32) hipLaunchKernelGGL((pass3_z<float, N0, N1, N2, WF, true, 1>), g3, dim3(YF::NT), 0, s, a, tasks);
    else if (gj > 1) hipLaunchKernelGGL((pass3_z<double, N0, N1, N2, WD, true, GD>), g3, dim3(YD::NT), 0, s, a, tasks);
    else hipLaunchKernelGGL((pass3_z<double, N0, N1, N2, WD, true, 1>), g3, dim3(YD::NT), 0, s, a, tasks);
  }
  if (ev) (void)hipEventRecord(ev[3], s);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && d.store_v) e = launch_pass4(fp32, a, d, gj, size_t(N0) * N1 * N2, tasks, s);
  if (ev) (void)hipEventRecord(ev[4], s);
  return e;
}

// Passes 1 to 4 of one chunk (tasks == nullptr, the chunk in `a`) or of the
// chunks of a task table in device memory, one per blockIdx.z (d: the largest
// sizes of the table).  ev (optional, 5 events) brackets the passes.
template <int N0, int N1, int N2>
hipError_t launch_chunk_t(bool fp32, const ChunkArgs& a, const ChunkDims& d, bool ex, int cfg,
                          hipStream_t s, hipEvent_t* ev, const ChunkArgs* tasks) {
  return cfg == 0 ? launch_chunk_cfg<N0, N1, N2, 0>(fp32, a, d, ex, s, ev, tasks)
                  : launch_chunk_cfg<N0, N1, N2, 1>(fp32, a, d, ex, s, ev, tasks);
}

}  // namespace px
