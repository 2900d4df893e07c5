// Plane passes of the Kohn-Sham Hamiltonian (HIP, gfx950): per m0 plane of
// the plane-wave sphere, z- and y-synthesis into T, and y- and z-analysis of
// U with the kinetic term and the Taylor-4 epilogue (Section
// "Implementation of the KS Hamiltonian"; Section "Real-time propagation").
#pragma once
#include "ks_common.hpp"

namespace ks {

// Work split of the plane passes by plane size, precision and direction:
// threads per block, columns per y-batch, columns per z-batch, orbitals
// transformed together.  A compute unit needs about three waves per SIMD here
// (a lone wave issues a vector instruction only every other slot), and every
// batch stage ends at a block barrier.  At 24 to 120 points the rows are the
// fastest of eight measured splits per size, precision and direction (spheres in
// the band, the analysis without the chained synthesis); at 8 to 20 points they
// follow the first rule, unswept; at 128 points the complex64 analysis is the
// fastest of eleven.  The rules:
//  - small planes take several orbitals at once (or a smaller block): a plane
//    of 8 to 40 points leaves most lanes of a 64-column batch without work;
//  - the z-batch follows the sphere's column count (about 0.45 N), not the
//    y-batch;
//  - in FP64 at 60, 64 and 72 points and for the synthesis at 80 the y-batch
//    shrinks until two blocks fit a compute unit (47 to 75 KB each); the analysis
//    at 80 and both passes from 96 on keep a larger one and one block (97 to 150 KB);
//  - a synthesis batch of complex64 stores rows of whole 32-byte sectors of T:
//    rows of 30 (240 bytes) took twice as long as rows of 60 or 20.
// Per launch, one block of 384 threads and 64 or 48 columns for all sizes
// against these rows, us: 8^2 FP64 / 512 orbitals (12 planes of n0) synthesis 9.8
// and 6.6, analysis 13.6 and 8.2; 16^2 FP64 / 512 16.3 and 10.7, 23.8 and 11.7; 20^2
// FP64 / 512 22.6 and 13.9, 34.7 and 23.7; 64^2 FP64 / 128 82 and 56, 93 and 70;
// 32^2 complex64, 262 orbitals in a batch 19 and 10, 33 and 13; 40^2 FP64 / 33 13.3
// and 9.4, 16.9 and 9.9; 96^2 complex64 / 512 398 and 376, 531 and 472; 120^2
// complex64 / 1024 1783 and 1717, 2752 and 2404; 128^2 complex64 / 160 (40 planes of
// n0) 120 and 110, 169 and 151, FP64 / 160 258 and 229, 350 and 352 (T or U streams
// at 3.6 and 2.9 TB/s at 120^2; 96^2 FP64 at 5.0 and 5.0, near the rate of a large
// copy, which bounds it).
// The four waves per SIMD asked for at 96 and 120 points in complex64 spill one to
// five registers of the analysis from FP64 orbitals (one of a step's four).
template <int N, bool F64, bool FWD> struct plane_cfg { static constexpr int NT = 384, YB = 16, ZB = 16, G = 1, W = 1; };
// (points, FP64, analysis) -> threads, y-batch, z-batch, orbitals, waves per SIMD to fit the registers to
#define KS_PLANE_CFG(n, f64, fwd, nt, yb, zb, g, w) \
  template <> struct plane_cfg<n, f64, fwd> { static constexpr int NT = nt, YB = yb, ZB = zb, G = g, W = w; };
KS_PLANE_CFG(8, true, false, 64, 64, 64, 8, 1)
KS_PLANE_CFG(8, true, true, 64, 64, 64, 8, 1)
KS_PLANE_CFG(8, false, false, 64, 64, 64, 8, 1)
KS_PLANE_CFG(8, false, true, 64, 64, 64, 8, 1)
KS_PLANE_CFG(12, true, false, 64, 48, 48, 4, 1)
KS_PLANE_CFG(12, true, true, 64, 48, 48, 4, 1)
KS_PLANE_CFG(12, false, false, 64, 48, 48, 4, 1)
KS_PLANE_CFG(12, false, true, 64, 48, 48, 4, 1)
KS_PLANE_CFG(16, true, false, 128, 16, 16, 1, 1)
KS_PLANE_CFG(16, true, true, 128, 16, 16, 1, 1)
KS_PLANE_CFG(16, false, false, 128, 16, 16, 1, 1)
KS_PLANE_CFG(16, false, true, 128, 16, 16, 1, 1)
KS_PLANE_CFG(20, true, false, 320, 60, 60, 3, 1)
KS_PLANE_CFG(20, true, true, 320, 60, 60, 3, 1)
KS_PLANE_CFG(20, false, false, 320, 60, 60, 3, 1)
KS_PLANE_CFG(20, false, true, 320, 60, 60, 3, 1)
KS_PLANE_CFG(24, true, false, 128, 24, 16, 1, 1)
KS_PLANE_CFG(24, true, true, 128, 24, 16, 1, 1)
KS_PLANE_CFG(24, false, false, 128, 24, 16, 1, 1)
KS_PLANE_CFG(24, false, true, 128, 24, 16, 1, 1)
KS_PLANE_CFG(32, true, false, 256, 64, 32, 2, 1)
KS_PLANE_CFG(32, true, true, 256, 64, 32, 2, 1)
KS_PLANE_CFG(32, false, false, 256, 32, 32, 2, 1)
KS_PLANE_CFG(32, false, true, 256, 32, 16, 1, 1)
KS_PLANE_CFG(40, true, false, 256, 40, 20, 1, 1)
KS_PLANE_CFG(40, true, true, 256, 40, 20, 1, 1)
KS_PLANE_CFG(40, false, false, 320, 40, 40, 2, 1)
KS_PLANE_CFG(40, false, true, 256, 40, 40, 2, 1)
KS_PLANE_CFG(48, true, false, 192, 24, 24, 1, 1)
KS_PLANE_CFG(48, true, true, 256, 24, 24, 1, 1)
KS_PLANE_CFG(48, false, false, 192, 48, 24, 1, 1)
KS_PLANE_CFG(48, false, true, 192, 48, 24, 1, 1)
KS_PLANE_CFG(60, true, false, 192, 20, 32, 1, 1)
KS_PLANE_CFG(60, true, true, 256, 30, 32, 1, 1)
KS_PLANE_CFG(60, false, false, 384, 60, 32, 1, 1)
KS_PLANE_CFG(60, false, true, 256, 60, 32, 1, 1)
KS_PLANE_CFG(64, true, false, 320, 32, 32, 1, 1)
KS_PLANE_CFG(64, true, true, 256, 32, 32, 1, 1)
KS_PLANE_CFG(64, false, false, 256, 64, 32, 1, 1)
KS_PLANE_CFG(64, false, true, 256, 32, 32, 1, 1)
KS_PLANE_CFG(72, true, false, 384, 24, 36, 1, 1)
KS_PLANE_CFG(72, true, true, 256, 24, 36, 1, 1)
KS_PLANE_CFG(72, false, false, 448, 72, 36, 1, 1)
KS_PLANE_CFG(72, false, true, 448, 72, 36, 1, 1)
KS_PLANE_CFG(80, true, false, 384, 20, 40, 1, 1)
KS_PLANE_CFG(80, true, true, 384, 40, 40, 1, 1)
KS_PLANE_CFG(80, false, false, 512, 40, 40, 1, 1)
KS_PLANE_CFG(80, false, true, 512, 40, 40, 1, 1)
KS_PLANE_CFG(96, true, false, 384, 48, 48, 1, 1)
KS_PLANE_CFG(96, true, true, 384, 48, 48, 1, 1)
KS_PLANE_CFG(96, false, false, 384, 48, 48, 1, 1)
KS_PLANE_CFG(96, false, true, 512, 48, 48, 1, 4)
KS_PLANE_CFG(120, true, false, 512, 24, 27, 1, 1)
KS_PLANE_CFG(120, true, true, 320, 24, 27, 1, 1)
KS_PLANE_CFG(120, false, false, 384, 24, 27, 1, 1)
KS_PLANE_CFG(120, false, true, 512, 24, 24, 1, 4)
KS_PLANE_CFG(128, true, false, 384, 16, 60, 1, 1)
KS_PLANE_CFG(128, true, true, 384, 16, 60, 1, 1)
KS_PLANE_CFG(128, false, false, 384, 16, 60, 1, 1)
KS_PLANE_CFG(128, false, true, 512, 16, 32, 1, 1)
#undef KS_PLANE_CFG
// The rows are for spheres inside the band.  Past it (not HB) a plane has up to
// 0.6 N columns at a spacing of 0.42 bohr; from 80 points on the z-batch takes
// those in one, and 80 FP64 the y-batch of 48 of its former split: a step of
// 160 orbitals there 10.4 -> 9.4 ms (80^3 FP64; 10.1 with the former split of 384
// threads and 48 columns), 5.6 -> 5.4 (80^3 complex64), 8.3 -> 7.8 (40 x 120^2
// complex64), 11.0 -> 10.3 ms (40 x 128^2 complex64).  Below, larger z-batches
// cost registers and were slower (48^3 complex64 1.41 -> 1.58 ms).
template <int N, bool F64, bool FWD, bool HB>
struct plane_split : plane_cfg<N, F64, FWD> {
  using row = plane_cfg<N, F64, FWD>;
  static constexpr int wide = (6 * N / 10 + 3) / 4 * 4;
  static constexpr int YB = !HB && F64 && N == 80 ? 48 : row::YB;
  static constexpr int ZB = !HB && N >= 80 && wide > row::ZB ? wide : row::ZB;
};
template <int N, typename R, bool FWD, bool HB> using pcfg = plane_split<N, sizeof(R) == 8, FWD, HB>;

// Packed coefficients of a plane that a thread holds in registers across an
// orbital's transforms: a band-limited plane has at most about 0.165 N^2.
constexpr int plane_ep(int n, int nt) {
  const int e = (165 * n * n / 1000 + nt - 1) / nt;
  return e < 1 ? 1 : e > 4 ? 4 : e;
}

// The column tables of plane pi in LDS; returns through the references.
struct PlaneCols {
  int c0, nc, m1lo, e0, npp;
};
template <int NT>
__device__ __forceinline__ PlaneCols plane_cols(const SphereTab& tab, int pi, int* s_off, int* s_m2lo) {
  PlaneCols p;
  p.c0 = tab.plane_col0[pi];
  p.nc = tab.plane_col0[pi + 1] - p.c0;
  p.m1lo = tab.plane_m1lo[pi];
  p.e0 = tab.col_off[p.c0];
  p.npp = tab.col_off[p.c0 + p.nc] - p.e0;
  for (int i = threadIdx.x; i <= p.nc; i += NT) s_off[i] = tab.col_off[p.c0 + i] - p.e0;
  for (int i = threadIdx.x; i < p.nc; i += NT) s_m2lo[i] = tab.col_m2lo[p.c0 + i];
  return p;
}

// z-synthesis of the columns of go <= G orbitals' plane into Z, then
// y-synthesis from Z, through Y, to T (out: this plane of the first orbital's
// T; gstride: bytes between orbitals).  coef(g, k, c, e): packed coefficient k
// of the plane of orbital g, which is point e of column c (it may live in Y: it
// is read before Y is written).
// Ends with a block barrier.
template <int N, int NTH, int YB, int ZB, int G, bool HB, typename C, class F>
__device__ __forceinline__ void plane_synthesis(C* Z, C* Y, const C* tw, const int* s_off, const int* s_m2lo,
                                                const PlaneCols& pc, int go, gbuf out, unsigned gstride, F&& coef) {
  const int nc = pc.nc, m1lo = pc.m1lo, nz = go * nc;
  for (int zb = 0; zb < nz; zb += ZB) {
    auto load = [&](int t, int e) -> C {
      int g = 0, c = zb + t;
#pragma unroll
      for (int i = 1; i < G; ++i) g += zb + t >= i * nc;
      c -= g * nc;
      const int idx = fold(e, N) - s_m2lo[c];
      return (idx >= 0 && idx < s_off[c + 1] - s_off[c]) ? coef(g, s_off[c] + idx, c, e) : czero<C>();
    };
    if constexpr (HB) fft_io<N, +1, ZB, NTH, SRC_FN, DST_LDS, C>(Z + zb * (N + 1), N + 1, nz - zb, tw, banded(load), no_store{});
    else fft_io<N, +1, ZB, NTH, SRC_FN, DST_LDS, C>(Z + zb * (N + 1), N + 1, nz - zb, tw, load, no_store{});
  }
  for (int y0 = 0; y0 < go * N; y0 += YB) {
    auto load = [&](int t, int e) -> C {
      const int y = y0 + t, g = G == 1 ? 0 : y / N, w = G == 1 ? y : y % N;
      const int c = fold(e, N) - m1lo;
      return (c >= 0 && c < nc) ? Z[(g * nc + c) * (N + 1) + w] : czero<C>();
    };
    auto store = [&](int t, int e, C v, int, int) {
      const int y = y0 + t, g = G == 1 ? 0 : y / N, w = G == 1 ? y : y % N;
      buf_store<true>(out, g * gstride + (unsigned)((e * N + w) * (int)sizeof(C)), v);
    };
    if constexpr (HB) fft_io<N, +1, YB, NTH, SRC_FN, DST_FN, C>(Y, N + 1, go * N - y0, tw, banded(load), store);
    else fft_io<N, +1, YB, NTH, SRC_FN, DST_FN, C>(Y, N + 1, go * N - y0, tw, load, store);
    __syncthreads();
  }
}

// ----------------------------------------------------------- plane synthesis
// Block (plane pi, orbital group).  G orbitals of the group at a time: their
// packed coefficients of the plane (contiguous, so the loads coalesce; fetched
// into registers one iteration ahead) are staged in LDS; z-synthesis of each
// disk column from the staging area into Z; y-synthesis of YB r2-columns at a
// time from Z straight into T.  Columns of the G orbitals are numbered through
// (orbital major), so a batch may hold columns of several orbitals.
// LDS: twiddles [N] | Z [G ncol][N+1] | Y [YB][N+1] (the staging area of the
// packed coefficients, consumed before the y-synthesis, shares Y).  `stage`
// = 0 when G planes' coefficients do not fit in Y: the z-synthesis then reads
// them from HBM directly.
//
// Bound: HBM writes of T for the largest planes (96^2 FP64: 5.1 of the 6.6
// TB/s that a fill reaches), LDS exchange and barrier latency for smaller ones.

// BOX: the orbitals are boxes [n0][N][N] (pk) of which the z-synthesis reads
// the sphere's points itself, without a packed copy.
//
// BATCH: one launch over several systems of the grid; the block's system
// (its input, T and orbital count) comes from jobs[rows[blockIdx.y].x].
template <int N, typename R, typename TIN, bool HB, bool BATCH = false, bool BOX = false>
__global__ __launch_bounds__((pcfg<N, R, false, HB>::NT)) __attribute__((amdgpu_waves_per_eu(pcfg<N, R, false, HB>::W))) void plane_inv_kernel(const TIN* __restrict__ pk, int nb, int pk_stride,
                                                                     cplx<R>* __restrict__ Tout, SphereTab tab,
                                                                     const cplx<R>* __restrict__ twN, int ncol_max,
                                                                     int stage,
                                                                     const BatchJob* __restrict__ jobs = nullptr,
                                                                     const int4* __restrict__ rows = nullptr) {
  using C = cplx<R>;
  constexpr int NTH = pcfg<N, R, false, HB>::NT, YB = pcfg<N, R, false, HB>::YB, ZB = pcfg<N, R, false, HB>::ZB, G = pcfg<N, R, false, HB>::G;
  constexpr int EP = plane_ep(N, NTH);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  C* tw = reinterpret_cast<C*>(smem_raw);
  C* Z = tw + N;
  C* Y = Z + G * ncol_max * (N + 1);
  C* S = Y;
  __shared__ int s_off[130];
  __shared__ int s_m2lo[129];
  const int pi = blockIdx.x, tid = threadIdx.x;
  int oa, ob;
  if constexpr (BATCH) {
    const int4 r = rows[blockIdx.y];
    pk = static_cast<const TIN*>(jobs[r.x].win);
    Tout = static_cast<cplx<R>*>(jobs[r.x].T);
    nb = jobs[r.x].nb;
    group_range(nb, r.y, r.z, oa, ob);
  } else {
    orbital_range(nb, oa, ob);
  }
  const PlaneCols pc = plane_cols<NTH>(tab, pi, s_off, s_m2lo);
  const int npp = pc.npp;
  // this thread's first EP coefficients of each of the next G orbitals
  TIN cin[G][EP];
  auto fetch = [&](int o) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const TIN* in = pk + (long long)(o + g) * pk_stride + pc.e0;
#pragma unroll
      for (int j = 0; j < EP; ++j) {
        const int k = tid + j * NTH;
        if (k < npp && (G == 1 || o + g < ob)) cin[g][j] = in[k];
      }
    }
  };
  if (!BOX && stage && oa < ob) fetch(oa);
  stage_twiddles<N, NTH>(tw, twN);
  __syncthreads();
  const unsigned gstride = (unsigned)(tab.nplanes * N * N * (int)sizeof(C));   // bytes between two orbitals' T
  for (int o = oa; o < ob; o += G) {
    const int go = G == 1 ? 1 : min(G, ob - o);
    if (!BOX && stage) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (G > 1 && g >= go) break;
#pragma unroll
        for (int j = 0; j < EP; ++j) {
          const int k = tid + j * NTH;
          if (k < npp) S[g * npp + k] = cvt<C>(cin[g][j]);
        }
        const TIN* in = pk + (long long)(o + g) * pk_stride + pc.e0;
        for (int k = tid + EP * NTH; k < npp; k += NTH) S[g * npp + k] = cvt<C>(in[k]);
      }
      if (o + G < ob) fetch(o + G);
      __syncthreads();
    }
    const gbuf out = make_gbuf(Tout + ((long long)o * tab.nplanes + pi) * N * N, OOB);
    if constexpr (BOX) {
      const long long plane = (long long)wrap(tab.m0lo + pi, tab.n0) * (N * N);
      plane_synthesis<N, NTH, YB, ZB, G, HB>(Z, Y, tw, s_off, s_m2lo, pc, go, out, gstride,
                                             [&](int g, int, int c, int e) {
        return cvt<C>((pk + (long long)(o + g) * tab.n0 * (N * N) + plane)[wrap(pc.m1lo + c, N) * N + e]);
      });
    } else if (stage) {
      plane_synthesis<N, NTH, YB, ZB, G, HB>(Z, Y, tw, s_off, s_m2lo, pc, go, out, gstride,
                                             [&](int g, int k, int, int) { return S[g * pc.npp + k]; });
    } else {
      plane_synthesis<N, NTH, YB, ZB, G, HB>(Z, Y, tw, s_off, s_m2lo, pc, go, out, gstride, [&](int g, int k, int, int) {
        return cvt<C>((pk + (long long)(o + g) * pk_stride + pc.e0)[k]);
      });
    }
  }
}

// ------------------------------------------------------------ plane analysis
// Block (plane pi, orbital group).  G orbitals of the group at a time:
// y-analysis of YB r2-columns of U at a time into the disk columns Z; the
// z-analysis of every column in place; then the epilogue over the plane's
// packed coefficients, which are contiguous, so its loads and stores
// coalesce: + 1/2|G|^2 c and the output mode.  The next U batch (also across
// orbitals) is loaded while the current one is transformed, and an orbital's
// epilogue operands are loaded before its transforms.  A thread's packed
// coefficients are the same for every orbital: their places in Z and kinetic
// energies are found once per block.
// LDS: twiddles [N] | Z [G ncol][N+1] | Y [YB][N+1].

// next: the block goes on to the plane synthesis of the next H psi: with 1 of
// the H psi just formed (the next power of H), with 2 of the
// accumulated state, from the coefficients in LDS into T (whose last reader,
// the x-apply pass, is done).  Saves a launch, a read of the coefficients and
// the start of a block (tables, twiddles): a step of 4 H psi measured 506 -> 451
// us (24^3, 10 orbitals, mixed), 1480 -> 1435 (60^3, 96, mixed), 2585 -> 2531
// (64^3, 128, FP64), 34.5 -> 33.7 ms (96^3, 512, FP64), 53.0 -> 51.1 ms (120^3,
// 1024, mixed).  The synthesis then runs in the analysis's work split;
// plane_next says for which sizes and launches.
//
// BOX: input and result are boxes [n0][N][N] (win, acc; the result alone, no
// mode).  The epilogue goes over all points of the plane, zero outside the
// sphere, and the grid over all n0 planes: those past the sphere's are filled
// with zeros.
//
// BATCH: as plane_inv_kernel; U, win, wout, acc, T and the orbital count come
// from the block's job (no second accumulator).
template <int N, typename R, typename TW, bool HB, bool BATCH = false, bool BOX = false>
__global__ __launch_bounds__((pcfg<N, R, true, HB>::NT)) __attribute__((amdgpu_waves_per_eu(pcfg<N, R, true, HB>::W))) void plane_fwd_kernel(
    const cplx<R>* __restrict__ Uin, int nb, const TW* win, cplx<R>* __restrict__ wout, double2* acc, double2* acc2,
    int pk_stride, int acc_stride, SphereTab tab, const double* __restrict__ kin, const cplx<R>* __restrict__ twN,
    int ncol_max, int mode, Taylor tay, int next, cplx<R>* __restrict__ Tout,
    const BatchJob* __restrict__ jobs = nullptr, const int4* __restrict__ rows = nullptr) {
  using C = cplx<R>;
  constexpr int NTH = pcfg<N, R, true, HB>::NT, YB = pcfg<N, R, true, HB>::YB, ZB = pcfg<N, R, true, HB>::ZB, G = pcfg<N, R, true, HB>::G;
  constexpr int EP = plane_ep(N, NTH);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  C* tw = reinterpret_cast<C*>(smem_raw);
  C* Z = tw + N;
  C* Y = Z + G * ncol_max * (N + 1);
  __shared__ int s_off[130];
  __shared__ int s_m2lo[129];
  const int pi = blockIdx.x, tid = threadIdx.x;
  int oa, ob;
  if constexpr (BATCH) {
    const int4 r = rows[blockIdx.y];
    Uin = static_cast<const cplx<R>*>(jobs[r.x].U);
    win = static_cast<const TW*>(jobs[r.x].win);
    wout = static_cast<cplx<R>*>(jobs[r.x].wout);
    acc = jobs[r.x].acc;
    acc2 = nullptr;
    Tout = static_cast<cplx<R>*>(jobs[r.x].T);
    nb = jobs[r.x].nb;
    group_range(nb, r.y, r.z, oa, ob);
  } else {
    orbital_range(nb, oa, ob);
  }
  double2* box = nullptr;   // this plane of the first orbital's result
  if constexpr (BOX) {
    box = acc + (long long)wrap(tab.m0lo + pi, tab.n0) * (N * N);
    if (pi >= tab.nplanes) {
      for (int o = oa; o < ob; ++o)
#pragma unroll 4
        for (int p = tid; p < N * N; p += NTH) st_stream(box + (long long)o * tab.n0 * (N * N) + p, double2{0.0, 0.0});
      return;
    }
  }
  const long long uplane = (long long)tab.nplanes * N * N;   // elements between two orbitals' U
  const unsigned gstride = (unsigned)(uplane * (int)sizeof(C));
  using FR = fft_regs<N, YB, NTH, C>;
  FR pre;
  // the columns y0 .. of the orbitals o .. (at most G, below ob) into pre
  auto load_batch = [&](int o, int y0) {
    const int left = (G == 1 ? 1 : min(G, ob - o)) * N - y0;
    const gbuf u = make_gbuf(Uin + (long long)o * uplane + (long long)pi * N * N, OOB);
    fft_preload<N, YB, NTH, C>(pre, left, [&](int t, int e) -> C {
      const int y = y0 + t, g = G == 1 ? 0 : y / N, w = G == 1 ? y : y % N;
      return buf_load<C, true>(u, g * gstride + (unsigned)((e * N + w) * (int)sizeof(C)));
    });
  };
  if (oa < ob) load_batch(oa, 0);
  const PlaneCols pc = plane_cols<NTH>(tab, pi, s_off, s_m2lo);
  const int nc = pc.nc, npp = pc.npp, m1lo = pc.m1lo;
  stage_twiddles<N, NTH>(tw, twN);
  __syncthreads();
  auto z_place = [&](int k) {
    const int c = find_col(s_off, nc, k);
    return c * (N + 1) + wrap(s_m2lo[c] + k - s_off[c], N);
  };
  // BOX: packed index of point p of the plane, -1 outside the sphere; its place in Z
  auto point = [&](int p, int& zp) {
    const int y = p / N, z = p - y * N, c = fold(y, N) - m1lo;
    if (c < 0 || c >= nc) return -1;
    const int t = fold(z, N) - s_m2lo[c];
    zp = c * (N + 1) + z;
    return t >= 0 && t < s_off[c + 1] - s_off[c] ? s_off[c] + t : -1;
  };
  int zk[EP], kb[EP];
#pragma unroll
  for (int j = 0; j < EP; ++j) {
    const int k = tid + j * NTH;
    if constexpr (BOX) kb[j] = k < N * N ? point(k, zk[j]) : -1;
    else zk[j] = k < npp ? z_place(k) : 0;
  }
  for (int o = oa; o < ob; o += G) {
    const int go = G == 1 ? 1 : min(G, ob - o);
    for (int y0 = 0; y0 < go * N; y0 += YB) {
      auto next = [&] {
        if (y0 + YB < go * N) load_batch(o, y0 + YB);
        else if (o + G < ob) load_batch(o + G, 0);
      };
      auto store = [&](int t, int e, C v, int, int) {
        const int y = y0 + t, g = G == 1 ? 0 : y / N, w = G == 1 ? y : y % N;
        const int c = fold(e, N) - m1lo;
        if (c >= 0 && c < nc) Z[(g * nc + c) * (N + 1) + w] = v;
      };
      if constexpr (HB) fft_io<N, -1, YB, NTH, SRC_PRE, DST_FN, C>(Y, N + 1, go * N - y0, tw, preloaded(pre, next), banded(store));
      else fft_io<N, -1, YB, NTH, SRC_PRE, DST_FN, C>(Y, N + 1, go * N - y0, tw, preloaded(pre, next), store);
      __syncthreads();
    }
    // epilogue operands of these orbitals, loaded while the columns are
    // transformed along z (held across the y-batches too they take the
    // complex64 form past the 128 registers of four waves per SIMD)
    double kk[EP];
#pragma unroll
    for (int j = 0; j < EP; ++j) {
      const int k = tid + j * NTH;
      if constexpr (BOX) kk[j] = kb[j] >= 0 ? kin[pc.e0 + kb[j]] : 0.0;
      else kk[j] = k < npp ? kin[pc.e0 + k] : 0.0;
    }
    TW wv[G][EP];
    double2 av[G][EP];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if constexpr (BOX) {
        const TW* in = win + (box - acc) + (long long)(o + g) * tab.n0 * (N * N);
#pragma unroll
        for (int j = 0; j < EP; ++j)
          if (kb[j] >= 0 && (G == 1 || g < go)) wv[g][j] = in[tid + j * NTH];
        continue;
      }
      const gbuf wp = make_gbuf(win + ((long long)(o + g) * pk_stride + pc.e0), OOB);
      const gbuf ap = make_gbuf(acc + ((long long)(o + g) * acc_stride + pc.e0), OOB);
#pragma unroll
      for (int j = 0; j < EP; ++j) {
        const int k = tid + j * NTH;
        if (k < npp && (G == 1 || g < go)) {
          wv[g][j] = buf_load<TW>(wp, k * (unsigned)sizeof(TW));
          if (mode != H_OUT) av[g][j] = buf_load<double2>(ap, k * (unsigned)sizeof(double2));
        }
      }
    }
    // z-analysis in place; with HB only the band |m2| < n2/4, which holds every column's run, is written
    for (int zb = 0; zb < go * nc; zb += ZB) {
      C* zp = Z + zb * (N + 1);
      if constexpr (HB)
        fft_io<N, -1, ZB, NTH, SRC_LDS, DST_FN_LDS, C>(zp, N + 1, go * nc - zb, tw, no_load{},
                                                       banded([&](int t, int e, C v, int, int) { zp[t * (N + 1) + e] = v; }));
      else
        fft_batch<N, -1, ZB, NTH, C>(zp, N + 1, go * nc - zb, tw);
    }
    // the second accumulator (ETRS predictor) is read where it is updated,
    // so the common single-accumulator path keeps its registers
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (G > 1 && g >= go) break;
      const long long ro = (long long)(o + g) * pk_stride + pc.e0, ra = (long long)(o + g) * acc_stride + pc.e0;
      const gbuf wp = make_gbuf(wout + ro, OOB);
      const gbuf ap = make_gbuf(acc + ra, OOB);
      const C* const zg = Z + g * nc * (N + 1);
      if constexpr (BOX) {
        const long long ro = (long long)(o + g) * tab.n0 * (N * N);
        auto put = [&](int p, int k, int zp, double K, TW w) {
          double2 v{0.0, 0.0};
          if (k >= 0) {
            const C ph = zg[zp];
            const double2 hw{K * double(w.x) + double(ph.x), K * double(w.y) + double(ph.y)};
            v = to_d(to_c<C>(hw));
          }
          st_stream(box + ro + p, v);
        };
#pragma unroll
        for (int j = 0; j < EP; ++j) {
          const int p = tid + j * NTH;
          if (p < N * N) put(p, kb[j], zk[j], kk[j], wv[g][j]);
        }
        for (int p = tid + EP * NTH; p < N * N; p += NTH) {
          int zp = 0;
          const int k = point(p, zp);
          put(p, k, zp, k >= 0 ? kin[pc.e0 + k] : 0.0, k >= 0 ? (win + (box - acc) + ro)[p] : TW{0.0, 0.0});
        }
        continue;
      }
      C* const sg = Y + g * npp;   // next: staged coefficients of the synthesis
      auto epilogue = [&](int k, int zp, double K, TW w, double2 a) {
        const C ph = zg[zp];
        const double2 hw{K * double(w.x) + double(ph.x), K * double(w.y) + double(ph.y)};
        if (mode == H_OUT) {
          buf_store(wp, k * (unsigned)sizeof(C), to_c<C>(hw));
        } else {
          if (tay.write_w) buf_store(wp, k * (unsigned)sizeof(C), to_c<C>(hw));
          a.x += tay.coef.x * hw.x - tay.coef.y * hw.y;
          a.y += tay.coef.x * hw.y + tay.coef.y * hw.x;
          buf_store(ap, k * (unsigned)sizeof(double2), a);
          if (next) sg[k] = to_c<C>(next == 1 ? hw : a);
          if (acc2) {
            double2 b = (acc2 + ra)[k];
            b.x += tay.coef2.x * hw.x - tay.coef2.y * hw.y;
            b.y += tay.coef2.x * hw.y + tay.coef2.y * hw.x;
            (acc2 + ra)[k] = b;
          }
        }
      };
#pragma unroll
      for (int j = 0; j < EP; ++j) {
        const int k = tid + j * NTH;
        if (k < npp) epilogue(k, zk[j], kk[j], wv[g][j], mode != H_OUT ? av[g][j] : double2{0.0, 0.0});
      }
      for (int k = tid + EP * NTH; k < npp; k += NTH)
        epilogue(k, z_place(k), kin[pc.e0 + k], (win + ro)[k],
                 mode != H_OUT ? (acc + ra)[k] : double2{0.0, 0.0});
    }
    __syncthreads();   // Z is rewritten by the next orbitals
    if (next)
      plane_synthesis<N, NTH, YB, ZB, G, HB>(Z, Y, tw, s_off, s_m2lo, pc, go,
                                             make_gbuf(Tout + ((long long)o * tab.nplanes + pi) * N * N, OOB), gstride,
                                             [&](int g, int k, int, int) { return Y[g * npp + k]; });
  }
}

// ------------------------------------------------------------------ launchers

// Plane size, precision, direction and band -> f(config, plane size)
template <bool FWD, class F>
void with_plane_cfg(const ks_system* s, F&& f) {
  switch (s->n[1]) {
#define KS_CASE(v)                                                                                         \
  case v:                                                                                                  \
    if (mixed(s)) s->yz_half ? f(plane_split<v, false, FWD, true>{}) : f(plane_split<v, false, FWD, false>{}); \
    else s->yz_half ? f(plane_split<v, true, FWD, true>{}) : f(plane_split<v, true, FWD, false>{});        \
    break;
    KS_SIZES(KS_CASE)
#undef KS_CASE
    default:
      break;
  }
}

// LDS of a plane block: the dynamic part, and the column tables s_off and
// s_m2lo that the kernels declare
constexpr size_t PLANE_TABLES = (130 + 129) * sizeof(int);
template <bool FWD>
size_t plane_smem(const ks_system* s) {
  size_t rows = 0;
  with_plane_cfg<FWD>(s, [&](auto c) { rows = (size_t)decltype(c)::G * s->ncol_max + decltype(c)::YB; });
  return (s->prec == KS_FP64 ? sizeof(double2) : sizeof(float2)) * ((size_t)s->n[1] + rows * (s->n[1] + 1));
}

inline int plane_groups(const ks_system* s, int nb) {
  const int g = plane_group_size(s, nb);
  return (nb + g - 1) / g;
}

}  // namespace ks
