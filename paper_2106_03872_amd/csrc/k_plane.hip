// Launches of the plane passes on packed orbitals (HIP, gfx950).
#include "plane_kernels.hpp"

namespace ks {

// The LDS that a sphere must leave within the 160 KB of a compute unit to be
// accepted: one plane's columns, a batch of 64 (n1 <= 64), 48, 24 or 16 rows
// and one byte per packed coefficient of the plane; and what the passes are
// launched with, which is more than that in some sizes (their largest splits,
// and the column tables beside the dynamic part).  Over the numbers of columns
// that a sphere can have, odd or the whole plane, no sphere that keeps the
// former exceeds 160 KB in the latter: it stands here for rows to come.
size_t plane_lds_bytes(const ks_system* s) {
  const int N = s->n[1];
  const int yb = N <= 64 ? 64 : (N <= 96 ? 48 : (N <= 120 ? 24 : 16));
  const size_t es = s->prec == KS_FP64 ? sizeof(double2) : sizeof(float2);
  const size_t bound =
      es * ((size_t)N + (size_t)s->ncol_max * (N + 1) + (size_t)yb * (N + 1)) + ((size_t)s->npp_max + 15) / 16 * 16;
  return std::max(bound, std::max(plane_smem<false>(s), plane_smem<true>(s)) + PLANE_TABLES);
}

// Orbitals per plane block for a launch over `total` orbitals: up to pg_max,
// fewer when the launch would have fewer than about 4 blocks per CU, but the
// G orbitals that a block transforms together, unless one orbital per block
// leaves compute units idle: up to 256 blocks, 768 in complex64 from 32 points
// on and 1024 of a wave each at 8 and 12 points.  A step of 4 H psi with and
// without that, us: 12 x 8 x 8 / 16 FP64 75 -> 70, / 160 78 -> 74; 20^3 / 16 77 ->
// 75 (/ 32, 288 blocks, 79 -> 81: not); 32^3 / 16 complex64 86 -> 75, / 48 103 -> 94;
// 40^3 / 8 complex64 104 -> 92, / 32 149 -> 140 (/ 64, 1088 blocks, 211 -> 224: not).
int plane_group_size(const ks_system* s, long long total) {
  int G = 1;
  with_plane_cfg<false>(s, [&](auto c) { G = decltype(c)::G; });
  with_plane_cfg<true>(s, [&](auto c) { G = std::max(G, decltype(c)::G); });
  G = std::min(G, s->pg_max);
  const int one = s->n[1] <= 12 ? 1024 : mixed(s) && s->n[1] >= 32 ? 768 : 256;
  if (s->nplanes * total <= one) return 1;
  long long g = (long long)s->nplanes * total / (256 * 4);
  g = g < G ? G : (g > s->pg_max ? s->pg_max : g);
  return (int)(g / G * G);
}

// Batched launches pass (rows, jobs, nrows): the grid's y extent is nrows
// and every per-system argument comes from the jobs; nb and the pointers
// below are then unused.
struct BatchRef {
  const BatchJob* jobs = nullptr;
  const int4* rows = nullptr;
  int nrows = 0;
};

template <int N, typename R, typename TIN, bool HB, bool B>
static void plane_inv_t(const ks_system* s, int nb, const void* pk, void* T, const void* tw, const BatchRef& b,
                        hipStream_t st) {
  using PC = pcfg<N, R, false, HB>;
  const int stage = PC::G * s->npp_max <= PC::YB * (N + 1) ? 1 : 0;
  const dim3 grid(s->nplanes, B ? b.nrows : plane_groups(s, nb));
  plane_inv_kernel<N, R, TIN, HB, B><<<grid, PC::NT, plane_smem<false>(s), st>>>(
      (const TIN*)pk, nb, s->npw_stride, (cplx<R>*)T, sphere_tab(s), (const cplx<R>*)tw, s->ncol_max, stage, b.jobs,
      b.rows);
}

template <int N, bool HB, bool B>
static void plane_inv_h(const ks_system* s, int nb, const void* pk, bool in_fp64, void* T, const BatchRef& b,
                        hipStream_t st) {
  if (!mixed(s)) plane_inv_t<N, double, double2, HB, B>(s, nb, pk, T, s->d_tw1, b, st);
  else if (in_fp64) plane_inv_t<N, float, double2, HB, B>(s, nb, pk, T, s->d_tw1f, b, st);
  else plane_inv_t<N, float, float2, HB, B>(s, nb, pk, T, s->d_tw1f, b, st);
}

template <int N, bool B>
static void plane_inv_n(const ks_system* s, int nb, const void* pk, bool in_fp64, void* T, const BatchRef& b,
                        hipStream_t st) {
  if (s->yz_half) plane_inv_h<N, true, B>(s, nb, pk, in_fp64, T, b, st);
  else plane_inv_h<N, false, B>(s, nb, pk, in_fp64, T, b, st);
}

bool launch_plane_inv(const ks_system* s, int nb, const void* pk, bool in_fp64, void* T, hipStream_t st) {
  switch (s->n[1]) {
#define KS_CASE(v) case v: plane_inv_n<v, false>(s, nb, pk, in_fp64, T, BatchRef{}, st); return true;
    KS_SIZES(KS_CASE)
#undef KS_CASE
    default:
      return false;
  }
}

bool launch_plane_inv_batch(const ks_system* s, const BatchJob* jobs, const int4* rows, int nrows, bool in_fp64,
                            hipStream_t st) {
  const BatchRef b{jobs, rows, nrows};
  switch (s->n[1]) {
#define KS_CASE(v) case v: plane_inv_n<v, true>(s, 0, nullptr, in_fp64, nullptr, b, st); return true;
    KS_SIZES(KS_CASE)
#undef KS_CASE
    default:
      return false;
  }
}

template <int N, typename R, typename TW, bool HB, bool B>
static void plane_fwd_t(const ks_system* s, int nb, const void* U, const void* win, void* wout, void* acc, void* acc2,
                        HMode mode, Taylor tay, int next, void* T, const void* tw, const BatchRef& b, hipStream_t st) {
  const dim3 grid(s->nplanes, B ? b.nrows : plane_groups(s, nb));
  plane_fwd_kernel<N, R, TW, HB, B><<<grid, pcfg<N, R, true, HB>::NT, plane_smem<true>(s), st>>>(
      (const cplx<R>*)U, nb, (const TW*)win, (cplx<R>*)wout, (double2*)acc, (double2*)acc2, s->npw_stride, s->npw_stride,
      sphere_tab(s), s->d_kin, (const cplx<R>*)tw, s->ncol_max, (int)mode, tay, next, (cplx<R>*)T, b.jobs,
      b.rows);
}

template <int N, bool HB, bool B>
static void plane_fwd_h(const ks_system* s, int nb, const void* U, const void* win, bool win_fp64, void* wout,
                        void* acc, void* acc2, HMode mode, Taylor tay, int next, void* T, const BatchRef& b,
                        hipStream_t st) {
  if (!mixed(s))
    plane_fwd_t<N, double, double2, HB, B>(s, nb, U, win, wout, acc, acc2, mode, tay, next, T, s->d_tw1, b, st);
  else if (win_fp64)
    plane_fwd_t<N, float, double2, HB, B>(s, nb, U, win, wout, acc, acc2, mode, tay, next, T, s->d_tw1f, b, st);
  else
    plane_fwd_t<N, float, float2, HB, B>(s, nb, U, win, wout, acc, acc2, mode, tay, next, T, s->d_tw1f, b, st);
}

template <int N, bool B>
static void plane_fwd_n(const ks_system* s, int nb, const void* U, const void* win, bool win_fp64, void* wout,
                        void* acc, void* acc2, HMode mode, Taylor tay, int next, void* T, const BatchRef& b,
                        hipStream_t st) {
  if (s->yz_half) plane_fwd_h<N, true, B>(s, nb, U, win, win_fp64, wout, acc, acc2, mode, tay, next, T, b, st);
  else plane_fwd_h<N, false, B>(s, nb, U, win, win_fp64, wout, acc, acc2, mode, tay, next, T, b, st);
}

bool launch_plane_fwd(const ks_system* s, int nb, const void* U, const void* win, bool win_fp64, void* wout,
                      void* acc, void* acc2, HMode mode, Taylor tay, int next, void* T, hipStream_t st) {
  switch (s->n[1]) {
#define KS_CASE(v) \
  case v: plane_fwd_n<v, false>(s, nb, U, win, win_fp64, wout, acc, acc2, mode, tay, next, T, BatchRef{}, st); return true;
    KS_SIZES(KS_CASE)
#undef KS_CASE
    default:
      return false;
  }
}

bool launch_plane_fwd_batch(const ks_system* s, const BatchJob* jobs, const int4* rows, int nrows, bool win_fp64,
                            Taylor tay, int next, hipStream_t st) {
  const BatchRef b{jobs, rows, nrows};
  switch (s->n[1]) {
#define KS_CASE(v)                                                                                              \
  case v:                                                                                                       \
    plane_fwd_n<v, true>(s, 0, nullptr, nullptr, win_fp64, nullptr, nullptr, nullptr, H_TAYLOR, tay, next, nullptr, b, st); \
    return true;
    KS_SIZES(KS_CASE)
#undef KS_CASE
    default:
      return false;
  }
}

// Whether the plane analyses of a launch over `orbitals` go on to the next
// synthesis (the results are the same, bit for bit).
// - The coefficients of the G orbitals' plane have to fit the y-batch's LDS,
//   which is free by then.  They do not on spheres wide for their plane: with
//   E_cut = 10 Ha from a spacing of 0.30 bohr on at 128 points, 0.36 at 120
//   in complex64, 0.48 at 72 in FP64, 0.58 at 40 and 96 in complex64, 48 and
//   60 in FP64, 64 and 80 in both.
// - In FP64 at 60, 72 and 80 points, in the band, the synthesis runs slower in the
//   analysis's work split than in its own, by more than a launch once the launch has over
//   about eight blocks per compute unit.  Steps of 4 H psi, two launches against
//   one, default group caps, us: 60^3 / 64 orbitals (1792 blocks) 706 and 697, /
//   96 (2688) 968 and 981, / 160 1531 and 1559; 72^3 / 48 (1584) 877 and 865, /
//   192 (6336) 2928 and 2970; 80^3 / 32 (1184) 775 and 773, / 48 (1776) 1054 and
//   1068, / 192 (7104) 3649 and 3704.
// Elsewhere one launch was faster or within the spread (see the kernel), but for
// 96 points in FP64 between 64 and 128 orbitals (2051 and 2067 us / 64, 3003 and
// 3072 / 96, 3889 and 3924 / 128; 1164 and 1144 / 32, 15258 and 15111 / 512), 40
// in complex64 at 512 (945 and 963) and 120 in complex64 at 96 (4522 and 4578;
// 22589 and 22098 / 512): no line between sizes or launches separates those.
bool plane_next(const ks_system* s, long long orbitals) {
  const int n = s->n[1];
  if (!mixed(s) && s->yz_half && (n == 60 || n == 72 || n == 80) && s->nplanes * orbitals > 2048) return false;
  bool fits = false;
  with_plane_cfg<true>(s, [&](auto c) {
    fits = (size_t)decltype(c)::G * s->npp_max <= (size_t)decltype(c)::YB * (n + 1);
  });
  return fits;
}

}  // namespace ks
