// Launches of the plane passes on orbitals in boxes (HIP, gfx950): H psi and
// the density of boxes without packed copies.  Bound: launches for small
// systems, the box itself for large ones.  With pack and unpack passes of their
// own and here: H psi of 16^3, 8 orbitals 28.4 and 23.3 us; 48 x 40 x 40, 33
// orbitals 61.9 and 57.6 us (the analysis that fills the box takes 18.2 us, as
// long as the packed one and the unpack); the reciprocal-space projections read
// packed orbitals and keep those passes.
#include "plane_kernels.hpp"

namespace ks {

template <int N, typename R, bool HB>
static void box_inv_h(const ks_system* s, int nb, const double2* box, void* T, const void* tw, hipStream_t st) {
  plane_inv_kernel<N, R, double2, HB, false, true>
      <<<dim3(s->nplanes, plane_groups(s, nb)), pcfg<N, R, false, HB>::NT, plane_smem<false>(s), st>>>(
          box, nb, 0, (cplx<R>*)T, sphere_tab(s), (const cplx<R>*)tw, s->ncol_max, 0, nullptr, nullptr);
}

template <int N, typename R>
static void box_inv_n(const ks_system* s, int nb, const double2* box, void* T, const void* tw, hipStream_t st) {
  if (s->yz_half) box_inv_h<N, R, true>(s, nb, box, T, tw, st);
  else box_inv_h<N, R, false>(s, nb, box, T, tw, st);
}

bool launch_plane_inv_box(const ks_system* s, int nb, const double2* box, void* T, hipStream_t st) {
  switch (s->n[1]) {
#define KS_CASE(v)                                               \
  case v:                                                        \
    if (mixed(s)) box_inv_n<v, float>(s, nb, box, T, s->d_tw1f, st); \
    else box_inv_n<v, double>(s, nb, box, T, s->d_tw1, st);      \
    return true;
    KS_SIZES(KS_CASE)
#undef KS_CASE
    default:
      return false;
  }
}

template <int N, typename R, bool HB>
static void box_fwd_h(const ks_system* s, int nb, const void* U, const double2* in, double2* out, const void* tw,
                      hipStream_t st) {
  plane_fwd_kernel<N, R, double2, HB, false, true>
      <<<dim3(s->n[0], plane_groups(s, nb)), pcfg<N, R, true, HB>::NT, plane_smem<true>(s), st>>>(
          (const cplx<R>*)U, nb, in, nullptr, out, nullptr, 0, 0, sphere_tab(s), s->d_kin, (const cplx<R>*)tw, s->ncol_max,
          (int)H_OUT, Taylor{{0.0, 0.0}, 0, {0.0, 0.0}}, 0, nullptr, nullptr, nullptr);
}

template <int N, typename R>
static void box_fwd_n(const ks_system* s, int nb, const void* U, const double2* in, double2* out, const void* tw,
                      hipStream_t st) {
  if (s->yz_half) box_fwd_h<N, R, true>(s, nb, U, in, out, tw, st);
  else box_fwd_h<N, R, false>(s, nb, U, in, out, tw, st);
}

bool launch_plane_fwd_box(const ks_system* s, int nb, const void* U, const double2* in, double2* out, hipStream_t st) {
  switch (s->n[1]) {
#define KS_CASE(v)                                                   \
  case v:                                                            \
    if (mixed(s)) box_fwd_n<v, float>(s, nb, U, in, out, s->d_tw1f, st); \
    else box_fwd_n<v, double>(s, nb, U, in, out, s->d_tw1, st);      \
    return true;
    KS_SIZES(KS_CASE)
#undef KS_CASE
    default:
      return false;
  }
}

}  // namespace ks
