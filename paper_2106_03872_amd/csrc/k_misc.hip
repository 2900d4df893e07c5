// Small kernels of the hot path (HIP, gfx950): box <-> packed sphere
// conversion at the boundary, the per-atom KB projection sums (Eq. vnl),
// norms and band energy reductions.
#include "ks_common.hpp"

namespace ks {

bool supported_size(int n) {
  switch (n) {
#define KS_CASE(v) case v:
    KS_SIZES(KS_CASE)
#undef KS_CASE
    return true;
    default:
      return false;
  }
}

int x_tile_nb(int n0) { return n0 <= 32 ? 64 : 32; }

// ------------------------------------------------------------ pack / unpack

template <typename T>
__global__ __launch_bounds__(NT) void pack_kernel(const double2* __restrict__ box, long long box_stride,
                                                  T* __restrict__ pk, int pk_stride, SphereTab tab) {
  __shared__ int s_off[130];
  __shared__ int s_m2lo[129];
  const int pi = blockIdx.x, o = blockIdx.y, tid = threadIdx.x;
  const int c0 = tab.plane_col0[pi], nc = tab.plane_col0[pi + 1] - c0;
  for (int i = tid; i <= nc; i += NT) s_off[i] = tab.col_off[c0 + i];
  for (int i = tid; i < nc; i += NT) s_m2lo[i] = tab.col_m2lo[c0 + i];
  __syncthreads();
  const int j0 = wrap(tab.m0lo + pi, tab.n0);
  const int m1lo = tab.plane_m1lo[pi];
  const double2* b = box + (long long)o * box_stride + (long long)j0 * tab.n1 * tab.n2;
  T* out = pk + (long long)o * pk_stride;
  for (int e = s_off[0] + tid; e < s_off[nc]; e += NT) {
    const int c = find_col(s_off, nc, e);
    const int m1 = m1lo + c, m2 = s_m2lo[c] + (e - s_off[c]);
    out[e] = to_c<T>(b[(long long)wrap(m1, tab.n1) * tab.n2 + wrap(m2, tab.n2)]);
  }
}

// Block (box plane j0, orbital): planes outside the sphere are a plain fill;
// in a plane of the sphere a thread finds its element's column in the plane's
// tables (in LDS).  Bound: HBM writes of the box.  One thread per element of
// the whole box, with its indices divided out of a 64-bit position and five
// dependent table loads, wrote 3.9 TB/s at 96^3 / 512 orbitals (1830 us); this
// form writes 5.0 TB/s (1450 us; 64^3 / 128: 148 and 108 us; 120^3 / 1024: 7080
// and 5890 us).
template <int N, typename T>
__global__ __launch_bounds__(NT) void unpack_kernel(const T* __restrict__ pk, int pk_stride,
                                                    double2* __restrict__ box, long long box_stride,
                                                    SphereTab tab) {
  __shared__ int s_off[130];
  __shared__ int s_m2lo[129];
  const int j0 = blockIdx.x, tid = threadIdx.x;
  const long long o = blockIdx.y;
  double2* out = box + o * box_stride + (long long)j0 * (N * N);
  const int pi = fold(j0, tab.n0) - tab.m0lo;
  if (pi < 0 || pi >= tab.nplanes) {
#pragma unroll 4
    for (int i = tid; i < N * N; i += NT) st_stream(out + i, double2{0.0, 0.0});
    return;
  }
  const int c0 = tab.plane_col0[pi], nc = tab.plane_col0[pi + 1] - c0, m1lo = tab.plane_m1lo[pi];
  for (int i = tid; i <= nc; i += NT) s_off[i] = tab.col_off[c0 + i];
  for (int i = tid; i < nc; i += NT) s_m2lo[i] = tab.col_m2lo[c0 + i];
  __syncthreads();
  const T* in = pk + o * pk_stride;
  for (int i = tid; i < N * N; i += NT) {
    const int j1 = i / N, j2 = i - j1 * N;
    const int c = fold(j1, N) - m1lo;
    double2 v{0.0, 0.0};
    if (c >= 0 && c < nc) {
      const int t = fold(j2, N) - s_m2lo[c], off = s_off[c];
      if (t >= 0 && t < s_off[c + 1] - off) v = to_d(in[off + t]);
    }
    st_stream(out + i, v);
  }
}

// Block = wave of projection lanes; thread = lane.
__global__ __launch_bounds__(64) void lane_rows_kernel(const int4* __restrict__ item, const int* __restrict__ lane_off,
                                                       const int* __restrict__ pt_lds, const double* __restrict__ beta,
                                                       int np, int n0, unsigned short* __restrict__ lane_pos,
                                                       double* __restrict__ lane_beta) {
  const int w = blockIdx.x, lane = threadIdx.x;
  const int4 it = item[(long long)w * 64 + lane];
  const int q = it.z % np;
  for (int r = lane_off[w], k = it.x; r < lane_off[w + 1]; ++r, ++k) {
    const bool in = k < it.y;
    lane_pos[(long long)r * 64 + lane] = (unsigned short)(in ? pt_lds[k] : n0);
    lane_beta[(long long)r * 64 + lane] = in ? beta[(long long)k * np + q] : 0.0;
  }
}

// KB projections: P_Ip = sum over the (tile, atom) slots of atom I in
// ascending tile order, DP = scale d_Ip P_Ip (Eq. vnl; scale is the analysis
// normalisation that the x-analysis leaves out).  One wavefront per (atom,
// orbital): lane = 8 * slot-lane + q; slot-lanes are combined in a fixed order.
// BATCH: block (I, y) reduces orbital rows[y].y of job rows[y].x (its
// partial sums, coefficients and tables); atoms beyond the job's count exit.
template <typename C, bool BATCH = false>
__global__ __launch_bounds__(64) void proj_reduce_kernel(const C* __restrict__ partial, double2* __restrict__ DP,
                                                         ProjTab pt, double scale,
                                                         const BatchJob* __restrict__ jobs = nullptr,
                                                         const int4* __restrict__ rows = nullptr) {
  __shared__ double2 red[64];
  const int I = blockIdx.x, lane = threadIdx.x;
  int o = blockIdx.y;
  if constexpr (BATCH) {
    const int4 r = rows[blockIdx.y];
    partial = static_cast<const C*>(jobs[r.x].partial);
    DP = jobs[r.x].DP;
    pt = jobs[r.x].pt;
    o = r.y;
    if (I >= pt.natoms) return;   // uniform per block
  }
  const int q = lane & 7, sl = lane >> 3;
  const int np = pt.nproj;
  double sx = 0.0, sy = 0.0;
  if (q < np) {
    for (int k = pt.atom_slot_off[I] + sl; k < pt.atom_slot_off[I + 1]; k += 8) {
      const C v = partial[((long long)o * pt.nslots + k) * np + q];
      sx += double(v.x);
      sy += double(v.y);
    }
  }
  red[lane] = double2{sx, sy};
  __syncthreads();
  if (lane < 8 && q < np) {
    double tx = 0.0, ty = 0.0;
    for (int j = 0; j < 8; ++j) {
      tx += red[j * 8 + lane].x;
      ty += red[j * 8 + lane].y;
    }
    const double dd = pt.d[I * np + q] * scale;
    DP[((long long)o * pt.natoms + I) * np + q] = double2{dd * tx, dd * ty};
  }
}

// sum over the lanes of a wave (a fixed butterfly: every lane gets the sum)
__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) x += __shfl_xor(x, m, 64);
  return x;
}

// per-orbital sums over the packed sphere: out[2o] = sum |a|^2, out[2o+1] =
// sum Re conj(a) b; norms (nullable): norms[o] = sum |a|^2 as well.
// Bound: HBM reads of the orbitals.  A block of 256 threads with one load in
// flight per thread took 15.7 us for 128 orbitals at 64^3 and 90 us for 512
// at 96^3 (3.7 TB/s), and the norms were gathered by a strided copy of 4 us;
// 512 threads with four loads each take 6.4 and 57 us.
constexpr int NT_DOT = 512, DOT_U = 4;
template <typename CA, typename CB_>
__global__ __launch_bounds__(NT_DOT) void dots_kernel(const CA* __restrict__ a, const CB_* __restrict__ b, int stride,
                                                      int npw, double* __restrict__ out, double* __restrict__ norms) {
  __shared__ double s0[NT_DOT / 64], s1[NT_DOT / 64];
  const int o = blockIdx.x, tid = threadIdx.x;
  const CA* pa = a + (long long)o * stride;
  const CB_* pb = b ? b + (long long)o * stride : nullptr;
  double x0[DOT_U], x1[DOT_U];
#pragma unroll
  for (int j = 0; j < DOT_U; ++j) x0[j] = x1[j] = 0.0;
  for (int e0 = tid; e0 < npw; e0 += DOT_U * NT_DOT) {
    CA u[DOT_U];
#pragma unroll
    for (int j = 0; j < DOT_U; ++j) {
      const int e = e0 + j * NT_DOT;
      u[j] = e < npw ? pa[e] : CA{0, 0};
    }
#pragma unroll
    for (int j = 0; j < DOT_U; ++j) x0[j] += double(u[j].x) * double(u[j].x) + double(u[j].y) * double(u[j].y);
    if (pb) {
      CB_ v[DOT_U];
#pragma unroll
      for (int j = 0; j < DOT_U; ++j) {
        const int e = e0 + j * NT_DOT;
        v[j] = e < npw ? pb[e] : CB_{0, 0};
      }
#pragma unroll
      for (int j = 0; j < DOT_U; ++j) x1[j] += double(u[j].x) * double(v[j].x) + double(u[j].y) * double(v[j].y);
    }
  }
  const double y0 = wave_sum((x0[0] + x0[1]) + (x0[2] + x0[3])), y1 = wave_sum((x1[0] + x1[1]) + (x1[2] + x1[3]));
  if ((tid & 63) == 0) {
    s0[tid >> 6] = y0;
    s1[tid >> 6] = y1;
  }
  __syncthreads();
  if (tid == 0) {
    double t0 = 0.0, t1 = 0.0;
    for (int w = 0; w < NT_DOT / 64; ++w) {
      t0 += s0[w];
      t1 += s1[w];
    }
    out[2 * o] = t0;
    out[2 * o + 1] = t1;
    if (norms) norms[o] = t0;
  }
}

// energy = sum_o occ[o] red[2o+1], in a fixed order (one wave)
__global__ __launch_bounds__(64) void energy_sum_kernel(int norb, const double* __restrict__ occ,
                                                        const double* __restrict__ red, double* __restrict__ energy) {
  double e = 0.0;
  for (int o = threadIdx.x; o < norb; o += 64) e += occ[o] * red[2 * o + 1];
  e = wave_sum(e);
  if (threadIdx.x == 0) energy[0] = e;
}

// ------------------------------------------------------------------ launchers

bool launch_pack(const ks_system* s, int nb, const double2* box, long long box_stride, void* pk, hipStream_t st) {
  pack_kernel<double2><<<dim3(s->nplanes, nb), NT, 0, st>>>(box, box_stride, (double2*)pk, s->npw_stride,
                                                             sphere_tab(s));
  return true;
}

bool launch_unpack(const ks_system* s, int nb, const void* pk, bool pk_fp64, double2* box, long long box_stride,
                   hipStream_t st) {
  const dim3 grid(s->n[0], nb);
  switch (s->n[1]) {
#define KS_CASE(v)                                                                                               \
  case v:                                                                                                        \
    if (pk_fp64)                                                                                                 \
      unpack_kernel<v, double2><<<grid, NT, 0, st>>>((const double2*)pk, s->npw_stride, box, box_stride, sphere_tab(s)); \
    else                                                                                                         \
      unpack_kernel<v, float2><<<grid, NT, 0, st>>>((const float2*)pk, s->npw_stride, box, box_stride, sphere_tab(s)); \
    return true;
    KS_SIZES(KS_CASE)
#undef KS_CASE
    default:
      return false;
  }
}

void launch_lane_rows(int nwaves, const int4* item, const int* lane_off, const int* pt_lds, const double* beta, int np,
                      int n0, unsigned short* lane_pos, double* lane_beta, hipStream_t st) {
  lane_rows_kernel<<<nwaves, 64, 0, st>>>(item, lane_off, pt_lds, beta, np, n0, lane_pos, lane_beta);
}

bool launch_proj_reduce(const ks_system* s, int nb, const void* partial, double2* DP, hipStream_t st) {
  if (s->natoms == 0 || nb == 0) return true;
  const double scale = sqrt(s->omega) / (double)s->N;
  if (!mixed(s))
    proj_reduce_kernel<double2><<<dim3(s->natoms, nb), 64, 0, st>>>((const double2*)partial, DP, proj_tab(s), scale);
  else
    proj_reduce_kernel<float2><<<dim3(s->natoms, nb), 64, 0, st>>>((const float2*)partial, DP, proj_tab(s), scale);
  return true;
}

bool launch_proj_reduce_batch(const ks_system* s, const BatchJob* jobs, const int4* rows, int nrows, int max_natoms,
                              hipStream_t st) {
  if (max_natoms == 0 || nrows == 0) return true;
  const double scale = sqrt(s->omega) / (double)s->N;
  if (!mixed(s))
    proj_reduce_kernel<double2, true><<<dim3(max_natoms, nrows), 64, 0, st>>>(nullptr, nullptr, ProjTab{}, scale, jobs,
                                                                             rows);
  else
    proj_reduce_kernel<float2, true><<<dim3(max_natoms, nrows), 64, 0, st>>>(nullptr, nullptr, ProjTab{}, scale, jobs,
                                                                            rows);
  return true;
}

// a: the FP64 state; b: H applied to it in the working precision (or null)
bool launch_dots(const ks_system* s, int nb, const void* a, const void* b, double* out, double* norms, hipStream_t st) {
  if (!mixed(s))
    dots_kernel<double2, double2><<<nb, NT_DOT, 0, st>>>((const double2*)a, (const double2*)b, s->npw_stride, s->npw,
                                                         out, norms);
  else
    dots_kernel<double2, float2><<<nb, NT_DOT, 0, st>>>((const double2*)a, (const float2*)b, s->npw_stride, s->npw,
                                                        out, norms);
  return true;
}

bool launch_energy_sum(int norb, const double* occ, const double* red, double* energy, hipStream_t st) {
  energy_sum_kernel<<<1, 64, 0, st>>>(norb, occ, red, energy);
  return true;
}

}  // namespace ks
