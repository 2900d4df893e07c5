// x-pencil passes of the Kohn-Sham Hamiltonian (HIP, gfx950): x-synthesis
// in LDS, Kleinman-Bylander projections (Eq. vnl), local potential and KB
// scatter, x-analysis; the density sum (Eq. density).
#include "ks_common.hpp"

namespace ks {

// -------------------------------------------------------------- x-pencil passes
// Block (tile of NB consecutive pencils p = j1*n2 + j2, orbital o).  The
// x-synthesis reads T (planes m0 of each pencil) straight into its first
// stage; LDS X[w][j0] holds one exchange buffer of the tile.

// T and U of one orbital are [nplanes][npl] (npl = n1 n2 pencils).  TPos
// gives the byte offset of element e of the tile's pencil t in that array, or
// OOB for an element outside the sphere's planes or a pencil beyond the last
// (buffer access then loads zero and drops stores).
//
// What bounds these passes: the x-tile makes two (xproj) or four (xapply)
// trips through LDS per orbital, each behind a barrier, at three (FP64) or
// four (complex64) waves per SIMD, so the SIMDs alternate between issue and
// waiting, and every instruction beside the transform's own counts.  With
// per-element branches, zero fills and 64-bit addresses the orbital loop of
// xproj had 131 integer and 170 scalar instructions beside 276 FP64 ones; it
// has 108 and 50.  Measured together with the projection reads in groups and
// the twiddle rows, per launch before and after: 96^3 / 512 orbitals FP64
// xproj 964 and 875 us, xapply 1543 and 1451 us (4.2 and 4.5 TB/s); complex64
// xapply 1074 and 987 us; 120^3 / 1024 complex64 xproj 2758 and 2502 us, xapply
// 4592 and 4377 us.
template <int N0, typename C>
struct TPos {
  int npl, nplanes, m0lo, p0;
  static constexpr unsigned BEYOND = 0x40000000u;   // past every array, also after adding a plane's offset
  __device__ TPos(const SphereTab& tab, int p0_) : npl(tab.n1 * tab.n2), nplanes(tab.nplanes), m0lo(tab.m0lo), p0(p0_) {}
  __device__ __forceinline__ unsigned bytes() const { return (unsigned)(nplanes * npl) * sizeof(C); }
  __device__ __forceinline__ unsigned pencil(int t) const {
    return t >= 0 && p0 + t < npl ? (unsigned)(p0 + t) * sizeof(C) : BEYOND;
  }
  // plane pi of the pencil at byte offset pb
  __device__ __forceinline__ unsigned plane(unsigned pb, int pi) const {
    const unsigned off = pb + (unsigned)__mul24(pi, npl * (int)sizeof(C));
    return (unsigned)pi < (unsigned)nplanes ? off : OOB;
  }
  __device__ __forceinline__ unsigned operator()(int t, int e) const { return plane(pencil(t), fold(e, N0) - m0lo); }
};

// Issue the loads of a thread's first-stage inputs of one orbital (T of
// `bytes` bytes) into r.  The offsets are formed anew for each orbital (four
// instructions per element): kept across orbitals they take the FP64 passes
// past the 168 registers of three waves per SIMD.
//
// Past the band (not FR::half) two fifths of the elements lie outside the
// sphere's planes at a spacing of 0.42 bohr, and their loads, though they only
// return zeros, take issue slots; a branch skips them: the density pass of 160
// orbitals in complex64 took 103 us at 80^3 before buffer access, 127 with it
// and 106 with the branch.
template <class FR, int N0, typename C>
__device__ __forceinline__ void load_inputs(FR& r, const TPos<N0, C>& pos, const C* T, unsigned bytes) {
  const gbuf b = make_gbuf(T, bytes);
  first_stage_positions<FR>([&](int it, int s, int t, int e) {
    const unsigned off = pos(t, e);
    if constexpr (FR::half) {
      r.v[it][s] = buf_load<C, true>(b, off);
    } else {
      r.v[it][s] = czero<C>();
      if (off < bytes) r.v[it][s] = buf_load<C, true>(b, off);
    }
  });
}

// x from another lane of the same row of 16 by the DPP permutation CTRL
// (quad_perm, row_half_mirror, row_mirror: every source lane is in the row)
template <int CTRL>
__device__ __forceinline__ double dpp_lane(double x) {
  const long long b = __builtin_bit_cast(long long, x);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, false);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}
constexpr int DPP_QUAD_XOR1 = 0xB1;   // quad_perm [1, 0, 3, 2]
constexpr int DPP_QUAD_XOR2 = 0x4E;   // quad_perm [2, 3, 0, 1]
constexpr int DPP_HALF_MIRROR = 0x141;
constexpr int DPP_MIRROR = 0x140;

// Orbital groups: block (tile, y) handles the orbitals [y*nb/ng, (y+1)*nb/ng)
// of its tile in order (ng = gridDim.y).  The next orbital's T is loaded into
// registers while the current one is transformed, and the per-tile data
// (twiddles, potential, KB tables) is fetched once per block.

// DENS: the block also accumulates the density sum_o occ_o |psi_o|^2 / Omega
// of its orbitals from the synthesis outputs and writes its group's partial
// density (as xdens does), so a propagation step gets the density of its
// input orbitals from its first H psi.
// BATCH: one launch over several systems of the grid (no density); the
// block's system (T, partial sums, projector tables, orbital count) comes
// from jobs[rows[blockIdx.y].x].
template <int N0, class SH, typename R, bool HB, bool DENS, bool BATCH = false>
__global__ __launch_bounds__(SH::XT) void xproj_kernel(const cplx<R>* __restrict__ Tin, int nb,
                                                   cplx<R>* __restrict__ partial, SphereTab tab, ProjTab pt,
                                                   const cplx<R>* __restrict__ tw0, double scale,
                                                   const double* __restrict__ occ, double* __restrict__ dpart,
                                                   double inv_omega, const BatchJob* __restrict__ jobs = nullptr,
                                                   const int4* __restrict__ rows = nullptr) {
  using C = cplx<R>;
  static_assert(!(BATCH && DENS), "batched launches carry no density");
  constexpr int NB = SH::NB, XT = SH::XT;
  using FR = fft_regs<N0, NB, XT, C, HB, SH::V>;
  using LS = last_shape<N0, NB, XT, SH::V>;
  __shared__ C X[NB * (N0 + 1)];
  __shared__ C tw[N0];
  const int tile = blockIdx.x, tid = threadIdx.x;
  int oa, ob;
  if constexpr (BATCH) {
    const int4 r = rows[blockIdx.y];
    Tin = static_cast<const C*>(jobs[r.x].T);
    partial = static_cast<C*>(jobs[r.x].partial);
    pt = jobs[r.x].pt;
    nb = jobs[r.x].nb;
    group_range(nb, r.y, r.z, oa, ob);
  } else {
    orbital_range(nb, oa, ob);
  }
  const int npl = tab.n1 * tab.n2;
  const int p0 = tile * NB;
  // the block's first loads, independent of each other, are issued together:
  // the first orbital, the work item, the slot range, the twiddles
  const TPos<N0, C> pos(tab, p0);
  const unsigned tbytes = pos.bytes();
  const long long tstride = (long long)tab.nplanes * npl;
  FR pre;
  if (oa < ob) load_inputs(pre, pos, Tin + oa * tstride, tbytes);
  const int wave = __builtin_amdgcn_readfirstlane(tile * (XT / 64) + tid / 64);
  int4 item;
  int row0, nrow;   // this wave's rows
  auto read_item = [&] {
    item = pt.item[(long long)tile * XT + tid];
    row0 = pt.lane_off[wave];
    nrow = pt.lane_off[wave + 1] - row0;
  };
  if constexpr (!BATCH) read_item();
  const int sA = pt.slot_off[tile], ns = pt.slot_off[tile + 1] - sA;
  if (!DENS && ns == 0) return;  // no sphere point in this tile (uniform per block)
  // A batch runs over all its systems, and one whose projectors were never set
  // has slot_off alone of these tables: the others are read after the return.
  if constexpr (BATCH) read_item();
  stage_twiddles<N0, XT, SH::V>(tw, tw0);
  double a[DENS ? LS::items : 1][DENS ? LS::radix : 1];
  if constexpr (DENS) {
#pragma unroll
    for (int it = 0; it < LS::items; ++it)
#pragma unroll
      for (int q = 0; q < LS::radix; ++q) a[it][q] = 0.0;
  }
  // Projections: each lane sums beta * psi over its rows of one (slot,
  // projector) pair of the tile (in point order); the 2^g lanes of a
  // pair, adjacent and aligned, are then added by a fixed butterfly and the
  // group's first lane writes the pair (work planned per tile on the host).
  // (the host plans XT projection lanes per tile)
  const int np = pt.nproj;
  const int glanes = 1 << (item.w & 0xff);
  const bool writer = (item.w & 256) != 0;
  // The first KP rows of the lanes (LDS position, beta) are the same for all
  // orbitals of the block and stay in registers.  Rows are read in groups of
  // KPG, with one coalesced load of each array per row (see build_proj); rows a
  // lane lacks add beta = 0 times the unused last word of the first pencil's row
  // (zero).
  constexpr int KP = KB_CACHED_POINTS, KPG = KB_ROW_GROUP;
  static_assert(KP % KPG == 0, "whole groups");
  const unsigned short* const lpos = pt.lane_pos + (long long)row0 * 64 + (tid & 63);
  const double* const lbeta = pt.lane_beta + (long long)row0 * 64 + (tid & 63);
  int cpos[KP];
  double cbeta[KP];
  if (tid == 0) X[N0] = czero<C>();
#pragma unroll
  for (int g = 0; g < KP; g += KPG) {
    if (g < nrow) {
#pragma unroll
      for (int c = g; c < g + KPG; ++c) {
        cpos[c] = lpos[c * 64];
        cbeta[c] = lbeta[c * 64];
      }
    } else {
#pragma unroll
      for (int c = g; c < g + KPG; ++c) {
        cpos[c] = 0;
        cbeta[c] = 0.0;
      }
    }
  }
  C* pout = partial + item.z;
  const long long pstride = (long long)pt.nslots * np;
  for (int o = oa; o < ob; ++o) {
    auto next = [&] {
      if (o + 1 < ob) load_inputs(pre, pos, Tin + (o + 1) * tstride, tbytes);
    };
    if constexpr (DENS) {
      const double f = occ[o] * inv_omega;
      fft_io<N0, +1, NB, XT, SRC_PRE, DST_FN_LDS, C, SH::V>(X, N0 + 1, NB, tw, preloaded(pre, next),
                                                   [&](int t, int e, C v, int it, int q) {
                                                     X[t * (N0 + 1) + e] = v;
                                                     a[it][q] += f * (double(v.x) * double(v.x) + double(v.y) * double(v.y));
                                                   });
      if (ns == 0) {
        __syncthreads();   // X is rewritten by the next orbital's first stage
        continue;
      }
    } else {
      fft_io<N0, +1, NB, XT, SRC_PRE, DST_LDS, C, SH::V>(X, N0 + 1, NB, tw, preloaded(pre, next), no_store{});
    }
    double sx = 0.0, sy = 0.0;
#pragma unroll
    for (int g = 0; g < KP; g += KPG) {
      if (g < nrow) {
        C x[KPG];
#pragma unroll
        for (int c = 0; c < KPG; ++c) x[c] = X[cpos[g + c]];
#pragma unroll
        for (int c = 0; c < KPG; ++c) {
          sx += cbeta[g + c] * double(x[c].x);
          sy += cbeta[g + c] * double(x[c].y);
        }
      }
    }
    for (int k = KP; k < nrow; k += KPG) {
      int p[KPG];
      double bv[KPG];
#pragma unroll
      for (int c = 0; c < KPG; ++c) {
        p[c] = lpos[(k + c) * 64];
        bv[c] = lbeta[(k + c) * 64];
      }
#pragma unroll
      for (int c = 0; c < KPG; ++c) {
        const C x = X[p[c]];
        sx += bv[c] * double(x.x);
        sy += bv[c] * double(x.y);
      }
    }
    // the group's lanes add their sums by a fixed butterfly (the partners of
    // stage m: lane pairs of a quad, then quads, then mirrored halves of 8 and
    // of 16 lanes; after stage m every lane of an aligned 2m-lane block holds
    // the block's sum, as with lane index xor m)
    static_assert(KB_MAX_GROUP_LOG == 4, "four butterfly stages");
    {
      double vx = dpp_lane<DPP_QUAD_XOR1>(sx), vy = dpp_lane<DPP_QUAD_XOR1>(sy);
      if (glanes > 1) {
        sx += vx;
        sy += vy;
      }
      vx = dpp_lane<DPP_QUAD_XOR2>(sx);
      vy = dpp_lane<DPP_QUAD_XOR2>(sy);
      if (glanes > 2) {
        sx += vx;
        sy += vy;
      }
      vx = dpp_lane<DPP_HALF_MIRROR>(sx);
      vy = dpp_lane<DPP_HALF_MIRROR>(sy);
      if (glanes > 4) {
        sx += vx;
        sy += vy;
      }
      vx = dpp_lane<DPP_MIRROR>(sx);
      vy = dpp_lane<DPP_MIRROR>(sy);
      if (glanes > 8) {
        sx += vx;
        sy += vy;
      }
    }
    if (writer) pout[o * pstride] = C{R(sx * scale), R(sy * scale)};
    __syncthreads();   // X is rewritten by the next orbital's first stage
  }
  if constexpr (DENS) {
    double* pb = dpart + (long long)blockIdx.y * tab.n0 * npl + p0;
    last_stage_positions<N0, NB, XT, SH::V>(NB, [&](int it, int q, int t, int e) {
      if (p0 + t < npl) pb[e * npl + t] = a[it][q];
    });
  }
}

// KB scatter (Eq. vnl): X[point] += sum over the point's entries (in atom
// order) of beta_entry . dP[slot].
template <typename C>
__device__ __forceinline__ void kb_add(C* X, int key, double fx, double fy) {
  C& x = X[key & ((1 << UP_POS_BITS) - 1)];
  x = C{decltype(x.x)(double(x.x) + fx), decltype(x.x)(double(x.y) + fy)};
}

// extra entries of a point where spheres overlap (rare)
__device__ __forceinline__ void kb_extra(const double2* dps, const ProjTab& pt, int np, int u, int key, double& fx,
                                         double& fy) {
  const int nx = key >> (UP_POS_BITS + UP_SLOT_BITS);
  if (nx == 0) return;
  const int x0 = pt.up_x[u];
  for (int e = x0; e < x0 + nx; ++e) {
    const double* b = pt.x_beta + (long long)e * np;
    const double2* dp = dps + pt.x_slot[e] * np;
    for (int q = 0; q < np; ++q) {
      fx += b[q] * dp[q].x;
      fy += b[q] * dp[q].y;
    }
  }
}

// NP projectors per atom fixed at compile time: two unique points per thread
// and pass, u and u + XT, with the table loads of both issued before either
// is used.
//
// A grid has at most 128^3 unique points of at most 8 projectors, so 32-bit
// byte offsets reach every row of the tables.
template <typename T>
__device__ __forceinline__ const T* row32(const T* base, unsigned index, unsigned row) {
  return reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + (index * row * (unsigned)sizeof(T)));
}
template <int NP, int XT, typename C>
__device__ __forceinline__ void kb_scatter_fixed(C* X, const double2* dps, const ProjTab& pt, int uA, int uB) {
  const int tid = threadIdx.x;
  for (int u = uA + tid; u < uB; u += 2 * XT) {
    const bool two = u + XT < uB;
    const int ub = two ? u + XT : u;
    const int ka = *row32(pt.up_key, u, 1);
    const int kb = *row32(pt.up_key, ub, 1);
    const double* rowa = row32(pt.up_beta, u, NP);
    const double* rowb = row32(pt.up_beta, ub, NP);
    double ba[NP], bb[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      ba[q] = rowa[q];
      bb[q] = rowb[q];
    }
    __builtin_amdgcn_sched_barrier(0);   // no use of a key before the rows' loads are issued
    const double2* da = dps + ((ka >> UP_POS_BITS) & UP_MAX_SLOT) * NP;
    const double2* db = dps + ((kb >> UP_POS_BITS) & UP_MAX_SLOT) * NP;
    double ax = 0.0, ay = 0.0, bx = 0.0, by = 0.0;
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const double2 pa = da[q], pb = db[q];
      ax += ba[q] * pa.x;
      ay += ba[q] * pa.y;
      bx += bb[q] * pb.x;
      by += bb[q] * pb.y;
    }
    kb_extra(dps, pt, NP, u, ka, ax, ay);
    kb_add(X, ka, ax, ay);
    if (two) {
      kb_extra(dps, pt, NP, ub, kb, bx, by);
      kb_add(X, kb, bx, by);
    }
  }
}

// any number of projectors per atom: one point at a time
template <int XT, typename C>
__device__ __forceinline__ void kb_scatter_any(C* X, const double2* dps, const ProjTab& pt, int uA, int uB) {
  const int np = pt.nproj, tid = threadIdx.x;
  for (int u = uA + tid; u < uB; u += XT) {
    const int key = pt.up_key[u];
    const double* b = pt.up_beta + (long long)u * np;
    const double2* dp = dps + ((key >> UP_POS_BITS) & UP_MAX_SLOT) * np;
    double fx = 0.0, fy = 0.0;
    for (int q = 0; q < np; ++q) {
      fx += b[q] * dp[q].x;
      fy += b[q] * dp[q].y;
    }
    kb_extra(dps, pt, np, u, key, fx, fy);
    kb_add(X, key, fx, fy);
  }
}

// SUMS: the block sums its atoms' projections itself from xproj's partial sums
// (the same sums in the same order as proj_reduce), which saves that launch
// where launches, not their work, bound the pass.
//
// BATCH: as xproj_kernel (T, U, V, d P, projector tables and orbital count
// from the block's job).
template <int N0, class SH, typename R, bool HB, bool SUMS, bool BATCH = false>
__global__ __launch_bounds__(SH::XT) void xapply_kernel(const cplx<R>* __restrict__ Tin, int nb,
                                                    cplx<R>* __restrict__ Uout, const double* __restrict__ V,
                                                    const double2* __restrict__ DP,
                                                    const cplx<R>* __restrict__ partial, double sc_p, SphereTab tab,
                                                    ProjTab pt, const cplx<R>* __restrict__ tw0, double sc_v,
                                                    const BatchJob* __restrict__ jobs = nullptr,
                                                    const int4* __restrict__ rows = nullptr) {
  using C = cplx<R>;
  constexpr int NB = SH::NB, XT = SH::XT;
  using LS = last_shape<N0, NB, XT, SH::V>;
  using FR = fft_regs<N0, NB, XT, C, HB, SH::V>;
  __shared__ C X[NB * (N0 + 1)];
  __shared__ double2 dps[KB_TILE_DP];
  __shared__ C tw[N0];
  const int tile = blockIdx.x, tid = threadIdx.x;
  int oa, ob;
  if constexpr (BATCH) {
    const int4 r = rows[blockIdx.y];
    Tin = static_cast<const C*>(jobs[r.x].T);
    Uout = static_cast<C*>(jobs[r.x].U);
    V = jobs[r.x].V;
    DP = jobs[r.x].DP;
    partial = static_cast<const C*>(jobs[r.x].partial);
    pt = jobs[r.x].pt;
    nb = jobs[r.x].nb;
    group_range(nb, r.y, r.z, oa, ob);
  } else {
    orbital_range(nb, oa, ob);
  }
  const int npl = tab.n1 * tab.n2;
  const int p0 = tile * NB;
  const TPos<N0, C> pos(tab, p0);
  const unsigned tbytes = pos.bytes();
  const long long tstride = (long long)tab.nplanes * npl;
  FR pre;
  if (oa < ob) load_inputs(pre, pos, Tin + oa * tstride, tbytes);
  // potential at the outputs of this thread's last synthesis stage, times the
  // synthesis and analysis scales Omega^-1/2 Omega^1/2 / N = 1/N
  double vr[LS::items][LS::radix];
  const double* vbase = V + p0;
  last_stage_positions<N0, NB, XT, SH::V>(NB, [&](int it, int q, int t, int e) {
    vr[it][q] = (p0 + t < npl) ? vbase[e * npl + t] * sc_v : 0.0;
  });
  // KB coefficients d*P of this tile's slots: thread tid < ns*np stages one
  // (slot, projector) value per orbital.
  const int np = pt.nproj;
  const int sA = pt.slot_off[tile], ns = pt.slot_off[tile + 1] - sA;
  const int ndp = ns * np;   // <= KB_TILE_DP <= XT
  const long long dp_stride = (long long)pt.natoms * np;
  long long dp_off = 0;
  int4 sd = make_int4(0, 0, 0, 0);   // SUMS: this thread's range of partial sums
  double dd = 0.0;
  const C* psum = nullptr;
  if (tid < ndp) {
    const int sl = tid / np, q = tid - sl * np;
    sd = pt.slot_desc[sA + sl];
    dp_off = (long long)sd.z * np + q;
    if constexpr (SUMS) {
      dd = pt.d[dp_off] * sc_p;
      psum = partial + q;
    }
  }
  // d P of this thread's pair for orbital o: its partial sums in eight strided
  // sums, added in order
  auto sum_projection = [&](int o) {
    double sx[8], sy[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) sx[j] = sy[j] = 0.0;
    const C* po = psum + (long long)o * pt.nslots * np;
    for (int k0 = sd.x; k0 < sd.y; k0 += 8) {
      C v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = k0 + j < sd.y ? po[(long long)(k0 + j) * np] : czero<C>();
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        sx[j] += double(v[j].x);
        sy[j] += double(v[j].y);
      }
    }
    double tx = 0.0, ty = 0.0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      tx += sx[j];
      ty += sy[j];
    }
    return double2{dd * tx, dd * ty};
  };
  const int uA = pt.up_off[tile], uB = pt.up_off[tile + 1];
  stage_twiddles<N0, XT, SH::V>(tw, tw0);
  double2 dnext = {0.0, 0.0};
  if (!SUMS && tid < ndp && oa < ob) dnext = DP[oa * dp_stride + dp_off];
  for (int o = oa; o < ob; ++o) {
    // this orbital's d*P (fetched one orbital ahead); the previous orbital's
    // scatter has finished reading dps, and the stage barriers publish it
    if (tid < ndp) {
      if constexpr (SUMS) dnext = sum_projection(o);
      dps[tid] = dnext;
    }
    auto next = [&] {
      if (o + 1 < ob) {
        load_inputs(pre, pos, Tin + (o + 1) * tstride, tbytes);
        if (!SUMS && tid < ndp) dnext = DP[(o + 1) * dp_stride + dp_off];
      }
    };
    // synthesis, then psi <- V psi as the outputs are written
    fft_io<N0, +1, NB, XT, SRC_PRE, DST_FN_LDS, C, SH::V>(X, N0 + 1, NB, tw, preloaded(pre, next), [&](int t, int e, C v, int it, int q) {
      X[t * (N0 + 1) + e] = C{R(vr[it][q] * double(v.x)), R(vr[it][q] * double(v.y))};
    });
    if (ns > 0) {
      if (np == 4) kb_scatter_fixed<4, XT>(X, dps, pt, uA, uB);
      else kb_scatter_any<XT>(X, dps, pt, uA, uB);
      __syncthreads();
    }
    // The stores stay behind branches: the compiler then rounds the last
    // butterfly's products before their sums.  Without the branches it fuses
    // some of them, and the complex64 results change in their last bits from
    // one plan to the next.
    const gbuf ub = make_gbuf(Uout + o * tstride, tbytes);
    auto store = [&](int t, int e, C v, int, int q) {
      // in the band the frequency of output q follows from q alone
      const int m0 = HB && LS::radix % 4 == 0 ? (q < LS::radix / 4 ? e : e - N0) : fold(e, N0);
      const int pi = m0 - pos.m0lo;
      if (pi >= 0 && pi < pos.nplanes && p0 + t < npl)
        buf_store<true>(ub, (unsigned)((p0 + t) * (int)sizeof(C) + __mul24(pi, npl * (int)sizeof(C))), v);
    };
    // only the sphere's planes are stored; with HB they all lie in the band |m0| < n0/4
    if constexpr (HB) fft_io<N0, -1, NB, XT, SRC_LDS, DST_FN, C, SH::V>(X, N0 + 1, NB, tw, no_load{}, banded(store));
    else fft_io<N0, -1, NB, XT, SRC_LDS, DST_FN, C, SH::V>(X, N0 + 1, NB, tw, no_load{}, store);
    __syncthreads();   // X and dps are rewritten for the next orbital
  }
}

// density: block (tile, orbital group); |psi|^2 is accumulated
// straight from the last synthesis stage over the group's orbitals in order
// and written to the group's partial density; dens_sum adds the groups in
// order.
// (The band-limited FP64 form is held to the 168 registers of three waves per
// SIMD up to 96 points: 32 x 256 tiles of 96 spill two registers for it.  Beyond,
// two blocks of that tile fill the LDS of a compute unit.)
template <int N0, class SH, typename R, bool HB>
__global__ __launch_bounds__(SH::XT) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 8 && HB && N0 <= 96 ? 3 : 1))) void xdens_kernel(const cplx<R>* __restrict__ Tin, int nb,
                                                   const double* __restrict__ occ, double* __restrict__ part,
                                                   SphereTab tab, const cplx<R>* __restrict__ tw0,
                                                   double inv_omega) {
  using C = cplx<R>;
  constexpr int NB = SH::NB, XT = SH::XT;
  using LS = last_shape<N0, NB, XT, SH::V>;
  __shared__ C X[NB * (N0 + 1)];
  __shared__ C tw[N0];
  const int tile = blockIdx.x, g = blockIdx.y, tid = threadIdx.x;
  const int npl = tab.n1 * tab.n2;
  const int p0 = tile * NB;
  stage_twiddles<N0, XT, SH::V>(tw, tw0);
  double a[LS::items][LS::radix];
#pragma unroll
  for (int it = 0; it < LS::items; ++it)
#pragma unroll
    for (int q = 0; q < LS::radix; ++q) a[it][q] = 0.0;
  int oa, ob;
  orbital_range(nb, oa, ob);
  // the next orbital's T is loaded once the first stage has consumed the current one
  using FR = fft_regs<N0, NB, XT, C, HB, SH::V>;
  const TPos<N0, C> pos(tab, p0);
  const unsigned tbytes = pos.bytes();
  const long long tstride = (long long)tab.nplanes * npl;
  FR pre;
  if (oa < ob) load_inputs(pre, pos, Tin + oa * tstride, tbytes);
  for (int o = oa; o < ob; ++o) {
    auto next = [&] {
      if (o + 1 < ob) load_inputs(pre, pos, Tin + (o + 1) * tstride, tbytes);
    };
    const double f = occ[o] * inv_omega;
    fft_io<N0, +1, NB, XT, SRC_PRE, DST_FN, C, SH::V>(X, N0 + 1, NB, tw, preloaded(pre, next), [&](int, int, C v, int it, int q) {
      a[it][q] += f * (double(v.x) * double(v.x) + double(v.y) * double(v.y));
    });
    __syncthreads();
  }
  double* pb = part + (long long)g * tab.n0 * npl + p0;
  last_stage_positions<N0, NB, XT, SH::V>(NB, [&](int it, int q, int t, int e) {
    if (p0 + t < npl) pb[e * npl + t] = a[it][q];
  });
}

// rho (+)= sum over groups g = 0..ng-1 of part[g] (in order)
__global__ __launch_bounds__(NT) void dens_sum_kernel(const double* __restrict__ part, int ng, long long N,
                                                      double* __restrict__ rho, int accumulate) {
  const long long i = (long long)blockIdx.x * NT + threadIdx.x;
  if (i >= N) return;
  double s = accumulate ? rho[i] : 0.0;
  for (int g = 0; g < ng; ++g) s += part[g * N + i];
  rho[i] = s;
}

// ------------------------------------------------------------------ launchers

// Orbital groups per x-pass launch: groups of at most xg_max orbitals (sizes
// differing by at most one), fewer orbitals per group when the launch would
// otherwise have too few blocks to fill the chip (about 12 per CU).
static int x_groups(const ks_system* s, int nb) {
  const long long blocks = (long long)s->ntiles * nb;
  long long g = blocks / (256 * 12);
  g = g < 1 ? 1 : (g > s->xg_max ? s->xg_max : g);
  return (int)((nb + g - 1) / g);
}

// Launch shapes of the x-pencil blocks: a tile (pencils NB x threads XT)
// and the factorisation of the x-transform (plan variant V, fft_device.hpp).
// Shape 0 is xnb<N0> pencils x NT threads; shape 1 is 16 pencils x 192
// threads, for the largest grids only (smaller LDS buffers, more blocks
// resident per CU); shapes 2 and 3 are shapes 0 and 1 with the second
// factorisation of n0 (n0 = 96: 8 x 12 instead of 12 x 8).  The autotuner
// picks the shape per grid and precision.
template <int NB_, int XT_>
struct XShape {
  static constexpr int NB = NB_, XT = XT_, V = 0;
};
template <int NB_, int XT_>
struct XShapeAlt {
  static constexpr int NB = NB_, XT = XT_, V = 1;
};
template <int N0> constexpr bool has_shape1 = N0 == 96 || N0 == 120;
template <int N0> constexpr bool has_alt_plan = N0 == 96;

template <int N0, class F>
static void with_shape(const ks_system* s, F&& f) {
  if constexpr (has_alt_plan<N0>) {
    if (s->xshape == 2) {
      f(XShapeAlt<xnb<N0>::value, NT>{});
      return;
    }
    if (s->xshape == 3) {
      f(XShapeAlt<16, 192>{});
      return;
    }
  }
  if constexpr (has_shape1<N0>) {
    if (s->xshape == 1) {
      f(XShape<16, 192>{});
      return;
    }
  }
  f(XShape<xnb<N0>::value, NT>{});
}

bool x_shape_available(int n0, int shape) {
  if (shape == 0) return true;
  if (shape < 1 || shape > 3) return false;
  switch (n0) {
#define KS_CASE(v) case v: return (shape == 1 || shape == 3 ? has_shape1<v> : true) && (shape < 2 || has_alt_plan<v>);
    KS_SIZES(KS_CASE)
#undef KS_CASE
    default:
      return false;
  }
}

int x_shape_nb(int n0, int shape) { return shape == 1 || shape == 3 ? 16 : x_tile_nb(n0); }
int x_shape_threads(int shape) { return shape == 1 || shape == 3 ? 192 : NT; }

// Orbital groups of a density pass (ng) and where they write their partial
// densities, which dens_sum adds in order: groups of at least DENS_GROUP
// orbitals, at most `most` of them.  A launch that leaves more than half of the
// compute units' block slots empty that way (fewer than 512 blocks: small
// grids, few orbitals) takes more and smaller groups, up to that number of blocks
// and as far as U, which is written only after a density pass, holds them.  A
// block's orbitals and the sum over groups are two chains, so the shortest are
// groups of about sqrt(nb) / 1.5 orbitals: a density pass of 24^3 with its
// synthesis took, in 1, 2, 3, 5, 8, 12, 24 groups, 30, 22, 19, 17.7, 17.7, 17.6,
// 20.6 us (24 orbitals, FP64); of 12 x 8 x 8 in 8, 12, 20, 32, 64, 128 groups 29, 26,
// 23, 23, 30, 45 us (160 orbitals); one group per orbital took twice the time of
// groups of 8 there.
struct DensPlan {
  int ng;
  double* part;
};
static DensPlan dens_plan(const ks_system* s, int nb, int most) {
  const int by_size = std::max(1, std::min(most, (nb + DENS_GROUP - 1) / DENS_GROUP));
  const int by_fill = (512 + s->ntiles - 1) / s->ntiles;
  const int orbitals = std::max(1, (int)lround(sqrt((double)nb) / 1.5));
  const int by_chain = (nb + orbitals - 1) / orbitals;
  const size_t es = mixed(s) ? sizeof(float2) : sizeof(double2);
  const size_t fit = (size_t)s->cb * s->nplanes * es / ((size_t)s->n[0] * sizeof(double));
  const int ng = (int)std::min<size_t>(fit, std::min({by_chain, most, by_fill}));
  if (ng > by_size) return {ng, static_cast<double*>(s->U)};
  return {by_size, s->dens_part};
}

template <int N0, bool HB>
static void xproj_n(const ks_system* s, int nb, const void* T, void* partial, const double* occ, double* rho,
                    int accumulate, hipStream_t st) {
  const double scale = s->dV / sqrt(s->omega);
  const double inv_omega = 1.0 / s->omega;
  const bool dens = rho != nullptr;
  const DensPlan dp = dens ? dens_plan(s, nb, x_groups(s, nb)) : DensPlan{x_groups(s, nb), nullptr};
  with_shape<N0>(s, [&](auto sh) {
    using SH = decltype(sh);
    const dim3 grid(s->ntiles, dp.ng);
    if (!dens) {
      if (!mixed(s))
        xproj_kernel<N0, SH, double, HB, false><<<grid, SH::XT, 0, st>>>(
            (const double2*)T, nb, (double2*)partial, sphere_tab(s), proj_tab(s), s->d_tw0, scale, nullptr, nullptr,
            inv_omega);
      else
        xproj_kernel<N0, SH, float, HB, false><<<grid, SH::XT, 0, st>>>(
            (const float2*)T, nb, (float2*)partial, sphere_tab(s), proj_tab(s), s->d_tw0f, scale, nullptr, nullptr,
            inv_omega);
    } else if (!mixed(s)) {
      xproj_kernel<N0, SH, double, HB, true><<<grid, SH::XT, 0, st>>>(
          (const double2*)T, nb, (double2*)partial, sphere_tab(s), proj_tab(s), s->d_tw0, scale, occ, dp.part,
          inv_omega);
    } else {
      xproj_kernel<N0, SH, float, HB, true><<<grid, SH::XT, 0, st>>>(
          (const float2*)T, nb, (float2*)partial, sphere_tab(s), proj_tab(s), s->d_tw0f, scale, occ, dp.part,
          inv_omega);
    }
  });
  if (dens)
    dens_sum_kernel<<<(unsigned)((s->N + NT - 1) / NT), NT, 0, st>>>(dp.part, dp.ng, s->N, rho, accumulate);
}

bool launch_xproj(const ks_system* s, int nb, const void* T, void* partial, const double* occ, double* rho,
                  int accumulate, hipStream_t st) {
  switch (s->n[0]) {
#define KS_CASE(v) \
  case v: s->x_half ? xproj_n<v, true>(s, nb, T, partial, occ, rho, accumulate, st) \
                    : xproj_n<v, false>(s, nb, T, partial, occ, rho, accumulate, st); return true;
    KS_SIZES(KS_CASE)
#undef KS_CASE
    default:
      return false;
  }
}

// Whether the x-apply blocks sum the projections themselves: every slot of a
// tile then re-reads all partial sums of its atom (`values` in all: orbitals x
// nproj x the sum over slots of their atom's slot count), at the head of each
// orbital, against one launch of proj_reduce.  Measured per step of 4 H psi,
// launch against head, 2 to 128 orbitals with atoms at one per 3000, 9000 and
// 20000 points:
// - 64-pencil tiles (n0 <= 32): 5 to 9 us less up to 1152 blocks, 1 to 3 at 2048
//   (blocks: a tile of an orbital each);
// - 32-pencil tiles in FP64: 4 to 8 us less while the blocks are resident at
//   once, four per compute unit at 40, 48 and 64 points (64^3 / 8, 1024: 146.6 and
//   140.2 us) and three elsewhere (72^3 / 4, 648: 165 and 160), and still 1 to 5
//   at 40 and 48 points up to 1792 (48^3 / 24, 1728: 173 and 169).  Beyond, each
//   further round pays the head's latency: 60^3 / 8, 904: 168 and 184; 72^3 / 16,
//   2592: 388 and 400; 96^3 / 8, 2304: 400 and 405.  On spheres past the band it
//   is three per compute unit from 32 points on (32^3 / 64, 1024: 186 and 194);
// - 32-pencil tiles in complex64: slower at every size in the band, by 1 us for
//   a few orbitals (64^3 / 2, 256: 98 and 102) and by 5 to 40 beyond one round
//   (40^3 / 24, 1200: 129 and 142; 96^3 / 8, 2304: 276 and 321), so never.
// And up to 6 MB of reads: 32^3 / 262 in a batch, 7 MB: 35.8 -> 40.9 us for the
// kernel, without 4.8 us; 60^3 / 96, 14 MB: 72 -> 110 us.
bool xapply_sums(const ks_system* s, long long orbitals, long long values) {
  const int n0 = s->n[0];
  if (s->xshape != 0 || (n0 > 32 && mixed(s))) return false;
  long long blocks = 768;
  if (n0 <= 24 || (n0 == 32 && (mixed(s) || s->x_half))) blocks = 2048;
  else if (s->x_half && n0 <= 48) blocks = 1792;
  else if (s->x_half && n0 == 64) blocks = 1024;
  return s->ntiles * orbitals <= blocks &&
         values * (long long)(mixed(s) ? sizeof(float2) : sizeof(double2)) <= (6ll << 20);
}

// the kernels that exist with the sums: the first tile shape, complex64 up to 32 points
template <int N0, class SH, typename R>
constexpr bool has_sums = SH::XT == NT && SH::V == 0 && (N0 <= 32 || sizeof(R) == 8);

template <int N0, bool HB, bool SUMS>
static void xapply_n(const ks_system* s, int nb, const void* T, const double2* DP, const void* partial, void* U,
                     hipStream_t st) {
  // synthesis scale Omega^-1/2 and analysis scale Omega^1/2/N folded into V
  // (the KB coefficients carry the analysis scale from the projection sums)
  const double sc_v = 1.0 / (double)s->N, sc_p = sqrt(s->omega) / (double)s->N;
  const int ng = x_groups(s, nb);
  with_shape<N0>(s, [&](auto sh) {
    using SH = decltype(sh);
    const dim3 grid(s->ntiles, ng);
    if (!mixed(s))
      xapply_kernel<N0, SH, double, HB, SUMS && has_sums<N0, SH, double>><<<grid, SH::XT, 0, st>>>((const double2*)T, nb, (double2*)U, s->d_v, DP,
                                                                   (const double2*)partial, sc_p, sphere_tab(s),
                                                                   proj_tab(s), s->d_tw0, sc_v);
    else
      xapply_kernel<N0, SH, float, HB, SUMS && has_sums<N0, SH, float>><<<grid, SH::XT, 0, st>>>((const float2*)T, nb, (float2*)U, s->d_v, DP,
                                                                  (const float2*)partial, sc_p, sphere_tab(s),
                                                                  proj_tab(s), s->d_tw0f, sc_v);
  });
}

bool launch_xapply(const ks_system* s, int nb, const void* T, const double2* DP, const void* partial, void* U,
                   hipStream_t st) {
  switch (s->n[0]) {
#define KS_CASE(v)                                                                                         \
  case v:                                                                                                  \
    if (partial) s->x_half ? xapply_n<v, true, true>(s, nb, T, DP, partial, U, st)                         \
                           : xapply_n<v, false, true>(s, nb, T, DP, partial, U, st);                       \
    else s->x_half ? xapply_n<v, true, false>(s, nb, T, DP, partial, U, st)                                \
                   : xapply_n<v, false, false>(s, nb, T, DP, partial, U, st);                              \
    return true;
    KS_SIZES(KS_CASE)
#undef KS_CASE
    default:
      return false;
  }
}

// Batched launches: one x-pass launch over several systems of the grid (all
// of one tile shape, that of s).
template <int N0, bool HB>
static void x_batch_n(const ks_system* s, const BatchJob* jobs, const int4* rows, int nrows, bool apply, bool sums,
                      hipStream_t st) {
  const dim3 grid(s->ntiles, nrows);
  const double scale = s->dV / sqrt(s->omega);
  const double sc_v = 1.0 / (double)s->N, sc_p = sqrt(s->omega) / (double)s->N;
  with_shape<N0>(s, [&](auto sh) {
    using SH = decltype(sh);
    if (!apply) {
      if (!mixed(s))
        xproj_kernel<N0, SH, double, HB, false, true><<<grid, SH::XT, 0, st>>>(
            nullptr, 0, nullptr, sphere_tab(s), ProjTab{}, s->d_tw0, scale, nullptr, nullptr, 0.0, jobs, rows);
      else
        xproj_kernel<N0, SH, float, HB, false, true><<<grid, SH::XT, 0, st>>>(
            nullptr, 0, nullptr, sphere_tab(s), ProjTab{}, s->d_tw0f, scale, nullptr, nullptr, 0.0, jobs, rows);
    } else if (!mixed(s)) {
      auto* k = sums ? xapply_kernel<N0, SH, double, HB, has_sums<N0, SH, double>, true> : xapply_kernel<N0, SH, double, HB, false, true>;
      k<<<grid, SH::XT, 0, st>>>(nullptr, 0, nullptr, nullptr, nullptr, nullptr, sc_p, sphere_tab(s), ProjTab{},
                                 s->d_tw0, sc_v, jobs, rows);
    } else {
      auto* k = sums ? xapply_kernel<N0, SH, float, HB, has_sums<N0, SH, float>, true> : xapply_kernel<N0, SH, float, HB, false, true>;
      k<<<grid, SH::XT, 0, st>>>(nullptr, 0, nullptr, nullptr, nullptr, nullptr, sc_p, sphere_tab(s), ProjTab{},
                                 s->d_tw0f, sc_v, jobs, rows);
    }
  });
}

bool launch_x_batch(const ks_system* s, const BatchJob* jobs, const int4* rows, int nrows, bool apply, bool sums,
                    hipStream_t st) {
  switch (s->n[0]) {
#define KS_CASE(v) \
  case v: s->x_half ? x_batch_n<v, true>(s, jobs, rows, nrows, apply, sums, st) \
                    : x_batch_n<v, false>(s, jobs, rows, nrows, apply, sums, st); return true;
    KS_SIZES(KS_CASE)
#undef KS_CASE
    default:
      return false;
  }
}

int x_group_size(const ks_system* s, long long total_orbitals) {
  long long g = (long long)s->ntiles * total_orbitals / (256 * 12);
  return (int)(g < 1 ? 1 : (g > s->xg_max ? s->xg_max : g));
}

template <int N0, bool HB>
static void xdens_n(const ks_system* s, int nb, const void* T, const double* occ, const DensPlan& dp, hipStream_t st) {
  with_shape<N0>(s, [&](auto sh) {
    using SH = decltype(sh);
    const dim3 grid(s->ntiles, dp.ng);
    if (!mixed(s))
      xdens_kernel<N0, SH, double, HB><<<grid, SH::XT, 0, st>>>((const double2*)T, nb, occ, dp.part, sphere_tab(s),
                                                               s->d_tw0, 1.0 / s->omega);
    else
      xdens_kernel<N0, SH, float, HB><<<grid, SH::XT, 0, st>>>((const float2*)T, nb, occ, dp.part, sphere_tab(s),
                                                              s->d_tw0f, 1.0 / s->omega);
  });
}

bool launch_xdens(const ks_system* s, int nb, const void* T, const double* occ, double* rho, int accumulate,
                  hipStream_t st) {
  // at most about 12 blocks per CU
  const DensPlan dp = dens_plan(s, nb, (256 * 12 + s->ntiles - 1) / s->ntiles);
  switch (s->n[0]) {
#define KS_CASE(v) \
  case v: s->x_half ? xdens_n<v, true>(s, nb, T, occ, dp, st) : xdens_n<v, false>(s, nb, T, occ, dp, st); break;
    KS_SIZES(KS_CASE)
#undef KS_CASE
    default:
      return false;
  }
  dens_sum_kernel<<<(unsigned)((s->N + NT - 1) / NT), NT, 0, st>>>(dp.part, dp.ng, s->N, rho, accumulate);
  return true;
}

}  // namespace ks
