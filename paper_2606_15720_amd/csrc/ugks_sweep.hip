// Fused velocity sweep for tensor-product, mirror-symmetric velocity sets.
//
// A work item is one cell with all of its velocities (or, where cells are
// too few, with one block of them).  Each lane owns a mirror pair of velocities
// (u, -u): for every face of the cell exactly one of the two leaves the cell, so
// the lane evaluates one time-integrated flux from the cell's own reconstruction
// (outgoing) and one from the neighbour's reconstruction (incoming); a wave
// diverges only where its pairs differ in which member leaves.  The face and cell
// data are wave-uniform:
//   * the Maxwellians g0, g_cell and the wall Maxwellian factor over the
//     velocity axes and are staged in LDS once per work item, so
//     exp(-lambda |u - U|^2) is a product of three table entries;
//   * every equilibrium term of the interface distribution (Eqs.
//     interface_distribution, c123, c45 integrated over the step) is g0(u)
//     times a cubic polynomial c + l.u + u^T Q u + (kappa . u)|u|^2, evaluated
//     with the even/odd split P(-u) = E(u) - O(u);
//   * those polynomials and the least-squares stencils of the cell and of
//     each neighbour are read from the face and cell records through the
//     scalar cache.
// The conservative update needs, per cell, sum_j sigma_j S_j F_j / V with
// F_j = sum_k w_k psi_k H_jk (Eqs. macro_update, macro_flux); the sweep
// regroups that sum by velocity, sum_k w_k psi_k (sum_j sigma_j S_j H_jk / V),
// accumulates it per lane and reduces it once per work item, so there are no
// atomics and the result is deterministic.  The first stage (Eq. f_tilde) is
// applied in the same pass.  All loads of an iteration (the cell's stencil at
// u and -u, each neighbour's stencil at the incoming member) are issued
// before any arithmetic so their latency overlaps.  In 2-D the b equation
// (same transport and relaxation, its own equilibrium polynomials) runs as a
// second pass over the cell's velocities after h, or in one pass with it: in the
// batched forms, and for a single case where the registers hold both
// (kBothPasses).  The work-group that has
// swept a whole cell goes on with the rest of the cell's step (conservative
// update, second stage of Eq. f_final, heat flux, the next step's cell
// record); the new state goes to the second of two buffers, which the host
// swaps, so neighbours keep reading h^n.
#include <algorithm>
#include <type_traits>

#include "ugks_device.h"

namespace ugks {

using namespace dev;

namespace {

constexpr int SWF = 4;      // faces per cell on the fused path (triangles, quads, tets)
constexpr int SWT = 256;    // lanes per work-group of the blocked form
constexpr int64_t kLdsPerCu = 160 * 1024, kLdsGrain = 1280;  // bytes; LDS is given out in grains
constexpr int CELLT = 512;  // most lanes per work-group of the whole-cell form
constexpr int NAX = 64;     // nodes per velocity axis (max)

// A wave-uniform row of f in the global address space, kept opaque in
// scalar registers, so that every load from it is one scalar base plus a
// 32-bit per-lane byte offset (no reassociated 64-bit vector addresses).
typedef const __attribute__((address_space(1))) char grow_t;

template <typename T>
__device__ __forceinline__ grow_t* srow(const T* p) {
  grow_t* g = (grow_t*)p;
  __asm__("" : "+s"(g));
  return g;
}

// The same of a pointer that need not be in scalar registers yet.
template <typename T>
__device__ __forceinline__ grow_t* srow_any(const T* p) {
  const uint64_t a = (uint64_t)p;
  return srow((const char*)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(a >> 32)) << 32 |
                            (uint32_t)__builtin_amdgcn_readfirstlane((int)a)));
}

// Per-cell and per-face records are read-only during the sweep; read
// through the constant address space their wave-uniform loads are always
// scalar loads, also where the record pointers themselves come from memory
// (the batched form).
typedef const __attribute__((address_space(4))) int32_t crec_i_t;
template <typename X>
using crec_t = const __attribute__((address_space(4))) X;

// N wave-uniform record values in scalar loads of 64 bytes (and one of what
// remains).
template <typename C, int N>
struct wide_t {
  typedef C vec __attribute__((ext_vector_type(N)));
  typedef vec type __attribute__((aligned(sizeof(C))));
};
template <typename C, int N>
__device__ __forceinline__ void load_rec(crec_t<C>* p, C (&v)[N]) {
  constexpr int W = 64 / sizeof(C);
  typedef typename wide_t<C, W>::type whole_t;
#pragma unroll
  for (int i = 0; i + W <= N; i += W) {
    const typename wide_t<C, W>::vec x = *(crec_t<whole_t>*)(p + i);
#pragma unroll
    for (int j = 0; j < W; ++j) v[i + j] = x[j];
  }
  constexpr int R = N % W;
  if constexpr (R > 0) {
    typedef typename wide_t<C, R>::type rest_t;
    const typename wide_t<C, R>::vec x = *(crec_t<rest_t>*)(p + N - R);
#pragma unroll
    for (int j = 0; j < R; ++j) v[N - R + j] = x[j];
  }
}

template <typename T, typename C>
__device__ __forceinline__ C ldo(grow_t* row, uint32_t off) {
  return static_cast<C>(*(const __attribute__((address_space(1))) T*)(row + off));
}

// The same for stores.
typedef __attribute__((address_space(1))) char gout_t;
template <typename T>
__device__ __forceinline__ gout_t* sout(T* p) {
  gout_t* g = (gout_t*)p;
  __asm__("" : "+s"(g));
  return g;
}
template <typename T>
__device__ __forceinline__ void sto(gout_t* row, uint32_t off, T v) {
  *(__attribute__((address_space(1))) T*)(row + off) = v;
}
template <typename T>
__device__ __forceinline__ void sto_nt(gout_t* row, uint32_t off, T v) {
  __builtin_nontemporal_store(v, (__attribute__((address_space(1))) T*)(row + off));
}

// Even and odd parts of a polynomial P = c + l.u + u^T Q u + (kappa . u)|u|^2 (a
// sweep record's values from SR_P on) at u, with v2 = |u|^2:
//   E = c + u^T Q u,  O = l.u + (kappa . u) v2,  P(u) = E + O,  P(-u) = E - O.
template <int D, typename C, typename PT>
__device__ __forceinline__ void cubic_eo(PT P, const C* v, C v2, C& E, C& O) {
  if constexpr (D == 3) {
    const C x = v[0], y = v[1], z = v[2];
    E = P[0] + x * (P[4] * x + P[7] * y + P[8] * z) + y * (P[5] * y + P[9] * z) + P[6] * z * z;
    O = (P[1] * x + P[2] * y + P[3] * z) + (P[10] * x + P[11] * y + P[12] * z) * v2;
  } else {
    const C x = v[0], y = v[1];
    E = P[0] + x * (P[3] * x + P[5] * y) + P[4] * y * y;
    O = (P[1] * x + P[2] * y) + (P[6] * x + P[7] * y) * v2;
  }
}

// Venkatakrishnan's limiter factor (Sec. 2.1 reconstruction with the
// optional limiter) of a gradient g of a field with cell value vi and stencil
// range [vmin, vmax]: at each of four faces with offsets off[q * stride + d]
// from the centroid, d- = g.off, d+ = vmax - vi (d- > 0) or vmin - vi,
// psi = (d+^2 + eps^2 + 2 d- d+) / (d+^2 + 2 d-^2 + d- d+ + eps^2) (psi = 1
// where d- = 0); returns min(1, min_faces psi).  On each side d+ is the same for
// every face and min(1, psi) falls as |d-| grows (below 1 its derivative has
// the sign of (d+^2 + eps^2) d+ - 4 d- (d+^2 + d+ d- + eps^2) < 0, as there
// d+ < 2 d-), so the largest and the smallest d- decide, and two of four psi are
// evaluated (101,376 tets x 28^3 FP32 with local steps, 2 steps: 47.4 ms with
// four, 41.4 so; 10,368 x 24^3 FP64 3.50 and 2.68 per step).  The minimum is kept as a fraction and divided once.
template <int D, typename C, typename PT>
__device__ __forceinline__ C venkat_phi(C vi, C vmin, C vmax, const C* g, PT off, int stride, C eps2) {
  C dmax = C(0), dmin = C(0);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    C dm = C(0);
#pragma unroll
    for (int d = 0; d < D; ++d) dm += g[d] * off[q * stride + d];
    dmax = fmax(dmax, dm);
    dmin = fmin(dmin, dm);
  }
  C Nm = C(1), Dm = C(1);
  auto side = [&](C dp, C dm) {
    const C a = dp * dp + eps2, t = dm * dp;
    const C N = a + C(2) * t, Dn = a + t + C(2) * dm * dm;
    const bool lt = N * Dm < Nm * Dn;  // (0 / 0 does not limit)
    Nm = lt ? N : Nm;
    Dm = lt ? Dn : Dm;
  };
  side(vmax - vi, dmax);
  side(vmin - vi, dmin);
  return Nm / Dm;
}

// Shakhov polynomials H+/H and B+/B of a cell's equilibrium with heat flux qc
// (Eqs. H_plus, B_plus).
template <int D>
__device__ __forceinline__ void shakhov_polys(const double* P, const GasP& g, const double* qc,
                                              double* SH, double* SB) {
  using Cb = Cubic<D>;
#pragma unroll
  for (int x = 0; x < Cb::N; ++x) SH[x] = SB[x] = 0.0;
  const double lam = P[4];
  const double sh = 4.0 * (1.0 - g.Pr) * lam * lam / ((g.K + 5.0) * P[0]);
  const double U[3] = {P[1], P[2], P[3]};
  Cb::add_shakhov(SH, sh, U, qc, lam, 2.0 + D);
  Cb::add_shakhov(SB, sh, U, qc, lam, (double)D);
}

// Per-step record of a cell with primitives P and heat flux qc.
template <int D, typename T>
__device__ __forceinline__ void cell_record(const double* P, const GasP& g, double dt, const double* qc,
                                            int nr, T* __restrict__ C) {
  constexpr int N = Cubic<D>::N;
  double SH[N], SB[N];
  shakhov_polys<D>(P, g, qc, SH, SB);
  const double cc = dt / (2.0 * P[5]), kap = (g.K + 3.0 - D) / (2.0 * P[4]);
  write_srec<D>(C, cc, kap, SH);
  if (nr == 2) write_srec<D>(C + SREC, cc, kap, SB);
}

// prim and the cell record of W^n, q before a first step (a step leaves the
// next one's).
template <int D, typename T>
__device__ __forceinline__ void cell_prep_at(int64_t i, const GasP& g, const double* __restrict__ W,
                                             const double* __restrict__ q, double* __restrict__ prim,
                                             int nr, T* __restrict__ cs, int32_t* flag) {
  if (*flag) return;
  double* P = &prim[i * NPRIM];
  if (!prim_of<D>(&W[i * (D + 2)], g, P)) {
    atomicOr(flag, 1);
    return;
  }
  const double qc[3] = {q[i * 3], q[i * 3 + 1], q[i * 3 + 2]};
  cell_record<D>(P, g, dt_cell(g, i), qc, nr, &cs[i * nr * SREC]);
}

template <int D, typename T>
__global__ __launch_bounds__(128) void k_cell_prep(int64_t nc, GasP g, const double* __restrict__ W,
                            const double* __restrict__ q, double* __restrict__ prim, int nr,
                            T* __restrict__ cs, int32_t* flag) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < nc) cell_prep_at<D>(i, g, W, q, prim, nr, cs, flag);
}

// LDS of one work item.  A table holds, for node n, the entry at n and the
// entry at its mirror na-1-n side by side: one read serves u and -u.
// During the sweep: the Maxwellian axis tables of the cell's four faces and of
// the cell, and the velocity nodes; afterwards: the new state's tables and
// Shakhov polynomials (FP64 in either form).
template <int D, typename C, int NF = SWF>
struct SweepTabs {
  alignas(16) C tab[NF + 1][D][NAX][2];  // the faces, then the cell
  C ax[NAX][2];
};
template <int D>
struct CellTabs {
  alignas(16) double tab[D][NAX][2];
  double ax[NAX][2];
  double poly[2][SREC];
  double par[8];  // lambda, U (3), the table's factor, 1/(1 + A), valid
};
template <int D, typename C, int NF = SWF>
struct SweepLds {
  union {
    SweepTabs<D, C, NF> s;
    CellTabs<D> c;
  };
  double red[5 * 16];
};

// Pair entry at a byte offset into one table row.
template <typename C>
__device__ __forceinline__ void tab_pair(const C (*row)[2], unsigned off, C& at_u, C& at_mu) {
  typedef C pair_t __attribute__((ext_vector_type(2)));
  const pair_t v = *(const pair_t*)((const char*)row + off);
  at_u = v.x;
  at_mu = v.y;
}

// Byte offset of a point's node on axis d in a table of C pairs (packed
// indices: 16 * node in 10 bits per axis).
template <typename C>
__device__ __forceinline__ unsigned node_off(int pk, int d) {
  return sizeof(C) == 8 ? ((unsigned)pk >> (10 * d)) & 1023u : ((unsigned)pk >> (10 * d + 1)) & 511u;
}
__device__ __forceinline__ int node_of(int pk, int d) { return (pk >> (10 * d + 4)) & 63; }

// One 64-lane sum, valid in lane 63: shifts within rows of 16, then the rows
// joined by broadcasts (no LDS round trips).
// (lanes without a source add 0; what the broadcasts add to other rows than the
// last does not reach lane 63)
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
  return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_total(double v) {
  v = dpp_add<0x111>(v);  // row_shr:1, 2, 4, 8
  v = dpp_add<0x112>(v);
  v = dpp_add<0x114>(v);
  v = dpp_add<0x118>(v);
  v = dpp_add<0x142>(v);  // row_bcast:15: each row's total to the next
  return dpp_add<0x143>(v);  // row_bcast:31: the first two rows' to the last two
}

// Work-group totals of N values, in every lane of the first wave: each wave's
// sum, then the waves in order.  A barrier for the whole work-group.
template <int N>
__device__ __forceinline__ void block_total(double (&v)[N], double* lds) {
#pragma unroll
  for (int n = 0; n < N; ++n) v[n] = wave_total(v[n]);
  const int wv = threadIdx.x / WAVE, nw = blockDim.x / WAVE;
  if (threadIdx.x % WAVE == WAVE - 1)
#pragma unroll
    for (int n = 0; n < N; ++n) lds[n * 16 + wv] = v[n];
  __syncthreads();
  if (threadIdx.x < WAVE) {
#pragma unroll
    for (int n = 0; n < N; ++n) {
      double t = lds[n * 16];
      for (int w = 1; w < nw; ++w) t += lds[n * 16 + w];
      v[n] = t;
    }
  }
}

// A wave-uniform double in scalar registers.
__device__ __forceinline__ double uniform(double v) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                          __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

// What a sweep reads besides f: every pointer wave-uniform.
template <typename C>
struct SweepIn {
  const int32_t* crec_i;
  const C* crec_d;
  const C* crec_l;
  const int32_t* vidx;
  const double* w;
  const C* cs;            // [nc*nr*SREC]
  const C* srec;          // [nf*nr*SREC]
  const double* frec;
  const double* prim;
  double dt;
  int64_t nvp;
  unsigned half;  // slots of the first members; the mirror of slot k is slot half + k
  unsigned full;  // sparse sets: slots (a multiple of 64) whose mirror may be a point; pads follow
  unsigned keep;  // whole-cell form: pairs (a multiple of 64) whose first stage stays in LDS
  int na;
  const double* axis;
};

// The Maxwellian axis tables of the cell's four faces (the interface g0, or
// on a wall the re-emitted Maxwellian scaled by rho_w dt) and of the cell,
// scale exp(-lambda (a_n - U_d)^2) with density and norm folded into the
// first axis, so that g(u) at a tensor point is a product of D entries.
// A half wave (a wave where an axis has more than 32 nodes) takes one
// (entity, axis) row at a time.  Computing them here takes about one exp per
// lane; as arrays written once per step and read by each cell they cost a
// launch and, with their FP32 copies, 1-3 % of the step.
template <int D, typename C, int NF = SWF>
__device__ __forceinline__ void sweep_tables(const SweepIn<C>& in, int64_t ic, SweepTabs<D, C, NF>& L) {
  constexpr unsigned FACE = NF == SWF ? CI_FACE : WI_FACE, KIND = NF == SWF ? CI_KIND : WI_KIND;
  const unsigned nthr = blockDim.x, na = (unsigned)in.na;
  const bool half = na <= 32;
  const unsigned n = half ? threadIdx.x & 31u : threadIdx.x & 63u;
  const unsigned r0 = half ? threadIdx.x >> 5 : threadIdx.x >> 6, rs = half ? nthr >> 5 : nthr >> 6;
  if (n < na) {
    const double a = in.axis[n];
    for (unsigned row = r0; row < (NF + 1u) * D; row += rs) {
      const unsigned e = row / D, d = row % D;
      double lam, U, scale = 1.0;
      if (e < NF) {
        const int32_t* ci = in.crec_i + ic * CRI;
        const double* R = in.frec + (uint64_t)(uint32_t)ci[FACE + e] * FREC;
        lam = R[FR_LAM];
        U = R[FR_U + d];
        if (d == 0) scale = ci[KIND + e] == UGKS_BC_WALL ? R[FR_C0] * R[FR_RHOW] * in.dt : R[FR_C0];
      } else {
        lam = in.prim[ic * NPRIM + 4];
        U = in.prim[ic * NPRIM + 1 + d];
        if (d == 0) scale = in.prim[ic * NPRIM] * maxw_norm<D>(lam);
      }
      const C v = (C)(scale * exp(-lam * (a - U) * (a - U)));
      L.tab[e][d][n][0] = v;
      L.tab[e][d][na - 1 - n][1] = v;
    }
    if (r0 == 0) L.ax[n][0] = (C)a;
  }
}

// A pair's share of the cell's moments of net outflow (acc0 at u, acc1 at -u,
// weights w0, w1) of distribution X (0: h, 1: b).
template <int D, typename C, int X>
__device__ __forceinline__ void add_moments(double w0, double w1, C acc0, C acc1, const C* vv, C v2,
                                            double (&mw)[D + 2]) {
  const double a0 = w0 * (double)acc0, a1 = w1 * (double)acc1;
  if (X == 0) {
    mw[0] += a0 + a1;
#pragma unroll
    for (int d = 0; d < D; ++d) mw[1 + d] += (double)vv[d] * (a0 - a1);
    mw[D + 1] += 0.5 * (double)v2 * (a0 + a1);
  } else {
    mw[D + 1] += 0.5 * (a0 + a1);
  }
}

// First stage (Eq. f_tilde) of a pair of distribution X: c0, c1 the cell's
// Maxwellian at u and -u, cc its record.
template <int D, typename C, int X, typename PT>
__device__ __forceinline__ void first_stage(PT cc, const C* vv, C v2, C c0, C c1, C f0, C f1, C acc0, C acc1,
                                            C& t0, C& t1) {
  C m0 = c0, m1 = c1;
  if (X == 1) {  // the b equilibrium carries the internal-energy factor
    const C kc = cc[1];
    m0 *= kc;
    m1 *= kc;
  }
  C E, O;
  cubic_eo<D>(cc + X * SREC + SR_P, vv, v2, E, O);
  E += C(1);
  const C ccoll = cc[0];
  t0 = f0 - acc0 + ccoll * (m0 * (E + O) - f0);
  t1 = f1 - acc1 + ccoll * (m1 * (E - O) - f1);
}

// One pass over the mirror pairs [kbeg, kend) of cell ic (multiples of 64
// except the lanes' stride) for NR reduced distributions, X0 the first:
// X = 0 is h (mass, momentum and its share of the energy), X = 1 is b (the
// rest of the energy).  The b equation has the same transport and relaxation
// as h with its own equilibrium polynomials.  Adds the lane's moments
// sum_k w_k psi_k (net outflow of the cell at u_k) to mw.
//
// The sign of u.n, which says which member leaves through a face, is a branch
// and not a select: a wave's 64 pairs are a compact block of the velocity
// lattice (4 x 4 x 4 or 8 x 8), so at most faces all lanes agree and one side
// is skipped.  With one table read for both members that leaves about 380 VALU
// instructions per pair of the 480 that selects took (3-D FP64).  Of 8.9 ms on
// 48,000 tets x 24^3, rows beyond the cell's own cost 1.7 (L2 misses), the
// first stage's stores 0.9 and the rest of the step 1.7; the loop alone is
// at 65 % of its VALU time.
//
// ONE: only the first members, for pairs whose second is a pad (points of a
// sparse set without a mirror): each face then has either its outgoing or its
// incoming side to do.  10,368 tets x 17,408 velocities, 3,456 of them without
// a mirror: 2.59 ms with whole pairs throughout, 2.30 so.
template <int D, typename T, typename C, int NR, int X0, bool LIM, bool HB, bool ONE = false>
__device__ __forceinline__ void sweep_pass(const SweepIn<C>& in, const T* __restrict__ h,
                                           const T* __restrict__ b, T* __restrict__ ht,
                                           T* __restrict__ bt, int64_t ic, unsigned kbeg, unsigned kend,
                                           const SweepTabs<D, C>& L, T* stage, double (&mw)[D + 2]) {
  crec_i_t* ci0 = (crec_i_t*)(in.crec_i + ic * CRI);
  crec_t<C>* cd0 = (crec_t<C>*)(in.crec_d + ic * CRD);
  constexpr int RS = (HB ? 2 : 1) * SREC;  // a face's or cell's records
  crec_t<C>* cc0 = (crec_t<C>*)(in.cs + ic * RS);
  crec_t<C>* frc = (crec_t<C>*)in.srec;
  crec_t<C>* cl0 = LIM ? (crec_t<C>*)(in.crec_l + ic * CRL) : nullptr;
  const unsigned nthr = blockDim.x;  // lanes of the work-group, one mirror pair each
  // Row r of h (or b) starts r * rowb bytes in.  Row indices are 32-bit and
  // non-negative, and a row is under 4 GiB, so the offset is one 32x32->64
  // scalar multiply.
  const uint32_t rowb = (uint32_t)in.nvp * (uint32_t)sizeof(T), halfb = in.half * (uint32_t)sizeof(T);
  auto row_of = [rowb](const T* base, int32_t r) {
    return srow((const char*)base + (uint64_t)(uint32_t)r * rowb);
  };
  const T* src[NR];
  gout_t* dst[NR];
  grow_t *own[NR], *wt = srow(in.w), *ix = srow(in.vidx);
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    src[r] = X0 + r ? b : h;
    dst[r] = sout((X0 + r ? bt : ht) + ic * in.nvp);
    own[r] = srow(src[r] + ic * in.nvp);
  }
  // the packed axis indices of the next pair are loaded one iteration ahead
  // (the array is padded for the read past the end)
  unsigned kp = kbeg + threadIdx.x;
  int pk_next = ldo<int32_t, int>(ix, kp * 4u);
  for (; kp < kend; kp += nthr) {
    // FP32: the wave takes a higher issue priority while it issues the
    // iteration's gathers, so that they start early (measured 2-6 % faster in
    // FP32, slower in FP64)
    if constexpr (sizeof(C) == 4) __builtin_amdgcn_s_setprio(1);
    // The cell and face records are loop invariant but too large to keep in
    // scalar registers for the whole loop: an opaque uniform zero added to
    // their addresses makes them scalar re-loads (scalar cache) each
    // iteration instead of hoisted, spilled registers.
    int z;
    __asm__ volatile("s_mov_b32 %0, 0" : "=s"(z));
    crec_i_t* ci = ci0 + z;
    crec_t<C>* cd = cd0 + z;
    crec_t<C>* cc = cc0 + z;
    const int pk = pk_next;
    pk_next = ldo<int32_t, int>(ix, (kp + nthr) * 4u);
    unsigned at[D];
    C vv[3] = {C(0), C(0), C(0)};
#pragma unroll
    for (int d = 0; d < D; ++d) {
      at[d] = node_off<C>(pk, d);
      vv[d] = *(const C*)((const char*)L.ax + at[d]);
    }
    int32_t rows[16];
    C nrm[12];
    load_rec<int32_t, 16>(ci + CI_OWN, rows);
    load_rec<C, 12>(cd + CD_N, nrm);
    // orientation of u against every outward normal
    C sp[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      C s = C(0);
#pragma unroll
      for (int d = 0; d < D; ++d) s += vv[d] * nrm[3 * p + d];
      sp[p] = s;
    }
    // ---- the cell's own stencil at u and -u (4 rows, padded) ----
    const uint32_t o0 = kp * (uint32_t)sizeof(T), o1 = o0 + halfb;
    C f0[NR], f1[NR], os0[NR][4], os1[NR][4];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      f0[r] = ldo<T, C>(own[r], o0);
      f1[r] = ONE ? C(0) : ldo<T, C>(own[r], o1);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        grow_t* rs = row_of(src[r], rows[CI_OWN + s]);
        os0[r][s] = ldo<T, C>(rs, o0);
        os1[r][s] = ONE ? C(0) : ldo<T, C>(rs, o1);
      }
    }
    // ---- every neighbour's stencil at the incoming member ----
    // Slot p of the own stencil is the row across face p, and slot 0 of
    // neighbour p's stencil is this cell: both are already in registers.
    C ns[NR][4][3] = {};
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      uint32_t oin = sp[p] > C(0) ? o1 : o0;  // u.n > 0: the incoming member is -u
      __asm__("" : "+v"(oin));  // keep the select on the offset, not on 64-bit addresses
      if (ONE && sp[p] > C(0)) continue;
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int r = 0; r < NR; ++r) ns[r][p][q] = ldo<T, C>(row_of(src[r], rows[CI_RING + 3 * p + q]), oin);
    }
    if constexpr (sizeof(C) == 4) __builtin_amdgcn_s_setprio(0);
    // ---- arithmetic ----
    C g0[NR][D], g1[NR][D], ug0[NR], ug1[NR], acc0[NR], acc1[NR];
    crec_t<C>* cl = LIM ? cl0 + z : nullptr;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
#pragma unroll
      for (int d = 0; d < D; ++d) g0[r][d] = g1[r][d] = C(0);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const C d0 = os0[r][s] - f0[r], d1 = os1[r][s] - f1[r];
#pragma unroll
        for (int d = 0; d < D; ++d) {
          const C G = cd[CD_G + d * 4 + s];
          g0[r][d] += G * d0;
          g1[r][d] += G * d1;
        }
      }
      if constexpr (LIM) {
        // the cell's own gradients at u and -u, limited (a wall slot's
        // zero row stands for the cell's own value in the bounds)
        C lo0 = f0[r], hi0 = f0[r], lo1 = f1[r], hi1 = f1[r];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const C wm = cl[1 + s];
          const C v0 = wm * f0[r] + os0[r][s], v1 = wm * f1[r] + os1[r][s];
          lo0 = fmin(lo0, v0);
          hi0 = fmax(hi0, v0);
          lo1 = fmin(lo1, v1);
          hi1 = fmax(hi1, v1);
        }
        const C e2 = cl[0];
        const C p0 = venkat_phi<D>(f0[r], lo0, hi0, g0[r], cd + CD_F0, CD_FS, e2);
        const C p1 = venkat_phi<D>(f1[r], lo1, hi1, g1[r], cd + CD_F0, CD_FS, e2);
#pragma unroll
        for (int d = 0; d < D; ++d) {
          g0[r][d] *= p0;
          g1[r][d] *= p1;
        }
      }
      ug0[r] = ug1[r] = acc0[r] = acc1[r] = C(0);
#pragma unroll
      for (int d = 0; d < D; ++d) {
        ug0[r] += vv[d] * g0[r][d];
        ug1[r] -= vv[d] * g1[r][d];
      }
    }
    C v2 = C(0);
#pragma unroll
    for (int d = 0; d < D; ++d) v2 += vv[d] * vv[d];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      // the face's geometry: in wide loads (FP32, and the pass of h and b), or,
      // where their 40 registers would spill others, value by value (FP64:
      // 7.75 against 7.89 ms on 48,000 x 24^3; FP32 x 28^3: 7.25 against 7.11)
      constexpr bool WIDE = sizeof(C) == 4 || NR == 2;
      crec_t<C>* fdp = cd + CD_F0 + CD_FS * p;
      C R[NR][SREC], fdw[CD_FS];
#pragma unroll
      for (int r = 0; r < NR; ++r)
        load_rec<C, SREC>(frc + (uint64_t)(uint32_t)ci[CI_FACE + p] * RS + (X0 + r) * SREC, R[r]);
      if constexpr (WIDE) load_rec<C, CD_FS>(fdp, fdw);
      auto fd = [&](int i) -> C {
        if constexpr (WIDE) return fdw[i];
        else return fdp[i];
      };
      const C G1 = R[0][0], G2 = R[0][1];
      const C eqm = fd(18);  // 0 on a wall: no equilibrium term going out
      // S/V |u.n|, in FP32 as two factors of every flux: their product rounded
      // beforehand is an error that each step repeats (state after 10 steps against
      // the FP64 form's: tets 0.7 % further off so, limited cylinder flow 4 %)
      const C as = fabs(sp[p]), sv = sizeof(C) == 4 ? fd(19) : C(1);
      const C sas = sizeof(C) == 4 ? as : fd(19) * as;
      // g0 (or the scaled wall Maxwellian) at u and -u from the axis tables
      C e0, e1;
      tab_pair(L.tab[p][0], at[0], e0, e1);
#pragma unroll
      for (int d = 1; d < D; ++d) {
        C a0, a1;
        tab_pair(L.tab[p][d], at[d], a0, a1);
        e0 *= a0;
        e1 *= a1;
      }
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        // times the equilibrium polynomial (constant on a wall)
        C E, O;
        cubic_eo<D>(R[r] + SR_P, vv, v2, E, O);
        const C q0 = e0 * (E + O), q1 = e1 * (E - O);
        // the neighbour's gradient from its value fj and this cell's value fi
        // (all zero rows on a wall)
        auto slope = [&](C fj, C fi, C* gj) {
#pragma unroll
          for (int d = 0; d < D; ++d) gj[d] = fd(6 + d * 4) * (fi - fj);
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            const C df = ns[r][p][q] - fj;
#pragma unroll
            for (int d = 0; d < D; ++d) gj[d] += fd(7 + d * 4 + q) * df;
          }
        };
        C gl[D];
        if constexpr (LIM) {
          // limited with the neighbour's own stencil bounds and face offsets
          const bool pos = sp[p] > C(0);
          const C fj = pos ? os1[r][p] : os0[r][p], fi = pos ? f1[r] : f0[r];
          slope(fj, fi, gl);
          crec_t<C>* Fr = cl + CRL_F0 + CRL_FS * p;
          C lo = fj, hi = fj;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const C vr = Fr[1 + q] * fj + (q ? ns[r][p][q - 1] : fi);
            lo = fmin(lo, vr);
            hi = fmax(hi, vr);
          }
          const C pj = venkat_phi<D>(fj, lo, hi, gl, Fr + 5, 3, Fr[0]);
#pragma unroll
          for (int d = 0; d < D; ++d) gl[d] *= pj;
        }
        // Fluxes at u and at -u along this cell's outward normal, times S/V:
        // the outgoing member's from the cell's own reconstruction (fo, go,
        // ugo), the incoming one's from the neighbour's (fj; fi is this cell's
        // value in its stencil; su u the incoming velocity).
        auto out = [&](C fo, const C* go, C ugo, C eqo, C& acco) {
          C ff = fo;
#pragma unroll
          for (int d = 0; d < D; ++d) ff += fd(d) * go[d];
          acco += sv * (sas * (G1 * ff + G2 * ugo + eqm * eqo));
        };
        auto into = [&](C fj, C fi, C su, C eqi, C& acci) {
          C gj[D];
          if constexpr (LIM) {
#pragma unroll
            for (int d = 0; d < D; ++d) gj[d] = gl[d];
          } else {
            slope(fj, fi, gj);
          }
          C ffj = fj, ugj = C(0);
#pragma unroll
          for (int d = 0; d < D; ++d) {
            ffj += fd(3 + d) * gj[d];
            ugj += vv[d] * gj[d];
          }
          acci -= sv * (sas * (G1 * ffj + G2 * (su * ugj) + eqi));
        };
        if (sp[p] > C(0)) {
          out(f0[r], g0[r], ug0[r], q0, acc0[r]);
          if constexpr (!ONE) into(os1[r][p], f1[r], C(-1), q1, acc1[r]);
        } else {
          if constexpr (!ONE) out(f1[r], g1[r], ug1[r], q1, acc1[r]);
          into(os0[r][p], f0[r], C(1), q0, acc0[r]);
        }
      }
    }
    // moments of the net outflow
    const double w0 = ldo<double, double>(wt, kp * 8u);
    const double w1 = ONE ? 0.0 : ldo<double, double>(wt, (kp + in.half) * 8u);
    add_moments<D, C, X0>(w0, w1, acc0[0], acc1[0], vv, v2, mw);
    if constexpr (NR == 2) add_moments<D, C, 1>(w0, w1, acc0[1], acc1[1], vv, v2, mw);
    // first stage with the cell's BGK-Shakhov equilibrium at u and -u
    C c0, c1;
    tab_pair(L.tab[4][0], at[0], c0, c1);
#pragma unroll
    for (int d = 1; d < D; ++d) {
      C a0, a1;
      tab_pair(L.tab[4][d], at[d], a0, a1);
      c0 *= a0;
      c1 *= a1;
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      C t0, t1;
      if (X0 + r == 0) first_stage<D, C, 0>(cc, vv, v2, c0, c1, f0[r], f1[r], acc0[r], acc1[r], t0, t1);
      else first_stage<D, C, 1>(cc, vv, v2, c0, c1, f0[r], f1[r], acc0[r], acc1[r], t0, t1);
      if (kp < in.keep) {
        stage[2 * (X0 + r) * in.keep + kp] = (T)t0;
        if constexpr (!ONE) stage[(2 * (X0 + r) + 1) * in.keep + kp] = (T)t1;
      } else {
        sto<T>(dst[r], o0, (T)t0);
        if constexpr (!ONE) sto<T>(dst[r], o1, (T)t1);
      }
    }
  }
}

// One work item of the fused sweep: the mirror pairs [kbeg, kend) of cell ic.
// Leaves the first stage in ht, bt and each lane's moment sums in mw.  h and b
// run as two passes (each pass's records and row addresses then fit the scalar
// registers, where h and b together spill them), or with BOTH in one (kBothPasses,
// and the batched forms, whose small cases run only a few iterations, whose
// dependent-load latency two passes would pay twice).  HB: b is carried.
// SPARSE: the pairs from in.full on have a pad for their second member.
template <int D, typename T, typename C, bool BOTH, bool LIM, bool HB, bool SPARSE = false>
__device__ __forceinline__ void sweep_item(const SweepIn<C>& in, const T* __restrict__ h,
                                           const T* __restrict__ b, T* __restrict__ ht,
                                           T* __restrict__ bt, int64_t ic, unsigned kbeg, unsigned kend,
                                           SweepTabs<D, C>& L, T* stage, double (&mw)[D + 2]) {
  sweep_tables<D, C>(in, ic, L);
  __syncthreads();
#pragma unroll
  for (int x = 0; x < D + 2; ++x) mw[x] = 0.0;
  if constexpr (SPARSE) {
    sweep_pass<D, T, C, 1, 0, LIM, HB>(in, h, b, ht, bt, ic, kbeg, in.full, L, stage, mw);
    sweep_pass<D, T, C, 1, 0, LIM, HB, true>(in, h, b, ht, bt, ic, in.full, kend, L, stage, mw);
    if constexpr (HB) {
      sweep_pass<D, T, C, 1, 1, LIM, HB>(in, h, b, ht, bt, ic, kbeg, in.full, L, stage, mw);
      sweep_pass<D, T, C, 1, 1, LIM, HB, true>(in, h, b, ht, bt, ic, in.full, kend, L, stage, mw);
    }
  } else if constexpr (HB && BOTH) {
    sweep_pass<D, T, C, 2, 0, LIM, HB>(in, h, b, ht, bt, ic, kbeg, kend, L, stage, mw);
  } else {
    sweep_pass<D, T, C, 1, 0, LIM, HB>(in, h, b, ht, bt, ic, kbeg, kend, L, stage, mw);
    if constexpr (HB) sweep_pass<D, T, C, 1, 1, LIM, HB>(in, h, b, ht, bt, ic, kbeg, kend, L, stage, mw);
  }
}

// The rest of a cell's step: the conservative update W^{n+1} = W^n - sum (tot,
// in the first wave), the second stage (Eq. f_final) with the equilibrium of
// W^{n+1} and q^n (reading R17) in place on the first stage's row, the heat
// flux of the result, and the next step's cell record.  Where the work-group
// has swept the cell, the first stage comes from LDS and from the row it wrote: a
// lane takes the pairs it swept, but for the single points of a sparse set, which
// are swept from `full` on and finished from 0 on, so by other lanes and waves.
// The barriers of block_total and of this function, between the sweep's stores and
// the loads here, make that right.  What is done once per cell is done by the first wave: by
// all eight it was a tenth of the kernel's VALU instructions.
template <int D, typename T, typename C, bool HB, bool SPARSE = false>
__device__ __forceinline__ void finish_cell(const GasP& g, const int32_t* __restrict__ vidx,
                                            const double* __restrict__ w, const CellOut& o, T* ht, T* bt,
                                            int64_t ic, int64_t nvp, unsigned half, int na,
                                            const double* __restrict__ axis, const T* stage, unsigned keep,
                                            double (&tot)[D + 2], CellTabs<D>& L, double* red,
                                            unsigned full = 0u) {
  constexpr int NM = D + 2, N = Cubic<D>::N, NP = Cubic<D>::C0 + D;
  double P[NPRIM], dt = 0.0;
  if (threadIdx.x < WAVE) {
    double Wn[NM];
    const double* Wi = o.W + ic * NM;
#pragma unroll
    for (int x = 0; x < NM; ++x) Wn[x] = Wi[x] - tot[x];
    const bool ok = prim_of<D>(Wn, g, P);
    dt = dt_cell(g, ic);
    if (threadIdx.x == 0) {
      const double lam = P[4], A = dt / (2.0 * P[5]), inv = 1.0 / (1.0 + A);
      const double kc = (g.K + 3.0 - D) / (2.0 * lam);
      const double qc[3] = {o.q[ic * 3], o.q[ic * 3 + 1], o.q[ic * 3 + 2]};
      // f^{n+1} = (f~ + A g (1 + P)) / (1 + A): the factor A / (1 + A) goes into
      // the first axis's table, the 1 into the polynomial's constant
      double SH[N], SB[N];
      shakhov_polys<D>(P, g, qc, SH, SB);
      SH[0] += 1.0;
      SB[0] += 1.0;
      write_srec<D>(L.poly[0], 0.0, 0.0, SH);
      if (HB) {
#pragma unroll
        for (int x = 0; x < N; ++x) SB[x] *= kc;
        write_srec<D>(L.poly[1], 0.0, 0.0, SB);
      }
      L.par[0] = lam;
      L.par[1] = P[1];
      L.par[2] = P[2];
      L.par[3] = P[3];
      L.par[4] = P[0] * maxw_norm<D>(lam) * A * inv;
      L.par[5] = inv;
      L.par[6] = ok ? 1.0 : 0.0;
      // (flag[2]: the other work-groups of this launch go on, on flag[0])
      if (!ok) atomicOr(&o.flag[2], 1);
      const double V = o.vol[ic], dr = Wn[0] - Wi[0];
      o.cellred[ic * 3 + 0] = V * dr * dr;
      o.cellred[ic * 3 + 1] = V;
      o.cellred[ic * 3 + 2] = V * Wi[0] * Wi[0];
#pragma unroll
      for (int x = 0; x < NM; ++x) o.Wn[ic * NM + x] = Wn[x];
    }
  }
  __syncthreads();
  if (L.par[6] == 0.0) return;  // the same in every lane
  const double lam = uniform(L.par[0]), inv = uniform(L.par[5]);
  const double U[3] = {uniform(L.par[1]), uniform(L.par[2]), uniform(L.par[3])};
  for (int t = threadIdx.x; t < D * NAX; t += blockDim.x) {
    const int d = t / NAX, n = t % NAX;
    if (n < na) {
      const double a = axis[n], Ud = d == 0 ? U[0] : d == 1 ? U[1] : U[2];
      const double v = (d == 0 ? L.par[4] : 1.0) * exp(-lam * (a - Ud) * (a - Ud));
      L.tab[d][n][0] = v;
      L.tab[d][na - 1 - n][1] = v;
      if (d == 0) L.ax[n][0] = a;
    }
  }
  double sh[NP], sb[NP];
#pragma unroll
  for (int x = 0; x < NP; ++x) {
    sh[x] = uniform(L.poly[0][SR_P + x]);
    sb[x] = HB ? uniform(L.poly[1][SR_P + x]) : 0.0;
  }
  __syncthreads();
  double acc[3] = {0.0, 0.0, 0.0};
  grow_t *hr = srow(ht + ic * nvp), *br = HB ? srow(bt + ic * nvp) : nullptr;
  grow_t *wt = srow(w), *ix = srow(vidx);
  gout_t *ho = sout(ht + ic * nvp), *bo = HB ? sout(bt + ic * nvp) : nullptr;
  const unsigned nthr = blockDim.x;
  // a few pairs per lane per pass, their loads issued together: as many as
  // the sweep's registers hold
  constexpr unsigned UN = sizeof(T) == 8 ? (HB ? 2 : 4) : (HB ? 1 : 2);
  for (unsigned kp = threadIdx.x; kp < half; kp += UN * nthr) {
    int pk[UN];
    T h0[UN], h1[UN], b0[UN], b1[UN];
    double w0[UN], w1[UN];
#pragma unroll
    for (unsigned u = 0; u < UN; ++u) {
      const unsigned k = kp + u * nthr;
      if (k < half) {  // whole waves: half is a multiple of 64
        const uint32_t o0 = k * (uint32_t)sizeof(T), o1 = o0 + half * (uint32_t)sizeof(T);
        const bool two = !SPARSE || k < full;  // not a pad
        h1[u] = b1[u] = T(0);
        w1[u] = 0.0;
        if (k < keep) {
          h0[u] = stage[k];
          if (two) h1[u] = stage[keep + k];
          b0[u] = HB ? stage[2 * keep + k] : T(0);
          if (two) b1[u] = HB ? stage[3 * keep + k] : T(0);
        } else {
          h0[u] = ldo<T, T>(hr, o0);
          if (two) h1[u] = ldo<T, T>(hr, o1);
          b0[u] = HB ? ldo<T, T>(br, o0) : T(0);
          if (two) b1[u] = HB ? ldo<T, T>(br, o1) : T(0);
        }
        pk[u] = ldo<int32_t, int>(ix, k * 4u);
        w0[u] = ldo<double, double>(wt, k * 8u);
        if (two) w1[u] = ldo<double, double>(wt, (k + half) * 8u);
      }
    }
#pragma unroll
    for (unsigned u = 0; u < UN; ++u) {
      const unsigned k = kp + u * nthr;
      if (k < half) {
        const uint32_t o0 = k * (uint32_t)sizeof(T), o1 = o0 + half * (uint32_t)sizeof(T);
        double vv[3] = {0, 0, 0}, c0 = 1.0, c1 = 1.0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
          const unsigned at = node_off<double>(pk[u], d);
          double a0, a1;
          vv[d] = *(const double*)((const char*)L.ax + at);
          tab_pair(L.tab[d], at, a0, a1);
          c0 *= a0;
          c1 *= a1;
        }
        const double v2 = vv[0] * vv[0] + vv[1] * vv[1] + vv[2] * vv[2];
        double E, O;
        cubic_eo<D>(sh, vv, v2, E, O);
        const double n0 = (double)h0[u] * inv + c0 * (E + O);
        const double n1 = (double)h1[u] * inv + c1 * (E - O);
        sto_nt<T>(ho, o0, (T)n0);
        const bool two = !SPARSE || k < full;
        if (two) sto_nt<T>(ho, o1, (T)n1);
        // heat flux of the new distribution about U^{n+1} (Eq. reduced_heat_flux)
        double x0[3], x1[3], e0 = 0.0, e1 = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
          x0[d] = vv[d] - U[d];
          x1[d] = -vv[d] - U[d];
          e0 += x0[d] * x0[d];
          e1 += x1[d] * x1[d];
        }
        double s0 = e0 * n0, s1 = e1 * n1;
        if constexpr (HB) {
          cubic_eo<D>(sb, vv, v2, E, O);
          const double m0 = (double)b0[u] * inv + c0 * (E + O);
          const double m1 = (double)b1[u] * inv + c1 * (E - O);
          sto_nt<T>(bo, o0, (T)m0);
          if (two) sto_nt<T>(bo, o1, (T)m1);
          s0 += m0;
          s1 += m1;
        }
        s0 *= w0[u];
        s1 *= w1[u];
#pragma unroll
        for (int d = 0; d < D; ++d) acc[d] += s0 * x0[d] + s1 * x1[d];
      }
    }
  }
  block_total<3>(acc, red);
  if (threadIdx.x == 0) {
    double qc[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) o.qn[ic * 3 + d] = qc[d] = d < D ? 0.5 * acc[d] : 0.0;
#pragma unroll
    for (int x = 0; x < NPRIM; ++x) o.prim[ic * NPRIM + x] = P[x];
    constexpr int nr = HB ? 2 : 1;
    cell_record<D>(P, g, dt, qc, nr, (C*)o.cs + ic * nr * SREC);
  }
}

// Single case: the sweep computes in the storage type T (FP32 storage uses
// FP32 copies of the records; moment sums stay FP64).  The FP32
// body fits in half the registers; its bound (kCellWaves) asks for the occupancy
// that hides the gathers' latency.  Every variant spills scalar registers (48 to
// 176), the limited 3-D FP64 ones 7 to 9 vector registers too.
//
// Whole-cell form: one work-group takes a cell through all of its velocities
// and then through the rest of the step, so the first stage's rows are read
// back by the compute unit that wrote them, and four launches and their passes
// over the cells go.  One step of 48,000 tets x 24^3, FP64: 10.27 ms as sweep
// (7.55) and second stage (2.11) of their own, 9.54 ms so, 9.18 ms with the
// slot order and the sign branches of the loop; FP32, 28^3: 9.60, 8.96, 8.07;
// cavity of 32^2 cells x 28^2: 0.088, 0.059, 0.056.
// In 2-D, FP32 without the limiter takes h and b in one pass (the registers of 5
// waves per SIMD hold it): 16,384 cells x 32^2 0.220 -> 0.208 ms, 4,096 x 28^2
// 0.067 -> 0.062.  FP64 would lose a resident wave: 1,024 x 28^2 0.031 -> 0.043.
template <typename T, int D, bool LIM>
constexpr bool kBothPasses = D == 2 && sizeof(T) == 4 && !LIM;
template <typename T, int D, bool LIM>
constexpr int kCellWaves = sizeof(T) == 8 ? 4 : kBothPasses<T, D, LIM> ? 5 : 6;  // per SIMD

template <int D, typename T, bool LIM, bool HB, bool SPARSE>
__global__ __launch_bounds__(CELLT, (kCellWaves<T, D, LIM>)) void k_step_cell(
    SweepIn<T> in, SweepSched sc, int64_t nc, GasP g, const T* __restrict__ h, const T* __restrict__ b,
    T* ht, T* bt, CellOut o) {
  __shared__ SweepLds<D, T> L;
  extern __shared__ __attribute__((aligned(16))) char stage_lds[];
  T* stage = (T*)stage_lds;
  // blocks are dealt round-robin to the 8 XCDs; XCD x takes tiles x, x+8, ...
  // of sc.tile consecutive (Z-order) cells, whose stencil rows its L2 shares
  const int64_t xcd = blockIdx.x % 8, local = blockIdx.x / 8;
  const int64_t ic = ((local / sc.tile) * 8 + xcd) * sc.tile + local % sc.tile;
  if (ic >= nc || *o.flag) return;
  double mw[D + 2];
  sweep_item<D, T, T, kBothPasses<T, D, LIM>, LIM, HB, SPARSE>(in, h, b, ht, bt, ic, 0u, in.half, L.s, stage,
                                                               mw);
  block_total<D + 2>(mw, L.red);
  finish_cell<D, T, T, HB, SPARSE>(g, in.vidx, in.w, o, ht, bt, ic, in.nvp, in.half, in.na, in.axis, stage,
                                   in.keep, mw, L.c, L.red, in.full);
}

// Blocked form, for a mesh too small to fill the GPU with whole cells (or a
// caller's block_v): work item = (cell, velocity block); the rest of the step
// runs in kernels of its own.
template <int D, typename T, bool LIM, bool HB>
__global__ __launch_bounds__(SWT, (sizeof(T) == 4 ? 6 : 4)) void k_sweep(
    SweepIn<T> in, SweepSched sc, int64_t nc, const T* __restrict__ h, const T* __restrict__ b,
    T* __restrict__ ht, T* __restrict__ bt, double* __restrict__ dWp,
    const int32_t* __restrict__ flag) {
  __shared__ SweepLds<D, T> L;
  // Blocks are dealt round-robin to the 8 XCDs; XCD x takes tiles x, x+8, ...
  // of sc.tile consecutive (Z-order) cells and runs all of a tile's cells
  // through velocity block 0, then 1, ..., so the stencil rows of one tile and
  // one velocity block are what its L2 must hold.
  const int64_t xcd = blockIdx.x % 8, local = blockIdx.x / 8;
  const int64_t per_tile = sc.nchunk * sc.tile;
  const int64_t tile = (local / per_tile) * 8 + xcd;
  const int64_t rem = local % per_tile;
  const int64_t chunk = rem / sc.tile;
  const int64_t ic = tile * sc.tile + rem % sc.tile;
  if (ic >= nc || *flag) return;
  double mw[D + 2];
  sweep_item<D, T, T, false, LIM, HB>(in, h, b, ht, bt, ic, (unsigned)(chunk * sc.chunk_pairs),
                                      (unsigned)min((int64_t)in.half, (chunk + 1) * sc.chunk_pairs), L.s,
                                      nullptr, mw);
  block_total<D + 2>(mw, L.red);
  if (threadIdx.x == 0)
    for (int x = 0; x < 5; ++x) dWp[(ic * sc.nchunk + chunk) * 5 + x] = x < D + 2 ? mw[x] : 0.0;
}

// One case of a batch as the cells' kernels read it.  The work list and the case
// table are read-only for the whole launch: read through the constant address
// space they are scalar loads, so the case's pointers and sizes land in scalar
// registers as kernel arguments do.  An FP32 batch computes in FP32, as the single
// case does, from the FP32 copies of its records.
typedef const __attribute__((address_space(4))) int32_t citem_t;
typedef const __attribute__((address_space(4))) CaseDev ccase_t;

template <typename T>
__device__ __forceinline__ void case_in(ccase_t& c, SweepIn<T>& in) {
  in.crec_i = c.fm.crec_i;
  in.crec_l = nullptr;
  in.vidx = c.fm.vidx;
  in.w = c.v.w;
  in.frec = c.B.frec;
  in.cs = (const T*)c.B.cs;
  in.srec = (const T*)c.B.srec;
  in.prim = c.B.prim;
  in.dt = c.g.dt;
  in.nvp = c.v.nvp;
  in.half = (unsigned)c.fm.half;
  in.keep = 0;
  in.na = c.fm.na;
  in.axis = c.fm.axis;
  if constexpr (sizeof(T) == 4) in.crec_d = c.fm.crec_d32;
  else in.crec_d = c.fm.crec_d;
}

__device__ __forceinline__ void case_out(ccase_t& c, GasP& g, CellOut& o) {
  g.Pr = c.g.Pr;
  g.R = c.g.R;
  g.Tref = c.g.Tref;
  g.muref = c.g.muref;
  g.omega = c.g.omega;
  g.dt = c.g.dt;
  o.vol = c.m.vol;
  o.W = c.B.W;
  o.q = c.B.q;
  o.Wn = c.B.Wn;
  o.qn = c.B.qn;
  o.prim = c.B.prim;
  o.cs = c.B.cs;
  o.cellred = c.B.cellred;
  o.flag = c.B.flag;
}

// The whole-cell step over a batch of cases: a persistent grid walks a list of
// (case, cell) work items; item w runs on block w mod the grid size, and the
// host orders the list so that the blocks of one XCD (block index mod 8) take
// whole tiles of one case.  Measured on the 64-case batch, one pass for h and b
// against two: 9.2 against 10.4 ms FP64 (9.5 with the registers of 4 waves per
// SIMD), 4.7 against 5.4 FP32 (5.5).
template <int D, typename T>
__global__ __launch_bounds__(SWT, (D == 3 ? 4 : 3)) void k_step_b(BatchDev bd) {
  __shared__ SweepLds<D, T> L;
  citem_t* items = (citem_t*)bd.items;
  ccase_t* cases = (ccase_t*)bd.cases;
  for (int64_t it = blockIdx.x; it < bd.nitems; it += gridDim.x) {
    const int c = items[4 * it];
    if (c < 0) continue;  // padding
    const int64_t ic = items[4 * it + 1];
    GasP g;
    CellOut o;
    SweepIn<T> in;
    case_out(cases[c], g, o);
    case_in<T>(cases[c], in);
    const T* h = (const T*)cases[c].B.h;
    const T* b = (const T*)cases[c].B.b;
    T* ht = (T*)cases[c].B.ht;
    T* bt = (T*)cases[c].B.bt;
    if (*o.flag) continue;
    __syncthreads();  // the previous item's readers of LDS are done
    double mw[D + 2];
    sweep_item<D, T, T, true, false, D == 2>(in, h, b, ht, bt, ic, 0u, in.half, L.s, nullptr, mw);
    block_total<D + 2>(mw, L.red);
    finish_cell<D, T, T, D == 2>(g, in.vidx, in.w, o, ht, bt, ic, in.nvp, in.half, in.na, in.axis, nullptr, 0u,
                              mw, L.c, L.red);
  }
}

// Blocked form of the batch, for one of few cells (or a caller's block_v): items
// (case, cell, block of the case's mirror pairs), then the rest of the step.  One
// work-group per cell leaves compute units idle: 6 tets x 28^3 0.403 ms per step
// whole, 0.080 in 8 blocks; 4 x 750 x 40^3 4.6 (64 lanes; 3.1 with 256) and 3.1;
// 16 x 162 x 32^3 2.22 and 1.34.
template <int D, typename T>
__global__ __launch_bounds__(SWT, (D == 3 ? 4 : 3)) void k_sweep_b(BatchDev bd) {
  __shared__ SweepLds<D, T> L;
  citem_t* items = (citem_t*)bd.items;
  ccase_t* cases = (ccase_t*)bd.cases;
  for (int64_t it = blockIdx.x; it < bd.nitems; it += gridDim.x) {
    const int c = items[4 * it];
    if (c < 0) continue;  // padding
    const int64_t ic = items[4 * it + 1], chunk = items[4 * it + 2];
    if (*cases[c].B.flag) continue;
    SweepIn<T> in;
    case_in<T>(cases[c], in);
    const int64_t nchunk = cases[c].sc.nchunk, pairs = cases[c].sc.chunk_pairs;
    double* dW = cases[c].B.dW + (ic * nchunk + chunk) * 5;
    __syncthreads();  // the previous item's readers of LDS are done
    double mw[D + 2];
    sweep_item<D, T, T, true, false, D == 2>(in, (const T*)cases[c].B.h, (const T*)cases[c].B.b,
                                             (T*)cases[c].B.ht, (T*)cases[c].B.bt, ic, (unsigned)(chunk * pairs),
                                             (unsigned)min((int64_t)in.half, (chunk + 1) * pairs), L.s, nullptr,
                                             mw);
    block_total<D + 2>(mw, L.red);
    if (threadIdx.x == 0)
      for (int x = 0; x < D + 2; ++x) dW[x] = mw[x];
  }
}

// ---- cells of more than four faces ------------------------------------------
// One pass over the mirror pairs of a wide cell for distribution X, from the
// stored gradients (gr): as sweep_pass, but a face's incoming side is read as
// the neighbour's value and gradient (four rows) where its stencil would be
// MAXF rows.  Faces go in groups of WGF, a group's rows loaded together (groups of
// 2, 3, 4 and 6: 0.562, 0.552, 0.552 and 0.554 ms on 4,096 hexahedra x 20^3).
constexpr int WGF = 3;

template <int D, typename T, bool HB, bool GH, int X>
__device__ __forceinline__ void wide_pass(const SweepIn<double>& in, const T* __restrict__ f,
                                          const double* __restrict__ gr, const double* __restrict__ gg,
                                          T* __restrict__ ft, int64_t ic, int32_t ghost0,
                                          const SweepTabs<D, double, MAXF>& L, T* stage,
                                          double (&mw)[D + 2]) {
  typedef double C;
  crec_i_t* ci0 = (crec_i_t*)(in.crec_i + ic * CRI);
  crec_t<C>* cd0 = (crec_t<C>*)(in.crec_d + ic * CRD);
  constexpr int RS = (HB ? 2 : 1) * SREC;
  crec_t<C>* cc0 = (crec_t<C>*)(in.cs + ic * RS);
  crec_t<C>* frc = (crec_t<C>*)in.srec;
  const int nf = ci0[WI_NF];
  const uint32_t rowb = (uint32_t)in.nvp * (uint32_t)sizeof(T), growb = (uint32_t)in.nvp * 8u;
  auto row_of = [rowb, f](int32_t r) { return srow((const char*)f + (uint64_t)(uint32_t)r * rowb); };
  auto grad_of = [growb, gr](int32_t r, int d) {
    return srow((const char*)gr + (uint64_t)(uint32_t)(3 * r + d) * growb);
  };
  grow_t *own = row_of((int32_t)ic), *wt = srow(in.w), *ix = srow(in.vidx);
  gout_t* dst = sout(ft + ic * in.nvp);
  for (unsigned kp = threadIdx.x; kp < in.half; kp += blockDim.x) {
    const int pk = ldo<int32_t, int>(ix, kp * 4u);
    const uint32_t o0 = kp * (uint32_t)sizeof(T), o1 = o0 + in.half * (uint32_t)sizeof(T);
    const uint32_t q0 = kp * 8u, q1 = q0 + in.half * 8u;
    const C f0 = ldo<T, C>(own, o0), f1 = ldo<T, C>(own, o1);
    C g0[D], g1[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
      grow_t* gd = grad_of((int32_t)ic, d);
      g0[d] = ldo<double, C>(gd, q0);
      g1[d] = ldo<double, C>(gd, q1);
    }
    unsigned at[D];
    C vv[3] = {0.0, 0.0, 0.0}, v2 = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      at[d] = node_off<C>(pk, d);
      vv[d] = *(const C*)((const char*)L.ax + at[d]);
      v2 += vv[d] * vv[d];
    }
    C ug0 = 0.0, ug1 = 0.0, acc0 = 0.0, acc1 = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      ug0 += vv[d] * g0[d];
      ug1 -= vv[d] * g1[d];
    }
    for (int p0 = 0; p0 < nf; p0 += WGF) {
      crec_i_t* ci = ci0 + p0;
      crec_t<C>* cd = cd0 + WD_FS * p0;
      C sp[WGF], fj[WGF], gj[WGF][D];
#pragma unroll
      for (int p = 0; p < WGF; ++p)
        if (p0 + p < nf) {
          C s = 0.0;
#pragma unroll
          for (int d = 0; d < D; ++d) s += vv[d] * cd[WD_FS * p + d];
          sp[p] = s;
          const int32_t row = ci[WI_ROW + p];
          // u.n > 0: the incoming member is -u
          if (!GH || row < ghost0) fj[p] = ldo<T, C>(row_of(row), s > 0.0 ? o1 : o0);
          else fj[p] = ldo<double, C>(srow((const char*)gg + (uint64_t)(uint32_t)(row - ghost0) * growb), s > 0.0 ? q1 : q0);
          if (ci[WI_KIND + p] == UGKS_BC_INTERIOR) {
#pragma unroll
            for (int d = 0; d < D; ++d) gj[p][d] = ldo<double, C>(grad_of(row, d), s > 0.0 ? q1 : q0);
          } else {
#pragma unroll
            for (int d = 0; d < D; ++d) gj[p][d] = 0.0;
          }
        }
#pragma unroll
      for (int p = 0; p < WGF; ++p)
        if (p0 + p < nf) {
          crec_t<C>* fd = cd + WD_FS * p;
          C R[SREC];
          load_rec<C, SREC>(frc + (uint64_t)(uint32_t)ci[WI_FACE + p] * RS + X * SREC, R);
          const C sas = fd[10] * fabs(sp[p]);
          C e0, e1;
          tab_pair(L.tab[p0 + p][0], at[0], e0, e1);
#pragma unroll
          for (int d = 1; d < D; ++d) {
            C a0, a1;
            tab_pair(L.tab[p0 + p][d], at[d], a0, a1);
            e0 *= a0;
            e1 *= a1;
          }
          C E, O;
          cubic_eo<D>(R + SR_P, vv, v2, E, O);
          auto flux = [&](C fo, const C* go, C ugo, C eqo, C su, C eqi, C& acco, C& acci) {
            C ff = fo, ffj = fj[p], ugj = 0.0;
#pragma unroll
            for (int d = 0; d < D; ++d) {
              ff += fd[3 + d] * go[d];
              ffj += fd[6 + d] * gj[p][d];
              ugj += vv[d] * gj[p][d];
            }
            acco += sas * (R[0] * ff + R[1] * ugo + fd[9] * eqo);
            acci -= sas * (R[0] * ffj + R[1] * (su * ugj) + eqi);
          };
          if (sp[p] > 0.0) flux(f0, g0, ug0, e0 * (E + O), -1.0, e1 * (E - O), acc0, acc1);
          else flux(f1, g1, ug1, e1 * (E - O), 1.0, e0 * (E + O), acc1, acc0);
        }
    }
    add_moments<D, C, X>(ldo<double, double>(wt, kp * 8u), ldo<double, double>(wt, (kp + in.half) * 8u), acc0,
                         acc1, vv, v2, mw);
    C c0, c1;
    tab_pair(L.tab[MAXF][0], at[0], c0, c1);
#pragma unroll
    for (int d = 1; d < D; ++d) {
      C a0, a1;
      tab_pair(L.tab[MAXF][d], at[d], a0, a1);
      c0 *= a0;
      c1 *= a1;
    }
    C t0, t1;
    first_stage<D, C, X>(cc0, vv, v2, c0, c1, f0, f1, acc0, acc1, t0, t1);
    if (kp < in.keep) {
      stage[2 * X * in.keep + kp] = (T)t0;
      stage[(2 * X + 1) * in.keep + kp] = (T)t1;
    } else {
      sto<T>(dst, o0, (T)t0);
      sto<T>(dst, o1, (T)t1);
    }
  }
}

// A wide cell's step after the gradients and wall densities: fluxes, first
// stage and the rest of the step in one work-group, FP64 arithmetic in either
// storage form.  Every face's flux is evaluated from both of its cells, with the
// axis tables and polynomials of the fused sweep, so no flux goes through memory.
// 4,096 hexahedra x 20^3, FP64: 0.55 ms (2.4 TB/s of rows and gradients read once
// and states written), where face fluxes, two stages and heat flux as passes of
// their own take 2.0.
template <int D, typename T, bool HB, bool GH>
__global__ __launch_bounds__(CELLT, 4) void k_step_wide(SweepIn<double> in, SweepSched sc, int64_t nc, GasP g,
                                                        const T* __restrict__ h, const T* __restrict__ b,
                                                        const double* __restrict__ gh,
                                                        const double* __restrict__ gb,
                                                        const double* __restrict__ hg,
                                                        const double* __restrict__ bg, T* ht, T* bt,
                                                        CellOut o) {
  __shared__ SweepLds<D, double, MAXF> L;
  extern __shared__ __attribute__((aligned(16))) char stage_lds[];
  T* stage = (T*)stage_lds;
  const int64_t xcd = blockIdx.x % 8, local = blockIdx.x / 8;
  const int64_t ic = ((local / sc.tile) * 8 + xcd) * sc.tile + local % sc.tile;
  if (ic >= nc || *o.flag) return;
  sweep_tables<D, double, MAXF>(in, ic, L.s);
  __syncthreads();
  double mw[D + 2];
#pragma unroll
  for (int x = 0; x < D + 2; ++x) mw[x] = 0.0;
  const int32_t ghost0 = (int32_t)nc + 1;
  auto passes = [&](auto far) {
    constexpr bool FAR = decltype(far)::value;
    wide_pass<D, T, HB, FAR, 0>(in, h, gh, hg, ht, ic, ghost0, L.s, stage, mw);
    if constexpr (HB) wide_pass<D, T, HB, FAR, 1>(in, b, gb, bg, bt, ic, ghost0, L.s, stage, mw);
  };
  if constexpr (GH) {
    if (((crec_i_t*)(in.crec_i + ic * CRI))[WI_FAR]) passes(std::true_type{});
    else passes(std::false_type{});
  } else {
    passes(std::false_type{});
  }
  block_total<D + 2>(mw, L.red);
  finish_cell<D, T, double, HB>(g, in.vidx, in.w, o, ht, bt, ic, in.nvp, in.half, in.na, in.axis, stage,
                                in.keep, mw, L.c, L.red);
}

// The macroscopic flux F of every face (Eq. macro_flux) from h^n, b^n and the
// stored gradients, one work-group per face.  The step itself does not need
// it: it runs for the last step of a call, whose face fluxes can be asked for,
// and with boundary-flux tracking.
template <int D, typename T, bool HB, bool GH>
__global__ __launch_bounds__(SWT) void k_face_flux(DevMesh m, SweepIn<double> in,
                                                   const int32_t* __restrict__ frow,
                                                   const T* __restrict__ h, const T* __restrict__ b,
                                                   const double* __restrict__ gh,
                                                   const double* __restrict__ gb,
                                                   const double* __restrict__ hg,
                                                   const double* __restrict__ bg, double* __restrict__ F,
                                                   const int32_t* flag) {
  __shared__ double tab[D][NAX], red[5 * 16];
  if (*flag) return;
  const int64_t f = face_of_block(m);
  if (f < 0) return;
  const int na = in.na;
  const double* R = in.frec + f * FREC;
  const bool wall = m.fbc[f] == UGKS_BC_WALL;
  for (int t = threadIdx.x; t < D * na; t += SWT) {
    const int d = t / na, n = t % na;
    const double c = in.axis[n] - R[FR_U + d];
    const double sc = d > 0 ? 1.0 : wall ? R[FR_C0] * R[FR_RHOW] * in.dt : R[FR_C0];
    tab[d][n] = sc * exp(-R[FR_LAM] * c * c);
  }
  __syncthreads();
  const int64_t Lc = m.fL[f], Rr = frow[f], nvp = in.nvp, gm = Rr - m.nc - 1;  // gm: ghost row
  const bool inner = m.fbc[f] == UGKS_BC_INTERIOR;
  double n[3], dL[3], dR[3];
  for (int d = 0; d < 3; ++d) {
    n[d] = m.fnorm[f * 3 + d];
    dL[d] = m.fdxL[f * 3 + d];
    dR[d] = m.fdxR[f * 3 + d];
  }
  double acc[5] = {0, 0, 0, 0, 0};
  for (unsigned kp = threadIdx.x; kp < in.half; kp += SWT) {
    const int pk = in.vidx[kp];
    double vv[3] = {0, 0, 0}, un = 0.0, v2 = 0.0, e0 = 1.0, e1 = 1.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int id = node_of(pk, d);
      vv[d] = in.axis[id];
      un += vv[d] * n[d];
      v2 += vv[d] * vv[d];
      e0 *= tab[d][id];
      e1 *= tab[d][na - 1 - id];
    }
    const bool pos = un > 0.0;  // u leaves the left cell, -u enters it
    const int64_t kl = pos ? kp : kp + in.half, kr = pos ? kp + in.half : kp;
    const double sl = pos ? 1.0 : -1.0, wl = in.w[kl], wr = in.w[kr];
#pragma unroll
    for (int r = 0; r < (HB ? 2 : 1); ++r) {
      const T* fv = r ? b : h;
      const double* gr = r ? gb : gh;
      const double* S = in.srec + (f * (HB ? 2 : 1) + r) * SREC;
      double fl = ld(fv, Lc * nvp + kl), ul = 0.0, ur = 0.0;
      double fr = GH && gm >= 0 ? (r ? bg : hg)[gm * nvp + kr] : ld(fv, Rr * nvp + kr);
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const double a = gr[(Lc * 3 + d) * nvp + kl];
        fl += dL[d] * a;
        ul += sl * vv[d] * a;
        if (inner) {
          const double c = gr[(Rr * 3 + d) * nvp + kr];
          fr += dR[d] * c;
          ur -= sl * vv[d] * c;
        }
      }
      double E, O;
      cubic_eo<D>(S + SR_P, vv, v2, E, O);
      const double q0 = e0 * (E + O), q1 = e1 * (E - O);
      const double Hl = wl * fabs(un) * (S[0] * fl + S[1] * ul + (wall ? 0.0 : pos ? q0 : q1));
      const double Hr = -wr * fabs(un) * (S[0] * fr + S[1] * ur + (pos ? q1 : q0));
      if (r == 0) {
        acc[0] += Hl + Hr;
#pragma unroll
        for (int d = 0; d < D; ++d) acc[1 + d] += sl * vv[d] * (Hl - Hr);
        acc[D + 1] += 0.5 * v2 * (Hl + Hr);
      } else {
        acc[D + 1] += 0.5 * (Hl + Hr);
      }
    }
  }
  block_sum<5>(acc, red);
  if (threadIdx.x == 0)
    for (int x = 0; x < 5; ++x) F[f * 5 + x] = x < D + 2 ? acc[x] : 0.0;
}

// The rest of the step of the blocked form, one work-group per cell.  The
// partial sums of the velocity blocks are added in block order.
template <int D, typename T, bool HB>
__global__ __launch_bounds__(SWT) void k_finish(SweepIn<T> in, GasP g, int64_t nchunk,
                                                const double* __restrict__ dWp, T* ht, T* bt, CellOut o) {
  __shared__ SweepLds<D, T> L;
  const int64_t ic = blockIdx.x;
  if (*o.flag) return;
  double tot[D + 2];
#pragma unroll
  for (int x = 0; x < D + 2; ++x) {
    tot[x] = 0.0;
    for (int64_t c = 0; c < nchunk; ++c) tot[x] += dWp[(ic * nchunk + c) * 5 + x];
  }
  finish_cell<D, T, T, HB>(g, in.vidx, in.w, o, ht, bt, ic, in.nvp, in.half, in.na, in.axis, nullptr, 0u, tot,
                        L.c, L.red);
}

// The same over a batch, one work-group per cell.
__device__ __forceinline__ int case_of(const int64_t* __restrict__ off, int n, int64_t t);

template <int D, typename T>
__global__ __launch_bounds__(SWT) void k_finish_b(BatchDev bd) {
  __shared__ SweepLds<D, T> L;
  const int c = case_of(bd.cell_off, bd.n, blockIdx.x);
  const int64_t ic = (int64_t)blockIdx.x - bd.cell_off[c];
  ccase_t& C = ((ccase_t*)bd.cases)[c];
  GasP g;
  CellOut o;
  case_out(C, g, o);
  if (*o.flag) return;
  const int64_t nchunk = C.sc.nchunk;
  const double* dW = C.B.dW + ic * nchunk * 5;
  double tot[D + 2];
#pragma unroll
  for (int x = 0; x < D + 2; ++x) {
    tot[x] = 0.0;
    for (int64_t k = 0; k < nchunk; ++k) tot[x] += dW[k * 5 + x];
  }
  finish_cell<D, T, T, D == 2>(g, C.fm.vidx, C.v.w, o, (T*)C.B.ht, (T*)C.B.bt, ic, C.v.nvp, (unsigned)C.fm.half,
                               C.fm.na, C.fm.axis, nullptr, 0u, tot, L.c, L.red);
}

// Wall density with the wall cell's gradient evaluated in place.
struct WallLds {
  double ax[NAX];
  double wx[3][NAX];  // axis factors of the wall Maxwellian, C_w folded into the first
  double red[2 * 16];
  double red2[5 * 16];
};

// Wall density of one wall face: the incident free transport of the wall
// cell (its gradient evaluated in place) against the re-emitted wall
// Maxwellian, whose value at a tensor point is a product of D LDS axis
// factors.  A lane takes mirror pairs: exactly one member is incident, the
// other leaves, so the lanes do not diverge and each pair reads f once.  Bound
// by the five rows read of every wall cell: 4,800 walls x 28^3 FP32 0.42 ms
// with one slot per lane and turn, 0.19 so;
// 24^3 FP64 0.246 and 0.178.
template <int D, typename T, bool LIM = false, bool BF = false>
__device__ __forceinline__ void wall_rho_at(int64_t wi, const DevMesh& m, const DevVel& v,
                                            const FusedMesh& fm, const GasP& g,
                                            const T* __restrict__ h, double* __restrict__ frec,
                                            const int32_t* flag, WallLds& S,
                                            const T* __restrict__ b = nullptr) {
  if (*flag) return;
  const int f = m.walls[wi];
  const int64_t L = m.fL[f];
  const int64_t nvp = v.nvp;
  double* R = &frec[(int64_t)f * FREC];
  const double lamw = R[FR_LAM], Cw = R[FR_C0], dt = g.dt;
  const int na = fm.na;
  for (int t = threadIdx.x; t < D * na; t += blockDim.x) {
    const int d = t / na, n = t % na;
    const double c = fm.axis[n] - R[FR_U + d];
    S.wx[d][n] = (d == 0 ? Cw : 1.0) * exp(-lamw * c * c);
  }
  for (int t = threadIdx.x; t < na; t += blockDim.x) S.ax[t] = fm.axis[t];
  __syncthreads();
  double nrm[3] = {0, 0, 0}, dxl[3] = {0, 0, 0};
  for (int d = 0; d < D; ++d) {
    nrm[d] = m.fnorm[f * 3 + d];
    dxl[d] = m.fdxL[f * 3 + d];
  }
  // The wall cell's padded stencil from its fused record: the row across
  // each face (a neighbour, the zero row with coefficient 0 across a wall,
  // the ghost row across a far-field or outflow face) and the least-squares
  // coefficients, wave-uniform for the whole loop.
  crec_i_t* ci = (crec_i_t*)(fm.crec_i + L * CRI);
  crec_t<double>* cd = (crec_t<double>*)(fm.crec_d + L * CRD);
  crec_t<double>* cl = LIM ? (crec_t<double>*)(fm.crec_l + L * CRL) : nullptr;
  auto row_of = [nvp](const T* base, int64_t r) { return srow_any(base + r * nvp); };
  // value and u.gradient of the wall cell's reconstruction at the wall
  auto at_wall = [&](double fi, const double (&fs)[4], const double* u, double& ff, double& ug) {
    double gr[3] = {0, 0, 0};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double df = fs[s] - fi;
#pragma unroll
      for (int d = 0; d < D; ++d) gr[d] += cd[CD_G + d * 4 + s] * df;
    }
    if constexpr (LIM) {
      // limited as the sweep limits it
      double lo = fi, hi = fi;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const double vs = cl[1 + s] * fi + fs[s];
        lo = fmin(lo, vs);
        hi = fmax(hi, vs);
      }
      const double ph = venkat_phi<D>(fi, lo, hi, gr, cd + CD_F0, CD_FS, cl[0]);
#pragma unroll
      for (int d = 0; d < D; ++d) gr[d] *= ph;
    }
    ff = fi;
    ug = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      ff += dxl[d] * gr[d];
      ug += u[d] * gr[d];
    }
  };
  grow_t *own = row_of(h, L), *rs[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) rs[s] = row_of(h, ci[CI_OWN + s]);
  grow_t *wt = srow_any(v.w), *ix = srow_any(fm.vidx);
  double acc[2] = {0.0, 0.0};
  // with BF: the wall flux's moments, incident (time-integrated free transport
  // of the wall cell's h, and b in 2-D) and reflected (per unit rho_w dt)
  double bfi[D + 2], bfr[D + 2];
#pragma unroll
  for (int x = 0; x < D + 2; ++x) bfi[x] = bfr[x] = 0.0;
  // a few pairs per lane per pass, their rows loaded together (FP32 with 4: 0.207)
  constexpr unsigned UN = sizeof(T) == 8 ? 4 : 2;
  const unsigned nb = blockDim.x, half = (unsigned)fm.half;
  for (unsigned k0 = threadIdx.x; k0 < half; k0 += UN * nb) {
    int pk[UN];
#pragma unroll
    for (unsigned u = 0; u < UN; ++u) {
      const unsigned kp = k0 + u * nb;
      if (kp < half) pk[u] = ldo<int32_t, int>(ix, kp * 4u);
    }
    double uu[UN][3], un[UN], hl[UN], hs[UN][4], wi_[UN], wo[UN], M[UN];
    unsigned kin[UN];
#pragma unroll
    for (unsigned u = 0; u < UN; ++u) {
      const unsigned kp = k0 + u * nb;
      if (kp < half) {  // whole waves: half is a multiple of 64
        int id[3];
        un[u] = 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
          id[d] = node_of(pk[u], d);
          uu[u][d] = S.ax[id[d]];
          un[u] += uu[u][d] * nrm[d];
        }
        const bool pos = un[u] > 0.0;  // u is incident, else -u
        M[u] = 1.0;
#pragma unroll
        for (int d = 0; d < D; ++d) {
          M[u] *= S.wx[d][pos ? na - 1 - id[d] : id[d]];
          uu[u][d] = pos ? uu[u][d] : -uu[u][d];
        }
        un[u] = fabs(un[u]);
        const unsigned kout = pos ? kp + half : kp;
        kin[u] = pos ? kp : kp + half;
        const uint32_t off = kin[u] * (uint32_t)sizeof(T);
        hl[u] = ldo<T, double>(own, off);
#pragma unroll
        for (int s = 0; s < 4; ++s) hs[u][s] = ldo<T, double>(rs[s], off);
        wi_[u] = ldo<double, double>(wt, kin[u] * 8u);
        wo[u] = ldo<double, double>(wt, kout * 8u);
      }
    }
#pragma unroll
    for (unsigned u = 0; u < UN; ++u) {
      const unsigned kp = k0 + u * nb;
      if (kp < half) {
        double hf, ugh;
        at_wall(hl[u], hs[u], uu[u], hf, ugh);
        const double fi = wi_[u] * un[u] * (dt * hf - 0.5 * dt * dt * ugh);  // incident
        const double fo = -wo[u] * un[u] * M[u];                             // re-emitted, per rho_w dt
        acc[0] += fi;
        acc[1] += fo;
        if constexpr (BF) {
          double u2 = 0.0;
#pragma unroll
          for (int d = 0; d < D; ++d) {
            bfi[1 + d] += uu[u][d] * fi;
            bfr[1 + d] -= uu[u][d] * fo;
            u2 += uu[u][d] * uu[u][d];
          }
          bfi[0] += fi;
          bfi[D + 1] += 0.5 * u2 * fi;
          bfr[0] += fo;
          // the re-emitted b = K_xi/(2 lambda_w) H_w adds to the energy
          bfr[D + 1] += 0.5 * (u2 + v.kxi / (2.0 * lamw)) * fo;
          if (b != nullptr) {
            // the b part of the energy: the same free transport of the wall cell's b
            const uint32_t off = kin[u] * (uint32_t)sizeof(T);
            double bs[4], bf, ugb;
#pragma unroll
            for (int s = 0; s < 4; ++s) bs[s] = ldo<T, double>(row_of(b, ci[CI_OWN + s]), off);
            at_wall(ldo<T, double>(row_of(b, L), off), bs, uu[u], bf, ugb);
            bfi[D + 1] += 0.5 * wi_[u] * un[u] * (dt * bf - 0.5 * dt * dt * ugb);
          }
        }
      }
    }
  }
  block_sum<2>(acc, S.red);
  if constexpr (BF) {
    __syncthreads();
    block_sum<D + 2>(bfi, S.red2);
    __syncthreads();
    block_sum<D + 2>(bfr, S.red2);
  }
  if (threadIdx.x == 0) {
    const double rhow = -acc[0] / (dt * acc[1]);
    R[FR_RHOW] = rhow;
    // the wall face's time-integrated flux of mass, momentum and energy
    // (Eq. macro_flux): incident part plus rho_w dt times the re-emitted part
    if constexpr (BF)
      for (int x = 0; x < D + 2; ++x) R[FR_BF + x] = bfi[x] + rhow * dt * bfr[x];
  }
}

// Ghost rows of the far-field / outflow faces, from row `first` of h and b on: the Maxwellian of the face's
// ghost state W_g (written by the interface-equilibrium pass), h and, where
// b is stored, b = K_xi/(2 lambda_g) h, so the sweep reads them as neighbour rows.
template <int D, typename T>
__device__ __forceinline__ void ghost_row_at(int64_t m, int64_t first, const int32_t* __restrict__ ffaces,
                                             const DevVel& v, const double* __restrict__ frec,
                                             T* __restrict__ h, T* __restrict__ b,
                                             const int32_t* flag) {
  if (*flag) return;
  const double* R = &frec[(int64_t)ffaces[m] * FREC];
  const double C = R[FR_GC], lam = R[FR_GLAM];
  const double U[3] = {R[FR_GU], R[FR_GU + 1], R[FR_GU + 2]};
  const int64_t row = (first + m) * v.nvp;
  for (int64_t k = threadIdx.x; k < v.nvp; k += blockDim.x) {
    double c2 = 0.0;
    for (int d = 0; d < D; ++d) {
      const double c = v.u[d * v.nvp + k] - U[d];
      c2 += c * c;
    }
    const double hv = C * exp(-lam * c2);
    st(h, row + k, hv);
    if (v.has_b) st(b, row + k, v.kxi / (2.0 * lam) * hv);
  }
}

// One work-group per wall face (256 lanes measured faster than 1024).
constexpr int WALLT = 256;

// With BF (boundary-flux tracking) the pass also keeps each wall face's flux; b
// is the b array where b is stored (its part of the energy flux), else null.
// The work-groups after the walls' fill the ghost rows, where the launch has
// any: 960 cells x 24^2 with 48 walls and 48 far-field faces 13.9 us in two
// launches, 7.6 in one.
template <int D, typename T, bool LIM, bool BF>
__global__ __launch_bounds__(WALLT) void k_wall_rho_inline(DevMesh m, DevVel v, FusedMesh fm, GasP g,
                                                         T* h, T* b, double* frec, const int32_t* flag) {
  __shared__ WallLds S;
  const int64_t ghost = (int64_t)blockIdx.x - m.nwall;
  if (ghost >= 0) ghost_row_at<D, T>(ghost, m.nc + 1, fm.ffaces, v, frec, h, b, flag);
  else wall_rho_at<D, T, LIM, BF>(blockIdx.x, m, v, fm, g, h, frec, flag, S, b);
}

template <int D, typename T>
__global__ __launch_bounds__(SWT) void k_ghost_rows(int64_t first, const int32_t* __restrict__ ffaces,
                                                    DevVel v, const double* __restrict__ frec,
                                                    T* __restrict__ h, T* __restrict__ b,
                                                    const int32_t* flag) {
  ghost_row_at<D, T>(blockIdx.x, first, ffaces, v, frec, h, b, flag);
}

// ---- batched forms: one launch covers every case of a batch ---------------
// Element t of a flattened range belongs to case c with off[c] <= t < off[c+1].
__device__ __forceinline__ int case_of(const int64_t* __restrict__ off, int n, int64_t t) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (off[mid] <= t) lo = mid;
    else hi = mid;
  }
  return lo;
}

// W^n, q -> prim, cs before the first step (the step itself leaves the next one's)
template <int D, typename T>
__global__ __launch_bounds__(128) void k_cell_prep_b(BatchDev bd) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= bd.cell_off[bd.n]) return;
  const int c = case_of(bd.cell_off, bd.n, t);
  const CaseDev& C = bd.cases[c];
  cell_prep_at<D>(t - bd.cell_off[c], C.g, C.B.W, C.B.q, C.B.prim, C.fm.nr, (T*)C.B.cs, C.B.flag);
}

// one block per far-field / outflow face of the batch
template <int D, typename T>
__global__ __launch_bounds__(SWT) void k_ghost_rows_b(BatchDev bd) {
  const int64_t t = blockIdx.x;
  const int c = case_of(bd.ff_off, bd.n, t);
  const CaseDev& C = bd.cases[c];
  ghost_row_at<D, T>(t - bd.ff_off[c], C.m.nc + 1, C.fm.ffaces, C.v, C.B.frec, (T*)C.B.h, (T*)C.B.b,
                     C.B.flag);
}

// one block per wall face of the batch
template <int D, typename T>
__global__ __launch_bounds__(WALLT) void k_wall_rho_b(BatchDev bd) {
  __shared__ WallLds S;
  const int64_t t = blockIdx.x;
  const int c = case_of(bd.wall_off, bd.n, t);
  const CaseDev& C = bd.cases[c];
  wall_rho_at<D, T>(t - bd.wall_off[c], C.m, C.v, C.fm, C.g, (const T*)C.B.h, C.B.frec, C.B.flag,
                    S);
}

}  // namespace

#define UGKS_DISPATCH_D(D_, ...) \
  do {                           \
    if ((D_) == 2) {             \
      constexpr int DD = 2;      \
      __VA_ARGS__;               \
    } else {                     \
      constexpr int DD = 3;      \
      __VA_ARGS__;               \
    }                            \
  } while (0)

#define UGKS_DISPATCH_DT(D_, P_, ...)   \
  do {                                  \
    if ((P_) == UGKS_FP32) {            \
      using TT = float;                 \
      UGKS_DISPATCH_D(D_, __VA_ARGS__); \
    } else {                            \
      using TT = double;                \
      UGKS_DISPATCH_D(D_, __VA_ARGS__); \
    }                                   \
  } while (0)

// precision only (the dimension fixed by the kernel named)
#define UGKS_DISPATCH_T(P_, ...)      \
  do {                                \
    if ((P_) == UGKS_FP32) {          \
      using TT = float;               \
      __VA_ARGS__;                    \
    } else {                          \
      using TT = double;              \
      __VA_ARGS__;                    \
    }                                 \
  } while (0)

hipError_t launch_cell_prep(int D, int prec, int nr, int64_t nc, const GasP& g, const double* W,
                            const double* q, double* prim, void* cs, int32_t* flag, hipStream_t s) {
  const unsigned grid = (unsigned)((nc + 127) / 128);
  UGKS_DISPATCH_DT(D, prec, k_cell_prep<DD, TT><<<grid, 128, 0, s>>>(nc, g, W, q, prim, nr, (TT*)cs, flag));
  return hipGetLastError();
}

namespace {

template <typename T>
SweepIn<T> sweep_in(const FusedMesh& fm, const DevVel& v, const GasP& g, const StepBuffers& B) {
  SweepIn<T> in{};
  in.crec_i = fm.crec_i;
  in.vidx = fm.vidx;
  in.w = v.w;
  in.frec = B.frec;
  in.cs = (const T*)B.cs;
  in.srec = (const T*)B.srec;
  in.prim = B.prim;
  in.dt = g.dt;
  in.nvp = v.nvp;
  in.half = (unsigned)fm.half;
  in.full = (unsigned)fm.full;
  in.na = fm.na;
  in.axis = fm.axis;
  if constexpr (sizeof(T) == 4) {
    in.crec_d = fm.crec_d32;
    in.crec_l = fm.crec_l32;
  } else {
    in.crec_d = fm.crec_d;
    in.crec_l = fm.crec_l;
  }
  return in;
}

CellOut cell_out(const DevMesh& m, const StepBuffers& B) {
  CellOut o{};
  o.vol = m.vol;
  o.W = B.W;
  o.q = B.q;
  o.Wn = B.Wn;
  o.qn = B.qn;
  o.prim = B.prim;
  o.cs = B.cs;
  o.cellred = B.cellred;
  o.flag = B.flag;
  return o;
}

// Pairs (of `pair` bytes) whose first stage fits the LDS that `waves` resident
// waves per compute unit leave beside the work-groups' own `used` bytes.
unsigned kept_pairs(int waves, const SweepSched& sc, int64_t used, int64_t pair, unsigned half) {
  const int64_t groups = waves / (sc.lanes / WAVE);
  const int64_t room = kLdsPerCu / groups / kLdsGrain * kLdsGrain - used;
  return (unsigned)(std::max<int64_t>(0, std::min<int64_t>(half, room / pair)) / WAVE * WAVE);
}

template <int D, typename T, bool LIM, bool HB>
void launch_sweep_as(const FusedMesh& fm, const DevVel& v, const GasP& g, const SweepSched& sc,
                     const StepBuffers& B, hipStream_t s) {
  const int64_t ntile = (fm.nc + sc.tile - 1) / sc.tile;
  const unsigned grid = (unsigned)(((ntile + 7) / 8) * 8 * sc.nchunk * sc.tile);
  k_sweep<D, T, LIM, HB><<<grid, SWT, 0, s>>>(sweep_in<T>(fm, v, g, B), sc, fm.nc, (const T*)B.h,
                                              (const T*)B.b, (T*)B.ht, (T*)B.bt, B.dW, B.flag);
}

template <int D, typename T, bool LIM, bool HB>
void launch_step_as(const DevMesh& m, const FusedMesh& fm, const DevVel& v, const GasP& g,
                    const SweepSched& sc, const StepBuffers& B, hipStream_t s) {
  const int64_t ntile = (fm.nc + sc.tile - 1) / sc.tile;
  const unsigned grid = (unsigned)(((ntile + 7) / 8) * 8 * sc.tile);
  SweepIn<T> in = sweep_in<T>(fm, v, g, B);
  // The first stage stays in what LDS the resident work-groups leave free (4
  // kCellWaves waves per compute unit, the registers' bound), so that
  // much of it does not go to memory and back: 48,000 x 24^3 FP64 9.18 ->
  // 8.36 ms per step (58 % of the row kept), x 28^3 FP32 8.07 -> 7.90 (51 %),
  // 16,384 cells x 32^2 FP32 0.317 -> 0.283 (all).  One grain too many costs a
  // resident work-group: 8.48 on the second.
  const int64_t pair = (HB ? 4 : 2) * (int64_t)sizeof(T);
  in.keep = kept_pairs(4 * kCellWaves<T, D, LIM>, sc, sizeof(SweepLds<D, T>), pair, in.half);
  if (fm.sparse)
    k_step_cell<D, T, LIM, HB, true><<<grid, sc.lanes, (size_t)in.keep * pair, s>>>(
        in, sc, fm.nc, g, (const T*)B.h, (const T*)B.b, (T*)B.ht, (T*)B.bt, cell_out(m, B));
  else
    k_step_cell<D, T, LIM, HB, false><<<grid, sc.lanes, (size_t)in.keep * pair, s>>>(
        in, sc, fm.nc, g, (const T*)B.h, (const T*)B.b, (T*)B.ht, (T*)B.bt, cell_out(m, B));
}

}  // namespace

// dimension, limiter and whether b is carried (always in 2-D)
#define UGKS_SWEEP_AS(FN, ...)                                                       \
  do {                                                                              \
    if (D == 2) {                                                                   \
      if (fm.crec_l) UGKS_DISPATCH_T(prec, (FN<2, TT, true, true>(__VA_ARGS__)));   \
      else UGKS_DISPATCH_T(prec, (FN<2, TT, false, true>(__VA_ARGS__)));            \
    } else if (B.b) {                                                               \
      if (fm.crec_l) UGKS_DISPATCH_T(prec, (FN<3, TT, true, true>(__VA_ARGS__)));   \
      else UGKS_DISPATCH_T(prec, (FN<3, TT, false, true>(__VA_ARGS__)));            \
    } else {                                                                        \
      if (fm.crec_l) UGKS_DISPATCH_T(prec, (FN<3, TT, true, false>(__VA_ARGS__)));  \
      else UGKS_DISPATCH_T(prec, (FN<3, TT, false, false>(__VA_ARGS__)));           \
    }                                                                               \
  } while (0)

hipError_t launch_sweep(int D, int prec, const FusedMesh& fm, const DevVel& v, const GasP& g,
                        const SweepSched& sc, const StepBuffers& B, hipStream_t s) {
  UGKS_SWEEP_AS(launch_sweep_as, fm, v, g, sc, B, s);
  return hipGetLastError();
}

hipError_t launch_step_cell(int D, int prec, const DevMesh& m, const FusedMesh& fm, const DevVel& v,
                            const GasP& g, const SweepSched& sc, const StepBuffers& B, hipStream_t s) {
  if (sc.lanes % 64 != 0 || sc.lanes < 64 || sc.lanes > CELLT) return hipErrorInvalidValue;
  UGKS_SWEEP_AS(launch_step_as, m, fm, v, g, sc, B, s);
  return hipGetLastError();
}
#undef UGKS_SWEEP_AS

hipError_t launch_finish(int D, int prec, const DevMesh& m, const FusedMesh& fm, const DevVel& v,
                         const GasP& g, const SweepSched& sc, const StepBuffers& B, hipStream_t s) {
  const unsigned grid = (unsigned)fm.nc;
  if (D == 2)
    UGKS_DISPATCH_T(prec, (k_finish<2, TT, true><<<grid, SWT, 0, s>>>(
        sweep_in<TT>(fm, v, g, B), g, sc.nchunk, B.dW, (TT*)B.ht, (TT*)B.bt, cell_out(m, B))));
  else if (B.b)
    UGKS_DISPATCH_T(prec, (k_finish<3, TT, true><<<grid, SWT, 0, s>>>(
        sweep_in<TT>(fm, v, g, B), g, sc.nchunk, B.dW, (TT*)B.ht, (TT*)B.bt, cell_out(m, B))));
  else
    UGKS_DISPATCH_T(prec, (k_finish<3, TT, false><<<grid, SWT, 0, s>>>(
        sweep_in<TT>(fm, v, g, B), g, sc.nchunk, B.dW, (TT*)B.ht, (TT*)B.bt, cell_out(m, B))));
  return hipGetLastError();
}

namespace {
template <int D, typename T, bool HB>
void launch_wide_as(const DevMesh& m, const FusedMesh& fm, const DevVel& v, const GasP& g,
                    const SweepSched& sc, const StepBuffers& B, hipStream_t s) {
  const int64_t ntile = (fm.nc + sc.tile - 1) / sc.tile;
  const unsigned grid = (unsigned)(((ntile + 7) / 8) * 8 * sc.tile);
  SweepIn<double> in = sweep_in<double>(fm, v, g, B);
  const int64_t pair = (HB ? 4 : 2) * (int64_t)sizeof(T);
  in.keep = kept_pairs(16, sc, sizeof(SweepLds<D, double, MAXF>), pair, in.half);
  auto run = [&](auto gh) {
    k_step_wide<D, T, HB, decltype(gh)::value><<<grid, sc.lanes, (size_t)in.keep * pair, s>>>(
        in, sc, fm.nc, g, (const T*)B.h, (const T*)B.b, B.gradh, B.gradb, B.ghosth, B.ghostb, (T*)B.ht,
        (T*)B.bt, cell_out(m, B));
  };
  if constexpr (sizeof(T) == 4) {
    if (B.ghosth) return run(std::true_type{});
  }
  run(std::false_type{});
}
}  // namespace

hipError_t launch_step_wide(int D, int prec, const DevMesh& m, const FusedMesh& fm, const DevVel& v,
                            const GasP& g, const SweepSched& sc, const StepBuffers& B, hipStream_t s) {
  if (sc.lanes % 64 != 0 || sc.lanes < 64 || sc.lanes > CELLT) return hipErrorInvalidValue;
  if (D == 2) UGKS_DISPATCH_T(prec, (launch_wide_as<2, TT, true>(m, fm, v, g, sc, B, s)));
  else if (B.b) UGKS_DISPATCH_T(prec, (launch_wide_as<3, TT, true>(m, fm, v, g, sc, B, s)));
  else UGKS_DISPATCH_T(prec, (launch_wide_as<3, TT, false>(m, fm, v, g, sc, B, s)));
  return hipGetLastError();
}

namespace {
template <int D, typename T, bool HB>
void launch_face_flux_as(const DevMesh& m, const FusedMesh& fm, const DevVel& v, const GasP& g,
                         const StepBuffers& B, hipStream_t s) {
  auto run = [&](auto gh) {
    k_face_flux<D, T, HB, decltype(gh)::value><<<face_grid(m), SWT, 0, s>>>(
        m, sweep_in<double>(fm, v, g, B), fm.frow, (const T*)B.h, (const T*)B.b, B.gradh, B.gradb, B.ghosth,
        B.ghostb, B.F, B.flag);
  };
  if constexpr (sizeof(T) == 4) {
    if (B.ghosth) return run(std::true_type{});
  }
  run(std::false_type{});
}
}  // namespace

hipError_t launch_face_flux(int D, int prec, const DevMesh& m, const FusedMesh& fm, const DevVel& v,
                            const GasP& g, const StepBuffers& B, hipStream_t s) {
  if (D == 2) UGKS_DISPATCH_T(prec, (launch_face_flux_as<2, TT, true>(m, fm, v, g, B, s)));
  else if (B.b) UGKS_DISPATCH_T(prec, (launch_face_flux_as<3, TT, true>(m, fm, v, g, B, s)));
  else UGKS_DISPATCH_T(prec, (launch_face_flux_as<3, TT, false>(m, fm, v, g, B, s)));
  return hipGetLastError();
}

hipError_t launch_wall_rho_inline(int D, int prec, const DevMesh& m, const DevVel& v,
                                  const FusedMesh& fm, const GasP& g, void* h, void* b, double* frec,
                                  const int32_t* flag, hipStream_t s, bool track, bool ghosts) {
  if (m.nwall == 0) return hipSuccess;
  const unsigned grid = (unsigned)(m.nwall + (ghosts ? fm.nff : 0));
#define UGKS_WALL(LIM, BF)                                                            \
  UGKS_DISPATCH_DT(D, prec, (k_wall_rho_inline<DD, TT, LIM, BF><<<grid, WALLT, 0, s>>>( \
                                m, v, fm, g, (TT*)h, (TT*)b, frec, flag)))
  if (track && fm.crec_l) UGKS_WALL(true, true);
  else if (track) UGKS_WALL(false, true);
  else if (fm.crec_l) UGKS_WALL(true, false);
  else UGKS_WALL(false, false);
#undef UGKS_WALL
  return hipGetLastError();
}

// The step's boundary flux, added to the running sum acc[0..D+1]: the sum
// over boundary faces of S_f F_f, from the wall records' fluxes (fused path,
// FR_BF) or from the face fluxes (staged path, every boundary face).  One
// work-group; each lane adds its faces in order, then a fixed reduction.  Run
// after the rest of the step, so that a failed step's flux is left out.
template <int D>
__global__ __launch_bounds__(256) void k_bflux(DevMesh m, const double* __restrict__ frec,
                                               const double* __restrict__ F, int staged,
                                               double* __restrict__ acc, const int32_t* flag) {
  __shared__ double red[5 * 16];
  if (flag[0] | flag[2]) return;
  double s[D + 2];
  for (int x = 0; x < D + 2; ++x) s[x] = 0.0;
  if (staged) {
    for (int64_t f = threadIdx.x; f < m.nf; f += 256)
      if (m.fR[f] < 0)
        for (int x = 0; x < D + 2; ++x) s[x] += m.farea[f] * F[f * 5 + x];
  } else {
    for (int64_t wi = threadIdx.x; wi < m.nwall; wi += 256) {
      const int64_t f = m.walls[wi];
      for (int x = 0; x < D + 2; ++x) s[x] += m.farea[f] * frec[f * FREC + FR_BF + x];
    }
  }
  block_sum<D + 2>(s, red);
  if (threadIdx.x == 0)
    for (int x = 0; x < D + 2; ++x) acc[x] += s[x];
}

hipError_t launch_bflux(int D, const DevMesh& m, const double* frec, const double* F, int staged,
                        double* acc, const int32_t* flag, hipStream_t s) {
  UGKS_DISPATCH_D(D, k_bflux<DD><<<1, 256, 0, s>>>(m, frec, F, staged, acc, flag));
  return hipGetLastError();
}

// ---- batched launchers ------------------------------------------------------
hipError_t launch_cell_prep_b(int D, int prec, const BatchDev& bd, int64_t ncell, hipStream_t s) {
  if (ncell == 0) return hipSuccess;
  const unsigned grid = (unsigned)((ncell + 127) / 128);
  UGKS_DISPATCH_DT(D, prec, k_cell_prep_b<DD, TT><<<grid, 128, 0, s>>>(bd));
  return hipGetLastError();
}

hipError_t launch_wall_rho_b(int D, int prec, const BatchDev& bd, int64_t nwall, hipStream_t s) {
  if (nwall == 0) return hipSuccess;
  UGKS_DISPATCH_DT(D, prec, k_wall_rho_b<DD, TT><<<(unsigned)nwall, WALLT, 0, s>>>(bd));
  return hipGetLastError();
}

hipError_t launch_ghost_rows(int D, int prec, const FusedMesh& fm, const DevVel& v,
                             const double* frec, int64_t first, void* h, void* b, const int32_t* flag,
                             hipStream_t s) {
  if (fm.nff == 0) return hipSuccess;
  UGKS_DISPATCH_DT(D, prec, k_ghost_rows<DD, TT><<<(unsigned)fm.nff, SWT, 0, s>>>(
      first, fm.ffaces, v, frec, (TT*)h, (TT*)b, flag));
  return hipGetLastError();
}

hipError_t launch_ghost_rows_b(int D, int prec, const BatchDev& bd, int64_t nff, hipStream_t s) {
  if (nff == 0) return hipSuccess;
  UGKS_DISPATCH_DT(D, prec, k_ghost_rows_b<DD, TT><<<(unsigned)nff, SWT, 0, s>>>(bd));
  return hipGetLastError();
}

hipError_t launch_step_b(int D, int prec, const BatchDev& bd, int64_t grid, int threads,
                         hipStream_t s) {
  if (bd.nitems == 0) return hipSuccess;
  if (threads % 64 != 0 || threads < 64 || threads > SWT) return hipErrorInvalidValue;
  UGKS_DISPATCH_DT(D, prec, k_step_b<DD, TT><<<(unsigned)grid, threads, 0, s>>>(bd));
  return hipGetLastError();
}

hipError_t launch_sweep_b(int D, int prec, const BatchDev& bd, int64_t ncell, int64_t grid, int threads,
                          hipStream_t s) {
  if (bd.nitems == 0) return hipSuccess;
  if (threads % 64 != 0 || threads < 64 || threads > SWT) return hipErrorInvalidValue;
  UGKS_DISPATCH_DT(D, prec, k_sweep_b<DD, TT><<<(unsigned)grid, threads, 0, s>>>(bd));
  UGKS_DISPATCH_DT(D, prec, k_finish_b<DD, TT><<<(unsigned)ncell, SWT, 0, s>>>(bd));
  return hipGetLastError();
}

int batch_blocks_per_cu(int D, int prec, int threads, bool blocks) {
  int n = 0;
  hipError_t e = hipSuccess;
  UGKS_DISPATCH_DT(D, prec, e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
                                &n, blocks ? reinterpret_cast<const void*>(&k_sweep_b<DD, TT>)
                                           : reinterpret_cast<const void*>(&k_step_b<DD, TT>), threads, 0));
  return e == hipSuccess ? n : 0;
}

}  // namespace ugks
