// gfx950 kernels of the UGKS phase-space step (staged form).
//
// Each kernel is one numbered part of the one-step algorithm (Sec. 2.2) for
// the BGK-Shakhov model of Sec. 2.1.  Velocity is the fast (lane) index:
// h is stored [cell][k] with k contiguous, so every per-(cell, velocity)
// kernel issues coalesced 64-lane loads and stores, and every per-face or
// per-cell quantity (geometry, interface coefficients) is wave-uniform.
// Sums over velocity use wave shuffles plus LDS in a fixed order, so the
// results are deterministic.
#include "ugks_device.h"

namespace ugks {

using namespace dev;

namespace {

// ---------------------------------------------------------------------------
// (a null flag: a readout, which raises no error)
template <int D>
__global__ void k_prims(int64_t nc, GasP g, const double* __restrict__ W, double* __restrict__ prim,
                        int32_t* flag, int check) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= nc) return;
  if (check && *flag) return;
  bool ok = prim_of<D>(&W[i * (D + 2)], g, &prim[i * NPRIM]);
  if (!ok && flag) atomicOr(flag, 1);
}

// Heat flux q_i = 1/2 sum_k w_k c_k (|c_k|^2 h_ik + b_ik), c = u - U_i.
template <int D, typename T>
__global__ __launch_bounds__(TPB) void k_heatflux(DevVel v, const T* __restrict__ h,
                                                  const T* __restrict__ b,
                                                  const double* __restrict__ prim,
                                                  double* __restrict__ q, const int32_t* flag) {
  __shared__ double lds[3 * 16];
  if (*flag) return;
  const int64_t i = blockIdx.x;
  const double* P = &prim[i * NPRIM];
  double acc[3] = {0.0, 0.0, 0.0};
  for (int64_t k = threadIdx.x; k < v.nvp; k += TPB) {
    double c[3], c2 = 0.0;
    for (int d = 0; d < D; ++d) {
      c[d] = v.u[d * v.nvp + k] - P[1 + d];
      c2 += c[d] * c[d];
    }
    double hv = ld(h, i * v.nvp + k);
    double bv = v.has_b ? ld(b, i * v.nvp + k) : 0.0;
    double s = v.w[k] * (c2 * hv + bv);
    for (int d = 0; d < D; ++d) acc[d] += s * c[d];
  }
  block_sum<3>(acc, lds);
  if (threadIdx.x == 0) {
    for (int d = 0; d < 3; ++d) q[i * 3 + d] = d < D ? 0.5 * acc[d] : 0.0;
  }
}

// Venkatakrishnan's limiter factor of one cell field (Sec. 2.1 reconstruction
// with an optional limiter): vi is the cell's value, [vmin, vmax] the range
// of the cell and its stencil values, g its least-squares gradient.  At each
// face d- = g.(x_f - x_i) and d+ the room left toward the bound on its side;
// psi = (d+^2 + eps^2 + 2 d- d+) / (d+^2 + 2 d-^2 + d- d+ + eps^2); the
// factor is min(1, min_faces psi).  d+ is one value per side and min(1, psi)
// falls as |d-| grows, so the largest and the smallest d- decide.
__device__ __forceinline__ double venkat_of(double vi, double vmin, double vmax, double dmax, double dmin,
                                            double eps2) {
  // (fmin drops the 0 / 0 of a side without slope or room)
  auto psi = [eps2](double dp, double dm) {
    return (dp * dp + eps2 + 2.0 * dm * dp) / (dp * dp + 2.0 * dm * dm + dm * dp + eps2);
  };
  return fmin(fmin(1.0, psi(vmax - vi, dmax)), psi(vmin - vi, dmin));
}

template <int D>
__device__ __forceinline__ double venkat_phi(const DevMesh& m, int64_t i, int nfc, double vi,
                                             double vmin, double vmax, const double* g) {
  double dmax = 0.0, dmin = 0.0;
  for (int p = 0; p < nfc; ++p) {
    const int f = m.cface[i * MAXF + p];
    const double* dx = m.csign[i * MAXF + p] > 0.0 ? &m.fdxL[f * 3] : &m.fdxR[f * 3];
    double dm = 0.0;
    for (int d = 0; d < D; ++d) dm += g[d] * dx[d];
    dmax = fmax(dmax, dm);
    dmin = fmin(dmin, dm);
  }
  return venkat_of(vi, vmin, vmax, dmax, dmin, m.veps2[i]);
}

// Macroscopic least-squares gradients of W (step 4), one lane per (cell,
// component).  A chain of dependent loads bounds it, so each kind is issued
// together: ids, neighbours, coefficients, offsets; slots past the cell's faces
// (NF per cell here, those of the mesh's largest cell or more) repeat its own
// value, with coefficient 0.  With the limiter 960 cells took 13.4 us with one
// lane per cell and face by face, 7.1 so; 48,000 tets without it 14.3 and 10.6.
template <int D, int NF>
__device__ __forceinline__ void gradW_at(int64_t t, const DevMesh& m, const DevBC* __restrict__ bcs,
                                         const GasP& g, const double* __restrict__ W,
                                         double* __restrict__ gW, int32_t* flag, int count) {
  constexpr int NV = D + 2;
  // the first kernel of a step (count): takes over the error of the step before,
  // and counts the steps begun without one (a failed step's results are dropped)
  if (count) {
    const bool bad = flag[0] | flag[2];
    if (t == 0) {
      if (bad) flag[0] = 1;
      else flag[1] += 1;
    }
    if (bad) return;
  }
  const int64_t i = t / NV;
  const int v = (int)(t % NV);
  const int nfc = m.nfc[i];
  int nbr[NF], face[NF];
#pragma unroll
  for (int p = 0; p < NF; ++p) {
    nbr[p] = m.cnbr[i * MAXF + p];
    face[p] = m.cface[i * MAXF + (p < nfc ? p : 0)];
  }
  const double wi = W[i * NV + v];
  double nb[NF];
#pragma unroll
  for (int p = 0; p < NF; ++p) nb[p] = W[(nbr[p] >= 0 ? (int64_t)nbr[p] : i) * NV + v];
#pragma unroll
  for (int p = 0; p < NF; ++p)
    if (p < nfc && nbr[p] < 0 && m.fbc[face[p]] != UGKS_BC_WALL) {  // (a wall's ghost is the cell itself)
      double Wi[5], Wg[5];
      for (int x = 0; x < NV; ++x) Wi[x] = W[i * NV + x];
      ghost_state<D>(m.fbc[face[p]], bcs[m.fbcid[face[p]]], &m.fnorm[(int64_t)face[p] * 3], Wi, g.R, g.K, Wg);
      for (int x = 0; x < NV; ++x)
        if (x == v) nb[p] = Wg[x];
    }
  double gr[D], lo = wi, hi = wi;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    gr[d] = 0.0;
#pragma unroll
    for (int p = 0; p < NF; ++p) gr[d] += m.lsG[(i * 3 + d) * MAXF + p] * (nb[p] - wi);
  }
  if (m.limiter) {
    double dmax = 0.0, dmin = 0.0;
#pragma unroll
    for (int p = 0; p < NF; ++p) {
      lo = fmin(lo, nb[p]);
      hi = fmax(hi, nb[p]);
      const double* dx = (m.csign[i * MAXF + (p < nfc ? p : 0)] > 0.0 ? m.fdxL : m.fdxR) + (int64_t)face[p] * 3;
      double dm = 0.0;
#pragma unroll
      for (int d = 0; d < D; ++d) dm += gr[d] * dx[d];
      dmax = fmax(dmax, dm);
      dmin = fmin(dmin, dm);
    }
    const double phi = venkat_of(wi, lo, hi, dmax, dmin, m.veps2[i]);
#pragma unroll
    for (int d = 0; d < D; ++d) gr[d] *= phi;
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    gW[(i * 3 + d) * 5 + v] = d < D ? gr[d < D ? d : 0] : 0.0;
    if (v == NV - 1)
      for (int x = NV; x < 5; ++x) gW[(i * 3 + d) * 5 + x] = 0.0;
  }
}

template <int D, int NF>
__global__ __launch_bounds__(128) void k_gradW(DevMesh m, const DevBC* __restrict__ bcs, GasP g, const double* __restrict__ W,
                        double* __restrict__ gW, int32_t* flag, int count) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t < m.nc * (D + 2)) gradW_at<D, NF>(t, m, bcs, g, W, gW, flag, count);
}

template <int D, typename T>
__device__ __forceinline__ void face_eq_at(int64_t f, const DevMesh& m, const DevBC* __restrict__ bcs,
                                           const GasP& g, const double* __restrict__ W,
                                           const double* __restrict__ gW,
                                           const double* __restrict__ q, double* __restrict__ frec,
                                           int nr, T* __restrict__ srec, int32_t* flag) {
  if (*flag) return;
  double* R = &frec[f * FREC];
  T* S = srec ? &srec[f * nr * SREC] : nullptr;
  const int kind = m.fbc[f];
  const int L = m.fL[f];
  if (kind == UGKS_BC_WALL) {
    const DevBC& bc = bcs[m.fbcid[f]];
    double lamw = 1.0 / (2.0 * g.R * bc.T);
    R[FR_C0] = maxw_norm<D>(lamw);
    R[FR_LAM] = lamw;
    for (int d = 0; d < 3; ++d) R[FR_U + d] = d < D ? bc.U[d] : 0.0;
    // free transport of the incident member over the step (h_f - t u.grad h),
    // and the re-emitted Maxwellian as g(u) times a constant polynomial
    if (S) {
      double P[Cubic<D>::N];
      for (int x = 0; x < Cubic<D>::N; ++x) P[x] = 0.0;
      P[0] = 1.0;
      write_srec<D>(S, g.dt, -0.5 * g.dt * g.dt, P);
      P[0] = (g.K + 3.0 - D) / (2.0 * lamw);
      if (nr == 2) write_srec<D>(S + SREC, g.dt, -0.5 * g.dt * g.dt, P);
    }
    return;
  }
  const bool ghost = kind != UGKS_BC_INTERIOR;
  const int Rc = ghost ? -1 : m.fR[f];
  // everything the face reads, loaded together (a ghost side: the cell's, unused)
  const int Rl = ghost ? L : Rc;
  double n[3], wl[5], wr[5], gl[3][5], gr[3][5], dl[3], dr[3], ql[3], qr[3];
  for (int d = 0; d < 3; ++d) {
    n[d] = m.fnorm[f * 3 + d];
    dl[d] = m.fdxL[f * 3 + d];
    dr[d] = m.fdxR[f * 3 + d];
    ql[d] = q[(int64_t)L * 3 + d];
    qr[d] = ghost ? 0.0 : q[(int64_t)Rl * 3 + d];
  }
  for (int v = 0; v < D + 2; ++v) {
    wl[v] = W[(int64_t)L * (D + 2) + v];
    wr[v] = W[(int64_t)Rl * (D + 2) + v];
    for (int d = 0; d < D; ++d) {
      gl[d][v] = gW[((int64_t)L * 3 + d) * 5 + v];
      gr[d][v] = gW[((int64_t)Rl * 3 + d) * 5 + v];
    }
  }
  double Wg[5];
  if (ghost) {
    ghost_state<D>(kind, bcs[m.fbcid[f]], n, wl, g.R, g.K, Wg);
    double Pg[NPRIM];
    prim_of<D>(Wg, g, Pg);
    R[FR_GRHO] = Pg[0];
    for (int d = 0; d < 3; ++d) R[FR_GU + d] = Pg[1 + d];
    R[FR_GLAM] = Pg[4];
    R[FR_GC] = Pg[0] * maxw_norm<D>(Pg[4]);
  }
  // 6.1 reconstructed states on both sides
  double Wl[5], Wr[5];
  for (int v = 0; v < D + 2; ++v) {
    double sl = wl[v], sr = wr[v];
    for (int d = 0; d < D; ++d) {
      sl += dl[d] * gl[d][v];
      sr += dr[d] * gr[d][v];
    }
    Wl[v] = sl;
    Wr[v] = ghost ? Wg[v] : sr;
  }
  double Pl[NPRIM], Pr[NPRIM];
  if (!prim_of<D>(Wl, g, Pl)) {
    for (int v = 0; v < D + 2; ++v) Wl[v] = wl[v];
    prim_of<D>(Wl, g, Pl);
  }
  if (!prim_of<D>(Wr, g, Pr)) {
    for (int v = 0; v < D + 2; ++v) Wr[v] = ghost ? Wg[v] : wr[v];
    prim_of<D>(Wr, g, Pr);
  }
  // 6.2 interface state from the two half-range Maxwellians
  double W0[5] = {0, 0, 0, 0, 0};
  const double* Ps[2] = {Pl, Pr};
  for (int s = 0; s < 2; ++s) {
    const double* P = Ps[s];
    double rho = P[0], lam = P[4];
    double Un = 0.0;
    for (int d = 0; d < D; ++d) Un += P[1 + d] * n[d];
    double Ut2 = 0.0, Ut[3];
    for (int d = 0; d < D; ++d) {
      Ut[d] = P[1 + d] - Un * n[d];
      Ut2 += Ut[d] * Ut[d];
    }
    double mo[3];
    half_range(Un, lam, s == 0 ? 1.0 : -1.0, mo);
    W0[0] += rho * mo[0];
    for (int d = 0; d < D; ++d) W0[1 + d] += rho * (mo[1] * n[d] + mo[0] * Ut[d]);
    W0[D + 1] += 0.5 * rho * (mo[2] + mo[0] * (Ut2 + (g.K + 2.0) / (2.0 * lam)));
  }
  // 6.3 interface primitives, relaxation time and time coefficients
  double P0[NPRIM];
  if (!prim_of<D>(W0, g, P0)) {
    atomicOr(flag, 2);
    return;
  }
  const double rho0 = P0[0], lam0 = P0[4];
  double U0[3] = {P0[1], P0[2], P0[3]};
  R[FR_C0] = rho0 * maxw_norm<D>(lam0);
  R[FR_LAM] = lam0;
  for (int d = 0; d < 3; ++d) R[FR_U + d] = U0[d];
  const double sh = 4.0 * (1.0 - g.Pr) * lam0 * lam0 / ((g.K + 5.0) * rho0);
  const double kxi = g.K + 3.0 - D;
  double G[5];
  time_coeffs(g.dt, P0[5], G);
  // 6.4 spatial slopes from the averaged gradient
  double a[3][5];
  for (int d = 0; d < 3; ++d)
    for (int v = 0; v < 5; ++v) a[d][v] = 0.0;
  for (int d = 0; d < D; ++d) {
    double bvec[5];
    for (int v = 0; v < D + 2; ++v) bvec[v] = 0.5 * (gl[d][v] + (ghost ? 0.0 : gr[d][v])) / rho0;
    slope_solve<D>(bvec, U0, lam0, g.K + 3.0, a[d]);
  }
  // 6.5 time slope from compatibility
  Moments<D> M;
  M.init(U0, lam0, kxi);
  double r[5], At[5];
  time_slope_rhs<D>(M, a, r);
  slope_solve<D>(r, U0, lam0, g.K + 3.0, At);
  // 6.6 interface heat flux
  double q0[3] = {0.0, 0.0, 0.0};
  for (int d = 0; d < 3; ++d) {
    q0[d] = d < D ? 0.5 * (ql[d] + qr[d]) : 0.0;
  }
  if (!S) {  // the staged path evaluates the terms one by one
    R[FR_SH] = sh;
    for (int x = 0; x < 5; ++x) R[FR_G + x] = G[x];
    for (int d = 0; d < 3; ++d) R[FR_Q + d] = q0[d];
    for (int d = 0; d < 3; ++d)
      for (int v = 0; v < 5; ++v) R[FR_A + d * 5 + v] = (d < D && v < D + 2) ? a[d][v] : 0.0;
    for (int v = 0; v < 5; ++v) R[FR_AT + v] = v < D + 2 ? At[v] : 0.0;
    return;
  }
  // All equilibrium terms of the time-integrated interface distribution,
  //   Gamma3 (g0 + g0+) + Gamma4 u.grad g0 + Gamma5 d_t g0,
  // equal g0(u) times a cubic polynomial in u: PH for h, PB for b.
  {
    using Cb = Cubic<D>;
    double PH[Cb::N], PB[Cb::N];
    for (int x = 0; x < Cb::N; ++x) PH[x] = PB[x] = 0.0;
    const double kap = kxi / (2.0 * lam0);                             // B0 / H0
    const double xi4 = kxi * (kxi + 2.0) / (4.0 * lam0 * lam0);       // int xi^4 g / H0
    const double G3 = G[2], G4 = G[3], G5 = G[4];
    double a0v[3], a4v[3], Am[9], Atl[3];
    for (int d = 0; d < D; ++d) {
      a0v[d] = a[d][0];
      a4v[d] = a[d][D + 1];
      Atl[d] = At[1 + d];
      for (int e = 0; e < D; ++e) Am[d * 3 + e] = a[d][1 + e];
    }
    // Gamma3 (1 + H0+/H0)
    Cb::add_const(PH, G3);
    Cb::add_shakhov(PH, G3 * sh, U0, q0, lam0, 2.0 + D);
    // Gamma4 sum_d u_d (P_d + a_d4 kap / 2), P_d = a_d0 + a_d.u + a_d4 |u|^2 / 2
    Cb::add_lin(PH, G4, a0v);
    Cb::add_mat(PH, G4, Am, 3);
    Cb::add_lin_u2(PH, 0.5 * G4, a4v);
    Cb::add_lin(PH, 0.5 * G4 * kap, a4v);
    // Gamma5 (P_A + A4 kap / 2)
    Cb::add_const(PH, G5 * (At[0] + 0.5 * At[D + 1] * kap));
    Cb::add_lin(PH, G5, Atl);
    Cb::add_u2(PH, 0.5 * G5 * At[D + 1]);
    if (kxi > 0.0) {
      Cb::add_const(PB, G3 * kap);
      Cb::add_shakhov(PB, G3 * sh * kap, U0, q0, lam0, (double)D);
      Cb::add_lin(PB, G4 * kap, a0v);
      Cb::add_mat(PB, G4 * kap, Am, 3);
      Cb::add_lin_u2(PB, 0.5 * G4 * kap, a4v);
      Cb::add_lin(PB, 0.5 * G4 * xi4, a4v);
      Cb::add_const(PB, G5 * (kap * At[0] + 0.5 * At[D + 1] * xi4));
      Cb::add_lin(PB, G5 * kap, Atl);
      Cb::add_u2(PB, 0.5 * G5 * kap * At[D + 1]);
    }
    write_srec<D>(S, G[0], G[1], PH);
    if (nr == 2) write_srec<D>(S + SREC, G[0], G[1], PB);
  }
}

// One lane per face, a long serial chain: its reads are issued together and the
// launch bound leaves it the registers that it needs (95,520 faces of tets 33.5
// us spilling, 27 so; 2,112 of quads 13.2 and 12.0).
template <int D, typename T>
__global__ __launch_bounds__(64) void k_face_eq(DevMesh m, const DevBC* __restrict__ bcs, GasP g,
                          const double* __restrict__ W, const double* __restrict__ gW,
                          const double* __restrict__ q, double* __restrict__ frec,
                          int nr, T* __restrict__ srec, int32_t* flag) {
  const int64_t f = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (f < m.nf) face_eq_at<D, T>(f, m, bcs, g, W, gW, q, frec, nr, srec, flag);
}

// Microscopic gradients of h (and b) for every (cell, velocity) (step 5).
// Bound by the three gradients it writes and by the neighbour rows it reads.
// A lane takes two adjacent velocities (16-byte accesses) and issues all of its
// neighbour rows before any arithmetic; the work-groups of one XCD take
// GRAD_TILE cells through one block of velocities, then the next, so that the
// rows the cells share are read from HBM once.  Gradients that the last-level cache
// cannot hold bypass the caches, which are left to the rows.  4,096 hexahedra x
// 20^3, FP64: 0.50 ms with one velocity per lane in cell order, 0.35 (3.0 TB/s) so;
// plain stores 0.355 and the wall pass that follows 0.084 instead of 0.065.  Smaller
// ones stay: 27 x 48^3 (72 MB) 0.41 for the wall pass bypassing, 0.33 plain.
constexpr int64_t GRAD_TILE = 32;
constexpr int64_t kLastLevel = 256 << 20;  // bytes

// (NT: a template argument, as a branch over the two kinds of store becomes one plain one)
template <int D, typename T, bool NT>
__global__ __launch_bounds__(TPB) void k_grad_micro(DevMesh m, DevVel v,
                                                    const double* __restrict__ frec,
                                                    const T* __restrict__ h, const T* __restrict__ b,
                                                    double* __restrict__ gh, double* __restrict__ gb,
                                                    const int32_t* flag) {
  typedef T pair_t __attribute__((ext_vector_type(2)));
  typedef double dpair_t __attribute__((ext_vector_type(2)));
  const int64_t nvp = v.nvp, nch = (nvp + 2 * TPB - 1) / (2 * TPB);
  const uint32_t xcd = blockIdx.x % 8, local = blockIdx.x / 8;
  uint32_t tile = 0, rem = local, run = GRAD_TILE;
  if (m.nc >= 8 * GRAD_TILE) {
    const uint32_t per_tile = (uint32_t)nch * GRAD_TILE;
    tile = local / per_tile;
    rem = local - tile * per_tile;
  } else {
    run = (uint32_t)xcd_run(m.nc, GRAD_TILE);
  }
  const int64_t i = (int64_t)(tile * 8 + xcd) * run + rem % run;
  const int64_t k = 2 * ((int64_t)(rem / run) * TPB + threadIdx.x);  // nvp is even
  if (i >= m.nc || k >= nvp || *flag) return;
  const int nfc = m.nfc[i];
  for (int r = 0; r < (v.has_b ? 2 : 1); ++r) {
    const T* __restrict__ f = r ? b : h;
    const pair_t fi = *(const pair_t*)&f[i * nvp + k];
    pair_t fn[MAXF];
#pragma unroll
    for (int p = 0; p < MAXF; ++p) {
      fn[p] = fi;
      if (p < nfc) {
        const int j = m.cnbr[i * MAXF + p];
        if (j >= 0) fn[p] = *(const pair_t*)&f[(int64_t)j * nvp + k];
      }
    }
    double a[2][3] = {{0, 0, 0}, {0, 0, 0}}, lo[2], hi[2], vi[2];
    for (int e = 0; e < 2; ++e) lo[e] = hi[e] = vi[e] = (double)fi[e];
#pragma unroll
    for (int p = 0; p < MAXF; ++p)
      if (p < nfc) {
        double x[2] = {(double)fn[p][0], (double)fn[p][1]};
        if (m.cnbr[i * MAXF + p] < 0) {
          const int fc = m.cface[i * MAXF + p];
          if (m.fbc[fc] != UGKS_BC_WALL) {  // (a wall's ghost value is the cell's own)
            const double* R = &frec[(int64_t)fc * FREC];
            for (int e = 0; e < 2; ++e) {
              double c2 = 0.0;
              for (int d = 0; d < D; ++d) {
                const double c = v.u[d * nvp + k + e] - R[FR_GU + d];
                c2 += c * c;
              }
              x[e] = R[FR_GC] * exp(-R[FR_GLAM] * c2);
              if (r) x[e] *= v.kxi / (2.0 * R[FR_GLAM]);
            }
          }
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          lo[e] = fmin(lo[e], x[e]);
          hi[e] = fmax(hi[e], x[e]);
          for (int d = 0; d < D; ++d) a[e][d] += m.lsG[(i * 3 + d) * MAXF + p] * (x[e] - vi[e]);
        }
      }
    if (m.limiter)
      for (int e = 0; e < 2; ++e) {
        const double ph = venkat_phi<D>(m, i, nfc, vi[e], lo[e], hi[e], a[e]);
        for (int d = 0; d < D; ++d) a[e][d] *= ph;
      }
    double* __restrict__ g = r ? gb : gh;
    for (int d = 0; d < D; ++d) {
      const dpair_t o = {a[0][d], a[1][d]};
      if constexpr (NT) __builtin_nontemporal_store(o, (dpair_t*)&g[(i * 3 + d) * nvp + k]);
      else *(dpair_t*)&g[(i * 3 + d) * nvp + k] = o;
    }
  }
}

// Wall density from the zero normal mass flux condition (step 7).
template <int D, typename T>
__global__ __launch_bounds__(TPB) void k_wall_rho(DevMesh m, DevVel v, GasP g,
                                                  const T* __restrict__ h,
                                                  const double* __restrict__ gh,
                                                  double* __restrict__ frec, const int32_t* flag) {
  __shared__ double lds[2 * 16];
  if (*flag) return;
  const int f = m.walls[blockIdx.x];
  const int L = m.fL[f];
  const int64_t nvp = v.nvp;
  double* R = &frec[(int64_t)f * FREC];
  const double lamw = R[FR_LAM], Cw = R[FR_C0];
  const double dt = g.dt;
  double acc[2] = {0.0, 0.0};
  for (int64_t k = threadIdx.x; k < nvp; k += TPB) {
    double un = 0.0;
    for (int d = 0; d < D; ++d) un += v.u[d * nvp + k] * m.fnorm[f * 3 + d];
    if (un > 0.0) {
      double hf = ld(h, (int64_t)L * nvp + k), ugh = 0.0;
      for (int d = 0; d < D; ++d) {
        double gd = gh[((int64_t)L * 3 + d) * nvp + k];
        hf += m.fdxL[f * 3 + d] * gd;
        ugh += v.u[d * nvp + k] * gd;
      }
      acc[0] += v.w[k] * un * (dt * hf - 0.5 * dt * dt * ugh);
    } else if (un < 0.0) {
      double c2 = 0.0;
      for (int d = 0; d < D; ++d) {
        double c = v.u[d * nvp + k] - R[FR_U + d];
        c2 += c * c;
      }
      acc[1] += v.w[k] * un * Cw * exp(-lamw * c2);
    }
  }
  block_sum<2>(acc, lds);
  if (threadIdx.x == 0) R[FR_RHOW] = -acc[0] / (dt * acc[1]);
}

// Time-integrated microscopic flux of one (face, velocity) (steps 6.7, 7).
template <int D, typename T>
__device__ __forceinline__ void face_flux(const DevMesh& m, const DevVel& v, const GasP& g,
                                          const double* R, int64_t f, int64_t k,
                                          const T* __restrict__ h, const T* __restrict__ b,
                                          const double* __restrict__ gh,
                                          const double* __restrict__ gb, double& FH, double& FB) {
  const int64_t nvp = v.nvp;
  const int kind = m.fbc[f];
  const int L = m.fL[f];
  double uk[3] = {0, 0, 0};
  double un = 0.0;
  for (int d = 0; d < D; ++d) {
    uk[d] = v.u[d * nvp + k];
    un += uk[d] * m.fnorm[f * 3 + d];
  }
  const double dt = g.dt;
  const double KXI = v.kxi;
  const bool hb = v.has_b;
  double ih = 0.0, ib = 0.0;
  if (kind == UGKS_BC_WALL) {
    if (un > 0.0) {
      double hf = ld(h, (int64_t)L * nvp + k), bf = hb ? ld(b, (int64_t)L * nvp + k) : 0.0;
      double ugh = 0.0, ugb = 0.0;
      for (int d = 0; d < D; ++d) {
        double gd = gh[((int64_t)L * 3 + d) * nvp + k];
        hf += m.fdxL[f * 3 + d] * gd;
        ugh += uk[d] * gd;
        if (hb) {
          double gbd = gb[((int64_t)L * 3 + d) * nvp + k];
          bf += m.fdxL[f * 3 + d] * gbd;
          ugb += uk[d] * gbd;
        }
      }
      ih = dt * hf - 0.5 * dt * dt * ugh;
      ib = dt * bf - 0.5 * dt * dt * ugb;
    } else if (un < 0.0) {
      double c2 = 0.0;
      for (int d = 0; d < D; ++d) {
        double c = uk[d] - R[FR_U + d];
        c2 += c * c;
      }
      double Hw = R[FR_C0] * exp(-R[FR_LAM] * c2);
      ih = dt * R[FR_RHOW] * Hw;
      ib = dt * R[FR_RHOW] * KXI / (2.0 * R[FR_LAM]) * Hw;
    }
    FH = un * ih;
    FB = un * ib;
    return;
  }
  const bool ghost = kind != UGKS_BC_INTERIOR;
  double hf, bf = 0.0, ugh = 0.0, ugb = 0.0;
  if (un <= 0.0 && ghost) {
    double c2 = 0.0;
    for (int d = 0; d < D; ++d) {
      double c = uk[d] - R[FR_GU + d];
      c2 += c * c;
    }
    hf = R[FR_GC] * exp(-R[FR_GLAM] * c2);
    bf = KXI / (2.0 * R[FR_GLAM]) * hf;
  } else {
    const bool left = un > 0.0;
    const int64_t up = left ? L : m.fR[f];
    const double* dx = left ? &m.fdxL[f * 3] : &m.fdxR[f * 3];
    hf = ld(h, up * nvp + k);
    if (hb) bf = ld(b, up * nvp + k);
    for (int d = 0; d < D; ++d) {
      double gd = gh[(up * 3 + d) * nvp + k];
      hf += dx[d] * gd;
      ugh += uk[d] * gd;
      if (hb) {
        double gbd = gb[(up * 3 + d) * nvp + k];
        bf += dx[d] * gbd;
        ugb += uk[d] * gbd;
      }
    }
  }
  // interface equilibrium, its Shakhov correction and derivative terms
  const double lam0 = R[FR_LAM];
  double c2 = 0.0, cq = 0.0, u2 = v.u2[k];
  for (int d = 0; d < D; ++d) {
    double c = uk[d] - R[FR_U + d];
    c2 += c * c;
    cq += c * R[FR_Q + d];
  }
  const double H0 = R[FR_C0] * exp(-lam0 * c2);
  const double B0 = KXI / (2.0 * lam0) * H0;
  const double sh = R[FR_SH] * cq;
  const double H0p = sh * (2.0 * lam0 * c2 - 2.0 - D) * H0;
  const double B0p = sh * (2.0 * lam0 * c2 - D) * KXI / (2.0 * lam0) * H0;
  const double xi4 = KXI * (KXI + 2.0) / (4.0 * lam0 * lam0);
  double uH = 0.0, uB = 0.0;
  for (int d = 0; d < D; ++d) {
    const double* ad = &R[FR_A + d * 5];
    double Pd = ad[0] + 0.5 * ad[D + 1] * u2;
    for (int c = 0; c < D; ++c) Pd += ad[1 + c] * uk[c];
    uH += uk[d] * (Pd * H0 + 0.5 * ad[D + 1] * B0);
    uB += uk[d] * (Pd * B0 + 0.5 * ad[D + 1] * xi4 * H0);
  }
  const double* At = &R[FR_AT];
  double PA = At[0] + 0.5 * At[D + 1] * u2;
  for (int c = 0; c < D; ++c) PA += At[1 + c] * uk[c];
  const double tH = PA * H0 + 0.5 * At[D + 1] * B0;
  const double tB = PA * B0 + 0.5 * At[D + 1] * xi4 * H0;
  const double* G = &R[FR_G];
  ih = G[0] * hf + G[1] * ugh + G[2] * (H0 + H0p) + G[3] * uH + G[4] * tH;
  ib = G[0] * bf + G[1] * ugb + G[2] * (B0 + B0p) + G[3] * uB + G[4] * tB;
  FH = un * ih;
  FB = un * ib;
}

// Microscopic fluxes of one face for every velocity, and the face's
// macroscopic flux F = sum_k w_k (H, u H, (|u|^2 H + B)/2) (Eq. macro_flux).
template <int D, typename T>
__global__ __launch_bounds__(TPB) void k_flux(DevMesh m, DevVel v, GasP g,
                                              const double* __restrict__ frec,
                                              const T* __restrict__ h, const T* __restrict__ b,
                                              const double* __restrict__ gh,
                                              const double* __restrict__ gb,
                                              double* __restrict__ fh, double* __restrict__ fb,
                                              double* __restrict__ F, const int32_t* flag) {
  __shared__ double lds[5 * 16];
  if (*flag) return;
  const int64_t f = face_of_block(m);
  if (f < 0) return;
  const double* R = &frec[f * FREC];
  const int64_t nvp = v.nvp;
  double acc[5] = {0, 0, 0, 0, 0};
  for (int64_t k = threadIdx.x; k < nvp; k += TPB) {
    double FH, FB;
    face_flux<D, T>(m, v, g, R, f, k, h, b, gh, gb, FH, FB);
    fh[f * nvp + k] = FH;
    if (v.has_b) fb[f * nvp + k] = FB;
    const double wk = v.w[k];
    acc[0] += wk * FH;
    for (int d = 0; d < D; ++d) acc[1 + d] += wk * v.u[d * nvp + k] * FH;
    acc[D + 1] += wk * 0.5 * (v.u2[k] * FH + FB);
  }
  block_sum<5>(acc, lds);
  if (threadIdx.x == 0)
    for (int x = 0; x < 5; ++x) F[f * 5 + x] = x < D + 2 ? acc[x] : 0.0;
}

// Reduced Maxwellian and Shakhov correction of a cell at one velocity.
template <int D>
__device__ __forceinline__ void cell_equilibrium(const double* P, const double* qv, const GasP& g,
                                                 const double* uk, double& Hs, double& Bs) {
  const double KXI = g.K + 3.0 - D, Pr = g.Pr;
  const double rho = P[0], lam = P[4];
  double c2 = 0.0, cq = 0.0;
  for (int d = 0; d < D; ++d) {
    double c = uk[d] - P[1 + d];
    c2 += c * c;
    cq += c * qv[d];
  }
  const double H = rho * maxw_norm<D>(lam) * exp(-lam * c2);
  const double pre = 4.0 * (1.0 - Pr) * lam * lam / ((g.K + 5.0) * rho) * cq;
  const double Hp = pre * (2.0 * lam * c2 - 2.0 - D) * H;
  const double Bp = pre * (2.0 * lam * c2 - D) * KXI / (2.0 * lam) * H;
  Hs = H + Hp;
  Bs = KXI / (2.0 * lam) * H + Bp;
}

// First stage (Eq. f_tilde).
template <int D, typename T>
__global__ __launch_bounds__(TPB) void k_stage1(DevMesh m, DevVel v, GasP g,
                                                const double* __restrict__ prim,
                                                const double* __restrict__ q,
                                                const T* __restrict__ h, const T* __restrict__ b,
                                                const double* __restrict__ fh,
                                                const double* __restrict__ fb, T* __restrict__ ht,
                                                T* __restrict__ bt, const int32_t* flag) {
  const int64_t nch = (v.nvp + TPB - 1) / TPB;
  const int64_t i = blockIdx.x / nch;
  const int64_t k = (blockIdx.x % nch) * TPB + threadIdx.x;
  if (k >= v.nvp || *flag) return;
  const int64_t nvp = v.nvp;
  double sh = 0.0, sb = 0.0;
  const int nfc = m.nfc[i];
  for (int p = 0; p < nfc; ++p) {
    const int64_t f = m.cface[i * MAXF + p];
    const double s = m.csign[i * MAXF + p] * area_for(g, i, m.farea[f]);
    sh += s * fh[f * nvp + k];
    if (v.has_b) sb += s * fb[f * nvp + k];
  }
  const double* P = &prim[i * NPRIM];
  double uk[3] = {0, 0, 0};
  for (int d = 0; d < D; ++d) uk[d] = v.u[d * nvp + k];
  double Hs, Bs;
  cell_equilibrium<D>(P, &q[i * 3], g, uk, Hs, Bs);
  const double c = dt_cell(g, i) / (2.0 * P[5]);
  const double iv = 1.0 / m.vol[i];
  const double hv = ld(h, i * nvp + k);
  st(ht, i * nvp + k, hv - sh * iv + c * (Hs - hv));
  if (v.has_b) {
    const double bv = ld(b, i * nvp + k);
    st(bt, i * nvp + k, bv - sb * iv + c * (Bs - bv));
  }
}

// Conservative update (Eq. macro_update) and per-cell residual parts.
template <int D>
__global__ void k_macro_update(DevMesh m, GasP g, const double* __restrict__ W, const double* __restrict__ F,
                               double* __restrict__ Wn, double* __restrict__ cellred,
                               const int32_t* flag) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= m.nc || *flag) return;
  double acc[5] = {0, 0, 0, 0, 0};
  const int nfc = m.nfc[i];
  for (int p = 0; p < nfc; ++p) {
    const int64_t f = m.cface[i * MAXF + p];
    const double s = m.csign[i * MAXF + p] * area_for(g, i, m.farea[f]);
    for (int x = 0; x < D + 2; ++x) acc[x] += s * F[f * 5 + x];
  }
  const double V = m.vol[i];
  for (int x = 0; x < D + 2; ++x) Wn[i * (D + 2) + x] = W[i * (D + 2) + x] - acc[x] / V;
  const double dr = Wn[i * (D + 2)] - W[i * (D + 2)];
  cellred[i * 3 + 0] = V * dr * dr;
  cellred[i * 3 + 1] = V;
  cellred[i * 3 + 2] = V * W[i * (D + 2)] * W[i * (D + 2)];
}

// Second stage (Eq. f_final) with the equilibrium of W^{n+1} and q^n.
template <int D, typename T>
__global__ __launch_bounds__(TPB) void k_stage2(DevVel v, GasP g, const double* __restrict__ primn,
                                                const double* __restrict__ q,
                                                const T* __restrict__ ht, const T* __restrict__ bt,
                                                T* __restrict__ h, T* __restrict__ b,
                                                const int32_t* flag) {
  const int64_t nch = (v.nvp + TPB - 1) / TPB;
  const int64_t i = blockIdx.x / nch;
  const int64_t k = (blockIdx.x % nch) * TPB + threadIdx.x;
  if (k >= v.nvp || *flag) return;
  const int64_t nvp = v.nvp;
  const double* P = &primn[i * NPRIM];
  double uk[3] = {0, 0, 0};
  for (int d = 0; d < D; ++d) uk[d] = v.u[d * nvp + k];
  double Hs, Bs;
  cell_equilibrium<D>(P, &q[i * 3], g, uk, Hs, Bs);
  const double a = dt_cell(g, i) / (2.0 * P[5]);
  const double inv = 1.0 / (1.0 + a);
  st(h, i * nvp + k, (ld(ht, i * nvp + k) + a * Hs) * inv);
  if (v.has_b) st(b, i * nvp + k, (ld(bt, i * nvp + k) + a * Bs) * inv);
}

// Residual of the density: one block, fixed summation order.
__device__ __forceinline__ void residual_of(int64_t nc, const double* __restrict__ cellred,
                                            double* __restrict__ resid, const int32_t* flag,
                                            double* lds) {
  if (flag[0] | flag[2]) return;
  double acc[3] = {0, 0, 0};
  for (int64_t i = threadIdx.x; i < nc; i += blockDim.x)
    for (int x = 0; x < 3; ++x) acc[x] += cellred[i * 3 + x];
  block_sum<3>(acc, lds);
  if (threadIdx.x == 0) {
    double nrm = sqrt(acc[0] / acc[1]);
    if (resid[3] == 0.0) resid[3] = nrm;
    resid[0] = resid[3] > 0.0 ? nrm / resid[3] : 0.0;
    resid[1] = nrm / sqrt(acc[2] / acc[1]);
  }
}

__global__ __launch_bounds__(1024) void k_residual(int64_t nc, const double* __restrict__ cellred,
                                                   double* __restrict__ resid, const int32_t* flag) {
  __shared__ double lds[3 * 16];
  residual_of(nc, cellred, resid, flag, lds);
}

template <int D>
__global__ void k_commit_W(int64_t nc, const double* __restrict__ Wn, double* __restrict__ W,
                           const int32_t* flag) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= nc * (D + 2) || *flag) return;
  W[i] = Wn[i];
}

template <int D, typename T>
__global__ __launch_bounds__(TPB) void k_init_maxwellian(DevVel v, const double* __restrict__ prim,
                                                         T* __restrict__ h, T* __restrict__ b) {
  const int64_t nch = (v.nvp + TPB - 1) / TPB;
  const int64_t i = blockIdx.x / nch;
  const int64_t k = (blockIdx.x % nch) * TPB + threadIdx.x;
  if (k >= v.nvp) return;
  const double* P = &prim[i * NPRIM];
  double c2 = 0.0;
  for (int d = 0; d < D; ++d) {
    double c = v.u[d * v.nvp + k] - P[1 + d];
    c2 += c * c;
  }
  const double H = P[0] * maxw_norm<D>(P[4]) * exp(-P[4] * c2);
  st(h, i * v.nvp + k, H);
  if (v.has_b) st(b, i * v.nvp + k, v.kxi / (2.0 * P[4]) * H);
}

// Rows of h or b in slots (own) and in the caller's order of cells and velocities
// (user): vel[k] is the velocity of slot k, -1 for a pad, which reads as 0.
template <typename T>
__global__ __launch_bounds__(TPB) void k_reorder(int64_t nv, int64_t nvp, const int32_t* __restrict__ cell,
                                                 const int32_t* __restrict__ vel, T* __restrict__ own,
                                                 T* __restrict__ user, int in) {
  const int64_t nch = (nvp + TPB - 1) / TPB;
  const int64_t i = blockIdx.x / nch;
  const int64_t k = (blockIdx.x % nch) * TPB + threadIdx.x;
  if (k >= nvp) return;
  const int32_t kk = vel[k];
  const int64_t at = (int64_t)cell[i] * nv + kk;
  if (in) own[i * nvp + k] = kk >= 0 ? user[at] : T(0);
  else if (kk >= 0) user[at] = own[i * nvp + k];
}

// Discrete moments sum_k w_k psi_k (h, b) per cell.
template <int D, typename T>
__global__ __launch_bounds__(TPB) void k_moments(DevVel v, const T* __restrict__ h,
                                                 const T* __restrict__ b, double* __restrict__ out) {
  __shared__ double lds[5 * 16];
  const int64_t i = blockIdx.x;
  double acc[5] = {0, 0, 0, 0, 0};
  for (int64_t k = threadIdx.x; k < v.nvp; k += TPB) {
    double wh = v.w[k] * ld(h, i * v.nvp + k);
    double wb = v.has_b ? v.w[k] * ld(b, i * v.nvp + k) : 0.0;
    acc[0] += wh;
    for (int d = 0; d < D; ++d) acc[1 + d] += wh * v.u[d * v.nvp + k];
    acc[D + 1] += 0.5 * (wh * v.u2[k] + wb);
  }
  block_sum<5>(acc, lds);
  if (threadIdx.x == 0)
    for (int x = 0; x < D + 2; ++x) out[i * (D + 2) + x] = acc[x];
}

// Per-cell CFL bound 2 V_i / max_k sum_j S_j |u_k . n_j|.
template <int D>
__global__ __launch_bounds__(TPB) void k_dt_cells(DevMesh m, DevVel v, double* __restrict__ out) {
  __shared__ double lds[16];
  const int64_t i = blockIdx.x;
  const int nfc = m.nfc[i];
  double mx = 0.0;
  for (int64_t k = threadIdx.x; k < v.nvp; k += TPB) {
    double s = 0.0;
    for (int p = 0; p < nfc; ++p) {
      const int64_t f = m.cface[i * MAXF + p];
      double un = 0.0;
      for (int d = 0; d < D; ++d) un += v.u[d * v.nvp + k] * m.fnorm[f * 3 + d];
      s += m.farea[f] * fabs(un);
    }
    mx = fmax(mx, s);
  }
  mx = block_max(mx, lds);
  if (threadIdx.x == 0) out[i] = 2.0 * m.vol[i] / mx;
}

inline unsigned blocks_for(int64_t n, int tpb) { return (unsigned)((n + tpb - 1) / tpb); }

// ---- batched forms: one launch covers every case of a batch ---------------
__device__ __forceinline__ int case_of(const int64_t* __restrict__ off, int n, int64_t t) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (off[mid] <= t) lo = mid;
    else hi = mid;
  }
  return lo;
}

template <int D>
__global__ __launch_bounds__(128) void k_gradW_b(BatchDev bd) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t cell = t / (D + 2);
  if (cell >= bd.cell_off[bd.n]) return;
  const int c = case_of(bd.cell_off, bd.n, cell);
  const CaseDev& C = bd.cases[c];
  gradW_at<D, 4>(t - bd.cell_off[c] * (D + 2), C.m, C.bcs, C.g, C.B.W, C.B.gW, C.B.flag, 1);
}

template <int D, typename T>
__global__ __launch_bounds__(64) void k_face_eq_b(BatchDev bd) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= bd.face_off[bd.n]) return;
  const int c = case_of(bd.face_off, bd.n, t);
  const CaseDev& C = bd.cases[c];
  face_eq_at<D, T>(t - bd.face_off[c], C.m, C.bcs, C.g, C.B.W, C.B.gW, C.B.q, C.B.frec, C.fm.nr,
                   (T*)C.B.srec, C.B.flag);
}

// one block per case
__global__ __launch_bounds__(1024) void k_residual_b(BatchDev bd) {
  __shared__ double lds[3 * 16];
  const CaseDev& C = bd.cases[blockIdx.x];
  residual_of(C.m.nc, C.B.cellred, C.B.resid, C.B.flag, lds);
}

}  // namespace

#define UGKS_DISPATCH_D(D_, ...)          \
  do {                                    \
    if ((D_) == 2) {                      \
      constexpr int DD = 2;               \
      __VA_ARGS__;                        \
    } else {                              \
      constexpr int DD = 3;               \
      __VA_ARGS__;                        \
    }                                     \
  } while (0)

#define UGKS_DISPATCH_DT(D_, P_, ...)                  \
  do {                                                 \
    if ((P_) == UGKS_FP32) {                           \
      using TT = float;                                \
      UGKS_DISPATCH_D(D_, __VA_ARGS__);                \
    } else {                                           \
      using TT = double;                               \
      UGKS_DISPATCH_D(D_, __VA_ARGS__);                \
    }                                                  \
  } while (0)

hipError_t launch_prims(int D, const DevMesh& m, const GasP& g, const double* W, double* prim,
                        int32_t* flag, int checkflag, hipStream_t s) {
  UGKS_DISPATCH_D(D, k_prims<DD><<<blocks_for(m.nc, 256), 256, 0, s>>>(m.nc, g, W, prim, flag, checkflag));
  return hipGetLastError();
}

hipError_t launch_heatflux(int D, int prec, const DevMesh& m, const DevVel& v, const void* h,
                           const void* b, const double* prim, double* q, const int32_t* flag,
                           hipStream_t s) {
  UGKS_DISPATCH_DT(D, prec, k_heatflux<DD, TT><<<(unsigned)m.nc, TPB, 0, s>>>(
      v, (const TT*)h, (const TT*)b, prim, q, flag));
  return hipGetLastError();
}

hipError_t launch_gradW(int D, const DevMesh& m, const DevBC* bcs, const GasP& g, const double* W,
                        double* gW, int32_t* flag, int count, hipStream_t s) {
  if (m.most <= 4)
    UGKS_DISPATCH_D(D, k_gradW<DD, 4><<<blocks_for(m.nc * (DD + 2), 128), 128, 0, s>>>(m, bcs, g, W, gW, flag, count));
  else
    UGKS_DISPATCH_D(D, k_gradW<DD, MAXF><<<blocks_for(m.nc * (DD + 2), 128), 128, 0, s>>>(m, bcs, g, W, gW, flag, count));
  return hipGetLastError();
}

hipError_t launch_face_eq(int D, const DevMesh& m, const DevBC* bcs, const GasP& g,
                          const double* W, const double* gW, const double* q, double* frec,
                          int prec, int nr, void* srec, int32_t* flag, hipStream_t s) {
  UGKS_DISPATCH_DT(D, prec, k_face_eq<DD, TT><<<blocks_for(m.nf, 64), 64, 0, s>>>(
      m, bcs, g, W, gW, q, frec, nr, (TT*)srec, flag));
  return hipGetLastError();
}

hipError_t launch_grad_micro(int D, int prec, const DevMesh& m, const DevVel& v,
                             const double* frec, const void* h, const void* b, double* gh,
                             double* gb, const int32_t* flag, hipStream_t s) {
  const int64_t per = 8 * xcd_run(m.nc, GRAD_TILE);
  const unsigned grid = (unsigned)((m.nc + per - 1) / per * per) * blocks_for(v.nvp, 2 * TPB);
  if (m.nc * v.nvp * D * (v.has_b ? 2 : 1) * (int64_t)sizeof(double) > kLastLevel)
    UGKS_DISPATCH_DT(D, prec, k_grad_micro<DD, TT, true><<<grid, TPB, 0, s>>>(
        m, v, frec, (const TT*)h, (const TT*)b, gh, gb, flag));
  else
    UGKS_DISPATCH_DT(D, prec, k_grad_micro<DD, TT, false><<<grid, TPB, 0, s>>>(
        m, v, frec, (const TT*)h, (const TT*)b, gh, gb, flag));
  return hipGetLastError();
}

hipError_t launch_flux(int D, int prec, const DevMesh& m, const DevVel& v, const GasP& g,
                       const double* frec, const void* h, const void* b, const double* gh,
                       const double* gb, double* fh, double* fb, double* F, const int32_t* flag,
                       hipStream_t s) {
  UGKS_DISPATCH_DT(D, prec, k_flux<DD, TT><<<face_grid(m), TPB, 0, s>>>(
      m, v, g, frec, (const TT*)h, (const TT*)b, gh, gb, fh, fb, F, flag));
  return hipGetLastError();
}

hipError_t launch_stage1(int D, int prec, const DevMesh& m, const DevVel& v, const GasP& g,
                         const double* prim, const double* q, const void* h, const void* b,
                         const double* fh, const double* fb, void* ht, void* bt,
                         const int32_t* flag, hipStream_t s) {
  const unsigned grid = blocks_for(v.nvp, TPB) * (unsigned)m.nc;
  UGKS_DISPATCH_DT(D, prec, k_stage1<DD, TT><<<grid, TPB, 0, s>>>(
      m, v, g, prim, q, (const TT*)h, (const TT*)b, fh, fb, (TT*)ht, (TT*)bt, flag));
  return hipGetLastError();
}

hipError_t launch_macro_update(int D, const DevMesh& m, const GasP& g, const double* W, const double* F,
                               double* Wn, double* cellred, const int32_t* flag, hipStream_t s) {
  UGKS_DISPATCH_D(D, k_macro_update<DD><<<blocks_for(m.nc, 256), 256, 0, s>>>(m, g, W, F, Wn, cellred, flag));
  return hipGetLastError();
}

hipError_t launch_stage2(int D, int prec, const DevMesh& m, const DevVel& v, const GasP& g,
                         const double* primn, const double* q, const void* ht, const void* bt,
                         void* h, void* b, const int32_t* flag, hipStream_t s) {
  const unsigned grid = blocks_for(v.nvp, TPB) * (unsigned)m.nc;
  UGKS_DISPATCH_DT(D, prec, k_stage2<DD, TT><<<grid, TPB, 0, s>>>(
      v, g, primn, q, (const TT*)ht, (const TT*)bt, (TT*)h, (TT*)b, flag));
  return hipGetLastError();
}

hipError_t launch_residual(const DevMesh& m, const double* cellred, double* resid,
                           const int32_t* flag, hipStream_t s) {
  k_residual<<<1, 1024, 0, s>>>(m.nc, cellred, resid, flag);
  return hipGetLastError();
}

hipError_t launch_commit_W(int D, const DevMesh& m, const double* Wn, double* W,
                           const int32_t* flag, hipStream_t s) {
  UGKS_DISPATCH_D(D, k_commit_W<DD><<<blocks_for(m.nc * (DD + 2), 256), 256, 0, s>>>(m.nc, Wn, W, flag));
  return hipGetLastError();
}

hipError_t launch_init_maxwellian(int D, int prec, const DevMesh& m, const DevVel& v,
                                  const double* prim, void* h, void* b, hipStream_t s) {
  const unsigned grid = blocks_for(v.nvp, TPB) * (unsigned)m.nc;
  UGKS_DISPATCH_DT(D, prec, k_init_maxwellian<DD, TT><<<grid, TPB, 0, s>>>(v, prim, (TT*)h, (TT*)b));
  return hipGetLastError();
}

hipError_t launch_moments(int D, int prec, const DevMesh& m, const DevVel& v, const void* h,
                          const void* b, double* out, hipStream_t s) {
  UGKS_DISPATCH_DT(D, prec, k_moments<DD, TT><<<(unsigned)m.nc, TPB, 0, s>>>(v, (const TT*)h, (const TT*)b, out));
  return hipGetLastError();
}

hipError_t launch_reorder(int prec, int64_t nc, int64_t nv, int64_t nvp, const int32_t* cell, const int32_t* vel,
                          void* own, void* user, bool in, hipStream_t s) {
  const unsigned grid = blocks_for(nvp, TPB) * (unsigned)nc;
  if (prec == UGKS_FP32)
    k_reorder<float><<<grid, TPB, 0, s>>>(nv, nvp, cell, vel, (float*)own, (float*)user, in);
  else
    k_reorder<double><<<grid, TPB, 0, s>>>(nv, nvp, cell, vel, (double*)own, (double*)user, in);
  return hipGetLastError();
}

hipError_t launch_dt_cells(int D, const DevMesh& m, const DevVel& v, double* cellval,
                           hipStream_t s) {
  UGKS_DISPATCH_D(D, k_dt_cells<DD><<<(unsigned)m.nc, TPB, 0, s>>>(m, v, cellval));
  return hipGetLastError();
}

hipError_t launch_wall_rho(int D, int prec, const DevMesh& m, const DevVel& v, const GasP& g,
                           const void* h, const double* gh, double* frec, const int32_t* flag,
                           hipStream_t s) {
  if (m.nwall == 0) return hipSuccess;
  UGKS_DISPATCH_DT(D, prec, k_wall_rho<DD, TT><<<(unsigned)m.nwall, TPB, 0, s>>>(
      m, v, g, (const TT*)h, gh, frec, flag));
  return hipGetLastError();
}

hipError_t launch_gradW_b(int D, const BatchDev& bd, int64_t ncell, hipStream_t s) {
  if (ncell == 0) return hipSuccess;
  const unsigned grid = (unsigned)((ncell * (D + 2) + 127) / 128);
  if (D == 2) k_gradW_b<2><<<grid, 128, 0, s>>>(bd);
  else k_gradW_b<3><<<grid, 128, 0, s>>>(bd);
  return hipGetLastError();
}

hipError_t launch_face_eq_b(int D, int prec, const BatchDev& bd, int64_t nface, hipStream_t s) {
  if (nface == 0) return hipSuccess;
  const unsigned grid = (unsigned)((nface + 63) / 64);
  UGKS_DISPATCH_DT(D, prec, k_face_eq_b<DD, TT><<<grid, 64, 0, s>>>(bd));
  return hipGetLastError();
}

hipError_t launch_residual_b(const BatchDev& bd, hipStream_t s) {
  if (bd.n == 0) return hipSuccess;
  k_residual_b<<<(unsigned)bd.n, 1024, 0, s>>>(bd);
  return hipGetLastError();
}

}  // namespace ugks
