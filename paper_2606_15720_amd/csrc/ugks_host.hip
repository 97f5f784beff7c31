// Host side of the gfx950 UGKS library: the C ABI declared in ugks.h.
//
// ugks_create validates the mesh and velocity set, renumbers nothing the
// caller can see (all outputs come back in the caller's order), precomputes
// the least-squares coefficients of every cell (unweighted, one row per face
// neighbour or mirror ghost), lays the velocity set out in slots (mirror pairs
// where it is symmetric; zero-weight pads to whole waves), fixes the time step
// from the CFL bound and allocates every device buffer once.  ugks_step only
// enqueues kernels and reads their status back.
#include "ugks_device.h"
#include "ugks_host_util.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <exception>
#include <fstream>
#include <map>
#include <set>
#include <memory>
#include <mutex>
#include <sstream>

using namespace ugks;
using namespace ugks::host;

namespace {

thread_local std::string g_create_error;

// Solve the D x D SPD normal system by Cholesky; returns false if singular.
bool chol_inverse(int D, const double* N, double* Ninv) {
  double Lm[9] = {0};
  for (int j = 0; j < D; ++j) {
    double s = N[j * 3 + j];
    for (int k = 0; k < j; ++k) s -= Lm[j * 3 + k] * Lm[j * 3 + k];
    if (!(s > 0.0)) return false;
    Lm[j * 3 + j] = std::sqrt(s);
    for (int i = j + 1; i < D; ++i) {
      double t = N[i * 3 + j];
      for (int k = 0; k < j; ++k) t -= Lm[i * 3 + k] * Lm[j * 3 + k];
      Lm[i * 3 + j] = t / Lm[j * 3 + j];
    }
  }
  for (int col = 0; col < D; ++col) {
    double y[3], x[3];
    for (int i = 0; i < D; ++i) {
      double t = (i == col) ? 1.0 : 0.0;
      for (int k = 0; k < i; ++k) t -= Lm[i * 3 + k] * y[k];
      y[i] = t / Lm[i * 3 + i];
    }
    for (int i = D - 1; i >= 0; --i) {
      double t = y[i];
      for (int k = i + 1; k < D; ++k) t -= Lm[k * 3 + i] * x[k];
      x[i] = t / Lm[i * 3 + i];
    }
    for (int i = 0; i < D; ++i) Ninv[i * 3 + col] = x[i];
  }
  return true;
}


// The checks of a case's arguments that need no mesh traversal: pointers,
// sizes, dimension and gas constants.
void check_case_args(const ugks_mesh* mesh, const ugks_velocity* vel, const ugks_gas* gas,
                     const double* W0) {
  fail_if(!mesh || !vel || !gas || !W0, "null argument");
  const int D = mesh->dim;
  fail_if(D != 2 && D != 3, "mesh.dim must be 2 or 3");
  fail_if(gas->K < 0, "gas.K (internal degrees of freedom) must be >= 0");
  const int64_t nc = mesh->n_cells, nf = mesh->n_faces, nv = vel->nv;
  fail_if(nc <= 0 || nf <= 0 || nv <= 0, "empty mesh or velocity set");
  fail_if(nc >= (int64_t)INT32_MAX || nf >= (int64_t)INT32_MAX, "mesh too large for 32-bit indices");
  fail_if(!mesh->cell_volume || !mesh->cell_centroid || !mesh->face_cells || !mesh->face_area ||
              !mesh->face_normal || !mesh->face_centroid || !mesh->face_bc || !mesh->face_bc_id ||
              !vel->u || !vel->w,
          "null mesh or velocity array");
  fail_if(!(gas->Pr > 0.0) || !(gas->R > 0.0) || !(gas->T_ref > 0.0) || !(gas->mu_ref > 0.0),
          "gas constants must be positive");
}

// The velocity slots of the fused path (see FusedMesh): the caller's point of
// every slot (-1: pad), and vidx the packed node indices of all of them.  ax:
// the sorted symmetric nodes that every coordinate is one of.
std::vector<int64_t> pair_slots(int D, const ugks_velocity* vel, const std::vector<double>& ax,
                                std::vector<int32_t>& vidx, int64_t* full) {
  const int64_t nv = vel->nv, na = (int64_t)ax.size();
  std::vector<int32_t> id(nv * D);
  int64_t cube = 1;
  for (int d = 0; d < D; ++d) cube *= na;
  std::vector<int64_t> at(cube, -1);
  auto cell = [&](const int32_t* i) {
    int64_t r = 0;
    for (int d = 0; d < D; ++d) r = r * na + i[d];
    return r;
  };
  for (int64_t k = 0; k < nv; ++k) {
    for (int d = 0; d < D; ++d)
      id[k * D + d] = (int32_t)(std::lower_bound(ax.begin(), ax.end(), vel->u[k * D + d]) - ax.begin());
    at[cell(&id[k * D])] = k;
  }
  struct Pair {
    int64_t key, k, m;  // order, first member, its mirror (-1: pad)
  };
  std::vector<Pair> pairs;
  std::vector<char> done(nv, 0);
  const int sh = D == 3 ? 2 : 3;  // blocks of 4 x 4 x 4 or 8 x 8 nodes
  for (int64_t k = 0; k < nv; ++k) {
    if (done[k]) continue;
    int32_t mi[3];
    for (int d = 0; d < D; ++d) mi[d] = (int32_t)na - 1 - id[k * D + d];
    int64_t first = k, m = at[cell(mi)];
    if (m >= 0 && (m == k || done[m])) m = -1;
    done[k] = 1;
    if (m >= 0) {
      done[m] = 1;
      // the member on the far side of the first axis that tells them apart
      if (std::lexicographical_compare(&id[k * D], &id[k * D] + D, mi, mi + D)) std::swap(first, m);
    }
    int64_t block = 0, in = 0;
    for (int d = 0; d < D; ++d) {
      // blocks are counted from the middle of the first axis
      const int64_t i = id[first * D + d] + (d == 0 ? (1 << 10) - na / 2 : 0);
      block = (block << 10) | (i >> sh);
      in = (in << sh) | (i & ((1 << sh) - 1));
    }
    pairs.push_back({(block << 10) | in, first, m});
  }
  // points without a mirror last: their waves need not do the second member
  std::sort(pairs.begin(), pairs.end(), [](const Pair& a, const Pair& b) {
    if ((a.m < 0) != (b.m < 0)) return b.m < 0;
    return a.key != b.key ? a.key < b.key : a.k < b.k;
  });
  const int64_t with = std::count_if(pairs.begin(), pairs.end(), [](const Pair& a) { return a.m >= 0; });
  *full = (with + WAVE - 1) / WAVE * WAVE;
  const int64_t half = ((int64_t)pairs.size() + WAVE - 1) / WAVE * WAVE;
  std::vector<int64_t> slots(2 * half, -1);
  vidx.assign(2 * half, 0);
  for (int64_t j = 0; j < half; ++j) {
    const bool real = j < (int64_t)pairs.size();
    const Pair& p = pairs[real ? j : pairs.size() - 1];  // pads repeat the last pair's velocities
    if (real) {
      slots[j] = p.k;
      slots[half + j] = p.m;
    }
    for (int d = 0; d < D; ++d) {
      const int32_t i = id[p.k * D + d];
      vidx[j] |= (i * 16) << (10 * d);
      vidx[half + j] |= (((int32_t)na - 1 - i) * 16) << (10 * d);
    }
  }
  return slots;
}

// Fewest cells that take the whole-cell form where a cell has more than one
// velocity block.  Measured per step, whole cells against blocks of 4096: 6
// cells x 28^3 130 / 128 us, 48 x 28^3 148 / 160, 384 x 28^3 193 / 226, 750 x
// 20^3 135 / 150, 1,296 x 24^3 316 / 349, 2,058 x 28^3 736 / 737 us.
constexpr int64_t kWholeCells = 48;

constexpr int64_t kPinnedCells = 4 << 20;  // bytes of cell data read back through pinned memory, at most

// Lanes per work-group of the whole-cell form (one mirror pair each): enough
// pairs per lane that the cell's fixed costs (tables, sums, the new
// equilibrium) are spread, yet as much of the row as can be in the
// work-groups' LDS and in flight; more lanes than that only while the cells do
// not fill the GPU's 4,096 resident waves.  The lines lie where the next size
// becomes faster, ms per step by lanes 64 / 128 / 256 / 512 (24,576 tets, and
// 9,216 quads at 13 and 7 waves of pairs):
//   FP64   4 waves 0.368 0.298 0.384 0.669;  7: 0.273 0.233 0.242 0.323;
//         13: 0.494 0.423 0.390 0.466;  22: 1.377 1.041 0.978 1.228;
//         54: - - 2.144 2.165;  63: - - 2.435 2.395
//   FP32   7: 0.141 0.147 0.163 0.260;  8: 0.326 0.306 0.349 0.505;
//         13: 0.236 0.218 0.237 0.331;  32 (48,000 tets): 1.834 1.572 1.524 1.768;
//         83: - - 1.839 1.846;  172: - - 3.647 3.592
// Wide cells' tables take the LDS of two to four narrow ones', so that small groups
// leave compute units short of waves.  Their kernel alone (4,096 hexahedra, and
// 13,824 at 54 and 63 waves):
//   FP64   1: 0.075 0.067 0.067 0.122;  2: 0.093 0.070 0.069 0.124;
//          3: 0.109 0.087 0.073 0.124;  8: 0.192 0.132 0.104 0.139;
//         32: 0.655 0.430 0.318 0.331;  54: - - 1.744 1.651;  63: - - 1.998 1.859
//   FP32   1: 0.078 0.070 0.070 0.130;  3: 0.123 0.094 0.075 0.136;
//         32: 0.840 0.505 0.343 0.361;  54: - - 1.878 1.889;  63: - - 2.112 2.096
int cell_lanes(int64_t nc, int64_t pairs, int prec, bool wide) {
  // waves of pairs from which 2, 4, 8 waves take a cell
  static const int64_t from[3][3] = {{3, 13, 58}, {8, 20, 128}, {1, 3, 54}};
  const int64_t waves = pairs / WAVE, *line = from[wide ? 2 : prec == UGKS_FP32 ? 1 : 0];
  int64_t w = 1;
  for (int i = 0; i < 3 && (waves >= line[i] || (nc * w < 4096 && 2 * w <= waves)); ++i) w *= 2;
  return (int)(w * WAVE);
}

void build(ugks_ctx* c, const ugks_mesh* mesh, const ugks_velocity* vel, const ugks_gas* gas,
           const ugks_bc* bcs, int32_t n_bc, const double* W0, const ugks_options* opt, bool host) {
  check_case_args(mesh, vel, gas, W0);
  const int D = mesh->dim;
  const int64_t nc = mesh->n_cells, nf = mesh->n_faces, nv = vel->nv;
  int prec = opt && opt->precision ? opt->precision : UGKS_FP64;
  fail_if(prec != UGKS_FP64 && prec != UGKS_FP32, "precision must be 64 or 32");
  int Bv = opt && opt->block_v ? opt->block_v : 0;
  fail_if(Bv < 0 || Bv % WAVE != 0, "block_v must be 0 or a positive multiple of 64");
  const int tile = opt && opt->tile_cells ? opt->tile_cells : 0;
  fail_if(tile < 0, "tile_cells must be >= 0");
  const int lim = opt ? opt->limiter : 0;
  const double limk = opt ? opt->limiter_k : 0.0;
  fail_if(lim != 0 && lim != 1, "limiter must be 0 (none) or 1 (Venkatakrishnan)");
  fail_if(lim == 1 && !(limk >= 0.0 && std::isfinite(limk)), "limiter_k must be finite and >= 0");
  c->D = D;
  // K_xi = K + 3 - D internal and out-of-plane dimensions (Eq. Kxi_def); b
  // is carried when there are any (always in 2-D)
  c->kxi = gas->K + 3 - D;
  c->nr = c->kxi > 0 ? 2 : 1;
  c->prec = prec;
  c->Bv = Bv;
  c->flags = opt ? opt->flags : 0;
  c->nc = nc;
  c->nf = nf;
  c->nv = nv;
  // ---- mesh validation and cell -> face tables --------------------------
  for (int64_t i = 0; i < nc; ++i)
    fail_if(!(mesh->cell_volume[i] > 0.0), "non-positive cell volume");
  std::vector<int32_t> nfc(nc, 0), cface(nc * MAXF, -1), cnbr(nc * MAXF, -1);
  std::vector<double> csign(nc * MAXF, 0.0);
  std::vector<int32_t> fL(nf), fR(nf), fbc(nf), fbcid(nf), walls;
  std::vector<double> farea(nf), fnorm(nf * 3, 0.0), fdxL(nf * 3, 0.0), fdxR(nf * 3, 0.0),
      fmir(nf * 3, 0.0);
  // ---- cell renumbering: Z-order (Morton) of the centroids, so that cells
  // with nearby indices are spatial neighbours (they run together and share
  // stencil rows in cache); the caller never sees this order
  std::vector<int64_t> perm(nc), inv(nc);
  {
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int64_t i = 0; i < nc; ++i)
      for (int d = 0; d < D; ++d) {
        lo[d] = std::min(lo[d], mesh->cell_centroid[i * D + d]);
        hi[d] = std::max(hi[d], mesh->cell_centroid[i * D + d]);
      }
    std::vector<std::pair<uint64_t, int64_t>> key(nc);
    for (int64_t i = 0; i < nc; ++i) {
      uint64_t code = 0;
      for (int d = 0; d < D; ++d) {
        const double span = hi[d] > lo[d] ? hi[d] - lo[d] : 1.0;
        uint64_t qd = (uint64_t)std::min(1048575.0, std::floor((mesh->cell_centroid[i * D + d] - lo[d]) / span * 1048576.0));
        for (int bit = 0; bit < 20; ++bit) code |= ((qd >> bit) & 1ull) << (bit * D + d);
      }
      key[i] = {(c->flags & 4) ? (uint64_t)i : code, i};
    }
    std::stable_sort(key.begin(), key.end());
    for (int64_t i = 0; i < nc; ++i) {
      perm[i] = key[i].second;
      inv[key[i].second] = i;
    }
  }
  std::vector<double> cen(nc * 3, 0.0), vol(nc);
  for (int64_t i = 0; i < nc; ++i) {
    vol[i] = mesh->cell_volume[perm[i]];
    for (int d = 0; d < D; ++d) cen[i * 3 + d] = mesh->cell_centroid[perm[i] * D + d];
  }
  std::vector<double> closure(nc * 3, 0.0), asum(nc, 0.0);
  for (int64_t f = 0; f < nf; ++f) {
    int64_t L = mesh->face_cells[2 * f], R = mesh->face_cells[2 * f + 1];
    int kind = mesh->face_bc[f];
    fail_if(L < 0 || L >= nc, "face_cells L out of range");
    fail_if(kind < 0 || kind > 3, "unknown face_bc");
    fail_if(kind == UGKS_BC_INTERIOR && (R < 0 || R >= nc || R == L), "interior face needs a distinct R");
    fail_if(kind != UGKS_BC_INTERIOR && R != -1, "boundary face must have R = -1");
    L = inv[L];
    if (R >= 0) R = inv[R];
    fail_if(!(mesh->face_area[f] > 0.0), "non-positive face area");
    double nn = 0.0;
    for (int d = 0; d < D; ++d) nn += mesh->face_normal[f * D + d] * mesh->face_normal[f * D + d];
    fail_if(std::fabs(nn - 1.0) > 1e-10, "face normal is not a unit vector");
    if (kind != UGKS_BC_INTERIOR) {
      int id = mesh->face_bc_id[f];
      fail_if(id < 0 || id >= n_bc || !bcs, "face_bc_id out of range");
      fail_if(bcs[id].kind != kind, "face_bc does not match the boundary table kind");
      if (kind == UGKS_BC_WALL) {
        double un = 0.0;
        for (int d = 0; d < D; ++d) un += bcs[id].U[d] * mesh->face_normal[f * D + d];
        fail_if(std::fabs(un) > 1e-12, "wall velocity must be tangential");
        walls.push_back((int32_t)f);
      }
    }
    fL[f] = (int32_t)L;
    fR[f] = (int32_t)R;
    fbc[f] = kind;
    fbcid[f] = mesh->face_bc_id[f];
    farea[f] = mesh->face_area[f];
    double dn = 0.0;
    for (int d = 0; d < D; ++d) {
      double n = mesh->face_normal[f * D + d];
      double xf = mesh->face_centroid[f * D + d];
      double sh = mesh->face_shift ? mesh->face_shift[f * D + d] : 0.0;
      fnorm[f * 3 + d] = n;
      fdxL[f * 3 + d] = xf - cen[L * 3 + d];
      if (R >= 0) fdxR[f * 3 + d] = xf - sh - cen[R * 3 + d];
      dn += (xf - cen[L * 3 + d]) * n;
    }
    for (int d = 0; d < D; ++d) fmir[f * 3 + d] = 2.0 * dn * fnorm[f * 3 + d];
    auto add = [&](int64_t cell, int64_t nb, double s) {
      fail_if(nfc[cell] >= MAXF, "a cell has more than 8 faces");
      int p = nfc[cell]++;
      cface[cell * MAXF + p] = (int32_t)f;
      cnbr[cell * MAXF + p] = (int32_t)nb;
      csign[cell * MAXF + p] = s;
      for (int d = 0; d < D; ++d) closure[cell * 3 + d] += s * farea[f] * fnorm[f * 3 + d];
      asum[cell] += farea[f];
    };
    add(L, R, 1.0);
    if (R >= 0) add(R, L, -1.0);
  }
  for (int64_t i = 0; i < nc; ++i) {
    fail_if(nfc[i] < D + 1, "a cell has fewer than D+1 faces");
    double cl = 0.0;
    for (int d = 0; d < D; ++d) cl += closure[i * 3 + d] * closure[i * 3 + d];
    fail_if(std::sqrt(cl) > 1e-9 * asum[i], "a cell is not closed (sum S n != 0)");
  }
  // ---- least-squares coefficients --------------------------------------
  std::vector<double> lsG(nc * 3 * MAXF, 0.0);
  for (int64_t i = 0; i < nc; ++i) {
    double off[MAXF][3] = {{0}};
    for (int p = 0; p < nfc[i]; ++p) {
      int f = cface[i * MAXF + p];
      int j = cnbr[i * MAXF + p];
      for (int d = 0; d < D; ++d) {
        if (j >= 0) {
          // offset to the neighbour's centroid (periodic image for a shifted face)
          double sh = mesh->face_shift ? mesh->face_shift[f * D + d] : 0.0;
          double s = csign[i * MAXF + p];
          off[p][d] = cen[j * 3 + d] + s * sh - cen[i * 3 + d];
        } else {
          off[p][d] = fmir[f * 3 + d];
        }
      }
    }
    double N[9] = {0}, Ni[9];
    for (int p = 0; p < nfc[i]; ++p)
      for (int r = 0; r < D; ++r)
        for (int s = 0; s < D; ++s) N[r * 3 + s] += off[p][r] * off[p][s];
    fail_if(!chol_inverse(D, N, Ni), "degenerate least-squares stencil");
    for (int d = 0; d < D; ++d)
      for (int p = 0; p < nfc[i]; ++p) {
        double s = 0.0;
        for (int e = 0; e < D; ++e) s += Ni[d * 3 + e] * off[p][e];
        lsG[(i * 3 + d) * MAXF + p] = s;
      }
  }
  // first-order reconstruction: every gradient of the step, macroscopic and
  // microscopic, is zero (piecewise-constant states on both sides of each
  // face); the true coefficients are kept for the warm start's features
  std::vector<double> lsG_true;
  if (opt && (opt->flags & 16)) {
    lsG_true = lsG;
    std::fill(lsG.begin(), lsG.end(), 0.0);
  }
  // ---- velocity set -----------------------------------------------------
  for (int64_t k = 0; k < nv; ++k) {
    fail_if(!(vel->w[k] > 0.0), "velocity weights must be positive");
    for (int d = 0; d < D; ++d) fail_if(!std::isfinite(vel->u[k * D + d]), "non-finite velocity");
  }
  // ---- fused-path eligibility ----------------------------------------------
  // A tensor product of one symmetric 1-D node set, first axis slowest, so
  // that point k and its mirror -u_k = u_{nv-1-k} are known by index.
  std::vector<double> ax;
  {
    std::vector<double> a0;
    for (int64_t k = 0; k < nv; ++k) a0.push_back(vel->u[k * D]);
    std::sort(a0.begin(), a0.end());
    a0.erase(std::unique(a0.begin(), a0.end()), a0.end());
    bool ok = !(c->flags & 2);
    const int64_t na = (int64_t)a0.size();
    int64_t prod = 1;
    for (int d = 0; d < D; ++d) prod *= na;
    ok = ok && prod == nv && na <= 64;
    for (int64_t n = 0; ok && n < na; ++n) ok = a0[na - 1 - n] == -a0[n];
    for (int64_t k = 0; ok && k < nv; ++k) {
      int64_t r = k;
      for (int d = D - 1; d >= 0 && ok; --d) {
        ok = vel->u[k * D + d] == a0[r % na];
        r /= na;
      }
    }
    bool mesh_ok = !(c->flags & 2);
    for (int64_t f = 0; mesh_ok && f < nf; ++f)
      mesh_ok = mesh->face_bc[f] >= UGKS_BC_INTERIOR && mesh->face_bc[f] <= UGKS_BC_OUTFLOW;
    const bool wide = *std::max_element(nfc.begin(), nfc.end()) > 4;
    // Cells of more faces are taken whole, one work-group each, unless they are
    // few and have many velocities (hexahedra, ms per step whole and staged: 27
    // cells x 16^3 0.070 and 0.097; 64 x 24^3 0.158 and 0.223, by then bound by
    // the number of work-groups).
    mesh_ok = mesh_ok && (!wide || nc >= kWholeCells || nv <= 4096);
    ok = ok && mesh_ok;
    if (ok) {
      ax = a0;
      c->fmesh.na = (int)na;
    } else if (mesh_ok) {
      // Sparse tensor set: every coordinate of every point is a node of one
      // 1-D set A = -A of at most 64 nodes (a locally refined set whose levels
      // are lattices is one), so the Maxwellians still factor over the axes.
      std::vector<double> aa;
      for (int64_t k = 0; k < nv * D; ++k) {
        aa.push_back(vel->u[k]);
        aa.push_back(-vel->u[k]);
      }
      std::sort(aa.begin(), aa.end());
      aa.erase(std::unique(aa.begin(), aa.end()), aa.end());
      if ((int64_t)aa.size() <= 64) {
        ax = aa;
        c->fmesh.na = (int)aa.size();
        c->fmesh.sparse = true;
        ok = true;
      }
    }
    c->fused = ok && !wide;
    c->wide = ok && wide;
  }
  // ---- velocity slots -------------------------------------------------------
  std::vector<int32_t> vidx;
  c->vel_perm = c->slots() ? pair_slots(D, vel, ax, vidx, &c->fmesh.full) : std::vector<int64_t>();
  if (!c->slots()) {
    // the caller's order, rows padded to whole waves
    c->vel_perm.assign((nv + WAVE - 1) / WAVE * WAVE, -1);
    for (int64_t k = 0; k < nv; ++k) c->vel_perm[k] = k;
  }
  const int64_t nvp = c->nvp = (int64_t)c->vel_perm.size();
  std::vector<double> u(3 * nvp, 0.0), w(nvp, 0.0), u2(nvp, 0.0);
  for (int64_t k = 0; k < nvp; ++k) {
    const int64_t kk = c->vel_perm[k];
    if (kk >= 0) w[k] = vel->w[kk];
    for (int d = 0; d < D; ++d) {
      if (kk >= 0) u[d * nvp + k] = vel->u[kk * D + d];
      else if (c->slots()) u[d * nvp + k] = ax[((uint32_t)vidx[k] >> (10 * d + 4)) & 63];
      u2[k] += u[d * nvp + k] * u[d * nvp + k];
    }
  }
  // ---- initial state check ---------------------------------------------
  for (int64_t i = 0; i < nc; ++i) {
    const double* Wi = &W0[i * (D + 2)];
    double rho = Wi[0], m2 = 0.0;
    for (int d = 0; d < D; ++d) m2 += Wi[1 + d] * Wi[1 + d];
    fail_if(!(rho > 0.0), "initial density must be positive");
    fail_if(!(Wi[D + 1] - 0.5 * m2 / rho > 0.0), "initial internal energy must be positive");
  }
  // ---- stream -------------------------------------------------------------
  if (opt && opt->stream) {
    c->stream = (hipStream_t)opt->stream;
    c->own_stream = false;
  } else {
    HIP_TRY(hipStreamCreateWithFlags(&c->stream, hipStreamNonBlocking));
    c->own_stream = true;
  }
  // ---- device buffers ---------------------------------------------------
  DevMesh& m = c->mesh;
  m.nc = nc;
  m.nf = nf;
  m.vol = upload(c, vol);
  m.cen = upload(c, cen);
  m.nfc = upload(c, nfc);
  m.most = *std::max_element(nfc.begin(), nfc.end());
  m.cface = upload(c, cface);
  m.cnbr = upload(c, cnbr);
  m.csign = upload(c, csign);
  m.lsG = upload(c, lsG);
  c->lsG_exact = lsG_true.empty() ? m.lsG : upload(c, lsG_true);
  m.fL = upload(c, fL);
  m.fR = upload(c, fR);
  std::vector<int32_t> ford(nf);
  for (int64_t f = 0; f < nf; ++f) ford[f] = (int32_t)f;
  std::stable_sort(ford.begin(), ford.end(), [&](int32_t a, int32_t b) { return fL[a] < fL[b]; });
  m.ford = upload(c, ford);
  m.fbc = upload(c, fbc);
  m.fbcid = upload(c, fbcid);
  m.farea = upload(c, farea);
  m.fnorm = upload(c, fnorm);
  m.fdxL = upload(c, fdxL);
  m.fdxR = upload(c, fdxR);
  m.fmir = upload(c, fmir);
  m.walls = upload(c, walls);
  m.nwall = (int64_t)walls.size();
  m.limiter = lim;
  if (lim) {
    std::vector<double> veps2(nc);
    for (int64_t i = 0; i < nc; ++i) veps2[i] = std::pow(limk * std::pow(vol[i], 1.0 / D), 3);
    m.veps2 = upload(c, veps2);
  }
  DevVel& v = c->vel;
  v.nv = nv;
  v.nvp = nvp;
  v.u = upload(c, u);
  v.w = upload(c, w);
  v.u2 = upload(c, u2);
  v.kxi = (double)c->kxi;
  v.has_b = c->nr == 2 ? 1 : 0;
  std::vector<DevBC> hb(std::max(n_bc, 1));
  for (int i = 0; i < n_bc; ++i) {
    hb[i].kind = bcs[i].kind;
    hb[i].rho = bcs[i].rho;
    for (int d = 0; d < 3; ++d) hb[i].U[d] = bcs[i].U[d];
    hb[i].T = bcs[i].T;
    fail_if(bcs[i].kind != UGKS_BC_OUTFLOW && !(bcs[i].T > 0.0), "boundary temperature must be positive");
  }
  c->bcs = upload(c, hb);
  // ---- time step (R5), and the local steps of reading R26 -------------------
  c->gas.Pr = gas->Pr;
  c->gas.R = gas->R;
  c->gas.Tref = gas->T_ref;
  c->gas.muref = gas->mu_ref;
  c->gas.omega = gas->omega;
  c->gas.K = (double)gas->K;
  const bool lts = (c->flags & 128) != 0;
  fail_if(lts && (c->flags & 64),
          "local time steps (flags bit 7) and boundary-flux tracking (bit 6) exclude each other");
  std::vector<double> dtc;
  {
    fail_if(!(gas->dt > 0.0) && !(gas->cfl > 0.0), "cfl must be positive when dt = 0");
    // each cell's bound 2 V_i / max_k sum_j S_j |u_k . n_j|
    std::vector<double> bound;
    double mn = INFINITY;
    if (!(gas->dt > 0.0) || lts) {
      double* cellv = dalloc<double>(c, nc);
      HIP_TRY(launch_dt_cells(D, m, v, cellv, c->stream));
      bound.resize(nc);
      HIP_TRY(hipMemcpyAsync(bound.data(), cellv, nc * sizeof(double), hipMemcpyDeviceToHost, c->stream));
      HIP_TRY(hipStreamSynchronize(c->stream));
      for (double x : bound) mn = std::min(mn, x);
      fail_if(!(mn > 0.0) || !std::isfinite(mn), "could not derive a time step");
    }
    c->gas.dt = gas->dt > 0.0 ? gas->dt : gas->cfl * mn;
    if (lts) {
      // cell i advances by dt b_i / min b (the most restrictive cell keeps dt)
      dtc.resize(nc);
      for (int64_t i = 0; i < nc; ++i) dtc[i] = c->gas.dt * (bound[i] / mn);
      c->gas.dtc = upload(c, dtc);
    }
  }
  // Rows of h and b beyond the cells': row nc is all zero (a wall face's
  // "neighbour"), then one ghost row per far-field or outflow face.
  std::vector<int32_t> ghost_row(nf, -1), ffaces;
  if (c->slots()) {
    for (int64_t f = 0; f < nf; ++f)
      if (fbc[f] == UGKS_BC_FARFIELD || fbc[f] == UGKS_BC_OUTFLOW) {
        ghost_row[f] = (int32_t)(nc + 1 + (int64_t)ffaces.size());
        ffaces.push_back((int32_t)f);
      }
    c->fmesh.nff = (int64_t)ffaces.size();
    c->fmesh.ffaces = upload(c, ffaces);
    c->fmesh.apart = true;
    for (int32_t f : walls)
      for (int p = 0; p < nfc[fL[f]]; ++p)
        if (ghost_row[cface[(int64_t)fL[f] * MAXF + p]] >= 0) c->fmesh.apart = false;
    c->fmesh.half = nvp / 2;
    c->fmesh.nr = c->nr;
    // the sweep reads one iteration ahead
    vidx.resize(vidx.size() + 512, 0);
    c->fmesh.nc = nc;
    c->fmesh.nv = nv;
    c->fmesh.axis = upload(c, ax);
    c->fmesh.vidx = upload(c, vidx);
  }
  if (c->wide) {
    std::vector<int32_t> ci(nc * CRI, 0), frow(nf);
    std::vector<double> cdr(nc * CRD, 0.0);
    for (int64_t f = 0; f < nf; ++f) frow[f] = fR[f] >= 0 ? fR[f] : ghost_row[f] >= 0 ? ghost_row[f] : (int32_t)nc;
    for (int64_t i = 0; i < nc; ++i) {
      int32_t* I = &ci[i * CRI];
      I[WI_NF] = nfc[i];
      for (int p = 0; p < MAXF; ++p) {
        // (slots past the cell's faces: face 0, for the tables only)
        const int pp = p < nfc[i] ? p : 0;
        double* fd = &cdr[i * CRD + WD_FS * p];
        const int f = cface[i * MAXF + pp];
        const int j = cnbr[i * MAXF + pp];
        const double sg = csign[i * MAXF + pp];
        I[WI_ROW + p] = j >= 0 ? j : ghost_row[f] >= 0 ? ghost_row[f] : (int32_t)nc;
        I[WI_FACE + p] = f;
        I[WI_KIND + p] = fbc[f];
        if (p < nfc[i] && ghost_row[f] >= 0) I[WI_FAR] = 1;
        for (int d = 0; d < 3; ++d) {
          fd[d] = sg * fnorm[f * 3 + d];
          fd[3 + d] = sg > 0.0 ? fdxL[f * 3 + d] : fdxR[f * 3 + d];
          fd[6 + d] = j >= 0 ? (sg > 0.0 ? fdxR[f * 3 + d] : fdxL[f * 3 + d]) : 0.0;
        }
        fd[9] = fbc[f] == UGKS_BC_WALL ? 0.0 : 1.0;
        fd[10] = p < nfc[i] ? farea[f] / vol[i] : 0.0;
        if (lts) fd[10] *= dtc[i] / c->gas.dt;
      }
    }
    c->fmesh.crec_i = upload(c, ci);
    c->fmesh.crec_d = upload(c, cdr);
    c->fmesh.frow = upload(c, frow);
    c->sched.lanes = cell_lanes(nc, c->fmesh.half, prec, true);
    c->sched.tile = dev::xcd_run(nc, 32);  // (as the gradients' runs)
  }
  if (c->fused) {
    // Static records of the fused sweep: the cell's faces, its least-squares
    // stencil and, per face, the neighbour's stencil, all wave-uniform.
    // Every cell is padded to the same shape (4 faces, 4-row stencils) so the
    // sweep runs one straight-line body:
    //   * a missing stencil row points at a real row with coefficient 0;
    //   * a wall face's "neighbour" rows point at the all-zero row nc (so the
    //     incoming free transport vanishes) and its equilibrium polynomial is
    //     the constant 1 (or K_xi/(2 lambda_w) for b), so the incoming flux
    //     is the re-emitted wall Maxwellian; the outgoing member's
    //     equilibrium term is switched off by the multiplier 0;
    //   * a far-field or outflow face's neighbour is a ghost row (rows
    //     nc+1 ... of h and b, refilled every step with the ghost Maxwellian)
    //     whose stencil is itself with coefficient 0, i.e. the ghost value
    //     with zero gradient; the ghost row also enters the least-squares
    //     stencil of the cell that owns the face, as its mirror-ghost row;
    //   * a missing face (cells with 3 faces) repeats face 0 with S/V = 0.
    const int32_t zero_row = (int32_t)nc;
    std::vector<int32_t> ci(nc * CRI, 0);
    std::vector<double> cdr(nc * CRD, 0.0);
    // Stencil slot p of a cell is its face p: the neighbour's row with the
    // least-squares coefficients of that face, the ghost row of a far-field
    // face, or the zero row with coefficient 0 at a wall (the wall ghost is the
    // cell's own value and adds nothing); slots past the cell's faces carry
    // the cell itself with coefficient 0.  So slot p of the cell's own stencil
    // is also the neighbour row read through face p.
    auto stencil = [&](int64_t cell, int32_t* cells, double* G /* [d*4 + s] */) {
      for (int p = 0; p < 4; ++p) {
        int32_t row = (int32_t)cell;
        bool coef = false;
        if (p < nfc[cell]) {
          const int f = cface[cell * MAXF + p];
          const int j = cnbr[cell * MAXF + p];
          if (j >= 0) {
            row = j;
            coef = true;
          } else if (ghost_row[f] >= 0) {
            row = ghost_row[f];
            coef = true;
          } else {
            row = zero_row;
          }
        }
        cells[p] = row;
        for (int d = 0; d < 3; ++d) G[d * 4 + p] = coef ? lsG[(cell * 3 + d) * MAXF + p] : 0.0;
      }
    };
    for (int64_t i = 0; i < nc; ++i) {
      int32_t* I = &ci[i * CRI];
      double* Dd = &cdr[i * CRD];
      stencil(i, &I[CI_OWN], &Dd[CD_G]);
      for (int p = 0; p < 4; ++p) {
        const int pp = p < nfc[i] ? p : 0;
        double* fd = &Dd[CD_F0 + CD_FS * p];
        const int f = cface[i * MAXF + pp];
        const double sg = csign[i * MAXF + pp];
        const int j = cnbr[i * MAXF + pp];
        I[CI_FACE + p] = f;
        I[CI_KIND + p] = fbc[f];
        const int32_t gr = ghost_row[f];
        if (j >= 0) {
          // the neighbour's stencil with this cell's row (through the shared
          // face) moved to slot 0: the sweep reads that value from registers
          int32_t rows[4];
          stencil(j, rows, &fd[6]);
          int q = 0;
          for (int t = 0; t < nfc[j]; ++t)
            if (cface[j * MAXF + t] == f) q = t;
          if (q != 0) {
            std::swap(rows[0], rows[q]);
            for (int d = 0; d < 3; ++d) std::swap(fd[6 + d * 4], fd[6 + d * 4 + q]);
          }
          for (int r = 1; r < 4; ++r) I[CI_RING + 3 * p + r - 1] = rows[r];
        } else {
          // zero or ghost row: its own value with zero gradient
          for (int r = 0; r < 3; ++r) I[CI_RING + 3 * p + r] = gr >= 0 ? gr : zero_row;
        }
        for (int d = 0; d < 3; ++d) {
          Dd[CD_N + 3 * p + d] = sg * fnorm[f * 3 + d];
          fd[0 + d] = sg > 0.0 ? fdxL[f * 3 + d] : fdxR[f * 3 + d];
          fd[3 + d] = j >= 0 ? (sg > 0.0 ? fdxR[f * 3 + d] : fdxL[f * 3 + d]) : 0.0;
        }
        double& sv = fd[19];
        sv = p < nfc[i] ? farea[f] / vol[i] : 0.0;
        // local steps: the face's integral over dt, applied for dt_i
        if (lts && p < nfc[i]) sv *= dtc[i] / c->gas.dt;
        // equilibrium term of the outgoing member: none at a wall
        fd[18] = (j >= 0 || gr >= 0) ? 1.0 : 0.0;
      }
    }
    c->fmesh.crec_i = upload(c, ci);
    c->fmesh.crec_d = upload(c, cdr);
    if (prec == UGKS_FP32) c->fmesh.crec_d32 = upload(c, std::vector<float>(cdr.begin(), cdr.end()));
    if (lim) {
      // Limiter record (reading R7): what the sweep needs beyond the stencil
      // to limit the cell's gradient and each neighbour's.
      std::vector<double> lr(nc * CRL, 0.0);
      auto eps2_of = [&](int64_t cell) { return std::pow(limk * std::pow(vol[cell], 1.0 / D), 3); };
      auto wall_slot = [&](int64_t cell, int p) {
        if (p >= nfc[cell]) return false;
        return cnbr[cell * MAXF + p] < 0 && ghost_row[cface[cell * MAXF + p]] < 0;
      };
      for (int64_t i = 0; i < nc; ++i) {
        double* Lr = &lr[i * CRL];
        Lr[0] = eps2_of(i);
        for (int p = 0; p < 4; ++p) Lr[1 + p] = wall_slot(i, p) ? 1.0 : 0.0;
        for (int p = 0; p < 4 && p < nfc[i]; ++p) {
          const int f = cface[i * MAXF + p];
          const int j = cnbr[i * MAXF + p];
          if (j < 0) continue;  // wall or ghost: the incoming side has no gradient
          double* Fr = &Lr[CRL_F0 + CRL_FS * p];
          Fr[0] = eps2_of(j);
          // the neighbour's slots in record order: the shared face at slot 0
          int order[4] = {0, 1, 2, 3};
          for (int t = 0; t < nfc[j]; ++t)
            if (cface[j * MAXF + t] == f) std::swap(order[0], order[t]);
          for (int r = 0; r < 4; ++r) {
            const int t = order[r];
            Fr[1 + r] = wall_slot(j, t) ? 1.0 : 0.0;
            if (t >= nfc[j]) continue;
            const int fj = cface[j * MAXF + t];
            const bool left = csign[j * MAXF + t] > 0.0;
            for (int d = 0; d < 3; ++d) Fr[5 + 3 * r + d] = left ? fdxL[fj * 3 + d] : fdxR[fj * 3 + d];
          }
        }
      }
      c->fmesh.crec_l = upload(c, lr);
      if (prec == UGKS_FP32) c->fmesh.crec_l32 = upload(c, std::vector<float>(lr.begin(), lr.end()));
    }
  }
  c->cell_perm = perm;
  c->cell_dev = upload(c, std::vector<int32_t>(perm.begin(), perm.end()));
  c->vel_dev = upload(c, std::vector<int32_t>(c->vel_perm.begin(), c->vel_perm.end()));
  c->face_perm.resize(nf);
  for (int64_t f = 0; f < nf; ++f) c->face_perm[f] = f;

  StepBuffers& B = c->buf;
  const size_t esz = prec == UGKS_FP32 ? sizeof(float) : sizeof(double);
  const int NW = D + 2;
  B.W = dalloc<double>(c, nc * NW);
  B.Wn = dalloc<double>(c, nc * NW);
  B.prim = dalloc<double>(c, nc * NPRIM);
  B.primn = dalloc<double>(c, nc * NPRIM);
  B.q = dalloc<double>(c, nc * 3);
  B.qn = dalloc<double>(c, nc * 3);
  B.gW = dalloc<double>(c, nc * 15);
  B.frec = dalloc<double>(c, nf * FREC);
  B.F = dalloc<double>(c, nf * 5);
  if (c->fused) {
    const int64_t npairs = c->fmesh.half;
    // Whole cells per work-group, unless the caller fixes a velocity block or
    // the cells are too few for the GPU and a cell has more than one block of
    // 4096 velocities
    int64_t cp = Bv ? Bv / 2 : 2048;
    cp = std::max<int64_t>(std::min<int64_t>(32, npairs), std::min<int64_t>(cp, npairs));
    c->sched.whole = cp >= npairs || (!Bv && nc >= kWholeCells) ? 1 : 0;
    if (c->sched.whole) cp = npairs;
    c->sched.lanes = cell_lanes(nc, npairs, prec, false);
    c->sched.chunk_pairs = cp;
    c->sched.nchunk = (npairs + cp - 1) / cp;
    c->sched.tile = tile ? tile : 32;
    c->Bv = (int)(2 * cp);
    if (!c->sched.whole) B.dW = dalloc<double>(c, nc * c->sched.nchunk * 5);
    B.srec = dalloc<char>(c, (size_t)nf * c->nr * SREC * esz);
    B.cs = dalloc<char>(c, (size_t)nc * c->nr * SREC * esz);
  } else if (c->wide) {
    B.srec = dalloc<double>(c, (size_t)nf * c->nr * SREC);
    B.cs = dalloc<double>(c, (size_t)nc * c->nr * SREC);
  } else {
    B.dW = dalloc<double>(c, nc * 5);
  }
  // row nc of h and b stays zero: the fused sweep's wall faces read it;
  // rows nc+1 ... are the fused sweep's far-field ghost rows.  On the fused
  // path h and ht (b and bt) trade places every step, so both have them.
  // (Wide cells' ghost rows in the FP32 form are FP64 arrays of their own.)
  const bool apart = c->wide && prec == UGKS_FP32;
  const int64_t rows = nc + 1 + (c->slots() && !apart ? c->fmesh.nff : 0), trows = c->slots() ? rows : nc;
  B.h = dalloc<char>(c, (size_t)rows * nvp * esz);
  B.ht = dalloc<char>(c, (size_t)trows * nvp * esz);
  B.b = c->nr == 2 ? (void*)dalloc<char>(c, (size_t)rows * nvp * esz) : nullptr;
  B.bt = c->nr == 2 ? (void*)dalloc<char>(c, (size_t)trows * nvp * esz) : nullptr;
  // The initial state and each step write every slot of the cells' rows, but for
  // the pads that a step of a sparse set leaves out.
  auto clear = [&](void* f, int64_t from, int64_t to) {
    if (f && to > from)
      HIP_TRY(hipMemsetAsync((char*)f + (size_t)from * nvp * esz, 0, (size_t)(to - from) * nvp * esz, c->stream));
  };
  clear(B.h, nc, rows);
  clear(B.b, nc, rows);
  if (c->slots()) {
    clear(B.ht, c->fmesh.sparse ? 0 : nc, rows);
    clear(B.bt, c->fmesh.sparse ? 0 : nc, rows);
  }
  if (!c->fused) {
    // the staged sweep keeps every gradient and microscopic flux in HBM, the
    // wide cells' step the gradients
    B.gradh = dalloc<double>(c, (size_t)nc * 3 * nvp);
    B.gradb = c->nr == 2 ? dalloc<double>(c, (size_t)nc * 3 * nvp) : nullptr;
  }
  if (apart && c->fmesh.nff) {
    B.ghosth = dalloc<double>(c, (size_t)c->fmesh.nff * nvp);
    B.ghostb = c->nr == 2 ? dalloc<double>(c, (size_t)c->fmesh.nff * nvp) : nullptr;
  }
  if (!c->slots()) {
    B.fluxh = dalloc<double>(c, (size_t)nf * nvp);
    B.fluxb = c->nr == 2 ? dalloc<double>(c, (size_t)nf * nvp) : nullptr;
  }
  B.resid = dalloc<double>(c, kStatus);
  B.cellred = dalloc<double>(c, nc * 3);
  B.flag = (int32_t*)(B.resid + 8);
  B.bflux = dalloc<double>(c, 5);
  HIP_TRY(hipMemsetAsync(B.frec, 0, nf * FREC * sizeof(double), c->stream));
  HIP_TRY(hipMemsetAsync(B.F, 0, nf * 5 * sizeof(double), c->stream));
  HIP_TRY(hipMemsetAsync(B.resid, 0, kStatus * sizeof(double), c->stream));
  HIP_TRY(hipMemsetAsync(B.bflux, 0, 5 * sizeof(double), c->stream));
  // Results go to the caller through pinned memory: to pageable memory each copy
  // is a wait of its own (a one-step call of 1,024 cells x 28^2 and its W: 108 us
  // with three such copies, 86 with two pinned ones).  Larger states are copied
  // at full rate either way.
  // (The cases of a batch share one piece of it.)
  c->host_room = nc * NW * 8 <= kPinnedCells ? nc * std::max(NW, 3) : 0;
  if (host) HIP_TRY(hipHostMalloc((void**)&c->host, (kStatus + c->host_room) * sizeof(double), hipHostMallocDefault));
  HIP_TRY(hipMemsetAsync(B.q, 0, nc * 3 * sizeof(double), c->stream));
  std::vector<double> W0p(nc * NW);
  for (int64_t i = 0; i < nc; ++i)
    for (int x = 0; x < NW; ++x) W0p[i * NW + x] = W0[perm[i] * NW + x];
  HIP_TRY(hipMemcpy(B.W, W0p.data(), nc * NW * sizeof(double), hipMemcpyHostToDevice));

  // ---- initial distributions: the reduced Maxwellian of W0 ---------------
  HIP_TRY(launch_prims(D, m, c->gas, B.W, B.prim, B.flag, 0, c->stream));
  HIP_TRY(launch_init_maxwellian(D, prec, m, v, B.prim, B.h, B.b, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
}

int set_err(ugks_ctx* c, int code, const std::string& msg) {
  if (c) c->err = msg;
  else g_create_error = msg;
  return code;
}

// Kernel kinds timed by ugks_profile_enable.
enum KernelKind {
  KK_PRIMS, KK_HEATFLUX, KK_GRADW, KK_FACE_EQ, KK_WALL, KK_SWEEP, KK_STAGE1, KK_GRAD_MICRO,
  KK_FLUX, KK_MACRO, KK_STAGE2, KK_RESID, KK_COMMIT, KK_COUNT
};
const char* const kKernelNames[KK_COUNT] = {
    "cell_prims", "heat_flux", "macro_gradient", "face_equilibrium", "wall_density",
    "sweep", "stage1", "micro_gradient", "face_flux", "macro_update", "stage2", "residual",
    "commit"};

hipEvent_t take_event(ugks_ctx* c) {
  if (!c->event_pool.empty()) {
    hipEvent_t e = c->event_pool.back();
    c->event_pool.pop_back();
    return e;
  }
  hipEvent_t e;
  HIP_TRY(hipEventCreate(&e));
  return e;
}

// Records an event pair around one launch when profiling is on.
struct Timed {
  ugks_ctx* c;
  int kind;
  hipEvent_t a = nullptr;
  Timed(ugks_ctx* c_, int k) : c(c_), kind(k) {
    if (c->profiling) {
      a = take_event(c);
      HIP_TRY(hipEventRecord(a, c->stream));
    }
  }
  ~Timed() noexcept(false) {
    // no second record while a failed launch is unwinding
    if (c->profiling && a && std::uncaught_exceptions() == 0) {
      hipEvent_t b = take_event(c);
      HIP_TRY(hipEventRecord(b, c->stream));
      c->prof_events.push_back({kind, {a, b}});
    }
  }
};
#define TIMED(kind, call)        \
  do {                           \
    Timed _t(c, kind);           \
    HIP_TRY(call);               \
  } while (0)

// The buffers that a step of the fused path leaves in each other's place.
void swap_buffers(StepBuffers& B) {
  std::swap(B.W, B.Wn);
  std::swap(B.q, B.qn);
  std::swap(B.h, B.ht);
  std::swap(B.b, B.bt);
}

// One time step of the fused path, enqueued.  (wide cells: from stored
// gradients, and the face fluxes only where they are asked for)
void enqueue_step_fused(ugks_ctx* c, bool residual, bool face_flux) {
  const int D = c->D, P = c->prec, R = c->wide ? UGKS_FP64 : P;  // R: the records' type
  const DevMesh& m = c->mesh;
  const DevVel& v = c->vel;
  const GasP& g = c->gas;
  StepBuffers& B = c->buf;
  hipStream_t s = c->stream;
  // 2 heat flux of h^n: left by the previous step once valid
  if (!c->q_valid) {
    TIMED(KK_PRIMS, launch_prims(D, m, g, B.W, B.prim, B.flag, 1, s));
    TIMED(KK_HEATFLUX, launch_heatflux(D, P, m, v, B.h, B.b, B.prim, B.q, B.flag, s));
    c->q_valid = true;
  }
  // 1 primitives of W^n and the cell equilibrium data of the first stage:
  // left by the previous step once valid
  if (!c->cs_valid)
    TIMED(KK_PRIMS, launch_cell_prep(D, R, c->nr, c->nc, g, B.W, B.q, B.prim, B.cs, B.flag, s));
  c->cs_valid = true;
  // 4 macroscopic reconstruction; 6.1-6.6 interface equilibrium
  TIMED(KK_GRADW, launch_gradW(D, m, c->bcs, g, B.W, B.gW, B.flag, 1, s));
  TIMED(KK_FACE_EQ, launch_face_eq(D, m, c->bcs, g, B.W, B.gW, B.q, B.frec, R, c->nr, B.srec, B.flag, s));
  // 7 far-field ghost rows (the wall cells' stencils may read them), then
  // the wall densities
  // (in one launch where neither reads what the other writes)
  const bool joint = c->fmesh.nff && c->fmesh.apart && m.nwall && !c->wide;
  if (c->fmesh.nff && B.ghosth)
    TIMED(KK_WALL, launch_ghost_rows(D, UGKS_FP64, c->fmesh, v, B.frec, 0, B.ghosth, B.ghostb, B.flag, s));
  else if (c->fmesh.nff && !joint)
    TIMED(KK_WALL, launch_ghost_rows(D, P, c->fmesh, v, B.frec, m.nc + 1, B.h, B.b, B.flag, s));
  // (with boundary-flux tracking the wall pass also keeps each wall face's flux)
  const bool track = (c->flags & 64) != 0;
  if (c->wide) {
    TIMED(KK_GRAD_MICRO, launch_grad_micro(D, P, m, v, B.frec, B.h, B.b, B.gradh, B.gradb, B.flag, s));
    TIMED(KK_WALL, launch_wall_rho(D, P, m, v, g, B.h, B.gradh, B.frec, B.flag, s));
    if (face_flux || track) TIMED(KK_FLUX, launch_face_flux(D, P, m, c->fmesh, v, g, B, s));
    TIMED(KK_SWEEP, launch_step_wide(D, P, m, c->fmesh, v, g, c->sched, B, s));
    if (track) TIMED(KK_RESID, launch_bflux(D, m, B.frec, B.F, 1, B.bflux, B.flag, s));
    if (residual) TIMED(KK_RESID, launch_residual(m, B.cellred, B.resid, B.flag, s));
    swap_buffers(B);
    return;
  }
  TIMED(KK_WALL, launch_wall_rho_inline(D, P, m, v, c->fmesh, g, B.h, B.b, B.frec, B.flag, s, track, joint));
  if (c->sched.whole) {
    // 5, 6.7-6.8, 8-11: the velocity sweep and the rest of every cell's step
    TIMED(KK_SWEEP, launch_step_cell(D, P, m, c->fmesh, v, g, c->sched, B, s));
  } else {
    // 5, 6.7-6.8, 9: the velocity sweep
    TIMED(KK_SWEEP, launch_sweep(D, P, c->fmesh, v, g, c->sched, B, s));
    // 8 conservative update; 10 new equilibrium (with q^n, reading R17); 11
    // second stage and the heat flux of h^{n+1}
    TIMED(KK_STAGE2, launch_finish(D, P, m, c->fmesh, v, g, c->sched, B, s));
  }
  if (track) TIMED(KK_RESID, launch_bflux(D, m, B.frec, B.F, 0, B.bflux, B.flag, s));
  if (residual) TIMED(KK_RESID, launch_residual(m, B.cellred, B.resid, B.flag, s));
  swap_buffers(B);
}

// The face fluxes of wide cells after a call that failed in the middle: such a
// call had not come to its last step, the one that computes them.  They are the
// failed step's, as the staged sweep leaves them: that step's records again, from
// the kept state.
void face_flux_after_failure(ugks_ctx* c) {
  StepBuffers B = c->buf;
  const int D = c->D, P = c->prec;
  hipStream_t s = c->stream;
  int32_t* const flags = B.flag;
  int32_t* const flag = B.flag = flags + 3;
  hipError_t e = launch_gradW(D, c->mesh, c->bcs, c->gas, B.W, B.gW, flags, 0, s);
  if (e == hipSuccess)
    e = launch_face_eq(D, c->mesh, c->bcs, c->gas, B.W, B.gW, B.q, B.frec, UGKS_FP64, c->nr, B.srec, flag, s);
  if (e == hipSuccess)
    e = B.ghosth ? launch_ghost_rows(D, UGKS_FP64, c->fmesh, c->vel, B.frec, 0, B.ghosth, B.ghostb, flag, s)
                 : launch_ghost_rows(D, P, c->fmesh, c->vel, B.frec, c->nc + 1, B.h, B.b, flag, s);
  if (e == hipSuccess)
    e = launch_grad_micro(D, P, c->mesh, c->vel, B.frec, B.h, B.b, B.gradh, B.gradb, flag, s);
  if (e == hipSuccess) e = launch_wall_rho(D, P, c->mesh, c->vel, c->gas, B.h, B.gradh, B.frec, flag, s);
  if (e == hipSuccess) e = launch_face_flux(D, P, c->mesh, c->fmesh, c->vel, c->gas, B, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) throw HipFail{e, "face fluxes after a failure"};
}

// One time step, enqueued (the one-step algorithm).
void enqueue_step(ugks_ctx* c, bool residual, bool face_flux) {
  if (c->slots()) {
    enqueue_step_fused(c, residual, face_flux);
    return;
  }
  const int D = c->D, P = c->prec;
  const DevMesh& m = c->mesh;
  const DevVel& v = c->vel;
  const GasP& g = c->gas;
  StepBuffers& B = c->buf;
  hipStream_t s = c->stream;
  // 1-2 primitives and heat flux of the current state
  TIMED(KK_PRIMS, launch_prims(D, m, g, B.W, B.prim, B.flag, 1, s));
  TIMED(KK_HEATFLUX, launch_heatflux(D, P, m, v, B.h, B.b, B.prim, B.q, B.flag, s));
  // 3-4 ghost states and macroscopic reconstruction
  TIMED(KK_GRADW, launch_gradW(D, m, c->bcs, g, B.W, B.gW, B.flag, 1, s));
  // 6.1-6.6 interface equilibrium data
  TIMED(KK_FACE_EQ, launch_face_eq(D, m, c->bcs, g, B.W, B.gW, B.q, B.frec, P, c->nr, nullptr, B.flag, s));
  // 5 microscopic reconstruction
  TIMED(KK_GRAD_MICRO, launch_grad_micro(D, P, m, v, B.frec, B.h, B.b, B.gradh, B.gradb, B.flag, s));
  // 7 wall densities
  TIMED(KK_WALL, launch_wall_rho(D, P, m, v, g, B.h, B.gradh, B.frec, B.flag, s));
  // 6.7-6.8 microscopic fluxes and their moments
  TIMED(KK_FLUX, launch_flux(D, P, m, v, g, B.frec, B.h, B.b, B.gradh, B.gradb, B.fluxh, B.fluxb,
                              B.F, B.flag, s));
  // 9 first stage
  TIMED(KK_STAGE1, launch_stage1(D, P, m, v, g, B.prim, B.q, B.h, B.b, B.fluxh, B.fluxb, B.ht,
                                B.bt, B.flag, s));
  // 8 conservative update, 10 new equilibrium
  TIMED(KK_MACRO, launch_macro_update(D, m, g, B.W, B.F, B.Wn, B.cellred, B.flag, s));
  TIMED(KK_PRIMS, launch_prims(D, m, g, B.Wn, B.primn, B.flag, 1, s));
  if (c->flags & 64) TIMED(KK_RESID, launch_bflux(D, m, B.frec, B.F, 1, B.bflux, B.flag, s));
  // 11 second stage
  TIMED(KK_STAGE2, launch_stage2(D, P, m, v, g, B.primn, B.q, B.ht, B.bt, B.h, B.b, B.flag, s));
  // 12 residual, commit W^{n+1}
  if (residual) TIMED(KK_RESID, launch_residual(m, B.cellred, B.resid, B.flag, s));
  TIMED(KK_COMMIT, launch_commit_W(D, m, B.Wn, B.W, B.flag, s));
}

}  // namespace

// ===========================================================================
// Batched form
// ===========================================================================
struct ugks_batch_impl;

namespace {

// Autotuner cache: case shape -> (pairs per work item: the whole set, a column of
// the file; tile cells; time) of the whole-cell form, batch shape list -> lanes
// per work-group and, where the blocked form is the faster one, its pairs per work
// item (else 0).
struct TuneCase {
  int64_t chunk_pairs = 0, tile = 0;
  double us = 0.0;
};
struct TuneBatch {
  int threads = 0;
  int64_t chunk_pairs = 0;
};
std::mutex g_tune_mu;
std::map<std::string, TuneCase> g_tune_case;
std::map<std::string, TuneBatch> g_tune_batch;

// (the w: timed on the whole-cell step.  Files written before there was one have
// keys without it; their entries are loaded and kept, but were measured on other
// kernels and match no case)
std::string case_key(int D, int prec, int threads, int64_t nc, int64_t nv) {
  char buf[128];
  std::snprintf(buf, sizeof buf, "%d %d %d %lld %lld w", D, prec, threads, (long long)nc, (long long)nv);
  return buf;
}

}  // namespace

struct ugks_batch {
  std::vector<ugks_ctx*> cases;
  int D = 0, prec = 64, flags = 0, nr = 1;
  int threads = 256;
  bool blocks = false;  // blocked form: sweep by velocity blocks, rest of the step in a launch of its own
  hipStream_t stream = nullptr;
  bool own_stream = false;
  std::vector<void*> allocations;
  CaseDev* cases_dev[2] = {nullptr, nullptr};  // even / odd step: the buffers a step swaps
  int64_t* offs = nullptr;                    // cell, face, wall, ghost offsets, [4][n+1]
  int32_t* items = nullptr;
  int64_t nitems = 0, grid = 0;
  int64_t ncell = 0, nface = 0, nwall = 0, nff = 0;
  int32_t* flags_dev = nullptr;  // [4*n], after resid_dev in one block
  std::vector<int> odd;          // per case: its state is in the second set of buffers
  std::vector<int64_t> dW_chunks;  // per case: velocity blocks that its dW has room for
  double* resid_dev = nullptr;   // [8*n]
  double* host = nullptr;        // pinned, [kStatus*n]: a copy of both; then what the cases share
  int parity = 0;
  hipGraph_t graph[2] = {nullptr, nullptr};
  hipGraphExec_t exec[2] = {nullptr, nullptr};
  bool use_graph = true, tuned = false;
  int64_t tune_timings = 0, steps_done = 0;
  std::string err;
};

namespace {

thread_local std::string g_batch_create_error;

template <typename T>
T* balloc(ugks_batch* b, size_t n) {
  if (n == 0) n = 1;
  void* p = nullptr;
  hipError_t e = hipMalloc(&p, n * sizeof(T));
  if (e != hipSuccess) throw HipFail{e, "hipMalloc"};
  b->allocations.push_back(p);
  return static_cast<T*>(p);
}

BatchDev batch_dev(const ugks_batch* b, int par) {
  BatchDev bd{};
  bd.cases = b->cases_dev[par];
  bd.n = (int32_t)b->cases.size();
  const int64_t n1 = bd.n + 1;
  bd.cell_off = b->offs;
  bd.face_off = b->offs + n1;
  bd.wall_off = b->offs + 2 * n1;
  bd.ff_off = b->offs + 3 * n1;
  bd.items = b->items;
  bd.nitems = b->nitems;
  return bd;
}

// Device case table of one parity from the sub-contexts' buffers.
void upload_cases(ugks_batch* b) {
  const size_t n = b->cases.size();
  for (int par = 0; par < 2; ++par) {
    std::vector<CaseDev> h(n);
    for (size_t i = 0; i < n; ++i) {
      const ugks_ctx* c = b->cases[i];
      CaseDev& d = h[i];
      d.m = c->mesh;
      d.v = c->vel;
      d.g = c->gas;
      d.fm = c->fmesh;
      d.sc = c->sched;
      d.bcs = c->bcs;
      d.B = c->buf;
      if (par) swap_buffers(d.B);
    }
    if (!b->cases_dev[par]) b->cases_dev[par] = balloc<CaseDev>(b, n);
    HIP_TRY(hipMemcpy(b->cases_dev[par], h.data(), n * sizeof(CaseDev), hipMemcpyHostToDevice));
  }
}

// Work list of the batched step.  The cells of a tile, with one velocity block
// of theirs, go to the XCD queue with the least work so far; queues are
// padded to one length and interleaved so that item w lands on a work-group
// with index = w (mod 8), i.e. on XCD w mod 8.
std::vector<int32_t> work_list(const ugks_batch* b, const std::vector<int64_t>& only) {
  std::vector<std::vector<int32_t>> q(8);
  std::vector<double> load(8, 0.0);
  auto add_case = [&](int64_t ci) {
    const ugks_ctx* c = b->cases[ci];
    const SweepSched& sc = c->sched;
    const int64_t ntile = (c->nc + sc.tile - 1) / sc.tile;
    for (int64_t t = 0; t < ntile; ++t)
      for (int64_t ch = 0; ch < sc.nchunk; ++ch) {
        const int x = (int)(std::min_element(load.begin(), load.end()) - load.begin());
        const int64_t c0 = t * sc.tile, c1 = std::min(c->nc, c0 + sc.tile);
        for (int64_t ic = c0; ic < c1; ++ic) {
          const int32_t item[4] = {(int32_t)ci, (int32_t)ic, (int32_t)ch, 0};
          q[x].insert(q[x].end(), item, item + 4);
        }
        load[x] += (double)(c1 - c0) * (double)std::min(sc.chunk_pairs, c->fmesh.half - ch * sc.chunk_pairs);
      }
  };
  if (only.empty())
    for (int64_t ci = 0; ci < (int64_t)b->cases.size(); ++ci) add_case(ci);
  else
    for (int64_t ci : only) add_case(ci);
  size_t len = 0;
  for (auto& v : q) len = std::max(len, v.size() / 4);
  std::vector<int32_t> out(8 * len * 4, 0);
  for (size_t j = 0; j < len; ++j)
    for (int x = 0; x < 8; ++x) {
      int32_t* o = &out[(8 * j + x) * 4];
      if (j < q[x].size() / 4) std::memcpy(o, &q[x][4 * j], 4 * sizeof(int32_t));
      else o[0] = -1;
    }
  return out;
}

int64_t sweep_grid(const ugks_batch* b, int64_t nitems) {
  int dev = 0, ncu = 0;
  HIP_TRY(hipGetDevice(&dev));
  HIP_TRY(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
  const int per = std::max(1, batch_blocks_per_cu(b->D, b->prec, b->threads, b->blocks));
  int64_t g = (int64_t)ncu * per;
  g = std::min<int64_t>(g, nitems);
  g = std::max<int64_t>(8, g / 8 * 8);
  return g;
}

void set_items(ugks_batch* b, const std::vector<int32_t>& items, int32_t** dst, int64_t* cap) {
  const int64_t n = (int64_t)items.size() / 4;
  if (n > *cap) {
    *dst = balloc<int32_t>(b, items.size());
    *cap = n;
  }
  HIP_TRY(hipMemcpy(*dst, items.data(), items.size() * sizeof(int32_t), hipMemcpyHostToDevice));
}

// 5, 6.7-6.8, 8-11: the velocity sweep and the rest of every cell's step
hipError_t launch_cells(const ugks_batch* b, const BatchDev& bd, int64_t grid) {
  if (b->blocks) return launch_sweep_b(b->D, b->prec, bd, b->ncell, grid, b->threads, b->stream);
  return launch_step_b(b->D, b->prec, bd, grid, b->threads, b->stream);
}

// The phases of one step for every case of the batch.
void enqueue_batch_step(ugks_batch* b, int par) {
  const int D = b->D, P = b->prec;
  const BatchDev bd = batch_dev(b, par);
  hipStream_t s = b->stream;
  // 4 macroscopic reconstruction; 6.1-6.6 interface equilibrium
  HIP_TRY(launch_gradW_b(D, bd, b->ncell, s));
  HIP_TRY(launch_face_eq_b(D, P, bd, b->nface, s));
  // 7 wall densities; far-field ghost rows
  HIP_TRY(launch_ghost_rows_b(D, P, bd, b->nff, s));
  HIP_TRY(launch_wall_rho_b(D, P, bd, b->nwall, s));
  HIP_TRY(launch_cells(b, bd, b->grid));
  // 12 residuals
  if (!(b->flags & 1)) HIP_TRY(launch_residual_b(bd, s));
}

// Average duration of `reps` launches of the batched step over `items`, after
// `warm` that are not counted.  They leave the state alone, but not the cell
// records and the error flags.
double time_sweep(ugks_batch* b, const std::vector<int32_t>& items, int32_t** buf, int64_t* cap, int warm,
                  int reps) {
  upload_cases(b);  // the kernels read each case's schedule from the case table
  set_items(b, items, buf, cap);
  BatchDev bd = batch_dev(b, 0);
  bd.items = *buf;
  bd.nitems = (int64_t)items.size() / 4;
  const int64_t g = sweep_grid(b, bd.nitems);
  hipEvent_t e0, e1;
  HIP_TRY(hipEventCreate(&e0));
  HIP_TRY(hipEventCreate(&e1));
  for (int r = 0; r < warm; ++r) HIP_TRY(launch_cells(b, bd, g));
  HIP_TRY(hipEventRecord(e0, b->stream));
  for (int r = 0; r < reps; ++r) HIP_TRY(launch_cells(b, bd, g));
  HIP_TRY(hipEventRecord(e1, b->stream));
  HIP_TRY(hipEventSynchronize(e1));
  float ms = 0.0f;
  HIP_TRY(hipEventElapsedTime(&ms, e0, e1));
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  b->tune_timings += reps + warm;
  return 1e3 * ms / reps;
}

// Pairs per work item (at least 32, or all) and cells per tile of one case.
void apply_sched(ugks_ctx* c, int64_t chunk_pairs, int64_t tile) {
  const int64_t half = c->fmesh.half;
  chunk_pairs = std::max(std::min<int64_t>(32, half), std::min(chunk_pairs, half));
  c->sched.whole = chunk_pairs == half;
  c->sched.chunk_pairs = chunk_pairs;
  c->sched.nchunk = (half + chunk_pairs - 1) / chunk_pairs;
  c->sched.tile = std::max<int64_t>(1, std::min(tile, c->nc));
  c->Bv = (int)(2 * chunk_pairs);
}
void apply_whole(ugks_ctx* c, int64_t tile) { apply_sched(c, c->fmesh.half, tile); }

// Blocked schedule of every case: the moment sums of its blocks get their room.
constexpr int64_t kBlockTile = 16;
void apply_blocks(ugks_batch* b, int64_t chunk_pairs, int64_t tile) {
  b->blocks = true;
  for (size_t i = 0; i < b->cases.size(); ++i) {
    ugks_ctx* c = b->cases[i];
    apply_sched(c, chunk_pairs, tile);
    if (c->sched.nchunk > b->dW_chunks[i]) {
      c->buf.dW = balloc<double>(b, (size_t)(c->nc * c->sched.nchunk * 5));
      b->dW_chunks[i] = c->sched.nchunk;
    }
  }
}

// Fewest cells of a batch that take the whole-cell form without a look at the
// blocked one.
constexpr int64_t kBatchCells = 8192;
constexpr int kMostBlocks = 32;

// Autotuner: the lanes per work-group by timing the whole batch's step, then each
// case's tile by timing that case's step alone; shapes found in the cache are not
// timed again.  A batch of few cells is timed in the blocked form too, by 2 to 32
// blocks of its largest velocity set.
void autotune(ugks_batch* b) {
  const int64_t n = (int64_t)b->cases.size();
  int32_t* buf = nullptr;
  int64_t cap = 0, half = 0;
  std::string bkey = "batch";
  for (ugks_ctx* c : b->cases) {
    bkey += " " + case_key(b->D, b->prec, 0, c->nc, c->nv);
    half = std::max(half, c->fmesh.half);
  }
  TuneBatch best;
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    auto it = g_tune_batch.find(bkey);
    if (it != g_tune_batch.end()) best = it->second;
  }
  if (!best.threads) {
    double best_t = INFINITY;
    // (another choice has to be faster by more than timings differ)
    auto take = [&](int64_t pairs, bool first) {
      const double t = time_sweep(b, work_list(b, {}), &buf, &cap, first ? 1 : 0, best_t > 300.0 ? 1 : 2);
      if (t < 0.95 * best_t) {
        best_t = t;
        best = {b->threads, pairs};
      }
      return t;
    };
    if (b->ncell < kBatchCells) {  // room for every list that is timed below
      cap = 4 * kBatchCells + 512;
      buf = balloc<int32_t>(b, 4 * (size_t)cap);
    }
    bool blocks_met = false;
    for (int th : {64, 128, 256}) {
      b->threads = th;
      b->blocks = false;
      for (ugks_ctx* c : b->cases) apply_whole(c, 32);
      take(0, th == 64);
      if (b->ncell >= kBatchCells || th == 64) continue;
      // (fewer pairs per block than lanes leave lanes idle, and more items than
      // fill the GPU a few times over gain nothing)
      double before = INFINITY;
      int64_t last = half;
      for (int nb = 2; nb <= kMostBlocks && b->ncell * nb <= 4 * kBatchCells; nb *= 2) {
        const int64_t pairs = ((half + nb - 1) / nb + WAVE - 1) / WAVE * WAVE;
        if (pairs == last || 2 * pairs < th) break;
        last = pairs;
        apply_blocks(b, pairs, kBlockTile);
        const double t = take(pairs, !blocks_met);
        blocks_met = true;
        if (t > 1.1 * before) break;
        before = t;
      }
    }
  }
  b->threads = best.threads;
  if (best.chunk_pairs) {
    apply_blocks(b, best.chunk_pairs, kBlockTile);
  } else {
    b->blocks = false;
    for (int64_t i = 0; i < n; ++i) {
      ugks_ctx* c = b->cases[i];
      const std::string key = case_key(b->D, b->prec, b->threads, c->nc, c->nv);
      TuneCase tc;
      {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        auto it = g_tune_case.find(key);
        if (it != g_tune_case.end()) tc = it->second;
      }
      if (!tc.tile) {
        tc.us = INFINITY;
        for (int64_t tile : {16, 64, 256}) {
          if (tile > 16 && tile / 4 >= c->nc) continue;
          apply_whole(c, tile);
          const double us = time_sweep(b, work_list(b, {i}), &buf, &cap, 1, 3);
          if (us < tc.us) tc = {c->sched.chunk_pairs, c->sched.tile, us};
        }
        std::lock_guard<std::mutex> lk(g_tune_mu);
        g_tune_case[key] = tc;
      }
      apply_whole(c, tc.tile);
    }
  }
  std::lock_guard<std::mutex> lk(g_tune_mu);
  g_tune_batch[bkey] = best;
}

void batch_build(ugks_batch* b, const ugks_case* cases, int32_t n, const ugks_options* opt) {
  fail_if(!cases || n < 1, "need at least one case");
  const int prec = opt && opt->precision ? opt->precision : UGKS_FP64;
  fail_if(prec != UGKS_FP64 && prec != UGKS_FP32, "precision must be 64 or 32");
  const int fixed_bv = opt ? opt->block_v : 0, fixed_tile = opt ? opt->tile_cells : 0;
  fail_if(fixed_bv < 0 || fixed_bv % WAVE != 0, "block_v must be 0 or a positive multiple of 64");
  fail_if(fixed_tile < 0, "tile_cells must be >= 0");
  if (opt && (opt->flags & 128))
    throw std::pair<int, std::string>(UGKS_EUNSUPPORTED,
                                      "the batched form runs one global step (no local time steps)");
  for (int32_t i = 0; i < n; ++i)
    if (cases && cases[i].gas && cases[i].gas->K != 0)
      throw std::pair<int, std::string>(UGKS_EUNSUPPORTED, "case " + std::to_string(i) +
                                        ": the batched form takes monatomic gases (K = 0) only");
  if (opt && opt->limiter)
    throw std::pair<int, std::string>(UGKS_EUNSUPPORTED,
                                      "the batched sweep has no limiter");
  // every case's arguments, and one dimension for all, before any device work
  for (int32_t i = 0; i < n; ++i) {
    const ugks_case& k = cases[i];
    try {
      check_case_args(k.mesh, k.vel, k.gas, k.W0);
    } catch (InvalidArg& e) {
      throw InvalidArg{"case " + std::to_string(i) + ": " + e.msg};
    } catch (std::pair<int, std::string>& e) {
      throw std::pair<int, std::string>(e.first, "case " + std::to_string(i) + ": " + e.second);
    }
    fail_if(k.mesh->dim != cases[0].mesh->dim,
            "case " + std::to_string(i) + ": every case needs the same dimension");
  }
  b->prec = prec;
  b->flags = opt ? opt->flags : 0;
  b->use_graph = !(b->flags & 8);
  if (opt && opt->stream) {
    b->stream = (hipStream_t)opt->stream;
  } else {
    HIP_TRY(hipStreamCreateWithFlags(&b->stream, hipStreamNonBlocking));
    b->own_stream = true;
  }
  b->resid_dev = balloc<double>(b, kStatus * (size_t)n);
  b->flags_dev = (int32_t*)(b->resid_dev + 8 * (size_t)n);
  HIP_TRY(hipMemset(b->flags_dev, 0, 4 * (size_t)n * sizeof(int32_t)));
  HIP_TRY(hipMemset(b->resid_dev, 0, 8 * (size_t)n * sizeof(double)));
  for (int32_t i = 0; i < n; ++i) {
    const ugks_case& k = cases[i];
    ugks_options o{};
    o.precision = prec;
    o.block_v = 0;
    o.tile_cells = 0;
    o.flags = b->flags & ~(2 | 8);
    o.stream = b->stream;
    std::unique_ptr<ugks_ctx> c(new ugks_ctx());
    try {
      build(c.get(), k.mesh, k.vel, k.gas, k.bcs, k.n_bc, k.W0, &o, false);
    } catch (InvalidArg& e) {
      ugks_destroy(c.release());
      throw InvalidArg{"case " + std::to_string(i) + ": " + e.msg};
    } catch (std::pair<int, std::string>& e) {
      ugks_destroy(c.release());
      throw std::pair<int, std::string>(e.first, "case " + std::to_string(i) + ": " + e.second);
    } catch (...) {
      ugks_destroy(c.release());
      throw;
    }
    ugks_ctx* cc = c.release();
    b->cases.push_back(cc);
    if (i == 0) {
      b->D = cc->D;
      b->nr = cc->nr;
    }
    fail_if(cc->D != b->D, "case " + std::to_string(i) + ": every case needs the same dimension");
    if (!cc->fused || cc->fmesh.sparse)
      throw std::pair<int, std::string>(
          UGKS_EUNSUPPORTED, "case " + std::to_string(i) +
                                 ": the batched form needs the fused sweep over a full tensor "
                                 "product velocity set (symmetric nodes, at most 4 faces per cell)");
    // flags and residuals of all cases side by side: one copy reads them all
    cc->buf.flag = b->flags_dev + 4 * i;
    cc->buf.resid = b->resid_dev + 8 * i;
    // heat flux of the initial state
    HIP_TRY(launch_prims(cc->D, cc->mesh, cc->gas, cc->buf.W, cc->buf.prim, cc->buf.flag, 1, b->stream));
    HIP_TRY(launch_heatflux(cc->D, cc->prec, cc->mesh, cc->vel, cc->buf.h, cc->buf.b, cc->buf.prim,
                            cc->buf.q, cc->buf.flag, b->stream));
    cc->q_valid = true;
    apply_whole(cc, 32);
  }
  int64_t room = 0;
  for (ugks_ctx* c : b->cases) room = std::max(room, c->host_room);
  HIP_TRY(hipHostMalloc((void**)&b->host, (kStatus * (n + 1) + room) * sizeof(double), hipHostMallocDefault));
  for (ugks_ctx* c : b->cases) c->host = b->host + kStatus * (int64_t)n;
  b->odd.assign(n, 0);
  b->dW_chunks.assign(n, 0);
  // case-offset tables
  const int64_t n1 = n + 1;
  std::vector<int64_t> off(4 * n1, 0);
  for (int32_t i = 0; i < n; ++i) {
    const ugks_ctx* c = b->cases[i];
    off[i + 1] = off[i] + c->nc;
    off[n1 + i + 1] = off[n1 + i] + c->nf;
    off[2 * n1 + i + 1] = off[2 * n1 + i] + c->mesh.nwall;
    off[3 * n1 + i + 1] = off[3 * n1 + i] + c->fmesh.nff;
  }
  b->ncell = off[n];
  b->nface = off[n1 + n];
  b->nwall = off[2 * n1 + n];
  b->nff = off[3 * n1 + n];
  b->offs = balloc<int64_t>(b, off.size());
  HIP_TRY(hipMemcpy(b->offs, off.data(), off.size() * sizeof(int64_t), hipMemcpyHostToDevice));
  upload_cases(b);
  // the step's phases up to the sweep once, so the autotuner times the step
  // on this batch's own records
  {
    const BatchDev bd = batch_dev(b, 0);
    HIP_TRY(launch_cell_prep_b(b->D, b->prec, bd, b->ncell, b->stream));
    HIP_TRY(launch_gradW_b(b->D, bd, b->ncell, b->stream));
    HIP_TRY(launch_face_eq_b(b->D, b->prec, bd, b->nface, b->stream));
    HIP_TRY(launch_ghost_rows_b(b->D, b->prec, bd, b->nff, b->stream));
    HIP_TRY(launch_wall_rho_b(b->D, b->prec, bd, b->nwall, b->stream));
  }
  HIP_TRY(hipStreamSynchronize(b->stream));
  {
    int32_t f0 = 0;
    std::vector<int32_t> fl(4 * (size_t)n);
    HIP_TRY(hipMemcpy(fl.data(), b->flags_dev, fl.size() * sizeof(int32_t), hipMemcpyDeviceToHost));
    for (int32_t i = 0; i < n; ++i) f0 |= fl[4 * i];
    fail_if(f0 != 0, "non-positive density or temperature in an initial state");
  }
  if (fixed_bv || fixed_tile) {
    b->threads = 256;
    const int64_t tile = fixed_tile ? fixed_tile : 256;
    bool blocks = false;
    for (const ugks_ctx* c : b->cases) blocks = blocks || (fixed_bv && fixed_bv / 2 < c->fmesh.half);
    if (blocks) apply_blocks(b, fixed_bv / 2, tile);
    else
      for (ugks_ctx* c : b->cases) apply_whole(c, tile);
  } else {
    autotune(b);
    b->tuned = true;
    HIP_TRY(hipStreamSynchronize(b->stream));
  }
  // the timed launches' traces: flags, step counts and the first step's records
  HIP_TRY(hipMemset(b->flags_dev, 0, 4 * (size_t)n * sizeof(int32_t)));
  upload_cases(b);
  HIP_TRY(launch_cell_prep_b(b->D, b->prec, batch_dev(b, 0), b->ncell, b->stream));
  const std::vector<int32_t> items = work_list(b, {});
  int64_t cap = 0;
  set_items(b, items, &b->items, &cap);
  b->nitems = (int64_t)items.size() / 4;
  b->grid = sweep_grid(b, b->nitems);
  HIP_TRY(hipStreamSynchronize(b->stream));
  if (b->use_graph) {
    for (int par = 0; par < 2; ++par) {
      HIP_TRY(hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal));
      try {
        enqueue_batch_step(b, par);
      } catch (...) {
        hipGraph_t g = nullptr;
        (void)hipStreamEndCapture(b->stream, &g);
        if (g) (void)hipGraphDestroy(g);
        throw;
      }
      HIP_TRY(hipStreamEndCapture(b->stream, &b->graph[par]));
      HIP_TRY(hipGraphInstantiate(&b->exec[par], b->graph[par], nullptr, nullptr, 0));
    }
  }
}

int batch_err(ugks_batch* b, int code, const std::string& msg) {
  if (b) b->err = msg;
  else g_batch_create_error = msg;
  return code;
}

// h and b between the caller's arrays and the device go through ht in the
// caller's order (between steps it holds nothing that is needed), so that the host
// copies in order: 1,024 cells x 28^2 (h, b, W) 0.73 and 1.2 ms to set and get from
// slots in the caller's order, 1.3 and 1.8 reordered by the CPU, 0.46 and 0.78 so.
// A few values are reordered by the CPU: 16 cells x 8^2 46 us, 78 with the GPU.
constexpr int64_t kFewValues = 1 << 14, kPiece = 1 << 20;  // kPiece: of the FP32 form's conversion

void reorder(ugks_ctx* c, void* own, bool in) {
  HIP_TRY(launch_reorder(c->prec, c->nc, c->nv, c->nvp, c->cell_dev, c->vel_dev, own, c->buf.ht, in, c->stream));
}

// A sparse set's steps leave its pads out: they are 0 in either buffer.
void clear_pads(ugks_ctx* c) {
  const size_t esz = c->prec == UGKS_FP32 ? sizeof(float) : sizeof(double);
  if (c->fmesh.sparse) HIP_TRY(hipMemsetAsync(c->buf.ht, 0, (size_t)c->nc * c->nvp * esz, c->stream));
}

template <typename T>
void read_rows(ugks_ctx* c, void* src, double* dst) {
  const int64_t n = c->nc * c->nv;
  if (n <= kFewValues) {
    std::vector<T> tmp(c->nc * c->nvp);
    HIP_TRY(hipMemcpy(tmp.data(), src, tmp.size() * sizeof(T), hipMemcpyDeviceToHost));
    for (int64_t i = 0; i < c->nc; ++i)
      for (int64_t k = 0; k < c->nvp; ++k)
        if (c->vel_perm[k] >= 0) dst[c->cell_perm[i] * c->nv + c->vel_perm[k]] = tmp[i * c->nvp + k];
    return;
  }
  reorder(c, src, false);
  if (sizeof(T) == sizeof(double)) {
    HIP_TRY(hipMemcpyAsync(dst, c->buf.ht, n * sizeof(T), hipMemcpyDeviceToHost, c->stream));
  } else {
    std::vector<T> tmp(std::min(n, kPiece));
    for (int64_t i = 0; i < n; i += kPiece) {
      const int64_t m = std::min(n - i, kPiece);
      HIP_TRY(hipMemcpyAsync(tmp.data(), (const T*)c->buf.ht + i, m * sizeof(T), hipMemcpyDeviceToHost, c->stream));
      HIP_TRY(hipStreamSynchronize(c->stream));
      std::copy(tmp.begin(), tmp.begin() + m, dst + i);
    }
  }
  clear_pads(c);
  HIP_TRY(hipStreamSynchronize(c->stream));
}

template <typename T>
void write_rows(ugks_ctx* c, const double* src, void* dst) {
  const int64_t n = c->nc * c->nv;
  if (n <= kFewValues) {
    std::vector<T> tmp(c->nc * c->nvp, T(0));
    for (int64_t i = 0; i < c->nc; ++i)
      for (int64_t k = 0; k < c->nvp; ++k)
        if (c->vel_perm[k] >= 0) tmp[i * c->nvp + k] = (T)src[c->cell_perm[i] * c->nv + c->vel_perm[k]];
    HIP_TRY(hipMemcpy(dst, tmp.data(), tmp.size() * sizeof(T), hipMemcpyHostToDevice));
    return;
  }
  if (sizeof(T) == sizeof(double)) {
    HIP_TRY(hipMemcpy(c->buf.ht, src, n * sizeof(T), hipMemcpyHostToDevice));
  } else {
    std::vector<T> tmp(std::min(n, kPiece));
    for (int64_t i = 0; i < n; i += kPiece) {
      const int64_t m = std::min(n - i, kPiece);
      for (int64_t j = 0; j < m; ++j) tmp[j] = (T)src[i + j];
      HIP_TRY(hipMemcpy((T*)c->buf.ht + i, tmp.data(), m * sizeof(T), hipMemcpyHostToDevice));
    }
  }
  reorder(c, dst, true);
  clear_pads(c);
  HIP_TRY(hipStreamSynchronize(c->stream));
}

}  // namespace


extern "C" {

int ugks_create(const ugks_mesh* mesh, const ugks_velocity* vel, const ugks_gas* gas,
                const ugks_bc* bcs, int32_t n_bc, const double* W0, const ugks_options* opt,
                ugks_ctx** out) {
  if (!out) return set_err(nullptr, UGKS_EINVAL, "out is NULL");
  Range range("ugks_create");
  std::unique_ptr<ugks_ctx> c(new ugks_ctx());
  try {
    build(c.get(), mesh, vel, gas, bcs, n_bc, W0, opt, true);
  } catch (const InvalidArg& e) {
    ugks_destroy(c.release());
    return set_err(nullptr, UGKS_EINVAL, e.msg);
  } catch (const std::pair<int, std::string>& e) {
    ugks_destroy(c.release());
    return set_err(nullptr, e.first, e.second);
  } catch (const HipFail& e) {
    ugks_destroy(c.release());
    int code = (e.e == hipErrorOutOfMemory) ? UGKS_ENOMEM : UGKS_EHIP;
    return set_err(nullptr, code, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } catch (const std::bad_alloc&) {
    ugks_destroy(c.release());
    return set_err(nullptr, UGKS_ENOMEM, "host memory allocation failed");
  } catch (...) {
    ugks_destroy(c.release());
    return set_err(nullptr, UGKS_EHIP, "internal error");
  }
  *out = c.release();
  return UGKS_OK;
}

namespace {

// The graph of the last step of a call (full: with the residual and wide cells'
// face fluxes), or of two steps that leave those out, from the buffers as they
// are; captured when it is first needed.  Kernels only (no memset or copy).
// A launch of a graph costs the GPU some 5 us: in graphs of one step, each with
// the last one's work, 1,024 cells x 24^2 took 53 us per step and 1,728 hexahedra
// x 16^3 358, where the kernels one by one take 42 and 248; 45 and 251 so.
hipGraphExec_t step_graph(ugks_ctx* c, bool full) {
  if (!c->graph_q0) c->graph_q0 = c->buf.q;
  const int par = c->buf.q == c->graph_q0 ? 0 : 1;
  hipGraphExec_t& exec = c->graph_exec[full][par];
  if (exec) return exec;
  const StepBuffers kept = c->buf;
  hipGraph_t g = nullptr;
  HIP_TRY(hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal));
  try {
    enqueue_step(c, full && !(c->flags & 1), full);
    if (!full) enqueue_step(c, false, false);
  } catch (...) {
    c->buf = kept;
    (void)hipStreamEndCapture(c->stream, &g);
    if (g) (void)hipGraphDestroy(g);
    throw;
  }
  c->buf = kept;
  HIP_TRY(hipStreamEndCapture(c->stream, &g));
  const hipError_t e = hipGraphInstantiate(&exec, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (e != hipSuccess) {
    exec = nullptr;
    throw HipFail{e, "hipGraphInstantiate"};
  }
  return exec;
}

// n steps: replayed from graphs where asked for (flags bit 5) and where that
// applies (not profiling, the heat flux of the current f known, a stream that can
// be captured), else the kernels one by one.  Both run the same kernels with the
// same arguments.
void run_steps(ugks_ctx* c, int32_t n) {
  const bool graphs = (c->flags & 32) && !c->profiling && c->stream != nullptr, nores = c->flags & 1;
  for (int32_t s = 0; s < n;) {
    // the residual is the last step's, in units of the first non-zero change:
    // the steps before the last need it only until that unit is known
    const bool last = s + 1 == n, residual = !nores && (last || !c->resid_set), full = last || residual;
    const bool replay = graphs && c->q_valid && (!c->slots() || c->cs_valid);
    if (replay && full) {
      HIP_TRY(hipGraphLaunch(step_graph(c, true), c->stream));
      if (c->slots()) swap_buffers(c->buf);  // as the fused step does on the host
      s += 1;
    } else if (replay && s + 2 < n) {
      HIP_TRY(hipGraphLaunch(step_graph(c, false), c->stream));
      s += 2;
    } else {
      enqueue_step(c, residual, last);
      s += 1;
    }
  }
}

}  // namespace

int ugks_step(ugks_ctx* c, int32_t n_steps, double* residual_out) {
  if (!c) return set_err(nullptr, UGKS_EINVAL, "ctx is NULL");
  if (n_steps < 0) return set_err(c, UGKS_EINVAL, "n_steps < 0");
  Range range("ugks_step");
  try {
    run_steps(c, n_steps);
    HIP_TRY(hipMemcpyAsync(c->host, c->buf.resid, kStatus * sizeof(double), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    const double* res = c->host;
    int32_t flag[4];
    std::memcpy(flag, c->host + 8, sizeof flag);
    c->resid_set = res[3] != 0.0;
    const int32_t begun = flag[1] - c->begun;
    c->begun = flag[1];
    if (flag[0] | flag[2]) {
      // The state is the one before the step that failed: of the steps begun,
      // all but the last are complete (the fused path swapped its buffers for
      // every step enqueued).  The flag stays set: further steps would repeat
      // the failure.
      const int32_t done = std::max(0, begun - 1);
      if (c->slots() && ((n_steps - done) & 1)) swap_buffers(c->buf);
      if (c->wide && begun > 0 && !(flag[0] & 2)) face_flux_after_failure(c);
      return set_err(c, UGKS_ENUMERIC, "non-positive density or temperature (flag " +
                                           std::to_string(flag[0] | flag[2]) + ")");
    }
    c->steps_done += n_steps;
    if (residual_out) {
      residual_out[0] = res[0];
      residual_out[1] = res[1];
    }
  } catch (const HipFail& e) {
    return set_err(c, UGKS_EHIP, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } UGKS_CATCH_REST(set_err, c)
  return UGKS_OK;
}

int ugks_moments(ugks_ctx* c, int32_t which, double* out, int32_t on_device) {
  if (!c || !out) return set_err(c, UGKS_EINVAL, "null argument");
  const int D = c->D;
  try {
    int64_t ncol = which == 2 ? D : D + 2;
    const int64_t n = c->nc * (which == 2 ? 3 : ncol);
    std::vector<double> pageable(n <= c->host_room ? 0 : n);
    double* lib = pageable.empty() ? c->host + kStatus : pageable.data();
    if (which == 0) {
      HIP_TRY(hipMemcpyAsync(lib, c->buf.W, c->nc * ncol * sizeof(double), hipMemcpyDeviceToHost, c->stream));
    } else if (which == 1) {
      double* tmp = c->buf.Wn;
      HIP_TRY(launch_moments(D, c->prec, c->mesh, c->vel, c->buf.h, c->buf.b, tmp, c->stream));
      HIP_TRY(hipMemcpyAsync(lib, tmp, c->nc * ncol * sizeof(double), hipMemcpyDeviceToHost, c->stream));
    } else if (which == 2) {
      // (of the state that is kept, after a failed call too)
      HIP_TRY(launch_prims(D, c->mesh, c->gas, c->buf.W, c->buf.primn, nullptr, 0, c->stream));
      HIP_TRY(launch_heatflux(D, c->prec, c->mesh, c->vel, c->buf.h, c->buf.b, c->buf.primn, c->buf.qn,
                              c->buf.flag + 3, c->stream));
      HIP_TRY(hipMemcpyAsync(lib, c->buf.qn, c->nc * 3 * sizeof(double), hipMemcpyDeviceToHost, c->stream));
    } else {
      return set_err(c, UGKS_EINVAL, "which must be 0, 1 or 2");
    }
    HIP_TRY(hipStreamSynchronize(c->stream));
    std::vector<double> ordered(on_device ? c->nc * ncol : 0);
    double* user = on_device ? ordered.data() : out;
    int64_t stride = which == 2 ? 3 : ncol;
    for (int64_t i = 0; i < c->nc; ++i)
      for (int64_t x = 0; x < ncol; ++x) user[c->cell_perm[i] * ncol + x] = lib[i * stride + x];
    if (on_device) HIP_TRY(hipMemcpy(out, user, ordered.size() * sizeof(double), hipMemcpyHostToDevice));
  } catch (const HipFail& e) {
    return set_err(c, UGKS_EHIP, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } UGKS_CATCH_REST(set_err, c)
  return UGKS_OK;
}


int ugks_boundary_flux(ugks_ctx* c, double* out, int32_t* complete) {
  if (!c || !out) return set_err(c, UGKS_EINVAL, "null argument");
  if (!(c->flags & 64))
    return set_err(c, UGKS_EINVAL, "boundary-flux tracking is off (options.flags bit 6)");
  try {
    double acc[5];
    HIP_TRY(hipMemcpyAsync(acc, c->buf.bflux, 5 * sizeof(double), hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
    for (int x = 0; x < c->D + 2; ++x) out[x] = acc[x];
    if (complete) *complete = (!c->fused || c->fmesh.nff == 0) ? 1 : 0;
  } catch (const HipFail& e) {
    return set_err(c, UGKS_EHIP, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } UGKS_CATCH_REST(set_err, c)
  return UGKS_OK;
}

int ugks_get_state(ugks_ctx* c, double* W, double* h, double* b) {
  if (!c) return set_err(nullptr, UGKS_EINVAL, "ctx is NULL");
  try {
    if (W) {
      int rc = ugks_moments(c, 0, W, 0);
      if (rc) return rc;
    }
    void* src[2] = {c->buf.h, c->buf.b};
    double* dst[2] = {h, b};
    for (int r = 0; r < 2; ++r) {
      if (!dst[r]) continue;
      if (r >= c->nr) std::fill(b, b + c->nc * c->nv, 0.0);
      else if (c->prec == UGKS_FP32) read_rows<float>(c, src[r], dst[r]);
      else read_rows<double>(c, src[r], dst[r]);
    }
  } catch (const HipFail& e) {
    return set_err(c, UGKS_EHIP, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } UGKS_CATCH_REST(set_err, c)
  return UGKS_OK;
}

int ugks_set_state(ugks_ctx* c, const double* W, const double* h, const double* b) {
  if (!c) return set_err(nullptr, UGKS_EINVAL, "ctx is NULL");
  try {
    const int64_t nc = c->nc;
    const int NW = c->D + 2;
    HIP_TRY(hipStreamSynchronize(c->stream));
    if (W) {
      std::vector<double> lib(nc * NW);
      for (int64_t i = 0; i < nc; ++i)
        for (int x = 0; x < NW; ++x) lib[i * NW + x] = W[c->cell_perm[i] * NW + x];
      HIP_TRY(hipMemcpy(c->buf.W, lib.data(), lib.size() * sizeof(double), hipMemcpyHostToDevice));
    }
    void* dst[2] = {c->buf.h, c->buf.b};
    const double* src[2] = {h, b};
    for (int r = 0; r < c->nr; ++r) {
      if (!src[r]) continue;
      if (c->prec == UGKS_FP32) write_rows<float>(c, src[r], dst[r]);
      else write_rows<double>(c, src[r], dst[r]);
    }
    // a new state restarts the residual normalisation and the boundary-flux
    // sum, and clears a failure
    HIP_TRY(hipMemset(c->buf.bflux, 0, 5 * sizeof(double)));
    c->q_valid = false;
    c->cs_valid = false;
    c->resid_set = false;
    c->begun = 0;
    HIP_TRY(hipMemset(c->buf.resid, 0, kStatus * sizeof(double)));  // (with the flags)
  } catch (const HipFail& e) {
    return set_err(c, UGKS_EHIP, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } UGKS_CATCH_REST(set_err, c)
  return UGKS_OK;
}

int ugks_face_data(ugks_ctx* c, double* F, double* rho_w) {
  if (!c) return set_err(nullptr, UGKS_EINVAL, "ctx is NULL");
  try {
    const int64_t nf = c->nf;
    const int NW = c->D + 2;
    HIP_TRY(hipStreamSynchronize(c->stream));
    if (F) {
      std::vector<double> lib(nf * 5);
      HIP_TRY(hipMemcpy(lib.data(), c->buf.F, lib.size() * sizeof(double), hipMemcpyDeviceToHost));
      for (int64_t f = 0; f < nf; ++f)
        for (int x = 0; x < NW; ++x) F[c->face_perm[f] * NW + x] = lib[f * 5 + x];
    }
    if (rho_w) {
      std::vector<double> lib(nf * FREC);
      HIP_TRY(hipMemcpy(lib.data(), c->buf.frec, lib.size() * sizeof(double), hipMemcpyDeviceToHost));
      std::vector<int32_t> kind(nf);
      HIP_TRY(hipMemcpy(kind.data(), c->mesh.fbc, nf * sizeof(int32_t), hipMemcpyDeviceToHost));
      for (int64_t f = 0; f < nf; ++f)
        rho_w[c->face_perm[f]] = kind[f] == UGKS_BC_WALL ? lib[f * FREC + FR_RHOW] : 0.0;
    }
  } catch (const HipFail& e) {
    return set_err(c, UGKS_EHIP, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } UGKS_CATCH_REST(set_err, c)
  return UGKS_OK;
}

int ugks_info(const ugks_ctx* c, ugks_info_t* out) {
  if (!c || !out) return UGKS_EINVAL;
  out->dim = c->D;
  out->n_r = c->nr;
  out->precision = c->prec;
  out->block_v = c->Bv;
  out->n_cells = c->nc;
  out->n_faces = c->nf;
  out->nv = c->nv;
  out->nv_padded = c->nvp;
  out->dt = c->gas.dt;
  out->steps_done = c->steps_done;
  out->device_bytes = c->bytes;
  out->fused = c->fused ? 1 : 0;
  out->tile_cells = c->fused ? (int32_t)c->sched.tile : 0;
  return UGKS_OK;
}

int ugks_profile_enable(ugks_ctx* c, int32_t on) {
  if (!c) return set_err(nullptr, UGKS_EINVAL, "ctx is NULL");
  try {
    HIP_TRY(hipStreamSynchronize(c->stream));
    for (auto& e : c->prof_events) {
      c->event_pool.push_back(e.second.first);
      c->event_pool.push_back(e.second.second);
    }
    c->prof_events.clear();
    c->profiling = on != 0;
  } catch (const HipFail& e) {
    return set_err(c, UGKS_EHIP, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } UGKS_CATCH_REST(set_err, c)
  return UGKS_OK;
}

int ugks_profile_read(ugks_ctx* c, ugks_kernel_time* out, int32_t max, int32_t* n_out) {
  if (!c) return set_err(nullptr, UGKS_EINVAL, "ctx is NULL");
  try {
    HIP_TRY(hipStreamSynchronize(c->stream));
    double tot[KK_COUNT] = {0};
    int64_t cnt[KK_COUNT] = {0};
    for (auto& e : c->prof_events) {
      float ms = 0.0f;
      HIP_TRY(hipEventElapsedTime(&ms, e.second.first, e.second.second));
      tot[e.first] += ms;
      cnt[e.first] += 1;
    }
    int n = 0;
    for (int k = 0; k < KK_COUNT; ++k) {
      if (!cnt[k]) continue;
      if (out && n < max) {
        std::memset(out[n].name, 0, sizeof(out[n].name));
        std::strncpy(out[n].name, kKernelNames[k], sizeof(out[n].name) - 1);
        out[n].launches = cnt[k];
        out[n].total_ms = tot[k];
      }
      ++n;
    }
    if (n_out) *n_out = n;
  } catch (const HipFail& e) {
    return set_err(c, UGKS_EHIP, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } UGKS_CATCH_REST(set_err, c)
  return UGKS_OK;
}

void ugks_destroy(ugks_ctx* c) {
  if (!c) return;
  if (c->stream) (void)hipStreamSynchronize(c->stream);
  for (auto& of : c->graph_exec)
    for (hipGraphExec_t exec : of)
      if (exec) (void)hipGraphExecDestroy(exec);
  for (auto& e : c->prof_events) {
    (void)hipEventDestroy(e.second.first);
    (void)hipEventDestroy(e.second.second);
  }
  for (hipEvent_t e : c->event_pool) (void)hipEventDestroy(e);
  for (void* p : c->allocations) (void)hipFree(p);
  if (c->host) (void)hipHostFree(c->host);
  if (c->own_stream && c->stream) (void)hipStreamDestroy(c->stream);
  delete c;
}

const char* ugks_last_error(const ugks_ctx* c) {
  return c ? c->err.c_str() : g_create_error.c_str();
}


int ugks_batch_create(const ugks_case* cases, int32_t n_cases, const ugks_options* opt,
                      ugks_batch** out) {
  if (!out) return batch_err(nullptr, UGKS_EINVAL, "out is NULL");
  Range range("ugks_batch_create");
  std::unique_ptr<ugks_batch> b(new ugks_batch());
  try {
    batch_build(b.get(), cases, n_cases, opt);
  } catch (const InvalidArg& e) {
    ugks_batch_destroy(b.release());
    return batch_err(nullptr, UGKS_EINVAL, e.msg);
  } catch (const std::pair<int, std::string>& e) {
    ugks_batch_destroy(b.release());
    return batch_err(nullptr, e.first, e.second);
  } catch (const HipFail& e) {
    ugks_batch_destroy(b.release());
    int code = (e.e == hipErrorOutOfMemory) ? UGKS_ENOMEM : UGKS_EHIP;
    return batch_err(nullptr, code, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } catch (const std::bad_alloc&) {
    ugks_batch_destroy(b.release());
    return batch_err(nullptr, UGKS_ENOMEM, "host memory allocation failed");
  } catch (...) {
    ugks_batch_destroy(b.release());
    return batch_err(nullptr, UGKS_EHIP, "internal error");
  }
  *out = b.release();
  return UGKS_OK;
}

int ugks_batch_step(ugks_batch* b, int32_t n_steps, double* residual_out) {
  if (!b) return batch_err(nullptr, UGKS_EINVAL, "batch is NULL");
  if (n_steps < 0) return batch_err(b, UGKS_EINVAL, "n_steps < 0");
  Range range("ugks_batch_step");
  const size_t n = b->cases.size();
  try {
    for (int32_t s = 0; s < n_steps; ++s) {
      if (b->use_graph) HIP_TRY(hipGraphLaunch(b->exec[b->parity], b->stream));
      else enqueue_batch_step(b, b->parity);
      b->parity ^= 1;
    }
    HIP_TRY(hipMemcpyAsync(b->host, b->resid_dev, kStatus * n * sizeof(double), hipMemcpyDeviceToHost, b->stream));
    HIP_TRY(hipStreamSynchronize(b->stream));
    const double* rs = b->host;
    std::vector<int32_t> fl(4 * n);
    std::memcpy(fl.data(), b->host + 8 * n, fl.size() * sizeof(int32_t));
    // where each case's state is: after the steps it has begun, or before the
    // one that failed
    for (size_t i = 0; i < n; ++i) {
      const bool bad = fl[4 * i] | fl[4 * i + 2];
      b->odd[i] = (bad ? std::max(0, fl[4 * i + 1] - 1) : fl[4 * i + 1]) & 1;
    }
    for (size_t i = 0; i < n; ++i)
      if (fl[4 * i] | fl[4 * i + 2]) {
        return batch_err(b, UGKS_ENUMERIC, "case " + std::to_string(i) +
                                               ": non-positive density or temperature");
      }
    b->steps_done += n_steps;
    for (ugks_ctx* c : b->cases) c->steps_done += n_steps;
    if (residual_out)
      for (size_t i = 0; i < n; ++i) {
        residual_out[2 * i] = rs[8 * i];
        residual_out[2 * i + 1] = rs[8 * i + 1];
      }
  } catch (const HipFail& e) {
    return batch_err(b, UGKS_EHIP, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } UGKS_CATCH_REST(batch_err, b)
  return UGKS_OK;
}

namespace {
// Case i as a context whose buffers hold its current state.
struct CaseView {
  ugks_ctx* c;
  bool odd;
  CaseView(ugks_batch* b, int32_t i) : c(b->cases[i]), odd(b->odd[i] != 0) {
    if (odd) swap_buffers(c->buf);
  }
  ~CaseView() {
    if (odd) swap_buffers(c->buf);
  }
};
}  // namespace

int ugks_batch_moments(ugks_batch* b, int32_t i, int32_t which, double* out, int32_t on_device) {
  if (!b) return batch_err(nullptr, UGKS_EINVAL, "batch is NULL");
  if (i < 0 || i >= (int32_t)b->cases.size()) return batch_err(b, UGKS_EINVAL, "case index out of range");
  CaseView v(b, i);
  int rc = ugks_moments(v.c, which, out, on_device);
  if (rc) batch_err(b, rc, v.c->err);
  return rc;
}

int ugks_batch_get_state(ugks_batch* b, int32_t i, double* W, double* h, double* bb) {
  if (!b) return batch_err(nullptr, UGKS_EINVAL, "batch is NULL");
  if (i < 0 || i >= (int32_t)b->cases.size()) return batch_err(b, UGKS_EINVAL, "case index out of range");
  CaseView v(b, i);
  int rc = ugks_get_state(v.c, W, h, bb);
  if (rc) batch_err(b, rc, v.c->err);
  return rc;
}

int ugks_batch_case_info(ugks_batch* b, int32_t i, ugks_info_t* out) {
  if (!b || !out) return UGKS_EINVAL;
  if (i < 0 || i >= (int32_t)b->cases.size()) return batch_err(b, UGKS_EINVAL, "case index out of range");
  return ugks_info(b->cases[i], out);
}

int ugks_batch_info(const ugks_batch* b, ugks_batch_info_t* out) {
  if (!b || !out) return UGKS_EINVAL;
  out->n_cases = (int32_t)b->cases.size();
  out->dim = b->D;
  out->precision = b->prec;
  out->threads = b->threads;
  out->work_items = b->nitems;
  out->grid = b->grid;
  out->graph = b->use_graph ? 1 : 0;
  out->tuned = b->tuned ? 1 : 0;
  out->tune_timings = b->tune_timings;
  out->steps_done = b->steps_done;
  return UGKS_OK;
}

void ugks_batch_destroy(ugks_batch* b) {
  if (!b) return;
  if (b->stream) (void)hipStreamSynchronize(b->stream);
  for (int par = 0; par < 2; ++par) {
    if (b->exec[par]) (void)hipGraphExecDestroy(b->exec[par]);
    if (b->graph[par]) (void)hipGraphDestroy(b->graph[par]);
  }
  for (ugks_ctx* c : b->cases) {
    c->host = nullptr;  // the batch's
    ugks_destroy(c);
  }
  for (void* p : b->allocations) (void)hipFree(p);
  if (b->host) (void)hipHostFree(b->host);
  if (b->own_stream && b->stream) (void)hipStreamDestroy(b->stream);
  delete b;
}

const char* ugks_batch_last_error(const ugks_batch* b) {
  return b ? b->err.c_str() : g_batch_create_error.c_str();
}

int ugks_autotune_save(const char* path) {
  try {
    if (!path) return UGKS_EINVAL;
    std::lock_guard<std::mutex> lk(g_tune_mu);
    std::ofstream f(path);
    if (!f) return UGKS_EINVAL;
    f << "ugks-autotune 1\n";
    for (auto& e : g_tune_case)
      f << "case " << e.first << " : " << e.second.chunk_pairs << " " << e.second.tile << " "
        << e.second.us << "\n";
    for (auto& e : g_tune_batch) {
      f << e.first << " : " << e.second.threads;
      if (e.second.chunk_pairs) f << " " << e.second.chunk_pairs;
      f << "\n";
    }
    return f.good() ? UGKS_OK : UGKS_EINVAL;
  } catch (...) {
    return UGKS_EHIP;  // no exception crosses the ABI
  }
}

int ugks_autotune_load(const char* path) {
  try {
    if (!path) return UGKS_EINVAL;
    std::ifstream f(path);
    if (!f) return UGKS_EINVAL;
    std::string line;
    if (!std::getline(f, line) || line != "ugks-autotune 1") return UGKS_EINVAL;
    std::map<std::string, TuneCase> cs;
    std::map<std::string, TuneBatch> bs;
    while (std::getline(f, line)) {
      if (line.empty()) continue;
      const size_t sep = line.find(" : ");
      if (sep == std::string::npos) return UGKS_EINVAL;
      const std::string key = line.substr(0, sep);
      std::istringstream val(line.substr(sep + 3));
      if (key.rfind("case ", 0) == 0) {
        TuneCase t;
        if (!(val >> t.chunk_pairs >> t.tile >> t.us) || t.chunk_pairs < 1 || t.tile < 1)
          return UGKS_EINVAL;
        cs[key.substr(5)] = t;
      } else if (key.rfind("batch", 0) == 0) {
        TuneBatch t;
        if (!(val >> t.threads) || (t.threads != 64 && t.threads != 128 && t.threads != 256)) return UGKS_EINVAL;
        if (!(val >> t.chunk_pairs)) t.chunk_pairs = 0;
        if (t.chunk_pairs < 0) return UGKS_EINVAL;
        bs[key] = t;
      } else {
        return UGKS_EINVAL;
      }
    }
    std::lock_guard<std::mutex> lk(g_tune_mu);
    for (auto& e : cs) g_tune_case[e.first] = e.second;
    for (auto& e : bs) g_tune_batch[e.first] = e.second;
    return UGKS_OK;
  } catch (...) {
    return UGKS_EHIP;  // no exception crosses the ABI
  }
}

void ugks_autotune_clear(void) {
  std::lock_guard<std::mutex> lk(g_tune_mu);
  g_tune_case.clear();
  g_tune_batch.clear();
}

}  // extern "C"
