// Internal declarations of the gfx950 UGKS library: the context, device
// records and the kernel launchers.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/ugks.h"

namespace ugks {

constexpr int MAXF = 8;    // faces per cell
constexpr int NPRIM = 8;   // rho, U[3], lambda, tau, p, spare
constexpr int FREC = 48;   // doubles per face record
constexpr int WAVE = 64;

// Face record layout (doubles).  Interior / far-field faces hold the
// interface equilibrium data; wall faces hold the wall Maxwellian data.
enum FaceRec : int {
  FR_C0 = 0,     // rho0 (lambda0/pi)^(D/2)   | wall: (lambda_w/pi)^(D/2)
  FR_LAM = 1,    // lambda0                    | wall: lambda_w
  FR_U = 2,      // U0[3]                      | wall: U_w[3]
  FR_SH = 5,     // 4 (1-Pr) lambda0^2 / (5 rho0)
  FR_Q = 6,      // q0[3]
  FR_G = 9,      // Gamma_1..5
  FR_A = 14,     // a[d][0..4], d < 3 (15)
  FR_AT = 29,    // A[0..4]
  FR_RHOW = 34,  // wall: rho_w (written by the wall pass)
  FR_GRHO = 35,  // ghost: rho_g, U_g[3], lambda_g (far field / outflow)
  FR_GU = 36,
  FR_GLAM = 39,
  FR_GC = 40,    // ghost: rho_g (lambda_g/pi)^(D/2)
  FR_BF = 41,    // wall: the step's flux of mass, momentum, energy (boundary-flux tracking)
};

struct DevMesh {
  int64_t nc, nf;
  // cells
  const double* vol;        // [nc]
  const double* cen;        // [nc*3]
  const int32_t* nfc;       // [nc] faces per cell
  int32_t most;             // faces of the cell with most
  const int32_t* cface;     // [nc*MAXF] face ids
  const int32_t* cnbr;      // [nc*MAXF] neighbour cell, -1 for a boundary face
  const double* csign;      // [nc*MAXF] +1 if the cell is L of the face, -1 if R
  const double* lsG;        // [nc*3*MAXF] least-squares coefficients G[d][p]
  // faces
  const int32_t* ford;      // [nf] the faces in the order of their left cells
  const int32_t* fL;        // [nf]
  const int32_t* fR;        // [nf] (-1 boundary)
  const int32_t* fbc;       // [nf]
  const int32_t* fbcid;     // [nf]
  const double* farea;      // [nf]
  const double* fnorm;      // [nf*3]
  const double* fdxL;       // [nf*3] x_f - x_L
  const double* fdxR;       // [nf*3] x_f - shift - x_R
  const double* fmir;       // [nf*3] mirror ghost offset from L: 2((x_f-x_L).n) n
  const int32_t* walls;     // [nwall] ids of the wall faces
  int64_t nwall;
  int32_t limiter = 0;      // 1: Venkatakrishnan's limiter on every reconstruction gradient
  const double* veps2 = nullptr;  // [nc] its eps^2 = (K V^(1/D))^3
};

// Static per-cell records of the fused sweep (built once at create), laid out
// in the order of their use, so that each step of the sweep's loop reads its
// wave-uniform values in one or two wide scalar loads.
// Integer record (CRI ints per cell):
//   [CI_OWN + s] rows of the own stencil, slot s across face s; [CI_RING + 3p + q]
//   rows 1..3 of the stencil of the neighbour across face p (its row 0 is this
//   cell); [CI_FACE + p] face ids; [CI_KIND + p] face kinds.
// Double record (CRD doubles per cell):
//   [CD_N + 3p + d] outward unit normal of face p;
//   [CD_G + 4d + s] own least-squares coefficients G[d][s];
//   face p at CD_F0 + CD_FS p: [0..2] x_f - x_cell, [3..5] x_f - x_neighbour,
//   [6 + 4d + r] the neighbour's coefficients G[d][r], [18] 1 (0 on a wall: the
//   outgoing member has no equilibrium term), [19] S/V.
constexpr int CRI = 32, CI_OWN = 0, CI_RING = 4, CI_FACE = 16, CI_KIND = 20;
constexpr int CRD = 112, CD_N = 0, CD_G = 16, CD_F0 = 32, CD_FS = 20;
// Limiter record of the fused path (CRL doubles per cell, only with the
// limiter): [0] eps^2 of the cell, [1..4] 1 where own stencil slot s is a
// wall (its row is the zero row; its value for the bounds is the cell's own),
// then per face p at CRL_F0 + CRL_FS p: [0] eps^2 of the neighbour, [1..4]
// the neighbour's wall slots, [5 + 3 r + d] the offset of the neighbour's
// face in its stencil slot r from its centroid (slot order of the record).
constexpr int CRL = 88, CRL_F0 = 8, CRL_FS = 20;
// Records of cells with more than four faces (the wide form of the fused
// step, up to MAXF faces, FP64), in the same arrays with strides CRI and CRD:
//   [WI_ROW + p] the row across face p (a neighbour, the zero row nc at a wall, or
//   nc + 1 + m for ghost row m, in the FP32 form a row of FP64 arrays of their own); [WI_FACE + p]; [WI_KIND + p]; [WI_NF] the cell's faces; [WI_FAR] 1 if one has a ghost row;
//   face p at WD_FS p: [0..2] outward unit normal, [3..5] x_f - x_cell,
//   [6..8] x_f - x_neighbour, [9] as [18] above, [10] S/V.
constexpr int WI_ROW = 0, WI_FACE = 8, WI_KIND = 16, WI_NF = 24, WI_FAR = 25;
constexpr int WD_FS = 12;
static_assert(WD_FS * MAXF <= CRD && WI_FAR < CRI, "records of wide cells");
// Per-step records of the fused path in its compute type, SREC values per
// face or cell and distribution (h, then b where it is carried):
//   face: [0..1] Gamma_1, Gamma_2; cell: [0] dt/(2 tau), [1] K_xi/(2 lambda);
//   [SR_P ...] the equilibrium polynomial c + l.u + u^T Q u + (kappa . u)|u|^2 as
//   c | l (D) | quadratics (xx yy zz xy xz yz, or xx yy xy) | kappa (D).
constexpr int SREC = 16, SR_P = 2;
// Velocity slots of the fused path: mirror pairs are kept as slot k and slot
// half + k (k < half = half a row), the first members ordered by compact blocks
// of the node lattice, so that 64 consecutive slots have mostly one sign of
// u.n.  A point whose mirror is not in the set (or is the point itself) has a
// pad slot there: the mirrored velocity with weight 0; such slots come last, and
// the whole-cell form leaves out the second members of their waves.
struct FusedMesh {
  int64_t nc, nv;
  int na;                   // nodes per velocity axis
  int64_t half;             // mirror pairs with padding (a multiple of 64)
  int64_t full;             // the first of them with a point for either member (up to a multiple of 64)
  const double* axis;       // [na] symmetric 1-D nodes
  const int32_t* vidx;      // [2*half + padding] 16 * node index of every slot, 10 bits per axis, first axis low
  const int32_t* crec_i;    // [nc*CRI]
  const double* crec_d;     // [nc*CRD]
  const float* crec_d32;    // [nc*CRD] FP32 copy (FP32 compute form), else null
  int nr = 1;               // distributions carried (records per face and cell)
  bool sparse = false;      // points on the tensor product of `axis`, not all of it
  const double* crec_l = nullptr;  // [nc*CRL] limiter record, null without the limiter
  const float* crec_l32 = nullptr; // its FP32 copy (FP32 compute form)
  const int32_t* ffaces;    // [nff] far-field / outflow faces; face m owns ghost row nc+1+m
  int64_t nff;
  bool apart = false;              // no wall cell's stencil reads a ghost row
  const int32_t* frow = nullptr;   // wide cells: [nf] the row right of a face (cell, ghost row or zero row)
};

// Schedule of the fused sweep: work item = a cell with all of its velocities
// (whole), or (cell, velocity block of chunk_pairs mirror pairs); tiles of
// `tile` consecutive cells per XCD.
struct SweepSched {
  int32_t whole = 0;      // 1: whole cells
  int32_t lanes = 256;    // lanes per work-group of the whole-cell form
  int64_t tile;           // cells per tile
  int64_t nchunk;         // velocity blocks
  int64_t chunk_pairs;    // mirror pairs per velocity block
};

struct DevVel {
  int64_t nv, nvp;          // points, and slots of a row (pads have weight 0)
  const double* u;          // [3*nvp] SoA: u[d*nvp + k]
  const double* w;          // [nvp]
  const double* u2;         // [nvp]
  // internal and out-of-plane dimensions of the full velocity space,
  // K_xi = K + 3 - D (Eq. Kxi_def); b is carried when K_xi > 0
  double kxi = 0.0;
  int32_t has_b = 0;
};

struct DevBC {
  int32_t kind;
  double rho, U[3], T;
};

struct GasP {
  double Pr, R, Tref, muref, omega, dt;
  double K = 0.0;  // internal degrees of freedom (0: monatomic)
  // local time steps (flags bit 7): per-cell steps dt_i [nc], or null for
  // the global dt everywhere.  Faces always integrate over the global dt.
  const double* dtc = nullptr;
};

// The step cell i advances by.
__host__ __device__ inline double dt_cell(const GasP& g, int64_t i) { return g.dtc ? g.dtc[i] : g.dt; }
// S_f as cell i applies it: times dt_i / dt under local steps
__host__ __device__ inline double area_for(const GasP& g, int64_t i, double S) {
  return g.dtc ? S * (g.dtc[i] / g.dt) : S;
}

constexpr int kStatus = 10;  // doubles of a context's resid and flag

// Kernel launchers (ugks_kernels.hip).  Each returns hipGetLastError().
struct StepBuffers {
  // (on the fused path a step ends with W and Wn, q and qn, h and ht, b and
  // bt trading places)
  double* W;       // [nc*(D+2)] state W^n
  double* Wn;      // [nc*(D+2)] W^{n+1}
  double* prim;    // [nc*NPRIM] of W^n
  double* primn;   // [nc*NPRIM] of W^{n+1} (staged form); readouts' own
  double* q;       // [nc*3] heat flux of h^n
  double* qn;      // [nc*3] heat flux of h^{n+1} (fused path)
  double* gW;      // [nc*3*5]
  double* frec;    // [nf*FREC]
  double* F;       // [nf*5] face fluxes (staged sweep)
  double* dW;      // [nc*nchunk*5] per-(cell, velocity block) net outflow moments (fused sweep)
  // per-step records of the fused path, in its compute type (SREC)
  void* srec;      // [nf*nr*SREC] faces
  void* cs;        // [nc*nr*SREC] cells
  void* h;         // [nc*nvp] storage type
  void* b;         // [nc*nvp] where b is carried
  void* ht;        // [nc*nvp] first-stage result; on the fused path then h^{n+1}
  void* bt;
  double* gradh;   // [nc*3*nvp] microscopic gradients (staged sweep)
  double* gradb;
  double* ghosth;  // [nff*nvp] ghost rows of wide cells in the FP32 form
  double* ghostb;
  double* fluxh;   // [nf*nvp] time-integrated microscopic fluxes (staged sweep)
  double* fluxb;
  double* resid;   // [8] residual accumulators and state, then flag: one block, read back in one copy
  double* bflux;   // [5] running boundary flux (with boundary-flux tracking)
  double* cellred; // [nc*3] per-cell residual contributions
  // [0] numeric error; [1] steps begun without one; [2] numeric error of the
  // whole-cell step now running (taken over into [0] by the next step, so that
  // every wave of that launch sees one value of [0]); [3] always 0: the flag of
  // readouts, which heed no error
  int32_t* flag;
};

// What the rest of a cell's step reads and writes (whole-cell form).
struct CellOut {
  const double *vol, *W, *q;
  double *Wn, *qn, *prim;
  void* cs;
  double* cellred;
  int32_t* flag;
};

// One case of a batch as the batched kernels see it (an array of these in
// device memory; the pointers are the case's own buffers).
struct CaseDev {
  DevMesh m;
  DevVel v;
  GasP g;
  FusedMesh fm;
  SweepSched sc;
  const DevBC* bcs;
  StepBuffers B;
};

// A batch of cases run by one launch per phase: flattened element ranges
// with case-offset tables (prefix sums) and the sweep's work list.
struct BatchDev {
  const CaseDev* cases;     // [n]
  int32_t n;
  const int64_t* cell_off;  // [n+1] cells
  const int64_t* face_off;  // [n+1] faces
  const int64_t* wall_off;  // [n+1] wall faces
  const int64_t* ff_off;    // [n+1] far-field / outflow faces (ghost rows)
  const int32_t* items;     // [4*nitems] work items: case (-1 = padding), cell, velocity block, unused
  int64_t nitems;
};

hipError_t launch_prims(int D, const DevMesh& m, const GasP& g, const double* W, double* prim,
                        int32_t* flag, int checkflag, hipStream_t s);
hipError_t launch_heatflux(int D, int prec, const DevMesh& m, const DevVel& v, const void* h,
                           const void* b, const double* prim, double* q, const int32_t* flag,
                           hipStream_t s);
hipError_t launch_gradW(int D, const DevMesh& m, const DevBC* bcs, const GasP& g, const double* W,
                        double* gW, int32_t* flag, int count, hipStream_t s);
hipError_t launch_face_eq(int D, const DevMesh& m, const DevBC* bcs, const GasP& g,
                          const double* W, const double* gW, const double* q, double* frec,
                          int prec, int nr, void* srec, int32_t* flag, hipStream_t s);
hipError_t launch_grad_micro(int D, int prec, const DevMesh& m, const DevVel& v,
                             const double* frec, const void* h, const void* b, double* gh,
                             double* gb, const int32_t* flag, hipStream_t s);
hipError_t launch_wall_rho(int D, int prec, const DevMesh& m, const DevVel& v, const GasP& g,
                           const void* h, const double* gh, double* frec, const int32_t* flag,
                           hipStream_t s);
hipError_t launch_flux(int D, int prec, const DevMesh& m, const DevVel& v, const GasP& g,
                       const double* frec, const void* h, const void* b, const double* gh,
                       const double* gb, double* fh, double* fb, double* F, const int32_t* flag,
                       hipStream_t s);
hipError_t launch_stage1(int D, int prec, const DevMesh& m, const DevVel& v, const GasP& g,
                         const double* prim, const double* q, const void* h, const void* b,
                         const double* fh, const double* fb, void* ht, void* bt,
                         const int32_t* flag, hipStream_t s);
hipError_t launch_macro_update(int D, const DevMesh& m, const GasP& g, const double* W, const double* F,
                               double* Wn, double* cellred, const int32_t* flag, hipStream_t s);
hipError_t launch_stage2(int D, int prec, const DevMesh& m, const DevVel& v, const GasP& g,
                         const double* primn, const double* q, const void* ht, const void* bt,
                         void* h, void* b, const int32_t* flag, hipStream_t s);
hipError_t launch_residual(const DevMesh& m, const double* cellred, double* resid,
                           const int32_t* flag, hipStream_t s);
hipError_t launch_commit_W(int D, const DevMesh& m, const double* Wn, double* W,
                           const int32_t* flag, hipStream_t s);
hipError_t launch_init_maxwellian(int D, int prec, const DevMesh& m, const DevVel& v,
                                  const double* prim, void* h, void* b, hipStream_t s);
hipError_t launch_moments(int D, int prec, const DevMesh& m, const DevVel& v, const void* h,
                          const void* b, double* out, hipStream_t s);
// rows between slots and the caller's order (in: to the slots)
hipError_t launch_reorder(int prec, int64_t nc, int64_t nv, int64_t nvp, const int32_t* cell, const int32_t* vel,
                          void* own, void* user, bool in, hipStream_t s);
hipError_t launch_dt_cells(int D, const DevMesh& m, const DevVel& v, double* cellval,
                           hipStream_t s);
// fused sweep (ugks_sweep.hip)
hipError_t launch_cell_prep(int D, int prec, int nr, int64_t nc, const GasP& g, const double* W,
                            const double* q, double* prim, void* cs, int32_t* flag, hipStream_t s);
hipError_t launch_sweep(int D, int prec, const FusedMesh& fm, const DevVel& v, const GasP& g,
                        const SweepSched& sc, const StepBuffers& B, hipStream_t s);
hipError_t launch_step_cell(int D, int prec, const DevMesh& m, const FusedMesh& fm, const DevVel& v,
                            const GasP& g, const SweepSched& sc, const StepBuffers& B, hipStream_t s);
// wide cells (more than four faces), from the stored gradients
hipError_t launch_step_wide(int D, int prec, const DevMesh& m, const FusedMesh& fm, const DevVel& v,
                            const GasP& g, const SweepSched& sc, const StepBuffers& B, hipStream_t s);
hipError_t launch_face_flux(int D, int prec, const DevMesh& m, const FusedMesh& fm, const DevVel& v,
                            const GasP& g, const StepBuffers& B, hipStream_t s);
hipError_t launch_finish(int D, int prec, const DevMesh& m, const FusedMesh& fm, const DevVel& v,
                         const GasP& g, const SweepSched& sc, const StepBuffers& B, hipStream_t s);
hipError_t launch_wall_rho_inline(int D, int prec, const DevMesh& m, const DevVel& v,
                                  const FusedMesh& fm, const GasP& g, void* h, void* b, double* frec,
                                  const int32_t* flag, hipStream_t s, bool track, bool ghosts);
hipError_t launch_bflux(int D, const DevMesh& m, const double* frec, const double* F, int staged,
                        double* acc, const int32_t* flag, hipStream_t s);
hipError_t launch_ghost_rows(int D, int prec, const FusedMesh& fm, const DevVel& v,
                             const double* frec, int64_t first, void* h, void* b,
                             const int32_t* flag, hipStream_t s);

// batched forms (one launch per phase over every case of a batch)
hipError_t launch_cell_prep_b(int D, int prec, const BatchDev& bd, int64_t ncell, hipStream_t s);
hipError_t launch_gradW_b(int D, const BatchDev& bd, int64_t ncell, hipStream_t s);
hipError_t launch_face_eq_b(int D, int prec, const BatchDev& bd, int64_t nface, hipStream_t s);
hipError_t launch_wall_rho_b(int D, int prec, const BatchDev& bd, int64_t nwall, hipStream_t s);
hipError_t launch_ghost_rows_b(int D, int prec, const BatchDev& bd, int64_t nff, hipStream_t s);
hipError_t launch_step_b(int D, int prec, const BatchDev& bd, int64_t grid, int threads,
                         hipStream_t s);
// blocked form: the sweep of (case, cell, block) items, then the rest of the step
hipError_t launch_sweep_b(int D, int prec, const BatchDev& bd, int64_t ncell, int64_t grid, int threads,
                          hipStream_t s);
// resident work-groups of either form's sweep per CU at `threads` lanes
int batch_blocks_per_cu(int D, int prec, int threads, bool blocks);
hipError_t launch_residual_b(const BatchDev& bd, hipStream_t s);

}  // namespace ugks

struct ugks_ctx {
  int D = 0, kxi = 0, nr = 0, prec = 64, Bv = 64, flags = 0;
  bool fused = false;       // tensor-product symmetric velocity set, cells of up to four faces
  bool wide = false;        // the same with cells of more faces: gradients stored, one pass per cell
  bool slots() const { return fused || wide; }  // mirror-pair velocity slots, two sets of state buffers
  bool q_valid = false;     // buf.q holds the heat flux of the current h
  bool cs_valid = false;    // buf.prim, buf.cs hold the records of the current W and q
  bool resid_set = false;   // the residual's unit (its first non-zero change) is known
  int32_t begun = 0;        // buf.flag[1] when last read
  // HIP graphs of two steps, and (1) of one with what only the last step of a call
  // computes, each per order of the buffers that a step swaps; graph_q0 is buf.q
  // in the first order
  hipGraphExec_t graph_exec[2][2] = {};
  const double* graph_q0 = nullptr;
  ugks::FusedMesh fmesh{};  // static records of the fused sweep
  ugks::SweepSched sched{};
  int64_t nc = 0, nf = 0, nv = 0, nvp = 0;
  int64_t steps_done = 0;
  ugks::GasP gas{};
  std::vector<int64_t> cell_perm;   // library cell c -> caller cell
  std::vector<int64_t> face_perm;   // library face f -> caller face
  std::vector<int64_t> vel_perm;    // velocity slot k < nvp -> caller velocity (-1: pad)
  const int32_t *cell_dev = nullptr, *vel_dev = nullptr;  // both on the device
  ugks::DevMesh mesh{};
  const double* lsG_exact = nullptr;  // least-squares coefficients even under first-order reconstruction
  ugks::DevVel vel{};
  ugks::DevBC* bcs = nullptr;
  ugks::StepBuffers buf{};
  std::vector<void*> allocations;
  int64_t bytes = 0;
  // Pinned host memory that results are copied through: the status block
  // (kStatus doubles), then room for host_room doubles of cell data (in a batch
  // a piece that its cases share).
  double* host = nullptr;
  int64_t host_room = 0;
  hipStream_t stream = nullptr;
  bool own_stream = false;
  // kernel timing (ugks_profile_enable): event pairs per launch, in order
  bool profiling = false;
  std::vector<std::pair<int, std::pair<hipEvent_t, hipEvent_t>>> prof_events;
  std::vector<hipEvent_t> event_pool;
  std::string err;
};
