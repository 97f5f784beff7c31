// Learned warm start on gfx950: per-cell features, stress / heat-flux
// targets, a 9-64-64-9 tanh network (bf16 MFMA inference, FP32 training
// kernels with Adam) and the Grad-type initial distribution.
//
// The network closes the moment hierarchy the way a Chapman-Enskog
// expansion does (Sec. 2.1: the BGK-Shakhov relaxation toward H+, B+ carries
// the stress and heat flux of f); it maps dimensionless gradients of the
// macroscopic state to sigma/p and q/(p sqrt(2RT)), and the initial f is
// Grad's 13-moment form about the Maxwellian of W built from them.
//
// Inference is one wave per 16 cells on v_mfma_f32_16x16x16_bf16 in the
// transposed form Z^T = W Z_prev^T: a layer's 16x16 output tile (hidden
// units x cells) lands in exactly the register layout the next layer's B
// operand needs, so the three layers chain in registers without LDS.
#include "ugks_device.h"
#include "ugks_host_util.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <mutex>

// Device memory of ugks_mlp_forward_noalloc: a copy of the input rows where a
// caller's output rows overlap them (2.25 MiB).  Each GPU holds its own
// array until the process ends.  Host code never uses this name as an
// address: it takes the device address that hipGetSymbolAddress returns on
// each device.
static __device__ __align__(256) float scratch[UGKS_NOALLOC_MAX_ROWS * 9];

namespace ugks {

using namespace dev;

namespace {

constexpr int NFEAT = 9, NOUT = 9, HID = 64;
constexpr int P_W1 = 0, P_B1 = P_W1 + HID * NFEAT, P_W2 = P_B1 + HID, P_B2 = P_W2 + HID * HID,
              P_W3 = P_B2 + HID, P_B3 = P_W3 + NOUT * HID, NPARAM = P_B3 + NOUT;
static_assert(NPARAM == 5385, "parameter layout");
constexpr int FS = 16;  // padded row of features and outputs (floats)

typedef short short4_t __attribute__((ext_vector_type(4)));
typedef float float4_t __attribute__((ext_vector_type(4)));

// float -> bfloat16 bits, round to nearest, ties to even (finite inputs)
__device__ __forceinline__ short bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (short)(u >> 16);
}

// ---------------------------------------------------------------------------
// Features of every cell from W and its least-squares gradient gW
// (gW[(i*3 + d)*5 + v] = dW_v/dx_d), in FP64, stored as float rows of 16.
template <int D>
__global__ void k_features(int64_t nc, GasP g, const double* __restrict__ W,
                           const double* __restrict__ gW, float* __restrict__ feat) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= nc) return;
  const double* Wi = &W[i * (D + 2)];
  double P[NPRIM];
  const bool ok = prim_of<D>(Wi, g, P);
  float* F = &feat[i * FS];
  for (int j = 0; j < FS; ++j) F[j] = 0.0f;
  if (!ok) {
    F[0] = NAN;  // outside every training box: the cell falls back to the Maxwellian
    return;
  }
  const double rho = P[0], tau = P[5], lam = P[4];
  const double RT = 0.5 / lam;
  const double E = Wi[D + 1] / rho;
  double dU[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};  // dU[d][a] = dU_a/dx_d
  double dTT[3] = {0, 0, 0}, dr[3] = {0, 0, 0};
  for (int d = 0; d < D; ++d) {
    const double* G = &gW[(i * 3 + d) * 5];
    dr[d] = G[0];
    double UdU = 0.0;
    for (int a = 0; a < D; ++a) {
      dU[d][a] = (G[1 + a] - P[1 + a] * G[0]) / rho;
      UdU += P[1 + a] * dU[d][a];
    }
    const double dE = (G[D + 1] - E * G[0]) / rho;
    dTT[d] = (dE - UdU) / (1.5 * RT);
  }
  const double div = dU[0][0] + dU[1][1] + dU[2][2];
  const double L = tau * sqrt(2.0 * RT);
  F[0] = (float)(tau * (dU[0][0] - div / 3.0));
  F[1] = (float)(tau * (dU[1][1] - div / 3.0));
  F[2] = (float)(tau * 0.5 * (dU[0][1] + dU[1][0]));
  F[3] = (float)(tau * 0.5 * (dU[0][2] + dU[2][0]));
  F[4] = (float)(tau * 0.5 * (dU[1][2] + dU[2][1]));
  for (int d = 0; d < 3; ++d) F[5 + d] = (float)(L * dTT[d]);
  F[8] = (float)(L * sqrt(dr[0] * dr[0] + dr[1] * dr[1] + dr[2] * dr[2]) / rho);
}

// Targets of every cell from its distribution: sigma/p (xx yy zz xy xz yz)
// and q/(p sqrt(2RT)), one work-group per cell, sums over velocity in a
// fixed order (wave shuffles, then waves in order).
template <int D, typename T>
__global__ __launch_bounds__(TPB) void k_targets(DevVel v, GasP g, const double* __restrict__ W,
                                                 const T* __restrict__ h, const T* __restrict__ b,
                                                 float* __restrict__ targ) {
  __shared__ double red[9 * 16];
  const int64_t i = blockIdx.x;
  double P[NPRIM];
  prim_of<D>(&W[i * (D + 2)], g, P);
  const double p = P[6], RT = 0.5 / P[4];
  double acc[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};  // Pxx Pyy Pzz Pxy Pxz Pyz qx qy qz
  for (int64_t k = threadIdx.x; k < v.nvp; k += TPB) {
    double c[3] = {0, 0, 0};
    double c2 = 0.0;
    for (int d = 0; d < D; ++d) {
      c[d] = v.u[d * v.nvp + k] - P[1 + d];
      c2 += c[d] * c[d];
    }
    const double wk = v.w[k];
    const double hk = wk * ld(h, i * v.nvp + k);
    const double bk = D == 2 ? wk * ld(b, i * v.nvp + k) : 0.0;
    acc[0] += c[0] * c[0] * hk;
    acc[1] += c[1] * c[1] * hk;
    acc[2] += D == 2 ? bk : c[2] * c[2] * hk;
    acc[3] += c[0] * c[1] * hk;
    acc[4] += c[0] * c[2] * hk;
    acc[5] += c[1] * c[2] * hk;
    const double e = c2 * hk + bk;
    for (int d = 0; d < 3; ++d) acc[6 + d] += 0.5 * c[d] * e;
  }
  block_sum<9>(acc, red);
  if (threadIdx.x == 0) {
    float* o = &targ[i * FS];
    for (int j = 0; j < FS; ++j) o[j] = 0.0f;
    for (int j = 0; j < 6; ++j) o[j] = (float)((acc[j] - (j < 3 ? p : 0.0)) / p);
    const double s = p * sqrt(2.0 * RT);
    for (int d = 0; d < 3; ++d) o[6 + d] = (float)(acc[6 + d] / s);
  }
}

// ---------------------------------------------------------------------------
// Network inference: y = out_scale * N(in_scale * x), N with bf16 weights and
// layer inputs, FP32 accumulation, FP32 biases and tanh.  One wave per tile
// of 16 rows; pb holds the weights as bf16, each matrix zero-padded to
// whole 16x16 tiles: W1 64x16, W2 64x64, W3 16x64.
struct MlpDev {
  const short* w1;     // [64*16]
  const short* w2;     // [64*64]
  const short* w3;     // [16*64]
  const float* p;      // FP32 parameters (biases read from here)
  const float* in_scale;
  const float* out_scale;
};

// Rows of x and y are xs and ys floats apart: the caller's dense rows of 9 are
// read and written in place, without staging copies.  A call of a few
// thousand rows is bound by its fixed latency (weights, one tile per wave,
// the launch), so the weights come in 8-byte pieces.  Measured on 11,520 rows:
// 9.4 us per call with padded staging rows before and after (three kernels),
// 4.3 us in place.
__global__ __launch_bounds__(256) void k_mlp_infer(MlpDev net, const float* x, int xs, int64_t n,
                                                   float* y, int ys) {
  const int lane = threadIdx.x & 63;
  const int row = lane & 15, grp = lane >> 4;  // A: row i = lane%16, k = 4*(lane/16)+e
  // weights of this lane, per 16x16 tile
  short4_t a1[4], a2[4][4], a3[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    a1[t] = *(const short4_t*)&net.w1[(16 * t + row) * 16 + 4 * grp];
#pragma unroll
    for (int s = 0; s < 4; ++s) a2[t][s] = *(const short4_t*)&net.w2[(16 * t + row) * 64 + 16 * s + 4 * grp];
    a3[t] = *(const short4_t*)&net.w3[row * 64 + 16 * t + 4 * grp];
  }
  // biases in the output layout: D[unit = 4*(lane/16)+r][cell = lane%16]
  float4_t c1[4], c2[4], c3;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    c1[t] = *(const float4_t*)&net.p[P_B1 + 16 * t + 4 * grp];
    c2[t] = *(const float4_t*)&net.p[P_B2 + 16 * t + 4 * grp];
  }
  float si[4], so[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int u = 4 * grp + r;
    c3[r] = u < NOUT ? net.p[P_B3 + u] : 0.0f;
    si[r] = u < NFEAT ? net.in_scale[u] : 0.0f;
    so[r] = u < NOUT ? net.out_scale[u] : 0.0f;
  }
  const int64_t ntile = (n + 15) / 16;
  const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  const int64_t nwave = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t tile = wave; tile < ntile; tile += nwave) {
    const int64_t cell = tile * 16 + row;  // B operand / output column of this lane
    const bool live = cell < n;
    // B = X^T: features 4*grp .. 4*grp+3 of this lane's cell
    short4_t bx;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int f = 4 * grp + e;
      const float v = (live && f < NFEAT) ? x[cell * xs + f] * si[e] : 0.0f;
      bx[e] = bf16_bits(v);
    }
    short4_t b2[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      float4_t z = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a1[t], bx, c1[t], 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) b2[t][r] = bf16_bits(tanhf(z[r]));
    }
    short4_t b3[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      float4_t z = c2[t];
#pragma unroll
      for (int s = 0; s < 4; ++s) z = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a2[t][s], b2[s], z, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) b3[t][r] = bf16_bits(tanhf(z[r]));
    }
    float4_t z = c3;
#pragma unroll
    for (int s = 0; s < 4; ++s) z = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a3[s], b3[s], z, 0, 0, 0);
    if (live)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int u = 4 * grp + r;
        if (u < NOUT) y[cell * ys + u] = z[r] * so[r];
      }
  }
}

__global__ void k_copy_rows(const float* x, int64_t n, float* y) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t < n) y[t] = x[t];
}

// FP32 parameters -> the padded bf16 tiles of k_mlp_infer
__global__ void k_mlp_pack(const float* __restrict__ p, short* __restrict__ w1,
                           short* __restrict__ w2, short* __restrict__ w3) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < 64 * 16) {
    const int j = t / 16, k = t % 16;
    w1[t] = k < NFEAT ? bf16_bits(p[P_W1 + j * NFEAT + k]) : (short)0;
  }
  if (t < 64 * 64) w2[t] = bf16_bits(p[P_W2 + t]);
  if (t < 16 * 64) {
    const int j = t / 64, k = t % 64;
    w3[t] = j < NOUT ? bf16_bits(p[P_W3 + j * HID + k]) : (short)0;
  }
}

// ---------------------------------------------------------------------------
// Training, FP32, two kernels per step: k_mlp_grad leaves one partial
// gradient per work-group, k_mlp_adam adds the partials in order and updates.
//
// k_mlp_grad: a work-group takes tiles of 16 samples through forward, loss and
// back-propagation on v_mfma_f32_16x16x4_f32 (FP32 inputs and sums).  Wave w
// owns hidden units 16w..16w+15 of both layers; activations and layer errors
// pass between waves through LDS ([unit][sample], rows padded to 17 floats),
// weights and the partial gradient stay in registers for the whole kernel.
// A step of 1,024 samples is 31 MFLOP: it is bound by latency, not by
// arithmetic, so the split is the finest the tile allows (64 work-groups at
// 1,024 samples), and nothing but the 5,385 partial sums per work-group goes
// through memory.  Measured per step of 1,024 samples, both kernels:
// 13 us (10 + 3) against 171 us for one sample per lane with its layers in
// scratch and a second pass over stored activations.
constexpr int TS = 16;           // samples per tile
constexpr int TP = TS + 1;       // padded row of an LDS tile
constexpr int64_t MAX_WG = 128;  // most partial gradients of one step

// hidden unit (or input) of step kk for lane group g: each lane's four
// consecutive steps are four consecutive floats of its weight row
__device__ __forceinline__ int unit_of(int kk, int g) { return 16 * (kk >> 2) + 4 * g + (kk & 3); }

__global__ __launch_bounds__(256) void k_mlp_grad(const float* __restrict__ p,
                                                  const float* __restrict__ in_scale,
                                                  const float* __restrict__ out_scale,
                                                  const float* __restrict__ x,
                                                  const float* __restrict__ t, int64_t n,
                                                  float* __restrict__ partial,
                                                  double* __restrict__ lossp) {
  // X: features, a row of ones (its products are the first layer's biases), zeros
  __shared__ float X[16][TP], A1[HID][TP], A2[HID][TP], D1[HID][TP], D2[HID][TP], DY[16][TP];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i = lane & 15, g = lane >> 4;
  const int mine = 16 * w + i;  // this lane's row of an A operand
  float w1[3], w2[16], w2t[16], w3[16], w3t[4];
#pragma unroll
  for (int kk = 0; kk < 3; ++kk) {
    const int k = 4 * kk + g;
    w1[kk] = k < NFEAT ? p[P_W1 + mine * NFEAT + k] : (k == NFEAT ? p[P_B1 + mine] : 0.0f);
  }
#pragma unroll
  for (int kk = 0; kk < 16; ++kk) {
    const int k = unit_of(kk, g);
    w2[kk] = p[P_W2 + mine * HID + k];
    w2t[kk] = p[P_W2 + k * HID + mine];
    w3[kk] = i < NOUT ? p[P_W3 + i * HID + k] : 0.0f;
  }
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const int u = 4 * g + kk;
    w3t[kk] = u < NOUT ? p[P_W3 + u * HID + mine] : 0.0f;
  }
  float4_t bias2, bias3;
  float so[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int u = 4 * g + r;
    bias2[r] = p[P_B2 + 16 * w + u];
    bias3[r] = u < NOUT ? p[P_B3 + u] : 0.0f;
    so[r] = u < NOUT ? out_scale[u] : 1.0f;
  }
  const float4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
  float4_t gw1 = zero, gw2[4] = {zero, zero, zero, zero}, gw3 = zero, gb2 = zero, gb3 = zero;
  double loss = 0.0;
  const float inv_n = 1.0f / (float)n;
  for (int e = threadIdx.x; e < 16 * TS; e += 256)
    if (e / TS >= NFEAT) X[e / TS][e % TS] = e / TS == NFEAT ? 1.0f : 0.0f;
  const int64_t ntile = (n + TS - 1) / TS;
  for (int64_t tile = blockIdx.x; tile < ntile; tile += gridDim.x) {
    const int64_t s0 = tile * TS;
    if (threadIdx.x < NFEAT * TS) {
      const int s = threadIdx.x / NFEAT, k = threadIdx.x % NFEAT;
      X[k][s] = s0 + s < n ? x[(s0 + s) * NFEAT + k] * in_scale[k] : 0.0f;
    }
    const bool live = s0 + i < n;
    float tv[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
      tv[r] = live && 4 * g + r < NOUT ? t[(s0 + i) * NOUT + 4 * g + r] : 0.0f;
    __syncthreads();
    // forward; in an output tile this lane holds rows 4g..4g+3 of column i
    float4_t z = zero;
#pragma unroll
    for (int kk = 0; kk < 3; ++kk) z = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[kk], X[4 * kk + g][i], z, 0, 0, 0);
    float a1[4], a2[4], dy[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) A1[16 * w + 4 * g + r][i] = a1[r] = tanhf(z[r]);
    __syncthreads();
    z = bias2;
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) z = __builtin_amdgcn_mfma_f32_16x16x4f32(w2[kk], A1[unit_of(kk, g)][i], z, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) A2[16 * w + 4 * g + r][i] = a2[r] = tanhf(z[r]);
    __syncthreads();
    // every wave forms the outputs and their errors (no exchange needed)
    z = bias3;
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) z = __builtin_amdgcn_mfma_f32_16x16x4f32(w3[kk], A2[unit_of(kk, g)][i], z, 0, 0, 0);
    float ls = 0.0f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float res = live && 4 * g + r < NOUT ? z[r] - tv[r] / so[r] : 0.0f;
      ls += res * res;
      dy[r] = 2.0f * res * inv_n;
    }
    if (w == 0) {
      loss += ls;
#pragma unroll
      for (int r = 0; r < 4; ++r) DY[4 * g + r][i] = dy[r];
    }
    // back: an output tile's rows 4g + kk are the next product's inputs
    z = zero;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) z = __builtin_amdgcn_mfma_f32_16x16x4f32(w3t[kk], dy[kk], z, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) D2[16 * w + 4 * g + r][i] = z[r] * (1.0f - a2[r] * a2[r]);
    __syncthreads();
    z = zero;
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) z = __builtin_amdgcn_mfma_f32_16x16x4f32(w2t[kk], D2[unit_of(kk, g)][i], z, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 4; ++r) D1[16 * w + 4 * g + r][i] = z[r] * (1.0f - a1[r] * a1[r]);
    // gradients: sums over the tile's samples 4kk + g
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int s = 4 * kk + g;
      const float d2 = D2[mine][s], dyv = DY[i][s];
#pragma unroll
      for (int c = 0; c < 4; ++c) gw2[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(d2, A1[16 * c + i][s], gw2[c], 0, 0, 0);
      gb2 = __builtin_amdgcn_mfma_f32_16x16x4f32(d2, 1.0f, gb2, 0, 0, 0);
      gw3 = __builtin_amdgcn_mfma_f32_16x16x4f32(dyv, A2[mine][s], gw3, 0, 0, 0);
      gb3 = __builtin_amdgcn_mfma_f32_16x16x4f32(dyv, 1.0f, gb3, 0, 0, 0);
    }
    __syncthreads();  // D1 is whole
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      gw1 = __builtin_amdgcn_mfma_f32_16x16x4f32(D1[mine][4 * kk + g], X[i][4 * kk + g], gw1, 0, 0, 0);
    __syncthreads();  // the tile's readers are done
  }
  float* P = partial + (int64_t)blockIdx.x * NPARAM;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int u = 16 * w + 4 * g + r;
    if (i < NFEAT) P[P_W1 + u * NFEAT + i] = gw1[r];
    if (i == NFEAT) P[P_B1 + u] = gw1[r];
#pragma unroll
    for (int c = 0; c < 4; ++c) P[P_W2 + u * HID + 16 * c + i] = gw2[c][r];
    if (i == 0) P[P_B2 + u] = gb2[r];
    if (4 * g + r < NOUT) {
      P[P_W3 + (4 * g + r) * HID + mine] = gw3[r];
      if (w == 0 && i == 0) P[P_B3 + 4 * g + r] = gb3[r];
    }
  }
  if (w == 0) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) loss += __shfl_down(loss, off, WAVE);
    if (lane == 0) lossp[blockIdx.x] = loss;
  }
}

// gradient = partials added in a fixed order (four interleaved sums, then
// those in order); the loss; optional Adam update
__global__ __launch_bounds__(256) void k_mlp_adam(const float* __restrict__ partial,
                                                  const double* __restrict__ lossp, int nwg,
                                                  int64_t n, float* __restrict__ grad,
                                                  double* __restrict__ loss, float* __restrict__ p,
                                                  float* __restrict__ m, float* __restrict__ v,
                                                  int do_update, float lr, float beta1, float beta2,
                                                  float eps, float bc1, float bc2) {
  __shared__ float part[4][64];
  const int q = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int j = blockIdx.x * 64 + l;
  float s = 0.0f;
  if (j < NPARAM) {
#pragma unroll 8
    for (int c = q; c < nwg; c += 4) s += partial[(int64_t)c * NPARAM + j];
  }
  part[q][l] = s;
  __syncthreads();
  if (blockIdx.x == 0 && q == 1) {
    double ls = 0.0;
    for (int c = l; c < nwg; c += 64) ls += lossp[c];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) ls += __shfl_down(ls, off, WAVE);
    if (l == 0) *loss = ls / (double)n;
  }
  if (q != 0 || j >= NPARAM) return;
  const float gr = ((part[0][l] + part[1][l]) + part[2][l]) + part[3][l];
  grad[j] = gr;
  if (!do_update) return;
  const float mj = beta1 * m[j] + (1.0f - beta1) * gr;
  const float vj = beta2 * v[j] + (1.0f - beta2) * gr * gr;
  m[j] = mj;
  v[j] = vj;
  p[j] -= lr * (mj / bc1) / (sqrtf(vj / bc2) + eps);
}

// ---------------------------------------------------------------------------
// Grad-type initial distribution (reduced over the internal dimension in
// 2-D), one work-group per cell; a cell whose features leave the training
// box (or are not finite) keeps the Maxwellian.
template <int D, typename T>
__global__ __launch_bounds__(TPB) void k_grad_init(DevVel v, GasP g, const double* __restrict__ W,
                                                   const float* __restrict__ feat,
                                                   const float* __restrict__ out,
                                                   const float* __restrict__ lo,
                                                   const float* __restrict__ hi, T* __restrict__ h,
                                                   T* __restrict__ b, int32_t* __restrict__ nfall) {
  const int64_t i = blockIdx.x;
  double P[NPRIM];
  prim_of<D>(&W[i * (D + 2)], g, P);
  bool use = true;
  for (int j = 0; j < NFEAT; ++j) {
    const float f = feat[i * FS + j];
    use = use && (f >= lo[j]) && (f <= hi[j]);  // false for NaN
  }
  for (int j = 0; j < NOUT; ++j) use = use && isfinite(out[i * FS + j]);
  double s[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}}, r[3] = {0, 0, 0};
  if (use) {
    const float* o = &out[i * FS];
    s[0][0] = o[0];
    s[1][1] = o[1];
    s[2][2] = o[2];
    s[0][1] = s[1][0] = o[3];
    s[0][2] = s[2][0] = o[4];
    s[1][2] = s[2][1] = o[5];
    const double tr = (s[0][0] + s[1][1] + s[2][2]) / 3.0;
    for (int a = 0; a < 3; ++a) s[a][a] -= tr;
    for (int d = 0; d < 3; ++d) r[d] = o[6 + d];
    if (D == 2) {
      s[0][2] = s[2][0] = s[1][2] = s[2][1] = 0.0;
      r[2] = 0.0;
    }
  } else if (threadIdx.x == 0) {
    atomicAdd(nfall, 1);
  }
  const double rho = P[0], lam = P[4];
  const double nrm = rho * maxw_norm<D>(lam);
  const double sq = 2.0 * sqrt(lam);
  for (int64_t k = threadIdx.x; k < v.nvp; k += TPB) {
    double c[3] = {0, 0, 0};
    double c2 = 0.0;
    for (int d = 0; d < D; ++d) {
      c[d] = v.u[d * v.nvp + k] - P[1 + d];
      c2 += c[d] * c[d];
    }
    double quad = 0.0, rc = 0.0;
    for (int a = 0; a < D; ++a) {
      rc += r[a] * c[a];
      for (int bb = 0; bb < D; ++bb) quad += s[a][bb] * c[a] * c[bb];
    }
    const double H = nrm * exp(-lam * c2);
    if (D == 3) {
      st(h, i * v.nvp + k, H * (1.0 + lam * quad + sq * rc * (0.4 * lam * c2 - 1.0)));
    } else {
      st(h, i * v.nvp + k, H * (1.0 + lam * quad + 0.5 * s[2][2] + sq * rc * (0.4 * lam * c2 - 0.8)));
      st(b, i * v.nvp + k,
         H / (2.0 * lam) * (1.0 + lam * quad + 1.5 * s[2][2] + sq * rc * (0.4 * lam * c2 - 0.4)));
    }
  }
}

}  // namespace
}  // namespace ugks

// ===========================================================================
// C ABI of the learned warm start
// ===========================================================================
using namespace ugks;
using namespace ugks::host;

struct ugks_mlp {
  hipStream_t stream = nullptr;
  bool own_stream = false;
  int device = -1;  // the device the network's memory lives on
  std::vector<void*> allocations;
  float* p = nullptr;  // FP32 parameters
  float* m = nullptr;
  float* v = nullptr;
  float* grad = nullptr;
  short* w1 = nullptr;
  short* w2 = nullptr;
  short* w3 = nullptr;
  float* in_scale = nullptr;
  float* out_scale = nullptr;
  float* lo = nullptr;
  float* hi = nullptr;
  int64_t adam_steps = 0;
  // partial gradients and losses of one step, and the losses of a call's steps
  float* partial = nullptr;
  double* lossp = nullptr;
  double* loss = nullptr;
  int64_t loss_cap = 0;
  // device copies of host rows (x, t) and device rows for host outputs,
  // grown on demand
  float* rows[3] = {nullptr, nullptr, nullptr};
  int64_t rows_cap[3] = {0, 0, 0};
  std::string err;
};

namespace {

thread_local std::string g_mlp_create_error;

template <typename T>
T* malloc_into(std::vector<void*>& list, size_t n) {
  if (n == 0) n = 1;
  void* p = nullptr;
  hipError_t e = hipMalloc(&p, n * sizeof(T));
  if (e != hipSuccess) throw HipFail{e, "hipMalloc"};
  list.push_back(p);
  return static_cast<T*>(p);
}

int mlp_err(ugks_mlp* n, int code, const std::string& msg) {
  if (n) n->err = msg;
  else g_mlp_create_error = msg;
  return code;
}

int ctx_err(ugks_ctx* c, int code, const std::string& msg) {
  if (c) c->err = msg;
  return code;
}

MlpDev mlp_dev(const ugks_mlp* n) {
  MlpDev d;
  d.w1 = n->w1;
  d.w2 = n->w2;
  d.w3 = n->w3;
  d.p = n->p;
  d.in_scale = n->in_scale;
  d.out_scale = n->out_scale;
  return d;
}

void mlp_pack(ugks_mlp* n) {
  hipLaunchKernelGGL(k_mlp_pack, dim3(16), dim3(256), 0, n->stream, n->p, n->w1, n->w2, n->w3);
  HIP_TRY(hipGetLastError());
}

// rows of x and y are xs and ys floats apart
void mlp_infer(const ugks_mlp* n, const float* x, int xs, int64_t rows, float* y, int ys, hipStream_t s) {
  if (rows == 0) return;
  const int64_t tiles = (rows + 15) / 16;
  const int64_t blocks = std::min<int64_t>((tiles + 3) / 4, 4096);
  hipLaunchKernelGGL(k_mlp_infer, dim3((unsigned)blocks), dim3(256), 0, s, mlp_dev(n), x, xs, rows, y, ys);
  HIP_TRY(hipGetLastError());
}

// Whether dense rows at x and y overlap without being the same rows: a wave
// reads its 16 rows before it writes them, so equal pointers are safe in
// place, while another wave's rows must not be written before they are read.
bool rows_overlap(const float* x, const float* y, int64_t rows) {
  const uintptr_t a = (uintptr_t)x, b = (uintptr_t)y, len = (uintptr_t)rows * NFEAT * sizeof(float);
  return a != b && a < b + len && b < a + len;
}

// Device address of the file-scope scratch array on the current device,
// looked up once per device (every GPU holds its own copy of the array).
std::mutex g_scratch_mu;
float* g_scratch_dev[64] = {};

float* noalloc_scratch(int device) {
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_dev[device]) {
    void* ptr = nullptr;
    HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    g_scratch_dev[device] = static_cast<float*>(ptr);
  }
  return g_scratch_dev[device];
}

// The network's own device buffer `slot` for dense rows of 9 floats.
float* own_rows(ugks_mlp* n, int slot, int64_t rows) {
  if (rows > n->rows_cap[slot]) {
    float* grown = malloc_into<float>(n->allocations, (size_t)rows * NFEAT);
    if (n->rows[slot]) {
      HIP_TRY(hipStreamSynchronize(n->stream));
      n->allocations.erase(std::find(n->allocations.begin(), n->allocations.end(), (void*)n->rows[slot]));
      (void)hipFree(n->rows[slot]);
    }
    n->rows[slot] = grown;
    n->rows_cap[slot] = rows;
  }
  return n->rows[slot];
}

// Dense rows of 9 on the device: the caller's own, or a copy of host rows in
// one piece (a pitched copy from pageable memory goes row by row: 460 ms for
// the 25,344 rows of x and t, against 0.4 ms).
const float* device_rows(ugks_mlp* n, const float* src, int64_t rows, int on_device, int slot) {
  if (on_device || rows == 0) return src;
  float* d = own_rows(n, slot, rows);
  HIP_TRY(hipMemcpyAsync(d, src, (size_t)rows * NFEAT * sizeof(float), hipMemcpyHostToDevice, n->stream));
  return d;
}

void grow_loss(ugks_mlp* n, int64_t steps) {
  if (steps <= n->loss_cap) return;
  double* grown = malloc_into<double>(n->allocations, (size_t)steps);
  if (n->loss) {
    HIP_TRY(hipStreamSynchronize(n->stream));
    n->allocations.erase(std::find(n->allocations.begin(), n->allocations.end(), (void*)n->loss));
    (void)hipFree(n->loss);
  }
  n->loss = grown;
  n->loss_cap = steps;
}

// gradient (and optionally one Adam step) of the mean squared error over rows
// [0, rows) of x, t (device rows of 9); the loss goes to loss[at]
void mlp_grad_step(ugks_mlp* n, const float* x, const float* t, int64_t rows, bool update, float lr,
                   int64_t at) {
  const int nwg = (int)std::min<int64_t>((rows + TS - 1) / TS, MAX_WG);
  hipLaunchKernelGGL(k_mlp_grad, dim3((unsigned)nwg), dim3(256), 0, n->stream, n->p, n->in_scale,
                     n->out_scale, x, t, rows, n->partial, n->lossp);
  HIP_TRY(hipGetLastError());
  float bc1 = 1.0f, bc2 = 1.0f;
  if (update) {
    n->adam_steps += 1;
    bc1 = 1.0f - std::pow(0.9f, (float)n->adam_steps);
    bc2 = 1.0f - std::pow(0.999f, (float)n->adam_steps);
  }
  hipLaunchKernelGGL(k_mlp_adam, dim3((NPARAM + 63) / 64), dim3(256), 0, n->stream, n->partial,
                     n->lossp, nwg, rows, n->grad, n->loss + at, n->p, n->m, n->v, update ? 1 : 0,
                     lr, 0.9f, 0.999f, 1e-8f, bc1, bc2);
  HIP_TRY(hipGetLastError());
}

}  // namespace

extern "C" {

int ugks_mlp_create(const float* params, const float* in_scale, const float* out_scale, void* stream,
                    ugks_mlp** out) {
  if (!out || !params || !in_scale || !out_scale) return mlp_err(nullptr, UGKS_EINVAL, "null argument");
  for (int j = 0; j < NPARAM; ++j)
    if (!std::isfinite(params[j])) return mlp_err(nullptr, UGKS_EINVAL, "parameters must be finite");
  for (int j = 0; j < 9; ++j)
    if (!(in_scale[j] > 0.0f) || !(out_scale[j] > 0.0f) || !std::isfinite(in_scale[j]) ||
        !std::isfinite(out_scale[j]))
      return mlp_err(nullptr, UGKS_EINVAL, "scales must be positive and finite");
  std::unique_ptr<ugks_mlp> n(new ugks_mlp());
  try {
    HIP_TRY(hipGetDevice(&n->device));
    if (stream) {
      n->stream = (hipStream_t)stream;
    } else {
      HIP_TRY(hipStreamCreateWithFlags(&n->stream, hipStreamNonBlocking));
      n->own_stream = true;
    }
    auto& A = n->allocations;
    n->p = malloc_into<float>(A, NPARAM);
    n->m = malloc_into<float>(A, NPARAM);
    n->v = malloc_into<float>(A, NPARAM);
    n->grad = malloc_into<float>(A, NPARAM);
    n->w1 = malloc_into<short>(A, 64 * 16);
    n->w2 = malloc_into<short>(A, 64 * 64);
    n->w3 = malloc_into<short>(A, 16 * 64);
    n->in_scale = malloc_into<float>(A, 16);
    n->out_scale = malloc_into<float>(A, 16);
    n->lo = malloc_into<float>(A, 16);
    n->hi = malloc_into<float>(A, 16);
    n->partial = malloc_into<float>(A, (size_t)MAX_WG * NPARAM);
    n->lossp = malloc_into<double>(A, MAX_WG);
    grow_loss(n.get(), 1);
    HIP_TRY(hipMemcpy(n->p, params, NPARAM * sizeof(float), hipMemcpyHostToDevice));
    HIP_TRY(hipMemset(n->m, 0, NPARAM * sizeof(float)));
    HIP_TRY(hipMemset(n->v, 0, NPARAM * sizeof(float)));
    HIP_TRY(hipMemcpy(n->in_scale, in_scale, 9 * sizeof(float), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(n->out_scale, out_scale, 9 * sizeof(float), hipMemcpyHostToDevice));
    // until a box is set every finite feature is inside it
    std::vector<float> lo(16, -INFINITY), hi(16, INFINITY);
    HIP_TRY(hipMemcpy(n->lo, lo.data(), 16 * sizeof(float), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(n->hi, hi.data(), 16 * sizeof(float), hipMemcpyHostToDevice));
    mlp_pack(n.get());
    HIP_TRY(hipStreamSynchronize(n->stream));
  } catch (const HipFail& e) {
    ugks_mlp_destroy(n.release());
    return mlp_err(nullptr, e.e == hipErrorOutOfMemory ? UGKS_ENOMEM : UGKS_EHIP,
                   std::string(e.what) + ": " + hipGetErrorString(e.e));
  } catch (const std::bad_alloc&) {
    ugks_mlp_destroy(n.release());
    return mlp_err(nullptr, UGKS_ENOMEM, "host memory allocation failed");
  } catch (...) {
    ugks_mlp_destroy(n.release());
    return mlp_err(nullptr, UGKS_EHIP, "internal error");
  }
  *out = n.release();
  return UGKS_OK;
}

int ugks_mlp_get_params(ugks_mlp* n, float* params) {
  if (!n || !params) return mlp_err(n, UGKS_EINVAL, "null argument");
  try {
    HIP_TRY(hipMemcpyAsync(params, n->p, NPARAM * sizeof(float), hipMemcpyDeviceToHost, n->stream));
    HIP_TRY(hipStreamSynchronize(n->stream));
  } catch (const HipFail& e) {
    return mlp_err(n, UGKS_EHIP, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } UGKS_CATCH_REST(mlp_err, n)
  return UGKS_OK;
}

int ugks_mlp_set_box(ugks_mlp* n, const float* lo, const float* hi) {
  if (!n || !lo || !hi) return mlp_err(n, UGKS_EINVAL, "null argument");
  for (int j = 0; j < 9; ++j)
    if (!(lo[j] <= hi[j])) return mlp_err(n, UGKS_EINVAL, "box bounds must satisfy lo <= hi");
  try {
    HIP_TRY(hipMemcpyAsync(n->lo, lo, 9 * sizeof(float), hipMemcpyHostToDevice, n->stream));
    HIP_TRY(hipMemcpyAsync(n->hi, hi, 9 * sizeof(float), hipMemcpyHostToDevice, n->stream));
    HIP_TRY(hipStreamSynchronize(n->stream));
  } catch (const HipFail& e) {
    return mlp_err(n, UGKS_EHIP, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } UGKS_CATCH_REST(mlp_err, n)
  return UGKS_OK;
}

int ugks_mlp_forward(ugks_mlp* n, const float* x, int64_t rows, float* y, int32_t on_device) {
  if (!n || (rows > 0 && (!x || !y)) || rows < 0) return mlp_err(n, UGKS_EINVAL, "bad argument");
  try {
    const size_t bytes = (size_t)rows * NFEAT * sizeof(float);
    const float* xd = device_rows(n, x, rows, on_device, 0);
    if (on_device && rows > 0 && rows_overlap(x, y, rows)) {
      float* copy = own_rows(n, 0, rows);
      HIP_TRY(hipMemcpyAsync(copy, x, bytes, hipMemcpyDeviceToDevice, n->stream));
      xd = copy;
    }
    float* yd = on_device || rows == 0 ? y : own_rows(n, 2, rows);
    mlp_infer(n, xd, NFEAT, rows, yd, NOUT, n->stream);
    if (!on_device && rows > 0) HIP_TRY(hipMemcpyAsync(y, yd, bytes, hipMemcpyDeviceToHost, n->stream));
    HIP_TRY(hipStreamSynchronize(n->stream));
  } catch (const HipFail& e) {
    return mlp_err(n, UGKS_EHIP, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } UGKS_CATCH_REST(mlp_err, n)
  return UGKS_OK;
}

int ugks_mlp_forward_noalloc(ugks_mlp* n, const float* x, int64_t rows, float* y) {
  if (!n) return mlp_err(n, UGKS_EINVAL, "null network");
  if (rows < 0 || rows > UGKS_NOALLOC_MAX_ROWS)
    return mlp_err(n, UGKS_EINVAL, "rows must be in [0, " + std::to_string(UGKS_NOALLOC_MAX_ROWS) +
                                       "] for the allocation-free inference");
  if (rows > 0 && (!x || !y)) return mlp_err(n, UGKS_EINVAL, "null input or output");
  if (rows == 0) return UGKS_OK;
  try {
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != n->device || dev < 0 || dev >= 64)
      return mlp_err(n, UGKS_EINVAL, "the network's device must be the current device");
    if (rows_overlap(x, y, rows)) {
      float* copy = noalloc_scratch(dev);
      const int64_t k = rows * NFEAT;
      hipLaunchKernelGGL(k_copy_rows, dim3((unsigned)((k + 255) / 256)), dim3(256), 0, n->stream, x, k, copy);
      HIP_TRY(hipGetLastError());
      x = copy;
    }
    mlp_infer(n, x, NFEAT, rows, y, NOUT, n->stream);
  } catch (const HipFail& e) {
    return mlp_err(n, UGKS_EHIP, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } UGKS_CATCH_REST(mlp_err, n)
  return UGKS_OK;
}

int ugks_mlp_loss_grad(ugks_mlp* n, const float* x, const float* t, int64_t rows, float* grad,
                       double* loss, int32_t on_device) {
  if (!n || !x || !t || rows <= 0) return mlp_err(n, UGKS_EINVAL, "bad argument");
  try {
    const float* xd = device_rows(n, x, rows, on_device, 0);
    const float* td = device_rows(n, t, rows, on_device, 1);
    mlp_grad_step(n, xd, td, rows, false, 0.0f, 0);
    if (grad) HIP_TRY(hipMemcpyAsync(grad, n->grad, NPARAM * sizeof(float), hipMemcpyDeviceToHost, n->stream));
    if (loss) HIP_TRY(hipMemcpyAsync(loss, n->loss, sizeof(double), hipMemcpyDeviceToHost, n->stream));
    HIP_TRY(hipStreamSynchronize(n->stream));
  } catch (const HipFail& e) {
    return mlp_err(n, UGKS_EHIP, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } UGKS_CATCH_REST(mlp_err, n)
  return UGKS_OK;
}

int ugks_mlp_train(ugks_mlp* n, const float* x, const float* t, int64_t rows, int64_t batch,
                   int32_t steps, float lr, int32_t on_device, double* loss_out) {
  if (!n || !x || !t || rows <= 0 || batch <= 0 || steps < 0 || !(lr > 0.0f))
    return mlp_err(n, UGKS_EINVAL, "bad argument");
  Range range("ugks_mlp_train");
  try {
    const float* xd = device_rows(n, x, rows, on_device, 0);
    const float* td = device_rows(n, t, rows, on_device, 1);
    grow_loss(n, steps);
    batch = std::min(batch, rows);
    int64_t at = 0;
    for (int32_t k = 0; k < steps; ++k) {
      if (at + batch > rows) at = 0;  // consecutive slices of the caller's (shuffled) order
      mlp_grad_step(n, xd + at * NFEAT, td + at * NFEAT, batch, true, lr, k);
      at += batch;
    }
    mlp_pack(n);
    if (loss_out && steps > 0)
      HIP_TRY(hipMemcpyAsync(loss_out, n->loss, steps * sizeof(double), hipMemcpyDeviceToHost, n->stream));
    HIP_TRY(hipStreamSynchronize(n->stream));
  } catch (const HipFail& e) {
    return mlp_err(n, UGKS_EHIP, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } UGKS_CATCH_REST(mlp_err, n)
  return UGKS_OK;
}

void ugks_mlp_destroy(ugks_mlp* n) {
  if (!n) return;
  if (n->stream) (void)hipStreamSynchronize(n->stream);
  for (void* p : n->allocations) (void)hipFree(p);
  if (n->own_stream && n->stream) (void)hipStreamDestroy(n->stream);
  delete n;
}

const char* ugks_mlp_last_error(const ugks_mlp* n) {
  return n ? n->err.c_str() : g_mlp_create_error.c_str();
}

int ugks_snapshot(ugks_ctx* c, float* feat, float* targ) {
  if (!c || (!feat && !targ)) return ctx_err(c, UGKS_EINVAL, "null argument");
  if (c->gas.K != 0.0)
    return ctx_err(c, UGKS_EUNSUPPORTED, "the learned closure is defined for monatomic gases (K = 0)");
  const int D = c->D;
  try {
    StepBuffers& B = c->buf;
    hipStream_t s = c->stream;
    const int64_t nc = c->nc;
    float* fd = dalloc<float>(c, (size_t)nc * FS);
    float* td = dalloc<float>(c, (size_t)nc * FS);
    DevMesh mg = c->mesh;
    mg.lsG = c->lsG_exact;  // features use the true gradient at any reconstruction order
    mg.limiter = 0;         // and unlimited
    HIP_TRY(launch_gradW(D, mg, c->bcs, c->gas, B.W, B.gW, B.flag, 0, s));
    const unsigned g1 = (unsigned)((nc + 127) / 128);
    if (D == 2) hipLaunchKernelGGL(k_features<2>, dim3(g1), dim3(128), 0, s, nc, c->gas, B.W, B.gW, fd);
    else hipLaunchKernelGGL(k_features<3>, dim3(g1), dim3(128), 0, s, nc, c->gas, B.W, B.gW, fd);
    HIP_TRY(hipGetLastError());
    if (c->prec == UGKS_FP32) {
      if (D == 2) hipLaunchKernelGGL((k_targets<2, float>), dim3((unsigned)nc), dim3(TPB), 0, s, c->vel, c->gas, B.W, (const float*)B.h, (const float*)B.b, td);
      else hipLaunchKernelGGL((k_targets<3, float>), dim3((unsigned)nc), dim3(TPB), 0, s, c->vel, c->gas, B.W, (const float*)B.h, (const float*)B.b, td);
    } else {
      if (D == 2) hipLaunchKernelGGL((k_targets<2, double>), dim3((unsigned)nc), dim3(TPB), 0, s, c->vel, c->gas, B.W, (const double*)B.h, (const double*)B.b, td);
      else hipLaunchKernelGGL((k_targets<3, double>), dim3((unsigned)nc), dim3(TPB), 0, s, c->vel, c->gas, B.W, (const double*)B.h, (const double*)B.b, td);
    }
    HIP_TRY(hipGetLastError());
    std::vector<float> hf(nc * FS), ht(nc * FS);
    HIP_TRY(hipMemcpyAsync(hf.data(), fd, hf.size() * sizeof(float), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipMemcpyAsync(ht.data(), td, ht.size() * sizeof(float), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    for (int64_t i = 0; i < nc; ++i) {
      const int64_t u = c->cell_perm[i];
      for (int j = 0; j < 9; ++j) {
        if (feat) feat[u * 9 + j] = hf[i * FS + j];
        if (targ) targ[u * 9 + j] = ht[i * FS + j];
      }
    }
    // scratch: released now (the allocation list keeps the rest)
    for (float* p : {fd, td}) {
      (void)hipFree(p);
      c->allocations.erase(std::find(c->allocations.begin(), c->allocations.end(), (void*)p));
      c->bytes -= (int64_t)(nc * FS * sizeof(float));
    }
  } catch (const HipFail& e) {
    return ctx_err(c, UGKS_EHIP, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } UGKS_CATCH_REST(ctx_err, c)
  return UGKS_OK;
}

int ugks_warm_start(ugks_ctx* c, const ugks_mlp* net, const double* W, int64_t* n_fallback) {
  if (!c || !net) return ctx_err(c, UGKS_EINVAL, "null argument");
  if (c->gas.K != 0.0)
    return ctx_err(c, UGKS_EUNSUPPORTED, "the learned closure is defined for monatomic gases (K = 0)");
  const int D = c->D;
  Range range("ugks_warm_start");
  try {
    StepBuffers& B = c->buf;
    hipStream_t s = c->stream;
    const int64_t nc = c->nc;
    if (W) {
      int rc = ugks_set_state(c, W, nullptr, nullptr);
      if (rc) return rc;
    }
    HIP_TRY(hipStreamSynchronize(net->stream));  // the network's last update is done
    float* fd = dalloc<float>(c, (size_t)nc * FS);
    float* od = dalloc<float>(c, (size_t)nc * FS);
    int32_t* cnt = dalloc<int32_t>(c, 1);
    HIP_TRY(hipMemsetAsync(cnt, 0, sizeof(int32_t), s));
    HIP_TRY(launch_prims(D, c->mesh, c->gas, B.W, B.prim, B.flag, 0, s));
    DevMesh mg = c->mesh;
    mg.lsG = c->lsG_exact;  // features use the true gradient at any reconstruction order
    mg.limiter = 0;         // and unlimited
    HIP_TRY(launch_gradW(D, mg, c->bcs, c->gas, B.W, B.gW, B.flag, 0, s));
    const unsigned g1 = (unsigned)((nc + 127) / 128);
    if (D == 2) hipLaunchKernelGGL(k_features<2>, dim3(g1), dim3(128), 0, s, nc, c->gas, B.W, B.gW, fd);
    else hipLaunchKernelGGL(k_features<3>, dim3(g1), dim3(128), 0, s, nc, c->gas, B.W, B.gW, fd);
    HIP_TRY(hipGetLastError());
    mlp_infer(net, fd, FS, nc, od, FS, s);
    if (c->prec == UGKS_FP32) {
      if (D == 2) hipLaunchKernelGGL((k_grad_init<2, float>), dim3((unsigned)nc), dim3(TPB), 0, s, c->vel, c->gas, B.W, fd, od, net->lo, net->hi, (float*)B.h, (float*)B.b, cnt);
      else hipLaunchKernelGGL((k_grad_init<3, float>), dim3((unsigned)nc), dim3(TPB), 0, s, c->vel, c->gas, B.W, fd, od, net->lo, net->hi, (float*)B.h, (float*)B.b, cnt);
    } else {
      if (D == 2) hipLaunchKernelGGL((k_grad_init<2, double>), dim3((unsigned)nc), dim3(TPB), 0, s, c->vel, c->gas, B.W, fd, od, net->lo, net->hi, (double*)B.h, (double*)B.b, cnt);
      else hipLaunchKernelGGL((k_grad_init<3, double>), dim3((unsigned)nc), dim3(TPB), 0, s, c->vel, c->gas, B.W, fd, od, net->lo, net->hi, (double*)B.h, (double*)B.b, cnt);
    }
    HIP_TRY(hipGetLastError());
    int32_t nf = 0;
    HIP_TRY(hipMemcpyAsync(&nf, cnt, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    if (n_fallback) *n_fallback = nf;
    c->q_valid = false;  // the next step takes the heat flux of the new f
    c->cs_valid = false;
    c->resid_set = false;
    HIP_TRY(hipMemsetAsync(B.resid, 0, 8 * sizeof(double), s));  // residuals restart from here
    for (void* p : {(void*)fd, (void*)od, (void*)cnt}) {
      (void)hipFree(p);
      c->allocations.erase(std::find(c->allocations.begin(), c->allocations.end(), p));
    }
    c->bytes -= (int64_t)(2 * nc * FS * sizeof(float) + sizeof(int32_t));
  } catch (const HipFail& e) {
    return ctx_err(c, UGKS_EHIP, std::string(e.what) + ": " + hipGetErrorString(e.e));
  } UGKS_CATCH_REST(ctx_err, c)
  return UGKS_OK;
}

}  // extern "C"
