// Reverse-mode kernels of the COLA step (Koda et al. 2015, Sec. 2.2, eqs.
// cola-kick and cola-drift with the PM force) and of the density output (Sec.
// 3.3); those of P(k) are in k_pk.hip, of the 2LPT source (Sec. 2.1) in k_fft.hip.
//
// Step, per particle (mesh units, x = q + d at the step start):
//   vt = vbar' + I dbar';  Psi1bar += e1 dbar' - c1 vt;  Psi2bar += e2 dbar' - c2 vt
//   vbar = vt;  Fbar = K vt
//   dbar = dbar' + sum_d Fbar_d sum_s grad w_s(x) g_d[c + s]     (readout weights)
// and, after the transpose deposit and the Green transpose, the deposit
// weight gradient dbar += sum_s grad w_s(x) rhobar[c + s].
// CIC weight gradient: d w_s / d u_e = (s_e ? +1 : -1) prod_{e' != e} w_{s_e'}(f_e').
#include "cola_device.h"
#include "cola_internal.h"

namespace cola {

__device__ __forceinline__ void weight_grads(const float f[3], int k, float gw[3]) {
  const float wx = (k & 4) ? f[0] : 1.0f - f[0];
  const float wy = (k & 2) ? f[1] : 1.0f - f[1];
  const float wz = (k & 1) ? f[2] : 1.0f - f[2];
  const float sx = (k & 4) ? 1.0f : -1.0f, sy = (k & 2) ? 1.0f : -1.0f, sz = (k & 1) ? 1.0f : -1.0f;
  gw[0] = sx * wy * wz;
  gw[1] = wx * sy * wz;
  gw[2] = wx * wy * sz;
}

__device__ __forceinline__ long node_index(const int c[3], int k, int nm, long row_stride) {
  int x = c[0] + ((k >> 2) & 1), y = c[1] + ((k >> 1) & 1), z = c[2] + (k & 1);
  if (x == nm) x = 0;
  if (y == nm) y = 0;
  if (z == nm) z = 0;
  return ((long)x * nm + y) * row_stride + z;
}

__global__ __launch_bounds__(256) void k_adj_readout_kick(
    const float* __restrict__ disp, const float* __restrict__ g, long row_stride, int np, int nm, long np3,
    KickDrift kd,
    float* __restrict__ dbar, float* __restrict__ vbar, float* __restrict__ p1bar,
    float* __restrict__ p2bar, float* __restrict__ fbar) {
  // particles of a block share mesh lines; neighbouring blocks stay on one XCD (L2)
  const long i = readout_particle(xcd_remap(blockIdx.x, gridDim.x), threadIdx.x, np, nm);
  if (i >= np3) return;
  float F[3];
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    const long j = e * np3 + i;
    const float db = dbar[j];
    const float vt = vbar[j] + kd.I * db;
    p1bar[j] += kd.e1 * db - kd.c1 * vt;
    p2bar[j] += kd.e2 * db - kd.c2 * vt;
    vbar[j] = vt;
    F[e] = kd.K * vt;
    fbar[j] = F[e];
  }
  int c[3];
  float f[3];
  home_cell(disp, np3, (uint32_t)i, np, nm, 1.0f, c, f);
  const ForceCorners fc(c, nm, row_stride);  // the force field interleaved by node
  float xb[3] = {0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    float gw[3];
    weight_grads(f, k, gw);
    const float* q = g + fc.at(k);
    const float s = F[0] * q[0] + F[1] * q[1] + F[2] * q[2];
#pragma unroll
    for (int e = 0; e < 3; ++e) xb[e] += gw[e] * s;
  }
#pragma unroll
  for (int e = 0; e < 3; ++e) dbar[e * np3 + i] += xb[e];
}

void launch_adj_readout_kick(const float* disp, const float* g, long row_stride, int np, int nm,
                             const KickDrift& kd, float* dbar, float* vbar, float* p1bar, float* p2bar,
                             float* fbar, hipStream_t s) {
  const long np3 = (long)np * np * np;
  hipLaunchKernelGGL(k_adj_readout_kick, dim3((unsigned)((np3 + 255) / 256)), dim3(256), 0, s, disp,
                     g, row_stride, np, nm, np3, kd, dbar, vbar, p1bar, p2bar, fbar);
}

// dbar += coef * dscale * sum_s grad w_s(u) field[c + s]  on an ng^3 grid.
__global__ __launch_bounds__(256) void k_adj_deposit_grad(const float* __restrict__ disp,
                                                          const float* __restrict__ field,
                                                          long row_stride, int np, int ng,
                                                          float dscale, long np3, float coef,
                                                          float* __restrict__ dbar) {
  // particles of a block share mesh lines; neighbouring blocks stay on one XCD (L2)
  const long i = readout_particle(xcd_remap(blockIdx.x, gridDim.x), threadIdx.x, np, ng);
  if (i >= np3) return;
  int c[3];
  float f[3];
  home_cell(disp, np3, (uint32_t)i, np, ng, dscale, c, f);
  float xb[3] = {0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    float gw[3];
    weight_grads(f, k, gw);
    const float v = field[node_index(c, k, ng, row_stride)];
#pragma unroll
    for (int e = 0; e < 3; ++e) xb[e] += gw[e] * v;
  }
  const float s = coef * dscale;
#pragma unroll
  for (int e = 0; e < 3; ++e) dbar[e * np3 + i] += s * xb[e];
}

void launch_adj_deposit_grad(const float* disp, const float* field, long row_stride, int np, int ng,
                             float dscale, float coef, float* dbar, hipStream_t s) {
  const long np3 = (long)np * np * np;
  hipLaunchKernelGGL(k_adj_deposit_grad, dim3((unsigned)((np3 + 255) / 256)), dim3(256), 0, s, disp,
                     field, row_stride, np, ng, dscale, np3, coef, dbar);
}

// mesh_q = a_q + alpha * b_q for the three components of particle arrays.
__global__ void k_axpy_to_mesh(const float* __restrict__ a, const float* __restrict__ b, float alpha,
                               int n, long n3, float* __restrict__ mesh, long row_stride,
                               long mesh_stride) {
  for (long p = blockIdx.x * (long)blockDim.x + threadIdx.x; p < n3;
       p += (long)gridDim.x * blockDim.x) {
    const long row = p / n, col = p - row * n;
  #pragma unroll
    for (int q = 0; q < 3; ++q)
      mesh[q * mesh_stride + row * row_stride + col] = a[q * n3 + p] + alpha * (b ? b[q * n3 + p] : 0.f);
  }
}

void launch_axpy_to_mesh(const float* a, const float* b, float alpha, int n, float* mesh,
                         long row_stride, long mesh_stride_floats, hipStream_t s) {
  const long n3 = (long)n * n * n;
  hipLaunchKernelGGL(k_axpy_to_mesh, dim3(grid_1d(n3)), dim3(256), 0, s, a, b, alpha,
                     n, n3, mesh, row_stride, mesh_stride_floats);
}

}  // namespace cola
