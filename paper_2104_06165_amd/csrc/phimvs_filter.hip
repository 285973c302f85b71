// Geometric-consistency filter of a depth map against its neighbours' maps (PHI-MVS
// Sec. III-D).  One thread per reference pixel; per neighbour the point is carried from
// the reference camera to the world and into the neighbour camera, compared with the
// neighbour's bilinear depth and its normal at the rounded position, and the neighbour's
// point is carried back to test the re-projection error.  FP64 throughout; the written-out
// form (`consistent`, no contraction) takes the decision of a sequential evaluation, in
// about 250 FP64 instructions and 30 bytes of gathers per pixel and neighbour, which the FP64
// instruction stream bounds (the vector ALU about 80% busy).
//
// Its outcome is a row of comparisons, so it is decided by a shorter form first
// (`consistent_short`): products of the cameras taken once per call (the neighbour's image of
// a reference pixel, the reference image of a neighbour's pixel, the normals' relative
// rotation), fused operations, reciprocals refined instead of divisions, squared distances.
// A bound of the difference between the two forms comes with each comparison, and a lane that
// any of them leaves open takes the written-out form, so every decision is that form's.
// 1600 x 1066 against eight neighbours: the kernel 111 us in the written-out form alone, 85 us so
// (about 170 instructions a neighbour, the vector ALU busy two thirds of the time, 3.2 TB/s of
// the bytes it cannot do without; two neighbours in flight at a time cost occupancy and took
// 113 us); the call 123 -> 90 us, the neighbour table now going with the launch.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "phimvs_internal.h"

namespace pmf {

using namespace phimvs_internal;

__device__ __forceinline__ void mat_vec(const double* M, const double* v, double* o) {
#pragma unroll
  for (int i = 0; i < 3; ++i) o[i] = M[3 * i] * v[0] + M[3 * i + 1] * v[1] + M[3 * i + 2] * v[2];
}

// camera -> world: R^T (X - t)
__device__ __forceinline__ void to_world(const double* R, const double* t, const double* X, double* Xw) {
  const double d0 = X[0] - t[0], d1 = X[1] - t[1], d2 = X[2] - t[2];
#pragma unroll
  for (int i = 0; i < 3; ++i) Xw[i] = R[i] * d0 + R[3 + i] * d1 + R[6 + i] * d2;
}

// world -> camera: R Xw + t
__device__ __forceinline__ void to_cam(const double* R, const double* t, const double* Xw, double* X) {
#pragma unroll
  for (int i = 0; i < 3; ++i) X[i] = R[3 * i] * Xw[0] + R[3 * i + 1] * Xw[1] + R[3 * i + 2] * Xw[2] + t[i];
}

// R^T n
__device__ __forceinline__ void normal_world(const double* R, float n0, float n1, float n2, double* nw) {
#pragma unroll
  for (int i = 0; i < 3; ++i) nw[i] = R[i] * (double)n0 + R[3 + i] * (double)n1 + R[6 + i] * (double)n2;
}

__device__ bool consistent(const FilterArgs& a, const FilterNbr& nb, int x, int y, double d, float n0, float n1,
                           float n2) {
  const double pix[3] = {(double)x, (double)y, 1.0};
  double ray[3], Xi[3], Xw[3], Xj[3], p[3];
  mat_vec(a.Kinv, pix, ray);
#pragma unroll
  for (int k = 0; k < 3; ++k) Xi[k] = d * ray[k];
  to_world(a.R, a.t, Xi, Xw);
  to_cam(nb.R, nb.t, Xw, Xj);
  mat_vec(nb.K, Xj, p);
  if (!(p[2] > 0.0)) return false;
  const double u = p[0] / p[2], v = p[1] / p[2];
  if (!(u >= 0.0 && u <= (double)(nb.W - 1) && v >= 0.0 && v <= (double)(nb.H - 1))) return false;
  const int x0 = (int)floor(u), y0 = (int)floor(v);
  const int x1 = min(x0 + 1, nb.W - 1), y1 = min(y0 + 1, nb.H - 1);
  const double fx = u - (double)x0, fy = v - (double)y0;
  const double d00 = nb.depth[(size_t)y0 * nb.W + x0], d01 = nb.depth[(size_t)y0 * nb.W + x1];
  const double d10 = nb.depth[(size_t)y1 * nb.W + x0], d11 = nb.depth[(size_t)y1 * nb.W + x1];
  if (!(d00 > 0.0 && d01 > 0.0 && d10 > 0.0 && d11 > 0.0)) return false;
  const double top = d00 + fx * (d01 - d00), bot = d10 + fx * (d11 - d10);
  const double dj = top + fy * (bot - top);
  if (!(fabs(Xj[2] - dj) < a.tau_d * dj)) return false;
  const int xr = min((int)floor(u + 0.5), nb.W - 1), yr = min((int)floor(v + 0.5), nb.H - 1);
  const float* nj = nb.normal + 3 * ((size_t)yr * nb.W + xr);
  double niw[3], njw[3];
  normal_world(a.R, n0, n1, n2, niw);
  normal_world(nb.R, nj[0], nj[1], nj[2], njw);
  const double dot = niw[0] * njw[0] + niw[1] * njw[1] + niw[2] * njw[2];
  if (!(dot > a.cos_n)) return false;
  const double pj[3] = {u, v, 1.0};
  double rj[3], Yj[3], Yw[3], Yi[3], q[3];
  mat_vec(nb.Kinv, pj, rj);
#pragma unroll
  for (int k = 0; k < 3; ++k) Yj[k] = dj * rj[k];
  to_world(nb.R, nb.t, Yj, Yw);
  to_cam(a.R, a.t, Yw, Yi);
  mat_vec(a.K, Yi, q);
  if (!(q[2] > 0.0)) return false;
  const double ex = q[0] / q[2] - (double)x, ey = q[1] / q[2] - (double)y;
  return sqrt(ex * ex + ey * ey) < a.tau_r;
}

// 1 / x to within 2^-40 (x normal): one step from the hardware's estimate
__device__ __forceinline__ double rcp_near(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  return __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
}

// 1 consistent, 0 not, -1 too close to call.  The table's bounds are described where it is
// filled (FilterNbr).
__device__ __forceinline__ int consistent_short(const FilterNbr& nb, double px, double py, double d, float n0, float n1,
                                                float n2, double tau_d, float cos_n, double tau2) {
  double p[3];
#pragma unroll
  for (int k = 0; k < 3; ++k)
    p[k] = __builtin_fma(d, __builtin_fma(nb.P[3 * k], px, __builtin_fma(nb.P[3 * k + 1], py, nb.P[3 * k + 2])), nb.s[k]);
  const double delta = __builtin_fma(nb.c1, d, nb.c0);
  const double e2 = nb.kw * delta;
  if (!(p[2] > e2)) return p[2] < -e2 ? 0 : -1;
  const double r = rcp_near(p[2]);
  const double u = p[0] * r, v = p[1] * r;
  // the position is within nb.m of the other form's; the texels taken and the rounded position
  // are the same unless it is that close to a whole or a half pixel
  if (!(delta * r * nb.cuv < nb.m)) return -1;
  const double hu = fabs(__builtin_amdgcn_fract(u + u) - 0.5), hv = fabs(__builtin_amdgcn_fract(v + v) - 0.5);
  if (!(fmax(hu, hv) < nb.half)) return -1;
  const double xf = floor(u), yf = floor(v);
  const int x0 = (int)xf, y0 = (int)yf;
  if (!((unsigned)x0 < (unsigned)(nb.W - 1) && (unsigned)y0 < (unsigned)(nb.H - 1))) return 0;
  const double fx = u - xf, fy = v - yf;
  const unsigned at = (unsigned)(y0 * nb.W + x0);
  const float* __restrict__ dp = nb.depth + at;
  const float f00 = dp[0], f01 = dp[1], f10 = dp[nb.W], f11 = dp[nb.W + 1];
  const unsigned an = at + (fx >= 0.5 ? 1u : 0u) + (fy >= 0.5 ? (unsigned)nb.W : 0u);
  const float* __restrict__ nj = nb.normal + 3 * (size_t)an;
  const float m0 = nj[0], m1 = nj[1], m2 = nj[2];
  if (!(f00 > 0.0f && f01 > 0.0f && f10 > 0.0f && f11 > 0.0f)) return 0;
  const float most = fmaxf(fmaxf(f00, f01), fmaxf(f10, f11)), least = fminf(fminf(f00, f01), fminf(f10, f11));
  // of the bilinear depth: the position's difference on the cell's slopes, and rounding
  const double ed = __builtin_fma(nb.m2, (double)(most - least), 0x1p-38 * (double)most);
  const double d00 = f00, d10 = f10;
  const double top = __builtin_fma(fx, (double)f01 - d00, d00), bot = __builtin_fma(fx, (double)f11 - d10, d10);
  const double dj = __builtin_fma(fy, bot - top, top);
  const double z = __builtin_fma(d, __builtin_fma(nb.zr[0], px, __builtin_fma(nb.zr[1], py, nb.zr[2])), nb.zr[3]);
  const double gap = __builtin_fma(-tau_d, dj, fabs(z - dj));
  if (!(fabs(gap) > __builtin_fma(2.0 + tau_d, ed, delta))) return -1;
  if (gap > 0.0) return 0;
  // n_0 . N n_j in FP32: off by less than 2e-6 of the magnitudes' product
  const float w0 = __builtin_fmaf(nb.N[0], m0, __builtin_fmaf(nb.N[1], m1, nb.N[2] * m2));
  const float w1 = __builtin_fmaf(nb.N[3], m0, __builtin_fmaf(nb.N[4], m1, nb.N[5] * m2));
  const float w2 = __builtin_fmaf(nb.N[6], m0, __builtin_fmaf(nb.N[7], m1, nb.N[8] * m2));
  const float gapn = __builtin_fmaf(n0, w0, __builtin_fmaf(n1, w1, n2 * w2)) - cos_n;
  const float en = __builtin_fmaf(2e-6f, (fabsf(n0) + fabsf(n1) + fabsf(n2)) * (fabsf(m0) + fabsf(m1) + fabsf(m2)), 5e-7f);
  if (!(fabsf(gapn) > en)) return -1;
  if (gapn < 0.0f) return 0;
  // neighbour j's point back on the reference image
  double q[3];
#pragma unroll
  for (int k = 0; k < 3; ++k)
    q[k] = __builtin_fma(dj, __builtin_fma(nb.Q[3 * k], u, __builtin_fma(nb.Q[3 * k + 1], v, nb.Q[3 * k + 2])), nb.w[k]);
  const double db = __builtin_fma(nb.cb, dj, __builtin_fma(nb.b2, ed, nb.b0));
  const double eq = nb.qw * db;
  if (!(q[2] > eq)) return q[2] < -eq ? 0 : -1;
  const double rq = rcp_near(q[2]);
  const double ex = __builtin_fma(q[0], rq, -px), ey = __builtin_fma(q[1], rq, -py);
  const double err2 = __builtin_fma(ex, ex, ey * ey);
  // m bounds either coordinate's difference inside the image or within twice the threshold of
  // it; below 1/4, a position further out is beyond the threshold in either form, as is one
  // with err2 > 4 (tau2 + 1); nearer, err2 differs by at most 6 m sqrt(tau2 + 1) + 2 m^2, and m
  // counts four times
  const double m = __builtin_fma(db * rq, nb.qu, nb.qe);
  if (!(m < 0.25)) return -1;
  if (!(fabs(err2 - tau2) > m * __builtin_fma(4.0, tau2, 5.0))) return err2 > __builtin_fma(4.0, tau2, 4.0) ? 0 : -1;
  return err2 < tau2 ? 1 : 0;
}

__global__ __launch_bounds__(256) void filter_kernel(FilterArgs a) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x, y = blockIdx.y;
  if (x >= a.W || y >= a.H) return;
  const size_t p = (size_t)y * a.W + x;
  const float df = a.depth[p];
  const float n0 = a.normal[3 * p], n1 = a.normal[3 * p + 1], n2 = a.normal[3 * p + 2];
  const double d = (double)df;
  int count = 0;
  if (d > 0.0)
    for (int k = 0; k < a.n_nbrs; ++k) {
      int c = consistent_short(a.nbrs[k], (double)x, (double)y, d, n0, n1, n2, a.tau_d, (float)a.cos_n,
                               a.tau_r * a.tau_r);
      if (c < 0) c = consistent(a, a.nbrs[k], x, y, d, n0, n1, n2) ? 1 : 0;
      count += c;
    }
  const bool keep = d > 0.0 && count >= a.min_consistent;
  a.count_out[p] = (uint8_t)min(count, 255);
  a.depth_out[p] = keep ? df : 0.0f;
  a.normal_out[3 * p] = keep ? n0 : 0.0f;
  a.normal_out[3 * p + 1] = keep ? n1 : 0.0f;
  a.normal_out[3 * p + 2] = keep ? n2 : 0.0f;
}

}  // namespace pmf

namespace phimvs_internal {

hipError_t launch_filter(const FilterArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(pmf::filter_kernel, dim3((a.W + 255) / 256, a.H), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace phimvs_internal
