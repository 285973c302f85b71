// Depth-map fusion (PHI-MVS Sec. III-F) as a sequence of data-parallel steps.  The paper
// walks the maps in order and, within a map, its pixels one by one; a later pixel only
// sees what earlier ones deleted.  Within one map's step the only state that changes is
// the deletion of pixels of later maps, and a pixel of map j is deleted by the first pixel
// (row-major) of map i that passes the test against it.  With a pixel's key its index in the
// concatenated maps, the pixel that deletes q is therefore the live one of the smallest key
// that passes, and one atomic minimum per test settles it for good: a claim of an earlier
// step is smaller than any later one's, and a claimed pixel is dead from the next step on.
// So each step is one launch (every live pixel of map i claims its candidates), and one
// launch at the end turns every pixel that nobody claimed into a point with the candidates
// it won, and writes each output once.  The result equals the sequential walk.
//
// All results are FP64 evaluations of the expressions in the order written (back_project,
// project_round, the squared distance).  The tests bound the work: FP64 instructions, about
// 200 for a pixel and a later map in that form (two camera chains through the world and two
// divisions).  They are decided by a shorter one, the same products in another order from
// tables (a pixel's position on image j; its point in the world, where the distance is taken:
// nothing is assumed of the rotations, which need not be orthonormal to the last digit),
// together with a bound of the difference between the two; a lane whose test lies within that
// bound of the other outcome (a rounding boundary of the pixel position, the distance limit)
// takes the expressions as written, so the decisions are theirs.  Nine 961 x 640 maps (5.5 M pixels):
// 404-422 us a call with both launches in every step (init 47, claims refilled 64, claim 142, merge
// 154 us) and the written form throughout, 273-298 us so, depending on the machine (init 12, claim
// 180, merge 84 us: the merge issues FP64 on 75% of its cycles; the first claim launch, 50 us, has
// 18 us of atomics, which memory carries out).

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "phimvs_internal.h"

namespace pmu {

using namespace phimvs_internal;

constexpr int kBlock = 256;
constexpr int kGroup = 4;
constexpr uint64_t kFree = ~0ull;  // claim of a pixel nobody has taken

// pixel (x, y) at depth d of a map's camera -> world point: R^T (d K^-1 (x, y, 1) - t)
__device__ __forceinline__ void back_project(const FuseMap& m, int x, int y, double d, double* Xw) {
  const double px = (double)x, py = (double)y;
  double X[3];
  for (int k = 0; k < 3; ++k) X[k] = d * (m.Kinv[3 * k] * px + m.Kinv[3 * k + 1] * py + m.Kinv[3 * k + 2] * 1.0);
  const double d0 = X[0] - m.t[0], d1 = X[1] - m.t[1], d2 = X[2] - m.t[2];
  for (int k = 0; k < 3; ++k) Xw[k] = m.R[k] * d0 + m.R[3 + k] * d1 + m.R[6 + k] * d2;
}

// nearest pixel of map m that world point Xw projects to; false when behind the camera
// or outside the image
__device__ __forceinline__ bool project_round(const FuseMap& m, const double* Xw, int& qx, int& qy) {
  double X[3], p[3];
  for (int k = 0; k < 3; ++k) X[k] = m.R[3 * k] * Xw[0] + m.R[3 * k + 1] * Xw[1] + m.R[3 * k + 2] * Xw[2] + m.t[k];
  for (int k = 0; k < 3; ++k) p[k] = m.K[3 * k] * X[0] + m.K[3 * k + 1] * X[1] + m.K[3 * k + 2] * X[2];
  if (!(p[2] > 0.0)) return false;
  const double xr = floor(p[0] / p[2] + 0.5), yr = floor(p[1] / p[2] + 0.5);
  if (!(xr >= 0.0 && xr <= (double)(m.W - 1) && yr >= 0.0 && yr <= (double)(m.H - 1))) return false;
  qx = (int)xr;
  qy = (int)yr;
  return true;
}

// ---------------------------------------------------------------------------- the short form
// Pair (i, j): pixel (x, y) of map i at depth d is p = d P (x, y, 1) + s on image j, P = K_j A, s =
// K_j t, A = R_j R_i^T K_i^-1, t = t_j - R_j R_i^T t_i.  A point in camera j differs between the two
// forms by at most delta = c0 + c1 d in any coordinate: 512 x 2^-53 of the magnitudes that enter
// (the forms are a few 3-term products of them, each within a few units), and p by kn delta with
// kn the row's sum of magnitudes in K_j, counted four times here.  cu and cv bound the position's
// share of that for positions inside image j or within a pixel of it, eu and ev the quotient's
// own rounding.  The way to the world (FuseMap's B, w, e0, e1) is bounded in the same way.
__device__ void make_pair(const FuseMap& a, const FuseMap& b, FusePair& o) {
  double R[9], A[9], t[3], kn[3];
  for (int r = 0; r < 3; ++r)
    for (int c = 0; c < 3; ++c)
      R[3 * r + c] = b.R[3 * r] * a.R[3 * c] + b.R[3 * r + 1] * a.R[3 * c + 1] + b.R[3 * r + 2] * a.R[3 * c + 2];
  double ray = 0.0, ti = 0.0, tj = 0.0;
  for (int r = 0; r < 3; ++r) {
    for (int c = 0; c < 3; ++c)
      A[3 * r + c] = R[3 * r] * a.Kinv[c] + R[3 * r + 1] * a.Kinv[3 + c] + R[3 * r + 2] * a.Kinv[6 + c];
    t[r] = b.t[r] - (R[3 * r] * a.t[0] + R[3 * r + 1] * a.t[1] + R[3 * r + 2] * a.t[2]);
    ray += fabs(a.Kinv[3 * r]) * a.W + fabs(a.Kinv[3 * r + 1]) * a.H + fabs(a.Kinv[3 * r + 2]);
    ti += fabs(a.t[r]);
    tj += fabs(b.t[r]);
    kn[r] = fabs(b.K[3 * r]) + fabs(b.K[3 * r + 1]) + fabs(b.K[3 * r + 2]);
  }
  for (int r = 0; r < 3; ++r) {
    for (int c = 0; c < 3; ++c)
      o.P[3 * r + c] = b.K[3 * r] * A[c] + b.K[3 * r + 1] * A[3 + c] + b.K[3 * r + 2] * A[6 + c];
    o.s[r] = b.K[3 * r] * t[0] + b.K[3 * r + 1] * t[1] + b.K[3 * r + 2] * t[2];
  }
  o.c0 = 512.0 * 0x1p-53 * (ti + tj);
  o.c1 = 512.0 * 0x1p-53 * ray;
  o.kw = 4.0 * kn[2];
  o.cu = 4.0 * (kn[0] + (b.W + 1) * kn[2]);
  o.cv = 4.0 * (kn[1] + (b.H + 1) * kn[2]);
  o.eu = 0x1p-46 * (b.W + 2);
  o.ev = 0x1p-46 * (b.H + 2);
}

// 1 / x to within a few units in the last place (x normal)
__device__ __forceinline__ double rcp_near(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
  return __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
}

// The pixel of map j nearest to the projection of pixel (x, y) of map i at depth d: 1 found
// (qx, qy), 0 none, -1 too close to call.
__device__ __forceinline__ int project_short(const FuseMap& mj, const FusePair& P, double px, double py, double d,
                                             double delta, int& qx, int& qy) {
  double p[3];
#pragma unroll
  for (int k = 0; k < 3; ++k)
    p[k] = __builtin_fma(d, __builtin_fma(P.P[3 * k], px, __builtin_fma(P.P[3 * k + 1], py, P.P[3 * k + 2])), P.s[k]);
  const double e2 = P.kw * delta;
  if (!(p[2] > e2)) return p[2] < -e2 ? 0 : -1;
  const double r = rcp_near(p[2]);
  const double u = p[0] * r, v = p[1] * r, rd = delta * r;
  const double mu = __builtin_fma(rd, P.cu, P.eu), mv = __builtin_fma(rd, P.cv, P.ev);
  // with these below 1/4, a position more than a pixel outside is outside in either form
  if (!(mu < 0.25 && mv < 0.25)) return -1;
  if (!(u >= -1.0 && u <= (double)mj.W && v >= -1.0 && v <= (double)mj.H)) return 0;
  const double xs = u + 0.5, ys = v + 0.5;
  const double xr = floor(xs), yr = floor(ys);
  const double fx = xs - xr, fy = ys - yr;
  if (!(fx >= mu && fx <= 1.0 - mu && fy >= mv && fy <= 1.0 - mv)) return -1;
  qx = (int)xr;
  qy = (int)yr;
  return (unsigned)qx < (unsigned)mj.W && (unsigned)qy < (unsigned)mj.H ? 1 : 0;
}

// s / n, rounded once: a quotient by the rounded reciprocal and one correction by its remainder
// is the correctly rounded quotient (Markstein) where nothing over- or underflows
__device__ __forceinline__ double div_by(double s, double n, double rn) {
  const double q = s * rn;
  const double c = __builtin_fma(__builtin_fma(-n, q, s), rn, q);
  return fabs(s) < 0x1p900 && fabs(s) > 0x1p-900 ? c : s / n;
}

__global__ __launch_bounds__(kBlock) void fuse_pairs_kernel(const FuseMap* __restrict__ maps, int n_maps, int row0,
                                                            int rows, FusePair* __restrict__ pairs) {
  const int k = blockIdx.x * kBlock + threadIdx.x;
  const int i = row0 + k / n_maps, j = k % n_maps;
  if (k < rows * n_maps && j > i) make_pair(maps[i], maps[j], pairs[k]);
}

// claims of every pixel free; the first rows of the pair table
__global__ __launch_bounds__(kBlock) void fuse_init_kernel(const FuseMap* __restrict__ maps, int n_maps, int rows,
                                                           FusePair* __restrict__ pairs, uint64_t* __restrict__ claim,
                                                           int64_t total) {
  const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (k < (int64_t)rows * n_maps) {
    const int i = (int)(k / n_maps), j = (int)(k % n_maps);
    if (j > i) make_pair(maps[i], maps[j], pairs[k]);
  }
  if (2 * k + 1 < total) {
    reinterpret_cast<ulonglong2*>(claim)[k] = make_ulonglong2(kFree, kFree);
  } else if (2 * k < total) {
    claim[2 * k] = kFree;
  }
}

// every live pixel of map i claims, in each later map, the candidate that passes the test;
// passed: which of the next 32 maps it found one in
__global__ __launch_bounds__(kBlock) void fuse_claim_kernel(const FuseMap* __restrict__ maps, int n_maps, int i,
                                                            const FusePair* __restrict__ row, double tau,
                                                            uint64_t* __restrict__ claim,
                                                            uint32_t* __restrict__ passed) {
  const FuseMap& mi = maps[i];
  const int x = blockIdx.x * kBlock + threadIdx.x, y = blockIdx.y;
  if (x >= mi.W) return;
  const int64_t p = (int64_t)y * mi.W + x, g = mi.off + p;
  const float df = mi.depth[p];
  if (!(df > 0.0f) || claim[g] != kFree) return;
  const double d = df, px = (double)x, py = (double)y;
  const double lim = tau * d, lim2 = lim * lim, ei = __builtin_fma(mi.e1, d, mi.e0);
  double Xs[3];  // the pixel's point
#pragma unroll
  for (int r = 0; r < 3; ++r)
    Xs[r] = __builtin_fma(d, __builtin_fma(mi.B[3 * r], px, __builtin_fma(mi.B[3 * r + 1], py, mi.B[3 * r + 2])), mi.w[r]);
  uint32_t bits = 0;
  // kGroup maps at a time, so that their gathers are in flight together and no gather waits
  // for an atomic of the map before
  for (int j0 = i + 1; j0 < n_maps; j0 += kGroup) {
    int found[kGroup];
    int64_t at[kGroup];
    int qx[kGroup], qy[kGroup];
    float dq[kGroup];
    uint64_t cl[kGroup];
#pragma unroll
    for (int k = 0; k < kGroup; ++k) {
      found[k] = 0;
      dq[k] = 0.0f;
      cl[k] = 0;
      at[k] = 0;
      if (j0 + k >= n_maps) continue;
      const FuseMap& mj = maps[j0 + k];
      const FusePair& P = row[j0 + k];
      found[k] = project_short(mj, P, px, py, d, __builtin_fma(P.c1, d, P.c0), qx[k], qy[k]);
      if (found[k] < 0) {
        double Xi[3];
        back_project(mi, x, y, d, Xi);
        found[k] = project_round(mj, Xi, qx[k], qy[k]) ? 2 : 0;
      }
      if (found[k]) {
        const int q = qy[k] * mj.W + qx[k];
        dq[k] = mj.depth[q];
        at[k] = mj.off + q;
        // a claim only ever gets smaller, so one below this pixel's key already has the
        // candidate (an ordinary load, which may show an older value)
        cl[k] = claim[at[k]];
      }
    }
    bool pass[kGroup];
#pragma unroll
    for (int k = 0; k < kGroup; ++k) {
      pass[k] = false;
      if (!found[k] || !(dq[k] > 0.0f) || cl[k] < (uint64_t)g) continue;
      const FuseMap& mj = maps[j0 + k];
      if (found[k] == 1) {
        // the candidate's point
        const double dd = dq[k], qxd = (double)qx[k], qyd = (double)qy[k];
        double e2 = 0.0;
#pragma unroll
        for (int r = 0; r < 3; ++r) {
          const double Y = __builtin_fma(
              dd, __builtin_fma(mj.B[3 * r], qxd, __builtin_fma(mj.B[3 * r + 1], qyd, mj.B[3 * r + 2])), mj.w[r]);
          const double e = Y - Xs[r];
          e2 = __builtin_fma(e, e, e2);
        }
        // both points through both forms; |e| is near lim where it matters, or below 21 dl
        const double dl = ei + __builtin_fma(mj.e1, dd, mj.e0);
        const double m = 64.0 * dl * lim + 0x1p-40 * lim2 + 512.0 * dl * dl;
        pass[k] = e2 < lim2;
        if (!(fabs(e2 - lim2) > m)) found[k] = 2;
      }
      if (found[k] == 2) {
        double Xi[3], Yw[3];
        back_project(mi, x, y, d, Xi);
        back_project(mj, qx[k], qy[k], (double)dq[k], Yw);
        const double e0 = Yw[0] - Xi[0], e1 = Yw[1] - Xi[1], ez = Yw[2] - Xi[2];
        pass[k] = e0 * e0 + e1 * e1 + ez * ez < lim * lim;
      }
    }
#pragma unroll
    for (int k = 0; k < kGroup; ++k) {
      if (!pass[k]) continue;
      atomicMin((unsigned long long*)&claim[at[k]], (unsigned long long)g);
      if (j0 + k - i <= 32) bits |= 1u << (j0 + k - i - 1);
    }
  }
  passed[g] = bits;
}

// every pixel of maps [i0, i0 + gridDim.z) that nobody claimed becomes a point with the
// candidates it won
__global__ __launch_bounds__(kBlock) void fuse_merge_kernel(const FuseMap* __restrict__ maps, int n_maps, int i0,
                                                            const FusePair* __restrict__ pairs,
                                                            const uint64_t* __restrict__ claim,
                                                            const uint32_t* __restrict__ passed,
                                                            float* __restrict__ points, int32_t* __restrict__ support,
                                                            int64_t* __restrict__ owner) {
  const int i = i0 + blockIdx.z;
  const FuseMap& mi = maps[i];
  const int x = blockIdx.x * kBlock + threadIdx.x, y = blockIdx.y;
  if (x >= mi.W || y >= mi.H) return;
  const int64_t p = (int64_t)y * mi.W + x, g = mi.off + p;
  const float df = mi.depth[p];
  const uint64_t c = claim[g];
  float o[3] = {0.0f, 0.0f, 0.0f};
  int count = 0;
  int64_t own = df > 0.0f ? (int64_t)c : -1;
  if (df > 0.0f && c == kFree) {
    own = g;
    const double d = df;
    double Xi[3];
    back_project(mi, x, y, d, Xi);
    double sum[3] = {Xi[0], Xi[1], Xi[2]};
    count = 1;
    const uint32_t bits = i + 1 < n_maps ? passed[g] : 0u;
    // as above, the gathers of kGroup maps in flight together
    for (int j0 = i + 1; j0 < n_maps; j0 += kGroup) {
      int qx[kGroup], qy[kGroup];
      uint64_t cl[kGroup];
      float dq[kGroup];
#pragma unroll
      for (int k = 0; k < kGroup; ++k) {
        cl[k] = kFree;
        dq[k] = 0.0f;
        const int j = j0 + k;
        if (j >= n_maps || (j - i <= 32 && !(bits >> (j - i - 1) & 1u))) continue;
        const FuseMap& mj = maps[j];
        const FusePair& P = pairs[(int64_t)(i - i0) * n_maps + j];
        int found = project_short(mj, P, (double)x, (double)y, d, __builtin_fma(P.c1, d, P.c0), qx[k], qy[k]);
        if (found < 0) found = project_round(mj, Xi, qx[k], qy[k]) ? 1 : 0;
        if (!found) continue;
        const int q = qy[k] * mj.W + qx[k];
        cl[k] = claim[mj.off + q];
        dq[k] = mj.depth[q];
      }
#pragma unroll
      for (int k = 0; k < kGroup; ++k) {
        // a claim by this pixel means q was live and passed the test
        if (cl[k] != (uint64_t)g) continue;
        double Yw[3];
        back_project(maps[j0 + k], qx[k], qy[k], (double)dq[k], Yw);
        for (int r = 0; r < 3; ++r) sum[r] = sum[r] + Yw[r];
        ++count;
      }
    }
    const double n = (double)count, rn = 1.0 / n;
    for (int k = 0; k < 3; ++k) o[k] = (float)div_by(sum[k], n, rn);
  }
  owner[g] = own;
  support[g] = count;
  for (int k = 0; k < 3; ++k) points[3 * g + k] = o[k];
}

}  // namespace pmu

namespace phimvs_internal {

// rows of the pair table held at a time
static int fuse_rows(int n_maps) { return std::min(n_maps, std::max(1, 65536 / n_maps)); }

size_t fuse_pairs(int n_maps) { return (size_t)fuse_rows(n_maps) * n_maps; }

hipError_t launch_fuse(const FuseMap* h_maps, const FuseMap* d_maps, int n_maps, double tau, FusePair* pairs,
                       uint64_t* claim, uint32_t* passed, float* points, int32_t* support, int64_t* owner,
                       hipStream_t st) {
  using pmu::kBlock;
  const int64_t total = h_maps[n_maps - 1].off + (int64_t)h_maps[n_maps - 1].W * h_maps[n_maps - 1].H;
  const int rows = fuse_rows(n_maps);
  const int64_t init = std::max<int64_t>((total + 1) / 2, (int64_t)rows * n_maps);
  hipLaunchKernelGGL(pmu::fuse_init_kernel, dim3((unsigned)((init + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, d_maps,
                     n_maps, rows, pairs, claim, total);
  for (int i0 = 0; i0 < n_maps; i0 += rows) {
    const int nr = std::min(rows, n_maps - i0);
    if (i0 > 0)
      hipLaunchKernelGGL(pmu::fuse_pairs_kernel, dim3((unsigned)((nr * n_maps + kBlock - 1) / kBlock)), dim3(kBlock), 0,
                         st, d_maps, n_maps, i0, nr, pairs);
    int wmax = 1, hmax = 1;
    for (int i = i0; i < i0 + nr; ++i) {
      wmax = std::max(wmax, h_maps[i].W);
      hmax = std::max(hmax, h_maps[i].H);
      if (i + 1 < n_maps)
        hipLaunchKernelGGL(pmu::fuse_claim_kernel, dim3((unsigned)((h_maps[i].W + kBlock - 1) / kBlock), h_maps[i].H),
                           dim3(kBlock), 0, st, d_maps, n_maps, i, pairs + (size_t)(i - i0) * n_maps, tau, claim, passed);
    }
    hipLaunchKernelGGL(pmu::fuse_merge_kernel, dim3((unsigned)((wmax + kBlock - 1) / kBlock), hmax, nr), dim3(kBlock), 0,
                       st, d_maps, n_maps, i0, pairs, claim, passed, points, support, owner);
  }
  return hipGetLastError();
}

}  // namespace phimvs_internal
