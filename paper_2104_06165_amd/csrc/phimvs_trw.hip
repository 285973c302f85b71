// Selection step of plane hypothesis inference on the GPU (PHI-MVS Sec. III-E): the graph
// model of phimvs_mrf.hip (node states, potentials, sequential tree-reweighted message passing
// in raster order, labelling in raster order), with the same FP64 operations in the same order
// per node.  Only the logarithms are each platform's own (3% of them differ, by an ulp), which
// can tell apart labels that tie to within rounding; where a node has such a tie the host takes
// the logarithms (trw_ties_kernel, launch_trw_potentials) and the sweeps run again, so the labels are the
// host decoder's.
//
// A node of a forward sweep needs its left and upper neighbours of the same sweep, so W + H - 1
// steps follow one another: a sweep is a chain, and what bounds it is the time of a step.  One
// wave takes 32 rows, two lanes per node (lane h: states 2h and 2h + 1), and walks them in a
// skewed order: step s holds (x, y) with x + (row in the band) = s.  What a node sends to the
// right stays in its lanes for the next step, what it sends down moves two lanes on (no LDS, no
// barrier on the way), and from a band's last row to the next band it goes through memory: slots
// that hold a value no message has until they are filled, taken kChunk columns at a time.  All the
// rest (unary terms, edge energies, the other sweep's messages) lies in memory in the order of the
// steps and is loaded kAhead steps ahead.  A backward sweep is the same walk with s, rows and
// bands descending.  Each band takes its number from a counter, so the band it waits for has
// always started before it and does not wait for it: every wait ends.
// At 1600 x 1066 pixels (426400 nodes, 36% of them with two to four states) the selection took
// 47-58 ms with the host decoder and takes 8.9 ms: 0.9 ms before and after the sweeps, 0.50 ms for
// each of 16 sweeps of 1584 steps.  A step is 0.31 us, about 135 instructions that one wave issues
// alone.  Measured before: four lanes per node, 64 rows in four waves with a barrier per step
// 0.52 us (17.3 ms, the columns announced by a counter with fences; 13.9 with slots); this form
// with 64-bit addresses in the vector unit 0.39 us (10.8 ms).  Chunks of 8 columns or 3 or 5 steps
// ahead change nothing (8.9-9.2 ms).

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "phimvs_internal.h"

namespace pmt {

using namespace phimvs_internal;

constexpr int kRows = 32;   // rows of a band: two lanes each
constexpr int kChunk = 16;  // columns taken from band to band at a time
constexpr int kAhead = 4;   // steps between a load and its use

// what a slot between two bands holds until it is filled: a signalling NaN, which no FP64 operation
// returns
constexpr double kEmpty = __builtin_nans("0x5e9d");
__device__ __forceinline__ bool is_empty(double x) {
  return __builtin_bit_cast(unsigned long long, x) == __builtin_bit_cast(unsigned long long, kEmpty);
}

__device__ __forceinline__ double edge_distance(double h1, double h2) {
  const double rel = h1 > h2 ? (h1 - h2) / h2 : (h2 - h1) / h1;
  return rel < 1.0 ? rel : 1.0;
}
__device__ __forceinline__ double edge_potential(double h1, double h2, double k3) {
  const double m = edge_distance(h1, h2);
  return (k3 - m) * (k3 - m);
}

// labels within this of each other (for up to 8 iterations, and times the largest energy, taken to
// be at least kTieScale) are settled with the host's logarithms (trw_ties_kernel)
constexpr double kTieGap = 1e-14, kTieScale = 4.0;

// info of a node: its states (3 bits), whether its upper and left neighbours have any
constexpr int kLiveUp = 8, kLiveLeft = 16;

struct Nodes {
  const float* depth;
  const float* hyp;
  const float* cost;
  int W, H;  // full size
};

// states of node (X, Y): its depth, or the hypotheses present, in order
__device__ __forceinline__ int node_states(const Nodes& g, int W2, int H2, int X, int Y, float* v) {
  if (X < 0 || Y < 0 || X >= W2 || Y >= H2) return 0;
  const size_t p = (size_t)(2 * Y) * g.W + 2 * X, plane = (size_t)g.W * g.H;
  const float d = g.depth[p];
  if (d > 0.0f) {
    v[0] = d;
    return 1;
  }
  int n = 0;
  for (int k = 0; k < 4; ++k) {
    const float h = g.hyp[k * plane + p];
    if (h > 0.0f) v[n++] = h;
  }
  return n;
}

// one quad of lanes per position of the skewed layout (lane l: state l): node data, edge
// energies, messages 0; and the slots between the bands empty
__global__ __launch_bounds__(256) void trw_setup_kernel(Nodes g, TrwBuffers B, double k1, double k2, double k3,
                                                        double cost_max) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, at = t >> 2;
  if (at >= B.positions) return;
  const int l = (int)threadIdx.x & 3;
  if (t < (int64_t)B.NB * B.S * 4) B.edge[t] = kEmpty;
  const int r = (int)(at % kRows);
  const int64_t bs = at / kRows;
  const int s = (int)(bs % B.S), b = (int)(bs / B.S);
  const int X = s - r, Y = b * kRows + r;
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  const int n = node_states(g, B.W, B.H, X, Y, v);
  const float mine = l == 0 ? v[0] : (l == 1 ? v[1] : (l == 2 ? v[2] : v[3]));
  double un = __builtin_inf();
  double gamma = 1.0;
  int info = 0;
  double er[4], ed[4];
  for (int j = 0; j < 4; ++j) er[j] = ed[j] = __builtin_inf();
  if (n) {
    const size_t p = (size_t)(2 * Y) * g.W + 2 * X, plane = (size_t)g.W * g.H;
    if (g.depth[p] > 0.0f) {
      if (l == 0) un = 0.0;
    } else if (l < n) {
      int i = 0, mk = 0;
      for (int k = 0; k < 4; ++k)
        if (g.hyp[k * plane + p] > 0.0f && i++ == l) mk = k;
      const double phi = (cost_max - (double)g.cost[mk * plane + p]) / k1 + k2;
      un = -log(phi);
      if (!(phi > 0.0)) atomicOr(B.flag, kTrwInvalid);
      else if (!(fabs(un) < __builtin_inf())) atomicOr(B.flag, kTrwInfinite);
      else if (fabs(un) > kTieScale) atomicMax(B.flag + 1, __float_as_int((float)fabs(un)));
    }
    float w[4];
    const int up = node_states(g, B.W, B.H, X, Y - 1, w), left = node_states(g, B.W, B.H, X - 1, Y, w);
    const int right = node_states(g, B.W, B.H, X + 1, Y, w);
    if (l < n)
      for (int j = 0; j < right; ++j) er[j] = n * right > 1 ? -log(edge_potential(mine, w[j], k3)) : 0.0;
    const int down = node_states(g, B.W, B.H, X, Y + 1, w);
    if (l < n)
      for (int j = 0; j < down; ++j) ed[j] = n * down > 1 ? -log(edge_potential(mine, w[j], k3)) : 0.0;
    if ((up && left) || (right && down)) gamma = 0.5;
    info = n | (up ? kLiveUp : 0) | (left ? kLiveLeft : 0);
  }
  if (l == 0) {
    B.gamma[at] = gamma;
    B.info[at] = info;
  }
  B.un[t] = un;
  B.val[t] = mine;
  for (int d = 0; d < 4; ++d) B.msg[d][t] = 0.0;
  for (int j = 0; j < 4; ++j) {
    B.er[4 * t + j] = er[j];
    B.ed[4 * t + j] = ed[j];
  }
}

template <int CTRL>
__device__ __forceinline__ double dpp(double old, double x) {
  const int2 o = __builtin_bit_cast(int2, old), v = __builtin_bit_cast(int2, x);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_update_dpp(o.x, v.x, CTRL, 0xf, 0xf, false),
                                              __builtin_amdgcn_update_dpp(o.y, v.y, CTRL, 0xf, 0xf, false)));
}
__device__ __forceinline__ int pick_other(int x) { return __builtin_amdgcn_update_dpp(x, x, 0xB1, 0xf, 0xf, false); }
// the other lane of the node (quad_perm [1, 0, 3, 2])
__device__ __forceinline__ double other(double x) {
  const int2 v = __builtin_bit_cast(int2, x);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_update_dpp(0, v.x, 0xB1, 0xf, 0xf, true),
                                              __builtin_amdgcn_update_dpp(0, v.y, 0xB1, 0xf, 0xf, true)));
}
// 16 bytes at lane offset v + wave offset s (in bytes) of a buffer
using Words4 = int __attribute__((ext_vector_type(4)));
__device__ __forceinline__ double2 load16(__amdgpu_buffer_rsrc_t b, unsigned v, unsigned s) {
  return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(b, (int)v, (int)s, 0));
}
__device__ __forceinline__ void store16(__amdgpu_buffer_rsrc_t b, unsigned v, unsigned s, double2 x) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(Words4, x), b, (int)v, (int)s, 0);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const void* p) {
  // the compiler sees no constants, or it puts each descriptor together anew at each use
  int size = -1, flags = 0x00027000;
  asm volatile("" : "+s"(size), "+s"(flags));
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, size, flags);
}
// two lanes on (a wave's lanes shifted by one, twice); the first row takes its states' values of e
template <bool BWD>
__device__ __forceinline__ double2 next_row(double2 x, const double (&e)[4]) {
  constexpr int c = BWD ? 0x130 : 0x138;  // wave_shl:1, wave_shr:1
  constexpr int i = BWD ? 0 : 2;          // of the value shifted in first, which ends one lane further
  return make_double2(dpp<c>(e[2 - i], dpp<c>(e[i], x.x)), dpp<c>(e[3 - i], dpp<c>(e[i + 1], x.y)));
}

// a message: for states m = 2h, 2h + 1 there the min over the states here of a + e, less the least
// over m.  Energies of states that a node does not have are +inf, as are the unary terms, so inf
// and NaN (which lose in fmin) stand for "none", and where there is no neighbour at all or no node
// the difference of two infinities becomes 0.
struct Energies {
  double2 v[4];
};
template <bool BWD>
__device__ __forceinline__ double2 message(double2 a, const Energies& e) {
  const double o0 = other(a.x), o1 = other(a.y);
  double x, y;
  if (BWD) {
    x = fmin(fmin(a.x + e.v[0].x, a.y + e.v[0].y), fmin(o0 + e.v[2].x, o1 + e.v[2].y));
    y = fmin(fmin(a.x + e.v[1].x, a.y + e.v[1].y), fmin(o0 + e.v[3].x, o1 + e.v[3].y));
  } else {
    x = fmin(fmin(a.x + e.v[0].x, a.y + e.v[1].x), fmin(o0 + e.v[2].x, o1 + e.v[3].x));
    y = fmin(fmin(a.x + e.v[0].y, a.y + e.v[1].y), fmin(o0 + e.v[2].y, o1 + e.v[3].y));
  }
  double lo = fmin(x, y);
  lo = fmin(lo, other(lo));
  return make_double2(fmax(x - lo, 0.0), fmax(y - lo, 0.0));
}

// MODE 0: forward sweep, 1: backward sweep, 2: labelling (forward order)
template <int MODE>
__global__ __launch_bounds__(2 * kRows) void trw_sweep_kernel(TrwBuffers B, int sweep, float* __restrict__ dec) {
  constexpr bool BWD = MODE == 1;
  __shared__ double taken[kChunk][4];  // from the band before, for the first row
  const int t = (int)threadIdx.x, r = t >> 1, h = t & 1;
  int o = 0;
  if (t == 0) o = (int)(atomicAdd(B.ticket, 1ull) - (unsigned long long)sweep * B.NB);
  o = __builtin_amdgcn_readfirstlane(o);
  const int b = BWD ? B.NB - 1 - o : o;
  constexpr int last = BWD ? 0 : kRows - 1;  // the row that sends to the next band
  const bool from = o > 0, to = o + 1 < B.NB;
  const int S = B.S, W = B.W;
  struct Step {
    double g;
    int info;
    double2 un, m0, m1;
    Energies e0, e1;
    float2 v;
  };
  // The band's part of each array: the lane's offset stays, the step moves the wave's.
  const int64_t band = (int64_t)b * S * kRows;
  const auto un = buffer(B.un + 4 * band), m0 = buffer(B.msg[BWD ? 0 : 2] + 4 * band),
             m1 = buffer(B.msg[BWD ? 1 : 3] + 4 * band), out0 = buffer(B.msg[BWD ? 2 : 1] + 4 * band),
             out1 = buffer(B.msg[BWD ? 3 : 0] + 4 * band), gamma = buffer(B.gamma + band);
  // Forward: the node's own edges.  Else those of the left and the upper node, which hold them as
  // their right and down: one step before, and there the row above or the band before's last row,
  // as offsets from the band before's place.  Ahead of the first band lies room that is read but
  // not used.
  const auto er = buffer(B.er + 16 * (MODE == 0 ? band : band - kRows));
  const auto ed = buffer(B.ed + 16 * (MODE == 0 ? band : band - (int64_t)S * kRows));
  const unsigned up = r > 0 || b == 0 ? (unsigned)(S * kRows - kRows + r - 1) : (unsigned)(kRows * kRows - 1);
  // The pairs of energies of a lane, in doubles from an edge's first: forward, rows of this node's
  // states (the lane's two, then the other lane's) at columns 2h, 2h + 1; backward, rows 2h, 2h + 1
  // at the columns of the lane's states, then of the other's; labelling, rows 0..3
  unsigned at0[4], at1[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = MODE == 0 ? 4 * (2 * (i < 2 ? h : 1 - h) + (i & 1)) + 2 * h
                            : (MODE == 1 ? 4 * (2 * h + (i & 1)) + 2 * (i < 2 ? h : 1 - h) : 4 * i + 2 * h);
    at0[i] = 128u * r + 8u * c;
    at1[i] = 128u * (MODE == 0 ? (unsigned)r : up) + 8u * c;
  }
  // what step k needs from memory
  auto load = [&](int k, Step& q) {
    k = min(k, S - 1);
    const unsigned row = (unsigned)(BWD ? S - 1 - k : k) * kRows;  // position of row 0
    q.un = load16(un, 16u * t, 32 * row);
    q.m0 = load16(m0, 16u * t, 32 * row);
    q.m1 = load16(m1, 16u * t, 32 * row);
    if (MODE == 2) {
      q.v = *reinterpret_cast<const float2*>(B.val + 4 * (band + row) + 2 * t);
      q.info = (B.info + band + row)[r];
    } else {
      q.g = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(gamma, 8 * r, (int)(8 * row), 0));
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      q.e0.v[i] = load16(er, at0[i], 128 * row);
      q.e1.v[i] = load16(ed, at1[i], 128 * row);
    }
  };
  // The slots between two bands: one per step of the band before, whose last row is kRows - 1
  // steps behind its first.  The one for this band's step k0 + t / 4:
  auto slot = [&](int k0) -> double* {
    const int k = k0 + (t >> 2) + kRows - 1;
    return t < 4 * kChunk && k < S ? &B.edge[((size_t)o * S + k) * 4 + (t & 3)] : nullptr;
  };
  auto take = [&](const double* p) {
    return p ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0;
  };
  const bool sends = to && r == last;
  double* send = B.edge + (size_t)(to ? o + 1 : o) * S * 4 + 2 * h;
  if (t < 4 * kChunk) (&taken[0][0])[t] = 0.0;
  double2 pass = make_double2(0.0, 0.0), down = pass;  // to the row's next node, to the next row: messages, or the state taken
  double got = 0.0;
  if (from) got = take(slot(0));
  Step q[kAhead];
#pragma unroll
  for (int i = 0; i < kAhead; ++i) load(i, q[i]);
  for (int k0 = 0; k0 < S; k0 += kChunk) {
    if (from) {
      // what the band before sends to the first row in the next kChunk steps: each slot is taken
      // when it is filled, and left empty for the next sweep
      double* p = slot(k0);
      while (__any(is_empty(got))) {
        __builtin_amdgcn_s_sleep(1);
        got = take(p);
      }
      if (p) __hip_atomic_store(p, kEmpty, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (t < 4 * kChunk) (&taken[0][0])[t] = got;
    }
    __builtin_amdgcn_wave_barrier();
    double e[4];
    for (int i = 0; i < 4; ++i) e[i] = taken[0][i];
#pragma unroll
    for (int kk = 0; kk < kChunk; ++kk) {
      const int k = k0 + kk;
      Step& c = q[kk % kAhead];
      const int s = BWD ? S - 1 - k : k;
      const unsigned row = (unsigned)s * kRows;
      const double2 in = next_row<BWD>(down, e);
      if (kk + 1 < kChunk)
        for (int i = 0; i < 4; ++i) e[i] = taken[kk + 1][i];
      if (MODE < 2) {
        // messages from (up, left, right, down)
        const double2 mu = BWD ? c.m0 : in, ml = BWD ? c.m1 : pass;
        const double2 mr = BWD ? pass : c.m0, md = BWD ? in : c.m1;
        const double gx = c.g * ((((c.un.x + mu.x) + ml.x) + mr.x) + md.x);
        const double gy = c.g * ((((c.un.y + mu.y) + ml.y) + mr.y) + md.y);
        store16(out0, 16u * t, 32 * row, pass);
        store16(out1, 16u * t, 32 * row, in);
        const double2 sv = BWD ? mu : md, ss = BWD ? ml : mr;
        down = message<BWD>(make_double2(gx - sv.x, gy - sv.y), c.e1);
        pass = message<BWD>(make_double2(gx - ss.x, gy - ss.y), c.e0);
      } else {
        // earlier neighbours by the state they took, later ones by their messages; the first
        // least state
        const int x = s - r, n = c.info & 7;
        const float vx = c.v.x, vy = c.v.y;
        const int pu = (int)in.x, pl = (int)pass.x;
        double2 eu = c.e1.v[0], el = c.e0.v[0];
#pragma unroll
        for (int i = 1; i < 4; ++i) {
          eu = make_double2(pu == i ? c.e1.v[i].x : eu.x, pu == i ? c.e1.v[i].y : eu.y);
          el = make_double2(pl == i ? c.e0.v[i].x : el.x, pl == i ? c.e0.v[i].y : el.y);
        }
        double ex = c.un.x, ey = c.un.y;
        if (c.info & kLiveUp) ex += eu.x, ey += eu.y;
        if (c.info & kLiveLeft) ex += el.x, ey += el.y;
        ex = (ex + c.m0.x) + c.m1.x;
        ey = (ey + c.m0.y) + c.m1.y;
        if (2 * h >= n) ex = __builtin_inf();
        if (2 * h + 1 >= n) ey = __builtin_inf();
        double least = ey < ex ? ey : ex;
        int pick = ey < ex ? 2 * h + 1 : 2 * h;
        const double theirs = other(least);
        const int their = pick_other(pick);
        if (theirs < least || (theirs == least && their < pick)) pick = their;
        if (x >= 0 && x < W && b * kRows + r < B.H && (n ? h == pick >> 1 : h == 0))
          dec[(size_t)(b * kRows + r) * W + x] = n ? (pick & 1 ? vy : vx) : 0.0f;
        pass = down = make_double2((double)pick, (double)pick);
      }
      if (sends) {
        __hip_atomic_store(send + 4 * kk, down.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(send + 4 * kk + 1, down.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (kk == kChunk / 2 && from) got = take(slot(k0 + kChunk));
      load(k + kAhead, c);
    }
    send += 4 * kChunk;
  }
}

// Whether the labels hang on rounding.  The energies here and on the host differ by an ulp of a
// logarithm; the messages then by 1e-15 of the largest energy after 8 iterations and by up to 1e-14
// of it after 200 (measured on the CPU, one-ulp changes of every energy, k3 from 1 + 1e-7 to 1000).
// So a node decides alike in both unless another state's energy lies within kTieGap times that
// energy (at least 4, the common potentials' 2.3 among them) of the least, 10 times what was
// measured.  Left out: states of the same depth (the label does not show), and states that nothing
// tells apart in either: the same cost, and what the neighbours contribute goes through equal
// relative distances (saturated ones as a rule), so they tie exactly in both.  What remains in
// filled maps are hypotheses that agree to six digits, on either side of which the energy is flat:
// one map of 24 (960 x 640 to 3200 x 2130), none of 80 of 1600 x 1066.  One quad of lanes per
// position, lane l: state l.  23 us at 1600 x 1066.
__device__ float state_cost(const Nodes& g, int X, int Y, int l) {
  const size_t p = (size_t)(2 * Y) * g.W + 2 * X, plane = (size_t)g.W * g.H;
  int i = 0;
  for (int k = 0; k < 4; ++k)
    if (g.hyp[k * plane + p] > 0.0f && i++ == l) return g.cost[k * plane + p];
  return 0.0f;
}
__global__ __launch_bounds__(256) void trw_ties_kernel(Nodes g, TrwBuffers B, double gap, double scale, bool sent,
                                                       const float* __restrict__ dec) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, at = t >> 2;
  if (at >= B.positions) return;  // whole quads
  const int l = (int)threadIdx.x & 3;
  const int r = (int)(at % kRows);
  const int64_t bs = at / kRows;
  const int X = (int)(bs % B.S) - r, Y = (int)(bs / B.S) * kRows + r;
  const int info = B.info[at], n = info & 7;
  if (n < 2) return;
  // the state a node took: the first of its depth (states of one depth have the same edges)
  auto taken = [&](int64_t a, int x, int y) {
    const float d = dec[(size_t)y * B.W + x];
    int k = 0;
    while (k < 3 && B.val[4 * a + k] != d) ++k;
    return k;
  };
  double e = B.un[t];
  const int64_t above = r > 0 ? at - kRows - 1 : at - ((int64_t)B.S - kRows + 1) * kRows + kRows - 1;
  if (info & kLiveUp) e += B.ed[16 * above + 4 * taken(above, X, Y - 1) + l];
  if (info & kLiveLeft) e += B.er[16 * (at - kRows) + 4 * taken(at - kRows, X - 1, Y) + l];
  e = (e + B.msg[2][t]) + B.msg[3][t];
  const float v = B.val[t];
  const int p = taken(at, X, Y);
  const double ep = __shfl(e, p, 4);
  const float vp = __shfl(v, p, 4);
  const double near = gap * fmax(scale, (double)__int_as_float(B.flag[1]));
  if (l >= n || v == vp || fabs(e - ep) > near) return;
  bool differs = state_cost(g, X, Y, l) != state_cost(g, X, Y, p);
  float w[4] = {0.f, 0.f, 0.f, 0.f};
  if (info & kLiveUp) {
    node_states(g, B.W, B.H, X, Y - 1, w);
    const float u = w[taken(above, X, Y - 1)];
    differs = differs || edge_distance(v, u) != edge_distance(vp, u);
  }
  if (info & kLiveLeft) {
    node_states(g, B.W, B.H, X - 1, Y, w);
    const float u = w[taken(at - kRows, X - 1, Y)];
    differs = differs || edge_distance(v, u) != edge_distance(vp, u);
  }
  // the last messages from the right and from below: every state there that is, or nearly is, the
  // least for either state here has to lie at the same distance from both
  for (int d = 2; d < 4 && sent; ++d) {
    const int m = node_states(g, B.W, B.H, X + (d == 2), Y + (d == 3), w);
    const int64_t a = d == 2 ? at + kRows : (r < kRows - 1 ? at + kRows + 1 : at + ((int64_t)B.S - kRows + 1) * kRows - kRows + 1);
    double to_l[4], to_p[4], least_l = __builtin_inf(), least_p = __builtin_inf();
    for (int k = 0; k < m; ++k) {
      const int64_t q = 4 * a + k;
      const double back = B.msg[d == 2 ? 1 : 0][q];
      const double sends = B.gamma[a] * ((((B.un[q] + B.msg[0][q]) + B.msg[1][q]) + B.msg[2][q]) + B.msg[3][q]) - back;
      const double* e = (d == 2 ? B.er : B.ed) + 16 * at + k;
      to_l[k] = sends + e[4 * l];
      to_p[k] = sends + e[4 * p];
      least_l = fmin(least_l, to_l[k]);
      least_p = fmin(least_p, to_p[k]);
    }
    for (int k = 0; k < m; ++k)
      if (to_l[k] <= least_l + near || to_p[k] <= least_p + near)
        differs = differs || edge_distance(v, w[k]) != edge_distance(vp, w[k]);
  }
  if (differs) atomicOr(B.flag, kTrwTie);
}

// The arguments of all logarithms of the energies, in any order: where each energy lies (in doubles
// from er) and its potential.  at null: counted only.
__global__ __launch_bounds__(256) void trw_potentials_kernel(Nodes g, TrwBuffers B, double k1, double k2, double k3,
                                                             double cost_max, unsigned long long* __restrict__ n_out,
                                                             int64_t* __restrict__ at_out, double* __restrict__ out) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, at = t >> 2;
  const int l = (int)threadIdx.x & 3;
  const int r = (int)(at % kRows);
  const int64_t bs = at / kRows;
  const int X = (int)(bs % B.S) - r, Y = (int)(bs / B.S) * kRows + r;
  double x[9];
  int64_t to[9];
  int count = 0;
  float v[4] = {0.f, 0.f, 0.f, 0.f}, w[4];
  const int n = at < B.positions ? node_states(g, B.W, B.H, X, Y, v) : 0;
  if (l < n) {
    const float mine = l == 0 ? v[0] : (l == 1 ? v[1] : (l == 2 ? v[2] : v[3]));
    if (!(g.depth[(size_t)(2 * Y) * g.W + 2 * X] > 0.0f)) {
      x[count] = (cost_max - (double)state_cost(g, X, Y, l)) / k1 + k2;
      to[count++] = B.un + t - B.er;
    }
    for (int d = 0; d < 2; ++d) {
      const int m = node_states(g, B.W, B.H, X + (d == 0), Y + (d == 1), w);
      for (int j = 0; j < m && n * m > 1; ++j) {
        x[count] = edge_potential(mine, w[j], k3);
        to[count++] = (d == 0 ? B.er : B.ed) + 4 * t + j - B.er;
      }
    }
  }
  // places in the list: a wave's entries together
  const int lane = threadIdx.x & 63;
  int before = count;
  for (int o = 1; o < 64; o <<= 1) {
    const int other = __shfl_up(before, o);
    if (lane >= o) before += other;
  }
  const int all = __shfl(before, 63);
  unsigned long long base = 0;
  if (lane == 0 && all) base = atomicAdd(n_out, (unsigned long long)all);
  base = __shfl(base, 0) + (before - count);
  if (!at_out) return;
  for (int i = 0; i < count; ++i) {
    at_out[base + i] = to[i];
    out[base + i] = x[i];
  }
}

__global__ __launch_bounds__(256) void trw_energies_kernel(double* __restrict__ er, const int64_t* __restrict__ at,
                                                           const double* __restrict__ energy, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) er[at[i]] = energy[i];
}

}  // namespace pmt

namespace phimvs_internal {

// steps of a band's walk: whole chunks
static int64_t trw_steps(int64_t W2) { return (W2 + pmt::kRows - 1 + pmt::kChunk - 1) / pmt::kChunk * pmt::kChunk; }
static int64_t trw_positions(int W2, int H2) {
  return (int64_t)((H2 + pmt::kRows - 1) / pmt::kRows) * trw_steps(W2) * pmt::kRows;
}

// The GPU's time goes with the steps that follow one another, 0.31 us each whatever they hold; the
// host's goes with the nodes, 5 (16 threads) to 20 ns (one thread) each.  At 8 iterations, GPU and
// host, with the nodes per step: 31 x 33 pixels (6) 0.36 and 0.11 ms, 60 x 1600 (21) 6.4 and 11.5,
// 128 x 64 (21) 0.54 and 0.66, 1600 x 42 (21) 4.1 and 7.9, 128 x 128 (29) 0.80 and 1.38, 320 x 240
// (45) 1.9 and 4.3, 1600 x 1066 (269) 8.9 and 58, 3200 x 2130 19.5 and 194.
// Longer walks than 2^19 steps do not fit the kernels' 32-bit offsets into a band.
bool trw_on_gpu(int W2, int H2) {
  const int64_t nb = ((int64_t)H2 + pmt::kRows - 1) / pmt::kRows;
  const int64_t steps = trw_steps(W2) + (nb - 1) * (pmt::kRows - 1 + pmt::kChunk);
  return trw_steps(W2) <= (1 << 19) && (int64_t)W2 * H2 >= 20 * steps;
}

// 64-bit words per position: er 16, ed 16, un 4, four messages of 4, val 2, gamma
// 1, info 1 (half used)
static constexpr int kWordsPerPosition = 16 + 16 + 4 + 16 + 2 + 1 + 1;

// room read before the first place of er (a step) and of ed (a band and a step)
static size_t trw_room_er() { return 16 * pmt::kRows; }
static size_t trw_room_ed(int W2) { return 16 * (size_t)(trw_steps(W2) + 1) * pmt::kRows; }

size_t trw_words(int W2, int H2) {
  const size_t nb = (size_t)(H2 + pmt::kRows - 1) / pmt::kRows;
  return (size_t)trw_positions(W2, H2) * kWordsPerPosition + trw_room_er() + trw_room_ed(W2) + nb * trw_steps(W2) * 4 + 2;
}

static TrwBuffers trw_buffers(int W, int H, uint64_t* words) {
  TrwBuffers B{};
  B.W = (W + 1) / 2;
  B.H = (H + 1) / 2;
  B.NB = (B.H + pmt::kRows - 1) / pmt::kRows;
  B.S = (int)trw_steps(B.W);
  B.positions = trw_positions(B.W, B.H);
  const size_t n = (size_t)B.positions;
  uint64_t* p = words;
  auto take = [&p](size_t k) {
    uint64_t* q = p;
    p += k;
    return q;
  };
  (void)take(trw_room_er());
  B.er = reinterpret_cast<double*>(take(16 * n));
  (void)take(trw_room_ed(B.W));
  B.ed = reinterpret_cast<double*>(take(16 * n));
  B.un = reinterpret_cast<double*>(take(4 * n));
  for (int d = 0; d < 4; ++d) B.msg[d] = reinterpret_cast<double*>(take(4 * n));
  B.val = reinterpret_cast<float*>(take(2 * n));
  B.edge = reinterpret_cast<double*>(take((size_t)B.NB * B.S * 4));
  B.ticket = reinterpret_cast<unsigned long long*>(take(1));
  B.flag = reinterpret_cast<int*>(take(1));
  B.gamma = reinterpret_cast<double*>(take(n));
  B.info = reinterpret_cast<int*>(take(n));
  return B;
}

hipError_t launch_trw(const float* depth, const float* hyp, const float* cost, int W, int H, const TrwParams& p,
                      uint64_t* words, const TrwLogs* logs, float* dec, int** flag, hipStream_t st) {
  const TrwBuffers B = trw_buffers(W, H, words);
  *flag = B.flag;
  // the flag lies after the ticket
  hipError_t e = launch_zero(reinterpret_cast<unsigned int*>(B.ticket), 4, st);
  if (e != hipSuccess) return e;
  const pmt::Nodes g{depth, hyp, cost, W, H};
  const dim3 places((unsigned)((4 * B.positions + 255) / 256));
  hipLaunchKernelGGL(pmt::trw_setup_kernel, places, dim3(256), 0, st, g, B, p.k1, p.k2, p.k3, p.cost_max);
  if (logs)
    hipLaunchKernelGGL(pmt::trw_energies_kernel, dim3((unsigned)((logs->n + 255) / 256)), dim3(256), 0, st, B.er, logs->at,
                       logs->x, logs->n);
  const dim3 grid(B.NB), block(2 * pmt::kRows);
  // a launch that failed ends it: the ones after it would take their band numbers from its share
  // of the ticket
  if ((e = hipGetLastError()) != hipSuccess) return e;
  int sweep = 0;
  for (int it = 0; it < p.iterations; ++it) {
    hipLaunchKernelGGL(pmt::trw_sweep_kernel<0>, grid, block, 0, st, B, sweep++, dec);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(pmt::trw_sweep_kernel<1>, grid, block, 0, st, B, sweep++, dec);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(pmt::trw_sweep_kernel<2>, grid, block, 0, st, B, sweep, dec);
  if ((e = hipGetLastError()) != hipSuccess || logs) return e;
  const double edge = 2.0 * std::max(std::fabs(std::log(p.k3 - 1.0)), std::log(p.k3));  // the largest of an edge
  hipLaunchKernelGGL(pmt::trw_ties_kernel, places, dim3(256), 0, st, g, B,
                     pmt::kTieGap * std::max(1.0, p.iterations / 8.0), std::max(pmt::kTieScale, edge), p.iterations > 0, dec);
  return hipGetLastError();
}

hipError_t launch_trw_potentials(const float* depth, const float* hyp, const float* cost, int W, int H, const TrwParams& p,
                                 uint64_t* words, const TrwLogs* logs, unsigned long long** n, hipStream_t st) {
  const TrwBuffers B = trw_buffers(W, H, words);
  *n = B.ticket;
  const hipError_t e = launch_zero(reinterpret_cast<unsigned int*>(B.ticket), 2, st);
  if (e != hipSuccess) return e;
  const pmt::Nodes g{depth, hyp, cost, W, H};
  hipLaunchKernelGGL(pmt::trw_potentials_kernel, dim3((unsigned)((4 * B.positions + 255) / 256)), dim3(256), 0, st, g, B, p.k1,
                     p.k2, p.k3, p.cost_max, B.ticket, logs ? logs->at : nullptr, logs ? logs->x : nullptr);
  return hipGetLastError();
}

}  // namespace phimvs_internal
