// Learned initial-plane proposal: a 5-layer 3x3 convolutional network (5 -> 32 -> 32 ->
// 32 -> 32 -> 4 channels, ReLU between layers) over a 1/4-resolution input (the
// reference and four source views warped by the fronto-parallel plane at the middle of
// the depth range).  Its output seeds the random initialisation of Sec. III-B: each
// pixel keeps the proposed plane only when its matching cost is not higher than the
// random plane's (the gate lives in the initialisation kernel).
//
// Numerics: weights and activations are bfloat16, every convolution accumulates in FP32
// on the matrix cores.  Activations are NHWC with the channel count padded to 16 or 32.  A
// convolution is an implicit GEMM over K = 9 taps x input channels; one wave walks down a
// strip of 16 columns with the layer's weights in registers, so that an input row is read
// once for the three output rows it enters.  Training runs on the same kernel: the data
// gradient is the forward convolution with flipped, transposed weights; the weight
// gradient accumulates (input patch)^T x (output gradient) over strips of 32 columns,
// summed over the waves of a workgroup and then over the workgroups in a fixed order.

#include <hip/hip_runtime.h>
#include <hip/hip_bfloat16.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "phimvs_net_internal.h"

namespace pmn {

using namespace phimvs_net_internal;

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f2bf(float f) {
  // round to nearest even (NaN not expected)
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
// two of them in one dword; the hardware's conversion rounds the same way (checked on every
// float that is not NaN)
typedef __bf16 v2b __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f{lo, hi}), v2b));
}
__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// ---------------------------------------------------------------------------- convolution
// y[b, r, c, co] = bias[co] + sum_{t, ci} x[b, r + dy_t, c + dx_t, ci] * w[t][co][ci]
// (zero outside the image), optionally ReLU; x: bf16 NHWC with CI channels; w: bf16
// [9][CO][CI].  Output: bf16 (y16, CO channels) and / or fp32 (y32, the first 4 channels).
// If mask16 is given the result is multiplied by (mask16 > 0) (ReLU backward of the
// producing layer) before storing.  FIRST: the input is the network's own, fp32 with 5
// channels (x32), rounded to bf16 here and stored as the layer's 16-channel bf16 input.
//
// Memory bounds the layer (54 MB at 800 x 533 x 32 channels: 11 us at the 5.0 TB/s of a
// large copy; the matrix work is 3 us), so the work is split to read each row once: a wave
// takes 16 columns x `rb` rows, holds all 9 x CI x CO weights in registers (72 VGPRs for
// 32 x 32) and keeps three output rows in flight; a row's three shifted fragments feed all
// of them (the columns beside a lane's own come from its neighbours), and two rows are in
// flight beyond the one in use.  The weights
// are the A operand, rows permuted, so that a lane ends with consecutive channels of one pixel
// (one 16-byte store for 32 channels).  The order of every accumulation is taps, then input channels: 16x16x32 equals
// two chained 16x16x16 over the lower and the upper 16 channels, bit for bit.
// 800 x 533, 32 -> 32 channels: 47 us with a wave per 16 pixels of one row (each pixel read
// for all nine taps, weights from LDS), 18 us so (3.0 TB/s; 21 us with three overlapping loads a
// row and one row in flight); 8 x 267 x 400: 91 -> 29 us (3.8 TB/s).
typedef __bf16 v8b __attribute__((ext_vector_type(8)));
template <int CI>
struct Frag;  // one lane's share of 16 columns (or output channels) x CI input channels
template <>
struct Frag<16> {
  uint2 v;
};
template <>
struct Frag<32> {
  uint4 v;
};
__device__ __forceinline__ v4f mfma(const Frag<16>& a, const Frag<16>& b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(v4s, a.v), __builtin_bit_cast(v4s, b.v), c, 0, 0,
                                                   0);
}
__device__ __forceinline__ v4f mfma(const Frag<32>& a, const Frag<32>& b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8b, a.v), __builtin_bit_cast(v8b, b.v), c, 0, 0, 0);
}

// src of the lane before (0x111) or after (0x101) within 16 lanes; `edge` at the end lane
template <int CTRL>
__device__ __forceinline__ uint32_t shift1(uint32_t edge, uint32_t src) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)edge, (int)src, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ __forceinline__ uint2 shift(uint2 e, uint2 s) {
  return make_uint2(shift1<CTRL>(e.x, s.x), shift1<CTRL>(e.y, s.y));
}
template <int CTRL>
__device__ __forceinline__ uint4 shift(uint4 e, uint4 s) {
  return make_uint4(shift1<CTRL>(e.x, s.x), shift1<CTRL>(e.y, s.y), shift1<CTRL>(e.z, s.z), shift1<CTRL>(e.w, s.w));
}

typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kConvBlock = 256;  // 4 waves on neighbouring strips
template <int CI, int CO, bool FIRST>
__global__ __launch_bounds__(kConvBlock) __attribute__((amdgpu_waves_per_eu(3))) void conv3x3_kernel(ConvArgs a, int rb, int segs, int bands) {
  constexpr int NCO = CO / 16, KL = CI / 4;  // output blocks; input channels of one lane
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int task = blockIdx.x * (kConvBlock / 64) + wave;  // (b, band, seg)
  if (task >= a.B * bands * segs) return;
  const int seg = task % segs;
  const int bb = task / segs;
  const int band = bb % bands, b = bb / bands;
  const int r0 = band * rb, r1 = min(r0 + rb, a.h);
  const int lr = lane & 15, lk = lane >> 4;
  const int c = seg * 16 + lr;  // this lane's column
  Frag<CI> W[9][NCO];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int i = 0; i < NCO; ++i)
      W[t][i].v = *reinterpret_cast<const decltype(W[t][i].v)*>(
          a.wt + (size_t)(t * CO + (lr >> 2) * 4 * NCO + i * 4 + (lr & 3)) * CI + lk * KL);
  float bias[NCO][4];
#pragma unroll
  for (int i = 0; i < NCO; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int co = lk * 4 * NCO + i * 4 + j;
      bias[i][j] = (a.bias && co < a.n_bias) ? a.bias[co] : 0.f;
    }
  // A row is loaded once: each lane its own column, and the lanes at the strip's ends the
  // column beside it; the shifted fragments come from the neighbouring lanes.
  const bool mine = c < a.w;
  const int ch = lr == 0 ? c - 1 : c + 1;
  const bool edge = (lr == 0 || lr == 15) && ch >= 0 && ch < a.w;
  // FIRST: lanes of the first K group hold channels 0..3, the second's channel 4 (the last of
  // the four it loads), the rest 0; 16-byte loads at 4-byte alignment, rounded when used
  typedef std::conditional_t<FIRST, f4u, decltype(Frag<CI>::v)> Raw;
  struct Row {
    Raw own, halo;
  };
  auto load_px = [&](int i, int col, bool ok, Raw& f) {
    f = Raw{};
    if (!ok) return;
    const size_t pix = ((size_t)b * a.h + i) * a.w + col;
    if constexpr (FIRST) {
      if (lk < 2) f = *reinterpret_cast<const f4u*>(a.x32 + pix * 5 + lk);
    } else {
      f = *reinterpret_cast<const Raw*>(a.x + pix * CI + lk * KL);
    }
  };
  auto rounded = [&](const Raw& f) {
    if constexpr (FIRST)
      return make_uint2(lk == 0 ? pack_bf(f[0], f[1]) : pack_bf(f[3], 0.f), lk == 0 ? pack_bf(f[2], f[3]) : 0u);
    else
      return f;
  };
  auto load_row = [&](int i, Row& r) {
    const bool rin = i >= 0 && i < a.h;
    load_px(i, c, rin && mine, r.own);
    load_px(i, ch, rin && edge, r.halo);
  };
  Row R0, R1, R2;
  load_row(r0 - 1, R0);
  load_row(r0, R1);
  v4f a0[NCO], a1[NCO], a2[NCO];  // output rows i + 1, i, i - 1 of the row being read
#pragma unroll
  for (int i = 0; i < NCO; ++i) a1[i] = a2[i] = v4f{0.f, 0.f, 0.f, 0.f};
  for (int i = r0 - 1; i <= r1; ++i) {
    const bool store = i - 1 >= r0 && c < a.w;
    const size_t p = ((size_t)b * a.h + (store ? i - 1 : 0)) * a.w + (store ? c : 0);
    Frag<CO> m;  // the mask at this lane's pixel and output channels
    m.v = decltype(m.v){};
    if (a.mask16 && store) m.v = *reinterpret_cast<const decltype(m.v)*>(a.mask16 + p * CO + lk * 4 * NCO);
    if (i + 2 <= r1) load_row(i + 2, R2);
    Frag<CI> F[3];  // columns c - 1, c, c + 1
    F[1].v = rounded(R0.own);
    F[0].v = shift<0x111>(rounded(R0.halo), F[1].v);
    F[2].v = shift<0x101>(rounded(R0.halo), F[1].v);
    if constexpr (FIRST) {
      if (i >= r0 && i < r1 && c < a.w)
        *reinterpret_cast<uint2*>(a.x16 + (((size_t)b * a.h + i) * a.w + c) * 16 + lk * 4) = F[1].v;
    }
#pragma unroll
    for (int k = 0; k < NCO; ++k) {
      a0[k] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        a0[k] = mfma(W[d][k], F[d], a0[k]);
        a1[k] = mfma(W[3 + d][k], F[d], a1[k]);
        a2[k] = mfma(W[6 + d][k], F[d], a2[k]);
      }
    }
    if (store) {
      // a2[k][j]: pixel (i - 1, c), output channel 4 NCO lk + 4 k + j
      uint32_t mw[2 * NCO], o[2 * NCO];
      __builtin_memcpy(mw, &m, sizeof mw);
#pragma unroll
      for (int k = 0; k < NCO; ++k) {
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          v[j] = a2[k][j] + bias[k][j];
          if (a.relu) v[j] = fmaxf(v[j], 0.f);
          if (a.mask16 && !(bf2f((uint16_t)(mw[2 * k + j / 2] >> (j & 1 ? 16 : 0))) > 0.f)) v[j] = 0.f;
        }
        o[2 * k] = pack_bf(v[0], v[1]);
        o[2 * k + 1] = pack_bf(v[2], v[3]);
        if (a.y32 && k == 0 && lk == 0) {
          if (a.y32_aligned) {
            *reinterpret_cast<float4*>(a.y32 + p * 4) = make_float4(v[0], v[1], v[2], v[3]);
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) a.y32[p * 4 + j] = v[j];
          }
        }
      }
      if (a.y16) {
        Frag<CO> y;
        __builtin_memcpy(&y, o, sizeof o);
        *reinterpret_cast<decltype(y.v)*>(a.y16 + p * CO + lk * 4 * NCO) = y.v;
      }
    }
#pragma unroll
    for (int k = 0; k < NCO; ++k) {
      a2[k] = a1[k];
      a1[k] = a0[k];
    }
    R0 = R1;
    R1 = R2;
  }
}

// Weight gradient partials: dW[t][ci][co] = sum_{b, r, c} x[b, r + dy, c + dx, ci] * g[b, r, c, co]
// and the bias gradient's sums of g.  One wave takes a strip of 32 columns x rb rows and all
// 9 x CI x CO sums (144 accumulator registers for 32 x 32); walking down, each input row meets
// the gradients of the three rows it enters.  The contraction runs over columns, which NHWC
// scatters, so a wave stages each row (34 input and 32 gradient pixels, 16-byte loads, the
// next row's in flight) in its own part of LDS and reads it back through the transposing LDS
// read: lane lr of 16 gets channel lr of 4 columns.  The waves of a workgroup add their sums in
// LDS in wave order; workgroup k's go to partial + k * stride ([9][CI][CO], then [CO] bias sums).
// 8 x 267 x 400, 32 x 32 channels: 176 us with a workgroup per image row (2136 partial sums of
// 36 KB to write and reduce, another 14 us); 81 us with these strips and dwords of two channels
// gathered and paired up per lane; 56 us through the transposing read; 28 us (234 partial sums)
// with the waves' sums added by the whole workgroup instead of by one wave after the other.
constexpr int kWgBlock = 512;
typedef __attribute__((address_space(3))) v4s* LdsV4s;
// columns 8 lk + p0 .. + 7 of channels ch0 + lr from a staged row of C channels per pixel
template <int C>
__device__ __forceinline__ Frag<32> read_columns(const uint16_t* row, int p0, int ch0, int lr, int lk) {
  const uint16_t* at = row + (8 * lk + p0 + lr / 4) * C + ch0 + 4 * (lr & 3);
  const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsV4s)at);
  const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsV4s)(at + 4 * C));
  Frag<32> f;
  __builtin_memcpy(&f.v.x, &lo, 8);
  __builtin_memcpy(&f.v.z, &hi, 8);
  return f;
}
template <int CI, int CO>
__global__ __launch_bounds__(kWgBlock) void conv3x3_wgrad_kernel(WgradArgs a, int rb, int segs, int bands) {
  constexpr int NCI = CI / 16, NCO = CO / 16, kSums = 9 * CI * CO;
  // 16-byte chunks of a staged row: the input's 34 pixels, the gradient's 32; per lane
  constexpr int kXc = 34 * CI / 8, kGc = 32 * CO / 8, kXl = (kXc + 63) / 64, kGl = kGc / 64;
  // a wave's staged rows; after the last row, the sums of three taps of every wave
  constexpr int kWaves = kWgBlock / 64, kRegs = 3 * NCI * NCO * 4;
  constexpr int kStageBytes = kWaves * (kXc + kGc) * 16, kRedBytes = kWaves * (kRegs + NCO) * 64 * 4;
  __shared__ uint4 lds[(kStageBytes > kRedBytes ? kStageBytes : kRedBytes) / 16];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int lr = lane & 15, lk = lane >> 4;
  uint4* xs = lds + wave * (kXc + kGc);
  uint4* gs = xs + kXc;
  v4f acc[9][NCI][NCO], accb[NCO];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int u = 0; u < NCI; ++u)
#pragma unroll
      for (int v = 0; v < NCO; ++v) acc[t][u][v] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int v = 0; v < NCO; ++v) accb[v] = v4f{0.f, 0.f, 0.f, 0.f};
  Frag<32> ones;
  ones.v = make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u);
  // (b, band, seg): one for a wave, more where there are more strips than waves
  const int tasks = a.B * bands * segs;
  for (int task = blockIdx.x * (kWgBlock / 64) + wave; task < tasks; task += gridDim.x * (kWgBlock / 64)) {
    const int seg = task % segs;
    const int bb = task / segs;
    const int band = bb % bands, b = bb / bands;
    const int r0 = band * rb, r1 = min(r0 + rb, a.h);
    // this lane's chunks of a row: element offset from the strip's first column (a row can hold more
    // than 2^31 elements), and whether the column exists
    int xo[kXl], go[kGl];
    bool xi[kXl], gi[kGl];
#pragma unroll
    for (int k = 0; k < kXl; ++k) {
      const int q = lane + 64 * k, c = q / (CI / 8) - 1;
      xi[k] = q < kXc && seg * 32 + c >= 0 && seg * 32 + c < a.w;
      xo[k] = xi[k] ? c * CI + (q % (CI / 8)) * 8 : 0;
    }
#pragma unroll
    for (int k = 0; k < kGl; ++k) {
      const int q = lane + 64 * k, c = q / (CO / 8);
      gi[k] = seg * 32 + c < a.w;
      go[k] = gi[k] ? c * CO + (q % (CO / 8)) * 8 : 0;
    }
    uint4 xr[kXl], gr[kGl];
    // input row i and gradient row i + 1 (zero outside the image, and outside the band)
    auto load_rows = [&](int i) {
      const bool xin = i >= 0 && i < a.h, gin = i + 1 >= r0 && i + 1 < r1;
      const uint16_t* xp = a.x + (((size_t)b * a.h + (xin ? i : 0)) * a.w + seg * 32) * CI;
      const uint16_t* gp = a.g + (((size_t)b * a.h + (gin ? i + 1 : 0)) * a.w + seg * 32) * CO;
#pragma unroll
      for (int k = 0; k < kXl; ++k) {
        xr[k] = make_uint4(0u, 0u, 0u, 0u);
        if (xin && xi[k]) xr[k] = *reinterpret_cast<const uint4*>(xp + xo[k]);
      }
#pragma unroll
      for (int k = 0; k < kGl; ++k) {
        gr[k] = make_uint4(0u, 0u, 0u, 0u);
        if (gin && gi[k]) gr[k] = *reinterpret_cast<const uint4*>(gp + go[k]);
      }
    };
    Frag<32> g0[NCO], g1[NCO], g2[NCO];  // gradient rows i + 1, i, i - 1
#pragma unroll
    for (int v = 0; v < NCO; ++v) g1[v].v = g2[v].v = make_uint4(0u, 0u, 0u, 0u);
    load_rows(r0 - 1);
    for (int i = r0 - 1; i <= r1; ++i) {
      // the staged row is this wave's own: its LDS operations stay in order
#pragma unroll
      for (int k = 0; k < kXl; ++k)
        if (lane + 64 * k < kXc) xs[lane + 64 * k] = xr[k];
#pragma unroll
      for (int k = 0; k < kGl; ++k) gs[lane + 64 * k] = gr[k];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (i < r1) load_rows(i + 1);
      Frag<32> X[3][NCI];
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int u = 0; u < NCI; ++u)
          X[d][u] = read_columns<CI>(reinterpret_cast<const uint16_t*>(xs), d, 16 * u, lr, lk);
#pragma unroll
      for (int v = 0; v < NCO; ++v)
        g0[v] = read_columns<CO>(reinterpret_cast<const uint16_t*>(gs), 0, 16 * v, lr, lk);
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int v = 0; v < NCO; ++v) {
        accb[v] = mfma(ones, g0[v], accb[v]);
#pragma unroll
        for (int u = 0; u < NCI; ++u)
#pragma unroll
          for (int d = 0; d < 3; ++d) {
            acc[d][u][v] = mfma(X[d][u], g0[v], acc[d][u][v]);
            acc[3 + d][u][v] = mfma(X[d][u], g1[v], acc[3 + d][u][v]);
            acc[6 + d][u][v] = mfma(X[d][u], g2[v], acc[6 + d][u][v]);
          }
        g2[v] = g1[v];
        g1[v] = g0[v];
      }
    }
  }
  // The waves' sums, three taps at a time: every wave lays its registers out lane by lane, then
  // the workgroup adds them in wave order.  Register ((t, u, v), j) of lane (lr, lk) is the sum of
  // tap t, ci = 16 u + 4 lk + j, co = 16 v + lr; accb[v] of a lane with lk = 0 the bias's co.
  float* red = reinterpret_cast<float*>(lds);
  float* P = a.partial + (size_t)blockIdx.x * (kSums + CO);
#pragma unroll
  for (int ty = 0; ty < 3; ++ty) {
    __syncthreads();
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int u = 0; u < NCI; ++u)
#pragma unroll
        for (int v = 0; v < NCO; ++v)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            red[(wave * (kRegs + NCO) + ((d * NCI + u) * NCO + v) * 4 + j) * 64 + lane] = acc[3 * ty + d][u][v][j];
#pragma unroll
    for (int v = 0; v < NCO; ++v) red[(wave * (kRegs + NCO) + kRegs + v) * 64 + lane] = accb[v][0];
    __syncthreads();
    for (int i = threadIdx.x; i < (kRegs + (ty == 0 ? NCO : 0)) * 64; i += kWgBlock) {
      float s = red[i];
      for (int w = 1; w < kWaves; ++w) s = s + red[w * (kRegs + NCO) * 64 + i];
      const int reg = i >> 6, l15 = i & 15, l4 = (i >> 4) & 3;
      if (reg >= kRegs) {
        if (l4 == 0) P[kSums + 16 * (reg - kRegs) + l15] = s;
        continue;
      }
      const int j = reg & 3, v = (reg >> 2) % NCO, u = (reg >> 2) / NCO % NCI, d = (reg >> 2) / (NCO * NCI);
      P[((3 * ty + d) * CI + 16 * u + 4 * l4 + j) * CO + 16 * v + l15] = s;
    }
  }
}

// The gradient of every layer from its workgroups' partial sums, in a fixed order: a
// workgroup of 16 waves takes 64 parameters of one layer, wave g sums the partials g, g + 16,
// g + 32, ... in turn, and the 16 sums are added in wave order, so the result does not depend
// on scheduling.  Parameter i of a layer: weight [t][ci][co] of the unpadded shape, then bias.
constexpr int kReduceGroups = 16;
__global__ __launch_bounds__(kReduceGroups * 64) void reduce_grads_kernel(ReduceArgs a) {
  __shared__ float part[kReduceGroups][64];
  const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
  int l = 0;
  while (l + 1 < a.n_layers && (int)blockIdx.x >= a.layer[l + 1].block0) ++l;
  const ReduceLayer& L = a.layer[l];
  const int i = ((int)blockIdx.x - L.block0) * 64 + lane;
  const int nw = 9 * L.cin * L.cout;
  const bool use = i < nw + L.cout;
  int e = 9 * L.CI * L.CO + (i - nw);
  if (i < nw) {
    const int t = i / (L.cin * L.cout);
    const int rem = i - t * L.cin * L.cout;
    const int ci = rem / L.cout;
    e = (t * L.CI + ci) * L.CO + (rem - ci * L.cout);
  }
  const int stride = (9 * L.CI + 1) * L.CO;
  float s = 0.f;
  if (use) {
#pragma unroll 4
    for (int k = g; k < L.n_partial; k += kReduceGroups) s += L.partial[(size_t)k * stride + e];
  }
  part[g][lane] = s;
  __syncthreads();
  if (g == 0 && use) {
    float t = 0.f;
    for (int q = 0; q < kReduceGroups; ++q) t += part[q][lane];
    L.grad[i] = t;
  }
}

// bf16 NHWC with CP channels -> fp32 NHWC with the first C
__global__ void bf16_unpad_kernel(const uint16_t* __restrict__ x, int n_pix, int CP, int C, float* __restrict__ y) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)n_pix * C) return;
  const size_t p = i / C, c = i - p * C;
  y[i] = bf2f(x[p * CP + c]);
}

// master fp32 weights [9][CIN][COUT] -> bf16 forward [9][COP][CIP] and flipped [9][CIP][COP]
__global__ void pack_weights_kernel(const float* __restrict__ w, int CIN, int COUT, int CIP, int COP,
                                    uint16_t* __restrict__ fwd, uint16_t* __restrict__ flip) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= 9 * CIP * COP) return;
  const int t = i / (CIP * COP);
  const int rem = i - t * CIP * COP;
  const int co = rem / CIP, ci = rem - co * CIP;
  const float v = (ci < CIN && co < COUT) ? w[((size_t)t * CIN + ci) * COUT + co] : 0.f;
  fwd[((size_t)t * COP + co) * CIP + ci] = f2bf(v);
  // data gradient: g_in[ci] = sum_{t, co} g[p - off_t][co] w[t][ci][co] = conv with w'[8 - t][ci][co]
  flip[((size_t)(8 - t) * CIP + ci) * COP + co] = f2bf(v);
}

// ---------------------------------------------------------------------------- loss
// out: B*h*w*4 fp32 (o0: depth logit, o1..o3: normal); target: B*h*w*4 (depth, normal);
// mask: B*h*w; drange: B*2.  Per pixel: depth = lo + (hi - lo) sigmoid(o0), n = o / |o|;
// loss = m (|log depth - log depth_t| + lambda (1 - n . n_t)) / sum(mask).
// Writes the output gradient (bf16, 16 channels) and per-block loss partials.
__global__ void loss_kernel(LossArgs a) {
  __shared__ float red[256];
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  float l = 0.f;
  if (i < a.n_pix) {
    const int b = i / (a.h * a.w);
    const float lo = a.drange[2 * b], hi = a.drange[2 * b + 1];
    const float* o = a.out + (size_t)i * 4;
    const float* tg = a.target + (size_t)i * 4;
    const float m = a.mask[i] * a.inv_count;
    float g[4] = {0.f, 0.f, 0.f, 0.f};
    if (m > 0.f) {
      const float s = 1.f / (1.f + expf(-o[0]));
      const float d = lo + (hi - lo) * s;
      const float diff = logf(d) - logf(tg[0]);
      const float nrm = sqrtf(o[1] * o[1] + o[2] * o[2] + o[3] * o[3]) + 1e-6f;
      const float nx = o[1] / nrm, ny = o[2] / nrm, nz = o[3] / nrm;
      const float dotp = nx * tg[1] + ny * tg[2] + nz * tg[3];
      l = m * (fabsf(diff) + a.lambda * (1.f - dotp));
      const float sg = diff > 0.f ? 1.f : (diff < 0.f ? -1.f : 0.f);
      g[0] = m * sg * (hi - lo) * s * (1.f - s) / d;
      const float k = -m * a.lambda / nrm;
      g[1] = k * (tg[1] - dotp * nx);
      g[2] = k * (tg[2] - dotp * ny);
      g[3] = k * (tg[3] - dotp * nz);
    }
    uint4* o16 = reinterpret_cast<uint4*>(a.grad16 + (size_t)i * 16);
    o16[0] = make_uint4(pack_bf(g[0], g[1]), pack_bf(g[2], g[3]), 0u, 0u);
    o16[1] = make_uint4(0u, 0u, 0u, 0u);
  }
  red[threadIdx.x] = l;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) a.loss_partial[blockIdx.x] = red[0];
}

// Adam on the fp32 master weights, and the bf16 copies of the weights it changes (their
// padding is zero since pack_weights_kernel and stays so)
__global__ void adam_kernel(AdamArgs a) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const float gi = a.g[i];
  const float mi = a.b1 * a.m[i] + (1.f - a.b1) * gi;
  const float vi = a.b2 * a.v[i] + (1.f - a.b2) * gi * gi;
  a.m[i] = mi;
  a.v[i] = vi;
  const float w = a.w[i] - a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
  a.w[i] = w;
  int l = 0;
  while (l + 1 < a.n_layers && i >= a.layer[l + 1].first) ++l;
  const PackLayer& L = a.layer[l];
  const int k = i - L.first;
  if (k >= 9 * L.cin * L.cout) return;  // a bias
  const int t = k / (L.cin * L.cout);
  const int rem = k - t * L.cin * L.cout;
  const int ci = rem / L.cout, co = rem - ci * L.cout;
  L.fwd[((size_t)t * L.CO + co) * L.CI + ci] = f2bf(w);
  L.flip[((size_t)(8 - t) * L.CI + ci) * L.CO + co] = f2bf(w);
}

// ---------------------------------------------------------------------------- proposal
// 1/4-resolution network input for reference pixel block (X, Y): channel 0 = mean of the
// 4x4 reference block, channels 1..4 = source k sampled (bilinear) at the image of the block
// centre under H_k (fronto-parallel plane at the middle of the depth range); 0 outside the
// source.  Values are (I - 127.5) / 64.
__global__ void proposal_inputs_kernel(ProposalInputs a) {
  const int X = blockIdx.x * blockDim.x + threadIdx.x, Y = blockIdx.y;
  if (X >= a.w || Y >= a.h) return;
  float s = 0.f;
  for (int dy = 0; dy < 4; ++dy)
    for (int dx = 0; dx < 4; ++dx) {
      const int x = min(4 * X + dx, a.W - 1), y = min(4 * Y + dy, a.H - 1);
      s += __half2float(a.ref[(size_t)y * a.W + x]);
    }
  float* o = a.out + ((size_t)Y * a.w + X) * 5;
  o[0] = (s / 16.f - 127.5f) / 64.f;
  const float px = 4.f * X + 1.5f, py = 4.f * Y + 1.5f;
  for (int k = 0; k < 4; ++k) {
    const float* Hm = a.Hmid + 9 * k;
    const float u = Hm[0] * px + Hm[1] * py + Hm[2];
    const float v = Hm[3] * px + Hm[4] * py + Hm[5];
    const float w = Hm[6] * px + Hm[7] * py + Hm[8];
    float val = 0.f;
    if (a.quad[k] && w > 0.f) {
      const float up = u / w, vp = v / w;
      if (up >= 0.f && vp >= 0.f && up <= (float)(a.sw[k] - 1) && vp <= (float)(a.sh[k] - 1)) {
        const int x0 = (int)up, y0 = (int)vp;
        const float fx = up - x0, fy = vp - y0;
        const uint32_t q = a.quad[k][(size_t)y0 * a.sw[k] + x0];
        const float t00 = (float)(q & 0xFF), t01 = (float)((q >> 8) & 0xFF);
        const float t10 = (float)((q >> 16) & 0xFF), t11 = (float)(q >> 24);
        const float top = t00 + fx * (t01 - t00), bot = t10 + fx * (t11 - t10);
        val = ((top + fy * (bot - top)) - 127.5f) / 64.f;
      }
    }
    o[1 + k] = val;
  }
}

// full-resolution planes from the 1/4-resolution network output: bilinear upsampling of the
// four raw outputs, depth = lo + (hi - lo) sigmoid(o0), normal = o / |o| turned to face the camera
__global__ void proposal_decode_kernel(ProposalDecode a) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x, y = blockIdx.y;
  if (x >= a.W || y >= a.H) return;
  const float X = fminf(fmaxf(((float)x - 1.5f) * 0.25f, 0.f), (float)(a.w - 1));
  const float Y = fminf(fmaxf(((float)y - 1.5f) * 0.25f, 0.f), (float)(a.h - 1));
  const int x0 = (int)X, y0 = (int)Y;
  const int x1 = min(x0 + 1, a.w - 1), y1 = min(y0 + 1, a.h - 1);
  const float fx = X - x0, fy = Y - y0;
  float o[4];
  for (int c = 0; c < 4; ++c) {
    const float v00 = a.net_out[((size_t)y0 * a.w + x0) * 4 + c], v01 = a.net_out[((size_t)y0 * a.w + x1) * 4 + c];
    const float v10 = a.net_out[((size_t)y1 * a.w + x0) * 4 + c], v11 = a.net_out[((size_t)y1 * a.w + x1) * 4 + c];
    const float top = v00 + fx * (v01 - v00), bot = v10 + fx * (v11 - v10);
    o[c] = top + fy * (bot - top);
  }
  const float d = a.d_lo + (a.d_hi - a.d_lo) / (1.f + expf(-o[0]));
  float nx = o[1], ny = o[2], nz = o[3];
  const float nrm = sqrtf(nx * nx + ny * ny + nz * nz);
  if (nrm > 1e-6f) {
    nx /= nrm;
    ny /= nrm;
    nz /= nrm;
  } else {
    nx = 0.f;
    ny = 0.f;
    nz = -1.f;
  }
  const float rx = a.Kinv[0] * x + a.Kinv[1] * y + a.Kinv[2];
  const float ry = a.Kinv[3] * x + a.Kinv[4] * y + a.Kinv[5];
  const float rz = a.Kinv[6] * x + a.Kinv[7] * y + a.Kinv[8];
  if (nx * rx + ny * ry + nz * rz > 0.f) {
    nx = -nx;
    ny = -ny;
    nz = -nz;
  }
  float* p = a.planes + ((size_t)y * a.W + x) * 4;
  p[0] = nx;
  p[1] = ny;
  p[2] = nz;
  p[3] = d;
}

// training targets at network resolution from a full-resolution plain PatchMatch result:
// block (X, Y) looks at the 2x2 full-resolution pixels around its centre (4X + 1.5, 4Y + 1.5);
// it is kept (mask 1) when all four are valid with cost below max_cost, with the mean depth
// and the normalised mean normal as target
__global__ void targets_kernel(TargetArgs a) {
  const int X = blockIdx.x * blockDim.x + threadIdx.x, Y = blockIdx.y;
  if (X >= a.w || Y >= a.h) return;
  float d = 0.f, nx = 0.f, ny = 0.f, nz = 0.f;
  bool ok = true;
  for (int dy = 1; dy <= 2; ++dy)
    for (int dx = 1; dx <= 2; ++dx) {
      const int x = min(4 * X + dx, a.W - 1), y = min(4 * Y + dy, a.H - 1);
      const size_t p = (size_t)y * a.W + x;
      const float c = a.cost[p], dd = a.depth[p];
      ok = ok && dd > 0.f && c < a.max_cost;
      d += dd;
      nx += a.normal[3 * p];
      ny += a.normal[3 * p + 1];
      nz += a.normal[3 * p + 2];
    }
  const float nrm = sqrtf(nx * nx + ny * ny + nz * nz);
  ok = ok && nrm > 1e-6f;
  float* t = a.target + ((size_t)Y * a.w + X) * 4;
  t[0] = ok ? 0.25f * d : 1.f;
  t[1] = ok ? nx / nrm : 0.f;
  t[2] = ok ? ny / nrm : 0.f;
  t[3] = ok ? nz / nrm : -1.f;
  a.mask[(size_t)Y * a.w + X] = ok ? 1.f : 0.f;
}

}  // namespace pmn

namespace phimvs_net_internal {

namespace {
// rows a wave walks so that `units` strip rows make at most `waves` waves (and at least one
// row each): enough waves to fill the chip once, as long as there are rows for them
int band_rows(int64_t strips, int h, int64_t waves) {
  int rb = (int)std::max<int64_t>(1, (strips * h + waves - 1) / waves);
  while (rb < h && strips * ((h + rb - 1) / rb) > waves) ++rb;
  return std::min(rb, h);
}

template <int CI, int CO, bool FIRST>
hipError_t conv_launch(const ConvArgs& a, hipStream_t st) {
  const int segs = (a.w + 15) / 16;
  // 3 waves per SIMD by registers
  const int rb = band_rows((int64_t)a.B * segs, a.h, 3072);
  const int bands = (a.h + rb - 1) / rb;
  const int64_t tasks = (int64_t)a.B * bands * segs;
  constexpr int wpb = pmn::kConvBlock / 64;
  hipLaunchKernelGGL((pmn::conv3x3_kernel<CI, CO, FIRST>), dim3((unsigned)((tasks + wpb - 1) / wpb)),
                     dim3(pmn::kConvBlock), 0, st, a, rb, segs, bands);
  return hipGetLastError();
}

template <int CI, int CO>
hipError_t wgrad_launch(const WgradArgs& a, int n_partial, hipStream_t st) {
  int rb, segs, bands;
  if (wgrad_partials(a.B, a.h, a.w, &rb, &segs, &bands) != n_partial) return hipErrorInvalidValue;
  hipLaunchKernelGGL((pmn::conv3x3_wgrad_kernel<CI, CO>), dim3(n_partial), dim3(pmn::kWgBlock), 0, st, a, rb, segs,
                     bands);
  return hipGetLastError();
}
}  // namespace

int wgrad_partials(int B, int h, int w, int* rb, int* segs, int* bands) {
  *segs = (w + 31) / 32;
  constexpr int waves = 2048, per_wg = pmn::kWgBlock / 64;  // 2 waves per SIMD by registers
  *rb = band_rows((int64_t)B * *segs, h, waves);
  *bands = (h + *rb - 1) / *rb;
  // more strips than waves are walked by these, so that the partial sums (148 KB for all layers of
  // one) do not grow with the images
  return (int)((std::min<int64_t>((int64_t)B * *bands * *segs, waves) + per_wg - 1) / per_wg);
}

hipError_t launch_conv(const ConvArgs& a, hipStream_t st) {
  if (a.x32) return a.CI == 16 && a.CO == 32 ? conv_launch<16, 32, true>(a, st) : hipErrorInvalidValue;
  if (a.CI == 32 && a.CO == 32) return conv_launch<32, 32, false>(a, st);
  if (a.CI == 32 && a.CO == 16) return conv_launch<32, 16, false>(a, st);
  if (a.CI == 16 && a.CO == 32) return conv_launch<16, 32, false>(a, st);
  return hipErrorInvalidValue;
}

hipError_t launch_wgrad(const WgradArgs& a, int n_partial, hipStream_t st) {
  if (a.CI == 32 && a.CO == 32) return wgrad_launch<32, 32>(a, n_partial, st);
  if (a.CI == 32 && a.CO == 16) return wgrad_launch<32, 16>(a, n_partial, st);
  if (a.CI == 16 && a.CO == 32) return wgrad_launch<16, 32>(a, n_partial, st);
  return hipErrorInvalidValue;
}

hipError_t launch_bf16_unpad(const uint16_t* x, int n_pix, int CP, int C, float* y, hipStream_t st) {
  const size_t n = (size_t)n_pix * C;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(pmn::bf16_unpad_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, x, n_pix, CP, C, y);
  return hipGetLastError();
}

hipError_t launch_reduce_grads(const ReduceArgs& a, int n_blocks, hipStream_t st) {
  hipLaunchKernelGGL(pmn::reduce_grads_kernel, dim3(n_blocks), dim3(pmn::kReduceGroups * 64), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_pack_weights(const float* w, int CIN, int COUT, int CIP, int COP, uint16_t* fwd, uint16_t* flip,
                               hipStream_t st) {
  const int n = 9 * CIP * COP;
  hipLaunchKernelGGL(pmn::pack_weights_kernel, dim3((n + 255) / 256), dim3(256), 0, st, w, CIN, COUT, CIP, COP, fwd, flip);
  return hipGetLastError();
}

hipError_t launch_loss(const LossArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(pmn::loss_kernel, dim3((a.n_pix + 255) / 256), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_adam(const AdamArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(pmn::adam_kernel, dim3((a.n + 255) / 256), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_proposal_inputs(const ProposalInputs& a, hipStream_t st) {
  hipLaunchKernelGGL(pmn::proposal_inputs_kernel, dim3((a.w + 127) / 128, a.h), dim3(128), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_proposal_decode(const ProposalDecode& a, hipStream_t st) {
  hipLaunchKernelGGL(pmn::proposal_decode_kernel, dim3((a.W + 255) / 256, a.H), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_targets(const TargetArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(pmn::targets_kernel, dim3((a.w + 127) / 128, a.h), dim3(128), 0, st, a);
  return hipGetLastError();
}

}  // namespace phimvs_net_internal
