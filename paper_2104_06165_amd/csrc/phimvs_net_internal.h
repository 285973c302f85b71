// Kernel-argument blocks and launchers of the learned-proposal network (not part of the
// public C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

namespace phimvs_net_internal {

constexpr int kMaxLayers = 8;

// one 3x3 convolution (zero padding), NHWC bf16 activations
struct ConvArgs {
  int B, h, w;               // images, rows, columns
  int CI, CO;                // input / output channels (16 or 32)
  const uint16_t* x;         // B*h*w*CI bf16 (null: x32)
  const float* x32;          // or the network's input, B*h*w*5 fp32 (CI 16)
  uint16_t* x16;             // with x32: receives it as B*h*w*16 bf16, zero padded
  const uint16_t* wt;        // [9][CO][CI] bf16
  const float* bias;         // n_bias values or null (channels co >= n_bias get no bias)
  int n_bias;
  int relu;
  const uint16_t* mask16;    // B*h*w*CO bf16 or null: zero the output where mask <= 0
  uint16_t* y16;             // B*h*w*CO bf16 or null
  float* y32;                // B*h*w*4 fp32 (the first 4 channels) or null
  int y32_aligned;           // y32 is 16-byte aligned (the caller's array need not be)
};

// weight gradient of one convolution, as partial sums of workgroups
struct WgradArgs {
  int B, h, w, CI, CO;
  const uint16_t* x;         // layer input, B*h*w*CI bf16
  const uint16_t* g;         // output gradient, B*h*w*CO bf16
  float* partial;            // per workgroup: [9][CI][CO], then the bias's [CO]
};

// the sum of every layer's partials into the flat gradient
struct ReduceLayer {
  const float* partial;
  float* grad;               // weights [9][cin][cout], then biases [cout]
  int n_partial, CI, CO, cin, cout, block0;
};
struct ReduceArgs {
  int n_layers;
  ReduceLayer layer[kMaxLayers];
};

// one Adam step and the bf16 weights' refresh
struct PackLayer {
  int first, CI, CO, cin, cout;  // first: the layer's first parameter
  uint16_t* fwd;
  uint16_t* flip;
};
struct AdamArgs {
  float* w;
  const float* g;
  float* m;
  float* v;
  int n;
  float lr, b1, b2, eps, c1, c2;
  int n_layers;
  PackLayer layer[kMaxLayers];
};

struct LossArgs {
  int n_pix, h, w;           // n_pix = B*h*w
  const float* out;          // network output, n_pix*4
  const float* target;       // n_pix*4 (depth, normal)
  const float* mask;         // n_pix
  const float* drange;       // B*2
  float inv_count;           // loss normaliser (1 / n_pix)
  float lambda;              // normal-term weight
  uint16_t* grad16;          // n_pix*16 bf16 output gradient (channels >= 4 zero)
  float* loss_partial;       // one per 256-pixel block
};

struct ProposalInputs {
  int W, H, w, h;            // reference size and network input size (ceil(W/4), ceil(H/4))
  const __half* ref;         // reference grey values H*W
  const uint32_t* quad[4];   // source texel quads (null: channel stays 0)
  int sw[4], sh[4];          // source sizes
  float Hmid[36];            // per source: reference pixel -> source pixel, fronto-parallel plane at mid depth
  float* out;                // h*w*5
};

struct ProposalDecode {
  int W, H, w, h;
  const float* net_out;      // h*w*4
  float Kinv[9];
  float d_lo, d_hi;
  float* planes;             // H*W*4
};

struct TargetArgs {
  int W, H, w, h;
  const float* depth;        // H*W
  const float* normal;       // H*W*3
  const float* cost;         // H*W
  float max_cost;
  float* target;             // h*w*4
  float* mask;               // h*w
};

hipError_t launch_conv(const ConvArgs& a, hipStream_t st);
// workgroups (partial sums) of a weight gradient of that size, and its split
int wgrad_partials(int B, int h, int w, int* rb, int* segs, int* bands);
hipError_t launch_wgrad(const WgradArgs& a, int n_partial, hipStream_t st);
hipError_t launch_reduce_grads(const ReduceArgs& a, int n_blocks, hipStream_t st);
// bf16 NHWC with CP channels -> float32 NHWC with the first C channels
hipError_t launch_bf16_unpad(const uint16_t* x, int n_pix, int CP, int C, float* y, hipStream_t st);
hipError_t launch_pack_weights(const float* w, int CIN, int COUT, int CIP, int COP, uint16_t* fwd, uint16_t* flip,
                               hipStream_t st);
hipError_t launch_loss(const LossArgs& a, hipStream_t st);
hipError_t launch_adam(const AdamArgs& a, hipStream_t st);
hipError_t launch_proposal_inputs(const ProposalInputs& a, hipStream_t st);
hipError_t launch_proposal_decode(const ProposalDecode& a, hipStream_t st);
hipError_t launch_targets(const TargetArgs& a, hipStream_t st);

}  // namespace phimvs_net_internal
