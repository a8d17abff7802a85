// Learned corrector network (BF16 MFMA kernels): shared definitions and the
// launch interface used by the host runtime.
//
// The network maps a real-space orientation volume psi[N][H][W] (FP32,
// planar) to psi + r, r = conv3(relu(conv2(relu(conv1(psi))))), each conv a
// 3x3 cross-correlation with circular padding.  Channels are padded to 32:
// the input's channels N..31 are zero and so are the weights that read them
// (layer 1) or write output channels N..31 (layer 3).
//
// Layouts
//   activations, gradients between layers: bfloat16, channels last
//       act[b][y][x][32]  (64 bytes per pixel)
//   parameters (FP32 master copy, the order of the public parameter vector):
//       for l = 0, 1, 2:  W_l[o][c][tap] (32 x 32 x 9), then b_l[o] (32),
//       tap = (dy+1)*3 + (dx+1) for the input offset (dy, dx)
//   MFMA weights (bfloat16): A[l][tap][row][k] with row the output channel of
//       the product and k the reduced channel: forward A = W[o][c] (row o,
//       k c); input gradient A = W[o][c] of the mirrored tap (row c, k o).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace se2n {

constexpr int kCnnC = 32;                       // padded channels
constexpr int kCnnW = kCnnC * kCnnC * 9;        // weights per layer
constexpr int kCnnL = kCnnW + kCnnC;            // parameters per layer
constexpr int kCnnP = 3 * kCnnL;                // parameter vector length
constexpr int kCnnTile = 16;                    // pixel tile side of the conv kernels
constexpr int kCnnPart = kCnnW + kCnnC;         // one workgroup's weight + bias gradient partial
constexpr int kCnnWgradParts = 512;             // weight gradient partials per layer at most
constexpr int kCnnScaleBlocks = 512;            // partial sums of squares per image

using bf16 = __bf16;

// scale[b] = root mean square of psi[b] (1 if zero); parts: B*kCnnScaleBlocks floats of scratch
hipError_t cnn_rms(const float* psi, float* parts, float* scale, int N, int M, int B, hipStream_t st);
// psi planar FP32 [B][N][M][M] / scale[b] -> act bf16 channels-last [B][M][M][32] (zero channels >= N)
hipError_t cnn_pack(const float* psi, const float* scale, bf16* act, int N, int M, int B, hipStream_t st);
// The network on B images of side M (M % 16 == 0):
//   out = coarse + scale[b] (layer 3), channels < N   (FP32 planar)
// a0: the packed input, needed when out overlaps coarse (which it may then
// equal); nullptr: coarse / scale is packed on the way.
hipError_t cnn_forward(const bf16* a0, const bf16* wf, const float* params, const float* coarse, float* out,
                       const float* scale, int N, int M, int B, hipStream_t st);
// The same for training: the packed input a0 and the activations a1, a2 of the
// hidden layers (bf16, channels last) and, each image in units of scale[b],
// d = (out - target) / scale[b] as g = gscale d (bf16 channels last, zero
// channels >= N) and in sums of d^2 per tile (cnn_loss_blocks).
hipError_t cnn_forward_loss(const bf16* wf, const float* params, const float* coarse, const float* target,
                            const float* scale, bf16* a0, bf16* a1, bf16* a2, bf16* g, float* loss_parts, float gscale,
                            int N, int M, int B, hipStream_t st);
int cnn_loss_blocks(int M, int B);
// Input gradient of a layer: out = conv(g) * [mask > 0]   (bf16, channels last)
hipError_t cnn_dgrad(const bf16* g, const bf16* wd, const bf16* mask, bf16* out, int M, int B, hipStream_t st);
// Weight + bias gradient partials of one layer: g (bf16 CL, the layer's output
// gradient), a (bf16 CL, the layer's input); one partial of kCnnPart floats per
// workgroup (cnn_wgrad_parts of them).
int cnn_wgrad_parts(int M, int B);
hipError_t cnn_wgrad(const bf16* g, const bf16* a, float* parts, int M, int B, hipStream_t st);
// Sum the partials of the three layers (one after the other in parts) into the
// gradient vector (per layer W[o][c][tap], b[o]), in a fixed order.
hipError_t cnn_wgrad_reduce(const float* parts, int nparts, float* grads, hipStream_t st);
// loss = sum(parts) * inv_numel (one value, deterministic order)
hipError_t cnn_loss_reduce(const float* parts, int nparts, float inv_numel, float* loss, hipStream_t st);
// Adam on the FP32 parameters (step t >= 1, bias-corrected), then refresh the MFMA weights.
hipError_t cnn_adam(float* params, const float* grads, float* m, float* v, int t, float lr, float beta1,
                    float beta2, float eps, hipStream_t st);
hipError_t cnn_prep(const float* params, bf16* wfwd, bf16* wdgrad, hipStream_t st);

}  // namespace se2n
