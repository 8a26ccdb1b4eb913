// Internal launch interface of the learned-shrinkage kernels (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

namespace shear {

// One 3x3 layer launch. Layer 0 reads the FP32 coefficients, layers 1 and 2
// bfloat16 channel-last activations [b][y][x][32]. Layers 0 and 1 write
// relu(conv + bias) as bfloat16 channel-last activations (out_bf); layer 2
// writes the shrunk FP32 coefficients out_f (coef kept where
// |coef * scale| >= softplus(conv + bias), plane `lowpass` kept whole) and,
// if non-null, the thresholds tau.
struct ConvArgs {
    const void* in;
    const unsigned short* W;  // packed bfloat16 weights [coutp][9][cinp]
    const float* bias;
    const float* scale;       // [B][K] 1 / (sigma_b RMS_k)
    const float* coef;        // layer 2: the coefficients (B x K x N x M)
    void* out_bf;
    float* out_f;
    float* tau;
    int N, M;
    int cin, cout;            // real channel counts (K for the coefficient side)
    int lowpass;
    // training
    void* z;                           // layer 0 training: the normalised bfloat16 input, written
    const float* coef2;                // layer 2 training: coefficients of the clean images
    const unsigned short* mask_act;    // backward data: saved activation whose relu mask applies
    float* loss;                       // layer 2 training: each 8 x 32 tile's sum of squared residuals
    float gate_ehi, gate_elo, gate_c;  // log2(e) / temperature in two parts, -2 loss scale / temperature
    int cus;  // compute units of the device (grid of the persistent layers)
};

// Weight-gradient launch: dy bf16 channel-last with dy_ch channels; input x bf16 channel-last (the packed z
// for layer 0, else a hidden activation); per-block partials to part.
struct WgradArgs {
    const unsigned short* dy;
    int dy_ch;
    const unsigned short* xb;
    float* part;
    int batch, N, M;
};

// Byte offsets of the packed parameter block of a K-filter network.
struct ShrinkLayout {
    size_t w1, w2, w3, b1, b2, b3, bytes;
};

int shrink_cinp(int K);   // padded input channels of layer 0 (32 or 64)
int shrink_coutp(int K);  // padded output channels of layer 2 (multiple of 16)
bool shrink_supported(int K, int N, int M);
ShrinkLayout shrink_layout(int K);

// FP32 natural-layout parameters (device) -> packed block (device).
hipError_t launch_shrink_pack(int K, const float* W1, const float* b1, const float* W2, const float* b2,
                              const float* W3, const float* b3, void* packed, hipStream_t st);
hipError_t launch_inv_scale(const float* sigma, const float* rms, float* out, int B, int K, hipStream_t st);
// layer 0 of training and 6 of inference: layer 1 of the network, its input staged straight from the FP32
// coefficients (coef, scale, cin = K) as z = bf16(c x scale); layer 0 also writes z, channel-last
// [b][y][x][shrink_cinp(K)], zero padded. 1: the hidden layer; 2: the shrink layer; 3: the last layer with
// the training epilogue; 4: backward data from 32 gradient channels; 5: from shrink_cinp(K).
hipError_t launch_conv(int layer, int K, const ConvArgs& a, int batch, hipStream_t st);
// weight gradients of layer 0, 1 or 2 (partials of `blocks` blocks, a multiple of 8; N % 8 == 0, M % 32 == 0)
hipError_t launch_wgrad(int layer, int K, const WgradArgs& a, int blocks, hipStream_t st);
hipError_t launch_wgrad_reduce(const float* part, float* dW, float* db, int nblk, int cout, int cin, int coutp, int cinp,
                               hipStream_t st);
// loss = scale x the sum of the n tiles' squared residuals
hipError_t launch_loss_sum(const float* part, int n, float scale, float* loss, hipStream_t st);
hipError_t launch_pack_weights_t(const float* W, unsigned short* out, int cout, int cin, int rows, int cols,
                                 hipStream_t st);
hipError_t launch_adam(float* p, const float* g, float* m, float* v, int n, float lr, float b1, float b2, float eps,
                       int step, hipStream_t st);

}  // namespace shear
