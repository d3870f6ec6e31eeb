// Launch interface of the proposal network kernels (BF16 matrix products and
// the mixture head).
#pragma once

#include "qgbe_common.h"

namespace qgbe {

constexpr int kMlpIn = 8;
constexpr int kMlpHidden = 128;
constexpr int kMixK = 8;
constexpr int kMixD = 5;
constexpr int kMlpOut = kMixK * (1 + 2 * kMixD);    // 88
constexpr float kLsMin = -7.0f, kLsMax = 3.0f;       // clamp of the log scales
constexpr int kRecordWidth = kMlpIn + kMixD + 1;     // x[8], y[5], |g|
// flat parameter layout: W1 [8][128], b1, W2 [128][128], b2, W3 [128][88], b3
constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kMlpIn * kMlpHidden;
constexpr int kOffW2 = kOffB1 + kMlpHidden;
constexpr int kOffB2 = kOffW2 + kMlpHidden * kMlpHidden;
constexpr int kOffW3 = kOffB2 + kMlpHidden;
constexpr int kOffB3 = kOffW3 + kMlpHidden * kMlpOut;
constexpr int kMlpParams = kOffB3 + kMlpOut;

// BF16 weights transposed to [out][in], the head's 88 rows padded to 96
constexpr int kOffT1 = 0;
constexpr int kOffT2 = kOffT1 + kMlpHidden * kMlpIn;
constexpr int kOffT3 = kOffT2 + kMlpHidden * kMlpHidden;
constexpr int kMlpParamsT = kOffT3 + 96 * kMlpHidden;

constexpr int kMlpTileRows = 32;    // rows a workgroup takes at a time
constexpr int kMlpMaxTiles = 512;   // of a gradient
// What the gradient's tiles keep for the products over rows, kMlpTileRows values
// to a row: inputs, hidden activations and gradients in BF16 (act), gradients in
// FP32 for the biases, in the order of layers 1, 2, 3 (dz)
constexpr int kActX = 0;
constexpr int kActH1 = kActX + kMlpIn;
constexpr int kActH2 = kActH1 + kMlpHidden;
constexpr int kActDZ1 = kActH2 + kMlpHidden;
constexpr int kActDZ2 = kActDZ1 + kMlpHidden;
constexpr int kActDY = kActDZ2 + kMlpHidden;
constexpr int kActRows = kActDY + kMlpOut;
constexpr int kDzZ1 = 0;
constexpr int kDzZ2 = kDzZ1 + kMlpHidden;
constexpr int kDzY = kDzZ2 + kMlpHidden;
constexpr int kDzRows = kDzY + kMlpOut;

struct MlpTileArgs {
  long long rows;
  const float* X;          // row r: X[i * xs ..+7], i = idx ? idx[r] : r
  long long xs;
  const float* yw;         // gradient: row r: logits (5) and weight at yw[i * ys ..+5]
  long long ys;
  const int* idx;          // optional row order
  const __bf16* pb;        // weights, row-major
  const __bf16* pbt;       // weights, transposed
  const float* P;          // FP32 parameters (biases)
  float* Y;                // forward: head [rows][88]
  const double* wsum;      // gradient: sum of the rows' weights
  __bf16* act;             // gradient: [tiles][kActRows][kMlpTileRows]
  float* dz;               // gradient: [tiles][kDzRows][kMlpTileRows]
  double* loss_part;       // gradient: [tiles]
};

struct MlpGradArgs {
  const __bf16* act;
  const float* dz;
  const double* loss_part;
  int n_tiles;
  double* loss;            // the batch's loss is added
  float* grad;             // without adam: the gradient
  int adam;                // an Adam step in place of it
  float *p, *m, *v;
  __bf16 *pb, *pbt;
  float lr, b1, b2, eps, c1, c2;  // c1 = 1 - b1^t, c2 = 1 - b2^t
};

hipError_t launch_mlp_forward(const MlpTileArgs& g, hipStream_t st);
hipError_t launch_mlp_grad(const MlpTileArgs& g, hipStream_t st);
// The gradient (or Adam step) of the rows that launch_mlp_grad went through.
hipError_t launch_weight_grad(const MlpGradArgs& a, hipStream_t st);
hipError_t launch_refresh_weights(const float* p, __bf16* pb, __bf16* pbt, hipStream_t st);
// out[b] = sum of w[i * stride] over the rows of batch b
hipError_t launch_weight_sums(const float* w, long long stride, const int* idx, long long n, int batch, double* out,
                              hipStream_t st);
// Conditioning features of every (channel, node) row from the cell-averaged
// masses; mass7 receives those 7 averages.
hipError_t launch_features(const Grid& G, const Channel* chans, int nch, const double* mass2, double* mass7, float* X,
                           hipStream_t st);
// Network forward on X [rows][8] straight into the proposal table (thr, mu,
// sigma in the layout of qgbe_set_proposal_table), activations kept on chip.
hipError_t launch_mlp_table(const float* X, int rows, const __bf16* pb, const float* P, float alpha, uint32_t* thr,
                            float* mu, float* sigma, hipStream_t st);

}  // namespace qgbe
