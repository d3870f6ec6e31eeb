// The learned proposal's network on the matrix cores.
//
// x (8) -> Linear 8x128 -> SiLU -> Linear 128x128 -> SiLU -> Linear 128x88
// (head: 8 mixture logits, 8x5 locations, 8x5 log scales in logit space).
// Every product, forward and backward, is BF16 x BF16 -> FP32 on the matrix
// cores (v_mfma_f32_16x16x32_bf16).  Master weights and Adam moments are FP32.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "mlp.h"

namespace qgbe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kKStep = 32;   // K per MFMA

__device__ __forceinline__ float silu_f(float z) { return z / (1.0f + __expf(-z)); }
__device__ __forceinline__ float dsilu_f(float z) {
  const float s = 1.0f / (1.0f + __expf(-z));
  return s * (1.0f + z * (1.0f - s));
}

// ---------------------------------------------------------------------------
// The network on tiles of 32 rows: forward, and with kGrad the mixture head's
// weighted NLL and the backward pass down to the gradients of the layers'
// outputs, one kernel for what are nine products and elementwise passes.  A
// workgroup of 16 waves takes a tile through every layer; the activations stay
// in LDS, row-major, where they are the left operand of a product over features,
// so that every MFMA operand is one 16-byte read.  A wave owns 16 rows and one of
// the eight feature tiles of each layer and keeps their pre-activations in
// registers for the backward pass.  With kGrad the activations and gradients also
// go to global memory, transposed, for the products over rows
// (weight_grad_kernel).  Weights are read from L2: pb is row-major [in][out]
// (left factor of the backward products), pbt its transpose [out][in].
// A batch is bound by the chain of its phases (4096 rows are 128 workgroups), so
// a tile is low; the forward pass of 400,000 rows takes 262 us on tiles of 64
// rows and 213 on these (two workgroups per compute unit).
// Per row the arithmetic is that of the separate products: BF16 operands, FP32
// accumulation over K in steps of 32, FP32 bias, activations and head.
// ---------------------------------------------------------------------------
constexpr int kRows = kMlpTileRows;
constexpr int kBlocks = kRows / 16;       // row blocks of a tile; a wave owns one and one of 16 / kBlocks feature tiles
static_assert(16 / kBlocks == kMlpHidden / 16, "16 waves cover a layer");
static_assert(kRows == kKStep, "a tile is one K step of the products over rows");
constexpr int kHidPad = kMlpHidden + 8;   // row strides that spread the LDS banks
constexpr int kOut16 = 96;                // head columns rounded up to MFMA tiles
constexpr int kOutPad16 = kOut16 + 8;
constexpr int kHeadPad = kMlpOut + 4;

struct TileLds {
  __bf16 Xb[kRows][kKStep + 8];           // inputs, k >= 8 zero
  __bf16 H1[kRows][kHidPad];              // in the backward pass dZ2
  __bf16 H2[kRows][kHidPad];
};
struct GradLds {
  __bf16 dYb[kRows][kOutPad16];           // columns >= 88 zero
  float Y[kRows][kHeadPad];               // head, then its gradient
  float yw[kRows][kMixD + 1];
  double loss[kRows / 8];
};
static_assert(sizeof(TileLds) + sizeof(GradLds) <= 64 * 1024, "the default dynamic limit");

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// A fragment: lane l holds row l % 16, k = 8 (l / 16)..+7 of a row-major tile.
template <typename T>
__device__ __forceinline__ bf16x8 frag(const T* row, int k) { return *(const bf16x8*)(row + k); }

__device__ __forceinline__ floatx4 mfma(bf16x8 a, bf16x8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

template <bool kGrad>
__global__ __launch_bounds__(1024) void mlp_tile_kernel(MlpTileArgs g) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  TileLds& L = *reinterpret_cast<TileLds*>(lds_raw);
  GradLds& D = *reinterpret_cast<GradLds*>(lds_raw + sizeof(TileLds));  // kGrad only
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int r16 = lane & 15, kq = (lane >> 4) * 8, rq = (lane >> 4) * 4;
  const int m0 = 16 * (w % kBlocks);             // this wave's rows
  const int n = 16 * (w / kBlocks) + r16;        // this lane's feature column of a layer
  const bf16x8 zero8 = {};
  const floatx4 zero4 = floatx4{0.f, 0.f, 0.f, 0.f};
  const __bf16 *T1 = g.pbt + kOffT1, *T2 = g.pbt + kOffT2, *T3 = g.pbt + kOffT3;
  const float* P = g.P;
  // the paddings that no tile writes
  for (int e = tid; e < kRows * kKStep; e += 1024) L.Xb[e / kKStep][e % kKStep] = (__bf16)0.0f;
  if (kGrad)
    for (int e = tid; e < 8 * kRows; e += 1024) D.dYb[e % kRows][kMlpOut + e / kRows] = (__bf16)0.0f;
  __syncthreads();
  const long long n_tiles = (g.rows + kRows - 1) / kRows;
  for (long long tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    const long long row0 = tile * kRows;
    __bf16* act = kGrad ? g.act + tile * (kActRows * kRows) : nullptr;
    float* dz = kGrad ? g.dz + tile * (kDzRows * kRows) : nullptr;
    // four rows of column `row`, rows beyond the last as zero
    const auto keep_act = [&](int row, const floatx4& v) {
      bf16x4 b;
      for (int q = 0; q < 4; ++q) b[q] = (__bf16)(row0 + m0 + rq + q < g.rows ? v[q] : 0.f);
      *(bf16x4*)(act + row * kRows + m0 + rq) = b;
    };
    const auto keep_dz = [&](int row, const floatx4& v) {
      floatx4 z;
      for (int q = 0; q < 4; ++q) z[q] = row0 + m0 + rq + q < g.rows ? v[q] : 0.f;
      *(floatx4*)(dz + row * kRows + m0 + rq) = z;
    };
    // inputs; rows beyond the last are zero
    for (int e = tid; e < kRows * kMlpIn; e += 1024) {
      const int r = e / kMlpIn, c = e % kMlpIn;
      float x = 0.f;
      if (row0 + r < g.rows) x = g.X[(g.idx ? (long long)g.idx[row0 + r] : row0 + r) * g.xs + c];
      L.Xb[r][c] = (__bf16)x;
      if (kGrad) act[(kActX + c) * kRows + r] = (__bf16)x;
    }
    if (kGrad)
      for (int e = tid; e < kRows * (kMixD + 1); e += 1024) {
        const int r = e / (kMixD + 1), c = e % (kMixD + 1);
        float x = 0.f;
        if (row0 + r < g.rows) x = g.yw[(g.idx ? (long long)g.idx[row0 + r] : row0 + r) * g.ys + c];
        D.yw[r][c] = x;
      }
    __syncthreads();
    // layer 1 (K = 8 in one step, zeros beyond)
    floatx4 z1, z2;
    {
      const bf16x8 a = frag(L.Xb[m0 + r16], kq);
      z1 = mfma(a, kq == 0 ? frag(T1 + n * kMlpIn, 0) : zero8, zero4);
      const float bias = P[kOffB1 + n];
      floatx4 h;
      for (int q = 0; q < 4; ++q) {
        z1[q] += bias;
        h[q] = silu_f(z1[q]);
        L.H1[m0 + rq + q][n] = (__bf16)h[q];
      }
      if (kGrad) keep_act(kActH1 + n, h);
    }
    __syncthreads();
    // layer 2
    {
      bf16x8 a[4];
      for (int ks = 0; ks < 4; ++ks) a[ks] = frag(L.H1[m0 + r16], ks * kKStep + kq);
      z2 = zero4;
      for (int ks = 0; ks < 4; ++ks) z2 = mfma(a[ks], frag(T2 + n * kMlpHidden, ks * kKStep + kq), z2);
      const float bias = P[kOffB2 + n];
      floatx4 h;
      for (int q = 0; q < 4; ++q) {
        z2[q] += bias;
        h[q] = silu_f(z2[q]);
        L.H2[m0 + rq + q][n] = (__bf16)h[q];
      }
      if (kGrad) keep_act(kActH2 + n, h);
    }
    __syncthreads();
    // head: six column tiles, the last one half used
    if (n < kOut16) {  // wave-uniform
      bf16x8 a[4];
      for (int ks = 0; ks < 4; ++ks) a[ks] = frag(L.H2[m0 + r16], ks * kKStep + kq);
      floatx4 y = zero4;
      for (int ks = 0; ks < 4; ++ks) y = mfma(a[ks], frag(T3 + n * kMlpHidden, ks * kKStep + kq), y);
      if (n < kMlpOut) {
        const float bias = P[kOffB3 + n];
        for (int q = 0; q < 4; ++q) {
          const int r = m0 + rq + q;
          if (kGrad) D.Y[r][n] = y[q] + bias;
          else if (row0 + r < g.rows) g.Y[(row0 + r) * kMlpOut + n] = y[q] + bias;
        }
      }
    }
    __syncthreads();  // forward only: the next tile's inputs
    if (!kGrad) continue;
    // NLL of the mixture head and its gradient: eight lanes per row, one per
    // component; the sums over components in component order
    if (w < kRows / 8) {
      const int r = tid >> 3, k = tid & 7;
      const bool valid = row0 + r < g.rows;
      float* h = D.Y[r];
      const float s = valid ? (float)((double)D.yw[r][kMixD] / *g.wsum) : 0.f;
      const float hk = h[k];
      float mx = -INFINITY;
      for (int j = 0; j < kMixK; ++j) mx = fmaxf(mx, __shfl(hk, j, 8));
      const float ea = __expf(hk - mx);
      float se = 0.f;
      for (int j = 0; j < kMixK; ++j) se += __shfl(ea, j, 8);
      const float lse_a = mx + __logf(se);
      float l = hk - lse_a, z[kMixD], lr[kMixD];
      for (int e = 0; e < kMixD; ++e) {
        lr[e] = h[kMixK + kMixK * kMixD + k * kMixD + e];
        const float ls = fminf(fmaxf(lr[e], kLsMin), kLsMax);
        const float zz = (D.yw[r][e] - h[kMixK + k * kMixD + e]) * __expf(-ls);
        z[e] = zz;
        l += -0.5f * zz * zz - ls - 0.91893853320467274f;
      }
      float m2 = -INFINITY;
      for (int j = 0; j < kMixK; ++j) m2 = fmaxf(m2, __shfl(l, j, 8));
      const float eb = __expf(l - m2);
      float se2 = 0.f;
      for (int j = 0; j < kMixK; ++j) se2 += __shfl(eb, j, 8);
      const float lm = m2 + __logf(se2);
      double part = k == 0 && valid ? -(double)s * (double)lm : 0.0;
      const float resp = __expf(l - lm), pi = __expf(hk - lse_a);
      const auto put = [&](int c, float v) {
        if (!valid) v = 0.f;
        h[c] = v;
        D.dYb[r][c] = (__bf16)v;
      };
      put(k, -s * (resp - pi));
      for (int e = 0; e < kMixD; ++e) {
        const float ls = fminf(fmaxf(lr[e], kLsMin), kLsMax);
        const float gmu = -s * resp * z[e] * __expf(-ls);
        float gls = -s * resp * (z[e] * z[e] - 1.0f);
        if (lr[e] < kLsMin || lr[e] > kLsMax) gls = 0.f;
        put(kMixK + k * kMixD + e, gmu);
        put(kMixK + kMixK * kMixD + k * kMixD + e, gls);
      }
      for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off, 64);
      if (lane == 0) D.loss[w] = part;
    }
    __syncthreads();
    if (tid == 0) {
      double loss = 0.0;
      for (int i = 0; i < kRows / 8; ++i) loss += D.loss[i];
      g.loss_part[tile] = loss;
    }
    // the head's gradient, four rows of a column per thread
    for (int e = tid; e < kMlpOut * (kRows / 4); e += 1024) {
      const int c = e / (kRows / 4), r = e % (kRows / 4) * 4;
      floatx4 v;
      bf16x4 b;
      for (int q = 0; q < 4; ++q) {
        v[q] = D.Y[r + q][c];
        b[q] = (__bf16)v[q];
      }
      *(floatx4*)(dz + (kDzY + c) * kRows + r) = v;
      *(bf16x4*)(act + (kActDY + c) * kRows + r) = b;
    }
    // dZ2 = (dY W3^T) silu'(Z2)
    {
      bf16x8 a[3];
      for (int ks = 0; ks < 3; ++ks) a[ks] = frag(D.dYb[m0 + r16], ks * kKStep + kq);
      const __bf16* wr = g.pb + kOffW3 + n * kMlpOut;
      floatx4 dh = zero4;
      for (int ks = 0; ks < 3; ++ks)
        dh = mfma(a[ks], ks * kKStep + kq < kMlpOut ? frag(wr, ks * kKStep + kq) : zero8, dh);
      for (int q = 0; q < 4; ++q) {
        dh[q] = dh[q] * dsilu_f(z2[q]);
        L.H1[m0 + rq + q][n] = (__bf16)dh[q];
      }
      keep_act(kActDZ2 + n, dh);
      keep_dz(kDzZ2 + n, dh);
    }
    __syncthreads();
    // dZ1 = (dZ2 W2^T) silu'(Z1)
    {
      bf16x8 a[4];
      for (int ks = 0; ks < 4; ++ks) a[ks] = frag(L.H1[m0 + r16], ks * kKStep + kq);
      floatx4 dh = zero4;
      for (int ks = 0; ks < 4; ++ks) dh = mfma(a[ks], frag(g.pb + kOffW2 + n * kMlpHidden, ks * kKStep + kq), dh);
      for (int q = 0; q < 4; ++q) dh[q] = dh[q] * dsilu_f(z1[q]);
      keep_act(kActDZ1 + n, dh);
      keep_dz(kDzZ1 + n, dh);
    }
    __syncthreads();  // the next tile's inputs
  }
}

// Position of parameter i in the transposed BF16 weights, -1 for a bias.
__device__ __forceinline__ int transposed_at(int i) {
  if (i < kOffB1) return kOffT1 + i % kMlpHidden * kMlpIn + i / kMlpHidden;
  if (i < kOffW2) return -1;
  if (i < kOffB2) return kOffT2 + (i - kOffW2) % kMlpHidden * kMlpHidden + (i - kOffW2) / kMlpHidden;
  if (i < kOffW3) return -1;
  if (i < kOffB3) return kOffT3 + (i - kOffW3) % kMlpOut * kMlpHidden + (i - kOffW3) / kMlpOut;
  return -1;
}

__device__ __forceinline__ void put_weight(__bf16* pb, __bf16* pbt, int i, float w) {
  pb[i] = (__bf16)w;
  const int t = transposed_at(i);
  if (t >= 0) pbt[t] = (__bf16)w;
}

// BF16 copies of the master weights, row-major and transposed (head rows
// beyond 88 zero).
__global__ void refresh_weights_kernel(const float* __restrict__ p, __bf16* __restrict__ pb, __bf16* __restrict__ pbt) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kMlpParams) put_weight(pb, pbt, i, p[i]);
  if (i < (kOut16 - kMlpOut) * kMlpHidden) pbt[kOffT3 + kMlpOut * kMlpHidden + i] = (__bf16)0.0f;
}

// The gradient of a batch from what mlp_tile_kernel kept, and with adam the
// bias-corrected Adam step on the FP32 master weights and their BF16 copies.
// The sums over the rows are bracketed by kGradChunk rows for the weights, one
// chain of MFMAs each, and by kBiasChunk rows for the biases (four chains of
// every fourth row, added in pairs): the values that training has always had, up
// to the order in which the chunks are added, which is in FP64 here.  (On sums
// in other brackets the losses of two epochs move by some 3e-7: the BF16 weights
// round the other way now and then.)
// Block b < kGradTiles: a 16 x 16 tile of a weight matrix, a wave per chunk (in
// turn); the others: kBiasCols biases each.  206 workgroups, one round; bound by
// the latency of a chain (16 loads, 8 MFMAs) and of the Adam step behind it.  A
// batch of 4096 rows takes 18.4 us in mlp_tile_kernel and 7.6 here (with the
// products over rows inside the tiles, and their slices summed, 22.6 and 9; as
// separate products and passes 196 in 21 launches).
constexpr int kGradChunk = 256, kBiasChunk = 64;
constexpr int kTilesW2 = (kMlpHidden / 16) * (kMlpHidden / 16), kTilesW3 = kMlpHidden / 16 * (kOut16 / 16),
              kTilesW1 = kMlpHidden / 16;
constexpr int kGradTiles = kTilesW2 + kTilesW3 + kTilesW1;
constexpr int kBiasCols = 4;
static_assert(kDzRows % kBiasCols == 0, "whole groups of biases");

__global__ __launch_bounds__(1024) void weight_grad_kernel(MlpGradArgs a) {
  __shared__ float sums[16][256];  // weights: a chunk per wave
  __shared__ double wave_sums[16];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const auto apply = [&](int i, float g) {
    if (!a.adam) {
      a.grad[i] = g;
      return;
    }
    const float mi = a.b1 * a.m[i] + (1.f - a.b1) * g;
    const float vi = a.b2 * a.v[i] + (1.f - a.b2) * g * g;
    a.m[i] = mi;
    a.v[i] = vi;
    const float p = a.p[i] - a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
    a.p[i] = p;
    put_weight(a.pb, a.pbt, i, p);
  };
  if (blockIdx.x < kGradTiles) {
    const int r16 = lane & 15, kq = (lane >> 4) * 8;
    int t = blockIdx.x, m, n, left, right;  // the tile, and its operands' first rows of act
    bool in_a = true, in_b = true;          // this lane's rows exist
    if (t < kTilesW2) {  // H1^T dZ2
      m = t / (kMlpHidden / 16), n = t % (kMlpHidden / 16);
      left = kActH1, right = kActDZ2;
    } else if (t < kTilesW2 + kTilesW3) {  // H2^T dY
      t -= kTilesW2;
      m = t / (kOut16 / 16), n = t % (kOut16 / 16);
      left = kActH2, right = kActDY;
      in_b = 16 * n + r16 < kMlpOut;
    } else {  // X^T dZ1
      m = 0, n = t - kTilesW2 - kTilesW3;
      left = kActX, right = kActDZ1;
      in_a = r16 < kMlpIn;
    }
    const int tiles = a.n_tiles, chunk_tiles = kGradChunk / kRows, chunks = (tiles + chunk_tiles - 1) / chunk_tiles;
    const bf16x8 zero8 = {};
    double g = 0.0;
    for (int c0 = 0; c0 < chunks; c0 += 16) {
      const int c = c0 + w;
      const int k0 = c * chunk_tiles, k1 = min(tiles, k0 + chunk_tiles);
      const __bf16* pa = a.act + ((size_t)k0 * kActRows + left + 16 * m + r16) * kRows;
      const __bf16* pb = a.act + ((size_t)k0 * kActRows + right + 16 * n + r16) * kRows;
      floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < chunk_tiles; ++k) {
        if (k0 + k >= k1) break;
        const bf16x8 x = in_a ? frag(pa + (size_t)k * kActRows * kRows, kq) : zero8;
        const bf16x8 y = in_b ? frag(pb + (size_t)k * kActRows * kRows, kq) : zero8;
        acc = mfma(x, y, acc);
      }
      *(floatx4*)(sums[w] + 4 * lane) = acc;
      __syncthreads();
      if (tid < 256)
        for (int i = 0; i < 16 && c0 + i < chunks; ++i) g += (double)sums[i][tid];
      __syncthreads();
    }
    if (tid >= 256) return;
    // element tid: lane tid / 4's value tid % 4
    const int row = 16 * m + (tid >> 6) * 4 + (tid & 3), col = 16 * n + ((tid >> 2) & 15);
    if (left == kActH1) apply(kOffW2 + row * kMlpHidden + col, (float)g);
    else if (left == kActH2 && col < kMlpOut) apply(kOffW3 + row * kMlpOut + col, (float)g);
    else if (left == kActX && row < kMlpIn) apply(kOffW1 + row * kMlpHidden + col, (float)g);
    return;
  }
  // biases: wave w takes column w / 4; 16 chunks of rows side by side, four lanes each
  const int col = (blockIdx.x - kGradTiles) * kBiasCols + w / 4, ph = lane & 3;
  double g = 0.0;
  for (int c = (w & 3) * 16 + (lane >> 2); c * (kBiasChunk / kRows) < a.n_tiles; c += 64) {
    float s = 0.f;
    for (int t = 0; t < kBiasChunk / kRows; ++t) {
      const int tile = c * (kBiasChunk / kRows) + t;
      if (tile >= a.n_tiles) break;
      const float* d = a.dz + ((size_t)tile * kDzRows + col) * kRows + ph;
#pragma unroll
      for (int i = 0; i < kRows / 4; ++i) s += d[4 * i];
    }
    s += __shfl_xor(s, 1, 4);
    s += __shfl_xor(s, 2, 4);
    if (ph == 0) g += (double)s;
  }
  for (int off = 32; off > 0; off >>= 1) g += __shfl_xor(g, off, 64);
  if (lane == 0) wave_sums[w] = g;
  __syncthreads();
  if ((tid & 255) == 0) {
    const float sum = (float)((wave_sums[w] + wave_sums[w + 1]) + (wave_sums[w + 2] + wave_sums[w + 3]));
    if (col < kDzZ2) apply(kOffB1 + col, sum);
    else if (col < kDzY) apply(kOffB2 + col - kDzZ2, sum);
    else apply(kOffB3 + col - kDzY, sum);
  }
  if (blockIdx.x == kGradTiles && w == 0) {  // the batch's loss is added
    double l = 0.0;
    for (int k = lane; k < a.n_tiles; k += 64) l += a.loss_part[k];
    for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
    if (lane == 0) *a.loss += l;
  }
}

// Weight sums of the batches: block b sums the weights of rows b * batch.. of
// the order idx (or of the rows themselves).
__global__ __launch_bounds__(256) void weight_sum_kernel(const float* __restrict__ w, long long stride,
                                                         const int* __restrict__ idx, long long n, int batch,
                                                         double* __restrict__ out) {
  __shared__ double sh[4];
  const long long lo = (long long)blockIdx.x * batch, hi = lo + batch < n ? lo + batch : n;
  double s = 0.0;
  for (long long r = lo + threadIdx.x; r < hi; r += blockDim.x) s += w[(idx ? (long long)idx[r] : r) * stride];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) out[blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// Inference straight to the proposal table: each wave takes 16-row blocks of
// X through the network (layer 1 on the vector ALUs, K = 8; layers 2 and 3 on
// the matrix cores with the block's weights staged in LDS, transposed so the
// K index is contiguous) and turns its head rows into table rows; the
// activations never leave LDS.  Numerics as the staged GEMMs: BF16 inputs,
// weights and hidden activations, FP32 accumulation and head.
constexpr int kInfWaves = 4;
constexpr int kHPad = kMlpHidden + 8;     // row stride of the hidden tile (bank spread)
constexpr int kOutPad = 96;               // head columns rounded up to MFMA tiles
constexpr int kYPad = kMlpOut + 4;

__global__ __launch_bounds__(kInfWaves * 64) void mlp_table_kernel(const float* __restrict__ X, int rows,
                                                                    const __bf16* __restrict__ pb,
                                                                    const float* __restrict__ P, float alpha,
                                                                    uint32_t* __restrict__ thr, float* __restrict__ mu,
                                                                    float* __restrict__ sigma) {
  __shared__ __bf16 W2t[kMlpHidden][kHPad];   // [n][k]
  __shared__ __bf16 W3t[kOutPad][kHPad];      // [n][k], rows >= 88 zero
  __shared__ float W1s[kMlpIn][kMlpHidden];
  __shared__ float bias[2 * kMlpHidden + kMlpOut];
  __shared__ float Xs[kInfWaves][16][kMlpIn];
  __shared__ __bf16 H[kInfWaves][16][kHPad];
  __shared__ float Ys[kInfWaves][16][kYPad];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  for (int e = tid; e < kMlpHidden * kMlpHidden; e += blockDim.x) {
    const int k = e / kMlpHidden, n = e % kMlpHidden;
    W2t[n][k] = pb[kOffW2 + e];
  }
  for (int e = tid; e < kOutPad * kMlpHidden; e += blockDim.x) {
    const int n = e / kMlpHidden, k = e % kMlpHidden;
    W3t[n][k] = n < kMlpOut ? pb[kOffW3 + k * kMlpOut + n] : (__bf16)0.0f;
  }
  for (int e = tid; e < kMlpIn * kMlpHidden; e += blockDim.x) W1s[e / kMlpHidden][e % kMlpHidden] = (float)pb[kOffW1 + e];
  for (int e = tid; e < kMlpHidden; e += blockDim.x) {
    bias[e] = P[kOffB1 + e];
    bias[kMlpHidden + e] = P[kOffB2 + e];
  }
  for (int e = tid; e < kMlpOut; e += blockDim.x) bias[2 * kMlpHidden + e] = P[kOffB3 + e];
  __syncthreads();
  const int n_blocks = (rows + 15) / 16;
  const int r16 = lane & 15, kq = (lane >> 4) * 8, rq = (lane >> 4) * 4;
  for (int t = blockIdx.x * kInfWaves + w; t < n_blocks; t += gridDim.x * kInfWaves) {
    const int row0 = t * 16;
    // inputs, rounded to BF16 like the staged path
    for (int e = lane; e < 16 * kMlpIn; e += 64) {
      const int r = e / kMlpIn, c = e % kMlpIn;
      Xs[w][r][c] = row0 + r < rows ? (float)(__bf16)X[(size_t)(row0 + r) * kMlpIn + c] : 0.0f;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // layer 1: lane owns columns lane and lane + 64
    for (int h = 0; h < 2; ++h) {
      const int n = lane + 64 * h;
      float wcol[kMlpIn];
      for (int k = 0; k < kMlpIn; ++k) wcol[k] = W1s[k][n];
      for (int r = 0; r < 16; ++r) {
        float z = bias[n];
        for (int k = 0; k < kMlpIn; ++k) z = fmaf(Xs[w][r][k], wcol[k], z);
        H[w][r][n] = (__bf16)silu_f(z);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // layers 2 and 3 on the matrix cores
    for (int layer = 0; layer < 2; ++layer) {
      bf16x8 a[kMlpHidden / kKStep];
      for (int ks = 0; ks < kMlpHidden / kKStep; ++ks)
        for (int q = 0; q < 8; ++q) a[ks][q] = H[w][r16][ks * kKStep + kq + q];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const int n_tiles = layer == 0 ? kMlpHidden / 16 : kOutPad / 16;
      for (int j = 0; j < n_tiles; ++j) {
        floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
        for (int ks = 0; ks < kMlpHidden / kKStep; ++ks) {
          bf16x8 b;
          for (int q = 0; q < 8; ++q)
            b[q] = layer == 0 ? W2t[j * 16 + r16][ks * kKStep + kq + q] : W3t[j * 16 + r16][ks * kKStep + kq + q];
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks], b, acc, 0, 0, 0);
        }
        const int c = j * 16 + r16;
        for (int q = 0; q < 4; ++q) {
          if (layer == 0) {
            H[w][rq + q][c] = (__bf16)silu_f(acc[q] + bias[kMlpHidden + c]);
          } else if (c < kMlpOut) {
            Ys[w][rq + q][c] = acc[q] + bias[2 * kMlpHidden + c];
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    // head -> table: four lanes per row; lane part 0 also forms the thresholds
    const int r = lane >> 2, part = lane & 3;
    const int row = row0 + r;
    if (row < rows) {
      const float* h = Ys[w][r];
      if (part == 0) {
        double mx = -1e300;
        for (int k = 0; k < kMixK; ++k) mx = fmax(mx, (double)h[k]);
        double e[kMixK], se = 0.0;
        for (int k = 0; k < kMixK; ++k) { e[k] = exp((double)h[k] - mx); se += e[k]; }
        double cum = 0.0;
        for (int k = 0; k < kMixK; ++k) {
          const double lo = (double)alpha + (1.0 - (double)alpha) * cum;
          double tt = floor(lo * 4294967296.0);
          tt = tt > 4294967295.0 ? 4294967295.0 : tt;
          thr[(size_t)row * kMixK + k] = (uint32_t)tt;
          cum += e[k] / se;
        }
      }
      for (int k = part; k < kMixK; k += 4)
        for (int d = 0; d < kMixD; ++d) {
          mu[((size_t)row * kMixK + k) * kMixD + d] = h[kMixK + k * kMixD + d];
          const float lr = h[kMixK + kMixK * kMixD + k * kMixD + d];
          sigma[((size_t)row * kMixK + k) * kMixD + d] = expf(fminf(fmaxf(lr, kLsMin), kLsMax));
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// Per-species thermal mass squared averaged over the cells (one workgroup per
// species, fixed summation order).
__global__ void mass_mean_kernel(Grid G, const double* __restrict__ mass2, double* __restrict__ mean) {
  __shared__ double part[256];
  const int sp = blockIdx.x;
  double s = 0.0;
  for (int x = threadIdx.x; x < G.cells; x += blockDim.x) s += mass2[sp * G.cells + x];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) mean[sp] = part[0] / G.cells;
}

// Conditioning inputs of every (channel, node) row; the masses are the
// per-species values in mass7 (cell averages), so one table serves all cells.
__global__ void features_kernel(Grid G, const Channel* __restrict__ chans, int nch, const double* __restrict__ mass7,
                                float* __restrict__ X) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nch * G.nodes) return;
  const int ci = r / G.nodes, node = r % G.nodes;
  const int iz = node % G.np[2], iy = (node / G.np[2]) % G.np[1], ix = node / (G.np[2] * G.np[1]);
  const double p[3] = {node_coord(G.ph[0], G.dp[0], ix), node_coord(G.ph[1], G.dp[1], iy),
                       node_coord(G.ph[2], G.dp[2], iz)};
  const double pn = sqrt(G.ph[0] * G.ph[0] + G.ph[1] * G.ph[1] + G.ph[2] * G.ph[2]);
  const int sp = chans[ci].sp[0];
  const double a = sqrt(p[0] * p[0] + p[1] * p[1] + p[2] * p[2]);
  const double E1 = sqrt(a * a + mass7[sp]);
  float* x = X + (size_t)r * kMlpIn;
  x[0] = (float)(p[0] / G.ph[0]);
  x[1] = (float)(p[1] / G.ph[1]);
  x[2] = (float)(p[2] / G.ph[2]);
  x[3] = (float)(a / pn);
  x[4] = (float)(E1 / pn);
  x[5] = (float)(mass7[kGluon] / (pn * pn));
  x[6] = (float)(sp / 3.0 - 1.0);
  x[7] = nch > 1 ? (float)(2.0 * ci / (nch - 1) - 1.0) : 0.0f;
}

}  // namespace

hipError_t launch_mlp_forward(const MlpTileArgs& g, hipStream_t st) {
  if (g.rows <= 0) return hipSuccess;
  const long long tiles = (g.rows + kRows - 1) / kRows;
  hipLaunchKernelGGL(mlp_tile_kernel<false>, dim3((unsigned)std::min<long long>(tiles, 4096)), dim3(1024),
                     sizeof(TileLds), st, g);
  return hipGetLastError();
}

hipError_t launch_mlp_grad(const MlpTileArgs& g, hipStream_t st) {
  if (g.rows <= 0 || g.rows > (long long)kMlpMaxTiles * kRows) return hipErrorInvalidValue;
  hipLaunchKernelGGL(mlp_tile_kernel<true>, dim3((unsigned)((g.rows + kRows - 1) / kRows)), dim3(1024),
                     sizeof(TileLds) + sizeof(GradLds), st, g);
  return hipGetLastError();
}

hipError_t launch_weight_grad(const MlpGradArgs& a, hipStream_t st) {
  if (a.n_tiles <= 0 || a.n_tiles > kMlpMaxTiles) return hipErrorInvalidValue;
  hipLaunchKernelGGL(weight_grad_kernel, dim3(kGradTiles + kDzRows / kBiasCols), dim3(1024), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_refresh_weights(const float* p, __bf16* pb, __bf16* pbt, hipStream_t st) {
  hipLaunchKernelGGL(refresh_weights_kernel, dim3((kMlpParams + 255) / 256), dim3(256), 0, st, p, pb, pbt);
  return hipGetLastError();
}

hipError_t launch_weight_sums(const float* w, long long stride, const int* idx, long long n, int batch, double* out,
                              hipStream_t st) {
  const long long blocks = (n + batch - 1) / batch;
  if (blocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(weight_sum_kernel, dim3((unsigned)blocks), dim3(256), 0, st, w, stride, idx, n, batch, out);
  return hipGetLastError();
}

hipError_t launch_features(const Grid& G, const Channel* chans, int nch, const double* mass2, double* mass7, float* X,
                           hipStream_t st) {
  hipLaunchKernelGGL(mass_mean_kernel, dim3(kSpecies), dim3(256), 0, st, G, mass2, mass7);
  const int rows = nch * G.nodes;
  if (rows > 0)
    hipLaunchKernelGGL(features_kernel, dim3((rows + 127) / 128), dim3(128), 0, st, G, chans, nch, mass7, X);
  return hipGetLastError();
}

hipError_t launch_mlp_table(const float* X, int rows, const __bf16* pb, const float* P, float alpha, uint32_t* thr,
                            float* mu, float* sigma, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  const int n_blocks = (rows + 15) / 16;
  int grid = (n_blocks + kInfWaves - 1) / kInfWaves;
  grid = grid > 512 ? 512 : grid;
  hipLaunchKernelGGL(mlp_table_kernel, dim3(grid), dim3(kInfWaves * 64), 0, st, X, rows, pb, P, alpha, thr, mu, sigma);
  return hipGetLastError();
}

}  // namespace qgbe
