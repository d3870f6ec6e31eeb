// C ABI of the learned proposal: network weights, forward and backward
// passes, training with Adam, the proposal table, and the sample recorder.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>
#include <random>
#include <type_traits>
#include <vector>

#include "context.h"

using namespace qgbe;

namespace {

constexpr int kBatch = QGBE_MLP_BATCH;
static_assert(QGBE_MLP_PARAMS == kMlpParams, "header and kernels disagree on the parameter count");

qgbe_status mlp_ensure(qgbe_ctx* c) {
  MlpState& m = c->mlp;
  if (m.ready) return QGBE_OK;
  char* base = nullptr;
  size_t used = 0;
  const auto take = [&](auto** p, size_t n) {
    using T = std::remove_reference_t<decltype(**p)>;
    if (base) *p = reinterpret_cast<T*>(base + used);
    used += (n * sizeof(T) + 255) & ~size_t(255);
  };
  for (int pass = 0; pass < 2; ++pass) {  // first for the size
    used = 0;
    take(&m.params, kMlpParams);
    take(&m.m, kMlpParams);
    take(&m.v, kMlpParams);
    take(&m.grad, kMlpParams);
    take(&m.pb, kMlpParams);
    take(&m.pbt, kMlpParamsT);
    take(&m.X, (size_t)kBatch * kMlpIn);
    take(&m.yw, (size_t)kBatch * (kMixD + 1));
    take(&m.Y, (size_t)kBatch * kMlpOut);
    take(&m.act, (size_t)kMlpMaxTiles * kActRows * kMlpTileRows);
    take(&m.dz, (size_t)kMlpMaxTiles * kDzRows * kMlpTileRows);
    take(&m.loss_part, kMlpMaxTiles);
    take(&m.scalars, 2);
    if (pass == 0) {
      const qgbe_status s = dev_alloc(c, &m.arena, used, "proposal network");
      if (s) return s;
      base = m.arena;
    }
  }
  m.ready = true;
  return QGBE_OK;
}

// Tile arguments of rows in place: X (stride xs), and yw (stride ys) or NULL.
MlpTileArgs tile_args(const qgbe_ctx* c, long long rows, const float* X, long long xs, const float* yw, long long ys,
                      const int* idx) {
  const MlpState& m = c->mlp;
  MlpTileArgs g{};
  g.rows = rows;
  g.X = X; g.xs = xs;
  g.yw = yw; g.ys = ys;
  g.idx = idx;
  g.pb = m.pb; g.pbt = m.pbt; g.P = m.params;
  g.act = m.act; g.dz = m.dz; g.loss_part = m.loss_part;
  return g;
}

MlpGradArgs grad_args(const qgbe_ctx* c, long long rows, double* loss) {
  const MlpState& m = c->mlp;
  MlpGradArgs r{};
  r.act = m.act; r.dz = m.dz; r.loss_part = m.loss_part;
  r.n_tiles = (int)((rows + kMlpTileRows - 1) / kMlpTileRows);
  r.loss = loss;
  r.grad = m.grad;
  r.p = m.params; r.m = m.m; r.v = m.v;
  r.pb = m.pb; r.pbt = m.pbt;
  return r;
}

qgbe_status check_weights(qgbe_ctx* c) {
  if (!c->mlp.ready || !c->mlp.has_weights) return fail(QGBE_ESTATE, "proposal weights not set");
  return QGBE_OK;
}

qgbe_status ensure_masses(qgbe_ctx* c) {
  if (c->masses_valid) return QGBE_OK;
  return compute_masses(c);
}

}  // namespace

qgbe_status qgbe::install_proposal_table(qgbe_ctx* c, int K) {
  const size_t rows = (size_t)c->nch * c->G.nodes;
  if (c->d_thr && c->K == K) return QGBE_OK;
  (void)hipFree(c->d_thr);
  (void)hipFree(c->d_mu);
  (void)hipFree(c->d_sigma);
  c->d_thr = nullptr; c->d_mu = nullptr; c->d_sigma = nullptr; c->K = 0;
  qgbe_status s = dev_alloc(c, &c->d_thr, std::max<size_t>(1, rows * K), "proposal thresholds");
  if (!s) s = dev_alloc(c, &c->d_mu, std::max<size_t>(1, rows * K * 5), "proposal locations");
  if (!s) s = dev_alloc(c, &c->d_sigma, std::max<size_t>(1, rows * K * 5), "proposal scales");
  if (!s && !c->d_mix_on) s = dev_alloc(c, &c->d_mix_on, std::max(1, c->nch), "channel samplers");
  if (s) return s;
  c->K = K;
  return QGBE_OK;
}

qgbe_status qgbe::reset_channel_samplers(qgbe_ctx* c) {
  HIP_TRY(hipMemsetAsync(c->d_mix_on, 1, std::max(1, c->nch), c->stream), "channel samplers");
  return QGBE_OK;
}

qgbe_status qgbe::ensure_proposal_features(qgbe_ctx* c) {
  qgbe_status s = QGBE_OK;
  if (!c->d_feat) s = dev_alloc(c, &c->d_feat, std::max<size_t>(1, (size_t)c->nch * c->G.nodes) * kMlpIn, "features");
  if (!s && !c->d_mass7) s = dev_alloc(c, &c->d_mass7, kSpecies, "mean masses");
  return s;
}

// Features of the current (cell-averaged) masses -> network -> table, on the
// context's stream.  Needs the weights, the table buffers (K = kMixK) and the
// feature buffers in place.
qgbe_status qgbe::refresh_proposal_table(qgbe_ctx* c) {
  const int rows = c->nch * c->G.nodes;
  HIP_TRY(launch_features(c->G, c->d_chans, c->nch, c->d_mass2, c->d_mass7, c->d_feat, c->stream), "features");
  HIP_TRY(launch_mlp_table(c->d_feat, rows, c->mlp.pb, c->mlp.params, c->table_alpha, c->d_thr, c->d_mu, c->d_sigma,
                           c->stream), "proposal table");
  return QGBE_OK;
}

extern "C" {

qgbe_status qgbe_set_proposal_table(qgbe_ctx* c, int32_t K, const uint32_t* thr, const float* mu, const float* sigma,
                                    int32_t on_device) {
  if (!c || !thr || !mu || !sigma) return fail(QGBE_EINVAL, "NULL argument");
  if (K < 1 || K > 16) return fail(QGBE_EINVAL, "K must be in 1..16");
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  qgbe_status s = install_proposal_table(c, K);
  if (s) return s;
  c->table_net = false;
  s = reset_channel_samplers(c);
  if (s) return s;
  const size_t rows = (size_t)c->nch * c->G.nodes;
  const hipMemcpyKind kind = on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
  HIP_TRY(hipMemcpyAsync(c->d_thr, thr, rows * K * sizeof(uint32_t), kind, c->stream), "copy thresholds");
  HIP_TRY(hipMemcpyAsync(c->d_mu, mu, rows * K * 5 * sizeof(float), kind, c->stream), "copy locations");
  HIP_TRY(hipMemcpyAsync(c->d_sigma, sigma, rows * K * 5 * sizeof(float), kind, c->stream), "copy scales");
  HIP_TRY(hipStreamSynchronize(c->stream), "synchronise");
  return QGBE_OK;
}

qgbe_status qgbe_get_proposal_table(qgbe_ctx* c, int32_t* K, uint32_t* thr, float* mu, float* sigma) {
  if (!c || !K) return fail(QGBE_EINVAL, "NULL argument");
  if (!c->K) return fail(QGBE_ESTATE, "no proposal table installed");
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  *K = c->K;
  const size_t rows = (size_t)c->nch * c->G.nodes;
  if (thr) HIP_TRY(hipMemcpyAsync(thr, c->d_thr, rows * c->K * sizeof(uint32_t), hipMemcpyDeviceToHost, c->stream), "copy");
  if (mu) HIP_TRY(hipMemcpyAsync(mu, c->d_mu, rows * c->K * 5 * sizeof(float), hipMemcpyDeviceToHost, c->stream), "copy");
  if (sigma)
    HIP_TRY(hipMemcpyAsync(sigma, c->d_sigma, rows * c->K * 5 * sizeof(float), hipMemcpyDeviceToHost, c->stream), "copy");
  HIP_TRY(hipStreamSynchronize(c->stream), "synchronise");
  return QGBE_OK;
}

qgbe_status qgbe_proposal_set_weights(qgbe_ctx* c, const float* w, int64_t n) {
  if (!c || !w) return fail(QGBE_EINVAL, "NULL argument");
  if (n != kMlpParams) return fail(QGBE_EINVAL, "weight count must be QGBE_MLP_PARAMS");
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  qgbe_status s = mlp_ensure(c);
  if (s) return s;
  MlpState& m = c->mlp;
  HIP_TRY(hipMemcpyAsync(m.params, w, kMlpParams * sizeof(float), hipMemcpyHostToDevice, c->stream), "copy weights");
  HIP_TRY(launch_refresh_weights(m.params, m.pb, m.pbt, c->stream), "bf16 weights");
  HIP_TRY(hipMemsetAsync(m.m, 0, kMlpParams * sizeof(float), c->stream), "zero m");
  HIP_TRY(hipMemsetAsync(m.v, 0, kMlpParams * sizeof(float), c->stream), "zero v");
  HIP_TRY(hipStreamSynchronize(c->stream), "synchronise");
  m.adam_t = 0;
  m.has_weights = true;
  return QGBE_OK;
}

qgbe_status qgbe_proposal_get_weights(qgbe_ctx* c, float* w, int64_t n) {
  if (!c || !w) return fail(QGBE_EINVAL, "NULL argument");
  if (n != kMlpParams) return fail(QGBE_EINVAL, "weight count must be QGBE_MLP_PARAMS");
  qgbe_status s = check_weights(c);
  if (s) return s;
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  HIP_TRY(hipMemcpyAsync(w, c->mlp.params, kMlpParams * sizeof(float), hipMemcpyDeviceToHost, c->stream), "copy");
  HIP_TRY(hipStreamSynchronize(c->stream), "synchronise");
  return QGBE_OK;
}

qgbe_status qgbe_mlp_forward(qgbe_ctx* c, const float* X, int64_t rows, float* Y, int32_t on_device) {
  if (!c || !X || !Y) return fail(QGBE_EINVAL, "NULL argument");
  if (rows < 0) return fail(QGBE_EINVAL, "rows must be >= 0");
  qgbe_status s = check_weights(c);
  if (s) return s;
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  MlpState& m = c->mlp;
  // device rows in place, unless X and Y overlap: a tile would write what another has yet to read
  const bool overlap = X < Y + rows * kMlpOut && Y < X + rows * kMlpIn;
  const bool staged = !on_device || overlap;
  const hipMemcpyKind in = on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
  const hipMemcpyKind out = on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost;
  if (!staged) {
    MlpTileArgs g = tile_args(c, rows, X, kMlpIn, nullptr, 0, nullptr);
    g.Y = Y;
    HIP_TRY(launch_mlp_forward(g, c->stream), "forward");
  }
  for (int64_t r0 = 0; staged && r0 < rows; r0 += kBatch) {
    const int nr = (int)std::min<int64_t>(kBatch, rows - r0);
    HIP_TRY(hipMemcpyAsync(m.X, X + r0 * kMlpIn, (size_t)nr * kMlpIn * sizeof(float), in, c->stream), "copy X");
    MlpTileArgs g = tile_args(c, nr, m.X, kMlpIn, nullptr, 0, nullptr);
    g.Y = m.Y;
    HIP_TRY(launch_mlp_forward(g, c->stream), "forward");
    HIP_TRY(hipMemcpyAsync(Y + r0 * kMlpOut, m.Y, (size_t)nr * kMlpOut * sizeof(float), out, c->stream), "copy Y");
  }
  HIP_TRY(hipStreamSynchronize(c->stream), "synchronise");
  return QGBE_OK;
}

qgbe_status qgbe_mlp_loss_grad(qgbe_ctx* c, const float* X, const float* yw, int64_t rows, float* grad, double* loss,
                               int32_t on_device) {
  if (!c || !X || !yw || !grad || !loss) return fail(QGBE_EINVAL, "NULL argument");
  if (rows < 1 || rows > kBatch) return fail(QGBE_EINVAL, "rows must be in 1..QGBE_MLP_BATCH");
  qgbe_status s = check_weights(c);
  if (s) return s;
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  MlpState& m = c->mlp;
  if (!on_device) {
    HIP_TRY(hipMemcpyAsync(m.X, X, (size_t)rows * kMlpIn * sizeof(float), hipMemcpyHostToDevice, c->stream), "copy X");
    HIP_TRY(hipMemcpyAsync(m.yw, yw, (size_t)rows * (kMixD + 1) * sizeof(float), hipMemcpyHostToDevice, c->stream),
            "copy yw");
    X = m.X;
    yw = m.yw;
  }
  HIP_TRY(launch_fill(m.scalars, 0.0, 1, c->stream), "zero loss");
  HIP_TRY(launch_weight_sums(yw + kMixD, kMixD + 1, nullptr, rows, (int)rows, m.scalars + 1, c->stream), "weight sum");
  MlpTileArgs g = tile_args(c, rows, X, kMlpIn, yw, kMixD + 1, nullptr);
  g.wsum = m.scalars + 1;
  HIP_TRY(launch_mlp_grad(g, c->stream), "gradient");
  MlpGradArgs r = grad_args(c, rows, m.scalars);
  if (on_device) r.grad = grad;
  HIP_TRY(launch_weight_grad(r, c->stream), "gradient sum");
  if (!on_device)
    HIP_TRY(hipMemcpyAsync(grad, m.grad, kMlpParams * sizeof(float), hipMemcpyDeviceToHost, c->stream), "copy grad");
  HIP_TRY(hipMemcpyAsync(loss, m.scalars, sizeof(double), hipMemcpyDeviceToHost, c->stream), "copy loss");
  HIP_TRY(hipStreamSynchronize(c->stream), "synchronise");
  return QGBE_OK;
}

qgbe_status qgbe_proposal_features(qgbe_ctx* c, float* X, int32_t on_device) {
  if (!c || !X) return fail(QGBE_EINVAL, "NULL argument");
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  qgbe_status s = ensure_masses(c);
  if (!s) s = ensure_proposal_features(c);
  if (s) return s;
  const size_t rows = (size_t)c->nch * c->G.nodes;
  HIP_TRY(launch_features(c->G, c->d_chans, c->nch, c->d_mass2, c->d_mass7, c->d_feat, c->stream), "features");
  HIP_TRY(hipMemcpyAsync(X, c->d_feat, rows * kMlpIn * sizeof(float),
                         on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, c->stream), "copy features");
  HIP_TRY(hipStreamSynchronize(c->stream), "synchronise");
  return QGBE_OK;
}

qgbe_status qgbe_record_samples(qgbe_ctx* c, int32_t n_per_item, int64_t item_stride, float* rows, int64_t max_rows,
                                int64_t* n_rows, int32_t on_device) {
  if (!c || !rows || !n_rows) return fail(QGBE_EINVAL, "NULL argument");
  if (n_per_item < 1 || item_stride < 1) return fail(QGBE_EINVAL, "n_per_item and item_stride must be >= 1");
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  const long long items = (long long)c->G.cells * c->nch * c->G.nodes;
  const long long n_sel = (items + item_stride - 1) / item_stride;
  const long long total = n_sel * n_per_item;
  *n_rows = total;
  if (total > max_rows) return fail(QGBE_EINVAL, "rows buffer too small");
  if (total == 0) return QGBE_OK;
  qgbe_status s = ensure_masses(c);
  if (s) return s;
  float* dst = rows;
  if (!on_device) HIP_TRY(hipMalloc(&dst, (size_t)total * kRecordWidth * sizeof(float)), "record scratch");
  CollideArgs a = base_args(c, n_per_item, nullptr, nullptr, nullptr);
  hipError_t e = launch_record(a, n_per_item, item_stride, n_sel, dst, c->stream);
  if (e == hipSuccess && !on_device)
    e = hipMemcpyAsync(rows, dst, (size_t)total * kRecordWidth * sizeof(float), hipMemcpyDeviceToHost, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  if (!on_device) (void)hipFree(dst);
  if (e != hipSuccess) return hip_fail(e, "record samples");
  return QGBE_OK;
}

qgbe_status qgbe_proposal_build_table(qgbe_ctx* c, float alpha) {
  if (!c) return fail(QGBE_EINVAL, "NULL context");
  if (!(alpha > 0.0f && alpha < 1.0f)) return fail(QGBE_EINVAL, "alpha must be in (0,1)");
  qgbe_status s = check_weights(c);
  if (s) return s;
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  s = ensure_masses(c);
  if (!s) s = install_proposal_table(c, kMixK);
  if (!s) s = ensure_proposal_features(c);
  if (s) return s;
  c->table_alpha = alpha;
  c->table_net = true;
  s = reset_channel_samplers(c);
  if (!s) s = refresh_proposal_table(c);
  if (s) {
    c->table_net = false;
    return s;
  }
  HIP_TRY(hipStreamSynchronize(c->stream), "build proposal table");
  return QGBE_OK;
}

qgbe_status qgbe_set_channel_samplers(qgbe_ctx* c, const uint8_t* use_learned) {
  if (!c || !use_learned) return fail(QGBE_EINVAL, "NULL argument");
  if (!c->K) return fail(QGBE_ESTATE, "no proposal table installed");
  std::vector<uint8_t> v(std::max(1, c->nch), 1);
  for (int i = 0; i < c->nch; ++i) {
    if (use_learned[i] > 1) return fail(QGBE_EINVAL, "channel sampler flags must be 0 or 1");
    v[i] = use_learned[i];
  }
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  HIP_TRY(hipMemcpyAsync(c->d_mix_on, v.data(), v.size(), hipMemcpyHostToDevice, c->stream), "copy flags");
  HIP_TRY(hipStreamSynchronize(c->stream), "synchronise");
  return QGBE_OK;
}

qgbe_status qgbe_get_channel_samplers(qgbe_ctx* c, uint8_t* use_learned) {
  if (!c || !use_learned) return fail(QGBE_EINVAL, "NULL argument");
  if (!c->K) return fail(QGBE_ESTATE, "no proposal table installed");
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  HIP_TRY(hipMemcpyAsync(use_learned, c->d_mix_on, c->nch, hipMemcpyDeviceToHost, c->stream), "copy flags");
  HIP_TRY(hipStreamSynchronize(c->stream), "synchronise");
  return QGBE_OK;
}

qgbe_status qgbe_proposal_judge(qgbe_ctx* c, int32_t n_pilot, int32_t n_reps, uint8_t* use_learned,
                                double* ratio) {
  if (!c) return fail(QGBE_EINVAL, "NULL context");
  if (n_pilot < 2 || n_reps < 1) return fail(QGBE_EINVAL, "n_pilot >= 2 and n_reps >= 1 required");
  if (!c->K) return fail(QGBE_ESTATE, "no proposal table installed");
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  const int nch = std::max(1, c->nch);
  std::vector<double> var[2], h((size_t)kStripes * nch);
  double t_ms[2] = {0.0, 0.0};
  const uint32_t saved_step = c->step;
  qgbe_status s = reset_channel_samplers(c);
  for (int l = 0; l < 2 && !s; ++l) {
    var[l].assign(nch, 0.0);
    for (int r = 0; r < n_reps && !s; ++r) {
      // pilot draws use their own key range, apart from the run's steps
      c->step = 0xF0000000u + (uint32_t)r;
      qgbe_stats st;
      s = qgbe_collision_term_ex(c, n_pilot, l ? QGBE_SAMPLER_LEARNED : QGBE_SAMPLER_UNIFORM, c->d_A, 1, nullptr, &st);
      if (s) break;
      t_ms[l] += st.t_collide_ms;
      hipError_t e = hipMemcpyAsync(h.data(), c->d_chan_var, h.size() * sizeof(double), hipMemcpyDeviceToHost,
                                    c->stream);
      if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
      if (e != hipSuccess) { s = hip_fail(e, "copy channel variances"); break; }
      for (int k = 0; k < kStripes; ++k)  // the stripes in order
        for (int ci = 0; ci < nch; ++ci) var[l][ci] += h[(size_t)k * nch + ci];
    }
  }
  c->step = saved_step;
  if (s) return s;
  // per channel: pooled variance of the item estimates x the sampler's pilot time
  std::vector<uint8_t> flags(nch, 1);
  for (int ci = 0; ci < c->nch; ++ci) {
    const double cost_u = var[0][ci] * t_ms[0], cost_l = var[1][ci] * t_ms[1];
    flags[ci] = (cost_u > 0.0 && cost_l < cost_u) ? 1 : 0;
    if (ratio) ratio[ci] = cost_u > 0.0 ? cost_l / cost_u : (cost_l > 0.0 ? INFINITY : 1.0);
  }
  HIP_TRY(hipMemcpyAsync(c->d_mix_on, flags.data(), flags.size(), hipMemcpyHostToDevice, c->stream), "copy flags");
  HIP_TRY(hipStreamSynchronize(c->stream), "synchronise");
  if (use_learned) std::memcpy(use_learned, flags.data(), c->nch);
  return QGBE_OK;
}

qgbe_status qgbe_train_proposal(qgbe_ctx* c, const float* rows, int64_t n, const qgbe_train_cfg* cfg,
                                double* epoch_loss, int32_t on_device) {
  if (!c || !rows || !cfg) return fail(QGBE_EINVAL, "NULL argument");
  if (n < 1) return fail(QGBE_EINVAL, "no training rows");
  if (cfg->epochs < 1 || cfg->batch < 1 || cfg->batch > kBatch) return fail(QGBE_EINVAL, "bad epochs or batch");
  if (!(cfg->lr > 0.0f) || !(cfg->lr_final >= 0.0f)) return fail(QGBE_EINVAL, "bad learning rate");
  if (!(cfg->alpha > 0.0f && cfg->alpha < 1.0f)) return fail(QGBE_EINVAL, "alpha must be in (0,1)");
  qgbe_status s = check_weights(c);
  if (s) return s;
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  MlpState& m = c->mlp;
  const float* d_rows = rows;
  float* owned = nullptr;
  if (!on_device) {
    HIP_TRY(hipMalloc(&owned, (size_t)n * kRecordWidth * sizeof(float)), "rows scratch");
    HIP_TRY(hipMemcpyAsync(owned, rows, (size_t)n * kRecordWidth * sizeof(float), hipMemcpyHostToDevice, c->stream),
            "copy rows");
    d_rows = owned;
  }
  // Per epoch on the device: the row order (the host draws the next one while
  // the GPU works on this one), the weight sum of every batch, and the loss.
  const int steps_per_epoch = (int)((n + cfg->batch - 1) / cfg->batch);
  const size_t perm_b = ((size_t)n * sizeof(int) + 255) & ~size_t(255);
  const size_t sums_b = ((size_t)steps_per_epoch * sizeof(double) + 255) & ~size_t(255);
  char* scratch = nullptr;
  if (hipMalloc(&scratch, 2 * (perm_b + sums_b) + (size_t)cfg->epochs * sizeof(double)) != hipSuccess) {
    if (owned) (void)hipFree(owned);
    return fail(QGBE_ENOMEM, "training scratch");
  }
  double* d_loss = (double*)(scratch + 2 * (perm_b + sums_b));
  std::mt19937_64 rng(cfg->seed);
  std::vector<int> perm((size_t)n);
  std::iota(perm.begin(), perm.end(), 0);
  std::vector<int> sent[2];  // the orders on their way; one is written again when its copy has ended
  hipEvent_t copied[2] = {nullptr, nullptr};
  const long long total_steps = (long long)steps_per_epoch * cfg->epochs;
  long long step = 0;
  hipError_t e = launch_fill(d_loss, 0.0, cfg->epochs, c->stream);
  for (int i = 0; i < 2 && e == hipSuccess; ++i) e = hipEventCreateWithFlags(&copied[i], hipEventDisableTiming);
  for (int ep = 0; ep < cfg->epochs && e == hipSuccess; ++ep) {
    std::shuffle(perm.begin(), perm.end(), rng);
    int* d_perm = (int*)(scratch + (ep & 1) * (perm_b + sums_b));
    double* d_sums = (double*)(scratch + (ep & 1) * (perm_b + sums_b) + perm_b);
    if (ep >= 2) e = hipEventSynchronize(copied[ep & 1]);
    if (e != hipSuccess) break;
    sent[ep & 1] = perm;
    e = hipMemcpyAsync(d_perm, sent[ep & 1].data(), (size_t)n * sizeof(int), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = hipEventRecord(copied[ep & 1], c->stream);
    if (e == hipSuccess)
      e = launch_weight_sums(d_rows + kMlpIn + kMixD, kRecordWidth, d_perm, n, cfg->batch, d_sums, c->stream);
    for (int b = 0; b < steps_per_epoch && e == hipSuccess; ++b, ++step) {
      const long long r0 = (long long)b * cfg->batch;
      const int nr = (int)std::min<int64_t>(cfg->batch, n - r0);
      MlpTileArgs g = tile_args(c, nr, d_rows, kRecordWidth, d_rows + kMlpIn, kRecordWidth, d_perm + r0);
      g.wsum = d_sums + b;
      e = launch_mlp_grad(g, c->stream);
      if (e != hipSuccess) break;
      const double frac = total_steps > 1 ? (double)step / (double)(total_steps - 1) : 1.0;
      m.adam_t += 1;
      MlpGradArgs r = grad_args(c, nr, d_loss + ep);
      r.adam = 1;
      r.lr = (float)(cfg->lr_final + 0.5 * (cfg->lr - cfg->lr_final) * (1.0 + std::cos(kPi * frac)));
      r.b1 = 0.9f; r.b2 = 0.999f; r.eps = 1e-8f;
      r.c1 = 1.f - powf(r.b1, (float)m.adam_t);
      r.c2 = 1.f - powf(r.b2, (float)m.adam_t);
      e = launch_weight_grad(r, c->stream);
    }
  }
  if (e == hipSuccess && epoch_loss) {
    e = hipMemcpyAsync(epoch_loss, d_loss, (size_t)cfg->epochs * sizeof(double), hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    for (int ep = 0; ep < cfg->epochs; ++ep) epoch_loss[ep] /= steps_per_epoch;
  }
  // wait for the queued work before the scratch buffers go (also after an error)
  const hipError_t e_sync = hipStreamSynchronize(c->stream);
  if (e == hipSuccess) e = e_sync;
  for (hipEvent_t ev : copied)
    if (ev) (void)hipEventDestroy(ev);
  (void)hipFree(scratch);
  if (owned) (void)hipFree(owned);
  if (s) return s;
  if (e != hipSuccess) return hip_fail(e, "train proposal");
  return qgbe_proposal_build_table(c, cfg->alpha);
}

}  // extern "C"
