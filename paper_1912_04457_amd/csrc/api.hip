// C ABI of libqgbe: context management, validation and launch logic.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "context.h"

using namespace qgbe;

namespace {
thread_local std::string g_error;
}  // namespace

namespace qgbe {

qgbe_status fail(qgbe_status s, const std::string& msg) {
  g_error = msg;
  return s;
}

qgbe_status hip_fail(hipError_t e, const char* what) {
  return fail(e == hipErrorOutOfMemory ? QGBE_ENOMEM : QGBE_EDEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

size_t field_len(const qgbe_ctx* c) { return (size_t)kSpecies * c->G.cells * c->G.nodes; }

}  // namespace qgbe

namespace qgbe {

namespace {

TermStart mass_args(qgbe_ctx* c) {
  TermStart t{};
  t.G = c->G;
  t.f = c->d_f;
  t.lag = c->has_lag ? c->d_lag : nullptr;
  if (c->d.mass_mode == QGBE_MASS_CONSTANT)
    for (int s = 0; s < kSpecies; ++s) t.constant.v[s] = c->d.const_mass2[s];
  else
    t.part = c->d_mass_part;
  t.mass2 = c->d_mass2;
  t.done = c->d_done;
  return t;
}

}  // namespace

qgbe_status compute_masses(qgbe_ctx* c) {
  HIP_TRY(launch_term_start(mass_args(c), c->stream), "masses");
  c->masses_valid = true;
  return QGBE_OK;
}

qgbe_status start_term(qgbe_ctx* c, int sampler, double* A, bool f32) {
  TermStart t = mass_args(c);
  t.A = A;
  t.count = c->d_count;
  t.n_count = kStripes;
  t.totals = c->d_mc;  // and the channel variances behind it
  t.n_totals = kStripes * (2 + std::max(1, c->nch));
  const bool cm = sampler == QGBE_SAMPLER_UNIFORM || sampler == QGBE_SAMPLER_LEARNED;
  if (c->d.precision == QGBE_FP32 && cm) {
    if (f32) t.f32 = c->d_f32;
    if (c->need_quads[sampler == QGBE_SAMPLER_LEARNED ? 1 : 0]) t.quads = c->d_f32q;
  }
  HIP_TRY(launch_term_start(t, c->stream), "start of the collision term");
  c->masses_valid = true;
  return QGBE_OK;
}

CollideArgs base_args(qgbe_ctx* c, int n_samples, double* A, double* scale, double* items) {
  CollideArgs a{};
  a.G = c->G;
  a.chans = c->d_chans;
  a.n_channels = c->nch;
  a.n_samples = n_samples;
  a.symmetric = c->d.symmetric;
  a.key0 = (uint32_t)c->d.seed;
  a.key1 = (uint32_t)(c->d.seed >> 32) + c->step;
  a.f64 = c->d_f;
  a.f32 = c->d_f32;
  a.mass2 = c->d_mass2;
  a.win_lo = 0;
  a.win_n = c->G.nodes;
  a.msq_mask = c->msq_mask;
  a.msq = c->d_msq;
  a.A = A;
  a.scale = scale;
  a.items = items;
  a.n_accepted = c->d_count;
  a.mc_acc = c->d_mc;
  a.chan_var = c->d_chan_var;
  a.mix_K = c->K;
  a.mix_thr = c->d_thr;
  a.mix_mu = c->d_mu;
  a.mix_sigma = c->d_sigma;
  a.mix_on = c->d_mix_on;
  return a;
}


qgbe_status validate(const qgbe_grid_desc* d) {
  if (!d) return fail(QGBE_EINVAL, "descriptor is NULL");
  long long cells = 1, nodes = 1;
  for (int a = 0; a < 3; ++a) {
    if (d->n_x[a] < 1) return fail(QGBE_EINVAL, "n_x must be >= 1");
    if (d->n_p[a] < 2) return fail(QGBE_EINVAL, "n_p must be >= 2 on every axis");
    if (!(d->x_half[a] > 0.0) || !std::isfinite(d->x_half[a])) return fail(QGBE_EINVAL, "x_half must be > 0");
    if (!(d->p_half[a] > 0.0) || !std::isfinite(d->p_half[a])) return fail(QGBE_EINVAL, "p_half must be > 0");
    cells *= d->n_x[a];
    nodes *= d->n_p[a];
  }
  if (cells * nodes * kSpecies > (1LL << 31)) return fail(QGBE_EINVAL, "grid too large for 32-bit indexing");
  if (nodes > (1 << 23)) return fail(QGBE_EINVAL, "too many momentum nodes");
  if ((d->species_mask & ~0x7Fu) || d->species_mask == 0) return fail(QGBE_EINVAL, "species_mask must be in 1..0x7F");
  if (d->row_mask & ~0x7Fu) return fail(QGBE_EINVAL, "row_mask must be in 0..0x7F");
  if (!(d->alpha_s > 0.0) || !std::isfinite(d->alpha_s)) return fail(QGBE_EINVAL, "alpha_s must be > 0");
  if (d->precision != QGBE_FP64 && d->precision != QGBE_FP32) return fail(QGBE_EINVAL, "bad precision");
  if (d->symmetric != 0 && d->symmetric != 1) return fail(QGBE_EINVAL, "symmetric must be 0 or 1");
  if (d->drift != QGBE_DRIFT_UPWIND && d->drift != QGBE_DRIFT_CENTRAL) return fail(QGBE_EINVAL, "bad drift scheme");
  if (d->mass_mode != QGBE_MASS_DYNAMIC && d->mass_mode != QGBE_MASS_CONSTANT) return fail(QGBE_EINVAL, "bad mass_mode");
  if (d->mass_mode == QGBE_MASS_CONSTANT)
    for (int s = 0; s < kSpecies; ++s)
      if (!(d->const_mass2[s] >= 0.0) || !std::isfinite(d->const_mass2[s]))
        return fail(QGBE_EINVAL, "const_mass2 must be finite and >= 0");
  return QGBE_OK;
}

void make_grid(const qgbe_grid_desc* d, Grid& G) {
  G.cells = 1;
  G.nodes = 1;
  for (int a = 0; a < 3; ++a) {
    G.nx[a] = d->n_x[a];
    G.np[a] = d->n_p[a];
    G.xh[a] = d->x_half[a];
    G.ph[a] = d->p_half[a];
    G.dx[a] = 2.0 * d->x_half[a] / d->n_x[a];
    G.dp[a] = 2.0 * d->p_half[a] / d->n_p[a];
    G.inv_dp[a] = 1.0 / G.dp[a];
    G.pc[a] = G.ph[a] * G.inv_dp[a] - 0.5;
    G.cells *= d->n_x[a];
    G.nodes *= d->n_p[a];
  }
  G.oy = G.np[2];
  G.ox = G.np[1] * G.np[2];
  G.Vp = 8.0 * d->p_half[0] * d->p_half[1] * d->p_half[2];
  G.g2 = 4.0 * kPi * d->alpha_s;
  G.g4 = G.g2 * G.g2;
  G.species_mask = d->species_mask;
}

bool several_launches(const qgbe_ctx* c, const Group& g, int l) {
  return c->d.symmetric && (g.lds_acc[l] < g.nslot || g.win[l] < c->G.nodes);
}

// LDS plan of a group for sampler l within a budget: FP64 accumulators first
// (they replace global atomics), then FP32 f tiles in what is left; tiles that
// do not fit are read from global memory.
static void plan_lds(const qgbe_ctx* c, Group& g, int l, size_t budget, bool long_form) {
  const size_t acc_b = (size_t)c->G.nodes * sizeof(double), tile_b = (size_t)c->G.nodes * sizeof(float);
  g.budget[l] = budget;
  g.long_form[l] = long_form;
  g.win[l] = c->G.nodes;
  if (c->d.symmetric && budget < acc_b) {
    // one slot's FP64 accumulators exceed LDS: node windows, one launch
    // per window holding every slot's accumulators for that window, the
    // same samples in each; f from the quads
    const int fit = (int)(budget / (sizeof(double) * g.nslot));
    const int n_win = (c->G.nodes + fit - 1) / fit;
    g.win[l] = (c->G.nodes + n_win - 1) / n_win;
    g.lds_acc[l] = g.nslot;
    g.lds_tiles[l] = 0;
    return;
  }
  g.lds_acc[l] = c->d.symmetric ? (int)std::min<size_t>(g.nslot, budget / acc_b) : 0;
  // FP64 reads f from the FP64 field
  g.lds_tiles[l] = c->d.precision == QGBE_FP32 && l < 2
                       ? (int)std::min<size_t>(g.nslot, (budget - g.lds_acc[l] * acc_b) / tile_b) : 0;
}

// The plans of every group.  The short-item form's tables take 6 KB that the
// long form leaves to the accumulators: where they are what a single launch
// lacks, the long form runs whatever the items (gluons, 27x27x28 nodes x 512 and
// 2048 samples: 0.49 and 1.83 ms recorded, 0.26 and 0.84 in one launch; learned
// sampler, 26x27x27: 0.86 and 3.67, 0.50 and 1.80).
void plan_groups(qgbe_ctx* c, bool long_form) {
  const size_t acc_b = (size_t)c->G.nodes * sizeof(double);
  const bool f32 = c->d.precision == QGBE_FP32;
  c->group_index.clear();
  c->groups.clear();
  for (std::vector<int>& m : c->match) m.clear();
  c->need_quads[0] = c->need_quads[1] = false;
  for (int nslot = 1; nslot <= 3; ++nslot) {
    Group g{};
    g.start = (int)c->group_index.size();
    g.nslot = nslot;
    for (int l = 0; l < 3; ++l) {
      const size_t* form = l == 0 ? c->lds.plain : c->lds.learned;
      plan_lds(c, g, l, l == 2 ? c->lds.roots : form[1], false);
      if (!f32 || l == 2) continue;
      Group h = g;
      plan_lds(c, h, l, form[0], true);
      if ((l == 0 && long_form) || (several_launches(c, g, l) && !several_launches(c, h, l))) g = h;
    }
    for (int i = 0; i < 2; ++i)
      if (c->d.symmetric && g.lds_acc[0] == nslot && g.win[0] == c->G.nodes && !(long_form && i))
        g.queue[i] = nslot * acc_b <= c->lds.queue[0][i] ? kRing
                     : nslot * acc_b <= c->lds.queue[1][i] && !long_form ? kTight : 0;
    for (int i = 0; i < c->nch; ++i)
      if (c->chans[i].nslot == nslot) c->group_index.push_back(i);
    g.count = (int)c->group_index.size() - g.start;
    if (g.count) {
      c->groups.push_back(g);
      for (int l = 0; l < 2; ++l) c->need_quads[l] = f32 && (c->need_quads[l] || g.lds_tiles[l] < nslot);
      c->need_quads[0] = f32 && (c->need_quads[0] || g.queue[0] || g.queue[1]);
    }
  }
  for (int l = 0; l < 3; ++l) {
    Replay& r = c->replay[l];
    r = {};
    for (const Group& g : c->groups)
      if (several_launches(c, g, l)) {
        if (!r.count) r.start = g.start;
        r.count += g.count;
      }
  }
  // The lists that go to the device do not depend on the grid: calls without a
  // context share them, and a captured one reads them at each replay.
  for (int gi = 0; gi < c->nch; ++gi)
    for (int p = 1; p < 4; ++p) c->match[c->chans[c->group_index[gi]].sp[p]].push_back(4 * gi + p);
  c->group_index.resize(kMaxGroupIndex, 0);
  for (int y = 0; y < kSpecies; ++y)
    std::copy(c->match[y].begin(), c->match[y].end(), c->group_index.begin() + kMatchAt + (size_t)y * kMaxMatches);
}

// Observed nodes per workgroup; acc: entries a workgroup zeroes and flushes.
static Chunking plan_evenly(const qgbe_ctx* c, long long nodes, long long pairs, long long acc, int n_samples, bool queue,
                            bool learned, bool long_form) {
  const int waves = collide_waves(queue);
  if (pairs >= c->n_cu && acc > 0) {
    // Enough (cell, channel) pairs to give every compute unit one: the nodes
    // of a pair are split over at most two workgroups per compute unit in all,
    // as each zeroes and flushes its accumulators (on the pure-gluon 16x16x1
    // grid: 4096 -> 512 workgroups, 71.0 -> 68.0 ms).  A chunk is a multiple
    // of the waves; a small one of a variant that hands nodes to its waves in
    // blocks, whole blocks for every wave (36 nodes in blocks of 4 would leave
    // 3 of 12 waves idle).  Large chunks keep the finer multiple: C2's two
    // chunks per cell of 4032 and 3968 nodes instead of 4008 and 3992 cost
    // 0.5% (compute units that ran two long ones).
    const long long per_pair = std::max(1LL, 2LL * c->n_cu / pairs);
    long long chunk = std::max<long long>(waves, (nodes + per_pair - 1) / per_pair);
    int nb = collide_node_block(queue);
    if (!long_form && collide_short(c->d.precision, learned, 1, n_samples))  // the largest block that leaves every wave 4 turns
      for (nb = kMaxNodeBlock; nb > 1 && chunk < 4LL * waves * nb; nb /= 2) {}
    const int unit = chunk < 16LL * waves * nb ? waves * nb : waves;
    chunk = (chunk + unit - 1) / unit * unit;
    chunk = std::min(chunk, (nodes + unit - 1) / unit * unit);
    return {(int)chunk, 1, nb};
  }
  // Fewer pairs than compute units, or (direct sums) no accumulators to pay for: 516
  // pairs as one workgroup each are 2.02 rounds that take three (20^3 nodes x 300
  // samples, FP64 direct 29.8 -> 22.7 ms).  A workgroup has its compute unit to
  // itself (LDS and registers), so their number is chosen near a multiple of
  // the compute units (up to eight rounds), and with few nodes per workgroup
  // several waves share a node.  The estimate, in sample iterations of a lone
  // wave (1.7 us): turns of the waves times (iterations per node plus 0.4
  // for its sums and partly filled batches, plus 0.8 per block of nodes for
  // their constants), a turn 1.3 or 1.75
  // times as long with two or three waves at work on a SIMD, plus the
  // workgroup's start and the accumulators it zeroes and flushes (450 take
  // about an iteration), in every round; nodes differ in how many samples
  // they accept, which unbalances one round by about a tenth.  (20^3 nodes of one gluon cell,
  // 512 samples: 167 workgroups without sharing 156 us, 256 with it 120.)
  const auto turn = [](long long active) { return active <= 0 ? 0.0 : active <= 4 ? 1.0 : active <= 8 ? 1.3 : 1.75; };
  Chunking best{0, 1, 1};
  double least = 0.0;
  for (int rounds = 1; rounds <= 8; ++rounds) {
    const long long want = pairs >= c->n_cu ? rounds : std::max(1LL, rounds * c->n_cu / pairs);
    const long long even = (nodes + want - 1) / want;
    for (int split = 1; split <= waves; ++split) {
      if (waves % split || (long_form && split > 1)) continue;
      const bool is_short = !long_form && collide_short(c->d.precision, learned, split, n_samples);
      for (long long unit = is_short ? kMaxNodeBlock : collide_node_block(queue); unit >= 1; unit /= 2) {
        const long long group = unit * (waves / split);  // nodes the workgroup takes at a time
        for (const long long step : {is_short ? 1LL : unit, group}) {
          const long long chunk = std::min((even + step - 1) / step * step,
                                           is_short ? nodes : (nodes + unit - 1) / unit * unit);
          if (split > 1 && chunk > kSplitNodes) continue;
          const double iters = (double)((n_samples + 64LL * split - 1) / (64LL * split)) + 0.4 + 0.8 / (double)unit;
          const long long units = (chunk + unit - 1) / unit, per_turn = waves / split;
          const double busy = (double)unit * iters * ((double)(units / per_turn) * turn(per_turn * split) +
                                                      turn(units % per_turn * split));
          const long long wgs = pairs * ((nodes + chunk - 1) / chunk);
          const double r = (double)((wgs + c->n_cu - 1) / c->n_cu);
          const double cost = r * (busy * (1.0 + 0.1 / r) + 3.0 + (double)acc / 450.0);
          if (!best.chunk || cost < least) {
            best = {(int)chunk, split, (int)unit};
            least = cost;
          }
        }
        if (!is_short) break;
      }
    }
  }
  return best;
}

// The same; the short-item form counts the accepted samples of a wave's nodes in
// 32 bits (two per sample with the root samplers), so its workgroups take fewer
// nodes of very many samples, which cost them nothing.
Chunking plan_chunks(const qgbe_ctx* c, long long nodes, long long pairs, long long acc, int n_samples, bool queue,
                     bool learned, bool long_form) {
  Chunking ck = plan_evenly(c, nodes, pairs, acc, n_samples, queue, learned, long_form);
  if (!long_form && collide_short(c->d.precision, learned, ck.split, n_samples))
    ck.chunk = (int)std::min<long long>(ck.chunk, std::max(1LL, ((1LL << 30) - 1) / n_samples));
  return ck;
}

// Record buffers: for 128 samples per item (and an eighth more, as whole
// chunks of nodes count), between kRecMin and kRecMax samples (7 species at 30^3 x 128: 2 M samples 13.3 ms, 4 M 12.1, 8 M
// 9.6, 16 M 9.2, 64 M 8.8; 52 B a sample, 92 B in FP64).  They take at most a
// sixteenth of the memory that is free, so that contexts that hold them leave
// what a caller's own allocations had; without them every launch draws its
// samples again, or adds its deposits with global atomics.  A context asks once.
constexpr long long kRecMin = 1LL << 21, kRecMax = 1LL << 23, kRecLeast = 1LL << 19;

size_t record_tile(const qgbe_ctx* c, bool roots) {
  return roots || c->d.precision == QGBE_FP64 ? collide_f64_record_tile() : collide_f32_record_tile();
}

void carve_records(qgbe_ctx* c, unsigned char* p, size_t bytes) {
  const size_t wgs = 1 << 16, counts = wgs * sizeof(uint32_t);
  if (bytes < counts + (kRecLeast / 64) * record_tile(c, false)) return;
  c->d_rec = p;
  c->rec.count = (uint32_t*)p;
  c->rec.tiles = p + counts;
  c->rec_wgs = (long long)wgs;
  c->rec_bytes = bytes - counts;
}

// Bytes of a context's record tiles.
size_t record_buffer_bytes(const qgbe_ctx* c) {
  const long long items = (long long)c->G.cells * c->G.nodes *
                          std::max({c->replay[0].count, c->replay[1].count, c->replay[2].count});
  return (size_t)(std::max(kRecMin, std::min(kRecMax, items * 144)) + 63) / 64 * record_tile(c, false);
}

void alloc_records(qgbe_ctx* c) {
  c->rec_asked = true;
  const size_t bytes = record_buffer_bytes(c) + ((size_t)sizeof(uint32_t) << 16);
  // an allocation takes nothing from a capture that another stream or thread is in
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) {
    (void)hipGetLastError();
    return;
  }
  size_t free = 0, total = 0;
  void* p = nullptr;
  if (hipMemGetInfo(&free, &total) == hipSuccess && bytes <= free / 16 && hipMalloc(&p, bytes) == hipSuccess) {
    c->ws += bytes;
    carve_records(c, static_cast<unsigned char*>(p), bytes);
  }
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  (void)hipGetLastError();  // a refusal is none of the caller's
}

// Samples whose deposits buffers of these bytes hold for a sampler (the root
// samplers' records are FP64, up to two to a sample).
long long record_capacity(const qgbe_ctx* c, int l, size_t bytes) {
  return 64 * (long long)(bytes / record_tile(c, l == 2)) / (l == 2 ? 2 : 1);
}

int replay_windows(const qgbe_ctx* c) {
  const long long lds_nodes = (long long)(c->lds.replay / sizeof(double));
  return (int)((c->G.nodes + lds_nodes - 1) / lds_nodes);
}

// How the channels whose accumulators take more than one launch deposit in this
// call, estimated in microseconds per million samples: 26 to draw them (whole
// iterations of 64, and half a one for the item; 60 with the learned sampler in
// FP64), in every launch that draws them again, and 45 for such a launch; 14 to
// record and replay them in up to two windows and 13 for each window more, and
// 40 for a batch; global FP64 atomics 520 (20 G/s; 340 with the root samplers, which
// accept fewer).  Drawing again ends early: gluons at 30^3, 128 samples, 216 us
// and 156 recorded; only in the few MB of the call without allocation it wins
// there (1000 samples: 25 batches and 2.1 ms instead of 1.3).  Records end where
// the windows are many, global atomics (FP64) take over: one cell of gluons, 64
// samples, drawn again / recorded / global atomics, in ms:
//           48^3               64^3              80^3               96^3               128^3
//   uniform 1.58 / 0.79 / 4.2  8.6 / 2.8 / 9.4   31 / 6.3 / 18.4    131 / 30.9 / 31.9  1206 / 138 / 75
//   roots   2.5 / 0.76 / 2.8   12.9 / 2.5 / 6.3  49.7 / 5.5 / 12.4  163 / 29.7 / 21.3  1187 / 174 / 51
//   learned 4.9 / 1.2 / 4.0    25.5 / 3.9 / 9.1  104 / 8.2 / 17.8   336 / 33.5 / 30.7
// (512 samples at 96^3, uniform: 1037 / 398 / 255).  FP32 has no global form: its
// grids took the windows before, too (96^3: 98.5 / 28.0).
DepositRoute deposit_route(const qgbe_ctx* c, int l, int n_samples, bool scale, long long capacity) {
  if (!c->replay[l].count) return DepositRoute::kAgain;
  const double per_sample = 1e-6 * (double)c->G.cells * c->G.nodes, n = c->replay[l].count;
  const bool f64 = l == 2 || c->d.precision == QGBE_FP64;
  const double drawn = (l == 1 && f64 ? 60.0 : 26.0) * per_sample * (64.0 * ((n_samples + 63) / 64) + 32.0);
  const double samples = per_sample * n_samples * n;
  double again = 0.0;
  for (const Group& g : c->groups)
    if (several_launches(c, g, l)) {
      const int passes = (g.nslot + g.lds_acc[l] - 1) / g.lds_acc[l];
      const int windows = (c->G.nodes + g.win[l] - 1) / g.win[l];
      again += passes * windows * (drawn * g.count + 45.0);
    }
  DepositRoute best = DepositRoute::kAgain;
  double least = again;
  const auto offer = [&](DepositRoute r, double t) {
    if (t < least) {
      best = r;
      least = t;
    }
  };
  if (!scale && n_samples <= capacity)
    offer(DepositRoute::kRecord, drawn * n + (14.0 + 13.0 * std::max(0, replay_windows(c) - 2)) * samples +
                                     40.0 * std::ceil(1e6 * samples / (double)capacity));
  if (f64) offer(DepositRoute::kGlobal, drawn * n + (l == 2 ? 340.0 : 520.0) * samples + 45.0);
  return best;
}

// The route of this call.  (The record buffers are there from the start where the
// CM-angle samplers need them; for the root samplers alone they are made by the
// first call that uses them, unless its stream is being captured.)
DepositRoute choose_route(qgbe_ctx* c, int l, int n_samples, const double* scale) {
  if (!c->rec_asked && l == 2 && c->d_arena && !scale &&
      deposit_route(c, l, n_samples, false, record_capacity(c, l, record_buffer_bytes(c))) == DepositRoute::kRecord) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &cap) != hipSuccess) (void)hipGetLastError();
    else if (cap == hipStreamCaptureStatusNone) alloc_records(c);
  }
  return deposit_route(c, l, n_samples, scale != nullptr, c->d_rec ? record_capacity(c, l, c->rec_bytes) : 0);
}

// The recording launches of a call: workgroups of the kernel in batches that fit
// the record buffers.
ReplayPlan plan_replay(const qgbe_ctx* c, int l, int n_samples, long long capacity) {
  const Replay& rp = c->replay[l];
  ReplayPlan p{};
  const int per_sample = l == 2 ? 2 : 1;
  const long long nodes = c->G.nodes, all_pairs = (long long)c->G.cells * rp.count;
  const long long fit = capacity / n_samples;  // items a batch holds
  p.chunks = plan_chunks(c, std::min(nodes, fit), std::max(1LL, std::min(all_pairs, fit / nodes)), 0, n_samples, l == 0,
                         l != 0, false);
  p.chunks.chunk = (int)std::min<long long>(p.chunks.chunk, fit);
  p.n_chunks = (int)((nodes + p.chunks.chunk - 1) / p.chunks.chunk);
  p.n_group = rp.count;
  p.capacity = per_sample * capacity;
  p.region = (long long)p.chunks.chunk * n_samples * per_sample;
  p.wgs = all_pairs * p.n_chunks;
  p.per = std::min(c->rec_wgs, p.capacity / p.region);
  if (p.per > c->n_cu) p.per = p.per / c->n_cu * c->n_cu;
  return p;
}

ReplayBatch replay_batch(const ReplayPlan& p, long long wg) {
  ReplayBatch b;
  const long long per_cell = (long long)p.n_group * p.n_chunks, last = std::min(wg + p.per, p.wgs) - 1;
  b.n_wg = (int)(last - wg + 1);
  b.cell_lo = (int)(wg / per_cell);
  b.wg_base = (int)(wg % per_cell);
  b.n_cells = (int)(last / per_cell) - b.cell_lo + 1;
  b.gi_lo = b.n_cells > 1 ? 0 : b.wg_base / p.n_chunks;
  b.gi_hi = b.n_cells > 1 ? p.n_group - 1 : (int)(last % per_cell / p.n_chunks);
  return b;
}

// Their samples and deposits.
qgbe_status run_replay(qgbe_ctx* c, CollideArgs a, int l, bool alt) {
  const Replay& rp = c->replay[l];
  const bool roots = l == 2, f64 = roots || c->d.precision == QGBE_FP64;
  const ReplayPlan p = plan_replay(c, l, a.n_samples, record_capacity(c, l, c->rec_bytes));
  a.group = c->d_groups + rp.start;
  a.n_group = p.n_group;
  a.split = p.chunks.split;
  a.node_block = p.chunks.block;
  a.chunk_items = p.chunks.chunk;
  a.n_chunks = p.n_chunks;
  a.rec = c->rec;
  a.rec.capacity = p.capacity;
  a.rec.region = p.region;
  ReplayArgs r{};
  r.G = c->G;
  r.match = c->d_groups + kMatchAt;
  r.first = rp.start;
  r.n_group = rp.count;
  r.n_chunks = a.n_chunks;
  r.A = a.A;
  r.n_win = replay_windows(c);
  r.win_n = (c->G.nodes + r.n_win - 1) / r.n_win;
  // workgroups of a replay launch: two to a compute unit where their windows fit
  const double target = (double)c->n_cu * (2 * (size_t)r.win_n * sizeof(double) <= c->lds.replay ? 2 : 1);
  for (long long wg = 0; wg < p.wgs; wg += p.per) {
    const ReplayBatch b = replay_batch(p, wg);
    a.rec.cell_lo = b.cell_lo;
    a.rec.wg_base = b.wg_base;
    HIP_TRY(roots ? launch_record_roots(a, alt, b.n_wg, c->stream)
                  : f64 ? launch_record_f64(a, b.n_wg, c->stream) : launch_record_f32(a, b.n_wg, c->stream),
            "collide (record)");
    r.rec = a.rec;
    r.n_wg = b.n_wg;
    r.n_cells = b.n_cells;
    long long total = 0;
    for (int y = 0; y < kSpecies; ++y) {
      const std::vector<int>& m = c->match[y];
      r.m_lo[y] = (int)(std::lower_bound(m.begin(), m.end(), 4 * (rp.start + b.gi_lo)) - m.begin());
      r.m_hi[y] = (int)(std::lower_bound(m.begin(), m.end(), 4 * (rp.start + b.gi_hi + 1)) - m.begin());
      total += r.m_hi[y] - r.m_lo[y];
    }
    for (int y = 0; y < kSpecies; ++y) {
      const int m = r.m_hi[y] - r.m_lo[y];
      const double share = target * m / (double)std::max(1LL, total) / ((double)r.n_win * r.n_cells);
      r.parts[y] = m ? (int)std::max(1LL, std::min<long long>((long long)m * a.n_chunks, (long long)(share + 0.5))) : 0;
    }
    HIP_TRY(f64 ? launch_replay_f64(r, c->stream) : launch_replay_f32(r, c->stream), "collide (replay)");
    c->n_launches += 2;
  }
  return QGBE_OK;
}

// Enqueue the collision kernels accumulating into A.
qgbe_status run_collide(qgbe_ctx* c, int n_samples, int sampler, double* A, double* scale, double* items) {
  const bool learned = sampler == QGBE_SAMPLER_LEARNED;
  c->n_launches = 0;
  if (c->nch == 0) return QGBE_OK;
  CollideArgs a = base_args(c, n_samples, A, scale, items);
  a.learned = learned ? 1 : 0;
  a.slot_lo = 0;
  a.slot_hi = 3;
  a.direct = 1;
  const bool roots = sampler == QGBE_SAMPLER_ROOTS || sampler == QGBE_SAMPLER_ROOTS_ALT;
  const bool f64_path = c->d.precision == QGBE_FP64;
  const int l = roots ? 2 : learned ? 1 : 0;
  const DepositRoute route = choose_route(c, l, n_samples, scale);
  a.f32q = c->d_f32q;
  if (route == DepositRoute::kRecord) {
    const qgbe_status s = run_replay(c, a, l, sampler == QGBE_SAMPLER_ROOTS_ALT);
    if (s) return s;
  }
  for (const Group& g : c->groups) {
    const bool several = several_launches(c, g, l);
    if (several && route == DepositRoute::kRecord) continue;
    const bool global = several && route == DepositRoute::kGlobal;  // one launch without accumulators
    const int per = global ? 0 : g.lds_acc[l], win = global ? c->G.nodes : g.win[l];
    a.group = c->d_groups + g.start;
    a.n_group = g.count;
    // the compacting variant when the whole group fits in LDS next to its queues
    const bool is_short = roots || (!g.long_form[l] && collide_short(c->d.precision, learned, 1, n_samples));
    a.long_form = g.long_form[l];
    int queue = l == 0 ? g.queue[is_short] : 0;
    const long long acc = c->d.symmetric ? (long long)std::min(g.nslot, per) * win : 0;
    const Chunking ck = plan_chunks(c, c->G.nodes, (long long)c->G.cells * g.count, acc, n_samples, queue, learned || roots,
                                    g.long_form[l]);
    if (!is_short && ck.split > 1 && queue) queue = g.queue[1];  // waves that share nodes take the short form
    a.split = ck.split;
    a.node_block = ck.block;
    const int chunk = ck.chunk;
    a.chunk_items = chunk;
    a.n_chunks = (c->G.nodes + chunk - 1) / chunk;
    // Deposit slots whose FP64 accumulators do not all fit in LDS are split
    // over launches that each keep their slots' accumulators in LDS: the
    // samples are recomputed (same draws).  The first launch also writes the
    // direct sums.
    const int n_pass = (c->d.symmetric && per >= 1 && per < g.nslot) ? (g.nslot + per - 1) / per : 1;
    const size_t acc_b = (size_t)c->G.nodes * sizeof(double), tile_b = (size_t)c->G.nodes * sizeof(float);
    const int n_win = (c->G.nodes + win - 1) / win;
    for (int pass = 0; pass < n_pass; ++pass) {
      for (int w = 0; w < n_win; ++w) {
        a.slot_lo = n_pass > 1 ? pass * per : 0;
        a.slot_hi = n_pass > 1 ? std::min(g.nslot, a.slot_lo + per) : g.nslot;
        a.win_lo = w * win;
        a.win_n = std::min(win, c->G.nodes - a.win_lo);
        a.direct = pass == 0 && w == 0 ? 1 : 0;
        a.lds_acc = per;
        a.lds_tiles = g.lds_tiles[l];
        if (n_pass > 1 && n_win == 1) {
          const size_t used = (size_t)(a.slot_hi - a.slot_lo) * acc_b;
          a.lds_tiles = f64_path || roots ? 0 : (int)std::min<size_t>(g.nslot, (g.budget[l] - used) / tile_b);
        }
        if (queue) a.lds_tiles = 0;  // the compacting variant reads f from the node quads
        const int q = n_pass == 1 && n_win == 1 ? queue : 0;
        if (roots) HIP_TRY(launch_collide_roots(a, sampler == QGBE_SAMPLER_ROOTS_ALT, c->stream), "collide (roots)");
        else if (f64_path) HIP_TRY(launch_collide_f64(a, g.nslot, q, c->stream), "collide (fp64)");
        else HIP_TRY(launch_collide_f32(a, g.nslot, q, c->stream), "collide (fp32)");
        ++c->n_launches;
      }
    }
  }
  return QGBE_OK;
}

}  // namespace qgbe

namespace {

void fill_stats(qgbe_ctx* c, const double* obs, const double* mass2_host, qgbe_stats* st) {
  std::memset(st, 0, sizeof *st);
  double mass_term = 0.0;
  for (int s = 0; s < kSpecies; ++s) {
    st->N[s] = obs[s * kObsPer];
    st->E[s] = obs[s * kObsPer + 1];
    st->N_total += st->N[s];
    st->E_total += st->E[s];
    for (int k = 0; k < 3; ++k) st->P[k] += obs[s * kObsPer + 2 + k];
    mass_term += obs[s * kObsPer + 5];
    st->entropy += obs[s * kObsPer + 6];
    for (int k = 0; k < 3; ++k) st->T_ii[k] += obs[s * kObsPer + 7 + k];
    double m = 0.0;
    for (int x = 0; x < c->G.cells; ++x) m += mass2_host[s * c->G.cells + x];
    st->mass2_avg[s] = m / c->G.cells;
  }
  st->E_total_mod = st->E_total - 0.25 * mass_term;
  st->min_f = obs[kSpecies * kObsPer];
  st->max_fermion_f = obs[kSpecies * kObsPer + 1];
  if (st->min_f < 0.0) st->flags |= QGBE_FLAG_NEGATIVE_F;
  if (st->max_fermion_f > 1.0) st->flags |= QGBE_FLAG_PAULI;
  if (obs[kSpecies * kObsPer + 2] > 0.0) st->flags |= QGBE_FLAG_NONFINITE;
  st->step = c->step;
}

qgbe_status read_stats(qgbe_ctx* c, qgbe_stats* st, bool energy = false) {
  HIP_TRY(launch_observables(c->G, c->d_f, c->d_mass2, c->d_obs_scratch, c->d_obs, c->stream), "observables");
  // the totals, the energy budget, the observables and the masses lie side by side: one copy
  const char* base = (const char*)c->d_count;
  std::vector<char> host((const char*)(c->d_mass2 + (size_t)kSpecies * c->G.cells) - base);
  HIP_TRY(hipMemcpyAsync(host.data(), base, host.size(), hipMemcpyDeviceToHost, c->stream), "copy statistics");
  HIP_TRY(hipStreamSynchronize(c->stream), "synchronise");
  const auto at = [&](const void* d) { return host.data() + ((const char*)d - base); };
  const unsigned long long* counts = (const unsigned long long*)at(c->d_count);
  const double *mcs = (const double*)at(c->d_mc), *obs = (const double*)at(c->d_obs);
  const double* m2 = (const double*)at(c->d_mass2);
  double budget[2] = {0.0, 0.0};
  if (energy) std::memcpy(budget, at(c->d_energy), sizeof budget);
  unsigned long long accepted = 0;
  double mc[2] = {0.0, 0.0};
  for (int i = 0; i < kStripes; ++i) {  // in stripe order: the same sum for the same stripes
    accepted += counts[i];
    mc[0] += mcs[2 * i];
    mc[1] += mcs[2 * i + 1];
  }
  fill_stats(c, obs, m2, st);
  st->E_source = budget[0];
  st->E_collide = budget[1];
  st->n_accepted = (double)accepted;
  // sum S_i^2 estimates sum (E S_i)^2 + sum Var S_i; remove the variance part
  const double signal = mc[1] - mc[0];
  st->mc_err_est = mc[0] <= 0.0 ? 0.0 : (signal > 0.0 ? std::sqrt(mc[0] / signal) : INFINITY);
  return QGBE_OK;
}

// The kernels' dynamic LDS limits, raised once per GPU and precision: each of
// the some 50 kernel variants takes a query and a call of the runtime.
hipError_t lds_budget(int device, int precision, size_t lds_max, LdsBudget* out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static struct { bool ready; LdsBudget lds; } known[kMaxDevices][2];
  const auto raise = precision == QGBE_FP64 ? collide_f64_lds_limit : collide_f32_lds_limit;
  if (device >= kMaxDevices) {
    const hipError_t e = raise(lds_max, out);
    return e != hipSuccess ? e : collide_roots_lds_limit(lds_max, &out->roots);
  }
  std::lock_guard<std::mutex> lock(mu);
  auto& k = known[device][precision];
  if (!k.ready) {
    hipError_t e = raise(lds_max, &k.lds);
    if (e == hipSuccess) e = collide_roots_lds_limit(lds_max, &k.lds.roots);
    if (e != hipSuccess) return e;
    k.ready = true;
  }
  *out = k.lds;
  return hipSuccess;
}

bool species_ok(int s) { return s >= -1 && s < kSpecies; }

}  // namespace

extern "C" {

const char* qgbe_last_error(void) { return g_error.c_str(); }

size_t qgbe_workspace_bytes(const qgbe_ctx* ctx) { return ctx ? ctx->ws : 0; }

int32_t qgbe_channel_table(uint32_t species_mask, uint32_t row_mask, int32_t* rows, double* weights,
                           int32_t max) {
  Channel buf[kMaxChannels];
  const int n = build_channels(species_mask & 0x7Fu, row_mask & 0x7Fu, buf, kMaxChannels);
  if (n < 0) return QGBE_EINVAL;
  if (n > max) return fail(QGBE_EINVAL, "channel table larger than max");
  for (int i = 0; i < n; ++i) {
    if (rows) {
      rows[i * 5] = buf[i].row;
      for (int p = 0; p < 4; ++p) rows[i * 5 + 1 + p] = buf[i].sp[p];
    }
    if (weights) {
      weights[i * 2] = buf[i].w;
      weights[i * 2 + 1] = buf[i].sigma;
    }
  }
  return n;
}

void qgbe_philox4x32_10(const uint32_t ctr[4], const uint32_t key[2], uint32_t out[4]) {
  uint32_t x0 = ctr[0], x1 = ctr[1], x2 = ctr[2], x3 = ctr[3];
  philox4x32_10(x0, x1, x2, x3, key[0], key[1]);
  out[0] = x0; out[1] = x1; out[2] = x2; out[3] = x3;
}

qgbe_status qgbe_init_grid(const qgbe_grid_desc* desc, qgbe_ctx** out) {
  if (!out) return fail(QGBE_EINVAL, "out is NULL");
  *out = nullptr;
  qgbe_status st = validate(desc);
  if (st) return st;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev == 0) return fail(QGBE_EDEVICE, "no HIP device");
  if (desc->device < 0 || desc->device >= ndev) return fail(QGBE_EINVAL, "device ordinal out of range");
  HIP_TRY(hipSetDevice(desc->device), "hipSetDevice");
  int lds_max = 0;
  HIP_TRY(hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, desc->device),
          "query LDS size");
  LdsBudget lds;
  const size_t lds_bytes = (size_t)std::max(lds_max, 0);
  HIP_TRY(lds_budget(desc->device, desc->precision, lds_bytes, &lds), "raise the dynamic LDS limit");
  qgbe_ctx* c = new qgbe_ctx();
  c->d = *desc;
  c->stream = (hipStream_t)desc->stream;
  make_grid(desc, c->G);
  c->chans.resize(kMaxChannels);
  c->nch = build_channels(desc->species_mask, desc->row_mask, c->chans.data(), kMaxChannels);
  c->chans.resize(c->nch);
  c->lds = lds;
  int n_cu = 0;
  if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, desc->device) == hipSuccess && n_cu > 0)
    c->n_cu = n_cu;
  plan_groups(c);
  const size_t n = field_len(c);
  // One allocation, carved: twice, first for its size.
  char* arena = nullptr;
  size_t used = 0;
  const auto take = [&](auto** p, size_t cnt) {
    using T = std::remove_reference_t<decltype(**p)>;
    if (arena) *p = reinterpret_cast<T*>(arena + used);
    used += (cnt * sizeof(T) + 255) & ~size_t(255);
  };
  const auto carve = [&]() {
    used = 0;
    take(&c->d_chans, std::max(1, c->nch));  // the channel tables side by side: one upload
    take(&c->d_groups, std::max<size_t>(1, c->group_index.size()));
    take(&c->d_f, n);                        // the zeroed fields side by side: one fill
    take(&c->d_f_next, n);
    take(&c->d_f32, n);
    take(&c->d_done, c->G.cells);            // zeroed with them
    if (c->d.precision == QGBE_FP32 && (c->need_quads[0] || c->need_quads[1])) take(&c->d_f32q, n);
    take(&c->d_A, n);
    take(&c->d_lag, (size_t)kSpecies * c->G.cells);
    take(&c->d_obs_scratch, observables_scratch(c->G));
    take(&c->d_msq, 1);
    take(&c->d_mass_part, mass_scratch(c->G));
    take(&c->d_count, kStripes);             // what the statistics read, side by side: one copy
    take(&c->d_mc, kStripes * (2 + std::max(1, c->nch)));  // and the channel variances
    c->d_chan_var = c->d_mc + 2 * kStripes;
    take(&c->d_energy, 2);
    take(&c->d_obs, (size_t)observables_len);
    take(&c->d_mass2, (size_t)kSpecies * c->G.cells);
  };
  carve();
  if (const qgbe_status s = dev_alloc(c, &c->d_arena, used, "context")) {
    qgbe_destroy(c);
    return s;
  }
  arena = c->d_arena;
  carve();
  if (c->replay[0].count || c->replay[1].count) alloc_records(c);
  std::vector<char> tables((char*)c->d_f - arena);
  std::memcpy(tables.data(), c->chans.data(), c->nch * sizeof(Channel));
  std::memcpy(tables.data() + ((char*)c->d_groups - arena), c->group_index.data(), c->group_index.size() * sizeof(int));
  const char* what = "copy channel tables";
  hipError_t e = hipMemcpy(arena, tables.data(), tables.size(), hipMemcpyHostToDevice);
  for (int i = 0; i < 4 && e == hipSuccess; ++i) {
    what = "create events";
    e = hipEventCreate(&c->ev[i]);
  }
  if (e == hipSuccess) {
    what = "zero f";
    // both buffers, as a step updates only the evolving species, and the FP32 shadow
    e = launch_fill(c->d_f, 0.0, ((char*)(c->d_done + c->G.cells) - (char*)c->d_f + 7) / sizeof(double), c->stream);
  }
  if (e == hipSuccess) {
    what = "synchronise";
    e = hipStreamSynchronize(c->stream);
  }
  if (e != hipSuccess) {
    qgbe_status s = hip_fail(e, what);
    qgbe_destroy(c);
    return s;
  }
  *out = c;
  g_error.clear();
  return QGBE_OK;
}

void qgbe_destroy(qgbe_ctx* c) {
  if (!c) return;
  (void)hipSetDevice(c->d.device);
  (void)hipStreamSynchronize(c->stream);
  (void)hipFree(c->d_arena);
  (void)hipFree(c->d_rec);
  (void)hipFree(c->d_thr);
  (void)hipFree(c->d_mu);
  (void)hipFree(c->d_sigma);
  (void)hipFree(c->d_feat);
  (void)hipFree(c->d_mix_on);
  (void)hipFree(c->d_mass7);
  (void)hipFree(c->mlp.arena);
  for (auto& e : c->ev)
    if (e) (void)hipEventDestroy(e);
  delete c;
}

qgbe_status qgbe_set_distribution(qgbe_ctx* c, int32_t species, const double* f, int32_t on_device) {
  if (!c || !f) return fail(QGBE_EINVAL, "NULL argument");
  if (!species_ok(species)) return fail(QGBE_EINVAL, "species must be -1 or 0..6");
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  const size_t per = (size_t)c->G.cells * c->G.nodes;
  double* dst = species < 0 ? c->d_f : c->d_f + (size_t)species * per;
  const size_t cnt = species < 0 ? field_len(c) : per;
  if (!on_device)
    HIP_TRY(hipMemcpyAsync(dst, f, cnt * sizeof(double), hipMemcpyHostToDevice, c->stream), "copy f in");
  // the second buffer of f too: a step updates only the evolving species
  const size_t at = dst - c->d_f;
  HIP_TRY(launch_set_field(on_device ? f : dst, dst, c->d_f_next + at, c->d_f32 + at, cnt, c->stream), "set f");
  if (!on_device) HIP_TRY(hipStreamSynchronize(c->stream), "synchronise");
  c->has_lag = false;
  c->masses_valid = false;
  return QGBE_OK;
}

qgbe_status qgbe_get_distribution(qgbe_ctx* c, int32_t species, double* f, int32_t on_device) {
  if (!c || !f) return fail(QGBE_EINVAL, "NULL argument");
  if (!species_ok(species)) return fail(QGBE_EINVAL, "species must be -1 or 0..6");
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  const size_t per = (size_t)c->G.cells * c->G.nodes;
  const double* src = species < 0 ? c->d_f : c->d_f + (size_t)species * per;
  const size_t cnt = species < 0 ? field_len(c) : per;
  HIP_TRY(hipMemcpyAsync(f, src, cnt * sizeof(double), on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost,
                         c->stream), "copy f out");
  if (!on_device) HIP_TRY(hipStreamSynchronize(c->stream), "synchronise");
  return QGBE_OK;
}

qgbe_status qgbe_get_masses(qgbe_ctx* c, double* mass2) {
  if (!c || !mass2) return fail(QGBE_EINVAL, "NULL argument");
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  HIP_TRY(hipMemcpyAsync(mass2, c->d_mass2, (size_t)kSpecies * c->G.cells * sizeof(double), hipMemcpyDeviceToHost,
                         c->stream), "copy masses");
  HIP_TRY(hipStreamSynchronize(c->stream), "synchronise");
  return QGBE_OK;
}

qgbe_status qgbe_set_step_index(qgbe_ctx* c, uint32_t step) {
  if (!c) return fail(QGBE_EINVAL, "NULL context");
  c->step = step;
  return QGBE_OK;
}

qgbe_status qgbe_get_step_index(const qgbe_ctx* c, uint32_t* step) {
  if (!c || !step) return fail(QGBE_EINVAL, "NULL argument");
  *step = c->step;
  return QGBE_OK;
}

qgbe_status qgbe_collision_term_ex(qgbe_ctx* c, int32_t n_samples, int32_t sampler, double* A_out,
                                   int32_t on_device, const qgbe_collide_extras* ex, qgbe_stats* st) {
  if (!c || !A_out) return fail(QGBE_EINVAL, "NULL argument");
  if (n_samples < 1) return fail(QGBE_EINVAL, "n_samples must be >= 1");
  if (sampler < QGBE_SAMPLER_UNIFORM || sampler > QGBE_SAMPLER_ROOTS_ALT) return fail(QGBE_EINVAL, "bad sampler");
  if (sampler == QGBE_SAMPLER_LEARNED && !c->K) return fail(QGBE_ESTATE, "no proposal table installed");
  if (sampler == QGBE_SAMPLER_LEARNED && c->d.precision == QGBE_FP32 && c->K > kMixKF32)
    return fail(QGBE_EUNSUPPORTED, "the FP32 learned sampler takes at most 8 mixture components (FP64 takes 16)");
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  const size_t n = field_len(c);
  double* A = on_device ? A_out : c->d_A;
  double* scale = nullptr;
  double* items = nullptr;
  const bool ex_host = ex && !ex->on_device;
  const size_t n_items = (size_t)c->G.cells * c->nch * c->G.nodes;
  if (ex && ex->scale) {
    if (ex_host) HIP_TRY(hipMalloc(&scale, n * sizeof(double)), "scale scratch");
    else scale = ex->scale;
  }
  if (ex && ex->item_sums && n_items) {
    if (ex_host) HIP_TRY(hipMalloc(&items, n_items * sizeof(double)), "item scratch");
    else items = ex->item_sums;
  }
  qgbe_status s = start_term(c, sampler, A, false);
  if (!s && sampler == QGBE_SAMPLER_LEARNED && c->table_net) s = refresh_proposal_table(c);
  if (!s) {
    hipError_t e = scale ? launch_fill(scale, 0.0, n, c->stream) : hipSuccess;
    if (e == hipSuccess && st) e = hipEventRecord(c->ev[0], c->stream);
    if (e != hipSuccess) s = hip_fail(e, "zero outputs");
  }
  if (!s) s = run_collide(c, n_samples, sampler, A, scale, items);
  if (!s) {
    hipError_t e = st ? hipEventRecord(c->ev[1], c->stream) : hipSuccess;
    if (e == hipSuccess && !on_device)
      e = hipMemcpyAsync(A_out, A, n * sizeof(double), hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess && ex_host && scale)
      e = hipMemcpyAsync(ex->scale, scale, n * sizeof(double), hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess && ex_host && items)
      e = hipMemcpyAsync(ex->item_sums, items, n_items * sizeof(double), hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess && (!on_device || ex_host || st)) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) s = hip_fail(e, "collision term");
  }
  if (ex_host) {
    (void)hipFree(scale);
    (void)hipFree(items);
  }
  if (s) return s;
  if (st) {
    s = read_stats(c, st);
    if (s) return s;
    float ms = 0.0f;
    (void)hipEventElapsedTime(&ms, c->ev[0], c->ev[1]);
    st->t_collide_ms = ms;
    st->n_collide_launches = (uint32_t)c->n_launches;
    st->n_evals = (double)c->G.cells * c->nch * c->G.nodes * n_samples;
  }
  return QGBE_OK;
}

qgbe_status qgbe_set_matrix_element(qgbe_ctx* c, int32_t row, int32_t n_terms, const double* coef,
                                    const int32_t* powers) {
  if (!c) return fail(QGBE_EINVAL, "NULL context");
  if (row < 1 || row > 7) return fail(QGBE_EINVAL, "row must be 1..7");
  if (n_terms < 0 || n_terms > kMsqMaxTerms) return fail(QGBE_EINVAL, "0..8 terms per row");
  if (n_terms > 0 && (!coef || !powers)) return fail(QGBE_EINVAL, "NULL terms");
  for (int k = 0; k < n_terms; ++k) {
    if (!std::isfinite(coef[k])) return fail(QGBE_EINVAL, "non-finite coefficient");
    for (int i = 0; i < 6; ++i)
      if (powers[6 * k + i] < 0 || powers[6 * k + i] > kMsqMaxPower) return fail(QGBE_EINVAL, "powers must be 0..4");
  }
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  c->msq.n[row] = n_terms;
  for (int k = 0; k < kMsqMaxTerms; ++k) {
    c->msq.c[row][k] = k < n_terms ? coef[k] : 0.0;
    for (int i = 0; i < 6; ++i) c->msq.p[row][k][i] = (int8_t)(k < n_terms ? powers[6 * k + i] : 0);
  }
  if (n_terms > 0) c->msq_mask |= 1u << row;
  else c->msq_mask &= ~(1u << row);
  // the table is read by kernels already queued on the stream: wait for them
  HIP_TRY(hipStreamSynchronize(c->stream), "synchronise");
  HIP_TRY(hipMemcpyAsync(c->d_msq, &c->msq, sizeof(MsqTable), hipMemcpyHostToDevice, c->stream),
          "copy matrix elements");
  HIP_TRY(hipStreamSynchronize(c->stream), "synchronise");
  return QGBE_OK;
}

qgbe_status qgbe_collision_term(qgbe_ctx* c, int32_t n_samples, int32_t sampler, double* A_out, int32_t on_device,
                                qgbe_stats* st) {
  return qgbe_collision_term_ex(c, n_samples, sampler, A_out, on_device, nullptr, st);
}

qgbe_status qgbe_step(qgbe_ctx* c, double dt_fm, int32_t n_samples, int32_t sampler, int32_t n_steps,
                      qgbe_stats* per_step) {
  if (!c) return fail(QGBE_EINVAL, "NULL context");
  if (!(dt_fm > 0.0) || !std::isfinite(dt_fm)) return fail(QGBE_EINVAL, "dt must be > 0");
  if (n_samples < 1 || n_steps < 0) return fail(QGBE_EINVAL, "n_samples >= 1 and n_steps >= 0 required");
  if (sampler < QGBE_SAMPLER_UNIFORM || sampler > QGBE_SAMPLER_ROOTS_ALT) return fail(QGBE_EINVAL, "bad sampler");
  if (sampler == QGBE_SAMPLER_LEARNED && !c->K) return fail(QGBE_ESTATE, "no proposal table installed");
  if (sampler == QGBE_SAMPLER_LEARNED && c->d.precision == QGBE_FP32 && c->K > kMixKF32)
    return fail(QGBE_EUNSUPPORTED, "the FP32 learned sampler takes at most 8 mixture components (FP64 takes 16)");
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  qgbe_status result = QGBE_OK;
  for (int k = 0; k < n_steps; ++k) {
    if (per_step) HIP_TRY(hipEventRecord(c->ev[2], c->stream), "event");
    qgbe_status s = start_term(c, sampler, c->d_A, false);
    if (!s && sampler == QGBE_SAMPLER_LEARNED && c->table_net) s = refresh_proposal_table(c);
    if (s) return s;
    if (per_step) HIP_TRY(hipEventRecord(c->ev[0], c->stream), "event");
    s = run_collide(c, n_samples, sampler, c->d_A, nullptr, nullptr);
    if (s) return s;
    if (per_step) HIP_TRY(hipEventRecord(c->ev[1], c->stream), "event");
    if (per_step)  // before the update: f_k, its masses, the step before's masses
      HIP_TRY(launch_energy_budget(c->G, c->d_f, c->d_A, c->d_mass2, c->has_lag ? c->d_lag : nullptr, dt_fm,
                                   c->d_obs_scratch, c->d_energy, c->stream),
              "energy budget");
    HIP_TRY(launch_update(c->G, c->d_f, c->d_A, c->d_mass2, dt_fm, c->d.drift, c->d_f_next, c->d_f32, c->d_lag,
                          c->stream), "update");
    std::swap(c->d_f, c->d_f_next);
    c->masses_valid = false;
    c->has_lag = c->d.mass_mode == QGBE_MASS_DYNAMIC;
    if (per_step) HIP_TRY(hipEventRecord(c->ev[3], c->stream), "event");
    c->step += 1;
    if (per_step) {
      s = read_stats(c, &per_step[k], true);
      if (s) return s;
      float ms = 0.0f;
      (void)hipEventElapsedTime(&ms, c->ev[0], c->ev[1]);
      per_step[k].t_collide_ms = ms;
      per_step[k].n_collide_launches = (uint32_t)c->n_launches;
      (void)hipEventElapsedTime(&ms, c->ev[2], c->ev[3]);
      per_step[k].t_step_ms = ms;
      per_step[k].n_evals = (double)c->G.cells * c->nch * c->G.nodes * n_samples;
      if (per_step[k].flags & QGBE_FLAG_NONFINITE) result = fail(QGBE_ENUMERIC, "non-finite f after step");
    }
  }
  return result;
}

qgbe_status qgbe_observables(qgbe_ctx* c, qgbe_stats* st) {
  if (!c || !st) return fail(QGBE_EINVAL, "NULL argument");
  HIP_TRY(hipSetDevice(c->d.device), "hipSetDevice");
  qgbe_status s = compute_masses(c);
  if (s) return s;
  return read_stats(c, st);
}


}  // extern "C"
