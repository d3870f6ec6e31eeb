// Context of libqgbe shared by the host-side translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <string>
#include <vector>

#include "collide.h"
#include "field.h"
#include "mlp.h"
#include "qgbe.h"
#include "qgbe_common.h"

namespace qgbe {

qgbe_status fail(qgbe_status s, const std::string& msg);
qgbe_status hip_fail(hipError_t e, const char* what);

#define HIP_TRY(expr, what)                                \
  do {                                                     \
    hipError_t _e = (expr);                                \
    if (_e != hipSuccess) return ::qgbe::hip_fail(_e, what); \
  } while (0)

// Channels grouped by their number of deposit slots.
struct Group {
  int start, count;   // range in the group index array
  int nslot;          // distinct species at positions 2..4
  int lds_acc[3];     // FP64 accumulators staged in LDS  [uniform, learned, root samplers]
  int lds_tiles[3];   // FP32 f tiles staged in LDS; none in FP64 and for the root samplers
  size_t budget[3];   // dynamic LDS of the launches
  bool long_form[3];  // the long-item form whatever the items: its budget is larger
  int win[3];         // nodes per accumulator window (= nodes unless one slot's FP64
                      // accumulators exceed LDS; then one launch per window and slot)
  int queue[2];       // the form of the uniform sampler's compacting variant that fits [long, short items]; 0: none
};

// Channels whose deposit accumulators need more than one launch (slots or node
// windows): their samples are drawn once and their deposits recorded, then
// replayed per (species, window).  A channel of more slots never needs fewer
// launches, so they are the last ones of the channels in order of their slots.
struct Replay {
  int start = 0, count = 0;        // range in the group index array
};

// Device buffers of the proposal network (one allocation, on first use).
struct MlpState {
  bool ready = false;
  bool has_weights = false;
  int adam_t = 0;
  char* arena = nullptr;
  float *params = nullptr, *m = nullptr, *v = nullptr, *grad = nullptr;
  __bf16 *pb = nullptr, *pbt = nullptr;   // BF16 weights, row-major and transposed
  float *X = nullptr, *yw = nullptr, *Y = nullptr;  // staging of host buffers
  __bf16* act = nullptr;                  // a gradient's activations and FP32 gradients (see mlp.h), losses per tile
  float* dz = nullptr;
  double* loss_part = nullptr;
  double* scalars = nullptr;              // [0] loss, [1] weight sum
};

}  // namespace qgbe

struct qgbe_ctx {
  qgbe_grid_desc d{};
  qgbe::Grid G{};
  hipStream_t stream = nullptr;
  int nch = 0;
  std::vector<qgbe::Channel> chans;
  std::vector<int> group_index;    // the channels in order of their slots, then match: of the masks alone
  std::vector<int> match[qgbe::kSpecies];  // as ReplayArgs::match, over all channels
  std::vector<qgbe::Group> groups;
  qgbe::Replay replay[3];          // [uniform, learned, root samplers]
  unsigned char* d_rec = nullptr;  // record buffers, an allocation of their own (NULL: none, every launch draws its samples again)
  bool rec_asked = false;          // whether they have been asked for
  qgbe::RecordArgs rec{};          // their parts
  long long rec_wgs = 0;           // counters in rec.count
  size_t rec_bytes = 0;            // of the tiles
  char* d_arena = nullptr;         // the allocation that holds the buffers below unless noted
  qgbe::Channel* d_chans = nullptr;
  int* d_groups = nullptr;
  double* d_f = nullptr;
  double* d_f_next = nullptr;
  float* d_f32 = nullptr;
  float4* d_f32q = nullptr;        // node quads of d_f32, for tiles read from global memory
  int n_launches = 0;                    // collision kernel launches of the last term
  bool need_quads[2] = {false, false};  // some group reads tiles globally [uniform, learned]
  double* d_mass2 = nullptr;
  double* d_lag = nullptr;
  bool has_lag = false;
  bool masses_valid = false;       // d_mass2 holds the masses of the current f
  double* d_A = nullptr;
  double* d_obs_scratch = nullptr;
  double* d_energy = nullptr;  // [E_source, E_collide] of the last step
  qgbe::MsqTable msq{};          // user matrix elements (host copy)
  uint32_t msq_mask = 0;         // rows replaced by them
  qgbe::MsqTable* d_msq = nullptr;  // device copy
  unsigned* d_done = nullptr;     // per cell: chunk sums that are in (zero between launches)
  double* d_mass_part = nullptr;  // per (cell, chunk, species) partial mass integrals
  double* d_obs = nullptr;
  unsigned long long* d_count = nullptr;
  double* d_mc = nullptr;          // [2] MC error accumulators of the last collision term
  double* d_chan_var = nullptr;    // [kStripes][channels] per-channel variance sums of the last collision term
  uint32_t step = 0;
  // allocated on first use
  int K = 0;                       // proposal table components (0 = none)
  uint32_t* d_thr = nullptr;
  float* d_mu = nullptr;
  float* d_sigma = nullptr;
  uint8_t* d_mix_on = nullptr;     // [channels] 1: learned sampler, 0: uniform fallback
  float* d_feat = nullptr;         // [nch * nodes][8] conditioning features
  double* d_mass7 = nullptr;       // cell-averaged masses behind d_feat
  bool table_net = false;          // table comes from the network: rebuilt whenever the masses change
  float table_alpha = 0.0f;        // defensive weight of that table
  qgbe::MlpState mlp;
  hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};
  size_t ws = 0;
  qgbe::LdsBudget lds;             // dynamic LDS per workgroup of the context's precision
  int n_cu = 256;                  // compute units of the device
};

namespace qgbe {

// How channels whose deposit accumulators need more than one launch deposit:
// every launch draws the samples again for its accumulators, the deposits are
// recorded and replayed, or (FP64) one launch adds them with global atomics.
enum class DepositRoute { kAgain, kRecord, kGlobal };
struct Chunking {
  int chunk;  // observed nodes per workgroup
  int split;  // waves that share a node
  int block;  // nodes a wave takes at a time
};
// Observed nodes per workgroup; acc: entries a workgroup zeroes and flushes.
Chunking plan_chunks(const qgbe_ctx* c, long long nodes, long long pairs, long long acc, int n_samples, bool queue,
                     bool learned, bool long_form);
// The recording launches of a call, and one of them: per workgroups from the
// wg-th of all wgs on, as its first cell, its first workgroup there, cells and
// (with one cell) channels of the group.
struct ReplayPlan {
  Chunking chunks;
  int n_chunks, n_group;
  long long capacity, region;  // as RecordArgs
  long long wgs, per;
};
struct ReplayBatch {
  int n_wg, cell_lo, wg_base, n_cells, gi_lo, gi_hi;
};
// capacity: samples whose deposits the record buffers hold (0: no buffers).
ReplayPlan plan_replay(const qgbe_ctx* c, int l, int n_samples, long long capacity);
ReplayBatch replay_batch(const ReplayPlan& p, long long wg);
DepositRoute deposit_route(const qgbe_ctx* c, int l, int n_samples, bool scale, long long capacity);

size_t field_len(const qgbe_ctx* c);
// Descriptor checks (QGBE_EINVAL with a message), the grid it describes, and
// the LDS plan of the channel groups (needs c->G, c->d, c->chans and the
// LDS budgets; long_form: the uniform sampler of FP32 in the long-item form and
// without the smaller queue, the plan that needs the node quads least).
qgbe_status validate(const qgbe_grid_desc* d);
void make_grid(const qgbe_grid_desc* d, Grid& G);
void plan_groups(qgbe_ctx* c, bool long_form = false);
// Whether a group's accumulators take more than one launch (slots or windows)
// with sampler l (0 uniform, 1 learned, 2 roots).
bool several_launches(const qgbe_ctx* c, const Group& g, int l);
// Entries of the group index array: the groups, and from kMatchAt on the
// species' matches, kMaxMatches apart.
constexpr size_t kMatchAt = kMaxChannels;
constexpr size_t kMaxGroupIndex = kMatchAt + (size_t)kSpecies * kMaxMatches;
// Record buffers in given memory (none if they would be too small to pay).
void carve_records(qgbe_ctx* c, unsigned char* p, size_t bytes);
// Masses, and the start of a collision term into A: A and the totals zeroed,
// the node quads of the sampler's kernels (f32: also the FP32 copy of f).
qgbe_status start_term(qgbe_ctx* c, int sampler, double* A, bool f32);
// Enqueue the collision kernels of one collision term, accumulating into A;
// start_term comes before.
qgbe_status run_collide(qgbe_ctx* c, int n_samples, int sampler, double* A, double* scale, double* items);
qgbe_status compute_masses(qgbe_ctx* c);
CollideArgs base_args(qgbe_ctx* c, int n_samples, double* A, double* scale, double* items);
// Enqueue features, network forward and table construction for the current
// masses (no allocation, no synchronisation).
qgbe_status refresh_proposal_table(qgbe_ctx* c);
// Device buffers of a K-component proposal table (reallocated if K changes).
qgbe_status install_proposal_table(qgbe_ctx* c, int K);
// Every channel back on the learned sampler (after a new table or network).
qgbe_status reset_channel_samplers(qgbe_ctx* c);
// Device buffers of the conditioning features.
qgbe_status ensure_proposal_features(qgbe_ctx* c);

template <typename T>
qgbe_status dev_alloc(qgbe_ctx* c, T** p, size_t n, const char* what) {
  hipError_t e = hipMalloc((void**)p, n * sizeof(T));
  if (e != hipSuccess) {
    *p = nullptr;
    return hip_fail(e, what);
  }
  c->ws += n * sizeof(T);
  return QGBE_OK;
}

}  // namespace qgbe
