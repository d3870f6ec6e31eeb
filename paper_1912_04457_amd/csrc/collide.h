// Launch interface of the collision kernels.
#pragma once

#include "qgbe_common.h"

namespace qgbe {

// Stripes of the per-launch totals: one global atomic per workgroup lands on
// one of kStripes addresses, so same-address atomics do not serialise.
constexpr int kStripes = 64;

// Mixture components the FP32 learned sampler takes (its per-wave LDS row of
// component constants is laid out for this many); the FP64 path takes 16.
constexpr int kMixKF32 = 8;

// Most observed nodes of a workgroup whose waves share nodes (split > 1).
constexpr int kSplitNodes = 64;
// Most consecutive nodes a wave takes at a time.
constexpr int kMaxNodeBlock = 8;

// Deposits of a launch's accepted samples, kept for replay_kernel: per sample
// the stencils of positions 2, 3, 4 (base node and weights) and the value, in
// the integrand's precision.  A workgroup of the sampling kernel owns `region`
// consecutive records (its nodes times the samples per node, all it can
// accept; twice that for the root samplers) and leaves their number in count.  Records lie in tiles of 64, field
// after field (see Record), so that a field of 64 consecutive records is one
// wide access and the fields of a record are constant offsets apart.
struct RecordArgs {
  unsigned char* tiles;
  uint32_t* count;    // [workgroups of the batch]
  long long capacity; // records the tiles hold, a multiple of 64
  long long region;   // records of a workgroup
  int cell_lo;       // first cell of the batch
  int wg_base;       // and its first workgroup there; workgroups run over (cell, channel, chunk)
};

struct CollideArgs {
  Grid G;
  const Channel* chans;   // device channel table (all channels)
  const int* group;       // channel indices processed by this launch
  int n_group;
  int n_channels;         // total channels (layout of items)
  int n_chunks;           // workgroups per (cell, channel)
  int chunk_items;        // observed nodes per workgroup
  int split;              // waves that share a node, each a part of its samples: divides
                          // the workgroup's waves; > 1 only with chunk_items <= kSplitNodes
  int node_block;         // consecutive nodes a wave takes at a time in the short-item form
  int long_form;          // the long-item form whatever the items (FP32): its own LDS is smaller
  int lds_tiles;          // f tiles staged in LDS
  int lds_acc;            // FP64 deposit accumulators in LDS (0: global atomics, FP64 only)
  int slot_lo, slot_hi;   // deposit slots [lo, hi) written by this launch, at most lds_acc
  int win_lo, win_n;      // LDS accumulators cover nodes [win_lo, win_lo + win_n);
                          // deposit corners outside belong to another launch
  int direct;             // this launch also writes the direct sums, items, scale and counts
  int n_samples;
  int symmetric;
  uint32_t key0, key1;    // Philox key
  const double* f64;      // [7][cells][nodes]
  const float* f32;       // FP32 shadow of f64
  const float4* f32q;     // node quads of f32 (global-memory tiles), see TermStart
  const double* mass2;    // [7][cells]
  double* A;              // [7][cells][nodes], accumulated into
  double* scale;          // optional, same shape
  double* items;          // optional [cells][n_channels][nodes]
  unsigned long long* n_accepted;  // [kStripes]: samples above threshold and inside the box
  double* mc_acc;         // [kStripes][2] (may be NULL): sum over items of the variance estimate
                          // of their direct sum, and of the squared direct sums
                          // (workgroup b adds into stripe b mod kStripes; the reader sums them)
  double* chan_var;       // [kStripes][n_channels] (may be NULL): variance sums per channel, striped
  uint32_t msq_mask;      // bit r: Table I row r replaced by the user terms in msq
  const MsqTable* msq;    // device copy of the user terms (NULL when msq_mask is 0)
  int learned;            // draw from the mixture table instead of uniformly
  int mix_K;              // mixture components
  const uint32_t* mix_thr;   // [channels*nodes][K]
  const float* mix_mu;       // [channels*nodes][K][5]
  const float* mix_sigma;    // [channels*nodes][K][5]
  const uint8_t* mix_on;     // [channels] 0: the channel falls back to the uniform sampler; NULL: all 1
  RecordArgs rec;            // launches that record only
};

// The (channel, position) pairs of a channel list that deposit into a species.
constexpr int kMaxMatches = 3 * kMaxChannels;
struct ReplayArgs {
  Grid G;
  RecordArgs rec;
  const int* match;       // [7][kMaxMatches]: 4 * (index in the list of all channels) + position (1..3), ascending
  int first;              // index there of the sampling launch's first channel
  int n_group, n_chunks;  // as the sampling launch
  int n_wg;               // workgroups of the batch
  int n_cells;            // cells of the batch, from rec.cell_lo on
  int win_n, n_win;       // nodes per LDS window, windows
  int m_lo[kSpecies], m_hi[kSpecies];  // matches of each species within the batch
  int parts[kSpecies];                 // workgroups per (cell, species, window)
  double* A;
};

// Dynamic LDS of one precision's kernel variants.
struct LdsBudget {
  size_t plain[2] = {}, learned[2] = {};  // uniform sampler, learned sampler: [long, short items]
  size_t queue[2][2] = {};        // the compacting variant: [kRing, kTight][long, short items]
  size_t replay = 0;              // replay_kernel
  size_t roots = 0;               // the root samplers
};

// The paper's root parameterisation (FP64; alt: the alternative elimination);
// a launch's slots and window as for the CM-angle samplers.
hipError_t launch_collide_roots(const CollideArgs& a, bool alt, hipStream_t stream);
// queue: a form of the compacting variant (0: none), used if the launch
// qualifies (uniform sampler, symmetric, every accumulator in LDS within the
// queue's budget): with its queue as a ring in LDS, or in fewer bytes.
constexpr int kRing = 1, kTight = 2;
hipError_t launch_collide_f32(const CollideArgs& a, int nslot, int queue, hipStream_t stream);
hipError_t launch_collide_f64(const CollideArgs& a, int nslot, int queue, hipStream_t stream);
// Sample a batch of n_wg workgroups (a.rec.wg_base onwards) and record the
// deposits instead of adding them: symmetric sampling without the scale
// output, short-item form.
hipError_t launch_record_f32(const CollideArgs& a, int n_wg, hipStream_t stream);
hipError_t launch_record_f64(const CollideArgs& a, int n_wg, hipStream_t stream);
// The root samplers record up to two deposits per sample, in FP64.
hipError_t launch_record_roots(const CollideArgs& a, bool alt, int n_wg, hipStream_t stream);
// Bytes of 64 records.
size_t collide_f32_record_tile();
size_t collide_f64_record_tile();
// Add the recorded deposits of a batch to A.
hipError_t launch_replay_f32(const ReplayArgs& a, hipStream_t stream);
hipError_t launch_replay_f64(const ReplayArgs& a, hipStream_t stream);
// Raise the kernels' dynamic LDS limit to what their static LDS leaves of
// lds_max; returns the dynamic budgets.
hipError_t collide_roots_lds_limit(size_t lds_max, size_t* out);
hipError_t collide_f32_lds_limit(size_t lds_max, LdsBudget* out);
hipError_t collide_f64_lds_limit(size_t lds_max, LdsBudget* out);
// Waves per workgroup of the kernel (chunks are multiples of it).
int collide_waves(bool queue);
// Consecutive observed nodes a wave of the long-item form takes at a time
// (its chunks must be multiples of it; multiples of the waves are).
int collide_node_block(bool queue);
// Whether a launch takes the short-item form.
bool collide_short(int precision, bool learned, int split, int n_samples);
hipError_t launch_record(const CollideArgs& a, int n_per_item, long long item_stride, long long n_sel, float* rows,
                         hipStream_t stream);

}  // namespace qgbe
