// The collision kernel: the CM-angle samplers in both precisions and the root
// samplers, and the replay of recorded deposits.
#pragma once

#include <algorithm>
#include <type_traits>
#include <vector>

#include "collide_device.h"

namespace qgbe {
namespace {

// ---------------------------------------------------------------------------
// A workgroup owns (cell, channel, a chunk of observed nodes).  LDS holds FP64
// accumulators for the deposit slots of the launch (all of the channel's, or a
// part of them, or a window of their nodes) and, in FP32, f tiles for the first
// `lds_tiles` slots; the others are read from global memory.  The accumulators
// are flushed into the FP64 output once per workgroup.  On the largest grids the
// FP64 kernels deposit with global atomics instead (see deposit_route).
//
// R = double is the reference precision: the integrand in FP64 and f from the
// FP64 field in global memory.  It is bound as FP32 is, by VALU issue and the
// LDS atomics; with every deposit a global FP64 atomic, which the XCDs' shared
// rows send past the L2 (20 G atomics/s), it took 38.3 instead of 2.3 ms on 7
// species, 12 cells of 11x12x10 nodes, 64 samples; 1510 instead of 82 us on a
// 20^3 gluon cell, 256 samples; 6.2 instead of 0.8 ms with the learned sampler
// (7 species, 12^3, 64 samples).
// ---------------------------------------------------------------------------
// Trilinear read from the node quads: the same corners and the same
// arithmetic as interpolate, in two 16-byte loads.
template <typename R>
__device__ __forceinline__ R interpolate_quads(const float4* __restrict__ q4, const Stencil<R>& st, int ox) {
  typedef float V4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(1))) const V4 GlobalV4;
  const V4 lo = ((GlobalV4*)q4)[st.base];
  const V4 hi = ((GlobalV4*)q4)[st.base + ox];
  const R a00 = (R)lo.x + st.wz * ((R)lo.y - (R)lo.x);
  const R a01 = (R)lo.z + st.wz * ((R)lo.w - (R)lo.z);
  const R a10 = (R)hi.x + st.wz * ((R)hi.y - (R)hi.x);
  const R a11 = (R)hi.z + st.wz * ((R)hi.w - (R)hi.z);
  const R b0 = a00 + st.wy * (a01 - a00);
  const R b1 = a10 + st.wy * (a11 - a10);
  return b0 + st.wx * (b1 - b0);
}

// Trilinear read from the FP64 field: the corners in pairs along z, four
// 16-byte loads (8-byte aligned) instead of eight.
__device__ __forceinline__ double interpolate_pairs(const double* __restrict__ f, const Stencil<double>& st, int ox,
                                                    int oy) {
  typedef double V2 __attribute__((ext_vector_type(2), aligned(8)));
  typedef __attribute__((address_space(1))) const V2 GlobalV2;
  const double* q = f + st.base;
  const V2 f00 = *(GlobalV2*)q, f01 = *(GlobalV2*)(q + oy), f10 = *(GlobalV2*)(q + ox), f11 = *(GlobalV2*)(q + ox + oy);
  const double a00 = f00.x + st.wz * (f00.y - f00.x);
  const double a01 = f01.x + st.wz * (f01.y - f01.x);
  const double a10 = f10.x + st.wz * (f10.y - f10.x);
  const double a11 = f11.x + st.wz * (f11.y - f11.x);
  const double b0 = a00 + st.wy * (a01 - a00);
  const double b1 = a10 + st.wy * (a11 - a10);
  return b0 + st.wx * (b1 - b0);
}

template <bool kAllLds, typename R>
__device__ __forceinline__ R interp_slot(int k, int n_tiles, const float* tiles, const float4* __restrict__ f32q,
                                         size_t off, const Stencil<R>& st, int nodes, int ox, int oy) {
  // an address-space-qualified view keeps the LDS reads ds_read instructions
  // instead of generic flat loads
  typedef __attribute__((address_space(3))) const float LdsF32;
  if (kAllLds || k < n_tiles) return interpolate<R>((LdsF32*)(tiles + k * nodes), st, ox, oy);
  return interpolate_quads<R>(f32q + off, st, ox);
}

// The corner values are split in FP64 from the FP32 value and weights (both
// convert exactly), so the deposits of a sample cancel to FP64 rounding.
__device__ __forceinline__ Stencil<double> widen(const Stencil<float>& st) {
  return Stencil<double>{st.base, (double)st.wx, (double)st.wy, (double)st.wz};
}
__device__ __forceinline__ const Stencil<double>& widen(const Stencil<double>& st) { return st; }

template <bool kAccLds, bool kWin, typename R>
__device__ __forceinline__ void deposit_slot(int k, int slot_lo, int slot_hi, double* acc,
                                             double* __restrict__ out, size_t off, const Stencil<R>& st,
                                             R v, int nodes, int ox, int oy, int win_lo, int win_n) {
  if (k < slot_lo || k >= slot_hi) return;  // deposited by another launch
  const int j = k - slot_lo;
  if (kAccLds) {
    if (!kWin || win_n == nodes)  // (wave-uniform) the whole grid in LDS
      deposit<double, double, __HIP_MEMORY_SCOPE_WORKGROUP>(acc + j * win_n, widen(st), (double)v, ox, oy);
    else
      deposit_window(acc + j * win_n, widen(st), (double)v, ox, oy, win_lo, win_n);
  } else {
    deposit<double, double>(out + off, widen(st), (double)v, ox, oy);
  }
}

// Workgroups are dispatched to the 8 XCDs in turn (workgroup b to XCD b mod
// 8), and each XCD has its own L2.  The logical index hands each XCD a
// contiguous range of (cell, channel, chunk) work, so the workgroups that
// read a cell's f quads and flush into its output rows share one L2.
__device__ __forceinline__ int xcd_local_block(int b, int n) {
  constexpr int kXcd = 8;
  const int q = n / kXcd, r = n % kXcd, x = b % kXcd;
  return x * q + min(x, r) + b / kXcd;
}

// Workgroup size: 12 waves, 3 per SIMD (the register budget is then 168
// VGPRs; the learned variant spills a few to scratch and still runs faster
// than with 8 waves), for both samplers.
constexpr int kSlotThreads = 768;
// The compacting variant (below) keeps a sample queue per wave in LDS next to
// the accumulators and reads f from the global node quads.  Two forms: kRing
// has room for a batch and 64 more (52 B x 128 per wave in FP32); kTight holds
// one batch, its p2 words in registers (40 B x 64), for accumulators that fit
// only so.  Where both fit the ring is faster (256 gluon cells of 20^3, 2048
// samples: 60.0 and 62.0 ms); against no queue kTight gains what compaction
// does (7 species at 20^3, 4096 samples, the two-slot channels: 29.8 -> 24.1
// ms, the term 48.4 -> 42.7).
constexpr int kQueueWaves = 12;
constexpr int kQueueLen = 128;  // kRing: entries per wave (>= 63 pending + 64 new)
constexpr int queue_len(int queue) { return queue == kRing ? kQueueLen : queue == kTight ? kWave : 1; }
constexpr int slots_block(bool queue) { return queue ? kQueueWaves * 64 : kSlotThreads; }
// Long items, compacting variant: observed nodes go to the waves of a
// workgroup in blocks of 4 consecutive nodes; a wave stages the direct sums
// of its block in LDS and adds them to the output with one atomic
// instruction over one 32-byte sector, instead of one single-lane atomic
// (counted as a whole sector) per node.  The plain long variants keep one
// node per wave in turn and one atomic per node: there the block order cost
// 5% (the three-slot variant's sample loop compiled to more instructions).
constexpr int kNodeBlock = 4;

// kQueue (uniform sampler, every deposit slot in LDS, f from the global node
// quads): each wave first runs the sample geometry for 64 samples, appends
// the accepted ones (the three 23-bit uniforms of p2, p3 in FP64, s, t, u and
// the prefactor in FP32) to its queue, and evaluates |M|^2, f, bracket
// and deposits 64 queued samples at a time, so that long path runs on full
// wavefronts.  The deposits of one such batch are issued while the geometry
// of the next 64 samples runs, a third before, between and after it, so the
// LDS works off the atomics behind VALU work.  Same arithmetic per sample as
// the direct loop.
// kUser: some row of the matrix-element table is replaced by user terms; the
// variants without them carry no code for the user-term evaluation (which
// otherwise holds registers across the sample loop: 6% of the 7-species term).
// kShort: short items, bound by the latency of an item's serial parts (three
// wavefronts per SIMD): its constants, its sums, its partly filled batches.
// The (cell, channel) constants are computed once per workgroup; a wave takes
// A.node_block consecutive nodes at a time, computes their constants side by
// side, a node per lane, and keeps them and the nodes' sums in LDS, so that
// the variances and outputs of the block are side by side too; and several
// waves may share a node (A.split).  The learned sampler is in this form at any
// length (unless A.long_form); a long uniform item is not: what it holds across
// its item loop costs more spilled registers in the sample loop than it saves.  One gluon cell,
// collision term: 10^3 nodes x 1000 samples 255 -> 46 us, 16^3 x 2048 547 ->
// 190 us, 20^3 x 256 98 -> 78 us; 7 species, 30^3 x 128 20.9 -> 19.5 ms.
// ---------------------------------------------------------------------------
// The paper's own parameterisation (Eq. work out delta E, Eq. delta replace):
// momentum conservation eliminates one momentum, energy conservation fixes
// one z component at the two roots of a quadratic, and each root carries
// 1/|J|.  In channel order k1 + k2 <-> k3 + k4 with k1 observed (the
// paper's p):
//   kAlt = false, the paper's choice: k2 uniform in the box, k3x and k3y
//     uniform, k4 = k1 + k2 - k3; E1 + E2 = E3 + E4 has the roots
//     z = (c Qz +- W sqrt(c^2 - 4 a (W^2 - Qz^2))) / (2 (W^2 - Qz^2)) with
//     W = E1 + E2 > 0, Q = k1 + k2, a = k3x^2 + k3y^2 + m3^2,
//     c = W^2 + a - (Qx - k3x)^2 - (Qy - k3y)^2 - m4^2 - Qz^2; a root holds
//     when c + 2 Qz z > 0 and E3 < W;
//   kAlt = true, the alternative the paper tests (Sec. IV A): k4 uniform in
//     the box, k3x and k3y uniform, k2 = k3 + k4 - k1; E3 - E2 = D = E1 - E4
//     gives z = (-C Qz +- |D| sqrt(C^2 + 4 a (Qz^2 - D^2))) / (2 (Qz^2 - D^2))
//     with Q = k4 - k1, C = 2 (k3x Qx + k3y Qy) + Q^2 + m2^2 - m3^2 - D^2; a
//     root holds when (C + 2 Qz z) D < 0 and E3 > D.  Its leading
//     coefficient has no fixed sign: the instability the paper reports.
// The value of a root is w V5 / N |M|^2 B / ((2 pi)^5 16 E1 E2 E3 E4 |J|),
// V5 = (2 P)^3 (2 Px) (2 Py), J the z derivative of the energy sum.  FP64
// throughout (f from the FP64 field, FP64 accumulators): the reference method.
// Every lane draws a sample and solves for its roots; samples with a valid
// root go to a per-wavefront queue in LDS (five 23-bit uniforms, both roots and
// which hold: 36 B), and whenever 64 are queued (and at the end of the item)
// the wavefront evaluates them on full lanes, the first valid root of every
// sample and then the second of those that have two.
// Deposits and launches as for the CM-angle samplers.  Bound by VALU issue
// (three wavefronts per SIMD; with workgroups of four and two per SIMD, and
// global FP64 atomics beyond 1170 points, before): 64000 gluon nodes x 100
// samples, direct, 262 -> 184 us a call; 7 species at 15^3 x 100, symmetric,
// 10.6 ms -> 0.76 ms, at 20^3 23.5 -> 2.5 ms, at 30^3 x 20 15.0 -> 5.6 ms.
// ---------------------------------------------------------------------------
constexpr double kRootNorm = 1.0 / (32.0 * kPi * kPi * kPi * kPi * kPi * 16.0);

// A sample's two root candidates: z and whether each holds (bits 0 and 1).
template <bool kAlt>
__device__ __forceinline__ uint32_t solve_roots(const Item& it, const Grid& G, const double u[5], double zr[2]) {
  double q[3];
  for (int a = 0; a < 3; ++a) q[a] = fma(2.0 * G.ph[a], u[a], -G.ph[a]);
  const double k3x = fma(2.0 * G.ph[0], u[3], -G.ph[0]);
  const double k3y = fma(2.0 * G.ph[1], u[4], -G.ph[1]);
  const double a3 = k3x * k3x + k3y * k3y + it.m3sq;
  const double Eq = sqrt64(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + (kAlt ? it.m4sq : it.m2sq));
  double Q[3], lin, half, den, W = 0.0, D = 0.0, C = 0.0;
  bool any;
  if (!kAlt) {
    W = it.E1 + Eq;
    for (int a = 0; a < 3; ++a) Q[a] = it.p1[a] + q[a];
    const double b = (Q[0] - k3x) * (Q[0] - k3x) + (Q[1] - k3y) * (Q[1] - k3y) + it.m4sq;
    C = W * W + a3 - b - Q[2] * Q[2];
    den = W * W - Q[2] * Q[2];
    const double H = C * C - 4.0 * a3 * den;
    any = H >= 0.0 && den > 0.0;
    lin = C * Q[2];
    half = any ? W * sqrt64(H) : 0.0;
  } else {
    D = it.E1 - Eq;
    for (int a = 0; a < 3; ++a) Q[a] = q[a] - it.p1[a];
    C = 2.0 * (k3x * Q[0] + k3y * Q[1]) + (Q[0] * Q[0] + Q[1] * Q[1] + Q[2] * Q[2]) + it.m2sq - it.m3sq - D * D;
    den = Q[2] * Q[2] - D * D;
    const double H = C * C + 4.0 * a3 * den;
    any = H >= 0.0 && den != 0.0 && D != 0.0;
    lin = -C * Q[2];
    half = any ? fabs(D) * sqrt64(H) : 0.0;
  }
  const double inv_2den = any ? rcp64(2.0 * den) : 0.0;
  uint32_t roots = 0;
  for (int r = 0; r < 2; ++r) {
    const double z = (lin + (r == 0 ? half : -half)) * inv_2den;
    const double E3 = sqrt64(a3 + z * z);
    bool ok = any;
    if (!kAlt) ok = ok && (C + 2.0 * Q[2] * z > 0.0) && (E3 < W);
    else ok = ok && ((C + 2.0 * Q[2] * z) * D < 0.0) && (E3 - D > 0.0);
    const double p3[3] = {k3x, k3y, z};
    for (int a = 0; a < 3; ++a) {
      const double other = kAlt ? p3[a] + Q[a] : Q[a] - p3[a];  // p2 or p4
      ok = ok && fabs(p3[a]) <= G.ph[a] && fabs(other) <= G.ph[a];
    }
    zr[r] = z;
    if (ok) roots |= 1u << r;
  }
  return roots;
}

// Momenta of the root z of a sample, and 1 / (E2 E3 E4 |J|) in place of the
// prefactor's p*/(sqrt s E2); s, t, u.
template <bool kAlt>
__device__ __forceinline__ double root_geometry(const Item& it, const Grid& G, const double u[5], double z, Geo& g) {
  double q[3];
  for (int a = 0; a < 3; ++a) q[a] = fma(2.0 * G.ph[a], u[a], -G.ph[a]);
  g.p3[0] = fma(2.0 * G.ph[0], u[3], -G.ph[0]);
  g.p3[1] = fma(2.0 * G.ph[1], u[4], -G.ph[1]);
  g.p3[2] = z;
  const double Eq = sqrt64(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + (kAlt ? it.m4sq : it.m2sq));
  const double E3 = sqrt64(g.p3[0] * g.p3[0] + g.p3[1] * g.p3[1] + it.m3sq + z * z);
  double E2, E4, J;
  if (!kAlt) {
    for (int a = 0; a < 3; ++a) {
      g.p2[a] = q[a];
      g.p4[a] = it.p1[a] + q[a] - g.p3[a];
    }
    E2 = Eq;
    E4 = sqrt64(g.p4[0] * g.p4[0] + g.p4[1] * g.p4[1] + g.p4[2] * g.p4[2] + it.m4sq);
    J = fabs(z * rcp64(E3) - g.p4[2] * rcp64(E4));
  } else {
    for (int a = 0; a < 3; ++a) {
      g.p4[a] = q[a];
      g.p2[a] = g.p3[a] + (q[a] - it.p1[a]);
    }
    E4 = Eq;
    E2 = sqrt64(g.p2[0] * g.p2[0] + g.p2[1] * g.p2[1] + g.p2[2] * g.p2[2] + it.m2sq);
    J = fabs(g.p2[2] * rcp64(E2) - z * rcp64(E3));
  }
  double Pq[3], d13[3], d14[3];
  for (int a = 0; a < 3; ++a) {
    Pq[a] = it.p1[a] + g.p2[a];
    d13[a] = it.p1[a] - g.p3[a];
    d14[a] = it.p1[a] - g.p4[a];
  }
  const double E12 = it.E1 + E2, E13 = it.E1 - E3, E14 = it.E1 - E4;
  g.s = E12 * E12 - (Pq[0] * Pq[0] + Pq[1] * Pq[1] + Pq[2] * Pq[2]);
  g.t = E13 * E13 - (d13[0] * d13[0] + d13[1] * d13[1] + d13[2] * d13[2]);
  g.u = E14 * E14 - (d14[0] * d14[0] + d14[1] * d14[1] + d14[2] * d14[2]);
  return rcp64(E2 * E3 * E4 * J);
}

// One record of RecordArgs: three weights per position and the value, then
// the three base nodes.
template <typename R>
struct Record {
  static constexpr size_t kTileBytes = 64 * (10 * sizeof(R) + 3 * sizeof(uint32_t));
  R* w;            // [10][64]
  uint32_t* base;  // [3][64]
  __device__ __forceinline__ Record(unsigned char* tiles, long long i) {
    unsigned char* t = tiles + (i >> 6) * (long long)kTileBytes;
    w = (R*)t + (i & 63);
    base = (uint32_t*)(t + 640 * sizeof(R)) + (i & 63);
  }
  __device__ __forceinline__ void store(int pos, const Stencil<R>& st) const {
    base[pos * 64] = (uint32_t)st.base;
    w[(3 * pos) * 64] = st.wx;
    w[(3 * pos + 1) * 64] = st.wy;
    w[(3 * pos + 2) * 64] = st.wz;
  }
  __device__ __forceinline__ Stencil<R> load(int pos) const {
    return Stencil<R>{(int)base[pos * 64], w[(3 * pos) * 64], w[(3 * pos + 1) * 64], w[(3 * pos + 2) * 64]};
  }
};

// kRec: the deposits go to A.rec instead of accumulators (see replay_kernel).
// kRoot: 0 the CM-angle samplers, 1 the root parameterisation, 2 its
// alternative (FP64, short form, their own queue; deposits issued at once).
template <typename R, bool kSym, bool kScale, bool kAllLds, bool kLearned, int kQueue, bool kUser, bool kShort,
          bool kRec = false, int kRoot = 0>
__global__ __launch_bounds__(slots_block(kQueue)) void collide_slots_kernel(CollideArgs A) {
  constexpr bool kF64 = std::is_same<R, double>::value;
  static_assert(!kRoot || (kF64 && kShort && !kLearned && !kQueue), "the root samplers: FP64, short form");
  static_assert(!kQueue || (kSym && kAllLds && !kLearned), "the queue serves the uniform sampler, slots in LDS");
  static_assert(!kRec || (kSym && !kScale && kShort), "deposits are recorded in the short form");
  // kAllLds: FP32: every f tile in LDS (not in the queue variant: f from the
  // quads); FP64: the accumulators in LDS
  constexpr bool kTilesLds = kAllLds && !kQueue && !kF64 && !kRec;
  constexpr bool kAccLds = kAllLds || !kF64;
  extern __shared__ double lds[];
  __shared__ R mix_rows[kLearned ? kSlotThreads / kWave : 1][kLearned ? (kF64 ? kMixRowF64 : kMixRow) : 1];
  __shared__ uint32_t q_v[kQueue == kRing ? kQueueWaves : 1][3][kQueue == kRing ? kQueueLen : 1];  // 23-bit uniforms of p2
  __shared__ double q_p3[kQueue ? kQueueWaves : 1][3][queue_len(kQueue)];
  __shared__ R q_f[kQueue ? kQueueWaves : 1][4][queue_len(kQueue)];    // s, t, u, prefactor
  __shared__ uint32_t r_v[kRoot ? kQueueWaves : 1][5][kRoot ? kQueueLen : 1];  // 23-bit uniforms; which roots hold
  __shared__ double r_z[kRoot ? kQueueWaves : 1][2][kRoot ? kQueueLen : 1];    // the roots
  __shared__ double mc_wg[2];  // this workgroup's item variances and squared item sums
  __shared__ unsigned long long ok_wg;  // and its accepted samples
  __shared__ unsigned rec_n;            // kRec: records of this workgroup
  constexpr int kNB = kQueue && !kShort ? kNodeBlock : 1;  // nodes per block (as collide_node_block)
  __shared__ double d_stage[kNB > 1 ? kSlotThreads / kWave : 1][kNB];  // direct sums of a wave's current block
  static_assert(slots_block(kQueue) % (kWave * kNB) == 0, "a multiple of the waves is one of the block");
  // kShort: constants (p1, E1, f1, prefactor) of a wave's current nodes; a node that is done holds its sums (S_i,
  // sum v^2, gain + loss) in the last three
  __shared__ double node_tab[kShort ? kSlotThreads / kWave : 1][6][kShort ? kMaxNodeBlock : 1];
  __shared__ double it_sum[3][kShort ? kSplitNodes : 1];  // A.split > 1: S_i, sum v^2 and the gain+loss sum of the chunk's items
  const Grid& G = A.G;
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = threadIdx.x / kWave;
  const int nw = blockDim.x / kWave;
  const int lb = (kRec ? A.rec.wg_base : 0) + xcd_local_block(blockIdx.x, gridDim.x);
  const int chunk = lb % A.n_chunks;
  // Uniform sampler: the chunks and channels of one cell follow each other
  // (they share its f quads and output rows in the XCD's L2).  Learned
  // sampler: blocks of 32 cells (the workgroups one XCD holds at a time),
  // and within a block the cells of one channel follow each other, so the
  // channel's proposal rows, shared by all cells, are read from HBM about
  // once per block instead of once per cell, and the block's f rows serve
  // every channel.
  int gi, cell;
  if (kLearned && !kRec) {
    constexpr int kCellBlock = 32;
    const int u = lb / A.n_chunks;
    const int per = A.n_group * kCellBlock;
    const int cb = u / per;
    const int S = min(kCellBlock, G.cells - cb * kCellBlock);  // the last block may be short
    const int r = u - cb * per;
    gi = r / S;
    cell = cb * kCellBlock + r % S;
  } else {
    gi = (lb / A.n_chunks) % A.n_group;
    cell = (kRec ? A.rec.cell_lo : 0) + lb / (A.n_chunks * A.n_group);
  }
  const int ci = A.group[gi];
  const Channel ch = A.chans[ci];
  const int nslot = ch.nslot;
  const int nodes = G.nodes;
  const int n_acc = kSym && !kRec ? min(A.slot_hi - A.slot_lo, A.lds_acc) : 0;
  const int n_tiles = kRec ? 0 : min(nslot, A.lds_tiles);
  const int win_lo = A.win_lo, win_n = A.win_n;
  double* acc = lds;                                          // [n_acc][win_n], slots slot_lo..
  float* tiles = reinterpret_cast<float*>(lds + (size_t)n_acc * win_n);  // [n_tiles][nodes]
  size_t goff[3];  // offsets of the slots' (species, cell) rows in f32 and A
  for (int k = 0; k < 3; ++k) {
    const int sp = k < nslot ? ch.slot_sp[k] : ch.slot_sp[0];
    goff[k] = ((size_t)sp * G.cells + cell) * nodes;
  }
  for (int i = threadIdx.x; i < n_acc * win_n; i += blockDim.x) acc[i] = 0.0;
  if (threadIdx.x < 2) mc_wg[threadIdx.x] = 0.0;
  if (threadIdx.x == 0) {
    ok_wg = 0ull;
    rec_n = 0u;
  }
  if (kNB > 1 && lane < kNB) d_stage[wid][lane] = 0.0;
  const int split = kShort ? A.split : 1;
  if (kShort && split > 1)
    for (int i = threadIdx.x; i < 3 * kSplitNodes; i += blockDim.x) it_sum[i / kSplitNodes][i % kSplitNodes] = 0.0;
  for (int k = 0; k < n_tiles; ++k)
    for (int i = threadIdx.x; i < nodes; i += blockDim.x) tiles[k * nodes + i] = A.f32[goff[k] + i];
  __syncthreads();
  const int k2 = ch.pos_slot[0], k3 = ch.pos_slot[1], k4 = ch.pos_slot[2];
  // row offsets of positions 2, 3, 4 (scalars: no dynamically indexed array in the loop)
  const size_t off2 = goff[k2], off3 = goff[k3], off4 = goff[k4];
  // 1 + f (gluons) or 1 - f, as one fma(+-1, f, 1): a select of the two is a
  // branch per factor (256 gluon cells of 20^3, 2048 samples: 59.6 -> 59.0 ms).
  // Not where the learned sampler records: there the signs' registers cost 0.6%.
  auto occupied = [&](int sp, R f) {
    if constexpr (kRec && kLearned) return is_gluon(sp) ? R(1) + f : R(1) - f;
    else return fma(is_gluon(sp) ? R(1) : R(-1), f, R(1));
  };
  const int first = chunk * A.chunk_items;
  const int last = min(first + A.chunk_items, nodes);
  Item pair;
  if (kShort) item_pair(pair, A, ch, cell);
  if (kRoot)  // V5 and the norm of a root's value in place of the CM form's
    pair.coef = (A.symmetric ? ch.w : ch.sigma) * (G.Vp * (2.0 * G.ph[0]) * (2.0 * G.ph[1])) / (double)A.n_samples *
                (kRootNorm / kNorm);
  // After the item at node p, the last of its node block (or of the chunk):
  // the wave adds the block's staged direct sums to the output, the lanes of
  // one atomic instruction covering consecutive nodes.
  auto flush_block = [&](int p) {
    if (kNB == 1 || !A.direct || ((p & (kNB - 1)) != kNB - 1 && p + 1 < last)) return;
    wave_lds_sync();
    if (lane < kNB) {
      const double d = d_stage[wid][lane];
      if (d != 0.0) atomicAdd(A.A + ((size_t)ch.sp[0] * G.cells + cell) * nodes + (p & ~(kNB - 1)) + lane, d);
      d_stage[wid][lane] = 0.0;
    }
    wave_lds_sync();
  };
  const long long rec0 = kRec ? (long long)(lb - A.rec.wg_base) * A.rec.region : 0;
  // kRec: the active lanes append their samples' deposits to the workgroup's records.
  auto record = [&](const Stencil<R>& s2, const Stencil<R>& s3, const Stencil<R>& s4, R v) {
    const unsigned long long m = __ballot(1);
    const int rank = __popcll(m & ((1ull << lane) - 1ull));
    unsigned at = 0;
    if (rank == 0) at = __hip_atomic_fetch_add(&rec_n, (unsigned)__popcll(m), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    at = (unsigned)__builtin_amdgcn_readfirstlane((int)at);
    const Record<R> r(A.rec.tiles, rec0 + at + rank);
    r.store(0, s2);
    r.store(1, s3);
    r.store(2, s4);
    r.w[9 * 64] = v;
  };
  int n_ok = 0;  // accepted samples: of the item, kShort of the wave
  const int s_first = split > 1 ? (wid % split) * kWave : 0, s_step = split * kWave;
  const size_t row1 = ((size_t)ch.sp[0] * G.cells + cell) * nodes;  // the observed species' output row
  // The samples of the observed node p1_lin; kShort: the j-th of the wave's
  // block, its constants in node_tab, where it leaves its sums.
  auto run_node = [&](const int p1_lin, const int j) __attribute__((always_inline)) {
    Item it;
    if (kShort) {
      it = pair;
      it.p1_lin = p1_lin;
      for (int a = 0; a < 3; ++a) it.p1[a] = node_tab[wid][a][j];
      it.E1 = node_tab[wid][3][j];
      it.f1 = node_tab[wid][4][j];
      it.pref = node_tab[wid][5][j];
    } else {
      load_item(it, A, ch, cell, p1_lin);
    }
    if (!(it.E1 > 0.0)) {  // massless p = 0 node: zero measure
      if (kShort) {
        if (lane < 3) node_tab[wid][3 + lane][j] = 0.0;
        return;
      }
      if (lane == 0 && A.items && A.direct) A.items[((size_t)cell * A.n_channels + ci) * nodes + p1_lin] = 0.0;
      flush_block(p1_lin);
      return;
    }
    const R f1 = (R)it.f1;
    const R F1 = occupied(ch.sp[0], f1);
    double dsum = 0.0, ssum = 0.0, dsq = 0.0;
    if (!kShort) n_ok = 0;
    const size_t mrow = (size_t)ci * nodes + p1_lin;
    const bool mix = kLearned && (!A.mix_on || A.mix_on[ci]);
    if (mix) {
      const uint32_t* thr = A.mix_thr + mrow * A.mix_K;
      const float *mu = A.mix_mu + mrow * A.mix_K * 5, *sg = A.mix_sigma + mrow * A.mix_K * 5;
      if constexpr (kF64) mix_prepare_f64(thr, mu, sg, A.mix_K, mix_rows[wid], lane);
      else mix_prepare_f32(thr, mu, sg, A.mix_K, mix_rows[wid], lane);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    // Queue mode: the deposits of the last evaluated batch, issued while the
    // next samples' geometry runs.
    Stencil<R> pd2{}, pd3{}, pd4{};
    R pdv = R(0);
    bool pending = false;
    // Integrand, direct sum and deposits of an accepted sample (wnb = value
    // without the bracket).
    auto finish = [&](const Geo& g, R wnb) {
      ++n_ok;
      const Stencil<R> s2 = make_stencil<R>(g.p2, G);
      const Stencil<R> s3 = make_stencil<R>(g.p3, G);
      const Stencil<R> s4 = make_stencil<R>(g.p4, G);
      R f2, f3, f4;
      if constexpr (kF64) {
        f2 = interpolate_pairs(A.f64 + off2, s2, G.ox, G.oy);
        f3 = interpolate_pairs(A.f64 + off3, s3, G.ox, G.oy);
        f4 = interpolate_pairs(A.f64 + off4, s4, G.ox, G.oy);
      } else {
        f2 = interp_slot<kTilesLds, R>(k2, n_tiles, tiles, A.f32q, off2, s2, nodes, G.ox, G.oy);
        f3 = interp_slot<kTilesLds, R>(k3, n_tiles, tiles, A.f32q, off3, s3, nodes, G.ox, G.oy);
        f4 = interp_slot<kTilesLds, R>(k4, n_tiles, tiles, A.f32q, off4, s4, nodes, G.ox, G.oy);
      }
      const R F2 = occupied(ch.sp[1], f2);
      const R F3 = occupied(ch.sp[2], f3);
      const R F4 = occupied(ch.sp[3], f4);
      const R gain = f3 * f4 * F1 * F2, loss = f1 * f2 * F3 * F4;
      const R v = wnb * (gain - loss);
      dsum += (double)v;
      if (!kRoot) dsq = fma((double)v, (double)v, dsq);  // a root sample's value is the sum over its roots
      const R vs = (wnb < R(0) ? -wnb : wnb) * (gain + loss);
      if (kScale) ssum += (double)vs;
      if (kSym) {
        if (kRec) {
          record(s2, s3, s4, v);
        } else if (kQueue) {
          pd2 = s2; pd3 = s3; pd4 = s4; pdv = v;
        } else {
          deposit_slot<kAccLds, true, R>(k2, A.slot_lo, A.slot_hi, acc, A.A, off2, s2, v,
                                nodes, G.ox, G.oy, win_lo, win_n);
          deposit_slot<kAccLds, true, R>(k3, A.slot_lo, A.slot_hi, acc, A.A, off3, s3, -v,
                                nodes, G.ox, G.oy, win_lo, win_n);
          deposit_slot<kAccLds, true, R>(k4, A.slot_lo, A.slot_hi, acc, A.A, off4, s4, -v,
                                nodes, G.ox, G.oy, win_lo, win_n);
        }
        if (kScale && A.direct) {
          deposit<double, double>(A.scale + ((size_t)ch.sp[1] * G.cells + cell) * nodes, widen(s2), (double)vs, G.ox, G.oy);
          deposit<double, double>(A.scale + ((size_t)ch.sp[2] * G.cells + cell) * nodes, widen(s3), (double)vs, G.ox, G.oy);
          deposit<double, double>(A.scale + ((size_t)ch.sp[3] * G.cells + cell) * nodes, widen(s4), (double)vs, G.ox, G.oy);
        }
      }
    };
    if constexpr (kRoot != 0) {
      constexpr bool kAlt = kRoot == 2;
      // The value of one queued sample: the sum over its valid roots, with
      // their deposits.
      auto finish_roots = [&](int slot) {
        const uint32_t v0 = r_v[wid][0][slot];
        double u[5];
        u[0] = unif23(v0 & 0x7FFFFFu);
        for (int a = 1; a < 5; ++a) u[a] = unif23(r_v[wid][a][slot]);
        const uint32_t roots = v0 >> 23;
        const double z0 = r_z[wid][0][slot], z1 = r_z[wid][1][slot];
        const double d0 = dsum;
        double vs2 = 0.0;
#pragma unroll 1
        for (int r = 0; r < 2; ++r) {
          if (r == 1 && roots != 3u) continue;
          const double z = r == 0 && (roots & 1u) ? z0 : z1;
          Geo g;
          const double w = root_geometry<kAlt>(it, G, u, z, g);
          const double m = msq_row<double, kUser>(A.msq_mask, A.msq, ch.row, g.s, g.t, g.u, it.mu);
          finish(g, it.pref * m * w);
        }
        vs2 = dsum - d0;
        dsq = fma(vs2, vs2, dsq);
      };
      unsigned head = 0, tail = 0;  // ring positions (wave-uniform)
      for (int base = s_first; base < A.n_samples; base += s_step) {
        const int s = base + lane;
        uint32_t x0 = (uint32_t)s, x1 = (uint32_t)p1_lin, x2 = (uint32_t)cell, x3 = ((uint32_t)ch.code << 8) | 2u;
        philox4x32_10(x0, x1, x2, x3, A.key0, A.key1);
        double u[5], zr[2];
        five_uniforms(x0, x1, x2, x3, u);
        uint32_t roots = 0;
        if (s < A.n_samples) roots = solve_roots<kAlt>(it, G, u, zr);
        const unsigned long long mask = __ballot(roots != 0u);
        if (roots) {
          const unsigned slot = (tail + (unsigned)__popcll(mask & ((1ull << lane) - 1ull))) & (kQueueLen - 1);
          r_v[wid][0][slot] = (x0 >> 9) | (roots << 23);
          r_v[wid][1][slot] = x1 >> 9;
          r_v[wid][2][slot] = x2 >> 9;
          r_v[wid][3][slot] = x3 >> 9;
          r_v[wid][4][slot] = fifth_word(x0, x1, x2);
          r_z[wid][0][slot] = zr[0];
          r_z[wid][1][slot] = zr[1];
        }
        tail += (unsigned)__popcll(mask);
        if (tail - head >= (unsigned)kWave) {
          wave_lds_sync();
          finish_roots((head + lane) & (kQueueLen - 1));
          head += kWave;
          wave_lds_sync();
        }
      }
      if (tail != head) {  // the last, partial batch
        wave_lds_sync();
        if ((unsigned)lane < tail - head) finish_roots((head + lane) & (kQueueLen - 1));
        wave_lds_sync();
      }
    } else {
    auto evaluate = [&](const SampleMap& m, R inv_q) {
      Geo g;
      if (!geometry(it, G, m, g)) return;
      finish(g, weight_no_bracket<R, kUser>(A, it, g, ch.row) * inv_q);
    };
    if (kQueue) {
      // A queued sample: the words of p2, p3, and s, t, u and the prefactor.
      struct Queued {
        uint32_t v[3];
        double p3[3];
        R f[4];
      };
      auto push = [&](unsigned i, const Geo& g) {
        for (int a = 0; a < 3; ++a) q_p3[wid][a][i] = g.p3[a];
        q_f[wid][0][i] = (R)g.s;
        q_f[wid][1][i] = (R)g.t;
        q_f[wid][2][i] = (R)g.u;
        q_f[wid][3][i] = prefactor<R>(it, g);
      };
      auto pop = [&](unsigned i, uint32_t v0, uint32_t v1, uint32_t v2) {
        return Queued{{v0, v1, v2},
                      {q_p3[wid][0][i], q_p3[wid][1][i], q_p3[wid][2][i]},
                      {q_f[wid][0][i], q_f[wid][1][i], q_f[wid][2][i], q_f[wid][3][i]}};
      };
      auto pop_ring = [&](unsigned i) {
        i &= kQueueLen - 1;
        return pop(i, q_v[wid][0][i], q_v[wid][1][i], q_v[wid][2][i]);
      };
      auto finish_queued = [&](const Queued& q) {
        Geo g;
        for (int a = 0; a < 3; ++a) {
          g.p2[a] = G.ph[a] * centred23(q.v[a]);  // as map_words formed it
          g.p3[a] = q.p3[a];
          g.p4[a] = (it.p1[a] + g.p2[a]) - g.p3[a];
        }
        const R m = msq_row<R, kUser>(A.msq_mask, A.msq, ch.row, q.f[0], q.f[1], q.f[2], (R)it.mu);
        finish(g, m * q.f[3]);
      };
      unsigned head = 0, tail = 0;      // kRing: positions; kTight: tail samples are queued (wave-uniform)
      uint32_t w0 = 0, w1 = 0, w2 = 0;  // kTight: lane i holds the words of queue entry i
      for (int base = s_first; base < A.n_samples; base += s_step) {
        const int s = base + lane;
        uint32_t x0 = (uint32_t)s, x1 = (uint32_t)p1_lin, x2 = (uint32_t)cell, x3 = ((uint32_t)ch.code << 8);
        philox4x32_10(x0, x1, x2, x3, A.key0, A.key1);
        if (pending) deposit_slot<true, false, R>(k2, A.slot_lo, A.slot_hi, acc, A.A, off2, pd2, pdv,
                                        nodes, G.ox, G.oy, win_lo, win_n);
        const SampleMap map = map_words(G, x0, x1, x2, x3);
        Geo g;
        const bool ok = s < A.n_samples && geometry(it, G, map, g);
        if (pending) deposit_slot<true, false, R>(k3, A.slot_lo, A.slot_hi, acc, A.A, off3, pd3, -pdv,
                                        nodes, G.ox, G.oy, win_lo, win_n);
        // The accepted samples take the next places of the queue.
        const unsigned long long mask = __ballot(ok);
        const unsigned cnt = (unsigned)__popcll(mask);
        const unsigned rank = (unsigned)__popcll(mask & ((1ull << lane) - 1ull));
        const unsigned at = tail + rank;
        uint32_t m0 = x0 >> 9, m1 = x1 >> 9, m2 = x2 >> 9;
        if constexpr (kQueue == kRing) {
          if (ok) {
            const unsigned slot = at & (kQueueLen - 1);
            q_v[wid][0][slot] = m0;
            q_v[wid][1][slot] = m1;
            q_v[wid][2][slot] = m2;
            push(slot, g);
          }
        } else {
          // Places from 64 up are the first of the next batch: their entries
          // wait in registers until this batch has been read.  The words go to
          // their lanes by a permutation (place mod 64); the rejected samples'
          // land on empty places.
          if (ok && at < (unsigned)kWave) push(at, g);
          const int to = (int)((ok ? at : tail + cnt + lane - rank) << 2);
          m0 = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)m0);
          m1 = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)m1);
          m2 = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)m2);
          if ((unsigned)lane >= tail) {
            w0 = m0;
            w1 = m1;
            w2 = m2;
          }
        }
        if (pending) deposit_slot<true, false, R>(k4, A.slot_lo, A.slot_hi, acc, A.A, off4, pd4, -pdv,
                                        nodes, G.ox, G.oy, win_lo, win_n);
        pending = false;
        tail += cnt;
        if (tail - head >= (unsigned)kWave) {
          wave_lds_sync();
          if constexpr (kQueue == kRing) {
            finish_queued(pop_ring(head + lane));
            head += kWave;
          } else {
            const Queued q = pop(lane, w0, w1, w2);
            wave_lds_sync();
            if (ok && at >= (unsigned)kWave) push(at - kWave, g);
            w0 = m0;
            w1 = m1;
            w2 = m2;
            tail -= kWave;
            finish_queued(q);
          }
          pending = !kRec;
          wave_lds_sync();
        }
      }
      auto flush = [&]() {
        deposit_slot<true, false, R>(k2, A.slot_lo, A.slot_hi, acc, A.A, off2, pd2, pdv,
                           nodes, G.ox, G.oy, win_lo, win_n);
        deposit_slot<true, false, R>(k3, A.slot_lo, A.slot_hi, acc, A.A, off3, pd3, -pdv,
                           nodes, G.ox, G.oy, win_lo, win_n);
        deposit_slot<true, false, R>(k4, A.slot_lo, A.slot_hi, acc, A.A, off4, pd4, -pdv,
                           nodes, G.ox, G.oy, win_lo, win_n);
      };
      if (pending) flush();  // the last full batch
      // the last, partial batch: only the lanes that hold a sample deposit (zeros
      // of the idle lanes, all at one address, took 60 us of an 88 us launch of
      // 7722 items x 100 samples)
      if (tail != head) {
        wave_lds_sync();
        if ((unsigned)lane < tail - head) {
          if constexpr (kQueue == kRing) finish_queued(pop_ring(head + lane));
          else finish_queued(pop(lane, w0, w1, w2));
          if (!kRec) flush();
        }
        wave_lds_sync();
      }
      pending = false;
    } else
    for (int s = s_first + lane; s < A.n_samples; s += s_step) {
      uint32_t x0 = (uint32_t)s, x1 = (uint32_t)p1_lin, x2 = (uint32_t)cell, x3 = ((uint32_t)ch.code << 8);
      philox4x32_10(x0, x1, x2, x3, A.key0, A.key1);
      SampleMap map;
      R inv_q = R(1);
      if (mix) {
        double u[5];
        uint32_t y0 = (uint32_t)s, y1 = (uint32_t)p1_lin, y2 = (uint32_t)cell, y3 = ((uint32_t)ch.code << 8) | 1u;
        philox4x32_10(y0, y1, y2, y3, A.key0, A.key1);
        const uint32_t xw[8] = {x0, x1, x2, x3, y0, y1, y2, y3};
        R yl[5];
        if constexpr (kF64) {
          mix_draw_row_f64(xw, A.mix_thr + mrow * A.mix_K, mix_rows[wid], A.mix_K, u, yl);
          const double q = mix_density_f64(mix_rows[wid], A.mix_K, yl);
          inv_q = q > 1e300 ? 0.0 : rcp64(q);  // q >= alpha > 0; rcp64 is for finite arguments
        } else {
          mix_draw_row(xw, A.mix_thr + mrow * A.mix_K, mix_rows[wid], A.mix_K, u, yl);
          inv_q = __builtin_amdgcn_rcpf(mix_density_f32(mix_rows[wid], A.mix_K, yl));  // about 1 ulp; q >= alpha
        }
        map = map_unit(G, u);
      } else {
        map = map_words(G, x0, x1, x2, x3);
      }
      evaluate(map, inv_q);
    }
    }  // CM-angle samplers
    if (!A.direct) return;
    if (kShort) {
      dsum = wave_sum_dpp(dsum);
      if (kScale) ssum = wave_sum_dpp(ssum);
      dsq = wave_sum_dpp(dsq);
      if (lane == 0) {
        node_tab[wid][3][j] = dsum;
        node_tab[wid][4][j] = dsq;
        if (kScale) node_tab[wid][5][j] = ssum;
      }
      return;
    }
    dsum = wave_sum(dsum);
    if (kScale) ssum = wave_sum(ssum);
    dsq = wave_sum(dsq);
    const int ok_total = wave_count(n_ok);
    if (lane == 0) {
      __hip_atomic_fetch_add(&ok_wg, (unsigned long long)ok_total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      __hip_atomic_fetch_add(&mc_wg[0], item_variance(dsum, dsq, A.n_samples), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_WORKGROUP);
      __hip_atomic_fetch_add(&mc_wg[1], dsum * dsum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (kNB > 1)
        d_stage[wid][p1_lin & (kNB - 1)] = dsum;
      else
        atomicAdd(A.A + row1 + p1_lin, dsum);
      if (kScale) atomicAdd(A.scale + row1 + p1_lin, ssum);
      if (A.items) A.items[((size_t)cell * A.n_channels + ci) * nodes + p1_lin] = dsum;
    }
    flush_block(p1_lin);
  };
  // An item's sums into the outputs and the workgroup's totals.
  auto finish_item = [&](int p1_lin, double dsum, double dsq, double ssum) {
    __hip_atomic_fetch_add(&mc_wg[0], item_variance(dsum, dsq, A.n_samples), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
    __hip_atomic_fetch_add(&mc_wg[1], dsum * dsum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (dsum != 0.0) atomicAdd(A.A + row1 + p1_lin, dsum);
    if (kScale) atomicAdd(A.scale + row1 + p1_lin, ssum);
    if (A.items) A.items[((size_t)cell * A.n_channels + ci) * nodes + p1_lin] = dsum;
  };
  if (kShort) {
    // The groups of `split` waves take blocks of node_block nodes in turn; the
    // waves of a group share the samples of each node.
    const int nb = A.node_block;
    for (int u0 = first + nb * (wid / split); u0 < last; u0 += nb * (nw / split)) {
      const int cnt = min(nb, last - u0);
      if (lane < cnt) {
        Item t = pair;
        item_node(t, A, ch, u0 + lane);
        for (int a = 0; a < 3; ++a) node_tab[wid][a][lane] = t.p1[a];
        node_tab[wid][3][lane] = t.E1;
        node_tab[wid][4][lane] = t.f1;
        node_tab[wid][5][lane] = t.pref;
      }
      wave_lds_sync();
      for (int j = 0; j < cnt; ++j) run_node(u0 + j, j);
      wave_lds_sync();
      if (A.direct && lane < cnt) {
        const double dsum = node_tab[wid][3][lane], dsq = node_tab[wid][4][lane];
        const double ssum = kScale ? node_tab[wid][5][lane] : 0.0;
        if (split == 1) {
          finish_item(u0 + lane, dsum, dsq, ssum);
        } else {  // this wave's part of the items
          const int i = u0 + lane - first;
          __hip_atomic_fetch_add(&it_sum[0][i], dsum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          __hip_atomic_fetch_add(&it_sum[1][i], dsq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          if (kScale) __hip_atomic_fetch_add(&it_sum[2][i], ssum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      }
      wave_lds_sync();
    }
    n_ok = wave_count_dpp(n_ok);
    if (lane == 0)
      __hip_atomic_fetch_add(&ok_wg, (unsigned long long)n_ok, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  } else {
    // Wave w takes the node blocks w, w + nw, w + 2 nw, ... of the chunk (the
    // chunk starts on a block boundary), the nodes of a block in turn.
    for (int p = first + kNB * wid; p < last; p += (p & (kNB - 1)) == kNB - 1 ? kNB * (nw - 1) + 1 : 1) run_node(p, 0);
  }
  __syncthreads();
  if (kShort && split > 1 && A.direct) {  // the chunk's items from their waves' parts, a node per lane
    const int i = threadIdx.x;
    if (first + i < last) finish_item(first + i, it_sum[0][i], it_sum[1][i], it_sum[2][i]);
    __syncthreads();
  }
  const int stripe = blockIdx.x % kStripes;
  if (threadIdx.x < 2 && A.mc_acc && A.direct) atomicAdd(&A.mc_acc[2 * stripe + threadIdx.x], mc_wg[threadIdx.x]);
  if (threadIdx.x == 0 && A.n_accepted && A.direct) atomicAdd(A.n_accepted + stripe, ok_wg);
  if (threadIdx.x == 0 && A.chan_var && A.direct)  // one channel per workgroup
    atomicAdd(&A.chan_var[(size_t)stripe * A.n_channels + ci], mc_wg[0]);
  if (kRec && threadIdx.x == 0) A.rec.count[lb - A.rec.wg_base] = rec_n;
  if (n_acc > 0) {
    for (int i = threadIdx.x; i < n_acc * win_n; i += blockDim.x) {
      const double v = acc[i];
      if (v != 0.0) {
        const int j = i / win_n;
        atomicAdd(A.A + goff[A.slot_lo + j] + win_lo + (i - j * win_n), v);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Replay.  A workgroup owns (cell, species, node window, part): it adds its
// part of the deposits that the batch's samples recorded for the species to
// LDS accumulators of the window and flushes them.  For grids whose deposit
// accumulators do not fit in LDS at once: drawing every sample again for each
// window or slot costs about 520 VALU instructions per 64 samples and launch,
// a record 52 B written once (92 B in FP64) and 20 B (36 B) read per deposit
// and window, and the sampling kernel then runs with its compacting queue.
// Bound: the sampling launch by VALU issue (378 instructions per 64 samples,
// 55% of the issue cycles), the replay by the LDS atomics (56% busy) and, with
// few records per workgroup, by the flush (13500 entries x 256 workgroups, 34
// us).  Terms with every launch drawing again, and recorded: 7 species at 30^3,
// 128 samples 18.8 and 9.0 ms (9 launches, 35 batches); gluons at 30^3, 128
// samples 216 and 156 us; 7 species at 20^3 (15 channels of three slots)
// learned, 256 samples 8.2 and 7.4 ms, plain, 4096 samples 44.0 and 42.7 ms.
// ---------------------------------------------------------------------------
constexpr int kReplayThreads = 1024;

template <typename R>
__global__ __launch_bounds__(kReplayThreads) void replay_kernel(ReplayArgs a) {
  extern __shared__ double lds[];
  const Grid& G = a.G;
  int per_cell = 0;
  for (int y = 0; y < kSpecies; ++y) per_cell += a.parts[y] * a.n_win;
  const int in_batch = blockIdx.x / per_cell, cell = a.rec.cell_lo + in_batch;  // the cell
  int r = blockIdx.x % per_cell, sp = 0;
  while (r >= a.parts[sp] * a.n_win) {
    r -= a.parts[sp] * a.n_win;
    ++sp;
  }
  const int part = r / a.n_win, lo = r % a.n_win * a.win_n;
  const int n = min(a.win_n, G.nodes - lo);
  for (int i = threadIdx.x; i < n; i += blockDim.x) lds[i] = 0.0;
  __syncthreads();
  const int jobs = (a.m_hi[sp] - a.m_lo[sp]) * a.n_chunks;
  for (int j = part; j < jobs; j += a.parts[sp]) {
    const int m = a.match[sp * kMaxMatches + a.m_lo[sp] + j / a.n_chunks];
    const int pos = (m & 3) - 1;  // 0, 1, 2: positions 2, 3, 4
    const long long wg = ((long long)in_batch * a.n_group + (m >> 2) - a.first) * a.n_chunks + j % a.n_chunks - a.rec.wg_base;
    if (wg < 0 || wg >= a.n_wg) continue;
    const int cnt = (int)a.rec.count[wg];
    const long long i0 = wg * a.rec.region;
    for (int i = threadIdx.x; i < cnt; i += blockDim.x) {
      const Record<R> rec(a.rec.tiles, i0 + i);
      const Stencil<R> st = rec.load(pos);
      const R x = rec.w[9 * 64];
      const double v = (double)(pos == 0 ? x : -x);
      if (a.n_win == 1)
        deposit<double, double, __HIP_MEMORY_SCOPE_WORKGROUP>(lds, widen(st), v, G.ox, G.oy);
      else
        deposit_window(lds, widen(st), v, G.ox, G.oy, lo, n);
    }
  }
  __syncthreads();
  double* out = a.A + ((size_t)sp * G.cells + cell) * G.nodes + lo;
  for (int i = threadIdx.x; i < n; i += blockDim.x)
    if (lds[i] != 0.0) atomicAdd(out + i, lds[i]);
}

// Uniform sampler: the short-item form when waves share nodes, and below
// kShortSamples samples per item (at 2048 samples on 256 cells of gluons the
// compiled long form is 0.9% faster, 59.75 against 60.3 ms; at 128 samples on
// the 70 channels of a 30^3 cell, every launch drawing again, the short one was
// 3.5%, 19.5 against 20.2 ms).
constexpr int kShortSamples = 1024;
inline bool short_items(int split, int n_samples) { return split > 1 || n_samples < kShortSamples; }

// One precision's kernel variants: the launch of one, and all of them with
// their LDS budget group (0 uniform sampler, 1 learned sampler, 2 to 5 the
// compacting variant: kRing and kTight, each for long and short items, 6 the
// replay kernel, 7 and 8 as 0 and 1, long items).
template <typename R>
struct SlotsVariants {
  // the reference precision keeps one form of an item
  static constexpr bool kF64 = std::is_same<R, double>::value;

  template <bool kSym, bool kScale, bool kAllLds, bool kLearned, int kQueue, bool kShort>
  static void launch_user(const CollideArgs& a, dim3 grid, dim3 block, size_t lds, hipStream_t st) {
    if (a.msq_mask)
      hipLaunchKernelGGL((collide_slots_kernel<R, kSym, kScale, kAllLds, kLearned, kQueue, true, kShort>), grid, block,
                         lds, st, a);
    else
      hipLaunchKernelGGL((collide_slots_kernel<R, kSym, kScale, kAllLds, kLearned, kQueue, false, kShort>), grid, block,
                         lds, st, a);
  }

  template <bool kSym, bool kScale, bool kLearned, bool kShort>
  static void launch_variant(const CollideArgs& a, bool all_lds, int queue, dim3 grid, dim3 block, size_t lds,
                             hipStream_t st) {
    if constexpr (kSym && !kLearned) {
      if (queue == kRing) {
        launch_user<true, kScale, true, false, kRing, kShort>(a, grid, block, lds, st);
        return;
      }
      if (queue == kTight) {
        launch_user<true, kScale, true, false, kTight, kShort>(a, grid, block, lds, st);
        return;
      }
    }
    if (all_lds) launch_user<kSym, kScale, true, kLearned, 0, kShort>(a, grid, block, lds, st);
    else if constexpr (!kF64 || kSym) launch_user<kSym, kScale, false, kLearned, 0, kShort>(a, grid, block, lds, st);
  }

  template <bool kSym, bool kScale>
  static void launch_sampler(const CollideArgs& a, bool all_lds, int queue, dim3 grid, dim3 block, size_t lds,
                             hipStream_t st) {
    if constexpr (!kF64)
      if (a.long_form && a.learned) {
        launch_variant<kSym, kScale, true, false>(a, all_lds, 0, grid, block, lds, st);
        return;
      }
    if (a.learned) launch_variant<kSym, kScale, true, true>(a, all_lds, 0, grid, block, lds, st);
    else if (kF64 || (!a.long_form && short_items(a.split, a.n_samples))) launch_variant<kSym, kScale, false, true>(a, all_lds, queue, grid, block, lds, st);
    else if constexpr (!kF64) launch_variant<kSym, kScale, false, false>(a, all_lds, queue, grid, block, lds, st);
  }

  struct Fn { const void* fn; int group; };

  template <bool kSym, bool kScale, bool kAllLds, bool kLearned, int kQueue, bool kShort>
  static void add(std::vector<Fn>& out, int group) {
    out.push_back({(const void*)collide_slots_kernel<R, kSym, kScale, kAllLds, kLearned, kQueue, false, kShort>, group});
    out.push_back({(const void*)collide_slots_kernel<R, kSym, kScale, kAllLds, kLearned, kQueue, true, kShort>, group});
  }
  template <bool kAllLds, bool kLearned, bool kShort>
  static void add_all(std::vector<Fn>& out, int group) {
    add<true, true, kAllLds, kLearned, 0, kShort>(out, group);
    add<true, false, kAllLds, kLearned, 0, kShort>(out, group);
    add<false, true, kAllLds, kLearned, 0, kShort>(out, group);
    add<false, false, kAllLds, kLearned, 0, kShort>(out, group);
  }
  template <int kQueue, bool kShort>
  static void add_queue(std::vector<Fn>& out) {
    const int group = 2 * kQueue + (kShort ? 1 : 0);
    add<true, true, true, false, kQueue, kShort>(out, group);
    add<true, false, true, false, kQueue, kShort>(out, group);
  }
  template <bool kLearned>
  static void launch_rec(const CollideArgs& a, dim3 grid, hipStream_t st) {
    const dim3 block(slots_block(!kLearned));
    if (a.msq_mask)
      hipLaunchKernelGGL((collide_slots_kernel<R, true, false, true, kLearned, kLearned ? 0 : kRing, true, true, true>), grid,
                         block, 0, st, a);
    else
      hipLaunchKernelGGL((collide_slots_kernel<R, true, false, true, kLearned, kLearned ? 0 : kRing, false, true, true>), grid,
                         block, 0, st, a);
  }
  static std::vector<Fn> all() {
    std::vector<Fn> fns;
    fns.push_back({(const void*)replay_kernel<R>, 6});
    add_all<true, false, true>(fns, 0);
    add_all<true, true, true>(fns, 1);
    add_queue<kRing, true>(fns);
    add_queue<kTight, true>(fns);
    if constexpr (!kF64) {
      add_all<false, false, true>(fns, 0);
      add_all<false, true, true>(fns, 1);
      add_all<true, false, false>(fns, 7);
      add_all<false, false, false>(fns, 7);
      add_all<true, true, false>(fns, 8);
      add_all<false, true, false>(fns, 8);
      add_queue<kRing, false>(fns);
      add_queue<kTight, false>(fns);
    }
    return fns;
  }
};

template <typename R>
hipError_t launch_slots(const CollideArgs& a, int nslot, int queue, hipStream_t stream) {
  constexpr bool kF64 = std::is_same<R, double>::value;
  const int n_acc = a.symmetric ? std::min(a.slot_hi - a.slot_lo, a.lds_acc) : 0;
  const int n_tiles = kF64 ? 0 : std::min(nslot, a.lds_tiles);
  const bool all_acc = !a.symmetric || n_acc == a.slot_hi - a.slot_lo;
  if (!all_acc && (!kF64 || n_acc || a.win_n != a.G.nodes)) return hipErrorInvalidValue;
  // FP32: every tile in LDS; FP64: the accumulators
  const bool all_lds = kF64 ? all_acc : n_tiles == nslot;
  if (!all_acc || !a.symmetric || a.learned || a.win_n != a.G.nodes) queue = 0;
  const int threads = slots_block(queue);
  const size_t lds = (size_t)n_acc * a.win_n * sizeof(double) + (size_t)n_tiles * a.G.nodes * sizeof(float);
  const long long blocks = (long long)a.G.cells * a.n_group * a.n_chunks;
  if (blocks <= 0) return hipSuccess;
  if (a.split < 1 || (threads / kWave) % a.split) return hipErrorInvalidValue;  // whole groups of waves
  if (a.split > 1 && a.chunk_items > kSplitNodes) return hipErrorInvalidValue;  // a shared chunk's sums fit in it_sum
  if (a.node_block < 1 || a.node_block > kMaxNodeBlock) return hipErrorInvalidValue;  // a block fits in node_tab
  if (a.long_form && (kF64 || a.split > 1)) return hipErrorInvalidValue;
  if (a.chunk_items % kNodeBlock != 0 && queue && !kF64 && !a.learned &&
      (a.long_form || !short_items(a.split, a.n_samples)))
    return hipErrorInvalidValue;  // the long form's chunks start on node blocks
  const dim3 grid((unsigned)blocks), block(threads);
  using V = SlotsVariants<R>;
  if (a.symmetric) {
    if (a.scale) V::template launch_sampler<true, true>(a, all_lds, queue, grid, block, lds, stream);
    else V::template launch_sampler<true, false>(a, all_lds, queue, grid, block, lds, stream);
  } else {
    if (a.scale) V::template launch_sampler<false, true>(a, all_lds, 0, grid, block, lds, stream);
    else V::template launch_sampler<false, false>(a, all_lds, 0, grid, block, lds, stream);
  }
  return hipGetLastError();
}

template <typename R>
size_t record_tile_bytes() {
  return Record<R>::kTileBytes;
}

// The launch plan of a recording launch: every workgroup's samples (per_sample
// records each) fit in its region, and the regions in the buffers.
inline bool record_fits(const CollideArgs& a, int n_wg, int per_sample) {
  const int waves = slots_block(true) / kWave;
  if (!a.symmetric || a.scale || a.split < 1 || waves % a.split) return false;
  if (a.split > 1 && a.chunk_items > kSplitNodes) return false;
  if (a.node_block < 1 || a.node_block > kMaxNodeBlock) return false;
  if ((long long)a.chunk_items * a.n_samples * per_sample > a.rec.region || a.rec.region * n_wg > a.rec.capacity)
    return false;
  // the kernel counts the batch's workgroups from its first cell in 32 bits
  const long long per_cell = (long long)a.n_group * a.n_chunks, end = (long long)a.rec.wg_base + n_wg;
  if (a.rec.cell_lo < 0 || a.rec.wg_base < 0 || a.rec.wg_base >= per_cell || end > 0x7FFFFFFF) return false;
  return a.rec.cell_lo * per_cell + end <= a.G.cells * per_cell;
}

template <typename R>
hipError_t launch_rec(const CollideArgs& a, int n_wg, hipStream_t stream) {
  if (n_wg <= 0) return hipSuccess;
  if (!record_fits(a, n_wg, 1)) return hipErrorInvalidValue;
  if (a.learned) SlotsVariants<R>::template launch_rec<true>(a, dim3((unsigned)n_wg), stream);
  else SlotsVariants<R>::template launch_rec<false>(a, dim3((unsigned)n_wg), stream);
  return hipGetLastError();
}

template <typename R>
hipError_t launch_replay(const ReplayArgs& a, hipStream_t stream) {
  long long per_cell = 0;
  for (int y = 0; y < kSpecies; ++y) per_cell += (long long)a.parts[y] * a.n_win;
  if (per_cell * a.n_cells <= 0) return hipSuccess;
  if ((long long)a.n_win * a.win_n < a.G.nodes) return hipErrorInvalidValue;  // the windows cover the grid
  hipLaunchKernelGGL(replay_kernel<R>, dim3((unsigned)(per_cell * a.n_cells)), dim3(kReplayThreads),
                     a.win_n * sizeof(double), stream, a);
  return hipGetLastError();
}

// A kernel may use what its static LDS leaves of lds_max.  Raising the
// per-kernel dynamic limit is only needed (and only accepted) above the
// runtime's default; after a refusal the budget is the limit in force.
inline hipError_t raise_lds_limit(const void* fn, size_t lds_max, size_t* budget) {
  hipFuncAttributes attr;
  if (hipFuncGetAttributes(&attr, fn) != hipSuccess) return hipGetLastError();
  const size_t stat = attr.sharedSizeBytes;
  size_t want = lds_max > stat ? lds_max - stat : 0;
  size_t have = attr.maxDynamicSharedSizeBytes > 0 ? (size_t)attr.maxDynamicSharedSizeBytes : 0;
  if (have < want) {
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)want) == hipSuccess)
      have = want;
    else
      (void)hipGetLastError();
  }
  *budget = std::min(*budget, std::min(have, want));
  return hipSuccess;
}

template <typename R>
hipError_t slots_lds_limit(size_t lds_max, LdsBudget* out) {
  size_t budget[9];
  for (size_t& b : budget) b = lds_max;
  for (const auto& f : SlotsVariants<R>::all())
    if (const hipError_t e = raise_lds_limit(f.fn, lds_max, &budget[f.group])) return e;
  out->plain[0] = budget[7];  // FP64 has the short form only: not used
  out->plain[1] = budget[0];
  out->learned[0] = budget[8];
  out->learned[1] = budget[1];
  for (int f = 0; f < 2; ++f) {
    out->queue[f][0] = std::is_same<R, double>::value ? 0 : budget[2 + 2 * f];  // FP64 has the short form only
    out->queue[f][1] = budget[3 + 2 * f];
  }
  out->replay = budget[6];
  return hipSuccess;
}

}  // namespace
}  // namespace qgbe
