// Field kernels around the collision term: thermal masses (Eq. mg, Eq. mq),
// the drift of Eq. left handside with the forward-Euler update (Sec. III),
// and the FP64 bookkeeping (Eq. particle numbers, Eq. energy momentum tensor).
// All of them are HBM-bound stencils or reductions in FP64.
#include <hip/hip_runtime.h>

#include "field.h"

namespace qgbe {
namespace {

constexpr int kBlock = 256;

__device__ __forceinline__ void node_p(const Grid& G, int node, double p[3]) {
  const int iz = node % G.np[2];
  const int iy = (node / G.np[2]) % G.np[1];
  const int ix = node / (G.np[2] * G.np[1]);
  p[0] = node_coord(G.ph[0], G.dp[0], ix);
  p[1] = node_coord(G.ph[1], G.dp[1], iy);
  p[2] = node_coord(G.ph[2], G.dp[2], iz);
}

__device__ __forceinline__ double block_sum(double v, double* sh) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  const int w = threadIdx.x / 64, lane = threadIdx.x & 63;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < (int)(blockDim.x / 64); ++i) t += sh[i];
  return t;  // valid in thread 0
}

// The start of a collision term, one pass over f: the thermal masses, the
// output and the term's totals zeroed, and for the FP32 kernels the FP32 shadow
// and the node quads.  (Apart, these were seven launches of 2 to 9 us, most of
// them latency: a step of 30^3 gluons spent 60 of 283 us in them.)
//
// Masses: I_Y = sum_p dV/(2pi)^3 f_Y / (2 E_Y) per cell, E_Y from the lagged
// masses (or |p| when there are none; a node at p = 0 then adds 0).  Block
// (cell, chunk) sums kMassChunk nodes of every species; the last block of a
// cell to finish adds the cell's chunks in a fixed order (deterministic) and
// applies Eq. mg / mq.  Without counters (`done`), or with more than
// kMaxFusedBlocks blocks, a second kernel does that: every block's release
// writes its XCD's L2 back, 1.3 ms for the 8192 blocks of 256 cells of 20^3
// against 0.2 ms with the second kernel (106 blocks of 30^3: the second kernel
// is 6 us and a gap more).
constexpr int kMaxFusedBlocks = 512;
constexpr int kMassChunk = kBlock;  // a node per thread: a single cell of 30^3 nodes fills 100+ CUs

__host__ __device__ inline int mass_chunks(const Grid& G) { return (G.nodes + kMassChunk - 1) / kMassChunk; }

// Sums of seven values over the block, in the order of block_sum: valid in
// thread sp < 7 for value sp.
__device__ __forceinline__ double block_sum7(const double v[kSpecies], double (*sh)[kSpecies]) {
  const int w = threadIdx.x / 64, lane = threadIdx.x & 63;
#pragma unroll
  for (int sp = 0; sp < kSpecies; ++sp) {
    double t = v[sp];
    for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
    if (lane == 0) sh[w][sp] = t;
  }
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x < kSpecies)
    for (int i = 0; i < (int)(blockDim.x / 64); ++i) t += sh[i][threadIdx.x];
  __syncthreads();
  return t;
}

// The masses of a cell from its chunk sums, by one block.
__device__ __forceinline__ void masses_of_cell(const Grid& G, const double* part, int chunks, int cell, double* mass2,
                                               double (*sh)[kSpecies]) {
  __shared__ double I[kSpecies];
  const double meas = G.dp[0] * G.dp[1] * G.dp[2] / (8.0 * kPi * kPi * kPi);
  double v[kSpecies] = {};
  for (int c = threadIdx.x; c < chunks; c += blockDim.x)
    for (int sp = 0; sp < kSpecies; ++sp) v[sp] += part[((size_t)cell * chunks + c) * kSpecies + sp];
  const double t = block_sum7(v, sh);
  if (threadIdx.x < kSpecies) I[threadIdx.x] = t * meas;
  __syncthreads();
  if (threadIdx.x != 0) return;
  // SU(3): dA = 8, CA = 3, CF = 4/3; N_g = 16, N_q = 6
  const double CF = 4.0 / 3.0;
  double q = 0.0;
  for (int i = 0; i < 3; ++i) q += 6.0 * CF * (I[i] + I[i + 3]);
  mass2[kGluon * G.cells + cell] = (2.0 * G.g2 / 8.0) * (16.0 * 3.0 * I[kGluon] + q);
  for (int i = 0; i < 3; ++i) {
    const double mq = 2.0 * CF * G.g2 * (2.0 * I[kGluon] + I[i] + I[i + 3]);
    mass2[i * G.cells + cell] = mq;
    mass2[(i + 3) * G.cells + cell] = mq;
  }
}

__global__ __launch_bounds__(kBlock) void term_start_kernel(TermStart a) {
  __shared__ double sh[kBlock / 64][kSpecies];
  __shared__ bool last;
  const Grid& G = a.G;
  const int chunks = mass_chunks(G);
  const int chunk = blockIdx.x % chunks, cell = blockIdx.x / chunks;
  const int node = chunk * kMassChunk + threadIdx.x;
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < a.n_count; i += blockDim.x) a.count[i] = 0ull;
    for (int i = threadIdx.x; i < a.n_totals; i += blockDim.x) a.totals[i] = 0.0;
  }
  double v[kSpecies] = {};
  if (node < G.nodes) {
    double p[3];
    node_p(G, node, p);
    const double p2 = p[0] * p[0] + p[1] * p[1] + p[2] * p[2];
    const int iz = node % G.np[2], iy = (node / G.np[2]) % G.np[1];
    const size_t dz = iz + 1 < G.np[2] ? 1 : 0;
    const size_t dy = iy + 1 < G.np[1] ? (size_t)G.oy : 0;
#pragma unroll
    for (int sp = 0; sp < kSpecies; ++sp) {
      const size_t i = ((size_t)sp * G.cells + cell) * G.nodes + node;
      const double x = a.f[i];
      if (a.A) a.A[i] = 0.0;
      if (a.f32) a.f32[i] = (float)x;
      if (a.quads) a.quads[i] = make_float4((float)x, (float)a.f[i + dz], (float)a.f[i + dy], (float)a.f[i + dy + dz]);
      if (a.part) {
        const double E = sqrt(p2 + (a.lag ? a.lag[sp * G.cells + cell] : 0.0));
        if (E > 0.0) v[sp] = x / (2.0 * E);
      }
    }
  }
  if (!a.part) {  // constant masses
    if (chunk == 0 && threadIdx.x < kSpecies) a.mass2[threadIdx.x * G.cells + cell] = a.constant.v[threadIdx.x];
    return;
  }
  const double t = block_sum7(v, sh);
  if (threadIdx.x < kSpecies) a.part[((size_t)cell * chunks + chunk) * kSpecies + threadIdx.x] = t;
  if (!a.done) return;
  if (chunks > 1) {
    // release the partial sums, count this block in, and let the cell's last one read them all
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(&a.done[cell], 1u) == (unsigned)chunks - 1u;
    __syncthreads();
    if (!last) return;
    __threadfence();
    if (threadIdx.x == 0) a.done[cell] = 0u;
  } else {
    __syncthreads();
  }
  masses_of_cell(G, a.part, chunks, cell, a.mass2, sh);
}

__global__ __launch_bounds__(kBlock) void mass_final(Grid G, const double* __restrict__ part, int chunks,
                                                     double* mass2) {
  __shared__ double sh[kBlock / 64][kSpecies];
  masses_of_cell(G, part, chunks, blockIdx.x, mass2, sh);
}

__device__ __forceinline__ int shift_cell(const Grid& G, int cell, int axis, int d) {
  int id[3] = {cell / (G.nx[1] * G.nx[2]), (cell / G.nx[2]) % G.nx[1], cell % G.nx[2]};
  id[axis] = (id[axis] + d + G.nx[axis]) % G.nx[axis];
  return (id[0] * G.nx[1] + id[1]) * G.nx[2] + id[2];
}

__device__ __forceinline__ int shift_node(const Grid& G, int node, int axis, int d) {
  int id[3] = {node / (G.np[1] * G.np[2]), (node / G.np[2]) % G.np[1], node % G.np[2]};
  id[axis] = (id[axis] + d + G.np[axis]) % G.np[axis];
  return (id[0] * G.np[1] + id[1]) * G.np[2] + id[2];
}

__device__ __forceinline__ double energy(const Grid& G, const double* mass2, int sp, int cell, int node) {
  double p[3];
  node_p(G, node, p);
  return sqrt(p[0] * p[0] + p[1] * p[1] + p[2] * p[2] + mass2[sp * G.cells + cell]);
}

__device__ __forceinline__ double upwind(double vel, double f_left, double f_right) {
  return vel > 0.0 ? vel * f_left : vel * f_right;
}

// D[f] at (sp, cell, node), flux form with periodic boundaries.
__device__ double drift_at(const Grid& G, const double* f, const double* mass2, int sp, int cell,
                           int node, int scheme) {
  const double* F = f + (size_t)sp * G.cells * G.nodes;
  double p[3];
  node_p(G, node, p);
  double D = 0.0;
  for (int a = 0; a < 3; ++a) {
    if (G.nx[a] == 1) continue;  // a single periodic cell has no gradient
    const int xp = shift_cell(G, cell, a, +1), xm = shift_cell(G, cell, a, -1);
    const int pp = shift_node(G, node, a, +1), pm = shift_node(G, node, a, -1);
    const double Ec = energy(G, mass2, sp, cell, node);
    const double Exp = energy(G, mass2, sp, xp, node), Exm = energy(G, mass2, sp, xm, node);
    const double inv2dx = 0.5 / G.dx[a];
    if (scheme == 0) {
      const double vc = p[a] / Ec, vp = p[a] / Exp, vm = p[a] / Exm;
      const double fR = upwind(0.5 * (vc + vp), F[(size_t)cell * G.nodes + node], F[(size_t)xp * G.nodes + node]);
      const double fL = upwind(0.5 * (vm + vc), F[(size_t)xm * G.nodes + node], F[(size_t)cell * G.nodes + node]);
      D += (fR - fL) / G.dx[a];
      // p-advection with the force -dE/dx_a (central in x)
      const double Fc = -(Exp - Exm) * inv2dx;
      const double Fp = -(energy(G, mass2, sp, xp, pp) - energy(G, mass2, sp, xm, pp)) * inv2dx;
      const double Fm = -(energy(G, mass2, sp, xp, pm) - energy(G, mass2, sp, xm, pm)) * inv2dx;
      const double gR = upwind(0.5 * (Fc + Fp), F[(size_t)cell * G.nodes + node], F[(size_t)cell * G.nodes + pp]);
      const double gL = upwind(0.5 * (Fm + Fc), F[(size_t)cell * G.nodes + pm], F[(size_t)cell * G.nodes + node]);
      D += (gR - gL) / G.dp[a];
    } else {
      D += (p[a] * F[(size_t)xp * G.nodes + node] / Exp - p[a] * F[(size_t)xm * G.nodes + node] / Exm) * inv2dx;
      const double dEp = (energy(G, mass2, sp, xp, pp) - energy(G, mass2, sp, xm, pp)) * inv2dx;
      const double dEm = (energy(G, mass2, sp, xp, pm) - energy(G, mass2, sp, xm, pm)) * inv2dx;
      D -= (F[(size_t)cell * G.nodes + pp] * dEp - F[(size_t)cell * G.nodes + pm] * dEm) * (0.5 / G.dp[a]);
    }
  }
  return D;
}

// The evolving species, in order (the update touches only these; the frozen
// species hold the same values in both buffers of f, set together).
struct Evolving {
  int n;
  int sp[kSpecies];
};

// f_out = f + dt (A / (N_Y hbar c) - D[f]) for the evolving species.
__global__ __launch_bounds__(kBlock) void update_kernel(Grid G, Evolving ev, const double* __restrict__ f,
                                                        const double* __restrict__ A,
                                                        const double* __restrict__ mass2, double dt,
                                                        int scheme, double* __restrict__ f_out,
                                                        float* __restrict__ f32, double* __restrict__ lag) {
  // the masses of this step are the lagged ones of the next
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < kSpecies * G.cells; i += gridDim.x * blockDim.x)
    lag[i] = mass2[i];
  const size_t per = (size_t)G.cells * G.nodes;
  const size_t total = (size_t)ev.n * per;
  for (size_t j = blockIdx.x * (size_t)blockDim.x + threadIdx.x; j < total; j += (size_t)gridDim.x * blockDim.x) {
    const int k = (int)(j / per);
    const size_t rem = j - (size_t)k * per;
    const int sp = ev.sp[k];
    const size_t i = (size_t)sp * per + rem;
    const int cell = (int)(rem / G.nodes), node = (int)(rem % G.nodes);
    const double D = drift_at(G, f, mass2, sp, cell, node, scheme);
    const double v = f[i] + dt * (A[i] / (degeneracy(sp) * kHbarC) - D);
    f_out[i] = v;
    f32[i] = (float)v;
  }
}

// Observables: per species N, E, P (3), M = sum m^2 f / E (the mass term of
// the modified tensor), the entropy S = sum [(1 + s f) ln(1 + s f)/s - f ln f]
// (s = +1 for gluons, -1 for quarks; a node adds only while 0 < f and
// 1 + s f > 0) and the diagonal T^ii = sum p_i^2 f / E of Eq. energy momentum
// tensor, then min f and max fermion f, and a non-finite counter.  Stage 1:
// per-block partials; stage 2: one block.
constexpr int kObs = kSpecies * kObsPer;

constexpr int kObsRow = kObsPer + 3;  // partials of a (block, species): the values, min f, max fermion f, non-finite

// Block (b, species): a block per species keeps the reductions of a block to
// kObsRow instead of seven times that (30^3 nodes, one cell: 41 -> 11 us).
__global__ __launch_bounds__(kBlock) void observables_partial(Grid G, const double* __restrict__ f,
                                                              const double* __restrict__ mass2,
                                                              double* partial) {
  __shared__ double sh[kBlock / 64][kObsRow];
  const size_t per = (size_t)G.cells * G.nodes;
  const int sp = blockIdx.y;
  double v[kObsPer] = {};
  double minf = 1e300, maxq = -1e300, bad = 0.0;
  const bool evolve = (G.species_mask >> sp) & 1u;
  const double sgn = sp == kGluon ? 1.0 : -1.0;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < per; i += (size_t)gridDim.x * blockDim.x) {
    const int cell = (int)(i / G.nodes), node = (int)(i % G.nodes);
    const double fv = f[(size_t)sp * per + i];
    double p[3];
    node_p(G, node, p);
    const double m2 = mass2[sp * G.cells + cell];
    const double En = sqrt(p[0] * p[0] + p[1] * p[1] + p[2] * p[2] + m2);
    v[0] += fv;
    v[1] += En * fv;
    for (int k = 0; k < 3; ++k) v[2 + k] += p[k] * fv;
    if (En > 0.0) {
      const double w = fv / En;
      v[5] += m2 * w;
      for (int k = 0; k < 3; ++k) v[7 + k] += p[k] * p[k] * w;
    }
    const double one = 1.0 + sgn * fv;
    if (fv > 0.0 && one > 0.0) v[6] += one * log(one) * sgn - fv * log(fv);
    if (evolve) {
      if (!isfinite(fv)) bad += 1.0;
      minf = fmin(minf, fv);
      if (sp != kGluon) maxq = fmax(maxq, fv);
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
    for (int k = 0; k < kObsPer; ++k) v[k] += __shfl_xor(v[k], off, 64);
    minf = fmin(minf, __shfl_xor(minf, off, 64));
    maxq = fmax(maxq, __shfl_xor(maxq, off, 64));
    bad += __shfl_xor(bad, off, 64);
  }
  const int w = threadIdx.x / 64;
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int k = 0; k < kObsPer; ++k) sh[w][k] = v[k];
    sh[w][kObsPer] = minf;
    sh[w][kObsPer + 1] = maxq;
    sh[w][kObsPer + 2] = bad;
  }
  __syncthreads();
  if (threadIdx.x < kObsRow) {
    const int k = threadIdx.x;
    double t = k == kObsPer ? 1e300 : (k == kObsPer + 1 ? -1e300 : 0.0);
    for (int i = 0; i < kBlock / 64; ++i)
      t = k == kObsPer ? fmin(t, sh[i][k]) : (k == kObsPer + 1 ? fmax(t, sh[i][k]) : t + sh[i][k]);
    partial[((size_t)blockIdx.x * kSpecies + sp) * kObsRow + k] = t;
  }
}

// Stage 2: one wave per value (min, max or sum over the block partials).
constexpr int kFinalThreads = 1024;

__global__ __launch_bounds__(kFinalThreads) void observables_final(Grid G, const double* partial, int nblocks,
                                                                   double* out) {
  const double meas = G.dx[0] * G.dx[1] * G.dx[2] * G.dp[0] * G.dp[1] * G.dp[2] / (8.0 * kPi * kPi * kPi);
  const int lane = threadIdx.x & 63, nw = blockDim.x / 64;
  for (int k = threadIdx.x / 64; k < kObs + 3; k += nw) {
    const bool is_min = k == kObs, is_max = k == kObs + 1;
    const bool whole = k >= kObs;  // over every species
    double v = is_min ? 1e300 : (is_max ? -1e300 : 0.0);
    const int n = whole ? nblocks * kSpecies : nblocks;
    for (int b = lane; b < n; b += 64) {
      const double x = whole ? partial[(size_t)b * kObsRow + kObsPer + (k - kObs)]
                             : partial[((size_t)b * kSpecies + k / kObsPer) * kObsRow + k % kObsPer];
      v = is_min ? fmin(v, x) : (is_max ? fmax(v, x) : v + x);
    }
    for (int off = 32; off > 0; off >>= 1) {
      const double o = __shfl_xor(v, off, 64);
      v = is_min ? fmin(v, o) : (is_max ? fmax(v, o) : v + o);
    }
    if (lane == 0) out[k] = (k < kObs) ? v * degeneracy(k / kObsPer) * meas : v;
  }
}

// Energy bookkeeping of a step, per-block partials [source, collide]:
// source  = sum N f (E(m^2) - E(m_prev^2)), the difference taken as
//           (m^2 - m_prev^2) / (E + E_prev) so it keeps its relative accuracy;
// collide = sum over evolved species of E(m^2) A.
__global__ __launch_bounds__(kBlock) void energy_partial(Grid G, const double* __restrict__ f,
                                                         const double* __restrict__ A,
                                                         const double* __restrict__ mass2,
                                                         const double* __restrict__ mass2_prev, double* partial) {
  __shared__ double sh[kBlock / 64];
  const size_t per = (size_t)G.cells * G.nodes;
  double src = 0.0, col = 0.0;
  for (int sp = 0; sp < kSpecies; ++sp) {
    const bool evolve = (G.species_mask >> sp) & 1u;
    double s_sp = 0.0;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < per; i += (size_t)gridDim.x * blockDim.x) {
      const int cell = (int)(i / G.nodes), node = (int)(i % G.nodes);
      double p[3];
      node_p(G, node, p);
      const double pp = p[0] * p[0] + p[1] * p[1] + p[2] * p[2];
      const double m2 = mass2[sp * G.cells + cell];
      const double E = sqrt(pp + m2);
      if (mass2_prev) {
        const double m2p = mass2_prev[sp * G.cells + cell];
        const double den = E + sqrt(pp + m2p);
        if (den > 0.0) s_sp += f[(size_t)sp * per + i] * (m2 - m2p) / den;
      }
      if (evolve) col += E * A[(size_t)sp * per + i];
    }
    src += degeneracy(sp) * s_sp;
  }
  const double t0 = block_sum(src, sh);
  const double t1 = block_sum(col, sh);
  if (threadIdx.x == 0) {
    partial[2 * (size_t)blockIdx.x] = t0;
    partial[2 * (size_t)blockIdx.x + 1] = t1;
  }
}

__global__ __launch_bounds__(kBlock) void energy_final(Grid G, const double* partial, int nblocks, double dt,
                                                       double* out) {
  __shared__ double sh[kBlock / 64];
  const double meas = G.dx[0] * G.dx[1] * G.dx[2] * G.dp[0] * G.dp[1] * G.dp[2] / (8.0 * kPi * kPi * kPi);
  for (int k = 0; k < 2; ++k) {
    double v = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += blockDim.x) v += partial[2 * (size_t)b + k];
    const double t = block_sum(v, sh);
    if (threadIdx.x == 0) out[k] = k == 0 ? t * meas : t * meas * dt / kHbarC;
  }
}

// f into both buffers and the FP32 shadow (src may be f itself).
__global__ void set_field_kernel(const double* src, double* f, double* __restrict__ f_next, float* __restrict__ f32,
                                 size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const double x = src[i];
    f[i] = x;
    f_next[i] = x;
    f32[i] = (float)x;
  }
}

__global__ void fill_kernel(double* __restrict__ dst, double v, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    dst[i] = v;
}

unsigned grid_for(size_t n) {
  size_t b = (n + kBlock - 1) / kBlock;
  if (b > 16384) b = 16384;
  return (unsigned)(b ? b : 1);
}

}  // namespace

size_t mass_scratch(const Grid& G) { return (size_t)G.cells * mass_chunks(G) * kSpecies; }

hipError_t launch_term_start(const TermStart& args, hipStream_t st) {
  TermStart a = args;
  const int chunks = mass_chunks(a.G);
  if ((long long)chunks * a.G.cells > kMaxFusedBlocks) a.done = nullptr;
  hipLaunchKernelGGL(term_start_kernel, dim3(chunks * a.G.cells), dim3(kBlock), 0, st, a);
  if (a.part && !a.done)
    hipLaunchKernelGGL(mass_final, dim3(a.G.cells), dim3(kBlock), 0, st, a.G, a.part, chunks, a.mass2);
  return hipGetLastError();
}

hipError_t launch_update(const Grid& G, const double* f, const double* A, const double* mass2, double dt,
                         int scheme, double* f_out, float* f32, double* lag, hipStream_t st) {
  Evolving ev{};
  for (int sp = 0; sp < kSpecies; ++sp)
    if ((G.species_mask >> sp) & 1u) ev.sp[ev.n++] = sp;
  const size_t n = (size_t)ev.n * G.cells * G.nodes;
  hipLaunchKernelGGL(update_kernel, dim3(grid_for(n)), dim3(kBlock), 0, st, G, ev, f, A, mass2, dt, scheme, f_out,
                     f32, lag);
  return hipGetLastError();
}

int observables_blocks(const Grid& G) {
  const size_t per = (size_t)G.cells * G.nodes;
  size_t b = (per + kBlock - 1) / kBlock;
  return (int)(b > 512 ? 512 : (b ? b : 1));
}

size_t observables_scratch(const Grid& G) { return (size_t)observables_blocks(G) * kSpecies * kObsRow; }

hipError_t launch_observables(const Grid& G, const double* f, const double* mass2, double* scratch,
                              double* out, hipStream_t st) {
  const int nb = observables_blocks(G);
  hipLaunchKernelGGL(observables_partial, dim3(nb, kSpecies), dim3(kBlock), 0, st, G, f, mass2, scratch);
  hipLaunchKernelGGL(observables_final, dim3(1), dim3(kFinalThreads), 0, st, G, scratch, nb, out);
  return hipGetLastError();
}

hipError_t launch_energy_budget(const Grid& G, const double* f, const double* A, const double* mass2,
                                const double* mass2_prev, double dt, double* scratch, double* out, hipStream_t st) {
  const int nb = observables_blocks(G);
  hipLaunchKernelGGL(energy_partial, dim3(nb), dim3(kBlock), 0, st, G, f, A, mass2, mass2_prev, scratch);
  hipLaunchKernelGGL(energy_final, dim3(1), dim3(kBlock), 0, st, G, scratch, nb, dt, out);
  return hipGetLastError();
}

hipError_t launch_set_field(const double* src, double* f, double* f_next, float* f32, size_t n, hipStream_t st) {
  hipLaunchKernelGGL(set_field_kernel, dim3(grid_for(n)), dim3(kBlock), 0, st, src, f, f_next, f32, n);
  return hipGetLastError();
}

hipError_t launch_fill(double* dst, double v, size_t n, hipStream_t st) {
  hipLaunchKernelGGL(fill_kernel, dim3(grid_for(n)), dim3(kBlock), 0, st, dst, v, n);
  return hipGetLastError();
}

}  // namespace qgbe
