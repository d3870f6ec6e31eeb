// The root-parameterisation kernel and the sample recorder.
#include "collide_device.h"

namespace qgbe {

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
// throughout (f from the FP64 field, FP64 atomics): the reference method.
// Every lane draws a sample and solves for its roots; samples with a valid
// root go to a per-wavefront queue in LDS, and whenever 64 are queued (and
// at the end of the item) the wavefront evaluates them on full lanes, so the
// value, f and deposits run once per valid sample, not on every lane.
// ---------------------------------------------------------------------------
constexpr double kRootNorm = 1.0 / (32.0 * kPi * kPi * kPi * kPi * kPi * 16.0);

constexpr int kRootWaves = 4;      // wavefronts per workgroup of the root kernel
constexpr int kRootQueueLen = 128;  // queued samples per wavefront (< 64 left + 64 new)

template <bool kAlt, bool kPriv>
__global__ __launch_bounds__(kRootWaves * kWave) void collide_roots_kernel(CollideArgs A) {
  const Grid& G = A.G;
  extern __shared__ double root_acc[];  // kPriv: [7][cells][nodes], as the output (see the FP64 kernel)
  const int n_out = kPriv ? kSpecies * G.cells * G.nodes : 0;
  for (int i = threadIdx.x; i < n_out; i += blockDim.x) root_acc[i] = 0.0;
  __shared__ unsigned long long blk_ok;
  __shared__ double blk_mc[2];
  __shared__ double blk_var[kMaxChannels];
  BlockTotals blk{&blk_ok, blk_mc, blk_var};
  __shared__ Channel s_ch[kMaxChannels];
  __shared__ int s_group[kMaxChannels];
  // Samples with at least one valid root, queued per wavefront: the uniform
  // momentum (k2 or k4), k3x, k3y, the two roots, and which roots hold.
  __shared__ double rq[kRootWaves][7][kRootQueueLen];
  __shared__ uint32_t rm[kRootWaves][kRootQueueLen];
  for (int i = threadIdx.x; i < A.n_group; i += blockDim.x) s_group[i] = A.group[i];
  for (int i = threadIdx.x; i < A.n_channels; i += blockDim.x) s_ch[i] = A.chans[i];
  blk.init();
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = threadIdx.x / kWave;
  const int wave = (blockIdx.x * blockDim.x + threadIdx.x) / kWave;
  const int nwaves = gridDim.x * blockDim.x / kWave;
  const long long n_items = (long long)G.cells * A.n_group * G.nodes;
  for (long long w = wave; w < n_items; w += nwaves) {
    const int p1_lin = (int)(w % G.nodes);
    const int gi = (int)((w / G.nodes) % A.n_group);
    const int cell = (int)(w / ((long long)G.nodes * A.n_group));
    const int ci = s_group[gi];
    const Channel ch = s_ch[ci];
    Item it;
    load_item(it, A, ch, cell, p1_lin);
    if (!(it.E1 > 0.0)) {  // massless p = 0 node: zero measure
      if (lane == 0 && A.items) A.items[((size_t)cell * A.n_channels + ci) * G.nodes + p1_lin] = 0.0;
      continue;
    }
    const double* fc[4];
    double* Ac[4];
    double* Sc[4];
    for (int p = 0; p < 4; ++p) {
      fc[p] = A.f64 + ((size_t)ch.sp[p] * G.cells + cell) * G.nodes;
      Ac[p] = A.A + ((size_t)ch.sp[p] * G.cells + cell) * G.nodes;
      Sc[p] = A.scale ? A.scale + ((size_t)ch.sp[p] * G.cells + cell) * G.nodes : nullptr;
    }
    const bool g1 = is_gluon(ch.sp[0]), g2 = is_gluon(ch.sp[1]);
    const bool g3 = is_gluon(ch.sp[2]), g4 = is_gluon(ch.sp[3]);
    const double F1 = g1 ? 1.0 + it.f1 : 1.0 - it.f1;
    const double V5 = G.Vp * (2.0 * G.ph[0]) * (2.0 * G.ph[1]);
    const double coef = (A.symmetric ? ch.w : ch.sigma) * V5 / (double)A.n_samples * G.g4 * kRootNorm / it.E1;
    double dsum = 0.0, ssum = 0.0, dsq = 0.0;
    int n_ok = 0;
    // The value of one queued sample: the sum over its valid roots, with
    // their deposits.
    auto finish = [&](unsigned slot) {
      const double q[3] = {rq[wid][0][slot], rq[wid][1][slot], rq[wid][2][slot]};
      const double k3x = rq[wid][3][slot], k3y = rq[wid][4][slot];
      const uint32_t roots = rm[wid][slot];
      const double a3 = k3x * k3x + k3y * k3y + it.m3sq;
      const double Eq = sqrt64(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + (kAlt ? it.m4sq : it.m2sq));
      double vsample = 0.0;
#pragma unroll 1
      for (int r = 0; r < 2; ++r) {
        if (!((roots >> r) & 1u)) continue;
        const double z = rq[wid][5 + r][slot];
        const double E3 = sqrt64(a3 + z * z);
        double p2[3], p3[3] = {k3x, k3y, z}, p4[3], E2, E4, J;
        if (!kAlt) {
          for (int a = 0; a < 3; ++a) {
            p2[a] = q[a];
            p4[a] = it.p1[a] + q[a] - p3[a];
          }
          E2 = Eq;
          E4 = sqrt64(p4[0] * p4[0] + p4[1] * p4[1] + p4[2] * p4[2] + it.m4sq);
          J = fabs(z * rcp64(E3) - p4[2] * rcp64(E4));
        } else {
          for (int a = 0; a < 3; ++a) {
            p4[a] = q[a];
            p2[a] = p3[a] + (q[a] - it.p1[a]);
          }
          E4 = Eq;
          E2 = sqrt64(p2[0] * p2[0] + p2[1] * p2[1] + p2[2] * p2[2] + it.m2sq);
          J = fabs(p2[2] * rcp64(E2) - z * rcp64(E3));
        }
        ++n_ok;
        double Pq[3], d13[3], d14[3];
        for (int a = 0; a < 3; ++a) {
          Pq[a] = it.p1[a] + p2[a];
          d13[a] = it.p1[a] - p3[a];
          d14[a] = it.p1[a] - p4[a];
        }
        const double E12 = it.E1 + E2, E13 = it.E1 - E3, E14 = it.E1 - E4;
        const double ms = E12 * E12 - (Pq[0] * Pq[0] + Pq[1] * Pq[1] + Pq[2] * Pq[2]);
        const double mt = E13 * E13 - (d13[0] * d13[0] + d13[1] * d13[1] + d13[2] * d13[2]);
        const double mu = E14 * E14 - (d14[0] * d14[0] + d14[1] * d14[1] + d14[2] * d14[2]);
        const double wnb = coef * msq_row<double>(A.msq_mask, A.msq, ch.row, ms, mt, mu, it.mu) *
                           rcp64(E2 * E3 * E4 * J);
        const Stencil<double> s2 = make_stencil<double>(p2, G);
        const Stencil<double> s3 = make_stencil<double>(p3, G);
        const Stencil<double> s4 = make_stencil<double>(p4, G);
        const double f2 = interpolate<double>(fc[1], s2, G.ox, G.oy);
        const double f3 = interpolate<double>(fc[2], s3, G.ox, G.oy);
        const double f4 = interpolate<double>(fc[3], s4, G.ox, G.oy);
        const double F2 = g2 ? 1.0 + f2 : 1.0 - f2;
        const double F3 = g3 ? 1.0 + f3 : 1.0 - f3;
        const double F4 = g4 ? 1.0 + f4 : 1.0 - f4;
        const double gain = f3 * f4 * F1 * F2, loss = it.f1 * f2 * F3 * F4;
        const double v = wnb * (gain - loss);
        const double vs = fabs(wnb) * (gain + loss);
        vsample += v;
        ssum += vs;
        if (kPriv) {
          deposit<double, double, __HIP_MEMORY_SCOPE_WORKGROUP>(root_acc + (Ac[1] - A.A), s2, v, G.ox, G.oy);
          deposit<double, double, __HIP_MEMORY_SCOPE_WORKGROUP>(root_acc + (Ac[2] - A.A), s3, -v, G.ox, G.oy);
          deposit<double, double, __HIP_MEMORY_SCOPE_WORKGROUP>(root_acc + (Ac[3] - A.A), s4, -v, G.ox, G.oy);
          if (A.scale) {
            deposit<double, double>(Sc[1], s2, vs, G.ox, G.oy);
            deposit<double, double>(Sc[2], s3, vs, G.ox, G.oy);
            deposit<double, double>(Sc[3], s4, vs, G.ox, G.oy);
          }
        } else if (A.symmetric) {
          deposit<double, double>(Ac[1], s2, v, G.ox, G.oy);
          deposit<double, double>(Ac[2], s3, -v, G.ox, G.oy);
          deposit<double, double>(Ac[3], s4, -v, G.ox, G.oy);
          if (A.scale) {
            deposit<double, double>(Sc[1], s2, vs, G.ox, G.oy);
            deposit<double, double>(Sc[2], s3, vs, G.ox, G.oy);
            deposit<double, double>(Sc[3], s4, vs, G.ox, G.oy);
          }
        }
      }
      dsum += vsample;
      dsq = fma(vsample, vsample, dsq);
    };
    unsigned head = 0, tail = 0;  // ring positions (wave-uniform)
    for (int base = 0; base < A.n_samples; base += kWave) {
      const int s = base + lane;
      uint32_t roots = 0;
      double q[3], k3x = 0.0, k3y = 0.0, zr[2] = {0.0, 0.0};
      if (s < A.n_samples) {
        uint32_t x0 = (uint32_t)s, x1 = (uint32_t)p1_lin, x2 = (uint32_t)cell, x3 = ((uint32_t)ch.code << 8) | 2u;
        philox4x32_10(x0, x1, x2, x3, A.key0, A.key1);
        double u[5];
        five_uniforms(x0, x1, x2, x3, u);
        for (int a = 0; a < 3; ++a) q[a] = fma(2.0 * G.ph[a], u[a], -G.ph[a]);
        k3x = fma(2.0 * G.ph[0], u[3], -G.ph[0]);
        k3y = fma(2.0 * G.ph[1], u[4], -G.ph[1]);
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
        for (int r = 0; r < 2 && any; ++r) {
          const double z = (lin + (r == 0 ? half : -half)) * inv_2den;
          const double E3 = sqrt64(a3 + z * z);
          bool ok;
          if (!kAlt) ok = (C + 2.0 * Q[2] * z > 0.0) && (E3 < W);
          else ok = ((C + 2.0 * Q[2] * z) * D < 0.0) && (E3 - D > 0.0);
          const double p3[3] = {k3x, k3y, z};
          for (int a = 0; a < 3; ++a) {
            const double other = kAlt ? p3[a] + Q[a] : Q[a] - p3[a];  // p2 or p4
            ok = ok && fabs(p3[a]) <= G.ph[a] && fabs(other) <= G.ph[a];
          }
          if (ok) {
            roots |= 1u << r;
            zr[r] = z;
          }
        }
      }
      const unsigned long long mask = __ballot(roots != 0u);
      if (roots) {
        const unsigned slot = (tail + (unsigned)__popcll(mask & ((1ull << lane) - 1ull))) & (kRootQueueLen - 1);
        for (int a = 0; a < 3; ++a) rq[wid][a][slot] = q[a];
        rq[wid][3][slot] = k3x;
        rq[wid][4][slot] = k3y;
        rq[wid][5][slot] = zr[0];
        rq[wid][6][slot] = zr[1];
        rm[wid][slot] = roots;
      }
      tail += (unsigned)__popcll(mask);
      if (tail - head >= (unsigned)kWave) {
        wave_lds_sync();
        finish((head + lane) & (kRootQueueLen - 1));
        head += kWave;
        wave_lds_sync();
      }
    }
    if (tail != head) {  // the last, partial batch
      wave_lds_sync();
      if ((unsigned)lane < tail - head) finish((head + lane) & (kRootQueueLen - 1));
      wave_lds_sync();
    }
    dsum = wave_sum_dpp(dsum);
    if (A.scale) ssum = wave_sum_dpp(ssum);
    dsq = wave_sum_dpp(dsq);
    const int ok_total = wave_count_dpp(n_ok);
    if (lane == 0) {
      blk.add(ok_total, item_variance(dsum, dsq, A.n_samples), dsum * dsum, ci);
      atomicAdd(Ac[0] + p1_lin, dsum);
      if (A.scale) atomicAdd(Sc[0] + p1_lin, ssum);
      if (A.items) A.items[((size_t)cell * A.n_channels + ci) * G.nodes + p1_lin] = dsum;
    }
  }
  blk.flush(A);  // (begins with a barrier: every wave's deposits are in)
  for (int i = threadIdx.x; i < n_out; i += blockDim.x)
    if (root_acc[i] != 0.0) atomicAdd(A.A + i, root_acc[i]);
}

// ---------------------------------------------------------------------------
// Training data for the proposal: for every item_stride-th work item
// (cell, channel, node; node fastest), n_per_item uniform samples are drawn
// exactly as the uniform sampler draws them and recorded as rows
// [x (8 features), y = logit(u) (5), |value|].  FP64 evaluation.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void record_kernel(CollideArgs A, int n_per_item, long long item_stride,
                                                     long long n_sel, float* __restrict__ rows) {
  const Grid& G = A.G;
  const long long total = n_sel * n_per_item;
  const double pn = sqrt(G.ph[0] * G.ph[0] + G.ph[1] * G.ph[1] + G.ph[2] * G.ph[2]);
  for (long long r = blockIdx.x * (long long)blockDim.x + threadIdx.x; r < total;
       r += (long long)gridDim.x * blockDim.x) {
    const long long j = r / n_per_item;
    const int s = (int)(r % n_per_item);
    const long long w = j * item_stride;
    const int p1_lin = (int)(w % G.nodes);
    const int ci = (int)((w / G.nodes) % A.n_channels);
    const int cell = (int)(w / ((long long)G.nodes * A.n_channels));
    const Channel ch = A.chans[ci];
    Item it;
    load_item(it, A, ch, cell, p1_lin);
    float* out = rows + (size_t)r * 14;
    const double a = sqrt(it.p1[0] * it.p1[0] + it.p1[1] * it.p1[1] + it.p1[2] * it.p1[2]);
    out[0] = (float)(it.p1[0] / G.ph[0]);
    out[1] = (float)(it.p1[1] / G.ph[1]);
    out[2] = (float)(it.p1[2] / G.ph[2]);
    out[3] = (float)(a / pn);
    out[4] = (float)(it.E1 / pn);
    out[5] = (float)(it.mu / (pn * pn));
    out[6] = (float)(ch.sp[0] / 3.0 - 1.0);
    out[7] = A.n_channels > 1 ? (float)(2.0 * ci / (A.n_channels - 1) - 1.0) : 0.0f;
    uint32_t x0 = (uint32_t)s, x1 = (uint32_t)p1_lin, x2 = (uint32_t)cell, x3 = ((uint32_t)ch.code << 8);
    philox4x32_10(x0, x1, x2, x3, A.key0, A.key1);
    double u[5];
    five_uniforms(x0, x1, x2, x3, u);
    for (int d = 0; d < 5; ++d) out[8 + d] = (float)log(u[d] / (1.0 - u[d]));
    double v = 0.0;
    Geo g;
    if (it.E1 > 0.0 && geometry(it, G, u, g)) {
      const double wnb = weight_no_bracket<double>(A, it, g, ch.row);
      const Stencil<double> s2 = make_stencil<double>(g.p2, G);
      const Stencil<double> s3 = make_stencil<double>(g.p3, G);
      const Stencil<double> s4 = make_stencil<double>(g.p4, G);
      const double* f = A.f64;
      const double f2 = interpolate<double>(f + ((size_t)ch.sp[1] * G.cells + cell) * G.nodes, s2, G.ox, G.oy);
      const double f3 = interpolate<double>(f + ((size_t)ch.sp[2] * G.cells + cell) * G.nodes, s3, G.ox, G.oy);
      const double f4 = interpolate<double>(f + ((size_t)ch.sp[3] * G.cells + cell) * G.nodes, s4, G.ox, G.oy);
      const double F1 = is_gluon(ch.sp[0]) ? 1.0 + it.f1 : 1.0 - it.f1;
      const double F2 = is_gluon(ch.sp[1]) ? 1.0 + f2 : 1.0 - f2;
      const double F3 = is_gluon(ch.sp[2]) ? 1.0 + f3 : 1.0 - f3;
      const double F4 = is_gluon(ch.sp[3]) ? 1.0 + f4 : 1.0 - f4;
      v = wnb * (f3 * f4 * F1 * F2 - it.f1 * f2 * F3 * F4);
    }
    out[13] = (float)fabs(v);
  }
}

hipError_t launch_record(const CollideArgs& a, int n_per_item, long long item_stride, long long n_sel, float* rows,
                         hipStream_t stream) {
  const long long total = n_sel * n_per_item;
  long long blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(record_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, a, n_per_item, item_stride, n_sel,
                     rows);
  return hipGetLastError();
}

hipError_t launch_collide_roots(const CollideArgs& a, bool alt, hipStream_t stream) {
  const long long items = (long long)a.G.cells * a.n_group * a.G.nodes;
  const int threads = kRootWaves * kWave;  // the per-wavefront queues are sized for this
  long long blocks = (items * kWave + threads - 1) / threads;
  if (blocks > 4096) blocks = 4096;  // 16 waves per CU; the rest by the grid-stride loop
  if (blocks < 1) blocks = 1;
  // a whole output that fits in 64 KB of dynamic LDS: workgroup-private deposits
  const size_t priv_b = (size_t)kSpecies * a.G.cells * a.G.nodes * sizeof(double);
  const bool priv = a.symmetric && priv_b <= 65536;
  const dim3 grid((unsigned)blocks), block(threads);
  if (priv) {
    if (alt) hipLaunchKernelGGL(HIP_KERNEL_NAME(collide_roots_kernel<true, true>), grid, block, priv_b, stream, a);
    else hipLaunchKernelGGL(HIP_KERNEL_NAME(collide_roots_kernel<false, true>), grid, block, priv_b, stream, a);
  } else {
    if (alt) hipLaunchKernelGGL(HIP_KERNEL_NAME(collide_roots_kernel<true, false>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL(HIP_KERNEL_NAME(collide_roots_kernel<false, false>), grid, block, 0, stream, a);
  }
  return hipGetLastError();
}

}  // namespace qgbe
