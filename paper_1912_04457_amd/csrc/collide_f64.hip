// The FP64 collision kernel.
#include "collide_device.h"

namespace qgbe {

// ---------------------------------------------------------------------------
// FP64 kernel: f read from the FP64 field in global memory, deposits as FP64
// atomics into the output.  This is the reference-precision path.  kPriv (a
// grid whose whole output fits in LDS): the symmetric deposits go to a
// workgroup-private FP64 copy of the output in LDS, in the output's layout,
// flushed once per workgroup, instead of every workgroup's atomics
// contending for the same few global addresses.
// ---------------------------------------------------------------------------
template <bool kLearned, bool kPriv>
__global__ __launch_bounds__(256) void collide_f64_kernel(CollideArgs A) {
  const Grid& G = A.G;
  extern __shared__ double f64_acc[];  // kPriv: [7][cells][nodes], as the output
  const int n_out = kPriv ? kSpecies * G.cells * G.nodes : 0;
  for (int i = threadIdx.x; i < n_out; i += blockDim.x) f64_acc[i] = 0.0;
  __shared__ unsigned long long blk_ok;
  __shared__ double blk_mc[2];
  __shared__ double blk_var[kMaxChannels];
  BlockTotals blk{&blk_ok, blk_mc, blk_var};
  __shared__ Channel s_ch[kMaxChannels];
  __shared__ int s_group[kMaxChannels];
  for (int i = threadIdx.x; i < A.n_group; i += blockDim.x) s_group[i] = A.group[i];
  for (int i = threadIdx.x; i < A.n_channels; i += blockDim.x) s_ch[i] = A.chans[i];
  blk.init();
  const int lane = threadIdx.x & (kWave - 1);
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
    double dsum = 0.0, ssum = 0.0, dsq = 0.0;
    int n_ok = 0;
    const size_t mrow = (size_t)ci * G.nodes + p1_lin;
    const bool mix = kLearned && (!A.mix_on || A.mix_on[ci]);
    for (int s = lane; s < A.n_samples; s += kWave) {
      uint32_t x0 = (uint32_t)s, x1 = (uint32_t)p1_lin, x2 = (uint32_t)cell, x3 = ((uint32_t)ch.code << 8);
      philox4x32_10(x0, x1, x2, x3, A.key0, A.key1);
      double u[5];
      double inv_q = 1.0;
      if (mix) {
        uint32_t y0 = (uint32_t)s, y1 = (uint32_t)p1_lin, y2 = (uint32_t)cell, y3 = ((uint32_t)ch.code << 8) | 1u;
        philox4x32_10(y0, y1, y2, y3, A.key0, A.key1);
        const uint32_t xw[8] = {x0, x1, x2, x3, y0, y1, y2, y3};
        double yl[5];
        const uint32_t* thr = A.mix_thr + mrow * A.mix_K;
        const float* mu = A.mix_mu + mrow * A.mix_K * 5;
        const float* sg = A.mix_sigma + mrow * A.mix_K * 5;
        mix_draw(xw, thr, mu, sg, A.mix_K, u, yl);
        inv_q = 1.0 / mix_density_f64(thr, mu, sg, A.mix_K, yl);
      } else {
        five_uniforms(x0, x1, x2, x3, u);
      }
      Geo g;
      if (!geometry(it, G, u, g)) continue;
      ++n_ok;
      const double wnb = weight_no_bracket<double>(A, it, g, ch.row) * inv_q;
      const Stencil<double> s2 = make_stencil<double>(g.p2, G);
      const Stencil<double> s3 = make_stencil<double>(g.p3, G);
      const Stencil<double> s4 = make_stencil<double>(g.p4, G);
      const double f2 = interpolate<double>(fc[1], s2, G.ox, G.oy);
      const double f3 = interpolate<double>(fc[2], s3, G.ox, G.oy);
      const double f4 = interpolate<double>(fc[3], s4, G.ox, G.oy);
      const double F2 = g2 ? 1.0 + f2 : 1.0 - f2;
      const double F3 = g3 ? 1.0 + f3 : 1.0 - f3;
      const double F4 = g4 ? 1.0 + f4 : 1.0 - f4;
      const double gain = f3 * f4 * F1 * F2, loss = it.f1 * f2 * F3 * F4;
      const double v = wnb * (gain - loss);
      dsum += v;
      dsq = fma(v, v, dsq);
      const double vs = fabs(wnb) * (gain + loss);
      ssum += vs;
      if (kPriv) {
        deposit<double, double, __HIP_MEMORY_SCOPE_WORKGROUP>(f64_acc + (Ac[1] - A.A), s2, v, G.ox, G.oy);
        deposit<double, double, __HIP_MEMORY_SCOPE_WORKGROUP>(f64_acc + (Ac[2] - A.A), s3, -v, G.ox, G.oy);
        deposit<double, double, __HIP_MEMORY_SCOPE_WORKGROUP>(f64_acc + (Ac[3] - A.A), s4, -v, G.ox, G.oy);
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
  for (int i = threadIdx.x; i < n_out; i += blockDim.x)  // kPriv: the same layout as the output
    if (f64_acc[i] != 0.0) atomicAdd(A.A + i, f64_acc[i]);
}

hipError_t launch_collide_f64(const CollideArgs& a, hipStream_t stream) {
  const long long items = (long long)a.G.cells * a.n_group * a.G.nodes;
  const int threads = 256;
  long long blocks = (items * kWave + threads - 1) / threads;
  if (blocks > 4096) blocks = 4096;  // 16 waves per CU; the rest by the grid-stride loop
  if (blocks < 1) blocks = 1;
  // a whole output that fits in the default dynamic LDS: workgroup-private deposits
  const size_t priv_b = (size_t)kSpecies * a.G.cells * a.G.nodes * sizeof(double);
  const bool priv = a.symmetric && priv_b <= 65536;
  const dim3 grid((unsigned)blocks), block(threads);
  if (priv) {
    if (a.learned) hipLaunchKernelGGL(HIP_KERNEL_NAME(collide_f64_kernel<true, true>), grid, block, priv_b, stream, a);
    else hipLaunchKernelGGL(HIP_KERNEL_NAME(collide_f64_kernel<false, true>), grid, block, priv_b, stream, a);
  } else {
    if (a.learned) hipLaunchKernelGGL(HIP_KERNEL_NAME(collide_f64_kernel<true, false>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL(HIP_KERNEL_NAME(collide_f64_kernel<false, false>), grid, block, 0, stream, a);
  }
  return hipGetLastError();
}

}  // namespace qgbe
