// The root-parameterisation samplers and the sample recorder.
#include "collide_slots.h"

namespace qgbe {
namespace {

// The root samplers' kernel variants: [direct, symmetric, symmetric with global
// atomics][scale][user terms].
template <int kRoot>
using RootFn = void (*)(CollideArgs);
template <int kRoot>
void root_variants(RootFn<kRoot> out[3][2][2]) {
  out[0][0][0] = collide_slots_kernel<double, false, false, true, false, 0, false, true, false, kRoot>;
  out[0][0][1] = collide_slots_kernel<double, false, false, true, false, 0, true, true, false, kRoot>;
  out[0][1][0] = collide_slots_kernel<double, false, true, true, false, 0, false, true, false, kRoot>;
  out[0][1][1] = collide_slots_kernel<double, false, true, true, false, 0, true, true, false, kRoot>;
  out[1][0][0] = collide_slots_kernel<double, true, false, true, false, 0, false, true, false, kRoot>;
  out[1][0][1] = collide_slots_kernel<double, true, false, true, false, 0, true, true, false, kRoot>;
  out[1][1][0] = collide_slots_kernel<double, true, true, true, false, 0, false, true, false, kRoot>;
  out[1][1][1] = collide_slots_kernel<double, true, true, true, false, 0, true, true, false, kRoot>;
  out[2][0][0] = collide_slots_kernel<double, true, false, false, false, 0, false, true, false, kRoot>;
  out[2][0][1] = collide_slots_kernel<double, true, false, false, false, 0, true, true, false, kRoot>;
  out[2][1][0] = collide_slots_kernel<double, true, true, false, false, 0, false, true, false, kRoot>;
  out[2][1][1] = collide_slots_kernel<double, true, true, false, false, 0, true, true, false, kRoot>;
}

template <int kRoot>
hipError_t launch_roots(const CollideArgs& a, hipStream_t stream) {
  const int n_acc = a.symmetric ? std::min(a.slot_hi - a.slot_lo, a.lds_acc) : 0;
  const bool all_acc = !a.symmetric || n_acc == a.slot_hi - a.slot_lo;
  if (!all_acc && (n_acc || a.win_n != a.G.nodes)) return hipErrorInvalidValue;
  const int waves = kSlotThreads / kWave;
  if (a.split < 1 || waves % a.split || (a.split > 1 && a.chunk_items > kSplitNodes)) return hipErrorInvalidValue;
  if (a.node_block < 1 || a.node_block > kMaxNodeBlock) return hipErrorInvalidValue;
  const long long blocks = (long long)a.G.cells * a.n_group * a.n_chunks;
  if (blocks <= 0) return hipSuccess;
  RootFn<kRoot> fns[3][2][2];
  root_variants<kRoot>(fns);
  hipLaunchKernelGGL(fns[!a.symmetric ? 0 : all_acc ? 1 : 2][a.scale ? 1 : 0][a.msq_mask ? 1 : 0], dim3((unsigned)blocks),
                     dim3(kSlotThreads), (size_t)n_acc * a.win_n * sizeof(double), stream, a);
  return hipGetLastError();
}

template <int kRoot>
hipError_t launch_roots_rec(const CollideArgs& a, int n_wg, hipStream_t stream) {
  if (n_wg <= 0) return hipSuccess;
  if (!record_fits(a, n_wg, 2)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)n_wg), block(kSlotThreads);
  if (a.msq_mask)
    hipLaunchKernelGGL((collide_slots_kernel<double, true, false, true, false, 0, true, true, true, kRoot>), grid,
                       block, 0, stream, a);
  else
    hipLaunchKernelGGL((collide_slots_kernel<double, true, false, true, false, 0, false, true, true, kRoot>), grid,
                       block, 0, stream, a);
  return hipGetLastError();
}

template <int kRoot>
hipError_t roots_lds_limit_of(size_t lds_max, size_t* out) {
  RootFn<kRoot> fns[3][2][2];
  root_variants<kRoot>(fns);
  for (int i = 0; i < 8; ++i)
    if (const hipError_t e = raise_lds_limit((const void*)fns[i >> 2][(i >> 1) & 1][i & 1], lds_max, out)) return e;
  return hipSuccess;
}

inline hipError_t roots_lds_limit(size_t lds_max, size_t* out) {
  *out = lds_max;
  const hipError_t e = roots_lds_limit_of<1>(lds_max, out);
  return e != hipSuccess ? e : roots_lds_limit_of<2>(lds_max, out);
}

}  // namespace

hipError_t launch_collide_roots(const CollideArgs& a, bool alt, hipStream_t stream) {
  return alt ? launch_roots<2>(a, stream) : launch_roots<1>(a, stream);
}

hipError_t launch_record_roots(const CollideArgs& a, bool alt, int n_wg, hipStream_t stream) {
  return alt ? launch_roots_rec<2>(a, n_wg, stream) : launch_roots_rec<1>(a, n_wg, stream);
}

hipError_t collide_roots_lds_limit(size_t lds_max, size_t* out) { return roots_lds_limit(lds_max, out); }

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
    if (it.E1 > 0.0 && geometry(it, G, map_words(G, x0, x1, x2, x3), g)) {
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

}  // namespace qgbe
