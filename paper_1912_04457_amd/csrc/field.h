// Launch interface of the field kernels (masses, drift + update, observables).
#pragma once

#include "qgbe_common.h"

namespace qgbe {

struct Mass7 {
  double v[kSpecies];
};

// Observables layout in `out` (length observables_len): per species
// [N, E, Px, Py, Pz, M, S, Txx, Tyy, Tzz] (7 x 10) with M = sum N dV m^2 f / E,
// S the entropy and Tii = sum N dV p_i^2 f / E, then min f, max fermion f,
// non-finite count.
constexpr int kObsPer = 10;
constexpr int observables_len = kSpecies * kObsPer + 3;

// The start of a collision term: thermal masses (Eq. mg, Eq. mq) of f into
// mass2, and what else is given, in one pass over f.
struct TermStart {
  Grid G;
  const double* f;
  const double* lag;         // lagged masses, or NULL: E = |p|
  double* part;              // mass_scratch(G) doubles; NULL: the constant masses
  Mass7 constant;
  double* mass2;
  unsigned* done;            // [cells] zero, left zero; NULL: the chunk sums are added by a second kernel
  double* A;                 // optional [7][cells][nodes]: zeroed
  unsigned long long* count; // optional: n_count zeroed
  int n_count;
  double* totals;            // optional: n_totals zeroed
  int n_totals;
  float* f32;                // optional: FP32 copy of f
  float4* quads;             // optional: node quads of the FP32 field: q[i] = (f[i], f[i+1], f[i+oy], f[i+oy+1])
                             // within each (species, cell) block, so a trilinear read takes two 16-byte loads;
                             // entries on the last z or y layer (never a stencil base) repeat f[i]
};
size_t mass_scratch(const Grid& G);
hipError_t launch_term_start(const TermStart& a, hipStream_t st);
// One step; lag receives mass2.
hipError_t launch_update(const Grid& G, const double* f, const double* A, const double* mass2, double dt,
                         int scheme, double* f_out, float* f32, double* lag, hipStream_t st);
size_t observables_scratch(const Grid& G);
hipError_t launch_observables(const Grid& G, const double* f, const double* mass2, double* scratch,
                              double* out, hipStream_t st);
// out[0] = E_source, out[1] = E_collide of a step (mass2_prev NULL: no
// source term); scratch as for launch_observables.
hipError_t launch_energy_budget(const Grid& G, const double* f, const double* A, const double* mass2,
                                const double* mass2_prev, double dt, double* scratch, double* out, hipStream_t st);
// src into f, its second buffer and its FP32 shadow.
hipError_t launch_set_field(const double* src, double* f, double* f_next, float* f32, size_t n, hipStream_t st);
hipError_t launch_fill(double* dst, double v, size_t n, hipStream_t st);

}  // namespace qgbe
