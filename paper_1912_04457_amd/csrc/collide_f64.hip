// The collision kernel of the CM-angle samplers, FP64 integrand.
#include "collide_slots.h"

namespace qgbe {

hipError_t launch_collide_f64(const CollideArgs& a, int nslot, int queue, hipStream_t stream) {
  return launch_slots<double>(a, nslot, queue, stream);
}

hipError_t launch_record_f64(const CollideArgs& a, int n_wg, hipStream_t stream) {
  return launch_rec<double>(a, n_wg, stream);
}

size_t collide_f64_record_tile() { return record_tile_bytes<double>(); }

hipError_t launch_replay_f64(const ReplayArgs& a, hipStream_t stream) { return launch_replay<double>(a, stream); }

hipError_t collide_f64_lds_limit(size_t lds_max, LdsBudget* out) { return slots_lds_limit<double>(lds_max, out); }

}  // namespace qgbe
