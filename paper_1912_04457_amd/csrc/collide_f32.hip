// The collision kernel of the CM-angle samplers, FP32 integrand.
#include "collide_slots.h"
#include "qgbe.h"

namespace qgbe {

int collide_waves(bool queue) { return slots_block(queue) / kWave; }
int collide_node_block(bool queue) { return queue ? kNodeBlock : 1; }
bool collide_short(int precision, bool learned, int split, int n_samples) {
  return precision == QGBE_FP64 || learned || short_items(split, n_samples);
}

hipError_t launch_collide_f32(const CollideArgs& a, int nslot, int queue, hipStream_t stream) {
  return launch_slots<float>(a, nslot, queue, stream);
}

hipError_t launch_record_f32(const CollideArgs& a, int n_wg, hipStream_t stream) {
  return launch_rec<float>(a, n_wg, stream);
}

size_t collide_f32_record_tile() { return record_tile_bytes<float>(); }

hipError_t launch_replay_f32(const ReplayArgs& a, hipStream_t stream) { return launch_replay<float>(a, stream); }

hipError_t collide_f32_lds_limit(size_t lds_max, LdsBudget* out) { return slots_lds_limit<float>(lds_max, out); }

}  // namespace qgbe
