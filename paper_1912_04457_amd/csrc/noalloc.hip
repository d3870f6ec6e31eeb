// Collision term without a context and without device allocation: the
// buffers that qgbe_init_grid would allocate (channel table and lists,
// masses and their partial sums, per-launch totals, the FP32 shadow of f and
// its node quads) are carved out of one statically sized device array.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "context.h"

using namespace qgbe;

namespace {

constexpr size_t kScratchBytes = size_t(QGBE_NOALLOC_SCRATCH_MIB) << 20;
constexpr int kMaxDevices = 64;

constexpr size_t align256(size_t n) { return (n + 255) & ~size_t(255); }

// The group lists lie beyond the declared bytes, of which they count 1 KB (as
// the two plain channel lists would): the grids that fit do not depend on
// their length.
constexpr size_t kListBytes = align256(kMaxGroupIndex * sizeof(int));
constexpr size_t kListCounted = 2 * align256(kMaxChannels * sizeof(int));

// One copy per GPU.  Host code never uses this name as an address: it takes
// the device address from hipGetSymbolAddress once per device.
__device__ __align__(256) unsigned char scratch[kScratchBytes + kListBytes];

struct DeviceState {
  bool ready = false;
  unsigned char* ptr = nullptr;   // this device's copy of scratch
  LdsBudget lds[2];               // dynamic LDS budgets [QGBE_FP64, QGBE_FP32]
  int n_cu = 256;
  // what the channel-table region holds (host copy of the last upload)
  std::vector<unsigned char> table;
};

std::mutex g_mu;
DeviceState g_dev[kMaxDevices];

// Once per device, with that device current.
qgbe_status setup(int device, DeviceState** out) {
  std::lock_guard<std::mutex> lock(g_mu);
  DeviceState& s = g_dev[device];
  if (!s.ready) {
    void* p = nullptr;
    HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "scratch address");
    int lds_max = 0;
    HIP_TRY(hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, device), "query LDS size");
    HIP_TRY(collide_f64_lds_limit((size_t)std::max(lds_max, 0), &s.lds[QGBE_FP64]), "raise the dynamic LDS limit");
    HIP_TRY(collide_f32_lds_limit((size_t)std::max(lds_max, 0), &s.lds[QGBE_FP32]), "raise the dynamic LDS limit");
    int n_cu = 0;
    if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess && n_cu > 0)
      s.n_cu = n_cu;
    for (LdsBudget& b : s.lds)
      HIP_TRY(collide_roots_lds_limit((size_t)std::max(lds_max, 0), &b.roots), "raise the dynamic LDS limit");
    s.ptr = static_cast<unsigned char*>(p);
    s.ready = true;
  }
  *out = &s;
  return QGBE_OK;
}

// Bump allocation inside the scratch array.
struct Carve {
  unsigned char* base;
  size_t used = 0;
  template <typename T>
  T* take(size_t n) {
    T* p = reinterpret_cast<T*>(base + used);
    used += align256(n * sizeof(T));
    return p;
  }
};

}  // namespace

extern "C" {

size_t qgbe_noalloc_scratch_bytes(void) { return kScratchBytes; }

qgbe_status qgbe_collision_term_noalloc(const qgbe_grid_desc* desc, const double* f, uint32_t step,
                                        int32_t n_samples, int32_t sampler, double* A) {
  if (!f || !A) return fail(QGBE_EINVAL, "NULL argument");
  qgbe_status st = validate(desc);
  if (st) return st;
  if (n_samples < 1) return fail(QGBE_EINVAL, "n_samples must be >= 1");
  if (sampler != QGBE_SAMPLER_UNIFORM && sampler != QGBE_SAMPLER_ROOTS && sampler != QGBE_SAMPLER_ROOTS_ALT)
    return fail(QGBE_EINVAL, "sampler must be uniform or one of the root samplers (no proposal table here)");
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev == 0) return fail(QGBE_EDEVICE, "no HIP device");
  if (desc->device < 0 || desc->device >= std::min(ndev, kMaxDevices))
    return fail(QGBE_EINVAL, "device ordinal out of range");
  HIP_TRY(hipSetDevice(desc->device), "hipSetDevice");
  DeviceState* dev = nullptr;
  st = setup(desc->device, &dev);
  if (st) return st;

  // A context on the stack: the launch plan of qgbe_init_grid, with every
  // device buffer inside scratch.
  qgbe_ctx c;
  c.d = *desc;
  c.stream = (hipStream_t)desc->stream;
  make_grid(desc, c.G);
  c.chans.resize(kMaxChannels);
  c.nch = build_channels(desc->species_mask, desc->row_mask, c.chans.data(), kMaxChannels);
  c.chans.resize(c.nch);
  c.lds = dev->lds[desc->precision];
  c.n_cu = dev->n_cu;
  c.step = step;
  plan_groups(&c);

  const size_t n = field_len(&c);
  const int nch1 = std::max(1, c.nch);
  const bool fp32 = desc->precision == QGBE_FP32 && sampler == QGBE_SAMPLER_UNIFORM;
  Carve cv{dev->ptr};
  c.d_chans = cv.take<Channel>(kMaxChannels);
  c.d_groups = cv.take<int>(kMaxGroupIndex);
  const size_t table_bytes = cv.used;
  c.d_mass2 = cv.take<double>((size_t)kSpecies * c.G.cells);
  c.d_mass_part = cv.take<double>(mass_scratch(c.G));
  c.d_count = cv.take<unsigned long long>(kStripes);
  c.d_mc = cv.take<double>((size_t)kStripes * (2 + nch1));
  c.d_chan_var = c.d_mc + 2 * kStripes;
  const size_t limit = kScratchBytes + kListBytes - kListCounted;
  if (fp32) {
    c.d_f32 = cv.take<float>(n);
    // Node quads that only the smaller sample queue would read (f tiles of every
    // slot fit in LDS) give way where they do not fit.
    bool tiles = true;
    for (const Group& g : c.groups)
      tiles = tiles && g.lds_tiles[0] == g.nslot && g.queue[0] != kRing && g.queue[1] != kRing;
    if (c.need_quads[0] && tiles && cv.used + align256(n * sizeof(float4)) > limit) {
      for (Group& g : c.groups) g.queue[0] = g.queue[1] = 0;
      c.need_quads[0] = false;
    }
    if (c.need_quads[0] && cv.used + align256(n * sizeof(float4)) > limit)
      plan_groups(&c, true);  // the tiles that only the long-item form's LDS holds: refused if they need quads too
    if (c.need_quads[0]) c.d_f32q = cv.take<float4>(n);
  }
  if (cv.used > limit)
    return fail(QGBE_EINVAL, "grid needs " + std::to_string(cv.used - (limit - kScratchBytes)) +
                                 " bytes of scratch, more than the " + std::to_string(kScratchBytes) +
                                 " of qgbe_collision_term_noalloc");
  carve_records(&c, dev->ptr + cv.used, limit - cv.used);  // what is left
  c.d_f = const_cast<double*>(f);  // read only: masses and the collision kernels

  // Channel table and group lists, uploaded when they differ
  // from what this device's scratch holds and waited for; the host record of
  // what the scratch holds changes only after the upload has completed, so a
  // failed upload is retried by the next call.
  std::vector<unsigned char> tab(table_bytes, 0);
  std::memcpy(tab.data(), c.chans.data(), c.chans.size() * sizeof(Channel));
  std::memcpy(tab.data() + ((unsigned char*)c.d_groups - dev->ptr), c.group_index.data(),
              c.group_index.size() * sizeof(int));
  {
    std::lock_guard<std::mutex> lock(g_mu);
    if (dev->table != tab) {
      dev->table.clear();
      HIP_TRY(hipMemcpyAsync(dev->ptr, tab.data(), table_bytes, hipMemcpyHostToDevice, c.stream),
              "copy channel table");
      HIP_TRY(hipStreamSynchronize(c.stream), "synchronise");
      dev->table = std::move(tab);
    }
  }

  st = start_term(&c, sampler, A, true);
  if (st) return st;
  return run_collide(&c, n_samples, sampler, A, nullptr, nullptr);
}

}  // extern "C"
