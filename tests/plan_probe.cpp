// Prints the launch plans that the library makes, for tests on the host: one
// line of numbers in (see main), one JSON object out.
#include <algorithm>
#include <cstdio>
#include <iostream>
#include <sstream>
#include <string>

#include "context.h"

using namespace qgbe;

static void print(const char* name, const std::vector<int>& v) {
  std::printf("\"%s\": [", name);
  for (size_t i = 0; i < v.size(); ++i) std::printf("%s%d", i ? ", " : "", v[i]);
  std::printf("], ");
}

int main() {
  std::string line;
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    qgbe_grid_desc d{};
    size_t plain[2], learned[2], roots, replay, queue[2][2];
    bool long_form;
    int n_samples;
    long long capacity;
    in >> d.species_mask >> d.n_x[0] >> d.n_x[1] >> d.n_x[2] >> d.n_p[0] >> d.n_p[1] >> d.n_p[2] >> d.precision >>
        d.symmetric >> long_form >> plain[0] >> plain[1] >> learned[0] >> learned[1] >> roots >> replay >> queue[0][0] >>
        queue[0][1] >> queue[1][0] >> queue[1][1] >> n_samples >> capacity;
    if (!in) return 2;
    d.row_mask = 0x7F;
    d.alpha_s = 0.5;
    for (int a = 0; a < 3; ++a) d.x_half[a] = d.p_half[a] = 1.0;
    if (validate(&d) != QGBE_OK) return 3;
    qgbe_ctx c;
    c.d = d;
    make_grid(&d, c.G);
    c.chans.resize(kMaxChannels);
    c.nch = build_channels(d.species_mask, d.row_mask, c.chans.data(), kMaxChannels);
    c.chans.resize(c.nch);
    for (int i = 0; i < 2; ++i) {
      c.lds.plain[i] = plain[i];
      c.lds.learned[i] = learned[i];
    }
    c.lds.roots = roots;
    c.lds.replay = replay;
    for (int i = 0; i < 4; ++i) c.lds.queue[i / 2][i % 2] = queue[i / 2][i % 2];
    plan_groups(&c, long_form);
    std::printf("{\"nch\": %d, ", c.nch);
    print("lists", c.group_index);
    std::vector<int> sp, slots;
    for (const Channel& ch : c.chans) {
      slots.push_back(ch.nslot);
      for (int p = 0; p < 4; ++p) sp.push_back(ch.sp[p]);
    }
    print("species", sp);
    print("nslot", slots);
    std::vector<int> start, count;
    for (const Replay& r : c.replay) {
      start.push_back(r.start);
      count.push_back(r.count);
    }
    print("replay_start", start);
    print("replay_count", count);
    std::printf("\"groups\": [");
    for (size_t i = 0; i < c.groups.size(); ++i) {
      const Group& g = c.groups[i];
      std::printf("%s{\"nslot\": %d, \"queue\": [%d, %d]", i ? ", " : "", g.nslot, g.queue[0], g.queue[1]);
      for (int l = 0; l < 3; ++l)
        std::printf(", \"%d\": {\"acc\": %d, \"tiles\": %d, \"win\": %d, \"long\": %d, \"several\": %d}", l,
                    g.lds_acc[l], g.lds_tiles[l], g.win[l], (int)g.long_form[l], (int)several_launches(&c, g, l));
      std::printf("}");
    }
    std::printf("], ");
    std::vector<int> route;  // of each sampler, without and with the scale output
    for (int l = 0; l < 3; ++l)
      for (int scale = 0; scale < 2; ++scale) route.push_back((int)deposit_route(&c, l, n_samples, scale, capacity));
    print("route", route);
    // chunks without a queue and with one, for the uniform and the learned (or a root) sampler
    std::vector<int> chunks;
    for (int i = 0; i < 4; ++i)
      chunks.push_back(plan_chunks(&c, c.G.nodes, (long long)c.G.cells * std::max(1, c.nch), c.G.nodes, n_samples, i & 1,
                                   i & 2, long_form && d.precision == QGBE_FP32).chunk);
    print("chunks", chunks);
    const Chunking direct = plan_chunks(&c, c.G.nodes, (long long)c.G.cells * std::max(1, c.nch), 0, n_samples, false,
                                        false, false);
    print("direct", {direct.chunk, direct.split, direct.block});
    // the recording launches: some of them as [first workgroup, those of replay_batch]
    std::printf("\"batches\": {");
    c.rec_wgs = 1 << 16;
    for (int l = 0; l < 3; ++l) {
      std::printf("%s\"%d\": [", l ? ", " : "", l);
      if (c.replay[l].count && n_samples <= capacity) {
        const ReplayPlan p = plan_replay(&c, l, n_samples, capacity);
        std::printf("[%d, %d, %d, %lld, %lld, %lld, %lld]", p.chunks.chunk, p.n_chunks, p.n_group, p.capacity, p.region, p.wgs,
                    p.per);
        const long long n = (p.wgs + p.per - 1) / p.per, step = std::max(1LL, n / 50);
        for (long long i = 0; i < n; i += i + step < n || i == n - 1 ? step : n - 1 - i) {
          const ReplayBatch b = replay_batch(p, i * p.per);
          std::printf(", [%lld, %d, %d, %d, %d, %d, %d]", i * p.per, b.n_wg, b.cell_lo, b.wg_base, b.n_cells, b.gi_lo, b.gi_hi);
        }
      }
      std::printf("]");
    }
    std::printf("}, ");
    std::printf("\"quads\": %d}\n", (int)c.need_quads[0]);
  }
  return 0;
}
