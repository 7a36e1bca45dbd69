// Host check of the geometry that untuned runs take (no GPU): over many extents,
// distances and requested tiles it never needs more tiles than the requested one,
// which the arena is sized for, stays within what the kernels stage, and keeps the
// requested tile where a run has few layers (one crowded spot in each is then what
// it waits for, and a query's lists grow with the tile).
#include "clue_api.hip"

#include <random>

namespace clue {
// the kernels' side of the library, which nothing here calls
const char* const kStageNames[S_COUNT] = {};
hipError_t launch_pipeline(const Geom&, const Arena&, const RunDesc&, const LaunchCfg&, hipStream_t, hipEvent_t*) {
  return hipErrorUnknown;
}
hipError_t launch_direct(const Geom&, const Arena&, const RunDesc&, hipStream_t, hipEvent_t*) { return hipErrorUnknown; }
hipError_t launch_set_desc(const RunDesc&, RunDesc*, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_read_out(const ReadOut&, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_event_ids(int32_t*, const int64_t*, int32_t, int32_t, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_validate(const Geom&, const Arena&, const RunDesc&, hipStream_t) { return hipErrorUnknown; }
int occupancy_blocks_per_cu(int, int) { return 1; }
int lds_bytes_for(const Geom&) { return 0; }
int lds_bytes_nh(const Geom&) { return 0; }
}  // namespace clue

int main() {
  std::mt19937 rng(7);
  auto uni = [&](double lo, double hi) { return std::uniform_real_distribution<double>(lo, hi)(rng); };
  auto logu = [&](double lo, double hi) { return std::exp(uni(std::log(lo), std::log(hi))); };
  int planned = 0, three = 0, coarser = 0;
  for (int i = 0; i < 200000; ++i) {
    clue_params p{};
    p.dc = (float)logu(1e-3, 1e2);
    p.delta_c = (float)(p.dc * uni(0.0, 4.0));
    p.delta_o = (float)(p.dc * uni(0.0, 4.0));
    const double wx = p.dc * logu(0.5, 500.0), wy = p.dc * logu(0.5, 500.0);
    // an origin at up to 10^6 dc: rounding of the coordinates then widens the windows
    const double ox = i % 3 ? 0.0 : p.dc * logu(1.0, 1e6), oy = i % 6 ? 0.0 : p.dc * logu(1.0, 1e6);
    p.x_min = (float)ox;
    p.y_min = (float)(i % 2 ? oy : -oy);
    p.x_max = (float)(ox + wx);
    p.y_max = (float)(p.y_min + wy);
    p.n_layers = 1 + i % 400;
    p.tile_size = i % 4 ? (float)(p.dc * uni(1.0, 6.0)) : 0.0f;
    Geom req{};
    std::string msg;
    if (plan_geom(p, p.tile_size, 1, 8, 8, kDefaultLdsCap, -1.0f, 1, 1, req, msg) != CLUE_OK) continue;
    ++planned;
    three += req.maxl > 2;
    for (double per_layer : {0.01, 1.0, 100.0, 1000.0, 1900.0, 10000.0, 1e6}) {
      const double units = p.n_layers;
      const Geom g = run_geom(p, req, 1, kDefaultLdsCap, -1.0f, 1, 1, per_layer * units, units);
      const int rw = std::min(g.bx + 2 * g.halo, g.nx), rh = std::min(g.by + 2 * g.halo, g.ny);
      const char* what = g.tpl > req.tpl ? "more tiles than the arena holds"
                         : g.inv_t > req.inv_t ? "a smaller tile than the requested one"
                         : g.maxl > req.maxl ? "a density window of more tiles"
                         : rh > kMaxRegionRows || rh * (rw + 1) > kMaxRegionTiles || g.ts_ints < rh * (rw + 1) + 1
                             ? "a region over the staged limit"
                         : req.maxl == 2 && units < 256.0 && g.inv_t != req.inv_t
                             ? "a grown tile in a run of fewer layers than CUs"
                         : g.bx > 24 || g.by > 24 || g.bx < 1 || g.by < 1 ? "a block over the walk's limit"
                                                                          : nullptr;
      if (what) {
        std::printf("%s: dc %g delta %g %g extent [%g, %g] x [%g, %g] tile %g -> %g, %d -> %d tiles a layer\n", what,
                    p.dc, p.delta_c, p.delta_o, p.x_min, p.x_max, p.y_min, p.y_max, 1.0 / req.inv_t, 1.0 / g.inv_t,
                    req.tpl, g.tpl);
        return 1;
      }
      coarser += g.inv_t < req.inv_t;
    }
  }
  if (planned < 10000 || three < 1000 || coarser < 1000) {
    std::printf("the draws miss a side of the rule: %d planned, %d of three tiles, %d coarser\n", planned, three, coarser);
    return 1;
  }
  std::printf("%d geometries\n", planned);
  return 0;
}
