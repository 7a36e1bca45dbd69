// Host check (no GPU): which LDS cap a tuned run takes. plain_lds_cap is tuned on one
// event and holds for runs of one event; batches of several take lds_cap.
#include "clue_api.hip"

#include "fake_hip.h"

int main() {
  constexpr int N = 3000000;
  std::vector<float> f(N);
  std::vector<int32_t> i(N), cid(N);
  std::vector<uint8_t> seed(N);
  clue_params p{};
  p.dc = 2.0f;
  p.delta_c = 2.0f;
  p.delta_o = 4.0f;
  p.x_max = p.y_max = 200.0f;
  p.n_layers = 100;
  clue_ctx* c = nullptr;
  if (clue_create(&c, &p, 0, N, 16, 0) != CLUE_OK) {
    std::printf("clue_create: %s\n", clue_last_error(nullptr));
    return 1;
  }
  clue_tuning t{};
  t.block_x = t.block_y = 10;
  t.lds_cap = 800;
  t.plain_lds_cap = 1024;
  t.nh_first_radius = -1.0f;
  if (clue_set_tuning(c, &t) != CLUE_OK) {
    std::printf("clue_set_tuning: %s\n", clue_last_error(c));
    return 1;
  }
  struct {
    int n, events;
    bool batched;
    int cap;
  } const cases[] = {{9000, 1, false, 1024},    {9000, 1, true, 1024},  {9000, 2, true, 800}, {480000, 16, true, 800},
                     {1000000, 1, false, 1024}, {1000000, 1, true, 1024}, {2000000, 2, true, 800}};
  for (const auto& k : cases) {
    const int rc = k.batched ? clue_run_batch(c, k.n, k.events, i.data(), f.data(), f.data(), i.data(), f.data(), cid.data(),
                                              seed.data(), nullptr)
                             : clue_run(c, k.n, f.data(), f.data(), i.data(), f.data(), cid.data(), seed.data(), nullptr);
    if (rc != CLUE_OK || g_graph || g_ran.lds_cap != k.cap) {
      std::printf("%d hits in %d events, batched %d: status %d, graph %d, cap %d, want %d\n", k.n, k.events, k.batched, rc,
                  g_graph, g_ran.lds_cap, k.cap);
      return 1;
    }
  }
  clue_destroy(c);
  std::printf("as tuned\n");
  return 0;
}
