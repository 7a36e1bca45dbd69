// Host check (no GPU): after clue_create, runs and read-outs allocate nothing, the
// first ones included; contexts after a process's first allocate their arena only,
// and give back what they took.
#include "clue_api.hip"

#include "fake_hip.h"

int main() {
  constexpr int N = 20000;
  std::vector<float> f(N), rho(N), d2(N);
  std::vector<int32_t> i(N), nh(N), cid(N), fstart(N + 1), flist(N);
  std::vector<uint8_t> seed(N);
  clue_params p{};
  p.dc = 2.0f;
  p.delta_c = 2.0f;
  p.delta_o = 4.0f;
  p.x_max = p.y_max = 50.0f;
  p.n_layers = 3;
  p.flags = CLUE_KEEP_INTERMEDIATES;
  int contexts = 0;
  for (int n : {100, N}) {  // the all-pairs and the tiled form
    for (int batched = 0; batched < 2; ++batched) {
      const int before = g_allocations;
      clue_ctx* c = nullptr;
      if (clue_create(&c, &p, 0, N, 2, 0) != CLUE_OK) {
        std::printf("clue_create: %s\n", clue_last_error(nullptr));
        return 1;
      }
      const int created = g_allocations;
      if (created - before != (contexts++ ? 1 : 2)) {  // the first one also the pinned words
        std::printf("context %d: %d allocations in clue_create\n", contexts, created - before);
        return 1;
      }
      int64_t total = -1;
      const int rc[] = {
          batched ? clue_run_batch(c, n, 2, i.data(), f.data(), f.data(), i.data(), f.data(), cid.data(), seed.data(), nullptr)
                  : clue_run(c, n, f.data(), f.data(), i.data(), f.data(), cid.data(), seed.data(), nullptr),
          clue_get_intermediates(c, rho.data(), nh.data(), d2.data(), nullptr),
          clue_get_followers(c, fstart.data(), flist.data(), nullptr, nullptr),
          clue_get_followers(c, fstart.data(), flist.data(), &total, nullptr),
      };
      const char* const what[] = {"the run", "clue_get_intermediates", "clue_get_followers", "clue_get_followers with its number"};
      for (int k = 0; k < 4; ++k)
        if (rc[k] != CLUE_OK) {
          std::printf("%s: %s\n", what[k], clue_last_error(c));
          return 1;
        }
      if (total != kFollowers) {
        std::printf("%lld followers, want %d\n", (long long)total, kFollowers);
        return 1;
      }
      if (g_allocations != created) {
        std::printf("%d hits, batched %d: %d allocations after clue_create\n", n, batched, g_allocations - created);
        return 1;
      }
      clue_destroy(c);
    }
  }
  // more contexts than there are words: the count is then copied
  std::vector<clue_ctx*> many(kPinnedWords + 3);
  for (int round = 0; round < 2; ++round) {
    for (auto& c : many)
      if (clue_create(&c, &p, 0, 10, 1, 0) != CLUE_OK) return 1;
    for (auto& c : many) {
      int64_t total = -1;
      if (clue_run(c, 10, f.data(), f.data(), i.data(), f.data(), cid.data(), seed.data(), nullptr) != CLUE_OK ||
          clue_get_followers(c, fstart.data(), flist.data(), &total, nullptr) != CLUE_OK || total != kFollowers) {
        std::printf("%zu contexts: %lld followers: %s\n", many.size(), (long long)total, clue_last_error(c));
        return 1;
      }
    }
    int without = 0;
    for (auto& c : many) without += c->total == nullptr;
    if (without != 3 || g_pinned.n_free != 0) {
      std::printf("%d contexts without a word, %d free\n", without, g_pinned.n_free);
      return 1;
    }
    for (auto& c : many) clue_destroy(c);
    if (g_pinned.n_free != kPinnedWords) {
      std::printf("%d words given back\n", g_pinned.n_free);
      return 1;
    }
  }
  std::printf("none\n");
  return 0;
}
