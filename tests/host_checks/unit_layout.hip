// Host check of the unit path's arrays (no GPU): for runs of many sizes, the ranges
// that one launch reads as its verdict or keeps for later are disjoint from those
// that the same launch, or one in between, writes. Prints the first overlap and
// exits with 1.
#include "clue_device.h"

#include <cstdio>
#include <initializer_list>

using namespace clue;

struct Span {
  const char* name;
  const void* lo;
  const void* hi;
};

template <typename T>
static Span span(const char* name, const T* p, int64_t from, int64_t to) {
  return Span{name, p + from, p + to};
}

static int fail(const RunDesc& d, const Geom& g, const Span& a, const Span& b, const char* when) {
  std::printf("n %d events %d layers %d workgroups %d: %s overlaps %s (%s)\n", d.n, d.n_events, g.L, g.units, a.name,
              b.name, when);
  return 1;
}

static bool meet(const Span& a, const Span& b) { return a.lo < b.hi && b.lo < a.hi; }

int main() {
  // the arena's buffers, each at an address of its own; rho and parent adjoin
  Arena a{};
  char* base = (char*)((uintptr_t)1 << 40);
  auto take = [&](int64_t bytes) {
    char* p = base;
    base += (bytes + 255) & ~(int64_t)255;
    return p;
  };
  const int64_t N = 1 << 26;
  a.key = (int32_t*)take(4 * N);
  a.rank = (int32_t*)take(4 * N);
  a.tile_start = (int32_t*)take((int64_t)1 << 33);
  a.xs = (float*)take(4 * N);
  a.ys = (float*)take(4 * N);
  a.es = (float*)take(4 * N);
  a.hs = (int32_t*)take(4 * N);
  a.rho = (float*)take(4 * N);
  a.parent = (int32_t*)take(4 * N);
  a.flags = (uint8_t*)take(N);
  a.seedbits = (uint32_t*)take(N);
  a.ev_start = (int32_t*)take(4 * N);
  a.fstart = (int32_t*)take(4 * N + 4);
  a.cap_chunks = N;
  a.scan_status = (unsigned long long*)take(16 * N);
  a.counters = (int32_t*)take(4 * C_COUNT);

  int taken = 0, refused = 0;
  for (int n : {1, 1000, 8193, 9000, 10000, 20011, 40000, 100000, 1000000, 9000000, 32000000})
    for (int events : {1, 2, 16, 33, 1000})
      for (int layers : {1, 3, 100, 186, 600})
        for (int units : {8, 16, 40, 104, 984, 1024})
          for (int halo : {1, 2, 3})
            for (int cap : {64, 960, 2048}) {
              RunDesc d{};
              d.n = n;
              d.n_events = events;
              Geom g{};
              g.L = layers;
              g.tpl = 2500;
              g.halo = halo;
              g.lds_cap = cap;
              g.units = units;
              if (!unit_space(g, d)) {
                ++refused;
                continue;
              }
              ++taken;
              const int64_t U = (int64_t)events * layers, side = 2 * halo + 1;
              const Span starts = span("unit starts", unit_starts(a, d, g), 0, U + 1);
              const Span counts = span("unit counts", unit_counts(a, d, g), 0, 2 * U);
              const Span verdict = span("verdict", unit_flags(a), 0, units);
              // what k_unit_sort writes: as the unit path ...
              const Span sorts[] = {span("tile_start", a.tile_start, 0, U * g.tpl + 1), span("xs", a.xs, 0, n),
                                    span("ys", a.ys, 0, n), span("es", a.es, 0, n), span("hs", a.hs, 0, n),
                                    span("counters", a.counters, 0, C_COUNT)};
              // ... and as the general path's histogram
              const Span hist[] = {span("key", a.key, 0, n), span("rank", a.rank, 0, n),
                                   span("event starts", a.ev_start, 0, events + 1),
                                   span("fstart", a.fstart, 0, (int64_t)n + 1),
                                   span("scan status", a.scan_status, 0, 2 * a.cap_chunks),
                                   span("seed bits", a.seedbits, 0, seed_words(n))};
              // the spill queues, which the density and nearest-higher stages fill later
              const int64_t chunks = n * side * side / (cap + 1) + n / kWG;
              const Span queue[] = {span("spilled tiles", a.key, 0, chunks), span("spilled slots", a.rank, 0, chunks)};
              for (const Span& s : sorts) {
                if (meet(verdict, s)) return fail(d, g, verdict, s, "read by k_unit_sort, written by the same launch");
                if (meet(starts, s)) return fail(d, g, starts, s, "read by k_unit_sort, written by the same launch");
                if (meet(counts, s)) return fail(d, g, counts, s, "cleared before k_unit_sort, added to after it");
              }
              for (const Span& s : hist)
                if (meet(verdict, s)) return fail(d, g, verdict, s, "read by k_unit_sort, written by the same launch");
              for (const Span& s : queue) {
                if (meet(starts, s)) return fail(d, g, starts, s, "read by k_unit_finish, written before it");
                if (meet(counts, s)) return fail(d, g, counts, s, "added to by the launch that writes it");
              }
              // k_units writes all three in one launch, and clears the counts
              if (meet(verdict, counts)) return fail(d, g, verdict, counts, "written by one launch");
              if (meet(verdict, starts)) return fail(d, g, verdict, starts, "written by one launch");
              // and each lies in its buffer's first n words
              if (starts.lo < a.key || starts.hi > a.key + n) return fail(d, g, starts, hist[0], "outside");
              if (counts.lo < a.rank || counts.hi > a.rank + n) return fail(d, g, counts, hist[1], "outside");
              const Span rho = span("rho and parent", a.rho, 0, 2 * (int64_t)n);
              if (meet(verdict, rho) && (verdict.lo < rho.lo || verdict.hi > rho.hi)) return fail(d, g, verdict, rho, "outside");
            }
  if (!taken || !refused) {
    std::printf("the sizes do not reach both sides of the rule: %d, %d\n", taken, refused);
    return 1;
  }
  std::printf("disjoint in %d runs\n", taken);
  return 0;
}
