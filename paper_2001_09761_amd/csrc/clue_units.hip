// The unit path: grid build, numbering, labels and follower lists of runs whose
// hits come grouped by (event, layer) unit.
//
// Neighbours and links never leave a unit, so when a unit's hits lie together
// in the caller's arrays, one workgroup can order them by tile, and later
// resolve their links, in LDS: the unit's first hit is also its first slot, no
// count or offset has to meet another unit's, and the scattered accesses stay
// within a few tens of KB. Whether the hits are grouped is known on the device
// only:
//   k_units        finds the units' first hits; a hit whose unit is smaller
//                  than the hit's before it, or a unit too large for LDS, rules
//                  the path out for the run
//   k_unit_sort    tile CSR and records of each unit; or, with the path ruled
//                  out, the general path's histogram
//   k_unit_finish  labels, seed flags and follower lists of each unit; or the
//                  general path's labels
// The general path's other stages (scans, scatter, placement, list sort) are
// launched too, and return at once in a run that takes the unit path (2 to 5 us
// each; merging the general stages into fewer launches with waits between their
// chunks cost such runs 36 us a wait, in L2 write-backs).
//
// What it measured, 32 events of 1M hits: grid build 846 -> 338 us (copying its
// inputs and outputs alone would take 240), labels and lists 617 -> 258 us, and
// the nearest-higher stage 1,025 -> 955 us without the follower-count atomics.
// The grid build is bound by the latency of its phases (count, scan, place, three
// columns), which two units per CU overlap; the finish by that of its LDS chases.
#include "clue_device.h"

#include <algorithm>

namespace clue {

namespace {

constexpr int kUWG = 1024;
constexpr int kUPer = kUnitMax / kUWG;  // hits per lane of a full unit
constexpr int kUWaves = kUWG / 64;
// Hits per lane of a general stage (the histogram's chunks are taken by four
// groups of kWG lanes side by side, the labels' by the workgroup). Every
// workgroup has an equal share of the hits, [return, end), and every XCD a
// contiguous run of shares: one or two large workgroups per CU leave no room for
// the dispatcher to even out whole chunks.
constexpr int kSideU = 2;
__device__ __forceinline__ int own_share(int n, int& end) {
  const int64_t per = gridDim.x / kQueues, i = (int)blockIdx.x % kQueues * per + (int)blockIdx.x / kQueues;
  end = (int)((i + 1) * n / gridDim.x);
  return (int)(i * n / gridDim.x);
}
static_assert(kUnitMax % kUWG == 0 && kUnitMax <= 16384, "unit-local indices are 16-bit, and 14 in k_unit_sort");
static_assert(kUnitTiles <= 4096 && kUnitTiles <= 4 * kUWG, "12-bit tiles, four to a lane in the scan");

// The same value, as far as the compiler knows a new one: the indices a phase
// derives from it are then not kept in registers for the next phase.
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

}  // namespace

// ---------------------------------------------------------------------------
// First hit of every unit and event, and this workgroup's verdict on the path
// in its slot of unit_flags. A unit of more than kUnitMax hits is seen by the
// hits at multiples of 64 whose unit is also that of the hit kUnitMax - 64
// before them.
// ---------------------------------------------------------------------------
template <bool G>
__global__ __launch_bounds__(kWG) void k_units(DescArg<G> dg, Geom g, Arena a) {
  const RunDesc d = dg.get();
  const int64_t stride = (int64_t)gridDim.x * kWG;
  const int64_t i0 = (int64_t)blockIdx.x * kWG + threadIdx.x;
  for (int64_t i = i0; i < C_COUNT; i += stride) a.counters[i] = 0;
  // event starts are written below too, so the tile counts alone are cleared here
  const int64_t tt = (int64_t)d.n_events * g.L * g.tpl + 1;
  for (int64_t i = i0; i < tt; i += stride) a.tile_start[i] = 0;
  if (!unit_space(g, d)) return;  // k_unit_sort sees the same
  const int U = d.n_events * g.L;
  int32_t* const us = unit_starts(a, d, g);
  int32_t* const uc = unit_counts(a, d, g);
  for (int64_t i = i0; i < 2 * U; i += stride) uc[i] = 0;
  bool bad = false;
  constexpr int V = 8, C = kWG * V;
  const int lane = threadIdx.x & 63;
  for (ChunkRun r = xcd_run(d.n, C); r.c < r.end; r.c += r.step) {
    const int h0 = r.c * C + (int)threadIdx.x, w0 = h0 - lane;
    // every load first: the hits' ids, those of the hit before each wave's
    // first and those kUnitMax - 64 before it
    int l[V], lp[V], lf[V], e[V], ep[V], ef[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
      l[j] = d.layer[min(h0 + j * kWG, d.n - 1)];
      lp[j] = d.layer[clampi(w0 + j * kWG - 1, 0, d.n - 1)];
      lf[j] = d.layer[clampi(w0 + j * kWG - (kUnitMax - 64), 0, d.n - 1)];
      e[j] = ep[j] = ef[j] = 0;
    }
    if (d.event) {
#pragma unroll
      for (int j = 0; j < V; ++j) {
        e[j] = d.event[min(h0 + j * kWG, d.n - 1)];
        ep[j] = d.event[clampi(w0 + j * kWG - 1, 0, d.n - 1)];
        ef[j] = d.event[clampi(w0 + j * kWG - (kUnitMax - 64), 0, d.n - 1)];
      }
#pragma unroll
      for (int j = 0; j < V; ++j) {
        e[j] = clampi(e[j] - d.event_base, 0, d.n_events - 1) * g.L;
        ep[j] = clampi(ep[j] - d.event_base, 0, d.n_events - 1) * g.L;
        ef[j] = clampi(ef[j] - d.event_base, 0, d.n_events - 1) * g.L;
      }
    }
#pragma unroll
    for (int j = 0; j < V; ++j) {
      const int h = h0 + j * kWG, w = w0 + j * kWG;
      const int u = e[j] + clampi(l[j], 0, g.L - 1);
      int up = __shfl_up(u, 1, 64);
      if (lane == 0) up = w == 0 ? -1 : ep[j] + clampi(lp[j], 0, g.L - 1);
      const int uf = w >= kUnitMax - 64 ? ef[j] + clampi(lf[j], 0, g.L - 1) : -1;
      bad |= h < d.n && (up > u || (lane == 0 && uf == u));
      if (__any(bad) || h >= d.n) continue;  // the run is ruled out: nothing here is read
      for (int v = up + 1; v <= u; ++v) {
        us[v] = h;
        if (v % g.L == 0) a.ev_start[v / g.L] = h;
      }
      if (h == d.n - 1) {
        for (int v = u + 1; v <= U; ++v) {
          us[v] = d.n;
          if (v % g.L == 0) a.ev_start[v / g.L] = d.n;
        }
      }
    }
  }
  bad = __syncthreads_or(bad);
  if (threadIdx.x == 0) unit_flags(a)[blockIdx.x] = bad;
}

// ---------------------------------------------------------------------------
// Tile CSR and records of each unit: a counting sort by tile that keeps the
// order of the hits.
//
// Each wave takes a contiguous sixteenth of the unit and counts its hits per
// tile in bytes of its own, by LDS atomics whose results rank its hits; a
// prefix over the waves and the tiles then gives every hit its slot. That the
// atomics of one wave's instruction are served in lane order is not promised,
// so the result is checked: if any tile's hits are out of order, or a byte
// overflows (more than 255 hits of one tile), each slot of the unit counts the
// smaller indices of its tile instead. The records then go through LDS one
// column at a time, so that all global accesses are in order.
// ---------------------------------------------------------------------------
template <bool G>
__global__ __launch_bounds__(kUWG, 8) void k_unit_sort(DescArg<G> dg, Geom g, Arena a) {
  // dynamic LDS: wave counts (bytes [16][tpl]), later a column [kUnitMax]; slot -> hit; tile offsets
  extern __shared__ __align__(16) unsigned char lds[];
  unsigned* const cnt4 = reinterpret_cast<unsigned*>(lds);  // four bytes a word
  float* const col = reinterpret_cast<float*>(lds);
  unsigned short* const alt = reinterpret_cast<unsigned short*>(lds);
  unsigned short* const srt = reinterpret_cast<unsigned short*>(lds + 4 * kUnitMax);
  unsigned short* const start = srt + kUnitMax;  // [kUnitTiles + 4]
  constexpr int W = kUnitMax / 32;
  __shared__ unsigned s_bit[W + 1];  // a tile's first slot
  __shared__ int s_part[kUWaves];
  __shared__ int s_over;
  const RunDesc d = dg.get();
  int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  bool bad = !unit_space(g, d);
  if (!bad)
    for (int i = tid; i < g.units; i += kUWG) bad |= unit_flags(a)[i] != 0;
  bad = __syncthreads_or(bad);
  if (blockIdx.x == 0 && tid == 0) a.counters[C_UNITS] = !bad;
  if (bad) {
    clear_lists(d, g, a, (int64_t)blockIdx.x * kUWG + tid, (int64_t)gridDim.x * kUWG);
    int end;
    for (int h = own_share(d.n, end); h < end; h += kUWG * kSideU)
      hist_chunk<kSideU>(d, g, a, h + tid / kWG * (kWG * kSideU), end, tid % kWG);
    return;
  }
  const int U = d.n_events * g.L;
  const int tw = (g.tpl + 3) >> 2;  // words of four tiles
  const int32_t* const us = unit_starts(a, d, g);
  for (int u = blockIdx.x; u < U; u += gridDim.x) {
    // in scalar registers, so that the accesses below take a scalar base
    const int s0 = __builtin_amdgcn_readfirstlane(us[u]), m = __builtin_amdgcn_readfirstlane(us[u + 1]) - s0;
    const int q = (m + kUWaves - 1) / kUWaves, i0 = wave * q, i1 = min(i0 + q, m);
    unsigned pk[kUPer];  // tile | rank << 12
    const float* const ux = d.x + s0;
    const float* const uy = d.y + s0;
    auto count = [&](bool bytes) {
      constexpr int V = (kUPer + 1) / 2;  // hits whose loads are in flight together
#pragma unroll
      for (int k0 = 0; k0 < kUPer; k0 += V) {
        float x[V], y[V];
#pragma unroll
        for (int k = 0; k < V; ++k)
          if ((k0 + k) * 64 < q) {  // uniform
            const unsigned i = max(min(i0 + (k0 + k) * 64 + lane, m - 1), 0);
            x[k] = ux[i];
            y[k] = uy[i];
          }
#pragma unroll
        for (int k = 0; k < V; ++k)
          if (k0 + k < kUPer && (k0 + k) * 64 < q) {
            const int t = tile_coord(y[k], g.y0, g.inv_t, g.ny) * g.nx + tile_coord(x[k], g.x0, g.inv_t, g.nx);
            if (i0 + (k0 + k) * 64 + lane < i1) {
              unsigned r;
              if (bytes) {
                const int sh = 8 * (t & 3);
                r = (atomicAdd(&cnt4[wave * tw + (t >> 2)], 1u << sh) >> sh) & 255u;
                if (r == 255u) s_over = 1;  // the byte wraps
              } else {
                r = atomicAdd(&cnt4[t], 1u);
              }
              pk[k0 + k] = (unsigned)t | (r << 12);
            }
          }
      }
    };
    for (int i = tid; i < kUWaves * tw; i += kUWG) cnt4[i] = 0u;
    for (int i = tid; i <= W; i += kUWG) s_bit[i] = 0u;
    if (tid == 0) s_over = 0;
    __syncthreads();
    count(true);
    __syncthreads();
    // four tiles per lane: prefix over the waves (kept in the bytes), then over the tiles
    unsigned lo = 0u, hi = 0u;  // tiles 0 and 2, 1 and 3, 16 bits each
    if (tid < tw) {
#pragma unroll
      for (int w = 0; w < kUWaves; ++w) {
        const unsigned c = cnt4[w * tw + tid];
        cnt4[w * tw + tid] = (lo & 0x00ff00ffu) | ((hi & 0x00ff00ffu) << 8);
        if ((lo | hi) & 0xff00ff00u) s_over = 1;
        lo += c & 0x00ff00ffu;
        hi += (c >> 8) & 0x00ff00ffu;
      }
    }
    __syncthreads();
    const bool over = s_over;  // uniform
    if (over) {
      __syncthreads();
      for (int i = tid; i < 4 * tw; i += kUWG) cnt4[i] = 0u;
      __syncthreads();
      count(false);
      __syncthreads();
      lo = hi = 0u;
      if (tid < tw) {
        lo = cnt4[4 * tid] | (cnt4[4 * tid + 2] << 16);
        hi = cnt4[4 * tid + 1] | (cnt4[4 * tid + 3] << 16);
      }
    }
    {
      const int c0 = lo & 0xffffu, c1 = hi & 0xffffu, c2 = lo >> 16, c3 = hi >> 16;
      int total;
      const int b0 = wg_excl<kUWG>(c0 + c1 + c2 + c3, s_part, total, fresh(tid));
      const int b1 = b0 + c0, b2 = b1 + c1, b3 = b2 + c2;
      if (tid < tw) {
        start[4 * tid] = (unsigned short)b0;
        start[4 * tid + 1] = (unsigned short)b1;
        start[4 * tid + 2] = (unsigned short)b2;
        start[4 * tid + 3] = (unsigned short)b3;
        atomicOr(&s_bit[b0 >> 5], c0 ? 1u << (b0 & 31) : 0u);
        atomicOr(&s_bit[b1 >> 5], c1 ? 1u << (b1 & 31) : 0u);
        atomicOr(&s_bit[b2 >> 5], c2 ? 1u << (b2 & 31) : 0u);
        atomicOr(&s_bit[b3 >> 5], c3 ? 1u << (b3 & 31) : 0u);
      }
    }
    __syncthreads();
    int32_t* const ts = a.tile_start + (int64_t)u * g.tpl;
    for (int t = tid; t < g.tpl; t += kUWG) ts[t] = s0 + start[t];
    if (u == U - 1 && tid == 0) ts[g.tpl] = d.n;
    tid = fresh(tid);
#pragma unroll
    for (int k = 0; k < kUPer; ++k) {
      const int i = i0 + k * 64 + lane;
      if (k * 64 < q && i < i1) {
        const int t = pk[k] & 4095u;
        int p = start[t] + (int)(pk[k] >> 12);
        if (!over) p += (cnt4[wave * tw + (t >> 2)] >> (8 * (t & 3))) & 255u;
        srt[p] = (unsigned short)i;
      }
    }
    __syncthreads();
    bool wrong = over;
    for (int p = tid + 1; p < m; p += kUWG)
      wrong |= srt[p - 1] > srt[p] && !((s_bit[p >> 5] >> (p & 31)) & 1u);
    if (__syncthreads_or(wrong)) {
      for (int p = tid; p < m; p += kUWG) {
        // the tile's slots [b, e), by the bits around p
        int w = p >> 5;
        unsigned v = s_bit[w] & (0xffffffffu >> (31 - (p & 31)));
        while (!v) v = s_bit[--w];  // slot 0 is a tile's first
        const int b = 32 * w + 31 - __clz((int)v);
        w = (p + 1) >> 5;
        v = s_bit[w] & (0xffffffffu << ((p + 1) & 31));
        while (!v && w < W) v = s_bit[++w];
        const int e = v ? min(32 * w + __ffs((int)v) - 1, m) : m;
        const int i = srt[p];
        int r = b;
        for (int c = b; c < e; ++c) r += srt[c] < i;
        alt[r] = (unsigned short)i;
      }
      __syncthreads();
      for (int p = tid; p < m; p += kUWG) srt[p] = alt[p];
      __syncthreads();
    }
    // the columns
    const float* const in[3] = {ux, uy, d.e + s0};
    float* const out[3] = {a.xs + s0, a.ys + s0, a.es + s0};
    int32_t* const oh = a.hs + s0;
    float v[kUPer];
    tid = fresh(tid);
#pragma unroll
    for (int k = 0; k < kUPer; ++k)
      if (k * kUWG < m) v[k] = in[0][(unsigned)min(k * kUWG + tid, m - 1)];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      tid = fresh(tid);
#pragma unroll
      for (int k = 0; k < kUPer; ++k)
        if (k * kUWG + tid < m) col[k * kUWG + tid] = v[k];
      if (c < 2) {
        tid = fresh(tid);
#pragma unroll
        for (int k = 0; k < kUPer; ++k)
          if (k * kUWG < m) v[k] = in[c < 2 ? c + 1 : 0][(unsigned)min(k * kUWG + tid, m - 1)];
      }
      __syncthreads();
      tid = fresh(tid);
#pragma unroll
      for (int k = 0; k < kUPer; ++k) {
        const unsigned p = k * kUWG + tid;
        if ((int)p < m) {
          const int i = srt[p];
          out[c][p] = col[i];
          if (c == 0) oh[p] = s0 + i;
        }
      }
      __syncthreads();  // the next column, or unit, overwrites it
    }
  }
}

// ---------------------------------------------------------------------------
// Labels, seed flags and follower lists of each unit. Seeds and followers of
// earlier units come from the counts of the nearest-higher stage; within the
// unit, links are followed in LDS (halving the path, which only ever moves a
// link to an ancestor, several hits' paths at a time), seeds are ranked by a
// bitmap in hit order, and follower lists are laid out by a scan of per-owner
// counts, each entry placed by counting the smaller entries of its list.
// ---------------------------------------------------------------------------
template <bool G>
__global__ __launch_bounds__(kUWG, 8) void k_unit_finish(DescArg<G> dg, Geom g, Arena a) {
  extern __shared__ __align__(16) unsigned char lds[];
  unsigned short* const par = reinterpret_cast<unsigned short*>(lds);  // links by slot, then list entries [kUnitMax]
  unsigned short* const idx = par + kUnitMax;                          // slot -> unit-local hit [kUnitMax]
  unsigned* const cnt2 = reinterpret_cast<unsigned*>(idx + kUnitMax);  // follower counts, two a word
  unsigned short* const off = reinterpret_cast<unsigned short*>(cnt2); // labels, then list offsets [kUnitMax + 2]
  constexpr int W = kUnitMax / 32;
  constexpr int V = 4;  // paths followed at a time
  __shared__ unsigned s_seed[W];
  __shared__ int s_rank[W];
  __shared__ int s_part[kUWaves];
  const RunDesc d = dg.get();
  int tid = threadIdx.x;
  if (!by_units(g, a)) {
    LabelChunk<kUWG * kSideU>& C = *reinterpret_cast<LabelChunk<kUWG * kSideU>*>(lds);
    int end;
    for (int s = own_share(d.n, end); s < end; s += kUWG * kSideU) label_chunk<kUWG, kSideU>(d, g, a, s, end, C);
    return;
  }
  const bool lists = !(g.flags & 8u);
  const int U = d.n_events * g.L;
  const int32_t* const us = unit_starts(a, d, g);
  const int32_t* const uc = unit_counts(a, d, g);
  int prev = 0, sb = 0, fb = 0;  // seeds of the event and followers of the run before unit prev
  for (int u = blockIdx.x; u < U; u += gridDim.x) {
    // in scalar registers, so that the accesses below take a scalar base
    const int s0 = __builtin_amdgcn_readfirstlane(us[u]), m = __builtin_amdgcn_readfirstlane(us[u + 1]) - s0;
    const int u0 = u - u % g.L;  // the event's first unit
    const int first = __builtin_amdgcn_readfirstlane(us[u0]);
    const int32_t* const uhs = a.hs + s0;
    const int32_t* const upar = a.parent + s0;
    const uint8_t* const uflags = a.flags + s0;
    unsigned lk[kUPer];  // the hit's link, a unit-local slot; then its owner | its arrival in the owner's list << 16
    unsigned fl = 0u;    // bit k: hit k is a follower
    tid = fresh(tid);
#pragma unroll
    for (int k = 0; k < kUPer; ++k)
      if (k * kUWG < m) lk[k] = upar[(unsigned)min(k * kUWG + tid, m - 1)] - s0;
    // the counts since this workgroup's previous unit, so that a run's units cost it
    // one pass over their counts (added up from the first for each of 100,000 units,
    // they took 3.2 ms)
    int ds = 0, df = 0;
    for (int v = prev + tid; v < u; v += kUWG) {
      if (v >= u0) ds += uc[2 * v];
      df += uc[2 * v + 1];
    }
    for (int i = tid; i < W; i += kUWG) s_seed[i] = 0u;
    wg_excl<kUWG>(ds, s_part, ds, threadIdx.x);
    wg_excl<kUWG>(df, s_part, df, threadIdx.x);
    sb = (prev < u0 ? 0 : sb) + __builtin_amdgcn_readfirstlane(ds);
    fb += __builtin_amdgcn_readfirstlane(df);
    prev = u;
    tid = fresh(tid);
#pragma unroll
    for (int k0 = 0; k0 < kUPer; k0 += V) {
      int i[V];
      unsigned f[V];
#pragma unroll
      for (int k = 0; k < V; ++k)
        if ((k0 + k) * kUWG < m) {
          const unsigned s = min((k0 + k) * kUWG + tid, m - 1);
          i[k] = uhs[s] - s0;
          f[k] = uflags[s];
        }
#pragma unroll
      for (int k = 0; k < V; ++k) {
        const int s = (k0 + k) * kUWG + tid;
        if (k0 + k < kUPer && s < m) {
          par[s] = (unsigned short)lk[k0 + k];
          idx[s] = (unsigned short)i[k];
          if (f[k] & F_FOLLOWER) fl |= 1u << (k0 + k);
          if (f[k] & F_SEED) atomicOr(&s_seed[i[k] >> 5], 1u << (i[k] & 31));
        }
      }
    }
    __syncthreads();
    {
      const int c = tid < W ? __popc(s_seed[tid]) : 0;
      int total;
      const int r = wg_excl<kUWG>(c, s_part, total, threadIdx.x);
      if (tid < W) s_rank[tid] = r;
    }
    __syncthreads();
    tid = fresh(tid);
#pragma unroll 1
    for (int k0 = 0; k0 * kUWG < m; k0 += V) {
      int r[V];
#pragma unroll
      for (int k = 0; k < V; ++k) r[k] = min((k0 + k) * kUWG + tid, m - 1);
      for (;;) {
        int p[V], q[V];
        bool more = false;
#pragma unroll
        for (int k = 0; k < V; ++k) p[k] = par[r[k]];
#pragma unroll
        for (int k = 0; k < V; ++k) q[k] = par[p[k]];
#pragma unroll
        for (int k = 0; k < V; ++k) {
          if (q[k] != p[k]) {
            par[r[k]] = (unsigned short)q[k];
            more = true;
          }
          r[k] = q[k];
        }
        if (!more) break;
      }
#pragma unroll
      for (int k = 0; k < V; ++k) {
        const int s = (k0 + k) * kUWG + tid;
        const unsigned ri = idx[r[k]], w = s_seed[ri >> 5];
        if (s < m)  // the root's seed number in the unit, by hit
          off[idx[s]] = (w >> (ri & 31)) & 1u
                            ? (unsigned short)(s_rank[ri >> 5] + __popc(w & ((1u << (ri & 31)) - 1u)))
                            : (unsigned short)0xffffu;
      }
    }
    __syncthreads();
    int32_t* const ucid = d.cluster_id + s0;
    uint8_t* const useed = d.is_seed + s0;
    for (int i = tid; i < m; i += kUWG) {
      ucid[(unsigned)i] = off[i] == 0xffffu ? -1 : sb + (int)off[i];
      useed[(unsigned)i] = (uint8_t)((s_seed[i >> 5] >> (i & 31)) & 1u);
    }
    if (lists) {
      __syncthreads();
      for (int i = tid; i <= m / 2; i += kUWG) cnt2[i] = 0u;
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kUPer; ++k)
        if (fl & (1u << k)) {
          const unsigned o = idx[lk[k]];
          const int sh = 16 * (o & 1u);
          lk[k] = o | (((atomicAdd(&cnt2[o >> 1], 1u << sh) >> sh) & 0xffffu) << 16);
        }
      __syncthreads();
      const int per = (m + kUWG) / kUWG;  // m + 1 offsets
      const int i0 = min(tid * per, m + 1), i1 = min(i0 + per, m + 1);
      int sum = 0, total;
      for (int i = i0; i < i1; ++i) sum += i < m ? off[i] : 0;
      int run = wg_excl<kUWG>(sum, s_part, total, threadIdx.x);
      for (int i = i0; i < i1; ++i) {
        const int c = i < m ? off[i] : 0;
        off[i] = (unsigned short)run;
        run += c;
      }
      __syncthreads();
      int32_t* const ufs = a.fstart + s0;
      int32_t* const ufl = a.flist + fb;
      for (int i = tid; i < m; i += kUWG) ufs[(unsigned)i] = fb + off[i];
      if (u == U - 1 && tid == 0) ufs[m] = fb + total;
      tid = fresh(tid);
#pragma unroll
      for (int k = 0; k < kUPer; ++k)
        if (fl & (1u << k)) par[off[lk[k] & 0xffffu] + (lk[k] >> 16)] = idx[k * kUWG + tid];
      __syncthreads();
      tid = fresh(tid);
#pragma unroll
      for (int k = 0; k < kUPer; ++k)
        if (fl & (1u << k)) {
          const int o = lk[k] & 0xffffu, i = idx[k * kUWG + tid];
          const int b = off[o], e = off[o + 1];
          int r = b;
          for (int c = b; c < e; ++c) r += par[c] < i;
          ufl[(unsigned)r] = s0 + i - first;
        }
    }
    __syncthreads();  // the next unit overwrites the lists
  }
}

constexpr int kSortLds = 6 * kUnitMax + 2 * (kUnitTiles + 4);
static_assert(kUWaves * kUnitTiles <= 4 * kUnitMax, "the wave counts fit the column");
constexpr int kFinishLds = 4 * kUnitMax + 2 * (kUnitMax + 2);

static_assert(sizeof(LabelChunk<kUWG * kSideU>) <= kFinishLds, "the general path's labels fit");

// Two workgroups per CU hold a unit each. A single event has a hundred units or
// so, and as a general run one or two shares per CU.
static int unit_grid(bool graph, const Geom& g, const RunDesc& d) {
  const int64_t units = (int64_t)d.n_events * g.L, chunks = ((int64_t)d.n + kUWG * kSideU - 1) / (kUWG * kSideU);
  int64_t wgs = chunks > 256 || graph ? 512 : std::min<int64_t>(chunks, 256);
  wgs = std::min<int64_t>(std::max(wgs, units), 512);
  return (int)((wgs + kQueues - 1) / kQueues * kQueues);
}

template <bool G>
void launch_units(const Geom& g, const Arena& a, DescArg<G> dg, const RunDesc&, hipStream_t s) {
  k_units<G><<<g.units, kWG, 0, s>>>(dg, g, a);
}
template <bool G>
void launch_unit_sort(const Geom& g, const Arena& a, DescArg<G> dg, const RunDesc& d, hipStream_t s) {
  k_unit_sort<G><<<unit_grid(G, g, d), kUWG, kSortLds, s>>>(dg, g, a);
}
template <bool G>
void launch_unit_finish(const Geom& g, const Arena& a, DescArg<G> dg, const RunDesc& d, hipStream_t s) {
  k_unit_finish<G><<<unit_grid(G, g, d), kUWG, kFinishLds, s>>>(dg, g, a);
}
template void launch_units<false>(const Geom&, const Arena&, DescArg<false>, const RunDesc&, hipStream_t);
template void launch_units<true>(const Geom&, const Arena&, DescArg<true>, const RunDesc&, hipStream_t);
template void launch_unit_sort<false>(const Geom&, const Arena&, DescArg<false>, const RunDesc&, hipStream_t);
template void launch_unit_sort<true>(const Geom&, const Arena&, DescArg<true>, const RunDesc&, hipStream_t);
template void launch_unit_finish<false>(const Geom&, const Arena&, DescArg<false>, const RunDesc&, hipStream_t);
template void launch_unit_finish<true>(const Geom&, const Arena&, DescArg<true>, const RunDesc&, hipStream_t);

}  // namespace clue
