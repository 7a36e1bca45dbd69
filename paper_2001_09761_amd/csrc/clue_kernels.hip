// HIP kernels of libclue for gfx950 (MI355X).
//
// Stage map (arXiv:2001.09761):
//   k_clear            clears counters, tile counts and scan status
//   (k_units, k_unit_sort and k_unit_finish, in clue_units.hip, take the place of
//   the other grid-build and label kernels when the hits come grouped by layer;
//   runs of few hits take the kernels of clue_direct.hip instead of all of these)
//   k_hist             fixed grid, part 1: atomic per-tile histogram (Sec. 2.1)
//   k_scan<TILES>      exclusive prefix scan of the tile counts (decoupled look-back)
//   k_scatter          fixed grid, part 2: hit ids into the tile CSR (arrival order)
//   k_place            fixed grid, part 3: each tile's records in ascending hit index
//   k_density          rho (Eq. 3, Algorithm 1) over LDS-staged tile windows,
//                      summed in ascending hit index along merged 2x2-tile
//                      lists of the index-ordered tiles
//   k_density_spill    rho of the queries in tiles too dense for LDS, queued by
//                      k_density and spread over the whole GPU
//   k_nearest_higher   nh / delta (Eq. 4, Algorithm 2) fused with the seed /
//                      outlier / follower decision (Sec. 2.2, Algorithm 3)
//   k_nh_spill         the same for the queries that k_nearest_higher queued
//   k_scan<SEEDS>      seed numbering by prefix scan over the seed bitmap (and
//                      follower list offsets); writes the caller-order seed flags
//   k_label            cluster ids: each hit follows nearest-higher links of
//                      followers to its root (pointer jumping with path
//                      compression); registers follower-list entries
//   k_expand_init      the k-way alternative to k_label (Algorithm 3): follower
//   k_expand_dfs       lists, seed list, then one depth-first walk per seed
//   k_follow_sort      sorts each follower list by hit index, event-local ids
//   k_event_ids        a host-resident chunk's event ids from its events' first hits
//   k_read_out         copies intermediates or follower lists to the caller
//
// Every float operation that decides a result is an explicit round-to-nearest
// intrinsic (no contraction), so results match a plain IEEE binary32
// evaluation of the same expressions.
#include "clue_device.h"

#include <algorithm>
#include <climits>

namespace clue {

const char* const kStageNames[S_COUNT] = {"clear",        "grid_hist",  "grid_scan",
                                          "grid_scatter", "grid_place", "density",
                                          "nearest_higher", "seed_scan", "labels",
                                          "follower_lists"};

// ---------------------------------------------------------------------------
// Geometry helpers.
// ---------------------------------------------------------------------------

// Half width of a query window: the radius inflated by 2^-10 relative plus
// 2^-20 |v|, so that rounding of v +- w can never exclude a hit whose float32
// squared distance passes the strict threshold.
__device__ __forceinline__ float window_half(float w, float v) {
  return __fadd_rn(w, __fmul_rn(fabsf(v), 0x1p-20f));
}

// ---------------------------------------------------------------------------
// k_clear
// ---------------------------------------------------------------------------
template <bool G>
__global__ __launch_bounds__(kWG) void k_clear(DescArg<G> dg, Geom g, Arena a) {
  const int64_t i0 = (int64_t)blockIdx.x * kWG + threadIdx.x, stride = (int64_t)gridDim.x * kWG;
  for (int64_t i = i0; i < C_COUNT; i += stride) a.counters[i] = 0;
  const RunDesc d = dg.get();
  clear_grid(d, g, a, i0, stride);
  clear_lists(d, g, a, i0, stride);
}

template <bool G>
__global__ __launch_bounds__(kWG) void k_hist(DescArg<G> dg, Geom g, Arena a) {
  const RunDesc d = dg.get();
  for (ChunkRun r = xcd_run(d.n, kHistChunk); r.c < r.end; r.c += r.step) hist_chunk<kPlaceU>(d, g, a, r.c * kHistChunk, d.n, (int)threadIdx.x);
}

// ---------------------------------------------------------------------------
// k_scatter: hit h's id and tile go to slot tile_start[tile] + rank (arrival
// order within a tile) as one eight-byte pair, so that hits in no order touch one
// line each, not two. The pairs lie in the rho and parent buffers, which are free
// until the density stage and adjoin.
// k_place: slot by slot, each hit counts the ids of its tile that are smaller
// than its own and writes its record at that position, so every tile of the
// CSR lists its hits in ascending hit index. Neighbouring slots share their
// tile, so the counting loads are broadcasts from lines just read.
// ---------------------------------------------------------------------------
template <bool G>
__device__ __forceinline__ void scatter_chunk(const RunDesc& d, const Geom& g, const Arena& a, int chunk) {
  int2* const pairs = reinterpret_cast<int2*>(a.rho);
  constexpr int U = G ? kBatchU : kPlaceU;
  const int h0 = chunk * kWG * U + (int)threadIdx.x;
  int t[U], r[U];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int h = h0 + j * kWG;
    t[j] = -1;
    if (h < d.n) {
      t[j] = a.key[h];
      r[j] = a.rank[h];
    }
  }
#pragma unroll
  for (int j = 0; j < U; ++j) {
    if (t[j] >= 0) {
      const int s = a.tile_start[t[j]] + r[j];
      pairs[s] = make_int2(h0 + j * kWG, t[j]);
    }
  }
}

template <bool G>
__global__ __launch_bounds__(kWG) void k_scatter(DescArg<G> dg, Geom g, Arena a) {
  if (by_units(g, a)) return;  // done unit by unit
  const RunDesc d = dg.get();
  for (ChunkRun r = xcd_run(d.n, stream_chunk(G)); r.c < r.end; r.c += r.step) scatter_chunk<G>(d, g, a, r.c);
}

template <bool G>
__device__ __forceinline__ void place_chunk(const RunDesc& d, const Geom& g, const Arena& a, int chunk) {
  const int2* const pairs = reinterpret_cast<const int2*>(a.rho);
  constexpr int U = G ? kBatchU : kPlaceU;
  constexpr int C = kWG * U;  // slots per chunk
  // the chunk's arrival-order ids in LDS: a hit's tile mostly lies inside
  // the chunk, so most of its counting reads are LDS reads
  __shared__ int s_ids[C];
  const int c0 = chunk * C;
  const int c1 = min(c0 + C, d.n);
  int tile[U];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int sl = c0 + (int)threadIdx.x + j * kWG;
    const int2 p = pairs[min(sl, d.n - 1)];
    s_ids[sl - c0] = p.x;
    tile[j] = p.y;
  }
  __syncthreads();
  // slots in groups of four: a group's loads are all issued before its
  // first store (which could alias them as far as the compiler knows)
  constexpr int V = 4;
#pragma unroll
  for (int j0 = 0; j0 < U; j0 += V) {
    int hv[V], s0v[V], s1v[V];
    float xv[V], yv[V], ev[V];
#pragma unroll
    for (int k = 0; k < V; ++k) {
      const int sl = c0 + (int)threadIdx.x + (j0 + k) * kWG;
      hv[k] = -1;
      if (sl < d.n) {
        const int h = s_ids[sl - c0];
        const int t = tile[j0 + k];
        hv[k] = h;
        xv[k] = d.x[h];
        yv[k] = d.y[h];
        ev[k] = d.e[h];
        s0v[k] = a.tile_start[t];
        s1v[k] = a.tile_start[t + 1];
      }
    }
#pragma unroll
    for (int k = 0; k < V; ++k) {
      if (hv[k] < 0) continue;
      const int h = hv[k], s0 = s0v[k], s1 = s1v[k];
      // the tile [s0, s1) in three parts: before the chunk, in it, after it
      const int m0 = min(max(s0, c0), s1), m1 = max(min(s1, c1), m0);
      int rk = 0;
      for (int c = s0; c < m0; ++c) rk += pairs[c].x < h;
      int c = m0;
      for (; c + 3 < m1; c += 4)
        rk += (s_ids[c - c0] < h) + (s_ids[c + 1 - c0] < h) + (s_ids[c + 2 - c0] < h) + (s_ids[c + 3 - c0] < h);
      for (; c < m1; ++c) rk += s_ids[c - c0] < h;
      for (c = m1; c < s1; ++c) rk += pairs[c].x < h;
      const int slot = s0 + rk;
      a.xs[slot] = xv[k];
      a.ys[slot] = yv[k];
      a.es[slot] = ev[k];
      a.hs[slot] = h;
    }
  }
  __syncthreads();  // the next chunk overwrites the staged ids
}

template <bool G>
__global__ __launch_bounds__(kWG) void k_place(DescArg<G> dg, Geom g, Arena a) {
  if (by_units(g, a)) return;  // done unit by unit
  const RunDesc d = dg.get();
  for (ChunkRun r = xcd_run(d.n, stream_chunk(G)); r.c < r.end; r.c += r.step) place_chunk<G>(d, g, a, r.c);
}

// ---------------------------------------------------------------------------
// Decoupled look-back exclusive scan, one or two channels.
// Status word: [63:62] flag (1 aggregate, 2 inclusive prefix), [61:31]
// channel 1, [30:0] channel 0. Every value is a count below 2^31.
// Chunk ids come from an atomic ticket, so every chunk a workgroup waits on
// was taken by a running workgroup that publishes without waiting: each wait
// ends.
// ---------------------------------------------------------------------------
enum ScanKind { SCAN_TILES = 0, SCAN_SEEDS = 1, SCAN_SEEDS_FOLLOW = 2 };

__device__ __forceinline__ unsigned long long st_pack(int flag, int v0, int v1) {
  return ((unsigned long long)flag << 62) | ((unsigned long long)(unsigned)(v1 & 0x7fffffff) << 31) |
         (unsigned long long)(unsigned)(v0 & 0x7fffffff);
}
__device__ __forceinline__ int st_flag(unsigned long long w) { return (int)(w >> 62); }
__device__ __forceinline__ int st_v0(unsigned long long w) { return (int)(w & 0x7fffffffull); }
__device__ __forceinline__ int st_v1(unsigned long long w) { return (int)((w >> 31) & 0x7fffffffull); }

template <bool G, int KIND>
__device__ __forceinline__ void scan_chunk(const RunDesc& d, const Geom& g, const Arena& a, int64_t chunk) {
  constexpr int NCH = KIND == SCAN_SEEDS_FOLLOW ? 2 : 1;
  constexpr int SI = scan_items(G), SC = kWG * SI;
  const int64_t nel = KIND == SCAN_TILES ? (int64_t)d.n_events * g.L * g.tpl : (int64_t)d.n;
  const int64_t nout = nel + 1;  // the last output is the total
  unsigned long long* status = a.scan_status + (KIND == SCAN_TILES ? 0 : a.cap_chunks);
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  __shared__ int s_wsum[NCH][kWG / 64];
  __shared__ int s_prefix[NCH];
  const int64_t base = chunk * SC + (int64_t)threadIdx.x * SI;

  int v[NCH][SI];
  if constexpr (KIND == SCAN_TILES) {
    if (base + SI <= nel) {
      const int4* p = reinterpret_cast<const int4*>(a.tile_start + base);
#pragma unroll
      for (int q = 0; q < SI / 4; ++q) {
        int4 w = p[q];
        v[0][4 * q] = w.x; v[0][4 * q + 1] = w.y; v[0][4 * q + 2] = w.z; v[0][4 * q + 3] = w.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < SI; ++i) v[0][i] = base + i < nel ? a.tile_start[base + i] : 0;
    }
  } else {
    // channel 0: the seeds of bitmap word w at element 32 w, zero elsewhere,
    // so that the prefix at 32 w counts the seeds before word w
    static_assert(SI % 32 == 0 || 32 % SI == 0, "a thread's elements hold whole words or none");
    const int64_t nw = seed_words(d.n);
    // the bitmap words of this thread's elements, loaded once
    constexpr int NW = (SI + 31) / 32;
    unsigned wv[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) wv[k] = (base >> 5) + k < nw ? a.seedbits[(base >> 5) + k] : 0u;
#pragma unroll
    for (int i = 0; i < SI; ++i) {
      const int64_t e = base + i;
      v[0][i] = (e & 31) == 0 ? __popc(wv[(e >> 5) - (base >> 5)]) : 0;
    }
    // the follower counts are loaded before the flag stores below, which
    // could alias them as far as the compiler knows
    if constexpr (NCH == 2) {
      if (base + SI <= nel) {
        const int4* p = reinterpret_cast<const int4*>(a.fstart + base);
#pragma unroll
        for (int q = 0; q < SI / 4; ++q) {
          int4 w = p[q];
          v[1][4 * q] = w.x; v[1][4 * q + 1] = w.y; v[1][4 * q + 2] = w.z; v[1][4 * q + 3] = w.w;
        }
      } else {
#pragma unroll
        for (int i = 0; i < SI; ++i) v[1][i] = base + i < nel ? a.fstart[base + i] : 0;
      }
    }
    // the caller-order seed flags, expanded from the bitmap 16 at a time
    // (one bit per hit -> one byte per hit), in coalesced stores
    static_assert(SI % 16 == 0, "flags are written 16 at a time");
#pragma unroll
    for (int q = 0; q < SI; q += 16) {
      const int64_t e0 = base + q;
      if (e0 >= nel) break;
      const unsigned w = (wv[(e0 >> 5) - (base >> 5)] >> (e0 & 31)) & 0xffffu;
      unsigned b4[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) b4[k] = (((w >> (4 * k)) & 0xfu) * 0x00204081u) & 0x01010101u;
      uint8_t* dst = d.is_seed + e0;
      if (e0 + 16 <= nel && ((uintptr_t)dst & 15u) == 0) {
        *reinterpret_cast<uint4*>(dst) = make_uint4(b4[0], b4[1], b4[2], b4[3]);
      } else {
        for (int k = 0; k < 16 && e0 + k < nel; ++k) dst[k] = (uint8_t)((w >> k) & 1u);
      }
    }
  }
  // thread-local exclusive prefix
  int tsum[NCH];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    int acc = 0;
#pragma unroll
    for (int i = 0; i < SI; ++i) {
      int t = v[c][i];
      v[c][i] = acc;
      acc += t;
    }
    tsum[c] = acc;
  }
  int texcl[NCH];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    int incl = wave_incl_scan(tsum[c], lane);
    texcl[c] = incl - tsum[c];
    if (lane == 63) s_wsum[c][wave] = incl;
  }
  __syncthreads();
  int agg[NCH];
  int wbase[NCH];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    int acc = 0;
    wbase[c] = 0;
#pragma unroll
    for (int w = 0; w < kWG / 64; ++w) {
      if (w == wave) wbase[c] = acc;
      acc += s_wsum[c][w];
    }
    agg[c] = acc;
  }
  // look-back by wave 0
  if (wave == 0) {
    int run[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) run[c] = 0;
    if (chunk == 0) {
      if (lane == 0)
        __hip_atomic_store(&status[0], st_pack(2, agg[0], NCH == 2 ? agg[NCH - 1] : 0), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    } else {
      if (lane == 0)
        __hip_atomic_store(&status[chunk], st_pack(1, agg[0], NCH == 2 ? agg[NCH - 1] : 0), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      int64_t look = chunk - 1;
      for (;;) {
        const int64_t j = look - lane;
        unsigned long long w = j >= 0 ? __hip_atomic_load(&status[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                      : st_pack(2, 0, 0);
        while (__any(st_flag(w) == 0)) {
          if (st_flag(w) == 0)
            w = __hip_atomic_load(&status[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        const unsigned long long incl_mask = __ballot(st_flag(w) == 2);
        const int stop = incl_mask ? __ffsll((long long)incl_mask) - 1 : 64;
        const bool take = lane <= stop;
        run[0] += wave_sum(take ? st_v0(w) : 0);
        if constexpr (NCH == 2) run[1] += wave_sum(take ? st_v1(w) : 0);
        if (incl_mask) break;
        look -= 64;
      }
      if (lane == 0)
        __hip_atomic_store(&status[chunk],
                           st_pack(2, run[0] + agg[0], NCH == 2 ? run[NCH - 1] + agg[NCH - 1] : 0),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (lane == 0) {
#pragma unroll
      for (int c = 0; c < NCH; ++c) s_prefix[c] = run[c];
    }
  }
  __syncthreads();
  // outputs
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int off = s_prefix[c] + wbase[c] + texcl[c];
    if (KIND != SCAN_TILES && c == 0) {  // one count per bitmap word
#pragma unroll
      for (int i = 0; i < SI; i += 32)
        if (base + i < nout && ((base + i) & 31) == 0) a.seed_wrank[(base + i) >> 5] = off + v[c][i];
      continue;
    }
    int* out = KIND == SCAN_TILES ? a.tile_start : a.fstart;
    if (base + SI <= nout) {
      int4* p = reinterpret_cast<int4*>(out + base);
#pragma unroll
      for (int q = 0; q < SI / 4; ++q)
        p[q] = make_int4(off + v[c][4 * q], off + v[c][4 * q + 1], off + v[c][4 * q + 2], off + v[c][4 * q + 3]);
    } else {
#pragma unroll
      for (int i = 0; i < SI; ++i)
        if (base + i < nout) out[base + i] = off + v[c][i];
    }
  }
  __syncthreads();
}

template <bool G, int KIND>
__host__ __device__ __forceinline__ int scan_chunks(const RunDesc& d, const Geom& g) {
  constexpr int SC = kWG * scan_items(G);
  const int64_t nel = KIND == SCAN_TILES ? (int64_t)d.n_events * g.L * g.tpl : (int64_t)d.n;
  return (int)((nel + SC) / SC);  // nel + 1 outputs
}

template <bool G, int KIND>
__global__ __launch_bounds__(kWG) void k_scan(DescArg<G> dg, Geom g, Arena a) {
  if (by_units(g, a)) return;  // done unit by unit
  const RunDesc d = dg.get();
  const int nchunks = scan_chunks<G, KIND>(d, g);
  int* ticket = &a.counters[KIND == SCAN_TILES ? C_TICKET_TILES : C_TICKET_SEEDS];
  __shared__ int s_chunk;
  for (;;) {
    if (threadIdx.x == 0) s_chunk = atomicAdd(ticket, 1);
    __syncthreads();
    const int chunk = s_chunk;
    __syncthreads();
    if (chunk >= nchunks) break;
    scan_chunk<G, KIND>(d, g, a, chunk);
  }
}

// ---------------------------------------------------------------------------
// Tile-block work items. An item is one (event, layer) unit and a block of
// bx*by tiles (the core); its staged region adds `halo` tiles around the core
// (clamped to the grid). A block whose region does not fit in LDS is halved
// along its longer side, and so on down to single tiles (BlockWalk); a tile
// whose own region does not fit is queued for the stage's spill kernel, which
// searches global memory.
// ---------------------------------------------------------------------------
struct Region {
  int unit;       // event * L + layer
  int e;          // event
  int rx0, ry0;   // region origin (tile coordinates)
  int rw, rh;     // region size in tiles
  int cx0, cy0;   // core origin relative to the region
  int cw, ch;     // core size in tiles
  int total;      // hits in the region
};

// Region metadata in LDS (pointers into the workgroup's shared memory; ts and
// qoff live in the dynamic part, sized for the configured block and halo):
//   ts[r*(rw+1) + c]  LDS offset of region tile (r, c); c = rw is the row end,
//                     and ts[rh*(rw+1)] repeats the last row's end
//   row_gs[r]         global slot of the first hit of region row r
//   row_lo[r]         LDS offset of region row r (row_lo[rh] = total)
//   core_lo[r]        prefix of core-hit counts over core rows
//   qoff[q]           density: offsets of the merged 2x2-tile lists
struct RegionLds {
  int* ts;
  int* row_gs;
  int* row_lo;
  int* core_lo;
  int* qoff;
  int* qtotal;
};
constexpr int kRowMetaInts = kMaxRegionRows + 2 * (kMaxRegionRows + 1) + 1;

__device__ __forceinline__ RegionLds region_lds(int* row_meta, int* ts, int* qoff) {
  RegionLds L;
  L.ts = ts;
  L.row_gs = row_meta;
  L.row_lo = row_meta + kMaxRegionRows;
  L.core_lo = row_meta + 2 * kMaxRegionRows + 1;
  L.qtotal = row_meta + 3 * kMaxRegionRows + 2;
  L.qoff = qoff;
  return L;
}

__device__ __forceinline__ void item_block(const Geom& g, int item, int& unit, int& tx0, int& ty0, int& tx1,
                                           int& ty1) {
  unit = item / g.bpu;
  const int b = item - unit * g.bpu;
  const int bj = b / g.nbx;
  const int bi = b - bj * g.nbx;
  tx0 = bi * g.bx;
  ty0 = bj * g.by;
  tx1 = min(tx0 + g.bx, g.nx) - 1;
  ty1 = min(ty0 + g.by, g.ny) - 1;
}

__device__ __forceinline__ void make_region(const Geom& g, int unit, int tx0, int ty0, int tx1, int ty1, Region& R) {
  R.unit = unit;
  R.e = unit / g.L;
  R.rx0 = max(tx0 - g.halo, 0);
  R.ry0 = max(ty0 - g.halo, 0);
  const int rx1 = min(tx1 + g.halo, g.nx - 1), ry1 = min(ty1 + g.halo, g.ny - 1);
  R.rw = rx1 - R.rx0 + 1;
  R.rh = ry1 - R.ry0 + 1;
  R.cx0 = tx0 - R.rx0;
  R.cy0 = ty0 - R.ry0;
  R.cw = tx1 - tx0 + 1;
  R.ch = ty1 - ty0 + 1;
}

// Loads the region's tile offsets and builds the LDS layout. Starts and ends
// with a barrier; R.total and the core counts are then valid everywhere.
__device__ __forceinline__ void region_setup(const Geom& g, const Arena& a, Region& R, RegionLds& L) {
  __syncthreads();
  const int64_t ubase = (int64_t)R.unit * g.tpl;
  const int per_row = R.rw + 1;
  const int ntile = R.rh * per_row;
  for (int k = threadIdx.x; k < ntile; k += kWG) {
    const int r = k / per_row, c = k - r * per_row;
    L.ts[k] = a.tile_start[ubase + (int64_t)(R.ry0 + r) * g.nx + R.rx0 + c];
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    const int r = threadIdx.x;
    const int len = r < R.rh ? L.ts[r * per_row + R.rw] - L.ts[r * per_row] : 0;
    const int incl = wave_incl_scan(len, r);
    if (r < R.rh) {
      L.row_gs[r] = L.ts[r * per_row];
      L.row_lo[r] = incl - len;
    }
    if (r == 63) L.row_lo[R.rh] = incl;
    const int cr = (R.cy0 + r) * per_row + R.cx0;
    const int clen = r < R.ch ? L.ts[cr + R.cw] - L.ts[cr] : 0;
    const int cincl = wave_incl_scan(clen, r);
    if (r < R.ch) L.core_lo[r] = cincl - clen;
    if (r == 63) L.core_lo[R.ch] = cincl;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < ntile; k += kWG) {
    const int r = k / per_row;
    L.ts[k] = L.row_lo[r] + (L.ts[k] - L.row_gs[r]);
  }
  // one entry past the last row's end, equal to it: (ntile - 1, ntile) is an
  // empty tile that searches may read in place of a tile they do not need
  if (threadIdx.x == 0) L.ts[ntile] = L.row_lo[R.rh];
  __syncthreads();
  R.total = L.row_lo[R.rh];
}

// Core query q -> (region row, LDS position). `cr` is a core row at or
// before q's, and is left at q's: a lane walking its queries in increasing
// order keeps it between calls.
__device__ __forceinline__ void core_query(const RegionLds& L, const Region& R, int q, int& cr, int& row, int& p) {
  while (cr + 1 < R.ch && L.core_lo[cr + 1] <= q) ++cr;
  row = R.cy0 + cr;
  p = L.ts[row * (R.rw + 1) + R.cx0] + (q - L.core_lo[cr]);
}

__device__ __forceinline__ int slot_of(const RegionLds& L, int row, int p) { return L.row_gs[row] + (p - L.row_lo[row]); }

// The rectangles that a block's core is processed in. Halving stages less halo
// than quartering did: a 10 x 10 block with a one-tile halo that overflows
// stages 2 x 84 tiles instead of 4 x 49 (one event of uneven layers, whose
// densest overflow a 10 x 10 block: density 67 -> 53 us, nearest-higher 76 ->
// 57 us; the paper's workload, 1M hits of 3 cm clusters: 828 -> 614 us a run).
// Rectangles are relative to the block (at most 32 tiles a side), eight bits per
// bound; those still to do wait on an LDS stack (each halving of at most 5 + 5
// leaves one). Every lane keeps the same state; lane 0 writes the stack, and
// region_setup's barriers lie between any write and read of one entry.
struct BlockWalk {
  int x0, y0, x1, y1;  // the current rectangle, inclusive
  int depth;
  unsigned* stack;
  static constexpr int kDepth = 10;
  __device__ __forceinline__ BlockWalk(unsigned* s, int w, int h)
      : x0(0), y0(0), x1(w - 1), y1(h - 1), depth(0), stack(s) {}
  __device__ __forceinline__ bool single() const { return x0 == x1 && y0 == y1; }
  // Keeps the first half as the current rectangle.
  __device__ __forceinline__ void split() {
    const bool wide = x1 - x0 >= y1 - y0;
    const int mx = (x0 + x1) >> 1, my = (y0 + y1) >> 1;
    if (threadIdx.x == 0)
      stack[depth] = (unsigned)((wide ? mx + 1 : x0) | (wide ? y0 : my + 1) << 8 | x1 << 16 | y1 << 24);
    ++depth;
    x1 = wide ? mx : x1;
    y1 = wide ? y1 : my;
  }
  // The next rectangle; false when none is left.
  __device__ __forceinline__ bool next() {
    if (depth == 0) return false;
    const unsigned v = stack[--depth];
    x0 = v & 255;
    y0 = (v >> 8) & 255;
    x1 = (v >> 16) & 255;
    y1 = v >> 24;
    return true;
  }
};

// Work-item scheduling. Items are (event, layer, tile block) triples in
// row-major block order, so consecutive items are spatially adjacent and
// share halo tiles. Plain launches take item = workgroup id: the dispatcher
// issues workgroups in order, so the items in flight stay adjacent.
// Persistent launches split the items into one contiguous run per XCD (each
// XCD has its own L2) and pop them from that XCD's queue head; an XCD whose
// run is exhausted steals from the others. The XCD comes from the hardware
// XCC_ID register.
__device__ __forceinline__ int xcc_id() {
  // s_getreg_b32 hwreg(HW_REG_XCC_ID = 20, offset 0, 4 bits)
  return __builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20) & (kQueues - 1);
}

__device__ __forceinline__ void queue_range(int n, int x, int& lo, int& cnt) {
  const int q = n / kQueues, r = n - q * kQueues;
  lo = x * q + min(x, r);
  cnt = q + (x < r ? 1 : 0);
}

struct ItemSched {
  int v;     // queues visited so far (persistent) / item taken (plain)
  int home;  // this workgroup's XCD
};

// Next work item, or -1 when none is left; uniform across the workgroup.
template <bool G>
__device__ __forceinline__ int next_item(ItemSched& st, int n_items, int* heads, int* s_item) {
  if constexpr (!G) {
    if (st.v++ > 0) return -1;
    return (int)blockIdx.x < n_items ? (int)blockIdx.x : -1;
  } else {
    while (st.v < kQueues) {  // own XCD's queue first, then steal
      const int x = (st.home + st.v) & (kQueues - 1);
      int lo, cnt;
      queue_range(n_items, x, lo, cnt);
      __syncthreads();
      if (threadIdx.x == 0) *s_item = atomicAdd(&heads[x * kCounterStride], 1);
      __syncthreads();
      const int k = *s_item;
      if (k < cnt) return lo + k;
      ++st.v;
    }
    return -1;
  }
}

// Query window [v - w', v + w'] in tile coordinates (w' from window_half).
struct Window {
  int x0, x1, y0, y1;
};
__device__ __forceinline__ Window query_window(const Geom& g, float w, float xi, float yi) {
  const float wx = window_half(w, xi), wy = window_half(w, yi);
  Window W;
  W.x0 = tile_coord(__fsub_rn(xi, wx), g.x0, g.inv_t, g.nx);
  W.x1 = tile_coord(__fadd_rn(xi, wx), g.x0, g.inv_t, g.nx);
  W.y0 = tile_coord(__fsub_rn(yi, wy), g.y0, g.inv_t, g.ny);
  W.y1 = tile_coord(__fadd_rn(yi, wy), g.y0, g.inv_t, g.ny);
  return W;
}

// ---------------------------------------------------------------------------
// Density (Eq. 3): rho_i = sum of E_j over same-layer j with d2 < dc2, added
// in ascending j. Tiles list their hits in ascending index; a query first marks
// the passing hits of each window tile in a 64-bit mask, then merges only the
// passing hits of the (at most MAXL x MAXL) sorted tile lists.
// Staged records: (x, y, E) and the hit index, laid out per instance (Staged).
// ---------------------------------------------------------------------------
// A staged record's position and energy.
struct Rec3 {
  float x, y, e;
};

// Staged density records, 16 bytes per hit in both layouts:
// * the two-tile instance keeps 12-byte records (x, y, E) with the hit
//   indices (the sort keys) in an array of their own, so that the records one
//   wave reads at once, and the keys the quad-list build probes, spread over
//   more LDS banks than 16-byte records would;
// * the three-tile instance keeps 16-byte records (x, y, E, hit index), whose
//   mask loop reads the (x, y) of two records in one 64-bit pair load.
template <int MAXL>
struct Staged {
  static constexpr bool kSplit = MAXL == 2;
  static constexpr int kRecBytes = kSplit ? 12 : 16;
  static constexpr int kKeyShift = kSplit ? 2 : 4;  // log2 of the LDS stride between keys
  unsigned char* base;
  int cap;
  __device__ __forceinline__ const float* rec(int j) const {
    return reinterpret_cast<const float*>(base + kRecBytes * j);
  }
  __device__ __forceinline__ float2 xy(int j) const {
    if constexpr (kSplit) {
      const float* r = rec(j);
      return make_float2(r[0], r[1]);
    } else {
      return *reinterpret_cast<const float2*>(rec(j));
    }
  }
  __device__ __forceinline__ const int* key_ptr(int j) const {
    if constexpr (kSplit) return reinterpret_cast<const int*>(base + 12 * cap) + j;
    else return reinterpret_cast<const int*>(base + 16 * j + 12);
  }
  __device__ __forceinline__ int key(int j) const { return *key_ptr(j); }
  __device__ __forceinline__ void put(int j, float x, float y, float en, int h) const {
    if constexpr (kSplit) {
      *reinterpret_cast<Rec3*>(base + 12 * j) = Rec3{x, y, en};
      *const_cast<int*>(key_ptr(j)) = h;
    } else {
      *reinterpret_cast<float4*>(base + 16 * j) = make_float4(x, y, en, __int_as_float(h));
    }
  }
  // The record at a quad-list entry (its byte offset). As one three- or
  // four-float vector; at the density kernel's occupancy bound the compiler
  // issues the split layout's as a two-word and a one-word LDS load from the
  // same address.
  __device__ __forceinline__ Rec3 at(int byte_off) const {
    if constexpr (kSplit) {
      typedef float Float3 __attribute__((ext_vector_type(3)));
      typedef Float3 Float3A4 __attribute__((aligned(4)));
      const Float3 v = *reinterpret_cast<const Float3A4*>(base + byte_off);
      return Rec3{v.x, v.y, v.z};
    } else {
      const float4 v = *reinterpret_cast<const float4*>(base + byte_off);
      return Rec3{v.x, v.y, v.z};
    }
  }
};

// Energy and hit index of a staged record, for both layouts (a 16-byte
// record carries its index in the fourth word; a 12-byte record's index is in
// the array beside the records).
__device__ __forceinline__ float rec_e(const float4& r) { return r.z; }
__device__ __forceinline__ float rec_e(const Rec3& r) { return r.e; }
__device__ __forceinline__ int rec_key(const float4* rec, const int*, int j) { return __float_as_int(rec[j].w); }
__device__ __forceinline__ int rec_key(const Rec3*, const int* keys, int j) { return keys[j]; }

template <int MAXL, int K, typename T>
__device__ __forceinline__ float density_merge_full(const T* __restrict__ rec, const int* __restrict__ keys, const int* lo,
                                                   const int* hi, float xi, float yi, float dc2, float ka) {
  constexpr int NL = MAXL * MAXL;
  int cur[NL], head[NL];
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    cur[k] = lo[k];
    head[k] = cur[k] < hi[k] ? rec_key(rec, keys, cur[k]) : INT_MAX;
  }
  float acc = 0.0f;
  for (;;) {
    int m = head[0];
#pragma unroll
    for (int k = 1; k < NL; ++k) m = min(m, head[k]);
    if (m == INT_MAX) break;
    int p = 0;
#pragma unroll
    for (int k = 0; k < NL; ++k)
      if (head[k] == m) p = cur[k];
    const T r = rec[p];
    const float d2 = dist2(xi, yi, r.x, r.y);
    if (d2 < dc2) acc = __fadd_rn(acc, kernel_term<K>(d2, ka, rec_e(r)));
    const int np = p + 1;
    int nh = INT_MAX;
    bool more = false;
#pragma unroll
    for (int k = 0; k < NL; ++k)
      if (head[k] == m) more = np < hi[k];
    if (more) nh = rec_key(rec, keys, np);
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      if (head[k] == m) {
        cur[k] = np;
        head[k] = nh;
      }
    }
  }
  return acc;
}

// Lowest set bit of a 64-bit mask kept as two 32-bit halves.
__device__ __forceinline__ int lowbit64(unsigned lo, unsigned hi) {
  return lo ? __builtin_ctz(lo) : 32 + __builtin_ctz(hi);
}

template <int MAXL, int K, typename T>
__device__ __forceinline__ float density_two_pass(const T* __restrict__ rec, const int* __restrict__ keys, const int* lo,
                                                  const int* hi, float xi, float yi, float dc2, float ka) {
  constexpr int NL = MAXL * MAXL;
  unsigned mlo[NL], mhi[NL];
  bool big = false;
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    mlo[k] = 0u;
    mhi[k] = 0u;
    const int len = hi[k] - lo[k];
    big |= len > 64;
    const T* base = rec + lo[k];
    const int n0 = min(len, 32);
    int c = 0;
    for (; c + 3 < n0; c += 4) {
      const float2 q0 = *reinterpret_cast<const float2*>(base + c);
      const float2 q1 = *reinterpret_cast<const float2*>(base + c + 1);
      const float2 q2 = *reinterpret_cast<const float2*>(base + c + 2);
      const float2 q3 = *reinterpret_cast<const float2*>(base + c + 3);
      const unsigned m4 = (dist2(xi, yi, q0.x, q0.y) < dc2 ? 1u : 0u) | (dist2(xi, yi, q1.x, q1.y) < dc2 ? 2u : 0u) |
                          (dist2(xi, yi, q2.x, q2.y) < dc2 ? 4u : 0u) | (dist2(xi, yi, q3.x, q3.y) < dc2 ? 8u : 0u);
      mlo[k] |= m4 << c;
    }
    for (; c < n0; ++c) {
      const float2 q = *reinterpret_cast<const float2*>(base + c);
      mlo[k] |= (dist2(xi, yi, q.x, q.y) < dc2 ? 1u : 0u) << c;
    }
    const int n1 = min(len, 64);
#pragma unroll 4
    for (int c = 32; c < n1; ++c) {
      const float2 q = *reinterpret_cast<const float2*>(base + c);
      mhi[k] |= (dist2(xi, yi, q.x, q.y) < dc2 ? 1u : 0u) << (c - 32);
    }
  }
  if (big) return density_merge_full<MAXL, K>(rec, keys, lo, hi, xi, yi, dc2, ka);
  // heads of the lists; with the flat kernel the head's energy is kept,
  // otherwise the selected head is re-read from LDS when it is added
  int hh[NL];
  float ee[K == 0 ? NL : 1];
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    hh[k] = INT_MAX;
    if constexpr (K == 0) ee[k] = 0.0f;
    if (mlo[k] | mhi[k]) {
      const int j = lo[k] + lowbit64(mlo[k], mhi[k]);
      hh[k] = rec_key(rec, keys, j);
      if constexpr (K == 0) ee[k] = rec_e(rec[j]);
    }
  }
  float acc = 0.0f;
  for (;;) {
    int m = hh[0];
#pragma unroll
    for (int k = 1; k < NL; ++k) m = min(m, hh[k]);
    if (m == INT_MAX) break;
    // the selected list: take its head, drop its lowest passing bit
    float e = 0.0f;
    if constexpr (K == 0) e = ee[0];
    unsigned ml = mlo[0], mh = mhi[0];
    int base = lo[0];
#pragma unroll
    for (int k = 1; k < NL; ++k) {
      if (hh[k] == m) {
        if constexpr (K == 0) e = ee[k];
        ml = mlo[k];
        mh = mhi[k];
        base = lo[k];
      }
    }
    if constexpr (K == 0) {
      acc = __fadd_rn(acc, e);
    } else {
      const T rs = rec[base + lowbit64(ml, mh)];
      acc = __fadd_rn(acc, kernel_term<K>(dist2(xi, yi, rs.x, rs.y), ka, rec_e(rs)));
    }
    if (ml)
      ml &= ml - 1u;
    else
      mh &= mh - 1u;
    const bool more = (ml | mh) != 0u;
    int nk = INT_MAX;
    float ne = 0.0f;
    if (more) {
      const int j = base + lowbit64(ml, mh);
      nk = rec_key(rec, keys, j);
      ne = rec_e(rec[j]);
    }
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      if (hh[k] == m) {
        mlo[k] = ml;
        mhi[k] = mh;
        hh[k] = nk;
        if constexpr (K == 0) ee[k] = ne;
      }
    }
  }
  return acc;
}

// Global-memory density (tiles too dense to stage): the window's tile lists,
// each in ascending hit index in the CSR, are merged on the fly (cursors and
// head indices in registers), so each query passes over its window once.
template <int K>
__device__ __forceinline__ float density_global(const Geom& g, const Arena& a, int64_t ubase, float xi, float yi) {
  const Window W = query_window(g, g.win_dc, xi, yi);
  constexpr int NL = 9;  // the density window spans at most 3 x 3 tiles
  int cur[NL], end[NL], head[NL];
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    const int ty = W.y0 + k / 3, tx = W.x0 + k % 3;
    cur[k] = end[k] = 0;
    if (ty <= W.y1 && tx <= W.x1) {
      const int64_t t = ubase + (int64_t)ty * g.nx + tx;
      cur[k] = a.tile_start[t];
      end[k] = a.tile_start[t + 1];
    }
    head[k] = cur[k] < end[k] ? a.hs[cur[k]] : INT_MAX;
  }
  float acc = 0.0f;
  for (;;) {
    int m = head[0];
#pragma unroll
    for (int k = 1; k < NL; ++k) m = min(m, head[k]);
    if (m == INT_MAX) break;
    int s = 0;
#pragma unroll
    for (int k = 0; k < NL; ++k)
      if (head[k] == m) s = cur[k];
    const float d2 = dist2(xi, yi, a.xs[s], a.ys[s]);
    if (d2 < g.dc2) acc = __fadd_rn(acc, kernel_term<K>(d2, g.ka, a.es[s]));
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      if (head[k] == m) {
        ++cur[k];
        head[k] = cur[k] < end[k] ? a.hs[cur[k]] : INT_MAX;
      }
    }
  }
  return acc;
}

// Quad-list entries are byte offsets of records (a staged position times the
// record size, below 2^15 for every LDS cap), so a scan adds no index scaling.
static_assert(kMaxLdsCap * 16 <= 65536, "quad-list byte offsets are 16-bit");
// Byte address of a shared-memory object in the workgroup's LDS, and a load
// from such an address: loops that step through LDS by byte address then need
// no base register added per access.
__device__ __forceinline__ unsigned lds_address(const void* p) {
  return (unsigned)(size_t)(const __attribute__((address_space(3))) void*)p;
}
__device__ __forceinline__ int lds_load_int(unsigned addr) {
  return *(const __attribute__((address_space(3))) int*)(size_t)addr;
}
static_assert(kMaxRegionRows <= 64 && kMaxRegionTiles <= 1024, "a staged tile id is (row << 10) | column in 16 bits");

// Density over a staged region (records x, y, E and their hit indices; each
// tile in ascending hit index). With MAXL == 2 every query window lies inside the
// 2x2 tile quad anchored at its lower-left window tile; the quads a core
// query can use are merged once per region into index-ordered lists (byte
// offsets of the records), so each query is one linear scan in ascending
// hit index. Where the quads do not fit, false is returned with nothing done and
// the caller halves the block (the merges below cost more than the second
// staging: 100 layers with 900 of 1000 hits in 10 cm, 620 -> 165 us); a `single`
// tile, or a window of three tiles, takes those: a query merges its window's
// tile lists itself.
template <int MAXL, int K>
__device__ __forceinline__ bool density_staged(const Geom& g, const Arena& a, const Region& R, RegionLds& L,
                                               const Staged<MAXL>& S, unsigned short* stile, unsigned short* qidx,
                                               unsigned short sent, bool keep, bool single) {
  const int per_row = R.rw + 1;
  const int64_t ubase = (int64_t)R.unit * g.tpl;
  const int ntl = R.rh * per_row;
  // region tile of every staged position as (row << 10) | column (rows
  // < 64, columns < 1024), two lanes per tile
  for (int k = threadIdx.x; k < 2 * ntl; k += kWG) {
    const int tl = k >> 1;
    const int tr = tl / per_row, tc = tl - tr * per_row;
    if (tc == R.rw) continue;  // row-end entry
    const unsigned short code = (unsigned short)((tr << 10) | tc);
    const int end = L.ts[tl + 1];
    for (int p = L.ts[tl] + (k & 1); p < end; p += 2) stile[p] = code;
  }
  __syncthreads();
  // copy the records (tiles are already in ascending hit index); every
  // global load of a lane is issued before its first LDS store
  for (int base = 0; base < R.total; base += kStagePer * kWG) {
    Rec3 v[kStagePer];
    int h[kStagePer];
#pragma unroll
    for (int k = 0; k < kStagePer; ++k) {
      const int p = base + (int)threadIdx.x + k * kWG;
      if (p < R.total) {
        const int sl = slot_of(L, stile[p] >> 10, p);
        v[k] = Rec3{a.xs[sl], a.ys[sl], a.es[sl]};
        h[k] = a.hs[sl];
      }
    }
#pragma unroll
    for (int k = 0; k < kStagePer; ++k) {
      const int p = base + (int)threadIdx.x + k * kWG;
      if (p < R.total) S.put(p, v[k].x, v[k].y, v[k].e, h[k]);
    }
  }
  // quads anchored at region tiles [qx0, qx1] x [qy0, qy1]
  const int qx0 = max(R.cx0 - 1, 0), qx1 = min(R.cx0 + R.cw - 1, R.rw - 1);
  const int qy0 = max(R.cy0 - 1, 0), qy1 = min(R.cy0 + R.ch - 1, R.rh - 1);
  const int qw = qx1 - qx0 + 1;
  const int nquad = qw * (qy1 - qy0 + 1);
  bool use_quads = MAXL == 2 && g.density_quads && nquad < g.q_ints;
  if (use_quads) {
    if (threadIdx.x < 64) {
      // quad sizes -> offsets, 64 quads per wave step. Each list is padded
      // with the sentinel to a multiple of four entries, so the queries read
      // their lists four entries at a time with no remainder loop (pads past
      // the array are not written: the quads are then not used).
      int run = 0;
      for (int q0 = 0; q0 < nquad; q0 += 64) {
        const int q = q0 + (int)threadIdx.x;
        int len = 0;
        if (q < nquad) {
          const int ax = qx0 + q % qw, ay = qy0 + q / qw;
          const int bx1 = min(ax + 1, R.rw - 1), by1 = min(ay + 1, R.rh - 1);
          for (int ty = ay; ty <= by1; ++ty) len += L.ts[ty * per_row + bx1 + 1] - L.ts[ty * per_row + ax];
        }
        const int plen = (len + 3) & ~3;
        const int incl = wave_incl_scan(plen, threadIdx.x);
        if (q < nquad) {
          const int o = run + incl - plen;
          L.qoff[q] = o;
          for (int i = o + len; i < o + plen && i < 4 * g.lds_cap; ++i) qidx[i] = sent;
        }
        run += __builtin_amdgcn_readlane(incl, 63);
      }
      if (threadIdx.x == 0) {
        L.qoff[nquad] = run;
        *L.qtotal = run;
      }
    }
  }
  __syncthreads();
  if (use_quads && *L.qtotal > 4 * g.lds_cap && !single) return false;
  if (use_quads && *L.qtotal <= 4 * g.lds_cap && g.density_quads == 2) {
    // one lane per quad: a sequential merge of its (up to four) index-sorted
    // tile lists
    for (int q = threadIdx.x; q < nquad; q += kWG) {
      const int ax = qx0 + q % qw, ay = qy0 + q / qw;
      const int bx1 = min(ax + 1, R.rw - 1), by1 = min(ay + 1, R.rh - 1);
      int cur[4], end[4], key[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int tx = (k & 1) ? bx1 : ax, ty = (k & 2) ? by1 : ay;
        const bool dup = ((k & 1) && bx1 == ax) || ((k & 2) && by1 == ay);
        const int t = ty * per_row + tx;
        cur[k] = dup ? 0 : L.ts[t];
        end[k] = dup ? 0 : L.ts[t + 1];
        key[k] = cur[k] < end[k] ? S.key(cur[k]) : INT_MAX;
      }
      const int out = L.qoff[q], n = (end[0] - cur[0]) + (end[1] - cur[1]) + (end[2] - cur[2]) + (end[3] - cur[3]);
      for (int i = 0; i < n; ++i) {
        const int m = min(min(key[0], key[1]), min(key[2], key[3]));
        const bool s0 = key[0] == m, s1 = !s0 && key[1] == m, s2 = !s0 && !s1 && key[2] == m;
        const int pk = s0 ? cur[0] : (s1 ? cur[1] : (s2 ? cur[2] : cur[3]));
        const int ek = s0 ? end[0] : (s1 ? end[1] : (s2 ? end[2] : end[3]));
        qidx[out + i] = (unsigned short)(pk * S.kRecBytes);
        const int np = pk + 1;
        const int nk = np < ek ? S.key(np) : INT_MAX;
        const bool s3 = !s0 && !s1 && !s2;
        cur[0] = s0 ? np : cur[0];
        key[0] = s0 ? nk : key[0];
        cur[1] = s1 ? np : cur[1];
        key[1] = s1 ? nk : key[1];
        cur[2] = s2 ? np : cur[2];
        key[2] = s2 ? nk : key[2];
        cur[3] = s3 ? np : cur[3];
        key[3] = s3 ? nk : key[3];
      }
    }
    __syncthreads();
  } else if (use_quads && *L.qtotal <= 4 * g.lds_cap) {
    // place every sorted record into each quad that holds its tile: its
    // position there is its rank in its own tile plus, for each other tile
    // of the quad, the entries with a smaller hit index (each of the up to
    // eight neighbour tiles is counted once and shared by the quads)
    for (int p = threadIdx.x; p < R.total; p += kWG) {
      const int tr = stile[p] >> 10, tc = stile[p] & 1023;
      const int tl = tr * per_row + tc;
      const int hp = S.key(p);
      const int own = p - L.ts[tl];
      bool qv[2][2];
#pragma unroll
      for (int dy = 0; dy < 2; ++dy)
#pragma unroll
        for (int dx = 0; dx < 2; ++dx) {
          const int ax = tc - dx, ay = tr - dy;
          qv[dy][dx] = ax >= qx0 && ax <= qx1 && ay >= qy0 && ay <= qy1;
        }
      // lower bounds in the needed neighbour tiles. The tile offsets are read
      // without a branch: a neighbour that is not needed (or lies outside the
      // region) reads the empty pair after the last row's end.
      const int rm = max(tr - 1, 0) * per_row, r0 = tl - tc, rp = min(tr + 1, R.rh - 1) * per_row;
      const int cm = max(tc - 1, 0), cp = min(tc + 1, R.rw - 1);
      const int empty = R.rh * per_row - 1;
      int lo[9], len[9];
#pragma unroll
      for (int oy = -1; oy <= 1; ++oy)
#pragma unroll
        for (int ox = -1; ox <= 1; ++ox) {
          const int k = (oy + 1) * 3 + ox + 1;
          lo[k] = 0;
          len[k] = 0;
          if (k == 4) continue;  // the hit's own tile
          bool need = false;
#pragma unroll
          for (int dy = 0; dy < 2; ++dy)
#pragma unroll
            for (int dx = 0; dx < 2; ++dx)
              need |= qv[dy][dx] && (ox == -dx || ox == 1 - dx) && (oy == -dy || oy == 1 - dy);
          const int nx = tc + ox, ny = tr + oy;
          need &= nx >= 0 && nx < R.rw && ny >= 0 && ny < R.rh;
          const int nt = need ? (oy < 0 ? rm : oy > 0 ? rp : r0) + (ox < 0 ? cm : ox > 0 ? cp : tc) : empty;
          lo[k] = L.ts[nt];
          len[k] = L.ts[nt + 1] - lo[k];
        }
      // The searches share one power-of-two step sequence, from the largest
      // of the tiles down to one record. Each holds the LDS address of its
      // last counted key (at first, the key before its tile); a step probes
      // the key `step` records further on, clamped to the tile's last key. A
      // clamped probe is taken only when every key of the tile is smaller,
      // which is then the count. So no search branches, and all loads of a
      // step are issued before its compares. An empty tile starts and ends
      // at record 0's key, so every probe reads a staged key.
      int maxlen = 0;
#pragma unroll
      for (int k = 0; k < 9; ++k) maxlen = max(maxlen, len[k]);
      constexpr int ks = Staged<MAXL>::kKeyShift;
      const unsigned key0 = lds_address(S.key_ptr(0));  // LDS address of record 0's key
      unsigned at[9], end[9];
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        at[k] = len[k] > 0 ? key0 + (((unsigned)lo[k] - 1u) << ks) : key0;
        end[k] = at[k] + ((unsigned)len[k] << ks);
      }
      // per quad, the sum of its three searches' starting addresses
      unsigned start3[2][2];
#pragma unroll
      for (int dy = 0; dy < 2; ++dy)
#pragma unroll
        for (int dx = 0; dx < 2; ++dx) {
          start3[dy][dx] = 0u;
#pragma unroll
          for (int oy = -dy; oy <= 1 - dy; ++oy)
#pragma unroll
            for (int ox = -dx; ox <= 1 - dx; ++ox)
              if (ox != 0 || oy != 0) start3[dy][dx] += at[(oy + 1) * 3 + ox + 1];
        }
      // at least one step (one key): with every tile empty it changes nothing
      unsigned step = (1u << ks) << max(31 - __clz(maxlen), 0);
      do {
        unsigned pr[9];
        int kv[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) {
          if (k == 4) continue;
          pr[k] = min(at[k] + step, end[k]);
          kv[k] = lds_load_int(pr[k]);
        }
#pragma unroll
        for (int k = 0; k < 9; ++k)
          if (k != 4) at[k] = kv[k] < hp ? pr[k] : at[k];
        step >>= 1;
      } while (step >= (1u << ks));
      // each quad: the own rank plus the three neighbour counts (one key
      // stride of address per counted key)
#pragma unroll
      for (int dy = 0; dy < 2; ++dy)
#pragma unroll
        for (int dx = 0; dx < 2; ++dx) {
          if (!qv[dy][dx]) continue;
          unsigned below = 0u - start3[dy][dx];
#pragma unroll
          for (int oy = -dy; oy <= 1 - dy; ++oy)
#pragma unroll
            for (int ox = -dx; ox <= 1 - dx; ++ox)
              if (ox != 0 || oy != 0) below += at[(oy + 1) * 3 + ox + 1];
          qidx[L.qoff[(tr - dy - qy0) * qw + (tc - dx - qx0)] + own + (int)(below >> ks)] =
              (unsigned short)(p * S.kRecBytes);
        }
    }
    __syncthreads();
  } else {
    use_quads = false;
  }
  const int nq = L.core_lo[R.ch];
  int cr = 0;
  for (int q = threadIdx.x; q < nq; q += kWG) {
    int row, p;
    core_query(L, R, q, cr, row, p);
    const int slot = slot_of(L, row, p);
    const float2 me = S.xy(p);
    const float xi = me.x, yi = me.y;
    const Window W = query_window(g, g.win_dc, xi, yi);
    const int tx0 = W.x0 - R.rx0, tx1 = W.x1 - R.rx0, ty0 = W.y0 - R.ry0, ty1 = W.y1 - R.ry0;
    const bool ok = tx0 >= 0 && ty0 >= 0 && tx1 < R.rw && ty1 < R.rh && tx1 - tx0 < MAXL && ty1 - ty0 < MAXL;
    float rho = 0.0f;
    if (ok && use_quads) {
      const int qq = (ty0 - qy0) * qw + (tx0 - qx0);
      const unsigned short* qp = qidx + L.qoff[qq];
      const unsigned short* const qe = qidx + L.qoff[qq + 1];
      // four entries at a time (the lists are padded to a multiple of four);
      // additions stay in ascending index order
      for (; qp < qe; qp += 4) {
        const int i0 = qp[0], i1 = qp[1], i2 = qp[2], i3 = qp[3];
        const Rec3 r0 = S.at(i0), r1 = S.at(i1), r2 = S.at(i2), r3 = S.at(i3);
        const float d0 = dist2(xi, yi, r0.x, r0.y), d1 = dist2(xi, yi, r1.x, r1.y);
        const float d2 = dist2(xi, yi, r2.x, r2.y), d3 = dist2(xi, yi, r3.x, r3.y);
        const float a0 = __fadd_rn(rho, kernel_term<K>(d0, g.ka, r0.e));
        rho = d0 < g.dc2 ? a0 : rho;
        const float a1 = __fadd_rn(rho, kernel_term<K>(d1, g.ka, r1.e));
        rho = d1 < g.dc2 ? a1 : rho;
        const float a2 = __fadd_rn(rho, kernel_term<K>(d2, g.ka, r2.e));
        rho = d2 < g.dc2 ? a2 : rho;
        const float a3 = __fadd_rn(rho, kernel_term<K>(d3, g.ka, r3.e));
        rho = d3 < g.dc2 ? a3 : rho;
      }
    } else if (ok) {
      int lo[MAXL * MAXL], hi[MAXL * MAXL];
#pragma unroll
      for (int jy = 0; jy < MAXL; ++jy)
#pragma unroll
        for (int jx = 0; jx < MAXL; ++jx) {
          const int k = jy * MAXL + jx;
          const int ty = ty0 + jy, tx = tx0 + jx;
          if (ty <= ty1 && tx <= tx1) {
            lo[k] = L.ts[ty * per_row + tx];
            hi[k] = L.ts[ty * per_row + tx + 1];
          } else {
            lo[k] = 0;
            hi[k] = 0;
          }
        }
      if constexpr (Staged<MAXL>::kSplit)
        rho = density_two_pass<MAXL, K>(reinterpret_cast<const Rec3*>(S.base), S.key_ptr(0), lo, hi, xi, yi, g.dc2, g.ka);
      else
        rho = density_two_pass<MAXL, K>(reinterpret_cast<const float4*>(S.base), nullptr, lo, hi, xi, yi, g.dc2, g.ka);
    } else {
      atomicOr(a.err, (uint32_t)E_WINDOW);
      rho = density_global<K>(g, a, ubase, xi, yi);
    }
    a.rho[slot] = rho;
    if (keep) a.rho_out[S.key(p)] = rho;
  }
  return true;
}

// Regions whose tiles are too dense for LDS are not searched by the workgroup
// that meets them: their core queries are queued, tile by tile in chunks of
// `per` consecutive slots (the tile and the chunk's first slot, in the key and
// rank buffers, which are free after the grid build), and a spill kernel after
// the stage spreads the chunks over every workgroup of the GPU. Each tile is a
// core tile of one region, and a chunk holds at least one hit, so there are at
// most n chunks.
__device__ __forceinline__ void spill_region(const Geom& g, const Arena& a, const Region& R, int counter, int per) {
  const int64_t ubase = (int64_t)R.unit * g.tpl;
  for (int k = threadIdx.x; k < R.cw * R.ch; k += kWG) {
    const int cy = k / R.cw, cx = k - cy * R.cw;
    const int64_t t = ubase + (int64_t)(R.ry0 + R.cy0 + cy) * g.nx + R.rx0 + R.cx0 + cx;
    const int s0 = a.tile_start[t], s1 = a.tile_start[t + 1];
    const int nch = (s1 - s0 + per - 1) / per;
    if (nch == 0) continue;
    const int i0 = atomicAdd(&a.counters[counter], nch);
    for (int c = 0; c < nch; ++c) {
      a.key[i0 + c] = (int)t;
      a.rank[i0 + c] = s0 + c * per;
    }
  }
}

// Density of the spilled queries, one lane per query. The tile lists around the
// chunk's tile are staged in rounds: each round takes a share of what is left of
// every list, cut at one hit index, so that its hits come before all later ones,
// and ranks them into one list in ascending hit index that every lane scans. The
// scan is bound by its additions, where a merge of the lists in global memory by
// every lane for itself waited for each hit's loads (100 layers with 1700 hits in
// 10 cm: density 2596 -> 451 us).
constexpr int kSpillHits = 1024;  // staged per round
constexpr int kSpillShare = 32;   // least share of a list in a round

// Entries of the ascending list v[0 .. n) below `key`.
__device__ __forceinline__ int lower_bound_lds(const int* v, int n, int key) {
  int lo = 0;
  while (n > 0) {
    const int half = n >> 1;
    const bool below = v[lo + half] < key;
    lo = below ? lo + half + 1 : lo;
    n = below ? n - half - 1 : half;
  }
  return lo;
}

template <bool G, int K>
__global__ __launch_bounds__(kWG) void k_density_spill(DescArg<G> dg, Geom g, Arena a) {
  constexpr int NL = 9;  // the density window spans at most 3 x 3 tiles
  __shared__ float4 s_rec[kSpillHits + 4];
  __shared__ int s_idx[kSpillHits];
  __shared__ int s_cur[NL], s_end[NL], s_off[NL + 1], s_cut[NL], s_next[NL];
  const int nch = a.counters[C_SPILL_RHO];
  const bool keep = g.flags & 2u;
  const int tid = threadIdx.x;
  for (int i = blockIdx.x; i < nch; i += gridDim.x) {
    const int64_t t = a.key[i];
    const int slot = a.rank[i] + tid;
    const int tu = (int)(t % g.tpl);
    const int64_t ubase = t - tu;
    const int ty = tu / g.nx, tx = tu - ty * g.nx;
    const bool active = slot < a.tile_start[t + 1];
    float xi = 0.0f, yi = 0.0f, acc = 0.0f;
    bool inside = true;
    if (active) {
      xi = a.xs[slot];
      yi = a.ys[slot];
      const Window W = query_window(g, g.win_dc, xi, yi);
      inside = W.x0 >= tx - 1 && W.x1 <= tx + 1 && W.y0 >= ty - 1 && W.y1 <= ty + 1;
    }
    __syncthreads();  // every lane has left the previous chunk's rounds
    if (tid < NL) {
      const int y = ty + tid / 3 - 1, x = tx + tid % 3 - 1;
      const bool in = y >= 0 && y < g.ny && x >= 0 && x < g.nx;
      const int64_t n = ubase + (int64_t)y * g.nx + x;
      s_cur[tid] = in ? a.tile_start[n] : 0;
      s_end[tid] = in ? a.tile_start[n + 1] : 0;
    }
    for (;;) {
      __syncthreads();
      int left = 0;
#pragma unroll
      for (int l = 0; l < NL; ++l) left += s_end[l] - s_cur[l];
      if (left == 0) break;  // uniform
      // shares of the lists; the first hit index that a list leaves out
      if (tid < NL) {
        int off = 0, take = 0, first = INT_MAX;
        for (int l = 0; l <= tid; ++l) {
          const int rem = s_end[l] - s_cur[l];
          off += take;
          take = left <= kSpillHits
                     ? rem
                     : min(rem, kSpillShare + (int)((int64_t)(kSpillHits - NL * kSpillShare) * rem / left));
        }
        if (take < s_end[tid] - s_cur[tid]) first = a.hs[s_cur[tid] + take];
        s_off[tid] = off;
        s_next[tid] = first;
        if (tid == NL - 1) s_off[NL] = off + take;
      }
      __syncthreads();
      int off[NL + 1];
#pragma unroll
      for (int l = 0; l <= NL; ++l) off[l] = s_off[l];
      const int staged = off[NL];
      constexpr int U = kSpillHits / kWG;
      int list[U], pos[U], idx[U];
      float4 rec[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int p = u * kWG + tid;
        int l = 0;
#pragma unroll
        for (int q = 1; q < NL; ++q) l = p >= off[q] ? q : l;
        list[u] = l;
        pos[u] = p - s_off[l];
        if (p < staged) {
          const int s = s_cur[l] + pos[u];
          idx[u] = a.hs[s];
          rec[u] = make_float4(a.xs[s], a.ys[s], a.es[s], 0.0f);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (u * kWG + tid < staged) s_idx[u * kWG + tid] = idx[u];
      __syncthreads();
      if (tid < NL) {
        int cut = INT_MAX;
#pragma unroll
        for (int l = 0; l < NL; ++l) cut = min(cut, s_next[l]);
        // the list that sets the cut gives its whole share: every round advances
        const int share = s_off[tid + 1] - s_off[tid];
        s_cut[tid] = s_next[tid] == cut ? share : lower_bound_lds(s_idx + s_off[tid], share, cut);
      }
      __syncthreads();
      int m = 0;
#pragma unroll
      for (int l = 0; l < NL; ++l) m += s_cut[l];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (u * kWG + tid >= staged || pos[u] >= s_cut[list[u]]) continue;
        int r = pos[u];
#pragma unroll 1
        for (int l = 0; l < NL; ++l)
          if (l != list[u]) r += lower_bound_lds(s_idx + s_off[l], s_cut[l], idx[u]);
        s_rec[r] = rec[u];
      }
      // to a multiple of four with records at an infinite distance
      if (tid < 4) s_rec[m + tid] = make_float4(__int_as_float(0x7f800000), 0.0f, 0.0f, 0.0f);
      __syncthreads();
      if (tid < NL) s_cur[tid] += s_cut[tid];
      if (active)
        for (int q = 0; q < m; q += 4) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float4 c = s_rec[q + v];
            const float d2 = dist2(xi, yi, c.x, c.y);
            if (d2 < g.dc2) acc = __fadd_rn(acc, kernel_term<K>(d2, g.ka, c.z));
          }
        }
    }
    if (active) {
      if (!inside) acc = density_global<K>(g, a, ubase, xi, yi);
      a.rho[slot] = acc;
      if (keep) a.rho_out[a.hs[slot]] = acc;
    }
  }
}

// The flat-kernel quad path is built for seven waves per SIMD (72 VGPRs), so
// that an LDS cap of up to 768 staged hits fits seven workgroups per CU; the
// compiler then keeps one item-level value in scratch, reloaded once per work
// item. The other instances keep their registers (they would spill in loops).
constexpr int density_min_waves(int maxl, int k) { return maxl == 2 && k == 0 ? 7 : 1; }

template <bool G, int MAXL, int K>
__global__ __launch_bounds__(kWG, density_min_waves(MAXL, K)) void k_density(DescArg<G> dg, Geom g, Arena a) {
  const RunDesc d = dg.get();
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int s_rows[kRowMetaInts];
  __shared__ int s_item;
  __shared__ unsigned s_stack[BlockWalk::kDepth];
  const Staged<MAXL> S{smem, g.lds_cap};
  unsigned short* stile = reinterpret_cast<unsigned short*>(smem + 16 * g.lds_cap);  // both layouts: 16 B per hit
  unsigned short* qidx = reinterpret_cast<unsigned short*>(smem + density_qidx_offset(g.lds_cap));
  // the record every quad list is padded with, to a multiple of four entries:
  // x = +inf puts it at an infinite squared distance from every query
  const unsigned short sent = (unsigned short)density_sentinel_offset(g.lds_cap);
  if (threadIdx.x == 0)
    *reinterpret_cast<float4*>(smem + sent) = make_float4(__int_as_float(0x7f800000), 0.0f, 0.0f, 0.0f);
  int* meta = reinterpret_cast<int*>(smem + lds_records_density(g.lds_cap));
  RegionLds L = region_lds(s_rows, meta, meta + g.ts_ints);
  const int n_items = d.n_events * g.L * g.bpu;
  const bool keep = g.flags & 2u;
  ItemSched st{0, G ? xcc_id() : 0};
  for (int item; (item = next_item<G>(st, n_items, &a.counters[C_QUEUE_RHO], &s_item)) >= 0;) {
    int unit, tx0, ty0, tx1, ty1;
    item_block(g, item, unit, tx0, ty0, tx1, ty1);
    BlockWalk B(s_stack, tx1 - tx0 + 1, ty1 - ty0 + 1);
    for (bool more = true; more;) {
      Region R;
      make_region(g, unit, tx0 + B.x0, ty0 + B.y0, tx0 + B.x1, ty0 + B.y1, R);
      region_setup(g, a, R, L);
      if (L.core_lo[R.ch] > 0) {
        if (R.total <= g.lds_cap) {
          if (!density_staged<MAXL, K>(g, a, R, L, S, stile, qidx, sent, keep, B.single())) {
            B.split();
            continue;
          }
        } else if (B.single()) {
          spill_region(g, a, R, C_SPILL_RHO, kWG);
        } else {
          B.split();
          continue;
        }
      }
      more = B.next();
    }
  }
}

// ---------------------------------------------------------------------------
// Nearest-higher (Eq. 4) and the decision (Sec. 2.2, Algorithm 3).
// Phase 1 searches a small window of radius r1 <= d_m; when its best
// higher hit lies strictly within r1, no hit outside that window can be
// closer, so the query is done. Other queries are queued in LDS and searched
// over the full d_m window with `tpq` lanes each (phase 2).
// Records: (x, y, hit index as bits, ord(rho)); the last two halves form
// the 64-bit (ord(rho), index) key in register order.
// ---------------------------------------------------------------------------
__device__ __forceinline__ unsigned long long key64(unsigned hi, unsigned lo) {
  return ((unsigned long long)hi << 32) | lo;
}

struct NhBest {
  unsigned long long k;  // (d2 bits, caller index) of the best so far
  int p;                 // LDS position >= 0, or global slot s encoded as -2 - s; -1 none
  __device__ __forceinline__ float d2() const { return __uint_as_float((unsigned)(k >> 32)); }
  __device__ __forceinline__ int h() const { return (int)(unsigned)(k & 0xffffffffu); }
};

// Search state before any candidate, for the squared radius thr: the key
// (thr, 0) is beaten exactly by the keys (d2, index) with d2 < thr, so the
// radius test needs no comparison of its own.
__device__ __forceinline__ NhBest nh_start(float thr) { return NhBest{key64(__float_as_uint(thr), 0u), -1}; }

// One candidate j for query i: eligible when j is higher (ord/index keys);
// keeps the lexicographic minimum of (d2, index), which starts at
// nh_start(thr), and the candidate's position pq. d2 >= 0, so its bit
// pattern orders like its value.
template <bool STRICT>
__device__ __forceinline__ void nh_consider(NhBest& b, float d2, unsigned ordj, unsigned hj, int pq, unsigned ordi,
                                            unsigned hi) {
  const bool higher = STRICT ? ordj > ordi : key64(ordj, hj) > key64(ordi, hi);
  const unsigned long long ck = key64(__float_as_uint(d2), hj);
  const bool take = higher & (ck < b.k);  // branch-free select
  b.k = take ? ck : b.k;
  b.p = take ? pq : b.p;
}

// Staged records carry, in place of the caller index, the word
// (event-local index << kPosBits) | LDS position. Within one event it orders
// like the caller index, so the (rho, index) and (d2, index) keys compare as
// before, and the winner's LDS position comes back out of its key: the scan
// tracks no position of its own.
__device__ __forceinline__ unsigned nh_pack(int h, int ev_first, int p) {
  return ((unsigned)(h - ev_first) << kPosBits) | (unsigned)p;
}
__device__ __forceinline__ int nh_unpack_h(unsigned z, int ev_first) { return ev_first + (int)(z >> kPosBits); }
// After a staged scan from key k0: a found winner gets its LDS position in
// b.p and its caller index back in the key's low word.
__device__ __forceinline__ void nh_unpack(NhBest& b, unsigned long long k0, int ev_first) {
  if (b.p == -1 && b.k < k0) {
    const unsigned z = (unsigned)(b.k & 0xffffffffu);
    b.p = (int)(z & kPosMask);
    b.k = key64((unsigned)(b.k >> 32), (unsigned)nh_unpack_h(z, ev_first));
  }
}

__device__ __forceinline__ void nh_reduce(NhBest& b, int tpq) {
  for (int o = 1; o < tpq; o <<= 1) {
    const unsigned long long ok = __shfl_xor(b.k, o, 64);
    const int op = __shfl_xor(b.p, o, 64);
    if (ok < b.k) {
      b.k = ok;
      b.p = op;
    }
  }
}

// Writes the decision for the hit in `slot` with nearest-higher `b` (b.p
// already converted to a slot index, or -1).
//
// The unit path numbers seeds and builds follower lists unit by unit
// afterwards. It needs only each unit's counts of both here: the workgroup
// collects them in `counts` (the hits it decides together are in one unit).
__device__ __forceinline__ void decide_and_store(const Geom& g, const Arena& a, const RunDesc& d, int* counts, int slot,
                                                 int hi, float ri, const NhBest& b, int ev_first) {
  const bool has = b.p >= 0;
  const float d2 = has ? b.d2() : __int_as_float(0x7f800000);
  const bool seed = ri > g.rho_c && d2 > g.dcs2;
  const bool outlier = ri < g.rho_c && d2 > g.do2;
  const bool follower = !seed && !outlier && has;
  a.parent[slot] = follower ? b.p : slot;
  a.flags[slot] = (uint8_t)((seed ? F_SEED : 0) | (outlier ? F_OUTLIER : 0) | (follower ? F_FOLLOWER : 0));
  if (g.units) {
    const unsigned long long ms = __builtin_amdgcn_ballot_w64(seed), mf = __builtin_amdgcn_ballot_w64(follower);
    const unsigned long long on = __builtin_amdgcn_ballot_w64(true);
    if (((int)threadIdx.x & 63) == __ffsll((long long)on) - 1) {
      atomicAdd(&counts[0], __popcll(ms));
      atomicAdd(&counts[1], __popcll(mf));
    }
  } else {
    if (seed) atomicOr(&a.seedbits[hi >> 5], 1u << (hi & 31));
    if (follower && builds_lists(g)) a.frank[slot] = atomicAdd(&a.fstart[b.h()], 1);
  }
  if (g.flags & 2u) {
    a.nh_out[hi] = has ? b.h() - ev_first : -1;
    a.d2_out[hi] = d2;
  }
}

// One staged record r for query i, as nh_consider but tracking no position:
// the record's index word carries it (nh_pack). The eligibility test comes
// first, and the scheduling barrier keeps the distance arithmetic after it:
// the record's rho word is then dead when d2 is formed, so d2 takes its
// register and (index word, d2) is already the register pair of the key.
template <bool STRICT>
__device__ __forceinline__ void nh_consider_rec(NhBest& b, float4 r, float xi, float yi, unsigned ordi, unsigned hi) {
  const unsigned ordj = __float_as_uint(r.w), hj = __float_as_uint(r.z);
  const bool higher = STRICT ? ordj > ordi : key64(ordj, hj) > key64(ordi, hi);
  __builtin_amdgcn_sched_barrier(0);
  const unsigned long long ck = key64(__float_as_uint(dist2(xi, yi, r.x, r.y)), hj);
  const bool take = higher & (ck < b.k);
  b.k = take ? ck : b.k;
}

// Scans window tiles [tx0..tx1] x [ty0..ty1] (region coordinates) of the
// staged records (x, y, index, ord(rho)) with lanes sub, sub + step, ...
template <bool STRICT>
__device__ __forceinline__ void nh_scan_staged(const float4* __restrict__ rec, const int* ts, int per_row,
                                               int tx0, int tx1, int ty0, int ty1, int sub, int step, float xi,
                                               float yi, unsigned ordi, unsigned hi, NhBest& b) {
  for (int ty = ty0; ty <= ty1; ++ty) {
    const int q0 = ts[ty * per_row + tx0];
    const int q1 = ts[ty * per_row + tx1 + 1];
    int c = q0 + sub;
    const int c4 = q1 - 3 * step;
    // four independent LDS loads in flight per step
    for (; c < c4; c += 4 * step) {
      const float4 r0 = rec[c], r1 = rec[c + step], r2 = rec[c + 2 * step], r3 = rec[c + 3 * step];
      nh_consider_rec<STRICT>(b, r0, xi, yi, ordi, hi);
      nh_consider_rec<STRICT>(b, r1, xi, yi, ordi, hi);
      nh_consider_rec<STRICT>(b, r2, xi, yi, ordi, hi);
      nh_consider_rec<STRICT>(b, r3, xi, yi, ordi, hi);
    }
    for (; c < q1; c += step) nh_consider_rec<STRICT>(b, rec[c], xi, yi, ordi, hi);
  }
}

template <bool STRICT>
__device__ __forceinline__ void nh_global_scan(const Geom& g, const Arena& a, int64_t ubase, const Window& W, int sub, int step,
                               float xi, float yi, unsigned ordi, unsigned hi, NhBest& b) {
  for (int ty = W.y0; ty <= W.y1; ++ty) {
    const int64_t t = ubase + (int64_t)ty * g.nx;
    const int s0 = a.tile_start[t + W.x0], s1 = a.tile_start[t + W.x1 + 1];
    for (int c = s0 + sub; c < s1; c += step)
      nh_consider<STRICT>(b, dist2(xi, yi, a.xs[c], a.ys[c]), ord_f32(a.rho[c]), (unsigned)a.hs[c], -2 - c, ordi,
                          hi);
  }
}

// `base` is the hit that the packed indices count from: the event's first, but
// for events too large for the word. Returns false, having written nothing, when
// a staged hit's index from there does not fit; the caller then searches the
// region in global memory.
template <bool STRICT>
__device__ __forceinline__ bool nh_staged(const Geom& g, const Arena& a, const RunDesc& d, const Region& R, const RegionLds& L,
                          float4* rec, unsigned short* queue, unsigned char* prow, unsigned short* coreq, int* s_qn,
                          int* s_counts, int ev_first, int base) {
  const int per_row = R.rw + 1;
  const int64_t ubase = (int64_t)R.unit * g.tpl;
  // the region row of every staged position (it gives the staging loads
  // their slots and the winners theirs), and the LDS position of every core
  // query, 16 lanes per row
  for (int k = threadIdx.x; k < 16 * R.rh; k += kWG) {
    const int r = k >> 4;
    const int end = L.row_lo[r + 1];
    for (int p = L.row_lo[r] + (k & 15); p < end; p += 16) prow[p] = (unsigned char)r;
    const int cr = r - R.cy0;
    if (cr >= 0 && cr < R.ch) {
      const int p0 = L.ts[r * per_row + R.cx0];
      const int q1 = L.core_lo[cr + 1];
      for (int q = L.core_lo[cr] + (k & 15); q < q1; q += 16) coreq[q] = (unsigned short)(p0 + q - L.core_lo[cr]);
    }
  }
  __syncthreads();
  // every global load of a lane is issued before its first LDS store
  bool outside = false;  // a hit whose event-local index does not fit the packed word
  for (int p0 = 0; p0 < R.total; p0 += kStagePer * kWG) {
    float4 v[kStagePer];
#pragma unroll
    for (int k = 0; k < kStagePer; ++k) {
      const int p = p0 + (int)threadIdx.x + k * kWG;
      if (p < R.total) {
        const int s = slot_of(L, prow[p], p);
        v[k] = make_float4(a.xs[s], a.ys[s], a.rho[s], __int_as_float(a.hs[s]));
      }
    }
#pragma unroll
    for (int k = 0; k < kStagePer; ++k) {
      const int p = p0 + (int)threadIdx.x + k * kWG;
      if (p < R.total) {
        outside |= (unsigned)(__float_as_int(v[k].w) - base) >= (unsigned)kPackedEventMax;
        rec[p] = make_float4(v[k].x, v[k].y, __uint_as_float(nh_pack(__float_as_int(v[k].w), base, p)),
                             __uint_as_float(ord_f32(v[k].z)));
      }
    }
  }
  if (threadIdx.x == 0) *s_qn = 0;
  // Event ids that decrease (unvalidated input) can leave hits of this unit
  // before its event's first hit; their packed index would wrap. Such a
  // region is searched in global memory, where records carry caller indices.
  if (__syncthreads_or(outside)) return false;
  const int nq = L.core_lo[R.ch];
  // phase 1: radius r1; only hits strictly within r1 can settle a query here
  for (int q = threadIdx.x; q < nq; q += kWG) {
    const int p = coreq[q];
    const int row = prow[p];
    bool done = false;
    if (g.nh_phase1) {
      const float4 me = rec[p];
      const unsigned ordi = __float_as_uint(me.w), zi = __float_as_uint(me.z);
      const Window W = query_window(g, g.win_r1, me.x, me.y);
      const int tx0 = W.x0 - R.rx0, tx1 = W.x1 - R.rx0, ty0 = W.y0 - R.ry0, ty1 = W.y1 - R.ry0;
      if (tx0 >= 0 && ty0 >= 0 && tx1 < R.rw && ty1 < R.rh) {
        NhBest b = nh_start(g.r1sq);
        const unsigned long long k0 = b.k;
        nh_scan_staged<STRICT>(rec, L.ts, per_row, tx0, tx1, ty0, ty1, 0, 1, me.x, me.y, ordi, zi, b);
        nh_unpack(b, k0, base);
        if (b.p >= 0) {
          b.p = slot_of(L, prow[b.p], b.p);
          decide_and_store(g, a, d, s_counts, slot_of(L, row, p), nh_unpack_h(zi, base), ord_inv(ordi), b, ev_first);
          done = true;
        }
      }
    }
    if (!done) queue[atomicAdd(s_qn, 1)] = (unsigned short)p;  // its LDS position
  }
  __syncthreads();
  // phase 2: full d_m window, tpq lanes per query
  const int nu = *s_qn;
  const int tpq = g.tpq;
  const int sub = threadIdx.x & (tpq - 1);
  const int qpp = kWG / tpq;
  for (int q0 = 0; q0 < nu; q0 += qpp) {  // uniform trip count
    const int qi = q0 + threadIdx.x / tpq;
    const bool active = qi < nu;
    NhBest b = nh_start(g.dm2);
    const unsigned long long k0 = b.k;
    int slot = 0;
    unsigned hi = 0, ordi = 0;
    if (active) {
      const int p = queue[qi];
      slot = slot_of(L, prow[p], p);
      const float4 me = rec[p];
      ordi = __float_as_uint(me.w);
      const unsigned zi = __float_as_uint(me.z);
      hi = (unsigned)nh_unpack_h(zi, base);
      const Window W = query_window(g, g.win_dm, me.x, me.y);
      const int tx0 = W.x0 - R.rx0, tx1 = W.x1 - R.rx0, ty0 = W.y0 - R.ry0, ty1 = W.y1 - R.ry0;
      if (tx0 >= 0 && ty0 >= 0 && tx1 < R.rw && ty1 < R.rh) {
        nh_scan_staged<STRICT>(rec, L.ts, per_row, tx0, tx1, ty0, ty1, sub, tpq, me.x, me.y, ordi, zi, b);
      } else {
        // global records carry the caller index itself, and the found slot as -2 - s
        atomicOr(a.err, (uint32_t)E_WINDOW);
        nh_global_scan<STRICT>(g, a, ubase, W, sub, tpq, me.x, me.y, ordi, hi, b);
      }
    }
    nh_reduce(b, tpq);  // the lanes of one query all took the same branch
    nh_unpack(b, k0, base);
    if (active && sub == 0) {
      if (b.p >= 0)
        b.p = slot_of(L, prow[b.p], b.p);
      else if (b.p <= -2)
        b.p = -2 - b.p;
      decide_and_store(g, a, d, s_counts, slot, (int)hi, ord_inv(ordi), b, ev_first);
    }
  }
  return true;
}

template <bool STRICT>
__device__ __forceinline__ void nh_global_region(const Geom& g, const Arena& a, const RunDesc& d, const Region& R,
                                 const RegionLds& L, int* s_counts, int ev_first) {
  const int64_t ubase = (int64_t)R.unit * g.tpl;
  const int nq = L.core_lo[R.ch];
  const int tpq = g.tpq;
  const int sub = threadIdx.x & (tpq - 1);
  const int qpp = kWG / tpq;
  int cr = 0;
  for (int base = 0; base < nq; base += qpp) {
    const int q = base + threadIdx.x / tpq;
    const bool active = q < nq;
    NhBest b = nh_start(g.dm2);
    int slot = 0;
    unsigned hi = 0;
    if (active) {
      int row, p;
      core_query(L, R, q, cr, row, p);
      slot = slot_of(L, row, p);
      const float xi = a.xs[slot], yi = a.ys[slot];
      hi = (unsigned)a.hs[slot];
      const Window W = query_window(g, g.win_dm, xi, yi);
      nh_global_scan<STRICT>(g, a, ubase, W, sub, tpq, xi, yi, ord_f32(a.rho[slot]), hi, b);
    }
    nh_reduce(b, tpq);
    if (active && sub == 0) {
      if (b.p <= -2) b.p = -2 - b.p;
      decide_and_store(g, a, d, s_counts, slot, (int)hi, a.rho[slot], b, ev_first);
    }
  }
}

// The first of a region's hits, or -1 when they span more than the packed index
// word holds; uniform across the workgroup. region_setup's barriers lie between
// two calls.
__device__ __forceinline__ int region_first_hit(const Arena& a, const Region& R, const RegionLds& L) {
  __shared__ int s_first, s_last;
  if (threadIdx.x == 0) {
    s_first = INT_MAX;
    s_last = -1;
  }
  __syncthreads();
  int first = INT_MAX, last = -1;
  for (int r = 0; r < R.rh; ++r)
    for (int p = threadIdx.x; p < L.row_lo[r + 1] - L.row_lo[r]; p += kWG) {
      const int h = a.hs[L.row_gs[r] + p];
      first = min(first, h);
      last = max(last, h);
    }
  atomicMin(&s_first, first);
  atomicMax(&s_last, last);
  __syncthreads();
  const int f = __builtin_amdgcn_readfirstlane(s_first), e = __builtin_amdgcn_readfirstlane(s_last);
  return e - f < kPackedEventMax ? f : -1;
}

template <bool STRICT, bool LARGE>
__device__ __forceinline__ void nh_item(const Geom& g, const Arena& a, const RunDesc& d, int item, RegionLds& L,
                                        float4* rec, unsigned short* queue, unsigned char* prow, unsigned short* coreq,
                                        int* s_qn, int* s_counts, unsigned* s_stack, int& unit) {
  int tx0, ty0, tx1, ty1;
  item_block(g, item, unit, tx0, ty0, tx1, ty1);
  const int e = unit / g.L;
  const int ev_first = event_first_hit(a, d, e);
  // An event too large for the packed index word: the spill kernel searches
  // global memory, where records carry caller indices. In the LARGE instance,
  // regions whose hits span less than the word holds count from their first hit.
  const bool large = event_first_hit(a, d, e + 1) - ev_first > kPackedEventMax;
  BlockWalk B(s_stack, tx1 - tx0 + 1, ty1 - ty0 + 1);
  for (bool more = true; more;) {
    Region R;
    make_region(g, unit, tx0 + B.x0, ty0 + B.y0, tx0 + B.x1, ty0 + B.y1, R);
    region_setup(g, a, R, L);
    if (L.core_lo[R.ch] > 0) {
      bool spill = (!LARGE && large) || (R.total > g.lds_cap && B.single());
      int base = ev_first;
      if constexpr (LARGE) {
        if (R.total <= g.lds_cap) {
          base = region_first_hit(a, R, L);
          spill = base < 0;
        }
      }
      if (spill) {
        spill_region(g, a, R, C_SPILL_NH, kWG);
      } else if (R.total > g.lds_cap) {
        B.split();
        continue;
      } else if (!nh_staged<STRICT>(g, a, d, R, L, rec, queue, prow, coreq, s_qn, s_counts, ev_first, base)) {
        nh_global_region<STRICT>(g, a, d, R, L, s_counts, ev_first);
      }
    }
    more = B.next();
  }
}

// Nearest-higher of the spilled queries, with the decision. A row of region
// tiles is one run of slots; its hits are staged in LDS, and a query's lanes, up
// to 64 as the chunk has few queries, search them there (a search in global
// memory waits for its loads: 100 layers with 1700 hits in 10 cm, nearest-higher
// 1253 -> 499 us).
template <bool G, bool STRICT>
__global__ __launch_bounds__(kWG) void k_nh_spill(DescArg<G> dg, Geom g, Arena a) {
  __shared__ float4 s_rec[kSpillHits];
  __shared__ int s_counts[2];
  g.units = by_units(g, a);
  const RunDesc d = dg.get();
  const int nch = a.counters[C_SPILL_NH];
  const int tid = threadIdx.x;
  for (int i = blockIdx.x; i < nch; i += gridDim.x) {  // uniform per workgroup: the barriers and shuffles below
    if (tid < 2) s_counts[tid] = 0;
    const int64_t t = a.key[i];
    const int first = a.rank[i], nq = min(a.tile_start[t + 1] - first, kWG);
    int tpq = 1;
    while (tpq < 64 && nq * tpq * 2 <= kWG) tpq *= 2;
    const int sub = tid & (tpq - 1), slot = first + tid / tpq;
    const bool active = tid / tpq < nq;
    const int tu = (int)(t % g.tpl);
    const int64_t ubase = t - tu;
    const int ty = tu / g.nx, tx = tu - ty * g.nx;
    const int x0 = max(tx - g.halo, 0), x1 = min(tx + g.halo, g.nx - 1);
    const int y0 = max(ty - g.halo, 0), y1 = min(ty + g.halo, g.ny - 1);
    const int ev_first = event_first_hit(a, d, (int)(t / ((int64_t)g.L * g.tpl)));
    NhBest b = nh_start(g.dm2);
    float xi = 0.0f, yi = 0.0f;
    unsigned hi = 0, ordi = 0;
    bool inside = true;
    if (active) {
      xi = a.xs[slot];
      yi = a.ys[slot];
      hi = (unsigned)a.hs[slot];
      ordi = ord_f32(a.rho[slot]);
      const Window W = query_window(g, g.win_dm, xi, yi);
      inside = W.x0 >= x0 && W.x1 <= x1 && W.y0 >= y0 && W.y1 <= y1;
      if (!inside) nh_global_scan<STRICT>(g, a, ubase, W, sub, tpq, xi, yi, ordi, hi, b);
    }
    for (int y = y0; y <= y1; ++y) {
      const int64_t row = ubase + (int64_t)y * g.nx;
      const int s0 = a.tile_start[row + x0], s1 = a.tile_start[row + x1 + 1];
      for (int c0 = s0; c0 < s1; c0 += kSpillHits) {
        const int m = min(s1 - c0, kSpillHits);
        __syncthreads();  // the previous part has been searched
        for (int p = tid; p < m; p += kWG) {
          const int s = c0 + p;
          s_rec[p] = make_float4(a.xs[s], a.ys[s], __uint_as_float(ord_f32(a.rho[s])), __int_as_float(a.hs[s]));
        }
        __syncthreads();
        if (active && inside)
          for (int p = sub; p < m; p += tpq) {
            const float4 c = s_rec[p];
            nh_consider<STRICT>(b, dist2(xi, yi, c.x, c.y), __float_as_uint(c.z), __float_as_uint(c.w), -2 - (c0 + p),
                                ordi, hi);
          }
      }
    }
    nh_reduce(b, tpq);
    if (active && sub == 0) {
      if (b.p <= -2) b.p = -2 - b.p;
      decide_and_store(g, a, d, s_counts, slot, (int)hi, a.rho[slot], b, ev_first);
    }
    __syncthreads();
    if (g.units && tid < 2 && s_counts[tid]) atomicAdd(&unit_counts(a, d, g)[2 * (int)(t / g.tpl) + tid], s_counts[tid]);
    __syncthreads();  // the counts are read before the next chunk clears them
  }
}

// Built for eight waves per SIMD (64 VGPRs): the compiler then keeps one
// item-level value in scratch, reloaded once per work item, and the kernel
// runs 11% faster than at seven waves.
//
// LARGE is for one event of more hits than the packed index word holds. The regions
// of an event that comes layer by layer span less, and are staged all the same: 2.5M
// hits in 100 layers, 12.2 ms when every region was searched in global memory, 1.23
// when each was spilled, 0.23 now. It is an instance of its own because the same code
// in the others made nearest-higher of other runs 2% slower. The host takes it for
// runs of one event, but for an event of more than 4M hits in a batch, which the
// captured graph runs: that one, and one in a batch of several, is spilled.
template <bool G, bool STRICT, bool LARGE = false>
__global__ __launch_bounds__(kWG, 8) void k_nearest_higher(DescArg<G> dg, Geom g, Arena a) {
  __shared__ int s_counts[2];
  g.units = by_units(g, a);  // read once; the search functions see the answer
  if (threadIdx.x < 2) s_counts[threadIdx.x] = 0;  // barriers follow before the first decision
  const RunDesc d = dg.get();
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int s_rows[kRowMetaInts];
  __shared__ int s_qn;
  __shared__ int s_item;
  __shared__ unsigned s_stack[BlockWalk::kDepth];
  float4* rec = reinterpret_cast<float4*>(smem);
  unsigned short* queue = reinterpret_cast<unsigned short*>(rec + g.lds_cap);
  unsigned short* coreq = queue + g.lds_cap;
  unsigned char* prow = reinterpret_cast<unsigned char*>(coreq + g.lds_cap);
  RegionLds L = region_lds(s_rows, reinterpret_cast<int*>(smem + lds_records_nh(g.lds_cap)), nullptr);
  const int n_items = d.n_events * g.L * g.bpu;
  ItemSched st{0, G ? xcc_id() : 0};
  for (int item; (item = next_item<G>(st, n_items, &a.counters[C_QUEUE_NH], &s_item)) >= 0;)
  {
    int unit;
    nh_item<STRICT, LARGE>(g, a, d, item, L, rec, queue, prow, coreq, &s_qn, s_counts, s_stack, unit);
    if (g.units) {
      __syncthreads();
      if (threadIdx.x < 2) {
        const int c = s_counts[threadIdx.x];
        s_counts[threadIdx.x] = 0;
        if (c) atomicAdd(&unit_counts(a, d, g)[2 * unit + (int)threadIdx.x], c);
      }
    }
  }
}

template <bool G>
__global__ __launch_bounds__(kWG) void k_label(DescArg<G> dg, Geom g, Arena a) {
  constexpr int U = G ? kBatchU : kPlaceU;
  __shared__ LabelChunk<kWG * U> S;
  const RunDesc d = dg.get();
  for (ChunkRun r = xcd_run(d.n, stream_chunk(G)); r.c < r.end; r.c += r.step) label_chunk<kWG, U>(d, g, a, r.c * stream_chunk(G), d.n, S);
}

// ---------------------------------------------------------------------------
// Labels by k-way expansion (Sec. 2.2, Algorithm 3): one thread per seed walks
// the seed's follower tree depth first and gives every hit in it the seed's
// cluster id. The walk keeps no stack: each follower's owner and its position
// in the owner's list (key / rank, free after the grid build) lead back up to
// the next unvisited sibling, so a thread holds O(1) state whatever the tree's
// depth.
// ---------------------------------------------------------------------------

// Part 1: places follower-list entries (as k_label does), records owner and
// position per follower, labels seeds with their number within the event and
// every other hit -1, and lists the seeds by rank.
template <bool G>
__global__ __launch_bounds__(kWG) void k_expand_init(DescArg<G> dg, Geom g, Arena a) {
  const RunDesc d = dg.get();
  int* const seeds = reinterpret_cast<int*>(a.xs);
  constexpr int U = kPlaceU;
  for (ChunkRun rn = xcd_run(d.n, kWG * U); rn.c < rn.end; rn.c += rn.step) {
    const int sb = rn.c * kWG * U + (int)threadIdx.x;
    int p[U], h[U];
    unsigned f[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int s = sb + j * kWG;
      f[j] = 0;
      p[j] = 0;
      h[j] = 0;
      if (s < d.n) {
        f[j] = a.flags[s] | 0x100u;
        p[j] = a.parent[s];
        h[j] = a.hs[s];
      }
    }
#pragma unroll
    for (int j = 0; j < U; ++j) {
      if (!(f[j] & 0x100u)) continue;
      const int s = sb + j * kWG;
      int lab = -1;
      if (f[j] & F_FOLLOWER) {
        const int owner = a.hs[p[j]];
        const int r = a.frank[s];
        a.flist[a.fstart[owner] + r] = h[j];
        a.key[h[j]] = owner;
        a.rank[h[j]] = r;
      } else if (f[j] & F_SEED) {
        const int e = d.event ? clampi(d.event[h[j]] - d.event_base, 0, d.n_events - 1) : 0;
        const int rk = seed_rank(a, h[j]);
        lab = rk - seed_rank(a, event_first_hit(a, d, e));
        seeds[rk] = h[j];
      }
      d.cluster_id[h[j]] = lab;
    }
  }
}

// Part 2: the walks. Each visits its tree in preorder: down to a node's first
// follower, else up through owners to the first one with a next sibling. A
// walk takes at most 2 (n + 1) steps (each edge down once and up once); a walk
// that reached that bound would mean corrupt lists, so it stops and flags the
// run instead of looping.
template <bool G>
__global__ __launch_bounds__(kWG) void k_expand_dfs(DescArg<G> dg, Geom g, Arena a) {
  const RunDesc d = dg.get();
  const int* const seeds = reinterpret_cast<const int*>(a.xs);
  const int ns = seed_rank(a, d.n);
  const int64_t max_steps = 2 * ((int64_t)d.n + 1);
  for (int t = blockIdx.x * kWG + (int)threadIdx.x; t < ns; t += gridDim.x * kWG) {
    const int root = seeds[t];
    const int lab = d.cluster_id[root];
    int u = root;
    int b = a.fstart[u], e = a.fstart[u + 1];
    int64_t steps = 0;
    for (;;) {
      if (++steps > max_steps) {
        atomicOr(a.err, (uint32_t)E_WALK);
        break;
      }
      if (b < e) {
        u = a.flist[b];  // first follower
      } else {
        // climb to the nearest node (u or an ancestor) that has a next sibling
        bool found = false;
        while (u != root && steps <= max_steps) {
          ++steps;
          const int p = a.key[u];
          const int nx = a.fstart[p] + a.rank[u] + 1;
          if (nx < a.fstart[p + 1]) {
            u = a.flist[nx];
            found = true;
            break;
          }
          u = p;
        }
        if (!found) break;
      }
      d.cluster_id[u] = lab;
      b = a.fstart[u];
      e = a.fstart[u + 1];
    }
  }
}

// Follower lists: sort each list by hit index. k_label writes event-local
// entries, so lists of one entry are already final; after the depth-first
// expansion (which walks caller indices) every entry is made event-local
// here. Lists of up to kShortList entries are sorted in registers (odd-even
// transposition networks of four entries, when every list of the wave fits,
// or eight); longer ones by insertion in place.
constexpr int kShortList = 8;

template <bool G>
__device__ __forceinline__ void follow_sort_chunk(const RunDesc& d, const Geom& g, const Arena& a, int chunk) {
  constexpr int U = kPlaceU;
  const int hb = chunk * kWG * U + (int)threadIdx.x;
  int b[U], end[U];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int h = hb + j * kWG;
    b[j] = 0;
    end[j] = 0;
    if (h < d.n) {
      b[j] = a.fstart[h];
      end[j] = a.fstart[h + 1];
    }
  }
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int len = end[j] - b[j];
    // nearly every wave holds only lists of up to four entries: then the
    // whole wave takes the shorter network (a wave-uniform choice)
    const bool four = __all(len <= 4);
    if (len < (g.expand ? 1 : 2)) continue;
    int off = 0;
    if (g.expand) {
      const int h = hb + j * kWG;
      off = event_first_hit(a, d, d.event ? clampi(d.event[h] - d.event_base, 0, d.n_events - 1) : 0);
    }
    if (four) {
      int v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = i < len ? a.flist[b[j] + i] : INT_MAX;
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int i = r & 1; i + 1 < 4; i += 2) {
          const int lo = min(v[i], v[i + 1]), hi = max(v[i], v[i + 1]);
          v[i] = lo;
          v[i + 1] = hi;
        }
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (i < len) a.flist[b[j] + i] = v[i] - off;
      continue;
    }
    if (len <= kShortList) {
      int v[kShortList];
#pragma unroll
      for (int i = 0; i < kShortList; ++i) v[i] = i < len ? a.flist[b[j] + i] : INT_MAX;
#pragma unroll
      for (int r = 0; r < kShortList; ++r)
#pragma unroll
        for (int i = r & 1; i + 1 < kShortList; i += 2) {
          const int lo = min(v[i], v[i + 1]), hi = max(v[i], v[i + 1]);
          v[i] = lo;
          v[i + 1] = hi;
        }
#pragma unroll
      for (int i = 0; i < kShortList; ++i)
        if (i < len) a.flist[b[j] + i] = v[i] - off;
      continue;
    }
    for (int i = b[j] + 1; i < end[j]; ++i) {
      const int v = a.flist[i];
      int k = i - 1;
      while (k >= b[j] && a.flist[k] > v) {
        a.flist[k + 1] = a.flist[k];
        --k;
      }
      a.flist[k + 1] = v;
    }
    for (int i = b[j]; i < end[j]; ++i) a.flist[i] -= off;
  }
}

template <bool G>
__global__ __launch_bounds__(kWG) void k_follow_sort(DescArg<G> dg, Geom g, Arena a) {
  if (by_units(g, a)) return;  // done unit by unit
  const RunDesc d = dg.get();
  for (ChunkRun r = xcd_run(d.n, kHistChunk); r.c < r.end; r.c += r.step) follow_sort_chunk<G>(d, g, a, r.c);
}

// ---------------------------------------------------------------------------
// Input validation (CLUE_VALIDATE).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kWG) void k_validate(RunDesc d, int L, uint32_t* err) {
  const int stride = gridDim.x * kWG;
  bool bad = false;
  for (int h = blockIdx.x * kWG + threadIdx.x; h < d.n; h += stride) {
    bad |= !isfinite(d.x[h]) || !isfinite(d.y[h]) || !isfinite(d.e[h]);
    bad |= d.layer[h] < 0 || d.layer[h] >= L;
    if (d.event) {
      bad |= d.event[h] < d.event_base || d.event[h] - d.event_base >= d.n_events;
      if (h > 0) bad |= d.event[h] < d.event[h - 1];
    }
  }
  if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(err, (uint32_t)E_INPUT);
}

// Copies a run's arrays out, one row of workgroups each. Sixteen bytes a lane
// where the destination is aligned for it, as the sources are; bound by the
// launch below about a million hits, by memory above.
__global__ __launch_bounds__(kWG) void k_read_out(ReadOut r) {
  const int k = blockIdx.y;
  const int64_t first = (int64_t)blockIdx.x * kWG + threadIdx.x, step = (int64_t)gridDim.x * kWG, n = r.n[k];
  if (k == 0 && first == 0 && r.word_out) *r.word_out = *r.word;
  const uint32_t* const src = (const uint32_t*)r.src[k];
  uint32_t* const dst = (uint32_t*)r.dst[k];
  if (!dst) return;
  int64_t done = 0;
  if (((uintptr_t)src | (uintptr_t)dst) % 16 == 0) {
    done = n & ~(int64_t)3;
    for (int64_t i = first; i < n / 4; i += step) ((uint4*)dst)[i] = ((const uint4*)src)[i];
  }
  for (int64_t i = done + first; i < n; i += step) dst[i] = src[i];
}

// Event ids of a chunk of the host-resident form, for up to kIdEvents events a
// launch, whose first hits travel in the kernel's arguments. Bound by its
// stores (4 bytes a hit), which overlap the next chunk's copy.
constexpr int kIdEvents = 128;
struct EventStarts {
  int32_t start[kIdEvents + 1];
};
__global__ __launch_bounds__(kWG) void k_event_ids(int32_t* ids, EventStarts s, int32_t first, int events) {
  __shared__ int32_t st[kIdEvents + 1];
  for (int i = threadIdx.x; i <= events; i += kWG) st[i] = s.start[i];
  __syncthreads();
  for (int h = st[0] + blockIdx.x * kWG + threadIdx.x; h < st[events]; h += gridDim.x * kWG) {
    int lo = 0, hi = events - 1;  // the last event that starts at or before h
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (st[mid] <= h)
        lo = mid;
      else
        hi = mid - 1;
    }
    ids[h] = first + lo;
  }
}

__global__ void k_set_desc(RunDesc d, RunDesc* dd) {
  if (threadIdx.x == 0) *dd = d;
}

// ---------------------------------------------------------------------------
// Host launches.
// ---------------------------------------------------------------------------
// Dynamic LDS of the density kernel: per staged hit 16 bytes of record and
// hit index, a 16-bit tile id and four 16-bit quad-list entries, then the
// region's tile offsets and quad-list offsets.
int lds_bytes_for(const Geom& g) { return lds_records_density(g.lds_cap) + 4 * (g.ts_ints + g.q_ints); }
// Nearest-higher: per staged hit a float4 record, a 16-bit queue entry, a
// 16-bit core-query position and its region row (a byte), then the region's
// tile offsets.
int lds_bytes_nh(const Geom& g) { return lds_records_nh(g.lds_cap) + 4 * g.ts_ints; }

static inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

template <bool G>
static hipError_t launch_all(const Geom& g, const Arena& a, DescArg<G> dg, const RunDesc& host_d,
                             const LaunchCfg& cfg, hipStream_t s, hipEvent_t* ev) {
  // Grid sizes: plain launches are sized to the run; graph launches use
  // persistent grids (sizes are read from the descriptor on the device).
  const int64_t n = host_d.n;
  const int64_t tt = (int64_t)host_d.n_events * g.L * g.tpl + 1;
  const int64_t items = (int64_t)host_d.n_events * g.L * g.bpu;
  // streaming grids are a multiple of kQueues (one run of chunks per XCD)
  auto stream_grid = [&](int64_t work) {
    if (G) return cfg.persist_blocks_stream;
    const int64_t b = std::max<int64_t>(1, std::min<int64_t>(cdiv(work, kWG), 1 << 20));
    return (int)((b + kQueues - 1) / kQueues * kQueues);
  };
  const int g_clear = G ? cfg.persist_blocks_stream
                        : (int)std::max<int64_t>(1, std::min<int64_t>(cdiv(std::max(tt, n + 1), kWG), 1 << 16));
  const int g_rho = G ? cfg.persist_blocks_rho : (int)std::max<int64_t>(1, items);
  const int g_nh = G ? cfg.persist_blocks_nh : (int)std::max<int64_t>(1, items);
  const int g_scan_t = G ? cfg.persist_blocks_scan : cdiv(tt, kScanChunk);
  // spill kernels: four workgroups per CU in single launches (an empty queue
  // costs one counter read per workgroup)
  const int g_spill = G ? cfg.persist_blocks_stream : 1024;
  const int g_scan_s = G ? cfg.persist_blocks_scan : cdiv(n + 1, kScanChunk);
  const bool fol = !(g.flags & 8u);
  int k = 0;
  auto mark = [&]() {
    if (ev) (void)hipEventRecord(ev[k++], s);
  };
  mark();
  if (g.units)
    launch_units<G>(g, a, dg, host_d, s);
  else
    k_clear<G><<<g_clear, kWG, 0, s>>>(dg, g, a);
  mark();
  if (g.units)
    launch_unit_sort<G>(g, a, dg, host_d, s);  // or the histogram
  else
    k_hist<G><<<stream_grid(cdiv(n, kPlaceU)), kWG, 0, s>>>(dg, g, a);
  mark();
  k_scan<G, SCAN_TILES><<<g_scan_t, kWG, 0, s>>>(dg, g, a);
  mark();
  k_scatter<G><<<G ? cfg.persist_blocks_scatter : stream_grid(cdiv(n, kPlaceU)), kWG, 0, s>>>(dg, g, a);
  mark();
  k_place<G><<<stream_grid(cdiv(n, G ? kBatchU : kPlaceU)), kWG, 0, s>>>(dg, g, a);
  mark();
  const int lds = lds_bytes_for(g);
  if (g.kernel == 0) {
    if (g.maxl == 2)
      k_density<G, 2, 0><<<g_rho, kWG, lds, s>>>(dg, g, a);
    else
      k_density<G, 3, 0><<<g_rho, kWG, lds, s>>>(dg, g, a);
    k_density_spill<G, 0><<<g_spill, kWG, 0, s>>>(dg, g, a);
  } else if (g.kernel == 1) {
    if (g.maxl == 2)
      k_density<G, 2, 1><<<g_rho, kWG, lds, s>>>(dg, g, a);
    else
      k_density<G, 3, 1><<<g_rho, kWG, lds, s>>>(dg, g, a);
    k_density_spill<G, 1><<<g_spill, kWG, 0, s>>>(dg, g, a);
  } else {
    if (g.maxl == 2)
      k_density<G, 2, 2><<<g_rho, kWG, lds, s>>>(dg, g, a);
    else
      k_density<G, 3, 2><<<g_rho, kWG, lds, s>>>(dg, g, a);
    k_density_spill<G, 2><<<g_spill, kWG, 0, s>>>(dg, g, a);
  }
  mark();
  const int lds_nh = lds_bytes_nh(g);
  const bool large = !G && host_d.n_events == 1 && n > kPackedEventMax;
  if (g.flags & 4u) {
    if (large)
      k_nearest_higher<false, true, true><<<g_nh, kWG, lds_nh, s>>>(DescArg<false>{host_d}, g, a);
    else
      k_nearest_higher<G, true><<<g_nh, kWG, lds_nh, s>>>(dg, g, a);
    k_nh_spill<G, true><<<g_spill, kWG, 0, s>>>(dg, g, a);
  } else {
    if (large)
      k_nearest_higher<false, false, true><<<g_nh, kWG, lds_nh, s>>>(DescArg<false>{host_d}, g, a);
    else
      k_nearest_higher<G, false><<<g_nh, kWG, lds_nh, s>>>(dg, g, a);
    k_nh_spill<G, false><<<g_spill, kWG, 0, s>>>(dg, g, a);
  }
  mark();
  if (builds_lists(g))
    k_scan<G, SCAN_SEEDS_FOLLOW><<<g_scan_s, kWG, 0, s>>>(dg, g, a);
  else
    k_scan<G, SCAN_SEEDS><<<g_scan_s, kWG, 0, s>>>(dg, g, a);
  mark();
  if (g.units) {
    launch_unit_finish<G>(g, a, dg, host_d, s);  // or the labels
  } else if (g.expand) {
    k_expand_init<G><<<stream_grid(cdiv(n, kPlaceU)), kWG, 0, s>>>(dg, g, a);
    const int g_dfs = G ? cfg.persist_blocks_stream : std::min(stream_grid(n), std::max(1, cfg.persist_blocks_stream));
    k_expand_dfs<G><<<g_dfs, kWG, 0, s>>>(dg, g, a);
  } else {
    k_label<G><<<stream_grid(cdiv(n, G ? kBatchU : kPlaceU)), kWG, 0, s>>>(dg, g, a);
  }
  mark();
  if (fol) k_follow_sort<G><<<stream_grid(cdiv(n, kPlaceU)), kWG, 0, s>>>(dg, g, a);
  mark();
  return hipGetLastError();
}

hipError_t launch_pipeline(const Geom& g, const Arena& a, const RunDesc& d, const LaunchCfg& cfg, hipStream_t s,
                           hipEvent_t* ev) {
  if (cfg.graph_mode) {
    DescArg<true> dg{a.desc};
    return launch_all<true>(g, a, dg, d, cfg, s, ev);
  }
  DescArg<false> dg{d};
  return launch_all<false>(g, a, dg, d, cfg, s, ev);
}

hipError_t launch_set_desc(const RunDesc& d, RunDesc* dd, hipStream_t s) {
  k_set_desc<<<1, 64, 0, s>>>(d, dd);
  return hipGetLastError();
}

hipError_t launch_read_out(const ReadOut& r, hipStream_t s) {
  int64_t most = 1;
  for (int k = 0; k < 3; ++k)
    if (r.dst[k]) most = std::max(most, r.n[k]);
  const dim3 grid((unsigned)std::min<int64_t>(cdiv(cdiv(most, 4), kWG), 2048), r.src[2] ? 3 : 2);
  k_read_out<<<grid, kWG, 0, s>>>(r);
  return hipGetLastError();
}

hipError_t launch_event_ids(int32_t* ids, const int64_t* start, int32_t first, int32_t events, hipStream_t s) {
  for (int32_t e = 0; e < events; e += kIdEvents) {
    const int ne = std::min(events - e, kIdEvents);
    EventStarts st;
    for (int i = 0; i <= ne; ++i) st.start[i] = (int32_t)(start[e + i] - start[0]);
    const int64_t n = st.start[ne] - st.start[0];
    if (n == 0) continue;
    const int grid = (int)std::min<int64_t>(cdiv(n, kWG), 1024);
    k_event_ids<<<grid, kWG, 0, s>>>(ids, st, first + e, ne);
  }
  return hipGetLastError();
}

hipError_t launch_validate(const Geom& g, const Arena& a, const RunDesc& d, hipStream_t s) {
  const int grid = (int)std::max<int64_t>(1, std::min<int64_t>(cdiv(d.n, kWG), 4096));
  k_validate<<<grid, kWG, 0, s>>>(d, g.L, a.err);
  return hipGetLastError();
}

int occupancy_blocks_per_cu(int which, int lds_bytes) {
  int nb = 0;
  hipError_t e = hipSuccess;
  switch (which) {
    case 0: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_hist<true>, kWG, 0); break;
    case 1: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_density<true, 2, 0>, kWG, lds_bytes); break;
    case 2: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_scan<true, SCAN_SEEDS_FOLLOW>, kWG, 0); break;
    case 3: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_nearest_higher<true, false>, kWG, lds_bytes); break;
    default: break;
  }
  if (e != hipSuccess || nb < 1) nb = 1;
  return nb;
}

}  // namespace clue
