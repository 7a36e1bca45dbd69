// Device helpers shared by the tiled kernels and the all-pairs kernels.
//
// Every float operation that decides a result is an explicit round-to-nearest
// intrinsic (no contraction), so results match a plain IEEE binary32
// evaluation of the same expressions.
#pragma once

#include "clue_internal.h"

namespace clue {

// ---------------------------------------------------------------------------
// Run descriptor: by value (plain launches) or from device memory (graph).
// ---------------------------------------------------------------------------
template <bool G>
struct DescArg;
template <>
struct DescArg<false> {
  RunDesc d;
  __device__ __forceinline__ RunDesc get() const { return d; }
};
template <>
struct DescArg<true> {
  const RunDesc* p;
  __device__ __forceinline__ RunDesc get() const { return *p; }
};

// Tile coordinate of a position: floor((v - origin) / T) clamped to the grid.
// Monotone non-decreasing in v, which is what makes the query windows below
// supersets of the true neighbourhoods.
__device__ __forceinline__ int tile_coord(float v, float origin, float inv_t, int n) {
  float t = floorf(__fmul_rn(__fsub_rn(v, origin), inv_t));
  t = fminf(fmaxf(t, 0.0f), (float)(n - 1));
  return (int)t;
}

__device__ __forceinline__ float dist2(float xi, float yi, float xj, float yj) {
  float dx = __fsub_rn(xi, xj);
  float dy = __fsub_rn(yi, yj);
  return __fadd_rn(__fmul_rn(dx, dx), __fmul_rn(dy, dy));
}

__device__ __forceinline__ int ld_relaxed(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_relaxed(int32_t* p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

__device__ __forceinline__ int wave_incl_scan(int v, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int t = __shfl_up(v, o, 64);
    if (lane >= o) v += t;
  }
  return v;
}
// Exclusive sum over a workgroup of T lanes, and the total. `tid` is the lane's
// thread id; s_part holds T / 64 words.
template <int T>
__device__ __forceinline__ int wg_excl(int v, int* s_part, int& total, int tid) {
  const int lane = tid & 63, wave = tid >> 6;
  const int incl = wave_incl_scan(v, lane);
  __syncthreads();
  if (lane == 63) s_part[wave] = incl;
  __syncthreads();
  int base = 0, all = 0;
#pragma unroll
  for (int w = 0; w < T / 64; ++w) {
    const int s = s_part[w];
    base += w < wave ? s : 0;
    all += s;
  }
  total = all;
  return base + incl - v;
}
__device__ __forceinline__ int wave_sum(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Order-preserving map of a float to uint32 (-0 folds onto +0), so that
// (rho, index) compares as one 64-bit unsigned key.
__device__ __forceinline__ unsigned ord_f32(float v) {
  const unsigned u = __float_as_uint(__fadd_rn(v, 0.0f));
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
// Inverse of ord_f32 (gives +0 for a folded -0, which compares the same).
__device__ __forceinline__ float ord_inv(unsigned o) {
  return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}

// First caller-order hit of event e, clamped to [0, n] (memory safety for
// unvalidated event ids).
__device__ __forceinline__ int event_first_hit(const Arena& a, const RunDesc& d, int e) {
  return clampi(a.ev_start[e], 0, d.n);
}

// Seeds are marked by one bit per hit in caller order; the seed scan gives
// the count before each 32-bit word. Words cover hits 0..n, so the rank of
// n (the seed total) is defined too.
__host__ __device__ __forceinline__ int64_t seed_words(int64_t n) { return n / 32 + 1; }
// ---------------------------------------------------------------------------
// Streaming kernels cut their index range into chunks of `chunk` consecutive
// indices and give each XCD one contiguous run of chunks (workgroups are
// dispatched to the XCDs round-robin by id; the grid is a multiple of
// kQueues). Neighbouring indices share lines in the gathers and scattered
// writes that follow, so they are fetched into, and completed in, one L2.
// ---------------------------------------------------------------------------
struct ChunkRun {
  int c, end, step;
};
__device__ __forceinline__ ChunkRun xcd_run(int n, int chunk) {
  const int nch = (int)(((int64_t)n + chunk - 1) / chunk);
  const int x = (int)blockIdx.x % kQueues, i = (int)blockIdx.x / kQueues;
  return {(int)((int64_t)nch * x / kQueues) + i, (int)((int64_t)nch * (x + 1) / kQueues),
          (int)gridDim.x / kQueues};
}

// Bits of a staged nearest-higher record's index word that hold its LDS position;
// the others hold the event-local index.
constexpr int kPosBits = 11;
constexpr unsigned kPosMask = (1u << kPosBits) - 1u;
constexpr int kPackedEventMax = 1 << (32 - kPosBits);  // hits per event
static_assert(kMaxLdsCap <= (1 << kPosBits), "an LDS position must fit the packed index word");

// Seeds among caller hits 0..h-1 (h in [0, n]).
__device__ __forceinline__ int seed_rank(const Arena& a, int h) {
  return a.seed_wrank[h >> 5] + __popc(a.seedbits[h >> 5] & ((1u << (h & 31)) - 1u));
}

// Event of tile-CSR slot s: slots are ordered by (event, layer, tile), so the
// event is the last e whose first tile starts at or before s.
__device__ __forceinline__ int event_of_slot(const Geom& g, const Arena& a, const RunDesc& d, int s) {
  const int64_t per = (int64_t)g.L * g.tpl;
  int lo = 0, hi = d.n_events - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.tile_start[mid * per] <= s)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// ---------------------------------------------------------------------------
// The unit path's arrays. They lie in buffers that the path leaves free while it
// needs them, so they take no memory of their own; unit_space says whether a run
// has the room.
//   key   [n - U - 1, n)  first hit of each of the U units, and n
//   rank  [n - 2 U, n)    seeds and followers of each unit
//   rho   [0, units)      each k_units workgroup's verdict
// The key and rank buffers hold the spill queues at their beginnings. A spilled
// tile's own region (at most 2 halo + 1 tiles a side) holds more than lds_cap hits
// and a hit lies in at most as many regions, which bounds the tiles; each has one
// chunk more than its hits fill.
// Every workgroup of k_unit_sort reads the verdict for itself, the last perhaps
// after the first have finished, so it must lie where that launch writes nothing:
// the unit path writes tile_start and the slots' x, y, energy and hit, the general
// path key, rank, tile_start, event starts and what clear_lists clears. (The unit
// starts are read by the unit path alone, which does not write key.) The rho buffer
// is free until the launches after it: k_scatter's pairs, the density.
__host__ __device__ __forceinline__ bool unit_space(const Geom& g, const RunDesc& d) {
  const int64_t n = d.n, U = (int64_t)d.n_events * g.L, side = 2 * g.halo + 1;
  const int64_t spill = n * side * side / g.lds_cap + n / kWG + 1;
  return spill + 2 * U + 1 <= n && g.units <= n && (int64_t)g.L * kUnitMax <= (int64_t)kPackedEventMax &&
         unit_sizes(g, n, U);
}
__host__ __device__ __forceinline__ int32_t* unit_starts(const Arena& a, const RunDesc& d, const Geom& g) {
  return a.key + ((int64_t)d.n - (int64_t)d.n_events * g.L - 1);
}
__host__ __device__ __forceinline__ int32_t* unit_counts(const Arena& a, const RunDesc& d, const Geom& g) {
  return a.rank + ((int64_t)d.n - 2 * (int64_t)d.n_events * g.L);
}
__host__ __device__ __forceinline__ int32_t* unit_flags(const Arena& a) { return reinterpret_cast<int32_t*>(a.rho); }
// This run takes the unit path (uniform; valid after k_unit_sort).
__device__ __forceinline__ bool by_units(const Geom& g, const Arena& a) { return g.units && a.counters[C_UNITS]; }

// Clears the tile counts and event starts, which the general path's histogram
// reads and writes, and what its later stages read before they write.
__device__ __forceinline__ void clear_grid(const RunDesc& d, const Geom& g, const Arena& a, int64_t i0,
                                           int64_t stride) {
  const int64_t tt = (int64_t)d.n_events * g.L * g.tpl + 1;
  for (int64_t i = i0; i < tt; i += stride) a.tile_start[i] = 0;
  for (int64_t i = i0; i <= d.n_events; i += stride) a.ev_start[i] = 0;
}
__device__ __forceinline__ void clear_lists(const RunDesc& d, const Geom& g, const Arena& a, int64_t i0,
                                            int64_t stride) {
  const int64_t tt = (int64_t)d.n_events * g.L * g.tpl + 1;
  const int64_t n1 = (int64_t)d.n + 1;
  if (builds_lists(g))
    for (int64_t i = i0; i < n1; i += stride) a.fstart[i] = 0;
  constexpr int64_t SC = kScanChunk;  // the smaller chunk of the two forms
  const int64_t nchunk_t = (tt + SC - 1) / SC;
  const int64_t nchunk_s = (n1 + SC - 1) / SC;
  for (int64_t i = i0; i < nchunk_t && i < a.cap_chunks; i += stride) a.scan_status[i] = 0ull;
  for (int64_t i = i0; i < nchunk_s && i < a.cap_chunks; i += stride) a.scan_status[a.cap_chunks + i] = 0ull;
  for (int64_t i = i0; i < seed_words(d.n); i += stride) a.seedbits[i] = 0u;
}

template <bool G>
void launch_units(const Geom& g, const Arena& a, DescArg<G> dg, const RunDesc& d, hipStream_t s);
template <bool G>
void launch_unit_sort(const Geom& g, const Arena& a, DescArg<G> dg, const RunDesc& d, hipStream_t s);
template <bool G>
void launch_unit_finish(const Geom& g, const Arena& a, DescArg<G> dg, const RunDesc& d, hipStream_t s);

// Hits of a chunk of k_hist and k_follow_sort, and of the other streaming kernels.
constexpr int kHistChunk = kWG * kPlaceU;
__host__ __device__ constexpr int stream_chunk(bool graph) { return kWG * (graph ? kBatchU : kPlaceU); }

// ---------------------------------------------------------------------------
// k_hist: tile of every hit, atomic count per tile, arrival rank kept.
// Lanes of a wave that share a tile are grouped first, so each distinct tile
// costs one atomic per wave (hits of a cluster tend to be adjacent in input
// order); ranks within a group follow lane order. Each lane takes U
// hits per step so that their atomics are in flight together. `tid` counts the
// kWG lanes that share the chunk [h0, end), of at most kWG U hits.
// ---------------------------------------------------------------------------
template <int U>  // sub-batches per step; their atomics overlap
__device__ __forceinline__ void hist_chunk(const RunDesc& d, const Geom& g, const Arena& a, int h0, int end, int tid) {
  const int lane = tid & 63;
  // every load of a lane is issued before its first store (the event
  // starts below could alias the inputs as far as the compiler knows)
  int t[U], ev[U], evp[U];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int h = h0 + j * kWG + tid;
    t[j] = -1;
    ev[j] = evp[j] = 0;
    if (h < end) {
      if (d.event) {
        ev[j] = clampi(d.event[h] - d.event_base, 0, d.n_events - 1);
        evp[j] = h == 0 ? -1 : clampi(d.event[h - 1] - d.event_base, 0, d.n_events - 1);
      }
      const int l = clampi(d.layer[h], 0, g.L - 1);
      const int tx = tile_coord(d.x[h], g.x0, g.inv_t, g.nx);
      const int ty = tile_coord(d.y[h], g.y0, g.inv_t, g.ny);
      t[j] = l * g.tpl + ty * g.nx + tx;  // the event's part is added below
    }
  }
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int h = h0 + j * kWG + tid;
    if (h >= end) continue;
    const int e = ev[j];
    t[j] += e * g.L * g.tpl;
    if (d.event) {
      for (int k = evp[j] + 1; k <= e; ++k) a.ev_start[k] = h;
      if (h == d.n - 1)
        for (int k = e + 1; k <= d.n_events; ++k) a.ev_start[k] = d.n;
    } else if (h == 0) {
      a.ev_start[0] = 0;
      a.ev_start[1] = d.n;
    }
  }
  int base[U], off[U], leader[U];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const bool valid = t[j] >= 0;
    unsigned long long todo = __ballot(valid);
    int ld = lane, o = 0, cnt = 0;
    while (todo) {  // wave-uniform: one pass per distinct tile in the wave
      // the lowest unmatched lane leads; its tile is read into a scalar
      // register, and a lane's offset is the count of its peers below it
      const int l = __ffsll((long long)todo) - 1;
      const int lt = __builtin_amdgcn_readlane(t[j], l);
      const bool mine = t[j] == lt;  // invalid lanes (-1) never match a tile
      const unsigned long long peers = __ballot(mine);
      if (mine) {
        ld = l;
        o = __builtin_amdgcn_mbcnt_hi((unsigned)(peers >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)peers, 0u));
        cnt = __popcll(peers);
      }
      todo &= ~peers;
    }
    base[j] = 0;
    if (valid && lane == ld) base[j] = atomicAdd(&a.tile_start[t[j]], cnt);
    off[j] = o;
    leader[j] = ld;
  }
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int bs = __shfl(base[j], leader[j], 64);
    const int h = h0 + j * kWG + tid;
    if (t[j] >= 0) {
      a.key[h] = t[j];
      a.rank[h] = bs + off[j];
    }
  }
}

// ---------------------------------------------------------------------------
// Labels: follow the follower -> nearest-higher links to the root (pointer
// jumping with path compression; concurrent updates only ever store an
// ancestor, so every read is an ancestor and every chase ends at the root).
// A root that is a seed gives its seed number within the event; any other
// root (outlier, orphan) gives -1. Also places follower-list entries.
// ---------------------------------------------------------------------------
// The chunk is the slots [c0, end), the first T U of them.
template <int C>
struct LabelChunk {
  int par[C], hs[C];
  unsigned char fl[C];
  int ev[2];  // the chunk's event when it holds one event (else -1), its first hit
};
template <int T, int U>  // lanes, and hits per lane, whose chases are interleaved
__device__ __forceinline__ void label_chunk(const RunDesc& d, const Geom& g, const Arena& a, int c0, int end,
                                            LabelChunk<T * U>& S) {
  const bool fol = builds_lists(g);
  constexpr int C = T * U;  // slots per chunk
  const int tid = threadIdx.x;
  // the chunk's parent, caller index and flags, staged in LDS: a nearest-higher
  // lies within d_m, so most links stay inside the chunk. A staged parent may
  // be older than a compression stored since; it is still an ancestor.
  int* const s_par = S.par;
  int* const s_hs = S.hs;
  unsigned char* const s_fl = S.fl;
  int* const s_ev = S.ev;
  if (tid == 0) {
    const int e0 = event_of_slot(g, a, d, c0);
    const int e1 = event_of_slot(g, a, d, min(c0 + C, end) - 1);
    s_ev[0] = e0 == e1 ? e0 : -1;
    s_ev[1] = event_first_hit(a, d, e0);
  }
  const int sb = c0 + tid;
  int s[U], p0[U], hsj[U], r[U], p[U];
  unsigned f[U];
  bool v[U];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    s[j] = sb + j * T;
    v[j] = s[j] < end;
    p0[j] = s[j];
    hsj[j] = 0;
    f[j] = 0;
    if (v[j]) {
      p0[j] = a.parent[s[j]];
      f[j] = a.flags[s[j]];
      hsj[j] = a.hs[s[j]];
    }
    s_par[s[j] - c0] = p0[j];
    s_hs[s[j] - c0] = hsj[j];
    s_fl[s[j] - c0] = (unsigned char)f[j];
  }
  __syncthreads();
  const unsigned held = (unsigned)max(min(end - c0, C), 0);
  auto staged = [&](int x) { return (unsigned)(x - c0) < held; };
  // first hit of each hit's event, from its slot
  const int ev1 = s_ev[0], first1 = s_ev[1];
  int first[U];
#pragma unroll
  for (int j = 0; j < U; ++j)
    first[j] = ev1 >= 0 || !v[j] ? first1 : event_first_hit(a, d, event_of_slot(g, a, d, s[j]));
  if (fol) {
    // entries are event-local already: the list sort then leaves lists of
    // one entry alone. Every load of a lane comes before its first store
    // (the stores could alias them as far as the compiler knows).
    int at[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      at[j] = -1;
      if (v[j] && (f[j] & F_FOLLOWER)) {
        const int owner = staged(p0[j]) ? s_hs[p0[j] - c0] : a.hs[p0[j]];
        at[j] = a.fstart[owner] + a.frank[s[j]];
      }
    }
#pragma unroll
    for (int j = 0; j < U; ++j)
      if (at[j] >= 0) a.flist[at[j]] = hsj[j] - first[j];
  }
#pragma unroll
  for (int j = 0; j < U; ++j) {
    r[j] = s[j];
    p[j] = p0[j];
  }
  for (;;) {
    bool more = false;
#pragma unroll
    for (int j = 0; j < U; ++j) {
      if (p[j] != r[j]) {
        r[j] = p[j];
        p[j] = staged(r[j]) ? s_par[r[j] - c0] : ld_relaxed(&a.parent[r[j]]);
        more = true;
      }
    }
    if (!more) break;
  }
  int lab[U];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    lab[j] = -1;
    if (!v[j]) continue;
    const bool in = staged(r[j]);
    if ((in ? s_fl[r[j] - c0] : a.flags[r[j]]) & F_SEED)
      lab[j] = seed_rank(a, in ? s_hs[r[j] - c0] : a.hs[r[j]]) - seed_rank(a, first[j]);
  }
#pragma unroll
  for (int j = 0; j < U; ++j) {
    if (!v[j]) continue;
    if (r[j] != s[j] && r[j] != p0[j]) st_relaxed(&a.parent[s[j]], r[j]);
    d.cluster_id[hsj[j]] = lab[j];
  }
  __syncthreads();  // the next chunk overwrites the staged arrays
}

// ---------------------------------------------------------------------------
// Terms of Eq. 3.
// ---------------------------------------------------------------------------
// exp(x) for x <= 0 as one fixed binary32 evaluation, after Cody and Waite's
// range reduction: x = k ln2 + r with k = floor(x / ln2 + 1/2) and ln2 split
// into a high part with trailing zero bits (k * hi exact) and the remainder;
// exp(r) by its degree-7 Taylor polynomial in Horner form; then the scale by
// 2^k. Every step is an explicit binary32 rounding, so any IEEE evaluation of
// the same steps gives the same bits. 0 when k < -125.
__device__ __forceinline__ float exp32(float x) {
  constexpr float inv_ln2 = (float)(1.0 / 0.69314718055994530942);
  constexpr float ln2_hi = 0.693145751953125f;
  constexpr float ln2_lo = (float)(0.69314718055994530942 - 0.693145751953125);
  const float kf = floorf(__fadd_rn(__fmul_rn(x, inv_ln2), 0.5f));
  if (!(kf >= -125.0f)) return 0.0f;
  const float r = __fsub_rn(__fsub_rn(x, __fmul_rn(kf, ln2_hi)), __fmul_rn(kf, ln2_lo));
  float p = (float)(1.0 / 5040.0);
  p = __fadd_rn(__fmul_rn(p, r), (float)(1.0 / 720.0));
  p = __fadd_rn(__fmul_rn(p, r), (float)(1.0 / 120.0));
  p = __fadd_rn(__fmul_rn(p, r), (float)(1.0 / 24.0));
  p = __fadd_rn(__fmul_rn(p, r), (float)(1.0 / 6.0));
  p = __fadd_rn(__fmul_rn(p, r), 0.5f);
  p = __fadd_rn(__fmul_rn(p, r), 1.0f);
  p = __fadd_rn(__fmul_rn(p, r), 1.0f);
  return __fmul_rn(p, __uint_as_float((unsigned)((int)kf + 127) << 23));
}

// Correctly rounded binary32 square root of x >= 0: the hardware estimate
// (within an ulp) is corrected by comparing x with the squares of the
// midpoints to its neighbours, which are exact in binary64. Subnormal x is
// scaled by 2^64 first (exact, and exactly undone by 2^-32).
__device__ __forceinline__ float sqrt_rn(float x) {
  if (!(x > 0.0f) || x == __int_as_float(0x7f800000)) return x;
  const bool tiny = x < 1.17549435e-38f;
  const float xs = tiny ? __fmul_rn(x, 18446744073709551616.0f) : x;
  float s = __builtin_sqrtf(xs);
  const double xd = (double)xs;
  const float up = __uint_as_float(__float_as_uint(s) + 1u);
  const double mh = 0.5 * ((double)s + (double)up);
  if (mh * mh < xd) {
    s = up;
  } else {
    const float dn = __uint_as_float(__float_as_uint(s) - 1u);
    const double ml = 0.5 * ((double)dn + (double)s);
    if (ml * ml > xd) s = dn;
  }
  return tiny ? __fmul_rn(s, 2.3283064365386963e-10f) : s;
}

// One term of Eq. 3 for a neighbour at squared distance d2 with energy e:
// e (flat kernel), fl(exp(-fl(d2 a)) e) (Gaussian, a = 1 / (2 s^2)) or
// fl(exp(-fl(sqrt(d2) a)) e) (exponential, a = 1 / s).
template <int K>
__device__ __forceinline__ float kernel_term(float d2, float ka, float e) {
  if constexpr (K == 0) {
    return e;
  } else if constexpr (K == 1) {
    return __fmul_rn(exp32(-__fmul_rn(d2, ka)), e);
  } else {
    return __fmul_rn(exp32(-__fmul_rn(sqrt_rn(d2), ka)), e);
  }
}

}  // namespace clue
