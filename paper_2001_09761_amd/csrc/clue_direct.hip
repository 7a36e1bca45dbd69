// The all-pairs form of the pipeline for runs of up to kDirectMax hits.
//
// A small run spends its time in launches and in the latency of short
// dependent stages, not in pair tests: one layer of 1,000 hits took 72 us in
// the tiled form's twelve kernels. So no grid is built. Three kernels read the
// hits in the caller's order, which is the ascending index order that the
// density sum needs:
//   k_direct_density  rho of every hit (Eq. 3)
//   k_direct_nearest  nh and delta^2 of every hit (Eq. 4) and the decision
//                     (Sec. 2.2, Algorithm 3)
//   k_direct_finish   seed numbers, labels and follower lists
// Both search kernels give each wave one or two queries and stream all hits past
// them in LDS blocks; candidates of other (event, layer) units are skipped 256
// at a time.
//
// They are bound by VALU issue (about 15 instructions per 64 pairs, 8 of them
// the distance and its tests) from about 4,000 hits of one layer on, and by
// latency below. Time per run, tiled form -> this one, with one layer of uniform
// hits in 200 x 200 cm (in brackets: the hits in 20 x 20 cm):
//   1,000 hits  67 -> 20 us (770 -> 20)    4,000 hits  75 -> 38 us (1,740 -> 43)
//   6,000 hits  82 -> 59 us (1,520 -> 66)  8,000 hits  84 -> 74 us (1,480 -> 83)
//   10,000 hits 92 -> 140 us
// With ten layers in order 8,000 hits take 29 us (tiled 74). The work grows with
// the square of the largest unit, which the host does not know, so kDirectMax
// (8,192) is where a single layer still gains; it is also where two queries per
// wave fill the 256 CUs once.
#include "clue_device.h"

#include <algorithm>

namespace clue {

namespace {

// Each workgroup has 16 waves, because a wave's chain of test, ballot and list
// update is latency-bound, and 4,000 hits at one query per wave are 250
// workgroups, one per CU: the waves that hide it have to come from the
// workgroup itself. Runs of more than kDirQ1Max hits have waves enough and give
// each wave two queries, which share a candidate's loads.
constexpr int kDirWG = 1024;
constexpr int kDirWaves = kDirWG / 64;
constexpr int kDirList = 640;    // passing terms a wave's lists hold, shared by its queries
constexpr int kDirQ1Max = 4096;
constexpr int kDirStep = 256;    // candidates a wave tests at a time
constexpr int kDirChunks = (kDirectMax + kDirWG - 1) / kDirWG * kDirWaves;  // 64 candidates each
static_assert(kDirWaves == 16, "a block's chunk mask is 16 bits");

// Unit of a hit: its event and layer, clamped as the tiled kernels clamp them.
// The ids are loaded apart from the arithmetic, so that a prefetch does not
// wait for them. Hit h must be in range.
struct Ids {
  int e, l;
};
__device__ __forceinline__ Ids load_ids(const RunDesc& d, int h) {
  return Ids{d.event ? d.event[h] : d.event_base, d.layer[h]};
}
__device__ __forceinline__ int unit_of(const RunDesc& d, const Geom& g, Ids i) {
  return clampi(i.e - d.event_base, 0, d.n_events - 1) * g.L + clampi(i.l, 0, g.L - 1);
}

__device__ __forceinline__ float uniform_f(float v) {
  return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v)));
}

// A wave's queries, in scalar registers: hits h0 .. h0 + Q - 1. A query past
// the last hit has unit -1, which no candidate has.
template <int Q>
struct Queries {
  float x[Q], y[Q];
  int u[Q];
};
template <int Q>
__device__ __forceinline__ Queries<Q> load_queries(const RunDesc& d, const Geom& g, int h0) {
  Queries<Q> qs;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int h = min(h0 + q, d.n - 1);
    qs.x[q] = uniform_f(d.x[h]);
    qs.y[q] = uniform_f(d.y[h]);
    const int u = __builtin_amdgcn_readfirstlane(unit_of(d, g, load_ids(d, h)));
    qs.u[q] = h0 + q < d.n ? u : -1;
  }
  return qs;
}

// One candidate per thread of the workgroup. The weight is the energy
// (density) or the order-preserving integer of rho (nearest-higher).
struct Cand {
  float x, y;
  unsigned w;
  int u;
};
struct RawCand {
  float x, y, w;
  Ids id;
};
struct __align__(16) CandBlock {
  float x[kDirWG], y[kDirWG];
  unsigned w[kDirWG];
  int u[kDirWG];
};

// Past the last hit the last one is loaded again; its unit is then replaced.
template <bool RHO>
__device__ __forceinline__ RawCand load_cand(const RunDesc& d, const Arena& a, int b0) {
  const int j = min(b0 + (int)threadIdx.x, d.n - 1);
  return RawCand{d.x[j], d.y[j], RHO ? a.rho[j] : d.e[j], load_ids(d, j)};
}

// Streams the hits past the workgroup's queries: `visit(j, candidates)` is
// called for each step of 256 candidates to be searched, in ascending order,
// with this lane's four and the index of their first. First the units alone
// are read, all at once, and each chunk of 64 that holds none of the
// workgroup's units is marked: a step of four such chunks is skipped, and a
// block of 16 is not loaded (10 layers of 1,003 hits in order are ten blocks, of
// which a workgroup needs one or two). Two LDS blocks alternate, so one barrier
// per block is enough.
template <int Q, bool RHO, typename Visit>
__device__ __forceinline__ void stream_hits(const RunDesc& d, const Geom& g, const Arena& a,
                                            Visit visit) {
  __shared__ CandBlock B[2];
  __shared__ unsigned char s_act[kDirChunks];
  const int lane = threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  const int blocks = (d.n + kDirWG - 1) / kDirWG;
  unsigned need = 1u;  // bit b: block b has to be searched
  if (blocks > 1) {
    Ids id[kDirChunks / kDirWaves];
#pragma unroll
    for (int b = 0; b < kDirChunks / kDirWaves; ++b) id[b] = load_ids(d, min(b * kDirWG + (int)threadIdx.x, d.n - 1));
    const int u =
        unit_of(d, g, load_ids(d, min((int)blockIdx.x * kDirWaves * Q + (lane & (kDirWaves * Q - 1)), d.n - 1)));
    int lo = u, hi = u;
#pragma unroll
    for (int o = 1; o < kDirWaves * Q; o <<= 1) {
      lo = min(lo, __shfl_xor(lo, o, 64));
      hi = max(hi, __shfl_xor(hi, o, 64));
    }
#pragma unroll
    for (int b = 0; b < kDirChunks / kDirWaves; ++b) {
      const int uj = unit_of(d, g, id[b]);
      const bool act = __any(b * kDirWG + (int)threadIdx.x < d.n && uj >= lo && uj <= hi);
      if (lane == 0) s_act[b * kDirWaves + wave] = act;
    }
    __syncthreads();
    need = 0u;
#pragma unroll
    for (int c0 = 0; c0 < kDirChunks; c0 += 64) {
      const unsigned long long m = __ballot(c0 + lane < kDirChunks && s_act[min(c0 + lane, kDirChunks - 1)]);
#pragma unroll
      for (int k = 0; k < 4; ++k) need |= (((m >> (16 * k)) & 0xffffull) ? 1u : 0u) << (c0 / kDirWaves + k);
    }
  }
  if (!need) return;
  int b = __ffs((int)need) - 1;
  RawCand c = load_cand<RHO>(d, a, b * kDirWG);
  for (int k = 0; need; k ^= 1) {
    const int b0 = b * kDirWG;
    CandBlock& S = B[k];
    S.x[threadIdx.x] = c.x;
    S.y[threadIdx.x] = c.y;
    S.w[threadIdx.x] = RHO ? ord_f32(c.w) : __float_as_uint(c.w);
    S.u[threadIdx.x] = b0 + (int)threadIdx.x < d.n ? unit_of(d, g, c.id) : -2;  // past the last hit: no query's unit
    unsigned act = 0xffffu >> (16 - min((d.n - b0 + 63) >> 6, 16));
    if (blocks > 1) act = (unsigned)__ballot(lane < kDirWaves && s_act[b * kDirWaves + (lane & (kDirWaves - 1))]);
    need &= need - 1u;
    if (need) {
      b = __ffs((int)need) - 1;
      c = load_cand<RHO>(d, a, b * kDirWG);
    }
    __syncthreads();
    // a step is 256 candidates, four consecutive ones per lane
    for (int st = 0; st < kDirWG / kDirStep; ++st) {
      if (!((act >> (4 * st)) & 0xfu)) continue;  // uniform
      const int p = st * kDirStep + 4 * lane;
      const float4 x = *reinterpret_cast<const float4*>(S.x + p), y = *reinterpret_cast<const float4*>(S.y + p);
      const uint4 w = *reinterpret_cast<const uint4*>(S.w + p);
      const int4 u = *reinterpret_cast<const int4*>(S.u + p);
      const Cand c[4] = {{x.x, y.x, w.x, u.x}, {x.y, y.y, w.y, u.y}, {x.z, y.z, w.z, u.z}, {x.w, y.w, w.w, u.w}};
      visit(b0 + p, c);
    }
  }
}

// Orders LDS traffic between the lanes of one wave (which runs in lockstep
// and whose LDS accesses are performed in order): the compiler may not move
// accesses across it.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

}  // namespace

// ---------------------------------------------------------------------------
// Density. Each lane tests its candidate; the terms of the passing ones are
// compacted, in lane order and so in ascending hit index, to the query's list
// in LDS, which lane q then adds up in order for query q.
// ---------------------------------------------------------------------------
template <int Q, int K>
__global__ __launch_bounds__(kDirWG) void k_direct_density(RunDesc d, Geom g, Arena a) {
  __shared__ __align__(16) float lists[kDirWaves][Q][kDirList / Q];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int h0 = ((int)blockIdx.x * kDirWaves + wave) * Q;
  const Queries<Q> qs = load_queries<Q>(d, g, h0);
  int cnt[Q];        // terms in each list, wave-uniform
  float acc = 0.0f;  // lane q: query q's sum so far
#pragma unroll
  for (int q = 0; q < Q; ++q) cnt[q] = 0;
  auto flush = [&]() {
    wave_sync();
    int n = cnt[0];
#pragma unroll
    for (int q = 1; q < Q; ++q) n = lane == q ? cnt[q] : n;
    const float* const list = lists[wave][lane & (Q - 1)];
    int i = 0;
    for (; i + 8 <= n; i += 8) {
      const float4 v = *reinterpret_cast<const float4*>(list + i), w = *reinterpret_cast<const float4*>(list + i + 4);
      acc = __fadd_rn(__fadd_rn(__fadd_rn(__fadd_rn(acc, v.x), v.y), v.z), v.w);
      acc = __fadd_rn(__fadd_rn(__fadd_rn(__fadd_rn(acc, w.x), w.y), w.z), w.w);
    }
    for (; i < n; ++i) acc = __fadd_rn(acc, list[i]);
#pragma unroll
    for (int q = 0; q < Q; ++q) cnt[q] = 0;
    wave_sync();
  };
  stream_hits<Q, false>(
      d, g, a,
      [&](int, const Cand (&c)[4]) {
        int most = 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          float d2[4];
          bool pass[4];
          unsigned long long m[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            d2[k] = dist2(qs.x[q], qs.y[q], c[k].x, c[k].y);
            pass[k] = c[k].u == qs.u[q] && d2[k] < g.dc2;
            m[k] = __builtin_amdgcn_ballot_w64(pass[k]);
          }
          if ((m[0] | m[1]) | (m[2] | m[3])) {
            // the passing candidates of the lanes below, then this lane's in order
            int o = cnt[q];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              o = __builtin_amdgcn_mbcnt_hi((unsigned)(m[k] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m[k], (unsigned)o));
              cnt[q] += __popcll(m[k]);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
              if (pass[k]) lists[wave][q][o++] = kernel_term<K>(d2[k], g.ka, __uint_as_float(c[k].w));
          }
          most = max(most, cnt[q]);
        }
        if (most > kDirList / Q - kDirStep) flush();  // a step adds at most kDirStep terms
      });
  flush();
  const int h = h0 + lane;
  if (lane < Q && h < d.n) {
    a.rho[h] = acc;
    if (g.flags & 2u) a.rho_out[h] = acc;
  }
}

// ---------------------------------------------------------------------------
// Nearest-higher and the decision. Each lane keeps the nearest higher
// candidate of its own (candidates come in ascending index, so a strict
// comparison keeps the smallest index among equal distances); the wave then
// takes the lexicographic minimum of (d2, index). Parents and nh are caller
// indices here; nh goes to the key buffer for k_direct_finish.
// ---------------------------------------------------------------------------
template <int Q>
__global__ __launch_bounds__(kDirWG) void k_direct_nearest(RunDesc d, Geom g, Arena a) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int h0 = ((int)blockIdx.x * kDirWaves + wave) * Q;
  const Queries<Q> qs = load_queries<Q>(d, g, h0);
  const bool strict = g.flags & 4u;
  unsigned ordi[Q];
  float bd[Q];
  int bj[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    ordi[q] = __builtin_amdgcn_readfirstlane(ord_f32(a.rho[min(h0 + q, d.n - 1)]));
    bd[q] = g.dm2;  // beaten by d2 < dm2 only
    bj[q] = -1;
  }
  stream_hits<Q, true>(
      d, g, a,
      [&](int j, const Cand (&c)[4]) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float d2 = dist2(qs.x[q], qs.y[q], c[k].x, c[k].y);
            const bool higher = c[k].w > ordi[q] || (!strict && c[k].w == ordi[q] && j + k > h0 + q);
            const bool take = c[k].u == qs.u[q] && higher && d2 < bd[q];
            bd[q] = take ? d2 : bd[q];
            bj[q] = take ? j + k : bj[q];
          }
        }
      });
  // d2 >= 0 orders like its bits
  unsigned long long best = ~0ull;  // lane q: query q's
  unsigned ord = 0u;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    unsigned long long k = bj[q] >= 0 ? ((unsigned long long)__float_as_uint(bd[q]) << 32) | (unsigned)bj[q] : ~0ull;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned long long t = __shfl_xor(k, o, 64);
      k = t < k ? t : k;
    }
    best = lane == q ? k : best;
    ord = lane == q ? ordi[q] : ord;
  }
  const int h = h0 + lane;
  if (lane < Q && h < d.n) {
    const bool has = best != ~0ull;
    const int nh = has ? (int)(unsigned)(best & 0xffffffffu) : -1;
    const float ri = ord_inv(ord);
    const float d2 = has ? __uint_as_float((unsigned)(best >> 32)) : __int_as_float(0x7f800000);
    const bool seed = ri > g.rho_c && d2 > g.dcs2;
    const bool outlier = ri < g.rho_c && d2 > g.do2;
    const bool follower = !seed && !outlier && has;
    a.parent[h] = follower ? nh : h;
    a.flags[h] = (uint8_t)((seed ? F_SEED : 0) | (outlier ? F_OUTLIER : 0) | (follower ? F_FOLLOWER : 0));
    if (g.flags & 2u) {
      a.key[h] = nh;
      a.d2_out[h] = d2;
    }
  }
}

// ---------------------------------------------------------------------------
// Seed numbers, labels and follower lists. One workgroup writes the results of
// kFinWG hits, but each builds the whole run's seed bitmap, follower lists and
// links in its own LDS (4 bytes a hit and a few bits): that takes each lane
// only n / kFinWG hits more, and no step then needs another workgroup's result
// or another launch. PER is the hits per lane of those steps, a template
// argument so that the code of a small run stays short.
// ---------------------------------------------------------------------------
constexpr int kFinWG = 1024;
constexpr int kFinPer = (kDirectMax + kFinWG - 1) / kFinWG;
constexpr int kFinWords = kDirectMax / 32 + 1;
static_assert(kDirectMax <= 65535, "links, counts and list entries are 16-bit");
static_assert(kFinWords <= kFinWG, "one lane per bitmap word");

template <int PER>
__global__ __launch_bounds__(kFinWG) void k_direct_finish(RunDesc d, Geom g, Arena a) {
  // dynamic LDS, 16 bits each: list entries, then links [n]; follower counts, then offsets [n + 1]
  extern __shared__ __align__(16) unsigned short lds16[];
  __shared__ unsigned s_seed[kFinWords], s_first[kFinWords];  // bit per hit: a seed; the first hit of an event
  __shared__ int s_wrank[kFinWords];   // seeds before each word
  __shared__ int s_wfirst[kFinWords];  // first hit of the last event that starts before each word
  __shared__ int s_part[kFinWG / 64];
  const int n = d.n, tid = threadIdx.x, lane = tid & 63;
  const int nr = (n + 2) & ~1;  // n + 1 rounded up to a pair
  unsigned short* const par = lds16;
  unsigned short* const ent = lds16;
  unsigned* const cnt2 = reinterpret_cast<unsigned*>(lds16 + nr);  // two counts per word
  unsigned short* const off = lds16 + nr;
  const bool lists = !(g.flags & 8u);

  int own[PER];  // the hit's link, before any jump
  bool fol[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int h = k * kFinWG + tid;
    own[k] = h;
    unsigned f = 0u;
    bool first = h == 0;
    if (h < n) {
      own[k] = a.parent[h];
      f = a.flags[h];
      if (d.event && h > 0) first = d.event[h] != d.event[h - 1];
      if (lists && h < nr / 2) cnt2[h] = 0u;
    }
    fol[k] = f & F_FOLLOWER;
    const unsigned long long ms = __ballot(f & F_SEED), mf = __ballot(first);
    const int w = (k * kFinWG + (tid & ~63)) >> 5;
    if (lane < 2 && w + lane < kFinWords) {
      s_seed[w + lane] = (unsigned)(ms >> (32 * lane));
      s_first[w + lane] = (unsigned)(mf >> (32 * lane));
    }
  }
  __syncthreads();
  // seeds before each word; last event start before each word
  {
    const int words = n / 32 + 1;
    const unsigned ws = tid < words ? s_seed[tid] : 0u, wf = tid < words ? s_first[tid] : 0u;
    int total;
    const int r = wg_excl<kFinWG>(__popc(ws), s_part, total, tid);
    if (tid < words) {
      s_wrank[tid] = r;
      s_wfirst[tid] = 0;
    }
    if (d.event) {
      int m = wf ? 32 * tid + 31 - __clz((int)wf) : 0;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(m, o, 64);
        if (lane >= o) m = max(m, t);
      }
      __syncthreads();
      if (lane == 63) s_part[tid >> 6] = m;
      __syncthreads();
      int before = __shfl_up(m, 1, 64);
      if (lane == 0) before = 0;
      for (int w = 0; w < (tid >> 6); ++w) before = max(before, s_part[w]);
      if (tid < words) s_wfirst[tid] = before;
    }
  }
  const int h = (int)blockIdx.x * kFinWG + tid;  // the hit this lane writes
  auto rank = [&](int i) { return s_wrank[i >> 5] + __popc(s_seed[i >> 5] & ((1u << (i & 31)) - 1u)); };
  auto first_of = [&](int i) {
    const unsigned w = s_first[i >> 5] & (0xffffffffu >> (31 - (i & 31)));
    return w ? (i & ~31) + 31 - __clz((int)w) : s_wfirst[i >> 5];
  };

  // follower lists: arrival position by a 16-bit count per owner, offsets by a
  // scan, then each entry's place by counting the smaller entries of its list
  if (lists) {
    int at[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (fol[k]) {
        const int s = 16 * (own[k] & 1);
        at[k] = (int)((atomicAdd(&cnt2[own[k] >> 1], 1u << s) >> s) & 0xffffu);
      }
    __syncthreads();
    const int i0 = tid * PER;  // PER counts per lane, n + 1 in all
    int v[PER], sum = 0, total;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      v[k] = i0 + k < n ? off[i0 + k] : 0;
      sum += v[k];
    }
    int run = wg_excl<kFinWG>(sum, s_part, total, tid);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      if (i0 + k < n) off[i0 + k] = (unsigned short)run;
      run += v[k];
    }
    if (tid == 0) {
      off[n] = (unsigned short)total;
      if (blockIdx.x == 0) a.fstart[n] = total;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k)
      if (fol[k]) ent[off[own[k]] + at[k]] = (unsigned short)(k * kFinWG + tid);
  }
  __syncthreads();
  const int f0 = h < n ? first_of(h) : 0;
  if (lists && h < n) {
    a.fstart[h] = off[h];
    const int owner = a.parent[h];
    if (owner != h) {
      const int b = off[owner], e = off[owner + 1];
      int r = b;
      for (int i = b; i < e; ++i) r += ent[i] < h;
      a.flist[r] = h - f0;
    }
  }
  __syncthreads();  // the links take the entries' place
#pragma unroll
  for (int k = 0; k < PER; ++k)
    if (k * kFinWG + tid < n) par[k * kFinWG + tid] = (unsigned short)own[k];
  __syncthreads();
  if (h >= n) return;
  // the root: every lane halves the paths it walks, and a link only ever moves
  // to an ancestor, so long chains shorten for all lanes at once and each walk ends
  int r = h;
  for (;;) {
    const int p = par[r];
    if (p == r) break;
    const int q = par[p];
    if (q != p) par[r] = (unsigned short)q;
    r = q;
  }
  const bool seeded = (s_seed[r >> 5] >> (r & 31)) & 1u;
  d.cluster_id[h] = seeded ? rank(r) - rank(f0) : -1;
  d.is_seed[h] = (uint8_t)((s_seed[h >> 5] >> (h & 31)) & 1u);
  if (g.flags & 2u) {
    const int nh = a.key[h];
    a.nh_out[h] = nh >= 0 ? nh - f0 : -1;
  }
}

template <int Q>
static void launch_direct_search(const Geom& g, const Arena& a, const RunDesc& d, hipStream_t s, hipEvent_t mid) {
  const int grid = (d.n + kDirWaves * Q - 1) / (kDirWaves * Q);
  if (g.kernel == 0)
    k_direct_density<Q, 0><<<grid, kDirWG, 0, s>>>(d, g, a);
  else if (g.kernel == 1)
    k_direct_density<Q, 1><<<grid, kDirWG, 0, s>>>(d, g, a);
  else
    k_direct_density<Q, 2><<<grid, kDirWG, 0, s>>>(d, g, a);
  if (mid) (void)hipEventRecord(mid, s);
  k_direct_nearest<Q><<<grid, kDirWG, 0, s>>>(d, g, a);
}

hipError_t launch_direct(const Geom& g, const Arena& a, const RunDesc& d, hipStream_t s, hipEvent_t* ev) {
  auto mark = [&](int from, int to) {
    for (int k = from; ev && k <= to; ++k) (void)hipEventRecord(ev[k], s);
  };
  mark(0, S_RHO);  // no grid is built
  if (d.n <= kDirQ1Max)
    launch_direct_search<1>(g, a, d, s, ev ? ev[S_NH] : nullptr);
  else
    launch_direct_search<2>(g, a, d, s, ev ? ev[S_NH] : nullptr);
  mark(S_SCAN_SEEDS, S_LABEL);
  const int fin = (d.n + kFinWG - 1) / kFinWG, lds = 4 * ((d.n + 2) & ~1);
  if (fin == 1)
    k_direct_finish<1><<<fin, kFinWG, lds, s>>>(d, g, a);
  else if (fin <= 4)
    k_direct_finish<4><<<fin, kFinWG, lds, s>>>(d, g, a);
  else
    k_direct_finish<kFinPer><<<fin, kFinWG, lds, s>>>(d, g, a);
  mark(S_FOLLOW, S_COUNT);
  return hipGetLastError();
}

}  // namespace clue
