// Binning of visibilities by (w-plane, uv tile, edge region): the MI355X
// counterpart of the paper's per-slab linked lists (Sec. 3.2), which gather
// the visibilities of one slab, halo included, into contiguous arrays so
// that the gridding kernel reads them in order.  Here a counting sort builds
// one contiguous record range per key:
//   bin_count   FP64 placement, key and rank of every visibility; ranks
//               come from an LDS hash table per workgroup, so a hot key
//               costs one global atomic per workgroup, not per visibility
//   scan_*      exclusive scan of the key counts into record offsets
//   bin_scatter writes the packed record of every visibility at
//               offset[key] + rank
//   tile_work   per tile: records to process (own + neighbours' facing
//               strips), number of work items, split-tile scratch slots
#include "ws_kernels.h"

namespace ws {

namespace {

constexpr int kCountThreads = 256;
constexpr int kCountPerBlock = 4096;    // visibilities per workgroup
constexpr int kHashSize = 8192;         // >= 2 x kCountPerBlock
static_assert(kHashSize == 1 << 13, "hash_slot takes 13 bits");
constexpr int kCountPerThread = kCountPerBlock / kCountThreads;

__device__ __forceinline__ uint32_t hash_slot(uint32_t key) {
  return (key * 2654435761u) >> (32 - 13);  // 13 = log2(kHashSize)
}

// Speed of light (m/s): baseline-major uvw in metres becomes wavelengths
// at frequency f by the factor f / c0.
constexpr double kSpeedOfLight = 299792458.0;

// Baseline coordinates of visibility i in wavelengths.  Baseline-major:
// the scale f / c0 is one FP64 division, then one product per coordinate
// (contraction off, so the position rounds as the separate operations).
__device__ __forceinline__ void source_uvw(const VisSource& s, int64_t i,
                                           double& u, double& v, double& w) {
#pragma clang fp contract(off)
  if (s.rows) {
    const int64_t r = i / s.nchan;
    const int c = (int)(i - r * s.nchan);
    const double sc = s.freq[c] / kSpeedOfLight;
    u = s.uvw[3 * r] * sc;
    v = s.uvw[3 * r + 1] * sc;
    w = s.uvw[3 * r + 2] * sc;
  } else {
    u = s.uvw[3 * i];
    v = s.uvw[3 * i + 1];
    w = s.uvw[3 * i + 2];
  }
}

// Weighted value of visibility i (gridding).  Baseline-major: the
// correlations of row r, channel c combined in FP64 with the coefficients
// and the per-correlation weights, then rounded to the path precision.
template <typename R>
__device__ __forceinline__ cplx<R> source_value(const VisSource& s,
                                                int64_t i) {
  if (s.rows) {
    const int64_t r = i / s.nchan;
    const cplx<R>* v = static_cast<const cplx<R>*>(s.vis) + i * s.npol;
    double re = 0.0, im = 0.0;
    for (int p = 0; p < s.npol; ++p) {
      const double wt = s.weight != nullptr
                            ? (double)s.weight[r * s.npol + p] : 1.0;
      const double ar = s.coef[p][0] * wt, ai = s.coef[p][1] * wt;
      const cplx<R> x = v[p];
      re += ar * (double)x.re - ai * (double)x.im;
      im += ar * (double)x.im + ai * (double)x.re;
    }
    return {(R)re, (R)im};
  }
  const R wt = s.weight != nullptr ? (R)s.weight[i] : (R)1;
  if (s.vis == nullptr) return {wt, (R)0};  // unit visibilities
  const cplx<R> vv = static_cast<const cplx<R>*>(s.vis)[i];
  return {wt * vv.re, wt * vv.im};
}

// Weight of visibility i (degridding reads flat sources only).
__device__ __forceinline__ float source_weight(const VisSource& s,
                                               int64_t i) {
  return s.weight != nullptr ? s.weight[i] : 1.0f;
}

__global__ __launch_bounds__(kCountThreads) void k_bin_count(
    Geo g, VisSource src, int64_t m,
    uint32_t* __restrict__ copies, uint32_t nkeys,
    uint2* __restrict__ keyrank, unsigned long long* __restrict__ dropped) {
  uint32_t* __restrict__ counts =
      copies + (size_t)(blockIdx.x % kCountCopies) * nkeys;
  __shared__ uint32_t s_key[kHashSize];
  __shared__ uint32_t s_cnt[kHashSize];
  __shared__ unsigned long long s_drop;
  const int tid = threadIdx.x;
  for (int s = tid; s < kHashSize; s += kCountThreads) {
    s_key[s] = kNoKey;
    s_cnt[s] = 0;
  }
  if (tid == 0) s_drop = 0;
  __syncthreads();

  uint32_t my_key[kCountPerThread];
  uint32_t my_slot[kCountPerThread];
  uint32_t my_rank[kCountPerThread];
  unsigned long long my_drop = 0;
  const int64_t base = (int64_t)blockIdx.x * kCountPerBlock;
  // All coordinates first (indices clamped into range), so that the loads
  // overlap instead of each waiting behind the previous one's LDS atomics.
  double cu[kCountPerThread], cv[kCountPerThread], cw[kCountPerThread];
#pragma unroll
  for (int e = 0; e < kCountPerThread; ++e) {
    int64_t gi = base + e * kCountThreads + tid;
    gi = gi < m ? gi : m - 1;
    source_uvw(src, gi, cu[e], cv[e], cw[e]);
  }
#pragma unroll
  for (int e = 0; e < kCountPerThread; ++e) {
    const int64_t gi = base + e * kCountThreads + tid;
    my_key[e] = kNoKey;
    if (gi < m) {
      double x, y;
      int i0, j0, k;
      const double u = cu[e], v = cv[e], w = cw[e];
      if (place(g, u, v, w, x, y, i0, j0, k)) {
        my_drop += (unsigned long long)(g.K * g.K - taps_on_grid(g, i0, j0));
        const uint32_t key = bin_key(g, i0, j0, k);
        uint32_t s = hash_slot(key);
        while (true) {
          const uint32_t prev = atomicCAS(&s_key[s], kNoKey, key);
          if (prev == kNoKey || prev == key) break;
          s = (s + 1) & (kHashSize - 1);
        }
        my_key[e] = key;
        my_slot[e] = s;
        my_rank[e] = atomicAdd(&s_cnt[s], 1u);
      } else {
        my_drop += (unsigned long long)(g.K * g.K);
      }
    }
  }
  if (dropped != nullptr && my_drop != 0) atomicAdd(&s_drop, my_drop);
  __syncthreads();
  // One global atomic per distinct key of the workgroup; the returned old
  // count becomes the workgroup's base rank for that key (kept in s_cnt).
  // All of a thread's atomics are issued before any result is used, so
  // their round trips overlap.
  constexpr int kSlotsPerThread = kHashSize / kCountThreads;
  uint32_t old[kSlotsPerThread];
#pragma unroll
  for (int e = 0; e < kSlotsPerThread; ++e) {
    const int s = tid + e * kCountThreads;
    const uint32_t key = s_key[s];
    old[e] = key != kNoKey ? atomicAdd(&counts[key], s_cnt[s]) : 0u;
  }
#pragma unroll
  for (int e = 0; e < kSlotsPerThread; ++e) {
    const int s = tid + e * kCountThreads;
    if (s_key[s] != kNoKey) s_cnt[s] = old[e];
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kCountPerThread; ++e) {
    const int64_t gi = base + e * kCountThreads + tid;
    if (gi < m) {
      uint2 kr;
      kr.x = my_key[e];
      kr.y = my_key[e] == kNoKey ? 0u : s_cnt[my_slot[e]] + my_rank[e];
      keyrank[gi] = kr;
    }
  }
  if (tid == 0 && dropped != nullptr && s_drop != 0)
    atomicAdd(dropped, s_drop);
}

// Per-key totals of the count copies.
__global__ __launch_bounds__(256) void k_fold_copies(
    const uint32_t* __restrict__ copies, uint32_t nkeys,
    uint32_t* __restrict__ totals) {
  const uint32_t key = blockIdx.x * 256u + threadIdx.x;
  if (key >= nkeys) return;
  uint32_t c[kCountCopies];
#pragma unroll
  for (int x = 0; x < kCountCopies; ++x) c[x] = copies[(size_t)x * nkeys + key];
  uint32_t t = 0;
#pragma unroll
  for (int x = 0; x < kCountCopies; ++x) t += c[x];
  totals[key] = t;
}

// Copy x of key k becomes the offset of its first record: the key's offset
// plus the counts of the copies before x.
__global__ __launch_bounds__(256) void k_copy_offsets(
    uint32_t* __restrict__ copies, uint32_t nkeys,
    const uint32_t* __restrict__ offsets) {
  const uint32_t key = blockIdx.x * 256u + threadIdx.x;
  if (key >= nkeys) return;
  uint32_t c[kCountCopies];
#pragma unroll
  for (int x = 0; x < kCountCopies; ++x) c[x] = copies[(size_t)x * nkeys + key];
  uint32_t o = offsets[key];
#pragma unroll
  for (int x = 0; x < kCountCopies; ++x) {
    copies[(size_t)x * nkeys + key] = o;
    o += c[x];
  }
}

// ---- exclusive scan of uint32 counts (reduce, scan of block sums, apply) --

constexpr int kScanThreads = 256;
constexpr int kScanPerThread = 16;
constexpr int kScanBlock = kScanThreads * kScanPerThread;

__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v,
                                                         uint32_t* s_tmp,
                                                         uint32_t* total) {
  // Inclusive wave scan, then a scan of the wave totals.
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) s_tmp[wave] = x;
  __syncthreads();
  uint32_t wbase = 0;
  uint32_t all = 0;
  for (int w2 = 0; w2 < (int)(blockDim.x >> 6); ++w2) {
    const uint32_t t = s_tmp[w2];
    if (w2 < wave) wbase += t;
    all += t;
  }
  __syncthreads();
  *total = all;
  return wbase + x - v;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(
    const uint32_t* __restrict__ in, int64_t n, uint32_t* __restrict__ sums) {
  __shared__ uint32_t s_tmp[kScanThreads / 64];
  const int64_t base = (int64_t)blockIdx.x * kScanBlock;
  uint32_t acc = 0;
#pragma unroll
  for (int e = 0; e < kScanPerThread; ++e) {
    const int64_t i = base + (int64_t)e * kScanThreads + threadIdx.x;
    if (i < n) acc += in[i];
  }
  uint32_t total;
  block_exclusive_scan(acc, s_tmp, &total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(1024) void k_scan_sums(uint32_t* __restrict__ sums,
                                                    int64_t nb) {
  // One workgroup: exclusive scan of nb block sums in place; sums[nb] = total.
  __shared__ uint32_t s_tmp[16];
  uint32_t carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += 1024) {
    const int64_t i = b0 + threadIdx.x;
    const uint32_t v = i < nb ? sums[i] : 0u;
    uint32_t total;
    const uint32_t ex = block_exclusive_scan(v, s_tmp, &total);
    if (i < nb) sums[i] = carry + ex;
    carry += total;
    __syncthreads();
  }
  if (threadIdx.x == 0) sums[nb] = carry;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_apply(
    const uint32_t* in, uint32_t* out, int64_t n,
    const uint32_t* __restrict__ sums, int64_t nb) {
  // Each thread owns kScanPerThread consecutive elements.
  __shared__ uint32_t s_tmp[kScanThreads / 64];
  const int64_t base = (int64_t)blockIdx.x * kScanBlock +
                       (int64_t)threadIdx.x * kScanPerThread;
  uint32_t v[kScanPerThread];
  uint32_t acc = 0;
#pragma unroll
  for (int e = 0; e < kScanPerThread; ++e) {
    const int64_t i = base + e;
    v[e] = i < n ? in[i] : 0u;
    acc += v[e];
  }
  uint32_t total;
  uint32_t run = block_exclusive_scan(acc, s_tmp, &total) + sums[blockIdx.x];
#pragma unroll
  for (int e = 0; e < kScanPerThread; ++e) {
    const int64_t i = base + e;
    if (i < n) out[i] = run;
    run += v[e];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = sums[nb];
}

// The record of visibility gi (one that place() accepts).
template <typename R>
__device__ __forceinline__ Record<R> make_record(const Geo& g,
                                                 const VisSource& src,
                                                 int64_t gi, int degrid) {
  double x, y, u, v, w;
  int i0, j0, k;
  source_uvw(src, gi, u, v, w);
  place(g, u, v, w, x, y, i0, j0, k);
  Record<R> r;
  // Fractional offsets from the nearest cell, subtracted in FP64 first.
  r.dx = (R)(x - (double)i0);
  r.dy = (R)(y - (double)j0);
  if (!degrid) {
    const cplx<R> vv = source_value<R>(src, gi);
    r.vr = vv.re;
    r.vi = vv.im;
  } else {
    r.vr = (R)source_weight(src, gi);
    r.vi = (R)0;
  }
  r.cell = pack_cell(i0, j0);
  r.idx = (uint32_t)gi;
  return r;
}

template <typename R>
__global__ __launch_bounds__(256) void k_bin_scatter(
    Geo g, VisSource src, int64_t m,
    const uint2* __restrict__ keyrank, const uint32_t* __restrict__ offsets,
    uint32_t nkeys, Record<R>* __restrict__ rec, int degrid,
    cplx<R>* __restrict__ vis_out) {
  const int64_t gi = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gi >= m) return;
  const uint2 kr = keyrank[gi];
  if (kr.x == kNoKey) {
    // No tap on the grid: no record, and a degridded value of zero (the
    // gather writes only the visibilities it has records for).
    if (degrid) vis_out[gi] = cplx<R>{(R)0, (R)0};
    return;
  }
  // The copy the counting workgroup of this visibility added into.
  const int64_t copy = (gi / kCountPerBlock) % kCountCopies;
  const uint32_t pos = offsets[copy * nkeys + kr.x] + kr.y;
  rec[pos] = make_record<R>(g, src, gi, degrid);
}

// Appends to a list with one atomic per wavefront: returns this lane's slot
// (lanes with pred false get an unspecified value).
__device__ __forceinline__ uint32_t wave_append(uint32_t* counter, bool pred) {
  const unsigned long long mask = __ballot(pred);
  const int lane = threadIdx.x & 63;
  const int leader = mask ? (__ffsll((long long)mask) - 1) : 0;
  uint32_t base = 0;
  if (mask != 0 && lane == leader)
    base = atomicAdd(counter, (uint32_t)__popcll(mask));
  base = (uint32_t)__shfl((int)base, leader, 64);
  const unsigned long long below = mask & ((1ull << lane) - 1ull);
  return base + (uint32_t)__popcll(below);
}

// Records of tile t: its own (degridding), or those of its ten key ranges
// (gridding), whose first records and lengths stay in registers for the
// descriptors.  `off` is the key offset table.
struct TileRecords {
  uint32_t work;
  uint32_t first[kSegments], len[kSegments];
};

template <class Off>
__device__ __forceinline__ TileRecords tile_records(const Geo& g, int t,
                                                    int mode_degrid, Off off) {
  TileRecords r;
  r.work = 0;
  if (mode_degrid) {
    r.first[0] = off[(uint32_t)t * kRegions];
    r.work = off[(uint32_t)t * kRegions + kRegions] - r.first[0];
    return r;
  }
  uint32_t lo[kSegments], hi[kSegments];
  tile_segments(g, t, lo, hi);
#pragma unroll
  for (int s = 0; s < kSegments; ++s) {
    r.first[s] = off[lo[s]];
    r.len[s] = off[hi[s]] - r.first[s];
    r.work += r.len[s];
  }
  return r;
}

// Cuts tile t into work items and writes what later passes read about it: its
// chunk count (0 marks a tile without records, whose stack cells may be left
// unwritten by a fused grid-and-image call), its entry `at` in the busy or
// idle list, its column strip's mark and the scratch slots of a split tile.
// Returns the chunk count, and in e0 the first of its extra items.  ctr: [0]
// scratch slots taken, [1] split tiles, [2] extra items; in LDS or in device
// memory.
__device__ __forceinline__ uint32_t emit_tile(const Geo& g, const TileWork& w,
                                              int t, uint32_t work,
                                              uint32_t at, uint32_t* ctr,
                                              uint32_t& e0) {
  if (work == 0) {
    w.idle[at] = (uint32_t)t;
    w.tile_slot[t] = 0;
    w.tile_chunks[t] = 0u;
    return 0;
  }
  w.busy[at] = (uint32_t)t;
  if (w.tslot != nullptr) w.tslot[t] = at;  // its slot in the busy-tile store
  if (w.strips != nullptr) {
    // Column strip of this tile: plane k, tile column tx.
    const int per_plane = g.tiles_u * g.tiles_v;
    const int k = t / per_plane;
    const int tx = (t - k * per_plane) % g.tiles_u;
    w.strips[k * g.tiles_u + tx] = 1u;
  }
  uint32_t nch = (work + w.chunk - 1) / w.chunk;
  uint32_t slot = 0;
  if (nch > 1 && !w.degrid) {
    const uint32_t s0 = atomicAdd(&ctr[0], nch);
    if (s0 + nch <= w.max_slots) {
      slot = s0;
      w.split_list[atomicAdd(&ctr[1], 1u)] = (uint32_t)t;
    } else {
      nch = 1;  // scratch exhausted: one item grids the whole tile
    }
  }
  if (nch > 1) {
    e0 = atomicAdd(&ctr[2], nch - 1);
    if (e0 + (nch - 1) > w.max_extra)
      nch = 1;  // cannot happen with the sizes the plan reserves
  }
  w.tile_slot[t] = slot;
  w.tile_chunks[t] = nch;
  return nch;
}

// What the descriptors of one tile hold (see kDescWords in ws_kernels.h).
struct TileDesc {
  uint32_t tile, nch, work, at, e0;
  uint32_t first;                       // degridding: its first record
  uint32_t ranges[2 * kSegments - 1];   // gridding: words 5 ..
};

__device__ __forceinline__ TileDesc tile_desc(const TileWork& w, int t,
                                              const TileRecords& r,
                                              uint32_t nch, uint32_t at,
                                              uint32_t e0) {
  TileDesc d = {};
  d.tile = (uint32_t)t;
  d.nch = nch;
  d.work = r.work;
  d.at = at;
  d.e0 = e0;
  d.first = r.first[0];
  if (w.degrid || nch == 0) return d;
  uint32_t cum = 0, prev = 0;
#pragma unroll
  for (int s = 0; s < kSegments; ++s) {
    const uint32_t off = r.first[s] - cum;
    if (s == 0) {
      d.ranges[0] = off;
    } else {
      d.ranges[s] = cum;
      d.ranges[kSegments - 1 + s] = off - prev;
    }
    prev = off;
    cum += r.len[s];
  }
  return d;
}

// Descriptor of chunk c.
template <bool DEGRID>
__device__ __forceinline__ void put_desc(const Geo& g, const TileWork& w,
                                         const TileDesc& d, uint32_t c) {
  const size_t n = c == 0 ? (size_t)d.at : (size_t)g.ntiles + d.e0 + c - 1;
  uint4* p = reinterpret_cast<uint4*>(w.desc);
  if constexpr (DEGRID) {
    const uint32_t b = d.first + c * w.chunk, end = d.first + d.work;
    p[n] = make_uint4(d.tile, b, d.nch == 1 ? end : min(end, b + w.chunk), 0u);
  } else {
    p += n * (kDescWords / 4);
    p[0] = make_uint4(d.tile, d.nch, d.nch == 1 ? d.at : c, c * w.chunk);
    p[1] = make_uint4(d.nch == 1 ? d.work : min(d.work, (c + 1) * w.chunk),
                      d.ranges[0], d.ranges[1], d.ranges[2]);
#pragma unroll
    for (int q = 2; q < kDescWords / 4; ++q)
      p[q] = make_uint4(d.ranges[4 * q - 5], d.ranges[4 * q - 4],
                        d.ranges[4 * q - 3], d.ranges[4 * q - 2]);
  }
}

// Descriptors of the items of a wavefront's tiles (one a lane, nch = 0 for
// none; all 64 lanes call).  A lane writes its own tile's, but those of a tile
// of more than kOwnDescs chunks are spread over the wavefront: one lane takes
// 80 ns for each, and the hottest tile may have thousands (1221 chunks of
// 4096: 101 -> 11 us; 19 532 degridding chunks of 256: 708 -> 27).
// With 3, 6 and 16 of its own: 1024^2 x 16, 1e6 14.0 / 12.4 / 11.5, 128^2 x 4,
// 2e4 (whole sort) 20.4 / 19.4 / 18.7.
constexpr uint32_t kOwnDescs = 16;
template <bool DEGRID>
__device__ __forceinline__ void spread_descs(const Geo& g, const TileWork& w,
                                             const TileDesc& d) {
  const bool own = d.nch <= kOwnDescs;
  if (own)
    for (uint32_t c = 0; c < d.nch; ++c) put_desc<DEGRID>(g, w, d, c);
  unsigned long long rest = __ballot(!own);
  while (rest != 0) {
    const int l = __ffsll((long long)rest) - 1;
    rest &= rest - 1;
    auto of = [&](uint32_t v) {
      return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
    };
    TileDesc o;
    o.tile = of(d.tile);
    o.nch = of(d.nch);
    o.work = of(d.work);
    o.at = of(d.at);
    o.e0 = of(d.e0);
    o.first = of(d.first);
    if constexpr (!DEGRID) {
#pragma unroll
      for (int q = 0; q < 2 * kSegments - 1; ++q)
        o.ranges[q] = of(d.ranges[q]);
    }
    for (uint32_t c = threadIdx.x & 63u; c < o.nch; c += 64u)
      put_desc<DEGRID>(g, w, o, c);
  }
}

__device__ __forceinline__ void emit_descs(const Geo& g, const TileWork& w,
                                           const TileDesc& d) {
  if (w.degrid) spread_descs<true>(g, w, d);
  else spread_descs<false>(g, w, d);
}

// One thread per tile.  Same-address atomics are the cost of this kernel (11.5
// ns each, one after the other), so each list takes one per workgroup of
// kTileWorkThreads tiles, not one per wavefront: 131 072 tiles 40 -> 20 us,
// with degridding's lists behind it 84 -> 30; 524 288 tiles 118 -> 43.
constexpr int kTileWorkThreads = 512;

__global__ __launch_bounds__(kTileWorkThreads) void k_tile_work(
    Geo g, const uint32_t* __restrict__ offsets, TileWork w) {
  // counters[0]: scratch slots taken, [1]: split tiles, [2]: extra items,
  // [4]: tiles with records (listed in busy), [5]: tiles without (idle),
  // [6..7]: 64-bit sum of the records every tile reads.
  uint32_t* counters = w.counters;
  constexpr int NW = kTileWorkThreads / 64;
  __shared__ uint32_t s_cnt[2][NW];
  __shared__ unsigned long long s_reads[NW];
  __shared__ uint32_t s_base[2];
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  const bool live = t < g.ntiles;
  TileRecords r;
  r.work = 0;
  if (live) r = tile_records(g, t, w.degrid, offsets);
  const int wave = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
  const unsigned long long bmask = __ballot(live && r.work > 0);
  const unsigned long long imask = __ballot(live && r.work == 0);
  unsigned long long wsum = r.work;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
    wsum += (unsigned long long)__shfl_xor((long long)wsum, o, 64);
  if (lane == 0) {
    s_cnt[0][wave] = (uint32_t)__popcll(bmask);
    s_cnt[1][wave] = (uint32_t)__popcll(imask);
    s_reads[wave] = wsum;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    uint32_t n = 0;
    for (int q = 0; q < NW; ++q) n += s_cnt[threadIdx.x][q];
    s_base[threadIdx.x] =
        n != 0 ? atomicAdd(&counters[4 + threadIdx.x], n) : 0u;
  } else if (threadIdx.x == 2) {
    unsigned long long reads = 0;
    for (int q = 0; q < NW; ++q) reads += s_reads[q];
    if (reads != 0)
      atomicAdd(reinterpret_cast<unsigned long long*>(&counters[6]), reads);
  }
  __syncthreads();
  const int which = r.work > 0 ? 0 : 1;
  uint32_t at = s_base[which];
  for (int q = 0; q < wave; ++q) at += s_cnt[which][q];
  at += (uint32_t)__popcll((which == 0 ? bmask : imask) &
                           ((1ull << lane) - 1ull));
  uint32_t nch = 0, e0 = 0;
  if (live) nch = emit_tile(g, w, t, r.work, at, counters, e0);
  emit_descs(g, w, tile_desc(w, t, r, nch, at, e0));
}

// ---- two-level partition (no global atomics) ------------------------------
//
// Level 1 sorts the visibilities into coarse buckets (a plane and G rows of
// tiles: all the keys of one bucket are contiguous in key order), level 2
// sorts each bucket by its fine keys (tile column and region).  Both
// levels count in dense LDS histograms and publish one histogram per
// workgroup, so offsets come from scans, never from global atomics.  Both
// scatters first place their workgroup's records in LDS in output order
// (bucket by bucket, or key by key), then write them out as contiguous runs.
//
//   part_count1   placement, key, coarse bucket and the rank within the
//                 workgroup's bucket (LDS atomic); the workgroup's bucket
//                 histogram and its exclusive scan, block-major
//   col_*         bucket-major exclusive scan of the block-major
//                 histograms in place: offset of (bucket, block), and the
//                 bucket bounds
//   part_bounds   one workgroup: bucket bounds and the first level-2 chunk
//                 of every bucket (chunks of one staging area each)
//   part_scatter1 records built from the inputs, staged in LDS in bucket
//                 order, written to their bucket offsets, with their keys
//                 in a separate array (level 2 reads only the keys to
//                 count; the record's spare word carries the key through
//                 the staging)
//   part_count2   per chunk: fine key ranks (LDS atomic), the chunk's
//                 fine-key histogram and its exclusive scan
//   part_scan2    per bucket: chunk-major running sums of every fine key,
//                 the bucket's key offsets (the gridder's offsets table)
//   part_scatter2 records staged in LDS in key order, written to their
//                 key offsets
//
// Workgroups of level 1 and chunks of level 2 hold part_block<R>()
// visibilities: as many records as fit the LDS staging area.

constexpr int kPartThreads = 1024;
// Limits of the direct sort: keys (LDS words of its histogram), and
// visibilities (beyond, its scattered record writes cost more than the
// partition's second level).  Up to kDirectCols histogram words the key
// totals come from the one workgroup of direct_tiles, a thread a key and
// sixteen blocks a round of loads, else from a kernel of their own.  The sort
// in us, that workgroup / the kernel (keys x blocks): 9 x 245 39.6 / 41.2,
// 1152 x 4 18.2 / 19.6, 1008 x 16 17.9 / 18.3, 16128 x 1 41.9 / 42.8; 1152 x
// 15 23.3 / 21.6, 9216 x 2 29.0 / 27.7, 9216 x 7 40.9 / 29.7, 16128 x 4 53.9 /
// 43.2, 1008 x 65 35.0 / 32.7.
constexpr int64_t kDirectKeys = 16384;
constexpr int64_t kDirectVis = 1 << 20;
constexpr uint64_t kDirectCols = 16384;
constexpr int kPartSegs = 64;  // block segments of the level-1 scan

// In-place exclusive scan of n LDS counters (each thread a contiguous run);
// returns the total.  Called by every thread of the workgroup.
__device__ __forceinline__ uint32_t lds_exclusive_scan(uint32_t* s, uint32_t n,
                                                       uint32_t* s_tmp) {
  const uint32_t per = (n + blockDim.x - 1) / blockDim.x;
  const uint32_t f0 = threadIdx.x * per;
  const uint32_t f1 = min(f0 + per, n);
  uint32_t acc = 0;
  for (uint32_t f = f0; f < f1; ++f) acc += s[f];
  uint32_t total;
  uint32_t run = block_exclusive_scan(acc, s_tmp, &total);
  for (uint32_t f = f0; f < f1; ++f) {
    const uint32_t v = s[f];
    s[f] = run;
    run += v;
  }
  __syncthreads();
  return total;
}

template <int V>
__global__ __launch_bounds__(kPartThreads) void k_part_count1(
    Geo g, VisSource src, int64_t m, uint32_t span, uint32_t nbuckets,
    uint2* __restrict__ keyrank, uint32_t* __restrict__ hist1,
    uint32_t* __restrict__ hist1x, uint32_t* __restrict__ btot,
    unsigned long long* __restrict__ dropped) {
  constexpr int PER = V / kPartThreads;
  extern __shared__ uint32_t s_h[];  // nbuckets counters
  __shared__ unsigned long long s_drop;
  __shared__ uint32_t s_tmp[kPartThreads / 64];
  const int tid = threadIdx.x;
  for (uint32_t c = tid; c < nbuckets; c += kPartThreads) s_h[c] = 0u;
  if (tid == 0) s_drop = 0;
  __syncthreads();
  unsigned long long my_drop = 0;
  const int64_t base = (int64_t)blockIdx.x * V;
  double cu[PER], cv[PER], cw[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    int64_t gi = base + (int64_t)e * kPartThreads + tid;
    gi = gi < m ? gi : m - 1;
    source_uvw(src, gi, cu[e], cv[e], cw[e]);
  }
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int64_t gi = base + (int64_t)e * kPartThreads + tid;
    if (gi >= m) continue;
    double x, y;
    int i0, j0, k;
    uint2 kr = make_uint2(kNoKey, 0u);
    if (place(g, cu[e], cv[e], cw[e], x, y, i0, j0, k)) {
      my_drop += (unsigned long long)(g.K * g.K - taps_on_grid(g, i0, j0));
      const uint32_t key = bin_key(g, i0, j0, k);
      kr.x = key;
      kr.y = atomicAdd(&s_h[key / span], 1u);
    } else {
      my_drop += (unsigned long long)(g.K * g.K);
    }
    keyrank[gi] = kr;
  }
  if (dropped != nullptr && my_drop != 0) atomicAdd(&s_drop, my_drop);
  __syncthreads();
  const size_t row = (size_t)blockIdx.x * nbuckets;
  for (uint32_t c = tid; c < nbuckets; c += kPartThreads)
    hist1[row + c] = s_h[c];
  __syncthreads();
  const uint32_t total = lds_exclusive_scan(s_h, nbuckets, s_tmp);
  for (uint32_t c = tid; c < nbuckets; c += kPartThreads)
    hist1x[row + c] = s_h[c];
  if (tid == 0) {
    btot[blockIdx.x] = total;
    if (dropped != nullptr && s_drop != 0) atomicAdd(dropped, s_drop);
  }
}

// Bucket-major exclusive scan of the block-major level-1 histograms
// (hist[b][c], b < nb blocks, c < nc buckets) without a transpose: the
// blocks are cut into nseg segments; col_sum totals each (segment,
// bucket), col_seg scans those over the segments and leaves each bucket's
// total, and col_apply turns the histograms into offsets in place:
//   hist[b][c] <- bounds[c] + sum over b' < b of hist[b'][c],
// bounds[c] the exclusive scan of the bucket totals (computed between
// col_seg and col_apply).
__global__ __launch_bounds__(256) void k_col_sum(
    const uint32_t* __restrict__ hist, uint32_t nb, uint32_t nc,
    uint32_t seglen, uint32_t* __restrict__ seg) {
  const uint32_t c = blockIdx.x * 256u + threadIdx.x;
  const uint32_t s = blockIdx.y;
  if (c >= nc) return;
  const uint32_t b0 = s * seglen, b1 = min(b0 + seglen, nb);
  uint32_t acc = 0;
  for (uint32_t b = b0; b < b1; ++b) acc += hist[(size_t)b * nc + c];
  seg[(size_t)s * nc + c] = acc;
}

__global__ __launch_bounds__(256) void k_col_seg(uint32_t* __restrict__ seg,
                                                 uint32_t nseg, uint32_t nc,
                                                 uint32_t* __restrict__ tot) {
  const uint32_t c = blockIdx.x * 256u + threadIdx.x;
  if (c >= nc) return;
  uint32_t run = 0;
  for (uint32_t s = 0; s < nseg; ++s) {
    const uint32_t v = seg[(size_t)s * nc + c];
    seg[(size_t)s * nc + c] = run;
    run += v;
  }
  tot[c] = run;
}

__global__ __launch_bounds__(256) void k_col_apply(
    uint32_t* __restrict__ hist, uint32_t nb, uint32_t nc, uint32_t seglen,
    const uint32_t* __restrict__ seg, const uint32_t* __restrict__ bounds) {
  const uint32_t c = blockIdx.x * 256u + threadIdx.x;
  const uint32_t s = blockIdx.y;
  if (c >= nc) return;
  const uint32_t b0 = s * seglen, b1 = min(b0 + seglen, nb);
  uint32_t run = bounds[c] + seg[(size_t)s * nc + c];
  // Eight loads in flight before the eight stores.
  uint32_t b = b0;
  for (; b + 8 <= b1; b += 8) {
    uint32_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = hist[(size_t)(b + u) * nc + c];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      hist[(size_t)(b + u) * nc + c] = run;
      run += v[u];
    }
  }
  for (; b < b1; ++b) {
    uint32_t* p = hist + (size_t)b * nc + c;
    const uint32_t v = *p;
    *p = run;
    run += v;
  }
}

// offs1: the scanned (bucket, block) offsets, block-major (one row per
// workgroup); hist1x: the workgroup's own exclusive bucket offsets.
template <typename R, int V>
__global__ __launch_bounds__(kPartThreads) void k_part_scatter1(
    Geo g, VisSource src, int64_t m, const uint2* __restrict__ keyrank,
    const uint32_t* __restrict__ offs1, const uint32_t* __restrict__ hist1x,
    const uint32_t* __restrict__ btot, uint32_t span, uint32_t nbuckets,
    Record<R>* __restrict__ rec, uint32_t* __restrict__ keys, int degrid,
    cplx<R>* __restrict__ vis_out) {
  constexpr int PER = V / kPartThreads;
  extern __shared__ __align__(16) unsigned char s_raw[];
  Record<R>* s_rec = reinterpret_cast<Record<R>*>(s_raw);  // V records
  uint32_t* s_key = reinterpret_cast<uint32_t*>(s_rec + V);  // their keys
  const uint32_t b = blockIdx.x;
  const int64_t base = (int64_t)b * V;
  const uint32_t* ex = hist1x + (size_t)b * nbuckets;
  const uint32_t* off = offs1 + (size_t)b * nbuckets;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int64_t gi = base + (int64_t)e * kPartThreads + threadIdx.x;
    if (gi >= m) continue;
    const uint2 kr = keyrank[gi];
    if (kr.x == kNoKey) {
      if (degrid) vis_out[gi] = cplx<R>{(R)0, (R)0};
      continue;
    }
    const uint32_t slot = ex[kr.x / span] + kr.y;
    s_rec[slot] = make_record<R>(g, src, gi, degrid);
    s_key[slot] = kr.x;  // for the write-out and level 2
  }
  __syncthreads();
  const uint32_t n = btot[b];
  for (uint32_t i = threadIdx.x; i < n; i += kPartThreads) {
    const uint32_t key = s_key[i];
    const uint32_t c = key / span;
    const uint32_t pos = off[c] + (i - ex[c]);
    rec[pos] = s_rec[i];
    keys[pos] = key;
  }
}

// Zeros of the tile work counters and (where asked for) of the strip marks:
// one workgroup of a kernel that runs before the tile work pass.
__device__ __forceinline__ void bin_clear(const BinClear& c) {
  for (uint32_t i = threadIdx.x; i < 16u; i += blockDim.x) c.counters[i] = 0u;
  for (uint32_t i = threadIdx.x; i < c.nstrips; i += blockDim.x)
    c.strips[i] = 0u;
}

// One workgroup: bucket totals (in bounds[], from col_seg) -> bucket bounds
// (exclusive scan, bounds[nbuckets] = total), then chunks per bucket ->
// first chunk of every bucket (chunk0[nbuckets] = total chunks).  Each
// thread takes a contiguous run of buckets (nbuckets <= 16384).
__global__ __launch_bounds__(kPartThreads) void k_part_bounds(
    uint32_t* __restrict__ bounds, uint32_t nbuckets, uint32_t chunk,
    uint32_t* __restrict__ chunk0, BinClear clear) {
  __shared__ uint32_t s_tmp[kPartThreads / 64];
  bin_clear(clear);
  const uint32_t per = (nbuckets + kPartThreads - 1) / kPartThreads;
  const uint32_t c0 = threadIdx.x * per;
  const uint32_t c1 = min(c0 + per, nbuckets);
  uint32_t tot[16];
  uint32_t acc = 0;
  for (uint32_t c = c0; c < c1; ++c) {
    tot[c - c0] = bounds[c];
    acc += tot[c - c0];
  }
  uint32_t total;
  uint32_t run = block_exclusive_scan(acc, s_tmp, &total);
  uint32_t nch = 0;
  for (uint32_t c = c0; c < c1; ++c) {
    bounds[c] = run;
    run += tot[c - c0];
    nch += (tot[c - c0] + chunk - 1) / chunk;
  }
  uint32_t ntotal;
  uint32_t crun = block_exclusive_scan(nch, s_tmp, &ntotal);
  for (uint32_t c = c0; c < c1; ++c) {
    chunk0[c] = crun;
    crun += (tot[c - c0] + chunk - 1) / chunk;
  }
  if (threadIdx.x == 0) {
    bounds[nbuckets] = total;
    chunk0[nbuckets] = ntotal;
  }
}

// The whole level-1 scan (col_sum, col_seg, part_bounds, col_apply) in one
// workgroup, for histograms of at most kSmallScan words: four launches of a
// few microseconds each become one (28 -> 13 us for 244 workgroups of 256
// buckets).  Thread (segment, bucket) sums its run of blocks eight loads at
// a time; more than 1024 buckets take one segment and several turns.  At most
// kSmallSegs segments, which one thread a bucket adds up in turn (with a
// thread for every segment that fits, 1024 of them for one bucket, 27 us).
constexpr uint32_t kSmallScan = 65536;
constexpr uint32_t kSmallSegs = 32;

__global__ __launch_bounds__(kPartThreads) void k_part_scan1_small(
    uint32_t* __restrict__ hist, uint32_t nb, uint32_t nc, uint32_t chunk,
    uint32_t* __restrict__ bounds, uint32_t* __restrict__ chunk0,
    BinClear clear) {
  extern __shared__ uint32_t s_bkt[];  // nc words, then kPartThreads
  uint32_t* s_seg = s_bkt + nc;
  __shared__ uint32_t s_tmp[kPartThreads / 64];
  bin_clear(clear);
  const uint32_t nseg =
      nc >= kPartThreads ? 1u : min(kPartThreads / nc, kSmallSegs);
  const uint32_t seg = threadIdx.x / nc, c0 = threadIdx.x % nc;
  const bool on = nc >= kPartThreads || seg < nseg;
  const uint32_t first = nc >= kPartThreads ? threadIdx.x : c0;
  const uint32_t step = nc >= kPartThreads ? (uint32_t)kPartThreads : nc;
  const uint32_t sg = nc >= kPartThreads ? 0u : seg;
  const uint32_t seglen = (nb + nseg - 1) / nseg;
  const uint32_t b0 = min(sg * seglen, nb), b1 = min(b0 + seglen, nb);
  auto column = [&](uint32_t c) {
    uint32_t acc = 0, b = b0;
    for (; b + 8 <= b1; b += 8) {
      uint32_t v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = hist[(size_t)(b + u) * nc + c];
#pragma unroll
      for (int u = 0; u < 8; ++u) acc += v[u];
    }
    for (; b < b1; ++b) acc += hist[(size_t)b * nc + c];
    return acc;
  };
  if (on) {
    for (uint32_t c = first; c < nc; c += step) {
      const uint32_t v = column(c);
      if (nseg > 1) s_seg[sg * nc + c] = v;
      else s_bkt[c] = v;
    }
  }
  __syncthreads();
  if (nseg > 1 && threadIdx.x < nc) {
    uint32_t run = 0;
    for (uint32_t q = 0; q < nseg; ++q) {
      const uint32_t v = s_seg[q * nc + threadIdx.x];
      s_seg[q * nc + threadIdx.x] = run;
      run += v;
    }
    s_bkt[threadIdx.x] = run;
  }
  __syncthreads();
  // Level-2 chunks, then bucket bounds, both exclusive scans over buckets.
  const uint32_t per = (nc + kPartThreads - 1) / kPartThreads;
  const uint32_t k0 = min(threadIdx.x * per, nc), k1 = min(k0 + per, nc);
  uint32_t nch = 0;
  for (uint32_t c = k0; c < k1; ++c) nch += (s_bkt[c] + chunk - 1) / chunk;
  uint32_t ntotal;
  uint32_t crun = block_exclusive_scan(nch, s_tmp, &ntotal);
  for (uint32_t c = k0; c < k1; ++c) {
    chunk0[c] = crun;
    crun += (s_bkt[c] + chunk - 1) / chunk;
  }
  const uint32_t total = lds_exclusive_scan(s_bkt, nc, s_tmp);
  for (uint32_t c = threadIdx.x; c < nc; c += kPartThreads)
    bounds[c] = s_bkt[c];
  if (threadIdx.x == 0) {
    bounds[nc] = total;
    chunk0[nc] = ntotal;
  }
  if (on) {
    for (uint32_t c = first; c < nc; c += step) {
      uint32_t run = s_bkt[c] + (nseg > 1 ? s_seg[sg * nc + c] : 0u);
      uint32_t b = b0;
      for (; b + 8 <= b1; b += 8) {
        uint32_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = hist[(size_t)(b + u) * nc + c];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          hist[(size_t)(b + u) * nc + c] = run;
          run += v[u];
        }
      }
      for (; b < b1; ++b) {
        uint32_t* p = hist + (size_t)b * nc + c;
        const uint32_t v = *p;
        *p = run;
        run += v;
      }
    }
  }
}

// Bucket of chunk ch: the last c with chunk0[c] <= ch (chunk0 exclusive
// scan of the chunk counts, chunk0[nbuckets] = total), i.e. the bucket
// that owns the chunk even when empty buckets share its chunk0 value.
__device__ __forceinline__ uint32_t chunk_bucket(const uint32_t* chunk0,
                                                 uint32_t nbuckets,
                                                 uint32_t ch) {
  uint32_t lo = 0, hi = nbuckets;  // chunk0[lo] <= ch < chunk0[hi]
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (chunk0[mid] <= ch) lo = mid;
    else hi = mid;
  }
  return lo;
}

template <int V>
__global__ __launch_bounds__(kPartThreads) void k_part_count2(
    const uint32_t* __restrict__ keys, const uint32_t* __restrict__ bounds,
    const uint32_t* __restrict__ chunk0, uint32_t nbuckets, uint32_t span,
    uint32_t* __restrict__ rank2, uint32_t* __restrict__ hist2,
    uint32_t* __restrict__ hist2x) {
  extern __shared__ uint32_t s_h[];  // span counters
  __shared__ uint32_t s_tmp[kPartThreads / 64];
  const uint32_t ch = blockIdx.x;
  if (ch >= chunk0[nbuckets]) return;
  const uint32_t c = chunk_bucket(chunk0, nbuckets, ch);
  const uint32_t start = bounds[c] + (ch - chunk0[c]) * V;
  const uint32_t end = min(start + (uint32_t)V, bounds[c + 1]);
  for (uint32_t f = threadIdx.x; f < span; f += kPartThreads) s_h[f] = 0u;
  __syncthreads();
  const uint32_t kb = c * span;
  for (uint32_t r = start + threadIdx.x; r < end; r += kPartThreads)
    rank2[r] = atomicAdd(&s_h[keys[r] - kb], 1u);
  __syncthreads();
  const size_t row = (size_t)ch * span;
  for (uint32_t f = threadIdx.x; f < span; f += kPartThreads)
    hist2[row + f] = s_h[f];
  __syncthreads();
  lds_exclusive_scan(s_h, span, s_tmp);
  for (uint32_t f = threadIdx.x; f < span; f += kPartThreads)
    hist2x[row + f] = s_h[f];
}

// One workgroup per bucket: hist2 of its chunks becomes the offset of
// every (chunk, fine key) share, and offsets[] of its keys is written.
__global__ __launch_bounds__(kPartThreads) void k_part_scan2(
    const uint32_t* __restrict__ bounds, const uint32_t* __restrict__ chunk0,
    uint32_t nbuckets, uint32_t span, uint32_t* __restrict__ hist2,
    uint32_t* __restrict__ offsets) {
  extern __shared__ uint32_t s_tot[];  // span totals
  __shared__ uint32_t s_tmp[kPartThreads / 64];
  const uint32_t c = blockIdx.x;
  const uint32_t base = bounds[c];
  const uint32_t q0 = chunk0[c], q1 = chunk0[c + 1];
  for (uint32_t f = threadIdx.x; f < span; f += kPartThreads) {
    uint32_t run = 0;
    uint32_t q = q0;
    for (; q + 8 <= q1; q += 8) {  // eight loads in flight, then the stores
      uint32_t v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = hist2[(size_t)(q + u) * span + f];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        hist2[(size_t)(q + u) * span + f] = run;
        run += v[u];
      }
    }
    for (; q < q1; ++q) {
      uint32_t* p = hist2 + (size_t)q * span + f;
      const uint32_t v = *p;
      *p = run;
      run += v;
    }
    s_tot[f] = run;
  }
  __syncthreads();
  lds_exclusive_scan(s_tot, span, s_tmp);
  for (uint32_t f = threadIdx.x; f < span; f += kPartThreads) {
    const uint32_t o = base + s_tot[f];
    offsets[(size_t)c * span + f] = o;
    for (uint32_t q = q0; q < q1; ++q) hist2[(size_t)q * span + f] += o;
  }
  if (c + 1 == nbuckets && threadIdx.x == 0)
    offsets[(size_t)nbuckets * span] = bounds[nbuckets];
}

template <typename R, int V>
__global__ __launch_bounds__(kPartThreads) void k_part_scatter2(
    const uint32_t* __restrict__ keys, const uint32_t* __restrict__ bounds,
    const uint32_t* __restrict__ chunk0, uint32_t nbuckets, uint32_t span,
    const uint32_t* __restrict__ rank2, const uint32_t* __restrict__ hist2,
    const uint32_t* __restrict__ hist2x,
    const Record<R>* __restrict__ rec1, Record<R>* __restrict__ rec) {
  extern __shared__ __align__(16) unsigned char s_raw[];
  Record<R>* s_rec = reinterpret_cast<Record<R>*>(s_raw);  // V records
  uint32_t* s_fine = reinterpret_cast<uint32_t*>(s_rec + V);  // fine keys
  const uint32_t ch = blockIdx.x;
  if (ch >= chunk0[nbuckets]) return;
  const uint32_t c = chunk_bucket(chunk0, nbuckets, ch);
  const uint32_t start = bounds[c] + (ch - chunk0[c]) * V;
  const uint32_t end = min(start + (uint32_t)V, bounds[c + 1]);
  const uint32_t* off = hist2 + (size_t)ch * span;
  const uint32_t* ex = hist2x + (size_t)ch * span;
  const uint32_t kb = c * span;
  for (uint32_t r = start + threadIdx.x; r < end; r += kPartThreads) {
    const uint32_t f = keys[r] - kb;
    const uint32_t slot = ex[f] + rank2[r];
    s_rec[slot] = rec1[r];
    s_fine[slot] = f;
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < end - start; i += kPartThreads) {
    const uint32_t f = s_fine[i];
    rec[off[f] + (i - ex[f])] = s_rec[i];
  }
}

// ---- direct sort (small plans) --------------------------------------------
//
// Where all keys of a plan fit one dense LDS histogram (kDirectKeys) the
// partition needs no second level, and its single-workgroup scans no launches
// of their own.  Small calls are bound by the number of launches (~4 us
// each): this sort and the tile work take three or four of them, the
// partition and its tile work ten.
//
//   direct_count    placement, key and rank within the workgroup's key (LDS
//                   atomic); the workgroup's key histogram, block-major
//   direct_cols     histograms -> running sums over the blocks, key totals
//                   (only where direct_tiles would be slow to do it itself)
//   direct_tiles    one workgroup: key offsets, then the tile work pass
//   direct_scatter  records to offset[key] + sum of earlier blocks + rank

template <int V>
__global__ __launch_bounds__(kPartThreads) void k_direct_count(
    Geo g, VisSource src, int64_t m, uint32_t nkeys,
    uint2* __restrict__ keyrank, uint32_t* __restrict__ hist,
    unsigned long long* __restrict__ dropped) {
  constexpr int PER = V / kPartThreads;
  extern __shared__ uint32_t s_h[];  // nkeys counters
  __shared__ unsigned long long s_drop;
  const int tid = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.x * V;
  double cu[PER], cv[PER], cw[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    int64_t gi = base + (int64_t)e * kPartThreads + tid;
    gi = gi < m ? gi : m - 1;
    source_uvw(src, gi, cu[e], cv[e], cw[e]);
  }
  for (uint32_t c = tid; c < nkeys; c += kPartThreads) s_h[c] = 0u;
  if (tid == 0) s_drop = 0;
  __syncthreads();
  unsigned long long my_drop = 0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int64_t gi = base + (int64_t)e * kPartThreads + tid;
    if (gi >= m) continue;
    double x, y;
    int i0, j0, k;
    uint2 kr = make_uint2(kNoKey, 0u);
    if (place(g, cu[e], cv[e], cw[e], x, y, i0, j0, k)) {
      my_drop += (unsigned long long)(g.K * g.K - taps_on_grid(g, i0, j0));
      kr.x = bin_key(g, i0, j0, k);
      kr.y = atomicAdd(&s_h[kr.x], 1u);
    } else {
      my_drop += (unsigned long long)(g.K * g.K);
    }
    keyrank[gi] = kr;
  }
  if (dropped != nullptr && my_drop != 0) atomicAdd(&s_drop, my_drop);
  __syncthreads();
  const size_t row = (size_t)blockIdx.x * nkeys;
  for (uint32_t c = tid; c < nkeys; c += kPartThreads) hist[row + c] = s_h[c];
  if (tid == 0 && dropped != nullptr && s_drop != 0)
    atomicAdd(dropped, s_drop);
}

// Running sums of key c over the blocks, in place; returns its total.
__device__ __forceinline__ uint32_t direct_column(uint32_t* hist, uint32_t nb,
                                                  uint32_t nkeys, uint32_t c) {
  uint32_t run = 0, b = 0;
  for (; b + 16 <= nb; b += 16) {
    uint32_t v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = hist[(size_t)(b + u) * nkeys + c];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      hist[(size_t)(b + u) * nkeys + c] = run;
      run += v[u];
    }
  }
  for (; b < nb; ++b) {
    const uint32_t v = hist[(size_t)b * nkeys + c];
    hist[(size_t)b * nkeys + c] = run;
    run += v;
  }
  return run;
}

__global__ __launch_bounds__(64) void k_direct_cols(
    uint32_t* __restrict__ hist, uint32_t nb, uint32_t nkeys,
    uint32_t* __restrict__ totals) {
  const uint32_t c = blockIdx.x * 64u + threadIdx.x;
  if (c < nkeys) totals[c] = direct_column(hist, nb, nkeys, c);
}

// One workgroup.  offsets[] holds the key totals (direct_cols), or nothing
// yet (COLS: the running sums are formed here).
template <bool COLS>
__global__ __launch_bounds__(kPartThreads) void k_direct_tiles(
    Geo g, uint32_t* hist, uint32_t nb, uint32_t nkeys, uint32_t* offsets,
    TileWork w, BinClear clear) {
  extern __shared__ uint32_t s_off[];  // nkeys + 1
  __shared__ uint32_t s_tmp[kPartThreads / 64];
  __shared__ uint32_t s_ctr[8];
  __shared__ unsigned long long s_reads;
  for (uint32_t i = threadIdx.x; i < clear.nstrips; i += kPartThreads)
    clear.strips[i] = 0u;
  if (threadIdx.x < 8) s_ctr[threadIdx.x] = 0u;
  if (threadIdx.x == 0) s_reads = 0ull;
  for (uint32_t c = threadIdx.x; c < nkeys; c += kPartThreads)
    s_off[c] = COLS ? direct_column(hist, nb, nkeys, c) : offsets[c];
  __syncthreads();  // also orders the strip zeros before their marks
  const uint32_t total = lds_exclusive_scan(s_off, nkeys, s_tmp);
  if (threadIdx.x == 0) s_off[nkeys] = total;
  __syncthreads();
  for (uint32_t c = threadIdx.x; c <= nkeys; c += kPartThreads)
    offsets[c] = s_off[c];
  for (;;) {
    for (int t0 = 0; t0 < g.ntiles; t0 += kPartThreads) {
      const int t = t0 + (int)threadIdx.x;
      const bool live = t < g.ntiles;
      TileRecords r;
      r.work = 0;
      if (live) r = tile_records(g, t, w.degrid, s_off);
      const uint32_t ib = wave_append(&s_ctr[4], live && r.work > 0);
      const uint32_t ii = wave_append(&s_ctr[5], live && r.work == 0);
      if (r.work > 0) atomicAdd(&s_reads, (unsigned long long)r.work);
      const uint32_t at = r.work > 0 ? ib : ii;
      uint32_t nch = 0, e0 = 0;
      if (live) nch = emit_tile(g, w, t, r.work, at, s_ctr, e0);
      emit_descs(g, w, tile_desc(w, t, r, nch, at, e0));
    }
    __syncthreads();
    // Scratch slots ran out (never in degridding, which takes none): all
    // over again with larger items, rather than tiles of any size in one
    // item.  Ends at the latest where an item holds the largest tile.
    if (s_ctr[0] <= w.max_slots) break;
    __threadfence();
    __syncthreads();
    if (threadIdx.x < 8) s_ctr[threadIdx.x] = 0u;
    if (threadIdx.x == 0) s_reads = 0ull;
    w.chunk *= 2u;
    __syncthreads();
  }
  if (threadIdx.x < 6) w.counters[threadIdx.x] = s_ctr[threadIdx.x];
  if (threadIdx.x == 6) w.counters[6] = (uint32_t)s_reads;
  if (threadIdx.x == 7) w.counters[7] = (uint32_t)(s_reads >> 32);
}

template <typename R, int V>
__global__ __launch_bounds__(256) void k_direct_scatter(
    Geo g, VisSource src, int64_t m, const uint2* __restrict__ keyrank,
    const uint32_t* __restrict__ hist, uint32_t nkeys,
    const uint32_t* __restrict__ offsets, Record<R>* __restrict__ rec,
    int degrid, cplx<R>* __restrict__ vis_out) {
  const int64_t gi = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gi >= m) return;
  const uint2 kr = keyrank[gi];
  if (kr.x == kNoKey) {
    if (degrid) vis_out[gi] = cplx<R>{(R)0, (R)0};
    return;
  }
  const uint32_t pos =
      offsets[kr.x] + hist[(size_t)(gi / V) * nkeys + kr.x] + kr.y;
  rec[pos] = make_record<R>(g, src, gi, degrid);
}

}  // namespace

// Two-level partition of m visibilities (see the kernels above), in the
// phases the library times separately.
namespace {
template <typename R>
constexpr int part_block() {
  // LDS staging of one workgroup: 4096 24-byte (FP32) or 2048 40-byte
  // (FP64) records and their keys.
  return sizeof(R) == 4 ? 4096 : 2048;
}
int part_block_of(int elem) { return elem == 8 ? 4096 : 2048; }
uint32_t part_nb1(int64_t m, int V) {
  const int64_t nb = (m + V - 1) / V;
  return (uint32_t)(nb > 0 ? nb : 1);
}
uint32_t part_max_chunks(int64_t m, uint32_t nbuckets, int V) {
  return (uint32_t)((m + V - 1) / V) + nbuckets;
}
}  // namespace

template <typename R>
void launch_part_count1(const Geo& g, const VisSource& src, int64_t m,
                        const PartWork& w, unsigned long long* dropped,
                        hipStream_t st) {
  if (m == 0) return;
  constexpr int V = part_block<R>();
  hipLaunchKernelGGL(k_part_count1<V>, dim3(part_nb1(m, V)),
                     dim3(kPartThreads), (size_t)w.nbuckets * 4, st, g, src, m,
                     w.span, w.nbuckets, w.keyrank, w.hist1, w.hist1x, w.btot,
                     dropped);
}

template <typename R>
void launch_part_scan1(int64_t m, const PartWork& w, hipStream_t st) {
  constexpr int V = part_block<R>();
  const uint32_t C = w.nbuckets;
  if (m > 0 && (uint64_t)part_nb1(m, V) * C <= kSmallScan) {
    hipLaunchKernelGGL(k_part_scan1_small, dim3(1), dim3(kPartThreads),
                       (size_t)(C + kPartThreads) * 4, st, w.hist1,
                       part_nb1(m, V), C, (uint32_t)V, w.bounds, w.chunk0,
                       w.clear);
    return;
  }
  const dim3 cg((C + 255) / 256);
  if (m > 0) {
    const uint32_t nb1 = part_nb1(m, V);
    const uint32_t nseg = nb1 < (uint32_t)kPartSegs ? nb1 : (uint32_t)kPartSegs;
    const uint32_t seglen = (nb1 + nseg - 1) / nseg;
    hipLaunchKernelGGL(k_col_sum, dim3(cg.x, nseg), dim3(256), 0, st,
                       w.hist1, nb1, C, seglen, w.seg);
    hipLaunchKernelGGL(k_col_seg, cg, dim3(256), 0, st, w.seg, nseg, C,
                       w.bounds);
  } else {
    launch_zero_u32(w.bounds, (int64_t)C + 1, st);
  }
  hipLaunchKernelGGL(k_part_bounds, dim3(1), dim3(kPartThreads), 0, st,
                     w.bounds, C, (uint32_t)V, w.chunk0, w.clear);
  if (m > 0) {
    const uint32_t nb1 = part_nb1(m, V);
    const uint32_t nseg = nb1 < (uint32_t)kPartSegs ? nb1 : (uint32_t)kPartSegs;
    const uint32_t seglen = (nb1 + nseg - 1) / nseg;
    hipLaunchKernelGGL(k_col_apply, dim3(cg.x, nseg), dim3(256), 0, st,
                       w.hist1, nb1, C, seglen, w.seg, w.bounds);
  }
}

template <typename R>
void launch_part_scatter1(const Geo& g, const VisSource& src, int64_t m,
                          const PartWork& w, int degrid, void* vis_out,
                          hipStream_t st) {
  if (m == 0) return;
  constexpr int V = part_block<R>();
  hipLaunchKernelGGL((k_part_scatter1<R, V>), dim3(part_nb1(m, V)),
                     dim3(kPartThreads), (size_t)V * (sizeof(Record<R>) + 4),
                     st, g, src, m, w.keyrank, w.hist1, w.hist1x, w.btot,
                     w.span, w.nbuckets, (Record<R>*)w.rec1, w.keys, degrid,
                     (cplx<R>*)vis_out);
}

template <typename R>
void launch_part_count2(int64_t m, const PartWork& w, hipStream_t st) {
  if (m == 0) return;
  constexpr int V = part_block<R>();
  hipLaunchKernelGGL(k_part_count2<V>,
                     dim3(part_max_chunks(m, w.nbuckets, V)),
                     dim3(kPartThreads), (size_t)w.span * 4, st, w.keys,
                     w.bounds, w.chunk0, w.nbuckets, w.span, w.rank2, w.hist2,
                     w.hist2x);
}

template <typename R>
void launch_part_scan2(int64_t, const PartWork& w, hipStream_t st) {
  hipLaunchKernelGGL(k_part_scan2, dim3(w.nbuckets), dim3(kPartThreads),
                     (size_t)w.span * 4, st, w.bounds, w.chunk0, w.nbuckets,
                     w.span, w.hist2, w.offsets);
}

template <typename R>
void launch_part_scatter2(int64_t m, const PartWork& w, hipStream_t st) {
  if (m == 0) return;
  constexpr int V = part_block<R>();
  hipLaunchKernelGGL((k_part_scatter2<R, V>),
                     dim3(part_max_chunks(m, w.nbuckets, V)),
                     dim3(kPartThreads), (size_t)V * (sizeof(Record<R>) + 4),
                     st, w.keys, w.bounds, w.chunk0, w.nbuckets, w.span, w.rank2,
                     w.hist2, w.hist2x, (const Record<R>*)w.rec1,
                     (Record<R>*)w.rec);
}

#define WS_INST(R)                                                           \
  template void launch_part_count1<R>(const Geo&, const VisSource&, int64_t, \
                                      const PartWork&, unsigned long long*, \
                                      hipStream_t);                         \
  template void launch_part_scan1<R>(int64_t, const PartWork&, hipStream_t); \
  template void launch_part_scatter1<R>(const Geo&, const VisSource&,       \
                                        int64_t, const PartWork&, int,      \
                                        void*, hipStream_t);                \
  template void launch_part_count2<R>(int64_t, const PartWork&,             \
                                      hipStream_t);                         \
  template void launch_part_scan2<R>(int64_t, const PartWork&, hipStream_t); \
  template void launch_part_scatter2<R>(int64_t, const PartWork&,           \
                                        hipStream_t);
WS_INST(float)
WS_INST(double)
#undef WS_INST

namespace {
// Visibilities of one counting workgroup: few enough workgroups that the
// histograms stay smaller than the records, enough of them for small calls.
constexpr int kDirectSmall = 1024, kDirectLarge = 4096;
bool direct_large(int64_t max_vis, int64_t nkeys) {
  return max_vis > 65536 || nkeys > 4096;
}
}  // namespace

int64_t direct_hist_words(int64_t max_vis, int64_t nkeys) {
  const int V = direct_large(max_vis, nkeys) ? kDirectLarge : kDirectSmall;
  return (max_vis + V - 1) / V * nkeys;
}

bool direct_fits(int64_t max_vis, int64_t nkeys) {
  return nkeys <= kDirectKeys && max_vis <= kDirectVis;
}

template <typename R>
void launch_direct_sort(const Geo& g, const VisSource& src, int64_t m,
                        int64_t max_vis, const DirectWork& w,
                        const TileWork& tw, const BinClear& clear,
                        unsigned long long* dropped, void* vis_out,
                        hipStream_t st) {
  const bool large = direct_large(max_vis, w.nkeys);
  const int V = large ? kDirectLarge : kDirectSmall;
  const uint32_t nb = (uint32_t)((m + V - 1) / V);
  if (m > 0) {
    if (large)
      hipLaunchKernelGGL(k_direct_count<kDirectLarge>, dim3(nb),
                         dim3(kPartThreads), (size_t)w.nkeys * 4, st, g, src,
                         m, w.nkeys, w.keyrank, w.hist, dropped);
    else
      hipLaunchKernelGGL(k_direct_count<kDirectSmall>, dim3(nb),
                         dim3(kPartThreads), (size_t)w.nkeys * 4, st, g, src,
                         m, w.nkeys, w.keyrank, w.hist, dropped);
  }
  const size_t lds = (size_t)(w.nkeys + 1) * 4;
  if ((uint64_t)nb * w.nkeys <= kDirectCols) {
    hipLaunchKernelGGL(k_direct_tiles<true>, dim3(1), dim3(kPartThreads), lds,
                       st, g, w.hist, nb, w.nkeys, w.offsets, tw, clear);
  } else {
    hipLaunchKernelGGL(k_direct_cols, dim3((w.nkeys + 63) / 64), dim3(64), 0,
                       st, w.hist, nb, w.nkeys, w.offsets);
    hipLaunchKernelGGL(k_direct_tiles<false>, dim3(1), dim3(kPartThreads),
                       lds, st, g, w.hist, nb, w.nkeys, w.offsets, tw, clear);
  }
  if (m == 0) return;
  const dim3 sg((unsigned)((m + 255) / 256));
  if (large)
    hipLaunchKernelGGL((k_direct_scatter<R, kDirectLarge>), sg, dim3(256), 0,
                       st, g, src, m, w.keyrank, w.hist, w.nkeys, w.offsets,
                       (Record<R>*)w.rec, tw.degrid, (cplx<R>*)vis_out);
  else
    hipLaunchKernelGGL((k_direct_scatter<R, kDirectSmall>), sg, dim3(256), 0,
                       st, g, src, m, w.keyrank, w.hist, w.nkeys, w.offsets,
                       (Record<R>*)w.rec, tw.degrid, (cplx<R>*)vis_out);
}

template void launch_direct_sort<float>(const Geo&, const VisSource&, int64_t,
                                        int64_t, const DirectWork&,
                                        const TileWork&, const BinClear&,
                                        unsigned long long*, void*,
                                        hipStream_t);
template void launch_direct_sort<double>(const Geo&, const VisSource&,
                                         int64_t, int64_t, const DirectWork&,
                                         const TileWork&, const BinClear&,
                                         unsigned long long*, void*,
                                         hipStream_t);

int64_t partition_blocks(int64_t max_vis, int elem) {
  const int V = part_block_of(elem);
  return (max_vis + V - 1) / V;
}
int64_t partition_chunks(int64_t max_vis, int64_t nbuckets, int elem) {
  const int V = part_block_of(elem);
  return (max_vis + V - 1) / V + nbuckets;
}

void launch_bin_count(const Geo& g, const VisSource& src, int64_t m,
                      uint32_t* copies, uint32_t nkeys, uint2* keyrank,
                      unsigned long long* dropped, hipStream_t st) {
  if (m == 0) return;
  const int64_t nb = (m + kCountPerBlock - 1) / kCountPerBlock;
  hipLaunchKernelGGL(k_bin_count, dim3((unsigned)nb), dim3(kCountThreads), 0,
                     st, g, src, m, copies, nkeys, keyrank, dropped);
}

void launch_fold_copies(const uint32_t* copies, uint32_t nkeys,
                        uint32_t* totals, hipStream_t st) {
  hipLaunchKernelGGL(k_fold_copies, dim3((nkeys + 255) / 256), dim3(256), 0,
                     st, copies, nkeys, totals);
}

void launch_copy_offsets(uint32_t* copies, uint32_t nkeys,
                         const uint32_t* offsets, hipStream_t st) {
  hipLaunchKernelGGL(k_copy_offsets, dim3((nkeys + 255) / 256), dim3(256), 0,
                     st, copies, nkeys, offsets);
}

int64_t scan_sums_len(int64_t n) { return (n + kScanBlock - 1) / kScanBlock + 1; }

void launch_exclusive_scan(const uint32_t* in, uint32_t* out, int64_t n,
                           uint32_t* sums, hipStream_t st) {
  // out has n + 1 entries; out[n] = total.  in may alias out.
  const int64_t nb = (n + kScanBlock - 1) / kScanBlock;
  hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(kScanThreads), 0,
                     st, in, n, sums);
  hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(1024), 0, st, sums, nb);
  hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nb), dim3(kScanThreads), 0,
                     st, in, out, n, sums, nb);
}

template <typename R>
void launch_bin_scatter(const Geo& g, const VisSource& src, int64_t m,
                        const uint2* keyrank, const uint32_t* offsets,
                        uint32_t nkeys, void* records, int degrid,
                        void* vis_out, hipStream_t st) {
  if (m == 0) return;
  const int64_t nb = (m + 255) / 256;
  hipLaunchKernelGGL(k_bin_scatter<R>, dim3((unsigned)nb), dim3(256), 0, st, g,
                     src, m, keyrank, offsets, nkeys, (Record<R>*)records,
                     degrid, (cplx<R>*)vis_out);
}

template void launch_bin_scatter<float>(const Geo&, const VisSource&, int64_t,
                                        const uint2*, const uint32_t*,
                                        uint32_t, void*, int, void*,
                                        hipStream_t);
template void launch_bin_scatter<double>(const Geo&, const VisSource&,
                                         int64_t, const uint2*,
                                         const uint32_t*, uint32_t, void*,
                                         int, void*, hipStream_t);

void launch_tile_work(const Geo& g, const uint32_t* offsets,
                      const TileWork& w, hipStream_t st) {
  const int nb = (g.ntiles + kTileWorkThreads - 1) / kTileWorkThreads;
  hipLaunchKernelGGL(k_tile_work, dim3(nb), dim3(kTileWorkThreads), 0, st, g,
                     offsets, w);
}

}  // namespace ws
