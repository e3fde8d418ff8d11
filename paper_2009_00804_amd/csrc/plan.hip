// Graph layout on the GPU: CSR validation, in/out degrees, degree-sorted row
// order (stable LSD radix sort, largest degree first), row segments of at
// most seg_len edges and row blocks of bounded cost.
//
// The degree skew of real graphs follows a power law (Sec. 3.2, Fig. 8a of
// the paper); batching vertices by degree as the profiled library did left
// the GPU idle (Fig. 8b/c).  Here the sorted order only schedules work: rows
// of similar degree share a workgroup, the heaviest rows start first, and a
// row longer than seg_len is split across several lanes groups so that no
// single wave walks a hub row alone.
#include "saga_device.h"
#include "saga_internal.h"

namespace saga {
namespace {

constexpr int kThreads = 256;
constexpr int kItems = 8;
constexpr int kTile = kThreads * kItems;  // 2048 items per workgroup tile
constexpr int kBins = 256;                // 8-bit radix digits

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// ------------------------------------------------------------------------
// block-wide scans (blockDim.x == NT)
// ------------------------------------------------------------------------
__device__ __forceinline__ int32_t wave_incl_scan(int32_t v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    int32_t y = __shfl_up(v, off, 64);
    if (lane >= off) v += y;
  }
  return v;
}

template <int NT>
__device__ __forceinline__ int32_t block_excl_scan(int32_t v, int32_t* total) {
  __shared__ int32_t ws[NT / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int32_t incl = wave_incl_scan(v);
  if (lane == 63) ws[wave] = incl;
  __syncthreads();
  int32_t off = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < NT / 64; ++k) {
    if (k < wave) off += ws[k];
    tot += ws[k];
  }
  __syncthreads();
  *total = tot;
  return off + incl - v;
}

// the in-degree behind a degree-order sort key (key = 0x7fffffff - d_in)
__device__ __forceinline__ int32_t key_degree(uint32_t key) { return (int32_t)(0x7fffffffu - key); }
// number of segments of a row of d edges
__device__ __forceinline__ int32_t seg_count(int32_t d, int32_t T) { return d > T ? (d + T - 1) / T : 1; }

// ------------------------------------------------------------------------
// kernels
// ------------------------------------------------------------------------
// The out-degree count and the row order may run on two streams at once, so
// neither looks at the errors the other can raise meanwhile: the count at a bad
// col_idx only, the row order (which never reads col_idx) at everything else.
// Both were raised by earlier kernels of the reader's own stream, so that every
// wave reads the same.
__device__ __forceinline__ bool count_stops(const int32_t* counts) { return counts[kErrFlags] & kErrCol; }
__device__ __forceinline__ bool order_stops(const int32_t* counts) { return counts[kErrFlags] & ~kErrCol; }
// for kernels that may themselves raise kErrInternal: one answer per workgroup
__device__ __forceinline__ bool order_stops_wg(const int32_t* counts) {
  return __syncthreads_or(threadIdx.x == 0 && order_stops(counts));
}

__global__ void k_zero(int32_t* p, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0;
}

// d_in, d_out (with global atomics) and CSR validation; error bits go to
// counts[kErrFlags].  Only for graphs without the bucketed count below.
__global__ __launch_bounds__(kThreads) void k_degrees(const int32_t* __restrict__ rp,
                                                      const int32_t* __restrict__ col, int32_t V,
                                                      int32_t Vs, int64_t E, int32_t* d_in,
                                                      int32_t* d_out, int32_t* counts) {
  int err = 0;
  int maxd = 0;
  const int64_t n = V > E ? (int64_t)V : E;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    if (i < V) {
      int32_t a = rp[i], b = rp[i + 1];
      if (b < a) err |= 2;
      int32_t d = b - a;
      d = d < 0 ? 0 : d;
      d_in[i] = d;
      maxd = d > maxd ? d : maxd;
      if (i == 0) {
        if (a != 0) err |= 1;
        if ((int64_t)rp[V] != E) err |= 4;
      }
    }
    if (i < E) {
      int32_t c = col[i];
      if (c < 0 || c >= Vs)
        err |= kErrCol;
      else
        atomicAdd(&d_out[c], 1);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    err |= __shfl_xor(err, off, 64);
    int m = __shfl_xor(maxd, off, 64);
    maxd = m > maxd ? m : maxd;
  }
  // one atomic per workgroup (same-address atomics serialize)
  __shared__ int s_err[kThreads / 64], s_max[kThreads / 64];
  if ((threadIdx.x & 63) == 0) {
    s_err[threadIdx.x >> 6] = err;
    s_max[threadIdx.x >> 6] = maxd;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < kThreads / 64; ++k) {
      err |= s_err[k];
      maxd = s_max[k] > maxd ? s_max[k] : maxd;
    }
    if (err) atomicOr(&counts[kErrFlags], err);
    // most workgroups already see a larger maximum: skip their atomic
    if (maxd > __hip_atomic_load(&counts[kMaxDegree], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(&counts[kMaxDegree], maxd);
  }
}

// d_in, row_ptr validation and, per tile of kTile rows, the histogram of the
// first radix digit (graphs whose out-degrees are counted in buckets)
__global__ __launch_bounds__(kThreads) void k_degrees_hist(const int32_t* __restrict__ rp, int32_t V,
                                                           int64_t E, int32_t* __restrict__ d_in,
                                                           int32_t* __restrict__ hist, int64_t ntiles,
                                                           int32_t* counts) {
  __shared__ int32_t h[kBins];
  __shared__ int s_err[kThreads / 64], s_max[kThreads / 64];
  const int64_t tile = blockIdx.x;
  h[threadIdx.x] = 0;
  __syncthreads();
  int err = 0, maxd = 0;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int64_t i = tile * kTile + j * kThreads + threadIdx.x;
    if (i < V) {
      const int32_t a = rp[i], b = rp[i + 1];
      if (b < a) err |= 2;
      int32_t d = b - a;
      d = d < 0 ? 0 : d;
      d_in[i] = d;
      maxd = d > maxd ? d : maxd;
      if (i == 0) {
        if (a != 0) err |= 1;
        if ((int64_t)rp[V] != E) err |= 4;
      }
      atomicAdd(&h[(0x7fffffffu - (uint32_t)d) & (kBins - 1)], 1);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    err |= __shfl_xor(err, off, 64);
    const int m = __shfl_xor(maxd, off, 64);
    maxd = m > maxd ? m : maxd;
  }
  if ((threadIdx.x & 63) == 0) {
    s_err[threadIdx.x >> 6] = err;
    s_max[threadIdx.x >> 6] = maxd;
  }
  __syncthreads();
  hist[(int64_t)threadIdx.x * ntiles + tile] = h[threadIdx.x];
  if (threadIdx.x == 0) {
    for (int k = 1; k < kThreads / 64; ++k) {
      err |= s_err[k];
      maxd = s_max[k] > maxd ? s_max[k] : maxd;
    }
    if (err) atomicOr(&counts[kErrFlags], err);
    if (maxd > __hip_atomic_load(&counts[kMaxDegree], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(&counts[kMaxDegree], maxd);
  }
}

// ------------------------------------------------------------------------
// Out-degrees without global atomics.  A power-law graph sends a large share
// of all edges to a few hub sources, and same-address atomics serialize, so
// instead: (1) each tile of kOdTile CSR entries is sorted by bucket (the
// source id's high bits, kOdBucket ids per bucket) in LDS and written back
// to its own place in one contiguous piece, as 16-bit offsets within the
// bucket, with the start of every bucket's run in the tile; (2) per bucket,
// workgroups count their share of the tiles' runs into an LDS histogram and
// store it; (3) the partial histograms are summed.  Counting is order-free,
// so no global scan is needed and every global write is contiguous.
// ------------------------------------------------------------------------
// Tile of this workgroup in an XCD-blocked order.  Workgroups are handed to
// the eight XCDs in turn (w % 8), so with tile = w the tiles one L2 sees are
// eight apart, and the tile-minor entries of neighbouring tiles (32 to a
// 128-byte line) are written and read as partial lines through eight
// different L2s.  Here XCD x takes the contiguous run [x * per, (x + 1) *
// per) of tiles.  The grid is xcd_grid(ntiles) workgroups; the spare ones
// get -1.  Any dispatch order gives the same result; only the locality
// depends on it.
constexpr int kXcds = 8;
__device__ __forceinline__ int64_t xcd_tile(int64_t ntiles) {
  const int64_t per = (ntiles + kXcds - 1) / kXcds;
  const int64_t w = blockIdx.x, t = (w % kXcds) * per + w / kXcds;
  return t < ntiles ? t : -1;
}
inline unsigned xcd_grid(int64_t ntiles) {
  return (unsigned)(kXcds * ((ntiles + kXcds - 1) / kXcds));
}

// Shapes measured on the 2^21-source R-MAT graph (E = 1.07e8), whole
// out-degree count: 16,384 ids per bucket and tiles of 16,384 entries; the
// count with about 1024 workgroups (two per CU, 64 KB of LDS each), each
// wave reading 4 tiles' runs at a time, 256 entries of each before counting.
// 8,192 or 32,768 ids per bucket, 256 or 512 count workgroups, 8 x 2 or
// 16 x 1 runs x loads, 32-bit loads of entry pairs, and persistent bin
// workgroups that prefetch their next tile were all slower.
constexpr int kOdBits = 14;
constexpr int kOdBucket = 1 << kOdBits;
constexpr int64_t kOdMaxSources = int64_t(1) << 23;  // larger graphs count in k_degrees
constexpr int kOdMaxBuckets = (int)(kOdMaxSources >> kOdBits);
constexpr int kOdThreads = 512, kOdWaves = kOdThreads / 64;
constexpr int kOdItems = 32;
constexpr int kOdTile = kOdThreads * kOdItems;  // 16384 entries per tile
constexpr int kOdCountWgs = 1024, kOdRuns = 4, kOdLoads = 4;
static_assert(kOdBits <= 15, "the count's LDS histogram holds 2^15 counters");
static_assert(kOdTile <= 65536, "16-bit offsets");
static_assert(64 * kOdItems < 0xffff, "16-bit ranks within a wave");
// workgroups per bucket in the count: about kOdCountWgs workgroups in all, at
// most 16 a bucket (each leaves a partial histogram to add up), or with few
// buckets up to 64 where each still has 2^16 entries (16,000 sources, 2.4e7
// edges: whole plan 738 -> 345 us; with 19 buckets, 6e6 edges: 131 -> 165)
inline int outdeg_split(int64_t nb, int64_t E) {
  const int64_t s = nb >= kOdCountWgs || nb < 1 ? 1 : kOdCountWgs / nb;
  const int64_t most = nb > 8 || E >> 16 < 16 ? 16 : E >> 16 > 64 ? 64 : E >> 16;
  return (int)(s > most ? most : s);
}
// Few buckets and few edges: no tile sort; every bucket's workgroups read all
// of col_idx and count their own ids.  The re-reads come from L2; the tile
// sort costs two launches and gives a bucket's few workgroups long runs.
// Measured (us, tile sort / direct): the count alone, 100,000 sources, 1.3e6
// edges 80 / 21; 15,000 sources, 1.65e5 edges 94 / 9; the whole plan, 100,000
// sources, 1e7 edges 127 / 87; 40,000 sources, 2.4e7 edges 279 / 111; 262,144
// sources, 1.3e6 edges 173 / 59; but 300,000 sources, 6e6 edges 131 / 164 and
// 10^6 sources, 2e6 edges 105 / 145.
inline bool outdeg_direct(int64_t nb, int64_t E) {
  return nb * E <= (nb <= 8 ? int64_t(256) << 20 : int64_t(32) << 20);
}
inline size_t outdeg_bin_lds(int nb) {
  return (size_t)kOdWaves * nb * 4 + (size_t)kOdTile * 2;
}
static_assert((size_t)kOdWaves * kOdMaxBuckets * 4 + (size_t)kOdTile * 2 + 64 <= 65536,
              "the bin kernel's LDS stays within 64 KB");

// Sort one tile by bucket.  Each wave ranks its own entries with counters
// of its own, laid out wave-major (a wave's lanes hit nb consecutive words);
// the bucket-major scan over (bucket, wave) then places bucket b's entries of
// wave 0, 1, ... one after another.  loc[b * ntiles + tile] is the start of
// bucket b's run within the tile, loc[nb * ntiles + tile] the tile's valid
// entries.  Source ids outside [0, Vs) raise error bit 8 and are left out.
// The loads are unconditional (E > 0, so a tile holds at least one entry):
// an entry past the tile's end reads the tile's last one and is then
// ignored, so no branch splits the batch of loads.
__global__ __launch_bounds__(kOdThreads) void k_outdeg_bin(const int32_t* __restrict__ col,
                                                           int64_t E, int32_t Vs, int nb,
                                                           int64_t ntiles,
                                                           uint16_t* __restrict__ out,
                                                           int32_t* __restrict__ loc,
                                                           int32_t* counts) {
  extern __shared__ int32_t sm[];
  int32_t* cnt = sm;  // [kOdWaves][nb]
  uint16_t* sval = reinterpret_cast<uint16_t*>(sm + kOdWaves * nb);  // [kOdTile]
  __shared__ int32_t wsum[kOdWaves];
  const int64_t tile = xcd_tile(ntiles);
  if (tile < 0) return;
  const int tx = threadIdx.x, wave = tx >> 6, lane = tx & 63;
  const int64_t base = tile * (int64_t)kOdTile;
  const int n = E - base < kOdTile ? (int)(E - base) : kOdTile;
  for (int b = tx; b < kOdWaves * nb; b += kOdThreads) cnt[b] = 0;
  const int32_t* p = col + base;
  int32_t c[kOdItems];
  if (n == kOdTile) {
#pragma unroll
    for (int j = 0; j < kOdItems; ++j) c[j] = __builtin_nontemporal_load(p + j * kOdThreads + tx);
  } else {
#pragma unroll
    for (int j = 0; j < kOdItems; ++j) {
      const int i = j * kOdThreads + tx;
      c[j] = __builtin_nontemporal_load(p + (i < n ? i : n - 1));
    }
  }
  __syncthreads();
  // rank within (wave, bucket), two 16-bit ranks to a register (a wave
  // ranks at most 64 * kOdItems entries); 0xffff marks no entry
  int32_t* cw = cnt + wave * nb;
  uint32_t r[kOdItems / 2];
  int err = 0;
#pragma unroll
  for (int j = 0; j < kOdItems; ++j) {
    const bool in = j * kOdThreads + tx < n;
    const bool ok = in && c[j] >= 0 && c[j] < Vs;
    err |= in && !ok;
    const uint32_t rj = ok ? (uint32_t)atomicAdd(&cw[c[j] >> kOdBits], 1) : 0xffffu;
    r[j / 2] = j % 2 ? r[j / 2] | rj << 16 : rj;
  }
  if (__any(err) && lane == 0) atomicOr(&counts[kErrFlags], kErrCol);
  __syncthreads();
  {  // exclusive scan over k = b * kOdWaves + w (entry cnt[w * nb + b]):
     // thread t owns k in [t * pk, (t + 1) * pk), then a wave scan and a
     // cross-wave pass
    const int m = kOdWaves * nb;
    const int pk = (m + kOdThreads - 1) / kOdThreads;
    const int k0 = tx * pk;
    int32_t own = 0;
    for (int k = k0; k < k0 + pk && k < m; ++k) own += cnt[(k % kOdWaves) * nb + k / kOdWaves];
    int32_t inc = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int32_t y = __shfl_up(inc, off, 64);
      if (lane >= off) inc += y;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    int32_t run = inc - own;
    for (int w = 0; w < wave; ++w) run += wsum[w];
    for (int k = k0; k < k0 + pk && k < m; ++k) {
      const int a = (k % kOdWaves) * nb + k / kOdWaves;
      const int32_t v = cnt[a];
      cnt[a] = run;
      if (k % kOdWaves == 0) loc[(int64_t)(k / kOdWaves) * ntiles + tile] = run;
      run += v;
    }
    if (tx == kOdThreads - 1) loc[(int64_t)nb * ntiles + tile] = run;
  }
  __syncthreads();
  int32_t total = 0;
  for (int w = 0; w < kOdWaves; ++w) total += wsum[w];
#pragma unroll
  for (int j = 0; j < kOdItems; ++j) {
    const uint32_t rj = r[j / 2] >> (16 * (j % 2)) & 0xffffu;
    if (rj != 0xffffu) sval[cw[c[j] >> kOdBits] + (int)rj] = (uint16_t)(c[j] & (kOdBucket - 1));
  }
  __syncthreads();
  // the tile's sorted entries, 8 to a 16-byte store
  const int nv = total >> 3;
  uint4* out4 = reinterpret_cast<uint4*>(out + base);
  const uint4* s4 = reinterpret_cast<const uint4*>(sval);
  for (int i = tx; i < nv; i += kOdThreads) out4[i] = s4[i];
  for (int i = nv * 8 + tx; i < total; i += kOdThreads) out[base + i] = sval[i];
}

// Bucket b's entries, from the runs of tiles [t0, t1) (slice s of
// outdeg_split), counted into LDS; the histogram goes to
// part[s][b * kOdBucket + i].  Each wave takes R tiles at a time and reads
// the first J * 64 entries of each run before counting, so that R * J loads
// are in flight; longer runs finish in a loop.
__global__ __launch_bounds__(1024) void k_outdeg_count(const uint16_t* __restrict__ bk,
                                                       const int32_t* __restrict__ loc,
                                                       int64_t ntiles, int nb, int64_t E,
                                                       int32_t* __restrict__ part,
                                                       const int32_t* counts) {
  if (count_stops(counts)) return;
  __shared__ int32_t h[kOdBucket];
  constexpr int R = kOdRuns, J = kOdLoads, NW = 1024 / 64;
  // buckets in an XCD-blocked order (gridDim.x = xcd_grid(nb)): XCD x takes
  // the contiguous buckets [x * per, (x + 1) * per), so that neighbouring
  // buckets, whose runs share the 128-byte lines where they meet, read them
  // through one L2
  const int per = (int)((nb + kXcds - 1) / kXcds);
  const int b = (int)(blockIdx.x % kXcds) * per + (int)(blockIdx.x / kXcds);
  const int s = blockIdx.y, S = gridDim.y;
  if (b >= nb) return;
  for (int i = threadIdx.x; i < kOdBucket; i += 1024) h[i] = 0;
  __syncthreads();
  const int64_t t0 = ntiles * s / S, t1 = ntiles * (s + 1) / S;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int32_t* lb = loc + (int64_t)b * ntiles;
  const int32_t* le = loc + (int64_t)(b + 1) * ntiles;
  for (int64_t tg = t0 + (int64_t)wave * R; tg < t1; tg += (int64_t)NW * R) {
    int64_t beg[R];
    int32_t len[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int64_t t = tg + q;
      len[q] = 0;
      beg[q] = 0;
      if (t < t1) {
        const int64_t tbase = t * (int64_t)kOdTile;
        const int32_t n = (int32_t)(E - tbase < kOdTile ? E - tbase : kOdTile);
        int32_t lo = lb[t], hi = le[t];
        lo = lo < 0 ? 0 : (lo > n ? n : lo);
        hi = hi < lo ? lo : (hi > n ? n : hi);
        beg[q] = tbase + lo;
        len[q] = hi - lo;
      }
    }
    uint32_t v[R][J];
#pragma unroll
    for (int q = 0; q < R; ++q)
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int k = j * 64 + lane;
        v[q][j] = k < len[q] ? (uint32_t)bk[beg[q] + k] : 0xffffffffu;
      }
#pragma unroll
    for (int q = 0; q < R; ++q)
#pragma unroll
      for (int j = 0; j < J; ++j)
        if (v[q][j] != 0xffffffffu) atomicAdd(&h[v[q][j] & (kOdBucket - 1)], 1);
#pragma unroll
    for (int q = 0; q < R; ++q)
      for (int k = J * 64 + lane; k < len[q]; k += 64)
        atomicAdd(&h[bk[beg[q] + k] & (kOdBucket - 1)], 1);
  }
  __syncthreads();
  int32_t* pw = part + (int64_t)s * nb * kOdBucket + (int64_t)b * kOdBucket;
  for (int i = threadIdx.x; i < kOdBucket; i += 1024) pw[i] = h[i];
}

// The direct count: workgroup (b, s) counts the ids of bucket b among slice s
// of col_idx; the workgroups of bucket 0 also check every id.
__global__ __launch_bounds__(1024) void k_outdeg_direct(const int32_t* __restrict__ col, int64_t E,
                                                        int32_t Vs, int nb, int32_t* __restrict__ part,
                                                        int32_t* counts) {
  __shared__ int32_t h[kOdBucket];
  const int b = blockIdx.x, s = blockIdx.y, S = gridDim.y;
  for (int i = threadIdx.x; i < kOdBucket; i += 1024) h[i] = 0;
  __syncthreads();
  const int64_t e0 = E * s / S, e1 = E * (s + 1) / S;
  constexpr int J = 8;  // loads in flight per thread
  bool bad = false;
  for (int64_t e = e0 + threadIdx.x; e < e1; e += 1024 * J) {
    int32_t c[J];
#pragma unroll
    for (int j = 0; j < J; ++j) c[j] = e + j * 1024 < e1 ? col[e + j * 1024] : -2;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      if (c[j] >= 0 && c[j] < Vs) {
        if (c[j] >> kOdBits == b) atomicAdd(&h[c[j] & (kOdBucket - 1)], 1);
      } else {
        bad |= e + j * 1024 < e1;
      }
    }
  }
  if (b == 0 && __any(bad) && (threadIdx.x & 63) == 0) atomicOr(&counts[kErrFlags], kErrCol);
  __syncthreads();
  int32_t* pw = part + (int64_t)s * nb * kOdBucket + (int64_t)b * kOdBucket;
  for (int i = threadIdx.x; i < kOdBucket; i += 1024) pw[i] = h[i];
}

// d_out[v] = the sum of the S partial counts, four sources per thread as
// 16-byte loads (part and d_out are 256-byte aligned, stride a multiple of 4)
__global__ __launch_bounds__(kThreads) void k_outdeg_reduce(const int32_t* __restrict__ part,
                                                            int nb, int S, int32_t Vs,
                                                            int32_t* __restrict__ d_out,
                                                            const int32_t* counts) {
  if (count_stops(counts)) return;
  const int64_t stride = (int64_t)nb * kOdBucket;
  const int64_t n4 = Vs / 4;
  const int64_t g0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, gs = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = g0; i < n4; i += gs) {
    int4 sum = make_int4(0, 0, 0, 0);
#pragma unroll 8
    for (int w = 0; w < S; ++w) {
      const int4 x = reinterpret_cast<const int4*>(part + w * stride)[i];
      sum.x += x.x;
      sum.y += x.y;
      sum.z += x.z;
      sum.w += x.w;
    }
    reinterpret_cast<int4*>(d_out)[i] = sum;
  }
  for (int64_t v = 4 * n4 + g0; v < Vs; v += gs) {
    int32_t sum = 0;
    for (int w = 0; w < S; ++w) sum += part[w * stride + v];
    d_out[v] = sum;
  }
}

// A pass over digit `shift` moves nothing when no in-degree reaches it: the
// digits of 0x7fffffff - d are then all the same.  Such passes are skipped on
// the device (the first never is), so the order ends in the buffers of the
// last pass that ran.
__device__ __forceinline__ bool radix_skips(const int32_t* counts, int shift) {
  return shift > 0 && (counts[kMaxDegree] >> shift) == 0;
}
// passes that ran
__device__ __forceinline__ int radix_passes(const int32_t* counts) {
  const int m = counts[kMaxDegree];
  return m >> 8 == 0 ? 1 : m >> 16 == 0 ? 2 : m >> 24 == 0 ? 3 : 4;
}

// per-tile digit histogram, stored digit-major: hist[digit * ntiles + tile]
template <bool FIRST>
__global__ __launch_bounds__(kThreads) void k_radix_hist(const int32_t* __restrict__ d_in,
                                                         const uint32_t* __restrict__ keys,
                                                         int32_t n, int shift,
                                                         int32_t* __restrict__ hist, int64_t ntiles,
                                                         const int32_t* counts) {
  if (order_stops(counts) || radix_skips(counts, shift)) return;
  __shared__ int32_t h[kBins];
  const int64_t tile = xcd_tile(ntiles);
  if (tile < 0) return;
  h[threadIdx.x] = 0;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    int64_t i = tile * kTile + j * kThreads + threadIdx.x;
    if (i < n) {
      uint32_t k = FIRST ? (0x7fffffffu - (uint32_t)d_in[i]) : keys[i];
      atomicAdd(&h[(k >> shift) & (kBins - 1)], 1);
    }
  }
  __syncthreads();
  hist[(int64_t)threadIdx.x * ntiles + tile] = h[threadIdx.x];
}

// Stable scatter.  Wave w of a tile takes its w-th quarter, 64 items at a time
// in index order: an item's rank among the wave's equal digits is the wave's
// count so far plus a match within the 64 (8 ballots).  The waves' counts are
// then added up in wave order, so equal keys keep their input order, with
// three workgroup barriers a tile (a barrier per 256 items: 13.5 against 11.3
// us for 49 tiles).
// Each item carries a second value, its row's first CSR entry (row_ptr[v]
// on the first pass), so that the segment builder reads it in perm order
// instead of gathering row_ptr at random.
// INSCAN: `offsets` holds the plain histograms, and each workgroup derives its
// own digit offsets from them (at most kInscanTiles tiles: one thread reads
// its digit's row), instead of from a scan in launches of its own.
constexpr int64_t kInscanTiles = 128;
template <bool FIRST, bool INSCAN>
__global__ __launch_bounds__(kThreads) void k_radix_scatter(
    const int32_t* __restrict__ d_in, const uint32_t* __restrict__ keys_in,
    const int32_t* __restrict__ vals_in, const int32_t* __restrict__ rb_in, int32_t n, int shift,
    const int32_t* __restrict__ offsets, int64_t ntiles, uint32_t* __restrict__ keys_out,
    int32_t* __restrict__ vals_out, int32_t* __restrict__ rb_out, const int32_t* counts) {
  if (order_stops_wg(counts) || radix_skips(counts, shift)) return;
  constexpr int NW = kThreads / 64;
  __shared__ int32_t wcnt[NW][kBins];
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  const int64_t tile = xcd_tile(ntiles);
  if (tile < 0) return;
#pragma unroll
  for (int k = 0; k < NW; ++k) wcnt[k][t] = 0;
  uint32_t key[kItems];
  int32_t val[kItems], rb[kItems], rank[kItems];
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int64_t i = tile * kTile + (w * kItems + j) * 64 + lane;
    if (i < n) {
      key[j] = FIRST ? (0x7fffffffu - (uint32_t)d_in[i]) : keys_in[i];
      val[j] = FIRST ? (int32_t)i : vals_in[i];
      rb[j] = rb_in[i];
    }
  }
  int32_t start;  // of digit t in the output, then of this tile's items of it
  if constexpr (INSCAN) {
    int32_t before = 0, all = 0;
    const int32_t* row = offsets + (int64_t)t * ntiles;
#pragma unroll 8
    for (int64_t k = 0; k < ntiles; ++k) {
      const int32_t x = row[k];
      before += k < tile ? x : 0;
      all += x;
    }
    int32_t tot;
    start = block_excl_scan<kThreads>(all, &tot) + before;
  } else {
    start = offsets[(int64_t)t * ntiles + tile];
    __syncthreads();
  }
  const uint64_t lt = lanemask_lt();
  int32_t* cnt = wcnt[w];
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int64_t i = tile * kTile + (w * kItems + j) * 64 + lane;
    const bool valid = i < n;
    const int dg = valid ? (key[j] >> shift) & (kBins - 1) : 0;
    uint64_t m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (dg >> b) & 1;
      uint64_t bal = __ballot(valid && bit);
      m &= bit ? bal : ~bal;
    }
    const int r = __popcll(m & lt);
    const int32_t have = valid ? cnt[dg] : 0;
    rank[j] = have + r;
    // the wave's LDS accesses complete in program order: every lane has read
    // the count before its group's first lane moves it on
    asm volatile("" ::: "memory");
    if (valid && r == 0) cnt[dg] = have + __popcll(m);
    asm volatile("" ::: "memory");
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NW; ++k) {  // thread t: digit t
    const int32_t x = wcnt[k][t];
    wcnt[k][t] = start;
    start += x;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int64_t i = tile * kTile + (w * kItems + j) * 64 + lane;
    if (i < n) {
      const int32_t pos = cnt[(key[j] >> shift) & (kBins - 1)] + rank[j];
      if (pos >= 0 && pos < n) {
        keys_out[pos] = key[j];
        vals_out[pos] = val[j];
        rb_out[pos] = rb[j];
      } else {
        atomicOr(const_cast<int32_t*>(counts) + kErrFlags, kErrInternal);
      }
    }
  }
}

__global__ __launch_bounds__(kThreads) void k_scan_reduce(const int32_t* __restrict__ in, int64_t n,
                                                          int32_t* tile_sums, int shift,
                                                          const int32_t* counts) {
  if (order_stops(counts) || radix_skips(counts, shift)) return;
  const int64_t base = blockIdx.x * (int64_t)kTile + threadIdx.x * kItems;
  int32_t s = 0;
#pragma unroll
  for (int k = 0; k < kItems; ++k)
    if (base + k < n) s += in[base + k];
  int32_t tot;
  block_excl_scan<kThreads>(s, &tot);
  if (threadIdx.x == 0) tile_sums[blockIdx.x] = tot;
}

// exclusive scan of the tile sums by one workgroup of 1024 threads
__global__ __launch_bounds__(1024) void k_scan_tilesums(int32_t* ts, int64_t nt, int shift,
                                                        const int32_t* counts) {
  if (order_stops(counts) || radix_skips(counts, shift)) return;
  __shared__ int32_t carry_s;
  if (threadIdx.x == 0) carry_s = 0;
  __syncthreads();
  for (int64_t base = 0; base < nt; base += 1024) {
    const int64_t i = base + threadIdx.x;
    const int32_t v = i < nt ? ts[i] : 0;
    int32_t tot;
    const int32_t ex = block_excl_scan<1024>(v, &tot);
    const int32_t carry = carry_s;
    if (i < nt) ts[i] = carry + ex;
    __syncthreads();
    if (threadIdx.x == 0) carry_s = carry + tot;
    __syncthreads();
  }
}

__global__ __launch_bounds__(kThreads) void k_scan_apply(const int32_t* in, int64_t n,
                                                         const int32_t* tile_sums,
                                                         int32_t* out, int shift,
                                                         const int32_t* counts) {
  if (order_stops(counts) || radix_skips(counts, shift)) return;
  const int64_t base = blockIdx.x * (int64_t)kTile + threadIdx.x * kItems;
  int32_t v[kItems];
  int32_t s = 0;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    v[k] = base + k < n ? in[base + k] : 0;
    s += v[k];
  }
  int32_t tot;
  int32_t run = block_excl_scan<kThreads>(s, &tot) + tile_sums[blockIdx.x];
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    if (base + k < n) out[base + k] = run;
    run += v[k];
  }
}

// ------------------------------------------------------------------------
// Segments and row blocks, from the degree order.  Position i of the order has
// ns(i) segments of total cost d_i + ns(i) row_cost, so one prefix sum over
// the rows gives both the first segment of every row and the cost before it;
// the segments inside a row follow from those.  k_seg_sums: each tile's totals
// (y: the tile sums of segments and of cost).  k_seg_emit: a workgroup adds up
// the tiles before its own (or reads them scanned), scans its rows in LDS and
// writes its segments slot by slot, so that a hub row's hundreds of segments
// are spread over the workgroup.  The first tile, the hubs', takes longest; 512
// rows and a shift for the default power-of-two block cost keep it short.
// ------------------------------------------------------------------------
struct Order {  // the degree order's buffers: pass p ends in keys[p % 2] ..
  const uint32_t* keys[2];
  const int32_t* vals[2];
  const int32_t* rbeg[2];
};
constexpr int kSegTile = 512;        // rows per workgroup, one per thread
constexpr int64_t kSumTiles = 4096;  // more tiles: their sums are scanned by a launch of its own

__global__ __launch_bounds__(kSegTile) void k_seg_sums(Order o, int32_t V, int32_t T, int32_t c,
                                                       int32_t* __restrict__ sums, int64_t ntiles,
                                                       const int32_t* counts) {
  if (order_stops(counts)) return;
  const uint32_t* __restrict__ keys = o.keys[(radix_passes(counts) - 1) & 1];
  int32_t ns = 0, cost = 0;
  const int64_t i = blockIdx.x * (int64_t)kSegTile + threadIdx.x;
  if (i < V) {
    const int32_t d = key_degree(keys[i]);
    ns = seg_count(d, T);
    cost = d + ns * c;
  }
  int32_t tn, tc;
  block_excl_scan<kSegTile>(ns, &tn);
  block_excl_scan<kSegTile>(cost, &tc);
  if (threadIdx.x == 0) {
    sums[blockIdx.x] = tn;
    sums[ntiles + blockIdx.x] = tc;
  }
}

__global__ __launch_bounds__(kSegTile) void k_seg_emit(Order o, int32_t V, int32_t T, int32_t c, int32_t B,
                                                       int bshift,
                                                       const int32_t* __restrict__ sums, int64_t ntiles,
                                                       int scanned, int64_t max_seg, int64_t max_blocks,
                                                       int32_t* __restrict__ perm,
                                                       int32_t* __restrict__ first,
                                                       int32_t* __restrict__ seg_row,
                                                       int32_t* __restrict__ seg_beg,
                                                       int32_t* __restrict__ seg_end,
                                                       int32_t* __restrict__ block_ptr, int32_t* counts) {
  if (order_stops_wg(counts)) return;
  __shared__ int32_t s_deg[kSegTile], s_row[kSegTile], s_rb[kSegTile], s_first[kSegTile + 1], s_cost[kSegTile];
  const int64_t tile = blockIdx.x;
  const int t = threadIdx.x;
  const int last_pass = (radix_passes(counts) - 1) & 1;
  const uint32_t* __restrict__ keys = o.keys[last_pass];
  const int32_t* __restrict__ vals = o.vals[last_pass];
  const int32_t* __restrict__ rbeg = o.rbeg[last_pass];
  int32_t base_n, base_c;  // segments and cost before this tile
  if (scanned) {
    base_n = sums[tile];
    base_c = sums[ntiles + tile];
  } else {
    int32_t a = 0, b = 0;
    for (int64_t k = t; k < tile; k += kSegTile) {
      a += sums[k];
      b += sums[ntiles + k];
    }
    block_excl_scan<kSegTile>(a, &base_n);
    block_excl_scan<kSegTile>(b, &base_c);
  }
  const int64_t i0 = tile * kSegTile;
  const int n = V - i0 < kSegTile ? (int)(V - i0) : kSegTile;
  bool bad = false;
  int32_t ns = 0, cost = 0;
  if (t < n) {
    const int32_t v = vals[i0 + t], d = key_degree(keys[i0 + t]);
    bad = v < 0 || v >= V;
    s_deg[t] = d;
    s_row[t] = v;
    s_rb[t] = rbeg[i0 + t];
    perm[i0 + t] = v;
    ns = seg_count(d, T);
    cost = d + ns * c;
  }
  int32_t tile_n, tile_c;
  s_first[t] = block_excl_scan<kSegTile>(ns, &tile_n);
  s_cost[t] = block_excl_scan<kSegTile>(cost, &tile_c) + base_c;
  if (t == 0 && n == kSegTile) s_first[n] = tile_n;  // (a short tile's scan holds it)
  bad |= base_n < 0 || tile_n < n || (int64_t)base_n + tile_n > max_seg;
  if (__syncthreads_or(bad)) {
    if (t == 0) atomicOr(&counts[kErrFlags], kErrInternal);
    return;
  }
  const bool last_tile = i0 + n == V;
  if (const int r = t; r < n) {
    first[i0 + r] = base_n + s_first[r];
    // the last split row: the next one fits a segment
    if (s_deg[r] > T) {
      const int32_t next = r + 1 < n ? s_deg[r + 1] : last_tile ? 0 : key_degree(keys[i0 + n]);
      if (next <= T) {
        counts[kNSplit] = (int32_t)(i0 + r + 1);
        counts[kSSplit] = base_n + s_first[r + 1];
      }
    }
  }
  if (last_tile && t == 0) {
    first[V] = base_n + tile_n;
    counts[kNumSegments] = base_n + tile_n;
  }
  // block b holds the segments s with floor(P(s) / B) == b; consecutive
  // segments differ in P by at most seg_len + row_cost <= B, so no block id
  // is skipped
  auto block_of = [&](int32_t P) { return bshift >= 0 ? P >> bshift : P / B; };
  for (int q = t; q < tile_n; q += kSegTile) {
    int r = q;
    if (tile_n != n) {  // rows of several segments: the row whose range holds q
      r = 0;
#pragma unroll
      for (int step = kSegTile / 2; step > 0; step >>= 1)
        if (r + step < n && s_first[r + step] <= q) r += step;
    }
    const int32_t j = q - s_first[r], d = s_deg[r], s = base_n + q;
    const int32_t b = s_rb[r] + j * T, left = d - j * T;
    seg_row[s] = s_row[r];
    seg_beg[s] = b;
    seg_end[s] = b + (left > T ? T : left);
    const int32_t P = s_cost[r] + j * (T + c), blk = block_of(P);
    int32_t prev = T + c;  // cost of segment s - 1
    if (j == 0 && s > 0) {
      const int32_t dp = r > 0 ? s_deg[r - 1] : key_degree(keys[i0 - 1]);
      prev = dp - (seg_count(dp, T) - 1) * T + c;
    }
    if (blk < 0 || blk >= max_blocks) {
      atomicOr(&counts[kErrFlags], kErrInternal);
    } else {
      if (s == 0 || block_of(P - prev) != blk) block_ptr[blk] = s;
      if (last_tile && q == tile_n - 1) {
        block_ptr[blk + 1] = s + 1;
        counts[kNumBlocks] = blk + 1;
      }
    }
  }
}

// exclusive scan of n ints, in launches of its own (skipped with the pass)
void scan(const int32_t* in, int64_t n, int32_t* out, int32_t* tile_sums, int shift, const int32_t* counts,
          hipStream_t st) {
  const int64_t nt = cdiv(n, kTile);
  if (nt == 0) return;
  hipLaunchKernelGGL(k_scan_reduce, dim3(nt), dim3(kThreads), 0, st, in, n, tile_sums, shift, counts);
  hipLaunchKernelGGL(k_scan_tilesums, dim3(1), dim3(1024), 0, st, tile_sums, nt, shift, counts);
  hipLaunchKernelGGL(k_scan_apply, dim3(nt), dim3(kThreads), 0, st, in, n, tile_sums, out, shift, counts);
}

inline unsigned grid_for(int64_t n, int64_t cap = 16384) {
  int64_t g = cdiv(n, kThreads);
  if (g < 1) g = 1;
  return (unsigned)(g < cap ? g : cap);
}

}  // namespace

bool plan_layout(int32_t V, int32_t Vs, int64_t E, int32_t T, int32_t B, int32_t c,
                 PlanLayout* L) {
  if (V < 0 || Vs < 0 || E < 0 || E >= (int64_t(1) << 31) || T <= 0 || c <= 0 || B < T + c)
    return false;
  L->max_segments = (int64_t)V + cdiv(E, T);
  const int64_t ptot = E + (int64_t)c * L->max_segments;
  if (ptot >= (int64_t(1) << 31) - 1) return false;
  L->max_blocks = ptot / B + 1;
  L->max_split = E / (int64_t(T) + 1) < V ? E / (int64_t(T) + 1) : V;
  L->max_split_segments = cdiv(E, T) + L->max_split;
  L->radix_tiles = cdiv(V, kTile);
  L->scan_tiles_rows = cdiv(V, kSegTile);
  const int64_t hist_n = (int64_t)kBins * L->radix_tiles;
  L->outdeg_nb = cdiv(Vs, kOdBucket);
  L->edge_tiles = cdiv(E, kOdTile);
  L->outdeg_bucketed = L->outdeg_nb > 0 && L->outdeg_nb <= kOdMaxBuckets && E > 0;
  int64_t scan_tiles = cdiv(hist_n, kTile);
  if (2 * L->scan_tiles_rows > scan_tiles) scan_tiles = 2 * L->scan_tiles_rows;

  size_t o = 0;
  auto take = [&](int64_t n_int) {
    size_t at = o;
    o = align256(o + (size_t)n_int * 4);
    return at;
  };
  L->off_d_in = take(V);
  L->off_d_out = take(Vs);
  L->off_perm = take(V);
  L->off_first = take((int64_t)V + 1);
  L->off_seg_row = take(L->max_segments);
  L->off_seg_beg = take(L->max_segments);
  L->off_seg_end = take(L->max_segments);
  L->off_block_ptr = take(L->max_blocks + 1);
  L->off_counts = take(kCountSlots);
  L->off_scratch = o;
  // scratch: keysA, valsA, keysB, valsB, row begins A and B, hist, tile
  // sums, bucketed source ids, bucket run starts, partial out-degree histograms
  const bool bk = L->outdeg_bucketed, sorted = bk && !outdeg_direct(L->outdeg_nb, E);
  take(V); take(V); take(V); take(V); take(V); take(V);
  take(hist_n);
  take(scan_tiles + 1);
  take(sorted ? cdiv(E, 2) : 0);
  take(sorted ? (L->outdeg_nb + 1) * L->edge_tiles : 0);
  take(bk ? (int64_t)outdeg_split(L->outdeg_nb, E) * L->outdeg_nb * kOdBucket : 0);
  L->scratch_bytes = o - L->off_scratch;
  L->total = o;
  return true;
}

hipError_t launch_plan_build(const saga_plan& p, const PlanLayout& L, hipStream_t st,
                             hipStream_t order_st, hipEvent_t fork, hipEvent_t join) {
  const int32_t V = p.num_dst, Vs = p.num_src, T = p.seg_len;
  const int64_t E = p.num_edges;
  char* sc = static_cast<char*>(p.scratch);
  size_t o = 0;
  auto take = [&](int64_t n_int) {
    char* at = sc + o;
    o = align256(o + (size_t)n_int * 4);
    return at;
  };
  uint32_t* keysA = reinterpret_cast<uint32_t*>(take(V));
  int32_t* valsA = reinterpret_cast<int32_t*>(take(V));
  uint32_t* keysB = reinterpret_cast<uint32_t*>(take(V));
  int32_t* valsB = reinterpret_cast<int32_t*>(take(V));
  int32_t* rbA = reinterpret_cast<int32_t*>(take(V));
  int32_t* rbB = reinterpret_cast<int32_t*>(take(V));
  const int64_t ntiles = L.radix_tiles;
  int32_t* hist = reinterpret_cast<int32_t*>(take((int64_t)kBins * ntiles));
  int64_t scan_tiles = cdiv((int64_t)kBins * ntiles, kTile);
  if (2 * L.scan_tiles_rows > scan_tiles) scan_tiles = 2 * L.scan_tiles_rows;
  int32_t* tile_sums = reinterpret_cast<int32_t*>(take(scan_tiles + 1));
  const bool bk = L.outdeg_bucketed, sorted = bk && !outdeg_direct(L.outdeg_nb, E);
  uint16_t* bucketed = reinterpret_cast<uint16_t*>(take(sorted ? cdiv(E, 2) : 0));
  int32_t* oloc = reinterpret_cast<int32_t*>(take(sorted ? (L.outdeg_nb + 1) * L.edge_tiles : 0));
  int32_t* opart = reinterpret_cast<int32_t*>(
      take(bk ? (int64_t)outdeg_split(L.outdeg_nb, E) * L.outdeg_nb * kOdBucket : 0));

  hipLaunchKernelGGL(k_zero, dim3(1), dim3(64), 0, st, p.counts, (int64_t)kCountSlots);
  if (Vs > 0 && !L.outdeg_bucketed)
    hipLaunchKernelGGL(k_zero, dim3(grid_for(Vs)), dim3(kThreads), 0, st, p.d_out, (int64_t)Vs);
  // Two independent branches: the out-degree count (col_idx only) and the
  // row order (row_ptr only: in-degrees, CSR validation, degree sort,
  // segments, row blocks).  With an order stream, the row order runs there
  // after the counters are cleared, so that whatever the caller enqueues on
  // `st` after the out-degrees (the d_out-scaled transform) overlaps it.
  // The graphs whose out-degrees are counted inside k_degrees (no buckets)
  // run both on `st`.
  const bool split = order_st && fork && join && L.outdeg_bucketed && V > 0;
  hipStream_t qst = st;
  if (split) {
    hipError_t e = hipEventRecord(fork, st);
    if (e == hipSuccess) e = hipStreamWaitEvent(order_st, fork, 0);
    if (e != hipSuccess) return e;
    qst = order_st;
  }
  if (V == 0) {
    if (join) {
      hipError_t e = hipEventRecord(join, st);
      if (e != hipSuccess) return e;
    }
    return hipGetLastError();
  }
  if (L.outdeg_bucketed) {
    hipLaunchKernelGGL(k_degrees_hist, dim3(ntiles), dim3(kThreads), 0, qst, p.row_ptr, V, E, p.d_in,
                       hist, ntiles, p.counts);
    const int nb = (int)L.outdeg_nb;
    const int64_t et = L.edge_tiles;
    const int S = outdeg_split(nb, E);
    if (sorted) {
      hipLaunchKernelGGL(k_outdeg_bin, dim3(xcd_grid(et)), dim3(kOdThreads), outdeg_bin_lds(nb), st,
                         p.col_idx, E, Vs, nb, et, bucketed, oloc, p.counts);
      hipLaunchKernelGGL(k_outdeg_count, dim3(xcd_grid(nb), S), dim3(1024), 0, st, bucketed, oloc, et,
                         nb, E, opart, p.counts);
    } else {
      hipLaunchKernelGGL(k_outdeg_direct, dim3(nb, S), dim3(1024), 0, st, p.col_idx, E, Vs, nb, opart,
                         p.counts);
    }
    hipLaunchKernelGGL(k_outdeg_reduce, dim3(grid_for((Vs + 3) / 4)), dim3(kThreads), 0, st, opart, nb,
                       S, Vs, p.d_out, p.counts);
  } else {
    hipLaunchKernelGGL(k_degrees, dim3(grid_for(E > V ? E : V, 2048)), dim3(kThreads), 0, qst, p.row_ptr,
                       p.col_idx, V, Vs, E, p.d_in, p.d_out, p.counts);
    hipLaunchKernelGGL(k_radix_hist<true>, dim3(xcd_grid(ntiles)), dim3(kThreads), 0, qst, p.d_in,
                       static_cast<const uint32_t*>(nullptr), V, 0, hist, ntiles, p.counts);
  }
  st = qst;  // the row order

  // degree order: stable passes of 8 bits over key = 0x7fffffff - d_in, as
  // many as an in-degree of at most E has digits
  const uint32_t* kin[4] = {nullptr, keysA, keysB, keysA};
  const int32_t* vin[4] = {nullptr, valsA, valsB, valsA};
  const int32_t* rin[4] = {p.row_ptr, rbA, rbB, rbA};
  uint32_t* kout[4] = {keysA, keysB, keysA, keysB};
  int32_t* vout[4] = {valsA, valsB, valsA, valsB};
  int32_t* rout[4] = {rbA, rbB, rbA, rbB};
  const bool inscan = ntiles <= kInscanTiles;
  const dim3 rg(xcd_grid(ntiles)), rb(kThreads);
  for (int pass = 0; pass < 4 && (pass == 0 || E >> (8 * pass) > 0); ++pass) {
    const int shift = 8 * pass;
    if (pass > 0)
      hipLaunchKernelGGL(k_radix_hist<false>, rg, rb, 0, st, p.d_in, kin[pass], V, shift, hist, ntiles,
                         p.counts);
    if (!inscan) scan(hist, (int64_t)kBins * ntiles, hist, tile_sums, shift, p.counts, st);
#define SAGA_SCATTER(FIRST, IN)                                                                    \
  hipLaunchKernelGGL((k_radix_scatter<FIRST, IN>), rg, rb, 0, st, p.d_in, kin[pass], vin[pass],     \
                     rin[pass], V, shift, hist, ntiles, kout[pass], vout[pass], rout[pass], p.counts)
    if (pass == 0 && inscan) SAGA_SCATTER(true, true);
    else if (pass == 0) SAGA_SCATTER(true, false);
    else if (inscan) SAGA_SCATTER(false, true);
    else SAGA_SCATTER(false, false);
#undef SAGA_SCATTER
  }

  // segments per row in perm order, their cost, row blocks
  const int64_t nst = L.scan_tiles_rows;
  const Order ord = {{keysA, keysB}, {valsA, valsB}, {rbA, rbB}};
  hipLaunchKernelGGL(k_seg_sums, dim3(nst), dim3(kSegTile), 0, st, ord, V, T, p.row_cost, tile_sums, nst,
                     p.counts);
  const int scanned = nst > kSumTiles ? 1 : 0;
  if (scanned) {
    hipLaunchKernelGGL(k_scan_tilesums, dim3(1), dim3(1024), 0, st, tile_sums, nst, 0, p.counts);
    hipLaunchKernelGGL(k_scan_tilesums, dim3(1), dim3(1024), 0, st, tile_sums + nst, nst, 0,
                       p.counts);
  }
  int bshift = -1;
  for (int k = 0; k < 31; ++k)
    if (p.block_cost == 1 << k) bshift = k;
  hipLaunchKernelGGL(k_seg_emit, dim3(nst), dim3(kSegTile), 0, st, ord, V, T, p.row_cost, p.block_cost, bshift, tile_sums,
                     nst, scanned, L.max_segments, L.max_blocks, p.perm, p.row_seg_first, p.seg_row,
                     p.seg_beg, p.seg_end, p.block_ptr, p.counts);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && join) e = hipEventRecord(join, st);
  return e;
}

}  // namespace saga
