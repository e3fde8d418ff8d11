// Device code shared by the ApplyVertex kernels: matrix-core element types,
// waits and barriers of the LDS rings, row offsets, and the fused epilogue.
#pragma once

#include "saga_device.h"
#include "saga_internal.h"

namespace saga {
namespace {

constexpr int kThreads = 256;
constexpr int kXcds = 8;

typedef __attribute__((address_space(3))) void* lds_ptr;

template <typename T> struct Mma;

template <> struct Mma<float> {
  static constexpr int EPL = 4;     // elements per 16-byte fragment
  static constexpr int KC = 32;     // k per 128-byte chunk
  typedef f32x4 Frag;
  __device__ __forceinline__ static float to_f(float x) { return x; }
  __device__ __forceinline__ static float from_f(float x) { return x; }
};

template <> struct Mma<uint16_t> {
  static constexpr int EPL = 8;
  static constexpr int KC = 64;
  typedef bf16x8 Frag;
  __device__ __forceinline__ static float to_f(uint16_t x) { return bf16_to_f32(x); }
  __device__ __forceinline__ static uint16_t from_f(float x) { return f32_to_bf16(x); }
};

__device__ __forceinline__ int swz(int r, int p) { return r * 8 + (p ^ ((r >> 1) & 7)); }

// s_waitcnt vmcnt(N) (gfx9 encoding; expcnt and lgkmcnt left at their maxima)
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt out of range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Workgroup barrier for the LDS ring.  A plain __syncthreads() would also
// wait for every direct-to-LDS load in flight (its release fence covers LDS
// writes, and those loads write LDS), which would drain the ring at every
// chunk.  Here the caller has already waited for the stage it needs; the
// barrier only orders this wave's own LDS reads and writes.
__device__ __forceinline__ void ring_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// element offsets of this lane's A rows r0 + 16 mt + lane % 16.  Rows >=
// M read row M - 1 (their results are never stored).  With a row map, row
// q is row arow[q] of A; a negative entry reads row 0 (the caller writes
// zeros for it).
template <int MT>
__device__ __forceinline__ void row_offsets(const int32_t* __restrict__ arow, int64_t lda,
                                                   int64_t M, int64_t r0, int64_t (&off)[MT]) {
  const int lr = threadIdx.x & 15;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int64_t row = r0 + mt * 16 + lr;
    int64_t rr = row < M ? row : M - 1;
    if (arow) {
      const int32_t s = arow[rr];
      rr = s >= 0 ? s : 0;
    }
    off[mt] = rr * lda;
  }
}

// ---------------------------------------------------------------------------
// epilogue.  Lane l of a wave holds rows 4 (l / 16) + r (r < 4), column
// l % 16 of each 16 x 16 accumulator tile (mt, nt).
// ---------------------------------------------------------------------------

template <int ACT, int MT, int NT>
__device__ __forceinline__ void act_tile(f32x4 (&acc)[MT][NT]) {
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[mt][nt][r] = apply_act(ACT, acc[mt][nt][r]);
}

// Row scale, biases and activation applied to the accumulators in place,
// in that order (v = acc * rs + b1 + b2, then act).  Each optional step is
// one uniform branch around the whole tile, and every load happens before
// the first store (the compiler cannot tell the output from the loaded
// arrays, so a load after a store would wait for it).
template <int MT, int NT>
__device__ __forceinline__ void finish_tile(const GemmArgs& g, int64_t row0, int64_t n0,
                                            f32x4 (&acc)[MT][NT]) {
  const int lane = threadIdx.x & 63;
  if (g.row_scale_deg) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t row = row0 + mt * 16 + 4 * (lane >> 4) + r;
        const float rs = row < g.M ? rsqrt_deg(g.row_scale_deg[row]) : 0.0f;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt][r] *= rs;
      }
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const float* bias = k == 0 ? g.bias : g.bias2;
    if (!bias) continue;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int64_t c = n0 + nt * 16 + (lane & 15);
      const float b = c < g.N ? bias[c] : 0.0f;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[mt][nt][r] += b;
    }
  }
  switch (g.act) {
    case SAGA_ACT_RELU: act_tile<SAGA_ACT_RELU>(acc); break;
    case SAGA_ACT_ELU: act_tile<SAGA_ACT_ELU>(acc); break;
    case SAGA_ACT_SIGMOID: act_tile<SAGA_ACT_SIGMOID>(acc); break;
    case SAGA_ACT_TANH: act_tile<SAGA_ACT_TANH>(acc); break;
    default: break;
  }
}

// output element (row, c) of the finished tile: columns >= split go to out2
template <typename T>
__device__ __forceinline__ void store_elem(const GemmArgs& g, int64_t row, int64_t c, float v) {
  if (g.split > 0 && c >= g.split)
    static_cast<T*>(g.out2)[row * g.ldo2 + (c - g.split)] = Mma<T>::from_f(v);
  else
    static_cast<T*>(g.out)[row * g.ldo + c] = Mma<T>::from_f(v);
}

// element by element, straight from the accumulators
template <typename T, int MT, int NT>
__device__ __forceinline__ void store_direct(const GemmArgs& g, int64_t row0, int64_t n0,
                                             const f32x4 (&acc)[MT][NT]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = row0 + mt * 16 + 4 * (lane >> 4) + r;
      if (row >= g.M) continue;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int64_t c = n0 + nt * 16 + (lane & 15);
        if (c < g.N) store_elem<T>(g, row, c, acc[mt][nt][r]);
      }
    }
}

// Through LDS: the wave writes its 16 MT rows x 16 NT columns (already in
// the output type) to its own region, then each lane reads back whole
// 16-byte pieces of rows, so one store instruction covers 1 KB of whole
// row pieces instead of 64-byte pieces of four rows.  A piece is stored
// whole when it lies inside the output, on one side of the split column,
// and both outputs allow 16-byte accesses; otherwise element by element.
// For 128-column tiles, piece p of local row lr sits at piece
// p ^ (((lr >> 2) & 3) << SH) of the row in LDS: the four rows one write
// instruction touches then fall on different banks (narrower tiles keep
// the plain order).  Only this wave's region is touched, so no workgroup
// barrier is needed once every wave is past the last read of the ring.
template <typename T, int MT, int NT>
__device__ __forceinline__ void store_staged(const GemmArgs& g, int64_t row0, int64_t n0,
                                             const f32x4 (&acc)[MT][NT], T* region) {
  constexpr int BN = 16 * NT, EPL = Mma<T>::EPL, PR = BN / EPL, ROWS = 16 * MT;
  constexpr int SH = NT == 8 ? (EPL == 4 ? 2 : 1) : 0;  // log2 pieces per 16 columns
  constexpr int SW = NT == 8 ? 3 : 0;                    // row bits that pick the swizzle
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int lr = mt * 16 + 4 * (lane >> 4) + r;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int col = nt * 16 + (lane & 15);
        const int pp = (col / EPL) ^ (((lr >> 2) & SW) << SH);
        region[lr * BN + pp * EPL + col % EPL] = Mma<T>::from_f(acc[mt][nt][r]);
      }
    }
  // the region is written as T and read back as 16-byte vectors: keep the
  // compiler from moving a read above a write (the wave's LDS accesses then
  // complete in program order)
  asm volatile("" ::: "memory");
  const size_t es = sizeof(T);
  const bool vec = (reinterpret_cast<uintptr_t>(g.out) & 15) == 0 && (g.ldo * es) % 16 == 0 &&
                   (g.split <= 0 || ((reinterpret_cast<uintptr_t>(g.out2) & 15) == 0 &&
                                     (g.ldo2 * es) % 16 == 0));
  const uint4* src = reinterpret_cast<const uint4*>(region);
#pragma unroll
  for (int i = 0; i < (ROWS * PR + 63) / 64; ++i) {
    const int k = i * 64 + lane, lr = k / PR, p = k % PR;
    if (k >= ROWS * PR) break;
    const uint4 v = src[lr * PR + (p ^ (((lr >> 2) & SW) << SH))];
    const int64_t row = row0 + lr, c = n0 + (int64_t)p * EPL;
    if (row >= g.M) continue;
    const bool whole = c + EPL <= g.N && (g.split <= 0 || c + EPL <= g.split || c >= g.split);
    if (vec && whole) {
      T* dst = g.split > 0 && c >= g.split
                   ? static_cast<T*>(g.out2) + row * g.ldo2 + (c - g.split)
                   : static_cast<T*>(g.out) + row * g.ldo + c;
      *reinterpret_cast<uint4*>(dst) = v;
    } else {
      T e[EPL];
      __builtin_memcpy(e, &v, 16);
#pragma unroll
      for (int j = 0; j < EPL; ++j)
        if (c + j < g.N) {
          if (g.split > 0 && c + j >= g.split)
            static_cast<T*>(g.out2)[row * g.ldo2 + (c + j - g.split)] = e[j];
          else
            static_cast<T*>(g.out)[row * g.ldo + c + j] = e[j];
        }
    }
  }
}

// staged stores need room in the ring for every wave's rows (kStaged), or
// at least for 16 rows of every wave, staged one 16-row slab at a time
template <typename T, int MT, int NT, typename R>
constexpr bool kStaged =
    (size_t)(R::THREADS / 64) * 16 * MT * 16 * NT * sizeof(T) <= R::LDS_BYTES;
template <typename T, int NT, typename R>
constexpr bool kStagedSlab = (size_t)(R::THREADS / 64) * 16 * 16 * NT * sizeof(T) <= R::LDS_BYTES;

template <typename T, int MT, int NT, typename R>
__device__ __forceinline__ void store_tile(const GemmArgs& g, int64_t row0, int64_t n0,
                                           const f32x4 (&acc)[MT][NT], uint4* ring) {
  const int wave = threadIdx.x >> 6;
  if constexpr (kStaged<T, MT, NT, R>) {
    store_staged<T, MT, NT>(g, row0, n0, acc,
                            reinterpret_cast<T*>(ring) + (size_t)wave * 16 * MT * 16 * NT);
  } else if constexpr (kStagedSlab<T, NT, R>) {
    T* region = reinterpret_cast<T*>(ring) + (size_t)wave * 16 * 16 * NT;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      // the previous slab's read-back stays ahead of this slab's writes
      asm volatile("" ::: "memory");
      store_staged<T, 1, NT>(g, row0 + mt * 16, n0,
                             reinterpret_cast<const f32x4(&)[1][NT]>(acc[mt]), region);
    }
  } else {
    store_direct<T, MT, NT>(g, row0, n0, acc);
  }
}

}  // namespace
}  // namespace saga
