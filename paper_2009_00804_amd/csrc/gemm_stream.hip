// ApplyVertex in bfloat16, PLAIN and CONCAT with more than 80 columns: all
// columns of a row block (up to 208) in one workgroup, so that A is read once
// (which products take it: gemm_streams).  Measured (us, against 128-column tiles
// with swizzled weights): 232965 x (300 + 300) x 200 199 -> 122, 600000 x 300 x 300
// 402 -> 266, 600000 x 128 x 96 72 -> 58.  Loads bound it: 2.7 to 4.5 TB/s of the
// bytes it cannot do without.
#include <algorithm>

#include "gemm_device.h"

namespace saga {
namespace {

typedef __attribute__((address_space(3))) uint4 lds_uint4;

// A straight from global memory into registers, the packed weights through two
// LDS stages.  A chunk is 64 k: 128 bytes of an A row, and for every 16-column
// tile two 1 KB planes of Wt (32 k each) whose 16-byte pieces lie in the order
// the lanes read them, so a stage is one contiguous copy and a fragment read is
// free of bank conflicts.
//
// At the top of step i the weights of chunk i + 1 start on their way into the
// other stage and the A rows of chunk i + 2 into the registers chunk i leaves.
// The direct-to-LDS loads are written in assembly: the compiler would otherwise
// wait for every one in flight before any LDS read.  Loads return in order, so
// waiting until only the newest chunk's A loads are pending covers the weights.
// As built, the loop moves registers of pending A loads at its end, so every
// second step first waits for all loads in flight.
template <int MT, int NT, int NW>
struct Stream {
  typedef uint16_t T;
  static constexpr int THREADS = 64 * NW;
  static constexpr int BM = 16 * MT * NW, BN = 16 * NT;
  static constexpr int STAGE = NT * 128;  // 16-byte slots per stage
  static constexpr int RING_SLOTS = 2 * STAGE;
  static constexpr size_t LDS_BYTES = (size_t)RING_SLOTS * 16;
  static constexpr int LB = (STAGE + THREADS - 1) / THREADS;
  static constexpr int KC = 64;

  struct Ctx {
    const T* row[MT];
    int64_t K;
    const uint4* Wi;  // this column block's image: chunk c at c * STAGE
    lds_uint4* ring;
    int last, kmax;   // last chunk; first column of a row's last 16-byte piece
  };
  typedef uint4 AChunk[MT][2];

  // a piece that starts at or past K reads the row's last piece instead and is
  // masked before use
  __device__ __forceinline__ static void load_a(const Ctx& c, int chunk, AChunk& a) {
    const int lg = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = min(chunk * KC + (h * 4 + lg) * 8, c.kmax);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) a[mt][h] = *reinterpret_cast<const uint4*>(c.row[mt] + k);
    }
  }
  __device__ __forceinline__ static void mask(const Ctx& c, int chunk, AChunk& a) {
    const int lg = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t left = c.K - (chunk * KC + (h * 4 + lg) * 8);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        uint32_t w[4];
        __builtin_memcpy(w, &a[mt][h], 16);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          if (left <= 2 * d) w[d] = 0;
          else if (left == 2 * d + 1) w[d] &= 0xffffu;
        }
        __builtin_memcpy(&a[mt][h], w, 16);
      }
    }
  }
  __device__ __forceinline__ static void issue_b(const Ctx& c, int chunk) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint4* src = c.Wi + (int64_t)chunk * STAGE;
    const uint32_t dst = (uint32_t)(uintptr_t)(c.ring + (chunk & 1) * STAGE);
#pragma unroll
    for (int j = 0; j < LB; ++j) {
      const int s0 = j * THREADS + wave * 64;
      if (STAGE % THREADS == 0 || s0 < STAGE)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :
                     : "s"(__builtin_amdgcn_readfirstlane(dst + s0 * 16)), "v"((uint32_t)(s0 + lane) * 16u),
                       "s"(src)
                     : "memory", "m0");
    }
  }
  // U: register slot of chunk i
  template <int U>
  __device__ __forceinline__ static void step(const Ctx& c, int i, AChunk (&a)[2], f32x4 (&acc)[MT][NT]) {
    const int lane = threadIdx.x & 63;
    wait_vm<2 * MT>();  // chunk i landed (the newest loads are chunk i + 1's A)
    ring_barrier();     // for every wave; the other stage is free again
    const lds_uint4* Bs = c.ring + (i & 1) * STAGE;
    AChunk cur;  // (copied, so that the slot can be refilled at once)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int h = 0; h < 2; ++h) cur[mt][h] = a[U][mt][h];
    if (i < c.last) issue_b(c, i + 1);
    load_a(c, i + 2, a[U]);  // past the last chunk: its last piece again, never used
    __builtin_amdgcn_sched_barrier(0);
    if (i == c.last) mask(c, i, cur);
    // a column tile's fragments are read while the tile before it is multiplied
    bf16x8 b[2][2];
    auto read_b = [&](int nt) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        b[nt & 1][h] = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(
            Bs + (nt * 2 + h) * 64 + lane);
    };
    read_b(0);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      if (nt + 1 < NT) read_b(nt + 1);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          bf16x8 av;
          __builtin_memcpy(&av, &cur[mt][h], 16);
          acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, b[nt & 1][h], acc[mt][nt], 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  __device__ __forceinline__ static void phase(const T* __restrict__ A, int64_t lda, int64_t M, int64_t K,
                                               const uint4* __restrict__ Wi, int64_t tile0, uint4* ring,
                                               f32x4 (&acc)[MT][NT]) {
    Ctx c;
    int64_t off[MT];
    row_offsets(nullptr, lda, M, tile0 + (threadIdx.x >> 6) * MT * 16, off);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) c.row[mt] = A + off[mt];
    c.K = K;
    c.Wi = Wi;
    c.ring = (lds_uint4*)ring;
    c.last = (int)((K + KC - 1) / KC) - 1;
    c.kmax = (int)((K - 1) / 8 * 8);
    AChunk a[2];
    issue_b(c, 0);
    load_a(c, 0, a[0]);
    load_a(c, 1, a[1]);
    for (int i = 0;; i += 2) {
      step<0>(c, i, a, acc);
      if (i == c.last) break;
      step<1>(c, i + 1, a, acc);
      if (i + 1 == c.last) break;
    }
    ring_barrier();  // the stages may be refilled by a following phase
  }
};

// PLAIN / CONCAT.  The column blocks of one row block run on one XCD one after
// another (workgroup w goes to XCD w % 8).
template <int MT, int NT, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void k_gemm_stream(GemmArgs g, int ny) {
  typedef Stream<MT, NT, NW> R;
  __shared__ uint4 ring[R::RING_SLOTS];
  const int wave = threadIdx.x >> 6;
  const unsigned w = blockIdx.x / kXcds;
  const int y = (int)(w % (unsigned)ny);
  const int64_t tile0 = ((int64_t)(w / (unsigned)ny) * kXcds + blockIdx.x % kXcds) * R::BM;
  const int64_t n0 = (int64_t)y * R::BN;
  if (tile0 >= g.M) return;
  f32x4 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  const bool concat = g.mode == SAGA_GEMM_CONCAT;
  for (int ph = 0; ph < (concat ? 2 : 1); ++ph) {
    const int64_t K = ph ? g.K2 : g.K;
    const uint4* img = static_cast<const uint4*>(ph ? g.wt2 : g.wt);
    R::phase(static_cast<const uint16_t*>(ph ? g.a2 : g.a), ph ? g.lda2 : g.lda, g.M, K,
             img + (int64_t)y * ((K + 63) / 64) * R::STAGE, tile0, ring, acc);
  }
  const int64_t row0 = tile0 + wave * MT * 16;
  finish_tile(g, row0, n0, acc);
  store_tile<uint16_t, MT, NT, R>(g, row0, n0, acc, ring);
}

// The image Stream reads: column block b, chunk c, tile t of the block, half h
// of the chunk: 64 pieces of 8 k (piece p of column r at slot 16 p + r), zeros
// past N and K.  One thread per piece; blockIdx.y: the operand.
struct PackIn {
  const uint16_t* w;
  int64_t ldw, K;
  uint4* img;
};
__global__ __launch_bounds__(kThreads) void k_pack_stream(PackIn i1, PackIn i2, int64_t N, int nt, int ny) {
  const PackIn in = blockIdx.y ? i2 : i1;
  const int nch = (int)((in.K + 63) / 64);
  const int64_t s = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  if (s >= (int64_t)ny * nch * nt * 128) return;
  const int r = s & 15, p = (s >> 4) & 3, h = (s >> 6) & 1;
  const int64_t q = s >> 7;  // (b nch + c) nt + t
  const int t = (int)(q % nt), c = (int)(q / nt % nch), b = (int)(q / nt / nch);
  const int64_t n = ((int64_t)b * nt + t) * 16 + r, k0 = (int64_t)c * 64 + (h * 4 + p) * 8;
  const int64_t kn = n < N ? in.K : 0;
  uint32_t v[4];
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const uint32_t lo = k0 + 2 * d < kn ? in.w[(k0 + 2 * d) * in.ldw + n] : 0;
    const uint32_t hi = k0 + 2 * d + 1 < kn ? in.w[(k0 + 2 * d + 1) * in.ldw + n] : 0;
    v[d] = lo | hi << 16;
  }
  in.img[s] = make_uint4(v[0], v[1], v[2], v[3]);
}

// Column blocks of nt 16-column tiles, of equal width.  One block up to 13
// tiles: with long K or many rows it saves the second read of A (us, one block /
// two: 232965 x (300 + 300) x 140 109 / 132, x 170 115 / 135, x 200 122 / 140;
// 600000 x 300 x 190 187 / 206), but 9, 11 and 12 tiles of one short operand over
// fewer rows lose some of it (232965 x 300 x 190 75 / 63, 100000 x 72 x 170 29 /
// 24; x 160 20 / 20).  Past that blocks of at most ten (66211 x 524 x 250, 16
// tiles: one block 68, two 44 to 49; 600000 x 300 x 300, 19 tiles: two blocks 266,
// three 297).  Over few rows blocks of at most seven, for more workgroups (13864 x
// 55 x 196, tanh: 18 -> 15; 40000 x 72 x 190 17.4 / 15.1).
constexpr int64_t kFewRows = 32768;
struct StreamShape {
  int nt, ny;
};
StreamShape stream_shape(int64_t N, bool few) {
  StreamShape s;
  const int tiles = (int)((N + 15) / 16);
  s.ny = few ? (tiles + 6) / 7 : tiles <= 13 ? 1 : (tiles + 9) / 10;
  s.nt = (tiles + s.ny - 1) / s.ny;
  return s;
}
int64_t image_bytes(const StreamShape& s, int64_t K) {
  return (int64_t)s.ny * s.nt * ((K + 63) / 64) * 2048;
}

template <int MT, int NT, int NW>
hipError_t launch_stream(const GemmArgs& g, int ny, hipStream_t st) {
  typedef Stream<MT, NT, NW> R;
  const int64_t mt = (g.M + R::BM - 1) / R::BM;
  hipLaunchKernelGGL((k_gemm_stream<MT, NT, NW>), dim3((unsigned)((mt + kXcds - 1) / kXcds * kXcds * ny)),
                     dim3(R::THREADS), 0, st, g, ny);
  return hipGetLastError();
}
// Up to eight column tiles: 32 rows a wave over many rows, which halves the LDS
// reads per product (600000 x 256 x 128: 116 us, 121 with 16; 131072 x 512 x
// 256: 68, 74), else 16 (111353 x 173 x 119: 28, 34; 197125 x 345 x 236: 79,
// 83).  More: their accumulators leave room for 16 rows, and over many rows
// eight waves share the weights (us, eight / four: 600000 x (300 + 300) x 140 250 /
// 266, x 200 287 / 304, 232965 x (300 + 300) x 200 125 / 125, but one short operand
// at 131072 to 250000 rows 232965 x 300 x 160 58 / 51).
template <int NT>
hipError_t dispatch_stream(const GemmArgs& g, int ny, hipStream_t st) {
  if constexpr (NT > 8) {
    return g.M >= 131072 ? launch_stream<1, NT, 8>(g, ny, st) : launch_stream<1, NT, 4>(g, ny, st);
  } else {
    const int64_t k = g.K + (g.mode == SAGA_GEMM_CONCAT ? g.K2 : 0);
    const bool tall = g.M >= 400000 || (g.M >= 65536 && k > 448);
    return tall ? launch_stream<2, NT, 4>(g, ny, st) : launch_stream<1, NT, 4>(g, ny, st);
  }
}

}  // namespace

size_t stream_workspace_bytes(int64_t N, int64_t K, int64_t K2) {
  size_t most = 0;  // enough for any M
  for (const bool few : {false, true}) {
    const StreamShape s = stream_shape(N, few);
    most = std::max(most, (size_t)(image_bytes(s, K) + image_bytes(s, K2)));
  }
  return most;
}

// Workspace: the image of w, then of w2
hipError_t launch_gemm_stream(const GemmArgs& g0, hipStream_t st) {
  const bool cat = g0.mode == SAGA_GEMM_CONCAT;
  const StreamShape s = stream_shape(g0.N, g0.M < kFewRows);
  if (!g0.ws || g0.ws_bytes < stream_workspace_bytes(g0.N, g0.K, cat ? g0.K2 : 0)) return hipErrorInvalidValue;
  GemmArgs g = g0;
  char* ws = static_cast<char*>(g.ws);
  g.wt = ws;
  g.wt2 = ws + image_bytes(s, g.K);
  const int64_t most = std::max(image_bytes(s, g.K), cat ? image_bytes(s, g.K2) : 0) / 16;
  hipLaunchKernelGGL(k_pack_stream, dim3((unsigned)((most + kThreads - 1) / kThreads), cat ? 2 : 1),
                     dim3(kThreads), 0, st,
                     PackIn{static_cast<const uint16_t*>(g.w), g.ldw, g.K, reinterpret_cast<uint4*>(ws)},
                     PackIn{static_cast<const uint16_t*>(g.w2), g.ldw2, g.K2,
                            reinterpret_cast<uint4*>(ws + image_bytes(s, g.K))},
                     g.N, s.nt, s.ny);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  switch (s.nt) {
    case 3: return dispatch_stream<3>(g, s.ny, st);
    case 4: return dispatch_stream<4>(g, s.ny, st);
    case 5: return dispatch_stream<5>(g, s.ny, st);
    case 6: return dispatch_stream<6>(g, s.ny, st);
    case 7: return dispatch_stream<7>(g, s.ny, st);
    case 8: return dispatch_stream<8>(g, s.ny, st);
    case 9: return dispatch_stream<9>(g, s.ny, st);
    case 10: return dispatch_stream<10>(g, s.ny, st);
    case 11: return dispatch_stream<11>(g, s.ny, st);
    case 12: return dispatch_stream<12>(g, s.ny, st);
    case 13: return dispatch_stream<13>(g, s.ny, st);
    default: return hipErrorInvalidValue;  // (over 80 columns: 3 to 13 tiles a block)
  }
}

}  // namespace saga
