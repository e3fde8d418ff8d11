// ApplyVertex: the dense per-vertex transform (Sec. 3.2 "ApplyVertex" of
// the paper: all vertices batched into one GEMM, Table III) on the CDNA4
// matrix cores, with the layer's epilogue fused (degree row scaling, bias,
// activation, the two-operand concat form [a | a2][w ; w2], and the GRU
// gate math of GGNN's ApplyVertex, Fig. 2).
//
// Tiling: a workgroup of NW waves owns BM = 16 MT NW rows and BN = 16 NT
// columns; wave w computes rows [16 MT w, 16 MT (w + 1)) of the tile as
// MT x NT blocks of 16 x 16 with
//   float32 : v_mfma_f32_16x16x4f32   (4 k per instruction; narrow products
//             only, see gemm_splits; the others are in gemm_split.hip)
//   bfloat16: v_mfma_f32_16x16x32_bf16 (32 k per instruction)
//
// Data path.  K is cut into chunks of 128 bytes per row (32 float32 or 64
// bfloat16 values).  Each wave owns its A rows, so A needs no sharing: it goes
// straight from global memory into registers.  The BN rows of the packed
// weights Wt (W transposed, zero-padded to whole tiles, built in the workspace
// by k_pack_wt) go into one stage of an S-stage LDS ring with direct-to-LDS
// loads (global_load_lds_dwordx4); a chunk's A and Wt loads are issued
// together, S - 1 chunks ahead, so one vmcnt wait covers both.  Inside a
// 128-byte row the eight 16-byte pieces are XOR swizzled (piece p of row r at
// slot 8 r + (p ^ ((r >> 1) & 7))), so that a fragment read -- 16 rows at one
// k offset -- touches every LDS bank once.  A lane's 16-byte fragment holds
// EPL consecutive k of one row; A and Wt use the same k order, so the products
// are exact sums over k.  The chunk holding the end of K is masked with zeros
// past column K.
#include <algorithm>
#include <type_traits>

#include "gemm_device.h"

namespace saga {
namespace {

template <typename T, int MT, int NT, int S, int NW = 4>
struct RegA {
  typedef typename Mma<T>::Frag Frag;
  static constexpr int THREADS = 64 * NW;  // NW waves, each 16 MT rows
  static constexpr int BM = 16 * MT * NW, BN = 16 * NT;
  static constexpr int B_SLOTS = BN * 8;
  static constexpr int STAGE = B_SLOTS;
  static constexpr int RING_SLOTS = S * STAGE;
  static constexpr int LA = 2 * MT;  // 16-byte A loads per lane per chunk
  static constexpr int LB = (B_SLOTS + THREADS - 1) / THREADS;
  static constexpr int LMIN = LA + B_SLOTS / THREADS;
  static_assert(B_SLOTS % 64 == 0, "B tile must be whole wave loads");
  static_assert(S >= 2 && (S - 2) * LMIN < 64, "vmcnt range");
  static constexpr size_t LDS_BYTES = (size_t)RING_SLOTS * 16;

  // fragment (h, mt) of chunk k0: the lane's row mt, columns
  // k0 + (4 h + lane / 16) EPL ..  A piece that starts at or past K reads
  // the last piece of the row instead and is zeroed by mask() before use.  A
  // piece that starts below K ends within the row's ld (a multiple of 16
  // bytes).
  __device__ __forceinline__ static void load_a(const T* __restrict__ A,
                                                const int64_t (&off)[MT], int64_t K, int64_t k0,
                                                Frag (&a)[2][MT]) {
    constexpr int EPL = Mma<T>::EPL;
    const int lane = threadIdx.x & 63, lg = lane >> 4;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const int64_t k = k0 + (h * 4 + lg) * EPL;
        const int64_t kk = k < K ? k : (K - 1) / EPL * EPL;
        const uint4 v = *reinterpret_cast<const uint4*>(A + off[mt] + kk);
        __builtin_memcpy(&a[h][mt], &v, 16);
      }
  }
  // zero the values at columns >= K (the tail chunk)
  __device__ __forceinline__ static void mask(int64_t K, int64_t k0, Frag (&a)[2][MT]) {
    constexpr int EPL = Mma<T>::EPL;
    const int lg = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t left = K - (k0 + (h * 4 + lg) * EPL);
      const int nv = left <= 0 ? 0 : left >= EPL ? EPL : (int)left;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        uint32_t w[4];
        __builtin_memcpy(w, &a[h][mt], 16);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          if constexpr (EPL == 4) {
            if (d >= nv) w[d] = 0;
          } else {
            if (2 * d >= nv) w[d] = 0;
            else if (2 * d + 1 >= nv) w[d] &= 0xffffu;
          }
        }
        __builtin_memcpy(&a[h][mt], w, 16);
      }
    }
  }
  __device__ __forceinline__ static void issue_b(const T* __restrict__ Wt, int64_t kp, int64_t n0,
                                                 int64_t k0, uint4* st) {
    constexpr int EPL = Mma<T>::EPL;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < LB; ++j) {
      const int s0 = j * THREADS + wave * 64;
      if (s0 < B_SLOTS) {
        const int s = s0 + lane, n = s >> 3, p = (s & 7) ^ ((n >> 1) & 7);
        __builtin_amdgcn_global_load_lds(Wt + (n0 + n) * kp + k0 + p * EPL, (lds_ptr)(st + s0), 16, 0, 0);
      }
    }
  }
  __device__ __forceinline__ static void wait_stages(int later) {
    if constexpr (S >= 4) {
      if (later >= 2) { wait_vm<2 * LMIN>(); return; }
    }
    if constexpr (S >= 3) {
      if (later == 1) { wait_vm<LMIN>(); return; }
    }
    wait_vm<0>();
  }
  __device__ __forceinline__ static void compute(const uint4* Bs, const Frag (&a)[2][MT],
                                                 f32x4 (&acc)[MT][NT]) {
    const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
    Frag b[2][NT];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const uint4 v = Bs[swz(nt * 16 + lr, h * 4 + lg)];
        __builtin_memcpy(&b[h][nt], &v, 16);
      }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
              acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[h][mt][c], b[h][nt][c], acc[mt][nt], 0, 0, 0);
      } else {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[h][mt], b[h][nt], acc[mt][nt], 0, 0, 0);
      }
    }
  }

  struct Ctx {
    const T* A; int64_t K;
    const T* Wt; int64_t kp, n0;
    int64_t off[MT];
    uint4* ring;
    int nch, last;
  };

  // chunk i = i0 + U: uses register slot U and ring stage U
  template <int U>
  __device__ __forceinline__ static void step(const Ctx& c, int i0, Frag (&a)[S][2][MT],
                                              f32x4 (&acc)[MT][NT]) {
    constexpr int KC = Mma<T>::KC;
    constexpr int NU = (U + S - 1) % S;
    const int i = i0 + U;
    if (i >= c.nch) return;
    wait_stages(c.last - i < S - 2 ? c.last - i : S - 2);  // chunk i's loads landed
    ring_barrier();  // every wave's; stage i - 1 is free again
    if (i + S - 1 < c.nch) {
      load_a(c.A, c.off, c.K, (int64_t)(i + S - 1) * KC, a[NU]);
      issue_b(c.Wt, c.kp, c.n0, (int64_t)(i + S - 1) * KC, c.ring + NU * STAGE);
    }
    if (i == c.last) mask(c.K, (int64_t)i * KC, a[U]);
    compute(c.ring + U * STAGE, a[U], acc);
  }

  // acc += A[tile0 .. tile0 + BM) x W[:, n0 .. n0 + BN); chunk i uses
  // register slot i % S and ring stage i % S (the loop is unrolled by S so
  // both are compile-time)
  __device__ __forceinline__ static void phase(const T* __restrict__ A, int64_t lda, int64_t M,
                                               int64_t K, const T* __restrict__ Wt, int64_t kp,
                                               int64_t tile0, int64_t n0, uint4* ring,
                                               f32x4 (&acc)[MT][NT],
                                               const int32_t* __restrict__ arow = nullptr) {
    static_assert(S <= 4, "unrolled for at most four stages");
    constexpr int KC = Mma<T>::KC;
    Ctx c;
    c.A = A; c.K = K; c.Wt = Wt; c.kp = kp; c.n0 = n0;
    row_offsets(arow, lda, M, tile0 + (threadIdx.x >> 6) * MT * 16, c.off);
    c.ring = ring;
    c.nch = (int)((K + KC - 1) / KC);
    c.last = c.nch - 1;
    Frag a[S][2][MT];
#pragma unroll
    for (int j = 0; j < S - 1; ++j)
      if (j < c.nch) {
        load_a(A, c.off, K, (int64_t)j * KC, a[j]);
        issue_b(Wt, kp, n0, (int64_t)j * KC, ring + j * STAGE);
      }
    for (int i0 = 0; i0 < c.nch; i0 += S) {
      step<0>(c, i0, a, acc);
      step<1>(c, i0, a, acc);
      if constexpr (S > 2) step<2>(c, i0, a, acc);
      if constexpr (S > 3) step<3>(c, i0, a, acc);
    }
    ring_barrier();  // the ring may be refilled by a following phase
  }
};

// Wt[n][k] = W[k][n] for n < N, k < K, else 0; Wt is Np x Kp with ld Kp
template <typename T>
__global__ __launch_bounds__(kThreads) void k_pack_wt(const T* __restrict__ W, int64_t ldw,
                                                      int64_t K, int64_t N, T* __restrict__ Wt,
                                                      int64_t Kp, int64_t Np) {
  const int64_t total = Np * Kp;
  for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * kThreads) {
    const int64_t n = i / Kp, k = i - n * Kp;
    Wt[i] = (n < N && k < K) ? W[k * ldw + n] : T(0);
  }
}

// bfloat16, 128 columns from column 0, through registers: three lane
// exchanges (partners lr ^ 1 and lr ^ 2 by DPP, lr ^ 4 by swizzle; lr =
// lane % 16 with bits b0..b3, lg = lane / 16) turn the accumulator layout
// (rows 4 lg + r of column 16 t + lr) into whole 16-byte row pieces: the
// lane then holds, for q = 0..3, row 4 lg + 2 b0 + b1 at columns
// 16 (2 q + b2) + 8 b3 .. + 7, and stores each with one 16-byte store
// (element by element where the piece is not whole, as for the staged
// stores).  For callers whose LDS is taken.
__device__ __forceinline__ uint32_t pack_bf2(uint32_t lo, uint32_t hi) {
  return (lo & 0xffffu) | (hi << 16);
}
template <int MT>
__device__ __forceinline__ void store_shuffled(const GemmArgs& g, int64_t row0,
                                               const f32x4 (&acc)[MT][8]) {
  typedef uint16_t T;
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const bool b0 = lr & 1, b1 = (lr >> 1) & 1, b2 = (lr >> 2) & 1, b3 = (lr >> 3) & 1;
  const bool vec = (reinterpret_cast<uintptr_t>(g.out) & 15) == 0 && (g.ldo * 2) % 16 == 0 &&
                   (g.split <= 0 || ((reinterpret_cast<uintptr_t>(g.out2) & 15) == 0 &&
                                     (g.ldo2 * 2) % 16 == 0));
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    uint32_t z[8][2];  // row 4 lg + 2 b0 + b1, columns 16 t + 4 (lr / 4) .. + 3
#pragma unroll
    for (int nt = 0; nt < 8; ++nt) {
      uint32_t x[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] = Mma<T>::from_f(acc[mt][nt][r]);
      // lanes with b0 = 0 keep rows 0, 1 and those with b0 = 1 rows 2, 3,
      // now for the column pair (lr & ~1, + 1)
      const uint32_t r1 = (uint32_t)__builtin_amdgcn_mov_dpp(
          (int)(b0 ? pack_bf2(x[0], x[1]) : pack_bf2(x[2], x[3])), 0xB1, 0xF, 0xF, true);
      const uint32_t y0 = b0 ? pack_bf2(r1, x[2]) : pack_bf2(x[0], r1);
      const uint32_t y1 = b0 ? pack_bf2(r1 >> 16, x[3]) : pack_bf2(x[1], r1 >> 16);
      // lanes with b1 = 0 keep the first of the two rows, b1 = 1 the second,
      // now for four columns from lr & ~3
      const uint32_t r2 = (uint32_t)__builtin_amdgcn_mov_dpp((int)(b1 ? y0 : y1), 0x4E, 0xF, 0xF, true);
      z[nt][0] = b1 ? r2 : y0;
      z[nt][1] = b1 ? y1 : r2;
    }
    const int64_t row = row0 + mt * 16 + 4 * lg + 2 * b0 + b1;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      // lanes with b2 = 0 keep tile 2 q and those with b2 = 1 tile 2 q + 1,
      // now for eight columns from 8 b3
      const uint32_t s0 = b2 ? z[2 * q][0] : z[2 * q + 1][0];
      const uint32_t s1 = b2 ? z[2 * q][1] : z[2 * q + 1][1];
      const uint32_t r0 = (uint32_t)__builtin_amdgcn_ds_swizzle((int)s0, 0x101F);
      const uint32_t r3 = (uint32_t)__builtin_amdgcn_ds_swizzle((int)s1, 0x101F);
      const uint4 w = b2 ? uint4{r0, r3, z[2 * q + 1][0], z[2 * q + 1][1]}
                         : uint4{z[2 * q][0], z[2 * q][1], r0, r3};
      const int64_t c = 16 * (2 * q + (int)b2) + 8 * (int)b3;
      if (row >= g.M) continue;
      const bool whole = c + 8 <= g.N && (g.split <= 0 || c + 8 <= g.split || c >= g.split);
      if (vec && whole) {
        T* dst = g.split > 0 && c >= g.split
                     ? static_cast<T*>(g.out2) + row * g.ldo2 + (c - g.split)
                     : static_cast<T*>(g.out) + row * g.ldo + c;
        *reinterpret_cast<uint4*>(dst) = w;
      } else {
        T e[8];
        __builtin_memcpy(e, &w, 16);
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (c + j < g.N) {
            if (g.split > 0 && c + j >= g.split)
              static_cast<T*>(g.out2)[row * g.ldo2 + (c + j - g.split)] = e[j];
            else
              static_cast<T*>(g.out)[row * g.ldo + c + j] = e[j];
          }
      }
    }
  }
}

// PLAIN / CONCAT
template <typename T, int MT, int NT, typename R>
__global__ __launch_bounds__(R::THREADS) void k_gemm(GemmArgs g) {
  __shared__ uint4 ring[R::RING_SLOTS];
  const int wave = threadIdx.x >> 6;
  const int64_t tile0 = (int64_t)blockIdx.x * R::BM;
  const int64_t n0 = (int64_t)blockIdx.y * R::BN;
  f32x4 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  R::phase(static_cast<const T*>(g.a), g.lda, g.M, g.K, static_cast<const T*>(g.wt), g.kp, tile0,
           n0, ring, acc);
  if (g.mode == SAGA_GEMM_CONCAT)
    R::phase(static_cast<const T*>(g.a2), g.lda2, g.M, g.K2, static_cast<const T*>(g.wt2), g.kp2,
             tile0, n0, ring, acc);
  const int64_t row0 = tile0 + wave * MT * 16;
  finish_tile(g, row0, n0, acc);
  store_tile<T, MT, NT, R>(g, row0, n0, acc, ring);
}

// bfloat16 PLAIN with the weights resident: one workgroup per CU holds
// all of W^T for its 128 output columns in LDS (k in half chunks of 32,
// column n = 16 t + r: piece p of 8 k at slot ((h * 8 + t) * 4 + p) * 16 + r,
// so the 16 lanes that read one piece of 16 columns read 256 contiguous
// bytes, free of bank conflicts), loaded once.  Each wave
// then streams its own 16 MT-row tiles (tile q = wave id, wave id + all
// waves, ...) through D register slots of A chunks; the stream runs on
// across tiles, so the next tile's first chunks are in flight during the
// last chunks and the epilogue of the current one.  No workgroup barrier
// after the weights land, and only A loads on the vmcnt counter, so a wait
// for one chunk never drains the chunks behind it.  The LDS being taken,
// the epilogue stores through lane exchanges (store_shuffled).
constexpr int kResHalfChunks = 19;  // half chunks of 32 k: K <= 608, 152 KB of LDS

template <int MT, int NW, int D>
__global__ __launch_bounds__(64 * NW) void k_gemm_bres(GemmArgs g) {
  typedef uint16_t T;
  typedef RegA<T, MT, 8, 2, NW> R;
  typedef typename Mma<T>::Frag Frag;
  constexpr int NT = 8, KC = Mma<T>::KC;
  static_assert(D >= 2 && D <= 8, "A slots");
  __shared__ uint4 wres[kResHalfChunks * 128 * 4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const T* A = static_cast<const T*>(g.a);
  const T* Wt = static_cast<const T*>(g.wt);
  const int hc = (int)((g.K + 31) / 32);  // half chunks held (<= kResHalfChunks, checked by the host)
  // weights: slot s of half chunk h, column n, piece p
  {
    const int slots = hc * 128 * 4;
    for (int s0 = wave * 64; s0 < slots; s0 += NW * 64) {
      const int s = s0 + lane, h = s / 512, p = (s / 16) % 4;
      // columns past N (not packed when N < 128) repeat column N - 1; their
      // outputs are never stored
      const int n = min((s / 64) % 8 * 16 + s % 16, (int)g.N - 1);
      __builtin_amdgcn_global_load_lds(Wt + (int64_t)n * g.kp + h * 32 + p * 8, (lds_ptr)(wres + s0),
                                       16, 0, 0);
    }
    wait_vm<0>();
    ring_barrier();
  }
  const int nch = (int)((g.K + KC - 1) / KC);
  const int64_t ntile = (g.M + 16 * MT - 1) / (16 * MT);
  const int64_t gw = (int64_t)blockIdx.x * NW + wave, stride = (int64_t)gridDim.x * NW;
  if (gw >= ntile) return;
  const int64_t mytiles = (ntile - gw + stride - 1) / stride;
  const int64_t total = mytiles * nch;  // chunks in this wave's stream
  // the stream's read position (tile q_pf, chunk c_pf) and compute position
  // (tile q_cur, chunk c_cur), advanced one chunk at a time
  int64_t q_pf = gw, q_cur = gw;
  int c_pf = 0, c_cur = 0;
  int64_t off_pf[MT];
  row_offsets(nullptr, g.lda, g.M, q_pf * 16 * MT, off_pf);
  auto issue_next = [&](Frag (&a)[2][MT]) {
    R::load_a(A, off_pf, g.K, (int64_t)c_pf * KC, a);
    if (++c_pf == nch) {  // rows of tiles past the last are clamped to row M - 1
      c_pf = 0;
      q_pf += stride;
      row_offsets(nullptr, g.lda, g.M, q_pf * 16 * MT, off_pf);
    }
  };
  Frag a[D][2][MT];
  f32x4 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  // chunk i of the stream from register slot U; FULL: the read of chunk
  // i + D - 1 exists (the steady state: no conditional loads, so the
  // compiler's waits count exactly the D - 1 chunks in flight)
  auto step = [&](auto u_c, auto full_c, int64_t i) {
    constexpr int U = decltype(u_c)::value;
    constexpr bool FULL = decltype(full_c)::value;
    if constexpr (FULL) {
      issue_next(a[(U + D - 1) % D]);
    } else {
      if (i >= total) return;
      if (i + D - 1 < total) issue_next(a[(U + D - 1) % D]);
    }
    const int c = c_cur;
    if (c == nch - 1) R::mask(g.K, (int64_t)c * KC, a[U]);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int hh = 2 * c + h;
      if (hh >= hc) break;  // past K: the A values there are zero, the weights not held
      Frag b[NT];
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const uint4 v = wres[((hh * 8 + nt) * 4 + lg) * 16 + lr];
        __builtin_memcpy(&b[nt], &v, 16);
      }
      __builtin_amdgcn_sched_barrier(0);  // every fragment read ahead of the MFMAs
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[U][h][mt], b[nt], acc[mt][nt], 0, 0, 0);
    }
    if (++c_cur == nch) {
      const int64_t row0 = q_cur * 16 * MT;
      finish_tile(g, row0, 0, acc);
      store_shuffled<MT>(g, row0, acc);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
      c_cur = 0;
      q_cur += stride;
    }
  };
  using T1 = std::true_type;
  using T0 = std::false_type;
  int64_t i0 = 0;
  if (total >= 2 * D - 1) {
    // the first D - 1 chunks, unconditionally: the steady loop below is
    // entered only from here, with exactly D - 1 chunks in flight
#pragma unroll
    for (int j = 0; j < D - 1; ++j) issue_next(a[j]);
    // steady state: every step's read exists (i + D - 1 < total)
    for (; i0 + 2 * D - 1 <= total; i0 += D) {
      step(std::integral_constant<int, 0>{}, T1{}, i0);
      step(std::integral_constant<int, 1>{}, T1{}, i0 + 1);
      if constexpr (D > 2) step(std::integral_constant<int, 2>{}, T1{}, i0 + 2);
      if constexpr (D > 3) step(std::integral_constant<int, 3>{}, T1{}, i0 + 3);
      if constexpr (D > 4) step(std::integral_constant<int, 4>{}, T1{}, i0 + 4);
      if constexpr (D > 5) step(std::integral_constant<int, 5>{}, T1{}, i0 + 5);
      if constexpr (D > 6) step(std::integral_constant<int, 6>{}, T1{}, i0 + 6);
      if constexpr (D > 7) step(std::integral_constant<int, 7>{}, T1{}, i0 + 7);
    }
  } else {
#pragma unroll
    for (int j = 0; j < D - 1; ++j)
      if (j < total) issue_next(a[j]);
  }
  // the last chunks, fewer or no reads
  for (; i0 < total; i0 += D) {
    step(std::integral_constant<int, 0>{}, T0{}, i0);
    step(std::integral_constant<int, 1>{}, T0{}, i0 + 1);
    if constexpr (D > 2) step(std::integral_constant<int, 2>{}, T0{}, i0 + 2);
    if constexpr (D > 3) step(std::integral_constant<int, 3>{}, T0{}, i0 + 3);
    if constexpr (D > 4) step(std::integral_constant<int, 4>{}, T0{}, i0 + 4);
    if constexpr (D > 5) step(std::integral_constant<int, 5>{}, T0{}, i0 + 5);
    if constexpr (D > 6) step(std::integral_constant<int, 6>{}, T0{}, i0 + 6);
    if constexpr (D > 7) step(std::integral_constant<int, 7>{}, T0{}, i0 + 7);
  }
}

// GRU: acc1 = a w (input gates), acc2 = a2 w2 (hidden gates), column blocks
// (r, z, n) of width F = NT3 * 16; hidden state h = a2
template <typename T, int NT3, int S>
__global__ __launch_bounds__(kThreads) void k_gemm_gru(GemmArgs g) {
  constexpr int NT = 3 * NT3;
  typedef RegA<T, 1, NT, S> R;
  __shared__ uint4 ring[R::RING_SLOTS];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t tile0 = (int64_t)blockIdx.x * R::BM;
  f32x4 acc1[1][NT], acc2[1][NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    acc1[0][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    acc2[0][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const T* h = static_cast<const T*>(g.a2);
  R::phase(static_cast<const T*>(g.a), g.lda, g.M, g.K, static_cast<const T*>(g.wt), g.kp, tile0,
           0, ring, acc1);
  R::phase(h, g.lda2, g.M, g.K2, static_cast<const T*>(g.wt2), g.kp2, tile0, 0, ring, acc2);
  const int F = NT3 * 16;
  const int64_t row0 = tile0 + wave * 16;
  T* out = static_cast<T*>(g.out);
  // biases and previous states are all loaded before the first store (a
  // load after a store the compiler cannot tell apart from it would wait)
  float bi[3][NT3], bh[3][NT3], hp[4][NT3];
#pragma unroll
  for (int t = 0; t < NT3; ++t) {
    const int c = t * 16 + (lane & 15);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      bi[q][t] = g.bias ? g.bias[q * F + c] : 0.f;
      bh[q][t] = g.bias2 ? g.bias2[q * F + c] : 0.f;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = row0 + 4 * (lane >> 4) + r;
      hp[r][t] = row < g.M ? Mma<T>::to_f(h[row * g.lda2 + c]) : 0.f;
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t row = row0 + 4 * (lane >> 4) + r;
    if (row >= g.M) continue;
#pragma unroll
    for (int t = 0; t < NT3; ++t) {
      const int c = t * 16 + (lane & 15);
      const float rr = sigmoidf_(acc1[0][t][r] + bi[0][t] + acc2[0][t][r] + bh[0][t]);
      const float zz = sigmoidf_(acc1[0][t + NT3][r] + bi[1][t] + acc2[0][t + NT3][r] + bh[1][t]);
      const float nn =
          tanhf(acc1[0][t + 2 * NT3][r] + bi[2][t] + rr * (acc2[0][t + 2 * NT3][r] + bh[2][t]));
      out[row * g.ldo + c] = Mma<T>::from_f((1.0f - zz) * nn + zz * hp[r][t]);
    }
  }
}

// Grouped: row q of the output is row arow[q] of A times the weight of the
// group whose row range holds q (R-GCN's per-relation transform of the
// distinct (relation, source) pairs).  Group ranges are whole tiles, so a
// tile finds its group by a binary search of grp_ptr and multiplies by that
// group's packed weight; tiles from grp_ptr[groups] on are idle.  Rows whose
// map entry is negative (range padding) are written as zeros.
template <typename T, int MT, int NT, typename R>
__global__ __launch_bounds__(R::THREADS) void k_gemm_grouped(GemmArgs g) {
  static_assert(R::BM == kRelTile, "grouped tiles must match the row-range padding");
  __shared__ uint4 ring[R::RING_SLOTS];
  if ((g.err1 && *g.err1) || (g.err2 && *g.err2)) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t tile0 = (int64_t)blockIdx.x * R::BM;
  const int64_t rows = g.grp_ptr[g.groups];
  if (tile0 >= rows) return;
  int lo = 0, hi = g.groups;  // grp_ptr[lo] <= tile0 < grp_ptr[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (g.grp_ptr[mid] <= tile0) lo = mid;
    else hi = mid;
  }
  const int64_t n0 = (int64_t)blockIdx.y * R::BN;
  f32x4 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  R::phase(static_cast<const T*>(g.a), g.lda, g.M, g.K,
           static_cast<const T*>(g.wt) + (int64_t)lo * g.wt_group_stride, g.kp, tile0, n0, ring,
           acc, g.arow);
  const int64_t row0 = tile0 + wave * MT * 16;
  // rows of range padding (map entry < 0) are written as zeros
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (g.arow[row0 + mt * 16 + 4 * (lane >> 4) + r] < 0) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt][r] = 0.0f;
      }
  store_tile<T, MT, NT, R>(g, row0, n0, acc, ring);
}

// Wt[grp][n][k] = W[grp K + k][n] for n < N, k < K, else 0; each group's
// packed weight is Np x Kp with ld Kp
template <typename T>
__global__ __launch_bounds__(kThreads) void k_pack_wt_grouped(const T* __restrict__ W,
                                                              int64_t ldw, int64_t K, int64_t N,
                                                              int groups, T* __restrict__ Wt,
                                                              int64_t Kp, int64_t Np) {
  const int64_t per = Np * Kp, total = per * groups;
  for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * kThreads) {
    const int64_t grp = i / per, j = i - grp * per;
    const int64_t n = j / Kp, k = j - n * Kp;
    Wt[i] = (n < N && k < K) ? W[(grp * K + k) * ldw + n] : T(0);
  }
}

// ---------------------------------------------------------------------------
// host side: tiling choice, weight packing, launch
// ---------------------------------------------------------------------------
struct Tiling {
  int nt, stages;  // column tiles; stages of the weight ring
};

// k chunks of a K-long operand
int64_t chunks(int dtype, int64_t K) {
  const int64_t kc = dtype == SAGA_BF16 ? Mma<uint16_t>::KC : Mma<float>::KC;
  return (K + kc - 1) / kc;
}

Tiling choose(int dtype, int mode, int64_t N, int64_t K) {
  if (mode == SAGA_GEMM_GRU) return Tiling{(int)(N / 16), 4};
  const int64_t nt = (N + 15) / 16;
  // narrow tiles: with at most four k chunks two stages suffice (the
  // registers two more A slots would hold buy occupancy instead; measured
  // on the 2^21 x 128 x 41 bfloat16 transform: 0.175 -> 0.162 ms)
  if (nt <= 5) return Tiling{(int)nt, chunks(dtype, K) <= 4 ? 2 : 4};
  return Tiling{8, 4};  // 128-column tiles; also the weight-resident kernel's packed rows
}

int kc_of(int dtype) { return dtype == SAGA_BF16 ? Mma<uint16_t>::KC : Mma<float>::KC; }

struct Packed {
  int64_t np, kp, kp2;
  size_t off2, bytes;
};

Packed packed_layout(int dtype, int mode, int64_t N, int64_t K, int64_t K2) {
  const Tiling t = choose(dtype, mode, N, K);
  const int64_t bn = 16 * t.nt, kc = kc_of(dtype);
  const size_t es = dtype == SAGA_BF16 ? 2 : 4;
  Packed p;
  p.np = (N + bn - 1) / bn * bn;
  p.kp = (K + kc - 1) / kc * kc;
  p.kp2 = mode == SAGA_GEMM_PLAIN ? 0 : (K2 + kc - 1) / kc * kc;
  const size_t b1 = ((size_t)p.np * p.kp * es + 255) / 256 * 256;
  p.off2 = b1;
  p.bytes = b1 + ((size_t)p.np * p.kp2 * es + 255) / 256 * 256;
  return p;
}

template <typename T, int MT, int NT, typename R>
hipError_t launch_plain(const GemmArgs& g, hipStream_t st) {
  static_assert(R::LDS_BYTES <= 160 * 1024, "LDS ring too large");
  dim3 grid((unsigned)((g.M + R::BM - 1) / R::BM), (unsigned)((g.N + R::BN - 1) / R::BN));
  hipLaunchKernelGGL((k_gemm<T, MT, NT, R>), grid, dim3(R::THREADS), 0, st, g);
  return hipGetLastError();
}

template <typename T, int NT>
hipError_t launch_nt(const GemmArgs& g, const Tiling& t, hipStream_t st) {
  if (t.stages == 2) return launch_plain<T, 2, NT, RegA<T, 2, NT, 2>>(g, st);
  return launch_plain<T, 2, NT, RegA<T, 2, NT, 4>>(g, st);
}

// weight-resident bfloat16 kernel: one workgroup per CU (its LDS holds the
// weights), or fewer when there are fewer tiles than waves
template <int MT, int NW, int D>
hipError_t launch_bres(const GemmArgs& g, hipStream_t st) {
  static int cus = [] {
    int dev = 0, n = 256;
    if (hipGetDevice(&dev) == hipSuccess)
      (void)hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
    return n > 0 ? n : 256;
  }();
  const int64_t tiles = (g.M + 16 * MT - 1) / (16 * MT);
  const int64_t wgs = std::max<int64_t>(1, std::min<int64_t>(cus, (tiles + NW - 1) / NW));
  hipLaunchKernelGGL((k_gemm_bres<MT, NW, D>), dim3((unsigned)wgs), dim3(64 * NW), 0, st, g);
  return hipGetLastError();
}

// The weight-resident kernel takes bfloat16 PLAIN products with 80 < N <= 128
// (narrower outputs use the narrow tiles) and K up to 608: from K = 256 on
// always, two 16-row tiles per wave and three A slots (2^21 rows x 128 columns
// against streamed weights, gemm_stream.hip: 0.353 / 0.362 ms at K = 256, 0.454 /
// 0.477 at 384, 0.663 / 0.679 at 602; four slots spill registers); from K = 192
// on over many rows, one tile per wave and four slots (us, resident / streamed:
// 500,000 x 208 x 128 81 / 89, x 240 x 96 85 / 89, x 192 x 128 79 / 83, but x 192 x
// 96 74 / 79 the other way; 400,000 x 240 x 128 70 / 78, but x 192 x 128 67 / 61).
bool takes_bres(int dtype, int mode, int64_t M, int64_t N, int64_t K) {
  if (dtype != SAGA_BF16 || mode != SAGA_GEMM_PLAIN || N <= 80 || N > 128 || K > 32 * kResHalfChunks) return false;
  if (K >= 256) return true;
  return N > 112 ? K >= 192 && M >= (K >= 224 ? 350000 : 450000) : K > 192 && M >= 450000;
}

template <typename T>
hipError_t dispatch(const GemmArgs& g, hipStream_t st) {
  if constexpr (sizeof(T) == 2)
    if (takes_bres(g.dtype, g.mode, g.M, g.N, g.K))
      return g.K < 256 ? launch_bres<1, 8, 4>(g, st) : launch_bres<2, 8, 3>(g, st);
  const Tiling t = choose(g.dtype, g.mode, g.N, g.mode == SAGA_GEMM_CONCAT ? g.K + g.K2 : g.K);
  if constexpr (sizeof(T) == 2) {  // float32: gemm_split.hip
    if (g.mode == SAGA_GEMM_GRU) {
      dim3 grid((unsigned)((g.M + 63) / 64));
      // two stages when both products have at most four k chunks (as for the
      // narrow plain tiles)
      const bool two = chunks(g.dtype, std::max(g.K, g.K2)) <= 4;
#define SAGA_GRU(N3)                                                                     \
    if (two) hipLaunchKernelGGL((k_gemm_gru<T, N3, 2>), grid, dim3(kThreads), 0, st, g);  \
    else hipLaunchKernelGGL((k_gemm_gru<T, N3, 4>), grid, dim3(kThreads), 0, st, g)
      switch (t.nt) {
        case 3: SAGA_GRU(1); break;
        case 6: SAGA_GRU(2); break;
        case 9: SAGA_GRU(3); break;
        case 12: SAGA_GRU(4); break;
        default: return hipErrorInvalidValue;
      }
#undef SAGA_GRU
      return hipGetLastError();
    }
  }
  switch (t.nt) {
    case 1: return launch_nt<T, 1>(g, t, st);
    case 2: return launch_nt<T, 2>(g, t, st);
  }
  if constexpr (sizeof(T) == 2) {  // float32 past two column tiles: gemm_splits
    switch (t.nt) {
      case 3: return launch_nt<T, 3>(g, t, st);
      case 4: return launch_nt<T, 4>(g, t, st);
      case 5: return launch_nt<T, 5>(g, t, st);
      default: return launch_plain<T, 1, 8, RegA<T, 1, 8, 4, 8>>(g, st);
    }
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t pack(const void* w, int64_t ldw, int64_t K, int64_t N, void* wt, int64_t kp,
                int64_t np, hipStream_t st) {
  const int64_t total = np * kp;
  const unsigned blocks = (unsigned)std::min<int64_t>((total + kThreads - 1) / kThreads, 2048);
  hipLaunchKernelGGL((k_pack_wt<T>), dim3(blocks), dim3(kThreads), 0, st, static_cast<const T*>(w),
                     ldw, K, N, static_cast<T*>(wt), kp, np);
  return hipGetLastError();
}

// grouped GEMM tiling: 128-row tiles (RegA, 2 x 16 rows per wave, 4 waves,
// 4 stages), up to 128 columns per tile
inline int grouped_nt(int64_t N) { return (int)std::min<int64_t>(8, (N + 15) / 16); }

template <typename T, int NT>
hipError_t launch_grouped_nt(const GemmArgs& g, hipStream_t st) {
  auto go = [&](auto r) {
    typedef decltype(r) R;
    dim3 grid((unsigned)(g.M / R::BM), (unsigned)((g.N + R::BN - 1) / R::BN));
    hipLaunchKernelGGL((k_gemm_grouped<T, 2, NT, R>), grid, dim3(R::THREADS), 0, st, g);
    return hipGetLastError();
  };
  // two stages for at most four k chunks, as for the plain narrow tiles
  if (chunks(g.dtype, g.K) <= 4) return go(RegA<T, 2, NT, 2>{});
  return go(RegA<T, 2, NT, 4>{});
}

template <typename T>
hipError_t dispatch_grouped(const GemmArgs& g, hipStream_t st) {
  switch (grouped_nt(g.N)) {
    case 1: return launch_grouped_nt<T, 1>(g, st);
    case 2: return launch_grouped_nt<T, 2>(g, st);
  }
  if constexpr (sizeof(T) == 2) {  // float32 past two column tiles: gemm_splits
    switch (grouped_nt(g.N)) {
      case 3: return launch_grouped_nt<T, 3>(g, st);
      case 4: return launch_grouped_nt<T, 4>(g, st);
      case 5: return launch_grouped_nt<T, 5>(g, st);
      case 6: return launch_grouped_nt<T, 6>(g, st);
      case 7: return launch_grouped_nt<T, 7>(g, st);
      default: return launch_grouped_nt<T, 8>(g, st);
    }
  }
  return hipErrorInvalidValue;
}

void grouped_packed(int dtype, int64_t N, int64_t K, int64_t* np, int64_t* kp) {
  const int64_t bn = 16 * grouped_nt(N), kc = kc_of(dtype);
  *np = (N + bn - 1) / bn * bn;
  *kp = (K + kc - 1) / kc * kc;
}

}  // namespace

// Whether the 128-column tiles (eight waves, four stages) beat streamed weights.
// With few k chunks their prefetch covers the whole product, and they waste little
// where N is close below one or two tiles (times as tiles / streamed):
//  - 113 to 128 columns, one operand, K < 192: with whole chunks from 24,000 rows
//    (60,000 x 128 x 128 13.1 / 14.7 us, 600,000 x 64 x 128 52 / 58; 20,000 rows
//    1.03 to 1.10), else where the streamed workgroups of 64 rows come to an
//    unlucky number of rounds (K = 20 to 176: 0.90 to 0.97 at 50,000 and 65,000
//    rows, 0.93 to 0.99 at 400,000, but 1.00 to 1.06 at 80,000 to 250,000 and 0.96
//    to 1.07 past 800,000); two operands of whole chunks, up to four in all, over
//    many rows (128 + 128: 0.95 at 400,000 rows, 1.02 at 300,000)
//  - two tiles over few rows, where the streamed column blocks are cut to seven
//    tiles (up to four chunks, 256 columns: 0.82 to 0.95 at 9,000 to 25,000 rows;
//    one operand, K <= 128, 208 columns: 0.90 to 0.98)
//  - 177 to 207 columns, one operand, whose single streamed block of 12 or 13
//    tiles leaves few waves in flight (200 columns, 50,000 / 130,000 rows: K = 64
//    0.83 / 0.94, K = 128 0.88 / 0.97, K = 192 0.91 / 1.02, K = 256 0.96 / 1.11);
//    209 to 256, two whole chunks (240 columns, 65,000 rows 0.94, 130,000 0.90 on
//    new inputs each call, 1.00 on the same)
bool tiles_win(int mode, int64_t M, int64_t N, int64_t K, int64_t K2) {
  const bool plain = mode == SAGA_GEMM_PLAIN, whole = K % 64 == 0 && K2 % 64 == 0;
  const int64_t ch = (K + 63) / 64 + (K2 + 63) / 64;
  if (N > 112 && N <= 128) {
    if (!plain) return whole && ch <= 4 && M >= 400000;
    return K < 192 && (whole ? M >= 24000 : (M >= 40000 && M < 75000) || (M >= 300000 && M < 700000));
  }
  if (M < 32768) return M >= 9000 && ((N > 240 && N <= 256 && ch <= 4) || (plain && N > 192 && N <= 208 && K <= 128));
  if (!plain || M < 40000 || M >= (K <= 128 ? 150000 : 75000)) return false;
  return (N > 176 && N < 208 && K <= 192) || (N > 208 && N <= 256 && K == 128);
}

// Whether a product streams its weights.  One k chunk an operand (K, K2 <= 64) and
// a concat or more than 208 columns: the tiles, whose single step prefetches
// nothing, stay (578959 x (31 + 31) x 250: 202 us, streamed 230; 575339 x (64 +
// 64) x 98: 91, 97; but 300000 x 20 x 160: 59, 37).  M < 0: for some M.
bool gemm_streams(int dtype, int mode, int64_t M, int64_t N, int64_t K, int64_t K2) {
  if (dtype != SAGA_BF16 || mode == SAGA_GEMM_GRU || N <= 80 || takes_bres(dtype, mode, M, N, K)) return false;
  if (tiles_win(mode, M, N, K, K2)) return false;
  return K > 64 || K2 > 64 || (mode == SAGA_GEMM_PLAIN && N <= 208);
}

size_t gemm_workspace_bytes(int dtype, int mode, int64_t N, int64_t K, int64_t K2) {
  if (mode != SAGA_GEMM_CONCAT && mode != SAGA_GEMM_GRU) K2 = 0;
  if (gemm_splits(dtype, mode, N, K + K2)) return split_workspace_bytes(mode, N, K, K2, 1);
  const size_t packed = packed_layout(dtype, mode, N, K, K2).bytes;
  return gemm_streams(dtype, mode, -1, N, K, K2) ? std::max(packed, stream_workspace_bytes(N, K, K2)) : packed;
}

hipError_t launch_gemm(const GemmArgs& g0, hipStream_t st) {
  if (g0.M == 0) return hipSuccess;
  if (gemm_streams(g0.dtype, g0.mode, g0.M, g0.N, g0.K, g0.mode == SAGA_GEMM_PLAIN ? 0 : g0.K2))
    return launch_gemm_stream(g0, st);
  if (g0.forms() || gemm_splits(g0.dtype, g0.mode, g0.N, g0.K + (g0.mode == SAGA_GEMM_CONCAT ? g0.K2 : 0)))
    return launch_gemm_split(g0, st);
  const Packed pk = packed_layout(g0.dtype, g0.mode, g0.N, g0.K, g0.K2);
  if (!g0.ws || g0.ws_bytes < pk.bytes) return hipErrorInvalidValue;
  GemmArgs g = g0;
  char* ws = static_cast<char*>(g.ws);
  g.wt = ws;
  g.kp = pk.kp;
  g.wt2 = pk.kp2 ? ws + pk.off2 : nullptr;
  g.kp2 = pk.kp2;
  const bool bf = g.dtype == SAGA_BF16;
  hipError_t e = bf ? pack<uint16_t>(g.w, g.ldw, g.K, g.N, ws, pk.kp, pk.np, st)
                    : pack<float>(g.w, g.ldw, g.K, g.N, ws, pk.kp, pk.np, st);
  if (e == hipSuccess && pk.kp2)
    e = bf ? pack<uint16_t>(g.w2, g.ldw2, g.K2, g.N, ws + pk.off2, pk.kp2, pk.np, st)
           : pack<float>(g.w2, g.ldw2, g.K2, g.N, ws + pk.off2, pk.kp2, pk.np, st);
  if (e != hipSuccess) return e;
  return bf ? dispatch<uint16_t>(g, st) : dispatch<float>(g, st);
}

size_t gemm_grouped_workspace_bytes(int dtype, int groups, int64_t N, int64_t K) {
  if (gemm_splits(dtype, SAGA_GEMM_PLAIN, N, K)) return split_workspace_bytes(SAGA_GEMM_PLAIN, N, K, 0, groups);
  int64_t np, kp;
  grouped_packed(dtype, N, K, &np, &kp);
  const size_t es = dtype == SAGA_BF16 ? 2 : 4;
  return ((size_t)groups * np * kp * es + 255) / 256 * 256;
}

hipError_t launch_gemm_grouped(const GemmArgs& g0, hipStream_t st) {
  if (g0.M == 0) return hipSuccess;
  if (g0.M % kRelTile != 0 || g0.groups < 1 || !g0.arow || !g0.grp_ptr) return hipErrorInvalidValue;
  if (!g0.ws || g0.ws_bytes < gemm_grouped_workspace_bytes(g0.dtype, g0.groups, g0.N, g0.K))
    return hipErrorInvalidValue;
  GemmArgs g = g0;
  if (gemm_splits(g.dtype, SAGA_GEMM_PLAIN, g.N, g.K)) return launch_gemm_split(g, st);
  int64_t np, kp;
  grouped_packed(g.dtype, g.N, g.K, &np, &kp);
  g.wt = g.ws;
  g.kp = kp;
  g.wt_group_stride = np * kp;
  const bool bf = g.dtype == SAGA_BF16;
  const int64_t total = np * kp * g.groups;
  const unsigned blocks = (unsigned)std::min<int64_t>((total + kThreads - 1) / kThreads, 4096);
  if (bf)
    hipLaunchKernelGGL((k_pack_wt_grouped<uint16_t>), dim3(blocks), dim3(kThreads), 0, st,
                       static_cast<const uint16_t*>(g.w), g.ldw, g.K, g.N, g.groups,
                       static_cast<uint16_t*>(g.ws), kp, np);
  else
    hipLaunchKernelGGL((k_pack_wt_grouped<float>), dim3(blocks), dim3(kThreads), 0, st,
                       static_cast<const float*>(g.w), g.ldw, g.K, g.N, g.groups,
                       static_cast<float*>(g.ws), kp, np);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return bf ? dispatch_grouped<uint16_t>(g, st) : dispatch_grouped<float>(g, st);
}

}  // namespace saga
