// ApplyVertex in float32: PLAIN, CONCAT, GRU and grouped products on the bfloat16
// matrix cores, every float32 operand as an exact sum of three bfloat16 values.
#include <type_traits>

#include "gemm_device.h"

namespace saga {
namespace {

// ---------------------------------------------------------------------------
// float32 products on the bfloat16 matrix cores.  Scaled by 2^16, every float32
// value below 2^110, subnormals included, is the exact sum of three bfloat16
// values, x = x1 + x2 + x3 (round to nearest, then the remainders: 8 + 8 + 8
// bits of significand; the scale keeps the last bit at 2^-133 or above, and the
// instruction takes subnormal bfloat16 values as they are).  Then
//   a w = a1 w1 + (a1 w2 + a2 w1) + (a1 w3 + a2 w2 + a3 w1) + rest
// with |rest| <= 2^-24.2 |a w|, 2^-27.5 |a w| in the root mean square, and the
// six products are accumulated in float32 by v_mfma_f32_16x16x32_bf16.  One such
// instruction takes 32 k at 16 times the rate of v_mfma_f32_16x16x4f32, so six of
// them take 3/8 of its time.  Up to four k the rest is not small beside the sum's own
// rounding; such a product, which memory bounds, takes all nine terms.
//
// What bounds it: the matrix cores.  2^21 x 602 x 128 takes 1.81 ms (float32
// instruction 2.89), 1,085 TFLOP/s of bfloat16 products where an 8192^3 product
// reaches 1,202; with one accumulator the products alone took 1.15 ms at the 1.87
// GHz the power limit leaves under this load, the A loads added 0.35, the weights
// 0.27, the stores 0.14.
//
// Accumulation.  The instruction adds its 32 products to the accumulator eight
// at a time and rounds after each eight, v_mfma_f32_16x16x4f32 after each
// product.  a1 w1 has accumulators of its own, the five small terms (2^-8 of it)
// others, added at the end: the large accumulator is then rounded at most once
// per eight k, and not at all where a and w are zero, so that no input has more
// roundings of its full magnitude than with the float32 instruction.  (All six in
// one accumulator are six roundings a chunk: nearer to float64 than the float32
// instruction on dense rows, but up to 2.1 times further off on rows with one to
// three nonzeros per 32 k.)  Relative error against float64, float32 instruction /
// one accumulator / two, 8192 rows x 128: K = 602 normal 4.4e-7 / 3.7e-7 / 1.3e-7,
// after ReLU 3.1e-7 / 3.5e-7 / 1.0e-7, 2 % of values nonzero 6.7e-8 / 1.3e-7 /
// 3.0e-8; K = 1 2.5e-8 / 3.3e-8 / 2.5e-8.
//
// Range.  The scaled sums must stay finite: with m the largest magnitude of a
// wave's rows and w of its columns, m < 2^110, w < 2^110 and m w K < 2^94.  The
// kernel tracks the rows' as it loads them, k_pack_split notes the columns'; a
// wave that meets more (infinities included), or NaN weights, recomputes its
// tile with the float32 instruction (native_phase; 262144 x 256 x 128, us: 114,
// every 1000th row infinite 198, every row 443).  NaN in A gives NaN either way.
// ---------------------------------------------------------------------------
constexpr int kAllTerms = 4;
constexpr float kSplitScale = 65536.0f;
constexpr float kSplitUnscale = 1.0f / (kSplitScale * kSplitScale);
constexpr float kSplitMax = 1298074214633706907132624082305024.0f;  // 2^110
constexpr float kSplitSum = 19807040628566084398385987584.0f;       // 2^94
__device__ __forceinline__ bool split_special(float m, float w, float k) {
  return !(m < kSplitMax && w < kSplitMax && m * w * k < kSplitSum);
}

typedef __attribute__((address_space(3))) uint4 lds_uint4;

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// kSplitScale x = p[0] + p[1] + p[2], two values at a time
__device__ __forceinline__ void split3(f32x2 x, uint32_t (&p)[3]) {
  x *= kSplitScale;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const bf16x2 h = __builtin_convertvector(x, bf16x2);
    __builtin_memcpy(&p[q], &h, 4);
    x -= f32x2{__uint_as_float(p[q] << 16), __uint_as_float(p[q] & 0xffff0000u)};
  }
}

// One operand's weights, K x N, as the caller holds them (GemmArgs)
struct WSrc {
  const float* w;
  int64_t ldw, K, N;
  int64_t cb, cbs;  // cb > 0: column n is column n % cb of the block at w + n / cb * cbs
  // fold > 0: columns from `fold` on are the attention vectors folded into the
  // first `fold`: column fold + h is sum_d w[:, h D + d] al[h D + d], then ar
  int fold, heads;
  const float *al, *ar;
  __device__ float at(int64_t k, int64_t n) const {
    if (k >= K || n >= N) return 0.0f;
    if (fold > 0 && n >= fold) {
      const int D = fold / heads, h = (int)(n - fold) % heads;
      const float* att = (n - fold < heads ? al : ar) + h * D;
      const float* row = w + k * ldw + h * D;
      float v = 0.0f;
      for (int d = 0; d < D; ++d) v += row[d] * att[d];
      return v;
    }
    return cb > 0 ? w[n / cb * cbs + k * ldw + n % cb] : w[k * ldw + n];
  }
};
__host__ __device__ inline WSrc wsrc1(const GemmArgs& g) {
  return WSrc{static_cast<const float*>(g.w), g.ldw, g.K, g.N, g.wcb, g.wcbs, g.fold, g.fold_heads,
              g.fold_al, g.fold_ar};
}
__host__ __device__ inline WSrc wsrc2(const GemmArgs& g) {
  return WSrc{static_cast<const float*>(g.w2), g.ldw2, g.K2, g.N, 0, 0, 0, 0, nullptr, nullptr};
}

// A straight from global memory into registers and split there; the packed
// weights, split by k_pack_split, through two LDS stages.  A chunk is 32 k:
// 128 bytes of an A row, and for every 16-column tile three 1 KB planes of Wt
// whose 16-byte pieces (8 k of one column: 4 p .. 4 p + 3 and 16 further on)
// lie in the order the lanes read them, piece p of column r at slot 16 p + r, so the stage is one contiguous
// copy and every fragment read covers 1 KB free of bank conflicts.
//
// Step i multiplies chunk i.  At its top the weights of chunk i + 1 start on
// their way into the other stage and the A rows of chunk i + 2 into registers;
// in its second half the A rows of chunk i + 1, which have had a whole step to
// land, are split, so that the vector instructions of the split issue between
// the matrix instructions.  The direct-to-LDS loads are written in assembly:
// the compiler would otherwise wait for every one in flight before any LDS
// read.  Loads return in order, so the explicit wait at the top of a step, at
// most the newest A loads pending, covers the older weight loads.
//
// CONCAT: the chunks of both operands make one stream, the second operand's from
// chunk n1 on, and their images lie one after another.
template <int MT, int NT, int NW, bool CONCAT = false>
struct Split3 {
  typedef float T;
  static constexpr int THREADS = 64 * NW;
  static constexpr int BM = 16 * MT * NW, BN = 16 * NT;
  static constexpr int STAGE = 3 * NT * 64;  // 16-byte slots per stage
  static constexpr int RING_SLOTS = 2 * STAGE;
  static constexpr size_t LDS_BYTES = (size_t)RING_SLOTS * 16;
  static constexpr int LB = (STAGE + THREADS - 1) / THREADS;
  static constexpr int KC = 32;

  // rows of one operand
  struct Rows {
    const float* a;
    int64_t lda, K;
    const int32_t* arow;
    __device__ int chunks() const { return (int)((K + KC - 1) / KC); }
  };
  struct Ctx {
    const float* row[MT];  // this lane's A rows
    int k0, kmax;          // their operand's first chunk; first column of a row's last 16-byte piece
    const uint4* Wi;       // this column block's image: chunk c at c * STAGE
    lds_uint4* ring;
    int last, n1;          // last chunk; the second operand's first
    Rows op2;              // CONCAT
    int64_t M, row0;
  };
  __device__ __forceinline__ static void set_rows(Ctx& c, const Rows& o, int first) {
    int64_t off[MT];
    row_offsets(o.arow, o.lda, c.M, c.row0, off);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) c.row[mt] = o.a + off[mt];
    c.k0 = first;
    c.kmax = (int)((o.K - 1) / 4 * 4);
  }

  // A values of chunk c: columns 32 c + 4 (lane / 16) .. + 3 and the same 16
  // further on (a load instruction then covers 64 contiguous bytes of every
  // row; k_pack_split orders its k alike).  A piece that starts at or past K
  // reads the row's last piece instead (masked when split).
  __device__ __forceinline__ static void load_a(Ctx& c, int chunk, uint4 (&a)[MT][2]) {
    if (CONCAT && chunk == c.n1) set_rows(c, c.op2, c.n1);
    const int lg = (threadIdx.x & 63) >> 4;
    const int k = (chunk - c.k0) * KC + lg * 4;
    const int k0 = min(k, c.kmax), k1 = min(k + 16, c.kmax);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      a[mt][0] = *reinterpret_cast<const uint4*>(c.row[mt] + k0);
      a[mt][1] = *reinterpret_cast<const uint4*>(c.row[mt] + k1);
    }
  }
  // zeros past column K, for the chunk-th chunk of an operand
  __device__ __forceinline__ static void mask(int64_t K, int chunk, uint4 (&a)[MT][2]) {
    const int lg = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t left = K - (chunk * KC + lg * 4 + h * 16);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        if (left < 4) a[mt][h].w = 0;
        if (left < 3) a[mt][h].z = 0;
        if (left < 2) a[mt][h].y = 0;
        if (left < 1) a[mt][h].x = 0;
      }
    }
  }
  __device__ __forceinline__ static void issue_b(const Ctx& c, int chunk, int stage) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint4* src = c.Wi + (int64_t)chunk * STAGE;
    const uint32_t dst = (uint32_t)(uintptr_t)(c.ring + stage * STAGE);
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

  struct Parts { uint32_t p[MT][3][4]; };
  // values 2 d and 2 d + 1 of row mt
  __device__ __forceinline__ static void split_pair(const uint4 (&a)[MT][2], int mt, int d,
                                                    float (&amax)[MT], Parts& o) {
    const uint4& v = a[mt][d / 2];
    const f32x2 x = d % 2 == 0 ? f32x2{__uint_as_float(v.x), __uint_as_float(v.y)}
                               : f32x2{__uint_as_float(v.z), __uint_as_float(v.w)};
    amax[mt] = fmaxf(fmaxf(fabsf(x.x), fabsf(x.y)), amax[mt]);
    uint32_t p[3];
    split3(x, p);
#pragma unroll
    for (int q = 0; q < 3; ++q) o.p[mt][q][d] = p[q];
  }
  __device__ __forceinline__ static bf16x8 part(const Parts& ap, int mt, int q) {
    bf16x8 r;
    __builtin_memcpy(&r, ap.p[mt][q], 16);
    return r;
  }

  // One step.  A column tile's weight fragments are read while the tile before
  // it is multiplied; in the second half (LAST: no next chunk) the pairs of
  // chunk i + 1's A values are split a few at a time between the matrix
  // instructions.  The scheduling barriers keep that order.
  static constexpr int G0 = NT / 2;             // first column tile of the second half
  static constexpr int SLOTS = (NT - G0) * 6;   // places to split at
  typedef bf16x8 BFrag[3];
  __device__ __forceinline__ static void read_b(const lds_uint4* Bs, int g, BFrag& b) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < 3; ++q)
      b[q] = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(
          Bs + (q * NT + g) * 64 + lane);
  }
  // Column tile g goes to accumulator g, or g + SHIFT from tile FROM on.  NQ: of
  // the nine products, smallest first, the last NQ; all but the last into `lo`.
  template <int U, bool LOAD, bool MASK, bool LAST, int FROM, int SHIFT, int NA, int NQ = 6>
  __device__ __forceinline__ static void step(Ctx& c, int i, const Rows& op1, uint4 (&a)[2][MT][2], Parts (&ap)[2],
                                              float (&amax)[MT], f32x4 (&acc)[MT][NA], f32x4 (&lo)[MT][NA]) {
    // chunk i's weights landed (only chunk i + 1's A loads are newer), for
    // every wave; the other stage is free again
    wait_vm<LAST ? 0 : 2 * MT>();
    ring_barrier();
    const lds_uint4* Bs = c.ring + U * STAGE;
    BFrag b[2];
    read_b(Bs, 0, b[0]);
    if constexpr (!LAST) issue_b(c, i + 1, U ^ 1);
    if constexpr (LOAD) load_a(c, i + 2, a[U]);
    __builtin_amdgcn_sched_barrier(0);
    constexpr int QA[9] = {2, 2, 1, 2, 1, 0, 1, 0, 0}, QB[9] = {2, 1, 2, 0, 1, 2, 0, 1, 0};
#pragma unroll
    for (int g = 0; g < NT; ++g) {
      if (g + 1 < NT) read_b(Bs, g + 1, b[(g + 1) & 1]);
      if constexpr (MASK) {
        if (g == G0) mask(CONCAT ? c.op2.K : op1.K, i + 1 - (CONCAT ? c.n1 : 0), a[U ^ 1]);
      }
      if constexpr (CONCAT && !LAST) {
        if (g == G0 && i + 2 == c.n1) mask(op1.K, i + 1, a[U ^ 1]);
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          f32x4& d = (q == NQ - 1 ? acc : lo)[mt][g + (g >= FROM ? SHIFT : 0)];
          d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(part(ap[U], mt, QA[9 - NQ + q]), b[g & 1][QB[9 - NQ + q]], d,
                                                      0, 0, 0);
        }
        if (!LAST && g >= G0) {
          const int slot = (g - G0) * 6 + q;
#pragma unroll
          for (int d = slot * MT * 4 / SLOTS; d < (slot + 1) * MT * 4 / SLOTS; ++d)
            split_pair(a[U ^ 1], d / 4, d % 4, amax, ap[U ^ 1]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  // acc, lo += A[tile0 .. tile0 + BM) x the column block's image; amax: this
  // lane's part of its rows' largest magnitudes.  CH > 0: the number of chunks.
  template <int FROM = NT, int SHIFT = 0, int CH = 0, int NA = NT>
  __device__ __forceinline__ static void phase(const Rows& op1, const Rows& op2, int64_t M,
                                               const uint4* __restrict__ Wi, int64_t tile0, uint4* ring,
                                               float (&amax)[MT], f32x4 (&acc)[MT][NA], f32x4 (&lo)[MT][NA]) {
    Ctx c;
    c.M = M;
    c.row0 = tile0 + (threadIdx.x >> 6) * MT * 16;
    set_rows(c, op1, 0);
    c.n1 = op1.chunks();
    c.op2 = op2;
    c.Wi = Wi;
    c.ring = (lds_uint4*)ring;
    c.last = (CH > 0 ? CH : CONCAT ? c.n1 + op2.chunks() : c.n1) - 1;
    uint4 a[2][MT][2];
    Parts ap[2];
    // chunk 0 into slot U
    auto first = [&](auto u) {
      constexpr int U = decltype(u)::value;
      issue_b(c, 0, U);
      load_a(c, 0, a[U]);
      if (c.last > 0) load_a(c, 1, a[U ^ 1]);
      if (c.n1 == 1) mask(op1.K, 0, a[U]);
#pragma unroll
      for (int d = 0; d < MT * 4; ++d) split_pair(a[U], d / 4, d % 4, amax, ap[U]);
    };
    // The last chunk is always in slot 1, so that there is one tail: with three,
    // one per remainder, the accumulators of a tail took registers beside the
    // loop's (213 instead of 145 for 1 x 8 tiles).
    typedef std::integral_constant<int, 0> Slot0;
    typedef std::integral_constant<int, 1> Slot1;
    int i = 0;
    if (!CONCAT && c.last == 0) {
      first(Slot0{});
      if (op1.K <= kAllTerms) step<0, false, false, true, FROM, SHIFT, NA, 9>(c, i, op1, a, ap, amax, acc, lo);
      else step<0, false, false, true, FROM, SHIFT, NA>(c, i, op1, a, ap, amax, acc, lo);
    } else {
      if (c.last % 2 == 0) {
        first(Slot1{});
        step<1, true, false, false, FROM, SHIFT, NA>(c, i++, op1, a, ap, amax, acc, lo);
      } else {
        first(Slot0{});
      }
      for (; i + 1 < c.last; i += 2) {
        step<0, true, false, false, FROM, SHIFT, NA>(c, i, op1, a, ap, amax, acc, lo);
        step<1, true, false, false, FROM, SHIFT, NA>(c, i + 1, op1, a, ap, amax, acc, lo);
      }
      step<0, false, true, false, FROM, SHIFT, NA>(c, i, op1, a, ap, amax, acc, lo);
      step<1, false, false, true, FROM, SHIFT, NA>(c, i + 1, op1, a, ap, amax, acc, lo);
    }
    ring_barrier();  // the stages may be refilled by a following phase
  }

  // acc += lo, without the scale
  template <int NA>
  __device__ __forceinline__ static void finish(f32x4 (&acc)[MT][NA], const f32x4 (&lo)[MT][NA]) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int t = 0; t < NA; ++t) acc[mt][t] = (acc[mt][t] + lo[mt][t]) * kSplitUnscale;
  }
  // does this wave meet values outside the split's range (uniform); wbits: this
  // lane's part of the columns' largest magnitude.  Ordinary ones take two
  // comparisons, without the columns' reduction over the lanes.
  __device__ __forceinline__ static bool special(const float (&amax)[MT], uint32_t wbits, int64_t k) {
    constexpr float kOrdinary = 140737488355328.0f;  // 2^47
    bool sp = !(__uint_as_float(wbits) * (float)k < kOrdinary);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) sp |= !(amax[mt] < kOrdinary);
    if (!__any(sp)) return false;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) wbits = max(wbits, (uint32_t)__shfl_xor((int)wbits, off, 64));
    sp = false;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) sp |= split_special(amax[mt], __uint_as_float(wbits), (float)k);
    return __any(sp);
  }

  // acc += A rows x W with the float32 instruction, operands straight from
  // memory: the waves whose values the split does not take (rare, not tuned)
  template <int FROM = NT, int SHIFT = 0, int NA = NT>
  __device__ __forceinline__ static void native_phase(const Rows& o, int64_t M, const WSrc& w, int64_t n0,
                                                      int64_t tile0, f32x4 (&acc)[MT][NA]) {
    const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
    int64_t off[MT];
    row_offsets(o.arow, o.lda, M, tile0 + (threadIdx.x >> 6) * MT * 16, off);
    for (int64_t k0 = 0; k0 < w.K; k0 += 4) {
      const int64_t k = k0 + lg;
      float a[MT], b[NT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) a[mt] = k < w.K ? o.a[off[mt] + k] : 0.0f;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) b[nt] = w.at(k, n0 + nt * 16 + lr);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          f32x4& c = acc[mt][nt + (nt >= FROM ? SHIFT : 0)];
          c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[mt], b[nt], c, 0, 0, 0);
        }
    }
  }
};

// The image Split3 streams, for one group of weights (blockIdx.y < groups) or
// the second operand (the next one): for column block b, chunk c, plane q, tile
// t of the block: 64 pieces of 8 k.  A workgroup takes kPackChunks chunks of a
// 16-column tile and notes their largest magnitude (one workgroup per tile ran 5
// to 6 us; a folded tile of 512 x 16, eight terms each, 20).  A tile of few folded
// columns divides every sum among its lanes (one head of 64 columns on two lanes
// alone: a pair of GAT layers at 1,785 vertices, 40 features 68.3 us, now 50.0).
constexpr int kPackThreads = 256, kPackChunks = kPackThreads / 64;
__host__ __device__ inline int64_t pack_parts(int64_t nch) { return (nch + kPackChunks - 1) / kPackChunks; }
struct PackOut {
  uint4* img;  // column block b's image begins b * stride chunks further on
  int stride;
  uint32_t* wmax;
};
__global__ __launch_bounds__(kPackThreads) void k_pack_split(WSrc w1, PackOut o1, WSrc w2, PackOut o2,
                                                             int groups, int nt) {
  __shared__ uint32_t tmax;
  const bool second = (int)blockIdx.y >= groups;
  const int grp = second ? 0 : blockIdx.y;
  WSrc w = second ? w2 : w1;
  const PackOut o = second ? o2 : o1;
  w.w += (int64_t)grp * w.K * w.ldw;
  const int nch = (int)((w.K + 31) / 32), tile = blockIdx.x, tiles = gridDim.x;
  const int b = tile / nt, t = tile % nt;
  uint4* im = o.img + ((int64_t)grp * (tiles / nt) + b) * o.stride * nt * 192;
  const int part = blockIdx.z;
  if (part >= pack_parts(nch)) return;
  if (threadIdx.x == 0) tmax = 0;
  __syncthreads();
  const int r = threadIdx.x & 15;
  const int64_t n = (int64_t)tile * 16 + r;
  // folded columns [f0, f0 + fc) of this tile, fs of its 16 lanes to a sum
  const int f0 = max(w.fold - tile * 16, 0), fc = w.fold > 0 ? (int)min(w.N - (int64_t)tile * 16, (int64_t)16) - f0 : 0;
  const bool folded = fc > 0 && r >= f0 && n < w.N;
  const float* col = w.w + (w.cb > 0 ? (int)n / (int)w.cb * w.cbs + (int)n % (int)w.cb : n);
  const int64_t kn = n < w.N ? w.K : 0;
  uint32_t m = 0;
  const int c = part * kPackChunks + threadIdx.x / 64, p = (threadIdx.x / 16) % 4;
  if (c < nch) {
    const int64_t k0 = (int64_t)c * 32 + p * 4;  // and k0 + 16
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = 0.0f;
    if (fc > 0) {  // (uniform in the workgroup)
      const int fs = fc > 8 ? 1 : fc > 4 ? 2 : fc > 2 ? 4 : 8, D = w.fold / w.heads;
      const int f = tile * 16 + f0 - w.fold + min(r / fs, fc - 1), h = f % w.heads;
      const float* wf = w.w + h * D;
      const float* att = (f < w.heads ? w.al : w.ar) + h * D;
      // eight k at a time, so that their loads overlap
#pragma unroll 4
      for (int d = r % fs; d < D; d += fs)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int64_t k = k0 + e % 4 + 16 * (e / 4);
          x[e] += (k < w.K ? wf[k * w.ldw + d] : 0.0f) * att[d];
        }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        for (int off = fs / 2; off > 0; off >>= 1) x[e] += __shfl_xor(x[e], off, 16);
        x[e] = __shfl(x[e], max(r - f0, 0) * fs, 16);
      }
    }
    if (!folded) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int64_t k = k0 + e % 4 + 16 * (e / 4);
        x[e] = k < kn ? col[k * w.ldw] : 0.0f;
      }
    }
    uint32_t q[3][4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      m = max(m, max(__float_as_uint(fabsf(x[2 * d])), __float_as_uint(fabsf(x[2 * d + 1]))));
      uint32_t o3[3];
      split3(f32x2{x[2 * d], x[2 * d + 1]}, o3);
#pragma unroll
      for (int k = 0; k < 3; ++k) q[k][d] = o3[k];
    }
#pragma unroll
    for (int k = 0; k < 3; ++k)
      im[((int64_t)c * 3 + k) * nt * 64 + t * 64 + p * 16 + r] = make_uint4(q[k][0], q[k][1], q[k][2], q[k][3]);
  }
  // (as bits: NaN is larger than any value)
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
  if ((threadIdx.x & 63) == 0) atomicMax(&tmax, m);
  __syncthreads();
  if (threadIdx.x == 0) o.wmax[((int64_t)grp * tiles + tile) * pack_parts(nch) + part] = tmax;
}

// this lane's part of the largest magnitude k_pack_split noted for column block b
template <int NT>
__device__ __forceinline__ uint32_t block_max(const uint32_t* __restrict__ wmax, int64_t b, int64_t nch) {
  const int n = NT * (int)pack_parts(nch);
  uint32_t m = 0;
  for (int i = threadIdx.x & 63; i < n; i += 64) m = max(m, wmax[b * n + i]);
  return m;
}

// float32 PLAIN / CONCAT / grouped through Split3.  The column blocks of one
// row block run on one XCD one after another (workgroup w goes to XCD w % 8),
// so that its rows of A come from HBM once.  GROUPED as k_gemm_grouped below.
template <int MT, int NT, int NW, bool GROUPED, bool CONCAT>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2))) void k_gemm_split(GemmArgs g, int ny) {
  typedef Split3<MT, NT, NW, CONCAT> R;
  __shared__ uint4 ring[R::RING_SLOTS];
  if constexpr (GROUPED)
    if ((g.err1 && *g.err1) || (g.err2 && *g.err2)) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const unsigned w = blockIdx.x / kXcds;
  const int y = (int)(w % (unsigned)ny);
  const int64_t tile0 = ((int64_t)(w / (unsigned)ny) * kXcds + blockIdx.x % kXcds) * R::BM;
  const int64_t n0 = (int64_t)y * R::BN;
  int grp = 0;
  if constexpr (GROUPED) {
    static_assert(R::BM == kRelTile, "grouped tiles must match the row-range padding");
    if (tile0 >= g.grp_ptr[g.groups]) return;
    int hi = g.groups;  // grp_ptr[grp] <= tile0 < grp_ptr[hi]
    while (hi - grp > 1) {
      const int mid = (grp + hi) >> 1;
      if (g.grp_ptr[mid] <= tile0) grp = mid;
      else hi = mid;
    }
  } else if (tile0 >= g.M) {
    return;
  }
  f32x4 acc[MT][NT], lo[MT][NT];
  float amax[MT];
  auto clear = [](f32x4 (&x)[MT][NT]) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) x[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  clear(acc);
  clear(lo);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) amax[mt] = 0.0f;
  const typename R::Rows op1{static_cast<const float*>(g.a), g.lda, g.K, GROUPED ? g.arow : nullptr};
  const typename R::Rows op2{static_cast<const float*>(g.a2), g.lda2, CONCAT ? g.K2 : 0, nullptr};
  const int64_t nch = (g.K + 31) / 32, nch2 = CONCAT ? (g.K2 + 31) / 32 : 0;
  const int64_t blk = (int64_t)grp * ny + y;
  R::phase(op1, op2, g.M, static_cast<const uint4*>(g.wt) + blk * (nch + nch2) * R::STAGE, tile0, ring, amax, acc, lo);
  R::finish(acc, lo);
  uint32_t wm = block_max<NT>(g.wmax, blk, nch);
  if (CONCAT) wm = max(wm, block_max<NT>(g.wmax2, y, nch2));
  if (R::special(amax, wm, g.K + op2.K)) {
    clear(acc);
    WSrc w = wsrc1(g);
    w.w += (int64_t)grp * g.K * g.ldw;
    R::native_phase(op1, g.M, w, n0, tile0, acc);
    if (CONCAT) R::native_phase(op2, g.M, wsrc2(g), n0, tile0, acc);
  }
  const int64_t row0 = tile0 + wave * MT * 16;
  if constexpr (GROUPED) {
    // rows of range padding (map entry < 0) are written as zeros
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (g.arow[row0 + mt * 16 + 4 * (lane >> 4) + r] < 0) {
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) acc[mt][nt][r] = 0.0f;
        }
  } else {
    finish_tile(g, row0, n0, acc);
  }
  store_tile<float, MT, NT, R>(g, row0, n0, acc, ring);
}

// GRU through Split3 (GGNN's ApplyVertex, Fig. 2): a wave's 16 rows of a w and
// a2 w2, column blocks (r, z, n) of F = 16 NT3.  Both products' r and z columns
// add up in the same accumulators; only the n blocks are kept apart.
template <int NT3>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_gru_split(GemmArgs g) {
  constexpr int NT = 3 * NT3, NA = 4 * NT3, F = 16 * NT3;
  typedef Split3<1, NT, 4> R;
  __shared__ uint4 ring[R::RING_SLOTS];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t tile0 = (int64_t)blockIdx.x * R::BM;
  const float* h = static_cast<const float*>(g.a2);
  f32x4 acc[1][NA], lo[1][NA];
  auto clear = [](f32x4 (&x)[1][NA]) {
#pragma unroll
    for (int t = 0; t < NA; ++t) x[0][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  clear(acc);
  clear(lo);
  float amax[1] = {0.0f};
  const typename R::Rows op1{static_cast<const float*>(g.a), g.lda, g.K, nullptr}, op2{h, g.lda2, F, nullptr};
  // (K2 = F, so the second product's chunks are known here)
  R::template phase<NT, 0, 0, NA>(op1, op2, g.M, static_cast<const uint4*>(g.wt), tile0, ring, amax, acc, lo);
  R::template phase<2 * NT3, NT3, (F + 31) / 32, NA>(op2, op2, g.M, static_cast<const uint4*>(g.wt2), tile0, ring, amax,
                                                     acc, lo);
  R::finish(acc, lo);
  const uint32_t wm = max(block_max<NT>(g.wmax, 0, (g.K + 31) / 32), block_max<NT>(g.wmax2, 0, (F + 31) / 32));
  if (R::special(amax, wm, g.K + F)) {
    clear(acc);
    R::template native_phase<NT, 0, NA>(op1, g.M, wsrc1(g), 0, tile0, acc);
    R::template native_phase<2 * NT3, NT3, NA>(op2, g.M, wsrc2(g), 0, tile0, acc);
  }
  const int64_t row0 = tile0 + wave * 16;
  float* out = static_cast<float*>(g.out);
  // biases and previous states are all loaded before the first store (a
  // load after a store the compiler cannot tell apart from it would wait)
  float br[NT3], bz[NT3], bi[NT3], bh[NT3], hp[4][NT3];
#pragma unroll
  for (int t = 0; t < NT3; ++t) {
    const int c = t * 16 + (lane & 15);
    const float* b1 = g.bias;
    const float* b2 = g.bias2;
    br[t] = (b1 ? b1[c] : 0.f) + (b2 ? b2[c] : 0.f);
    bz[t] = (b1 ? b1[F + c] : 0.f) + (b2 ? b2[F + c] : 0.f);
    bi[t] = b1 ? b1[2 * F + c] : 0.f;
    bh[t] = b2 ? b2[2 * F + c] : 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = row0 + 4 * (lane >> 4) + r;
      hp[r][t] = row < g.M ? h[row * g.lda2 + c] : 0.f;
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t row = row0 + 4 * (lane >> 4) + r;
    if (row >= g.M) continue;
#pragma unroll
    for (int t = 0; t < NT3; ++t) {
      const float rr = sigmoidf_(acc[0][t][r] + br[t]);
      const float zz = sigmoidf_(acc[0][NT3 + t][r] + bz[t]);
      const float nn = tanhf(acc[0][2 * NT3 + t][r] + bi[t] + rr * (acc[0][3 * NT3 + t][r] + bh[t]));
      out[row * g.ldo + t * 16 + (lane & 15)] = (1.0f - zz) * nn + zz * hp[r][t];
    }
  }
}

// ---- float32 through Split3 ----
// column blocks of NT 16-column tiles: as few blocks of at most eight as
// cover N, of equal width
struct SplitShape {
  int nt, ny;
  int64_t nch, img_bytes, max_bytes;  // per K operand (and group, for the image)
};
SplitShape split_shape(int64_t N, int64_t K, int groups, int mode) {
  SplitShape s;
  const int tiles = (int)((N + 15) / 16);
  s.ny = mode == SAGA_GEMM_GRU ? 1 : (tiles + 7) / 8;  // a GRU row needs all its columns
  s.nt = (tiles + s.ny - 1) / s.ny;
  s.nch = (K + 31) / 32;
  s.img_bytes = (int64_t)groups * s.ny * s.nt * s.nch * 3072;
  s.max_bytes = ((int64_t)groups * s.ny * s.nt * pack_parts(s.nch) * 4 + 255) / 256 * 256;
  return s;
}

template <int MT, int NT, int NW, bool GROUPED, bool CONCAT = false>
hipError_t launch_split(const GemmArgs& g, int ny, hipStream_t st) {
  typedef Split3<MT, NT, NW, CONCAT> R;
  static_assert(R::LDS_BYTES <= 160 * 1024, "LDS ring too large");
  const int64_t mt = (g.M + R::BM - 1) / R::BM;
  const unsigned grid = (unsigned)((mt + kXcds - 1) / kXcds * kXcds * ny);
  hipLaunchKernelGGL((k_gemm_split<MT, NT, NW, GROUPED, CONCAT>), dim3(grid), dim3(R::THREADS), 0, st, g,
                     ny);
  return hipGetLastError();
}

// Tile shape, measured (us, float32 matrix instructions / 32 rows per wave /
// 16 rows per wave; four waves): long K over many rows takes 32 rows a wave,
// which halves the LDS reads per product (2^21 x 602 x 128: 2888 / 1806 / 1949;
// 131072 x 512 x 256 in two operands: 312 / 185 / 196; 600000 x 300 x 300: 1411 /
// 722 / 734).  Up to seven k chunks, or too few tiles to fill the chip twice over,
// 16 rows: more waves in flight (100000 x 64 x 64: 20.2 / 20.9 / 18.2; 500000 x
// 100 x 48: 90.9 / 75.9 / 76.9; 5000 x 602 x 256: 51.9 / 32.2 / 23.8; 20000 x 512 x
// 80: 33.7 / 24.8 / 22.5).
template <int NT, bool GROUPED>
hipError_t dispatch_split_nt(const GemmArgs& g, const SplitShape& s, int64_t chunks, hipStream_t st) {
  const bool tall = chunks >= 8 && (GROUPED || (g.M + 127) / 128 * s.ny >= 1024);
  if constexpr (GROUPED)  // tiles of exactly kRelTile rows
    return tall ? launch_split<2, NT, 4, true>(g, s.ny, st) : launch_split<1, NT, 8, true>(g, s.ny, st);
  else
    if (g.mode == SAGA_GEMM_CONCAT)
      return tall ? launch_split<2, NT, 4, false, true>(g, s.ny, st) : launch_split<1, NT, 4, false, true>(g, s.ny, st);
    else
      return tall ? launch_split<2, NT, 4, false>(g, s.ny, st) : launch_split<1, NT, 4, false>(g, s.ny, st);
}

template <bool GROUPED>
hipError_t dispatch_split(const GemmArgs& g, const SplitShape& s, int64_t chunks, hipStream_t st) {
  switch (s.nt) {
    case 1: return dispatch_split_nt<1, GROUPED>(g, s, chunks, st);
    case 2: return dispatch_split_nt<2, GROUPED>(g, s, chunks, st);
    case 3: return dispatch_split_nt<3, GROUPED>(g, s, chunks, st);
    case 4: return dispatch_split_nt<4, GROUPED>(g, s, chunks, st);
    case 5: return dispatch_split_nt<5, GROUPED>(g, s, chunks, st);
    case 6: return dispatch_split_nt<6, GROUPED>(g, s, chunks, st);
    case 7: return dispatch_split_nt<7, GROUPED>(g, s, chunks, st);
    default: return dispatch_split_nt<8, GROUPED>(g, s, chunks, st);
  }
}

}  // namespace

bool gemm_splits(int dtype, int mode, int64_t N, int64_t K) {
  return dtype == SAGA_F32 && (mode == SAGA_GEMM_GRU || N > 32 || K > 256);
}

size_t split_workspace_bytes(int mode, int64_t N, int64_t K, int64_t K2, int groups) {
  const SplitShape s = split_shape(N, K, groups, mode), s2 = split_shape(N, K2, groups, mode);
  return (size_t)(s.img_bytes + s2.img_bytes + s.max_bytes + s2.max_bytes);
}

// Workspace: the images of w and w2 (column block by column block), then the largest magnitudes of each
hipError_t launch_gemm_split(const GemmArgs& g0, hipStream_t st) {
  const bool grouped = g0.groups > 0, gru = !grouped && g0.mode == SAGA_GEMM_GRU;
  const bool two = !grouped && g0.mode != SAGA_GEMM_PLAIN;
  const int groups = grouped ? g0.groups : 1;
  const int64_t K2 = two ? g0.K2 : 0;
  const SplitShape s = split_shape(g0.N, g0.K, groups, g0.mode);
  const SplitShape s2 = split_shape(g0.N, K2, groups, g0.mode);
  if (!g0.ws || g0.ws_bytes < split_workspace_bytes(g0.mode, g0.N, g0.K, K2, groups))
    return hipErrorInvalidValue;
  GemmArgs g = g0;
  char* ws = static_cast<char*>(g.ws);
  uint32_t* m1 = reinterpret_cast<uint32_t*>(ws + s.img_bytes + s2.img_bytes);
  uint32_t* m2 = m1 + s.max_bytes / 4;
  g.wmax = m1;
  g.wmax2 = m2;
  uint4* img = reinterpret_cast<uint4*>(ws);
  uint4* img2 = img + s.nch * s.nt * 192;  // behind the first column block of w
  g.wt = img;
  g.wt2 = img2;
  const int stride = (int)(s.nch + s2.nch);
  const unsigned parts = (unsigned)pack_parts(s.nch > s2.nch ? s.nch : s2.nch);
  hipLaunchKernelGGL(k_pack_split, dim3((unsigned)(s.ny * s.nt), (unsigned)(groups + (two ? 1 : 0)), parts),
                     dim3(kPackThreads), 0, st, wsrc1(g), PackOut{img, stride, m1}, wsrc2(g),
                     PackOut{img2, stride, m2}, groups, s.nt);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (gru) {
    const dim3 grid((unsigned)((g.M + 63) / 64));
    switch (s.nt) {
      case 3: hipLaunchKernelGGL(k_gru_split<1>, grid, dim3(kThreads), 0, st, g); break;
      case 6: hipLaunchKernelGGL(k_gru_split<2>, grid, dim3(kThreads), 0, st, g); break;
      case 9: hipLaunchKernelGGL(k_gru_split<3>, grid, dim3(kThreads), 0, st, g); break;
      case 12: hipLaunchKernelGGL(k_gru_split<4>, grid, dim3(kThreads), 0, st, g); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  const int64_t chunks = s.nch + s2.nch;
  return grouped ? dispatch_split<true>(g, s, chunks, st) : dispatch_split<false>(g, s, chunks, st);
}

}  // namespace saga
