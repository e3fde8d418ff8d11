// LSTM Gather of GraphSAGE (Table I, GraphSAGE row; Sec. 3.2, Gather
// paragraph): the in-edges of a destination, in CSR order, are the input
// sequence of an LSTM that starts from h = c = 0; the aggregate is its last
// hidden state.  The paper singles this Gather out as the one that cannot be
// fused: it is a recurrence along each row.
//
// Split of the work:
//   * the input half of every gate pre-activation depends only on the
//     source vertex, so it is one dense product over all vertices,
//     P = X W_ih + b_ih + b_hh (the caller's ApplyVertex GEMM), not a
//     product per edge;
//   * what is left per edge is the recurrent step
//       z = P[u_t] + h W_hh;  i, f, o = sigmoid, g = tanh (blocks i|f|g|o);
//       c = f c + i g;  h = o tanh(c)
//     which this kernel runs.
//
// Schedule.  Instead of one launch per distinct degree (the degree traversal
// the paper measured), a persistent grid pulls rows from a work queue in
// degree-sorted order (the plan's perm: longest rows first, so the longest
// recurrence starts at once while the short rows fill the other CUs).  One
// workgroup of 4H threads runs one row at a time; the longest row's d
// sequential steps bound the time, so a step is kept as short as the vector
// ALU allows (4H x H multiply-adds per step):
//   * thread t serves gate q = t % 4 of hidden unit i = t / 4.  Eight lanes
//     share the recurrent sums of their eight (unit, gate) columns: each keeps
//     an eighth of all eight columns of W_hh in registers, so every h value it
//     reads from LDS feeds eight multiply-adds, and seven DPP adds hand each
//     lane the sum of its own column;
//   * the thread applies that gate's activation; the four activations are then
//     broadcast within the quad, every lane updates its copy of (c, h), and
//     lane 0 writes h to a double-buffered LDS vector -- one workgroup
//     barrier per step;
//   * the P rows of the next PF steps are loaded straight into an LDS ring
//     (global_load_lds_dwordx4) by the first waves, so the recurrence never
//     waits on memory; the neighbour ids come in chunks through LDS.  A step's
//     load is issued, with scalar addresses, before its multiply-adds and not
//     at the end of the step, where every wave would wait for it at the barrier.
// Measured, GraphSAGE-LSTM layer at 131,072 vertices, H = 128, longest row about
// 19,800 in-edges (ms): groups of 4 lanes 12.35, 8 12.18 (12.0 as built now), 16 12.74; before, with
// groups of 4, selects in the exchange, the loads at the end of a step and a
// chain of scalar branches around every wait, 15.70.  One column a lane with h
// broadcast by a DPP modifier on every multiply-add reads the least LDS but took
// 15.78: such multiply-adds issue more slowly.  The vector ALU's own bound is
// 1,024 cycles a step, 8.5 ms for that row at 2.4 GHz.
// The same kernel takes a range of perm positions, so a caller can also run
// the degree traversal (one launch per run of equal degrees) for comparison.
#include <algorithm>

#include "saga_device.h"
#include "saga_internal.h"

namespace saga {
namespace {

constexpr int kGates = 4;    // threads per hidden unit, and gates
constexpr int kGroup = 8;    // lanes that share a recurrent sum
constexpr int kPF = 12;      // P rows in flight ahead of the recurrence
constexpr int kUch = 1024;   // neighbour ids per LDS chunk
constexpr int kLone = 2048;  // the longest rows are handed out one by one
constexpr int kBatch = 8;    // then batches of rows per ticket

typedef __attribute__((address_space(3))) void* lds_ptr;

template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt out of range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// wait until at most n (0 <= n < kPF) of this wave's loads are pending
__device__ __forceinline__ void wait_vm_le(int n) {
  switch (n) {
    case 0: wait_vm<0>(); break;
    case 1: wait_vm<1>(); break;
    case 2: wait_vm<2>(); break;
    case 3: wait_vm<3>(); break;
    case 4: wait_vm<4>(); break;
    case 5: wait_vm<5>(); break;
    case 6: wait_vm<6>(); break;
    case 7: wait_vm<7>(); break;
    case 8: wait_vm<8>(); break;
    case 9: wait_vm<9>(); break;
    case 10: wait_vm<10>(); break;
    default: wait_vm<11>(); break;
  }
  static_assert(kPF == 12, "wait_vm_le covers 0 .. kPF - 1");
}

// A workgroup barrier that orders LDS only: the direct-to-LDS loads in
// flight are waited for explicitly by the waves that issued them.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Gate functions with the hardware reciprocal (about 1 ulp) instead of a
// correctly rounded division, which costs ten instructions:
// sigmoid(x) = 1 / (1 + exp(-x)); tanh(x) = 1 - 2 / (exp(2x) + 1) (saturates
// to +-1 for large |x|; near 0 its absolute error is at the float32 rounding
// level).
__device__ __forceinline__ float sigmoid_fast(float x) {
  return __builtin_amdgcn_rcpf(1.0f + __expf(-x));
}
__device__ __forceinline__ float tanh_fast(float x) {
  return 1.0f - 2.0f * __builtin_amdgcn_rcpf(__expf(2.0f * x) + 1.0f);
}

// The value of lane K of the quad, through DPP; a generic shuffle would go
// through the LDS crossbar (ds_bpermute) and add its latency to every step.
template <int K>
__device__ __forceinline__ float quad_bcast(float x) {
  static_assert(K >= 0 && K < 4, "quad lane");
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), K * 0x55, 0xF, 0xF, false));
}

__global__ void k_lstm_zero(int32_t* q) {
  if (threadIdx.x == 0) q[0] = 0;
}

template <int H>
struct LstmCfg {
  static constexpr int G = 4 * H;                // gate columns
  static constexpr int THREADS = kGates * H;     // 128, 256 or 512
  static constexpr int L = kGroup;
  static constexpr int HPL = H / L;              // values of h a lane holds: 4, 8 or 16
  static constexpr int HV = 4;                   // of them, contiguous in h
  static constexpr int PV = G / 4;               // 16-byte pieces of one P row
  static_assert(HPL * L == H && HPL % HV == 0, "shape");
  static_assert(PV % 64 == 0 || PV < 64, "P row = whole waves or one partial wave");
  static_assert(PV <= THREADS, "P row loaders");
};

// The lane that bit BIT of an index stands for, as the mask one DPP modifier
// exchanges: quad permutations (1, 2) and the half-row mirror (7, for 4).
constexpr int lane_mask(int j) { return (j & 3) ^ (j & 4 ? 7 : 0); }
template <int BIT>
__device__ __forceinline__ float lane_xor(float x) {
  static_assert(BIT == 1 || BIT == 2 || BIT == 4, "index bit");
  constexpr int ctrl = BIT == 1 ? 0xB1 : BIT == 2 ? 0x4E : 0x141;
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), ctrl, 0xF, 0xF, true));
}
// z[j] of a lane belongs to lane ^ lane_mask(j): z[0] ends as the lane's own
// column summed over the group, without a select
template <int BIT, int L>
__device__ __forceinline__ void reduce_scatter(float (&z)[L]) {
#pragma unroll
  for (int j = 0; j < BIT; ++j) z[j] += lane_xor<BIT>(z[j + BIT]);
  if constexpr (BIT > 1) reduce_scatter<BIT / 2>(z);
}

template <int H>
__global__ __launch_bounds__(LstmCfg<H>::THREADS) void k_lstm_gather(LstmArgs a) {
  typedef LstmCfg<H> C;
  constexpr int G = C::G, L = C::L, HPL = C::HPL, HV = C::HV, PV = C::PV, NT = C::THREADS;
  __shared__ __attribute__((aligned(16))) float ring[(kPF + 1) * G];
  __shared__ __attribute__((aligned(16))) float hbuf[2][H];
  __shared__ int32_t ucache[2][kUch];
  __shared__ int s_item[2];
  if (a.counts[kErrFlags]) return;

  const int t = threadIdx.x;
  const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int i = t / kGates, q = t % kGates;  // hidden unit, gate
  float w[L][HPL];  // w[j]: column of lane ^ lane_mask(j)
#pragma unroll
  for (int j = 0; j < L; ++j) {
    const int tj = t ^ lane_mask(j);
#pragma unroll
    for (int r = 0; r < HPL; ++r)
      w[j][r] = a.w_hh[(int64_t)(r / HV * L * HV + lane % L * HV + r % HV) * a.ld_whh + tj % kGates * H + tj / kGates];
  }
  // P row pieces: lane l of wave w (w * 64 + l < PV) loads piece w * 64 + l
  const bool p_loader = wave * 64 < PV;
  const bool p_lane = wave * 64 + lane < PV;
  const int64_t npos = (int64_t)a.perm_end - a.perm_begin;
  const uint32_t ring_base = __builtin_amdgcn_readfirstlane((uint32_t)reinterpret_cast<uintptr_t>((lds_ptr)ring));

  // This wave's pieces of row u into a ring slot.  In assembly: told that the
  // ring is written, the compiler would wait for every load in flight before
  // each read of it, stalling each step on the newest prefetch.
  auto load_p = [&](int u, int slot) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :
                 : "s"(ring_base + (uint32_t)(slot * G + wave * 256) * 4), "v"(a.gates_x + (int64_t)u * a.ld_gx + (wave * 64 + lane) * 4)
                 : "memory", "m0");
  };

  int par = 0;
  for (;;) {
    // ticket k: the single row k for the kLone longest rows, then batches of
    // kBatch consecutive rows (fewer same-address atomics for the many
    // short rows, while no long row waits behind another)
    if (t == 0) s_item[par] = atomicAdd(a.queue, 1);
    lds_barrier();
    const int ticket = s_item[par];
    par ^= 1;
    const int64_t first = ticket < kLone ? ticket : kLone + (int64_t)(ticket - kLone) * kBatch;
    if (first >= npos) break;  // uniform: every thread read the same ticket
    const int64_t last = ticket < kLone ? first + 1 : std::min<int64_t>(first + kBatch, npos);
    for (int64_t item = first; item < last; ++item) {
      const int v = a.perm[a.perm_begin + item];
      const int64_t beg = a.row_ptr[v];
      const int d = a.row_ptr[v + 1] - a.row_ptr[v];
      float* orow = a.out + (int64_t)v * a.ld_out;
      if (d <= 0) {
        if (t < H) orow[t] = 0.0f;
        continue;
      }
      // the previous row's output stores have drained, so the vmcnt waits
      // below count this row's ring loads only; the previous row is done
      // with hbuf and ucache
      wait_vm<0>();
      lds_barrier();
      // neighbour ids of chunks 0 and 1; h = 0
      for (int j = t; j < 2 * kUch; j += NT)
        if (j < d) ucache[j / kUch][j % kUch] = a.col_idx[beg + j];
      if (t < H) hbuf[0][t] = 0.0f;
      float c = 0.0f;
      lds_barrier();
      // P rows of the first kPF steps into ring slots 0 .. kPF-1
      if (p_loader) {
        for (int s = 0; s < kPF; ++s) {
          if (s < d) {
            const int u = __builtin_amdgcn_readfirstlane(ucache[0][s]);
            if (p_lane) load_p(u, s);
          }
        }
      }
      for (int s = 0; s < d; ++s) {
        // this wave's P row of step s has landed (the loads of at most the
        // kPF - 1 later steps may still be pending), then everyone's; h of
        // step s - 1 is in hbuf[s & 1]
        if (p_loader) {
          if (d - s >= kPF) wait_vm<kPF - 1>();  // (the switch is a chain of scalar branches)
          else wait_vm_le(d - 1 - s);
        }
        lds_barrier();
        // this lane's values of h: r is h[r / HV * L HV + lane % L * HV + r % HV]
        const float* hb = hbuf[s & 1] + lane % L * HV;
        float hk[HPL];
#pragma unroll
        for (int r = 0; r < HPL; r += HV) {
          typedef float vec __attribute__((ext_vector_type(HV)));
          const vec hv = *reinterpret_cast<const vec*>(hb + r * L);
#pragma unroll
          for (int j = 0; j < HV; ++j) hk[r + j] = hv[j];
        }
        // this lane's gate-q entry of the step's P row; the slot has landed: its
        // loader waves waited for it before the barrier
        const float pq = ring[(s % (kPF + 1)) * G + q * H + i];
        // the P row of step s + kPF goes to the slot step s - 1 used (read
        // before this step's barrier)
        const int sn = s + kPF;
        if (p_loader && sn < d) {
          const int u = __builtin_amdgcn_readfirstlane(ucache[(sn / kUch) & 1][sn % kUch]);
          if (p_lane) load_p(u, sn % (kPF + 1));
        }
        __builtin_amdgcn_sched_barrier(0);  // keep every read ahead of the multiply-adds
        float z[L];
#pragma unroll
        for (int j = 0; j < L; ++j) z[j] = w[j][0] * hk[0];
#pragma unroll
        for (int r = 1; r < HPL; ++r)
#pragma unroll
          for (int j = 0; j < L; ++j) z[j] = fmaf(w[j][r], hk[r], z[j]);
        reduce_scatter<L / 2>(z);
        const float zq = z[0] + pq;
        // gate q's activation: tanh for g (q == 2, as 2 sigmoid(2x) - 1),
        // sigmoid for i, f, o; then all four to every lane of the quad
        const float sg = sigmoid_fast(q == 2 ? 2.0f * zq : zq);
        const float aq = q == 2 ? 2.0f * sg - 1.0f : sg;
        const float gi = quad_bcast<0>(aq), gf = quad_bcast<1>(aq), gg = quad_bcast<2>(aq),
                    go = quad_bcast<3>(aq);
        c = gf * c + gi * gg;
        const float hn = go * tanh_fast(c);
        if (q == 0) {
          hbuf[(s + 1) & 1][i] = hn;
          if (s == d - 1) orow[i] = hn;
        }
        // entering chunk cc: chunk cc + 1 replaces chunk cc - 1, whose ids
        // were last read for the load of step cc * kUch - 1 (issued kPF
        // steps, and barriers, ago)
        if ((s + 1) % kUch == 0) {
          const int cc = (s + 1) / kUch;
          for (int j = t; j < kUch; j += NT) {
            const int64_t e = (int64_t)(cc + 1) * kUch + j;
            if (e < d) ucache[(cc + 1) & 1][j] = a.col_idx[beg + e];
          }
        }
      }
    }  // rows of the ticket
  }
}

template <int H>
hipError_t launch_h(const LstmArgs& a, hipStream_t st) {
  // one workgroup per CU: the longest row's step time is what bounds the
  // call, so it does not share its CU's vector ALUs with a second row
  static int grid = [] {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess)
      (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    return cus > 0 ? cus : 256;
  }();
  const int64_t n = (int64_t)a.perm_end - a.perm_begin;
  const unsigned g = (unsigned)std::min<int64_t>(grid, n);
  hipLaunchKernelGGL(k_lstm_zero, dim3(1), dim3(64), 0, st, a.queue);
  hipLaunchKernelGGL((k_lstm_gather<H>), dim3(g), dim3(LstmCfg<H>::THREADS), 0, st, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_lstm_gather(const LstmArgs& a, hipStream_t st) {
  if (a.perm_end <= a.perm_begin) return hipSuccess;
  switch (a.hidden) {
    case 32: return launch_h<32>(a, st);
    case 64: return launch_h<64>(a, st);
    case 128: return launch_h<128>(a, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace saga
