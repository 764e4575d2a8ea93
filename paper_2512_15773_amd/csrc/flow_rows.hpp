// Forward pass of a few rows in ONE launch: the layers are cut into phases and the phases into tasks, a workgroup per
// task, and a task waits until the tasks of the phase before it have delivered.
//
//   phase A  residual -> LayerNorm + FiLM -> q | k | v of 16 features                  (layer 0: embedding first)
//   phase B  attention of all heads (one per wavefront) -> output projection of 16 features, added to the residual
//   phase X, Y  the same for cross-attention: queries; attention over the observation tokens and projection
//   phase C  residual -> LayerNorm + FiLM -> 64 hidden features, GELU
//   phase D  down projection of 16 features, added to the residual
//   head     LayerNorm -> output projection; in a rollout the sampler step, done by phase A of the next transition
//
// For the fewest rows (flow_forward_pays, flow_draft_pays): fp32 networks, whose products are worth sixteen units a row, rollouts
// with cross-attention, and bf16 networks (one environment, K = 8: d = 256 with a conditioning vector round 250 -> 214 us, d = 512
// with cross-attention 801 -> 601).
// What bounds a few rows is the chain of dependent steps, not their work.  With two launches per layer a step was 6 to
// 12 us: 2.4 us between dependent launches, the weights requested only then, and partial sums of the whole row (up to 272 KB)
// read by every workgroup.  Here a step is an exchange of 16 to 64 KB through the L2 (0.4 to 0.9 us), workgroups of the
// next phases wait with their weights in registers, and a product's contraction is split over the wavefronts of its
// workgroup (a wavefront owns one head's columns), so that nothing but finished activations leaves a workgroup.
// C2, one environment, K = 8: verify 177 -> 105 us, rollout 208 -> 147, round 390 -> 257; the split also shortens the
// chains of additions.  More rows: 16, 32, 64, 96, 128 rows 134, 186, 300, 414, 527 us against 181, 218, 288, 432, 511.
//
// Waiting.  The buffers that phases hand to each other hold the pattern FLOW_EMPTY (a NaN that no task stores) until their
// data arrives: a task reads its operands again until none of them is empty, which costs one way through the L2 (a counter
// or flag costs three: stores complete, flag, data).  Every buffer exists twice, for even and odd passes through the layers
// (i = number of the pass), and is emptied again when all its readers are known to be done:
//   phase C (X where there is one) of pass i has seen every output of B, so A and B of pass i are done with
//     the residual before A, q | k | v and the embedding; it empties its share of them;
//   (C with cross-attention: the residual before X and the cross queries, which X and Y have read);
//   phase A of pass i + 1 has seen every output of D and empties the residual before C and the hidden layer of pass i;
//   after the last pass the head / the last sampler step does, so a launch leaves everything empty, as it found it.
// A task starts to poll only when the phase two before its own is complete (guard): all of that phase's tasks have added
// to its counter, behind their stores and emptyings.  That is two phases of slack, so it costs nothing, keeps the polls to the
// one phase that is next, and is why nobody meets data of pass i - 2: what a task of pass i polls or writes was emptied by C / X
// of pass i - 2 or A of pass i - 1 at the latest, A of pass i starts behind the counter of C(i-1), C(i-1) behind A(i-1)
// (X(i-1)), and every other task of pass i behind data or a counter of A(i).
// Every eighth row is a set; a set belongs to one XCD, and its tasks are drawn from the set's ticket in the order of the
// phases and depend on earlier tickets only.  The earliest unfinished task has been drawn by a workgroup that is running, and
// waits for nothing: the launch makes progress with any number of resident workgroups, also beside other launches of this
// kind.  The rows of a set are its own, so the XCDs do not wait for each other.  Every wait is bounded all the same
// (flow_turn): past the bound the status word reports it, the waits of the other tasks end too, and the launch drains.
// A workgroup asks the hardware which XCD it is on and takes the set of that number for it (owner word); a set whose XCD has
// no workgroup of this launch for FLOW_LATE looks (another partition mode, an XCD busy with other work) is taken by one whose
// tickets have run out, and every workgroup of that XCD which waits or comes by joins it (flow_next_set).  So every set is
// worked off, each by one XCD, at the rate of an XCD: pairs of C2 rounds (one environment, K = 7 / K = 8) of two contexts on two
// streams 271 / 336 us, 346 / 417 where only the workgroup that took a set works on it (439 / 472 one after the other).
// Visibility: what one workgroup writes for another in the same launch therefore meets in one L2.  Stores are plain (the L1
// writes through), loads of device scope (sc1) pass the L1 by.  One way between two units of an XCD 0.26 us; with stores of
// device scope, which go on to memory, 0.49 (0.65 to another XCD): one C2 environment 258 -> 230 us a round, four C4 914 -> 862.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "fused_mfma.hpp"
#include "few_plan.hpp"
#include "few_rows.hpp"
#include "round_kernels.hpp"

namespace tsdp {

constexpr int FLOW_NAP = 3;                       // x 64 cycles between the first words of a store and all of them
constexpr int FLOW_KINDS = 6;                     // counters of a row: one per kind of phase
constexpr int FLOW_LATE = 64;                     // looks at a set that nobody has taken (about half a microsecond each) before another XCD takes it
// lines of the tickets (one per set), of the word that ends all waits, of the sets' owners and of the counters of `rows` rows
constexpr int FLOW_SETS = 8, FLOW_OVER_LINE = 8, FLOW_OWNER_LINE = 9, FLOW_CNT_LINE = 17;
inline int flow_lines(size_t rows) { return (int)(FLOW_CNT_LINE + rows * FLOW_KINDS); }
constexpr int FLOW_STATUS = 16;                   // status bit: a wait ran into its bound

// Feature blocks of a task.  fp32: one, its products are bound by a unit's matrix rate (one C2 environment 260 us a round, with two
// blocks 312).  bf16: two, half as many tasks then read a row's activations (eight rows of d = 256 91 us a pass, 137 with one).
template <class TT, int D> constexpr int flow_blocks() { return sizeof(typename TT::elem) == 2 && D % 32 == 0 ? 2 : 1; }

template <class TT_, int D_, int H_, int HEADS_, int SX_ = 0, int FS_ = flow_blocks<TT_, D_>()>
struct FlowCfg {
  typedef TT_ TT;
  static constexpr int D = D_, H = H_, HEADS = HEADS_, SX = SX_, FS = FS_, DH = D / HEADS, NB = H / 16, NW = HEADS, TH = NW * 64;
  static constexpr int G = D / 16 / FS;           // tasks of a phase and row
  static constexpr int KW = DH / TT::KSTEP, KWM = 4 * KW, CF = DH / 16, VQ = TT::VW / 4;   // a wavefront's k-steps of D, of 4 D
  static constexpr int NPH = SX ? 6 : 4;
  static constexpr int NHF = H == 16 ? 2 : 1;     // fragment rows of the output projection at most (H A <= 512)
  // a row's buffers, one of two sets: embedding, residual before A, after B, (after Y), q | k | v, hidden layer, (cross queries)
  static constexpr int HB = H * D * 4, XB = H * D * (int)sizeof(typename TT::elem);
  static constexpr int O_E = 0, O_H0 = HB, O_H1 = 2 * HB, O_H2 = SX ? 3 * HB : O_H1, O_Q = O_H2 + HB, O_U = O_Q + 3 * XB, O_XQ = O_U + 4 * XB,
                       SET_B = O_XQ + (SX ? XB : 0);
  static constexpr int STAT_B = 2 * NW * H * 4, RED_B = NW * 4 * FS * NB * 1024, STEP_B = 2 * 512 * 4;
  // LDS: statistics, sums, a step's outputs and latents, token embedding.  Wide rows: the embedding (32 KB) lies over the last quarter
  // of the sums, which phase A does not use: 134 KB with A = 16, one after the other 166 KB.  (512 threads leave 256 registers: before
  // its rows phase A of the wide shape keeps 26 of its operands' in scratch, 108 bytes a lane; no other shape spills vectors.)
  static constexpr bool WIDE = D * H >= FEW_WIDE;
  static constexpr int O_ET = WIDE ? STAT_B : STAT_B + RED_B, O_RED = WIDE ? STAT_B + STEP_B : STAT_B, O_TOK = WIDE ? O_RED + RED_B / 4 * 3 : O_ET + STEP_B;
  static constexpr int lds(int A) { return O_TOK + D * A * 4 > O_RED + RED_B ? O_TOK + D * A * 4 : O_RED + RED_B; }
  static_assert(DH % TT::KSTEP == 0 && H % 16 == 0 && D % (16 * FS) == 0, "shape");
};

struct FlowIO {
  int R_cap, groups, phases;     // groups: the rows of a set are dealt to this many tasks of a phase and slice
  const int32_t* word;           // live row count; rollout: K_eff of every environment
  int32_t* ticket; int32_t* over; int32_t* owner; int32_t* cnt; int32_t* status;
  const float* x;                // latents of the rows
  const int32_t* row_t; const int32_t* row_env; int T;
  const float* mod; int mod_row, by_t;           // FiLM vectors: floats between rows; by_t: rows are timesteps
  unsigned char* buf;            // [row][2][SET_B]: residuals as [D/16][H][16]; q, k, transposed v and the hidden layer as MFMA operands
  float* eps_out;
  int A;
  int k_max; float* y[2];        // rollout
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t flow_rsrc(const void* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
typedef unsigned flow_u4 __attribute__((ext_vector_type(4)));
typedef unsigned flow_u2 __attribute__((ext_vector_type(2)));
constexpr int FLOW_SC1 = 16;                      // device scope
constexpr unsigned FLOW_EMPTY = 0xFFFFFFFFu;      // an fp32 NaN, two bf16 NaNs; writers store the usual one instead
__device__ __forceinline__ unsigned flow_word(unsigned w) { return w == FLOW_EMPTY ? 0x7FC07FC0u : w; }
__device__ __forceinline__ void flow_st(__amdgpu_buffer_rsrc_t r, int off, f32x4 v) {
  flow_u4 w = __builtin_bit_cast(flow_u4, v);
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = flow_word(w[i]);
  __builtin_amdgcn_raw_buffer_store_b128(w, r, off, 0, 0);
}
__device__ __forceinline__ void flow_st(__amdgpu_buffer_rsrc_t r, int off, bf16x4 v) {
  flow_u2 w = __builtin_bit_cast(flow_u2, v);
  w[0] = flow_word(w[0]); w[1] = flow_word(w[1]);
  __builtin_amdgcn_raw_buffer_store_b64(w, r, off, 0, 0);
}
template <class F> __device__ __forceinline__ F flow_ld(__amdgpu_buffer_rsrc_t r, int off) {   // 16 or 8 bytes
  if constexpr (sizeof(F) == 16) return __builtin_bit_cast(F, (flow_u4)__builtin_amdgcn_raw_buffer_load_b128(r, off, 0, FLOW_SC1));
  else return __builtin_bit_cast(F, (flow_u2)__builtin_amdgcn_raw_buffer_load_b64(r, off, 0, FLOW_SC1));
}
// the largest word of everything in v (arrays of vectors)
template <class F> __device__ __forceinline__ void flow_max(unsigned& m, const F& v) {
  if constexpr (std::is_array<F>::value) {
#pragma unroll
    for (auto& e : v) flow_max(m, e);
  } else if constexpr (sizeof(F) == 16) {
    const flow_u4 w = __builtin_bit_cast(flow_u4, v);
    m = max(max(max(m, w[0]), max(w[1], w[2])), w[3]);
  } else {
    const flow_u2 w = __builtin_bit_cast(flow_u2, v);
    m = max(max(m, w[0]), w[1]);
  }
}
// behind poll n of a wait that found its data missing: true ends the wait (cannot happen; lets the launch drain)
__device__ __forceinline__ bool flow_over(const FlowIO& io, int n, int lane) {
  const FlowTurn turn = flow_turn(n);
  if (turn == FLOW_POLL) return false;
  if (turn == FLOW_ASK) return __builtin_amdgcn_readfirstlane(__hip_atomic_load(io.over, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != 0;
  if (lane == 0) {
    atomicOr(io.status, FLOW_STATUS);
    __hip_atomic_store(io.over, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  return true;
}
// Waits for N pieces of BYTES each at off (what one store instruction writes, or several): every lane looks at one word, so that
// 64 / N lanes look at each piece.  Cheap to repeat, where reading everything is not; who reads the pieces afterwards still checks them whole.
template <int N, int BYTES>
__device__ __forceinline__ void flow_sample(const FlowIO& io, __amdgpu_buffer_rsrc_t r, int off, int lane) {
  static_assert(64 % N == 0 && BYTES % (64 / N) == 0, "lanes per piece");
  const int at = off + lane % N * BYTES + lane / N * (BYTES / (64 / N)) + 4 * (lane & 1);
  for (int n = 0;; ++n) {
    asm volatile("" ::: "memory");
    if (!__any(__builtin_amdgcn_raw_buffer_load_b32(r, at, 0, FLOW_SC1) == FLOW_EMPTY) || flow_over(io, n, lane)) break;
  }
  __builtin_amdgcn_s_sleep(FLOW_NAP);
}
// empties `bytes` (a multiple of 16) at off
__device__ __forceinline__ void flow_clear(__amdgpu_buffer_rsrc_t r, int off, int bytes, int tid, int threads) {
  for (int i = tid * 16; i < bytes; i += threads * 16)
    __builtin_amdgcn_raw_buffer_store_b128(flow_u4{FLOW_EMPTY, FLOW_EMPTY, FLOW_EMPTY, FLOW_EMPTY}, r, off + i, 0, 0);
}

__device__ __forceinline__ int flow_xcc() { return __builtin_amdgcn_s_getreg(20 | 3 << 11); }   // HW_REG_XCC_ID, 4 bits
__device__ __forceinline__ int32_t flow_word_at(const int32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// (one thread) takes the set for the XCD: true if it is the XCD's now
__device__ __forceinline__ bool flow_take(const FlowIO& io, int set, int xcc) {
  int32_t had = 0;
  __hip_atomic_compare_exchange_strong(io.owner + set * SYNC_LINE, &had, xcc + 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return had == 0 || had == xcc + 1;
}
// (wavefront 0, all lanes) the set to draw from next, or FLOW_LEAVE: one of this XCD's that is not among `done`, or one that nobody
// has taken although its own XCD had time to.  looks: so far in this launch (a workgroup that has waited once does not wait again)
__device__ __forceinline__ int flow_other_set(const FlowIO& io, int rows, int xcc, unsigned done, int& looks, int lane) {
  const int n = min(rows, FLOW_SETS);
  for (;; ++looks) {
    const int32_t owner = flow_word_at(io.owner + min(lane, FLOW_SETS - 1) * SYNC_LINE);
    const unsigned open = (unsigned)__ballot(lane < n && owner == 0), ours = (unsigned)__ballot(lane < n && owner == xcc + 1) & ~done;
    const int set = flow_next_set(open, ours, looks >= FLOW_LATE);
    if (set == FLOW_LEAVE || (set >= 0 && __builtin_amdgcn_readfirstlane(lane == 0 ? flow_take(io, set, xcc) : 0))) return set;
    __builtin_amdgcn_s_sleep(8);
  }
}

// wavefront 0 waits until counter `kind` of the row has reached `target`, the others at the barrier
__device__ __forceinline__ void flow_guard(const FlowIO& io, int row, int kind, int target, int wave, int lane) {
  if (wave == 0 && target > 0) {
    int32_t* c = io.cnt + (row * FLOW_KINDS + kind) * SYNC_LINE;
    for (int n = 0;; ++n) {
      if (__builtin_amdgcn_readfirstlane(__hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >= target) break;
      if (flow_over(io, n, lane)) break;
      __builtin_amdgcn_s_sleep(2);
    }
  }
  asm volatile("" ::: "memory");
  lds_barrier();
}
// reads the operands v.. with load() until none is empty
template <class F, class... V>
__device__ __forceinline__ void flow_poll(const FlowIO& io, int lane, F&& load, const V&... v) {
  for (int n = 0;; ++n) {
    asm volatile("" ::: "memory");
    load();
    __builtin_amdgcn_sched_barrier(0);                   // (all loads in flight before the first is looked at: 64 KB 3.6 -> 1 us)
    unsigned m = 0;
    (flow_max(m, v), ...);
    if (!__any(m == FLOW_EMPTY)) break;
    if (flow_over(io, n, lane)) break;
  }
}
// the task's stores are complete: count it
__device__ __forceinline__ void flow_signal(const FlowIO& io, int row, int kind) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  lds_barrier();
  if (threadIdx.x == 0)
    __hip_atomic_fetch_add(io.cnt + (row * FLOW_KINDS + kind) * SYNC_LINE, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A wavefront's columns of the residual (those of its head) of all tokens: lane -> token l16, VW neighbouring columns
// of every k-step, which is the layout of an MFMA operand.
template <class C> using FlowV = f32x4[C::KW][C::NB][C::VQ];

template <class C>
struct FlowTask {
  typedef typename C::TT TT;
  typedef typename TT::elem elem;
  typedef typename TT::frag frag;
  typedef typename TT::vec4 vec4;
  static constexpr int D = C::D, H = C::H, DH = C::DH, NB = C::NB, NW = C::NW, KW = C::KW, KWM = C::KWM, CF = C::CF, VQ = C::VQ, VW = TT::VW,
                       KSTEP = TT::KSTEP, FS = C::FS, ES = sizeof(elem);
  const FusedNet& net;
  const FlowIO& io;
  const int slice, tid, wave, lane, l16, lg;
  float* stat; f32x4* red; float* et; float* yt; float* tokw;

  __device__ FlowTask(const FusedNet& n, const FlowIO& i, int s, int t, unsigned char* lds)
      : net(n), io(i), slice(s), tid(t), wave(__builtin_amdgcn_readfirstlane(t >> 6)), lane(t & 63), l16(t & 15), lg((t & 63) >> 4) {
    stat = reinterpret_cast<float*>(lds);
    red = reinterpret_cast<f32x4*>(lds + C::O_RED);
    et = reinterpret_cast<float*>(lds + C::O_ET);
    yt = et + 512;
    tokw = reinterpret_cast<float*>(lds + C::O_TOK);
  }
  __device__ int col(int ks, int q) const { return wave * DH + ks * KSTEP + lg * VW + q * 4; }
  __device__ __amdgpu_buffer_rsrc_t bufs(int row, int pass) const {
    return flow_rsrc(io.buf + ((size_t)row * 2 + (pass & 1)) * C::SET_B, C::SET_B);
  }

  // ---- operands ---------------------------------------------------------------------------------------------------
  template <int MF, int NK>
  __device__ void weights(frag (&w)[MF][NK], const void* p, int ks_total, const int (&row)[MF], int ks0) const {
#pragma unroll
    for (int m = 0; m < MF; ++m)
#pragma unroll
      for (int k = 0; k < NK; ++k) w[m][k] = reinterpret_cast<const frag*>(p)[((size_t)row[m] * ks_total + ks0 + k) * 64 + lane];
  }
  __device__ void residual(__amdgpu_buffer_rsrc_t r, int at, FlowV<C>& v) const {
    flow_poll(io, lane, [&]() {
#pragma unroll
      for (int ks = 0; ks < KW; ++ks)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int q = 0; q < VQ; ++q) {
            const int c = col(ks, q);
            v[ks][nb][q] = flow_ld<f32x4>(r, at + ((c >> 4) * H * 16 + (nb * 16 + l16) * 16 + (c & 15)) * 4);
          }
    }, v);
  }
  struct Film { f32x4 g[KW][VQ], b[KW][VQ]; };
  __device__ void film(Film& f, const float* m) const {
#pragma unroll
    for (int ks = 0; ks < KW; ++ks)
#pragma unroll
      for (int q = 0; q < VQ; ++q) {
        f.g[ks][q] = *reinterpret_cast<const f32x4*>(m + col(ks, q));
        f.b[ks][q] = *reinterpret_cast<const f32x4*>(m + D + col(ks, q));
      }
  }
  // LayerNorm of v as the product's operand.  A wavefront sums its columns of a token and their squared deviations from its
  // own mean; the NW pairs are combined after one barrier.
  template <bool FILM>
  __device__ void norm(const FlowV<C>& v, const Film& f, frag (&a)[KW][NB]) const {
    constexpr float NC = (float)DH;
    float* s1 = stat;
    float* s2 = stat + NW * H;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      float s = 0.0f, m2 = 0.0f;
#pragma unroll
      for (int ks = 0; ks < KW; ++ks)
#pragma unroll
        for (int q = 0; q < VQ; ++q) s += (v[ks][nb][q][0] + v[ks][nb][q][1]) + (v[ks][nb][q][2] + v[ks][nb][q][3]);
      s = add_half32(add_row16(s));
      const float mw = net.rms ? 0.0f : s * (1.0f / NC);
#pragma unroll
      for (int ks = 0; ks < KW; ++ks)
#pragma unroll
        for (int q = 0; q < VQ; ++q)
#pragma unroll
          for (int i = 0; i < 4; ++i) { const float d = v[ks][nb][q][i] - mw; m2 = fmaf(d, d, m2); }
      m2 = add_half32(add_row16(m2));
      if (lg == 0) { s1[wave * H + nb * 16 + l16] = s; s2[wave * H + nb * 16 + l16] = m2; }
    }
    lds_barrier();
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      float sw[NW], s = 0.0f, m2 = 0.0f;
#pragma unroll
      for (int w = 0; w < NW; ++w) { sw[w] = s1[w * H + nb * 16 + l16]; s += sw[w]; m2 += s2[w * H + nb * 16 + l16]; }
      const float mean = net.rms ? 0.0f : s * (1.0f / D);
      if (!net.rms) {
#pragma unroll
        for (int w = 0; w < NW; ++w) { const float d = sw[w] * (1.0f / NC) - mean; m2 = fmaf(NC * d, d, m2); }
      }
      const float rs = rsqrtf(m2 * (1.0f / D) + 1e-5f);
#pragma unroll
      for (int ks = 0; ks < KW; ++ks) {
        f32x4 y[VQ];
#pragma unroll
        for (int q = 0; q < VQ; ++q) {
          y[q] = (v[ks][nb][q] - mean) * rs;
          if (FILM) y[q] = y[q] * (1.0f + f.g[ks][q]) + f.b[ks][q];
        }
        if constexpr (VQ == 1) a[ks][nb] = y[0];
        else {
#pragma unroll
          for (int i = 0; i < 8; ++i) a[ks][nb][i] = (__bf16)y[i / 4][i % 4];
        }
      }
    }
  }

  // ---- a wavefront's share of a product, reduced over the wavefronts: item = (fragment row m, token fragment nb) -----
  template <int MF, int NK>
  __device__ void product(const frag (&w)[MF][NK], const frag (&a)[NK][NB], f32x4 (&acc)[MF][NB]) const {
#pragma unroll
    for (int m = 0; m < MF; ++m)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        acc[m][nb] = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < NK; ++k) TT::mma(w[m][k], a[k][nb], acc[m][nb]);
      }
  }
  template <int MF>
  __device__ void deposit(const f32x4 (&acc)[MF][NB]) const {
#pragma unroll
    for (int m = 0; m < MF; ++m)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) red[(wave * MF * NB + m * NB + nb) * 64 + lane] = acc[m][nb];
    lds_barrier();
  }
  template <int MF>
  __device__ f32x4 collect(int it) const {
    f32x4 s = red[it * 64 + lane];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += red[(w * MF * NB + it) * 64 + lane];
    return s;
  }
  // the task's items are dealt to the wavefronts round-robin
  template <int MF, class F>
  __device__ void items(F&& f) const {
    constexpr int N = MF * NB, PW = (N + NW - 1) / NW;
#pragma unroll
    for (int j = 0; j < PW; ++j) {
      const int it = wave + j * NW;
      if (it < N) f(j, it / NB, it % NB, it);
    }
  }
  template <int MF> static __device__ constexpr int per_wave() { return (MF * NB + NW - 1) / NW; }
  __device__ int hoff(int blk, int nb) const { return ((blk * H + nb * 16 + l16) * 16 + lg * 4) * 4; }   // item's 16 bytes in a residual

  // the task's blocks of 16 features (slice * FS ..): their bias, their residual, the sum of both and the product
  __device__ void own_bias(const float* b, f32x4 (&bias)[per_wave<FS>()]) const {
    items<FS>([&](int j, int m, int, int) { bias[j] = *reinterpret_cast<const f32x4*>(b + (slice * FS + m) * 16 + lg * 4); });
  }
  __device__ void own_residual(__amdgpu_buffer_rsrc_t r, int at, f32x4 (&res)[per_wave<FS>()]) const {
    items<FS>([&](int j, int mf, int nb, int) { res[j] = flow_ld<f32x4>(r, at + hoff(slice * FS + mf, nb)); });
  }
  __device__ void add_residual(__amdgpu_buffer_rsrc_t r, int at, const f32x4 (&res)[per_wave<FS>()], const f32x4 (&bias)[per_wave<FS>()]) const {
    items<FS>([&](int j, int m, int nb, int it) { flow_st(r, at + hoff(slice * FS + m, nb), collect<FS>(it) + res[j] + bias[j]); });
  }
  // empties the task's share of a residual, of n activations per feature
  __device__ void clear_residual(__amdgpu_buffer_rsrc_t r, int at) const { flow_clear(r, at + slice * (C::HB / C::G), C::HB / C::G, tid, C::TH); }
  __device__ void clear_act(__amdgpu_buffer_rsrc_t r, int at, int n) const {
    flow_clear(r, at + slice * (n * C::XB / C::G), n * C::XB / C::G, tid, C::TH);
  }
  // what phase A of the next pass, the head or the last sampler step empties
  __device__ void clear_pass(int row, int pass) const {
    const auto r = bufs(row, pass);
    clear_residual(r, C::O_H2);
    clear_act(r, C::O_U, 4);
  }

  // byte offset of features f .. f+3 (f a multiple of 4) of token fragment nb in an operand of k-steps: [ks][nb][64 lanes][VW]
  __device__ int foff(int f, int nb) const {
    return (((f / KSTEP * NB + nb) * 64 + l16 + 16 * (f % KSTEP / VW)) * VW + f % VW) * ES;
  }

  // output projection of the attention's result: weights of the wavefront's head, 16 columns at a time
  __device__ void proj_weights(const void* p, vec4 (&w)[FS][CF]) const {
    constexpr int KS = D / KSTEP;
#pragma unroll
    for (int m = 0; m < FS; ++m)
#pragma unroll
      for (int cf = 0; cf < CF; ++cf) {
        const int c = wave * DH + cf * 16 + lg * 4;      // lane: row l16, columns c .. c+3
        w[m][cf] = *reinterpret_cast<const vec4*>(reinterpret_cast<const elem*>(p) +
                                                  (((size_t)(slice * FS + m) * KS + c / KSTEP) * 64 + l16 + 16 * (c % KSTEP / VW)) * VW + c % VW);
      }
  }
  // softmax(q k^T) v of the wavefront's head (kk[ks][kf], vv[cf][kf]) times its columns of the output projection
  template <int N>
  __device__ void attend(const frag (&q)[KW][NB], const frag (&kk)[KW][N], const vec4 (&vv)[CF][N], const vec4 (&w)[FS][CF],
                         f32x4 (&acc)[FS][NB]) const {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
      for (int m = 0; m < FS; ++m) acc[m][nb] = f32x4{0, 0, 0, 0};
      f32x4 s[N];
#pragma unroll
      for (int kf = 0; kf < N; ++kf) {
        s[kf] = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < KW; ++ks) TT::mma(kk[ks][kf], q[ks][nb], s[kf]);
      }
      vec4 p[N];
      softmax_keys<TT, N>(s, p, DH);
#pragma unroll
      for (int cf = 0; cf < CF; ++cf) {
        f32x4 o = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int kf = 0; kf < N; ++kf) TT::mma16(vv[cf][kf], p[kf], o);
        const vec4 ob = TT::cvt(o);
#pragma unroll
        for (int m = 0; m < FS; ++m) TT::mma16(w[m][cf], ob, acc[m][nb]);
      }
    }
  }
};

// groups of eight workgroups, one per XCD (consecutive workgroups go to the XCDs in turn); ROLL: the drafter's rollout,
// rows are environments
template <class C, bool ROLL>
__global__ __launch_bounds__(C::TH) void k_flow(FusedNet net, FlowIO io, std::conditional_t<ROLL, DraftIO, FewNone> dr) {
  typedef typename C::TT TT;
  typedef typename TT::elem elem;
  typedef typename TT::frag frag;
  typedef typename TT::vec4 vec4;
  typedef FlowTask<C> Task;
  constexpr int D = C::D, H = C::H, DH = C::DH, NB = C::NB, KW = C::KW, KWM = C::KWM, CF = C::CF, VQ = C::VQ, VW = TT::VW, KSTEP = TT::KSTEP,
                FS = C::FS, ES = sizeof(elem), KD = D / KSTEP, G = C::G;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  __shared__ int32_t drawn[4];                           // ticket; next set; sets whose tickets ran out, looks (registers across tasks: 0.5 % of a round)
  const int xcc = flow_xcc();
  const bool first_wave = threadIdx.x < 64;
  int set = xcc % FLOW_SETS;
  if (threadIdx.x == 0) { drawn[1] = flow_take(io, set, xcc); drawn[2] = drawn[3] = 0; }
  const int rows = ROLL ? io.R_cap : min(*io.word, io.R_cap), A = io.A;
  if (rows == 0) return;
  int phases = io.phases, n_tasks = 0;
  auto enter = [&]() {                                   // the set's tasks; rollout: its longest one and the phase that ends it
    if (ROLL) {
      int k_max = 0;
      for (int row = set; row < rows; row += FLOW_SETS) k_max = max(k_max, io.word[row]);
      phases = k_max == 0 ? 0 : min(io.phases, k_max * net.L * C::NPH + 1);
    }
    n_tasks = set < rows ? phases * io.groups * G : 0;
  };
  lds_barrier();
  if (__builtin_amdgcn_readfirstlane(drawn[1])) enter();
  for (;;) {
    lds_barrier();                                       // the task before has read its LDS
    if (threadIdx.x == 0) drawn[0] = n_tasks ? __hip_atomic_fetch_add(io.ticket + set * SYNC_LINE, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    lds_barrier();
    const int ticket = __builtin_amdgcn_readfirstlane(drawn[0]);
    if (ticket >= n_tasks) {
      if (first_wave) {                                  // (only now: the owners' words are other XCDs', and far)
        const int done = drawn[2] | 1 << set;
        int looks = drawn[3];
        const int other = flow_other_set(io, rows, xcc, done, looks, threadIdx.x);
        if (threadIdx.x == 0) { drawn[1] = other; drawn[2] = done; drawn[3] = looks; }
      }
      lds_barrier();
      set = __builtin_amdgcn_readfirstlane(drawn[1]);
      if (set < 0) return;
      enter();
      continue;
    }
    const int slice = ticket % G, group = ticket / G % io.groups, phase = ticket / G / io.groups;
    const int row0 = set + FLOW_SETS * group, row_step = FLOW_SETS * io.groups;
    if (row0 >= rows) continue;
    const int pass = phase / C::NPH, layer = pass % net.L, k = ROLL ? pass / net.L + 1 : 1;   // k: the drafted transition
    const bool end = !ROLL && pass == net.L;             // behind the last layer
    const int kind0 = phase % C::NPH, kind = kind0 < 2 || C::SX ? kind0 : kind0 + 2;           // 0 A, 1 B, 2 X, 3 Y, 4 C, 5 D
    // guard: the phase two before
    const int guard = kind == 0 ? 4 : kind == 1 ? 5 : kind == 4 && !C::SX ? 0 : kind == 5 && !C::SX ? 1 : kind - 2;
    const int target = (kind < 2 ? pass : pass + 1) * G;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                        // (addresses are derived per task, not kept across tasks)
    Task t(net, io, slice, tid, lds);
    const int lane = t.lane, wave = t.wave, l16 = t.l16, lg = t.lg;
    const FusedLayer& W = net.layer[layer];
    auto wait = [&](int row) { flow_guard(io, row, guard, target, wave, lane); };
    auto drafts = [&](int row) { return !ROLL || k <= io.word[row]; };   // rollout: transition k runs while k <= K_eff
    auto mod_row = [&](int row) {
      const int r0 = min(io.row_t[row], io.T - 1), tt = max(ROLL ? r0 - (k - 1) : r0, 0);
      return io.mod + (size_t)(io.by_t ? tt : (ROLL ? row * io.k_max + min(k, io.k_max) - 1 : row)) * io.mod_row + (size_t)layer * 4 * D;
    };

    if (kind == 0 && !end) {
      frag w[3 * FS][KW];
      int fr[3 * FS];
#pragma unroll
      for (int m = 0; m < 3 * FS; ++m) {
        const int blk = slice * FS + m % FS, head = blk * 16 / DH;
        fr[m] = head * (3 * CF) + m / FS * CF + blk % CF;
      }
      t.weights(w, W.qkv, KD, fr, wave * KW);
      f32x4 bias[Task::template per_wave<3 * FS>()];
      t.template items<3 * FS>([&](int j, int m, int, int) {
        const float* b = W.qkv_b + fr[m] * 16;           // (values: one feature per lane)
        bias[j] = m / FS == 2 ? f32x4{b[l16], b[l16], b[l16], b[l16]} : *reinterpret_cast<const f32x4*>(b + lg * 4);
      });
      frag wh[C::NHF][KW];
      FlowV<C> pe;                                       // embedding of an all-zero latent
      const bool first = layer == 0, step = ROLL && first && k > 1;
      if (first) {
#pragma unroll
        for (int ks = 0; ks < KW; ++ks)
#pragma unroll
          for (int q = 0; q < VQ; ++q) {
            const f32x4 tb = *reinterpret_cast<const f32x4*>(net.tok_b + t.col(ks, q));
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
              pe[ks][nb][q] = tb + *reinterpret_cast<const f32x4*>(net.pos + (size_t)(nb * 16 + l16) * D + t.col(ks, q));
          }
        for (int i = tid; i < A * (D / 4); i += C::TH) reinterpret_cast<f32x4*>(t.tokw)[i] = reinterpret_cast<const f32x4*>(net.tok_wt)[i];
        if (step) {
          int hr[C::NHF];
#pragma unroll
          for (int i = 0; i < C::NHF; ++i) hr[i] = min(i, (A + 15) / 16 - 1);
          t.weights(wh, net.head, KD, hr, wave * KW);
        }
      }
      for (int row = row0; row < rows; row += row_step) {
        const int ke = ROLL ? io.word[row] : 0;
        const bool ends = ROLL && step && ke == k - 1;   // the environment's last drafted transition ends here
        if (ROLL && k > ke && !ends) continue;
        if (ends && slice != 0) {                        // D of the last pass is complete: empty the buffers
          flow_guard(io, row, 5, pass * G, wave, lane);
          t.clear_pass(row, pass - 1);
          continue;
        }
        typename Task::Film f;
        t.film(f, mod_row(row));
        const auto r = t.bufs(row, pass);
        FlowV<C> v;
        frag a[KW][NB];
        if (first) {
          if constexpr (ROLL) {
            if (step) {
              // transition k - 1 ends here: output projection, sampler step; every slice for itself
              const int done = k - 1, i = tid, nblk = H * A / 4;
              int tt = dr.t0[row];
              tt = (tt >= dr.tb.T ? dr.tb.T - 1 : tt) - done + 1;
              float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
              if (i < nblk) z = xi_block(dr.seed, dr.env_id ? dr.env_id[row] : row, tt, i);
              const float sa = dr.tb.sqrt_abar[tt], s1 = dr.tb.sqrt_1m[tt], c0 = dr.tb.c0[tt], cx = dr.tb.cx[tt], ce = dr.tb.ce[tt];
              const float sig = dr.sigma_scale[row] * dr.tb.sigma[tt];
              const size_t o_row = ((size_t)dr.row_ptr[row] + done - 1) * (H * A);
              // the latents before the step: complete since the pass after their step (behind its q | k | v)
              const float* yin = (k == 2 ? dr.y : io.y[(k - 1) & 1]) + (size_t)row * (H * A);
              wait(row);
              f32x4 y = f32x4{0, 0, 0, 0};
              if (i < nblk) y = flow_ld<f32x4>(flow_rsrc(yin, H * A * 4), i * 16);
              t.residual(r, C::O_H0, v);
              t.template norm<false>(v, f, a);
              f32x4 e[C::NHF][NB];
              t.product(wh, a, e);
              t.deposit(e);
              t.template items<C::NHF>([&](int, int m, int nb, int it) {
                const f32x4 s = t.template collect<C::NHF>(it);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                  const int c = m * 16 + lg * 4 + j;
                  if (c < A) t.et[(nb * 16 + l16) * A + c] = s[j] + net.head_b[c];
                }
              });
              lds_barrier();
              if (i < nblk) {
                const f32x4 ev = *reinterpret_cast<const f32x4*>(t.et + 4 * i), zv = {z.x, z.y, z.z, z.w};
                f32x4 o;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                  float x0 = (y[j] - s1 * ev[j]) / sa;
                  if (dr.clip) x0 = fminf(fmaxf(x0, -dr.clip_val), dr.clip_val);
                  o[j] = c0 * x0 + cx * y[j] + ce * ev[j] + sig * zv[j];
                }
                *reinterpret_cast<f32x4*>(t.yt + 4 * i) = o;
                if (slice == 0) {
                  *reinterpret_cast<f32x4*>(dr.states + o_row + 4 * i) = y;
                  *reinterpret_cast<f32x4*>(dr.eps_p + o_row + 4 * i) = ev;
                  if (dr.xi) *reinterpret_cast<f32x4*>(dr.xi + o_row + 4 * i) = zv;
                  float* yo = (ends ? dr.y : io.y[k & 1]) + (size_t)row * (H * A);
                  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(flow_u4, o), flow_rsrc(yo, H * A * 4), i * 16, 0, 0);
                  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // complete before this task's q | k | v (barriers between)
                }
              }
              if (ends) {
                flow_clear(r, C::O_H0, C::HB, tid, C::TH);
                t.clear_pass(row, pass - 1);
                lds_barrier();
                continue;
              }
            }
          }
          if (!step) {
            wait(row);                                   // (a barrier: the row before has read its latents)
            const float* xr = io.x + (size_t)row * (H * A);
            for (int i = tid; i < H * A; i += C::TH) t.yt[i] = xr[i];
          }
          lds_barrier();
#pragma unroll
          for (int ks = 0; ks < KW; ++ks)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
              for (int q = 0; q < VQ; ++q) v[ks][nb][q] = pe[ks][nb][q];
          for (int c = 0; c < A; ++c)
#pragma unroll
            for (int ks = 0; ks < KW; ++ks)
#pragma unroll
              for (int q = 0; q < VQ; ++q) {
                const f32x4 tw = *reinterpret_cast<const f32x4*>(t.tokw + c * D + t.col(ks, q));
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                  const float xv = t.yt[(nb * 16 + l16) * A + c];
#pragma unroll
                  for (int j = 0; j < 4; ++j) v[ks][nb][q][j] = fmaf(xv, tw[j], v[ks][nb][q][j]);
                }
              }
#pragma unroll
          for (int ks = 0; ks < KW; ++ks)                // every slice stores its own blocks
#pragma unroll
            for (int q = 0; q < VQ; ++q) {
              const int c = t.col(ks, q), blk = c >> 4;
              if (blk >= slice * FS && blk < (slice + 1) * FS) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) flow_st(r, C::O_E + ((blk * H + nb * 16 + l16) * 16 + (c & 15)) * 4, v[ks][nb][q]);
              }
            }
        } else {
          wait(row);
          t.residual(r, C::O_H0, v);
        }
        t.template norm<true>(v, f, a);
        f32x4 acc[3 * FS][NB];
#pragma unroll
        for (int m = 0; m < 3 * FS; ++m)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            acc[m][nb] = f32x4{0, 0, 0, 0};
#pragma unroll
            for (int ks = 0; ks < KW; ++ks) {
              if (m / FS == 2) TT::mma(a[ks][nb], w[m][ks], acc[m][nb]);   // values tokens x features: stored transposed
              else TT::mma(w[m][ks], a[ks][nb], acc[m][nb]);
            }
          }
        t.deposit(acc);
        t.template items<3 * FS>([&](int j, int m, int nb, int it) {
          const vec4 o = TT::cvt(t.template collect<3 * FS>(it) + bias[j]);
          const int cls = m / FS, blk = slice * FS + m % FS;
          if (cls < 2) flow_st(r, C::O_Q + cls * C::XB + t.foff(blk * 16 + lg * 4, nb), o);
          else flow_st(r, C::O_Q + 2 * C::XB + ((blk * NB + nb) * 64 + lane) * 4 * ES, o);
        });
        if (pass > 0) t.clear_pass(row, pass - 1);
        flow_signal(io, row, kind);
      }
    } else if (kind == 1 || (C::SX > 0 && kind == 3)) {
      // attention of the wavefront's head, then its share of the output projection
      const bool cross = kind == 3;
      vec4 w[FS][CF];
      t.proj_weights(cross ? W.co : W.o, w);
      f32x4 bias[Task::template per_wave<FS>()] = {}, res[Task::template per_wave<FS>()] = {};
      t.own_bias(cross ? W.co_b : W.o_b, bias);
      for (int row = row0; row < rows; row += row_step) {
        if (!drafts(row)) continue;
        const auto r = t.bufs(row, pass);
        frag q[KW][NB];
        f32x4 acc[FS][NB];
        if (C::SX == 0 || !cross) {
          frag kk[KW][NB];
          vec4 vv[CF][NB];
          wait(row);
          flow_poll(io, lane, [&]() {
#pragma unroll
            for (int ks = 0; ks < KW; ++ks)
#pragma unroll
              for (int nb = 0; nb < NB; ++nb) {
                const int o = C::O_Q + ((wave * KW + ks) * NB + nb) * 64 * VW * ES + lane * VW * ES;
                q[ks][nb] = flow_ld<frag>(r, o);
                kk[ks][nb] = flow_ld<frag>(r, o + C::XB);
              }
#pragma unroll
            for (int cf = 0; cf < CF; ++cf)
#pragma unroll
              for (int nb = 0; nb < NB; ++nb)
                vv[cf][nb] = flow_ld<vec4>(r, C::O_Q + 2 * C::XB + (((wave * CF + cf) * NB + nb) * 64 + lane) * 4 * ES);
            t.own_residual(r, layer == 0 ? C::O_E : C::O_H0, res);
          }, q, kk, vv, res);
          t.attend(q, kk, vv, w, acc);
        } else if constexpr (C::SX > 0) {
          constexpr int SF = C::SX / 16;
          const int env = ROLL ? row : (io.row_env ? io.row_env[row] : row);
          const size_t eh = ((size_t)env * net.L + layer) * C::HEADS + wave;
          const bf16x8* kp = net.kc + eh * (SF * KW) * 64 + lane;
          const bf16x4* vp = net.vct + eh * (CF * SF) * 64 + lane;
          frag kk[KW][SF];
          vec4 vv[CF][SF];
#pragma unroll
          for (int ks = 0; ks < KW; ++ks)
#pragma unroll
            for (int kf = 0; kf < SF; ++kf) kk[ks][kf] = kp[(kf * KW + ks) * 64];
#pragma unroll
          for (int cf = 0; cf < CF; ++cf)
#pragma unroll
            for (int kf = 0; kf < SF; ++kf) vv[cf][kf] = vp[(cf * SF + kf) * 64];
          wait(row);
          flow_poll(io, lane, [&]() {
#pragma unroll
            for (int ks = 0; ks < KW; ++ks)
#pragma unroll
              for (int nb = 0; nb < NB; ++nb) q[ks][nb] = flow_ld<frag>(r, C::O_XQ + (((wave * KW + ks) * NB + nb) * 64 + lane) * VW * ES);
            t.own_residual(r, C::O_H1, res);
          }, q, res);
          t.attend(q, kk, vv, w, acc);
        }
        t.deposit(acc);
        t.add_residual(r, cross ? C::O_H2 : C::O_H1, res, bias);
        flow_signal(io, row, kind);
      }
    } else if (C::SX > 0 && kind == 2) {
      if constexpr (C::SX > 0) {
        frag w[FS][KW];
        int fr[FS];
#pragma unroll
        for (int m = 0; m < FS; ++m) fr[m] = slice * FS + m;
        t.weights(w, W.cq, KD, fr, wave * KW);
        f32x4 bias[Task::template per_wave<FS>()];
        t.own_bias(W.cq_b, bias);
        for (int row = row0; row < rows; row += row_step) {
          if (!drafts(row)) continue;
          const auto r = t.bufs(row, pass);
          FlowV<C> v;
          frag a[KW][NB];
          f32x4 acc[FS][NB];
          typename Task::Film f;
          wait(row);
          t.residual(r, C::O_H1, v);
          t.template norm<false>(v, f, a);
          t.product(w, a, acc);
          t.deposit(acc);
          t.template items<FS>([&](int j, int m, int nb, int it) {
            flow_st(r, C::O_XQ + t.foff((slice * FS + m) * 16 + lg * 4, nb), TT::cvt(t.template collect<FS>(it) + bias[j]));
          });
          t.clear_residual(r, C::O_H0);
          if (layer == 0) t.clear_residual(r, C::O_E);
          t.clear_act(r, C::O_Q, 3);
          flow_signal(io, row, kind);
        }
      }
    } else if (kind == 4) {
      frag w[4 * FS][KW];
      int fr[4 * FS];
#pragma unroll
      for (int m = 0; m < 4 * FS; ++m) fr[m] = slice * 4 * FS + m;
      t.weights(w, W.up, KD, fr, wave * KW);
      f32x4 bias[Task::template per_wave<4 * FS>()];
      t.template items<4 * FS>([&](int j, int m, int, int) { bias[j] = *reinterpret_cast<const f32x4*>(W.up_b + fr[m] * 16 + lg * 4); });
      for (int row = row0; row < rows; row += row_step) {
        if (!drafts(row)) continue;
        typename Task::Film f;
        t.film(f, mod_row(row) + 2 * D);
        const auto r = t.bufs(row, pass);
        FlowV<C> v;
        frag a[KW][NB];
        f32x4 acc[4 * FS][NB];
        wait(row);
        t.residual(r, C::O_H2, v);
        t.template norm<true>(v, f, a);
        t.product(w, a, acc);
        t.deposit(acc);
        t.template items<4 * FS>([&](int j, int m, int nb, int it) {
          f32x4 s = t.template collect<4 * FS>(it) + bias[j];
#pragma unroll
          for (int i = 0; i < 4; ++i) s[i] = gelu_fast(s[i]);
          flow_st(r, C::O_U + t.foff(fr[m] * 16 + lg * 4, nb), TT::cvt(s));
        });
        if constexpr (C::SX > 0) {
          t.clear_residual(r, C::O_H1);
          t.clear_act(r, C::O_XQ, 1);
        } else {
          t.clear_residual(r, C::O_H0);
          if (layer == 0) t.clear_residual(r, C::O_E);
          t.clear_act(r, C::O_Q, 3);
        }
        flow_signal(io, row, kind);
      }
    } else if (kind == 5) {
      frag w[FS][KWM];
      int fr[FS];
#pragma unroll
      for (int m = 0; m < FS; ++m) fr[m] = slice * FS + m;
      t.weights(w, W.dn, 4 * KD, fr, wave * KWM);
      f32x4 bias[Task::template per_wave<FS>()] = {}, res[Task::template per_wave<FS>()] = {};
      t.own_bias(W.dn_b, bias);
      for (int row = row0; row < rows; row += row_step) {
        if (!drafts(row)) continue;
        const auto r = t.bufs(row, pass);
        frag a[KWM][NB];
        f32x4 acc[FS][NB];
        wait(row);
        flow_sample<KWM * NB, 64 * VW * ES>(io, r, C::O_U + wave * KWM * NB * 64 * VW * ES, lane);
        flow_poll(io, lane, [&]() {
#pragma unroll
          for (int ks = 0; ks < KWM; ++ks)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) a[ks][nb] = flow_ld<frag>(r, C::O_U + (((wave * KWM + ks) * NB + nb) * 64 + lane) * VW * ES);
          t.own_residual(r, C::O_H2, res);
        }, a, res);
        t.product(w, a, acc);
        t.deposit(acc);
        t.add_residual(t.bufs(row, pass + 1), C::O_H0, res, bias);
        flow_signal(io, row, kind);
      }
    } else if (!ROLL) {                                  // behind the last layer: output head, buffers emptied
      frag w[C::NHF][KW];
      int hr[C::NHF];
#pragma unroll
      for (int i = 0; i < C::NHF; ++i) hr[i] = min(i, (A + 15) / 16 - 1);
      if (slice == 0) t.weights(w, net.head, KD, hr, wave * KW);
      for (int row = row0; row < rows; row += row_step) {
        if (slice != 0) {
          flow_guard(io, row, 5, pass * G, wave, lane);
          t.clear_pass(row, pass - 1);
          continue;
        }
        const auto r = t.bufs(row, pass);
        FlowV<C> v;
        frag a[KW][NB];
        f32x4 e[C::NHF][NB];
        typename Task::Film f;
        wait(row);
        t.residual(r, C::O_H0, v);
        t.template norm<false>(v, f, a);
        t.product(w, a, e);
        t.deposit(e);
        float* out = io.eps_out + (size_t)row * (H * A);
        t.template items<C::NHF>([&](int, int m, int nb, int it) {
          const f32x4 s = t.template collect<C::NHF>(it);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int c = m * 16 + lg * 4 + j;
            if (c < A) out[(nb * 16 + l16) * A + c] = s[j] + net.head_b[c];
          }
        });
        flow_clear(r, C::O_H0, C::HB, tid, C::TH);
        t.clear_pass(row, pass - 1);
      }
    }
  }
}

}  // namespace tsdp
