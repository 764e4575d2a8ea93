// Forward pass of a few rows, spread over the chip: two launches per layer (three with cross-attention) instead of one
// workgroup that carries a row through all layers.
//
//   k_few_attn   one workgroup per (row, head): residual, LayerNorm + FiLM, the head's q | k | v, attention, and the
//                head's share of the output projection
//   k_few_cross  the same for the cross-attention block (fused bf16 networks with observation tokens)
//   k_few_mlp    one workgroup per (row, slice of the hidden layer): residual, LayerNorm + FiLM, up, GELU, down
//   k_few_head   one workgroup per row: residual, LayerNorm, output projection
//   k_few_out    wide rows only: output / down projection of a row, 64 features per workgroup
//
// A workgroup leaves its share of the block's output as an fp32 partial sum [slice][row][token][D]; the next launch
// starts by adding the shares of all slices (in slice order: the result does not depend on timing) to the residual
// stream, which slice 0 writes back.  Launch boundaries are the only synchronisation.
// Wide rows (64 KB of residual: 32 tokens x 512): eight such sums per workgroup would be 576 KB of reading, twice its
// weights; there the attention output / hidden activations themselves go to memory (bf16, as the product reads them) and
// k_few_out contracts them over their whole width: twice the launches, an eighth of the traffic.
//
// What bounds it: with R rows the one-workgroup-per-tile kernels keep R / rows-per-tile compute units busy, each of
// which streams every weight of the network (or, fp32, multiplies at one unit's matrix rate).  Here a launch has
// R x heads or R x slices workgroups that read each weight once per row, request their weights right behind the residual
// and its partial sums, before the first of these is used, and do a few microseconds of work; the rest is the launch itself.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "fused_mfma.hpp"
#include "kernels_f32.hpp"

namespace tsdp {

// Compile-time sizes of a network; NCH slices of the MLP's hidden layer.  Four wavefronts, one per SIMD, whose up to 512
// registers hold weights in flight; eight for wide rows.
// Slices: one unit's fp32 matrix rate bounds a slice of d = 256 (16 slices of 64 instead of 8 of 128: round of one C2
// environment 402 -> 389 us), in bf16 the sums that the next launch reads do (4 instead of 8: 128 rows 172 instead of 232 us).
constexpr int FEW_WIDE = 16384;                   // numbers of a wide row's residual
template <class TT, int D, int H>
constexpr int few_slices() { return D * H >= FEW_WIDE ? 8 : sizeof(typename TT::elem) == 2 ? 4 : D >= 256 ? 16 : 8; }

template <class TT_, int D_, int H_, int HEADS_, int SX_ = 0, int NCH_ = few_slices<TT_, D_, H_>()>
struct FewCfg {
  typedef TT_ TT;
  static constexpr bool DYN = false;
  static constexpr int D = D_, H = H_, HEADS = HEADS_, SX = SX_, NCH = NCH_, DH = D / HEADS, CH = 4 * D / NCH, NB = H / 16;
  static constexpr bool WIDE = D * H >= FEW_WIDE;
  static constexpr int NW = WIDE ? 8 : 4, TH = NW * 64;
  static constexpr int NPA = WIDE ? 0 : HEADS, NPM = WIDE ? 0 : NCH;   // partial sums an attention / MLP block leaves
  static constexpr int JV = (D / 4 + 63) / 64;    // 16-byte vectors per lane and token
  // MLP workgroups of a unit: two where they fit (136 rows are 544 of them; d = 256 in bf16 with 264 registers 435 us a round, 256 425)
  static constexpr int MLP_WGS = sizeof(typename TT::elem) == 2 && H == 16 && D <= 256 ? 2 : 1;
  static_assert(D % 32 == 0 && H % 16 == 0 && CH % TT_::KSTEP == 0 && CH % 16 == 0 && DH % TT_::KSTEP == 0, "shape");
};

// Run-time sizes (fp32, with the exact functions of the operator kernels): any D, head width and hidden width that are
// multiples of 16; H = 16 NB.
template <int NB_>
struct FewDyn {
  typedef TF32 TT;
  static constexpr bool DYN = true, WIDE = false;
  static constexpr int D = 0, H = NB_ * 16, HEADS = 0, SX = 0, NCH = 0, DH = 0, CH = 0, NB = NB_, JV = 4, NW = 4, TH = 256, MLP_WGS = 1;
  static constexpr int NPA = 1, NPM = 1;           // (the number is in FewIO)
};

struct FewIO {
  int by_row;
  int R_cap, safe_rows;          // rows below safe_rows start loading before the live row count is known
  const int32_t* word; int roll;   // roll = 0: the live row count; 1: K_eff of every environment
  // residual stream: h_in + bias_in + sum of n_part partial sums, part_in + i * pstride
  const float* h_in; const float* part_in; const float* bias_in; float* h_out;
  float* part_out; size_t pstride; int n_part;
  // FiLM pair of this block (gamma at +0, beta at +D), per row or per timestep
  const float* mod; int mod_stride, by_t; const int32_t* row_t; int t_sub, T;
  const int32_t* row_env;
  const void* w1; const float* b1; const void* w2;   // projection in (q|k|v, q or up) and out (o or down)
  // embedding of the first layer; output projection of the last
  const float* x; const float* tok_wt; const float* tok_b; const float* pos; int A;
  const void* head; const float* head_b; float* eps_out;
  const bf16x8* kc; const bf16x4* vct; int layer, L;
  int rms;
  int D, DH, heads, M, CH;       // sizes (run-time configuration only)
  int step;                      // rollout: the drafted transition of this launch (rows are environments)
  const float* y_in; float* y_out;
};

// Workgroup -> (slice, row).  Consecutive workgroups go to the eight XCDs in turn.
__device__ __forceinline__ void few_place(const FewIO& io, int slices, int& slice, int& row) {
  const int i = blockIdx.x;
  if (io.by_row) { row = i / (8 * slices) * 8 + i % 8; slice = i / 8 % slices; }
  else { row = i / slices; slice = i % slices; }
}

// What the launch knows of its row: rows of the ragged batch exist below the live row count, environments of a rollout
// while they still draft.  (Straight-line: the two scalar loads travel together with everything else the row needs.)
struct FewRow { bool live; int t; int k_eff; };
__device__ __forceinline__ FewRow few_row(const FewIO& io, int row) {
  const int r = min(row, io.R_cap - 1);
  const int w = io.word[r * io.roll], t = io.row_t[r];
  FewRow f;
  f.live = row < io.R_cap && (io.roll ? w >= io.step : row < w);
  f.t = t; f.k_eff = row < io.R_cap ? w : -1;
  return f;
}

// sums over lanes without LDS: neighbours inside 16 lanes by DPP, rows of 16 and halves of 32 by lane swaps
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
  return x + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
// every lane receives the sum over its group of N consecutive lanes (8 <= N <= 64)
template <int N>
__device__ __forceinline__ float lane_sum(float x) {
  x = dpp_add<0xB1>(x);                                  // quad_perm 1,0,3,2
  x = dpp_add<0x4E>(x);                                  // quad_perm 2,3,0,1
  x = dpp_add<0x141>(x);                                 // mirror in 8
  if (N >= 16) x = dpp_add<0x140>(x);                    // mirror in 16
  if (N >= 32) x = add_row16(x);
  if (N >= 64) x = add_half32(x);
  return x;
}

template <class C> __device__ __forceinline__ int few_d(const FewIO& io) { return C::DYN ? io.D : C::D; }

// Token-major walk of the row's H x D residual: a wave takes whole tokens, LPT lanes per token with JV vectors each.
template <class C>
struct FewWalk {
  static constexpr bool P2 = !C::DYN && (C::D / 4 & (C::D / 4 - 1)) == 0 && C::D / 4 <= 64;
  static constexpr int LPT = P2 ? C::D / 4 : 64, TPP = 64 / LPT, NPASS = (C::H + C::NW * TPP - 1) / (C::NW * TPP);
  static constexpr bool FULL = !C::DYN && C::D == C::JV * LPT * 4;   // no lane is beyond the feature dimension
  static __device__ __forceinline__ int tok(int pass, int wave, int lane) { return (pass * C::NW + wave) * TPP + lane / LPT; }
  static __device__ __forceinline__ int col(int j, int lane) { return (lane % LPT + j * LPT) * 4; }
};

template <class C>
using FewRes = f32x4[FewWalk<C>::NPASS][C::JV];

// v = residual of the row, NP partial sums and the bias of their projection added (NP = 0: as it is).  after_first() requests the weights.
template <class C, int NP, class F>
__device__ __forceinline__ void few_residual(const FewIO& io, int row, int wave, int lane, FewRes<C>& v, F&& after_first) {
  typedef FewWalk<C> W;
  constexpr int JV = C::JV, NPASS = W::NPASS;
  const int D = few_d<C>(io);
  const size_t base = (size_t)min(row, io.R_cap - 1) * C::H * D;
  int c[JV];
#pragma unroll
  for (int j = 0; j < JV; ++j) c[j] = W::FULL ? W::col(j, lane) : min(W::col(j, lane), D - 4);
  f32x4 bias[JV];
#pragma unroll
  for (int j = 0; j < JV; ++j) bias[j] = NP > 0 ? *reinterpret_cast<const f32x4*>(io.bias_in + c[j]) : f32x4{0, 0, 0, 0};
  if constexpr (!C::DYN) {
    // Batches of passes whose loads (residual and all partial sums) are in flight together, the next batch requested
    // before the current one is added; 36 vectors a lane in all.  The weights are requested behind the last batch: loads
    // complete in order.  (The empty asm keeps the compiler from moving a request down to its first use.)
    constexpr int ALL = NPASS * JV * (NP + 1), PB0 = (ALL <= 36 ? 36 : 18) / (JV * (NP + 1));
    constexpr bool DB = C::NW == 4;                       // (eight wavefronts: the other one's loads fill the gap)
    constexpr int PB = PB0 < 1 ? 1 : (PB0 > NPASS ? NPASS : PB0), NBAT = (NPASS + PB - 1) / PB;
    f32x4 t[NBAT > 1 && DB ? 2 : 1][PB][JV][NP + 1];
    auto request = [&](int bt) {
#pragma unroll
      for (int i = 0; i < PB; ++i) {
        const int tk = min(W::tok(min(bt * PB + i, NPASS - 1), wave, lane), C::H - 1);
#pragma unroll
        for (int j = 0; j < JV; ++j) {
          const size_t o = base + (size_t)tk * D + c[j];
          t[DB ? bt & 1 : 0][i][j][0] = *reinterpret_cast<const f32x4*>(io.h_in + o);
#pragma unroll
          for (int s = 0; s < NP; ++s) t[DB ? bt & 1 : 0][i][j][s + 1] = *reinterpret_cast<const f32x4*>(io.part_in + s * io.pstride + o);
        }
      }
      if (bt == NBAT - 1) after_first();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    };
    if (DB) request(0);
#pragma unroll
    for (int bt = 0; bt < NBAT; ++bt) {
      if (!DB) request(bt);
      else if (bt + 1 < NBAT) request(bt + 1);
#pragma unroll
      for (int i = 0; i < PB; ++i)
#pragma unroll
        for (int j = 0; j < JV; ++j) {
          f32x4 a = t[DB ? bt & 1 : 0][i][j][0];
#pragma unroll
          for (int s = 0; s < NP; ++s) a += t[DB ? bt & 1 : 0][i][j][s + 1];
          if (bt * PB + i < NPASS) v[bt * PB + i][j] = NP > 0 ? a + bias[j] : a;
        }
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
    after_first();
#pragma unroll
    for (int p = 0; p < NPASS; ++p) {
      const int tk = min(W::tok(p, wave, lane), C::H - 1);
#pragma unroll
      for (int j = 0; j < JV; ++j) {
        if (j * 256 >= D) break;
        v[p][j] = *reinterpret_cast<const f32x4*>(io.h_in + base + (size_t)tk * D + c[j]);
      }
    }
    for (int s0 = 0; s0 < io.n_part; s0 += 4) {           // four partial sums of every token in flight
#pragma unroll
      for (int p = 0; p < NPASS; ++p) {
        const int tk = min(W::tok(p, wave, lane), C::H - 1);
#pragma unroll
        for (int j = 0; j < JV; ++j) {
          if (j * 256 >= D) break;
          f32x4 t[4];
#pragma unroll
          for (int s = 0; s < 4; ++s)
            t[s] = *reinterpret_cast<const f32x4*>(io.part_in + min(s0 + s, io.n_part - 1) * io.pstride + base + (size_t)tk * D + c[j]);
#pragma unroll
          for (int s = 0; s < 4; ++s) if (s0 + s < io.n_part) v[p][j] += t[s];
        }
      }
    }
#pragma unroll
    for (int p = 0; p < NPASS; ++p)
#pragma unroll
      for (int j = 0; j < JV; ++j) {
        if (j * 256 >= D) break;
        v[p][j] += bias[j];
      }
  }
}

// v = token embedding of the row's latent xr [H, A] in LDS: tok_w x + tok_b + pos; io.tok_wt is tok_w as [A][D]
template <class C>
__device__ __forceinline__ void few_embed(const FewIO& io, const float* xr, int wave, int lane, FewRes<C>& v) {
  typedef FewWalk<C> W;
  const int D = few_d<C>(io), A = io.A;
#pragma unroll
  for (int j = 0; j < C::JV; ++j) {
    if (C::DYN && j * 256 >= D) break;
    const int c = W::FULL ? W::col(j, lane) : min(W::col(j, lane), D - 4);
    const f32x4 tb = *reinterpret_cast<const f32x4*>(io.tok_b + c);
#pragma unroll
    for (int p = 0; p < W::NPASS; ++p) {
      const int tk = min(W::tok(p, wave, lane), C::H - 1);
      v[p][j] = tb + *reinterpret_cast<const f32x4*>(io.pos + (size_t)tk * D + c);
    }
    for (int a0 = 0; a0 < A; a0 += 8) {
      f32x4 w[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) w[u] = *reinterpret_cast<const f32x4*>(io.tok_wt + (size_t)min(a0 + u, A - 1) * D + c);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (a0 + u < A) {
#pragma unroll
          for (int p = 0; p < W::NPASS; ++p) {
            const float xv = xr[min(W::tok(p, wave, lane), C::H - 1) * A + a0 + u];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[p][j][i] = fmaf(xv, w[u][i], v[p][j][i]);
          }
        }
      }
    }
  }
}

// The lanes' share of a FiLM pair; requested before the weights (loads complete in order).
template <class C>
struct FewFilm {
  f32x4 g[C::JV], b[C::JV];
  __device__ __forceinline__ void none() {
#pragma unroll
    for (int j = 0; j < C::JV; ++j) { g[j] = f32x4{0, 0, 0, 0}; b[j] = f32x4{0, 0, 0, 0}; }
  }
  // (rows beyond the live ones hold any timestep: it is clamped before the table is read)
  __device__ __forceinline__ void load(const FewIO& io, int row, int t, int lane) {
    typedef FewWalk<C> W;
    const int D = few_d<C>(io);
    t = max(min(t, io.T - 1) - io.t_sub, 0);
    const int r = io.by_t ? t : min(row, io.R_cap - 1);
    const float* mp = io.mod + (size_t)r * io.mod_stride;
#pragma unroll
    for (int j = 0; j < C::JV; ++j) {
      if (C::DYN && j * 256 >= D) break;
      const int c = W::FULL ? W::col(j, lane) : min(W::col(j, lane), D - 4);
      g[j] = *reinterpret_cast<const f32x4*>(mp + c); b[j] = *reinterpret_cast<const f32x4*>(mp + D + c);
    }
  }
};

// act[token][D] = LN(v) (1 + gamma) + beta.  Statistics of a token stay inside the lanes that hold it (two passes:
// mean, then squared deviations).
template <class C>
__device__ __forceinline__ void few_norm(const FewIO& io, const FewFilm<C>& fm, int wave, int lane, const FewRes<C>& v,
                                         typename C::TT::elem* act, int stride) {
  typedef FewWalk<C> W;
  typedef typename C::TT TT;
  constexpr int JV = C::JV;
  const int D = few_d<C>(io);
  const float rD = 1.0f / (float)D;
  float mean[W::NPASS], rstd[W::NPASS];
#pragma unroll
  for (int p = 0; p < W::NPASS; ++p) {
    float s = 0.0f;
#pragma unroll
    for (int j = 0; j < JV; ++j) {
      if (C::DYN && j * 256 >= D) break;
      if (W::FULL || W::col(j, lane) < D) s += (v[p][j][0] + v[p][j][1]) + (v[p][j][2] + v[p][j][3]);
    }
    mean[p] = s;
  }
#pragma unroll
  for (int p = 0; p < W::NPASS; ++p) mean[p] = lane_sum<W::LPT>(mean[p]);
#pragma unroll
  for (int p = 0; p < W::NPASS; ++p) {
    mean[p] = io.rms ? 0.0f : mean[p] * rD;              // RMSNorm: no centring
    float q = 0.0f;
#pragma unroll
    for (int j = 0; j < JV; ++j) {
      if (C::DYN && j * 256 >= D) break;
      if (W::FULL || W::col(j, lane) < D) {
#pragma unroll
        for (int i = 0; i < 4; ++i) { const float dv = v[p][j][i] - mean[p]; q = fmaf(dv, dv, q); }
      }
    }
    rstd[p] = q;
  }
#pragma unroll
  for (int p = 0; p < W::NPASS; ++p) rstd[p] = lane_sum<W::LPT>(rstd[p]);
#pragma unroll
  for (int p = 0; p < W::NPASS; ++p) {
    const float rs = C::DYN ? 1.0f / sqrtf(rstd[p] * rD + 1e-5f) : rsqrtf(rstd[p] * rD + 1e-5f);
    const int tk = W::tok(p, wave, lane);
#pragma unroll
    for (int j = 0; j < JV; ++j) {
      if (C::DYN && j * 256 >= D) break;
      const int c = W::col(j, lane);
      if ((C::NW * W::TPP * W::NPASS == C::H || tk < C::H) && (W::FULL || c < D)) {
        f32x4 y = (v[p][j] - mean[p]) * rs;
        y = y * (1.0f + fm.g[j]) + fm.b[j];
        *reinterpret_cast<typename TT::vec4*>(act + tk * stride + c) = TT::cvt(y);
      }
    }
  }
}

template <class C>
__device__ __forceinline__ void few_store_residual(const FewIO& io, int row, int wave, int lane, const FewRes<C>& v) {
  typedef FewWalk<C> W;
  const int D = few_d<C>(io);
#pragma unroll
  for (int p = 0; p < W::NPASS; ++p) {
    const int tk = W::tok(p, wave, lane);
#pragma unroll
    for (int j = 0; j < C::JV; ++j) {
      const int c = W::col(j, lane);
      if ((C::NW * W::TPP * W::NPASS == C::H || tk < C::H) && (W::FULL || c < D))
        *reinterpret_cast<f32x4*>(io.h_out + ((size_t)row * C::H + tk) * D + c) = v[p][j];
    }
  }
}

// One product of a workgroup: MF fragment rows dealt to the waves round-robin, contraction over NKS k-steps of a matrix
// with ks_total.  begin() requests weights (compile-time sizes), run() multiplies and
// hands every finished fragment row to epi(index, accumulators).
template <class C, int MF, int NKS>
struct FewGemm {
  typedef typename C::TT TT;
  static constexpr int MB = (MF + C::NW - 1) / C::NW;
  static_assert(MF % C::NW == 0 || MB <= 2, "at most the last fragment of a wave may be missing");
  // Fragments of weights that a wavefront requests ahead.  A unit takes 16 cycles for each, and a wavefront does nothing else until
  // its requests are issued: with 40 the four held up the normalisation for 2500 cycles; too few, and the product waits.  us with 40,
  // 20, 12, 9, 6, 4: fp32 verify of 128 rows of d = 256 503, 495, 471, 455, 450, 452; bf16 128 rows 179, 173, 171, 173, 171, 169, 64 rows
  // 124, 124, 120, 121, 127, 130, a plain chain of eight (few workgroups a unit) 12 230, 12 240, 11 885, 12 050, 12 620, 12 920.
  static constexpr int AHEAD = C::NW == 8 ? 20 : std::is_same<TT, TF32>::value ? 8 : 12;
  static constexpr int DEEP0 = AHEAD / MB, DEEP = DEEP0 < 1 ? 1 : DEEP0;
  typedef FragGemm<TT, MB, C::NB, NKS, 2, DEEP> G;
  G g;
  f32x4 bias[MB];
  // requested ahead of the weights: in the epilogue nothing covers its way through the L2 (with k_few_out's residual: rounds of
  // four C4 environments 857 -> 840 us (846 -> 765 with the weights in the Infinity Cache), eight C2 448 -> 424, a plain chain of eight
  // C3 13.05 -> 12.37 ms)
  __device__ __forceinline__ void with_bias(const float* b, int wave, int lane) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) bias[mb] = *reinterpret_cast<const f32x4*>(b + min(wave + mb * C::NW, MF - 1) * 16 + (lane >> 4) * 4);
  }
  __device__ __forceinline__ void begin(const void* w, int ks_total, int mf0, int ks0, int wave, int lane) {
    // a wave without a last fragment repeats its first one (its result is dropped): every load stays inside the slice
    g.prime_begin(w, ks_total, mf0 + min(wave, MF - 1), ks0, lane, wave + (MB - 1) * C::NW < MF ? C::NW : 0);
#pragma unroll
    for (int p = 0; p < G::PF; ++p) g.prime_stage(p);
    asm volatile("" ::: "memory");
  }
  template <bool BIAS = false, class E>
  __device__ __forceinline__ void run(const typename TT::elem* act, int stride, int wave, int lane, E&& epi) {
    f32x4 acc[MB][C::NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < C::NB; ++nb) acc[mb][nb] = f32x4{0, 0, 0, 0};
    g.run(act, stride, acc, lane, NoSide{}, std::integral_constant<int, G::PF>{});
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int f = wave + mb * C::NW;
      if (BIAS) {
#pragma unroll
        for (int nb = 0; nb < C::NB; ++nb) acc[mb][nb] += bias[mb];
      }
      if (MF % C::NW == 0 || f < MF) epi(f, acc[mb]);
    }
  }
};

// run-time sizes: one fragment row at a time, eight k-steps of weights in flight
template <int NB, class E>
__device__ __forceinline__ void few_gemm_dyn(const void* w, int ks_total, int mf0, int MF, int ks0, int KS, const float* act,
                                             int stride, int wave, int lane, E&& epi) {
  const float* al = act + (lane & 15) * stride + (lane >> 4) * 4;
  for (int f = wave; f < MF; f += 4) {
    const f32x4* wl = reinterpret_cast<const f32x4*>(w) + ((size_t)(mf0 + f) * ks_total + ks0) * 64 + lane;
    f32x4 acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = f32x4{0, 0, 0, 0};
    for (int k0 = 0; k0 < KS; k0 += 8) {
      f32x4 a[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) a[u] = wl[(size_t)min(k0 + u, KS - 1) * 64];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (k0 + u < KS) {
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
            TF32::mma(a[u], *reinterpret_cast<const f32x4*>(al + nb * 16 * stride + (k0 + u) * 16), acc[nb]);
        }
    }
    epi(f, acc);
  }
}

// a workgroup's share of the block's output: fragment row f of slice `slice`
template <class C>
__device__ __forceinline__ void few_store_part(const FewIO& io, int slice, int row, int f, int lane, const f32x4 (&acc)[C::NB]) {
  const int D = few_d<C>(io);
  float* o = io.part_out + slice * io.pstride + ((size_t)row * C::H + (lane & 15)) * D + f * 16 + (lane >> 4) * 4;
#pragma unroll
  for (int nb = 0; nb < C::NB; ++nb) *reinterpret_cast<f32x4*>(o + (size_t)nb * 16 * D) = acc[nb];
}

// wide rows: four neighbouring activations of a token, [row][token][width] in operand precision
template <class C>
__device__ __forceinline__ void few_store_act(const FewIO& io, int row, int tok, int width, int col, typename C::TT::vec4 v) {
  *reinterpret_cast<typename C::TT::vec4*>(reinterpret_cast<typename C::TT::elem*>(io.part_out) +
                                           ((size_t)row * C::H + tok) * width + col) = v;
}

// LDS of the kernels in bytes; DH and CH as the kernel uses them
template <class TT>
constexpr int few_lds_attn(int D, int H, int DH) {
  return (int)sizeof(typename TT::elem) * (H * (D + TT::PAD) + 2 * H * (DH + TT::PAD) + DH * (H + 4));
}
template <class TT>
constexpr int few_lds_mlp(int D, int H, int CH) { return (int)sizeof(typename TT::elem) * (H * (D + TT::PAD) + H * (CH + TT::PAD)); }

// eps of the row's tokens from the normalised activations: one fragment row (16 outputs) a wave, A <= 64
template <class C, class E>
__device__ __forceinline__ void few_head(const FewIO& io, const typename C::TT::elem* act, int AS, int wave, int lane, E&& put) {
  typedef typename C::TT TT;
  constexpr int NB = C::NB;
  const int D = few_d<C>(io), KD = D / TT::KSTEP, lg = lane >> 4, l16 = lane & 15;
  if (wave * 16 >= io.A) return;
  f32x4 e[1][NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) e[0][nb] = f32x4{0, 0, 0, 0};
  if constexpr (!C::DYN) {
    constexpr int NKS = C::D / TT::KSTEP;
    FragGemm<TT, 1, NB, NKS, 2, (NKS < 32 ? NKS : 32)> gh;
    gh.issue(io.head, KD, wave, 0, lane);
    gh.run(act, AS, e, lane);
  } else {
    few_gemm_dyn<NB>(io.head, KD, wave, 1, 0, KD, reinterpret_cast<const float*>(act), AS, 0, lane, [&](int, const f32x4 (&acc)[NB]) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) e[0][nb] = acc[nb];
    });
  }
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int a = wave * 16 + lg * 4 + i;
      if (a < io.A) put((nb * 16 + l16) * io.A + a, e[0][nb][i] + io.head_b[a]);
    }
}

constexpr int FEW_EMBED = -1;
struct FewNone {};
constexpr int FEW_STEP_LDS = 3 * 512 * 4;         // latents (first layer); drafter output, latents and noise (STEP); H A <= 512

// NP: partial sums to add; FEW_EMBED: the row's residual is its token embedding (run-time configuration: any NP > 0 stands
// for the number in FewIO).
// STEP (rollout): the launch first ends the previous transition -- output projection, then the DDPM / DDIM step with
// its noise, whose results slice 0 writes to the transition's row -- and embeds the new latents; every head of the
// environment does this for itself, which costs less than the two launches it replaces.
template <class C, int NP, bool STEP = false>
__global__ __launch_bounds__(C::TH, 1) void k_few_attn(FewIO io, std::conditional_t<STEP, DraftIO, FewNone> dr) {
  typedef typename C::TT TT;
  typedef typename TT::elem elem;
  typedef typename TT::vec4 vec4;
  typedef typename TT::frag frag;
  constexpr int H = C::H, NB = C::NB, KSTEP = TT::KSTEP, VW = TT::VW, VS = H + 4, UNR = C::DYN ? 1 : 8;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int D = few_d<C>(io), DH = C::DYN ? io.DH : C::DH, heads = C::DYN ? io.heads : C::HEADS;
  const int AS = D + TT::PAD, QS = DH + TT::PAD, KD = D / KSTEP, KH = DH / KSTEP;
  elem* act = reinterpret_cast<elem*>(lds);
  elem* q = act + H * AS;
  elem* k = q + H * QS;
  elem* vt = k + H * QS;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, lg = lane >> 4;
  int head, row;
  few_place(io, heads, head, row);
  const FewRow me = few_row(io, row);
  // STEP: transition `done` ends here, if it was drafted at all; below safe_rows the others decide once the first loads
  // are under way
  const int ke = me.k_eff, done = io.step - 1;
  if (STEP ? ke < done || (ke == done && head != 0) : row >= io.safe_rows && !me.live) return;
  constexpr bool ST = !C::DYN;
  typedef FewGemm<C, ST ? 3 * C::DH / 16 : 4, ST ? C::D / KSTEP : 1> GQ;
  typedef FewGemm<C, ST ? C::D / 16 : 4, ST ? C::DH / KSTEP : 1> GO;
  GQ gq;
  const float* bq = io.b1 + head * 3 * DH;
  auto weights = [&]() {
    if constexpr (ST) {
      gq.with_bias(bq, wave, lane);
      gq.begin(io.w1, KD, head * (3 * DH / 16), 0, wave, lane);
    }
  };
  FewRes<C> v;
  FewFilm<C> fm;
  fm.load(io, row, me.t, lane);
  if constexpr (STEP) {
    few_residual<C, NP>(io, row, wave, lane, v, weights);
    FewFilm<C> none;
    none.none();
    few_norm<C>(io, none, wave, lane, v, act, AS);
    const int DE = H * io.A, nblk = DE >> 2;
    float* et = reinterpret_cast<float*>(vt + DH * VS);
    float* yt = et + 512;
    float* zt = yt + 512;
    int t = dr.t0[row];
    t = (t >= dr.tb.T ? dr.tb.T - 1 : t) - done + 1;
    lds_barrier();
    for (int i = (threadIdx.x + C::TH - 64) % C::TH; i < nblk; i += C::TH) {   // beside the product of wave 0
      const float4 z = xi_block(dr.seed, dr.env_id ? dr.env_id[row] : row, t, i);
      *reinterpret_cast<f32x4*>(zt + 4 * i) = f32x4{z.x, z.y, z.z, z.w};
    }
    few_head<C>(io, act, AS, wave, lane, [&](int i, float e) { et[i] = e; });
    lds_barrier();
    const size_t o_row = ((size_t)dr.row_ptr[row] + done - 1) * DE, o_env = (size_t)row * DE;
    const float sa = dr.tb.sqrt_abar[t], s1 = dr.tb.sqrt_1m[t], c0 = dr.tb.c0[t], cx = dr.tb.cx[t], ce = dr.tb.ce[t];
    const float sig = dr.sigma_scale[row] * dr.tb.sigma[t];
    for (int i = threadIdx.x; i < nblk; i += C::TH) {
      const f32x4 y = *reinterpret_cast<const f32x4*>(io.y_in + o_env + 4 * i), e = *reinterpret_cast<const f32x4*>(et + 4 * i),
                  z = *reinterpret_cast<const f32x4*>(zt + 4 * i);
      f32x4 o;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float x0 = (y[j] - s1 * e[j]) / sa;
        if (dr.clip) x0 = fminf(fmaxf(x0, -dr.clip_val), dr.clip_val);
        o[j] = c0 * x0 + cx * y[j] + ce * e[j] + sig * z[j];
      }
      *reinterpret_cast<f32x4*>(yt + 4 * i) = o;
      if (head == 0) {
        *reinterpret_cast<f32x4*>(dr.states + o_row + 4 * i) = y;
        *reinterpret_cast<f32x4*>(dr.eps_p + o_row + 4 * i) = e;
        if (dr.xi) *reinterpret_cast<f32x4*>(dr.xi + o_row + 4 * i) = z;
        *reinterpret_cast<f32x4*>((ke == done ? dr.y : io.y_out) + o_env + 4 * i) = o;
      }
    }
    if (ke == done) return;                              // the environment's last drafted transition
    lds_barrier();
    few_embed<C>(io, yt, wave, lane, v);
  } else if constexpr (NP == FEW_EMBED) {
    float* xt = reinterpret_cast<float*>(vt + DH * VS);
    const float* xr = io.x + (size_t)min(row, io.R_cap - 1) * H * io.A;
    for (int i = threadIdx.x; i < H * io.A; i += C::TH) xt[i] = xr[i];
    weights();
    lds_barrier();
    few_embed<C>(io, xt, wave, lane, v);
  } else {
    few_residual<C, NP>(io, row, wave, lane, v, weights);
  }
  if (!STEP && !me.live) return;
  few_norm<C>(io, fm, wave, lane, v, act, AS);
  if (head == 0 && (NP != 0 || STEP)) few_store_residual<C>(io, row, wave, lane, v);
  lds_barrier();
  auto epi_qkv = [&](int f, const f32x4 (&acc)[NB]) {
    const int lr = f * 16, cls = lr / DH, c0 = lr % DH + lg * 4;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const f32x4 r = C::DYN ? acc[nb] + *reinterpret_cast<const f32x4*>(bq + lr + lg * 4) : acc[nb];
      const int t = nb * 16 + l16;
      if (cls < 2) {
        *reinterpret_cast<vec4*>((cls ? k : q) + t * QS + c0) = TT::cvt(r);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) vt[(c0 + i) * VS + t] = (elem)r[i];
      }
    }
  };
  GO go;
  if constexpr (ST) {
    gq.template run<true>(act, AS, wave, lane, epi_qkv);
    if constexpr (!C::WIDE) go.begin(io.w2, KD, 0, head * KH, wave, lane);   // travels during the attention
  } else {
    few_gemm_dyn<NB>(io.w1, KD, head * (3 * DH / 16), 3 * DH / 16, 0, KD, reinterpret_cast<const float*>(act), AS, wave, lane, epi_qkv);
  }
  lds_barrier();
  if (wave < NB) {                                       // 16 queries a wave; the result replaces them
    elem* qp = q + wave * 16 * QS;
    f32x4 s[NB];
#pragma unroll
    for (int kf = 0; kf < NB; ++kf) s[kf] = f32x4{0, 0, 0, 0};
#pragma unroll UNR
    for (int ks = 0; ks < KH; ++ks) {
      const frag qb = *reinterpret_cast<const frag*>(qp + l16 * QS + ks * KSTEP + lg * VW);
#pragma unroll
      for (int kf = 0; kf < NB; ++kf)
        TT::mma(*reinterpret_cast<const frag*>(k + (kf * 16 + l16) * QS + ks * KSTEP + lg * VW), qb, s[kf]);
    }
    vec4 p[NB];
    softmax_keys<TT, NB, C::DYN>(s, p, DH);
#pragma unroll UNR
    for (int cf = 0; cf < DH / 16; ++cf) {
      f32x4 o = f32x4{0, 0, 0, 0};
#pragma unroll
      for (int kf = 0; kf < NB; ++kf) TT::mma16(*reinterpret_cast<const vec4*>(vt + (cf * 16 + l16) * VS + kf * 16 + lg * 4), p[kf], o);
      if constexpr (C::WIDE) few_store_act<C>(io, row, wave * 16 + l16, D, head * DH + cf * 16 + lg * 4, TT::cvt(o));
      else *reinterpret_cast<vec4*>(qp + l16 * QS + cf * 16 + lg * 4) = TT::cvt(o);
    }
  }
  if constexpr (C::WIDE) return;
  lds_barrier();
  auto epi_o = [&](int f, const f32x4 (&acc)[NB]) { few_store_part<C>(io, head, row, f, lane, acc); };
  if constexpr (ST) { if constexpr (!C::WIDE) go.run(q, QS, wave, lane, epi_o); }
  else few_gemm_dyn<NB>(io.w2, KD, 0, D / 16, head * KH, KH, reinterpret_cast<const float*>(q), QS, wave, lane, epi_o);
}

// Cross-attention over the row's SX observation tokens: keys and transposed values arrive in fragment order.
template <class C, int NP>
__global__ __launch_bounds__(C::TH, 1) void k_few_cross(FewIO io) {
  typedef typename C::TT TT;
  constexpr int H = C::H, NB = C::NB, D = C::D, DH = C::DH, HEADS = C::HEADS, AS = D + TT::PAD, QS = DH + TT::PAD, KD = D / 32,
                KH = DH / 32, SF = C::SX / 16, CF = DH / 16;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  __bf16* act = reinterpret_cast<__bf16*>(lds);
  __bf16* q = act + H * AS;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, lg = lane >> 4;
  int head, row;
  few_place(io, HEADS, head, row);
  const FewRow me = few_row(io, row);
  if (row >= io.safe_rows && !me.live) return;           // (below that: decided once the first loads are under way)
  FewGemm<C, DH / 16, KD> gq;
  FewGemm<C, D / 16, KH> go;
  FewRes<C> v;
  few_residual<C, NP>(io, row, wave, lane, v, [&]() {
    gq.with_bias(io.b1 + head * DH, wave, lane);
    gq.begin(io.w1, KD, head * (DH / 16), 0, wave, lane);
  });
  if (!me.live) return;
  FewFilm<C> fm;
  fm.none();
  few_norm<C>(io, fm, wave, lane, v, act, AS);
  if (head == 0 && NP != 0) few_store_residual<C>(io, row, wave, lane, v);
  __builtin_amdgcn_sched_barrier(0);                     // (their registers are those of the residual)
  bf16x8 ka[KH][SF];
  bf16x4 va[CF][SF];
  if (wave < NB) {
    const size_t eh = ((size_t)(io.row_env ? io.row_env[row] : row) * io.L + io.layer) * HEADS + head;
    const bf16x8* kp = io.kc + eh * (SF * KH) * 64 + lane;
    const bf16x4* vp = io.vct + eh * (CF * SF) * 64 + lane;
#pragma unroll
    for (int kf = 0; kf < SF; ++kf)
#pragma unroll
      for (int ks = 0; ks < KH; ++ks) ka[ks][kf] = kp[(kf * KH + ks) * 64];
#pragma unroll
    for (int cf = 0; cf < CF; ++cf)
#pragma unroll
      for (int kf = 0; kf < SF; ++kf) va[cf][kf] = vp[(cf * SF + kf) * 64];
  }
  lds_barrier();
  gq.template run<true>(act, AS, wave, lane, [&](int f, const f32x4 (&acc)[NB]) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      *reinterpret_cast<bf16x4*>(q + (nb * 16 + l16) * QS + f * 16 + lg * 4) = to_bf16x4(acc[nb]);
  });
  if constexpr (!C::WIDE) go.begin(io.w2, KD, 0, head * KH, wave, lane);
  lds_barrier();
  if (wave < NB) {
    __bf16* qp = q + wave * 16 * QS;
    f32x4 s[SF];
#pragma unroll
    for (int kf = 0; kf < SF; ++kf) s[kf] = f32x4{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < KH; ++ks) {
      const bf16x8 qb = *reinterpret_cast<const bf16x8*>(qp + l16 * QS + ks * 32 + lg * 8);
#pragma unroll
      for (int kf = 0; kf < SF; ++kf) s[kf] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[ks][kf], qb, s[kf], 0, 0, 0);
    }
    bf16x4 p[SF];
    softmax_keys<TBF16, SF>(s, p, DH);
#pragma unroll
    for (int cf = 0; cf < CF; ++cf) {
      f32x4 o = f32x4{0, 0, 0, 0};
#pragma unroll
      for (int kf = 0; kf < SF; ++kf) TBF16::mma16(va[cf][kf], p[kf], o);
      if constexpr (C::WIDE) few_store_act<C>(io, row, wave * 16 + l16, D, head * DH + cf * 16 + lg * 4, to_bf16x4(o));
      else *reinterpret_cast<bf16x4*>(qp + l16 * QS + cf * 16 + lg * 4) = to_bf16x4(o);
    }
  }
  if constexpr (C::WIDE) return;
  lds_barrier();
  if constexpr (!C::WIDE) go.run(q, QS, wave, lane, [&](int f, const f32x4 (&acc)[NB]) { few_store_part<C>(io, head, row, f, lane, acc); });
}

template <class C, int NP>
__global__ __launch_bounds__(C::TH, C::MLP_WGS) void k_few_mlp(FewIO io) {
  typedef typename C::TT TT;
  typedef typename TT::elem elem;
  constexpr int H = C::H, NB = C::NB, KSTEP = TT::KSTEP;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int D = few_d<C>(io), CH = C::DYN ? io.CH : C::CH, M = C::DYN ? io.M : 4 * C::D, NCH = C::DYN ? M / CH : C::NCH;
  const int AS = D + TT::PAD, US = CH + TT::PAD, KD = D / KSTEP, KM = M / KSTEP, KC = CH / KSTEP;
  elem* act = reinterpret_cast<elem*>(lds);
  elem* u = act + H * AS;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, lg = lane >> 4;
  int slice, row;
  few_place(io, NCH, slice, row);
  const FewRow me = few_row(io, row);
  if (row >= io.safe_rows && !me.live) return;           // (below that: decided once the first loads are under way)
  constexpr bool ST = !C::DYN;
  FewGemm<C, ST ? C::CH / 16 : 4, ST ? C::D / KSTEP : 1> gu;
  FewGemm<C, ST ? C::D / 16 : 4, ST ? C::CH / KSTEP : 1> gd;
  FewRes<C> v;
  FewFilm<C> fm;
  fm.load(io, row, me.t, lane);
  few_residual<C, NP>(io, row, wave, lane, v, [&]() {
    if constexpr (ST) {
      gu.with_bias(io.b1 + slice * CH, wave, lane);
      gu.begin(io.w1, KD, slice * (CH / 16), 0, wave, lane);
    }
  });
  if (!me.live) return;
  few_norm<C>(io, fm, wave, lane, v, act, AS);
  if (slice == 0 && NP != 0) few_store_residual<C>(io, row, wave, lane, v);
  lds_barrier();
  auto epi_up = [&](int f, const f32x4 (&acc)[NB]) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      f32x4 r = C::DYN ? acc[nb] + *reinterpret_cast<const f32x4*>(io.b1 + slice * CH + f * 16 + lg * 4) : acc[nb];
#pragma unroll
      for (int i = 0; i < 4; ++i) r[i] = C::DYN ? gelu_tanh_f(r[i]) : gelu_fast(r[i]);
      if constexpr (C::WIDE) few_store_act<C>(io, row, nb * 16 + l16, M, slice * CH + f * 16 + lg * 4, TT::cvt(r));
      else *reinterpret_cast<typename TT::vec4*>(u + (nb * 16 + l16) * US + f * 16 + lg * 4) = TT::cvt(r);
    }
  };
  if constexpr (ST) {
    gu.template run<true>(act, AS, wave, lane, epi_up);
    if constexpr (C::WIDE) return;
    else gd.begin(io.w2, KM, 0, slice * KC, wave, lane);
  } else {
    few_gemm_dyn<NB>(io.w1, KD, slice * (CH / 16), CH / 16, 0, KD, reinterpret_cast<const float*>(act), AS, wave, lane, epi_up);
  }
  lds_barrier();
  auto epi_dn = [&](int f, const f32x4 (&acc)[NB]) { few_store_part<C>(io, slice, row, f, lane, acc); };
  if constexpr (ST) { if constexpr (!C::WIDE) gd.run(u, US, wave, lane, epi_dn); }
  else few_gemm_dyn<NB>(io.w2, KM, 0, D / 16, slice * KC, KC, reinterpret_cast<const float*>(u), US, wave, lane, epi_dn);
}

template <class C, int NP>
__global__ __launch_bounds__(C::TH, 1) void k_few_head(FewIO io) {
  typedef typename C::TT TT;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  typename TT::elem* act = reinterpret_cast<typename TT::elem*>(lds);
  const int AS = few_d<C>(io) + TT::PAD;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), row = blockIdx.x;
  if (row >= *io.word) return;
  FewRes<C> v;
  few_residual<C, NP>(io, row, wave, lane, v, []() {});
  FewFilm<C> fm;
  fm.none();
  few_norm<C>(io, fm, wave, lane, v, act, AS);
  lds_barrier();
  float* out = io.eps_out + (size_t)row * C::H * io.A;
  few_head<C>(io, act, AS, wave, lane, [&](int i, float e) { out[i] = e; });
}

// Wide rows: h += W act + bias for 64 features of a row, act = [row][token][K].  The contraction is split over the eight
// wavefronts, so every weight and every activation is read once per workgroup, straight into registers as MFMA
// operands; the eight sums meet in LDS (in wavefront order).  Bound by its reads: 96 KB (K = 512) or 384 KB (K = 2048).
template <class C, int K>
__global__ __launch_bounds__(C::TH, 1) void k_few_out(FewIO io) {
  typedef typename C::TT TT;
  typedef typename TT::frag frag;
  constexpr int H = C::H, NB = C::NB, D = C::D, SL = D / 64, KS = K / TT::KSTEP, KW = KS / C::NW;
  static_assert(KS % C::NW == 0 && C::TH * 4 % 64 == 0 && H * 64 % (C::TH * 4) == 0, "shape");
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  float* red = reinterpret_cast<float*>(lds);            // [wave][token][64], vectors of a token permuted against bank conflicts
  auto at = [&](int w, int tok, int c) { return red + (w * H + tok) * 64 + ((c >> 2 ^ (tok & 15)) << 2); };
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, lg = lane >> 4;
  int slice, row;
  few_place(io, SL, slice, row);
  const FewRow me = few_row(io, row);
  if (row >= io.safe_rows && !me.live) return;           // (below that: decided once the first loads are under way)
  const frag* wl = reinterpret_cast<const frag*>(io.w2) + ((size_t)slice * 4 * KS + wave * KW) * 64 + lane;
  const int row_in = min(row, io.R_cap - 1);
  const typename TT::elem* al = reinterpret_cast<const typename TT::elem*>(io.part_in) + ((size_t)row_in * H + l16) * K +
                                wave * KW * TT::KSTEP + lg * TT::VW;
  f32x4 acc[4][NB];
#pragma unroll
  for (int mb = 0; mb < 4; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x4{0, 0, 0, 0};
  constexpr int U = KW < 8 ? KW : 8;                     // k-steps in flight
  // the thread's share of the residual and of the bias, requested behind the first operands
  constexpr int NJ = H * 64 / (C::TH * 4);
  f32x4 res[NJ], bias[NJ];
#pragma unroll
  for (int k0 = 0; k0 < KW; k0 += U) {
    frag a[U][4], b[U][NB];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) b[u][nb] = *reinterpret_cast<const frag*>(al + (size_t)nb * 16 * K + (k0 + u) * TT::KSTEP);
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) a[u][mb] = wl[((size_t)mb * KS + k0 + u) * 64];
    }
    if (k0 == 0) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int i = threadIdx.x + j * C::TH;
        res[j] = *reinterpret_cast<const f32x4*>(io.h_in + ((size_t)row_in * H + i / 16) * D + slice * 64 + i % 16 * 4);
        bias[j] = *reinterpret_cast<const f32x4*>(io.bias_in + slice * 64 + i % 16 * 4);
      }
      asm volatile("" ::: "memory");
    }
    __builtin_amdgcn_sched_barrier(0);
    if (k0 == 0 && !me.live) return;
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) TT::mma(a[u][mb], b[u][nb], acc[mb][nb]);
  }
#pragma unroll
  for (int mb = 0; mb < 4; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      *reinterpret_cast<f32x4*>(at(wave, nb * 16 + l16, mb * 16 + lg * 4)) = acc[mb][nb];
  lds_barrier();
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int i = threadIdx.x + j * C::TH, tok = i / 16, c = (i % 16) * 4;
    const size_t o = ((size_t)row * H + tok) * D + slice * 64 + c;
    f32x4 v = res[j] + bias[j];
#pragma unroll
    for (int w = 0; w < C::NW; ++w) v += *reinterpret_cast<const f32x4*>(at(w, tok, c));
    *reinterpret_cast<f32x4*>(io.h_out + o) = v;
  }
}

template <class TT>
__device__ __forceinline__ f32x4 film_silu(f32x4 v) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if constexpr (std::is_same<TT, TF32>::value) v[j] = v[j] / (1.0f + expf(-v[j]));
    else v[j] = silu_fast(v[j]);
  }
  return v;
}

// FiLM vectors of a few rows, all layers at once: mod[r, :] = W_mod SiLU(temb[t_r] + cemb[env_r]) + b_mod.  A workgroup
// takes 16 rows and four fragment rows (64 outputs), so that one row tile already puts L*D/16 workgroups on the chip.
// k_max > 0: the rows are the transitions of a rollout, r = env * k_max + (k - 1) at timestep t_arr[env] - (k - 1).
// gate: 0 = nothing to do (no environment drafts), or null.  DC = 0: run-time D.
template <class TT, int DC>
__global__ __launch_bounds__(256, 1) void k_few_film(const void* __restrict__ modw, const float* __restrict__ modb,
                                                        const float* __restrict__ temb, const float* __restrict__ cemb,
                                                        const int32_t* __restrict__ t_arr, int t_sub,
                                                        const int32_t* __restrict__ env_arr, int k_max, int T, int Drt, int Nm,
                                                        const int32_t* __restrict__ d_R, const int32_t* __restrict__ gate,
                                                        int R_cap, float* __restrict__ mod) {
  typedef typename TT::elem elem;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  elem* sg = reinterpret_cast<elem*>(lds);
  const int D = DC ? DC : Drt, AS = D + TT::PAD, KD = D / TT::KSTEP;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, lg = lane >> 4;
  const int R = d_R ? min(*d_R, R_cap) : R_cap, row0 = blockIdx.y * 16;
  if (row0 >= R || (gate && *gate == 0)) return;
  const int f = min((int)blockIdx.x * 4 + wave, Nm / 16 - 1);   // (a wave past the last fragment row repeats it)
  typedef FragGemm<TT, 1, 1, (DC ? DC / TT::KSTEP : 1), 2, 16> G;
  G g;
  if constexpr (DC > 0) {
    g.prime_begin(modw, KD, f, 0, lane);
#pragma unroll
    for (int p = 0; p < G::PF; ++p) g.prime_stage(p);
  }
  for (int i = threadIdx.x; i < 16 * (D / 4); i += 256) {
    const int r = min(row0 + i / (D / 4), R - 1), c = (i % (D / 4)) * 4;
    int t = k_max ? min(t_arr[r / k_max], T - 1) - r % k_max : t_arr[r] - t_sub;
    t = t < 0 ? 0 : (t >= T ? T - 1 : t);
    f32x4 v = *reinterpret_cast<const f32x4*>(temb + (size_t)t * D + c);
    if (cemb) v += *reinterpret_cast<const f32x4*>(cemb + (size_t)(k_max ? r / k_max : (env_arr ? env_arr[r] : r)) * D + c);
    *reinterpret_cast<typename TT::vec4*>(sg + (i / (D / 4)) * AS + c) = TT::cvt(film_silu<TT>(v));
  }
  lds_barrier();
  f32x4 acc[1][1] = {{f32x4{0, 0, 0, 0}}};
  if constexpr (DC > 0) {
    g.run(sg, AS, acc, lane, NoSide{}, std::integral_constant<int, G::PF>{});
  } else {
    few_gemm_dyn<1>(modw, KD, f, 1, 0, KD, reinterpret_cast<const float*>(sg), AS, 0, lane,
                    [&](int, const f32x4 (&a)[1]) { acc[0][0] = a[0]; });
  }
  if (row0 + l16 < R)
    *reinterpret_cast<f32x4*>(mod + (size_t)(row0 + l16) * Nm + f * 16 + lg * 4) =
        acc[0][0] + *reinterpret_cast<const f32x4*>(modb + f * 16 + lg * 4);
}

}  // namespace tsdp
