// Run-time sizes, a row per workgroup: one launch carries a row through all layers (k_row), or an environment through all
// transitions of its rollout (ROLL), with the residual and every activation in LDS and fp32 operands on the matrix cores; the
// functions are those of the operator kernels.
//
// For networks whose layers are small (row_pays): one unit multiplies such a layer in less time than the two or more launches
// and the partial sums cost that spreading it takes.  256 rows and 32 rollouts of eight transitions (d = 96, two layers, and
// d = 48, one): round 307 -> 132 us.  What bounds it: seven barrier-separated phases a layer of 1000 to 3500 cycles each, of
// which the fp32 matrix rate is about half (a drafted transition of d = 48 8 us).  Eight wavefronts, two per SIMD; a wavefront's
// fragments of a product are one stream whose next block of weights is requested before the current one is multiplied, and whose
// first block is requested before the barrier ahead of the phase.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "fused_mfma.hpp"
#include "few_rows.hpp"
#include "kernels_f32.hpp"

namespace tsdp {

constexpr int ROW_NW = 8, ROW_TH = ROW_NW * 64;               // wavefronts
// fragments of a block; forward passes: 128 registers, two workgroups per unit
template <int NB, bool ROLL> constexpr int row_block() { return (ROLL ? 8 : 4) / NB; }
constexpr int ROW_JV = 2, ROW_MAX_D = ROW_JV * 128;           // 16-byte vectors of a token per lane (32 lanes a token)

constexpr int ROW_MAX_BIAS = 4 * ROW_TH;          // a layer's biases, 5 D + M floats: a vector per thread (row_pays allows 1728)
// LDS in floats: residual, normalised activations / attention output, q | k | v or the hidden layer, biases of a layer,
// drafter output, latents and noise; token embedding and the embedding of an all-zero latent (rollout)
struct RowLds { int h, act, scr, bias, hb, et, tok, total; };
constexpr RowLds row_lds(int D, int H, int M, int A, bool roll) {
  const int S = D + 4, qkv = 2 * H * S + D * (H + 4), u = H * (M + 4), scr = qkv > u ? qkv : u;
  RowLds l{};
  l.h = 0; l.act = H * S; l.scr = 2 * H * S; l.bias = l.scr + scr; l.hb = l.bias + 2 * (5 * D + M); l.et = l.hb + 64; l.tok = l.et + 3 * 512; l.total = l.tok + (roll ? (A + H) * D : 0);
  return l;
}

// i / d for i d < 2^20 by a multiplication (run-time divisors)
struct RowDiv {
  unsigned m;
  explicit RowDiv(unsigned d) : m(((1u << 20) + d - 1) / d) {}
  __device__ __forceinline__ int operator()(int i) const { return (int)((unsigned)i * m >> 20); }
};
struct RowIO {
  RowDiv by_cf, by_3cf, by_vec;  // a head's fragments, those of its q | k | v, 16-byte vectors of a token
  const int32_t* word;           // live row count; rollout: unused
  int R_cap, A, H, dh, k_max;
  const float* x; const float* mod; float* eps_out;
};

// A wavefront's fragments of one product: fragment rows wave, wave + 8, .. of the packed matrix in blocks of U k-steps.  A block's
// loads and LDS reads differ by immediate offsets only (address arithmetic of single fragments cost as much as their products);
// what lies beyond a row is not fetched and not multiplied.
template <int U>
struct RowStream {
  const char* w;
  int KS, MF;
  f32x4 a[U];
  __device__ __forceinline__ void request(f32x4 (&d)[U], int f, int k0, int lane) const {
    const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(w + (size_t)f * KS * 1024), 0, KS * 1024, 0x00020000);
    const int at = k0 * 1024 + lane * 16;
#pragma unroll
    for (int u = 0; u < U; ++u) d[u] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, at + u * 1024, 0, 0));
  }
  __device__ __forceinline__ void begin(const void* p, int rows, int ks, int wave, int lane) {
    w = reinterpret_cast<const char*>(p); KS = ks; MF = rows;
    if (wave < MF) request(a, wave, 0, lane);
    asm volatile("" ::: "memory");
  }
  // act [token][stride]; every finished fragment row f goes to epi(f, accumulators)
  template <int NB, class E>
  __device__ __forceinline__ void run(const float* act, int stride, int wave, int lane, E&& epi) {
    const float* al = act + (lane & 15) * stride + (lane >> 4) * 4;
    // every NC-th k-step adds to a sum of its own: shorter chains of roundings (error of a d = 96 network 4.0e-7 with one sum)
    constexpr int NC = 4 / NB;
    static_assert(U % NC == 0, "the sums do not depend on the block");
    f32x4 acc[NC][NB];
    auto clear = [&]() {
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[c][nb] = f32x4{0, 0, 0, 0};
    };
    clear();
    for (int f = wave, k0 = 0; f < MF;) {
      const bool ends = k0 + U >= KS;
      const int nf = ends ? f + ROW_NW : f, nk = ends ? 0 : k0 + U;
      f32x4 next[U], b[U][NB];
      const bool more = nf < MF;
      if (more) request(next, nf, nk, lane);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const float* bp = al + nb * 16 * stride + k0 * 16;
#pragma unroll
        for (int u = 0; u < U; ++u) b[u][nb] = *reinterpret_cast<const f32x4*>(bp + u * 16);   // (beyond K: other data of the row, unused)
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (u > 0 && k0 + u >= KS) break;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) TF32::mma(a[u], b[u][nb], acc[u % NC][nb]);
      }
      if (ends) {
        f32x4 sum[NB];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) sum[nb] = NC == 4 ? (acc[0][nb] + acc[1][nb]) + (acc[NC - 2][nb] + acc[NC - 1][nb]) : acc[0][nb] + acc[1][nb];
        epi(f, sum);
        clear();
      }
      if (more) {
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = next[u];
      }
      f = nf; k0 = nk;
    }
  }
};

// FiLM pair of a block: a lane's vectors of the 32 lanes that share a token; at = the pair's first byte in the row's vectors
struct RowFilm {
  f32x4 g[ROW_JV], b[ROW_JV];
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t mod, int at, int D, int lane) {
#pragma unroll
    for (int j = 0; j < ROW_JV; ++j) {
      const int c = (lane & 31) * 16 + j * 512;            // (past the pair: other vectors or nothing, unused)
      g[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(mod, c, at, 0));
      b[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(mod, c, at + D * 4, 0));
    }
  }
  __device__ __forceinline__ void none() {
#pragma unroll
    for (int j = 0; j < ROW_JV; ++j) { g[j] = f32x4{0, 0, 0, 0}; b[j] = f32x4{0, 0, 0, 0}; }
  }
};

// act = LN(h) (1 + g) + b, both [token][D + 4]; a token stays inside 32 lanes
template <int H>
__device__ __forceinline__ void row_norm(const float* h, float* act, int D, int rms, const RowFilm& fm, int wave, int lane) {
  constexpr int NP = H / (2 * ROW_NW);
  const int S = D + 4;
  const float rD = 1.0f / (float)D;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int tk = (p * ROW_NW + wave) * 2 + (lane >> 5);
    f32x4 v[ROW_JV];
    float s = 0.0f, q = 0.0f;
#pragma unroll
    for (int j = 0; j < ROW_JV; ++j) {
      const int c = (lane & 31) * 4 + j * 128;
      v[j] = f32x4{0, 0, 0, 0};
      if (c < D) { v[j] = *reinterpret_cast<const f32x4*>(h + tk * S + c); s += (v[j][0] + v[j][1]) + (v[j][2] + v[j][3]); }
    }
    s = lane_sum<32>(s);
    const float mean = rms ? 0.0f : s * rD;
#pragma unroll
    for (int j = 0; j < ROW_JV; ++j) {
      if ((lane & 31) * 4 + j * 128 < D) {
#pragma unroll
        for (int i = 0; i < 4; ++i) { const float d = v[j][i] - mean; q = fmaf(d, d, q); }
      }
    }
    q = lane_sum<32>(q);
    const float rs = 1.0f / sqrtf(q * rD + 1e-5f);
#pragma unroll
    for (int j = 0; j < ROW_JV; ++j) {
      const int c = (lane & 31) * 4 + j * 128;
      if (c < D) *reinterpret_cast<f32x4*>(act + tk * S + c) = (v[j] - mean) * rs * (1.0f + fm.g[j]) + fm.b[j];
    }
  }
}

// One forward pass of the row whose latents are xt [H, A] in LDS; mod: its FiLM vectors, all layers.  put(i, eps) receives
// element i of the prediction.  `idle(wave, lane)` runs on the wavefronts that have no part in the output head.
template <int NB, bool ROLL, class P, class I>
__device__ __forceinline__ void row_pass(const FusedNet& net, const RowIO& io, float* lds, const float* xt, const float* mod, P&& put, I&& idle) {
  constexpr int H = NB * 16, VS = H + 4;
  const int D = net.D, M = net.M, A = io.A, DH = io.dh, S = D + 4, US = M + 4, KD = D / 16, KM = M / 16, KH = DH / 16;
  const RowLds at = row_lds(D, H, M, A, ROLL);
  float* h = lds + at.h;
  float* act = lds + at.act;
  float* q = lds + at.scr;
  float* k = q + H * S;
  float* vt = k + H * S;
  float* u = q;
  float* biases = lds + at.bias;
  const float* tok = lds + at.tok;
  const float* hb = lds + at.hb;
  int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  asm volatile("" : "+v"(lane));
  const int l16 = lane & 15, lg = lane >> 4;

  RowStream<row_block<NB, ROLL>()> st;
  RowFilm fm;
  f32x4 bv;                                              // the next layer's biases: q|k|v, output projection, down, up
  const int NBIAS = 5 * D + M;
  auto load_bias = [&](const FusedLayer& W) {            // (packed behind q | k | v)
    const auto r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(W.qkv_b), 0, NBIAS * 4, 0x00020000);
    bv = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)threadIdx.x * 16, 0, 0));
  };
  auto store_bias = [&](int l) {                         // (two regions: the layer before may still read its own)
    const int i = threadIdx.x * 4;
    if (i < NBIAS) *reinterpret_cast<f32x4*>(biases + (l & 1) * NBIAS + i) = bv;
  };
  const int MROW = net.L * 4 * D * 4;
  const auto mrow = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(mod), 0, MROW, 0x00020000);
  fm.load(mrow, 0, D, lane);
  load_bias(net.layer[0]);
  // embedding: tok_w x + tok_b + pos
  for (int i = threadIdx.x; i < H * (D / 4); i += ROW_TH) {
    const int tk = io.by_vec(i), c = (i - tk * (D / 4)) * 4;
    f32x4 v;
    if constexpr (ROLL) {
      v = *reinterpret_cast<const f32x4*>(tok + A * D + tk * D + c);
      for (int a0 = 0; a0 < A; a0 += 4) {
        f32x4 w[4];
        float xv[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) { const int a = min(a0 + j, A - 1); w[j] = *reinterpret_cast<const f32x4*>(tok + a * D + c); xv[j] = xt[tk * A + a]; }
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (a0 + j < A) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = fmaf(xv[j], w[j][e], v[e]);
          }
      }
    } else {
      v = *reinterpret_cast<const f32x4*>(net.tok_b + c) + *reinterpret_cast<const f32x4*>(net.pos + (size_t)tk * D + c);
      for (int a0 = 0; a0 < A; a0 += 8) {
        f32x4 w[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) w[j] = *reinterpret_cast<const f32x4*>(net.tok_wt + (size_t)min(a0 + j, A - 1) * D + c);
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (a0 + j < A) {
            const float xv = xt[tk * A + a0 + j];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = fmaf(xv, w[j][e], v[e]);
          }
      }
    }
    *reinterpret_cast<f32x4*>(h + tk * S + c) = v;
  }
  store_bias(0);                                         // (before the request: nothing below waits for the weights with it)
  st.begin(net.layer[0].qkv, 3 * KD, KD, wave, lane);
  lds_barrier();
  auto add_to_h = [&](const float* b) {
    return [=](int f, const f32x4 (&acc)[NB]) {
      const int c = f * 16 + lg * 4;
      const f32x4 bv = *reinterpret_cast<const f32x4*>(b + c);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        f32x4* o = reinterpret_cast<f32x4*>(h + (nb * 16 + l16) * S + c);
        *o = *o + (acc[nb] + bv);
      }
    };
  };
  for (int l = 0; l < net.L; ++l) {
    const FusedLayer& W = net.layer[l];
    const float* bias = biases + (l & 1) * NBIAS;
    row_norm<H>(h, act, D, net.rms, fm, wave, lane);
    lds_barrier();
    st.template run<NB>(act, S, wave, lane, [&](int f, const f32x4 (&acc)[NB]) {
      const int head = io.by_3cf(f), in = f - head * 3 * KH, cls = io.by_cf(in), c0 = head * DH + (in - cls * KH) * 16 + lg * 4;
      const f32x4 b = *reinterpret_cast<const f32x4*>(bias + f * 16 + lg * 4);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const f32x4 r = acc[nb] + b;
        const int t = nb * 16 + l16;
        if (cls < 2) {
          *reinterpret_cast<f32x4*>((cls ? k : q) + t * S + c0) = r;
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) vt[(c0 + i) * VS + t] = r[i];
        }
      }
    });
    st.begin(W.o, KD, KD, wave, lane);
    lds_barrier();
    for (int task = wave; task < net.heads * NB; task += ROW_NW) {     // 16 queries of a head
      const int head = task / NB, qf = task % NB;
      const float* qp = q + (qf * 16 + l16) * S + head * DH + lg * 4;
      f32x4 s[NB], p[NB];
#pragma unroll
      for (int kf = 0; kf < NB; ++kf) s[kf] = f32x4{0, 0, 0, 0};
      for (int ks = 0; ks < KH; ++ks) {
        const f32x4 qb = *reinterpret_cast<const f32x4*>(qp + ks * 16);
#pragma unroll
        for (int kf = 0; kf < NB; ++kf)
          TF32::mma(*reinterpret_cast<const f32x4*>(k + (kf * 16 + l16) * S + head * DH + ks * 16 + lg * 4), qb, s[kf]);
      }
      softmax_keys<TF32, NB, true>(s, p, DH);
      for (int cf = 0; cf < KH; ++cf) {
        f32x4 o = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int kf = 0; kf < NB; ++kf) TF32::mma16(*reinterpret_cast<const f32x4*>(vt + (head * DH + cf * 16 + l16) * VS + kf * 16 + lg * 4), p[kf], o);
        *reinterpret_cast<f32x4*>(act + (qf * 16 + l16) * S + head * DH + cf * 16 + lg * 4) = o;
      }
    }
    fm.load(mrow, (l * 4 + 2) * D * 4, D, lane);
    lds_barrier();
    st.template run<NB>(act, S, wave, lane, add_to_h(bias + 3 * D));
    st.begin(W.up, KM, KD, wave, lane);
    lds_barrier();
    row_norm<H>(h, act, D, net.rms, fm, wave, lane);
    lds_barrier();
    st.template run<NB>(act, S, wave, lane, [&](int f, const f32x4 (&acc)[NB]) {
      const int c = f * 16 + lg * 4;
      const f32x4 b = *reinterpret_cast<const f32x4*>(bias + 5 * D + c);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        f32x4 r = acc[nb] + b;
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = gelu_tanh_f(r[i]);   // (gelu_fast: 3.5 of 133 us less, error of the function 4.5e-8 for 3.9e-8)
        *reinterpret_cast<f32x4*>(u + (nb * 16 + l16) * US + c) = r;
      }
    });
    const bool more = l + 1 < net.L;
    const int next = more ? l + 1 : l;
    fm.load(mrow, next * 4 * D * 4, D, lane);            // (unused behind the last layer)
    load_bias(net.layer[next]);
    st.begin(W.dn, KD, KM, wave, lane);
    lds_barrier();
    st.template run<NB>(u, US, wave, lane, add_to_h(bias + 4 * D));
    const int AF = (A + 15) / 16;
    store_bias(l + 1);
    if (more) st.begin(net.layer[l + 1].qkv, 3 * KD, KD, wave, lane);
    else st.begin(net.head, AF, KD, wave, lane);
    lds_barrier();
  }
  fm.none();
  row_norm<H>(h, act, D, net.rms, fm, wave, lane);
  lds_barrier();
  if (wave * 16 >= A) idle(wave, lane);
  st.template run<NB>(act, S, wave, lane, [&](int f, const f32x4 (&acc)[NB]) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int a = f * 16 + lg * 4 + i;
        if (a < A) put((nb * 16 + l16) * A + a, acc[nb][i] + hb[a]);
      }
  });
}

// ROLL: rows are environments; mod holds the FiLM vectors of [env][k_max] transitions
template <int NB, bool ROLL>
__global__ __launch_bounds__(ROW_TH, ROLL ? 2 : 4) void k_row(FusedNet net, RowIO io, std::conditional_t<ROLL, DraftIO, FewNone> dr) {
  constexpr int H = NB * 16;
  extern __shared__ __attribute__((aligned(16))) float row_mem[];
  const int row = blockIdx.x, A = io.A, n = H * A;
  const RowLds at = row_lds(net.D, H, net.M, A, ROLL);
  float* et = row_mem + at.et;
  float* yt = et + 512;
  float* zt = yt + 512;
  const int mod_row = net.L * 4 * net.D;
  if ((int)threadIdx.x < A) row_mem[at.hb + threadIdx.x] = net.head_b[threadIdx.x];
  if constexpr (!ROLL) {
    if (row >= min(*io.word, io.R_cap)) return;
    for (int i = threadIdx.x; i < n; i += ROW_TH) yt[i] = io.x[(size_t)row * n + i];
    lds_barrier();
    float* out = io.eps_out + (size_t)row * n;
    row_pass<NB, ROLL>(net, io, row_mem, yt, io.mod + (size_t)row * mod_row, [&](int i, float e) { out[i] = e; }, [](int, int) {});
  } else {
    const int ke = dr.K_eff[row], nblk = n / 4;
    if (ke == 0) return;
    for (int i = threadIdx.x; i < n; i += ROW_TH) yt[i] = dr.y[(size_t)row * n + i];
    const int D = net.D;
    f32x4* tok = reinterpret_cast<f32x4*>(row_mem + at.tok);
    for (int i = threadIdx.x; i < A * (D / 4); i += ROW_TH) tok[i] = reinterpret_cast<const f32x4*>(net.tok_wt)[i];
    for (int i = threadIdx.x; i < H * (D / 4); i += ROW_TH)
      tok[A * (D / 4) + i] = reinterpret_cast<const f32x4*>(net.tok_b)[i % (D / 4)] + reinterpret_cast<const f32x4*>(net.pos)[i];
    lds_barrier();
    int t = dr.t0[row];
    t = t >= dr.tb.T ? dr.tb.T - 1 : t;
    const int env = dr.env_id ? dr.env_id[row] : row;
    const size_t o_row = (size_t)dr.row_ptr[row] * n;
    const float s = dr.sigma_scale[row];
    for (int k = 0; k < ke; ++k, --t) {
      // the next transition's FiLM vectors are brought into the L2 (another launch left them in memory: 2000 cycles)
      const float touched = io.mod[((size_t)row * io.k_max + min(k + 1, ke - 1)) * mod_row + min((int)threadIdx.x * 32, mod_row - 1)];
      const float sa = dr.tb.sqrt_abar[t], s1 = dr.tb.sqrt_1m[t], c0 = dr.tb.c0[t], cx = dr.tb.cx[t], ce = dr.tb.ce[t], sig = s * dr.tb.sigma[t];
      row_pass<NB, ROLL>(net, io, row_mem, yt, io.mod + ((size_t)row * io.k_max + k) * mod_row, [&](int i, float e) { et[i] = e; },
                   [&](int wave, int lane) {              // A <= 64: at least four wavefronts, 256 lanes for up to 128 blocks of noise
                     const int i = (ROW_NW - 1 - wave) * 64 + lane;
                     if (i < nblk) {
                       const float4 z = xi_block(dr.seed, env, t, i);
                       *reinterpret_cast<f32x4*>(zt + 4 * i) = f32x4{z.x, z.y, z.z, z.w};
                     }
                   });
      asm volatile("" ::"v"(touched));
      lds_barrier();
      const int i = threadIdx.x;
      if (i < nblk) {
        const f32x4 y = *reinterpret_cast<const f32x4*>(yt + 4 * i), e = *reinterpret_cast<const f32x4*>(et + 4 * i),
                    z = *reinterpret_cast<const f32x4*>(zt + 4 * i);
        f32x4 o;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float x0 = (y[j] - s1 * e[j]) / sa;
          if (dr.clip) x0 = fminf(fmaxf(x0, -dr.clip_val), dr.clip_val);
          o[j] = c0 * x0 + cx * y[j] + ce * e[j] + sig * z[j];
        }
        const size_t o_at = o_row + (size_t)k * n + 4 * i;
        *reinterpret_cast<f32x4*>(dr.states + o_at) = y;
        *reinterpret_cast<f32x4*>(dr.eps_p + o_at) = e;
        if (dr.xi) *reinterpret_cast<f32x4*>(dr.xi + o_at) = z;
        *reinterpret_cast<f32x4*>(yt + 4 * i) = o;
      }
      lds_barrier();
    }
    for (int i = threadIdx.x; i < n; i += ROW_TH) dr.y[(size_t)row * n + i] = yt[i];
  }
}

}  // namespace tsdp
