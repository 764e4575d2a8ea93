// Cross-attention keys / values of new observations, for the fused bf16 networks: every layer's K and V projection of
// both networks in one launch, written straight in the fragment order the attention reads.
//
// The sums are k_linear's, bit for bit: fp32 fused multiply-adds over the features in ascending order, then the bias,
// then one rounding to bf16.  mfma_f32_16x16x4_f32 adds its four products to the accumulator one after the other, each
// with one rounding, in the order of the lane groups (checked on hardware, denormals included), so a chain of them over
// ascending features is that sum.  Another order (three bf16 planes per observation: 0.92 ms instead of 2.83) rounds a few
// keys to the other bf16 number, and at the first timesteps of a squared-cosine chain, where a noise prediction is
// multiplied by 31, that is enough for a nearly tied draft to fall on the other side of its test.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "fused_mfma.hpp"

namespace tsdp {

// Conditioning vectors: both networks' embeddings W cond + b in one launch.  A workgroup takes 16 output features and 16
// environments, one thread per number: fp32 fused multiply-adds over the components in ascending order, then the bias --
// k_linear's sum, bit for bit, so an environment's embedding does not depend on which of the two a batch takes.  Weights
// and vectors come through LDS in pieces of 256 components, the next piece travels in registers meanwhile.  Bound in small
// batches by the chain of dependent multiply-adds, in large ones by the LDS (two 16-byte reads per four of them).
// C = 1024, both networks of d = 256 + 128 (384 + 192): 1, 64, 256, 1024 environments 7.7 (7.6), 8.9 (9.0), 13 (18),
// 31 (43) us; k_linear, whose C / 16 barrier steps take the same time for any batch up to 1024, 117 (131) us, so beyond 1024
// environments that one stays.
constexpr int COND_VEC_B = 1024, COND_VEC_C = 256, COND_VEC_S = COND_VEC_C + 4;   // (stride: 16 rows on different banks)
struct CondVecNet { const float* w; const float* b; float* out; int d; };
__global__ __launch_bounds__(256) void k_cond_vec(const float* __restrict__ cond, CondVecNet n0, CondVecNet n1, int B, int C) {
  __shared__ __attribute__((aligned(16))) float ws[16 * COND_VEC_S], xs[16 * COND_VEC_S];
  const int tiles0 = (n0.d + 15) / 16;
  const bool second = (int)blockIdx.x >= tiles0;
  const CondVecNet n = second ? n1 : n0;
  const int f0 = ((int)blockIdx.x - (second ? tiles0 : 0)) * 16, e0 = blockIdx.y * 16;
  const int fl = threadIdx.x & 15, el = threadIdx.x >> 4, f = f0 + fl, e = e0 + el;
  f32x4 rw[4], rx[4];                                   // thread i brings 16 bytes of rows i / 64 + 0, 4, 8, 12
  const int row = threadIdx.x >> 6, col = (threadIdx.x & 63) * 4;
  auto request = [&](int c0) {
    const int c = min(c0 + col, C - 4);                 // (C is a multiple of 4; what lies beyond it is not summed)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      rw[j] = *reinterpret_cast<const f32x4*>(n.w + (size_t)min(f0 + row + 4 * j, n.d - 1) * C + c);
      rx[j] = *reinterpret_cast<const f32x4*>(cond + (size_t)min(e0 + row + 4 * j, B - 1) * C + c);
    }
  };
  float acc = 0.0f;
  request(0);
  for (int c0 = 0; c0 < C; c0 += COND_VEC_C) {
    if (c0) __syncthreads();                            // the piece before has been read
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      *reinterpret_cast<f32x4*>(ws + (row + 4 * j) * COND_VEC_S + col) = rw[j];
      *reinterpret_cast<f32x4*>(xs + (row + 4 * j) * COND_VEC_S + col) = rx[j];
    }
    __syncthreads();
    if (c0 + COND_VEC_C < C) request(c0 + COND_VEC_C);
    if (e0 + (el & ~3) < B) {                           // (a wavefront without an environment only brings data)
      const int nc = min(COND_VEC_C, C - c0);
#pragma unroll 8
      for (int c = 0; c < nc; c += 4) {
        const f32x4 w = *reinterpret_cast<const f32x4*>(ws + fl * COND_VEC_S + c), x = *reinterpret_cast<const f32x4*>(xs + el * COND_VEC_S + c);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = fmaf(x[j], w[j], acc);
      }
    }
  }
  if (e < B && f < n.d) n.out[(size_t)e * n.d + f] = acc + n.b[f];
}

struct CondNet {                 // one network's share of the launch
  const bf16x8* w;               // [L*2*d/16][KS][64] fragments: per layer the key rows, then the value rows
  const float* bias;             // [L*2*d]
  __bf16* kc; __bf16* vct;       // FusedNet::kc / vct
  int L, d, heads, tiles;        // tiles = L*2*d / 256
};
struct CondIO { CondNet net[2]; const float* cond; int M, C, KS, SF; };   // cond [M = B*S, C]

// Tile: 256 features (16 fragments, all keys or all values of one layer because d is a multiple of 256) x 128 tokens
// (8 fragments).  8 waves as 4 x 2, each 64 features x 64 tokens.  Per k-step the workgroup brings 16 KB of weights and
// 16 KB of observations into LDS and does 1024 MFMAs, 8192 cycles of each matrix core: they bound it.  Two LDS buffers,
// the next k-step travels through registers while the current one is multiplied; one barrier per k-step.  Two workgroups
// per CU (128 registers, a few spilled before the loop and read back after it), one multiplies while the other waits at
// its barrier: 2.83 ms instead of 3.04.
// Lane group g supplies features 4m + g of a k-step to MFMA m: the weights are packed in that order (build_fused).
// Keys are computed features x tokens, values tokens x features, so that in both cases a lane's four accumulators are
// the neighbouring entries of one 8-byte piece of the attention operand.
// Measured, 256 environments x 64 tokens x 768, 12 layers of d = 512 and 2 of d = 256: 2.83 ms = 118 TFLOP/s (nominal fp32
// matrix rate 157), against 4.9 ms of fp32 products on the vector units in 28 launches, each followed by two that rounded
// and reordered its output.
constexpr int COND_FF = 16, COND_TF = 8, COND_XS = 36;   // floats per token in LDS: 32 and the bank padding
constexpr int COND_W_B = COND_FF * 64 * 16, COND_STAGE_B = COND_W_B + COND_TF * 16 * COND_XS * 4, COND_LDS = 2 * COND_STAGE_B;

__global__ __launch_bounds__(512, 4) void k_cond_kv(CondIO io) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wf = wave & 3, wt = wave >> 2, l16 = lane & 15, lg = lane >> 4;
  // consecutive workgroups share the feature tile and walk the tokens
  const int MF = io.M / 16, tt = (MF + COND_TF - 1) / COND_TF;
  int ft = blockIdx.x / tt;
  const int tf0 = (blockIdx.x % tt) * COND_TF;
  const int which = ft >= io.net[0].tiles ? 1 : 0;
  const CondNet& n = io.net[which];
  if (which) ft -= io.net[0].tiles;
  const int KS = io.KS;
  // a thread fetches two pieces of weights (fragments 2 wave, 2 wave + 1) and of observations (tokens xr, xr + 64)
  const bf16x8* wsrc = n.w + ((size_t)ft * COND_FF + wave * 2) * KS * 64 + lane;
  const int xr = threadIdx.x >> 3, xc = (threadIdx.x & 7) * 4;
  const float* xsrc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) xsrc[j] = io.cond + (size_t)min(tf0 * 16 + xr + j * 64, io.M - 1) * io.C;
  bf16x8 rw[2];
  f32x4 rx[2];
  auto request = [&](int k) {
    k = min(k, KS - 1);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      rw[j] = wsrc[((size_t)j * KS + k) * 64];
      rx[j] = *reinterpret_cast<const f32x4*>(xsrc[j] + min(k * 32 + xc, io.C - 4));
    }
    __builtin_amdgcn_sched_barrier(0);                  // (the scheduler would sink the loads to their use)
  };
  auto deposit = [&](int k) {
    unsigned char* st = lds + (k & 1) * COND_STAGE_B;
    const bool in = k * 32 + xc < io.C;                 // (C is a multiple of 4; features beyond it are zero)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      reinterpret_cast<bf16x8*>(st)[(wave * 2 + j) * 64 + lane] = rw[j];
      *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(st + COND_W_B) + (xr + j * 64) * COND_XS + xc) =
          in ? rx[j] : f32x4{0, 0, 0, 0};
    }
  };
  request(0);
  deposit(0);
  request(1);
  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0, 0, 0, 0};
  const int per_layer = 2 * n.d, f_tile = ft * COND_FF * 16;       // first feature of the tile in [layer][k|v][d]
  const int layer = f_tile / per_layer, cls = (f_tile % per_layer) / n.d;   // 0 keys, 1 values
  auto product = [&](auto KEYS) {
    constexpr bool keys = decltype(KEYS)::value;
    for (int k = 0; k < KS; ++k) {
      __syncthreads();                                  // stage k is in LDS; stage k-1 has been read by every wave
      const unsigned char* st = lds + (k & 1) * COND_STAGE_B;
      const float* xs = reinterpret_cast<const float*>(st + COND_W_B) + (wt * 64 + l16) * COND_XS + lg;
      bf16x8 a[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = reinterpret_cast<const bf16x8*>(st)[(wf * 4 + i) * 64 + lane];
      deposit(k + 1);
      request(k + 2);
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        float b[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) b[j] = xs[j * 16 * COND_XS + 4 * m];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[i][j] = keys ? __builtin_amdgcn_mfma_f32_16x16x4f32((float)a[i][m], b[j], acc[i][j], 0, 0, 0)
                             : __builtin_amdgcn_mfma_f32_16x16x4f32(b[j], (float)a[i][m], acc[i][j], 0, 0, 0);
      }
    }
  };
  if (cls == 0) product(std::true_type{}); else product(std::false_type{});
  const int DH = n.d / n.heads, KH = DH / 32, CF = DH / 16, SF = io.SF;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int fr = f_tile + (wf * 4 + i) * 16;          // first feature of the fragment, [layer][k|v][d]
    const int fd = fr % n.d, head = fd / DH, fh = fd % DH;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int tf = tf0 + wt * 4 + j;
      if (tf >= MF) continue;
      const int env = tf / SF, sf = tf % SF;
      const size_t eh = ((size_t)env * n.L + layer) * n.heads + head;
      if (cls == 0) {
        const f32x4 b = *reinterpret_cast<const f32x4*>(n.bias + fr + lg * 4);
        const int ks = fh / 32, g = (fh % 32) / 8 + lg / 2;      // a fragment is half of a 32-deep k-step
        __bf16* dst = n.kc + (((eh * SF + sf) * KH + ks) * 64 + l16 + 16 * g) * 8 + (lg & 1) * 4;
        *reinterpret_cast<bf16x4*>(dst) = to_bf16x4(acc[i][j] + b);
      } else {
        const float b = n.bias[fr + l16];
        __bf16* dst = n.vct + (((eh * CF + fh / 16) * SF + sf) * 64 + lane) * 4;
        *reinterpret_cast<bf16x4*>(dst) = to_bf16x4(acc[i][j] + b);
      }
    }
  }
}

}  // namespace tsdp
