// Cross-attention keys / values of new observations, for the fused bf16 networks: every layer's K and V projection of
// both networks in one launch, written straight in the fragment order the attention reads.
//
// The observations are fp32 and stay so: a float is the exact sum of three bf16 numbers (3 x 8 significant bits), the
// weights are bf16 already, so three bf16 MFMAs per fragment pair give the fp32 x bf16 products exactly and add them
// in fp32 -- at a third of the bf16 matrix rate, five times the fp32 matrix rate.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "fused_mfma.hpp"

namespace tsdp {

// Conditioning vectors: both networks' embeddings W cond + b in one launch.  One wavefront per
// output feature and eight environments: it reads its weight row once, 16 bytes a lane, and sums over the lanes.  Bound by
// the latency of two dependent reads, in large batches by the environments each wavefront reads again.  C = 1024, both
// networks of d = 256 + 128 (384 + 192): 1, 64, 256, 1024 environments 6.9 (6.5), 7.9 (10), 19 (27), 66 (94) us; the tiled
// product (C / 16 barrier steps whatever the batch) 117 us, so beyond 1024 environments that one stays.
constexpr int COND_VEC_B = 1024;
struct CondVecNet { const float* w; const float* b; float* out; int d; };
__global__ __launch_bounds__(256) void k_cond_vec(const float* __restrict__ cond, CondVecNet n0, CondVecNet n1, int B, int C) {
  constexpr int NE = 8;
  const int lane = threadIdx.x & 63;
  int f = blockIdx.x * 4 + (threadIdx.x >> 6);
  const CondVecNet n = f < n0.d ? n0 : n1;
  if (f >= n0.d) f -= n0.d;
  if (f >= n.d) return;
  const int e0 = blockIdx.y * NE;
  float acc[NE] = {};
  for (int c = lane * 4; c < C; c += 256) {             // (C is a multiple of 4)
    const f32x4 w = *reinterpret_cast<const f32x4*>(n.w + (size_t)f * C + c);
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(cond + (size_t)min(e0 + e, B - 1) * C + c);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[e] = fmaf(w[j], x[j], acc[e]);
    }
  }
#pragma unroll
  for (int e = 0; e < NE; ++e) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc[e] += __shfl_xor(acc[e], o);
    if (lane == 0 && e0 + e < B) n.out[(size_t)(e0 + e) * n.d + f] = acc[e] + n.b[f];
  }
}

// cond [M, C] fp32 -> planes [ceil(M/16)][KS][3][64][8] bf16 in MFMA operand order (lane l: row l%16, columns
// ks*32 + (l/16)*8 ..), zero beyond M and C.  One thread per (fragment, k-step, lane); C is a multiple of 4.
__global__ __launch_bounds__(256) void k_split_cond(const float* __restrict__ cond, int M, int C, int KS,
                                                    bf16x8* __restrict__ planes) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  const int MF = (M + 15) / 16;
  if (i >= (long long)MF * KS * 64) return;
  const int lane = (int)(i & 63);
  const long long fk = i >> 6;
  const int ks = (int)(fk % KS), mf = (int)(fk / KS);
  const int row = mf * 16 + (lane & 15), col = ks * 32 + (lane >> 4) * 8;
  float v[8];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    f32x4 x = f32x4{0, 0, 0, 0};
    if (row < M && col + 4 * h < C) x = *reinterpret_cast<const f32x4*>(cond + (size_t)row * C + col + 4 * h);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[4 * h + j] = x[j];
  }
  bf16x8 p[3];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const __bf16 a = (__bf16)v[j];
    const float r1 = v[j] - (float)a;
    const __bf16 b = (__bf16)r1;
    p[0][j] = a; p[1][j] = b; p[2][j] = (__bf16)(r1 - (float)b);
  }
  bf16x8* out = planes + fk * 3 * 64 + lane;
#pragma unroll
  for (int q = 0; q < 3; ++q) out[q * 64] = p[q];
}

struct CondNet {                 // one network's share of the launch
  const bf16x8* w;               // [L*2*d/16][KS][64] fragments: per layer the key rows, then the value rows
  const float* bias;             // [L*2*d]
  __bf16* kc; __bf16* vct;       // FusedNet::kc / vct
  int L, d, heads, tiles;        // tiles = L*2*d / 256
};
struct CondIO { CondNet net[2]; const bf16x8* planes; int MF, KS, SF; };   // MF = B*SF token fragments

// Tile: 256 features (16 fragments, all keys or all values of one layer because d is a multiple of 256) x 128 tokens
// (8 fragments, three planes each).  8 waves as 4 x 2, each 64 features x 64 tokens.  Per k-step the workgroup brings
// 16 KB of weights and 24 KB of planes into LDS and does 384 MFMAs (1536 cycles): 27 B per cycle and CU, half of what
// the L2 delivers, so the matrix cores bound it.  Two LDS buffers, the next k-step travels through registers while
// the current one is multiplied; one barrier per k-step.
// Keys are computed features x tokens, values tokens x features, so that in both cases a lane's four accumulators are
// the neighbouring entries of one 8-byte piece of the attention operand.
// Measured, 256 environments x 64 tokens x 768, 12 layers of d = 512 and 2 of d = 256: 0.90 ms = 1.12 PFLOP/s of bf16
// products (k_split_cond before it: 0.024 ms), against 4.9 ms of fp32 products on the vector units in 28 launches, each
// followed by two that rounded and reordered its output.
constexpr int COND_FF = 16, COND_TF = 8, COND_STAGE = (COND_FF + 3 * COND_TF) * 64;   // stage size in 16-byte units
constexpr int COND_LDS = 2 * COND_STAGE * 16;

__global__ __launch_bounds__(512, 1) void k_cond_kv(CondIO io) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  bf16x8* lds = reinterpret_cast<bf16x8*>(lds_raw);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wf = wave & 3, wt = wave >> 2, l16 = lane & 15, lg = lane >> 4;
  // consecutive workgroups share the feature tile and walk the tokens
  const int tt = (io.MF + COND_TF - 1) / COND_TF;
  int ft = blockIdx.x / tt;
  const int tf0 = (blockIdx.x % tt) * COND_TF;
  const int which = ft >= io.net[0].tiles ? 1 : 0;
  const CondNet& n = io.net[which];
  if (which) ft -= io.net[0].tiles;
  const int KS = io.KS;
  const bf16x8* wsrc = n.w + (size_t)ft * COND_FF * KS * 64;
  // a wave fetches 5 of the 40 fragments of a stage: fragment id 0..15 weights, 16.. planes (token fragment, plane)
  constexpr int PW = (COND_FF + 3 * COND_TF) / 8;
  const bf16x8* src[PW];
  int step[PW];
#pragma unroll
  for (int j = 0; j < PW; ++j) {
    const int id = wave * PW + j;
    if (id < COND_FF) {
      src[j] = wsrc + (size_t)id * KS * 64 + lane; step[j] = 64;
    } else {
      const int tf = min(tf0 + (id - COND_FF) / 3, io.MF - 1), q = (id - COND_FF) % 3;
      src[j] = io.planes + ((size_t)tf * KS * 3 + q) * 64 + lane; step[j] = 3 * 64;
    }
  }
  bf16x8 r[PW];
#pragma unroll
  for (int j = 0; j < PW; ++j) r[j] = src[j][0];
#pragma unroll
  for (int j = 0; j < PW; ++j) lds[(wave * PW + j) * 64 + lane] = r[j];
#pragma unroll
  for (int j = 0; j < PW; ++j) r[j] = src[j][(size_t)min(1, KS - 1) * step[j]];
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
      const bf16x8* st = lds + (k & 1) * COND_STAGE;
      bf16x8 a[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = st[(wf * 4 + i) * 64 + lane];
#pragma unroll
      for (int q = 2; q >= 0; --q) {                    // small pieces first
        bf16x8 b[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) b[j] = st[(COND_FF + (wt * 4 + j) * 3 + q) * 64 + lane];
        if (q == 2) {
          bf16x8* nx = lds + ((k + 1) & 1) * COND_STAGE;
#pragma unroll
          for (int j = 0; j < PW; ++j) nx[(wave * PW + j) * 64 + lane] = r[j];
#pragma unroll
          for (int j = 0; j < PW; ++j) r[j] = src[j][(size_t)min(k + 2, KS - 1) * step[j]];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[i][j] = keys ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0)
                             : __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
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
      if (tf >= io.MF) continue;
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
