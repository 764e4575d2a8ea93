// Cross-attention keys / values of new observations, for the fused bf16 networks: every layer's K and V projection of
// both networks in one launch, written straight in the fragment order the attention reads.
//
// The sums are k_linear's: fp32 fused multiply-adds over the features in ascending order, then the bias, then one rounding to
// bf16.  Any other order rounds a few keys to the other bf16 number, and at the first timesteps of a squared-cosine chain,
// where a noise prediction is multiplied by 31, that is enough for a nearly tied draft to fall on the other side of its test.
// So the product runs on the bf16 matrix cores, where it is ordered otherwise, and the numbers that lie so close to a rounding
// boundary that the order may matter (of Gaussian observations one in a hundred) are added up again, feature by feature.  How close
// that is follows from how far apart the two sums were measured to end up: it is no bound for every input (that would list one number in seven).
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

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

struct CondNet {                 // one network's share of the launch
  const bf16x8* w;               // [L*2*d/16][KS][64] fragments: per layer the key rows, then the value rows
  const float* bias;             // [L*2*d], behind them the 2-norms of the weight rows
  __bf16* kc; __bf16* vct;       // FusedNet::kc / vct
  int L, d, heads, tiles;        // tiles = L*2*d / 256
};
constexpr int COND_FEW = 10;
struct CondIO { CondNet net[2]; const float* cond; float* size; int M, C, KS, SF; };   // cond [M = B*S, C], size [M]

// size[m] = 2-norm of token m, negative where the kernel below would add most of its numbers again: an infinity among its features,
// or a few features of two leading bits each (a mask, an index), whose sums end on rounding boundaries.  A wavefront a token.
__global__ __launch_bounds__(256) void k_cond_size(CondIO io) {
  const int m = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (m >= io.M) return;
  float q = 0.0f;
  unsigned bits = 0;
  int count = 0;
#pragma unroll 4
  for (int i = lane * 4; i < io.C; i += 256) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(io.cond + (size_t)m * io.C + i);
    q += (x[0] * x[0] + x[1] * x[1]) + (x[2] * x[2] + x[3] * x[3]);
#pragma unroll
    for (int e = 0; e < 4; ++e) { bits |= __builtin_bit_cast(unsigned, x[e]); count += x[e] != 0.0f; }
  }
#pragma unroll
  for (int o = 1; o < 64; o *= 2) { q += __shfl_xor(q, o); bits |= __shfl_xor(bits, o); count += __shfl_xor(count, o); }
  const bool again = q == INFINITY || (count > 1 && count <= COND_FEW && (bits & 0x1FFFFF) == 0);
  if (lane == 0) io.size[m] = again ? -sqrtf(q) : sqrtf(q);
}

// Tile: 256 features (16 fragments, all keys or all values of one layer because d is a multiple of 256) x 128 tokens
// (8 fragments).  8 waves as 4 x 2, each 64 features x 64 tokens.  An observation is the sum of three bf16 numbers (its leading,
// middle and last eight bits), the weights are bf16: three products on the bf16 matrix cores, each exact, summed in fp32.  Per
// k-step of 32 features the workgroup brings 16 KB of weights and 24 KB of observation planes into LDS and does 384 MFMAs, 1536
// cycles of each matrix core: they bound it.  Two LDS buffers, the next k-step travels through registers while the current one
// is multiplied; one barrier per k-step; two workgroups per CU, one multiplies while the other waits or adds again.
// Keys are computed features x tokens, values tokens x features, so that in both cases a lane's four accumulators are
// the neighbouring entries of one 8-byte piece of the attention operand.
//
// Which numbers are added again: those v that round differently with the largest of three terms on either side, u = 2^-24.
//   3 u |x| |w|       terms of either sign: a chain of fp32 additions ends 0.30 u |x| |w| away from the exact sum (standard deviation), the
//                     matrix cores' sum 0.18.  With 1.5 35 numbers of the 2.2e8 of 256 observations round the other way, with 2 ten, with 3 none to two.
//   2.2 r u |v|       r = sqrt(C) + C / 128.  Sums that grow steadily, as of one sign: standard deviation of the difference 8.5 u |v| at C = 768, 16.5
//                     (mean 38) at 3072, 2.4 at 64, so seven and more of them (at 3072 five beyond the mean).
//   3.5 r u |x| |w| s sums that were far larger on the way and cancel: s is the largest of the thread's 64 partial sums after a quarter, half
//                     and three quarters of the features in units of their |x| |w|.  Only where r s > 5.4, 4.5 standard deviations of a sum
//                     of either sign: most wavefronts only compare their largest partial sum with the least that could be that.
// The deviations are those of 2.6e5 sums each against fp64 (Gaussian; of one sign; half of each sign in turn; large in the first eighth).  With all
// three the noise predictions of 60 batches of 256 environments (six of each of ten kinds, weights of either and of one sign) had no bit other than
// with every number added in order; with the first alone those of one or two environments of every second Gaussian batch had.
// The workgroup lists the numbers in LDS, a thread takes one, and a second pass over the k-steps brings weights and observations
// through the LDS as before, 512 numbers at a time: 0.35 ms each where all tiles take one.
// Observations of a few features of two leading bits (masks, indices) list 8 to 22 % of their numbers, since their sums end on boundaries,
// and infinities all of them.  Beyond 3072 numbers a tile is multiplied once more with fp32 operands on the fp32 matrix cores, whose
// chains are the sums in order themselves (2.5 ms where all tiles do), and a tile with 16 marked tokens (k_cond_size) at once.
// Measured, 256 environments x 64 tokens x 768, 12 layers of d = 512 and 2 of d = 256, with k_cond_size, Gaussian observations: 1.31 ms
// (1.28 ms and 71 us with the first term alone); of one sign 1.3, a mask of 5 % 1.62, of 1 %, four or two features set, infinities 2.54, sums
// that cancel 3.55; 4 environments 77 us, at most 173 us.  With every tile in order 2.50 ms and 112 us; without the fp32 tiles 3.6, 4.5, 5.9, 19.8
// (infinities, not-a-numbers), 4.0 and up to 1.1 ms.  Of the 128 registers 42 are spilled before and after the loop over the k-steps, none in it.
constexpr int COND_FF = 16, COND_TF = 8, COND_XS = 36;   // floats per token in LDS (second pass): 32 and the bank padding
constexpr int COND_W_B = COND_FF * 64 * 16, COND_STAGE_B = COND_W_B + 3 * COND_TF * 64 * 16, COND_LDS = 2 * COND_STAGE_B;
constexpr int COND_AGAIN_B = COND_W_B + COND_TF * 16 * COND_XS * 4, COND_LIST = 512, COND_AGAIN = 6 * COND_LIST, COND_MARKED = 16;
constexpr float COND_ULP = 5.9604645e-8f, COND_TIE = 3.0f * COND_ULP, COND_OWN = 2.2f, COND_GROWN = 3.5f, COND_UNUSUAL = 5.4f;
static_assert(2 * COND_AGAIN_B + 4 * (COND_LIST + 1) <= COND_LDS && 2 * COND_LDS <= 160 * 1024, "LDS");

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
  const float* xsrc = io.cond + (size_t)tf0 * 16 * io.C;
  unsigned xat[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) xat[j] = (unsigned)min(xr + j * 64, io.M - 1 - tf0 * 16) * io.C;
  bf16x8 rw[2];
  f32x4 rx[2];
  auto request = [&](int k) {
    k = min(k, KS - 1);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      rw[j] = wsrc[((size_t)j * KS + k) * 64];
      rx[j] = *reinterpret_cast<const f32x4*>(xsrc + (xat[j] + min(k * 32 + xc, io.C - 4)));
    }
    __builtin_amdgcn_sched_barrier(0);                  // (the scheduler would sink the loads to their use)
  };
  auto observed = [&](int k, int j) { return k * 32 + xc < io.C ? rx[j] : f32x4{0, 0, 0, 0}; };   // (C is a multiple of 4; features beyond it are zero)
  auto deposit_weights = [&](unsigned char* st) {
#pragma unroll
    for (int j = 0; j < 2; ++j) reinterpret_cast<bf16x8*>(st)[(wave * 2 + j) * 64 + lane] = rw[j];
  };
  // planes as fragments [plane][token fragment][64][8]
  auto deposit = [&](int k) {
    unsigned char* st = lds + (k & 1) * COND_STAGE_B;
    deposit_weights(st);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      f32x4 x = observed(k, j);
      unsigned char* at = st + COND_W_B + ((j * 4 + xr / 16) * 64 + xr % 16 + 16 * (xc / 8)) * 16 + (xc % 8) * 2;
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        uint32_t b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float v = x[i];
          b[i] = __builtin_bit_cast(uint32_t, v) & 0xFFFF0000u;
          x[i] = v - __builtin_bit_cast(float, b[i]);    // exact
        }
        *reinterpret_cast<uint2*>(at + p * (COND_TF * 64 * 16)) = make_uint2(b[0] >> 16 | b[1], b[2] >> 16 | b[3]);
      }
    }
  };
  const int per_layer = 2 * n.d, f_tile = ft * COND_FF * 16;       // first feature of the tile in [layer][k|v][d]
  const int layer = f_tile / per_layer, cls = (f_tile % per_layer) / n.d;   // 0 keys, 1 values
  const float *bias0 = n.bias + f_tile + wf * 64, *norm0 = bias0 + n.L * per_layer, *size0 = io.size + tf0 * 16;
  // of the wave's feature fragment i the lane's four features, of its token fragment j the lane's four tokens (one of them four times)
  auto features = [&](bool keys, const float* v, int i) {
    return keys ? *reinterpret_cast<const f32x4*>(v + i * 16 + lg * 4) : f32x4{1, 1, 1, 1} * v[i * 16 + l16];
  };
  auto tokens = [&](bool keys, int j) {
    const float* v = size0 + min(wt * 4 + j, MF - 1 - tf0) * 16;
    const f32x4 x = keys ? f32x4{1, 1, 1, 1} * v[l16] : *reinterpret_cast<const f32x4*>(v + lg * 4);
    return f32x4{fabsf(x[0]), fabsf(x[1]), fabsf(x[2]), fabsf(x[3])};
  };
  // (the same without a branch, by addresses)
  const int fb = cls == 0 ? lg * 4 : l16, fs = cls == 0 ? 1 : 0, tb = cls == 0 ? l16 : lg * 4, ts = 1 - fs;
  auto features_of = [&](const float* v, int i) { v += i * 16 + fb; return f32x4{v[0], v[fs], v[2 * fs], v[3 * fs]}; };
  auto tokens_of = [&](int j) {
    const float* v = size0 + min(wt * 4 + j, MF - 1 - tf0) * 16 + tb;
    return f32x4{fabsf(v[0]), fabsf(v[ts]), fabsf(v[2 * ts]), fabsf(v[3 * ts])};
  };
  // Largest of the thread's partial sums on the way, in units of |x| |w|, where one is more than `unusual` of them; looked at three
  // times.  The least product of the thread's norms tells first whether there can be one.
  const float root = sqrtf((float)io.C) + io.C * (1.0f / 128), unusual = COND_UNUSUAL / root;
  float seen = 0.0f;
  auto limit = [&](auto KEYS) {
    constexpr bool keys = decltype(KEYS)::value;
    float lw = INFINITY, lx = INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f32x4 w = features(keys, norm0, i), x = tokens(keys, i);
#pragma unroll
      for (int e = 0; e < 4; ++e) { lw = fminf(lw, w[e] > 0.0f ? w[e] : INFINITY); lx = fminf(lx, x[e] > 0.0f ? x[e] : INFINITY); }
    }
    return lw * lx * unusual;
  };
  const float least = cls == 0 ? limit(std::true_type{}) : limit(std::false_type{});
  const int quarter = (KS + 3) / 4;
  f32x4 acc[4][4];
  auto zero = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0, 0, 0, 0};
  };
  auto product = [&](auto KEYS) {
    constexpr bool keys = decltype(KEYS)::value;
    auto look = [&]() {
      float most = 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) most = fmaxf(most, fabsf(acc[i][j][e]));
      if (!__any(most > least)) return;
      for (int j = 0; j < 4; ++j) {                      // (not unrolled: registers)
        const f32x4 x = tokens(keys, j);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f32x4 w = features(keys, norm0, i);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float s = j == 0 ? acc[i][0][e] : j == 1 ? acc[i][1][e] : j == 2 ? acc[i][2][e] : acc[i][3][e];
            seen = fmaxf(seen, fabsf(s) * __builtin_amdgcn_rcpf(w[e] * x[e]));   // (0 / 0 of an empty token or row: left out)
          }
        }
      }
    };
    int next = quarter - 1;
    request(0);
    deposit(0);
    request(1);
    zero();
    for (int k = 0; k < KS; ++k) {
      __syncthreads();                                  // stage k is in LDS; stage k-1 has been read by every wave
      const unsigned char* st = lds + (k & 1) * COND_STAGE_B;
      const bf16x8* xs = reinterpret_cast<const bf16x8*>(st + COND_W_B) + wt * 4 * 64 + lane;
      bf16x8 a[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = reinterpret_cast<const bf16x8*>(st)[(wf * 4 + i) * 64 + lane];
      deposit(k + 1);
      request(k + 2);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          const bf16x8 b = xs[(p * COND_TF + j) * 64];
#pragma unroll
          for (int i = 0; i < 4; ++i)
            acc[i][j] = keys ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b, acc[i][j], 0, 0, 0)
                             : __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, a[i], acc[i][j], 0, 0, 0);
        }
      if (k == next && k < KS - 1) { look(); next += quarter; }
    }
  };
  const int DH = n.d / n.heads, KH = DH / 32, CF = DH / 16, SF = io.SF;
  // where the four numbers of lane `ln` in feature fragment fi of the tile and token fragment tj go
  auto place = [&](int fi, int tj, int ln) {
    const int fr = f_tile + fi * 16, fd = fr % n.d, head = fd / DH, fh = fd % DH, g = ln / 16;
    const int tf = tf0 + tj, env = tf / SF, sf = tf % SF;
    const size_t eh = ((size_t)env * n.L + layer) * n.heads + head;
    return cls == 0 ? n.kc + (((eh * SF + sf) * KH + fh / 32) * 64 + ln % 16 + 16 * ((fh % 32) / 8 + g / 2)) * 8 + (g & 1) * 4   // a fragment is half of a 32-deep k-step
                    : n.vct + (((eh * CF + fh / 16) * SF + sf) * 64 + ln) * 4;
  };
  auto each = [&](auto&& f) {                           // f(i, j, sums with their biases) of the thread's pieces, stored as well
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f32x4 bias = features_of(bias0, i);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (tf0 + wt * 4 + j >= MF) continue;
        const f32x4 v = acc[i][j] + bias;
        *reinterpret_cast<bf16x4*>(place(wf * 4 + i, wt * 4 + j, lane)) = to_bf16x4(v);
        f(i, j, v);
      }
    }
  };
  // observations as they are, [token][COND_XS]
  auto deposit_x = [&](unsigned char* st, int k) {
#pragma unroll
    for (int j = 0; j < 2; ++j) *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(st + COND_W_B) + (xr + j * 64) * COND_XS + xc) = observed(k, j);
  };
  // how many of the tile's tokens had better be added in order right away
  int marked = 0;
#pragma unroll
  for (int j = 0; j < 2; ++j) marked += __builtin_popcountll(__ballot(lane + j * 64 < io.M - tf0 * 16 && size0[min(lane + j * 64, io.M - 1 - tf0 * 16)] < 0.0f));
  if (marked < COND_MARKED) {
    if (cls == 0) product(std::true_type{}); else product(std::false_type{});
    const float line = seen > unusual ? fmaxf(COND_TIE, COND_GROWN * COND_ULP * root * seen) : COND_TIE, own = (COND_OWN * root + 2.0f) * COND_ULP;
    uint64_t again = 0;                                 // bit (i * 4 + j) * 4 + e
    f32x4 x[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = tokens_of(j) * line;
    f32x4 wnorm;
    each([&](int i, int j, const f32x4& v) {
      if (j == 0) wnorm = features_of(norm0, i);
      const f32x4 drawn = wnorm * x[j];
      unsigned m = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float tie = fmaxf(drawn[e], own * fabsf(v[e]));
        // (drawn is a not-a-number where an observation or a weight is one, and the sum is one in any order)
        if (drawn[e] == drawn[e] && ((float)(__bf16)(v[e] - tie) != (float)(__bf16)(v[e] + tie) || !(fabsf(v[e]) + tie < 3.0e38f))) m |= 1u << e;
      }
      again |= (uint64_t)m << ((i * 4 + j) * 4);
    });
    int* list = reinterpret_cast<int*>(lds + 2 * COND_AGAIN_B);
    int* listed = list + COND_LIST;
    __syncthreads();                                    // the LDS is free, and what was stored above has left (the numbers added again are stored over it)
    if (threadIdx.x == 0) *listed = 0;
    __syncthreads();
    int slot = again ? atomicAdd(listed, __builtin_popcountll(again)) : 0;
    __syncthreads();
    const int total = *listed;
    if (total <= COND_AGAIN) {
      for (int from = 0; from < total; from += COND_LIST) {
        __syncthreads();                                // the list and both stages have been read
        for (; again && slot < from + COND_LIST; ++slot) {
          list[slot - from] = (int)threadIdx.x << 6 | __builtin_ctzll(again);
          again &= again - 1;
        }
        __syncthreads();
        const bool mine = (int)threadIdx.x < total - from;
        const int item = list[mine ? threadIdx.x : 0], ow = item >> 12, ol = item >> 6 & 63, p = item & 63;
        const int fi = (ow & 3) * 4 + p / 16, tj = (ow >> 2) * 4 + p / 4 % 4, four = (ol >> 4) * 4 + p % 4;
        const int fl = cls == 0 ? four : ol & 15, tk = tj * 16 + (cls == 0 ? ol & 15 : four);
        auto deposit_again = [&](int k) {
          unsigned char* st = lds + (k & 1) * COND_AGAIN_B;
          deposit_weights(st);
          deposit_x(st, k);
        };
        request(0);
        deposit_again(0);
        request(1);
        float sum = 0.0f;
        for (int k = 0; k < KS; ++k) {
          __syncthreads();
          const unsigned char* st = lds + (k & 1) * COND_AGAIN_B;
          deposit_again(k + 1);
          request(k + 2);
          if (mine) {
            const bf16x8* w = reinterpret_cast<const bf16x8*>(st) + fi * 64 + fl;
            const f32x4* x = reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(st + COND_W_B) + tk * COND_XS);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              const bf16x8 wv = w[g * 16];
              const f32x4 x0 = x[2 * g], x1 = x[2 * g + 1];
#pragma unroll
              for (int i = 0; i < 4; ++i) sum = fmaf(x0[i], (float)wv[i], sum);
#pragma unroll
              for (int i = 0; i < 4; ++i) sum = fmaf(x1[i], (float)wv[4 + i], sum);
            }
          }
        }
        if (mine) place(fi, tj, ol)[p % 4] = (__bf16)(sum + n.bias[f_tile + fi * 16 + fl]);
      }
      return;
    }
  }
  // The whole tile in order.  mfma_f32_16x16x4_f32 adds its four products to the accumulator one after the other, each with one
  // rounding, in the order of the lane groups (checked on hardware, denormals included): lane group g supplies features 4m + g of a
  // k-step to MFMA m, so its weights lie as entries m of lane 16 g + row.
  auto deposit_ordered = [&](int k) {
    unsigned char* st = lds + (k & 1) * COND_AGAIN_B;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<bf16x2*>(st + (((wave * 2 + j) * 64 + 16 * g + l16) * 8 + 2 * lg) * 2) = bf16x2{rw[j][g], rw[j][4 + g]};
    deposit_x(st, k);
  };
  auto ordered = [&](auto KEYS) {
    constexpr bool keys = decltype(KEYS)::value;
    __syncthreads();
    request(0);
    deposit_ordered(0);
    request(1);
    zero();
    for (int k = 0; k < KS; ++k) {
      __syncthreads();
      const unsigned char* st = lds + (k & 1) * COND_AGAIN_B;
      const float* xs = reinterpret_cast<const float*>(st + COND_W_B) + (wt * 64 + l16) * COND_XS + lg;
      bf16x8 a[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = reinterpret_cast<const bf16x8*>(st)[(wf * 4 + i) * 64 + lane];
      deposit_ordered(k + 1);
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
  if (cls == 0) ordered(std::true_type{}); else ordered(std::false_type{});
  each([](int, int, const f32x4&) {});
}

}  // namespace tsdp
