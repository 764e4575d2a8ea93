// C ABI of the speculative denoising round: context, weights, tables, workspace and launch sequences.
// Definitions of the operations: Section 3.1 (acceptance test, first rejection, reflection coupling)
// and Section 3.2 (drafter rollout, batched verification, log acceptance ratio) of the TS-DP paper.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/tsdp.h"
#include "kernels_f32.hpp"
#include "fused_mfma.hpp"
#include "cond_kernels.hpp"
#include "few_plan.hpp"
#include "few_rows.hpp"
#include "row_dyn.hpp"
#include "flow_rows.hpp"
#include "round_kernels.hpp"

using namespace tsdp;

namespace {

struct FewRun {                 // one forward pass of k_few_*
  const float* x; const int32_t* row_t; const int32_t* row_env; const int32_t* d_R;
  int R_cap, safe_rows, A, T;
  const float* mod;             // [R][L*4D], or the network's table over timesteps
  float* eps_out;
  float* h[2]; float* part[2]; size_t pstride;
  unsigned char* buf; int32_t* sync; int32_t* status;   // k_flow: buffers of the rows, tickets and counters
  int flow_wgs;                 // k_flow: workgroups of a launch at most, 0: as many as are of use
};

struct LayerOff {
  size_t mod_w, mod_b, qkv_w, qkv_b, o_w, o_b, cq_w, cq_b, ck_w, ck_b, cv_w, cv_b, co_w, co_b, up_w, up_b, dn_w, dn_b;
};

// a tile of the persistent rollout: `rpt` environments a workgroup; fits: its LDS suffices for this network
struct DraftTile {
  hipError_t (*launch)(const FusedNet&, const DraftIO&, int A, hipStream_t) = nullptr;
  bool (*fits_of)(int A, int L) = nullptr;
  int rpt = 0;
  bool fits = false;
};

struct Net {
  int L = 0, d = 0, heads = 0, m = 0;
  size_t n_floats = 0;
  size_t tok_w, tok_b, pos, t_w1, t_b1, t_w2, t_b2, c_w, c_b, head_w, head_b;
  std::vector<LayerOff> lay;
  float* blob = nullptr;        // device copy of the (rounded) canonical blob
  float* temb = nullptr;        // [T, d] timestep embedding of every timestep
  float* modtab = nullptr;      // [T, L*4d] FiLM vectors of every timestep (token conditioning, fused bf16 path)
  int32_t* t_iota = nullptr;    // [T] 0..T-1, the row timesteps of the table build
  float* modw = nullptr;        // [L*4d, d] FiLM projections of all layers, concatenated
  float* modb = nullptr;        // [L*4d]
  float* cemb = nullptr;        // [B_max, d] conditioning embedding (mode 0)
  float* kc = nullptr;          // [L, B_max*S, d] cross-attention keys (mode 1)
  float* vc = nullptr;          // [L, B_max*S, d] cross-attention values (mode 1)
  bool loaded = false;
  const char* path = "f32-ops";
  // fused bf16 MFMA path (bf16 networks of supported shape)
  bool fused = false;
  FusedNet fnet;
  hipError_t (*fused_verify)(const FusedNet&, const FusedIO&, int A, int R_cap, hipStream_t) = nullptr;
  hipError_t (*fused_verify_few)(const FusedNet&, const FusedIO&, int A, int R_cap, hipStream_t) = nullptr;
  int verify_rpt = 1;
  void (*fused_mod)(const FusedNet&, const int32_t*, int, const int32_t*, int, const int32_t*, int, float*, hipStream_t) = nullptr;
  DraftTile draft_small, draft_big;   // few, many environments per workgroup
  bool few = false;             // the forward pass of this context's rows is spread over the chip (k_few_*)
  bool few_roll = false;        // so is the drafter's rollout
  void (*few_forward)(const FusedNet&, const FewRun&, hipStream_t) = nullptr;
  void (*few_draft)(const FusedNet&, const FewRun&, const DraftIO&, int, float* const*, hipStream_t) = nullptr;
  void (*few_film)(const FusedNet&, const int32_t*, int, const int32_t*, int, int, const int32_t*, const int32_t*, int, float*, hipStream_t) = nullptr;
  int few_slices = 0;           // partial sums per row, 0: none (k_row)
  size_t flow_row = 0;          // bytes of a row's buffers (k_flow), 0: two launches per layer (k_few_*)
  float* tok_wt = nullptr;      // [A, d] token embedding, transposed
  uint16_t* kc_pk = nullptr;    // fragment-ordered bf16 keys / transposed values of every (env, layer, head)
  uint16_t* vct_pk = nullptr;
  uint8_t* kv_w = nullptr;      // key / value projections of all layers as MFMA fragments (fused bf16 cross-attention)
  float* kv_b = nullptr;        // their biases, [L][k|v][d], and the 2-norms of their rows
};

}  // namespace

// Scratch of tsdp_distill_loss_noalloc: the per-workgroup partial sums of the loss (three doubles each) live in a
// file-scope device array instead of context memory, so that entry point allocates nothing.  Every GPU holds its own
// copy; host code uses the address hipGetSymbolAddress returns for the current device, looked up once per device in
// tsdp_create, never the symbol itself.
constexpr int NOALLOC_MAX_ROWS = 65536;
constexpr int NOALLOC_MAX_DEVICES = 64;
static __device__ __align__(256) double scratch[3 * DISTILL_WGS];
static double* g_scratch_ptr[NOALLOC_MAX_DEVICES];   // device address of `scratch` on each device, null until looked up

struct tsdp_ctx {
  tsdp_config cfg;
  int device = -1;              // the device that was current in tsdp_create
  int D = 0;
  std::string err;
  float* tables = nullptr;      // 6 x T fp32: sqrt_abar, sqrt_1m, c0, cx, sigma, ce
  SchedTables tb;
  Net net[2];
  bool cond_set = false;
  int cond_B = 0;
  float* cond_size = nullptr;   // [B_max * tokens] their 2-norms (k_cond_kv)
  int32_t* status = nullptr;
  int32_t* live = nullptr;      // environments still running (chain driver)
  int32_t* K_sel = nullptr;     // [B_max] per-round picks from the stage tables (staged chain driver)
  float* s_sel = nullptr;
  float* lam_sel = nullptr;
  double* loss_partial = nullptr;   // per-workgroup partial sums of the distillation loss
  int32_t* K_eff = nullptr;     // [B_max]
  int32_t* n_draft = nullptr;   // [0] B while some environment has rows in the current plan, [1] B while one drafts; else 0
  // network workspace (lazy)
  bool ws_ready = false;
  float *h = nullptr, *a = nullptr, *qkv = nullptr, *ao = nullptr, *u = nullptr, *sg = nullptr, *mod = nullptr;
  // k_few_*: residual, partial sums, latents between two transitions, FiLM vectors of all transitions of a rollout
  FewSize few_have;             // floats of few_h / few_part
  unsigned char* flow_buf = nullptr; size_t flow_have = 0;   // k_flow: buffers of the rows, empty between launches
  int32_t* sync = nullptr;      // k_flow: tickets and counters of the verify rows, then of the rollout's environments
  int flow_wgs = 0;             // (FewRun::flow_wgs; tests)
  float *few_h[2] = {nullptr, nullptr}, *few_part[2] = {nullptr, nullptr}, *few_y[2] = {nullptr, nullptr}, *few_mod = nullptr;
  float* eps_tmp = nullptr;     // [B_max, D] drafter output of the current step
  int32_t *row_t_chk = nullptr, *row_env_chk = nullptr;   // [rows] range-checked copy of a caller's row table (tsdp_verify)
  int32_t* Bconst = nullptr;    // device ints holding B for row-count reads of dense (per-env) launches
  // round-owned ragged buffers (lazy)
  bool rb_ready = false;
  int32_t *row_ptr = nullptr, *row_t = nullptr, *row_env = nullptr, *t_next = nullptr, *n_acc = nullptr, *n_adv = nullptr;
  float *states = nullptr, *eps_p = nullptr, *eps_q = nullptr, *xi = nullptr, *y_last = nullptr;
  std::vector<void*> owned;
  // A round of more than a few rows computes the base network's per-row FiLM vectors (k_mod_gemm, bound by its output
  // stream) on a second stream of the same priority while the drafter rolls out: forked after the row table, joined
  // before the verify.
  hipStream_t aux = nullptr;
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;
  // optional kernel timing: events recorded around the dominant kernel of each stage
  bool timing = false;
  int timing_mask = 15;         // stages whose kernels are bracketed by events while timing is on (bit = stage)
  hipEvent_t ev[4][2] = {{nullptr, nullptr}, {nullptr, nullptr}, {nullptr, nullptr}, {nullptr, nullptr}};   // draft, verify, accept, FiLM GEMM
  bool ev_used[4] = {false, false, false, false};
};

namespace {

int fail(tsdp_ctx* c, int code, const std::string& msg) {
  if (c) c->err = msg;
  return code;
}

inline void tick(tsdp_ctx* c, int stage, int edge, hipStream_t s) {
  if (c->timing && ((c->timing_mask >> stage) & 1)) {
    (void)hipEventRecord(c->ev[stage][edge], s);
    c->ev_used[stage] = true;
  }
}

#define HIPCHK(c, expr)                                                                         \
  do {                                                                                          \
    hipError_t e_ = (expr);                                                                     \
    if (e_ != hipSuccess)                                                                       \
      return fail(c, e_ == hipErrorOutOfMemory ? TSDP_E_NOMEM : TSDP_E_HIP,                     \
                  std::string(#expr) + ": " + hipGetErrorString(e_));                           \
  } while (0)

template <typename T>
int dev_alloc(tsdp_ctx* c, T** p, size_t count) {
  void* v = nullptr;
  HIPCHK(c, hipMalloc(&v, (count ? count : 1) * sizeof(T)));
  c->owned.push_back(v);
  *p = static_cast<T*>(v);
  return TSDP_OK;
}

float bf16_round(float f) {
  uint32_t b;
  std::memcpy(&b, &f, 4);
  if ((b & 0x7F800000u) == 0x7F800000u) return f;     // inf / nan unchanged
  b = (b + 0x7FFFu + ((b >> 16) & 1u)) & 0xFFFF0000u;
  std::memcpy(&f, &b, 4);
  return f;
}


uint16_t bf16_bits(float f) {
  uint32_t b;
  std::memcpy(&b, &f, 4);
  b = (b + 0x7FFFu + ((b >> 16) & 1u)) >> 16;
  return (uint16_t)b;
}

// Fragment order of a logical [rows, K] matrix as MFMA A operands: [rows/16][Kpad/KSTEP][64 lanes][VW elements];
// lane l of fragment (mf, ks) holds row mf*16 + l%16, columns ks*KSTEP + (l/16)*VW .. +VW-1, with VW = 8 bf16
// (k-step 32) or VW = 4 fp32 (k-step 16).  src_row(lr) maps a logical row to a row of W (or -1 for a zero row).
// Offsets returned by the callers are in bytes of `out`.
template <typename RowMap>
void pack_frags(std::vector<uint8_t>& out, bool f32, const float* W, int K, int rows, RowMap src_row) {
  const int VW = f32 ? 4 : 8, KSTEP = 4 * VW, ES = f32 ? 4 : 2;
  const int mfs = (rows + 15) / 16, kss = (K + KSTEP - 1) / KSTEP;
  const size_t base = out.size();
  out.resize(base + (size_t)mfs * kss * 64 * VW * ES, 0);
  for (int mf = 0; mf < mfs; ++mf)
    for (int ks = 0; ks < kss; ++ks)
      for (int l = 0; l < 64; ++l) {
        const int lr = mf * 16 + (l & 15);
        const int sr = lr < rows ? src_row(lr) : -1;
        for (int i = 0; i < VW; ++i) {
          const int col = ks * KSTEP + (l >> 4) * VW + i;
          if (sr < 0 || col >= K) continue;
          const float v = W[(size_t)sr * K + col];
          uint8_t* dst = &out[base + ((((size_t)mf * kss + ks) * 64 + l) * VW + i) * ES];
          if (f32) {
            std::memcpy(dst, &v, 4);
          } else {
            const uint16_t b = bf16_bits(v);
            std::memcpy(dst, &b, 2);
          }
        }
      }
}

template <class C>
hipError_t launch_verify(const FusedNet& n, const FusedIO& io, int A, int R_cap, hipStream_t s) {
  auto kern = k_fused_forward<C>;
  static bool attr_set = false;
  if (!attr_set) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS_B);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  const int tiles = (R_cap + C::RPT - 1) / C::RPT;
  if (tiles > 0) hipLaunchKernelGGL(kern, dim3(tiles), dim3(C::THREADS), C::LDS_B, s, n, io, A);
  return hipSuccess;
}

template <class C, bool STAGED>
hipError_t launch_draft_as(const FusedNet& n, const DraftIO& io, int A, hipStream_t s) {
  auto kern = k_fused_draft<C, STAGED>;
  const int lds = DraftLds<C>::bytes(A, n.L, io.mod_cols, STAGED);
  static int attr_lds = 0;
  if (lds > attr_lds) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    attr_lds = lds;
  }
  const int tiles = (io.B + C::RPT - 1) / C::RPT;
  if (tiles > 0) hipLaunchKernelGGL(kern, dim3(tiles), dim3(C::THREADS), lds, s, n, io, A);
  return hipSuccess;
}

template <class C>
hipError_t launch_draft(const FusedNet& n, const DraftIO& io_in, int A, hipStream_t s) {
  typedef DraftLds<C> Lds;
  DraftIO io = io_in;
  // FiLM vectors of up to 16 / RPT steps per in-kernel product, as many as LDS has room for, then the token embedding
  io.mod_cols = C::RPT;
  for (int cols = 16; C::CM == 0 && cols > C::RPT; cols /= 2)
    if (cols % C::RPT == 0 && Lds::bytes(A, n.L, cols, Lds::ALWAYS) <= Lds::MOST) { io.mod_cols = cols; break; }
  if constexpr (!Lds::ALWAYS)
    if (Lds::bytes(A, n.L, io.mod_cols, true) > Lds::MOST) return launch_draft_as<C, false>(n, io, A, s);
  return launch_draft_as<C, true>(n, io, A, s);
}
template <class C>
bool draft_fits(int A, int L) { return DraftLds<C>::bytes(A, L, C::RPT, DraftLds<C>::ALWAYS) <= DraftLds<C>::MOST; }
template <class C, bool USED>
DraftTile draft_tile_of() {
  if constexpr (USED) return {launch_draft<C>, draft_fits<C>, C::RPT};
  else return {nullptr, nullptr, C::RPT};
}

template <int D>
void launch_mod(const FusedNet& n, const int32_t* t_arr, int t_sub, const int32_t* env_arr, int T, const int32_t* d_R,
                int R_cap, float* mod, hipStream_t s) {
  const int Nm = n.L * 4 * D;                           // a multiple of 256 because D is a multiple of 64
  constexpr int NR = 64;                                // rows per workgroup
  const int row_tiles = (R_cap + NR - 1) / NR;
  // output tiles of 256 features are dealt over blockIdx.x; enough workgroups for about twelve per CU at the row bound
  // (a ragged batch leaves the tiles beyond its live rows empty)
  const int fx = std::max(1, std::min(Nm / 256, (3072 + row_tiles - 1) / row_tiles));
  dim3 g(fx, row_tiles);
  hipLaunchKernelGGL((k_mod_gemm<D, NR>), g, dim3(256), 0, s, n.modw, n.modb, n.temb, n.cemb, t_arr, t_sub, env_arr, T, Nm, d_R,
                     R_cap, mod);
}

// slices of a run-time hidden width: eight where fragments of 16 allow it
inline int few_slices_dyn(int M) {
  int n = 8;
  while (M % (16 * n)) n /= 2;
  return n;
}

// From eight rows on all workgroups of a row sit on one XCD, whose L2 then holds the row's partial sums (32 rows of
// 32 x 512 with partial sums: round 2279 -> 1368 us; 8 rows of 16 x 256: no change); fewer rows are dealt over all of them.
constexpr int FEW_BY_ROW = 8;

// The launches of one spread forward pass: every kernel reads the residual and the partial sums its predecessor left
// and writes the other pair of buffers.
template <class C>
struct FewPass {
  typedef typename C::TT TT;
  const FusedNet& n;
  const FewRun& r;
  hipStream_t s;
  FewIO io{};
  DraftIO dr{};
  int at = 0;
  const int D = C::DYN ? n.D : C::D, heads = C::DYN ? n.heads : C::HEADS, nch = C::DYN ? few_slices_dyn(n.M) : C::NCH;
  const int la = few_lds_attn<TT>(D, C::H, D / heads), lm = few_lds_mlp<TT>(D, C::H, n.M / nch);

  FewPass(const FusedNet& n_, const FewRun& r_, hipStream_t s_) : n(n_), r(r_), s(s_) {
    io.by_row = r.R_cap >= FEW_BY_ROW;
    io.R_cap = r.R_cap; io.safe_rows = r.safe_rows; io.word = r.d_R; io.pstride = r.pstride;
    io.by_t = n.modtab != nullptr; io.mod_stride = n.L * 4 * D; io.row_t = r.row_t; io.T = r.T; io.row_env = r.row_env;
    io.x = r.x; io.tok_wt = n.tok_wt; io.tok_b = n.tok_b; io.pos = n.pos; io.A = r.A;
    io.head = n.head; io.head_b = n.head_b; io.eps_out = r.eps_out; io.kc = n.kc; io.vct = n.vct; io.L = n.L; io.rms = n.rms;
    io.D = D; io.DH = D / heads; io.heads = heads; io.M = n.M; io.CH = n.M / nch;
  }
  static constexpr int FIRST = C::WIDE ? 0 : C::NPM;   // residual that the previous MLP block left
  // buffers of the next launch: partial sums and residual change places; wide rows keep their residual where it is
  // (`move` where a launch starts a new one while its other workgroups may still read the old)
  void flip(bool move = false) {
    if (C::WIDE) {
      io.h_in = r.h[at];
      if (move) at ^= 1;
      io.h_out = r.h[at];
    } else {
      io.h_in = r.h[at]; io.part_in = r.part[at];
      at ^= 1;
      io.h_out = r.h[at]; io.part_out = r.part[at];
    }
  }
  int rows() const { return io.by_row ? (r.R_cap + 7) / 8 * 8 : r.R_cap; }
  // h += product of the activations the previous launch left, K of them per token
  template <int K>
  void out(const void* w, const float* bias) {
    if constexpr (C::WIDE) {
      flip();
      io.part_in = r.part[0]; io.w2 = w; io.bias_in = bias;
      hipLaunchKernelGGL((k_few_out<C, K>), dim3(rows() * (C::D / 64)), dim3(C::TH), C::NW * C::H * 64 * 4, s, io);
    } else {
      io.bias_in = bias;
    }
  }
  void start(bool ends_step) {
    const dim3 th(C::TH), ga(rows() * heads);
    if (ends_step) hipLaunchKernelGGL((k_few_attn<C, FIRST, true>), ga, th, la + FEW_STEP_LDS, s, io, dr);
    else hipLaunchKernelGGL((k_few_attn<C, FEW_EMBED>), ga, th, la + FEW_STEP_LDS, s, io, FewNone{});
  }
  // all layers; mod = FiLM vectors of row 0; ends_step: the first launch ends the rollout's previous transition
  void layers(const float* mod, bool ends_step) {
    const dim3 th(C::TH), ga(rows() * heads), gm(rows() * nch);
    if (C::WIDE) io.part_out = r.part[0];
    for (int l = 0; l < n.L; ++l) {
      const FusedLayer& w = n.layer[l];
      flip(l == 0);
      io.mod = mod + (size_t)l * 4 * D; io.w1 = w.qkv; io.b1 = w.qkv_b; io.w2 = w.o; io.layer = l; io.n_part = nch;
      if (l == 0) start(ends_step);
      else hipLaunchKernelGGL((k_few_attn<C, FIRST>), ga, th, la, s, io, FewNone{});
      out<C::D>(w.o, w.o_b);
      if constexpr (C::SX > 0) {
        flip();
        io.w1 = w.cq; io.b1 = w.cq_b; io.w2 = w.co;
        hipLaunchKernelGGL((k_few_cross<C, C::NPA>), ga, th, la, s, io);
        out<C::D>(w.co, w.co_b);
      }
      flip();
      io.mod += 2 * D; io.w1 = w.up; io.b1 = w.up_b; io.w2 = w.dn; io.n_part = heads;
      hipLaunchKernelGGL((k_few_mlp<C, C::NPA>), gm, th, lm, s, io);
      out<4 * C::D>(w.dn, w.dn_b);
    }
  }
  void head() {
    flip();
    io.n_part = nch;
    hipLaunchKernelGGL((k_few_head<C, FIRST>), dim3(r.R_cap), dim3(C::TH), lm, s, io);
  }
};

template <class C>
void few_forward(const FusedNet& n, const FewRun& r, hipStream_t s) {
  FewPass<C> p(n, r, s);
  p.layers(r.mod, false);
  p.head();
}

// The drafter's rollout as launches: 2 L per transition (3 L with cross-attention) and one that ends the last.  r.mod holds
// the FiLM vectors of every transition, [env][k_max] rows (unless they come from the table).
template <class C>
void few_draft(const FusedNet& n, const FewRun& r, const DraftIO& dr, int k_max, float* const* y, hipStream_t s) {
  FewPass<C> p(n, r, s);
  const int stride = n.L * 4 * p.D;
  p.dr = dr;
  p.io.word = dr.K_eff;
  p.io.roll = 1;
  p.io.x = dr.y;
  if (!p.io.by_t) p.io.mod_stride = k_max * stride;
  for (int k = 1; k <= k_max + 1; ++k) {
    p.io.step = k;
    p.io.t_sub = k - 1;
    p.io.y_in = k == 2 ? dr.y : y[(k - 1) & 1];
    p.io.y_out = y[k & 1];
    if (k <= k_max) {
      p.layers(p.io.by_t ? r.mod : r.mod + (size_t)(k - 1) * stride, k > 1);
    } else {
      p.flip(true);
      p.io.n_part = p.nch;
      p.start(true);
    }
  }
}

template <class TT, int D>
void launch_few_film(const FusedNet& n, const int32_t* t_arr, int t_sub, const int32_t* env_arr, int k_max, int T,
                     const int32_t* d_R, const int32_t* gate, int R_cap, float* mod, hipStream_t s) {
  const int d = D ? D : n.D, Nm = n.L * 4 * d;
  hipLaunchKernelGGL((k_few_film<TT, D>), dim3((Nm / 16 + 3) / 4, (R_cap + 15) / 16), dim3(256),
                     16 * (d + TT::PAD) * (int)sizeof(typename TT::elem), s, n.modw, n.modb, n.temb, n.cemb, t_arr, t_sub, env_arr,
                     k_max, T, d, Nm, d_R, gate, R_cap, mod);
}

// Workgroups of a one-launch pass, per XCD: four phases of its rows (one at work, the next ones waiting with their weights in
// registers; one C2 environment with 2, 3, 4 phases 282, 262, 260 us a round), two per compute unit at most.
// Up to eight rows (one per XCD) and in rollouts a workgroup asks for half a unit's LDS, so that no two share its matrix cores
// (8 rows 106 us a pass, 138 with two); with more rows the second one works while the first waits (64 rows 486 -> 300 us).
// The rows of an XCD are dealt to four groups of tasks: fewer leave units idle, eight have no row left to take in turn
// (64 rows of two layers 342, 385, 300, 351 us with 1, 2, 4, 8).
constexpr int FLOW_WGS = 64, FLOW_GROUPS = 4, FLOW_ALONE = 84 * 1024;
template <class C, bool ROLL> int flow_lds(int A, int R_cap) { return ROLL || R_cap <= 8 ? std::max(C::lds(A), FLOW_ALONE) : C::lds(A); }
template <class C, bool ROLL>
void flow_launch(const FusedNet& n, const FewRun& r, FlowIO& io, const std::conditional_t<ROLL, DraftIO, FewNone>& dr, int phases, hipStream_t s) {
  const int per_xcd = (r.R_cap + 7) / 8, lds = flow_lds<C, ROLL>(r.A, r.R_cap);
  io.R_cap = r.R_cap; io.phases = phases; io.groups = std::min(per_xcd, FLOW_GROUPS);
  io.ticket = r.sync; io.over = r.sync + FLOW_OVER_LINE * SYNC_LINE; io.owner = r.sync + FLOW_OWNER_LINE * SYNC_LINE; io.cnt = r.sync + FLOW_CNT_LINE * SYNC_LINE; io.status = r.status;
  io.x = r.x; io.row_t = r.row_t; io.row_env = r.row_env; io.T = r.T; io.A = r.A;
  io.mod = r.mod; io.mod_row = n.L * 4 * C::D; io.by_t = n.modtab != nullptr;
  io.buf = r.buf; io.eps_out = r.eps_out;
  const int wgs = 8 * std::min(4 * io.groups * C::G, FLOW_WGS);
  if (r.R_cap > 0)
    hipLaunchKernelGGL((k_flow<C, ROLL>), dim3(r.flow_wgs > 0 ? std::min(r.flow_wgs, wgs) : wgs), dim3(C::TH), lds, s, n, io, dr);
}
// Declares the largest LDS request of any context (H A <= 512) on the device that is current: at every load, so that a launch has
// nothing to set and contexts on several devices or with several A do not depend on each other.
template <class C, bool ROLL>
hipError_t flow_declare() {
  static_assert(C::lds(512 / C::H) + 16 <= 160 * 1024, "LDS");   // (16: the drawn ticket and set)
  return hipFuncSetAttribute((const void*)k_flow<C, ROLL>, hipFuncAttributeMaxDynamicSharedMemorySize, flow_lds<C, ROLL>(512 / C::H, 1));
}

template <class C>
void flow_forward(const FusedNet& n, const FewRun& r, hipStream_t s) {
  FlowIO io{};
  io.word = r.d_R;
  flow_launch<C, false>(n, r, io, FewNone{}, n.L * C::NPH + 1, s);
}

template <class C>
void flow_draft(const FusedNet& n, const FewRun& r, const DraftIO& dr, int k_max, float* const* y, hipStream_t s) {
  FlowIO io{};
  io.word = dr.K_eff; io.k_max = k_max; io.y[0] = y[0]; io.y[1] = y[1];
  FewRun rr = r;
  rr.x = dr.y;
  flow_launch<C, true>(n, rr, io, dr, k_max * n.L * C::NPH + 1, s);
}

// Run-time sizes, one workgroup per row or environment (k_row)
template <int NB>
RowIO row_io(const FusedNet& n, const FewRun& r, int k_max) {
  const unsigned cf = n.D / n.heads / 16;
  return RowIO{RowDiv(cf), RowDiv(3 * cf), RowDiv(n.D / 4), r.d_R, r.R_cap, r.A, NB * 16, n.D / n.heads, k_max, r.x, r.mod, r.eps_out};
}
template <int NB>
void row_forward(const FusedNet& n, const FewRun& r, hipStream_t s) {
  hipLaunchKernelGGL((k_row<NB, false>), dim3(r.R_cap), dim3(ROW_TH), row_lds(n.D, NB * 16, n.M, r.A, false).total * 4, s, n,
                     row_io<NB>(n, r, 0), FewNone{});
}
template <int NB>
void row_draft(const FusedNet& n, const FewRun& r, const DraftIO& dr, int k_max, float* const*, hipStream_t s) {
  hipLaunchKernelGGL((k_row<NB, true>), dim3(r.R_cap), dim3(ROW_TH), row_lds(n.D, NB * 16, n.M, r.A, true).total * 4, s, n,
                     row_io<NB>(n, r, k_max), dr);
}

struct FusedKernels {
  void (*few_forward)(const FusedNet&, const FewRun&, hipStream_t) = nullptr;
  void (*few_draft)(const FusedNet&, const FewRun&, const DraftIO&, int, float* const*, hipStream_t) = nullptr;
  void (*few_film)(const FusedNet&, const int32_t*, int, const int32_t*, int, int, const int32_t*, const int32_t*, int, float*, hipStream_t) = nullptr;
  int few_slices = 0;
  // the same in one launch, where a shape has it; bytes of a row's buffers
  void (*flow_forward)(const FusedNet&, const FewRun&, hipStream_t) = nullptr;
  void (*flow_draft)(const FusedNet&, const FewRun&, const DraftIO&, int, float* const*, hipStream_t) = nullptr;
  hipError_t (*flow_declare_forward)() = nullptr; hipError_t (*flow_declare_draft)() = nullptr;
  size_t flow_row = 0;
  // variant for batches of at most one tile per CU: one 8-wave workgroup per CU instead of two 4-wave ones
  hipError_t (*verify_few)(const FusedNet&, const FusedIO&, int, int, hipStream_t) = nullptr;
  int rpt_verify = 0;
  void (*mod)(const FusedNet&, const int32_t*, int, const int32_t*, int, const int32_t*, int, float*, hipStream_t) = nullptr;
  hipError_t (*verify)(const FusedNet&, const FusedIO&, int, int, hipStream_t) = nullptr;
  DraftTile draft_small, draft_big;
};

// The spread kernels of a compiled shape, where few_pays can choose them.
template <class TT, int D, int H, int HEADS, int SX>
void spread_kernels(FusedKernels& k) {
  constexpr bool F32 = std::is_same<TT, TF32>::value, NARROW = D * H < FEW_WIDE;
  if constexpr (layer_bytes(D, F32, SX > 0) >= FEW_LAYER_BYTES) {
    typedef FewCfg<TT, D, H, HEADS, SX> F;
    k.few_forward = few_forward<F>; k.few_draft = few_draft<F>; k.few_slices = std::max(F::NCH, F::HEADS);
    constexpr bool FORWARD = F32 || (SX == 0 && D >= 256 && NARROW) || (SX > 0 && !NARROW), DRAFT = F32 || (SX > 0 && NARROW);
    if constexpr (FORWARD || DRAFT) {
      typedef FlowCfg<TT, D, H, HEADS, SX> X;
      if constexpr (FORWARD) { k.flow_forward = flow_forward<X>; k.flow_declare_forward = flow_declare<X, false>; }
      if constexpr (DRAFT) { k.flow_draft = flow_draft<X>; k.flow_declare_draft = flow_declare<X, true>; }
      k.flow_row = 2 * X::SET_B;
    }
  }
}

// Measured tile choices of the compiled shapes.
constexpr int NWS128 = 8;        // waves of the one-environment drafter tile, d = 128
constexpr int NWS256X = 8;       // waves and heads per phase of the one-environment drafter tile, d = 256 with cross-attention
constexpr int HPS256X = 8;
constexpr int F256_NW = 8;       // fp32 d = 256 verify kernel: waves, heads per phase, hidden chunk
constexpr int F256_HP = 2;
constexpr int F256_CH = 256;
constexpr int FEW_TILES = 288;   // up to this many tiles the 8-wave verify variant (one workgroup per CU) is used
constexpr int V512_HPX = 8;      // heads per cross-attention phase of the d = 512 verify kernel
constexpr int V512_CH = 256;     // hidden-chunk width of the d = 512 verify kernel
// shapes with compiled fused kernels
bool find_fused(int dtype, int D, int H, int heads, int cm, int S, int mlp_ratio, int L, FusedKernels& k) {
  if (mlp_ratio != 4 || L > FUSED_MAX_LAYERS) return false;
#define TSDP_SHAPE(TT_, DT_, D_, H_, HD_, CM_, SX_, NTV, CHV, HPV, NWV, HPXV, NTS, CHS, HPS, NWS, NTB, CHB, HPB, NWD)  \
  if (dtype == DT_ && D == D_ && H == H_ && heads == HD_ && cm == CM_ && (CM_ == 0 || S == SX_)) {             \
    k.verify = launch_verify<FusedCfg<TT_, D_, NTV, H_, HD_, CM_, CHV, SX_, HPV, NWV, HPXV>>;                  \
    k.rpt_verify = NTV / H_;                                                                                   \
    spread_kernels<TT_, D_, H_, HD_, SX_>(k);                                                                  \
    k.few_film = launch_few_film<TT_, D_>;                                                                       \
    k.mod = DT_ == 1 ? launch_mod<D_> : nullptr;                                                               \
    k.draft_small = draft_tile_of<FusedCfg<TT_, D_, NTS, H_, HD_, CM_, CHS, SX_, HPS, NWS>, (D_ < 512)>();    \
    k.draft_big = draft_tile_of<FusedCfg<TT_, D_, NTB, H_, HD_, CM_, CHB, SX_, HPB, NWD>, DT_ == 0 || (D_ <= 192)>(); \
    return true;                                                                                               \
  }
  // The drafter's small tile (one environment per workgroup) is latency-bound: it takes all heads in one attention
  // phase and the whole MLP hidden layer in one chunk (d = 256 with cross-attention: half of it, 512; 1024 does not
  // fit the LDS), which minimises the number of barrier-separated phases; its four-environment tile at d = 192 takes
  // the hidden layer in two chunks of 384 (measured against 128 / 256: -15 % at d = 256, -3.5 % at d = 192).
  // Rollout tiles that lose to a forward pass per transition are not compiled: of many environments from d = 256 on (tsdp_draft, us, eight
  // transitions, two layers, tile / forward passes: 1024 environments of d = 256 671 / 656, four layers 1493 / 1171, d = 384 1341 / 1113; 512 of
  // d = 256 with cross-attention 880 / 870), of one at d = 512 (64 environments 1709 / 1513).
  //         type dtype  D   H heads cm  S | verify: NT  CH  HP NW HPX | draft small: NT CH HP NW | big: NT CH HP | NW
  if (dtype == 1 && D == 256 && H == 16 && heads == 4 && cm == 0)
    k.verify_few = launch_verify<FusedCfg<TBF16, 256, 64, 16, 4, 0, 256, 0, 2, 8>>;
  if (dtype == 1 && D == 384 && H == 16 && heads == 6 && cm == 0)
    k.verify_few = launch_verify<FusedCfg<TBF16, 384, 64, 16, 6, 0, 256, 0, 2, 8>>;
  TSDP_SHAPE(TBF16, 1, 256, 16, 4, 0, 0, 64, 128, 1, 4, 1, 16, 128, 1, 4, 64, 128, 1, 4)
  TSDP_SHAPE(TBF16, 1, 384, 16, 6, 0, 0, 64, 192, 1, 4, 1, 16, 128, 1, 4, 64, 128, 1, 4)
  TSDP_SHAPE(TBF16, 1, 128, 16, 4, 0, 0, 128, 128, 2, 4, 2, 16, 512, 4, NWS128, 64, 128, 2, 4)
  TSDP_SHAPE(TBF16, 1, 192, 16, 6, 0, 0, 128, 128, 2, 4, 2, 16, 768, 6, 4, 64, 384, 2, 4)
  TSDP_SHAPE(TBF16, 1, 512, 32, 8, 1, 64, 64, V512_CH, 2, 8, V512_HPX, 32, 128, 1, 4, 64, 128, 1, 4)
  TSDP_SHAPE(TBF16, 1, 256, 32, 8, 1, 64, 64, 256, 2, 4, 2, 32, 512, HPS256X, NWS256X, 64, 128, 2, 4)
  // fp32 networks on the fp32 matrix cores: one row (16 tokens) per workgroup, weights streamed per workgroup (d = 64: the hidden
  // layer in one phase, and the weights of a product requested before the phase ahead of it: tsdp_verify of 4 rows 23.4 -> 21.4 us)
  TSDP_SHAPE(TF32, 0, 256, 16, 4, 0, 0, 16, F256_CH, F256_HP, F256_NW, F256_HP, 16, 128, 1, 4, 16, 128, 1, 4)
  TSDP_SHAPE(TF32, 0, 128, 16, 4, 0, 0, 16, 128, 2, 4, 2, 16, 512, 4, NWS128, 16, 512, 4, 4)
  TSDP_SHAPE(TF32, 0, 64, 16, 2, 0, 0, 16, 256, 2, 4, 2, 16, 64, 2, 4, 16, 64, 2, 4)
  TSDP_SHAPE(TF32, 0, 32, 16, 2, 0, 0, 16, 32, 2, 2, 2, 16, 128, 2, 2, 16, 128, 2, 2)
#undef TSDP_SHAPE
  return false;
}

// rows of the ragged batch a context must hold: K_max per environment, one more with the bonus row
inline size_t rows_max(const tsdp_config& cf) { return (size_t)cf.B_max * (cf.K_max + (cf.bonus_row ? 1 : 0)); }

// A drafter of the base network's own shape takes the base network's kernels, so that equal weights give equal predictions.
inline bool twin_nets(const tsdp_config& cf) {
  return cf.base_d == cf.draft_d && cf.base_layers == cf.draft_layers && cf.base_heads == cf.draft_heads;
}
// tokens of the largest spread launch of a network with run-time sizes: the rollout has one row per environment
inline size_t dyn_tokens(const tsdp_config& cf, int which) {
  return (which == 1 && !twin_nets(cf) ? (size_t)cf.B_max : rows_max(cf)) * cf.H;
}

// Shapes without a compiled kernel: the kernels with run-time sizes where few_dyn_pays says so (vector conditioning, sizes in
// fragments of 16, a row's operands in the LDS; 48 and 64 tokens would spill the residual): one workgroup per row where row_pays
// says so, else the spread ones.
template <int NB>
hipError_t row_kernels(FusedKernels& k) {
  k.few_forward = row_forward<NB>; k.few_draft = row_draft<NB>; k.few_film = launch_few_film<TF32, 0>;
  for (const void* f : {(const void*)k_row<NB, false>, (const void*)k_row<NB, true>, (const void*)k_few_film<TF32, 0>})
    if (hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)) return e;
  return hipSuccess;
}
template <class C>
hipError_t few_dyn_kernels(FusedKernels& k) {
  k.few_forward = few_forward<C>; k.few_draft = few_draft<C>; k.few_film = launch_few_film<TF32, 0>;
  for (const void* f : {(const void*)k_few_attn<C, FEW_EMBED>, (const void*)k_few_attn<C, 1>, (const void*)k_few_attn<C, 1, true>,
                        (const void*)k_few_mlp<C, 1>, (const void*)k_few_head<C, 1>, (const void*)k_few_film<TF32, 0>})
    if (hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)) return e;
  return hipSuccess;
}

hipError_t find_few_dyn(const tsdp_config& cf, int which, const Net& n, FusedKernels& k) {
  const int dh = n.d / n.heads, ch = n.m % 16 ? 0 : n.m / few_slices_dyn(n.m);
  const size_t bytes = 4 * ((size_t)4 * n.d * n.d + (size_t)2 * n.d * n.m);
  if (cf.cond_mode != 0 || (cf.H != 16 && cf.H != 32) || n.d % 16 || dh % 16 || n.m % 16 || n.L > FUSED_MAX_LAYERS ||
      few_lds_attn<TF32>(n.d, cf.H, dh) + FEW_STEP_LDS > 160 * 1024 || few_lds_mlp<TF32>(n.d, cf.H, ch) > 160 * 1024 ||
      !few_dyn_pays(dyn_tokens(cf, which), n.heads, bytes))
    return hipSuccess;
  // (twins: both of them or neither)
  if (row_pays(dyn_tokens(cf, which), cf.H, bytes, n.heads) && n.d <= ROW_MAX_D && 5 * n.d + n.m <= ROW_MAX_BIAS &&
      row_lds(n.d, cf.H, n.m, cf.A, true).total * 4 <= 160 * 1024)
    return cf.H == 16 ? row_kernels<1>(k) : row_kernels<2>(k);
  k.few_slices = std::max(n.heads, few_slices_dyn(n.m));
  return cf.H == 16 ? few_dyn_kernels<FewDyn<1>>(k) : few_dyn_kernels<FewDyn<2>>(k);
}

size_t layout_net(const tsdp_config& cf, int which, Net& n) {
  n.L = which == 0 ? cf.base_layers : cf.draft_layers;
  n.d = which == 0 ? cf.base_d : cf.draft_d;
  n.heads = which == 0 ? cf.base_heads : cf.draft_heads;
  n.m = (which == 0 ? cf.base_mlp_ratio : cf.draft_mlp_ratio) * n.d;
  const size_t d = n.d, m = n.m, A = cf.A, H = cf.H, C = cf.cond_dim;
  size_t o = 0;
  auto take = [&](size_t cnt) { size_t r = o; o += cnt; return r; };
  n.tok_w = take(d * A); n.tok_b = take(d); n.pos = take(H * d);
  n.t_w1 = take(d * d); n.t_b1 = take(d); n.t_w2 = take(d * d); n.t_b2 = take(d);
  n.c_w = n.c_b = 0;
  if (cf.cond_mode == 0) { n.c_w = take(d * C); n.c_b = take(d); }
  n.lay.resize(n.L);
  for (auto& l : n.lay) {
    l.mod_w = take(4 * d * d); l.mod_b = take(4 * d);
    l.qkv_w = take(3 * d * d); l.qkv_b = take(3 * d);
    l.o_w = take(d * d); l.o_b = take(d);
    if (cf.cond_mode == 1) {
      l.cq_w = take(d * d); l.cq_b = take(d);
      l.ck_w = take(d * C); l.ck_b = take(d);
      l.cv_w = take(d * C); l.cv_b = take(d);
      l.co_w = take(d * d); l.co_b = take(d);
    }
    l.up_w = take(m * d); l.up_b = take(m);
    l.dn_w = take(d * m); l.dn_b = take(d);
  }
  n.head_w = take(A * d); n.head_b = take(A);
  n.n_floats = o;
  return o;
}


// Packs one network for the fused kernel (weights as bf16 MFMA fragments, q|k|v rows grouped per head
// group) and fills n.fnet.  `w` is the host copy of the bf16-rounded canonical blob.
int build_fused(tsdp_ctx* c, Net& n, const std::vector<float>& w, const std::vector<float>& modw_cat, const FusedKernels& fk) {
  const tsdp_config& cf = c->cfg;
  const int d = n.d, m = n.m, L = n.L, DH = d / n.heads;
  const bool dyn = !fk.verify, f32 = dyn || cf.dtype == 0;   // run-time sizes: fp32 operands, as in the operator kernels
  std::vector<uint8_t> pk;
  // q|k|v biases of a layer; run-time sizes: the other biases behind them (output projection, down, up)
  const size_t nb = dyn ? 5 * (size_t)d + m : 3 * (size_t)d;
  std::vector<float> qb(L * nb);
  struct Off { size_t qkv, o, up, dn, cq, co; };
  std::vector<Off> off(L);
  auto ident = [](int r) { return r; };
  for (int l = 0; l < L; ++l) {
    const LayerOff& o = n.lay[l];
    // logical row lr of the q|k|v matrix: per head [q(DH) k(DH) v(DH)]
    auto qkv_row = [&](int lr) {
      const int head = lr / (3 * DH), cls = (lr / DH) % 3, cdim = lr % DH;
      return cls * d + head * DH + cdim;
    };
    off[l].qkv = pk.size(); pack_frags(pk, f32, &w[o.qkv_w], d, 3 * d, qkv_row);
    for (int lr = 0; lr < 3 * d; ++lr) qb[l * nb + lr] = w[o.qkv_b + qkv_row(lr)];
    if (dyn) {
      std::copy_n(&w[o.o_b], d, &qb[l * nb + 3 * d]);
      std::copy_n(&w[o.dn_b], d, &qb[l * nb + 4 * d]);
      std::copy_n(&w[o.up_b], m, &qb[l * nb + 5 * d]);
    }
    off[l].o = pk.size(); pack_frags(pk, f32, &w[o.o_w], d, d, ident);
    off[l].up = pk.size(); pack_frags(pk, f32, &w[o.up_w], d, m, ident);
    off[l].dn = pk.size(); pack_frags(pk, f32, &w[o.dn_w], m, d, ident);
    if (cf.cond_mode == 1) {
      off[l].cq = pk.size(); pack_frags(pk, f32, &w[o.cq_w], d, d, ident);
      off[l].co = pk.size(); pack_frags(pk, f32, &w[o.co_w], d, d, ident);
    }
  }
  const size_t head_off = pk.size();
  pack_frags(pk, f32, &w[n.head_w], d, (cf.A + 15) / 16 * 16, [&](int r) { return r < cf.A ? r : -1; });
  const size_t mod_off = pk.size();
  pack_frags(pk, f32, modw_cat.data(), d, L * 4 * d, ident);
  uint8_t* dpk = nullptr;
  float* dqb = nullptr;
  int rc;
  if ((rc = dev_alloc(c, &dpk, pk.size()))) return rc;
  if ((rc = dev_alloc(c, &dqb, qb.size()))) return rc;
  HIPCHK(c, hipMemcpy(dpk, pk.data(), pk.size(), hipMemcpyHostToDevice));
  HIPCHK(c, hipMemcpy(dqb, qb.data(), qb.size() * sizeof(float), hipMemcpyHostToDevice));
  FusedNet& f = n.fnet;
  std::memset(&f, 0, sizeof(f));
  f.L = L; f.D = d; f.heads = n.heads; f.M = m;
  auto P = [&](size_t o) { return reinterpret_cast<const void*>(dpk + o); };
  for (int l = 0; l < L; ++l) {
    const LayerOff& o = n.lay[l];
    FusedLayer& fl = f.layer[l];
    fl.qkv = P(off[l].qkv); fl.o = P(off[l].o); fl.up = P(off[l].up); fl.dn = P(off[l].dn);
    fl.qkv_b = dqb + l * nb;
    fl.o_b = n.blob + o.o_b; fl.up_b = n.blob + o.up_b; fl.dn_b = n.blob + o.dn_b;
    if (cf.cond_mode == 1) {
      fl.cq = P(off[l].cq); fl.co = P(off[l].co);
      fl.cq_b = n.blob + o.cq_b; fl.co_b = n.blob + o.co_b;
    }
  }
  std::vector<float> tokt((size_t)cf.A * d);
  for (int i = 0; i < d; ++i)
    for (int a = 0; a < cf.A; ++a) tokt[(size_t)a * d + i] = w[n.tok_w + (size_t)i * cf.A + a];
  if (!n.tok_wt && (rc = dev_alloc(c, &n.tok_wt, tokt.size()))) return rc;
  HIPCHK(c, hipMemcpy(n.tok_wt, tokt.data(), tokt.size() * sizeof(float), hipMemcpyHostToDevice));
  f.tok_wt = n.tok_wt;
  f.tok_b = n.blob + n.tok_b; f.pos = n.blob + n.pos;
  f.head = P(head_off); f.head_b = n.blob + n.head_b;
  f.modtab = nullptr;
  f.rms = cf.norm;
  f.modw = P(mod_off); f.modb = n.modb; f.temb = n.temb; f.cemb = cf.cond_mode == 0 ? n.cemb : nullptr;
  if (cf.cond_mode == 1) {
    const size_t S = cf.cond_tokens, cnt = (size_t)cf.B_max * L * S * d;
    if (!n.kc_pk && (rc = dev_alloc(c, &n.kc_pk, cnt))) return rc;
    if (!c->cond_size && (rc = dev_alloc(c, &c->cond_size, (size_t)cf.B_max * S))) return rc;
    if (!n.vct_pk && (rc = dev_alloc(c, &n.vct_pk, cnt))) return rc;
    // key / value projections, per layer the key rows then the value rows (k_cond_kv)
    std::vector<uint8_t> kv;
    std::vector<float> kvb;
    for (int l = 0; l < L; ++l) {
      const LayerOff& o = n.lay[l];
      pack_frags(kv, false, &w[o.ck_w], cf.cond_dim, d, ident);
      pack_frags(kv, false, &w[o.cv_w], cf.cond_dim, d, ident);
      kvb.insert(kvb.end(), &w[o.ck_b], &w[o.ck_b] + d);
      kvb.insert(kvb.end(), &w[o.cv_b], &w[o.cv_b] + d);
    }
    for (int l = 0; l < L; ++l)
      for (const size_t at : {n.lay[l].ck_w, n.lay[l].cv_w})
        for (int r = 0; r < d; ++r) {
          double q = 0.0;
          for (int k = 0; k < cf.cond_dim; ++k) { const double v = w[at + (size_t)r * cf.cond_dim + k]; q += v * v; }
          kvb.push_back((float)std::sqrt(q));
        }
    if (!n.kv_w && (rc = dev_alloc(c, &n.kv_w, kv.size()))) return rc;
    if (!n.kv_b && (rc = dev_alloc(c, &n.kv_b, kvb.size()))) return rc;
    HIPCHK(c, hipMemcpy(n.kv_w, kv.data(), kv.size(), hipMemcpyHostToDevice));
    HIPCHK(c, hipMemcpy(n.kv_b, kvb.data(), kvb.size() * sizeof(float), hipMemcpyHostToDevice));
    HIPCHK(c, hipFuncSetAttribute(reinterpret_cast<const void*>(k_cond_kv), hipFuncAttributeMaxDynamicSharedMemorySize, COND_LDS));
    f.kc = reinterpret_cast<const bf16x8*>(n.kc_pk);
    f.vct = reinterpret_cast<const bf16x4*>(n.vct_pk);
  }
  n.fused = !dyn;
  n.fused_verify = fk.verify;
  n.fused_verify_few = fk.verify_few;
  n.verify_rpt = fk.rpt_verify;
  n.fused_mod = fk.mod;
  n.draft_small = fk.draft_small; n.draft_big = fk.draft_big;
  for (DraftTile* t : {&n.draft_small, &n.draft_big}) t->fits = t->fits_of && t->fits_of(cf.A, L);
  n.few_forward = fk.few_forward; n.few_draft = fk.few_draft; n.few_film = fk.few_film; n.few_slices = fk.few_slices; n.flow_row = 0;
  // Few rows: the spread kernels.  The capacity of the context decides, not the call: an environment's result must not
  // depend on the batch it is computed in.
  n.few = dyn || few_pays(rows_max(cf) * cf.H, f32, layer_bytes(d, f32, cf.cond_mode == 1));
  // The rollout: fp32 layers are bound by one unit's matrix rate (d = 128: 37 us per transition, in launches 23, in one launch
  // 17), and so are those with cross-attention by one unit's weight stream; bf16 drafters with a conditioning vector are not
  // (d = 192: spread 2 us per transition slower).  Twins are both in one launch, both in two launches per layer or neither.
  const bool base = &n == &c->net[0], twin = twin_nets(cf);
  const bool launches = dyn || few_rollout_pays(cf.draft_layers, (size_t)cf.draft_d * cf.H >= FEW_WIDE, cf.cond_mode == 1, cf.K_max);
  const bool one_forward = n.few && fk.flow_forward && flow_forward_pays(rows_max(cf) * cf.H, f32, d, L);
  const bool one_draft = (n.few || !f32) && fk.flow_draft && flow_draft_pays(cf.B_max, f32, d, L, cf.K_max, launches);
  // (twins whose rollout would be the persistent kernel: it gains a multiple of what the forward pass can lose -- four layers of
  // d = 256, 16 environments, K = 8: tsdp_draft 2240 -> 644 us, tsdp_verify 243 -> 279)
  const bool one = twin ? fk.flow_forward && one_draft && (one_forward || !launches) : base ? one_forward : one_draft;
  if (one) {
    if (base) {
      n.few_forward = fk.flow_forward;
      HIPCHK(c, fk.flow_declare_forward());
    } else {
      n.few_draft = fk.flow_draft;
      HIPCHK(c, fk.flow_declare_draft());
    }
    n.flow_row = fk.flow_row;
  }
  if (twin && !launches && !one) n.few = false;
  n.few_roll = !base && (one || (n.few && launches && (twin || f32)));
  if (!base) n.few = n.few_roll;
  if (!dyn) n.path = f32 ? "f32-mfma-fused" : "bf16-mfma-fused";
  return TSDP_OK;
}

inline dim3 grid1(long long n, int bs) { return dim3((unsigned)((n + bs - 1) / bs)); }

template <int EPI>
void linear(hipStream_t s, const float* in, const float* W, const float* bias, float* out, int units_cap,
            int rows_per_unit, int N, int K, const int32_t* d_R) {
  const long long M = (long long)units_cap * rows_per_unit;
  dim3 g((N + 63) / 64, (unsigned)((M + 63) / 64));
  hipLaunchKernelGGL(k_linear<EPI>, g, dim3(256), 0, s, in, W, bias, out, rows_per_unit, N, K, d_R, units_cap);
}

// eps[R,H,A] = network(x_rows; t, cond) with the fp32 operator kernels.
void forward_f32(tsdp_ctx* c, Net& n, const float* x_rows, int R_cap, const int32_t* d_R, const int32_t* t_arr,
                 int t_sub, const int32_t* env_arr, float* eps_out, hipStream_t s) {
  const tsdp_config& cf = c->cfg;
  const int H = cf.H, A = cf.A, d = n.d, L = n.L, m = n.m, dh = n.d / n.heads;
  const long long M = (long long)R_cap * H;
  const float* w = n.blob;
  hipLaunchKernelGGL(k_embed, grid1(M * d, 256), dim3(256), 0, s, x_rows, w + n.tok_w, w + n.tok_b, w + n.pos, c->h,
                     H, A, d, d_R, R_cap);
  hipLaunchKernelGGL(k_gvec, grid1((long long)R_cap * d, 256), dim3(256), 0, s, t_arr, t_sub, env_arr, n.temb,
                     cf.cond_mode == 0 ? n.cemb : nullptr, c->sg, d, cf.T, d_R, R_cap);
  const int ms = L * 4 * d;                         // modulation row stride
  linear<0>(s, c->sg, n.modw, n.modb, c->mod, R_cap, 1, ms, d, d_R);
  const dim3 lng((unsigned)((M + 3) / 4));
  for (int l = 0; l < L; ++l) {
    const LayerOff& o = n.lay[l];
    const float* mod = c->mod + (size_t)l * 4 * d;
    hipLaunchKernelGGL(k_lnmod, lng, dim3(256), 0, s, c->h, mod, mod + d, ms, c->a, H, d, cf.norm, d_R, R_cap);
    linear<0>(s, c->a, w + o.qkv_w, w + o.qkv_b, c->qkv, R_cap, H, 3 * d, d, d_R);
    hipLaunchKernelGGL(k_attn, dim3(R_cap, n.heads), dim3(256), H * H * sizeof(float), s, c->qkv, 3 * d, c->qkv + d,
                       c->qkv + 2 * d, 3 * d, (const int32_t*)nullptr, c->ao, d, H, H, dh, d_R, R_cap);
    linear<2>(s, c->ao, w + o.o_w, w + o.o_b, c->h, R_cap, H, d, d, d_R);
    if (cf.cond_mode == 1) {
      const int S = cf.cond_tokens;
      const size_t per_layer = (size_t)cf.B_max * S * d;
      hipLaunchKernelGGL(k_lnmod, lng, dim3(256), 0, s, c->h, (const float*)nullptr, (const float*)nullptr, 0, c->a, H, d, cf.norm, d_R, R_cap);
      linear<0>(s, c->a, w + o.cq_w, w + o.cq_b, c->qkv, R_cap, H, d, d, d_R);
      hipLaunchKernelGGL(k_attn, dim3(R_cap, n.heads), dim3(256), H * S * sizeof(float), s, c->qkv, d,
                         n.kc + l * per_layer, n.vc + l * per_layer, d, env_arr, c->ao, d, H, S, dh, d_R, R_cap);
      linear<2>(s, c->ao, w + o.co_w, w + o.co_b, c->h, R_cap, H, d, d, d_R);
    }
    hipLaunchKernelGGL(k_lnmod, lng, dim3(256), 0, s, c->h, mod + 2 * d, mod + 3 * d, ms, c->a, H, d, cf.norm, d_R, R_cap);
    linear<1>(s, c->a, w + o.up_w, w + o.up_b, c->u, R_cap, H, m, d, d_R);
    linear<2>(s, c->u, w + o.dn_w, w + o.dn_b, c->h, R_cap, H, d, m, d_R);
  }
  hipLaunchKernelGGL(k_lnmod, lng, dim3(256), 0, s, c->h, (const float*)nullptr, (const float*)nullptr, 0, c->a, H, d, cf.norm, d_R, R_cap);
  linear<0>(s, c->a, w + n.head_w, w + n.head_b, eps_out, R_cap, H, A, d, d_R);
}

FewRun few_run(tsdp_ctx* c, const Net& n, int R_cap, int safe_rows, const int32_t* t_arr, const int32_t* env_arr, const float* mod) {
  FewRun r{};
  r.row_t = t_arr; r.row_env = env_arr; r.R_cap = R_cap; r.safe_rows = safe_rows;
  r.A = c->cfg.A; r.T = c->cfg.T; r.mod = n.fnet.modtab ? n.fnet.modtab : mod;
  for (int i = 0; i < 2; ++i) { r.h[i] = c->few_h[i]; r.part[i] = c->few_part[i]; }
  r.pstride = (size_t)R_cap * c->cfg.H * n.d;
  r.sync = c->sync + (&n == &c->net[1] ? (size_t)flow_lines(rows_max(c->cfg)) * SYNC_LINE : 0);
  r.buf = c->flow_buf; r.status = c->status; r.flow_wgs = c->flow_wgs;
  return r;
}

// eps[R,H,A] = network(x_rows; t, cond): fused bf16 MFMA kernel where the shape has one, fp32 operators otherwise.
// mod_ready: the FiLM vectors of these rows are already in c->mod (computed on the auxiliary stream; the caller has
// made `s` wait for them)
int forward(tsdp_ctx* c, Net& n, const float* x_rows, int R_cap, const int32_t* d_R, const int32_t* t_arr,
            int t_sub, const int32_t* env_arr, float* eps_out, hipStream_t s, bool mod_ready = false, int safe_rows = 0) {
  if (!n.fused && !n.few) {
    forward_f32(c, n, x_rows, R_cap, d_R, t_arr, t_sub, env_arr, eps_out, s);
    return TSDP_OK;
  }
  const tsdp_config& cf = c->cfg;
  if (n.fnet.modtab || mod_ready) {
    // token conditioning: the FiLM vectors are a function of the timestep only and were tabulated at load time
  } else {
    const bool timed = &n == &c->net[0] && n.fused_mod;
    if (timed) tick(c, 3, 0, s);
    if (n.fused_mod && !n.few) n.fused_mod(n.fnet, t_arr, t_sub, env_arr, cf.T, d_R, R_cap, c->mod, s);
    else n.few_film(n.fnet, t_arr, t_sub, env_arr, 0, cf.T, d_R, nullptr, R_cap, c->mod, s);   // few rows; fp32 networks
    if (timed) tick(c, 3, 1, s);
  }
  const int stage = (&n == &c->net[0]) ? 1 : -1;          // only the base network's forward is the verify stage
  if (n.few) {                                        // (the base network: a drafter that is `few` rolls out in draft_impl)
    FewRun r = few_run(c, n, R_cap, safe_rows, t_arr, env_arr, c->mod);
    r.x = x_rows; r.d_R = d_R; r.eps_out = eps_out;
    tick(c, 1, 0, s);
    n.few_forward(n.fnet, r, s);
    tick(c, 1, 1, s);
    return TSDP_OK;
  }
  FusedIO io;
  io.x_rows = x_rows; io.mod = c->mod; io.row_t = t_arr; io.t_sub = t_sub; io.T = cf.T; io.row_env = env_arr; io.d_R = d_R; io.R_cap = R_cap; io.eps_out = eps_out;
  if (stage == 1) tick(c, 1, 0, s);
  const bool few = n.fused_verify_few && (R_cap + n.verify_rpt - 1) / n.verify_rpt <= FEW_TILES;
  HIPCHK(c, (few ? n.fused_verify_few : n.fused_verify)(n.fnet, io, cf.A, R_cap, s));
  if (stage == 1) tick(c, 1, 1, s);
  return TSDP_OK;
}

// Tile of the persistent rollout for B environments; null: a forward pass per transition, in the verify kernel's tiles.  From 192 of
// the tiles of many environments on these fill the chip; where a network is too large for one or has none, the verify kernel's tiles of 64 or 128
// tokens stream the weights less often than tiles of one environment.  tsdp_draft, us, eight transitions of 1024 environments, one / four
// environments a workgroup / forward passes: d = 128, 2 and 9 layers 443 / 283 / 569, 1577 / 1251 / 2017; d = 192, 2, 4 and 5 layers 877 / 449 / 883,
// 1600 / 958 / 1595, 2384 / - / 2048.
const DraftTile* draft_tile(const Net& n, int B) {
  if (!n.fused) return nullptr;
  const DraftTile& t = (B + n.draft_big.rpt - 1) / n.draft_big.rpt >= 192 ? n.draft_big : n.draft_small;
  return t.fits ? &t : nullptr;
}

int sync_lines(const tsdp_ctx* c) { return flow_lines(rows_max(c->cfg)) + flow_lines(c->cfg.B_max); }

int ensure_few(tsdp_ctx* c) {
  const tsdp_config& cf = c->cfg;
  int rc;
  const Net &bn = c->net[0], &dn = c->net[1];
  auto shape = [&](const Net& n, int which) { return FewShape{n.few && !n.flow_row && n.few_slices, n.fused ? rows_max(cf) * cf.H : dyn_tokens(cf, which), (size_t)n.d, (size_t)n.few_slices}; };
  const FewSize need = few_size(shape(bn, 0), shape(dn, 1));
  if (!few_fits(c->few_have, need)) {                  // (buffers that are replaced live as long as the context: a graph may hold them)
    const FewSize z{std::max(need.h, c->few_have.h), std::max(need.part, c->few_have.part)};
    float *h[2], *part[2];
    for (int i = 0; i < 2; ++i) {
      if ((rc = dev_alloc(c, &h[i], z.h))) return rc;
      if ((rc = dev_alloc(c, &part[i], z.part))) return rc;
    }
    for (int i = 0; i < 2; ++i) { c->few_h[i] = h[i]; c->few_part[i] = part[i]; }
    c->few_have = z;
  }
  for (float*& y : c->few_y)
    if (dn.few_roll && !y && (rc = dev_alloc(c, &y, (size_t)cf.B_max * c->D))) return rc;
  const size_t flow = std::max(bn.few ? rows_max(cf) * bn.flow_row : 0, dn.few ? cf.B_max * dn.flow_row : 0);
  if (flow > c->flow_have) {
    unsigned char* buf;
    if ((rc = dev_alloc(c, &buf, flow))) return rc;
    HIPCHK(c, hipMemset(buf, 0xFF, flow));               // FLOW_EMPTY
    HIPCHK(c, hipStreamSynchronize(nullptr));
    if (!c->sync && (rc = dev_alloc(c, &c->sync, (size_t)sync_lines(c) * SYNC_LINE))) return rc;
    c->flow_buf = buf;
    c->flow_have = flow;
  }
  if (dn.few_roll && cf.cond_mode == 0 && !c->few_mod &&
      (rc = dev_alloc(c, &c->few_mod, (size_t)cf.B_max * cf.K_max * dn.L * 4 * dn.d)))
    return rc;
  return TSDP_OK;
}

int ensure_workspace(tsdp_ctx* c) {
  if (int rc = ensure_few(c)) return rc;
  if (c->ws_ready) return TSDP_OK;
  const tsdp_config& cf = c->cfg;
  const size_t Rw = rows_max(cf), Mw = Rw * cf.H;
  const size_t dmax = std::max(cf.base_d, cf.draft_d);
  const size_t mmax = std::max(c->net[0].m, c->net[1].m);
  const size_t lmax = std::max(cf.base_layers, cf.draft_layers);
  int rc;
  if ((rc = dev_alloc(c, &c->h, Mw * dmax))) return rc;
  if ((rc = dev_alloc(c, &c->a, Mw * dmax))) return rc;
  if ((rc = dev_alloc(c, &c->qkv, Mw * 3 * dmax))) return rc;
  if ((rc = dev_alloc(c, &c->ao, Mw * dmax))) return rc;
  if ((rc = dev_alloc(c, &c->u, Mw * mmax))) return rc;
  if ((rc = dev_alloc(c, &c->sg, Rw * dmax))) return rc;
  if ((rc = dev_alloc(c, &c->mod, Rw * lmax * 4 * dmax))) return rc;
  if ((rc = dev_alloc(c, &c->eps_tmp, (size_t)cf.B_max * c->D))) return rc;
  if ((rc = dev_alloc(c, &c->row_t_chk, Rw))) return rc;
  if ((rc = dev_alloc(c, &c->row_env_chk, Rw))) return rc;
  c->ws_ready = true;
  return TSDP_OK;
}

int ensure_round_buffers(tsdp_ctx* c) {
  if (c->rb_ready) return TSDP_OK;
  const tsdp_config& cf = c->cfg;
  const size_t Rw = rows_max(cf), B = cf.B_max, D = c->D;
  int rc;
  if ((rc = dev_alloc(c, &c->row_ptr, B + 1))) return rc;
  if ((rc = dev_alloc(c, &c->row_t, Rw))) return rc;
  if ((rc = dev_alloc(c, &c->row_env, Rw))) return rc;
  if ((rc = dev_alloc(c, &c->t_next, B))) return rc;
  if ((rc = dev_alloc(c, &c->n_acc, B))) return rc;
  if ((rc = dev_alloc(c, &c->n_adv, B))) return rc;
  if ((rc = dev_alloc(c, &c->states, Rw * D))) return rc;
  if ((rc = dev_alloc(c, &c->eps_p, Rw * D))) return rc;
  if ((rc = dev_alloc(c, &c->eps_q, Rw * D))) return rc;
  if ((rc = dev_alloc(c, &c->xi, Rw * D))) return rc;
  if ((rc = dev_alloc(c, &c->y_last, B * D))) return rc;
  c->rb_ready = true;
  return TSDP_OK;
}

int check_ready(tsdp_ctx* c, int B, bool need_nets) {
  if (!c) return TSDP_E_INVAL;
  if (B < 0 || B > c->cfg.B_max) return fail(c, TSDP_E_SHAPE, "B outside 0..B_max");
  if (need_nets) {
    if (!c->net[0].loaded || !c->net[1].loaded) return fail(c, TSDP_E_STATE, "weights of both networks must be loaded");
    if (!c->cond_set) return fail(c, TSDP_E_STATE, "tsdp_set_cond has not been called");
    if (B > c->cond_B) return fail(c, TSDP_E_SHAPE, "B exceeds the batch given to tsdp_set_cond");
  }
  return TSDP_OK;
}

}  // namespace

extern "C" {

int tsdp_create(const tsdp_config* cfg, tsdp_ctx** out) {
  if (!cfg || !out) return TSDP_E_INVAL;
  *out = nullptr;
  const tsdp_config& f = *cfg;
  auto bad = [&](int d, int heads, int L, int mr) {
    return L < 1 || L > 64 || d < 8 || d > 1024 || d % 4 || heads < 1 || d % heads || (d / heads) > 128 || mr < 1 || mr > 8;
  };
  if (f.dtype < 0 || f.dtype > 1 || f.H < 1 || f.H > 64 || f.A < 1 || f.A > 64 || (f.H * f.A) % 4 || f.H * f.A > 512 || f.cond_mode < 0 ||
      f.cond_mode > 1 || f.cond_dim < 4 || f.cond_dim % 4 || (f.cond_mode == 1 && (f.cond_tokens < 1 || f.cond_tokens > 256)) ||
      bad(f.base_d, f.base_heads, f.base_layers, f.base_mlp_ratio) ||
      bad(f.draft_d, f.draft_heads, f.draft_layers, f.draft_mlp_ratio) || f.T < 1 || f.T > 4096 || f.schedule < 0 ||
      f.schedule > 1 || f.B_max < 1 || f.K_max < 1 || f.K_max > MAX_DRAFTS || (f.clip_x0 && !(f.clip_val > 0.0f)))
    return TSDP_E_INVAL;
  if (f.sampler < 0 || f.sampler > 1 || (f.sampler == 1 && !(f.eta > 0.0f && f.eta <= 1.0f))) return TSDP_E_INVAL;
  if (f.schedule == 0 && !(f.beta0 > 0.0f && f.beta1 >= f.beta0 && f.beta1 < 1.0f)) return TSDP_E_INVAL;
  if (f.bonus_row < 0 || f.bonus_row > 1 || f.norm < 0 || f.norm > 1) return TSDP_E_INVAL;
  if ((long long)f.B_max * (f.K_max + 1) > (1ll << 24)) return TSDP_E_SHAPE;
  tsdp_ctx* c = new (std::nothrow) tsdp_ctx();
  if (!c) return TSDP_E_NOMEM;
  c->cfg = f;
  c->D = f.H * f.A;
  layout_net(f, 0, c->net[0]);
  layout_net(f, 1, c->net[1]);
  // DDPM tables: textbook epsilon-prediction posterior with the fixed-small variance, fp64 then fp32
  const int T = f.T;
  std::vector<double> beta(T), abar(T);
  const double PI = 3.14159265358979323846;
  for (int i = 0; i < T; ++i) {
    if (f.schedule == 0) {
      beta[i] = T == 1 ? (double)f.beta0 : (double)f.beta0 + ((double)f.beta1 - (double)f.beta0) * i / (T - 1);
    } else {
      auto fc = [&](double j) { double v = std::cos(((j / T) + 0.008) / 1.008 * PI / 2.0); return v * v; };
      beta[i] = std::min(1.0 - fc(i + 1.0) / fc((double)i), 0.999);
    }
    abar[i] = (i ? abar[i - 1] : 1.0) * (1.0 - beta[i]);
  }
  std::vector<float> tab(6 * (size_t)T);
  for (int t = 0; t < T; ++t) {
    const double ap = t ? abar[t - 1] : 1.0;
    tab[0 * T + t] = (float)std::sqrt(abar[t]);
    tab[1 * T + t] = (float)std::sqrt(1.0 - abar[t]);
    if (f.sampler == 0) {                             // DDPM posterior: mu = c0 x0_hat + cx x
      tab[2 * T + t] = (float)(std::sqrt(ap) * beta[t] / (1.0 - abar[t]));
      tab[3 * T + t] = (float)(std::sqrt(1.0 - beta[t]) * (1.0 - ap) / (1.0 - abar[t]));
      tab[4 * T + t] = (float)std::sqrt(beta[t] * (1.0 - ap) / (1.0 - abar[t]));
      tab[5 * T + t] = 0.0f;
    } else {                                          // DDIM(eta): mu = sqrt(abar') x0_hat + sqrt(1 - abar' - sigma^2) eps
      const double sig = (double)f.eta * std::sqrt((1.0 - ap) / (1.0 - abar[t])) * std::sqrt(1.0 - abar[t] / ap);
      tab[2 * T + t] = (float)std::sqrt(ap);
      tab[3 * T + t] = 0.0f;
      tab[4 * T + t] = (float)sig;
      tab[5 * T + t] = (float)std::sqrt(std::max(1.0 - ap - sig * sig, 0.0));
    }
  }
  auto cleanup = [&](int code) { tsdp_destroy(c); return code; };
  if (dev_alloc(c, &c->tables, tab.size())) return cleanup(TSDP_E_NOMEM);
  if (hipMemcpy(c->tables, tab.data(), tab.size() * sizeof(float), hipMemcpyHostToDevice) != hipSuccess)
    return cleanup(TSDP_E_HIP);
  c->tb = {c->tables, c->tables + T, c->tables + 2 * T, c->tables + 3 * T, c->tables + 4 * T, c->tables + 5 * T, T};
  if (dev_alloc(c, &c->status, 1) || dev_alloc(c, &c->K_eff, (size_t)f.B_max) || dev_alloc(c, &c->n_draft, 2))
    return cleanup(TSDP_E_NOMEM);
  if (hipGetDevice(&c->device) != hipSuccess || c->device < 0 || c->device >= NOALLOC_MAX_DEVICES) return cleanup(TSDP_E_HIP);
  if (!g_scratch_ptr[c->device]) {
    double* p = nullptr;
    if (hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(scratch)) != hipSuccess || !p) return cleanup(TSDP_E_HIP);
    g_scratch_ptr[c->device] = p;
  }
  if (hipMemset(c->status, 0, sizeof(int32_t)) != hipSuccess) return cleanup(TSDP_E_HIP);
  if (hipStreamCreateWithFlags(&c->aux, hipStreamNonBlocking) != hipSuccess ||
      hipEventCreateWithFlags(&c->ev_fork, hipEventDisableTiming) != hipSuccess ||
      hipEventCreateWithFlags(&c->ev_join, hipEventDisableTiming) != hipSuccess)
    return cleanup(TSDP_E_HIP);
  *out = c;
  return TSDP_OK;
}

void tsdp_destroy(tsdp_ctx* c) {
  if (!c) return;
  (void)hipDeviceSynchronize();
  for (auto& st : c->ev)
    for (auto& e : st)
      if (e) (void)hipEventDestroy(e);
  if (c->ev_fork) (void)hipEventDestroy(c->ev_fork);
  if (c->ev_join) (void)hipEventDestroy(c->ev_join);
  if (c->aux) (void)hipStreamDestroy(c->aux);
  for (void* p : c->owned) (void)hipFree(p);
  delete c;
}

int tsdp_load_weights(tsdp_ctx* c, int which, const float* h_blob, size_t nbytes) {
  if (!c) return TSDP_E_INVAL;
  if (!h_blob || which < 0 || which > 1) return fail(c, TSDP_E_INVAL, "bad argument to tsdp_load_weights");
  Net& n = c->net[which];
  if (nbytes != n.n_floats * sizeof(float))
    return fail(c, TSDP_E_SHAPE, "weight blob has " + std::to_string(nbytes) + " bytes, expected " +
                                     std::to_string(n.n_floats * sizeof(float)));
  const tsdp_config& cf = c->cfg;
  std::vector<float> w(h_blob, h_blob + n.n_floats);
  if (cf.dtype == 1)
    for (auto& v : w) v = bf16_round(v);
  const int d = n.d, T = cf.T, L = n.L;
  // timestep embedding of every timestep (depends on the weights only): fp64 on the host
  std::vector<float> temb((size_t)T * d);
  {
    const int half = d / 2;
    std::vector<double> e(d), hdn(d);
    for (int t = 0; t < T; ++t) {
      for (int i = 0; i < half; ++i) {
        const double fr = std::exp(-std::log(10000.0) * i / half);
        e[i] = std::sin(t * fr);
        e[half + i] = std::cos(t * fr);
      }
      for (int i = 2 * half; i < d; ++i) e[i] = 0.0;
      for (int o = 0; o < d; ++o) {
        double acc = w[n.t_b1 + o];
        for (int i = 0; i < d; ++i) acc += (double)w[n.t_w1 + (size_t)o * d + i] * e[i];
        hdn[o] = acc / (1.0 + std::exp(-acc));
      }
      for (int o = 0; o < d; ++o) {
        double acc = w[n.t_b2 + o];
        for (int i = 0; i < d; ++i) acc += (double)w[n.t_w2 + (size_t)o * d + i] * hdn[i];
        temb[(size_t)t * d + o] = (float)acc;
      }
    }
  }
  std::vector<float> modw((size_t)L * 4 * d * d), modb((size_t)L * 4 * d);
  for (int l = 0; l < L; ++l) {
    std::memcpy(&modw[(size_t)l * 4 * d * d], &w[n.lay[l].mod_w], sizeof(float) * 4 * d * d);
    std::memcpy(&modb[(size_t)l * 4 * d], &w[n.lay[l].mod_b], sizeof(float) * 4 * d);
  }
  int rc;
  if (!n.blob) {
    if ((rc = dev_alloc(c, &n.blob, n.n_floats))) return rc;
    if ((rc = dev_alloc(c, &n.temb, temb.size()))) return rc;
    if ((rc = dev_alloc(c, &n.modw, modw.size()))) return rc;
    if ((rc = dev_alloc(c, &n.modb, modb.size()))) return rc;
    if (cf.cond_mode == 0) {
      if ((rc = dev_alloc(c, &n.cemb, (size_t)cf.B_max * d))) return rc;
    }
  }
  HIPCHK(c, hipDeviceSynchronize());
  HIPCHK(c, hipMemcpy(n.blob, w.data(), w.size() * sizeof(float), hipMemcpyHostToDevice));
  HIPCHK(c, hipMemcpy(n.temb, temb.data(), temb.size() * sizeof(float), hipMemcpyHostToDevice));
  HIPCHK(c, hipMemcpy(n.modw, modw.data(), modw.size() * sizeof(float), hipMemcpyHostToDevice));
  HIPCHK(c, hipMemcpy(n.modb, modb.data(), modb.size() * sizeof(float), hipMemcpyHostToDevice));
  if (c->flow_buf) HIPCHK(c, hipMemset(c->flow_buf, 0xFF, c->flow_have));   // FLOW_EMPTY, as every launch leaves it
  n.loaded = true;
  c->cond_set = false;
  n.fused = n.few = n.few_roll = false;
  n.path = "f32-ops";
  if (!std::getenv("TSDP_DISABLE_FUSED")) {
    FusedKernels fk;
    if (!find_fused(cf.dtype, n.d, cf.H, n.heads, cf.cond_mode, cf.cond_tokens, n.m / n.d, n.L, fk)) HIPCHK(c, find_few_dyn(cf, which, n, fk));
    if (fk.few_film && (rc = build_fused(c, n, w, modw, fk))) return rc;
  }
  if (!n.fused && cf.cond_mode == 1 && !n.kc) {        // fp32 keys / values of the operator kernels
    const size_t cnt = (size_t)L * cf.B_max * cf.cond_tokens * d;
    if ((rc = dev_alloc(c, &n.kc, cnt))) return rc;
    if ((rc = dev_alloc(c, &n.vc, cnt))) return rc;
  }
  if (n.fused && n.fused_mod && cf.cond_mode == 1) {
    // With token conditioning no conditioning vector enters the FiLM projections: they depend on the timestep
    // alone, so the vectors of all T timesteps are computed once, by the kernel that otherwise computes them per row.
    const int T = cf.T;
    if (!n.modtab) {
      if ((rc = dev_alloc(c, &n.modtab, (size_t)T * L * 4 * d))) return rc;
      if ((rc = dev_alloc(c, &n.t_iota, (size_t)T))) return rc;
      std::vector<int32_t> iota(T);
      for (int t = 0; t < T; ++t) iota[t] = t;
      HIPCHK(c, hipMemcpy(n.t_iota, iota.data(), sizeof(int32_t) * T, hipMemcpyHostToDevice));
    }
    n.fused_mod(n.fnet, n.t_iota, 0, nullptr, T, nullptr, T, n.modtab, nullptr);
    HIPCHK(c, hipGetLastError());
    HIPCHK(c, hipDeviceSynchronize());
    n.fnet.modtab = n.modtab;
  }
  return c->ws_ready ? ensure_few(c) : TSDP_OK;         // a context in use: the network may need larger buffers than before
}

int tsdp_set_cond(tsdp_ctx* c, const float* d_cond, int B, void* stream) {
  if (!c) return TSDP_E_INVAL;
  if (!d_cond) return fail(c, TSDP_E_INVAL, "d_cond is null");
  if (B < 1 || B > c->cfg.B_max) return fail(c, TSDP_E_SHAPE, "B outside 1..B_max");
  if (!c->net[0].loaded || !c->net[1].loaded) return fail(c, TSDP_E_STATE, "weights of both networks must be loaded");
  hipStream_t s = (hipStream_t)stream;
  const tsdp_config& cf = c->cfg;
  if (cf.cond_mode == 0 && B <= COND_VEC_B) {
    const Net &a = c->net[0], &b = c->net[1];
    hipLaunchKernelGGL(k_cond_vec, dim3((a.d + 15) / 16 + (b.d + 15) / 16, (B + 15) / 16), dim3(256), 0, s, d_cond,
                       CondVecNet{a.blob + a.c_w, a.blob + a.c_b, a.cemb, a.d}, CondVecNet{b.blob + b.c_w, b.blob + b.c_b, b.cemb, b.d},
                       B, cf.cond_dim);
    HIPCHK(c, hipGetLastError());
    c->cond_set = true;
    c->cond_B = B;
    return TSDP_OK;
  }
  CondIO io{};
  for (int which = 0; which < 2; ++which) {
    Net& n = c->net[which];
    const float* w = n.blob;
    if (cf.cond_mode == 0) {
      linear<0>(s, d_cond, w + n.c_w, w + n.c_b, n.cemb, B, 1, n.d, cf.cond_dim, nullptr);
    } else if (n.fused) {                             // bf16 (fused cross-attention is): one launch for both networks, below
      io.net[which] = {reinterpret_cast<const bf16x8*>(n.kv_w), n.kv_b, reinterpret_cast<__bf16*>(n.kc_pk),
                       reinterpret_cast<__bf16*>(n.vct_pk), n.L, n.d, n.heads, n.L * 2 * n.d / (COND_FF * 16)};
    } else {
      const int S = cf.cond_tokens;
      const size_t per_layer = (size_t)cf.B_max * S * n.d;
      for (int l = 0; l < n.L; ++l) {
        linear<0>(s, d_cond, w + n.lay[l].ck_w, w + n.lay[l].ck_b, n.kc + l * per_layer, B * S, 1, n.d, cf.cond_dim, nullptr);
        linear<0>(s, d_cond, w + n.lay[l].cv_w, w + n.lay[l].cv_b, n.vc + l * per_layer, B * S, 1, n.d, cf.cond_dim, nullptr);
      }
    }
  }
  if (const int tiles = io.net[0].tiles + io.net[1].tiles) {
    io.cond = d_cond; io.size = c->cond_size;
    io.M = B * cf.cond_tokens; io.C = cf.cond_dim; io.KS = (cf.cond_dim + 31) / 32; io.SF = cf.cond_tokens / 16;
    hipLaunchKernelGGL(k_cond_size, dim3((io.M + 3) / 4), dim3(256), 0, s, io);
    hipLaunchKernelGGL(k_cond_kv, dim3(tiles * ((io.M / 16 + COND_TF - 1) / COND_TF)), dim3(512), COND_LDS, s, io);
  }
  HIPCHK(c, hipGetLastError());
  c->cond_set = true;
  c->cond_B = B;
  return TSDP_OK;
}

enum BaseMod { MOD_NONE, MOD_DONE, MOD_BESIDE };   // the base network's FiLM vectors: not yet, on the caller's stream, on the auxiliary one

// gated: chain driver -- the row-table kernel also returns at once when no environment has rows (the drafter kernels
// always do: without rows there is nothing to draft)
static int draft_impl(tsdp_ctx* c, int B, const float* d_x, const int32_t* d_t0, const int32_t* d_K,
                      const float* d_sigma_scale, const int32_t* d_env_id, int32_t* d_row_ptr, int32_t* d_row_t,
                      int32_t* d_row_env, float* d_states, float* d_eps_p, float* d_xi, float* d_y_last, bool gated,
                      void* stream, int base_mod_rows = 0, BaseMod* base_mod = nullptr, int32_t* live = nullptr,
                      int32_t* rounds_run = nullptr) {
  // live: word that the round's k_accept counts the running environments in (cleared here), rounds_run: rounds that had rows, or null
  // base_mod_rows > 0 (whole rounds): the base network's per-row FiLM vectors of up to that many rows are computed with the row
  // table where the product is small, else, once the table exists, on the auxiliary stream beside the rollout; *base_mod says which
  int rc = check_ready(c, B, true);
  if (rc) return rc;
  if (B == 0) return TSDP_OK;                        // an empty batch is valid and touches nothing
  if (!d_x || !d_t0 || !d_K || !d_sigma_scale || !d_row_ptr || !d_row_t || !d_row_env || !d_states || !d_eps_p ||
      !d_y_last)
    return fail(c, TSDP_E_INVAL, "null pointer passed to tsdp_draft");
  if ((rc = ensure_workspace(c))) return rc;
  hipStream_t s = (hipStream_t)stream;
  const tsdp_config& cf = c->cfg;
  const int D = c->D;
  Net &dn = c->net[1], &bn = c->net[0];
  // persistent drafter kernel (or the spread launches), else a forward pass per transition
  const DraftTile* tile = draft_tile(dn, B);
  const bool kernel = dn.few_roll || tile;
  bool roll_film = false;                               // the rollout's FiLM vectors are part of the first launch
  if (B <= PLAN_ROWS_B) {
    const PlanIO plan{d_x, d_t0, d_K, d_sigma_scale, B, cf.K_max, cf.T, D, cf.bonus_row, gated ? 1 : 0, c->K_eff, d_row_ptr, c->status,
                      c->n_draft, live, rounds_run, d_row_t, d_row_env, d_y_last, d_states, d_eps_p, d_xi, c->sync, sync_lines(c)};
    // (bf16 networks and those with run-time sizes, which have fp32 operands, do not share a launch)
    auto f32 = [&](const Net& n) { return cf.dtype == 0 || !n.fused; };
    auto lds = [&](const Net& n) { return 16 * (n.d + (f32(n) ? TF32::PAD : TBF16::PAD)) * (f32(n) ? 4 : 2); };
    auto small = [&](const Net& n) { return n.few_film && !n.fnet.modtab && lds(n) <= 60 * 1024; };
    auto job = [&](const Net& n, int rows, int k_max, float* mod) {
      const int Nm = n.L * 4 * n.d;
      return FilmJob{n.fnet.modw, n.modb, n.temb, n.fnet.cemb, mod, n.d, Nm, (Nm / 16 + 3) / 4, (rows + 15) / 16, k_max};
    };
    auto timed = [&](int stage) { return c->timing && ((c->timing_mask >> stage) & 1); };   // (a product that a timed stage contains stays in it)
    FilmJob jb{}, jr{};
    jb.nx = jr.nx = 1;
    if (B <= PLAN_FILM_B) {
      if (dn.few_roll && small(dn) && !timed(0)) { jr = job(dn, B * cf.K_max, cf.K_max, c->few_mod); roll_film = true; }
      // (a rollout keeps its FiLM vectors in LDS or in few_mod; the operator kernels would use the buffer that the base network's go to)
      if (base_mod_rows > 0 && kernel && !timed(3) && (bn.few || (bn.fused && !bn.fused_mod)) && small(bn) && (!roll_film || f32(bn) == f32(dn))) {
        jb = job(bn, base_mod_rows, 0, c->mod);
        if (base_mod) *base_mod = MOD_DONE;
      }
    }
    const int wgs = jb.nx * jb.tiles + jr.nx * jr.tiles;
    if (wgs == 0) {
      hipLaunchKernelGGL(k_plan_rows, dim3(B), dim3(128), 0, s, plan);
    } else {
      const int bytes = std::max(jb.tiles ? lds(bn) : 0, jr.tiles ? lds(dn) : 0);
      const auto kern = f32(jr.tiles ? dn : bn) ? k_plan_film<TF32> : k_plan_film<TBF16>;
      hipLaunchKernelGGL(kern, dim3(B + wgs), dim3(256), bytes, s, plan, jb, jr);
    }
  } else {
    hipLaunchKernelGGL(k_plan, dim3(1), dim3(1024), 0, s, d_t0, d_K, d_sigma_scale, B, cf.K_max, cf.T, cf.bonus_row, c->K_eff,
                       d_row_ptr, c->status, c->n_draft, live, rounds_run);
    hipLaunchKernelGGL(k_rows, dim3(B), dim3(128), 0, s, d_x, d_t0, (const int32_t*)d_row_ptr, cf.T, D, d_row_t,
                       d_row_env, d_y_last, d_states, d_eps_p, d_xi, c->sync, sync_lines(c), gated ? (const int32_t*)c->n_draft : nullptr);
  }
  auto bonus_rows = [&]() {
    if (cf.bonus_row)
      hipLaunchKernelGGL(k_bonus_rows, dim3(B), dim3(128), 0, s, d_t0, (const int32_t*)c->K_eff, (const int32_t*)d_row_ptr,
                         d_env_id, cf.T, D, cf.seed, (const float*)d_y_last, d_states, d_eps_p, d_xi);
  };
  if (kernel) {
    if (base_mod_rows > 0 && bn.fused && bn.fused_mod && !bn.few && !bn.fnet.modtab) {
      // fork: a rollout keeps its FiLM vectors in LDS or in few_mod, so the shared buffer is free for the base network's.
      // (Not for few rows: their product takes 6 us, the fork and join about 30 us of every round of an enqueued chain.)
      HIPCHK(c, hipEventRecord(c->ev_fork, s));
      HIPCHK(c, hipStreamWaitEvent(c->aux, c->ev_fork, 0));
      bn.fused_mod(bn.fnet, d_row_t, 0, d_row_env, cf.T, d_row_ptr + B, base_mod_rows, c->mod, c->aux);
      HIPCHK(c, hipEventRecord(c->ev_join, c->aux));
      if (base_mod) *base_mod = MOD_BESIDE;
    }
    DraftIO io;
    io.B = B; io.t0 = d_t0; io.K_eff = c->K_eff; io.row_ptr = d_row_ptr; io.sigma_scale = d_sigma_scale;
    io.env_id = d_env_id;
    io.tb = {c->tb.sqrt_abar, c->tb.sqrt_1m, c->tb.c0, c->tb.cx, c->tb.sigma, c->tb.ce, c->tb.T};
    io.clip = cf.clip_x0; io.clip_val = cf.clip_val; io.seed = cf.seed;
    io.y = d_y_last; io.states = d_states; io.eps_p = d_eps_p; io.xi = d_xi;
    io.gate = c->n_draft + 1;
    io.bonus = cf.bonus_row;
    tick(c, 0, 0, s);
    if (dn.few_roll) {
      if (!dn.fnet.modtab && !roll_film) dn.few_film(dn.fnet, d_t0, 0, nullptr, cf.K_max, cf.T, nullptr, c->n_draft + 1, B * cf.K_max, c->few_mod, s);
      const FewRun r = few_run(c, dn, B, few_safe_rows(!gated, B, B), d_t0, nullptr, c->few_mod);   // (d_y_last has B rows)
      dn.few_draft(dn.fnet, r, io, cf.K_max, c->few_y, s);
    } else {
      HIPCHK(c, tile->launch(dn.fnet, io, cf.A, s));
    }
    tick(c, 0, 1, s);
    if (dn.few_roll) bonus_rows();
    HIPCHK(c, hipGetLastError());
    return TSDP_OK;
  }
  for (int k = 1; k <= cf.K_max; ++k) {
    // every environment runs the drafter at step k; the DDPM step masks those with K_eff < k
    if ((rc = forward(c, c->net[1], d_y_last, B, c->n_draft + 1, d_t0, k - 1, nullptr, c->eps_tmp, s))) return rc;
    hipLaunchKernelGGL(k_draft_step, grid1((long long)B * (D / 4), 256), dim3(256), 0, s, k, (const float*)c->eps_tmp,
                       d_t0, (const int32_t*)c->K_eff, (const int32_t*)d_row_ptr, d_sigma_scale, d_env_id, c->tb,
                       cf.clip_x0, cf.clip_val, cf.seed, B, D, d_y_last, d_states, d_eps_p, d_xi);
  }
  bonus_rows();
  HIPCHK(c, hipGetLastError());
  return TSDP_OK;
}

int tsdp_draft(tsdp_ctx* c, int B, const float* d_x, const int32_t* d_t0, const int32_t* d_K,
               const float* d_sigma_scale, const int32_t* d_env_id, int32_t* d_row_ptr, int32_t* d_row_t,
               int32_t* d_row_env, float* d_states, float* d_eps_p, float* d_xi, float* d_y_last, void* stream) {
  return draft_impl(c, B, d_x, d_t0, d_K, d_sigma_scale, d_env_id, d_row_ptr, d_row_t, d_row_env, d_states, d_eps_p, d_xi,
                    d_y_last, false, stream);
}

static int verify_impl(tsdp_ctx* c, int B, int R_cap, const int32_t* d_row_ptr, const int32_t* d_row_t,
                       const int32_t* d_row_env, const float* d_states, float* d_eps_q, bool own_table, void* stream,
                       BaseMod mod = MOD_NONE, bool gated = false) {
  int rc = check_ready(c, B, true);
  if (rc) return rc;
  if (B == 0 || R_cap == 0) return TSDP_OK;
  if (!d_row_ptr || !d_row_t || !d_row_env || !d_states || !d_eps_q)
    return fail(c, TSDP_E_INVAL, "null pointer passed to tsdp_verify");
  if (R_cap < 0 || (size_t)R_cap > rows_max(c->cfg))
    return fail(c, TSDP_E_SHAPE, "R_cap outside 0..B_max*(K_max+bonus_row)");
  if ((rc = ensure_workspace(c))) return rc;
  hipStream_t s = (hipStream_t)stream;
  if (!own_table) {
    // a caller's row table: timesteps and environment indices are clamped into range (the kernels index tables
    // with them) and the status word reports it
    hipLaunchKernelGGL(k_check_rows, grid1(R_cap, 256), dim3(256), 0, s, d_row_ptr + B, R_cap, d_row_t, d_row_env, c->cfg.T,
                       c->cond_B, c->row_t_chk, c->row_env_chk, c->status, c->sync, flow_lines(R_cap));
    d_row_t = c->row_t_chk;
    d_row_env = c->row_env_chk;
  }
  if (mod == MOD_BESIDE) HIPCHK(c, hipStreamWaitEvent(s, c->ev_join, 0));   // join: the FiLM vectors computed beside the rollout
  if ((rc = forward(c, c->net[0], d_states, R_cap, d_row_ptr + B, d_row_t, 0, d_row_env, d_eps_q, s, mod != MOD_NONE,
                    few_safe_rows(own_table && !gated, B, R_cap))))
    return rc;
  HIPCHK(c, hipGetLastError());
  return TSDP_OK;
}

int tsdp_verify(tsdp_ctx* c, int B, int R_cap, const int32_t* d_row_ptr, const int32_t* d_row_t,
                const int32_t* d_row_env, const float* d_states, float* d_eps_q, void* stream) {
  return verify_impl(c, B, R_cap, d_row_ptr, d_row_t, d_row_env, d_states, d_eps_q, false, stream);
}

static int accept_impl(tsdp_ctx* c, int B, const int32_t* d_row_ptr, const int32_t* d_row_t, const int32_t* d_env_id,
                       const float* d_sigma_scale, const float* d_lambda, const float* d_states, const float* d_eps_p,
                       const float* d_eps_q, const float* d_xi, const float* d_y_last, float* d_x_out, int32_t* d_t_next,
                       int32_t* d_n_accept, int32_t* d_n_adv, uint8_t* d_flags, float* d_logratio, float* d_logu,
                       const int32_t* d_gate, void* stream, const ChainAcc& chain = ChainAcc{}) {
  int rc = check_ready(c, B, false);
  if (rc) return rc;
  if (B == 0) return TSDP_OK;
  if (!d_row_ptr || !d_row_t || !d_sigma_scale || !d_states || !d_eps_p || !d_eps_q || !d_y_last || !d_x_out ||
      !d_t_next || !d_n_accept)
    return fail(c, TSDP_E_INVAL, "null pointer passed to tsdp_accept");
  hipStream_t s = (hipStream_t)stream;
  const tsdp_config& cf = c->cfg;
  const int wpb = 4;                                // environments (wavefronts) per workgroup
  const dim3 g((B + wpb - 1) / wpb), blk(64 * wpb);
  tick(c, 2, 0, s);
  // lanes per row: the D/4 vectors of a row should fill them (8 lanes x 5 at D = 160, 16 x 7 at D = 448); at most 8 per lane
  const int nb = c->D / 4;
  const int maxi8 = (nb + 7) / 8, maxi16 = (nb + 15) / 16;
  const bool g8 = maxi8 <= 8 && nb * 16 * maxi16 > nb * 8 * maxi8;   // the 8-lane mapping fits and idles fewer lanes
  const int maxi = g8 ? maxi8 : maxi16;
  const bool chained = chain.tot_accept || chain.tot_drafts || chain.tot_rounds || chain.live;   // (a chain stores its noise)
#define TSDP_ACCEPT(CL, GG, MI)                                                                                 \
  if (chained) TSDP_ACCEPT_X(CL, false, GG, MI, true, chain);                                                   \
  else if (d_xi) TSDP_ACCEPT_X(CL, false, GG, MI, false, NoChain{});                                            \
  else TSDP_ACCEPT_X(CL, true, GG, MI, false, NoChain{})
#define TSDP_ACCEPT_X(CL, RG, GG, MI, CH, ACC)                                                                           \
  hipLaunchKernelGGL((k_accept<CL, RG, GG, MI, CH>), g, blk, 0, s, B, c->D, d_row_ptr, d_row_t, d_env_id, d_sigma_scale, \
                     d_states, d_eps_p, d_eps_q, d_xi, d_y_last, c->tb, cf.clip_val, cf.seed, d_lambda, cf.bonus_row, d_x_out, d_t_next, \
                     d_n_accept, d_n_adv, d_flags, d_logratio, d_logu, d_gate, ACC)
#define TSDP_ACCEPT_MI(MI)                                                       \
  case MI:                                                                       \
    if (cf.clip_x0) { if (g8) TSDP_ACCEPT(true, 8, MI); else TSDP_ACCEPT(true, 16, MI); }    \
    else            { if (g8) TSDP_ACCEPT(false, 8, MI); else TSDP_ACCEPT(false, 16, MI); }  \
    break;
  switch (maxi) {
    TSDP_ACCEPT_MI(1) TSDP_ACCEPT_MI(2) TSDP_ACCEPT_MI(3) TSDP_ACCEPT_MI(4)
    TSDP_ACCEPT_MI(5) TSDP_ACCEPT_MI(6) TSDP_ACCEPT_MI(7) TSDP_ACCEPT_MI(8)
    default: return fail(c, TSDP_E_SHAPE, "H*A above 512 is not supported by the acceptance kernel");
  }
#undef TSDP_ACCEPT_MI
#undef TSDP_ACCEPT
#undef TSDP_ACCEPT_X
  tick(c, 2, 1, s);
  HIPCHK(c, hipGetLastError());
  return TSDP_OK;
}

int tsdp_accept(tsdp_ctx* c, int B, const int32_t* d_row_ptr, const int32_t* d_row_t, const int32_t* d_env_id,
                const float* d_sigma_scale, const float* d_states, const float* d_eps_p, const float* d_eps_q,
                const float* d_xi, const float* d_y_last, float* d_x_out, int32_t* d_t_next, int32_t* d_n_accept,
                int32_t* d_n_adv, uint8_t* d_flags, float* d_logratio, float* d_logu, void* stream) {
  return accept_impl(c, B, d_row_ptr, d_row_t, d_env_id, d_sigma_scale, nullptr, d_states, d_eps_p, d_eps_q, d_xi, d_y_last,
                     d_x_out, d_t_next, d_n_accept, d_n_adv, d_flags, d_logratio, d_logu, nullptr, stream);
}

int tsdp_accept_threshold(tsdp_ctx* c, int B, const int32_t* d_row_ptr, const int32_t* d_row_t,
                          const float* d_sigma_scale, const float* d_lambda, const float* d_states, const float* d_eps_p,
                          const float* d_eps_q, const float* d_xi, const float* d_y_last, float* d_x_out,
                          int32_t* d_t_next, int32_t* d_n_accept, int32_t* d_n_adv, uint8_t* d_flags, float* d_logratio,
                          void* stream) {
  if (c && B > 0 && !d_lambda) return fail(c, TSDP_E_INVAL, "d_lambda is null");
  if (c && B > 0 && !d_xi) return fail(c, TSDP_E_INVAL, "d_xi is null (no environment ids here to regenerate the noise from)");
  return accept_impl(c, B, d_row_ptr, d_row_t, nullptr, d_sigma_scale, d_lambda, d_states, d_eps_p, d_eps_q, d_xi, d_y_last,
                     d_x_out, d_t_next, d_n_accept, d_n_adv, d_flags, d_logratio, nullptr, nullptr, stream);
}

static int round_impl(tsdp_ctx* c, int B, float* d_x, int32_t* d_t, const int32_t* d_K, const float* d_sigma_scale,
                      const int32_t* d_env_id, const float* d_lambda, int32_t* d_n_accept, int32_t* d_n_advanced,
                      bool gated, void* stream, const ChainAcc& chain = ChainAcc{}, int32_t* rounds_run = nullptr) {
  int rc = check_ready(c, B, true);
  if (rc) return rc;
  if (B == 0) return TSDP_OK;
  if (!d_x || !d_t || !d_K || !d_sigma_scale) return fail(c, TSDP_E_INVAL, "null pointer passed to tsdp_round");
  if ((rc = ensure_round_buffers(c))) return rc;
  const int R_cap = B * (c->cfg.K_max + (c->cfg.bonus_row ? 1 : 0));
  BaseMod mod = MOD_NONE;
  if ((rc = draft_impl(c, B, d_x, d_t, d_K, d_sigma_scale, d_env_id, c->row_ptr, c->row_t, c->row_env, c->states,
                       c->eps_p, c->xi, c->y_last, gated, stream, R_cap, &mod, chain.live, rounds_run)))
    return rc;
  if ((rc = verify_impl(c, B, R_cap, c->row_ptr, c->row_t, c->row_env, c->states, c->eps_q, true, stream, mod, gated)))
    return rc;
  // x and t are overwritten in place: the acceptance kernel reads only the round's own buffers
  return accept_impl(c, B, c->row_ptr, c->row_t, d_env_id, d_sigma_scale, d_lambda, c->states, c->eps_p, c->eps_q, c->xi,
                     c->y_last, d_x, d_t, d_n_accept ? d_n_accept : c->n_acc, d_n_advanced ? d_n_advanced : c->n_adv,
                     nullptr, nullptr, nullptr, gated ? (const int32_t*)c->n_draft : nullptr, stream, chain);
}

int tsdp_round(tsdp_ctx* c, int B, float* d_x, int32_t* d_t, const int32_t* d_K, const float* d_sigma_scale,
               const int32_t* d_env_id, int32_t* d_n_accept, int32_t* d_n_advanced, void* stream) {
  return round_impl(c, B, d_x, d_t, d_K, d_sigma_scale, d_env_id, nullptr, d_n_accept, d_n_advanced, false, stream);
}

int tsdp_round_threshold(tsdp_ctx* c, int B, float* d_x, int32_t* d_t, const int32_t* d_K, const float* d_sigma_scale,
                         const int32_t* d_env_id, const float* d_lambda, int32_t* d_n_accept, int32_t* d_n_advanced,
                         void* stream) {
  if (c && B > 0 && !d_lambda) return fail(c, TSDP_E_INVAL, "d_lambda is null");
  return round_impl(c, B, d_x, d_t, d_K, d_sigma_scale, d_env_id, d_lambda, d_n_accept, d_n_advanced, false, stream);
}

static int ensure_chain_buffers(tsdp_ctx* c) {
  int rc;
  if ((rc = ensure_round_buffers(c))) return rc;
  if (!c->live && (rc = dev_alloc(c, &c->live, 1))) return rc;
  if (!c->K_sel) {
    if ((rc = dev_alloc(c, &c->K_sel, (size_t)c->cfg.B_max))) return rc;
    if ((rc = dev_alloc(c, &c->s_sel, (size_t)c->cfg.B_max))) return rc;
    if ((rc = dev_alloc(c, &c->lam_sel, (size_t)c->cfg.B_max))) return rc;
  }
  return TSDP_OK;
}

// host_checked: rounds are enqueued until the number of running environments, read back every check_every rounds,
// is zero (or max_rounds is reached).  Otherwise exactly max_rounds rounds are enqueued and nothing is read back:
// the kernels of a round return at once when the round's row table is empty (every environment has finished).
static int chain_impl(tsdp_ctx* c, int B, float* d_x, int32_t* d_t, const int32_t* d_K, const float* d_sigma_scale,
                      const int32_t* d_env_id, const float* d_lambda, bool staged, int t_hi, int t_lo, int max_rounds,
                      int check_every, bool host_checked, int32_t* d_tot_accept, int32_t* d_tot_drafts,
                      int32_t* d_tot_rounds, int32_t* h_rounds, int32_t* d_rounds_run, void* stream) {
  int rc = check_ready(c, B, true);
  if (rc) return rc;
  if (h_rounds) *h_rounds = 0;
  if (!host_checked && max_rounds < 0) return fail(c, TSDP_E_INVAL, "n_rounds must not be negative");
  hipStream_t s = (hipStream_t)stream;
  if (d_rounds_run) hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(1), 0, s, d_rounds_run, 1, 0);
  if (B == 0) return TSDP_OK;
  if (!d_x || !d_t || !d_K || !d_sigma_scale) return fail(c, TSDP_E_INVAL, "null pointer passed to tsdp_chain");
  if (host_checked && (max_rounds < 1 || check_every < 1))
    return fail(c, TSDP_E_INVAL, "max_rounds and check_every must be positive");
  if (staged && !(t_hi >= t_lo && t_lo >= 0)) return fail(c, TSDP_E_INVAL, "stage bounds must satisfy t_hi >= t_lo >= 0");
  if ((rc = ensure_chain_buffers(c))) return rc;
  const dim3 gb((B + 255) / 256), blk(256);
  for (int32_t* p : {d_tot_accept, d_tot_drafts, d_tot_rounds})
    if (p) hipLaunchKernelGGL(k_fill_i32, gb, blk, 0, s, p, B, 0);
  const ChainAcc chain{d_tot_accept, d_tot_drafts, d_tot_rounds, host_checked ? c->live : nullptr};
  int rounds = 0;
  while (rounds < max_rounds) {
    if (staged) {
      // the round's K, sigma scale and threshold are those of the stage each environment is in now
      hipLaunchKernelGGL(k_stage_select, gb, blk, 0, s, B, (const int32_t*)d_t, t_hi, t_lo, d_K, d_sigma_scale, d_lambda,
                         c->K_sel, c->s_sel, c->lam_sel);
      rc = round_impl(c, B, d_x, d_t, c->K_sel, c->s_sel, d_env_id, d_lambda ? c->lam_sel : nullptr, c->n_acc, c->n_adv,
                      !host_checked, stream, chain, d_rounds_run);
    } else {
      rc = round_impl(c, B, d_x, d_t, d_K, d_sigma_scale, d_env_id, d_lambda, c->n_acc, c->n_adv, !host_checked, stream, chain, d_rounds_run);
    }
    if (rc) return rc;
    ++rounds;
    if (host_checked && (rounds % check_every == 0 || rounds == max_rounds)) {
      int32_t live = 0;
      HIPCHK(c, hipMemcpyAsync(&live, c->live, sizeof(int32_t), hipMemcpyDeviceToHost, s));
      HIPCHK(c, hipStreamSynchronize(s));
      if (live == 0) break;
    }
  }
  if (h_rounds) *h_rounds = rounds;
  HIPCHK(c, hipGetLastError());
  return TSDP_OK;
}

int tsdp_chain(tsdp_ctx* c, int B, float* d_x, int32_t* d_t, const int32_t* d_K, const float* d_sigma_scale,
               const int32_t* d_env_id, const float* d_lambda, int max_rounds, int check_every, int32_t* d_tot_accept,
               int32_t* d_tot_drafts, int32_t* d_tot_rounds, int32_t* h_rounds, void* stream) {
  return chain_impl(c, B, d_x, d_t, d_K, d_sigma_scale, d_env_id, d_lambda, false, 0, 0, max_rounds, check_every, true,
                    d_tot_accept, d_tot_drafts, d_tot_rounds, h_rounds, nullptr, stream);
}

int tsdp_chain_staged(tsdp_ctx* c, int B, float* d_x, int32_t* d_t, const int32_t* d_K3, const float* d_sigma_scale3,
                      const float* d_lambda3, int t_hi, int t_lo, const int32_t* d_env_id, int max_rounds, int check_every,
                      int32_t* d_tot_accept, int32_t* d_tot_drafts, int32_t* d_tot_rounds, int32_t* h_rounds, void* stream) {
  return chain_impl(c, B, d_x, d_t, d_K3, d_sigma_scale3, d_env_id, d_lambda3, true, t_hi, t_lo, max_rounds, check_every,
                    true, d_tot_accept, d_tot_drafts, d_tot_rounds, h_rounds, nullptr, stream);
}

int tsdp_chain_enqueue(tsdp_ctx* c, int B, float* d_x, int32_t* d_t, const int32_t* d_K, const float* d_sigma_scale,
                       const float* d_lambda, int staged, int t_hi, int t_lo, const int32_t* d_env_id, int n_rounds,
                       int32_t* d_tot_accept, int32_t* d_tot_drafts, int32_t* d_tot_rounds, int32_t* d_rounds_run,
                       void* stream) {
  return chain_impl(c, B, d_x, d_t, d_K, d_sigma_scale, d_env_id, d_lambda, staged != 0, t_hi, t_lo, n_rounds, 0, false,
                    d_tot_accept, d_tot_drafts, d_tot_rounds, nullptr, d_rounds_run, stream);
}

int tsdp_prepare(tsdp_ctx* c) {
  if (!c) return TSDP_E_INVAL;
  if (!c->net[0].loaded || !c->net[1].loaded) return fail(c, TSDP_E_STATE, "weights of both networks must be loaded");
  int rc;
  if ((rc = ensure_workspace(c))) return rc;
  if ((rc = ensure_chain_buffers(c))) return rc;
  if (!c->loss_partial && (rc = dev_alloc(c, &c->loss_partial, 3 * DISTILL_WGS))) return rc;
  // the launch attributes of the fused kernels (dynamic LDS size): a launch over zero rows sets them and enqueues nothing
  FusedIO io{};
  DraftIO dio{};
  Net& bn = c->net[0];
  if (bn.fused) {
    if (bn.fused_verify) HIPCHK(c, bn.fused_verify(bn.fnet, io, c->cfg.A, 0, nullptr));
    if (bn.fused_verify_few) HIPCHK(c, bn.fused_verify_few(bn.fnet, io, c->cfg.A, 0, nullptr));
  }
  Net& dn = c->net[1];
  if (dn.fused)                                       // the tiles tsdp_draft may pick
    for (const DraftTile* t : {&dn.draft_small, &dn.draft_big})
      if (t->fits) HIPCHK(c, t->launch(dn.fnet, dio, c->cfg.A, nullptr));
  return TSDP_OK;
}

// partial: room for 3 * DISTILL_WGS doubles; every entry that is read is written first by the same call
static int distill_launch(tsdp_ctx* c, int R, const int32_t* d_row_t, const float* d_states, const float* d_eps_p,
                          const float* d_eps_q, float lambda1, float lambda2, double* partial, double* d_loss, hipStream_t s) {
  const int parts = std::min((R + 15) / 16, DISTILL_WGS);
  if (parts > 0) {
    if (c->cfg.clip_x0)
      hipLaunchKernelGGL(k_distill_partial<true>, dim3(parts), dim3(256), 0, s, R, c->D, d_row_t, d_states, d_eps_p, d_eps_q,
                         c->tb, c->cfg.clip_val, partial);
    else
      hipLaunchKernelGGL(k_distill_partial<false>, dim3(parts), dim3(256), 0, s, R, c->D, d_row_t, d_states, d_eps_p, d_eps_q,
                         c->tb, c->cfg.clip_val, partial);
  }
  hipLaunchKernelGGL(k_distill_final, dim3(1), dim3(256), 0, s, parts, R, (const double*)partial, lambda1, lambda2, d_loss);
  HIPCHK(c, hipGetLastError());
  return TSDP_OK;
}

int tsdp_distill_loss(tsdp_ctx* c, int R, const int32_t* d_row_t, const float* d_states, const float* d_eps_p,
                      const float* d_eps_q, float lambda1, float lambda2, double* d_loss, void* stream) {
  if (!c) return TSDP_E_INVAL;
  if (R < 0 || (size_t)R > rows_max(c->cfg)) return fail(c, TSDP_E_SHAPE, "R outside 0..B_max*(K_max+bonus_row)");
  if (!d_loss || (R > 0 && (!d_row_t || !d_states || !d_eps_p || !d_eps_q)))
    return fail(c, TSDP_E_INVAL, "null pointer passed to tsdp_distill_loss");
  if (!c->loss_partial) {
    int rc = dev_alloc(c, &c->loss_partial, 3 * DISTILL_WGS);
    if (rc) return rc;
  }
  return distill_launch(c, R, d_row_t, d_states, d_eps_p, d_eps_q, lambda1, lambda2, c->loss_partial, d_loss,
                        (hipStream_t)stream);
}

int tsdp_distill_loss_noalloc(tsdp_ctx* c, int R, const int32_t* d_row_t, const float* d_states, const float* d_eps_p,
                              const float* d_eps_q, float lambda1, float lambda2, double* d_loss, void* stream) {
  if (!c) return TSDP_E_INVAL;
  if (R < 0 || R > NOALLOC_MAX_ROWS)
    return fail(c, TSDP_E_SHAPE, "tsdp_distill_loss_noalloc: R outside 0.." + std::to_string(NOALLOC_MAX_ROWS) +
                                     " (the size of the static scratch)");
  if (!d_loss || (R > 0 && (!d_row_t || !d_states || !d_eps_p || !d_eps_q)))
    return fail(c, TSDP_E_INVAL, "null pointer passed to tsdp_distill_loss_noalloc");
  int dev = -1;
  HIPCHK(c, hipGetDevice(&dev));
  if (dev != c->device || !g_scratch_ptr[dev])
    return fail(c, TSDP_E_STATE, "tsdp_distill_loss_noalloc must run with the context's device current");
  return distill_launch(c, R, d_row_t, d_states, d_eps_p, d_eps_q, lambda1, lambda2, g_scratch_ptr[dev], d_loss,
                        (hipStream_t)stream);
}

int tsdp_status(tsdp_ctx* c, void* stream, int32_t* h_status) {
  if (!c || !h_status) return TSDP_E_INVAL;
  hipStream_t s = (hipStream_t)stream;
  HIPCHK(c, hipMemcpyAsync(h_status, c->status, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  HIPCHK(c, hipStreamSynchronize(s));
  // cleared with a tiny fill kernel-free path: a synchronous memset outside any capture
  HIPCHK(c, hipMemset(c->status, 0, sizeof(int32_t)));
  return TSDP_OK;
}

int tsdp_kernel_timing(tsdp_ctx* c, int enable) {
  if (!c) return TSDP_E_INVAL;
  if (enable && !c->ev[0][0]) {
    for (auto& st : c->ev)
      for (auto& e : st) HIPCHK(c, hipEventCreate(&e));
  }
  c->timing = enable != 0;
  c->timing_mask = enable <= 1 ? 15 : (enable >> 1) & 15;
  for (bool& u : c->ev_used) u = false;
  return TSDP_OK;
}

int tsdp_kernel_ms(tsdp_ctx* c, int stage, float* h_ms) {
  if (!c || !h_ms || stage < 0 || stage > 3) return TSDP_E_INVAL;
  if (!c->ev[0][0] || !c->ev_used[stage]) return fail(c, TSDP_E_STATE, "no timed launch of that stage since timing was enabled");
  HIPCHK(c, hipEventSynchronize(c->ev[stage][1]));
  HIPCHK(c, hipEventElapsedTime(h_ms, c->ev[stage][0], c->ev[stage][1]));
  return TSDP_OK;
}

const char* tsdp_path_name(const tsdp_ctx* c, int which) {
  if (!c || which < 0 || which > 1) return "";
  return c->net[which].path;
}

const char* tsdp_last_error(const tsdp_ctx* c) { return c ? c->err.c_str() : "null context"; }

// Not part of the interface, for tests: the kernels that a network's weights are loaded for.
const char* tsdp_internal_kernels(const tsdp_ctx* c, int which) {
  if (!c || which < 0 || which > 1) return "";
  const Net& n = c->net[which];
  return n.few ? (n.flow_row ? "k_flow" : n.few_slices ? "k_few" : "k_row") : n.fused ? "tiles" : "operators";
}

// Not part of the interface, for tests: environments per workgroup of the persistent rollout of B environments, 0: another kernel's.
int tsdp_internal_rollout_tile(const tsdp_ctx* c, int B) {
  const DraftTile* t = c && !c->net[1].few_roll ? draft_tile(c->net[1], B) : nullptr;
  return t ? t->rpt : 0;
}

// Not part of the interface, for tests: one-launch passes of this context with at most n workgroups (0: all), so that XCDs
// without one leave their sets to others.  A launch makes progress with any number of workgroups, one included.
int tsdp_internal_flow_workgroups(tsdp_ctx* c, int n) {
  if (!c || n < 0) return TSDP_E_INVAL;
  c->flow_wgs = n;
  return TSDP_OK;
}

}  // extern "C"
