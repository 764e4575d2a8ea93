// Host-side rules of the spread forward pass (few_rows.hpp); plain C++ without HIP.
#pragma once
#include <algorithm>
#include <cstddef>

namespace tsdp {

// Rows below this one a launch may start to read before it knows how many rows are live (`ahead`).  In the context's own
// row buffers any row up to their capacity exists, and every running environment has one: the loads of the first B rows
// travel together with the live row count, which is worth 1 % of a round.  Not so
//  - in a caller's buffers: they hold the live rows and no more -- finished environments own none, so not even the first B
//    need exist -- and nothing of them is read before the count is known;
//  - in the rounds of an enqueued chain, most of which have no live row: a launch without one costs 1.5 us where it asks
//    first and 2.6 us where it first requests the row's data and weights (an empty round of 54 launches 85 us, 142).
inline int few_safe_rows(bool ahead, int B, int R_cap) { return ahead ? std::min(B, R_cap) : 0; }

// Networks with compiled kernels.  One workgroup per tile takes the same time from 1 to 256 tiles, the spread launches grow
// with the rows; they meet at about 2100 tokens.  tsdp_verify of four layers, us, tile / spread: fp32 d = 256, 112, 128 rows of 16 tokens
// 241 / 214, 242 / 233; bf16 d = 256, 128, 136 rows 122 / 94, 122 / 117; bf16 d = 384, 112, 128 rows 205 / 189, 204 / 194, but 136 rows 204 / 244
// (the line is one for both); 48, 64, 68 rows of 32 tokens, d = 512: 364 / 263, 362 / 270, 362 / 356.  A layer of less than 700 KB passes through
// one compute unit faster than through two launches (fp32 d = 64, 393 KB in all: 21 us against 25, before either became faster); one
// launch was not measured there.
constexpr size_t FEW_LAYER_BYTES = 700000;
constexpr size_t layer_bytes(size_t d, bool f32, bool cross) { return (cross ? 14 : 12) * d * d * (f32 ? 4 : 2); }
inline bool few_pays(size_t tokens, bool f32, size_t layer_bytes) {
  return tokens <= (f32 ? 2048 : 2176) && layer_bytes >= FEW_LAYER_BYTES;
}

// Launches of a spread rollout (two bf16 networks of one shape; fp32 drafters beyond flow_draft_pays): every transition up to
// K_max has its own, whether drafted or not (the draft counts are on the device).  With half of K_max or more the spread rollout
// is the faster one, and what fewer drafts lose grows with K_max.  Rounds of one environment, two bf16 networks of d = 256, us,
// persistent rollout and tile kernels / all spread: two layers, K = 1, 4, 8 of 8 148 / 143, 264 / 197, 419 / 263; 1, 4, 9 of 9 149 / 154,
// 267 / 208, 457 / 291; 1, 8, 16 of 16 150 / 250, 419 / 346, 724 / 480; four layers 1, 2, 4 of 4 251 / 189, 338 / 218, 508 / 275, 1, 8
// of 8 251 / 272, 849 / 475.  With the fp32 drafter of d = 128, two layers, K = 1, 4, 8 of 8, persistent (and the forward pass in one
// launch) / all spread 155 / 246, 263 / 297, 402 / 361; 4, 64 of 64 (both spread) 319 / 826, 2030 / 1595.  So up to 40 launches (two layers:
// K_max = 9) the rollout is spread -- the two networks' loss stays below a quarter of a round -- and beyond it is one launch.
constexpr int FEW_ROLL_LAUNCHES = 40;
inline bool few_rollout_pays(int layers, bool wide, bool cross, int K_max) {
  return layers * (wide ? 2 : 1) * (cross ? 3 : 2) * K_max + 1 <= FEW_ROLL_LAUNCHES;
}

// Rollout in one launch (k_flow) instead of in launches (where that pays, `launches`) or in the persistent kernel.
// fp32: the XCDs work side by side, and from the third environment of an XCD on a transition grows by about a quarter with
// every other one, where the launches fill the chip at the same time.  tsdp_draft, us, launches / one launch, four transitions of
// 8, 12, 16, 18, 24, 32 environments, two layers: d = 128 103 / 76, 104 / 88, 104 / 88, 104 / 103, 110 / 109, 110 / 136 (one
// transition of 64, 128: 41 / 68, 56 / 115); d = 256 181 / 121, 184 / 183, 185 / 186, 210 / 258, 212 / 260, 219 / 344.  One layer of
// d = 128 is too short for the exchanges unless there are several transitions: 16 environments, K_max = 1, 2, 4, 7 27 / 28, 38 /
// 39, 64 / 60, 103 / 92 (eight environments 26 / 25, 37 / 33, 63 / 49, 102 / 72: there the line gives up to an eighth away).  Against the
// persistent kernel (four layers, K_max = 7, 8 / 18 environments) d = 128 506 / 205, 507 / 299, d = 256 1962 / 344, 1958 / 801.
// bf16 with cross-attention, d = 256, 32 tokens, two layers, eight transitions of 1, 4, 8, 16, 32 environments 277, 281, 304, 320, 523, the
// persistent kernel (one workgroup an environment) 399 to 434; tsdp_draft, persistent / one launch, 24 environments, K_max = 1, 2, 8, one
// layer 40 / 44, 66 / 70, 220 / 222, two 72 / 68, 123 / 116, 428 / 403; one layer, 16 environments 40 / 38, 66 / 59, 219 / 179.
inline bool flow_draft_pays(int environments, bool f32, size_t d, int layers, int K_max, bool launches) {
  if (!f32) return environments <= (layers >= 2 ? 24 : K_max >= 2 ? 16 : 8);
  return launches ? environments <= 16 && (layers * d >= 256 || K_max >= 4) : environments <= 32;
}

// Forward pass in one launch (k_flow): its dependent steps are shorter than two launches per layer, but a row costs it more of
// the chip (registers for one workgroup per unit, tasks that take their rows in turn).
// fp32, tsdp_verify, us, launches / one launch: d = 256, one layer, 16, 20, 32, 40, 48 rows of 16 tokens 33.0 / 32.7, 36 / 38, 39 / 42, 43 / 46,
// 43 / 49; two, 24, 28, 40, 48 rows 60 / 55, 61 / 64, 69 / 71, 70 / 78; four, 32, 40, 44, 56, 64 rows 107 / 105, 121 / 118, 121 / 133, 134 / 146,
// 138 / 161; eight 199 / 189, 226 / 215, 229 / 243, 254 / 270, 260 / 297.  d = 128, 8, 10, 12, 16 rows: one layer 20.2 / 20.0, 20.4 / 22.3 (8, 10
// rows); two 29.7 / 26.7, 29.8 / 31.9; four 49 / 41, 49.7 / 49.9, 49.7 / 49.1, 50 / 53; eight 90 / 68, 91 / 89, 91.2 / 88.4, 91.4 / 92.2.
// The lines of d = 256 were drawn where both met when the launches requested 40 fragments of weights ahead (40 rows, 56 from four layers on);
// they request fewer since (FewGemm::AHEAD), and meet at 16 to 24 rows and at 40.  Between, a pass is up to a tenth slower than it
// could be: the lines are where the bits of a result may change, which tsdp.h names, and stay.
// bf16, rows of 16 tokens: d = 256, one layer, 8, 10, 12 rows 22.1 / 21.3, 22.1 / 24.8, 22.5 / 25.1; two, 8, 16 rows 33 / 28, 35 / 34; four 62 / 44, 62 / 54;
// eight 111 / 71, 111 / 89; d = 384, 8, 16 rows, one layer 33 / 28, 35 / 33, two 55 / 37, 55 / 47, four 94 / 56, 95 / 72.  Rounds with the slower launches:
// d = 256 at 16, 32, 64, 128 rows 253 / 228, 256 / 273, 264 / 345, 311 / 490; d = 384 at 32 rows 642 / 675.
// With cross-attention (d = 512, 32 tokens), tsdp_verify of 1, 8 rows: one layer 48 / 40, 50 / 46; two 84 / 61, 87 / 68; twelve 447 / 277, 462 / 294, and 9, 16
// rows (when the launches were 1 % slower) 466 / 504, 472 / 524 (one group of tasks that take two rows in turn 466): beyond one row an XCD
// every further one adds the 3 us of a task to each of the phases.  Whole rounds of 1 x 8, 8 x 1 environments and drafts, twelve layers: 773 / 570,
// 521 / 351.
inline bool flow_forward_pays(size_t tokens, bool f32, size_t d, int layers) {
  if (!f32) return tokens <= (layers * d >= 384 ? 256 : 160);
  return tokens <= 16 * (d >= 256 ? (layers >= 4 ? 56 : 40) : (layers >= 4 ? 16 : 8));
}

// Waits of the one-launch kernels.  No wait polls more than FLOW_SPINS times (about half a microsecond each); every FLOW_LOOK
// polls it looks whether another wait of its launch has run into that bound, and ends if so: a launch whose data cannot arrive
// drains within one bound and FLOW_LOOK polls of every later wait, not one bound each.
constexpr int FLOW_SPINS = 1 << 22, FLOW_LOOK = 64;
enum FlowTurn { FLOW_POLL, FLOW_ASK, FLOW_GIVE_UP };   // behind poll n that found its data missing
constexpr FlowTurn flow_turn(int n) { return n >= FLOW_SPINS ? FLOW_GIVE_UP : n % FLOW_LOOK == FLOW_LOOK - 1 ? FLOW_ASK : FLOW_POLL; }

// Where a workgroup of a one-launch pass goes when the tickets it draws from have run out.  Sets as masks: `open` have rows and
// no XCD yet, `ours` are its XCD's and it has not seen their tickets run out; `late`: it has looked long enough for the XCD of
// an open set to have come.  A set of its own XCD comes first: one that changes hands is then worked by every workgroup of the
// XCD that is waiting, not by the one that took it.
constexpr int FLOW_LEAVE = -1, FLOW_STAY = -2;           // every set is in hand; look again
constexpr int flow_next_set(unsigned open, unsigned ours, bool late) {
  return ours ? __builtin_ctz(ours) : !open ? FLOW_LEAVE : late ? __builtin_ctz(open) : FLOW_STAY;
}

// Networks with run-time sizes: `tokens` a launch covers at most (the ragged batch's, the rollout's one row per environment).
// A spread launch streams its weights once per row and adds max(heads, slices) partial sums of the whole row in every
// workgroup; one launch per operator does neither but has six times the launches.  Rows at which both take the same time
// (two layers, 64 .. 2048 rows measured), 16 tokens: 3 heads d = 96 ~950, 8 d = 256 ~850, 10 d = 320 ~500, 16 d = 512 ~420,
// 20 d = 640 ~230, 32 d = 512 ~200, up to six heads at d = 512 .. 768 beyond 2048; 32 tokens: 8 d = 512 ~240, 12 d = 768 ~115.
// That is tokens x heads of 44 000 and more, near whose lower end the line is.  (64 rows, us, operators / spread: d = 96
// 187 / 57, d = 512 with 16 heads 663 / 309; 2048 rows 671 / 800, 7164 / 8634.)  A layer of more than the 32 MB of all L2s
// comes from beyond them for every row: d = 1024 meets at 90 rows (8 or 16 heads), 64 rows 1369 / 1182, 512 6434 / 9794.
// (k_row stands behind this line too, which was measured for the launches alone: it has no partial sums, and where it meets the
// operator kernels is not measured.)
inline bool few_dyn_pays(size_t tokens, size_t heads, size_t layer_bytes) {
  return layer_bytes <= (32u << 20) ? tokens * std::max<size_t>(heads, 5) <= 47000
                                    : tokens * std::max<size_t>(heads, 16) <= 16384;
}

// One workgroup per row or environment through all layers (k_row) instead of launches, for networks with run-time sizes.
// A unit's time for a layer grows with its weights times the fragments of 16 tokens (fp32 matrix rate), and not with the rows
// until every unit has one; a launch costs the same for any small layer, and grows with the rows.  Two layers, us, launches / one
// workgroup a row; tsdp_verify of 8, 256, 512 rows of 16 tokens: d = 48, 3 heads (0.1 MB a layer) 42 / 24, 67 / 25, 111 / 32; d = 96, 3
// heads (0.44 MB) 51 / 41, 122 / 43, 222 / 63; d = 128, 2 heads (0.79 MB) 55 / 51, 125 / 53, 230 / 82; d = 160, 5 heads (1.2 MB) 64 / 80,
// 212 / 82, 381 / 126; d = 256, 8 heads (3.1 MB) 90 / 165, 302 / 164.  tsdp_draft of one layer, eight transitions of 1, 64 environments:
// 169 / 82, 166 / 84; 213 / 140, 214 / 143; 233 / 185, 238 / 188; d = 160 272 / 294, 299 / 299.  32 tokens, verify of 8, 256 rows: d = 96, 3
// heads 72 / 67, 289 / 69, d = 128, 4 heads 76 / 92, 324 / 93.
// Layers of 0.9 to 1.6 MB, tsdp_verify of 64, 96, 128 rows of 16 tokens: d = 144, 3 heads 70 / 72, 81 / 73, 83 / 73; d = 160, 5 heads
// 77 / 81, 106 / 81, 124 / 80, 10 heads 87 / 81, 131 / 81, 146 / 81; d = 176, 11 heads 96 / 91, 117 / 91, 126 / 91; d = 208, 13 heads, hidden
// layer of twice the width 119 / 89, 131 / 90, 149 / 90; 32, 48, 64 rows of 32: d = 128, 4 heads 79 / 92, 102 / 92, 104 / 92, 8 heads 77 / 93,
// 119 / 94, 123 / 93.  So from 1536 tokens on, or where the launches have 2.5 workgroups and more per unit (rows x heads).
// What these lines give away: a context of which few rows live (4 of 128, d = 160: 64 / 80), which the capacity cannot tell.
inline bool row_pays(size_t tokens, size_t H, size_t layer_bytes, size_t heads = 1) {
  const size_t work = layer_bytes * H / 16;
  return work <= 900000 || (work <= 1600000 && (tokens >= 1536 || (tokens >= 1024 && tokens / H * heads >= 640)));
}

// Floats of the two residual and of the two partial-sum buffers, shared by both networks.  Which networks take the spread
// path can change with every tsdp_load_weights, so what a context holds is compared with what its networks need now, and
// replaced by a larger buffer where it is too small.
struct FewShape { bool few; size_t tokens, d, slices; };
struct FewSize { size_t h = 0, part = 0; };
inline FewSize few_size(const FewShape& base, const FewShape& draft) {
  FewSize z;
  for (const FewShape* n : {&base, &draft})
    if (n->few) {
      z.h = std::max(z.h, n->tokens * n->d);
      z.part = std::max(z.part, n->tokens * n->d * n->slices);
    }
  return z;
}
inline bool few_fits(const FewSize& have, const FewSize& need) { return need.h <= have.h && need.part <= have.part; }

}  // namespace tsdp
