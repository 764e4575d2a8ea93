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
// with the rows; they meet at about 2100 tokens.  Rounds, us, tile / spread at 64, 128, 144 rows of 16 tokens: bf16 d = 256
// 498 / 409, 498 / 443, 497 / 511; bf16 d = 384 880 / 729, 881 / 869, -; fp32 d = 256 799 / 504, 800 / 724, and at 136 rows
// 797 / 835; at 64, 128 rows of 32 tokens, d = 512: 1577 / 1252, 1591 / 1856.  A layer of less than 700 KB passes through one
// compute unit faster than through two launches (fp32 d = 64, 393 KB in all: 21 us against 25); one launch was not measured there.
constexpr size_t FEW_LAYER_BYTES = 700000;
constexpr size_t layer_bytes(size_t d, bool f32, bool cross) { return (cross ? 14 : 12) * d * d * (f32 ? 4 : 2); }
inline bool few_pays(size_t tokens, bool f32, size_t layer_bytes) {
  return tokens <= (f32 ? 2048 : 2176) && layer_bytes >= FEW_LAYER_BYTES;
}

// Launches of a spread rollout (two bf16 networks of one shape; fp32 drafters beyond flow_draft_pays): every transition up to
// K_max has its own, whether drafted or not (the draft counts are on the device).  With half of K_max or more the spread rollout
// is the faster one, and what fewer drafts lose grows with K_max.  Rounds of one environment, two bf16 networks of d = 256, us,
// persistent rollout and tile kernels / all spread: two layers, K = 1, 4, 8 of 8 170 / 164, 296 / 220, 464 / 293; 1, 4, 9 of 9 169 / 178,
// 296 / 232, 507 / 321; 1, 8, 16 of 16 170 / 279, 464 / 390, 802 / 532; four layers 1, 2, 4 of 4 283 / 213, 384 / 244, 589 / 307, 1, 8
// of 8 282 / 310, 1031 / 531.  With the fp32 drafter of d = 128, two layers (spread 23 us a drafted and 6 to 15 an undrafted transition,
// persistent 39), K = 1, 4, 8 of 8 226 / 277, 344 / 331, 495 / 396; 4, 64 of 64 344 / 1085, 2673 / 1888.  So up to 40 launches (two layers:
// K_max = 9) the rollout is spread -- the loss stays below a quarter of a round -- and beyond it is one launch.
constexpr int FEW_ROLL_LAUNCHES = 40;
inline bool few_rollout_pays(int layers, bool wide, bool cross, int K_max) {
  return layers * (wide ? 2 : 1) * (cross ? 3 : 2) * K_max + 1 <= FEW_ROLL_LAUNCHES;
}

// Rollout in one launch (k_flow) instead of in launches (where that pays, `launches`) or in the persistent kernel.
// fp32: the XCDs work side by side, and from the third environment of an XCD on a transition grows by about a quarter with
// every other one, where the launches fill the chip at the same time.  tsdp_draft, us, launches / one launch, four transitions of
// 8, 12, 16, 18, 24, 32 environments, two layers: d = 128 105 / 87, 107 / 95, 107 / 96, 108 / 113, 108 / 113, 109 / 137 (one
// transition of 64, 128: 40 / 69, 57 / 115); d = 256 197 / 124, 202 / 182, 202 / 183, 231 / 257, 232 / 256, 239 / 336.  One layer of
// d = 128 is too short for the exchanges unless there are several transitions: 16 environments, K_max = 1, 2, 4, 7 23 / 27, 37 /
// 39, 64 / 63, 105 / 98.  Against the persistent kernel (four layers, K_max = 7, 8 / 18 environments) d = 128 515 / 249, 515 / 335,
// d = 256 1992 / 357, 1972 / 797; it does not grow with the environments, and at 32 one launch takes 0.83 (0.55) of its time.
// bf16 with cross-attention, d = 256, 32 tokens: eight transitions of 1, 4, 8, 16, 32 environments 317, 346, 350, 373, 518, the
// persistent kernel (one workgroup an environment) 425 to 463; tsdp_draft, persistent / one launch, 24 environments, K_max = 1, 2, 8, one
// layer 38 / 42, 66 / 71, 236 / 236, two 67 / 66, 122 / 117, 459 / 420; one layer, 16 environments 36.8 / 38.5, 65 / 63, 235 / 208.
inline bool flow_draft_pays(int environments, bool f32, size_t d, int layers, int K_max, bool launches) {
  if (!f32) return environments <= (layers >= 2 ? 24 : K_max >= 2 ? 16 : 8);
  return launches ? environments <= 16 && (layers * d >= 256 || K_max >= 4) : environments <= 32;
}

// Forward pass in one launch (k_flow): its dependent steps are shorter than two launches per layer, but a row costs it more of
// the chip (registers for one workgroup per unit, tasks that take their rows in turn).
// fp32, tsdp_verify, us, launches / one launch: d = 256, one layer, 32, 40, 48, 64 rows of 16 tokens 41 / 39, 45 / 43, 45 / 49, 49 / 56;
// two 66 / 64, 73 / 69, 76 / 77, 83 / 93; four 117 / 104, 131 / 118, 135 / 133, 151 / 161; eight 219 / 186, 250 / 215, 254 / 244,
// 288 / 300, at 56 rows four 148 / 145, eight 284 / 271, eight at 80, 96, 112, 128 rows 401 / 357, 432 / 415, 468 / 471, 509 / 531.
// d = 128, 8, 12, 16, 20 rows: one layer 21.4 / 21.2, 22.0 / 22.7, 21.3 / 23.1, 21.8 / 25.0; two 32 / 29, 31.7 / 32.4, 31.9 / 32.7, 32 / 37;
// four 50 / 45, 53 / 53, 53 / 53, 52 / 59; eight 97 / 79, 98 / 93, 99 / 98, 99 / 106 (128 rows, four layers: 89 / 157).
// bf16, rounds, us, 8, 16, 32, 64, 128 rows of 16 tokens: d = 256 250 / 214, 253 / 228, 256 / 273, 264 / 345, 311 / 490; d = 384 at
// 4, 16, 32 rows 317 / 243, 634 / 579, 642 / 675 (328 / 363 with four drafts).  Two workgroups per unit at d = 256 meet at 32 rows
// (256 / 251) and lose 5 % at 16.  tsdp_verify of one layer, d = 256, 8, 10, 12, 16 rows 24.3 / 22.6, 24.2 / 23.8, 23.9 / 24.1, 24.1 / 24.9
// (two layers, 16 rows 37 / 34), d = 384, 16 rows 36 / 31.
// With cross-attention (d = 512, 32 tokens), tsdp_verify of 1, 8, 9, 16 rows: one layer 46 / 42, 50 / 47, 51 / 62; two 81 / 65, 88 / 70,
// 88 / 105; twelve 445 / 289, 462 / 307, 466 / 504, 472 / 524 (one group of tasks that take two rows in turn 466): beyond one row an XCD
// every further one adds the 3 us of a task to each of the phases.  Whole rounds with launches / one launch, of 1 x 1, 1 x 8, 2 x 4, 8 x 1
// environments and drafts: one layer 104 / 94, 373 / 324, 229 / 194, 113 / 102; two 139 / 110, 427 / 366, 271 / 227, 151 / 125; twelve 520 / 338,
// 801 / 601, 654 / 444, 538 / 350; of eight environments one that runs 102 / 90, 139 / 114, 489 / 334.
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
