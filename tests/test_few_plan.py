"""Host-side rules of the spread forward pass (csrc/few_plan.hpp, plain C++), compiled here and checked without a GPU."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_15773_amd", "csrc")
SHIM = """
#include "few_plan.hpp"
using namespace tsdp;
extern "C" {
int safe_rows(int own, int B, int R_cap) { return few_safe_rows(own != 0, B, R_cap); }
int rollout_pays(int layers, int wide, int cross, int K_max) { return few_rollout_pays(layers, wide != 0, cross != 0, K_max); }
int pays(long tokens, int f32, long layer_bytes) { return few_pays(tokens, f32 != 0, layer_bytes); }
int draft_pays(int environments, int f32, long d, int layers, int K_max, int launches) { return flow_draft_pays(environments, f32 != 0, d, layers, K_max, launches != 0); }
int forward_pays(long tokens, int f32, long d, int layers) { return flow_forward_pays(tokens, f32 != 0, d, layers); }
int dyn_pays(long tokens, long heads, long layer_bytes) { return few_dyn_pays(tokens, heads, layer_bytes); }
int one_workgroup_pays(long tokens, long H, long layer_bytes) { return row_pays(tokens, H, layer_bytes); }
int one_workgroup_pays_heads(long tokens, long H, long layer_bytes, long heads) { return row_pays(tokens, H, layer_bytes, heads); }
int next_set(unsigned open, unsigned ours, int late) { return flow_next_set(open, ours, late != 0); }
// polls of one workgroup's `waits` waits, one after the other, for data that never arrives
long drain(int waits) {
  long polls = 0;
  bool over = false;
  for (int w = 0; w < waits; ++w)
    for (int n = 0;; ++n) {
      ++polls;
      const FlowTurn turn = flow_turn(n);
      if (turn == FLOW_GIVE_UP) over = true;
      if (turn == FLOW_GIVE_UP || (turn == FLOW_ASK && over)) break;
    }
  return polls;
}
// the context's buffers after a sequence of loads: flags[2 * i] / [2 * i + 1] = base / drafter takes the spread path then
int buffers_hold(long tokens, long d0, long s0, long d1, long s1, const int* flags, int loads) {
  FewSize have;
  for (int i = 0; i < loads; ++i) {
    const FewSize need = few_size({flags[2 * i] != 0, (size_t)tokens, (size_t)d0, (size_t)s0}, {flags[2 * i + 1] != 0, (size_t)tokens, (size_t)d1, (size_t)s1});
    if (!few_fits(have, need)) have = {std::max(have.h, need.h), std::max(have.part, need.part)};
    const long d[2] = {d0, d1}, s[2] = {s0, s1};
    for (int n = 0; n < 2; ++n)
      if (flags[2 * i + n] && (have.h < (size_t)(tokens * d[n]) || have.part < (size_t)(tokens * d[n] * s[n]))) return 0;
  }
  return 1;
}
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    out = tmp_path_factory.mktemp("few_plan")
    src, lib = str(out / "shim.cpp"), str(out / "shim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", CSRC, src, "-o", lib], check=True)
    plan = C.CDLL(lib)
    plan.drain.restype = C.c_long
    return plan


def test_rows_of_a_callers_buffer_are_not_read_beyond_the_live_ones(plan):
    # a workgroup of row r loads r ahead of the live row count when r < safe_rows; a caller's buffer may end at the live
    # rows, of which there are fewer than environments once some have finished
    for B in (1, 3, 8):
        for R_cap in (1, B, 5 * B):
            for live in range(R_cap + 1):
                early = [r for r in range(R_cap) if r < plan.safe_rows(0, B, R_cap)]
                assert all(r < live for r in early), (B, R_cap, live)
            assert plan.safe_rows(1, B, R_cap) <= R_cap           # the context's own buffers hold R_cap rows


def test_buffers_hold_whatever_networks_take_the_spread_path(plan):
    # a reload can move either network to the spread path: the larger one after the smaller one, and back
    L = C.c_long
    for d0, s0, d1, s1 in ((256, 16, 128, 8), (128, 8, 256, 16), (512, 8, 512, 8)):
        for flags in ([0, 1, 1, 1], [1, 0, 1, 1], [0, 0, 0, 1, 1, 0], [1, 1, 0, 1, 1, 1]):
            a = (C.c_int * len(flags))(*flags)
            assert plan.buffers_hold(L(2048), L(d0), L(s0), L(d1), L(s1), a, len(flags) // 2), (d0, d1, flags)


def test_rollouts_of_many_possible_drafts_stay_in_one_launch(plan):
    # every transition up to K_max is launched, drafted or not: a context for 64 drafts that asks for four would pay for 64
    assert plan.rollout_pays(2, 0, 0, 8) and not plan.rollout_pays(2, 0, 0, 16)
    for layers in (1, 2, 8):
        for wide in (0, 1):
            for cross in (0, 1):
                pays = [plan.rollout_pays(layers, wide, cross, k) for k in range(1, 65)]
                assert pays == sorted(pays, reverse=True) and not pays[-1]


def test_run_time_sizes_are_spread_only_where_that_is_faster(plan):
    # (d, heads, rows of 16 tokens, spread was the faster one): both sides measured on networks of two layers
    layer = lambda d: 12 * d * d * 4
    pays = lambda d, heads, rows: bool(plan.dyn_pays(C.c_long(16 * rows), C.c_long(heads), C.c_long(layer(d))))
    for d, heads, rows in ((96, 3, 512), (96, 3, 576), (320, 5, 512), (256, 8, 256), (320, 10, 128), (512, 16, 128), (512, 32, 64), (1024, 16, 64)):
        assert pays(d, heads, rows), (d, heads, rows)
    for d, heads, rows in ((64, 4, 1024), (96, 3, 1024), (256, 16, 1024), (320, 20, 256), (512, 32, 256), (640, 20, 256),
                           (1024, 32, 64), (1024, 8, 128), (1024, 16, 512), (1024, 64, 2048)):
        assert not pays(d, heads, rows), (d, heads, rows)


def test_a_row_per_workgroup_only_where_that_is_faster(plan):
    # (d, tokens of a row, rows, one workgroup per row was the faster one): both sides measured on networks of two layers
    for d, H, rows, faster in ((48, 16, 8, 1), (96, 16, 512, 1), (128, 16, 8, 1), (160, 16, 8, 0), (160, 16, 256, 1), (256, 16, 8, 0),
                               (96, 32, 8, 1), (128, 32, 8, 0), (128, 32, 256, 1)):
        assert plan.one_workgroup_pays(C.c_long(H * rows), C.c_long(H), C.c_long(12 * d * d * 4)) == faster, (d, H, rows)


def test_larger_layers_take_a_workgroup_per_row_only_from_enough_rows_on(plan):
    # (d, heads, hidden layer, tokens of a row, rows, one workgroup per row was the faster one)
    for d, heads, ratio, H, rows, faster in (
            (144, 3, 4, 16, 64, 0), (144, 3, 4, 16, 96, 1), (160, 5, 4, 16, 64, 0), (160, 5, 4, 16, 96, 1), (160, 10, 4, 16, 64, 1), (176, 11, 4, 16, 64, 1),
            (208, 13, 2, 16, 64, 1), (112, 7, 4, 32, 32, 0), (112, 7, 4, 32, 48, 1), (128, 4, 4, 32, 32, 0), (128, 4, 4, 32, 48, 1), (128, 8, 4, 32, 32, 0), (128, 8, 4, 32, 48, 1)):
        layer = 4 * (4 + 2 * ratio) * d * d
        assert plan.one_workgroup_pays_heads(C.c_long(H * rows), C.c_long(H), C.c_long(layer), C.c_long(heads)) == faster, (d, heads, H, rows)


def test_compiled_kernels_are_spread_up_to_2048_and_2176_tokens(plan):
    # the GPU tests of the tile kernels take contexts just above these lines
    L = C.c_long
    big = L(12 * 256 * 256 * 2)
    assert plan.pays(L(2048), 1, big) and not plan.pays(L(2064), 1, big)
    assert plan.pays(L(2176), 0, big) and not plan.pays(L(2192), 0, big)
    assert not plan.pays(L(16), 1, L(12 * 64 * 64 * 4))


def test_rollouts_in_one_launch_only_where_that_is_faster(plan):
    # (d, layers, K_max, environments): tsdp_draft measured on every side of the line, in fp32 against the launches (all of K_max
    # up to 40 launches) and against the persistent kernel beyond, in bf16 (cross-attention) against the persistent kernel
    L = C.c_long
    pays = lambda f32, d, layers, K_max, B: bool(plan.draft_pays(B, f32, L(d), layers, K_max, plan.rollout_pays(layers, 0, 1 - f32, K_max)))
    for d, layers, K_max, B in ((128, 1, 7, 16), (128, 1, 4, 12), (128, 2, 1, 8), (128, 2, 4, 16), (128, 4, 2, 16), (256, 1, 1, 8), (256, 2, 7, 16), (256, 4, 1, 16),
                                (128, 2, 64, 2), (128, 2, 16, 8), (128, 4, 7, 18), (256, 4, 7, 18)):
        assert pays(1, d, layers, K_max, B), (d, layers, K_max, B)
    for d, layers, K_max, B in ((128, 1, 1, 8), (128, 1, 2, 16), (128, 1, 4, 18), (128, 2, 1, 24), (128, 2, 4, 18), (128, 2, 2, 64), (128, 2, 1, 128), (128, 4, 4, 32),
                                (256, 1, 1, 18), (256, 2, 4, 24), (256, 4, 4, 32), (256, 4, 2, 64)):
        assert not pays(1, d, layers, K_max, B), (d, layers, K_max, B)
    assert pays(0, 256, 2, 1, 24) and not pays(0, 256, 2, 8, 25)
    assert pays(0, 256, 1, 1, 8) and pays(0, 256, 1, 2, 16) and not pays(0, 256, 1, 1, 16) and not pays(0, 256, 1, 2, 24)


def test_forward_passes_in_one_launch_only_where_that_is_faster(plan):
    # (fp32, d, layers, rows of 16 tokens): tsdp_verify measured against two launches per layer
    L = C.c_long
    pays = lambda f32, d, layers, rows: bool(plan.forward_pays(L(16 * rows), f32, L(d), layers))
    for f32, d, layers, rows in ((1, 256, 1, 40), (1, 256, 2, 40), (1, 256, 4, 56), (1, 256, 8, 56), (1, 128, 1, 8), (1, 128, 2, 8), (1, 128, 4, 16),
                                 (1, 128, 8, 16), (0, 256, 1, 10), (0, 256, 2, 16), (0, 384, 1, 16), (0, 384, 8, 16)):
        assert pays(f32, d, layers, rows), (f32, d, layers, rows)
    for f32, d, layers, rows in ((1, 256, 1, 48), (1, 256, 2, 64), (1, 256, 4, 64), (1, 256, 8, 64), (1, 256, 8, 128), (1, 128, 1, 12), (1, 128, 2, 20), (1, 128, 4, 20),
                                 (1, 128, 8, 24), (1, 128, 4, 128), (0, 256, 1, 16), (0, 256, 8, 32), (0, 384, 8, 32)):
        assert not pays(f32, d, layers, rows), (f32, d, layers, rows)


def test_a_launch_whose_data_cannot_arrive_drains_after_one_bound(plan):
    # one wait may take its bound (about two seconds), the hundreds that follow in the same launch may not
    bound = plan.drain(1)
    assert 1 << 20 <= bound <= (1 << 22) + 1
    for waits in (2, 97, 10000):
        assert plan.drain(waits) <= bound + 64 * (waits - 1), waits


def _work_off(plan, first_at, wgs, tasks, late):
    """A one-launch pass in steps: XCD i's workgroups start one by one from step first_at[i] on; a draw takes a step, a task eight.  Returns the
    last step and, per set, the workgroups that worked on it."""
    owner = [-1] * 8; drawn = [0] * 8; workers = [set() for _ in range(8)]
    state = {(x, w): dict(at=first_at[x] + w, set=None, done=0, looks=0) for x in range(8) for w in range(wgs)}
    step = 0
    while state:
        assert step < 100000, "the launch does not end"
        seen = list(owner)                                # looks of one step see the words as they were
        for (x, w), s in list(state.items()):
            if s["at"] > step:
                continue
            if s["set"] is None:                          # the set of its own number
                if owner[x] < 0:
                    owner[x] = x
                s["set"] = x
            if s["set"] >= 0 and owner[s["set"]] == x and not s["done"] >> s["set"] & 1 and drawn[s["set"]] < tasks:
                drawn[s["set"]] += 1
                workers[s["set"]].add((x, w))
                s["at"] = step + 8
                continue
            s["done"] |= 1 << s["set"]
            open_ = sum(1 << i for i in range(8) if seen[i] < 0)
            ours = sum(1 << i for i in range(8) if seen[i] == x) & ~s["done"]
            n = plan.next_set(open_, ours, int(s["looks"] >= late))
            s["looks"] += 1
            if n == -1:
                del state[(x, w)]
            elif n >= 0:
                if owner[n] < 0:
                    owner[n] = x
                if owner[n] == x:
                    s["set"] = n
        step += 1
    assert all(d == tasks for d in drawn)
    return step, workers


def test_a_set_that_changes_hands_is_worked_by_the_whole_xcd(plan):
    # XCDs 0 .. 6 are busy for a long time: XCD 7 works off all eight sets with all of its workgroups, and not one after the other
    # with the workgroup that took the set; what the others find when they come is in hand
    for wgs in (1, 2, 16):
        steps, workers = _work_off(plan, [4000] * 7 + [0], wgs, tasks=256, late=64)
        assert all(len({w for _, w in s}) >= wgs - 1 and len({x for x, _ in s}) == 1 for s in workers), wgs
        assert steps <= max(4000, 8 * (256 // wgs + 2) * 8 + 64 * 2) + 8 * 2, (wgs, steps)
    # an XCD that comes while its set is still open takes it, and nobody waits for long where every XCD comes
    _, workers = _work_off(plan, [40] * 7 + [0], 16, tasks=256, late=64)
    assert all({x for x, _ in workers[i]} == {i} for i in range(8))
    steps, workers = _work_off(plan, [0] * 8, 16, tasks=256, late=64)
    assert steps <= 8 * 17 + 16 + 4 and all({x for x, _ in workers[i]} == {i} for i in range(8))


def test_no_kernel_is_compiled_that_no_network_reaches():
    # a layer of less than FEW_LAYER_BYTES never takes the spread kernels: fp32 d = 32, 64 and bf16 d = 128 have none
    lib = os.path.join(os.path.dirname(CSRC), "libtsdp.so")
    if not os.path.exists(lib):
        pytest.skip("the library is not built")
    names = subprocess.run(["nm", "-D", "--defined-only", lib], capture_output=True, text=True, check=True).stdout
    assert "FlowCfgINS_4TF32ELi256E" in names and "FewCfgINS_4TF32ELi128E" in names
    for cfg in ("FlowCfg", "FewCfg"):
        for shape in ("INS_4TF32ELi32E", "INS_4TF32ELi64E", "INS_5TBF16ELi128E"):
            assert cfg + shape not in names, cfg + shape
