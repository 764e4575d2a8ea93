"""Forward passes and rollouts in one launch (csrc/flow_rows.hpp): row counts where the tasks are dealt differently, and the
buffers that every launch has to leave empty."""
import ctypes

import numpy as np
import pytest

import tsdp_inputs as ti
from tests.helpers import gpu_side, kernels, to_dev
from tests.test_gpu_parity import _stage_parity

pytestmark = pytest.mark.gpu
STATE = ti.replace(ti.C2, base=ti.NetShape(2, 256, 4))


@pytest.mark.parametrize("wl, B, K_max", [
    (STATE, 7, 1), (STATE, 8, 1),                     # one row per XCD at most: a workgroup per unit
    (STATE, 33, 1), (STATE, 43, 3),                   # five rows of an XCD for its four groups of tasks; tile kernels
    (STATE, 40, 1), (STATE, 41, 1), (ti.replace(ti.C2, base=ti.NetShape(4, 256, 4)), 14, 4), (ti.replace(ti.C2, base=ti.NetShape(4, 256, 4)), 19, 3),
    (ti.replace(ti.C2, base=ti.NetShape(4, 128, 4)), 8, 2), (ti.replace(ti.C2, base=ti.NetShape(4, 128, 4)), 17, 1),   # fp32 forward passes: the most rows
    # in one launch, the fewest in two launches per layer
    (STATE, 16, 2), (STATE, 17, 2),                   # fp32 rollouts: the most environments in one launch, the fewest in launches
    (ti.replace(ti.C2, base=ti.NetShape(3, 128, 4), draft=ti.NetShape(4, 256, 4)), 18, 7),   # so many launches: in one beyond that too
    (ti.replace(ti.C2, base=ti.NetShape(1, 256, 4), draft=ti.NetShape(4, 128, 4)), 33, 3),   # and in launches
    (ti.replace(ti.C2, base=ti.NetShape(1, 256, 4), draft=ti.NetShape(1, 128, 4)), 2, 5),   # one layer: both sets of buffers in turn
    (ti.replace(ti.C2, base=ti.NetShape(3, 128, 4), draft=ti.NetShape(3, 256, 4)), 2, 4),   # an odd number of layers
    (ti.replace(ti.C4, base=ti.NetShape(1, 512, 8)), 24, 2), (ti.replace(ti.C4, base=ti.NetShape(1, 512, 8)), 25, 2),   # rollout with
    # cross-attention: the largest in one launch, the smallest beyond it; bf16 bases up to 16 rows (one layer: ten), and the first beyond
    (ti.replace(ti.C3, base=ti.NetShape(2, 256, 4)), 1, 9), (ti.replace(ti.C3, base=ti.NetShape(1, 256, 4)), 8, 2), (ti.replace(ti.C3, base=ti.NetShape(1, 256, 4)), 5, 2),
    (ti.replace(ti.C3, base=ti.NetShape(2, 256, 4)), 17, 1), (ti.replace(ti.C5, base=ti.NetShape(1, 384, 6)), 5, 3),
    (ti.replace(ti.C5, base=ti.NetShape(3, 384, 6)), 16, 1),
])
def test_rows_are_dealt_to_the_tasks(wl, B, K_max):
    wl = ti.small_variant(wl, B=B, K_max=K_max)
    rng = np.random.default_rng(B)
    t0 = rng.integers(0, wl.T, B); K = rng.integers(1, K_max + 1, B); s = rng.uniform(1.0, 1.5, B)
    t0[0] = wl.T - 1; K[0] = K_max; t0[-1] = 1
    _stage_parity(wl, B, t0, K, s, norm=B % 2)


def _context(wl, **kw):
    return gpu_side(wl, *(ti.make_weights(wl, which, b_std=0.02) for which in ("base", "draft")), ti.make_cond(wl, wl.B), B_max=wl.B, **kw)


def _stages(ctx, x, t0, K, s):
    B = len(t0)
    rows = ctx.alloc_rows(B)
    ctx.tsdp_draft(x, to_dev(t0.astype(np.int32)), to_dev(K.astype(np.int32)), to_dev(s.astype(np.float32)), None, rows)
    ctx.tsdp_verify(B, rows)
    n = int(rows["row_ptr"][B])
    return {k: rows[k][:n].clone() for k in ("states", "eps_p", "eps_q")} | {"y_last": rows["y_last"].clone()}


@pytest.mark.parametrize("wl, B, K_max", [
    (STATE, 8, 5), (STATE, 13, 3),                    # fp32: rows and environments of which a task has one or two
    (ti.replace(ti.C2, base=ti.NetShape(4, 256, 4)), 7, 8), (ti.replace(ti.C2, base=ti.NetShape(1, 256, 4), draft=ti.NetShape(1, 128, 4)), 6, 5),
    (ti.replace(ti.C2, base=ti.NetShape(3, 128, 4), draft=ti.NetShape(4, 256, 4)), 18, 7),
    (ti.replace(ti.C4, base=ti.NetShape(1, 512, 8)), 24, 2), (ti.replace(ti.C4, base=ti.NetShape(1, 512, 8), draft=ti.NetShape(3, 256, 8)), 11, 4),
    (ti.replace(ti.C3, base=ti.NetShape(3, 256, 4)), 4, 4), (ti.replace(ti.C5, base=ti.NetShape(1, 384, 6)), 16, 1),
    (ti.replace(ti.C4, base=ti.NetShape(1, 512, 8)), 2, 4), (ti.replace(ti.C4, base=ti.NetShape(2, 512, 8)), 8, 1),   # wide bases
])
def test_every_call_finds_the_buffers_empty(wl, B, K_max):
    # what a launch leaves behind shows in the next one: calls with fewer environments and rows, other inputs and finished
    # environments in between, after each of which the first call gives the same bits again
    import torch
    wl = ti.small_variant(wl, B=B, K_max=K_max)
    ctx = _context(wl)
    assert "k_flow" in kernels(ctx)
    rng = np.random.default_rng(B)
    x = to_dev(ti.make_latents(wl, B))
    first = (x, np.full(B, wl.T - 1), np.full(B, K_max), np.ones(B))
    ref = _stages(ctx, *first)
    for i in range(3):
        n = (B, 1, (B + 1) // 2)[i]
        t0 = rng.integers(-1, wl.T, n); t0[0] = wl.T - 1
        _stages(ctx, torch.randn_like(x[:n]), t0, rng.integers(1, K_max + 1, n), rng.uniform(1.0, 1.5, n))
        got = _stages(ctx, *first)
        for name in ref:
            assert torch.equal(got[name], ref[name]), (i, name)
    assert ctx.tsdp_status() == 0
    ctx.close()


@pytest.mark.parametrize("layers, d, B, K_max", [(2, 256, 3, 3), (2, 128, 2, 4), (4, 256, 3, 8), (2, 128, 12, 2), (2, 256, 20, 2)])
def test_equal_networks_in_fp32_give_equal_predictions(layers, d, B, K_max):
    # both in one launch (the third because its rollout would be too many launches), both in two launches per layer
    import torch
    net = ti.NetShape(layers, d, 4)
    wl = ti.small_variant(ti.C2, base=net, draft=net, B=B, K_max=K_max)
    wb = ti.make_weights(wl, "base", b_std=0.02)
    ctx = gpu_side(wl, wb, wb, ti.make_cond(wl, B), B_max=B)
    t0 = np.linspace(90, 9, B).astype(int); K = 1 + np.arange(B) % K_max
    got = _stages(ctx, to_dev(ti.make_latents(wl, B)), t0, K, np.ones(B))
    assert torch.equal(got["eps_p"], got["eps_q"])
    ctx.close()


def test_one_launch_passes_of_two_contexts_side_by_side():
    # contexts whose forward passes and rollouts are one launch each run rounds at the same time on streams of their own: the bits
    # of running them one after the other
    import torch
    wls = [ti.small_variant(ti.C2, B=7, K_max=8), ti.small_variant(ti.C4, B=9, K_max=4, base=ti.NetShape(2, 512, 8)), ti.small_variant(ti.C5, B=4, K_max=4),
           ti.small_variant(ti.C4, B=2, K_max=4, base=ti.NetShape(3, 512, 8))]
    ctxs = [_context(wl) for wl in wls]
    rng = np.random.default_rng(1)
    inputs = [(to_dev(ti.make_latents(wl, wl.B)), to_dev(rng.integers(30, wl.T, wl.B).astype(np.int32)), to_dev(rng.integers(1, wl.K_max + 1, wl.B).astype(np.int32)),
               torch.ones(wl.B, device="cuda")) for wl in wls]

    def rounds(i, x, t, stream):
        with torch.cuda.stream(stream):
            for _ in range(4):
                ctxs[i].tsdp_round(x, t, inputs[i][2], inputs[i][3], None)

    want = [(x.clone(), t.clone()) for x, t, _, _ in inputs]
    for i, (x, t) in enumerate(want):
        rounds(i, x, t, torch.cuda.current_stream())
        torch.cuda.synchronize()
    got = [(x.clone(), t.clone()) for x, t, _, _ in inputs]
    streams = [torch.cuda.Stream() for _ in wls]
    torch.cuda.synchronize()                          # (every tensor exists before a side stream reads it, and lives on)
    for i, (x, t) in enumerate(got):
        rounds(i, x, t, streams[i])
    torch.cuda.synchronize()
    for i in range(len(wls)):
        assert torch.equal(got[i][0], want[i][0]) and torch.equal(got[i][1], want[i][1]), i
        assert ctxs[i].tsdp_status() == 0
        ctxs[i].close()


@pytest.mark.parametrize("wl, B, K_max", [
    (STATE, 9, 3), (ti.replace(ti.C3, base=ti.NetShape(2, 256, 4)), 3, 5), (ti.replace(ti.C4, base=ti.NetShape(1, 512, 8)), 11, 2),
    (ti.replace(ti.C4, base=ti.NetShape(2, 512, 8)), 2, 4),
])
def test_sets_whose_xcd_does_not_come_are_worked_off_by_another(wl, B, K_max):
    # fewer workgroups than XCDs: the sets of the others are taken over, with the bits of an ordinary launch; and ordinary launches
    # in between, so that a set's owner changes from launch to launch
    import torch
    from paper_2512_15773_amd import load_library
    wl = ti.small_variant(wl, B=B, K_max=K_max)
    ctx = _context(wl)
    assert "k_flow" in kernels(ctx)
    limit = load_library().tsdp_internal_flow_workgroups
    limit.argtypes = [ctypes.c_void_p, ctypes.c_int]
    x = to_dev(ti.make_latents(wl, B))
    K = 1 + np.arange(B) % K_max; K[0] = K_max
    calls = (x, np.linspace(wl.T - 1, 2, B).astype(int), K, np.ones(B))
    ref = _stages(ctx, *calls)
    for wgs in (1, 3, 0, 2, 8, 9, 0):
        assert limit(ctx.ctx, wgs) == 0
        got = _stages(ctx, *calls)
        for name in ref:
            assert torch.equal(got[name], ref[name]), (wgs, name)
        assert ctx.tsdp_status() == 0, wgs
    ctx.close()


@pytest.mark.parametrize("wl, B", [(STATE, 3), (ti.replace(ti.C3, base=ti.NetShape(2, 256, 4)), 3), (ti.replace(ti.C4, base=ti.NetShape(1, 512, 8)), 3),
                                   (ti.replace(ti.C4, base=ti.NetShape(2, 512, 8)), 2)])
@pytest.mark.parametrize("payload", [0xFFFFFFFF, 0x7FC00000])
def test_not_a_number_passes_through_and_leaves_nothing_behind(wl, B, payload):
    # the pattern of an empty buffer, as a latent: its environment's results are not numbers, the others' and those of the
    # next calls have the same bits as without it (fp32, pairs of bf16, a rollout with cross-attention, a wide base)
    import torch
    wl = ti.small_variant(wl, B=B, K_max=4)
    ctx = _context(wl)
    x = to_dev(ti.make_latents(wl, B)); bad = x.clone()
    bad[1].view(torch.int32).fill_(payload - (1 << 32) if payload >= 1 << 31 else payload)
    calls = (np.array([99, 50, 3])[:B], np.array([4, 3, 4])[:B], np.ones(B))
    assert "k_flow" in kernels(ctx)
    ref = _stages(ctx, x, *calls)
    for latents in (bad, x, bad, bad, x):
        got = _stages(ctx, latents, *calls)
        keep = [0, 1, 2, 3, 7, 8, 9][:4 if B == 2 else 7]   # rows of environments 0 and 2
        for name in ("states", "eps_p", "eps_q"):
            assert torch.equal(got[name][keep], ref[name][keep]), name
            if latents is bad:
                assert bool(torch.isnan(got[name][4:7]).all()), name
            else:
                assert torch.equal(got[name], ref[name]), name
    assert ctx.tsdp_status() == 0
    ctx.close()


class _FuncAttributes(ctypes.Structure):              # hipFuncAttributes
    _fields_ = [(n, t) for n, t in (("binaryVersion", ctypes.c_int), ("cacheModeCA", ctypes.c_int), ("constSizeBytes", ctypes.c_size_t),
                                    ("localSizeBytes", ctypes.c_size_t), ("maxDynamicSharedSizeBytes", ctypes.c_int), ("maxThreadsPerBlock", ctypes.c_int),
                                    ("numRegs", ctypes.c_int), ("preferredShmemCarveout", ctypes.c_int), ("ptxVersion", ctypes.c_int), ("sharedSizeBytes", ctypes.c_size_t))]


def _declared(lib, symbol):
    attr = _FuncAttributes()
    assert ctypes.CDLL("libamdhip64.so").hipFuncGetAttributes(ctypes.byref(attr), ctypes.c_void_p(ctypes.addressof(ctypes.c_void_p.in_dll(lib, symbol)))) == 0
    return attr.maxDynamicSharedSizeBytes


def test_launches_declare_the_lds_that_they_ask_for():
    # the rollout of d = 256 with cross-attention asks for 134 KB and one KB per component of an action: more for A = 16, the most
    # that 32 tokens allow, than for the context that is loaded last
    from paper_2512_15773_amd import load_library
    wl = ti.replace(ti.C4, base=ti.NetShape(1, 512, 8))
    for A in (16, 2):
        wl = ti.small_variant(wl, B=2, K_max=2, A=A)
        ctx = gpu_side(wl, *(ti.make_weights(wl, which) for which in ("base", "draft")), ti.make_cond(wl, 2))
        ctx.tsdp_prepare()
        ctx.close()
    symbol = "_ZN4tsdp6k_flowINS_7FlowCfgINS_5TBF16ELi256ELi32ELi8ELi64ELi2EEELb1EEEvNS_8FusedNetENS_6FlowIOENSt11conditionalIXT0_ENS_7DraftIOENS_7FewNoneEE4typeE"
    assert _declared(load_library(), symbol) >= 2 * 8 * 32 * 4 + 8 * 4 * 2 * 2 * 1024 + 2 * 512 * 4 + 256 * 16 * 4


@pytest.mark.parametrize("A", [16, 6])
def test_rollouts_with_cross_attention_and_the_most_lds(A):
    wl = ti.small_variant(ti.C4, B=3, K_max=3, A=A, base=ti.NetShape(1, 512, 8))
    _stage_parity(wl, 3, np.array([99, 40, 2]), np.array([3, 1, 3]), np.ones(3))


@pytest.mark.parametrize("layers, B, K_max, A", [(1, 1, 1, 16), (2, 1, 8, 14), (3, 2, 4, 16), (2, 4, 2, 2), (1, 3, 3, 14)])
def test_wide_bases_with_cross_attention(layers, B, K_max, A):
    # up to eight rows of 32 x 512 in one launch (the last case: nine, in launches); A = 16 is the most embedding that shares the LDS of
    # the hidden layer's sums.  Again after another call: the same bits
    wl = ti.small_variant(ti.C4, B=B, K_max=K_max, A=A, base=ti.NetShape(layers, 512, 8))
    t0 = np.linspace(wl.T - 1, 2, B).astype(int); K = np.full(B, K_max)
    _stage_parity(wl, B, t0, K, np.ones(B), norm=layers % 2)
    ctx = _context(wl)
    assert kernels(ctx) == ("k_flow" if B * K_max <= 8 else "k_few", "k_flow")
    x = to_dev(ti.make_latents(wl, B))
    ref = _stages(ctx, x, t0, K, np.ones(B))
    _stages(ctx, x[:1] * 2, t0[:1], K[:1], np.ones(1))
    got = _stages(ctx, x, t0, K, np.ones(B))
    assert all(bool((got[name] == ref[name]).all()) for name in ref) and ctx.tsdp_status() == 0
    ctx.close()
