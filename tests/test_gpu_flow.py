"""Forward passes and rollouts in one launch (csrc/flow_rows.hpp): row counts where the tasks are dealt differently, and the
buffers that every launch has to leave empty."""
import ctypes

import numpy as np
import pytest

import tsdp_inputs as ti
from tests.helpers import gpu_side, to_dev
from tests.test_gpu_parity import _stage_parity

pytestmark = pytest.mark.gpu
STATE = ti.replace(ti.C2, base=ti.NetShape(2, 256, 4))


@pytest.mark.parametrize("wl, B, K_max", [
    (STATE, 7, 1), (STATE, 8, 1),                     # one row per XCD at most: a workgroup per unit
    (STATE, 33, 1), (STATE, 43, 3),                   # five tiles of rows for four groups; groups of four and five
    (STATE, 40, 1), (STATE, 41, 1), (ti.replace(ti.C2, base=ti.NetShape(4, 256, 4)), 14, 4), (ti.replace(ti.C2, base=ti.NetShape(4, 256, 4)), 19, 3),
    (ti.replace(ti.C2, base=ti.NetShape(4, 128, 4)), 8, 2), (ti.replace(ti.C2, base=ti.NetShape(4, 128, 4)), 17, 1),   # fp32 forward passes: the most rows
    # in one launch, the fewest in two launches per layer
    (STATE, 16, 2), (STATE, 17, 2),                   # fp32 rollouts: the most environments in one launch, the fewest in launches
    (ti.replace(ti.C2, base=ti.NetShape(3, 128, 4), draft=ti.NetShape(4, 256, 4)), 18, 7),   # so many launches: in one beyond that too
    (ti.replace(ti.C2, base=ti.NetShape(1, 256, 4), draft=ti.NetShape(4, 128, 4)), 33, 3),   # and in launches
    (ti.replace(ti.C2, base=ti.NetShape(1, 256, 4), draft=ti.NetShape(1, 128, 4)), 2, 5),   # one layer: both sets of buffers in turn
    (ti.replace(ti.C2, base=ti.NetShape(3, 128, 4), draft=ti.NetShape(3, 256, 4)), 2, 4),   # an odd number of layers
    (ti.replace(ti.C4, base=ti.NetShape(1, 512, 8)), 24, 2), (ti.replace(ti.C4, base=ti.NetShape(1, 512, 8)), 25, 2),   # rollout with
    # cross-attention: the largest in one launch, the smallest beyond it; bf16 bases up to 16 rows, and the first beyond
    (ti.replace(ti.C3, base=ti.NetShape(2, 256, 4)), 1, 9), (ti.replace(ti.C3, base=ti.NetShape(1, 256, 4)), 8, 2),
    (ti.replace(ti.C3, base=ti.NetShape(2, 256, 4)), 17, 1), (ti.replace(ti.C5, base=ti.NetShape(1, 384, 6)), 5, 3),
    (ti.replace(ti.C5, base=ti.NetShape(3, 384, 6)), 16, 1),
])
def test_rows_are_dealt_to_the_tasks(wl, B, K_max):
    wl = ti.small_variant(wl, B=B, K_max=K_max)
    rng = np.random.default_rng(B)
    t0 = rng.integers(0, wl.T, B); K = rng.integers(1, K_max + 1, B); s = rng.uniform(1.0, 1.5, B)
    t0[0] = wl.T - 1; K[0] = K_max; t0[-1] = 1
    _stage_parity(wl, B, t0, K, s, norm=B % 2)


@pytest.mark.parametrize("payload", [0xFFFFFFFF, 0x7FC00000])
def test_not_a_number_passes_through_and_leaves_nothing_behind(payload):
    # the pattern of an empty buffer, as a latent: its environment's results are not numbers, the others' and those of the
    # next calls have the same bits as without it
    import torch
    wl = ti.small_variant(STATE, B=3, K_max=4)
    nets = [ti.make_weights(wl, which, b_std=0.02) for which in ("base", "draft")]
    ctx = gpu_side(wl, *nets, ti.make_cond(wl, 3), B_max=3)
    x = to_dev(ti.make_latents(wl, 3)); bad = x.clone()
    bad[1].view(torch.int32).fill_(payload - (1 << 32) if payload >= 1 << 31 else payload)
    t0 = to_dev(np.array([99, 50, 3], np.int32)); K = to_dev(np.array([4, 3, 4], np.int32)); s = to_dev(np.ones(3, np.float32))

    def stages(latents):
        rows = ctx.alloc_rows(3)
        ctx.tsdp_draft(latents, t0, K, s, None, rows)
        ctx.tsdp_verify(3, rows)
        return {k: rows[k][:10].clone() for k in ("states", "eps_p", "eps_q")}
    ref = stages(x)
    for latents in (bad, x, bad, bad, x):
        got = stages(latents)
        keep = [0, 1, 2, 3, 7, 8, 9]                  # rows of environments 0 and 2
        for name in got:
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
