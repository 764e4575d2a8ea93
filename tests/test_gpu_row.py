"""One workgroup per row for networks with run-time sizes (csrc/row_dyn.hpp), at the sizes where its blocks, fragments and
vectors end, against the fp64 oracle."""
import numpy as np
import pytest

import tsdp_inputs as ti
from oracle.denoiser import Denoiser
from tests.helpers import gpu_side, kernels, to_dev
from tests.test_gpu_parity import _stage_parity

pytestmark = pytest.mark.gpu
N = ti.NetShape


@pytest.mark.parametrize("H, A, base, draft, B, K_max", [
    (16, 4, N(2, 96, 3), N(1, 48, 3), 5, 8),             # six and three k-steps; more wavefronts than fragment rows
    (16, 30, N(1, 112, 7), N(3, 16, 1), 3, 5),           # seven k-steps, heads of one fragment, two fragment rows of the head; one k-step
    (16, 5, N(1, 144, 3, 2), N(1, 128, 1), 2, 3),        # nine k-steps: a block and one; a head of eight fragments
    (32, 16, N(2, 80, 5, 3), N(1, 64, 2), 4, 4),         # two token fragments, hidden width of 15 fragments; the most latents of a row
    (16, 4, N(2, 160, 5), N(1, 160, 2), 64, 1),          # larger layers: a second vector on some lanes; 1024 tokens of few heads are in launches
    (16, 4, N(16, 32, 2), N(16, 48, 3), 1, 2),           # the most layers (a base with compiled kernels)
    (16, 4, N(16, 48, 1), N(16, 32, 1), 2, 2),           # the same in both networks
    (16, 4, N(2, 160, 5), N(1, 160, 2), 96, 1),          # the fewest tokens for larger layers of few heads
    (16, 4, N(2, 256, 4, 1), N(1, 256, 2, 1), 96, 1),    # the widest token: two vectors on every lane; a head of 128
    (32, 16, N(1, 96, 1, 8), N(1, 128, 4), 48, 1),       # two token fragments: the widest hidden layer, a head of six fragments
    (16, 32, N(1, 128, 2, 8), N(1, 96, 6, 8), 96, 1),    # the most biases of a layer (1664) and latents of a token
])
@pytest.mark.parametrize("bonus, clip, norm", [(False, None, 0), (True, 1.5, 1)])
def test_one_workgroup_per_row(H, A, base, draft, B, K_max, bonus, clip, norm):
    wl = ti.small_variant(ti.C2, H=H, A=A, cond_dim=32, B=B, K_max=K_max, base=base, draft=draft)
    rng = np.random.default_rng(B)
    t0 = rng.integers(0, wl.T, B); K = rng.integers(1, K_max + 1, B); s = rng.uniform(1.0, 1.5, B)
    t0[0] = wl.T - 1; K[0] = K_max
    if B > 2:
        t0[1], t0[2] = 0, -1                             # a lone base step; a finished environment
    ctx = gpu_side(wl, ti.make_weights(wl, "base"), ti.make_weights(wl, "draft"), ti.make_cond(wl, B), B_max=B, bonus_row=bonus)
    elsewhere = {64: ("k_row" if bonus else "k_few", "k_few"), 1: ("tiles", "k_row")}
    assert kernels(ctx) == elsewhere.get(B, ("k_row", "k_row"))
    ctx.close()
    _stage_parity(wl, B, t0, K, s, clip=clip, norm=norm, bonus=bonus)


def test_equal_networks_predict_the_same():
    wl = ti.small_variant(ti.C2, A=6, cond_dim=32, B=3, K_max=5, base=N(2, 96, 3), draft=N(2, 96, 3))
    w = ti.make_weights(wl, "base", b_std=0.02)
    ctx = gpu_side(wl, w, w, ti.make_cond(wl, 3), B_max=3)
    rows = ctx.alloc_rows(3)
    ctx.tsdp_draft(to_dev(ti.make_latents(wl, 3)), to_dev(np.array([99, 50, 9], np.int32)), to_dev(np.full(3, 5, np.int32)),
                   to_dev(np.ones(3, np.float32)), None, rows)
    ctx.tsdp_verify(3, rows)
    assert kernels(ctx) == ("k_row", "k_row")
    assert bool((rows["eps_p"][:15] == rows["eps_q"][:15]).all())
    ctx.close()


def test_the_activation_is_no_less_exact_than_the_operator_kernels(monkeypatch):
    # a network in which nothing before the activation rounds: latents of +-1024 that RMSNorm makes +-1, hidden features that are
    # sums of 20 of them times powers of two (uniform in +-0.5 .. +-4).  Behind it a power of two lifts the hidden layer above
    # the residual, and the scale of a token is fitted away.  10240 numbers: the two errors' ratio is known to 1 %
    net = N(1, 48, 3)
    B, A, d = 20, 32, net.d
    wl = ti.small_variant(ti.C2, H=16, A=A, cond_dim=32, B=B, K_max=1, base=net, draft=net)
    w = ti.make_weights(wl, "base", w_std=0.0)
    rng = np.random.default_rng(5)
    w["tok_w"][:A] = np.eye(A); w["head_w"][:, :A] = np.eye(A); w["pos"][:, A:] = 1024
    for j in range(A):
        w["l0.up_w"][j, rng.permutation(A)[:20]] = 2.0 ** (j % 4 - 2 - np.arange(20))
    w["l0.dn_w"][:A, :A] = 2.0 ** 26 * np.eye(A)
    x, t, cond = 1024 * rng.choice([-1.0, 1.0], (B, 16, A)).astype(np.float32), np.full(B, 50), ti.make_cond(wl, B)
    want = Denoiser(w, net.layers, net.heads, 0, norm=1)(x, t, cond)

    def errors(names):
        ctx = gpu_side(wl, w, w, cond, B_max=B, norm=1)
        rows = ctx.alloc_rows(B)
        ctx.tsdp_draft(to_dev(x), to_dev(t.astype(np.int32)), to_dev(np.ones(B, np.int32)), to_dev(np.ones(B, np.float32)), None, rows)
        ctx.tsdp_verify(B, rows)
        assert kernels(ctx) == (names, names)
        got = [rows[name][:B].cpu().numpy().reshape(want.shape).astype(np.float64) for name in ("eps_p", "eps_q")]
        ctx.close()
        fit = [g * ((g * want).sum(-1) / (g * g).sum(-1))[..., None] for g in got]
        return [float(np.linalg.norm(g - want) / np.linalg.norm(want)) for g in fit]

    one_workgroup = errors("k_row")
    monkeypatch.setenv("TSDP_DISABLE_FUSED", "1")
    operators = errors("operators")
    print("relative error of the rollout and of the forward pass", one_workgroup, operators)
    assert all(a <= 1.05 * b for a, b in zip(one_workgroup, operators))
