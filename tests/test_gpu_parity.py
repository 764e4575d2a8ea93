"""GPU parity: every C entry point against the CPU oracle on the same seeded inputs (needs an MI355X)."""
import numpy as np
import pytest

import tsdp_inputs as ti
from oracle import philox, spec_round as sr
from tests.helpers import assert_latents_close, drafted_rows, gpu_side, kernels, list_near_ties, oracle_side, scaled_err, to_dev

pytestmark = pytest.mark.gpu

# Tolerances.  Latents (drafted states, final actions): elementwise, rtol 1e-5 for fp32 networks and 2e-2 for bf16
# networks (tests/helpers.py: assert_latents_close).  Intermediate noise predictions: max error relative to the
# tensor's scale below the same numbers (the GPU accumulates dot products of length <= 4d in fp32 through L residual
# layers, the oracle in fp64; bf16 matrix-multiply inputs carry 2^-9 relative rounding).
TOL = {"fp32": 1e-5, "bf16": 2e-2}
TIE = 1e-5          # accept decisions may differ only where |log U - log alpha| is below this


def _setup(wl, B, clip=None, K_max=None, b_std=0.02, head_scale=1.0, seed=None, sampler=0, eta=1.0, bonus=False, norm=0):
    wb = ti.make_weights(wl, "base", b_std=b_std, head_scale=head_scale)
    wd = ti.make_weights(wl, "draft", b_std=b_std, head_scale=head_scale)
    cond = ti.make_cond(wl, B)
    x = ti.make_latents(wl, B)
    base, drafter, sched = oracle_side(wl, wb, wd, sampler=sampler, eta=eta, norm=norm)
    ctx = gpu_side(wl, wb, wd, cond, clip=clip, B_max=B, K_max=K_max, seed=seed, sampler=sampler, eta=eta,
                   bonus_row=bonus, norm=norm)
    return dict(wl=wl, B=B, cond=cond, x=x, base=base, drafter=drafter, sched=sched, ctx=ctx, clip=clip, bonus=bonus,
                seed=wl.philox_seed if seed is None else seed)


def _gpu_draft(S, t0, K, s, env):
    ctx, B = S["ctx"], S["B"]
    rows = ctx.alloc_rows(B)
    ctx.tsdp_draft(to_dev(S["x"]), to_dev(t0.astype(np.int32)), to_dev(K.astype(np.int32)), to_dev(s.astype(np.float32)),
                   None if env is None else to_dev(env.astype(np.int32)), rows)
    return rows


def _check_draft(S, rows, t0, K, s, env, tol):
    o = sr.draft(S["drafter"], S["sched"], S["x"], t0, K, s, env, S["seed"], S["cond"], S["clip"], S["bonus"])
    R = int(o["row_ptr"][-1])
    np.testing.assert_array_equal(rows["row_ptr"].cpu().numpy(), o["row_ptr"])
    np.testing.assert_array_equal(rows["row_t"].cpu().numpy()[:R], o["row_t"])
    np.testing.assert_array_equal(rows["row_env"].cpu().numpy()[:R], o["row_env"])
    xi = rows["xi"].cpu().numpy()[:R]
    np.testing.assert_allclose(xi, o["xi"], rtol=1e-5, atol=2e-6)      # fp32 Box-Muller vs fp64
    e = scaled_err(rows["eps_p"].cpu().numpy()[:R], o["eps_p"])
    print(f"[{S['wl'].name}] draft eps_p: scaled err {e:.3e}")
    assert e < tol, ("eps_p", e)
    w = assert_latents_close(rows["states"].cpu().numpy()[:R], o["states"], S["wl"].dtype, "drafted states")
    w2 = assert_latents_close(rows["y_last"].cpu().numpy(), o["y_last"], S["wl"].dtype, "y_last")
    print(f"[{S['wl'].name}] draft states / y_last: {w:.3f} / {w2:.3f} of the elementwise bound")
    return o


def _check_verify(S, rows, o, tol):
    ctx, B = S["ctx"], S["B"]
    ctx.tsdp_verify(B, rows)
    R = int(o["row_ptr"][-1])
    st = rows["states"].cpu().numpy()[:R]
    ref = sr.verify(S["base"], o["row_env"], o["row_t"], st, S["cond"])   # oracle on the GPU's own states
    got = rows["eps_q"].cpu().numpy()[:R]
    e = scaled_err(got, ref)
    print(f"[{S['wl'].name}] verify eps_q: scaled err {e:.3e}")
    assert e < tol, ("eps_q", e)
    return ref


def _check_accept(S, rows, o, s, env, window):
    """tsdp_accept against the oracle on the identical tensors: indices exact outside the near-tie
    window, latents to fp32 rounding."""
    ctx, B = S["ctx"], S["B"]
    out = ctx.tsdp_accept(B, to_dev(s.astype(np.float32)), None if env is None else to_dev(env.astype(np.int32)), rows)
    R = int(o["row_ptr"][-1])
    g = {k: v.cpu().numpy() for k, v in out.items()}
    ref = sr.accept(S["sched"], o["row_ptr"], o["row_t"], s.astype(np.float32), env, S["seed"],
                    rows["states"].cpu().numpy()[:R], rows["eps_p"].cpu().numpy()[:R], rows["eps_q"].cpu().numpy()[:R],
                    rows["xi"].cpu().numpy()[:R], rows["y_last"].cpu().numpy(), S["clip"], bonus=S["bonus"])
    np.testing.assert_allclose(g["logu"][:R], ref["logu"], rtol=1e-6, atol=1e-7)
    np.testing.assert_allclose(g["logratio"][:R], ref["logratio"], rtol=1e-6, atol=1e-6)
    near = list_near_ties(S["wl"].name, ref["logu"], ref["logratio"], o["row_ptr"], window,
                          drafted_rows(o["row_ptr"], o["row_t"], S["bonus"]))
    diff = g["flags"][:R] != ref["flags"]
    assert not np.any(diff & ~near), "accept flag differs outside the near-tie window"
    env_ok = np.array([not np.any(diff[o["row_ptr"][b]:o["row_ptr"][b + 1]]) for b in range(B)])
    for k in ("n_accept", "n_adv", "t_next"):
        np.testing.assert_array_equal(g[k][env_ok], ref[k][env_ok])
    np.testing.assert_allclose(g["x_out"][env_ok], ref["x_out"][env_ok], rtol=1e-5, atol=1e-6)
    return g, ref, env_ok


def _stage_parity(wl, B, t0, K, s, env=None, clip=None, b_std=0.02, paths=None, sampler=0, eta=1.0, bonus=False, norm=0):
    S = _setup(wl, B, clip=clip, b_std=b_std, sampler=sampler, eta=eta, bonus=bonus, norm=norm)
    if paths is not None:
        assert (S["ctx"].path_name(0), S["ctx"].path_name(1)) == paths
    tol = TOL[wl.dtype]
    rows = _gpu_draft(S, t0, K, s, env)
    o = _check_draft(S, rows, t0, K, s, env, tol)
    _check_verify(S, rows, o, tol)
    g, ref, _ = _check_accept(S, rows, o, s, env, 1e-9)
    S["ctx"].close()
    return g, ref


def test_c1_stages():
    wl = ti.C1
    g, ref = _stage_parity(wl, 1, np.array([9]), np.array([4]), np.array([1.0]), paths=("f32-mfma-fused", "f32-mfma-fused"))
    assert ref["n_adv"][0] >= 1


def test_c1_ragged_edges_with_clip():
    # K_eff = 0 (t0 = 0), finished env, t0 < K, K = 1, per-env sigma scale, env ids, clamped x0
    wl = ti.small_variant(ti.C1, B=8)
    t0 = np.array([9, 0, -1, 2, 5, 7, 1, 9]); K = np.array([4, 4, 4, 4, 1, 1, 3, 2])
    s = np.array([1.0, 1.0, 1.0, 1.3, 1.0, 1.5, 1.2, 1.1]); env = np.array([5, 900, 3, 77, 1, 0, 12345678, 42])
    for clip in (None, 1.0):
        g, ref = _stage_parity(wl, 8, t0, K, s, env, clip=clip)
        np.testing.assert_array_equal(ref["n_adv"][[1, 2, 4]], [1, 0, 1])


def test_c2_stages():
    wl = ti.C2
    _stage_parity(wl, 1, np.array([99]), np.array([8]), np.array([1.0]), paths=("f32-mfma-fused", "f32-mfma-fused"))
    _stage_parity(wl, 1, np.array([50]), np.array([8]), np.array([1.0]))


@pytest.mark.parametrize("name,B", [("C3", 3), ("C5", 6)])
def test_bf16_vector_cond_stages(name, B):
    wl = ti.small_variant(ti.WORKLOADS[name], B=B)
    t0, K, s = ti.make_schedule_inputs(wl, B, t0=None if wl.ragged else 60)
    _stage_parity(wl, B, t0, K, s, paths=("bf16-mfma-fused", "bf16-mfma-fused"))


def test_c4_cross_attention_stages():
    wl = ti.small_variant(ti.C4, B=2, base=ti.NetShape(3, 512, 8))
    t0, K, s = ti.make_schedule_inputs(wl, 2, t0=40)
    _stage_parity(wl, 2, t0, K, s, paths=("bf16-mfma-fused", "bf16-mfma-fused"))


@pytest.mark.parametrize("B, cond_dim, S", [(1, 768, 64), (3, 36, 64), (5, 768, 64)])
def test_cross_attention_operands_at_tile_edges(B, cond_dim, S):
    # the key / value product takes 128 tokens (two environments) at a time and 32 observation features per k-step: odd
    # batches end in half a tile, 36 features in a k-step of 4
    wl = ti.small_variant(ti.C4, B=B, cond_dim=cond_dim, cond_tokens=S, base=ti.NetShape(1, 512, 8), draft=ti.NetShape(1, 256, 8))
    t0 = np.full(B, 50); K = np.full(B, 2); s = np.ones(B)
    _stage_parity(wl, B, t0, K, s, paths=("bf16-mfma-fused", "bf16-mfma-fused"))


@pytest.mark.parametrize("cond_dim, S", [(36, 64), (768, 64)])
def test_keys_and_values_add_the_observation_features_in_order(cond_dim, S):
    # 2^24 + 1 + ... + 1 - 2^24 is zero in fp32 in ascending order (a tie to even every time), and cond_dim - 2 or something
    # between in any other order: an observation of these numbers must give the bits of an observation of zeros
    import torch
    wl = ti.small_variant(ti.C4, B=2, K_max=1, cond_dim=cond_dim, cond_tokens=S, base=ti.NetShape(1, 512, 8), draft=ti.NetShape(1, 256, 8))
    nets = [ti.make_weights(wl, which, b_std=0.02) for which in ("base", "draft")]
    for w in nets:
        for name in w:
            if name.endswith(("ck_w", "cv_w")):
                w[name][:] = 1.0
    cond = np.zeros((2, S, cond_dim), np.float32)
    cond[1, :, 1:-1] = 1.0; cond[1, :, 0] = 2.0 ** 24; cond[1, :, -1] = -2.0 ** 24
    ctx = gpu_side(wl, *nets, cond, B_max=2)
    rows = ctx.alloc_rows(2)
    x = np.repeat(ti.make_latents(wl, 2)[:1], 2, axis=0)
    one = np.ones(2, np.int32)
    ctx.tsdp_draft(to_dev(x), to_dev(50 * one), to_dev(one), to_dev(np.ones(2, np.float32)), to_dev(7 * one), rows)
    ctx.tsdp_verify(2, rows)
    for name in ("eps_p", "eps_q"):
        assert bool(torch.isfinite(rows[name]).all()) and torch.equal(rows[name][0], rows[name][1]), name
    ctx.close()


@pytest.mark.parametrize("cond_dim", [32, 36, 768])
def test_keys_and_values_round_as_their_sums_in_order_do(cond_dim):
    # with weights of one a key is an observation's features added up in ascending order.  The last feature puts that fp32 sum
    # halfway between two bf16 numbers or one unit beside it, so that a sum in any other order rounds the other way in about every
    # second token; the observation that holds the sum itself and zeros must give the same bits.  The last pair of environments: an
    # empty token among the others, a not-a-number and an overflow
    import torch
    n, S = 5, 64
    wl = ti.small_variant(ti.C4, B=2 * n, K_max=1, cond_dim=cond_dim, cond_tokens=S, base=ti.NetShape(1, 512, 8), draft=ti.NetShape(1, 256, 8))
    nets = [ti.make_weights(wl, which) for which in ("base", "draft")]
    for w in nets:
        for name in w:
            if name.endswith(("ck_w", "cv_w")):
                w[name][:] = 1.0
    rng = np.random.default_rng(cond_dim)
    x = rng.standard_normal((n, S, cond_dim)).astype(np.float32)
    part = np.zeros((n, S), np.float32)
    for c in range(cond_dim - 1):
        part += x[:, :, c]
    b = (part.view(np.uint32) & np.uint32(0xFFFF0000)) + np.uint32(0x8000) + rng.integers(0, 2, (n, S)).astype(np.uint32)
    x[:, :, -1] = b.view(np.float32) - part
    x[-1, :8] = 0.0
    total = np.zeros((n, S), np.float32)
    for c in range(cond_dim):
        total += x[:, :, c]
    cond = np.zeros((2 * n, S, cond_dim), np.float32)
    cond[0::2] = x
    cond[1::2, :, 0] = total
    ctx = gpu_side(wl, *nets, cond, B_max=2 * n)
    rows = ctx.alloc_rows(2 * n)
    one = np.ones(2 * n, np.int32)

    def run():
        ctx.tsdp_draft(to_dev(np.repeat(ti.make_latents(wl, 1), 2 * n, axis=0)), to_dev(50 * one), to_dev(one), to_dev(np.ones(2 * n, np.float32)),
                       to_dev(7 * one), rows)
        ctx.tsdp_verify(2 * n, rows)
        return {name: rows[name].clone() for name in ("eps_p", "eps_q")}

    finite = run()
    for name, e in finite.items():
        assert bool(torch.isfinite(e).all()) and torch.equal(e[0::2], e[1::2]), name
    cond[-1, 3, 1] = np.nan; cond[-2, 3, :2] = 3e38
    ctx.tsdp_set_cond(to_dev(cond))
    for name, e in run().items():
        assert torch.equal(e[:-2], finite[name][:-2]) and not bool(torch.isfinite(e[-1]).any()), name
    ctx.close()


def _summed_observations(kind, n, S, cond_dim, rng):
    """Observations [n, S, cond_dim] whose features, added up in ascending order in fp32, end halfway between two bf16 numbers or one
    unit beside, and these sums."""
    x = rng.standard_normal((n, S, cond_dim)).astype(np.float32)
    if kind != "either":
        x = np.abs(x)
    if kind == "cancelling":
        x[:, :, cond_dim // 2:] *= -1
    if kind == "early":                                     # large at once, then small terms of either sign
        x[:, :, cond_dim // 8:] = 0.02 * rng.standard_normal((n, S, cond_dim - cond_dim // 8)).astype(np.float32)
    part = np.zeros((n, S), np.float32)
    for c in range(cond_dim - 1):
        part += x[:, :, c]
    b = (part.view(np.uint32) & np.uint32(0xFFFF0000)) + np.uint32(0x8000) + rng.integers(0, 2, (n, S)).astype(np.uint32)
    x[:, :, -1] = b.view(np.float32) - part
    total = np.zeros((n, S), np.float32)
    for c in range(cond_dim):
        total += x[:, :, c]
    return x, total


@pytest.mark.parametrize("cond_dim", [32, 768, 3072])
@pytest.mark.parametrize("kind", ["either", "one sign", "cancelling", "early"])
def test_keys_and_values_round_as_their_sums_in_order_do_whatever_the_signs(kind, cond_dim):
    # as above (weights of one, an observation against one that holds its sum and zeros), but the sums of the matrix cores and those in order
    # lie up to 20 units of 2^-24 |x| |w| apart (45 with 3072 features); 256 tokens, so that a sum beyond the line is among them
    import torch
    n, S = 4, 64
    wl = ti.small_variant(ti.C4, B=2 * n, K_max=1, cond_dim=cond_dim, cond_tokens=S, base=ti.NetShape(1, 512, 8), draft=ti.NetShape(1, 256, 8))
    nets = [ti.make_weights(wl, which) for which in ("base", "draft")]
    for w in nets:
        for name in w:
            if name.endswith(("ck_w", "cv_w")):
                w[name][:] = 1.0
    x, total = _summed_observations(kind, n, S, cond_dim, np.random.default_rng(cond_dim))
    cond = np.zeros((2 * n, S, cond_dim), np.float32)
    cond[0::2] = x
    cond[1::2, :, 0] = total
    ctx = gpu_side(wl, *nets, cond, B_max=2 * n)
    rows = ctx.alloc_rows(2 * n)
    one = np.ones(2 * n, np.int32)
    ctx.tsdp_draft(to_dev(np.repeat(ti.make_latents(wl, 1), 2 * n, axis=0)), to_dev(50 * one), to_dev(one), to_dev(np.ones(2 * n, np.float32)),
                   to_dev(7 * one), rows)
    ctx.tsdp_verify(2 * n, rows)
    for name in ("eps_p", "eps_q"):
        e = rows[name]
        assert bool(torch.isfinite(e).all()) and torch.equal(e[0::2], e[1::2]), name
    ctx.close()


def _key_observations(kind, B, S, C, rng):
    import torch
    x = rng.standard_normal((B, S, C)).astype(np.float32)
    if kind == "cancelling":
        x = np.abs(x); x[:, :, C // 2:] *= -1
    if kind == "few features":
        x = np.zeros((B, S, C), np.float32); np.put_along_axis(x, rng.integers(0, C, (B, S, 4)), 1.5, axis=2)
    if kind == "not a number":
        x[:] = np.nan
    if kind == "infinite":
        x[:] = np.inf
    return to_dev(x)


def test_keys_and_values_take_a_bounded_time_whatever_the_observations_hold():
    # numbers near a rounding boundary are added up a second time: at worst a tile is multiplied twice, once of them with fp32 operands
    # (2.6 times the time of Gaussian observations; 4.3 with few features and 14.5 with infinities when any share of the numbers was
    # added again one by one).  The fastest of ten repetitions each
    import torch
    B, S, C = 32, 64, 768
    wl = ti.small_variant(ti.C4, B=B, K_max=1, draft=ti.NetShape(2, 256, 8))
    nets = [ti.make_weights(wl, which) for which in ("base", "draft")]
    for w in nets:
        for name in w:
            if name.endswith(("ck_w", "cv_w")):
                w[name] = np.abs(w[name])                   # (for the sums that cancel)
    ctx = gpu_side(wl, *nets, np.zeros((B, S, C), np.float32), B_max=B)
    rng, took = np.random.default_rng(5), {}
    for kind in ("gaussian", "few features", "cancelling", "not a number", "infinite"):
        x = _key_observations(kind, B, S, C, rng)
        ctx.tsdp_set_cond(x)
        took[kind] = np.inf
        for _ in range(10):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(); ctx.tsdp_set_cond(x); ctx.tsdp_set_cond(x); b.record()
            torch.cuda.synchronize()
            took[kind] = min(took[kind], a.elapsed_time(b))
    assert max(took.values()) < 4 * took["gaussian"], took
    ctx.close()


@pytest.mark.parametrize("cond_dim", [36, 768])
@pytest.mark.parametrize("marked, dense", [(16, 0), (15, 0), (128, 0), (0, 11), (0, 13), (0, 128)])
def test_tiles_in_order_give_the_bits_of_tiles_that_are_not(marked, dense, cond_dim):
    # weights of one.  2^24 + 1 + 1 + .. - 2^24 is zero in order and something else otherwise: as three numbers among zeros (a token that
    # counts as marked, 16 in a tile of 128 tokens take it to the fp32 matrix cores at once) or as all features of a token (256 numbers
    # listed for each; 12 of them still are added again one by one).  Each against zeros in its place; the other tokens are the same
    import torch
    wl = ti.small_variant(ti.C4, B=4, K_max=1, cond_dim=cond_dim, cond_tokens=64, base=ti.NetShape(1, 512, 8), draft=ti.NetShape(1, 256, 8))
    nets = [ti.make_weights(wl, which) for which in ("base", "draft")]
    for w in nets:
        for name in w:
            if name.endswith(("ck_w", "cv_w")):
                w[name][:] = 1.0
    rng = np.random.default_rng(marked + dense)
    cond = np.repeat(np.round(rng.standard_normal((1, 128, cond_dim)) * 64).astype(np.float32), 2, axis=0)   # (whole numbers: exact in any order)
    at = rng.permutation(128)[:marked + dense]
    cond[:, at] = 0.0
    few = np.zeros(cond_dim, np.float32); few[[0, cond_dim // 2, cond_dim - 1]] = (2.0 ** 24, 1.0, -2.0 ** 24)
    many = np.ones(cond_dim, np.float32); many[[0, -1]] = (2.0 ** 24, -2.0 ** 24)
    cond[1, at] = few if marked else many
    cond = cond.reshape(4, 64, cond_dim)                    # two tiles of two environments
    ctx = gpu_side(wl, *nets, cond, B_max=4)
    rows = ctx.alloc_rows(4)
    one = np.ones(4, np.int32)
    ctx.tsdp_draft(to_dev(np.repeat(ti.make_latents(wl, 1), 4, axis=0)), to_dev(50 * one), to_dev(one), to_dev(np.ones(4, np.float32)),
                   to_dev(7 * one), rows)
    ctx.tsdp_verify(4, rows)
    for name in ("eps_p", "eps_q"):
        e = rows[name]
        assert bool(torch.isfinite(e).all()) and torch.equal(e[:2], e[2:]), name
    ctx.close()


@pytest.mark.parametrize("wl, B, K_max", [
    (ti.small_variant(ti.C3, A=32, draft=ti.NetShape(16, 128, 4)), 2, 2),       # one row a workgroup, weights in flight: the most LDS
    (ti.small_variant(ti.C3, A=4, draft=ti.NetShape(1, 128, 4)), 1, 64),        # one layer; the most transitions
    (ti.small_variant(ti.C3, A=17, draft=ti.NetShape(3, 128, 4)), 3, 18),       # two fragments of components; more steps than a FiLM batch
    (ti.small_variant(ti.C1, A=32, draft=ti.NetShape(16, 32, 2)), 2, 4),        # the same in fp32
    (ti.small_variant(ti.C1, A=1, draft=ti.NetShape(3, 32, 2)), 2, 4),
    (ti.small_variant(ti.C4, A=16, draft=ti.NetShape(6, 256, 8)), 25, 2),       # token embedding not in LDS
    (ti.small_variant(ti.C5, A=32, ragged=False, draft=ti.NetShape(4, 192, 6)), 768, 1),   # four environments a workgroup, the same
])
@pytest.mark.parametrize("bonus, clip, norm", [(False, None, 0), (True, 1.5, 1)])
def test_rollouts_of_a_workgroup_an_environment(wl, B, K_max, bonus, clip, norm):
    wl = ti.replace(wl, B=B, K_max=K_max, base=ti.NetShape(1, wl.base.d, wl.base.heads))
    t0 = np.full(B, -1); t0[-1] = wl.T // 2; t0[:2] = (wl.T - 1, min(K_max, wl.T - 1) // 2 + 1)[:B]
    _stage_parity(wl, B, t0, np.full(B, K_max), np.full(B, 1.1), clip=clip, bonus=bonus, norm=norm)


@pytest.mark.parametrize("wl, B, rpt", [
    (ti.small_variant(ti.C5, A=8, draft=ti.NetShape(2, 192, 6)), 768, 4),       # four environments a workgroup with more components
    (ti.small_variant(ti.C5, A=7, draft=ti.NetShape(5, 192, 6)), 765, 4),       # and layers: the most that fit; the last workgroup of one environment
    (ti.small_variant(ti.C5, A=32, draft=ti.NetShape(4, 192, 6)), 768, 4),
    (ti.small_variant(ti.C5, A=32, draft=ti.NetShape(5, 192, 6)), 768, 0),      # one too many
    (ti.small_variant(ti.C5, A=32, draft=ti.NetShape(5, 192, 6)), 764, 1),
    (ti.small_variant(ti.C3, A=8, draft=ti.NetShape(11, 128, 4)), 768, 4),
    (ti.small_variant(ti.C3, A=8, draft=ti.NetShape(12, 128, 4)), 768, 0),
    (ti.small_variant(ti.C4, A=16, draft=ti.NetShape(9, 256, 8)), 25, 1),       # cross-attention
    (ti.small_variant(ti.C4, A=1, draft=ti.NetShape(10, 256, 8)), 25, 0),       # more layers than the LDS holds biases and vectors of
    (ti.small_variant(ti.C4, A=16, draft=ti.NetShape(16, 256, 8)), 25, 0),
    (ti.small_variant(ti.C5, A=16, draft=ti.NetShape(13, 384, 6)), 2, 1),
    (ti.small_variant(ti.C5, A=16, draft=ti.NetShape(14, 384, 6)), 2, 0),
    (ti.small_variant(ti.C2, A=32, draft=ti.NetShape(16, 256, 4)), 33, 1),      # fp32
])
def test_rollout_tile_is_the_one_whose_lds_suffices(wl, B, rpt):
    K = 2 if wl.dtype == "fp32" else 1                      # (fp32 rollouts of one transition are spread)
    wl = ti.replace(wl, B=B, K_max=K, ragged=False, base=ti.NetShape(1, wl.base.d, wl.base.heads))
    S = _setup(wl, B, K_max=K)
    lib = S["ctx"].lib
    assert lib.tsdp_internal_rollout_tile(S["ctx"].ctx, B) == rpt
    S["ctx"].close()
    t0 = np.full(B, -1); t0[-1] = wl.T // 2; t0[0] = wl.T - 1
    _stage_parity(wl, B, t0, np.full(B, K), np.full(B, 1.1))


@pytest.mark.parametrize("base, B, K_max", [
    (ti.replace(ti.C2, base=ti.NetShape(2, 256, 4)), 1, 1),       # one row
    (ti.replace(ti.C2, base=ti.NetShape(2, 256, 4)), 9, 1),       # rows not a multiple of the eight XCDs
    (ti.replace(ti.C2, base=ti.NetShape(1, 256, 4)), 16, 8),      # the largest fp32 capacity of the spread kernels (2048 tokens)
    (ti.replace(ti.C2, base=ti.NetShape(1, 256, 4)), 17, 8),      # and the smallest beyond it
    (ti.replace(ti.C5, ragged=False, base=ti.NetShape(2, 384, 6)), 3, 5),
    (ti.replace(ti.C4, base=ti.NetShape(2, 512, 8)), 3, 3),       # wide rows with cross-attention
])
def test_forward_of_few_rows_at_its_edges(base, B, K_max):
    wl = ti.small_variant(base, B=B, K_max=K_max)
    rng = np.random.default_rng(B)
    t0 = rng.integers(0, wl.T, B); K = rng.integers(1, K_max + 1, B); s = rng.uniform(1.0, 1.5, B)
    t0[-1] = min(1, wl.T - 1); K[0] = K_max; t0[0] = wl.T - 1
    _stage_parity(wl, B, t0, K, s, clip=1.5 if B == 9 else None, norm=B == 3, bonus=B == 9)


@pytest.mark.parametrize("dtype, H, base, draft, B", [
    ("fp32", 16, ti.NetShape(2, 112, 7), ti.NetShape(1, 48, 3), 1),      # seven k-steps, heads of one fragment
    ("fp32", 32, ti.NetShape(1, 144, 3, 3), ti.NetShape(1, 16, 1, 1), 3),   # nine k-steps, hidden width 27 fragments; one fragment in all
    ("fp32", 16, ti.NetShape(1, 272, 17), ti.NetShape(1, 96, 3), 2),     # 272 features: a second vector on some lanes
    ("bf16", 16, ti.NetShape(1, 320, 5), ti.NetShape(1, 64, 2), 9),      # bf16 weights, fp32 operands
    ("fp32", 16, ti.NetShape(2, 192, 6), ti.NetShape(2, 208, 13), 5),    # layers too large for a workgroup per row, in both networks
    ("fp32", 32, ti.NetShape(1, 160, 5), ti.NetShape(1, 176, 11), 3),    # the same with two token fragments
    ("bf16", 32, ti.NetShape(1, 192, 3), ti.NetShape(2, 144, 9, 8), 2),
])
def test_few_rows_of_run_time_sizes(dtype, H, base, draft, B):
    wl = ti.small_variant(ti.C2, dtype=dtype, H=H, A=6, cond_dim=32, K_max=3, base=base, draft=draft)
    t0 = np.full(B, 60); t0[-1] = 2
    K = np.full(B, 3); K[0] = 2
    ctx = gpu_side(wl, ti.make_weights(wl, "base"), ti.make_weights(wl, "draft"), ti.make_cond(wl, B), B_max=B)
    assert kernels(ctx) == ("k_row" if base.d == 112 else "k_few", "k_few" if draft.d > 128 else "k_row")
    ctx.close()
    _stage_parity(wl, B, t0, K, np.full(B, 1.1), bonus=B == 2, paths=("f32-ops", "f32-ops"))


def _runs_timed_kernel(ctx, stage):
    # operator sequences are not bracketed by events, every other path of a network is
    from paper_2512_15773_amd.binding import TsdpError
    try:
        ctx.tsdp_kernel_ms(stage)
        return True
    except TsdpError:
        return False


@pytest.mark.parametrize("B, K_max, spread", [(587, 1, (True, True)), (588, 1, (False, False)), (293, 2, (True, True)), (294, 2, (False, True))])
def test_run_time_sizes_on_both_sides_of_their_line(B, K_max, spread):
    # three heads: up to 9400 tokens, of the ragged batch for the base network and of the environments for the drafter
    wl = ti.small_variant(ti.C2, A=4, cond_dim=32, B=B, K_max=K_max, base=ti.NetShape(1, 96, 3), draft=ti.NetShape(1, 48, 3))
    S = _setup(wl, B)
    t0 = np.full(B, -1); t0[[0, B // 2, B - 1]] = (70, 0, 3)
    K = np.full(B, K_max); s = np.full(B, 1.1)
    S["ctx"].tsdp_kernel_timing(True)
    rows = _gpu_draft(S, t0, K, s, None)
    o = _check_draft(S, rows, t0, K, s, None, TOL["fp32"])
    _check_verify(S, rows, o, TOL["fp32"])
    assert (_runs_timed_kernel(S["ctx"], 1), _runs_timed_kernel(S["ctx"], 0)) == spread
    S["ctx"].close()


@pytest.mark.parametrize("dtype, H, base, draft", [
    ("fp32", 8, ti.NetShape(2, 96, 3), ti.NetShape(1, 48, 3)),         # eight tokens
    ("fp32", 16, ti.NetShape(1, 100, 5), ti.NetShape(1, 36, 3)),       # sizes that are not multiples of 16
    ("fp32", 48, ti.NetShape(1, 64, 4, 2), ti.NetShape(1, 32, 2)),     # 48 tokens
    ("bf16", 8, ti.NetShape(1, 256, 4), ti.NetShape(1, 128, 4)),       # bf16 weights
])
@pytest.mark.parametrize("bonus, clip, norm", [(False, None, 0), (True, 1.5, 1)])
def test_operator_kernels_with_vector_conditioning(dtype, H, base, draft, bonus, clip, norm):
    # shapes that neither a compiled kernel nor one with run-time sizes takes: one launch per operator, one pass per drafted transition
    wl = ti.small_variant(ti.C2, dtype=dtype, H=H, A=5, cond_dim=32, B=4, K_max=3, base=base, draft=draft)
    S = _setup(wl, 4, clip=clip, bonus=bonus, norm=norm)
    assert (S["ctx"].path_name(0), S["ctx"].path_name(1)) == ("f32-ops", "f32-ops")
    t0 = np.array([99, 0, -1, 2]); K = np.array([3, 2, 3, 3]); s = np.full(4, 1.1)
    S["ctx"].tsdp_kernel_timing(True)
    rows = _gpu_draft(S, t0, K, s, None)
    o = _check_draft(S, rows, t0, K, s, None, TOL[dtype])
    _check_verify(S, rows, o, TOL[dtype])
    assert not _runs_timed_kernel(S["ctx"], 0) and not _runs_timed_kernel(S["ctx"], 1)
    _check_accept(S, rows, o, s, None, 1e-9)
    S["ctx"].close()


@pytest.mark.parametrize("wl, B", [
    (ti.small_variant(ti.C2, base=ti.NetShape(2, 256, 4)), 129),                        # fp32: 2064 tokens with K_max = 1
    (ti.small_variant(ti.C3, base=ti.NetShape(2, 256, 4)), 137),                        # bf16: 2192
    (ti.small_variant(ti.C5, ragged=False, base=ti.NetShape(2, 384, 6)), 137),
    (ti.small_variant(ti.C4, base=ti.NetShape(1, 512, 8)), 69),                         # 2208 tokens of 32-token rows
])
@pytest.mark.parametrize("bonus, clip, norm", [(False, None, 1), (True, 1.5, 1)])
def test_tile_kernels_just_above_the_few_rows(wl, B, bonus, clip, norm):
    # the smallest contexts whose base network keeps one workgroup per tile; most environments are finished, so that the
    # live rows end inside a tile
    wl = ti.replace(wl, B=B, K_max=1)
    t0 = np.full(B, -1); t0[:5] = (wl.T - 1, 0, 60, 1, 30)
    K = np.ones(B, int); s = np.full(B, 1.1)
    _stage_parity(wl, B, t0, K, s, clip=clip, bonus=bonus, norm=norm)


@pytest.mark.parametrize("wl", [ti.small_variant(ti.C3, base=ti.NetShape(2, 256, 4), draft=ti.NetShape(2, 256, 4), K_max=3),
                                ti.small_variant(ti.C4, base=ti.NetShape(1, 512, 8), draft=ti.NetShape(1, 512, 8), K_max=3)])
def test_few_rows_of_equal_networks_give_equal_predictions(wl):
    # a drafter with the base network's weights: its rollout and the verify forward of the same states agree bit for bit
    import torch
    B = 3
    wb = ti.make_weights(wl, "base", b_std=0.02)
    ctx = gpu_side(wl, wb, wb, ti.make_cond(wl, B), B_max=B)
    rows = ctx.alloc_rows(B)
    K = to_dev(np.array([3, 1, 2], np.int32))
    ctx.tsdp_draft(to_dev(ti.make_latents(wl, B)), to_dev(np.array([90, 40, 9], np.int32)), K, to_dev(np.ones(B, np.float32)), None, rows)
    ctx.tsdp_verify(B, rows)
    assert torch.equal(rows["eps_p"][:6], rows["eps_q"][:6])
    ctx.close()


@pytest.mark.parametrize("B, cond_dim", [(1, 4), (9, 260), (1024, 64), (1025, 64)])
def test_conditioning_vectors_at_the_edges_of_their_kernel(B, cond_dim):
    # eight environments a wavefront, 256 components a step, another kernel beyond 1024 environments
    wl = ti.small_variant(ti.C1, B=B, cond_dim=cond_dim)
    wb = ti.make_weights(wl, "base", b_std=0.02); wd = ti.make_weights(wl, "draft", b_std=0.02)
    cond = ti.make_cond(wl, B)
    ctx = gpu_side(wl, wb, wd, cond, B_max=B)
    rows = ctx.alloc_rows(B)
    t0 = np.full(B, 5, np.int32); one = np.ones(B, np.int32)
    ctx.tsdp_draft(to_dev(ti.make_latents(wl, B)), to_dev(t0), to_dev(one), to_dev(np.ones(B, np.float32)), None, rows)
    ctx.tsdp_verify(B, rows)
    pick = np.unique([0, B // 2, B - 1])
    base, drafter, _ = oracle_side(wl, wb, wd)
    st = rows["states"].cpu().numpy()[pick]
    for net, name in ((drafter, "eps_p"), (base, "eps_q")):
        ref = sr.verify(net, pick, t0[pick], st, cond)
        assert scaled_err(rows[name].cpu().numpy()[pick], ref) < TOL["fp32"], name
    ctx.close()


@pytest.mark.parametrize("which", [0, 1])
def test_reload_of_a_network_onto_the_spread_path(which, monkeypatch):
    # TSDP_DISABLE_FUSED is read by every load: a context that has already run with one network on the operator kernels gets
    # larger buffers when that network returns, and then gives the bits of a fresh context
    import torch
    wl = ti.C2
    nets = [ti.make_weights(wl, name, b_std=0.02) for name in ("base", "draft")]
    cond = ti.make_cond(wl, 1)

    def predictions(ctx):
        rows = ctx.alloc_rows(1)
        ctx.tsdp_draft(to_dev(ti.make_latents(wl, 1)), to_dev(np.array([70], np.int32)), to_dev(np.array([8], np.int32)),
                       to_dev(np.ones(1, np.float32)), None, rows)
        ctx.tsdp_verify(1, rows)
        return torch.stack([rows["eps_p"], rows["eps_q"], rows["states"]])

    fresh = gpu_side(wl, *nets, cond, B_max=1)
    ref = predictions(fresh)
    fresh.close()
    monkeypatch.setenv("TSDP_DISABLE_FUSED", "1")
    ctx = gpu_side(wl, *nets, cond, B_max=1)
    monkeypatch.delenv("TSDP_DISABLE_FUSED")
    for load in (1 - which, which):
        ctx.tsdp_load_weights(load, ti.pack_blob(nets[load]))
        ctx.tsdp_set_cond(to_dev(cond))
        got = predictions(ctx)
        assert scaled_err(got.cpu().numpy(), ref.cpu().numpy()) < TOL[wl.dtype]
    assert torch.equal(got, ref)
    ctx.close()


@pytest.mark.parametrize("cond_dim, few", [(64, 3), (36, 17), (1024, 1)])
def test_conditioning_vectors_do_not_depend_on_the_batch(cond_dim, few):
    # batches of up to 1024 and larger ones take different kernels: the same environments give the same bits in both, and
    # both add the components in ascending order (2^24 + 1 + ... + 1 - 2^24 is zero in fp32 in that order only)
    import torch
    B = 1025
    wl = ti.small_variant(ti.C1, B=B, cond_dim=cond_dim)
    nets = [ti.make_weights(wl, which, b_std=0.02) for which in ("base", "draft")]
    cond = ti.make_cond(wl, B)
    cond[:2] = 0.0
    cond[1, 1:-1] = 1.0; cond[1, 0] = 2.0 ** 24; cond[1, -1] = -2.0 ** 24
    x = ti.make_latents(wl, B); x[1] = x[0]

    def predictions(ctx, n):
        ctx.tsdp_set_cond(to_dev(cond[:n]))
        rows = ctx.alloc_rows(n)
        one = np.ones(n, np.int32)
        ctx.tsdp_draft(to_dev(x[:n]), to_dev(5 * one), to_dev(one), to_dev(np.ones(n, np.float32)), None, rows)
        ctx.tsdp_verify(n, rows)
        return torch.stack([rows["eps_p"][:n], rows["eps_q"][:n]])

    ctx = gpu_side(wl, *nets, cond, B_max=B)
    assert torch.equal(predictions(ctx, B)[:, :few], predictions(ctx, few))
    for w in nets:
        w["c_w"][:] = 1.0
    for which, w in enumerate(nets):
        ctx.tsdp_load_weights(which, ti.pack_blob(w))
    for n in (2, B):
        got = predictions(ctx, n)
        assert torch.equal(got[:, 0], got[:, 1]), n
    ctx.close()


@pytest.mark.parametrize("B", [127, 129, 1024, 1025])
@pytest.mark.parametrize("bonus", [False, True])
def test_row_table_and_chain_totals_over_the_batch_size(B, bonus):
    # the row table is one launch up to 1024 environments and two beyond; a chain counts in its acceptance kernel
    import torch
    wl = ti.small_variant(ti.C1, B=B)
    rng = np.random.default_rng(B)
    t0 = rng.integers(-1, wl.T, B).astype(np.int32); K = rng.integers(0 if bonus else 1, wl.K_max + 1, B).astype(np.int32)
    ctx = gpu_side(wl, ti.make_weights(wl, "base"), ti.make_weights(wl, "draft"), ti.make_cond(wl, B), B_max=B, bonus_row=bonus)
    rows = ctx.alloc_rows(B)
    x = to_dev(ti.make_latents(wl, B)); s = to_dev(np.ones(B, np.float32))
    ctx.tsdp_draft(x, to_dev(t0), to_dev(K), s, None, rows)
    ke, ptr = sr.plan_rows(t0, K, bonus)[:2]
    np.testing.assert_array_equal(rows["row_ptr"].cpu().numpy(), ptr)
    first = np.repeat(np.asarray(ptr)[:-1], np.diff(ptr))
    np.testing.assert_array_equal(rows["row_t"].cpu().numpy()[:ptr[-1]], np.repeat(t0, np.diff(ptr)) - (np.arange(ptr[-1]) - first))
    assert ctx.tsdp_status() == 0
    td = to_dev(t0)
    rounds, tot = ctx.tsdp_chain(x, td, to_dev(np.maximum(K, 1)), s, None, check_every=1)
    live = np.asarray(t0) >= 0
    assert bool((td < 0).all().item()) and rounds == int(tot["rounds"].max().item())
    assert bool((tot["rounds"][~torch.from_numpy(live).cuda()] == 0).all().item())
    # every step is an accepted draft, a reflected one or a base step, at most one of the latter two a round
    adv = (tot["accept"] + tot["rounds"]).cpu().numpy()
    assert (adv[live] >= t0[live] + 1).all() and (tot["accept"].cpu().numpy() <= tot["drafts"].cpu().numpy()).all()
    ctx.close()


def _round_parity(wl, B, t0, K, s, env, head_scale=1.0):
    """tsdp_round against the oracle's round.  The same inputs also go through the three stages with diagnostics,
    which gives the GPU's own log alpha of every row: the fused round must equal the stages bit for bit, accept
    decisions must equal the oracle's outside the near-tie window (near-tie rows are printed), and the final actions
    of every compared environment must agree elementwise.  At least one environment must be compared."""
    import torch
    S = _setup(wl, B, head_scale=head_scale)
    ctx = S["ctx"]
    sd = to_dev(s.astype(np.float32)); ed = None if env is None else to_dev(env.astype(np.int32))
    rows = _gpu_draft(S, t0, K, s, env)
    ctx.tsdp_verify(B, rows)
    st = {k: v.cpu().numpy() for k, v in ctx.tsdp_accept(B, sd, ed, rows).items()}
    x = to_dev(S["x"]); t = to_dev(t0.astype(np.int32))
    nacc = torch.zeros(B, dtype=torch.int32, device="cuda"); nadv = torch.zeros_like(nacc)
    ctx.tsdp_round(x, t, to_dev(K.astype(np.int32)), sd, ed, nacc, nadv)
    g = dict(x=x.cpu().numpy(), t=t.cpu().numpy(), nacc=nacc.cpu().numpy(), nadv=nadv.cpu().numpy())
    np.testing.assert_array_equal(g["nacc"], st["n_accept"])
    np.testing.assert_array_equal(g["nadv"], st["n_adv"])
    np.testing.assert_array_equal(g["t"], st["t_next"])
    np.testing.assert_array_equal(g["x"], st["x_out"])
    ref = sr.spec_round(S["base"], S["drafter"], S["sched"], S["x"], t0, K, s, env, S["seed"], S["cond"])
    d = ref["draft"]; rp = d["row_ptr"]; R = int(rp[-1])
    drafted = d["row_t"] > 0
    near = list_near_ties(wl.name, ref["logu"], ref["logratio"], rp, TIE, drafted)
    dl = np.abs(st["logratio"][:R] - ref["logratio"])
    # rows up to the oracle's first rejection see the same states on both sides: there the decisions are comparable
    seen = np.zeros(R, bool)
    for b in range(B):
        seen[rp[b]:rp[b] + min(int(ref["n_accept"][b]) + 1, rp[b + 1] - rp[b])] = True
    print(f"[{wl.name}] round: max |log alpha (GPU) - log alpha (oracle)| on compared rows = {dl[seen & drafted].max(initial=0.0):.3e}")
    mism = (st["flags"][:R] != ref["flags"]) & seen & drafted
    # a decision may differ inside the near-tie window, or where the network's own rounding error on log alpha (the
    # GPU's fp32 / bf16 forward against the oracle's fp64, shown here per row) reaches the margin of that row
    margin = np.abs(ref["logu"] - ref["logratio"])
    for r in np.nonzero(mism)[0]:
        print(f"[{wl.name}] row {int(r)}: decision differs, margin {margin[r]:.3e}, network error on log alpha {dl[r]:.3e}")
    bad = mism & ~near & (margin > dl + TIE)
    assert not np.any(bad), ("accept decision differs outside the near-tie window", np.nonzero(bad)[0], margin[bad], dl[bad])
    ok = np.array([not np.any((near | mism)[rp[b]:rp[b + 1]] & seen[rp[b]:rp[b + 1]]) for b in range(B)])
    assert ok.any(), "every environment has a near-tie row: nothing was compared"
    np.testing.assert_array_equal(g["nacc"][ok], ref["n_accept"][ok])
    np.testing.assert_array_equal(g["nadv"][ok], ref["n_adv"][ok])
    np.testing.assert_array_equal(g["t"][ok], ref["t_next"][ok])
    w = assert_latents_close(g["x"][ok], ref["x_out"][ok], wl.dtype, "final actions of tsdp_round")
    print(f"[{wl.name}] round: {int(ok.sum())}/{B} environments compared, final actions at {w:.3f} of the elementwise bound")
    assert ctx.tsdp_status() == 0
    ctx.close()
    return ref, ~ok


def test_c1_round():
    ref, near = _round_parity(ti.C1, 1, np.array([9]), np.array([4]), np.array([1.0]), None)
    assert not near.any()


def test_c2_round_and_chain():
    wl = ti.C2
    for t0 in (99, 50, 8, 3):
        ref, near = _round_parity(wl, 1, np.array([t0]), np.array([8]), np.array([1.0]), None)
        assert not near.any()


def test_round_ragged_batch_fp32():
    wl = ti.small_variant(ti.C2, B=12, base=ti.NetShape(3, 256, 4))
    rng = np.random.default_rng(3)
    t0 = rng.integers(-1, 100, 12); K = rng.integers(1, 9, 12); s = rng.uniform(1, 1.5, 12)
    t0[:3] = [0, -1, 2]
    ref, near = _round_parity(wl, 12, t0, K, s, np.arange(12) + 1000, head_scale=0.5)
    assert near.sum() <= 2
    assert (ref["n_accept"] > 0).any() and (ref["n_accept"] < ref["draft"]["K_eff"]).any()


def test_device_status_reports_clamped_inputs():
    wl = ti.C1
    S = _setup(wl, 1)
    rows = S["ctx"].alloc_rows(1)
    S["ctx"].tsdp_draft(to_dev(S["x"]), to_dev(np.array([50], np.int32)), to_dev(np.array([9], np.int32)),
                        to_dev(np.array([1.0], np.float32)), None, rows)
    assert S["ctx"].tsdp_status() == 3                                # K > K_max and t0 >= T, both clamped
    assert rows["row_ptr"].cpu().numpy().tolist() == [0, 4]
    assert rows["row_t"].cpu().numpy()[:4].tolist() == [9, 8, 7, 6]
    assert S["ctx"].tsdp_status() == 0
    # K = 0 has no meaning without the bonus row: reported and run as K = 1
    S["ctx"].tsdp_draft(to_dev(S["x"]), to_dev(np.array([5], np.int32)), to_dev(np.array([0], np.int32)),
                        to_dev(np.array([1.0], np.float32)), None, rows)
    assert S["ctx"].tsdp_status() == 1
    assert rows["row_ptr"].cpu().numpy().tolist() == [0, 1] and rows["row_t"].cpu().numpy()[0] == 5
    np.testing.assert_array_equal(rows["states"].cpu().numpy()[0], np.asarray(S["x"][0], np.float32))
    S["ctx"].close()


def test_error_paths_return_codes():
    import torch
    from paper_2512_15773_amd import Tsdp, TsdpError
    wl = ti.C1
    ctx = Tsdp.from_workload(wl)
    x = torch.zeros(1, wl.H, wl.A, device="cuda"); i = torch.zeros(1, dtype=torch.int32, device="cuda")
    f = torch.ones(1, device="cuda")
    with pytest.raises(TsdpError) as e:
        ctx.tsdp_round(x, i, i, f, None)
    assert e.value.code == -5                                          # weights not loaded
    with pytest.raises(TsdpError) as e:
        ctx.tsdp_load_weights(0, np.zeros(7, np.float32))
    assert e.value.code == -2
    ctx.tsdp_load_weights(0, ti.pack_blob(ti.make_weights(wl, "base")))
    ctx.tsdp_load_weights(1, ti.pack_blob(ti.make_weights(wl, "draft")))
    with pytest.raises(TsdpError) as e:
        ctx.tsdp_round(x, i, i, f, None)
    assert e.value.code == -5                                          # conditioning not set
    ctx.tsdp_set_cond(torch.zeros(1, wl.cond_dim, device="cuda"))
    x2 = torch.zeros(2, wl.H, wl.A, device="cuda")
    with pytest.raises(TsdpError) as e:
        ctx.tsdp_round(x2, torch.zeros(2, dtype=torch.int32, device="cuda"), torch.zeros(2, dtype=torch.int32, device="cuda"),
                       torch.ones(2, device="cuda"), None)
    assert e.value.code == -2                                          # B > B_max
    ctx.tsdp_round(x, i, i, f, None)
    # the enqueue-only chain: negative round count, bad stage bounds, null latents
    with pytest.raises(TsdpError) as e:
        ctx.tsdp_chain_enqueue(x, i, i, f, None, None, -1)
    assert e.value.code == -1
    with pytest.raises(TsdpError) as e:
        ctx.tsdp_chain_enqueue(x, i, torch.zeros(1, 3, dtype=torch.int32, device="cuda"), torch.ones(1, 3, device="cuda"),
                               None, None, 2, stages=(2, 3))
    assert e.value.code == -1
    assert ctx.lib.tsdp_chain_enqueue(ctx.ctx, 1, None, None, None, None, None, 0, 0, 0, None, 1, None, None, None, None, None) == -1
    assert ctx.lib.tsdp_prepare(None) == -1
    ctx.close()


def test_threshold_rule_matches_oracle():
    # deterministic p >= lambda rule (Section 3.2) on identical tensors: flags exact outside the near-tie window
    wl = ti.small_variant(ti.C2, B=10, base=ti.NetShape(2, 256, 4))
    S = _setup(wl, 10, head_scale=0.5)
    rng = np.random.default_rng(4)
    t0 = rng.integers(0, 100, 10); K = rng.integers(1, 9, 10); s = rng.uniform(1, 1.5, 10); lam = rng.uniform(0.05, 1.0, 10)
    lam[0] = 1.0
    rows = _gpu_draft(S, t0, K, s, None)
    S["ctx"].tsdp_verify(10, rows)
    out = S["ctx"].tsdp_accept_threshold(10, to_dev(s.astype(np.float32)), to_dev(lam.astype(np.float32)), rows)
    g = {k: v.cpu().numpy() for k, v in out.items()}
    R = int(rows["row_ptr"].cpu().numpy()[-1])
    ref = sr.accept(S["sched"], rows["row_ptr"].cpu().numpy(), rows["row_t"].cpu().numpy()[:R], s.astype(np.float32), None,
                    S["seed"], rows["states"].cpu().numpy()[:R], rows["eps_p"].cpu().numpy()[:R],
                    rows["eps_q"].cpu().numpy()[:R], rows["xi"].cpu().numpy()[:R], rows["y_last"].cpu().numpy(),
                    lam=lam.astype(np.float32))
    near = np.abs(ref["logu"] - ref["logratio"]) < 1e-6
    assert not np.any((g["flags"][:R] != ref["flags"]) & ~near)
    assert not near.any()
    for k in ("n_accept", "n_adv", "t_next"):
        np.testing.assert_array_equal(g[k], ref[k])
    np.testing.assert_allclose(g["x_out"], ref["x_out"], rtol=1e-5, atol=1e-6)
    assert 0 < g["flags"][:R].sum() < R
    # the fused round with the same thresholds gives the same counters
    import torch
    x = to_dev(S["x"]); t = to_dev(t0.astype(np.int32)); na = torch.zeros(10, dtype=torch.int32, device="cuda"); nd = torch.zeros_like(na)
    S["ctx"].tsdp_round_threshold(x, t, to_dev(K.astype(np.int32)), to_dev(s.astype(np.float32)), None,
                                  to_dev(lam.astype(np.float32)), na, nd)
    np.testing.assert_array_equal(na.cpu().numpy(), ref["n_accept"])
    np.testing.assert_array_equal(t.cpu().numpy(), ref["t_next"])
    S["ctx"].close()


def test_chain_runs_rounds_until_every_environment_finishes():
    # fp32: the chain driver must equal the oracle's round applied repeatedly (same noise stream, same decisions)
    wl = ti.small_variant(ti.C1, B=6)
    S = _setup(wl, 6, head_scale=0.6)
    t0 = np.array([9, 9, 6, 3, 0, -1]); K = np.array([4, 2, 4, 3, 4, 4]); s = np.array([1.0, 1.2, 1.0, 1.0, 1.0, 1.0])
    x = to_dev(S["x"]); t = to_dev(t0.astype(np.int32))
    rounds, tot = S["ctx"].tsdp_chain(x, t, to_dev(K.astype(np.int32)), to_dev(s.astype(np.float32)), None, check_every=1)
    xr, tr = np.asarray(S["x"], float), t0.copy()
    acc = np.zeros(6, int); drafts = np.zeros(6, int); nr = np.zeros(6, int); n = 0
    while (tr >= 0).any():
        r = sr.spec_round(S["base"], S["drafter"], S["sched"], xr, tr, K, s, None, S["seed"], S["cond"])
        ran = tr >= 0
        acc += r["n_accept"]; drafts += r["draft"]["K_eff"]; nr += ran
        near = list_near_ties("C1 chain", r["logu"], r["logratio"], r["draft"]["row_ptr"], TIE, r["draft"]["row_t"] > 0)
        assert not near.any()                                             # no near-tie on this seed: decisions are comparable
        xr, tr = r["x_out"], r["t_next"]; n += 1
    assert rounds == n
    assert (t.cpu().numpy() == -1).all()
    np.testing.assert_array_equal(tot["accept"].cpu().numpy(), acc)
    np.testing.assert_array_equal(tot["drafts"].cpu().numpy(), drafts)
    np.testing.assert_array_equal(tot["rounds"].cpu().numpy(), nr)
    # up to four rounds compound their fp32 rounding in the final action: the per-round bound, once per round
    assert assert_latents_close(x.cpu().numpy(), xr, "fp32", "final actions of the chain") <= 1.0
    S["ctx"].close()


def test_chain_bf16_invariants():
    # every environment ends at t = -1 and the rounds it ran advance it by exactly t0 + 1 steps in total
    wl = ti.small_variant(ti.C3, B=12)
    S = _setup(wl, 12, head_scale=0.2, b_std=0.0)
    t0 = np.array([99, 99, 80, 64, 50, 33, 17, 16, 15, 1, 0, -1]); K = np.full(12, 16); s = np.ones(12)
    x = to_dev(S["x"]); t = to_dev(t0.astype(np.int32))
    rounds, tot = S["ctx"].tsdp_chain(x, t, to_dev(K.astype(np.int32)), to_dev(s.astype(np.float32)), None, check_every=3)
    assert (t.cpu().numpy() == -1).all() and np.isfinite(x.cpu().numpy()).all()
    a, d, r = (tot[k].cpu().numpy() for k in ("accept", "drafts", "rounds"))
    assert r[-1] == 0 and r[-2] == 1 and (r[:-1] >= 1).all() and rounds >= r.max()
    assert (a <= d).all() and (a[:4] > 0).all()
    # steps advanced = accepted drafts + one corrected / base step per round that did not accept everything;
    # at least one step per round and never more than t0 + 1 in total
    assert ((a + r >= t0 + 1) | (t0 < 0)).all()
    S["ctx"].close()


def test_operator_kernel_path_for_shapes_without_a_fused_kernel():
    # a width with no compiled fused kernel (d = 96) runs the general fp32 operator kernels, both conditioning modes
    for cm, extra in ((0, {}), (1, dict(cond_dim=24, cond_tokens=5))):
        wl = ti.small_variant(ti.C1, B=3, cond_mode=cm, base=ti.NetShape(2, 96, 3), draft=ti.NetShape(1, 48, 3), **extra)
        t0 = np.array([9, 4, 0]); K = np.array([4, 3, 2]); s = np.array([1.0, 1.3, 1.0])
        _stage_parity(wl, 3, t0, K, s, paths=("f32-ops", "f32-ops"))


def test_distillation_loss_matches_oracle():
    wl = ti.small_variant(ti.C2, B=9, base=ti.NetShape(2, 256, 4))
    for clip in (None, 1.5):
        S = _setup(wl, 9, clip=clip)
        t0 = np.array([99, 70, 40, 20, 9, 3, 1, 0, -1]); K = np.full(9, 8); s = np.ones(9)
        rows = _gpu_draft(S, t0, K, s, None)
        S["ctx"].tsdp_verify(9, rows)
        R = int(rows["row_ptr"].cpu().numpy()[-1])
        got = S["ctx"].tsdp_distill_loss(R, rows, 0.7, 0.3).cpu().numpy()
        ref = sr.distill_loss(S["sched"], rows["row_t"].cpu().numpy()[:R], rows["states"].cpu().numpy()[:R],
                              rows["eps_p"].cpu().numpy()[:R], rows["eps_q"].cpu().numpy()[:R],
                              float(np.float32(0.7)), float(np.float32(0.3)), clip)   # the ABI takes the weights as fp32
        np.testing.assert_allclose(got, ref, rtol=1e-10)
        again = S["ctx"].tsdp_distill_loss(R, rows, 0.7, 0.3).cpu().numpy()
        assert got.tobytes() == again.tobytes()                            # fixed reduction order
        assert got[0] > 0 and got[1] > 0
        S["ctx"].close()


def test_ddim_sampler_stages_and_loss():
    # DDIM(eta) transitions in the draft step, the acceptance ratio, the reflection, the last step and the loss
    wl = ti.small_variant(ti.C1, B=7)
    t0 = np.array([9, 6, 3, 1, 0, -1, 9]); K = np.array([4, 4, 4, 2, 4, 4, 1]); s = np.array([1.0, 1.3, 1.0, 1.0, 1.0, 1.0, 1.1])
    for clip in (None, 1.0):
        _stage_parity(wl, 7, t0, K, s, clip=clip, sampler=1, eta=0.6)
    wl = ti.small_variant(ti.C3, B=4)
    t0, K, s = ti.make_schedule_inputs(wl, 4, t0=45)
    _stage_parity(wl, 4, t0, K, s, sampler=1, eta=1.0, paths=("bf16-mfma-fused", "bf16-mfma-fused"))
    S = _setup(ti.small_variant(ti.C2, B=3, base=ti.NetShape(2, 256, 4)), 3, clip=2.0, sampler=1, eta=0.5)
    rows = _gpu_draft(S, np.array([60, 9, 0]), np.full(3, 8), np.ones(3), None)
    S["ctx"].tsdp_verify(3, rows)
    R = int(rows["row_ptr"].cpu().numpy()[-1])
    got = S["ctx"].tsdp_distill_loss(R, rows, 1.0, 1.0).cpu().numpy()
    ref = sr.distill_loss(S["sched"], rows["row_t"].cpu().numpy()[:R], rows["states"].cpu().numpy()[:R],
                          rows["eps_p"].cpu().numpy()[:R], rows["eps_q"].cpu().numpy()[:R], 1.0, 1.0, 2.0)
    np.testing.assert_allclose(got, ref, rtol=1e-10)
    S["ctx"].close()


def test_bonus_row_stages_rounds_and_chain():
    # K+1 candidate set: the extra base row in the row table, in verification and in the commit; K = 0 = plain base step
    wl = ti.small_variant(ti.C1, B=8)
    t0 = np.array([9, 0, -1, 2, 5, 7, 1, 9]); K = np.array([4, 4, 4, 4, 0, 1, 3, 2])
    s = np.array([1.0, 1.0, 1.0, 1.3, 1.0, 1.5, 1.2, 1.1]); env = np.array([5, 900, 3, 77, 1, 0, 12345678, 42])
    for clip in (None, 1.0):
        g, ref = _stage_parity(wl, 8, t0, K, s, env, clip=clip, bonus=True)
        np.testing.assert_array_equal(ref["n_adv"][[1, 2, 4]], [1, 0, 1])
        assert (ref["n_adv"] == ref["n_accept"] + 1)[t0 >= 0].all()     # a corrected or a base step ends every round
    wl = ti.small_variant(ti.C3, B=5)
    t0, K, s = ti.make_schedule_inputs(wl, 5, t0=45)
    t0[3] = 2; t0[4] = 0
    _stage_parity(wl, 5, t0, K, s, bonus=True, paths=("bf16-mfma-fused", "bf16-mfma-fused"))
    # identical networks: every draft passes and each round advances K_eff + 1 exact base steps
    wl = ti.small_variant(ti.C1, B=4)
    wb = ti.make_weights(wl, "base", b_std=0.02)
    cond = ti.make_cond(wl, 4); x0 = ti.make_latents(wl, 4)
    wl_same = ti.small_variant(wl, draft=wl.base)
    base, _, sched = oracle_side(wl_same, wb, wb)
    ctx = gpu_side(wl_same, wb, wb, cond, B_max=4, bonus_row=True)
    t0 = np.array([9, 9, 4, 1]); K = np.array([3, 2, 4, 4]); s = np.ones(4)
    x = to_dev(x0); t = to_dev(t0.astype(np.int32))
    rounds, tot = ctx.tsdp_chain(x, t, to_dev(K.astype(np.int32)), to_dev(s.astype(np.float32)), None, check_every=2)
    ref = sr.chain(base, base, sched, x0, t0, K, s, None, wl.philox_seed, cond, bonus=True)
    assert rounds >= ref["rounds"] and (t.cpu().numpy() == -1).all()
    np.testing.assert_array_equal(tot["rounds"].cpu().numpy(), ref["totals"]["rounds"])
    np.testing.assert_array_equal(tot["rounds"].cpu().numpy(), [3, 4, 1, 1])            # ceil((t0+1)/(K+1))
    np.testing.assert_array_equal(tot["accept"].cpu().numpy(), ref["totals"]["accept"])
    assert_latents_close(x.cpu().numpy(), ref["x"], "fp32", "final actions of the bonus-row chain")
    ctx.close()


@pytest.mark.parametrize("bonus", [False, True])
def test_row_table_of_a_batch_of_several_thousand_environments(bonus):
    # the plan kernel scans environments in chunks of 1024: a batch over several chunks with a ragged tail, finished
    # environments, t0 = 0 and (bonus row) K = 0 against the oracle's row table; the base rows' states are the inputs
    B = 2500
    wl = ti.small_variant(ti.C1, B=B)
    rng = np.random.default_rng(77)
    t0 = rng.integers(-1, wl.T, B); K = rng.integers(0 if bonus else 1, wl.K_max + 1, B)
    t0[1023:1026] = [0, -1, wl.T - 1]; K[1023:1026] = [wl.K_max, 1, 0 if bonus else 1]
    S = _setup(wl, B, bonus=bonus)
    rows = _gpu_draft(S, t0, K, np.ones(B), None)
    K_eff, row_ptr, row_env, row_t = sr.plan_rows(t0, K, bonus)
    R = int(row_ptr[-1])
    np.testing.assert_array_equal(rows["row_ptr"].cpu().numpy(), row_ptr)
    np.testing.assert_array_equal(rows["row_t"].cpu().numpy()[:R], row_t)
    np.testing.assert_array_equal(rows["row_env"].cpu().numpy()[:R], row_env)
    first = row_ptr[:-1][np.diff(row_ptr) > 0]                       # every running environment's first row holds x
    live = np.flatnonzero(np.diff(row_ptr) > 0)
    np.testing.assert_array_equal(rows["states"].cpu().numpy()[first], S["x"][live])
    assert S["ctx"].tsdp_status() == 0
    S["ctx"].close()


def test_two_contexts_on_two_streams_do_not_share_state():
    # two contexts (different shapes, both with a FiLM product on their own second stream) run whole rounds at the same
    # time on two streams; every result is bit-identical to the same rounds run one context after the other
    import torch
    specs = [(ti.small_variant(ti.C3, B=24), 24, 30), (ti.small_variant(ti.C5, B=40), 40, None)]
    S, inputs = [], []
    for wl, B, t_fix in specs:
        S.append(_setup(wl, B, head_scale=0.3))
        t0, K, s = ti.make_schedule_inputs(wl, B, t0=t_fix)
        inputs.append((t0.astype(np.int32), K.astype(np.int32), s.astype(np.float32)))

    def tensors(i):
        t0, K, s = inputs[i]
        return dict(x=to_dev(S[i]["x"]), t=to_dev(t0), K=to_dev(K), s=to_dev(s),
                    na=torch.zeros(len(t0), dtype=torch.int32, device="cuda"),
                    nd=torch.zeros(len(t0), dtype=torch.int32, device="cuda"))

    def rounds(i, T, stream, n=3):
        with torch.cuda.stream(stream):
            for _ in range(n):
                S[i]["ctx"].tsdp_round(T["x"], T["t"], T["K"], T["s"], None, T["na"], T["nd"])

    main = torch.cuda.current_stream()
    want = [tensors(0), tensors(1)]
    for i in range(2):
        rounds(i, want[i], main)
        torch.cuda.synchronize()
    # every input exists (and stays alive) before anything is enqueued on the side streams: a tensor freed while a
    # stream that the allocator does not know of still reads it would be handed out again
    got = [tensors(0), tensors(1)]
    torch.cuda.synchronize()
    st = [torch.cuda.Stream(), torch.cuda.Stream()]
    rounds(0, got[0], st[0]); rounds(1, got[1], st[1])         # enqueued back to back, nothing waits in between
    torch.cuda.synchronize()
    for i in range(2):
        for name in ("x", "t", "na", "nd"):
            assert torch.equal(got[i][name], want[i][name]), (i, name)
        assert S[i]["ctx"].tsdp_status() == 0
        S[i]["ctx"].close()


def test_timed_rollouts_contain_their_film_product():
    # 128 environments draft once; with K_max = 64 their FiLM product has 64 times the rows (100 MB of vectors), the rollout is the same
    import torch
    took = []
    for K_max in (1, 64):
        wl = ti.small_variant(ti.C2, A=4, B=128, K_max=K_max, cond_dim=64, base=ti.NetShape(1, 96, 3), draft=ti.NetShape(16, 48, 3))
        S = _setup(wl, 128, K_max=K_max)
        ctx = S["ctx"]
        assert kernels(ctx)[1] == "k_row"
        ctx.tsdp_kernel_timing(2)
        ms = []
        for _ in range(5):
            _gpu_draft(S, np.full(128, 50), np.ones(128), np.ones(128), None)
            ms.append(ctx.tsdp_kernel_ms(0))
        took.append(min(ms))
        ctx.close()
    assert took[1] > 1.15 * took[0], took


def test_kernel_timing_brackets_the_chosen_stages():
    # measurement aid: event pairs around the stage kernels; a stage without a timed launch is an error, not a number
    from paper_2512_15773_amd import TsdpError
    wl = ti.small_variant(ti.C3, B=6)
    S = _setup(wl, 6)
    ctx = S["ctx"]
    t0, K, s = ti.make_schedule_inputs(wl, 6, t0=40)
    rows = _gpu_draft(S, t0, K, s, None)
    ctx.tsdp_verify(6, rows)
    ctx.tsdp_accept(6, to_dev(s.astype(np.float32)), None, rows)
    before = {k: v.clone() for k, v in rows.items()}
    ctx.tsdp_kernel_timing(True)                               # all stages
    with pytest.raises(TsdpError):
        ctx.tsdp_kernel_ms(1)                                  # nothing launched since timing was switched on
    ctx.tsdp_draft(to_dev(S["x"]), to_dev(t0.astype(np.int32)), to_dev(K.astype(np.int32)), to_dev(s.astype(np.float32)),
                   None, rows)
    ctx.tsdp_verify(6, rows)
    ctx.tsdp_accept(6, to_dev(s.astype(np.float32)), None, rows)
    ms = [ctx.tsdp_kernel_ms(st) for st in range(4)]           # rollout, verify forward, acceptance, FiLM product
    assert all(0.0 < m < 1000.0 for m in ms), ms
    for k in ("states", "eps_p", "eps_q", "xi", "row_t"):      # timing changes no result
        assert torch_equal(rows[k], before[k]), k
    ctx.tsdp_kernel_timing(2 * 0b0010)                         # the verify forward only
    ctx.tsdp_verify(6, rows)
    assert ctx.tsdp_kernel_ms(1) > 0.0
    for st in (0, 2, 3):
        with pytest.raises(TsdpError):
            ctx.tsdp_kernel_ms(st)
    ctx.tsdp_kernel_timing(False)
    ctx.close()


def torch_equal(a, b):
    import torch
    return bool(torch.equal(a, b))


def test_draft_count_zero_is_the_plain_base_chain():
    # bonus-row context, K = 0 everywhere: every round is one base evaluation and one sampler step per environment
    # (no drafter work at all), so the chain is the base model's own reverse process with the round's noise stream
    for wl, B, dtype, paths in ((ti.small_variant(ti.C1, B=3), 3, "fp32", None),
                                (ti.small_variant(ti.C3, B=5), 5, "bf16", ("bf16-mfma-fused", "bf16-mfma-fused"))):
        S = _setup(wl, B, bonus=True)
        if paths is not None:
            assert (S["ctx"].path_name(0), S["ctx"].path_name(1)) == paths
        t0 = np.full(B, min(wl.T - 1, 9)); t0[-1] = 3           # a short chain: bf16 rounding adds up over the steps
        s = np.linspace(1.0, 1.4, B)
        x = to_dev(S["x"]); t = to_dev(t0.astype(np.int32))
        K0 = to_dev(np.zeros(B, dtype=np.int32))
        rounds, tot = S["ctx"].tsdp_chain(x, t, K0, to_dev(s.astype(np.float32)), None, check_every=1)
        assert rounds == t0.max() + 1 and (t.cpu().numpy() == -1).all()
        np.testing.assert_array_equal(tot["rounds"].cpu().numpy(), t0 + 1)
        np.testing.assert_array_equal(tot["drafts"].cpu().numpy(), 0)
        ref = S["x"].astype(np.float64); tt = t0.copy()
        while (tt >= 0).any():
            live = tt >= 0
            step = sr.base_chain_step(S["base"], S["sched"], ref[live], tt[live], s[live], np.arange(B)[live], S["seed"],
                                      S["cond"][live])
            ref[live] = step
            tt[live] -= 1
        assert_latents_close(x.cpu().numpy(), ref, dtype, "final actions of the plain chain")
        S["ctx"].close()


def test_staged_chain_follows_the_stage_tables():
    wl = ti.small_variant(ti.C1, B=6)
    S = _setup(wl, 6, head_scale=0.6)
    t0 = np.array([9, 9, 6, 3, 0, -1])
    K3 = np.array([[1, 4, 2], [2, 3, 1], [4, 4, 4], [1, 1, 3], [2, 2, 2], [1, 1, 1]])
    s3 = np.array([[1.0, 1.2, 1.0]] * 6); l3 = np.array([[0.3, 0.5, 0.9]] * 6)
    for lam in (None, l3):
        x = to_dev(S["x"]); t = to_dev(t0.astype(np.int32))
        rounds, tot = S["ctx"].tsdp_chain_staged(x, t, to_dev(K3.astype(np.int32)), to_dev(s3.astype(np.float32)),
                                                 None if lam is None else to_dev(lam.astype(np.float32)), 7, 3, None,
                                                 check_every=1)
        ref = sr.chain(S["base"], S["drafter"], S["sched"], S["x"], t0, K3, s3.astype(np.float32),
                       None, S["seed"], S["cond"], lam=None if lam is None else lam.astype(np.float32), stages=(7, 3))
        for r in ref["history"]:
            near = list_near_ties("C1 staged chain", r["logu"], r["logratio"], r["draft"]["row_ptr"], TIE, r["draft"]["row_t"] > 0)
            assert not near.any()
        assert rounds == ref["rounds"] and (t.cpu().numpy() == -1).all()
        for k in ("accept", "drafts", "rounds"):
            np.testing.assert_array_equal(tot[k].cpu().numpy(), ref["totals"][k])
        assert_latents_close(x.cpu().numpy(), ref["x"], "fp32", "final actions of the staged chain")
    import pytest as _pt
    from paper_2512_15773_amd import TsdpError
    with _pt.raises(TsdpError):
        S["ctx"].tsdp_chain_staged(x, t, to_dev(K3.astype(np.int32)), to_dev(s3.astype(np.float32)), None, 2, 3, None)
    S["ctx"].close()


def test_maximum_sizes_on_the_general_path():
    # the limits of the configuration: H*A = 512 elements per latent, K_max = 64 drafts, T = 4096 timesteps
    wl = ti.small_variant(ti.C1, B=3, H=32, A=16, T=4096, K_max=64, base=ti.NetShape(1, 96, 3), draft=ti.NetShape(1, 48, 3))
    t0 = np.array([4095, 2000, 40]); K = np.array([64, 64, 64]); s = np.array([1.0, 1.2, 1.0])
    g, ref = _stage_parity(wl, 3, t0, K, s, paths=("f32-ops", "f32-ops"))
    assert (ref["n_adv"] >= 1).all() and (ref["n_adv"] <= [64, 64, 40]).all()
    # past the limits the context is refused
    from paper_2512_15773_amd import Tsdp, TsdpError
    for kw in (dict(K_max=65), dict(T=4097), dict(A=17)):
        bad = ti.small_variant(wl, **kw)
        with pytest.raises(TsdpError):
            Tsdp.from_workload(bad, B_max=1)


def test_round_replays_from_a_captured_hip_graph():
    # a round is a fixed sequence of kernel launches on the caller's stream (no allocation after the first call, no
    # host synchronisation, no memset node): captured once, every replay must equal the eager round it stands for
    import torch
    wl = ti.small_variant(ti.C1, B=5)
    S = _setup(wl, 5, head_scale=0.6)
    ctx = S["ctx"]
    t0 = np.array([9, 9, 7, 5, 9], np.int32); K = to_dev(np.array([4, 2, 3, 4, 1], np.int32))
    s = to_dev(np.array([1.0, 1.1, 1.0, 1.2, 1.0], np.float32))

    def fresh():
        return to_dev(S["x"]), to_dev(t0), torch.zeros(5, dtype=torch.int32, device="cuda"), torch.zeros(5, dtype=torch.int32, device="cuda")

    # eager reference: four rounds in a row, with the state after each
    x, t, na, nd = fresh()
    eager = []
    for _ in range(4):
        ctx.tsdp_round(x, t, K, s, None, na, nd)
        torch.cuda.synchronize()
        eager.append((x.clone(), t.clone(), na.clone(), nd.clone()))
    # captured: the same buffers are updated in place by every replay
    x, t, na, nd = fresh()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        xw, tw, naw, ndw = fresh()
        ctx.tsdp_round(xw, tw, K, s, None, naw, ndw)              # warm-up on the capture stream
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.tsdp_round(x, t, K, s, None, na, nd)
    x.copy_(to_dev(S["x"])); t.copy_(to_dev(t0))                   # capture does not execute: start from the inputs
    for i in range(4):
        graph.replay()
        torch.cuda.synchronize()
        _ = (x * 2).sum().item()                                   # eager work and a synchronisation between replays
        for got, want in zip((x, t, na, nd), eager[i]):
            assert torch.equal(got, want), f"replay {i} differs from the eager round"
    assert ctx.tsdp_status() == 0
    ctx.close()


def test_round_does_not_depend_on_batch_composition():
    # sharding invariance: with global environment ids as Philox counters, an environment's round is bit-identical
    # whatever batch (order, neighbours, size) it is computed in
    import torch
    wl = ti.small_variant(ti.C3, B=12)
    S = _setup(wl, 12, head_scale=0.3)
    ctx = S["ctx"]
    rng = np.random.default_rng(5)
    t0 = rng.integers(0, 100, 12).astype(np.int32); K = rng.integers(1, 17, 12).astype(np.int32)
    s = rng.uniform(1, 1.5, 12).astype(np.float32); env = (np.arange(12) + 500).astype(np.int32)

    def run(idx):
        ctx.tsdp_set_cond(to_dev(S["cond"][idx]))
        x = to_dev(np.asarray(S["x"])[idx]); t = to_dev(t0[idx])
        na = torch.zeros(len(idx), dtype=torch.int32, device="cuda"); nd = torch.zeros_like(na)
        ctx.tsdp_round(x, t, to_dev(K[idx]), to_dev(s[idx]), to_dev(env[idx]), na, nd)
        return x.cpu().numpy(), t.cpu().numpy(), na.cpu().numpy()

    full = run(np.arange(12))
    perm = rng.permutation(12)
    shuffled = run(perm)
    part = run(np.array([7, 2, 9]))
    for got, idx in ((shuffled, perm), (part, np.array([7, 2, 9]))):
        for a, b in zip(got, full):
            np.testing.assert_array_equal(a, b[idx])
    ctx.close()
    # also across the drafter's tile variants: 800 environments take the four-environment tile, 5 the single one
    wl = ti.small_variant(ti.C5, B=800, base=ti.NetShape(1, 384, 6))
    wb = ti.make_weights(wl, "base", head_scale=0.3); wd = ti.make_weights(wl, "draft", head_scale=0.3)
    cond = ti.make_cond(wl, 800); x0 = np.asarray(ti.make_latents(wl, 800))
    t0, K, s = ti.make_schedule_inputs(wl, 800)
    env = np.arange(800, dtype=np.int32)
    ctx = gpu_side(wl, wb, wd, cond, B_max=800)

    def run5(idx):
        ctx.tsdp_set_cond(to_dev(cond[idx]))
        x = to_dev(x0[idx]); t = to_dev(t0[idx].astype(np.int32))
        na = torch.zeros(len(idx), dtype=torch.int32, device="cuda")
        ctx.tsdp_round(x, t, to_dev(K[idx].astype(np.int32)), to_dev(s[idx].astype(np.float32)), to_dev(env[idx]), na, None)
        return x.cpu().numpy(), t.cpu().numpy(), na.cpu().numpy()

    full = run5(np.arange(800))
    idx = np.array([3, 250, 251, 600, 799])
    for a, b in zip(run5(idx), full):
        np.testing.assert_array_equal(a, b[idx])
    ctx.close()


def test_acceptance_with_regenerated_noise_matches_stored_noise():
    # d_xi = NULL in tsdp_draft / tsdp_accept: the kernel redraws the Philox blocks of every row
    wl = ti.small_variant(ti.C1, B=8)
    t0 = np.array([9, 0, -1, 2, 5, 7, 1, 9]); K = np.array([4, 4, 4, 4, 1, 1, 3, 2])
    s = np.array([1.0, 1.0, 1.0, 1.3, 1.0, 1.5, 1.2, 1.1]); env = np.array([5, 900, 3, 77, 1, 0, 12345678, 42])
    for clip, bonus in ((None, False), (1.0, False), (None, True)):
        S = _setup(wl, 8, clip=clip, bonus=bonus)
        ctx = S["ctx"]
        rows = _gpu_draft(S, t0, K, s, env)
        ctx.tsdp_verify(8, rows)
        sd, ed = to_dev(s.astype(np.float32)), to_dev(env.astype(np.int32))
        stored = {k: v.cpu().numpy() for k, v in ctx.tsdp_accept(8, sd, ed, rows).items()}
        rows_nx = dict(rows); rows_nx["xi"] = None
        redrawn = {k: v.cpu().numpy() for k, v in ctx.tsdp_accept(8, sd, ed, rows_nx).items()}
        for k in ("flags", "n_accept", "n_adv", "t_next", "logratio", "logu", "x_out"):
            np.testing.assert_array_equal(redrawn[k], stored[k])     # the same fp32 noise, bit for bit
        # and a rollout that never stored the noise leaves the other outputs unchanged
        rows2 = ctx.alloc_rows(8); rows2["xi"] = None
        ctx.tsdp_draft(to_dev(S["x"]), to_dev(t0.astype(np.int32)), to_dev(K.astype(np.int32)), sd, ed, rows2)
        for k in ("row_ptr", "states", "eps_p", "y_last"):
            np.testing.assert_array_equal(rows2[k].cpu().numpy(), rows[k].cpu().numpy())
        ctx.close()


def test_rmsnorm_networks_on_every_path():
    # norm = 1: RMSNorm in place of LayerNorm in both networks (fused fp32, fused bf16 with either conditioning,
    # general operator kernels)
    wl = ti.small_variant(ti.C1, B=3)
    _stage_parity(wl, 3, np.array([9, 5, 0]), np.array([4, 4, 4]), np.ones(3), norm=1, paths=("f32-mfma-fused", "f32-mfma-fused"))
    wl = ti.small_variant(ti.C3, B=3)
    t0, K, s = ti.make_schedule_inputs(wl, 3, t0=60)
    _stage_parity(wl, 3, t0, K, s, norm=1, paths=("bf16-mfma-fused", "bf16-mfma-fused"))
    wl = ti.small_variant(ti.C4, B=2, base=ti.NetShape(2, 512, 8))
    t0, K, s = ti.make_schedule_inputs(wl, 2, t0=40)
    _stage_parity(wl, 2, t0, K, s, norm=1, paths=("bf16-mfma-fused", "bf16-mfma-fused"))
    wl = ti.small_variant(ti.C1, B=2, base=ti.NetShape(2, 96, 3), draft=ti.NetShape(1, 48, 3))
    _stage_parity(wl, 2, np.array([9, 4]), np.array([4, 4]), np.ones(2), norm=1, paths=("f32-ops", "f32-ops"))


def test_action_dim_above_one_head_fragment():
    # A = 20, 33: the output head spans two / three 16-row MFMA fragments in the fused kernels (verify and drafter)
    wl = ti.small_variant(ti.C3, B=3, A=20, base=ti.NetShape(2, 256, 4))
    t0, K, s = ti.make_schedule_inputs(wl, 3, t0=60)
    _stage_parity(wl, 3, t0, K, s, paths=("bf16-mfma-fused", "bf16-mfma-fused"))
    wl = ti.small_variant(ti.C2, B=2, H=16, A=20, base=ti.NetShape(2, 256, 4))
    _stage_parity(wl, 2, np.array([70, 5]), np.array([8, 8]), np.array([1.0, 1.2]), paths=("f32-mfma-fused", "f32-mfma-fused"))
    wl = ti.small_variant(ti.C1, B=2, H=16, A=32)
    _stage_parity(wl, 2, np.array([9, 3]), np.array([4, 4]), np.ones(2), paths=("f32-mfma-fused", "f32-mfma-fused"))


def _chain_both_ways(ctx, x0, t0, K, s, lam, env, stages, n_rounds, T):
    """Host-checked chain and enqueue-only chain (eager, then captured in a HIP graph and replayed three times with
    eager work between the replays) on the same inputs."""
    import torch
    dev = "cuda"
    Kd, sd = to_dev(K.astype(np.int32)), to_dev(s.astype(np.float32))
    ld = None if lam is None else to_dev(lam.astype(np.float32))
    ed = None if env is None else to_dev(env.astype(np.int32))
    x, t = to_dev(x0), to_dev(t0.astype(np.int32))
    if stages is None:
        rounds, tot = ctx.tsdp_chain(x, t, Kd, sd, ed, lam=ld, check_every=1)
    else:
        rounds, tot = ctx.tsdp_chain_staged(x, t, Kd, sd, ld, stages[0], stages[1], ed, check_every=1)
    want = dict(x=x.clone(), t=t.clone(), **{k: v.clone() for k, v in tot.items()})
    B = x.shape[0]
    x2, t2 = to_dev(x0), to_dev(t0.astype(np.int32))
    tot2 = {k: torch.full((B,), -5, dtype=torch.int32, device=dev) for k in ("accept", "drafts", "rounds")}
    run = torch.full((1,), -5, dtype=torch.int32, device=dev)
    ctx.tsdp_chain_enqueue(x2, t2, Kd, sd, ld, ed, n_rounds, stages=stages, totals=tot2, rounds_run=run)
    torch.cuda.synchronize()

    def check(tag):
        assert int(run.item()) == rounds, (tag, int(run.item()), rounds)
        assert torch.equal(x2, want["x"]) and torch.equal(t2, want["t"]), tag
        for k in tot2:
            assert torch.equal(tot2[k], want[k]), (tag, k)

    check("eager")
    # captured: kernel launches only, so the whole chain is one graph
    ctx.tsdp_prepare()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        xw, tw = to_dev(x0), to_dev(t0.astype(np.int32))
        ctx.tsdp_chain_enqueue(xw, tw, Kd, sd, ld, ed, 2, stages=stages)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.tsdp_chain_enqueue(x2, t2, Kd, sd, ld, ed, n_rounds, stages=stages, totals=tot2, rounds_run=run)
    for i in range(3):
        x2.copy_(to_dev(x0)); t2.copy_(to_dev(t0.astype(np.int32)))
        graph.replay()
        torch.cuda.synchronize()
        _ = (x2 * 2).sum().item()                                  # eager work and a synchronisation between replays
        check(f"replay {i}")
    assert rounds < n_rounds                                       # rounds past the end ran as empty launches
    return rounds


def test_enqueue_only_chain_is_bit_identical_to_the_host_checked_chain():
    # C1 (fp32) and C3 (bf16) shapes; plain, bonus row, stage tables with and without the threshold rule
    for name, B, bonus in (("C1", 6, False), ("C1", 6, True), ("C3", 12, False), ("C3", 12, True)):
        wl = ti.small_variant(ti.WORKLOADS[name], B=B)
        S = _setup(wl, B, head_scale=0.6 if name == "C1" else 0.2, bonus=bonus)
        rng = np.random.default_rng(17)
        t0 = rng.integers(-1, wl.T, B); t0[0] = wl.T - 1; t0[1] = 0
        K = rng.integers(0 if bonus else 1, wl.K_max + 1, B); s = rng.uniform(1.0, 1.3, B)
        env = rng.integers(0, 10 ** 6, B)
        n = _chain_both_ways(S["ctx"], S["x"], t0, K, s, None, env, None, wl.T + 3, wl.T)
        assert n >= 1
        K3 = rng.integers(0 if bonus else 1, wl.K_max + 1, (B, 3)); s3 = rng.uniform(1.0, 1.3, (B, 3))
        l3 = rng.uniform(0.2, 0.9, (B, 3))
        stages = (7 * wl.T // 10, 3 * wl.T // 10)
        _chain_both_ways(S["ctx"], S["x"], t0, K3, s3, None, None, stages, wl.T + 3, wl.T)
        _chain_both_ways(S["ctx"], S["x"], t0, K3, s3, l3, env, stages, wl.T + 3, wl.T)
        assert S["ctx"].tsdp_status() == 0
        S["ctx"].close()


@pytest.mark.parametrize("wl, B, bonus", [
    (ti.small_variant(ti.C2, T=30, base=ti.NetShape(2, 256, 4)), 5, False),                                 # one launch each
    (ti.small_variant(ti.C2, T=30, base=ti.NetShape(2, 256, 4)), 5, True),
    (ti.small_variant(ti.C2, T=30, K_max=4, base=ti.NetShape(2, 256, 4)), 18, False),                       # launches
    (ti.small_variant(ti.C2, T=30, K_max=4, base=ti.NetShape(2, 256, 4)), 17, True),
    (ti.small_variant(ti.C3, T=30, K_max=4, base=ti.NetShape(2, 256, 4), draft=ti.NetShape(2, 256, 4)), 3, True),   # bf16
    (ti.small_variant(ti.C3, T=30, K_max=4), 3, False),                                                     # persistent rollout
    (ti.small_variant(ti.C4, T=20, K_max=3, base=ti.NetShape(1, 512, 8)), 2, False),                        # wide rows
    (ti.small_variant(ti.C2, T=30, A=4, cond_dim=64, base=ti.NetShape(2, 96, 3), draft=ti.NetShape(1, 48, 3)), 5, True),
])
def test_enqueue_only_chain_of_few_rows(wl, B, bonus):
    # an enqueued chain looks at the live word before anything else, the host-checked one loads ahead of it; draft counts
    # from 0 or 1 to K_max end the rollouts at different transitions, and the last rounds have no live row
    rng = np.random.default_rng(B)
    S = _setup(wl, B, head_scale=0.3, bonus=bonus)
    t0 = rng.integers(-1, wl.T, B); t0[0] = wl.T - 1; t0[1] = 0
    K = rng.integers(0 if bonus else 1, wl.K_max + 1, B); K[0] = wl.K_max
    _chain_both_ways(S["ctx"], S["x"], t0, K, rng.uniform(1.0, 1.3, B), None, None, None, wl.T + 3, wl.T)
    assert S["ctx"].tsdp_status() == 0
    S["ctx"].close()


def test_layernorm_statistics_survive_a_large_mean_in_fp32():
    # a residual stream whose mean is 12x its spread (token-embedding bias 0.5 on features of spread 0.04): the
    # one-pass variance E[x^2] - mean^2 loses 2^-24 mean^2 / var = 1e-5 of the variance in fp32, at the fp32
    # tolerance; the fused fp32 kernels centre their statistics
    for wl in (ti.small_variant(ti.C1, B=3), ti.small_variant(ti.C2, B=2, base=ti.NetShape(2, 256, 4))):
        wb = ti.make_weights(wl, "base", b_std=0.02); wd = ti.make_weights(wl, "draft", b_std=0.02)
        for w in (wb, wd):
            w["tok_b"] = (w["tok_b"] + np.float32(0.5)).astype(np.float32)
        B = wl.B
        cond, x = ti.make_cond(wl, B), ti.make_latents(wl, B)
        base, drafter, sched = oracle_side(wl, wb, wd)
        ctx = gpu_side(wl, wb, wd, cond)
        assert ctx.path_name(0) == "f32-mfma-fused" and ctx.path_name(1) == "f32-mfma-fused"
        t0 = np.full(B, wl.T - 2); K = np.full(B, wl.K_max); s = np.ones(B)
        S = dict(wl=wl, B=B, cond=cond, x=x, base=base, drafter=drafter, sched=sched, ctx=ctx, clip=None, bonus=False,
                 seed=wl.philox_seed)
        rows = _gpu_draft(S, t0, K, s, None)
        o = _check_draft(S, rows, t0, K, s, None, TOL["fp32"])
        _check_verify(S, rows, o, TOL["fp32"])
        ctx.close()


def test_prepare_makes_a_fresh_context_capturable_and_short_chains_stop_where_asked():
    # tsdp_prepare on a context that has never run: the very first round is recorded into a HIP graph (an allocation
    # or a launch-attribute call during capture would fail it) and its replay equals the eager round of a second
    # context; an enqueue-only chain of 2 rounds equals the host-checked chain cut at max_rounds = 2
    import torch
    wl = ti.small_variant(ti.C3, B=9)
    wb = ti.make_weights(wl, "base", head_scale=0.2); wd = ti.make_weights(wl, "draft", head_scale=0.2)
    cond, x0 = ti.make_cond(wl, 9), ti.make_latents(wl, 9)
    t0 = np.array([99, 80, 60, 40, 20, 10, 3, 0, -1], np.int32); K = np.full(9, 16, np.int32); s = np.ones(9, np.float32)
    Kd, sd = to_dev(K), to_dev(s)
    ref_ctx = gpu_side(wl, wb, wd, cond)
    xr, tr = to_dev(x0), to_dev(t0)
    na_r = torch.zeros(9, dtype=torch.int32, device="cuda"); nd_r = torch.zeros_like(na_r)
    ref_ctx.tsdp_round(xr, tr, Kd, sd, None, na_r, nd_r)
    torch.cuda.synchronize()
    ctx = gpu_side(wl, wb, wd, cond)
    ctx.tsdp_prepare()
    x, t = to_dev(x0), to_dev(t0)
    na = torch.zeros(9, dtype=torch.int32, device="cuda"); nd = torch.zeros_like(na)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.tsdp_round(x, t, Kd, sd, None, na, nd)
    for i in range(2):
        x.copy_(to_dev(x0)); t.copy_(to_dev(t0))
        graph.replay()
        torch.cuda.synchronize()
        for got, want in ((x, xr), (t, tr), (na, na_r), (nd, nd_r)):
            assert torch.equal(got, want), f"replay {i}"
    # a chain cut short
    xa, ta = to_dev(x0), to_dev(t0)
    rounds, tot = ref_ctx.tsdp_chain(xa, ta, Kd, sd, None, max_rounds=2, check_every=1)
    assert rounds == 2 and (ta.cpu().numpy()[:5] >= 0).all()
    xb, tb = to_dev(x0), to_dev(t0)
    totb = {k: torch.zeros(9, dtype=torch.int32, device="cuda") for k in ("accept", "drafts", "rounds")}
    run = torch.zeros(1, dtype=torch.int32, device="cuda")
    ctx.tsdp_chain_enqueue(xb, tb, Kd, sd, None, None, 2, totals=totb, rounds_run=run)
    torch.cuda.synchronize()
    assert int(run.item()) == 2 and torch.equal(xa, xb) and torch.equal(ta, tb)
    for k in totb:
        assert torch.equal(totb[k], tot[k])
    ctx.tsdp_chain_enqueue(xb, tb, Kd, sd, None, None, 0, rounds_run=run)     # zero rounds: nothing but the counter
    torch.cuda.synchronize()
    assert int(run.item()) == 0 and torch.equal(xa, xb)
    ref_ctx.close(); ctx.close()


@pytest.mark.parametrize("wl", [
    ti.small_variant(ti.C2, B=3, K_max=4, base=ti.NetShape(2, 256, 4)),
    ti.small_variant(ti.C2, B=18, K_max=3, base=ti.NetShape(2, 256, 4)),
    ti.small_variant(ti.C4, B=2, K_max=3, base=ti.NetShape(1, 512, 8)),
    ti.small_variant(ti.C2, B=3, K_max=4, A=4, cond_dim=64, base=ti.NetShape(2, 96, 3), draft=ti.NetShape(1, 48, 3)),
    ti.small_variant(ti.C2, B=3, K_max=4, A=4, cond_dim=64, base=ti.NetShape(2, 192, 6), draft=ti.NetShape(1, 208, 13)),
])
def test_first_round_of_few_rows_can_be_captured(wl):
    # after tsdp_prepare the spread kernels need no allocation and no launch attribute: their first launch is recorded
    import torch
    B = wl.B
    nets = [ti.make_weights(wl, which, head_scale=0.3) for which in ("base", "draft")]
    cond, x0 = ti.make_cond(wl, B), to_dev(ti.make_latents(wl, B))
    t0 = to_dev(np.resize([50, 2, 0], B).astype(np.int32)); K = to_dev(np.resize([wl.K_max, 3, 1], B).astype(np.int32)); s = torch.ones(B, device="cuda")
    ctx = gpu_side(wl, *nets, cond)
    ctx.tsdp_prepare()
    x, t = x0.clone(), t0.clone()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.tsdp_round(x, t, K, s, None)
    eager = gpu_side(wl, *nets, cond)
    for i in range(3):
        x.copy_(x0); t.copy_(t0)
        graph.replay()
        torch.cuda.synchronize()
        xe, te = x0.clone(), t0.clone()
        eager.tsdp_round(xe, te, K, s, None)
        assert torch.equal(x, xe) and torch.equal(t, te), i
    del graph
    eager.close(); ctx.close()


@pytest.mark.parametrize("wl, B, K_max", [
    (ti.small_variant(ti.C1, draft=ti.NetShape(1, 32, 2)), 1, 1),                                     # one row
    (ti.small_variant(ti.C2, base=ti.NetShape(1, 256, 4), draft=ti.NetShape(1, 128, 4)), 5, 7),      # both networks' vectors, rows not a multiple of 16
    (ti.small_variant(ti.C3, base=ti.NetShape(1, 256, 4), draft=ti.NetShape(1, 128, 4)), 9, 9),      # bf16, the base network's alone
    (ti.small_variant(ti.C1, base=ti.NetShape(1, 64, 2), draft=ti.NetShape(1, 32, 2)), 256, 2),      # one environment a thread
    (ti.small_variant(ti.C1, base=ti.NetShape(1, 64, 2), draft=ti.NetShape(1, 32, 2)), 257, 2),      # one more: in launches of their own
    (ti.small_variant(ti.C2, A=4, base=ti.NetShape(1, 96, 3), draft=ti.NetShape(1, 48, 3)), 20, 5),  # run-time sizes
    (ti.small_variant(ti.C1, A=4, base=ti.NetShape(1, 64, 2), draft=ti.NetShape(1, 36, 3)), 3, 3),   # a drafter in operator kernels
])
@pytest.mark.parametrize("bonus", [False, True])
def test_a_round_finds_the_vectors_of_its_stages(wl, B, K_max, bonus):
    # a whole round makes the FiLM vectors with its row table, the three stages make them from the table: the same bits
    import torch
    S = _setup(wl, B, K_max=K_max, bonus=bonus)
    ctx, rng = S["ctx"], np.random.default_rng(B)
    t0 = rng.integers(-1, wl.T, B).astype(np.int32); t0[0] = wl.T - 1
    K = rng.integers(0 if bonus else 1, K_max + 1, B).astype(np.int32); s = rng.uniform(1, 1.5, B).astype(np.float32)
    x, t = to_dev(S["x"]), to_dev(t0)
    n_acc = torch.zeros(B, dtype=torch.int32, device="cuda"); n_adv = torch.zeros_like(n_acc)
    rows = ctx.alloc_rows(B)
    ctx.tsdp_draft(x, t, to_dev(K), to_dev(s), None, rows)
    ctx.tsdp_verify(B, rows)
    out = dict(x_out=torch.empty_like(x), **{k: torch.empty(B, dtype=torch.int32, device="cuda") for k in ("t_next", "n_accept", "n_adv")})
    ctx.tsdp_accept_into(B, to_dev(s), None, rows, out)
    ctx.tsdp_round(x, t, to_dev(K), to_dev(s), None, n_acc, n_adv)
    assert torch.equal(x, out["x_out"]) and torch.equal(t, out["t_next"]) and torch.equal(n_acc, out["n_accept"])
    ctx.close()
