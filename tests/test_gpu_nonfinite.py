"""Infinite, NaN and very large values in single envs and in the actor: what the
fp32 kernels make of them, and that the envs beside them keep their bits.

A NaN among an env's inputs, or a weight that is not finite, makes the actions NaN.
Infinite inputs (and magnitudes that round past bf16's largest) leave finite actions.
Finite inputs up to there: the actor in numpy float32 on the observed features.
"""
import numpy as np
import pytest

import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

VARIANTS = {"auto": 0, "plain": 1, "tile32": 3, "tile16": 4, "split": 5}
FP32_KERNELS = ["auto", "plain", "tile32", "tile16", "split"]
INF, NAN, HUGE = np.inf, np.nan, 3.2e38  # HUGE: below bf16's largest; 3.4e38 above it


@pytest.fixture(scope="module")
def pkg():
    import paper_2311_13081_amd as p
    p.load()
    return p


def np_(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def spoil(state, hist):
    """Sets single values; returns the envs with a NaN, with an infinite (or nearly) value
    and with a large finite one."""
    state[0, 3], state[7, 4], state[10, 5] = INF, -INF, INF
    state[0, 7], state[7, 8], state[10, 9] = 3.4e38, HUGE, -1e30
    hist[5, 2, 12], hist[0, 0, 14], hist[31, 3, 15] = INF, 1e30, -INF
    state[0, 40], state[12, 70], hist[30, 1, 33] = -INF, INF, HUGE
    state[0, 6], state[12, 20], hist[31, 1, 13], hist[0, 2, 65] = NAN, NAN, NAN, NAN
    return [6, 20, 13, 65], [3, 4, 5, 7, 12, 15, 40, 70], [8, 9, 14, 33]


def actor_f32(W, o):
    """Actions of the observations o [n][146], in float32."""
    w = W.astype(np.float32)
    layers = [(w[:9344].reshape(64, 146), w[9344:9408]), (w[9408:13504].reshape(64, 64), w[13504:13568]),
              (w[13568:13824].reshape(4, 64), w[13824:])]
    x = o.astype(np.float32)
    with np.errstate(all="ignore"):
        for i, (A, b) in enumerate(layers):
            x = (x[:, None, :] * A[None]).sum(-1, dtype=np.float32) + b
            if i < 2:
                x = np.where(x > 0, x, np.float32(0))
        return np.tanh(x)


def config(flags, extras=False, n=80, **kw):
    cfg = wl.crazyflie_config(n_envs=n, dr_enable=1, flags=flags, max_episode_steps=0, **kw)
    return wl.training_extras(cfg) if extras else cfg


def run(pkg, cfg, W, variant, T, bad):
    sim = pkg.QuadSim(cfg)
    sim.set_variant(VARIANTS[variant])
    a = sim.actor_tensor(W)
    sim.rollout(a, 3)
    g = {k: np_(v).copy() for k, v in sim.get_state().items()}
    if bad:
        spoil(g["state"], g["hist"])
        sim.set_state(state=g["state"], hist=g["hist"])
    o = np_(sim.observe(critic=False)["actor"]).T
    out = sim.rollout(a, T, states=True)
    out = {k: np_(v) for k, v in out.items()}
    out.update({k: np_(v) for k, v in sim.get_state().items()})
    sim.close()
    return o, out


@pytest.mark.parametrize("extras", [False, True])
@pytest.mark.parametrize("policy", ["random", "xavier"])
def test_spoiled_envs(pkg, extras, policy):
    W = wl.random_actor(5) if policy == "random" else wl.xavier_actor(0)
    cfg = config(wl.F_RENORM_Q | wl.F_TERMINATE, extras)
    nans, infs, large = spoil(np.zeros((17, 80)), np.zeros((32, 4, 80)))
    others = np.setdiff1d(np.arange(80), nans + infs + large)
    for T in (1, 4):
        first = None
        for v in FP32_KERNELS:
            o, out = run(pkg, cfg, W, v, T, True)
            _, clean = run(pkg, cfg, W, v, T, False)
            for k in out:  # neighbours of the same tiles
                assert np.array_equal(out[k][..., others], clean[k][..., others]), (v, k)
            if first is None:
                first = out
            for k in out:
                assert np.array_equal(out[k], first[k], equal_nan=True), (v, k)
            act = out["hist"][32 - T]  # the first step's
            assert np.isnan(act[:, nans]).all(), v
            assert (out["dones"][0, nans] == 1).all() and np.isnan(out["rewards"][0, nans]).all()
            assert np.isfinite(act[:, infs]).all() and (out["dones"][0, [3, 4, 5, 7, 40, 70]] == 1).all()
            # sums of roundings relative to the large feature; its actions saturate
            want = actor_f32(W, o[large]).T
            assert np.allclose(act[:, large], want, rtol=0, atol=1e-5), v


# layer 1, its bias, layers 2 and 3 and their biases; first and last
@pytest.mark.parametrize("where", [5, 9343, 9344 + 7, 9408 + 70, 13503, 13504 + 3, 13568, 13824])
def test_nan_weight_makes_actions_nan(pkg, where):
    W = wl.random_actor(5).copy()
    W[where] = NAN
    for v in FP32_KERNELS:
        _, out = run(pkg, config(wl.F_RENORM_Q | wl.F_TERMINATE), W, v, 2, False)
        rows = slice(None) if where < 13568 else [(where - 13568) // 64 if where < 13824 else 0]
        assert np.isnan(out["hist"][30][rows]).all() and np.isnan(out["hist"][31]).all(), v


@pytest.mark.parametrize("where", [5, 9344 + 7, 9408 + 70])
@pytest.mark.parametrize("value", [INF, -INF])
def test_infinite_weight_makes_actions_nan(pkg, where, value):
    W = wl.random_actor(5).copy()
    W[where] = value
    for v in FP32_KERNELS:
        _, out = run(pkg, config(wl.F_RENORM_Q), W, v, 1, False)
        assert np.isnan(out["hist"][31]).all(), v


# split-actor kernel, tile kernel of one and of two tiles; segments that the forward
# records and segments recomputed from a checkpoint
@pytest.mark.parametrize("n", [80, 5000, 33000])
@pytest.mark.parametrize("extras", [False, True])
def test_taped_rollout_beside_spoiled_envs(pkg, n, extras):
    W, T = wl.random_actor(5), 10
    cfg = config(wl.F_RENORM_Q, extras, n=n, max_tape_horizon=T, ckpt_every=1 if n == 80 else 2)
    nans, infs, large = spoil(np.zeros((17, 80)), np.zeros((32, 4, 80)))
    others = np.setdiff1d(np.arange(n), nans + infs + large)
    got = []
    for bad in (False, True):
        sim = pkg.QuadSim(cfg)
        a = sim.actor_tensor(W)
        g = {k: np_(v).copy() for k, v in sim.get_state().items()}
        if bad:
            spoil(g["state"], g["hist"])
            sim.set_state(state=g["state"], hist=g["hist"])
        out = sim.rollout(a, T, states=True, record_tape=True)
        ga, gp = (np_(x).copy() for x in sim.backward(a))
        gb, gq = (np_(x) for x in sim.backward(a))
        assert np.array_equal(ga, gb, equal_nan=True) and np.array_equal(gp, gq, equal_nan=True)
        got.append((np_(out["states"]), np_(out["rewards"]), gp, ga))
        sim.close()
    for x, y in zip(got[0][:3], got[1][:3]):
        assert np.array_equal(x[..., others], y[..., others])
    # an infinite history value reads the same in a recompute as in the forward
    assert np.isfinite(got[1][0][:, :, [12, 15]]).all() and np.isfinite(got[1][2][:, [12, 15]]).all()
    assert np.isnan(got[1][2][:, nans]).any(axis=0).all()  # not taken for finite
    assert np.isnan(got[1][3]).any() and np.isfinite(got[0][3]).all()
