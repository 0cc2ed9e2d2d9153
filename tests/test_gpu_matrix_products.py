"""The kernels whose fp32 products run on bf16 matrix cores from operands split
into three parts, at the sizes where tiles, waves and workgroups end.

Reference for a layer: the network in FP64 (numpy).  A split product drops terms
below 2^-24 of |w x| (three parts of 8 bits on both sides), so one output of
K products in fp32 accumulation is off by at most (K + 8) 2^-23 sum |w x|, counted
generously; the bound is carried through the layers element by element.
Reference for gradients: the FP64 oracle, block by block of the actor (a tile
that lands in the wrong place is wrong by all of its block).  Kernels that
promise the same arithmetic are compared bit for bit.
"""
import numpy as np
import pytest

import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

VARIANTS = {"auto": 0, "plain": 1, "tile32": 3, "tile16": 4, "split": 5}
NO, NH = 146, 64
BLOCKS = {"W1": (0, 9344), "b1": (9344, 9408), "W2": (9408, 13504), "b2": (13504, 13568),
          "W3": (13568, 13824), "b3": (13824, 13828)}


@pytest.fixture(scope="module")
def pkg():
    import paper_2311_13081_amd as p
    p.load()
    return p


def np_(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def run(pkg, cfg, variant, W, T):
    sim = pkg.QuadSim(cfg)
    sim.set_variant(VARIANTS[variant])
    o = sim.rollout(sim.actor_tensor(W), T, rewards=True, dones=True, states=True)
    out = {k: np_(v) for k, v in o.items() if v is not None}
    out.update({k: np_(v) for k, v in sim.get_state().items()})
    sim.close()
    return out


# one env to one past a whole wave of each tile kernel, and both sides of the
# batch sizes at which the default kernel changes (4096, 32768)
@pytest.mark.parametrize("n", [1, 15, 17, 31, 33, 63, 65, 129, 4096, 4097, 32768, 32769])
@pytest.mark.parametrize("extras", [False, True])
def test_rollout_kernels_agree_at_tile_edges(pkg, n, extras):
    """Tile kernels of one and two tiles, split-actor kernel and the default one,
    resets and both episode-end kinds on the way: equal bit for bit."""
    flags = wl.F_RENORM_Q | wl.F_TERMINATE | wl.F_AUTORESET
    if extras:
        flags |= wl.F_DISTURB | wl.F_OBS_NOISE
    cfg = wl.crazyflie_config(n_envs=n, dr_enable=1, flags=flags, max_episode_steps=5)
    W, T = wl.xavier_actor(1), 11
    names = ["auto", "tile32", "tile16"] + (["split"] if n <= 4097 else [])
    out = {v: run(pkg, cfg, v, W, T) for v in names}
    assert out["auto"]["dones"].any()
    for v in names[1:]:
        for k, x in out["auto"].items():
            assert np.array_equal(x, out[v][k], equal_nan=True), (v, k)


def layers_fp64(W, o):
    """z3 of the observations o [N][146] and a bound of the kernels' error on it."""
    w = W.astype(np.float64)
    u = 2.0 ** -23
    W1, b1 = w[:9344].reshape(NH, NO), w[9344:9408]
    W2, b2 = w[9408:13504].reshape(NH, NH), w[13504:13568]
    W3, b3 = w[13568:13824].reshape(4, NH), w[13824:]
    z1 = o @ W1.T + b1
    # the observation in fp32: rotation matrix entries to a few roundings
    eo = 8 * u * np.maximum(np.abs(o), 1.0)
    e1 = eo @ np.abs(W1).T + (NO + 9) * u * (np.abs(o) @ np.abs(W1).T + np.abs(b1))
    h1 = np.maximum(z1, 0)
    z2 = h1 @ W2.T + b2
    e2 = e1 @ np.abs(W2).T + (NH + 9) * u * ((h1 + e1) @ np.abs(W2).T + np.abs(b2))
    h2 = np.maximum(z2, 0)
    z3 = h2 @ W3.T + b3
    e3 = e2 @ np.abs(W3).T + (NH + 9) * u * ((h2 + e2) @ np.abs(W3).T + np.abs(b3))
    return z3, e3


@pytest.mark.parametrize("variant", ["plain", "tile32", "tile16", "split"])
@pytest.mark.parametrize("scale", [2.0 ** -20, 1.0, 2.0 ** 12])
def test_actor_products_against_fp64(pkg, variant, scale):
    """One step's actions (the newest history slot) against the FP64 network, the
    first layer scaled up and the second down by the same power of two and the
    reverse, so that operands of all magnitudes are split."""
    n = 70
    cfg = wl.crazyflie_config(n_envs=n, dr_enable=1, flags=wl.F_RENORM_Q)
    W = wl.random_actor(9).astype(np.float64)
    W[:9408] *= scale
    W[9408:13504] /= scale
    W = W.astype(np.float32)
    sim = pkg.QuadSim(cfg)
    sim.set_variant(VARIANTS[variant])
    a = sim.actor_tensor(W)
    sim.rollout(a, 40)  # a history of actions
    o = np_(sim.observe(critic=False)["actor"]).astype(np.float64).T
    sim.rollout(a, 1)
    hist = np_(sim.get_state()["hist"]).astype(np.float64).reshape(-1, n)[-4:].T
    z3, e3 = layers_fp64(W, o)
    # tanh is 1-Lipschitz; its own evaluation and the action to fp32
    bar = e3 + 8 * 2.0 ** -23
    assert np.all(np.abs(hist - np.tanh(z3)) <= bar), float((np.abs(hist - np.tanh(z3)) / bar).max())
    sim.close()


def oracle_batch(orc, cfg, sim):
    st = sim.get_state()
    n = cfg["n_envs"]
    ref = orc.Batch(cfg, n)
    ref.set_soa(np_(st["state"]), np_(st["hist"]),
                theta_soa=np_(sim.get_params()))
    return ref


# one env, waves and 64-env blocks that end early, both sides of the sizes where
# the reverse sweep changes (4096; 65536 is covered below), segments of odd length
# and a short last one
@pytest.mark.parametrize("n,T,K", [(1, 3, 2), (17, 5, 5), (63, 4, 1), (65, 7, 3), (130, 5, 4),
                                   (4097, 3, 2)])
def test_gradient_blocks_match_oracle(pkg, oracle_lib, n, T, K):
    """Each block of the actor gradient against the FP64 oracle within 1e-3 of the
    block's norm (the bar of the backward tests; a misplaced tile or a dropped
    environment is off by far more)."""
    cfg = wl.crazyflie_config(n_envs=n, dr_enable=1, flags=wl.F_RENORM_Q, max_episode_steps=0,
                              max_tape_horizon=T, ckpt_every=K)
    sim = pkg.QuadSim(cfg)
    ref = oracle_batch(oracle_lib, cfg, sim)
    W = wl.random_actor(5)
    a = sim.actor_tensor(W)
    sim.rollout(a, T, record_tape=True)
    ga, _ = sim.backward(a)
    ga = np_(ga).astype(np.float64)
    _, gW, _ = ref.grad(W, T, nthreads=8)
    for name, (lo, hi) in BLOCKS.items():
        d = np.linalg.norm(ga[lo:hi] - gW[lo:hi]) / np.linalg.norm(gW[lo:hi])
        assert d <= 1e-3, (name, d)
    sim.close()


@pytest.mark.parametrize("n", [16384, 65600])
def test_more_segments_than_buffers(pkg, n):
    """Ten segments on eight segment buffers (the first two are recomputed, into
    buffers of the last two): a second backward on the same tape gives the same
    gradients bit for bit, and the per-env parameter gradients equal those of a
    handle with one segment."""
    T = 10
    W = wl.xavier_actor(2)
    out = []
    for K in (1, T):
        cfg = wl.crazyflie_config(n_envs=n, dr_enable=1, flags=wl.F_RENORM_Q,
                                  max_episode_steps=0, max_tape_horizon=T, ckpt_every=K)
        sim = pkg.QuadSim(cfg)
        a = sim.actor_tensor(W)
        sim.rollout(a, T, record_tape=True)
        g1 = [np_(x).copy() for x in sim.backward(a)]
        g2 = [np_(x).copy() for x in sim.backward(a)]
        assert all(np.array_equal(x, y) for x, y in zip(g1, g2))
        out.append(g1)
        sim.close()
    assert np.array_equal(out[0][1], out[1][1])
    ga, gb = out[0][0].astype(np.float64), out[1][0].astype(np.float64)
    # the same terms summed in another order: fp32 sums over n envs and T steps in
    # blocks of 32, some 2^9 roundings in sequence at most
    assert np.linalg.norm(ga - gb) <= 2.0 ** -23 * 2 ** 9 * np.linalg.norm(gb)
