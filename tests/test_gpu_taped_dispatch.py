"""Taped rollouts and gradients on every path of the dispatch by size: with the training
extras on each kernel, and with more segments than segment buffers where recomputes
run beside the sweep and where they do not.

References: a handle with one segment for the whole horizon (everything recorded by
the forward, nothing recomputed) and, for per-env parameter gradients, the same env ids
on another kernel: the forward kernels agree bit for bit, and so do the sweeps up to
32768 envs.
"""
import numpy as np
import pytest

import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pkg():
    import paper_2311_13081_amd as p
    p.load()
    return p


def np_(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def config(n, T, K, extras):
    cfg = wl.crazyflie_config(n_envs=n, dr_enable=1, flags=wl.F_RENORM_Q, max_episode_steps=0,
                              max_tape_horizon=T, ckpt_every=K)
    return wl.training_extras(cfg) if extras else cfg


def taped(pkg, n, T, K, extras, times=1):
    sim = pkg.QuadSim(config(n, T, K, extras))
    a = sim.actor_tensor(wl.xavier_actor(2))
    o = sim.rollout(a, T, states=True, record_tape=True)
    fwd = [np_(o["states"]), np_(o["rewards"])]
    grads = [[np_(x).copy() for x in sim.backward(a)] for _ in range(times)]
    sim.close()
    return fwd, grads


# the kernels of taped rollouts: split actor, one tile, two tiles; ragged batches
@pytest.mark.parametrize("n", [1000, 5000, 33000])
def test_taped_extras_agree_across_kernels(pkg, n):
    T, K = 12, 2
    fwd, (g1, g2) = taped(pkg, n, T, K, True, times=2)
    assert all(np.array_equal(x, y) for x, y in zip(g1, g2))
    # untaped forward of the other kernels
    sim = pkg.QuadSim(config(n, T, K, True))
    for v in (3, 4):
        sim.reset()
        sim.set_variant(v)
        o = sim.rollout(sim.actor_tensor(wl.xavier_actor(2)), T, states=True)
        assert np.array_equal(np_(o["states"]), fwd[0]) and np.array_equal(np_(o["rewards"]), fwd[1])
    sim.close()
    # the first envs of the batch are those of a small handle (draws keyed by env id)
    m = 1000
    small_fwd, (small,) = taped(pkg, m, T, K, True)
    assert np.array_equal(small_fwd[0], fwd[0][..., :m])
    assert np.array_equal(small[1], g1[1][:, :m])


# 5000 envs: recomputes on a stream of their own, beside the sweep (four buffers);
# 16500 and 33000: in order (up to eight); more segments than buffers in each
@pytest.mark.parametrize("n,K", [(5000, 2), (16500, 1), (33000, 1)])
@pytest.mark.parametrize("extras", [False, True])
def test_more_segments_than_buffers_on_each_path(pkg, n, K, extras):
    T = 11  # a short last segment where K = 2
    _, (g1, g2) = taped(pkg, n, T, K, extras, times=2)
    assert all(np.array_equal(x, y) for x, y in zip(g1, g2))
    _, (whole,) = taped(pkg, n, T, T, extras)
    assert np.array_equal(g1[1], whole[1])
    ga, gb = g1[0].astype(np.float64), whole[0].astype(np.float64)
    # the same terms in another order of fp32 sums: 2^9 roundings in sequence at most
    assert np.linalg.norm(ga - gb) <= 2.0 ** -23 * 2 ** 9 * np.linalg.norm(gb)
