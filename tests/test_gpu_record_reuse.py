"""Record buffers of a handle reused by taped rollouts of other lengths: the
gradients of a tape do not depend on what an earlier, longer or shorter tape left
in the buffers.  The reference is a new handle, whose buffers are clear: equal
bit for bit."""
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


def all_on_actor():
    """Every hidden unit active, so each recorded ReLU mask word is all ones (a NaN
    when it is read as a float)."""
    W = wl.random_actor(5).copy()
    W[9344:9408] = 50.0     # b1
    W[13504:13568] = 1000.0  # b2
    W[13568:13824] *= 1e-3   # W3
    return W


# batches that end inside a 64-env block, on the split-actor kernel, the tile
# kernel of one and of two tiles, and with the bf16 actor
@pytest.mark.parametrize("n,flags", [(130, 0), (1000, 0), (5000, 0), (33001, 0),
                                     (130, wl.F_ACTOR_BF16), (1000, wl.F_ACTOR_BF16)])
def test_gradients_after_tapes_of_other_lengths(pkg, n, flags):
    cfg = wl.crazyflie_config(n_envs=n, dr_enable=1, flags=wl.F_RENORM_Q | flags,
                              max_episode_steps=0, max_tape_horizon=16, ckpt_every=8)
    W = all_on_actor()

    def grads(sim, T):
        sim.reset()
        a = sim.actor_tensor(W)
        sim.rollout(a, T, record_tape=True)
        g = sim.backward(a)
        torch.cuda.synchronize()
        return [x.cpu().numpy() for x in g]

    used = pkg.QuadSim(cfg)
    for T in (8, 1, 3, 16, 11, 2):  # whole and short last segments, one and two of them
        got = grads(used, T)
        new = pkg.QuadSim(cfg)
        want = grads(new, T)
        new.close()
        for g, w in zip(got, want):
            assert np.all(np.isfinite(w)) and np.array_equal(g, w), T
    used.close()
