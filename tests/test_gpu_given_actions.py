"""Steps under given actions one at a time (sim_step) and T at a time with held actions
run one kernel and are equal bit for bit, resets and the action history among them."""
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


# one env, both sides of a workgroup, two rounds of the chip
@pytest.mark.parametrize("n", [1, 255, 257, 140001])
@pytest.mark.parametrize("flags", [0, wl.F_DISTURB | wl.F_OBS_NOISE, wl.F_ACTOR_BF16])
def test_single_steps_equal_rollouts(pkg, n, flags):
    T = 36  # a launch that draws start states ahead; more steps than history slots
    cfg = wl.crazyflie_config(n_envs=n, dr_enable=1, max_episode_steps=11, dist_force=0.01,
                              dist_torque=3e-5, obs_noise=(0.001, 0.01, 0.02, 0.05),
                              flags=wl.F_RENORM_Q | wl.F_TERMINATE | wl.F_AUTORESET | flags)
    held = torch.as_tensor(wl.random_actions(n, seed=4)).cuda()
    got = {}
    for way in ("steps", "held"):
        sim = pkg.QuadSim(cfg)
        if way == "steps":
            o = [sim.step(actions=held) for _ in range(T)]
            r, d = torch.stack([x[0] for x in o]), torch.stack([x[1] for x in o])
        else:
            o = sim.rollout_actions(held, T)
            r, d = o["rewards"], o["dones"]
        got[way] = dict({k: np_(v) for k, v in sim.get_state().items()}, rewards=np_(r), dones=np_(d))
        sim.close()
    assert (got["steps"]["dones"] != 0).any()
    for k, v in got["steps"].items():
        assert np.array_equal(v, got["held"][k]), k
