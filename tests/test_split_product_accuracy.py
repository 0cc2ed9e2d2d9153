"""Accuracy of the fp32 products formed from bf16 parts (six of nine terms), in the
actions of one step against the network in FP64.

Bars: rms 2e-7 and 2e-6 at most.  An emulation on the CPU (exact products of the
parts, fp32 sums) gives 4e-8 and 3e-7 with all six terms, and without any one of them at
least 1.5e-6 and 8e-6: so a term lost in the kernels, which share their products and
would still agree with each other, shows.  An fp32 chain gives 3.4e-7 rms.

The weight gradients of one env and one step are single products, a unit's cotangent
(the bias gradient) times an input: their relative error is at most 2^-21 (omitted
terms 2^-26, a handful of roundings), and a lost term leaves up to 2^-18.
"""
import numpy as np
import pytest

import workloads as wl

torch = pytest.importorskip("torch")

N, SEED = 2048, 9
RMS_BAR, MAX_BAR = 2e-7, 2e-6
TERMS = [(2, 0), (0, 2), (1, 1), (1, 0), (0, 1), (0, 0)]  # (part of the weight, of the input)
VARIANTS = {"plain": 1, "tile32": 3, "tile16": 4, "split": 5}


def layers(W, dtype):
    w = W.astype(dtype)
    return [(w[:9344].reshape(64, 146), w[9344:9408]), (w[9408:13504].reshape(64, 64), w[13504:13568]),
            (w[13568:13824].reshape(4, 64), w[13824:])]


def fp64_actions(W, o):
    x = o.astype(np.float64)
    for i, (A, b) in enumerate(layers(W, np.float64)):
        x = x @ A.T + b
        x = np.maximum(x, 0) if i < 2 else np.tanh(x)
    return x


def exceeds(err):
    return np.sqrt((err ** 2).mean()) > RMS_BAR, np.abs(err).max() > MAX_BAR


def bf16(x):
    u = np.ascontiguousarray(x, np.float32).view(np.uint32).astype(np.uint64)
    return ((u + 0x7fff + ((u >> 16) & 1)) & 0xffff0000).astype(np.uint32).view(np.float32)


def split(x):
    p0 = bf16(x)
    p1 = bf16(x - p0)
    return p0, p1, bf16(x - p0 - p1)


def emulated_actions(W, o, terms):
    x = o.astype(np.float32)
    for i, (A, b) in enumerate(layers(W, np.float32)):
        if i == 2:  # the last layer's products are fp32
            return np.tanh(x.astype(np.float64) @ A.T.astype(np.float64) + b)
        w, p = split(A), split(x)
        acc = np.zeros((len(x), len(A)), np.float32)
        for lead in (False, True):  # small terms of every chunk first
            for c in range(0, A.shape[1], 32):
                for t in terms:
                    if (t == (0, 0)) == lead:
                        f = p[t[1]][:, c:c + 32].astype(np.float64) @ w[t[0]][:, c:c + 32].T.astype(np.float64)
                        acc = (acc + f).astype(np.float32)
        x = np.maximum(acc + b, 0)


def start_states():
    S, H = wl.random_states(N, seed=5)
    return S.astype(np.float32), H.astype(np.float32)


def test_every_term_counts():
    S, H = start_states()
    w, x, y, z = S[3:7]
    R = np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                  2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                  2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)])
    o = np.concatenate([S[:3], R, S[7:13], H.reshape(128, N)]).T
    W = wl.random_actor(SEED)
    want = fp64_actions(W, o)
    assert not any(exceeds(emulated_actions(W, o, TERMS) - want))
    for t in TERMS:
        assert all(exceeds(emulated_actions(W, o, [u for u in TERMS if u != t]) - want)), t


@pytest.mark.gpu
@pytest.mark.parametrize("variant", sorted(VARIANTS))
@pytest.mark.parametrize("scale", [2.0 ** -20, 1.0, 2.0 ** 12])
def test_kernel_actions(variant, scale):
    """The first layer scaled by a power of two and the second by its inverse: the same
    actions from operands of other magnitudes."""
    import paper_2311_13081_amd as pkg
    cfg = wl.crazyflie_config(n_envs=N, dr_enable=1, flags=wl.F_RENORM_Q, max_episode_steps=0)
    W = wl.random_actor(SEED).astype(np.float64)
    W[:9408] *= scale
    W[9408:13504] /= scale
    W = W.astype(np.float32)
    sim = pkg.QuadSim(cfg)
    sim.set_variant(VARIANTS[variant])
    S, H = start_states()
    sim.set_state(state=S, hist=H)
    o = sim.observe(critic=False)["actor"].cpu().numpy().T
    sim.rollout(sim.actor_tensor(W), 1)
    err = sim.get_state()["hist"].cpu().numpy()[31].T - fp64_actions(W, o)
    sim.close()
    print(f"{variant} x {scale}: rms {np.sqrt((err ** 2).mean()):.2e}, max {np.abs(err).max():.2e}")
    assert not any(exceeds(err))


PRODUCT_BAR = 2.0 ** -21


def test_every_term_counts_in_one_product():
    rng = np.random.default_rng(1)
    a, b = (rng.uniform(-1, 1, 5000).astype(np.float32) for _ in range(2))
    p, q = split(a), split(b)
    want = a.astype(np.float64) * b
    def worst(terms):
        acc = np.zeros(a.shape, np.float32)
        for i, j in terms:
            acc = (acc + p[i].astype(np.float64) * q[j]).astype(np.float32)
        return np.abs((acc - want) / want).max()
    assert worst(TERMS) <= PRODUCT_BAR / 2
    for t in TERMS:
        assert worst([u for u in TERMS if u != t]) > 4 * PRODUCT_BAR, t


@pytest.mark.gpu
@pytest.mark.parametrize("seed", range(4))
def test_weight_gradients_of_one_step(seed):
    import paper_2311_13081_amd as pkg
    sim = pkg.QuadSim(wl.crazyflie_config(n_envs=1, flags=wl.F_RENORM_Q, max_episode_steps=0,
                                          max_tape_horizon=1, ckpt_every=1))
    S, H = wl.random_states(8, seed=30 + seed)
    sim.set_state(state=S[:, :1].copy(), hist=H[:, :, :1].copy())
    o = sim.observe(critic=False)["actor"].cpu().numpy()[:, 0].astype(np.float64)
    W = wl.random_actor(SEED + seed)
    a = sim.actor_tensor(W)
    sim.rollout(a, 1, record_tape=True)
    g, _ = sim.backward(a)
    g = g.cpu().numpy().astype(np.float64)
    sim.close()
    (G1, d1), (G2, d2), (G3, d3) = layers(g, np.float64)

    def rel(got, want):
        keep = want != 0
        assert np.array_equal(got != 0, keep) and keep.any()
        return np.abs((got[keep] - want[keep]) / want[keep]).max()

    cols = np.r_[0:3, 12:146]  # inputs that are copied (rotation entries are formed twice)
    assert rel(G1[:, cols], d1[:, None] * o[cols]) <= PRODUCT_BAR
    for G, d in ((G2, d2), (G3, d3)):  # the layer's inputs from its largest row
        i = np.argmax(np.abs(d))
        x = G[i] / d[i]
        assert rel(G, d[:, None] * x[None]) <= 2 * PRODUCT_BAR
