"""Gradients of long horizons against their FP64 evaluation: 128 steps of a flying batch,
the cotangents a state loss that grows along the horizon, of one sign per env."""
import pytest

torch = pytest.importorskip("torch")


def gradients(n, steps, seed):
    import perf.cases as pc
    case = dict(kind="sysid", n=n, steps=steps, every=16)
    exact = pc.exact(case, seed)
    st = pc.prepare(case, seed)
    out = pc.run(st)
    torch.cuda.synchronize()
    st["sim"].close()
    return {k: (out[k].double(), torch.as_tensor(exact[k], device=out[k].device,
                                                 dtype=torch.float64).reshape(out[k].shape))
            for k in ("actor", "params")}


# the reverse sweeps: four waves per 16 envs, quarter-lane, one env per lane
SIZES = pytest.mark.parametrize("n,steps", [(4096, 128), (16384, 128), (65536, 96)])


@pytest.mark.gpu
@SIZES
def test_parameter_gradients(n, steps):
    """Relative error of all of them below 4.5e-6.  With the terms of each stage
    added to the adjoints one by one the three sizes give 5.4e-6 to 6.1e-6, with the
    stages' shares summed first 3.0e-6 to 3.3e-6 (the spread between seeds is 1%)."""
    got, want = gradients(n, steps, 1)["params"]
    assert ((got - want).norm() / want.norm()).item() < 4.5e-6


@pytest.mark.gpu
@SIZES
def test_no_drift(n, steps):
    """The median over the envs of the mass gradient's relative error, whose spread is
    1e-6 to 5e-6, is the sweep's drift: 1.1e-7 at most with products rounded to nearest,
    4.8e-7 to 6.1e-7 where every product is rounded the same way."""
    got, want = gradients(n, steps, 2)["params"]
    assert abs(((got - want)[0] / want[0]).median().item()) < 2e-7


@pytest.mark.gpu
def test_actor_gradient():
    """Relative error over four seeds.  Products and sums in single precision throughout
    give 9.8e-8 (16 seeds, spread 4e-9), so 1.0e-7 at most."""
    errs = []
    for seed in range(1, 5):
        got, want = gradients(16384, 32, seed)["actor"]
        errs.append(((got - want).norm() / want.norm()).item())
    print(errs)
    assert sum(errs) / len(errs) < 1.0e-7
