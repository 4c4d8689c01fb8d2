"""States outside what a plasma reaches: particles so fast that a coordinate in cells exceeds
what a double resolves.  A run may not be meaningful then, but its sums stay those of its
particles."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

ES = ("esec2", "esec1", "standard")
EM = ("emec_li", "emec_psatd", "emec_lf")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_09605_amd  # noqa: F401


def _say(msg):
    print(msg, flush=True)


def _workload(scheme, n, ng, order):
    if scheme in EM:
        wl = workloads.weibel(n_particles=n, n_cells=ng, order=order, steps=4)
        wl.dt = min(wl.dt, 0.9 * wl.length / ng)
        return wl
    return workloads.two_stream(n_particles=n, n_cells=ng, order=order, steps=4)


@pytest.mark.parametrize("which", [0, 500, 1000])
@pytest.mark.parametrize("scheme", ES + EM)
def test_a_runaway_particle_deposits_its_own_weight(scheme, which):
    """One particle at 1e25 lengths per unit time (x / h near 1e24, past 2^51): its stencil
    weights still lie in [0, 1], so no current exceeds w |v| / h and the field moves by at most
    dt w |v| / h a step (half as much again for the acceleration by that field); the standard
    scheme's density stays a density, with a Gauss field of at most the total charge L."""
    from paper_2411_09605_amd import Pic
    _say(f"case: runaway particle {which} in {scheme}")
    speed = 1e25
    wl = _workload(scheme, 1001, 32, 2)
    wl.v = wl.v.copy()
    wl.v[0, which] = speed
    gpu = Pic.from_workload(wl, scheme=scheme)
    e0 = gpu.state()["E"]
    steps = 1 if scheme in EM else 2
    gpu.step(steps)
    e1 = gpu.state()["E"]
    assert np.isfinite(e1).all()
    w, h = wl.length / wl.n_particles, wl.length / wl.n_cells
    bound = wl.length if scheme == "standard" else 1.5 * steps * wl.dt * w * speed / h
    assert np.abs(e1 - (0.0 if scheme == "standard" else e0)).max() <= bound
