"""States outside what a plasma reaches: particles so fast that a coordinate in cells exceeds
what a double resolves, values that are not finite, and deposits beyond the deterministic
mode's range.  A run may not be meaningful then, but its sums stay those of its particles and
its records say what happened."""
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


@pytest.mark.parametrize("scheme,order,knobs", [
    ("esec2", 1, {}), ("esec2", 2, {}), ("esec2", 1, dict(charge_conserving=True)),
    ("esec2", 2, dict(deterministic=True)), ("esec2", 2, dict(deposit_mode="window")),
    ("esec1", 1, {}), ("esec1", 2, {}), ("standard", 1, {}), ("standard", 2, {}),
    ("emec_li", 1, {}), ("emec_li", 2, {}), ("emec_psatd", 2, {}), ("emec_lf", 2, {})])
@pytest.mark.parametrize("weights", [False, True])
def test_non_finite_states_are_recorded(scheme, order, knobs, weights):
    """A position or a velocity that is not finite, in the first, a middle and the ragged last
    batch, also of a particle that carries no weight: the records of the steps that follow say
    so (and those of a clean run don't)."""
    import torch
    from paper_2411_09605_amd import Pic
    _say(f"case: non-finite {scheme} order {order} {knobs} weights {weights}")
    n, ng = 3001, 48
    wl = _workload(scheme, n, ng, order)
    if weights:
        wl.w = wl.length / n * np.ones(n)
    for which, array, value in [(None, None, None), (0, "x", np.nan), (1500, "x", np.nan), (n - 1, "x", np.nan),
                                (0, "v", np.nan), (1500, "v", np.inf), (n - 1, "v", -np.inf)]:
        if weights and which is not None:
            wl.w = wl.length / n * np.ones(n)
            wl.w[which] = 0.0
        gpu = Pic.from_workload(wl, scheme=scheme, block_threads=64, grid_blocks=7, **knobs)
        gpu.step(1)
        if which is not None:
            (gpu.x if array == "x" else gpu.v[0])[which] = value
            torch.cuda.synchronize()
        gpu.step(2)
        rec = gpu.diagnostics()
        assert list(rec["step"]) == [0, 1, 2, 3]
        assert list(rec["nonfinite"]) == [0, 0, 0, 0] if which is None else rec["nonfinite"][2:].min() == 1, \
            (which, array, value, rec["nonfinite"])


def test_deterministic_deposit_out_of_range_is_recorded():
    """The deterministic mode drops a contribution more than 2^12 times the range set by the
    initial particles and reports it.  Only the centred deposit is out of range here: the field
    of one node throws the particle that sits on it half a period away, where there is none."""
    from paper_2411_09605_amd import Pic
    _say("case: deterministic deposit out of range")
    n, ng, L, dt = 64, 64, 10.0, 0.1
    a = 2000.0 * 501                     # dt^2 a / 4 = 250.5 periods from x to x^{1/2}
    x = np.full(n, 7.5)
    x[0] = 20 * L / ng
    E0 = np.zeros((3, ng))
    E0[0, 20] = a
    for deterministic in (False, True):
        gpu = Pic.from_arrays(1, "esec2", 1, ng, L, dt, x, np.zeros((1, n)), E0=E0,
                              deterministic=deterministic)
        gpu.step(1)
        rec = gpu.diagnostics()
        assert list(rec["nonfinite"]) == [0, int(deterministic)]
        assert np.abs(gpu.state()["v"]).max() < 1.0 or not deterministic
