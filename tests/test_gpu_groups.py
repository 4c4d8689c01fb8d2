"""How many of a lane's particles a pass loads at once and computes on together: one or two
of each by the number of velocity components, the kind of deposit and the form (single or
batched).  Every combination against the oracle on counts around a batch (the 1e-10 bar of
tests/gpu_util.py)."""
import numpy as np
import pytest

import oracle
import workloads
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_09605_amd  # noqa: F401


def _say(msg):
    print(msg, flush=True)


def _weibel(n, ng, order, seed=11):
    wl = workloads.weibel(n_particles=n, n_cells=ng, order=order, steps=4, seed=seed)
    wl.dt = min(wl.dt, 0.9 * wl.length / ng)
    wl.B0 = wl.B0 * 50.0
    wl.w = wl.length / n * (1.0 + 0.5 * workloads.uniforms(31, 7, n))
    return wl


@pytest.mark.parametrize("n", [1, 64, 65, 128, 129, 4001])
@pytest.mark.parametrize("mode", ["window", "wave", "lds_f64", "lds_atomic"])
@pytest.mark.parametrize("scheme,order", [("emec_li", 1), ("emec_li", 2), ("emec_lf", 2), ("esec2", 1), ("esec2", 2)])
def test_three_components_by_deposit(scheme, order, mode, n):
    _say(f"case: {scheme} order {order} deposit {mode} particles {n}")
    wl = _weibel(n, 33, order)
    if scheme == "esec2":
        wl.E0 = wl.B0 = None
        wl.init_gauss, wl.b_ext = True, (0.3, 0.1, -0.2)
    gu.run_pair(wl, 3, scheme=scheme, deposit_mode=mode, block_threads=64, grid_blocks=5)


@pytest.mark.parametrize("scheme,order", [("emec_li", 1), ("emec_li", 2), ("esec2", 1), ("esec2", 2), ("esec1", 2)])
@pytest.mark.parametrize("threads", [64, 512])
def test_batched_three_components(scheme, order, threads):
    from paper_2411_09605_amd import PicBatch
    _say(f"case: batch of {scheme} order {order} threads {threads}")
    runs = []
    for n, ng in ((1, 5), (64, 33), (65, 64), (129, 65), (4001, 193)):
        wl = _weibel(n, ng, order, seed=40 + ng)
        wl.scheme, wl.dt = scheme, 0.01
        if scheme != "emec_li":
            wl.E0 = wl.B0 = None
            wl.init_gauss, wl.b_ext = True, (0.3, 0.1, -0.2)
        runs.append(wl)
    b = PicBatch(runs, block_threads=threads, chunk=1024)
    orcs = [oracle.State(wl) for wl in runs]
    for n in (1, 2, 3):
        b.step(n)
        for k, (wl, o) in enumerate(zip(runs, orcs)):
            o.run(n)
            gu.compare_state(b.state(k), o, wl.length, max(1.0, float(np.abs(wl.v).max())), scheme == "emec_li",
                             where=f"run {k}")


@pytest.mark.parametrize("scheme", ["esec2", "standard"])
@pytest.mark.parametrize("n", [1, 703, 1409, 8449, 30_001])
def test_eleven_wavefronts(scheme, n):
    """The workgroups of the largest runs (704 threads, interleaved batches) on small ones."""
    _say(f"case: 704 threads, {scheme}, {n} particles")
    wl = workloads.two_stream(n_particles=n, n_cells=77, steps=4)
    wl.w = wl.length / n * (1.0 + 0.5 * workloads.uniforms(31, 7, n))
    gu.run_pair(wl, 4, scheme=scheme, block_threads=704, grid_blocks=3, interleave=True)


@pytest.mark.parametrize("n,scheme,knobs,threads", [
    (50_000_000, "esec2", {}, 1024), (50_000_001, "esec2", {}, 704), (50_000_001, "standard", {}, 704),
    (50_000_001, "esec1", {}, 1024), (50_000_001, "esec2", dict(charge_conserving=True), 1024),
    (50_000_001, "esec2", dict(deposit_mode="window"), 1024), (50_000_001, "esec2", dict(block_threads=512), 512)])
def test_default_threads_of_the_largest_runs(n, scheme, knobs, threads):
    import torch
    from paper_2411_09605_amd import Pic, binding
    _say(f"case: default threads of {n} particles, {scheme} {knobs}")
    p = binding.make_params(1, scheme, 1, n, 64, 12.0, 0.1, init_gauss=True, **knobs)
    x = torch.arange(n, device="cuda", dtype=torch.float64) * (12.0 / n)
    gpu = Pic(p, x, torch.zeros(1, n, device="cuda", dtype=torch.float64),
              torch.zeros(3, 64, device="cuda", dtype=torch.float64))
    assert gpu.launch_shape()[0] == threads


@pytest.mark.parametrize("order,ng", [(1, 1842), (2, 1446)])
def test_esec1_on_the_largest_grids(order, ng):
    """The largest grids that ESEC1 accepts (its tiles in LDS end within the launch)."""
    from paper_2411_09605_amd import binding
    _say(f"case: ESEC1 order {order} on {ng} cells")
    wl = workloads.two_stream(n_particles=6001, n_cells=ng, order=order, steps=3)
    gu.run_pair(wl, 3, scheme="esec1")
    p = binding.make_params(1, "esec1", order, 6001, ng + 1, wl.length, wl.dt)
    assert binding.validate(p) == -6
