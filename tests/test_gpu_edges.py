"""The GPU kernels at the edges of how they split the grid's nodes, a lane's particles and
the Gauss solve over threads, wavefronts and workgroups, against the oracle on the same
inputs (the 1e-10 bar of tests/gpu_util.py; initial fields 1e-12, gradients 1e-8, as the
tests of each form have them)."""
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


def _weights(wl):
    wl.w = wl.length / wl.n_particles * (1.0 + 0.5 * workloads.uniforms(31, 7, wl.n_particles))
    return wl


@pytest.mark.parametrize("scheme", ["esec2", "esec1", "standard"])
@pytest.mark.parametrize("ng", [5, 63, 64, 65, 128, 129, 193, 513])
def test_nodes_over_one_wavefront(scheme, ng):
    """Workgroups of one wavefront on grids just below, at and just above one, two, three and
    eight nodes per thread; a ragged count, weights."""
    _say(f"case: {scheme} on {ng} cells, 64 threads")
    wl = _weights(workloads.two_stream(n_particles=3001, n_cells=ng, steps=5))
    gu.run_pair(wl, 5, scheme=scheme, block_threads=64, grid_blocks=9)


@pytest.mark.parametrize("scheme", ["emec_li", "emec_psatd", "emec_lf"])
@pytest.mark.parametrize("ng,threads", [(5, 0), (63, 64), (64, 0), (65, 64), (129, 64), (257, 0)])
def test_fields_over_wavefronts(scheme, ng, threads):
    """Field launches with a node to a wavefront, and the passes' copies of the field tiles with
    their periodic images, from the smallest grid to one past a whole number of wavefronts."""
    _say(f"case: {scheme} on {ng} cells, threads {threads}")
    wl = _weights(workloads.weibel(n_particles=4001, n_cells=ng, steps=5))
    wl.dt = min(wl.dt, 0.9 * wl.length / ng)
    wl.B0 = wl.B0 * 50.0
    gu.run_pair(wl, 5, scheme=scheme, block_threads=threads)


@pytest.mark.parametrize("ng,order", [(3, 1), (5, 2), (64, 1), (65, 2), (511, 2), (512, 2), (513, 2),
                                      (1024, 1), (1500, 2)])
def test_gauss_solve_segments(ng, order):
    """The initial Gauss solve over its segments of the grid (several up to 512 cells, whole
    above) with weights, also from the initial deposits of several workgroups."""
    from paper_2411_09605_amd import Pic
    _say(f"case: Gauss on {ng} cells, order {order}")
    wl = _weights(workloads.two_stream(n_particles=20_011, n_cells=ng, order=order, alpha=0.05))
    o = oracle.State(wl)
    orec = o.run(0)
    for knobs in ({}, dict(grid_blocks=300, block_threads=64), dict(deterministic=True)):
        gpu = Pic.from_workload(wl, **knobs)
        rec = gpu.diagnostics()
        E = gpu.state()["E"][0]
        assert np.abs(E - o.E[0]).max() < 1e-12 * np.abs(o.E[0]).max()
        assert abs(rec["total"][0] - orec["total"][0]) < 1e-13 * orec["total"][0]


@pytest.mark.parametrize("n,ng,dt,speed", [(1, 3, 0.4, 1.0), (65, 3, 3.0, 1.0), (200, 4, 2.0, 1.0),
                                           (3001, 16, 2.0, 1.0), (3001, 64, 0.4, 40.0)])
@pytest.mark.parametrize("threads", [64, 1024])
def test_cc_paths_of_many_cells(n, ng, dt, speed, threads):
    """Charge-conserving paths from less than a cell to several periods of the grid in a step,
    where the lanes of a wavefront cut their paths into very different numbers of pieces."""
    _say(f"case: charge conserving n {n} cells {ng} dt {dt} speed x{speed} threads {threads}")
    wl = _weights(workloads.two_stream(n_particles=n, n_cells=ng, dt=dt, steps=4, order=1, alpha=0.05,
                                       v_beam=3.0, v_spread=0.5))
    wl.v = wl.v.copy()
    wl.v[:, ::7] *= speed
    gu.run_pair(wl, 4, charge_conserving=True, block_threads=threads)


@pytest.mark.parametrize("n,ng,every", [(63, 5, 3), (1000, 7, 20), (4001, 130, 6), (4001, 515, 9),
                                        (4001, 1750, 20), (300_001, 64, 7)])
def test_adjoint_small_and_wide_grids(n, ng, every):
    """Reverse passes on grids narrower than their ghost cells and with more nodes than a
    workgroup has threads; ragged particle counts and a last segment of its own.  The segments'
    recompute on a grid whose fields fit the LDS once but not twice (1750 cells), and with
    several groups of particles to a workgroup (300001)."""
    from paper_2411_09605_amd import PicAdjoint
    _say(f"case: adjoint n {n} cells {ng} checkpoint every {every}")
    wl = workloads.adjoint_two_stream(n_particles=n, n_cells=ng, alphas=(2e-2, 1e-2), v_beam=1.5,
                                      v_spread=0.2, dt=0.1, steps=20, order=2, seed=23)
    adj = PicAdjoint.from_workload(wl, checkpoint_every=every)
    m = wl.meta
    J = adj.forward(m["alphas"], m["v_beam"], m["v_spread"])
    g = adj.backward(1.0)
    Jo, go, _ = oracle.two_stream_gradient(wl, wl.steps)
    assert abs(J - Jo) <= 1e-10 * abs(Jo), (J, Jo)
    assert np.abs(g - go).max() <= 1e-8 * np.abs(go).max(), (g, go)


@pytest.mark.parametrize("graph_steps", [0, 1, 3])
def test_batch_step_counts(graph_steps):
    """Batched runs of uneven grids advanced by odd and even numbers of steps, plain or from a
    graph of an odd length, each call leaving off where the next goes on."""
    import torch
    from paper_2411_09605_amd import PicBatch
    _say(f"case: batch, graph of {graph_steps} steps")
    runs = [workloads.landau(n_particles=n, n_cells=ng, order=2, alpha=0.1, seed=40 + ng)
            for n, ng in ((1, 5), (65, 64), (2049, 65), (3001, 513))]
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        b = PicBatch(runs, **(dict(graph_steps=graph_steps, stream=s) if graph_steps else {}))
        orcs = [oracle.State(wl) for wl in runs]
        done = 0
        for n in (1, 2, 3, 1, 4):
            b.step(n)
            done += n
            for k, (wl, o) in enumerate(zip(runs, orcs)):
                o.run(n)
                gu.compare_state(b.state(k), o, wl.length, max(1.0, float(np.abs(wl.v).max())), False,
                                 where=f"run {k} step {done}")
        for k in range(len(runs)):
            assert b.diagnostics(k)["step"][-1] == done


@pytest.mark.parametrize("n,ng,threads", [(10_000, 64, 64), (10_000, 65, 128), (10_000, 512, 512),
                                          (10_000, 1024, 512), (10_000_000, 64, 1024)])
def test_default_threads_cover_the_nodes(n, ng, threads):
    """Two particles per thread of 256 workgroups, but a thread per node up to 512."""
    from paper_2411_09605_amd import Pic
    _say(f"case: default threads n {n} cells {ng}")
    assert Pic.from_workload(workloads.landau(n_particles=n, n_cells=ng)).launch_shape()[0] == threads
