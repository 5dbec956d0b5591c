"""The LDS-resident loop's default launch shape on both sides of its lines: runs
of many replicas agree bit for bit with runs of few, whose shape is another."""
import numpy as np
import pytest

import synth
from _util import DT, ramp_schedule

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oim():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22631_amd as m
    m.lib()
    return m


def _t(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _check(oim, graphs, weights, R, q=2, few=3):
    big, off = synth.block_diagonal(graphs)
    if weights == "unit":
        J = -np.ones(big.nnz, np.float32)
    else:
        ei, ej, _ = big.upper_edges()
        rng = np.random.default_rng(1)
        big = synth.csr_from_edges(big.n, ei, ej, rng.standard_normal(ei.size))
        J = (-big.w).astype(np.float32)
    n, I, steps = big.n, len(graphs), 5
    th0, sd = synth.theta0(R, n, seed=R), synth.seeds(R, 2)
    outs = []
    with oim.Problem.from_csr_blocks(n, big.row_ptr, big.col, J, off) as prob:
        K, Ks, sg = (_t(x) for x in ramp_schedule(prob.info["max_abs_row_sum"], q, steps))
        for reps in (R, few):
            th = _t(th0[:reps])
            ph = oim.oim_phase_from_theta(th)
            out = oim.run(prob, th, K, Ks, sg, _t(sd[:reps]), q=q, dt=DT, readout_every=2, phase=ph,
                          want_best=True)
            outs.append([ph, out["best_colour"], out["best_h"].view(reps, I),
                         out["best_step"].view(reps, I), out["trace"].view(3, reps, I).transpose(0, 1)])
    for a, b in zip(*outs):
        assert bool((a[:few] == b).all())


# slices, waves per split shape, row length and workgroups per CU at the lines
@pytest.mark.parametrize("n,degree,R", [
    (400, 4, 2000), (600, 4, 600), (600, 4, 1000), (600, 4, 2000), (600, 4, 3000), (600, 30, 1000),
    (1000, 4, 600), (1000, 4, 1500), (800, 30, 4500), (1100, 4, 1000), (1100, 10, 300),
    (1500, 10, 300), (1500, 4, 700), (2049, 4, 300), (2049, 4, 600), (2049, 4, 2000),
    (2100, 30, 300), (2100, 30, 600), (2500, 30, 600), (3000, 10, 300), (3000, 10, 2000),
    (4000, 4, 1000), (12600, 4, 3), (200, 4, 3200), (400, 4, 1500), (400, 14, 1500), (600, 4, 3100),
    (600, 10, 1000), (600, 20, 1500), (800, 14, 1300), (800, 20, 600), (1500, 4, 400),
    (1500, 4, 1400), (2000, 10, 700), (2300, 30, 300), (3000, 14, 1400)])
@pytest.mark.parametrize("weights", ["unit", "real"])
def test_default_shape_same_bits(oim, n, degree, R, weights):
    _check(oim, [synth.gnp_avg_degree(n, degree, seed=n + degree)], weights, R)


@pytest.mark.parametrize("n,degree,R", [(2500, 6, 1000), (2500, 30, 1000), (4000, 30, 1000),
                                        (4100, 6, 300), (6000, 6, 300)])
@pytest.mark.parametrize("q", [2, 3, 5])
def test_default_shape_by_shil_order(oim, n, degree, R, q):
    _check(oim, [synth.gnp_avg_degree(n, degree, seed=n + degree)], "unit", R, q)


def test_default_shape_of_images_beyond_the_caches(oim):
    # few replicas of many graphs: 1024 of three slices
    sizes = np.random.default_rng(3).integers(300, 600, 1024).tolist()
    _check(oim, [synth.gnp_avg_degree(n, 4.6, seed=i) for i, n in enumerate(sizes)], "real", 3,
           few=1)


@pytest.mark.parametrize("R", [2, 4, 6, 17])
@pytest.mark.parametrize("weights", ["unit", "real"])
def test_default_shape_of_ragged_batches(oim, R, weights):
    sizes = np.random.default_rng(2).integers(60, 320, 255).tolist() + [599]
    _check(oim, [synth.gnp_avg_degree(n, 4.6, seed=n) for n in sizes], weights, R, q=3, few=1)
