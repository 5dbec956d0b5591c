"""The forms of the stepwise loop: entries from the CSR or the padded row image,
state words as buffer offsets or at 64-bit global addresses
(OIM_STEPWISE_GLOBAL_ADDR=1, at any number of replicas), several quads per wave
below 33 replicas."""
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


def _run(oim, prob, R, q, run):
    K, Ks, sg = (_t(x) for x in ramp_schedule(prob.info["max_abs_row_sum"], q, 150))
    th = _t(synth.theta0(R, prob.n, seed=R))
    ph = oim.oim_phase_from_theta(th)
    out = run(K, Ks, sg, th, ph)
    return [th.cpu().numpy(), ph.cpu().numpy()] + [v.cpu().numpy() for v in out.values()]


# several quads per wave: the padded image at any size here, the CSR below 33
# quads and from 1250 (4 replicas: 2000) on
@pytest.mark.parametrize("weights", ["pm1", "real"])
@pytest.mark.parametrize("n,R,q", [(203, 1, 2), (203, 5, 3), (203, 32, 5), (203, 33, 2), (203, 70, 3),
                                   (203, 70, 5), (97, 2, 5), (97, 4, 2), (97, 3, 3), (5003, 5, 5),
                                   (5003, 32, 3), (5003, 17, 2), (8003, 1, 3), (8003, 4, 5)])
def test_stepwise_addressing_same_bits(oim, n, R, q, weights, monkeypatch):
    # one problem for both ways of addressing, so that a graph captured for one
    # may not serve the other; the CSR and the padded row image
    if n < 1000:
        g = synth.random_small(n, 10 / n, seed=7, weights=weights)
    else:
        g = synth.gnp_avg_degree(n, 5, seed=7)
        if weights == "real":
            ei, ej, _ = g.upper_edges()
            g = synth.csr_from_edges(n, ei, ej, np.random.default_rng(3).standard_normal(ei.size))
    ref = None
    for image in ("0", "1"):
        monkeypatch.setenv("OIM_STEPWISE_ELL", image)
        with oim.Problem.from_csr(g.n, g.row_ptr, g.col, (-g.w).astype(np.float32)) as prob:
            assert (prob.info["stepwise_row_length"] > 0) == (image == "1")
            for addr in ("0", "1", "0"):
                monkeypatch.setenv("OIM_STEPWISE_GLOBAL_ADDR", addr)
                got = _run(oim, prob, R, q, lambda K, Ks, sg, th, ph: oim.run(
                    prob, th, K, Ks, sg, _t(synth.seeds(R, 8)), q=q, dt=DT, step0=5,
                    readout_every=23, want_best=True, flags=oim.OIM_LOOP_STEPWISE, phase=ph))
                if ref is None:
                    ref = got
                for a, b in zip(got, ref):
                    np.testing.assert_array_equal(a, b, err_msg=f"image {image} addr {addr}")


@pytest.mark.parametrize("rows,R", [(10, 3), (400, 32)])
def test_stepwise_global_addressing_at_any_size(oim, rows, R, monkeypatch):
    # the kernel that ran, by name
    import torch
    g = synth.torus(rows, 12, seed=3)
    with oim.Problem.from_csr(g.n, g.row_ptr, g.col, (-g.w).astype(np.float32)) as prob:
        for addr, kernel in (("0", "stepwise_packed_kernel"), ("1", "stepwise_step_kernel")):
            monkeypatch.setenv("OIM_STEPWISE_GLOBAL_ADDR", addr)
            K, Ks, sg = (_t(x) for x in ramp_schedule(prob.info["max_abs_row_sum"], 2, 3))
            th = _t(synth.theta0(R, g.n, seed=1))
            seeds = _t(synth.seeds(R, 2))
            torch.cuda.synchronize()
            with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
                oim.oim_run_noalloc(prob.handle, g.n, th, K, Ks, sg, seeds, q=2, dt=DT,
                                    flags=oim.OIM_LOOP_STEPWISE)
                torch.cuda.synchronize()
            steps = {k for e in prof.events()
                     for k in ("stepwise_packed_kernel", "stepwise_step_kernel") if k in e.name}
            assert steps == {kernel}


def _ring_of(n, degree):
    """n oscillators with `degree` neighbours each."""
    i = np.arange(n)
    ei, ej = zip(*[(i, (i + k) % n) for k in range(1, degree // 2 + 1)])
    return synth.csr_from_edges(n, np.concatenate(ei), np.concatenate(ej), np.ones(n * degree // 2))


@pytest.mark.parametrize("R", [1, 2, 16, 32, 40, 64, 200])
@pytest.mark.parametrize("n,degree", [(9, 2), (64, 4), (301, 6), (1003, 4), (5001, 4), (8192, 2),
                                      (8193, 2)])
def test_stepwise_readouts(oim, orc, n, degree, R):
    # in-run readouts with blocks of 16 to 256 rows, the colours of a best by
    # either kernel (up to 8192 oscillators, and above)
    q = 2 if R % 2 == 0 else 3
    g = _ring_of(n, degree)
    J = (-g.w).astype(np.float32)
    with oim.Problem.from_csr(n, g.row_ptr, g.col, J) as prob:
        K, Ks, sg = (_t(x) for x in ramp_schedule(prob.info["max_abs_row_sum"], q, 11))
        th = _t(synth.theta0(R, n, seed=R))
        ph = oim.oim_phase_from_theta(th)
        out = oim.run(prob, th, K, Ks, sg, _t(synth.seeds(R, 3)), q=q, dt=DT, readout_every=4,
                      want_best=True, flags=oim.OIM_LOOP_STEPWISE, phase=ph)
        out = {k: v.cpu().numpy() for k, v in out.items()}
        words = ph.cpu().numpy()
    np.testing.assert_array_equal(out["best_h"], out["trace"].min(axis=0))
    np.testing.assert_array_equal(out["best_step"],
                                  np.array([4, 8, 11])[out["trace"].argmin(axis=0)])
    for r in sorted({0, R // 2, R - 1}):
        assert out["best_h"][r] == orc.h_model_fixed(g.row_ptr, g.col, J, q, out["best_colour"][r])
        last = (((q * words[r].astype(np.uint64) + (1 << 31)) >> 32) % q).astype(np.int8)
        assert out["trace"][-1, r] == orc.h_model_fixed(g.row_ptr, g.col, J, q, last)
