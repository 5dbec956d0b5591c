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


@pytest.mark.parametrize("weights", ["pm1", "real"])
@pytest.mark.parametrize("R,q", [(1, 2), (5, 3), (32, 5), (33, 2), (70, 3), (70, 5)])
def test_stepwise_addressing_same_bits(oim, R, q, weights, monkeypatch):
    # one problem for both ways of addressing, so that a graph captured for one
    # may not serve the other; the CSR and the padded row image
    g = synth.random_small(203, 0.05, seed=7, weights=weights)
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


@pytest.mark.parametrize("R", [3, 32])
def test_stepwise_global_addressing_at_any_size(oim, R, monkeypatch):
    # the kernel that ran, by name
    import torch
    g = synth.torus(10, 12, seed=3)
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
