"""Problems created where device memory is short (OIM_IMAGE_LIMIT counts an
allocation above that many bytes as refused): what runs can do without is left
out, and the general kernel's shapes of one slice per wave group take the
sorted rows' place, bit for bit; the adjoint makes its rows on first use."""
import numpy as np
import pytest

import synth
from _util import DT, ramp_schedule
from test_gpu_adjoint import _gpu_adjoint, _schedules, dev, oim  # noqa: F401

pytestmark = pytest.mark.gpu

SHAPES = ((64, 1, 4), (128, 1, 4), (256, 1, 4), (512, 1, 4), (1024, 1, 4), (256, 1, 1), (256, 1, 2),
          (512, 1, 1), (512, 1, 2), (1024, 1, 1), (1024, 1, 2))


def _t(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _batch(sizes, weights):
    rng = np.random.default_rng(sum(sizes))
    graphs = []
    for n in sizes:
        a, b = rng.integers(0, n, (2, 8 * n))
        pairs = np.unique(np.stack([np.minimum(a, b), np.maximum(a, b)], 1)[a != b], axis=0)
        w = np.ones(len(pairs)) if weights == "unit" else rng.standard_normal(len(pairs))
        graphs.append(synth.csr_from_edges(n, pairs[:, 0], pairs[:, 1], w))
    big, off = synth.block_diagonal(graphs)
    return big, (-big.w).astype(np.float32), off


def _create(oim, monkeypatch, limit, big, J, off):  # noqa: F811
    if limit is None:
        monkeypatch.delenv("OIM_IMAGE_LIMIT", raising=False)
    else:
        monkeypatch.setenv("OIM_IMAGE_LIMIT", str(limit))
    try:
        return oim.Problem.from_csr_blocks(big.n, big.row_ptr, big.col, J, off)
    except oim.OimError as e:
        assert "OIM_E_NOMEM" in str(e)
        return None
    finally:
        monkeypatch.delenv("OIM_IMAGE_LIMIT", raising=False)


def _least(oim, monkeypatch, big, J, off):  # noqa: F811
    """The smallest limit a problem is created under: without optional images."""
    lo, hi = 0, 1 << 26
    while hi - lo > 1:
        mid = (lo + hi) // 2
        prob = _create(oim, monkeypatch, mid, big, J, off)
        if prob is None:
            lo = mid
        else:
            prob.close()
            hi = mid
    return hi


@pytest.mark.parametrize("q", [2, 3, 5])
@pytest.mark.parametrize("weights", ["unit", "real"])
@pytest.mark.parametrize("sizes", [[250, 3, 129], [500, 64], [1000], [1900], [4000]])
def test_runs_without_the_sorted_rows(oim, dev, monkeypatch, sizes, weights, q):  # noqa: F811
    import torch
    big, J, off = _batch(sizes, weights)
    R, steps = 2, 7
    least = _least(oim, monkeypatch, big, J, off)
    th0, sd = synth.theta0(R, big.n, seed=1), synth.seeds(R, 4)
    ref, ran = None, set()
    for limit in (None, least):
        with _create(oim, monkeypatch, limit, big, J, off) as prob:
            K, Ks, sg = (_t(x) for x in ramp_schedule(prob.info["max_abs_row_sum"], q, steps))
            for shape in (None,) + SHAPES:
                if shape:
                    try:
                        oim.oim_set_tuning(prob.handle, q, *shape)
                    except oim.OimError:
                        continue  # does not cover the largest instance
                th = _t(th0)
                ph = oim.oim_phase_from_theta(th)
                out = oim.run(prob, th, K, Ks, sg, _t(sd), q=q, dt=DT, readout_every=3, phase=ph,
                              want_best=True)
                got = [th, ph] + list(out.values())
                if ref is None:
                    ref = got
                for a, b in zip(got, ref):
                    assert torch.equal(a, b), (limit, shape)
                ran.add((limit, shape))
    assert len(ran) >= 4  # the default and at least one shape on either side


def test_which_kernel_ran(oim, dev, monkeypatch):  # noqa: F811
    import torch
    big, J, off = _batch([300], "unit")
    least = _least(oim, monkeypatch, big, J, off)
    for limit, kernel in ((None, "sorted_kernel"), (least, "persistent_sparse_kernel")):
        with _create(oim, monkeypatch, limit, big, J, off) as prob:
            args = [_t(x) for x in (*ramp_schedule(1.0, 2, 3), synth.seeds(1, 1))]
            th = _t(synth.theta0(1, big.n, seed=1))
            with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
                oim.run(prob, th, *args, q=2, dt=DT)
                torch.cuda.synchronize()
            names = {k for e in prof.events() for k in ("sorted_kernel", "persistent_sparse_kernel")
                     if k in e.name}
            assert names == {kernel}


@pytest.mark.parametrize("weights", ["unit", "real"])
@pytest.mark.parametrize("sizes", [[40], [300, 1, 517]])
def test_adjoint_makes_its_rows(oim, dev, monkeypatch, sizes, weights):  # noqa: F811
    big, J, off = _batch(sizes, weights)
    least = _least(oim, monkeypatch, big, J, off)
    K, Ks, sg = _schedules(20)
    th0, sd = synth.theta0(2, big.n, seed=5), synth.seeds(2, 6)
    outs = []
    for limit in (None, least, least):
        with _create(oim, monkeypatch, limit, big, J, off) as prob:
            outs.append(_gpu_adjoint(oim, prob, th0, K, Ks, sg, sd, 2, 6))
            outs.append(_gpu_adjoint(oim, prob, th0, K, Ks, sg, sd, 2, 6))
    for out in outs[1:]:
        for a, b in zip(out, outs[0]):
            np.testing.assert_array_equal(a, b)
