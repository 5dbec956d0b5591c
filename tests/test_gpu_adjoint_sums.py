"""The adjoint with the row sums formed again (as for segments whose sums take
more than 8 GiB, or where they cannot be had) against the oracle, and bit for
bit against the handed-over sums: every SHIL order class, unit and general
weights, rows in LDS and streamed from device memory."""
import numpy as np
import pytest

import synth
from _util import DT
from test_gpu_adjoint import _close_vec, _gpu_adjoint, _schedules, dev, oim  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q", [2, 3, 5])
@pytest.mark.parametrize("weights", ["unit", "real"])
@pytest.mark.parametrize("sizes", [[1, 65, 300], [1500, 129]])
def test_adjoint_forming_sums_again(oim, orc, dev, monkeypatch, sizes, weights, q):  # noqa: F811
    rng = np.random.default_rng(q)
    graphs = []
    for n in sizes:
        a, b = rng.integers(0, n, (2, 3 * n))
        pairs = np.unique(np.stack([np.minimum(a, b), np.maximum(a, b)], 1)[a != b], axis=0)
        w = np.ones(len(pairs)) if weights == "unit" else rng.standard_normal(len(pairs))
        w *= rng.choice([-1.0, 1.0], len(pairs))
        graphs.append(synth.csr_from_edges(n, pairs[:, 0], pairs[:, 1], w))
    big, off = synth.block_diagonal(graphs)
    J = (-big.w).astype(np.float32)
    steps, R, C = 30, 2, 11
    K, Ks, sg = _schedules(steps)
    K = (K / 4.0).astype(np.float32)
    th0 = synth.theta0(R, big.n, seed=8)
    sd = synth.seeds(R, 2)
    got = {}
    for sums in ("1", "0"):
        for rows in ("", "global"):
            monkeypatch.setenv("OIM_ADJ_SUMS", sums)
            monkeypatch.setenv("OIM_ADJ_ROWS", rows)
            with oim.Problem.from_csr_blocks(big.n, big.row_ptr, big.col, J, off) as prob:
                got[sums, rows] = _gpu_adjoint(oim, prob, th0, K, Ks, sg, sd, q, C)
    for key, out in got.items():
        for a, b in zip(out, got["0", ""]):
            np.testing.assert_array_equal(a, b, err_msg=str(key))
    loss, _, gK, gKs, gS = got["0", ""]
    L, oK, oKs, oS = orc.adjoint_csr(big.row_ptr, big.col, J.astype(np.float64),
                                     th0.astype(np.float64), q=q, dt=DT, K=K, Ks=Ks, sigma=sg,
                                     seeds=sd, inst_off=off)
    assert loss.sum() == pytest.approx(L, rel=1e-5)
    for g, ref, name in ((gK, oK, "K"), (gKs, oKs, "Ks"), (gS, oS, "sigma")):
        ok, rel = _close_vec(g, ref, 1e-4)
        assert ok, (name, rel)


def test_adjoint_sums_switch(oim, dev, monkeypatch):  # noqa: F811
    # the kernel that ran, by its last template argument
    import torch
    g = synth.torus(6, 6, seed=1)
    K, Ks, sg = _schedules(4)
    with oim.Problem.from_csr(g.n, g.row_ptr, g.col, (-g.w).astype(np.float32)) as prob:
        for sums, wide in (("1", "false"), ("0", "true")):
            monkeypatch.setenv("OIM_ADJ_SUMS", sums)
            with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
                _gpu_adjoint(oim, prob, synth.theta0(1, g.n, seed=1), K, Ks, sg, synth.seeds(1, 2),
                             2, 2)
            names = {e.name for e in prof.events() if "adjoint_segment_kernel" in e.name}
            assert names and all(f", {wide}>" in n for n in names), names
