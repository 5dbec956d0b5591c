"""Every shape of the scoring kernels (waves and replicas per workgroup, entries
one by one or in groups, lanes per row) where it can go wrong: one wave for
several replicas, ragged replica groups, rows around a block of 64, the first
and last replica of a launch that fills the chip."""
import numpy as np
import pytest

import synth

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


def _check(oim, orc, prob, csr, R, q, theta):
    """Replicas repeat 7 patterns: those of the first and of the last period
    equal the oracle, and every other one its pattern."""
    n, P = prob.n, 7
    rp, cl, J = csr
    rng = np.random.default_rng(n + R)
    col = rng.integers(0, q, (P, n)).astype(np.int8)
    th = synth.theta0(P, n, seed=n)
    rep = -(-R // P)
    dcol = _t(col).repeat(rep, 1)[:R].contiguous()
    dth = _t(th).repeat(rep, 1)[:R].contiguous() if theta else None
    hm, h6 = oim.oim_energy(prob.handle, q, dth, dcol)
    only6 = oim.oim_energy(prob.handle, q, dth, None)[1] if theta else None
    out = {"cut": oim.oim_cut(prob.handle, dcol, exact=False),
           "conf": oim.oim_conflicts(prob.handle, dcol), "hm": hm}
    if prob.info["integer_weights"]:
        out["cut_i"] = oim.oim_cut(prob.handle, dcol)
    if theta:
        out.update(h6=h6, only6=only6)
    out = {k: v.cpu().numpy() for k, v in out.items()}
    for k, v in out.items():
        np.testing.assert_array_equal(v, v[np.arange(R) % P], err_msg=k)
    bound = 2.0**-51 * np.abs(J).astype(np.float64).sum() / 2
    for r in range(min(R, P)):
        assert out["hm"][r] == orc.h_model_fixed(rp, cl, J, q, col[r])
        assert out["cut"][r] == orc.cut_fixed(rp, cl, J, col[r])
        assert out["conf"][r] == orc.conflicts(rp, cl, J, col[r])
        if "cut_i" in out:
            assert out["cut_i"][r] == out["cut"][r]
        if theta:
            assert out["h6"][r] == out["only6"][r]
            assert abs(out["h6"][r] - orc.h_eq6_fixed(rp, cl, J, th[r].astype(np.float64))) <= bound


# one, two and four replicas per workgroup of one, two and three waves
@pytest.mark.parametrize("n,R,q", [(1, 3, 2), (10, 2051, 2), (10, 16387, 3), (64, 2049, 3),
                                   (65, 1027, 2), (66, 8195, 2), (130, 703, 3), (130, 5463, 2),
                                   (1000, 2, 2), (1000, 257, 3), (150, 3, 2), (300, 1001, 3), (520, 257, 2),
                                   (520, 1003, 3), (960, 300, 2)])
@pytest.mark.parametrize("integer", [True, False])
def test_dense_shapes(oim, orc, n, R, q, integer):
    rng = np.random.default_rng(n)
    J = rng.integers(-3, 4, (n, n)) if integer else rng.standard_normal((n, n))
    J = np.triu(J, k=1).astype(np.float32)
    J = J + J.T
    with oim.Problem.from_dense(J) as prob:
        _check(oim, orc, prob, orc.dense_to_csr(J), R, q, True)


# (n, mean degree, replicas): 1 to 16 waves, entries one by one and in fours,
# long rows; whole-number sums of 64 to 1024 threads, 1, 4 and 16 lanes per row
@pytest.mark.parametrize("n,degree,R", [
    (25, 12, 88), (300, 20, 300), (300, 20, 400), (300, 20, 1001), (300, 20, 1600),
    (300, 16, 6200), (500, 40, 701), (500, 40, 1930), (700, 30, 30), (700, 30, 270),
    (9, 3, 5), (64, 6, 5000), (65, 6, 5000), (63, 4, 20001), (129, 5, 300), (200, 10, 1400),
    (300, 10, 4100), (600, 6, 601), (1100, 5, 300), (1025, 12, 700), (2100, 4, 12300),
    (4200, 12, 600), (9000, 12, 520), (9000, 4, 520), (130, 40, 600), (500, 60, 3), (500, 60, 200),
    (500, 40, 2100), (700, 30, 600)])
@pytest.mark.parametrize("weights", ["pm1", "real"])
def test_sparse_shapes(oim, orc, n, degree, R, weights):
    g = synth.gnp_avg_degree(n, min(degree, n - 1), seed=n + degree)
    if weights == "real":
        ei, ej, _ = g.upper_edges()
        rng = np.random.default_rng(n)
        w = rng.standard_normal(ei.size) * np.exp(rng.uniform(-4, 2, ei.size))
        g = synth.csr_from_edges(n, ei, ej, w.astype(np.float32))
    J = (-g.w).astype(np.float32)
    with oim.Problem.from_csr(n, g.row_ptr, g.col, J) as prob:
        _check(oim, orc, prob, (g.row_ptr, g.col, J), R, 2 if R % 2 else 3, n * R < 1e7)
