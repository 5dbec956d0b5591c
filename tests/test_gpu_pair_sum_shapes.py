"""Every shape of the scoring kernels (waves and replicas per workgroup) where it
can go wrong: one wave for several replicas, ragged replica groups, rows around
a block of 64, the first and last replica of a launch that fills the chip."""
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
                                   (65, 1027, 2), (66, 8195, 2), (130, 703, 3), (130, 5463, 2)])
@pytest.mark.parametrize("integer", [True, False])
def test_dense_shapes(oim, orc, n, R, q, integer):
    rng = np.random.default_rng(n)
    J = rng.integers(-3, 4, (n, n)) if integer else rng.standard_normal((n, n))
    J = np.triu(J, k=1).astype(np.float32)
    J = J + J.T
    with oim.Problem.from_dense(J) as prob:
        _check(oim, orc, prob, orc.dense_to_csr(J), R, q, True)
