"""GPU pair sums (cut, conflicts, Eq. 1 / 2 / 6 energies, in-run readouts) at
the sizes where their split can go wrong: partial row blocks and column
groups, every replica grouping of the dense sums, every lanes-per-row and
workgroup split of the whole-number sums, more than one round of blocks."""
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


def _dense(n, seed, integer):
    rng = np.random.default_rng(seed)
    J = rng.integers(-3, 4, (n, n)) if integer else rng.standard_normal((n, n)) * np.exp(
        rng.uniform(-6, 3, (n, n)))
    J = np.triu(J, k=1).astype(np.float32)
    return J + J.T


# 257 .. and 1025 .. replicas share a workgroup by two and by four
@pytest.mark.parametrize("n,R", [(1, 2), (2, 1), (63, 3), (64, 3), (65, 2), (80, 1), (1030, 2),
                                 (130, 301), (66, 1027)])
@pytest.mark.parametrize("integer", [True, False])
def test_dense_pair_sums(oim, orc, n, R, integer):
    J = _dense(n, 5 + n, integer)
    rp, cl, Jv = orc.dense_to_csr(J)
    np.fill_diagonal(J, np.nan)  # the diagonal is ignored
    rng = np.random.default_rng(n)
    th = synth.theta0(R, n, seed=n)
    check = sorted({0, R // 2, R - 1})
    with oim.Problem.from_dense(J) as prob:
        for q in (2, 3):
            col = rng.integers(0, q, (R, n)).astype(np.int8)
            hm, h6 = oim.oim_energy(prob.handle, q, _t(th) if R < 10 else None, _t(col))
            conf = oim.oim_conflicts(prob.handle, _t(col)).cpu().numpy()
            cutf = oim.oim_cut(prob.handle, _t(col), exact=False).cpu().numpy()
            cuti = oim.oim_cut(prob.handle, _t(col)).cpu().numpy() if integer else None
            for r in check:
                assert hm[r].item() == orc.h_model_fixed(rp, cl, Jv, q, col[r])
                assert cutf[r] == orc.cut_fixed(rp, cl, Jv, col[r])
                assert conf[r] == orc.conflicts(rp, cl, Jv, col[r])
                if integer:
                    assert cuti[r] == cutf[r]
                if h6 is not None:
                    want = orc.h_eq6_fixed(rp, cl, Jv, th[r].astype(np.float64))
                    assert abs(h6[r].item() - want) <= 2.0**-51 * np.abs(Jv).astype(np.float64).sum() / 2


@pytest.mark.parametrize("n,R,q", [(65, 2, 2), (200, 300, 2), (97, 1030, 3)])
def test_dense_in_run_readout_groups(oim, orc, n, R, q):
    J = _dense(n, n, False)
    rp, cl, Jv = orc.dense_to_csr(J)
    with oim.Problem.from_dense(J) as prob:
        K, Ks, sg = ramp_schedule(prob.info["max_abs_row_sum"], q, 5)
        th = _t(synth.theta0(R, n, seed=1))
        out = oim.run(prob, th, _t(K), _t(Ks), _t(sg), _t(synth.seeds(R, 9)), q=q, dt=DT,
                      readout_every=2, want_best=True)
        out = {k: v.cpu().numpy() for k, v in out.items()}
    np.testing.assert_array_equal(out["best_h"], out["trace"].min(axis=0))
    np.testing.assert_array_equal(out["best_step"],
                                  np.array([2, 4, 5])[out["trace"].argmin(axis=0)])
    for r in sorted({0, R // 2, R - 1}):
        assert out["best_h"][r] == orc.h_model_fixed(rp, cl, Jv, q, out["best_colour"][r])


# degrees for 1, 4 and 16 lanes per row; sizes for one and several workgroups
@pytest.mark.parametrize("degree", [2, 20, 60])
@pytest.mark.parametrize("n,R", [(70, 1), (257, 3), (6001, 2)])
def test_sparse_whole_number_sums(oim, degree, n, R):
    g = synth.gnp_avg_degree(n, degree, seed=degree + n)
    J = -g.w.copy()
    rows = np.repeat(np.arange(n), np.diff(g.row_ptr))
    J[(rows + g.col) % 5 == 0] = 0.0  # stored zeros are no conflicts
    col = np.random.default_rng(n).integers(-1, 3, (R, n)).astype(np.int8)
    with oim.Problem.from_csr(n, g.row_ptr, g.col, J) as prob:
        cut = oim.oim_cut(prob.handle, _t(col)).cpu().numpy()
        conf = oim.oim_conflicts(prob.handle, _t(col)).cpu().numpy()
    up = rows < g.col
    for r in range(R):
        same = col[r][rows[up]] == col[r][g.col[up]]
        assert cut[r] == int(-J[up][~same].astype(np.int64).sum())
        assert conf[r] == int((same & (J[up] != 0)).sum())


# one round of 1024 row blocks holds 65536 rows; colours and phases are staged
# in LDS up to about 28000 oscillators
@pytest.mark.parametrize("n", [1, 63, 64, 65, 3000, 65536, 66000])
def test_sparse_real_sums(oim, orc, n):
    if n == 1:
        g = synth.csr_from_edges(1, [], [], [])
    else:
        g = synth.gnp_avg_degree(n, 7.0, seed=n) if n < 4000 else synth.torus(n // 60, 60, seed=2)
    n = g.n
    rng = np.random.default_rng(n)
    ei, ej, _ = g.upper_edges()
    w = (rng.standard_normal(ei.size) * np.exp(rng.uniform(-6, 3, ei.size))).astype(np.float32)
    g = synth.csr_from_edges(n, ei, ej, w)
    J = (-g.w).astype(np.float32)
    R = 2
    th = synth.theta0(R, n, seed=4)
    with oim.Problem.from_csr(n, g.row_ptr, g.col, J) as prob:
        col = rng.integers(0, 2, (R, n)).astype(np.int8)
        hm, h6 = oim.oim_energy(prob.handle, 2, _t(th), _t(col))
        h3, _ = oim.oim_energy(prob.handle, 3, None, _t(col))
        cutf = oim.oim_cut(prob.handle, _t(col), exact=False).cpu().numpy()
    for r in range(R):
        assert hm[r].item() == orc.h_model_fixed(g.row_ptr, g.col, J, 2, col[r])
        assert h3[r].item() == orc.h_model_fixed(g.row_ptr, g.col, J, 3, col[r])
        assert cutf[r] == orc.cut_fixed(g.row_ptr, g.col, J, col[r])
        want = orc.h_eq6_fixed(g.row_ptr, g.col, J, th[r].astype(np.float64))
        assert abs(h6[r].item() - want) <= 2.0**-51 * np.abs(J).astype(np.float64).sum() / 2
