"""Calls at the edges of what one kernel launch takes: scoring where the staged
copies come near the LDS of a CU, and more workgroups than a launch of
1024-thread ones holds (a grid dimension ends at 2^32 threads)."""
import numpy as np
import pytest

import synth
from _util import DT

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


def _repeat(x, R):
    """[P][..] tiled to R rows on the GPU: row r is x[r % P]."""
    t = _t(x)
    P = x.shape[0]
    return t.repeat(*([-(-R // P)] + [1] * (x.ndim - 1)))[:R].contiguous()


def _same_period(out, P):
    """Every row r of out equals row r % P."""
    R = out.shape[0]
    head = R // P * P
    ref = out[:P].unsqueeze(0)
    assert bool((out[:head].view(-1, P, *out.shape[1:]) == ref).all())
    assert bool((out[head:] == out[:R - head]).all())


def _ring(n, weights, seed=0):
    """Rings of step 1 and 7 on n oscillators."""
    i = np.arange(n)
    ei, ej = np.concatenate([i, i]), np.concatenate([(i + 1) % n, (i + 7) % n])
    rng = np.random.default_rng(seed + n)
    w = np.ones(ei.size) if weights == "unit" else rng.standard_normal(ei.size) * np.exp(
        rng.uniform(-4, 2, ei.size))
    return synth.csr_from_edges(n, ei, ej, w.astype(np.float32))


# phases and colours, phases alone, colours alone: the smallest and largest
# sizes whose copies sit in more than 124 KiB of LDS, and the first beyond
@pytest.mark.parametrize("n,what", [(25293, "both"), (28672, "both"), (28673, "both"),
                                    (31617, "phases"), (35840, "phases"), (35841, "phases"),
                                    (126465, "cut"), (143360, "cut"), (143361, "cut")])
def test_scoring_near_the_lds_limit(oim, orc, n, what):
    g = _ring(n, "real")
    J = (-g.w).astype(np.float32)
    th = synth.theta0(1, n, seed=n)
    col = np.random.default_rng(n).integers(0, 2, (1, n)).astype(np.int8)
    with oim.Problem.from_csr(n, g.row_ptr, g.col, J) as prob:
        if what == "cut":
            cut = oim.oim_cut(prob.handle, _t(col), exact=False)
            assert cut[0].item() == orc.cut_fixed(g.row_ptr, g.col, J, col[0])
            return
        hm, h6 = oim.oim_energy(prob.handle, 2, _t(th), _t(col) if what == "both" else None)
        if hm is not None:
            assert hm[0].item() == orc.h_model_fixed(g.row_ptr, g.col, J, 2, col[0])
        want = orc.h_eq6_fixed(g.row_ptr, g.col, J, th[0].astype(np.float64))
        assert abs(h6[0].item() - want) <= 2.0**-51 * np.abs(J).astype(np.float64).sum() / 2


@pytest.mark.parametrize("form", ["sparse", "dense"])
def test_scoring_of_many_replicas(oim, orc, form):
    # 2^22 workgroups of 1024 threads and more
    n, P = 9, 50
    R = (1 << 22) + 3 if form == "sparse" else (1 << 24) + 5
    g = _ring(n, "real")
    J = (-g.w).astype(np.float32)
    rng = np.random.default_rng(3)
    col = rng.integers(0, 2, (P, n)).astype(np.int8)
    th = synth.theta0(P, n, seed=4)
    if form == "sparse":
        prob = oim.Problem.from_csr(n, g.row_ptr, g.col, J)
    else:
        Jd = np.zeros((n, n), np.float32)
        Jd[np.repeat(np.arange(n), np.diff(g.row_ptr)), g.col] = J
        prob = oim.Problem.from_dense(Jd)
    with prob:
        dcol, dth = _repeat(col, R), _repeat(th, R)
        hm, h6 = oim.oim_energy(prob.handle, 2, dth, dcol)
        cut = oim.oim_cut(prob.handle, dcol, exact=False)
        conf = oim.oim_conflicts(prob.handle, dcol)
        for out in (hm, h6, cut, conf):
            _same_period(out, P)
        bound = 2.0**-51 * np.abs(J).astype(np.float64).sum() / 2
        for r in range(P):
            assert hm[r].item() == orc.h_model_fixed(g.row_ptr, g.col, J, 2, col[r])
            assert cut[r].item() == orc.cut_fixed(g.row_ptr, g.col, J, col[r])
            assert conf[r].item() == orc.conflicts(g.row_ptr, g.col, J, col[r])
            want = orc.h_eq6_fixed(g.row_ptr, g.col, J, th[r].astype(np.float64))
            assert abs(h6[r].item() - want) <= bound


def _many_instances(big, count):
    """`count` single oscillators and one ring of `big`, as a batch."""
    g = _ring(big, "real")
    n = count + big
    ptr = np.concatenate([np.zeros(count, np.int64), g.row_ptr])
    off = np.concatenate([np.arange(count + 1), [n]]).astype(np.int32)
    return n, ptr, (g.col + count).astype(np.int32), (-g.w).astype(np.float32), off


def test_run_of_many_workgroups(oim):
    # 1028 replicas of 4097 instances: more than 2^22 workgroups, a default
    # or tuned shape of 1024 threads would not hold
    import torch
    n, ptr, col, J, off = _many_instances(2000, 4096)
    P, R, steps = 4, 1028, 3
    th0, sd = synth.theta0(P, n, seed=5), synth.seeds(P, 6)
    K, Ks, sg = (_t(x) for x in (synth.ramp(0, 2, steps), synth.ramp(0, 3, steps),
                                 synth.const(0.1, steps)))
    with oim.Problem.from_csr_blocks(n, ptr, col, J, off) as prob:
        ref = _t(th0)
        oim.run(prob, ref, K, Ks, sg, _t(sd), q=2, dt=DT)
        for tuned in (None, (1024, 1, 2)):
            if tuned:
                oim.oim_set_tuning(prob.handle, 2, *tuned)
            th = _repeat(th0, R)
            out = oim.run(prob, th, K, Ks, sg, _repeat(sd.view(np.int64), R).view(torch.uint64),
                          q=2, dt=DT, readout_every=2)
            assert torch.equal(th[:P], ref)
            _same_period(th, P)
            _same_period(out["best_h"].view(R, -1), P)


def test_adjoint_of_many_workgroups(oim):
    # the same number of workgroups of 1024 threads
    import torch
    n, ptr, col, J, off = _many_instances(1000, 4096)
    P, R, steps = 4, 1028, 2
    th0, sd = synth.theta0(P, n, seed=7), synth.seeds(P, 8)
    K, Ks, sg = (_t(x) for x in (synth.const(1.0, steps), synth.const(2.0, steps),
                                 synth.const(0.1, steps)))

    def adjoint(prob, th, seeds):
        reps = th.shape[0]
        words = oim.oim_adjoint_checkpoint_words(prob.handle, q=2, R=reps, steps=steps, dt=DT,
                                                 checkpoint_every=steps)
        ckpt = torch.empty(words, dtype=torch.uint32, device="cuda")
        thT = torch.empty_like(th)
        loss = torch.empty(reps * len(off[1:]), dtype=torch.float64, device="cuda")
        oim.oim_adjoint_forward(prob.handle, n, th, K, Ks, sg, seeds, ckpt, q=2, dt=DT,
                                checkpoint_every=steps, theta_T=thT, loss=loss)
        grad = [torch.full((steps,), float("nan"), dtype=torch.float64, device="cuda")
                for _ in range(3)]
        oim.oim_adjoint_backward(prob.handle, reps, K, Ks, sg, seeds, ckpt, *grad, q=2, dt=DT,
                                 checkpoint_every=steps)
        return thT, loss.view(reps, -1), [g.cpu().numpy() for g in grad]

    with oim.Problem.from_csr_blocks(n, ptr, col, J, off) as prob:
        thT1, loss1, g1 = adjoint(prob, _t(th0), _t(sd))
        thT, loss, g = adjoint(prob, _repeat(th0, R),
                               _repeat(sd.view(np.int64), R).view(torch.uint64))
    assert torch.equal(thT[:P], thT1) and torch.equal(loss[:P], loss1)
    _same_period(thT, P)
    _same_period(loss, P)
    for a, b in zip(g, g1):  # R / P times the same partials, summed in FP64
        np.testing.assert_allclose(a, (R // P) * b, rtol=1e-9)
