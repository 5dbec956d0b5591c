"""Every workgroup tile of the dense step in both precisions (OIM_DENSE_TILE
takes one at any size): the same bits, the large tile against the oracle, and
the kernel that ran by name."""
import numpy as np
import pytest

import synth
from _util import DT, ramp_schedule, wrapdiff
from test_gpu_dense import _check_bf16x3, oim  # noqa: F401

pytestmark = pytest.mark.gpu

TILES = ("128x64", "128x32", "64x32", "64x16", "32x16")


def _t(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


# ragged row and replica tiles; one row tile, several
@pytest.mark.parametrize("q", [2, 3, 5])
@pytest.mark.parametrize("prec", ["bf16x3", "fp32"])
@pytest.mark.parametrize("n,R", [(9, 3), (300, 70)])
def test_dense_tiles(oim, orc, monkeypatch, prec, q, n, R):  # noqa: F811
    J = synth.sk_dense(n, seed=6)
    flags = oim.OIM_PREC_BF16X3 if prec == "bf16x3" else oim.OIM_PREC_FP32
    th0, sd = synth.theta0(R, n, seed=3), synth.seeds(R, 5)
    ref = None
    with oim.Problem.from_dense(J) as prob:
        sched = ramp_schedule(prob.info["max_abs_row_sum"], q, 1000, 100)
        K, Ks, sg = (_t(x) for x in sched)
        for tile in TILES + ("",):
            monkeypatch.setenv("OIM_DENSE_TILE", tile)
            th = _t(th0)
            ph = oim.oim_phase_from_theta(th)
            out = oim.run(prob, th, K, Ks, sg, _t(sd), q=q, dt=DT, step0=50, flags=flags, phase=ph,
                          readout_every=40, want_best=True)
            got = [x.cpu().numpy() for x in (th, ph, *out.values())]
            if ref is None:
                ref = got
            for a, b in zip(got, ref):
                np.testing.assert_array_equal(a, b, err_msg=tile)
    pick = [0, R - 1]
    if prec == "bf16x3":
        _check_bf16x3(orc, ref[0][pick], J, th0[pick], *sched, sd[pick], q, step0=50, label=f"q={q}")
    else:
        want = orc.run_dense(J.astype(np.float64), th0[pick], q=q, dt=DT, K=sched[0], Ks=sched[1],
                             sigma=sched[2], seeds=sd[pick], step0=50)
        assert wrapdiff(ref[0][pick], want).max() < 1e-5


@pytest.mark.parametrize("prec", ["bf16x3", "fp32"])
def test_dense_tile_that_ran(oim, monkeypatch, prec):  # noqa: F811
    # large tile: a kernel of its own; others: rows = 16 RB WM, replicas = 16 CB WN
    # of dense_tile_kernel<QM, F32, RB, CB, WM, WN, ..>
    import torch
    flags = oim.OIM_PREC_BF16X3 if prec == "bf16x3" else oim.OIM_PREC_FP32
    with oim.Problem.from_dense(synth.sk_dense(70, seed=2)) as prob:
        K = _t(np.full(1, 0.5, np.float32))
        for tile in TILES:
            monkeypatch.setenv("OIM_DENSE_TILE", tile)
            th, sd = _t(synth.theta0(2, 70, seed=1)), _t(synth.seeds(2, 1))
            with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
                oim.run(prob, th, K, K, K, sd, q=2, dt=DT, flags=flags)
                torch.cuda.synchronize()
            names = {e.name for e in prof.events()
                     if any(k in e.name for k in ("dense_step", "dense_tile_kernel"))}
            assert len(names) == 1, names
            name = names.pop()
            if tile == "128x64":
                assert ("dense_step32_kernel" if prec == "fp32" else "dense_step_kernel") in name
            else:
                args = name[name.index("dense_tile_kernel<") + 18:].split(">")[0].split(", ")
                rb, cb, wm, wn = (int(x) for x in args[2:6])
                assert (args[1] == "true") == (prec == "fp32")
                assert f"{16 * rb * wm}x{16 * cb * wn}" == tile
