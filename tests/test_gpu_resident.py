"""Launch shapes of the LDS-resident loop that keep a row's first entries in
registers (one slice per wave group) against a shape that reads all of them
every step, bit for bit, at row lengths around the resident part and its
batches: 32 / 16 / 8 entries per row with unit weights for 1 / 2 / 4 rows per
lane, half of that with general ones, read in two batches."""
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


def _circulant(n, degree, weights):
    """n oscillators of `degree` neighbours each, the last third of the rows
    shorter by two."""
    i = np.arange(n)
    ei, ej = [], []
    for k in range(1, degree // 2 + 1):
        keep = i < (n if k < degree // 2 else 2 * n // 3)
        ei.append(i[keep])
        ej.append((i[keep] + k) % n)
    ei = np.concatenate(ei) if ei else np.zeros(0, np.int64)
    ej = np.concatenate(ej) if ej else np.zeros(0, np.int64)
    rng = np.random.default_rng(degree)
    w = np.ones(ei.size) if weights == "unit" else rng.standard_normal(ei.size)
    return synth.csr_from_edges(n, ei, ej, w)


@pytest.mark.parametrize("degree", [0, 2, 4, 8, 10, 16, 18, 32, 34, 50])
@pytest.mark.parametrize("weights", ["unit", "real"])
@pytest.mark.parametrize("n,q,steps", [(101, 2, 7), (254, 5, 8)])
def test_resident_rows_same_bits(oim, degree, weights, n, q, steps):
    import torch
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    g = _circulant(n, degree, weights)
    R = 3
    with oim.Problem.from_csr(g.n, g.row_ptr, g.col, (-g.w).astype(np.float32)) as prob:
        K, Ks, sg = ramp_schedule(max(prob.info["max_abs_row_sum"], 1.0), q, steps)
        th0 = synth.theta0(R, n, seed=1)
        ref = None
        for shape in ((64, 2, 4), (256, 1, 4), (256, 1, 2), (256, 1, 1), (1024, 1, 1)):
            oim.oim_set_tuning(prob.handle, q, *shape)
            th = t(th0)
            ph = oim.oim_phase_from_theta(th)
            out = oim.run(prob, th, t(K), t(Ks), t(sg), t(synth.seeds(R, 4)), q=q, dt=DT,
                          readout_every=3, phase=ph, want_best=True)
            got = [ph.cpu().numpy()] + [v.cpu().numpy() for v in out.values()]
            if ref is None:
                ref = got
            for a, b in zip(got, ref):
                np.testing.assert_array_equal(a, b, err_msg=f"shape {shape}")


@pytest.mark.parametrize("weights", ["unit", "real"])
@pytest.mark.parametrize("sizes,R,shapes", [
    ([1000], 2, ((1024, 1, 1), (512, 1, 2))),          # every wave holds rows
    ([770, 30, 255, 256, 257, 1], 2, ((1024, 1, 1), (512, 1, 2), (1024, 1, 2))),
    ([1700], 2, ((1024, 1, 2),)),                      # two idle waves for seven slices
    ([2048], 1, ((1024, 1, 2),)),
    ([510], 300, ((512, 1, 1), (256, 1, 2))),          # two workgroups per CU
    ([4095], 2, ((1024, 1, 4),)),
    ([3, 900, 64, 65], 2, ((256, 1, 4), (512, 1, 4), (512, 1, 2))),
    ([250], 600, ((256, 1, 1), (256, 1, 2), (512, 1, 1))),
])
def test_shared_noise_same_bits(oim, sizes, R, weights, shapes):
    """Split-row shapes whose noise is drawn by idle or added waves, or by one
    wave of each slice, against whole quads, which draw their own."""
    import torch
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    gs = [_circulant(n, 6 if n > 6 else 0, weights) for n in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)])
    ptr = np.concatenate([[0]] + [g.row_ptr[1:] + sum(h.row_ptr[-1] for h in gs[:k])
                                  for k, g in enumerate(gs)]).astype(np.int64)
    col = np.concatenate([g.col + off[k] for k, g in enumerate(gs)]).astype(np.int32)
    w = np.concatenate([g.w for g in gs])
    q, steps, n = 3, 6, int(off[-1])
    with oim.Problem.from_csr_blocks(n, ptr, col, (-w).astype(np.float32), off) as prob:
        K, Ks, sg = ramp_schedule(max(prob.info["max_abs_row_sum"], 1.0), q, steps)
        th0 = synth.theta0(R, n, seed=2)
        ref = None
        for shape in ((512, 4, 4),) + shapes:
            oim.oim_set_tuning(prob.handle, q, *shape)
            th = t(th0)
            ph = oim.oim_phase_from_theta(th)
            out = oim.run(prob, th, t(K), t(Ks), t(sg), t(synth.seeds(R, 5)), q=q, dt=DT,
                          readout_every=2, phase=ph, want_best=True)
            got = [ph.cpu().numpy()] + [v.cpu().numpy() for v in out.values()]
            if ref is None:
                ref = got
            for a, b in zip(got, ref):
                np.testing.assert_array_equal(a, b, err_msg=f"shape {shape}")
