"""Timed workloads of the simulated oscillator Ising/Potts machine.

Each case is a piece of work that a program using the package does through its
public entry points: whole solves on the three loop forms (LDS-resident,
stepwise, dense) with their readouts, the scoring of stored phases, and a
training step of the annealing schedule.  `listed()` holds named ones, `draw`
makes more of the same ranges, `prepare` builds what a program holds before the
call, `run` makes one pass, `exact` evaluates the same pass in 64 bits with
plain numpy / torch, and `work` counts what a pass cannot do without.

Keys of a case:
  kind     "sparse" (one graph, loop form chosen by the library), "batch" (many
           small graphs in one launch), "dense" (all-to-all coupling), "score"
           (readouts of given phases), "adjoint" (schedule gradient)
  graph    "gnp", "torus" (rows x cols), "planted" (q-colourable), "sk" (dense)
  n, degree, rows, cols, graphs, n_lo   sizes (graphs: instances of a batch with
           n_lo .. n oscillators each)
  weights  "unit" (+1), "pm1" (+-1) or "real" edge weights w; J = -w
  R, q, steps, readout, sweep (a schedule of its own per replica), prec, ckpt
"""
import math

import numpy as np
import torch

import paper_2505_22631_amd as oim
from paper_2505_22631_amd.autograd import relaxed_cut

DT = float(np.float32(0.01))
TWO_PI = 2.0 * math.pi


def listed():
    return [
        # the smallest call: a first solve of a small graph with two replicas,
        # as a service answering single requests makes it (latency)
        dict(name="first-solve", kind="sparse", graph="gnp", n=200, degree=10.0, weights="unit",
             R=2, q=2, steps=50, readout=0, sweep=False),
        # plain max-cut on an 800-node graph, one replica, read out often
        # enough to follow the best cut: the loop of one launch per replica
        dict(name="maxcut-one", kind="sparse", graph="gnp", n=800, degree=48.0, weights="unit",
             R=1, q=2, steps=1000, readout=10, sweep=False),
        # the same graph with a batch of replicas in one launch
        dict(name="maxcut-batched", kind="sparse", graph="gnp", n=800, degree=48.0,
             weights="unit", R=256, q=2, steps=1000, readout=10, sweep=False),
        # sparse max-cut at scale, the headline graph and replica count
        dict(name="torus-batched", kind="sparse", graph="torus", rows=100, cols=100,
             weights="pm1", R=256, q=2, steps=2000, readout=100, sweep=False),
        # a sweep of annealing schedules, one per replica, on a graph with
        # real weights and an odd number of oscillators
        dict(name="schedule-sweep", kind="sparse", graph="gnp", n=1999, degree=10.0,
             weights="real", R=96, q=2, steps=100, readout=25, sweep=True),
        # Potts colouring of many graphs of mixed sizes in one launch
        dict(name="colouring-batch", kind="batch", graph="planted", graphs=256, n_lo=100, n=600,
             degree=4.6, weights="unit", R=8, q=3, steps=1000, readout=50, sweep=False),
        # a graph beyond one workgroup's LDS: state in device memory
        dict(name="large-torus", kind="sparse", graph="torus", rows=200, cols=300, weights="pm1",
             R=64, q=2, steps=100, readout=50, sweep=False),
        # the all-to-all coupling at the benchmark's size
        dict(name="sk-large", kind="dense", graph="sk", n=4096, R=512, q=2, steps=100, readout=0,
             prec="bf16x3"),
        # an all-to-all problem of ordinary size with few replicas, followed
        # through its readouts and scored at the end
        dict(name="sk-ordinary", kind="dense", graph="sk", n=777, R=24, q=2, steps=100,
             readout=25, prec="bf16x3"),
        # the same kind of problem in full FP32, the paper's precision
        dict(name="sk-fp32", kind="dense", graph="sk", n=2000, R=128, q=2, steps=50, readout=25,
             prec="fp32"),
        # scoring of stored phases: thresholding, cut, conflicts and energies
        dict(name="score-torus", kind="score", graph="torus", rows=100, cols=100, weights="real",
             R=64, q=2),
        # one training step of the annealing schedule over a batch of graphs
        dict(name="train-schedule", kind="adjoint", graph="gnp", graphs=128, n_lo=2000, n=2000,
             degree=10.0, weights="pm1", R=1, q=2, steps=256, ckpt=64),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the same ranges: sizes spread over their logarithm,
    odd ones among them, replicas and steps bounded by the listed cases'."""
    kind = rng.choice(["sparse", "sparse", "batch", "large", "dense", "dense", "score", "adjoint"])
    if kind == "sparse":
        n = _log_int(rng, 64, 10000)
        if rng.random() < 0.3 and n >= 400:
            rows = _log_int(rng, 16, 100)
            c = dict(kind=kind, graph="torus", rows=rows, cols=max(5, min(100, n // rows)))
        else:
            c = dict(kind=kind, graph="gnp", n=n, degree=float(rng.randint(3, 12 if n > 2000 else
                                                                          min(48, n // 4))))
        c.update(weights=rng.choice(["unit", "pm1", "real"]), R=_log_int(rng, 1, 256),
                 q=rng.choice([2, 2, 3, 4]), steps=_log_int(rng, 50, 1000),
                 readout=rng.choice([0, 10, 50, 100]), sweep=rng.random() < 0.25)
    elif kind == "batch":
        hi = rng.randint(150, 1200)
        c = dict(kind=kind, graph="planted", graphs=_log_int(rng, 8, 256),
                 n_lo=rng.randint(40, hi), n=hi, degree=round(rng.uniform(3.5, 6.0), 1),
                 weights="unit", R=_log_int(rng, 1, 8), q=rng.choice([3, 3, 4]),
                 steps=_log_int(rng, 50, 500), readout=rng.choice([0, 25, 50]), sweep=False)
    elif kind == "large":
        c = dict(kind="sparse")
        if rng.random() < 0.5:
            c.update(graph="torus", rows=rng.randint(150, 250), cols=rng.randint(150, 250))
        else:
            c.update(graph="gnp", n=_log_int(rng, 20000, 60000), degree=float(rng.randint(3, 8)))
        c.update(weights=rng.choice(["unit", "pm1", "real"]), R=_log_int(rng, 1, 64),
                 q=rng.choice([2, 2, 3]), steps=_log_int(rng, 30, 100),
                 readout=rng.choice([0, 25, 50]), sweep=rng.random() < 0.2)
    elif kind == "dense":
        c = dict(kind=kind, graph="sk", n=_log_int(rng, 96, 4096), R=_log_int(rng, 1, 512),
                 q=rng.choice([2, 2, 2, 3]), steps=_log_int(rng, 20, 100),
                 prec=rng.choice(["bf16x3", "bf16x3", "fp32"]))
        # in-run readouts where a program follows the best state: up to the
        # sizes at which the listed cases do
        c["readout"] = rng.choice([0, 10, 25]) if c["n"] * c["R"] <= 2000 * 128 else 0
    elif kind == "score":
        c = dict(kind=kind, graph="gnp", n=_log_int(rng, 200, 20000),
                 degree=float(rng.randint(3, 24)), weights=rng.choice(["unit", "pm1", "real"]),
                 R=_log_int(rng, 1, 64), q=rng.choice([2, 2, 3]))
    else:
        n = _log_int(rng, 200, 2000)
        c = dict(kind=kind, graph="gnp", graphs=_log_int(rng, 1, 128), n_lo=n - n // 5, n=n,
                 degree=float(rng.randint(4, 10)), weights=rng.choice(["unit", "pm1", "real"]),
                 R=rng.choice([1, 1, 2]), q=rng.choice([2, 2, 3]), steps=_log_int(rng, 64, 256),
                 ckpt=rng.choice([16, 32, 64]))
    return c


# ------------------------------------------------------------ host inputs ----
def _csr(n, a, b, w):
    """Symmetric CSR of distinct undirected edges (a, b) of weight w."""
    rows, cols, vals = np.concatenate([a, b]), np.concatenate([b, a]), np.concatenate([w, w])
    order = np.argsort(rows * n + cols)
    row_ptr = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(rows, minlength=n), out=row_ptr[1:])
    return row_ptr, cols[order].astype(np.int32), vals[order].astype(np.float32)


def _graph(case, rng):
    """(n, row_ptr, col, w, instance offsets) of a sparse case."""
    off = None
    if case["graph"] == "torus":
        rows, cols = case["rows"], case["cols"]
        n = rows * cols
        r, c = np.meshgrid(np.arange(rows), np.arange(cols), indexing="ij")
        v = (cols * r + c).ravel()
        a = np.concatenate([v, v])
        b = np.concatenate([(cols * r + (c + 1) % cols).ravel(), (cols * ((r + 1) % rows) + c).ravel()])
    else:
        graphs = case.get("graphs", 1)
        lo, hi = case.get("n_lo", case["n"]), case["n"]
        # a case's sizes are its own; the graphs come from the seed
        sizes = np.random.default_rng([graphs, lo, hi]).integers(lo, hi + 1, size=graphs)
        off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        n = int(off[-1])
        # a share of the pairs is lost to loops, repeats and (planted) equal classes
        q = case["q"] if case["graph"] == "planted" else 0
        share = 1.0 - 1.0 / q if q else 1.0
        m = np.round(case["degree"] * sizes / 2.0 / share).astype(np.int64)
        of = np.repeat(np.arange(graphs), m)
        a = off[of] + (rng.random(of.size) * sizes[of]).astype(np.int64)
        b = off[of] + (rng.random(of.size) * sizes[of]).astype(np.int64)
        keep = a != b
        if q:
            colour = rng.integers(0, q, size=n)
            keep &= colour[a] != colour[b]
        key = np.unique(np.minimum(a, b)[keep] * n + np.maximum(a, b)[keep])
        a, b = key // n, key % n
    weights = case["weights"]
    if weights == "unit":
        w = np.ones(a.size)
    elif weights == "pm1":
        w = np.where(rng.random(a.size) < 0.5, 1.0, -1.0)
    else:
        w = rng.standard_normal(a.size)
    row_ptr, col, w = _csr(n, a, b, w.astype(np.float32))
    return n, row_ptr, col, w, off


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _sk(n, seed):
    """Sherrington-Kirkpatrick couplings N(0, 1/n), symmetric, zero diagonal."""
    g = torch.Generator(device=_device()).manual_seed(seed)
    J = torch.randn((n, n), generator=g, device=_device()) / math.sqrt(n)
    J = torch.triu(J, diagonal=1)
    return (J + J.T).cpu().numpy()


def _host(case, seed):
    """Everything of a case as host arrays, from the seed alone."""
    rng = np.random.default_rng([seed, 17])
    h = {}
    if case["kind"] == "dense":
        n = case["n"]
        h["J"] = _sk(n, seed)
        row_sum = float(np.abs(h["J"]).sum(axis=1).max())
    else:
        n, h["row_ptr"], h["col"], w, h["off"] = _graph(case, rng)
        h["J"] = -w  # max-cut and colouring couplings (the sign of "pm1" and "real" is symmetric)
        rows = np.repeat(np.arange(n), np.diff(h["row_ptr"]))
        row_sum = float(np.bincount(rows, np.abs(w), minlength=n).max()) if w.size else 1.0
    h["n"] = n
    R, q, steps = case["R"], case["q"], case.get("steps", 0)
    h["theta0"] = (rng.random((R, n)) * TWO_PI).astype(np.float32).clip(0, np.float32(6.283185))
    h["seeds"] = rng.integers(0, 2**62, size=R).astype(np.uint64)
    if steps:
        # linear K ramp and (q = 2) triangular or (q > 2) ramped Ks, as multiples
        # of the stability bounds 0.5 / (dt max row sum) and 0.5 / (dt q); the
        # all-to-all coupling's row sum grows with sqrt(n), its norm does not
        mult = {"dense": 32.0 * math.sqrt(n / 4096.0), "batch": 4.0, "adjoint": 1.0}.get(
            case["kind"], 8.0 if case.get("degree", 0) > 30 else 2.0)
        kmax = mult * 0.5 / (DT * max(row_sum, 1e-6))
        ksmax = (0.03 if case["kind"] == "dense" else 0.5) * 0.5 / (DT * q)
        t = np.arange(steps) / max(steps - 1, 1)
        K, Ks = kmax * t, ksmax * (1.0 - np.abs(2.0 * ((5.0 * t) % 1.0) - 1.0))
        if q > 2:
            Ks = ksmax * t
        sg = np.full(steps, 0.1)
        if case.get("sweep"):
            K = K[None] * rng.uniform(0.5, 2.0, (R, 1))
            Ks = Ks[None] * rng.uniform(0.25, 2.0, (R, 1))
            sg = np.repeat(rng.uniform(0.05, 0.2, (R, 1)), steps, axis=1)
        h["K"], h["Ks"], h["sigma"] = (np.ascontiguousarray(x, np.float32) for x in (K, Ks, sg))
    return h


# --------------------------------------------------------------- prepare ----
def prepare(case, seed):
    h = _host(case, seed)
    dev = torch.device("cuda")
    s = {"case": case}
    if case["kind"] == "dense":
        s["problem"] = oim.Problem.from_dense(h["J"])
    elif h["off"] is not None and h["off"].size > 2:
        s["problem"] = oim.Problem.from_csr_blocks(h["n"], h["row_ptr"], h["col"], h["J"], h["off"])
    else:
        s["problem"] = oim.Problem.from_csr(h["n"], h["row_ptr"], h["col"], h["J"])
    for k in ("theta0", "seeds", "K", "Ks", "sigma"):
        if k in h:
            s[k] = torch.from_numpy(h[k]).to(dev)
    s["theta"] = s["theta0"].clone()
    if case["kind"] == "adjoint":
        for k in ("K", "Ks", "sigma"):
            s[k].requires_grad_(True)
    return s


# ------------------------------------------------------------------- run ----
def run(state):
    c, problem, q = state["case"], state["problem"], state["case"]["q"]
    if c["kind"] == "adjoint":
        K, Ks, sigma = state["K"], state["Ks"], state["sigma"]
        K.grad = Ks.grad = sigma.grad = None
        loss = relaxed_cut(problem, state["theta0"], K, Ks, sigma, state["seeds"], q=q, dt=DT,
                           checkpoint_every=c["ckpt"])
        loss.backward()
        return {"loss": loss.detach(), "gK": K.grad, "gKs": Ks.grad, "gsigma": sigma.grad}
    if c["kind"] == "score":
        theta = state["theta"]
        colour = oim.oim_round(q, theta)
        h_model, h_eq6 = oim.oim_energy(problem.handle, q, theta, colour)
        return {"colour": colour, "conflicts": oim.oim_conflicts(problem.handle, colour),
                "cut": oim.oim_cut(problem.handle, colour, exact=c["weights"] != "real"),
                "h_model": h_model, "h_eq6": h_eq6}
    theta = state["theta"]
    theta.copy_(state["theta0"])
    flags = oim.OIM_PREC_BF16X3 if c.get("prec") == "bf16x3" else 0
    out = oim.run(problem, theta, state["K"], state["Ks"], state["sigma"], state["seeds"], q=q,
                  dt=DT, readout_every=c["readout"], flags=flags, want_best=True)
    out["theta"] = theta
    out["colour"] = oim.oim_round(q, theta)
    if c["kind"] == "batch":
        out["conflicts"] = oim.oim_conflicts(problem.handle, out["colour"])
    elif c["kind"] == "dense":
        out["h_model"] = oim.oim_energy(problem.handle, q, colour=out["colour"])[0]
    else:
        out["cut"] = oim.oim_cut(problem.handle, out["colour"], exact=c["weights"] != "real")
    return out


# ----------------------------------------------------------------- exact ----
def _mulhilo(m, a):
    p = m * a  # the wrapped 64-bit product has the right bits
    return (p >> 32) & 0xffffffff, p & 0xffffffff


def _normals(seeds, quad, inst, n_of_quad, t):
    """Standard normals [R][n] of step t: Philox4x32-10 on counter (quad, t,
    instance, 0) and Box-Muller on 24-bit uniforms, in 64 bits."""
    k0, k1 = (seeds & 0xffffffff)[:, None], ((seeds >> 32) & 0xffffffff)[:, None]
    shape = (seeds.shape[0], quad.shape[0])
    x = quad[None].expand(shape)
    y = torch.full(shape, t, dtype=torch.int64, device=quad.device)
    z = inst[None].expand(shape)
    w = torch.zeros(shape, dtype=torch.int64, device=quad.device)
    for _ in range(10):
        h0, l0 = _mulhilo(0xD2511F53, x)
        h1, l1 = _mulhilo(0xCD9E8D57, z)
        x, y, z, w = h1 ^ y ^ k0, l1, h0 ^ w ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & 0xffffffff, (k1 + 0xBB67AE85) & 0xffffffff
    out = []
    for a, b in ((x, y), (z, w)):
        u1 = ((a >> 8) + 1).double() / 2**24
        u2 = (b >> 8).double() / 2**24
        rho = torch.sqrt(-2.0 * torch.log(u1))
        out += [rho * torch.cos(TWO_PI * u2), rho * torch.sin(TWO_PI * u2)]
    z4 = torch.stack(out, dim=2).reshape(shape[0], -1)
    return z4[:, n_of_quad]


class _Exact:
    """The fixed-noise trajectory of a case in 64 bits."""

    def __init__(self, case, h):
        d = _device()
        self.q, self.n, self.h = case["q"], h["n"], h
        off = h.get("off")
        off = np.array([0, self.n]) if off is None else np.asarray(off, np.int64)
        i = np.arange(self.n)
        inst = np.searchsorted(off, i, side="right") - 1
        local = i - off[inst]
        nq = (np.diff(off) + 3) // 4
        q0 = np.concatenate([[0], np.cumsum(nq)])
        put = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(d)  # noqa: E731
        self.quad = put(np.concatenate([np.arange(k) for k in nq]))
        self.inst = put(np.repeat(np.arange(off.size - 1), nq))
        self.n_of_quad = put(4 * (q0[inst] + local // 4) + local % 4)
        self.seeds = put(h["seeds"].astype(np.int64))
        self.theta = put(h["theta0"].astype(np.float64))
        if case["kind"] == "dense":
            self.J = put(h["J"].astype(np.float64))
            self.rows = None
        else:
            self.rows = put(np.repeat(i, np.diff(h["row_ptr"])))
            self.cols = put(h["col"].astype(np.int64))
            self.J = put(h["J"].astype(np.float64))

    def coupling(self, theta):
        """sum_j J_ij sin(theta_i - theta_j)."""
        s, c = torch.sin(theta), torch.cos(theta)
        if self.rows is None:
            return s * (c @ self.J) - c * (s @ self.J)
        d = self.J * torch.sin(theta[:, self.rows] - theta[:, self.cols])
        return torch.zeros_like(theta).index_add(1, self.rows, d)

    def step(self, theta, t, K, Ks, sigma):
        xi = _normals(self.seeds, self.quad, self.inst, self.n_of_quad, t)
        f = -K * self.coupling(theta) - Ks * torch.sin(self.q * theta)
        return theta + DT * f + sigma * math.sqrt(DT) * xi


def _hamiltonian(e, colour, q):
    """Eq. 1 (q = 2) or Eq. 2 (q > 2) of colours [R][n]."""
    up = e.rows < e.cols
    same = colour[:, e.rows[up]] == colour[:, e.cols[up]]
    term = torch.where(same, 1.0, -1.0 if q == 2 else 0.0).double()
    return -(term * e.J[up]).sum(dim=1)


def exact(case, seed):
    steps = case.get("steps", 0)
    if case["kind"] not in ("score", "adjoint") and steps > 100:
        return None  # over a long run FP32 and FP64 trajectories part
    h = _host(case, seed)
    e = _Exact(case, h)
    q, theta = case["q"], e.theta
    if case["kind"] == "score":
        scale = np.float32(q / TWO_PI)
        th = h["theta0"]
        # the FP32 decision of the thresholding, fused multiply-add in 64 bits
        colour = np.floor((th.astype(np.float64) * np.float64(scale) + 0.5).astype(np.float32))
        colour = torch.from_numpy(colour.astype(np.int64) % q).to(theta.device)
        up = e.rows < e.cols
        i, j, w = e.rows[up], e.cols[up], -e.J[up]
        cut = ((colour[:, i] != colour[:, j]).double() * w).sum(dim=1)
        conflicts = (colour[:, i] == colour[:, j]).sum(dim=1)
        return {"colour": colour, "conflicts": conflicts,
                "cut": cut if case["weights"] == "real" else None,
                "h_model": _hamiltonian(e, colour, q),
                "h_eq6": (torch.cos(theta[:, i] - theta[:, j]) * w).sum(dim=1)}
    sched = [torch.from_numpy(h[k].astype(np.float64)).to(theta.device)
             for k in ("K", "Ks", "sigma")]
    if case["kind"] == "adjoint":
        for x in sched:
            x.requires_grad_(True)
        # checkpointed every few steps to bound the stored trajectory
        from torch.utils.checkpoint import checkpoint

        def span(th, t0, t1, K, Ks, sigma):
            for t in range(t0, t1):
                th = e.step(th, t, K[t], Ks[t], sigma[t])
            return th

        for t0 in range(0, steps, 16):
            theta = checkpoint(span, theta, t0, min(steps, t0 + 16), *sched, use_reentrant=False)
        up = e.rows < e.cols
        loss = (-e.J[up] * (1.0 - torch.cos(theta[:, e.rows[up]] - theta[:, e.cols[up]])) / 2).sum()
        loss.backward()
        return {"loss": loss.detach(), "gK": sched[0].grad, "gKs": sched[1].grad,
                "gsigma": sched[2].grad}
    K, Ks, sigma = (x[:, :, None] if x.dim() == 2 else x[None, :, None] for x in sched)
    for t in range(steps):
        theta = e.step(theta, t, K[:, t], Ks[:, t], sigma[:, t])
    # thresholded outputs follow from the phases; near a threshold 32 and 64
    # bits decide differently, so only the phases have a value here
    return {"theta": torch.remainder(theta, TWO_PI), "colour": None, "trace": None,
            "best_h": None, "best_step": None, "best_colour": None, "cut": None,
            "conflicts": None, "h_model": None}


# ------------------------------------------------------------------ work ----
def work(case):
    """Bytes: phases, schedules, seeds and coupling read once, results written
    once.  Operations: a multiply-add each for sine and cosine of every stored
    coupling (four operations), and about forty per oscillator and step for
    noise, injection locking and update; a gradient step is three passes."""
    R, q, steps = case["R"], case["q"], case.get("steps", 0)
    if case["kind"] == "dense":
        n = case["n"]
        nnz, coupling = n * n, 4 * n * n
    else:
        if case["graph"] == "torus":
            n = case["rows"] * case["cols"]
            nnz = 4 * n
        else:
            g = case.get("graphs", 1)
            n = g * (case.get("n_lo", case["n"]) + case["n"]) // 2
            nnz = int(case["degree"] * n)
        coupling = 8 * nnz + 8 * n
    bytes_ = coupling + 8 * R
    if case["kind"] == "score":
        # theta in, colours and five sums per replica out
        return {"bytes": bytes_ + 5 * R * n + 40 * R, "flops": R * nnz / 2 * 10}
    rows = R if case.get("sweep") else 1
    bytes_ += 12 * rows * steps
    flops = float(R) * steps * (4.0 * nnz + 40.0 * n)
    if case["kind"] == "adjoint":
        return {"bytes": bytes_ + 4 * R * n + 12 * steps, "flops": 3.0 * flops}
    nr = -(-steps // case["readout"]) if case["readout"] else 0
    return {"bytes": bytes_ + (8 + 1) * R * n + 8 * R * nr + (R * n if nr else 0), "flops": flops}
