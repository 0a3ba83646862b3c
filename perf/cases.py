"""Performance cases of the MI355X conic-QP solver: solves of one problem and
of batches over the instance families of this repository, the cone
projections, and the warm-start network, each through the calls that a
program makes.

listed() names the cases, draw() gives further ones of the same ranges,
prepare() makes what a program holds before the call (a set-up handle, device
tensors, a network with its weights), run() is one call, work() the bytes and
operations that the call cannot do without, and exact() its outputs in plain
64-bit numpy / torch.

Solves run a fixed budget of outer iterations from a cold start, as a
receding-horizon or interactive program uses the solver, and return the
primal-dual point and its objective.  The FP32 bulk mode is not listed: its
own measurements show that it does not pay on this hardware.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2608_09159_amd as pkg

# the warm-start network of the Fisher family (1,000 buyers x 500 goods) and
# of its smaller sibling (300 buyers x 150 goods)
NET_FULL = "51000,512,512,56500"
NET_MID = "4800,512,512,5450"


def listed():
    return [
        # the SOC blocks of the mixed-cone instance, projected in a metric by a
        # caller's own first-order method: latency of one small device call
        {"name": "project_soc_2000x20", "do": "project", "kind": "soc", "dim": 20, "count": 2000},
        # a Fisher-size set of exponential blocks: throughput of the root-finder
        {"name": "project_exp_400000", "do": "project", "kind": "exp", "dim": 3, "count": 400_000},
        # the smallest solve (tiny QP, sparse general Q), host arrays in and out
        {"name": "qp_200", "do": "qp", "n": 200, "m": 100, "power": 0.0, "iters": 256, "memory": "host"},
        # an ordinary sparse QP of odd size
        {"name": "qp_20011", "do": "qp", "n": 20_011, "m": 9_973, "power": 0.8, "iters": 48, "memory": "host"},
        # a large sparse QP with power-law columns, data resident on the device
        {"name": "qp_1200000", "do": "qp", "n": 1_200_000, "m": 600_000, "power": 0.8, "iters": 24,
         "memory": "device"},
        # implementation form: range, one-sided and equality rows, boxes, diagonal Q
        {"name": "bounded_60001", "do": "bounded", "n": 60_001, "m": 30_011, "iters": 192, "memory": "host"},
        # portfolio rebalancing: a batch of factor-model QPs, 50 to 2,000 assets
        {"name": "portfolio_batch_1000", "do": "batch", "count": 1000, "lo": 50, "hi": 2000, "iters": 48,
         "memory": "host"},
        # every cone type with a diagonal plus rank-10 Q (the benchmark's SOCP/QCQP)
        {"name": "mixed_cone_100000", "do": "mixed", "n": 100_000, "m": 50_000, "rank": 10, "iters": 48,
         "memory": "host"},
        # a Fisher market with exponential cones, Q = 0 (1,000 buyers x 500 goods)
        {"name": "fisher_exp_1000x500", "do": "fisher", "buyers": 1000, "goods": 500, "density": 0.1,
         "middle": "row", "iters": 256, "memory": "host"},
        # the paper-shaped Fisher market with 1e4 buyers (fixed-middle blocks)
        {"name": "fisher_fixed_10000x4000", "do": "fisher", "buyers": 10_000, "goods": 4_000, "density": 0.02,
         "middle": "fixed", "iters": 192, "memory": "device"},
        # a learned warm start for one instance: the network's forward pass, batch 1
        {"name": "network_predict_1", "do": "predict", "dims": NET_FULL, "rows": 1},
        # one epoch of training on 4,096 instances, then the weights read out
        {"name": "network_epoch", "do": "epoch", "dims": NET_MID, "rows": 4096, "batch": 256},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["project", "project", "qp", "qp", "qp", "bounded", "batch", "batch", "mixed", "fisher",
                     "fisher", "predict"])
    memory = rng.choice(["host", "device"])
    if do == "project":
        kind = rng.choice(["soc", "soc", "rsoc", "exp", "exp", "pow"])
        dim = rng.randint(3, 120) if kind in ("soc", "rsoc") else 3
        return {"do": do, "kind": kind, "dim": dim, "count": max(64, _log(rng, 500, 1_200_000) // dim)}
    if do == "qp":
        n = _log(rng, 150, 1_100_000)
        return {"do": do, "n": n, "m": int(n * rng.uniform(0.3, 0.7)), "power": rng.choice([0.0, 0.8]),
                "iters": rng.randint(8, 20) if n > 50_000 else rng.randint(16, 48), "memory": memory}
    if do == "bounded":
        n = _log(rng, 500, 300_000)
        return {"do": do, "n": n, "m": int(n * rng.uniform(0.3, 0.7)), "iters": rng.randint(32, 192),
                "memory": memory}
    if do == "batch":
        lo = rng.randint(40, 400)
        return {"do": do, "count": _log(rng, 2, 700), "lo": lo, "hi": lo + rng.randint(0, 1500),
                "iters": rng.randint(16, 48), "memory": "host"}
    if do == "mixed":
        n = _log(rng, 2_000, 100_000)
        return {"do": do, "n": n, "m": n // 2, "rank": rng.choice([0, 1, 5, 10, 17]), "iters": rng.randint(16, 48),
                "memory": memory}
    if do == "fisher":
        buyers = _log(rng, 60, 8_000)
        return {"do": do, "buyers": buyers, "goods": rng.randint(20, 600), "density": round(rng.uniform(0.05, 0.2), 3),
                "middle": rng.choice(["row", "fixed"]), "iters": rng.randint(64, 256), "memory": memory}
    return {"do": do, "dims": "%d,512,512,%d" % (_log(rng, 600, 51_000), _log(rng, 700, 56_500)),
            "rows": _log(rng, 1, 256)}


# ---------------------------------------------------------------------------
# instances (the families of this repository's generators, drawn with numpy)
# ---------------------------------------------------------------------------
class Csr:
    """A CSR matrix as the binding reads it."""

    def __init__(self, rows, cols, vals, shape):
        order = np.argsort(rows * np.int64(shape[1]) + cols, kind="stable")
        self.shape = shape
        self.rows = rows[order]
        self.indices = cols[order].astype(np.int32)
        self.data = np.ascontiguousarray(vals[order], dtype=np.float64)
        self.indptr = np.concatenate([[0], np.cumsum(np.bincount(self.rows, minlength=shape[0]))]).astype(np.int64)
        self.nnz = self.data.size

    def tocsr(self):
        return self


def _problem(n, m, A, b, c, cones, P=None, R=None, D=None, **bounds):
    p = SimpleNamespace(n=n, m=m, A=A, b=b, c=c, cones=cones, P=P, R=R, D=D, row_lo=None, row_hi=None, x_lo=None,
                        x_hi=None)
    vars(p).update(bounds)
    return p


def _pattern(rng, m, n, mean, power, extra=1):
    """(rows, cols) of m rows with extra + Poisson(mean) entries, columns
    uniform or by a power law over a random permutation, duplicates dropped."""
    k = np.minimum(extra + rng.poisson(mean, m), n)
    rows = np.repeat(np.arange(m, dtype=np.int64), k)
    if power > 0:
        top = (n + 1.0) ** (1.0 - power) - 1.0
        j = ((rng.random(rows.size) * top + 1.0) ** (1.0 / (1.0 - power)) - 1.0).astype(np.int64)
        cols = rng.permutation(n)[np.clip(j, 0, n - 1)]
    else:
        cols = rng.integers(0, n, rows.size)
    key = np.sort(rows * n + cols)
    key = key[np.concatenate([[True], key[1:] != key[:-1]])]
    return key // n, key % n


def _matvec(A, x):
    return np.bincount(A.rows, A.data * x[A.indices], minlength=A.shape[0])


def _diag(d):
    i = np.arange(d.size, dtype=np.int64)
    return Csr(i, i, d, (d.size, d.size))


def _qp(case, rng):
    """R+ columns, 10% of them slacks, sparse diagonally dominant Q."""
    n, m = case["n"], case["m"]
    slack = min(n // 10, m)
    rows, cols = _pattern(rng, m, n - slack, 9.0, case["power"])
    vals = np.concatenate([rng.standard_normal(rows.size), np.ones(slack)])
    rows = np.concatenate([rows, rng.permutation(m)[:slack]])
    cols = np.concatenate([cols, n - slack + np.arange(slack)])
    A = Csr(rows, cols, vals, (m, n))
    i, j = rng.integers(0, n, n), rng.integers(0, n, n)
    lo, hi = np.minimum(i, j), np.maximum(i, j)
    key = np.unique((lo * n + hi)[lo != hi])
    i, j = key // n, key % n
    v = 0.1 * rng.standard_normal(i.size)
    d = np.bincount(i, np.abs(v), minlength=n) + np.bincount(j, np.abs(v), minlength=n) + rng.uniform(0.01, 0.1, n)
    k = np.arange(n)
    P = Csr(np.concatenate([i, j, k]), np.concatenate([j, i, k]), np.concatenate([v, v, d]), (n, n))
    b = _matvec(A, np.abs(rng.standard_normal(n)))
    return _problem(n, m, A, b, rng.standard_normal(n), [("nonneg", 0, n, 0.0)], P=P)


def _bounded(case, rng):
    """Boxes (finite, lower only, upper only), R+ and free columns; range,
    equality and one-sided rows around an interior point; diagonal Q."""
    n, m = case["n"], case["m"]
    rows, cols = _pattern(rng, m, n, 5.0, 0.0)
    A = Csr(rows, cols, rng.standard_normal(rows.size), (m, n))
    nb, nf = (3 * n) // 5, n // 10
    x = rng.uniform(0.2, 0.8, n)
    xlo, xhi = np.full(n, -np.inf), np.full(n, np.inf)
    t = rng.integers(0, 3, nb)
    xlo[:nb] = np.where(t != 2, 0.0, -np.inf)
    xhi[:nb] = np.where(t != 1, 1.0, np.inf)
    ax = _matvec(A, x)
    t = rng.integers(0, 4, m)
    gap = rng.uniform(0.05, 1.0, (2, m))
    rlo = np.where(t == 3, ax, np.where(t != 2, ax - gap[0], -np.inf))
    rhi = np.where(t == 3, ax, np.where(t != 1, ax + gap[1], np.inf))
    q = np.where(rng.random(n) < 0.5, rng.uniform(0.0, 1.0, n), 0.0)
    cones = [("box", 0, nb, 0.0), ("free", nb, nf, 0.0), ("nonneg", nb + nf, n - nb - nf, 0.0)]
    return _problem(n, m, A, np.zeros(m), 0.3 * rng.standard_normal(n), cones, P=_diag(q), row_lo=rlo, row_hi=rhi,
                    x_lo=xlo, x_hi=xhi)


def _portfolio(rng, na, k):
    """One factor-model portfolio QP: budget row, ten sector caps."""
    ns = 10
    sector = rng.integers(0, ns, na)
    n, m, a = na + ns, 1 + ns, np.arange(na)
    A = Csr(np.concatenate([np.zeros(na, dtype=np.int64), 1 + sector, 1 + np.arange(ns)]),
            np.concatenate([a, a, na + np.arange(ns)]), np.ones(2 * na + ns), (m, n))
    R = np.zeros((k, n))
    R[:, :na] = 0.1 * rng.standard_normal((k, na))
    return _problem(n, m, A, np.concatenate([[1.0], np.full(ns, 0.3)]),
                    np.concatenate([-rng.normal(0.05, 0.02, na), np.zeros(ns)]), [("nonneg", 0, n, 0.0)],
                    P=_diag(np.concatenate([rng.uniform(0.01, 0.1, na), np.zeros(ns)])), R=R, D=np.eye(k))


def _mixed(case, rng):
    """SOC(20), RSOC(10), EXP, POW and R+ blocks, diagonal plus low-rank Q."""
    n, m, r = case["n"], case["m"], case["rank"]
    cones, x, at = [], np.abs(rng.standard_normal(n)) + 0.1, 0
    for kind, d, count in (("soc", 20, n // 50), ("rsoc", 10, n // 100), ("exp", 3, n // 200), ("pow", 3, n // 200)):
        al = rng.uniform(0.2, 0.8, count) if kind == "pow" else np.zeros(count)
        cones += [(kind, at + d * k, d, float(al[k])) for k in range(count)]
        z = x[at:at + d * count].reshape(count, d)
        v, g = rng.standard_normal((count, d)), np.abs(rng.standard_normal(count)) + 0.1
        if kind == "soc":
            z[:, :-1], z[:, -1] = v[:, :-1], np.linalg.norm(v[:, :-1], axis=1) + g
        elif kind == "rsoc":
            z[:, :-2] = v[:, :-2]
            z[:, -2] = z[:, -1] = np.linalg.norm(v[:, :-2], axis=1) / math.sqrt(2.0) + g
        elif kind == "exp":
            s = np.abs(v[:, 1]) + 0.1
            z[:, 0], z[:, 1], z[:, 2] = s * v[:, 0], s, s * np.exp(v[:, 0]) + g
        else:
            p = rng.uniform(0.5, 2.0, (2, count))
            z[:, 0], z[:, 1] = p
            z[:, 2] = 0.9 * rng.uniform(-1.0, 1.0, count) * p[0] ** al * p[1] ** (1.0 - al)
        at += d * count
    cones.append(("nonneg", at, n - at, 0.0))
    rows, cols = _pattern(rng, m, n, 19.0, 0.0)
    A = Csr(rows, cols, rng.standard_normal(rows.size), (m, n))
    R = rng.standard_normal((r, n)) / math.sqrt(n) if r else None
    return _problem(n, m, A, _matvec(A, x), rng.standard_normal(n), cones, P=_diag(rng.uniform(0.1, 1.0, n)), R=R,
                    D=np.eye(r) if r else None)


def _fisher(case, rng):
    """Quasilinear Fisher market: exponential blocks with the middle
    coordinate fixed by a row ("row") or by the set ("fixed")."""
    nb, ng = case["buyers"], case["goods"]
    fixed = case["middle"] == "fixed"
    # the graph is the case's (one market, changing valuations and budgets)
    graph = np.random.default_rng(nb + ng)
    mask = graph.random((nb, ng)) < case["density"]
    mask[np.arange(nb), graph.integers(0, ng, nb)] = True
    mask[graph.integers(0, nb, ng), np.arange(ng)] = True
    bi, gj = np.nonzero(mask)
    e = bi.size
    if fixed:
        u, w, supply = rng.uniform(0.1, 1.1, e), rng.uniform(0.1, 1.1, nb), np.full(ng, 0.2 * nb)
    else:
        u, w, supply = rng.lognormal(0.0, 1.0, e), rng.lognormal(0.0, 0.5, nb), np.ones(ng)
    k = np.arange(nb)
    n, m, z = e + 4 * nb, ng + (1 if fixed else 2) * nb, e + nb + 3 * k
    rows, cols = [gj, ng + bi, ng + k, ng + k], [np.arange(e), np.arange(e), e + k, z + 2]
    vals = [np.ones(e), -u, -np.ones(nb), np.ones(nb)]
    if not fixed:
        rows, cols, vals = rows + [ng + nb + k], cols + [z + 1], vals + [np.ones(nb)]
    A = Csr(np.concatenate(rows), np.concatenate(cols), np.concatenate(vals), (m, n))
    c = np.zeros(n)
    c[e:e + nb], c[z] = 1.0, -w
    b = np.concatenate([supply, np.zeros(nb), np.zeros(0) if fixed else np.ones(nb)])
    kind = "exp1" if fixed else "exp"
    return _problem(n, m, A, b, c, [("nonneg", 0, e + nb, 0.0)] + [(kind, int(i), 3, 0.0) for i in z])


MAKE = {"qp": _qp, "bounded": _bounded, "mixed": _mixed, "fisher": _fisher}


def _instances(case, seed):
    rng = np.random.default_rng(seed)
    if case["do"] == "batch":
        # the sizes are the case's, the data the seed's
        sizes = np.random.default_rng(case["count"])
        return [_portfolio(rng, int(sizes.integers(case["lo"], case["hi"] + 1)), int(sizes.integers(5, 21)))
                for _ in range(case["count"])]
    return [MAKE[case["do"]](case, rng)]


def _blocks(case, seed):
    """Blocks to project: points around the cone over a few magnitudes, a
    third of the metrics constant on their block."""
    rng = np.random.default_rng(seed)
    count, dim = case["count"], case["dim"]
    r = rng.standard_normal((count, dim)) * 10.0 ** rng.uniform(-1, 1, (count, 1))
    m = 10.0 ** rng.uniform(-0.5, 0.5, (count, dim))
    m[::3] = m[::3, :1]
    return r, m, rng.uniform(0.2, 0.8, count) if case["kind"] == "pow" else None


def _dims(case):
    return [int(d) for d in case["dims"].split(",")]


def _network(case, seed, device):
    """He-normal weights, zero biases, standardised inputs and targets."""
    g = torch.Generator(device=device).manual_seed(seed)
    dims = _dims(case)
    W = [torch.randn((a, b), generator=g, device=device) * math.sqrt(2.0 / a) for a, b in zip(dims, dims[1:])]
    x = torch.randn((case["rows"], dims[0]), generator=g, device=device)
    if case["do"] == "predict":
        return W, x, None
    mix = torch.randn((64, dims[-1]), generator=g, device=device) / 8.0
    return W, x, torch.tanh(x[:, :64]) @ mix


# ---------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------
def prepare(case, seed):
    if case["do"] == "project":
        r, m, al = (None if a is None else torch.from_numpy(a).cuda() for a in _blocks(case, seed))
        return SimpleNamespace(do="project", kind=case["kind"], r=r, m=m, al=al, out=torch.empty_like(r))
    if case["do"] in ("predict", "epoch"):
        W, x, y = _network(case, seed, "cuda")
        batch = case["rows"] if y is None else case["batch"]
        net = pkg.MLP(_dims(case), batch)
        for k, w in enumerate(W):
            net.set_params(k, w.cpu().numpy(), np.zeros(w.shape[1], np.float32))
        return SimpleNamespace(do=case["do"], net=net, x=x, y=y, batch=batch)
    probs = _instances(case, seed)
    opts = dict(max_iter=case["iters"], memory_kind=case["memory"])
    if case["do"] == "batch":
        # autotune off: the lane rule then depends on the instances alone and
        # every run gives the same bits
        return SimpleNamespace(do="batch", handle=pkg.setup_batch(probs, autotune=0, **opts))
    return SimpleNamespace(do="solve", handle=pkg.setup(probs[0], **opts))


def run(state):
    if state.do == "project":
        return pkg.project_cones_noalloc(state.kind, state.r, state.out, state.m, state.al,
                                         stream=torch.cuda.current_stream())
    if state.do == "predict":
        return state.net.forward(state.x)
    if state.do == "epoch":
        losses = [state.net.train_step(state.x[i:i + state.batch], state.y[i:i + state.batch], lr=1e-3)
                  for i in range(0, len(state.x), state.batch)]
        return losses, [state.net.get_params(k) for k in range(state.net.layers)]
    if state.do == "batch":
        res = state.handle.solve()
        return (np.concatenate([r["x"] for r in res]), np.concatenate([r["y"] for r in res]),
                np.array([r["primal_obj"] for r in res]))
    res = state.handle.solve()
    return res["x"], res["y"], np.array([res["primal_obj"]])


# ---------------------------------------------------------------------------
# what a call cannot do without
# ---------------------------------------------------------------------------
def work(case):
    """Inputs read once and outputs written once; for a solve, per outer
    iteration the products with A, its transpose and Q (12 bytes and 2 flops a
    nonzero), the state read and written (three vectors in x, four in y) and
    the same for one inner step (a second one is the data's choice)."""
    if case["do"] == "project":
        c = case["count"] * case["dim"]
        return {"bytes": 24 * c + (8 * case["count"] if case["kind"] == "pow" else 0), "flops": 30 * c}
    if case["do"] in ("predict", "epoch"):
        dims, rows = _dims(case), case["rows"]
        w = sum(a * b + b for a, b in zip(dims, dims[1:]))
        if case["do"] == "predict":
            return {"bytes": 2 * w + 4 * rows * (dims[0] + dims[-1]), "flops": 2 * rows * w}
        # BF16 weights twice, moments and master weights read and written,
        # gradients written, BF16 copy written; the weights read out once
        steps = rows // case["batch"]
        return {"bytes": steps * w * (4 + 24 + 4 + 2) + 4 * rows * (dims[0] + dims[-1]) + 4 * w,
                "flops": 6 * rows * w}
    it, r = case["iters"], 0
    if case["do"] == "qp":
        n, m, a, p = case["n"], case["m"], 10.1 * case["m"], 3.0 * case["n"]
    elif case["do"] == "bounded":
        n, m, a, p = case["n"], case["m"], 6.0 * case["m"], 0.0
    elif case["do"] == "mixed":
        n, m, a, p, r = case["n"], case["m"], 20.0 * case["m"], 0.0, case["rank"]
    elif case["do"] == "batch":
        n = case["count"] * (0.5 * (case["lo"] + case["hi"]) + 10)
        m, a, p, r = 11 * case["count"], 2.0 * n, 0.0, 12.5
    else:
        e = case["buyers"] * case["goods"] * case["density"]
        n, m, a, p = e + 4 * case["buyers"], case["goods"] + 2 * case["buyers"], 2 * e + 3 * case["buyers"], 0.0
    per = 24 * a + 60 * n + 116 * m + 12 * p + 16 * r * n + 92 * n
    return {"bytes": it * per, "flops": it * (4 * a + 2 * p + 4 * r * n + 20 * n)}


# ---------------------------------------------------------------------------
# the outputs in 64 bits
# ---------------------------------------------------------------------------
def _soc(r, m):
    """Metric projections onto {||v|| <= t}, rows (v, t)."""
    v, t, mv, mt = r[:, :-1], r[:, -1], m[:, :-1], m[:, -1]
    out = r.copy()
    zero = np.linalg.norm(mv * v, axis=1) <= -mt * t
    out[zero] = 0.0
    k = np.flatnonzero(~zero & (np.linalg.norm(v, axis=1) > t))
    if not k.size:
        return out
    v, t, mv, mt = v[k], t[k], mv[k], mt[k]
    mr, sg = mv * v, np.where(t < 0, -1.0, 1.0)

    def psi(d):          # with the multiplier mt - sg d
        inv = 1.0 / (mv + (mt - sg * d)[:, None])
        s2, s3 = ((mr * inv) ** 2).sum(1), ((mr * inv) ** 2 * inv).sum(1)
        nv = np.sqrt(s2)
        return d * nv - mt * np.abs(t), nv + d * sg * s3 / nv

    lo, hi = np.zeros(k.size), np.where(sg > 0, mt, np.inf)
    d = np.where(sg > 0, 0.5 * mt, mt)
    for _ in range(200):
        f, df = psi(d)
        lo, hi = np.where(f < 0, d, lo), np.where(f < 0, hi, d)
        dn = d - f / df
        mid = np.where(np.isfinite(hi), 0.5 * (lo + np.where(np.isfinite(hi), hi, 0.0)), 2.0 * d)
        dn = np.where((dn >= lo) & (dn <= hi), dn, mid)
        done = np.abs(dn - d) <= 4e-16 * d
        d = dn
        if done.all():
            break
    v = mr / (mv + (mt - sg * d)[:, None])
    out[k, :-1] = v
    out[k, -1] = np.linalg.norm(v, axis=1)
    return out


def _rsoc(r, m):
    """Rows (v, s, t) with ||v||^2 <= 2 s t: an SOC in the coordinates
    (sqrt(q) v, (s' - t')/sqrt 2, (s' + t')/sqrt 2)."""
    a, b = np.sqrt(m[:, -2]), np.sqrt(m[:, -1])
    q, h = (a * b)[:, None], math.sqrt(0.5)
    s, t = a * r[:, -2], b * r[:, -1]
    z = np.concatenate([np.sqrt(q) * r[:, :-2], ((s - t) * h)[:, None], ((s + t) * h)[:, None]], 1)
    z = _soc(z, np.concatenate([m[:, :-2] / q, np.ones((len(r), 2))], 1))
    return np.concatenate([z[:, :-2] / np.sqrt(q), ((z[:, -1:] + z[:, -2:-1]) * h) / a[:, None],
                           ((z[:, -1:] - z[:, -2:-1]) * h) / b[:, None]], 1)


RATIOS = np.sinh(np.linspace(-7.24, 7.24, 401))


def _exp(r, m):
    """Rows (r, s, t), closure of s exp(r/s) <= t, s > 0: of the rays
    (rho, 1, e^rho) the one that gains most, by a scan and bisection."""
    out = r.copy()
    a, b, c = -m[:, 0] * r[:, 0], -m[:, 1] * r[:, 1], -m[:, 2] * r[:, 2]
    with np.errstate(all="ignore"):
        inside = (r[:, 1] > 0) & (r[:, 1] * np.exp(r[:, 0] / r[:, 1]) <= r[:, 2])
        polar = (a < 0) & (-a * np.exp(b / a) <= math.e * c)
    face = ~inside & ~polar & (r[:, 0] <= 0) & (r[:, 1] <= 0)
    out[polar & ~inside] = 0.0
    out[face, 1], out[face, 2] = 0.0, np.maximum(r[face, 2], 0.0)
    k = np.flatnonzero(~inside & ~polar & ~face)
    for part in np.array_split(k, max(1, k.size // 20000)):
        if part.size:
            out[part] = _exp_ray(r[part], m[part])
    return out


def _exp_ray(r, m):
    r0, s0, t0, mr, ms, mt = (v[:, None] for v in (*r.T, *m.T))

    def gain(rho):       # squared length of the projection onto the ray, scaled free of overflow
        w = np.minimum(1.0, np.exp(-np.abs(rho)) ** (rho > 0))
        x = np.exp(np.minimum(rho, 0.0))
        num = mr * rho * r0 * w + ms * s0 * w + mt * t0 * x
        return np.where(num > 0, num, 0.0) ** 2 / (mr * (rho * w) ** 2 + ms * w * w + mt * x * x)

    def slope(rho):      # sign of the gain's derivative along the ray parameter
        e = np.exp(-np.abs(rho))
        A, B, C = mr * r0 * (rho - 1) + ms * s0, mr * rho * (rho - 1) + ms, rho * s0 - r0
        return np.where(rho > 0, mt * A - mt * t0 * e * B + mr * ms * C * e * e,
                        mt * A * e * e - mt * t0 * e * B + mr * ms * C)

    g, up = gain(RATIOS[None, :]), slope(RATIOS[None, :]) > 0
    j = np.argmax(g, axis=1)
    # the stationary interval next to the best ray (the gain is flat far out);
    # a block with none in the scanned range ends at its best ray
    turn = ~up[:, :-1] & up[:, 1:] & (np.maximum(g[:, :-1], g[:, 1:]) >= 0.9 * g.max(1)[:, None])
    k = np.argmin(np.where(turn, np.abs(np.arange(RATIOS.size - 1) + 0.5 - j[:, None]), np.inf), axis=1)
    some = turn.any(axis=1)
    lo, hi = RATIOS[np.where(some, k, j)][:, None], RATIOS[np.where(some, k + 1, j)][:, None]
    for _ in range(70):
        mid = 0.5 * (lo + hi)
        left = slope(mid) < 0
        lo, hi = np.where(left, mid, lo), np.where(left, hi, mid)
    rho = 0.5 * (lo + hi)
    w, x = np.exp(-np.maximum(rho, 0.0)), np.exp(np.minimum(rho, 0.0))
    eta = (mr * rho * r0 * w + ms * s0 * w + mt * t0 * x) / (mr * (rho * w) ** 2 + ms * w * w + mt * x * x)
    return np.concatenate([eta * w * rho, eta * w, eta * x], 1)


def _pow(r, m, al):
    """Rows (x, y, z) with x^al y^(1-al) >= |z|: bisection on |z|."""
    x, y, z, mx, my, mz = (*r.T, *m.T)
    out = r.copy()
    R = np.abs(z)
    with np.errstate(all="ignore"):
        inside = (x >= 0) & (y >= 0) & (x ** al * y ** (1 - al) >= R)
        p, q = -mx * x, -my * y
        polar = (p >= 0) & (q >= 0) & ((p / al) ** al * (q / (1 - al)) ** (1 - al) >= mz * R)
    lo, hi = np.zeros_like(R), R.copy()

    def at(rho):
        w = rho * (R - rho)

        def root(s, c):
            d = np.sqrt(s * s + 4 * c)
            with np.errstate(all="ignore"):
                return np.where(s >= 0, 0.5 * (s + d), 2 * c / (d - s))
        return root(x, al * mz / mx * w), root(y, (1 - al) * mz / my * w)

    with np.errstate(all="ignore"):
        for _ in range(80):
            mid = 0.5 * (lo + hi)
            u, v = at(mid)
            pos = al * np.log(u) + (1 - al) * np.log(v) - np.log(mid) > 0
            lo, hi = np.where(pos, mid, lo), np.where(pos, hi, mid)
        rho = 0.5 * (lo + hi)
        u, v = at(rho)
    mov = ~inside & ~polar
    out[mov, 0], out[mov, 1], out[mov, 2] = u[mov], v[mov], np.copysign(rho, z)[mov]
    out[polar & ~inside] = 0.0
    return out


def _exp1(r, m, kappa):
    """Rows (z, ., t) onto kappa {(z, 1, t): e^z <= t}."""
    z0, t0, mz, mt = r[:, 0] / kappa, r[:, 2] / kappa, m[:, 0], m[:, 2]
    inside = np.exp(np.minimum(z0, 700.0)) <= t0
    hi = np.minimum(z0, 700.0)
    lo = np.where(t0 > 0, np.minimum(np.log(np.where(t0 > 0, t0, 1.0)), hi), np.minimum(hi, 0.0) - 1.0)

    def f(z):
        return mz * (z - z0) + mt * (np.exp(z) - t0) * np.exp(z)

    for _ in range(60):
        bad = (f(lo) > 0) & (t0 <= 0)
        if not bad.any():
            break
        lo = np.where(bad, lo - 2.0 * (hi - lo), lo)
    for _ in range(75):
        mid = 0.5 * (lo + hi)
        pos = f(mid) > 0
        lo, hi = np.where(pos, lo, mid), np.where(pos, mid, hi)
    z = np.where(inside, z0, 0.5 * (lo + hi))
    t = np.where(inside, t0, np.exp(z))
    return kappa[:, None] * np.stack([z, np.ones_like(z), t], 1)


class _Sets:
    """The cones of a problem, grouped by kind and dimension."""

    def __init__(self, p):
        self.n, self.pos, self.box, groups = p.n, np.zeros(p.n, bool), np.zeros(p.n, bool), {}
        for kind, st, d, al in p.cones:
            if kind in ("free", "nonneg", "box"):
                self.pos[st:st + d] = kind == "nonneg"
                self.box[st:st + d] = kind == "box"
            else:
                groups.setdefault((kind, d), []).append((st, al))
        self.groups = [(k, np.array([s for s, _ in g])[:, None] + np.arange(d)[None, :], np.array([a for _, a in g]))
                       for (k, d), g in groups.items()]

    def project(self, z, m, kappa, lo, hi):
        out = np.where(self.pos, np.maximum(z, 0.0), z)
        if lo is not None:
            out = np.where(self.box, np.minimum(np.maximum(z, lo), hi), out)
        for kind, idx, al in self.groups:
            r, w = z[idx], m[idx]
            out[idx] = (_soc(r, w) if kind == "soc" else _rsoc(r, w) if kind == "rsoc" else _exp(r, w)
                        if kind == "exp" else _pow(r, w, al) if kind == "pow" else _exp1(r, w, kappa[idx[:, 0]]))
        return out


def _op(rows, cols, data, size):
    return lambda x: np.bincount(rows, data * x[cols], minlength=size)


def _reference(p, iters):
    """Restarted reflected-Halpern PDHG in numpy: Ruiz (10 passes) and
    Pock-Chambolle scaling with one factor per cone block, bound-objective
    scaling, 128 power iterations, projected Barzilai-Borwein prox for a
    general Q, restart test and PID primal weight at iteration 1 of an epoch
    and every 64 iterations."""
    n, m, A, S = p.n, p.m, p.A, _Sets(p)
    rows, cols, val = torch.from_numpy(A.rows), torch.from_numpy(A.indices.astype(np.int64)), np.abs(A.data)
    Sx, Sy = np.ones(n), np.ones(m)
    for step in range(11):
        v = torch.from_numpy(val)
        if step < 10:
            col = torch.zeros(n, dtype=torch.float64).scatter_reduce_(0, cols, v, "amax").numpy()
            row = torch.zeros(m, dtype=torch.float64).scatter_reduce_(0, rows, v, "amax").numpy()
        else:
            col, row = np.bincount(A.indices, val, minlength=n), np.bincount(A.rows, val, minlength=m)
        col, row = np.sqrt(col), np.sqrt(row)
        for _, idx, _ in S.groups:
            g = col[idx]
            col[idx] = (g.max(1) if step < 10 else np.sqrt((g * g).mean(1)))[:, None]
        col[col == 0], row[row == 0] = 1.0, 1.0
        val = val / row[A.rows] / col[A.indices]
        Sx, Sy = Sx * col, Sy / row
    data = A.data * Sy[A.rows] / Sx[A.indices]
    ax = _op(A.rows, A.indices, data, m)
    at = _op(A.indices, A.rows, data, n)
    c = p.c / Sx
    if p.row_lo is None:
        lo = hi = None
        b = p.b * Sy
    else:
        lo, hi = p.row_lo * Sy, p.row_hi * Sy
        fin = [np.where(np.isfinite(e), np.abs(e), 0.0) for e in (lo, hi)]
        b = np.where(lo == hi, lo, np.maximum(*fin))
    nu_b, nu_c = np.linalg.norm(b) + 1.0, np.linalg.norm(c) + 1.0
    b, c, ratio = b / nu_b, c / nu_c, nu_b / nu_c
    if lo is not None:
        lo, hi = lo / nu_b, hi / nu_b
    xlo, xhi = (None, None) if p.x_lo is None else (p.x_lo * Sx / nu_b, p.x_hi * Sx / nu_b)
    kappa = Sx / nu_b
    qd, pp, diag = np.zeros(n), None, p.R is None
    if p.P is not None:
        pv = ratio * p.P.data / Sx[p.P.rows] / Sx[p.P.indices]
        on = p.P.rows == p.P.indices
        qd = np.bincount(p.P.rows[on], pv[on], minlength=n)
        diag = diag and bool(on.all())
        pp = (lambda u: qd0 * u) if on.all() else _op(p.P.rows, p.P.indices, pv, n)
        qd0 = qd.copy()
    R = None if p.R is None else p.R / Sx[None, :]
    if R is not None:
        qd = qd + ratio * ((p.D @ R) * R).sum(0)

    def q(u):
        w = pp(u) if pp is not None else np.zeros(n)
        return w if R is None else w + R.T @ (ratio * (p.D @ (R @ u)))

    def proj(z, d):
        return S.project(z, d, kappa, xlo, xhi)

    z = np.full(n, 1.0 / math.sqrt(n))
    lam = 0.0
    for _ in range(128):
        w = at(ax(z))
        lam = np.linalg.norm(w)
        z = w / lam
    eta = 0.998 / math.sqrt(lam)
    bn, cn = np.linalg.norm(b), np.linalg.norm(c)
    omega = cn / bn if bn > 1e-10 and cn > 1e-10 else 1.0
    x, y = proj(np.zeros(n), np.ones(n)), np.zeros(m)
    x_a, y_a, eps, k, integ, e0, e_last = x, y, 1e-3, 0, 0.0, 0.0, 0.0
    for tot in range(1, iters + 1):
        tau, sigma = eta / omega, eta * omega
        v = x + tau * at(y)
        if diag:
            d = 1.0 + tau * qd
            wx = proj((v - tau * c) / d, d)
        else:
            d = qd + 1.0 / tau
            up, gp = x, q(x) + c + (x - v) / tau
            wx = proj(up - gp / d, d)
            for _ in range(499):
                if np.linalg.norm(wx - up) <= eps:
                    break
                g, s = q(wx) + c + (wx - v) / tau, wx - up
                den = s @ (g - gp)
                up, gp, wx = wx, g, proj(wx - ((s @ (d * s)) / den if den > 0 else 1.0) * g / d, d)
        over = ax(2.0 * wx - x)
        if lo is None:
            wy = y + sigma * (b - over)
        else:
            t = over - y / sigma
            wy = np.where(lo == hi, y + sigma * (b - over), sigma * (np.minimum(np.maximum(t, lo), hi) - t))
        restart = False
        if k == 0 or tot % 64 == 0:
            dx, dy = x - wx, y - wy
            e = math.sqrt(max(omega * (dx @ dx) + (dy @ dy) / omega + 2.0 * eta * (ax(dx) @ dy), 0.0))
            if k == 0:
                e0 = e
            else:
                restart = e <= 0.2 * e0 or (e <= 0.8 * e0 and e > e_last) or k + 1 >= 0.36 * tot
            e_last = e
        if restart:
            mx, my = np.linalg.norm(wx - x_a), np.linalg.norm(wy - y_a)
            if mx > 1e-12 and my > 1e-12:
                err = math.log(my / (omega * mx))
                integ = 0.3 * integ + err
                omega = math.exp(math.log(omega) + 0.99 * err + 0.01 * integ)
            x, y, x_a, y_a, k = wx, wy, wx, wy, 0
        else:
            c1, c3 = (k + 1.0) / (k + 2.0), 1.0 / (k + 2.0)
            xn = c1 * (2.0 * wx - x) + c3 * x_a
            y = c1 * (2.0 * wy - y) + c3 * y_a
            eps = min(eps, max(5e-4 * np.linalg.norm(xn - x) / tau, 1e-9))
            x, k = xn, k + 1
    return nu_b * wx / Sx, nu_c * Sy * wy, nu_b * nu_c * (0.5 * (wx @ q(wx)) + c @ wx)


def exact(case, seed):
    if case["do"] == "project":
        r, m, al = _blocks(case, seed)
        return {"soc": _soc, "rsoc": _rsoc, "exp": _exp}[case["kind"]](r, m) if al is None else _pow(r, m, al)
    if case["do"] in ("predict", "epoch"):
        W, x, y = _network(case, seed, "cuda")
        W = [w.double().cpu() for w in W]
        x = x.double().cpu()
        if y is None:
            for k, w in enumerate(W):
                x = torch.clamp(x, min=0.0) @ w if k else x @ w
            return x
        return None          # Adam divides by the size of a gradient: signs near zero decide, not precision
    it, n = case["iters"], case.get("n", 0)
    if case["do"] == "fisher":
        e = case["buyers"] * case["goods"] * case["density"]
        seconds = e * (256 + 2 * it) * 1e-8 + case["buyers"] * it * (2e-5 if case["middle"] == "row" else 6e-6)
    elif case["do"] == "batch":
        seconds = case["count"] * (0.005 + 0.5 * (case["lo"] + case["hi"]) * it * 1.5e-7)
    else:
        seconds = n * {"qp": (256 + 10 * it) * 4e-8, "bounded": (256 + 2 * it) * 3e-8, "mixed": it * 1.8e-6}[case["do"]]
    if seconds > 20:
        return None
    res = [_reference(p, case["iters"]) for p in _instances(case, seed)]
    return (np.concatenate([r[0] for r in res]), np.concatenate([r[1] for r in res]), np.array([r[2] for r in res]))
