"""Performance cases of the online tensor method on one GPU.

A case is a dict of plain values.  `listed()` names the ones that are timed
every time, `draw(rng)` gives more of the same ranges, `prepare(case, seed)`
makes the inputs and the state that a program holds before the call,
`run(state)` makes one pass through the package's entry points, `work(case)`
counts the bytes and operations that the pass cannot do without and
`exact(case, seed)` gives its results in 64 bits from plain torch.

The paths are the stages of a decomposition (sketch, whitener, whitening,
stochastic updates, memberships), one whole small decomposition, a batch of
decompositions with restarts, and a training step of the warm start's
perceptron.  The sizes are those of the repository's own workloads: the block
model graphs with 1000 and 100,000 nodes (k = 10 and 100), the document
collection with 10,000 words (k = 50), and the batch of uneven problems.
"""
from __future__ import annotations

import math

import torch

from paper_1309_0787_amd import otm, pipeline

DTYPES = {"fp32": otm.F32, "bf16": otm.BF16}
TORCH = {"fp32": torch.float32, "bf16": torch.bfloat16}
F64 = torch.float64


# ---------------------------------------------------------------- the cases
def listed() -> list[dict]:
    return [
        # a whole decomposition of the small graph workload (500 x 500 block, 50
        # passes): what an interactive user runs; launches and latency count
        dict(name="fit_graph_small", path="fit", nodes=1000, k=10, alpha0=0.1, p=0.3, q=0.05, passes=50),
        # power-iterated sketch of the large graph's second moment (FP64): the first
        # stage of the benchmark decomposition
        dict(name="sketch_graph", path="sketch", data="graph", n=50000, d=50000, k=100, alpha0=0.5, p=0.05, q=0.001,
             power=3),
        # the same stage on the document collection, whose rows are longer and whose
        # columns are few and very long
        dict(name="sketch_docs", path="sketch", data="docs", n=100000, d=10000, k=50, alpha0=1.0, length=200, power=3),
        # whitening matrix of the large graph from its sketch (FP64, BF16 copy)
        dict(name="whitener_graph", path="whitener", d=50000, k=100, width=200, dtype="bf16"),
        # the three document views whitened in FP32
        dict(name="whiten_docs", path="whiten", data="docs", n=100000, d=10000, k=50, alpha0=1.0, length=200,
             dtype="fp32"),
        # the large graph block whitened in BF16
        dict(name="whiten_graph", path="whiten", data="graph", n=50000, d=50000, k=100, alpha0=0.5, p=0.05, q=0.001,
             dtype="bf16"),
        # online updates on 10,000 newly arrived whitened rows of the large graph:
        # BF16, one view (single leaf set), plain update
        dict(name="stgd_graph_bf16", path="stgd", n=10000, k=100, alpha0=0.5, views=1, dtype="bf16", batch=100, passes=1,
             restarts=1, compensated=False, beta0=1e-3),
        # the four-partition form of it: three different views, compensated update
        dict(name="stgd_four_bf16", path="stgd", n=10000, k=100, alpha0=0.5, views=3, dtype="bf16", batch=100, passes=1,
             restarts=1, compensated=True, beta0=1e-3),
        # one pass over the whitened documents in FP32, three views
        dict(name="stgd_docs_fp32", path="stgd", n=100000, k=50, alpha0=1.0, views=3, dtype="fp32", batch=100, passes=1,
             restarts=1, compensated=True, beta0=1e-3),
        # many uneven problems with eight restarts each in one batched run (FP32)
        dict(name="batched_fp32", path="batched", problems=24, n_lo=1000, n_hi=20000, restarts=8, passes=2),
        # one training step of the warm start's perceptron: forward, loss,
        # backward, Adam
        dict(name="warm_train", path="train", batch=256),
        # memberships of the large graph's nodes and their validation
        dict(name="memberships_graph", path="members", n=50000, k=100, dtype="bf16"),
    ]


def _log(rng, lo: float, hi: float) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> dict:
    path = rng.choice(["fit", "sketch", "whitener", "whiten", "whiten", "stgd", "stgd", "stgd", "batched", "train",
                       "members"])
    if path == "fit":
        return dict(path=path, nodes=_log(rng, 600, 4000), k=rng.randint(3, 12), alpha0=0.1, p=0.3, q=0.05,
                    passes=rng.randint(10, 50))
    if path in ("sketch", "whiten"):
        if rng.random() < 0.5:
            n = _log(rng, 4000, 50000)
            k = rng.randint(20, 100) if n > 12000 else rng.randint(10, 30)
            c = dict(path=path, data="graph", n=n, d=n + rng.randint(-n // 10, n // 10) if n < 40000 else n, k=k,
                     alpha0=0.5, p=min(0.3, 2500.0 / n), q=min(0.006, 50.0 / n))
        else:
            c = dict(path=path, data="docs", n=_log(rng, 5000, 100000), d=_log(rng, 1500, 10000),
                     k=rng.randint(10, 50), alpha0=1.0, length=rng.randint(60, 200))
        if path == "sketch":
            c["power"] = rng.randint(1, 3)
        else:
            c["dtype"] = rng.choice(["fp32", "bf16"])
        return c
    if path == "whitener":
        k = rng.randint(8, 100)
        return dict(path=path, d=_log(rng, 2000, 50000), k=k, width=2 * k, dtype=rng.choice(["fp32", "bf16"]))
    if path == "stgd":
        dtype = rng.choice(["fp32", "bf16"])
        k = _log(rng, 8, 128)
        batch = rng.choice([100, 100, 128, 64, rng.randint(20, 127)])
        steps = rng.randint(20, 100) if dtype == "bf16" else rng.randint(50, 500)
        return dict(path=path, n=max(batch, steps * batch - rng.randint(0, batch - 1)), k=k,
                    alpha0=rng.choice([0.1, 0.5, 1.0]), views=rng.choice([1, 3]), dtype=dtype, batch=batch, passes=1,
                    restarts=rng.choice([1, 1, 8]), compensated=rng.choice([False, True]), beta0=1e-3)
    if path == "batched":
        return dict(path=path, problems=rng.randint(4, 24), n_lo=1000, n_hi=_log(rng, 3000, 20000),
                    restarts=rng.choice([2, 4, 8]), passes=rng.randint(1, 2))
    if path == "train":
        return dict(path=path, batch=_log(rng, 16, 256))
    return dict(path=path, n=_log(rng, 2000, 50000), k=rng.randint(8, 100), dtype=rng.choice(["fp32", "bf16"]))


# ------------------------------------------------------------ input recipes
def _gen(seed: int, sub: int, device):
    return torch.Generator(device=device).manual_seed((seed * 1000003 + sub * 7919 + 12345) % (1 << 62))


def _dirichlet(rows: int, k: int, conc: float, g, device) -> torch.Tensor:
    x = torch._standard_gamma(torch.full((rows, k), conc, dtype=F64, device=device), generator=g)
    x = x + 1e-290 * torch.rand((rows, k), dtype=F64, device=device, generator=g)   # rows whose draws all underflow
    return x / x.sum(1, keepdim=True)


def _haar(k: int, seed: int, sub: int) -> torch.Tensor:
    """Orthonormal k x k factor of a Gaussian, on the host in FP64."""
    q, r = torch.linalg.qr(torch.randn((k, k), dtype=F64, generator=_gen(seed, sub, "cpu")))
    return q * torch.sign(torch.diagonal(r))[None, :]


def _csr(rows, cols, n_rows: int, n_cols: int, counts=None):
    """(DeviceCSR, unique row-major keys, counts) of the entries (rows, cols)."""
    key, cnt = torch.unique(rows * n_cols + cols, return_counts=True)
    r = key // n_cols
    ptr = torch.zeros(n_rows + 1, dtype=torch.int64, device=rows.device)
    ptr[1:] = torch.cumsum(torch.bincount(r, minlength=n_rows), 0)
    vals = cnt.to(torch.float32) if counts else None
    return otm.DeviceCSR(n_rows, n_cols, ptr.to(torch.int32), (key % n_cols).to(torch.int32), vals), key, cnt


def _transposed(key, cnt, n_rows: int, n_cols: int, counts=None):
    r, c = key // n_cols, key % n_cols
    t, order = torch.sort(c * n_rows + r)
    ptr = torch.zeros(n_cols + 1, dtype=torch.int64, device=key.device)
    ptr[1:] = torch.cumsum(torch.bincount(c, minlength=n_cols), 0)
    vals = cnt[order].to(torch.float32) if counts else None
    return otm.DeviceCSR(n_cols, n_rows, ptr.to(torch.int32), (t % n_rows).to(torch.int32), vals)


def _flat_cum(w: torch.Tensor) -> torch.Tensor:
    """Row c of w as the cumulative distribution on [c, c + 1), summed on the host."""
    c = torch.cumsum(w.cpu(), 1)
    c = c / c[:, -1:] + torch.arange(w.shape[0], dtype=F64)[:, None]
    return c.reshape(-1).to(w.device)


def _pick(cum: torch.Tensor, group: torch.Tensor, width: int, g) -> torch.Tensor:
    """One index in [0, width) per entry from the distribution of its group."""
    u = torch.rand(group.shape, dtype=F64, device=group.device, generator=g) * (1 - 1e-9)
    at = torch.searchsorted(cum, group.to(F64) + u, right=True) - group * width
    return at.clamp_(0, width - 1)


def _graph(case, seed: int, device, transpose: bool = True):
    """Block G[X, A] of a mixed membership block model: within-community edges
    from Poisson counts per (node, community), background edges uniform."""
    n, d, k, p, q = case["n"], case["d"], case["k"], case["p"], case["q"]
    g = _gen(seed, 1, device)
    px, pa = _dirichlet(n, k, case["alpha0"] / k, g, device), _dirichlet(d, k, case["alpha0"] / k, g, device)
    size = pa.sum(0)
    cell = torch.poisson((p - q) * px * size[None, :], generator=g).to(torch.int64).reshape(-1)
    at = torch.repeat_interleave(torch.arange(n * k, device=device), cell)
    x, c = at // k, at % k
    a = _pick(_flat_cum(pa.T.contiguous()), c, d, g)
    bg = torch.poisson(torch.full((n,), q * d, dtype=F64, device=device), generator=g).to(torch.int64)
    xb = torch.repeat_interleave(torch.arange(n, device=device), bg)
    ab = torch.randint(0, d, xb.shape, device=device, generator=g)
    C, key, cnt = _csr(torch.cat([x, xb]), torch.cat([a, ab]), n, d)
    return C, (_transposed(key, cnt, n, d) if transpose else None)


def _documents(case, seed: int, device, views: bool):
    """Word counts of documents from a topic model: the whole collection with its
    transpose, or the three views (token position modulo 3)."""
    n, d, k = case["n"], case["d"], case["k"]
    g = _gen(seed, 2, device)
    mu = _dirichlet(k, d, 0.05, g, device)
    h = _dirichlet(n, k, case["alpha0"] / k, g, device)
    length = torch.poisson(torch.full((n,), float(case["length"]), dtype=F64, device=device), generator=g)
    length = length.clamp_(min=6).to(torch.int64)
    doc = torch.repeat_interleave(torch.arange(n, device=device), length)
    topic = _pick(_flat_cum(h), doc, k, g)
    word = _pick(_flat_cum(mu), topic, d, g)
    if not views:
        C, key, cnt = _csr(doc, word, n, d, True)
        return C, _transposed(key, cnt, n, d, True)
    start = torch.cumsum(length, 0) - length
    view = (torch.arange(doc.numel(), device=device) - start[doc]) % 3
    return [_csr(doc[view == v], word[view == v], n, d, True)[0] for v in range(3)]


def _rows(n: int, k: int, alpha0: float, views: int, dtype: str, seed: int, sub: int, device):
    """Whitened rows of a planted mixture, y = sqrt(k) U h + noise, each view with
    noise of its own; ([YA, YB, YC], ybar (3 x k), U, h)."""
    g = _gen(seed, 10 + sub, device)
    U = _haar(k, seed, 20 + sub)
    h = _dirichlet(n, k, alpha0 / k, g, device)
    mean = h @ (math.sqrt(k) * U.to(device)).T
    out = []
    for _ in range(views):
        y = torch.zeros((n, otm.default_ldy(k)), dtype=TORCH[dtype], device=device)
        y[:, :k] = (mean + 0.3 / math.sqrt(k) * torch.randn((n, k), dtype=F64, device=device, generator=g)).to(y.dtype)
        out.append(y)
    out = out * 3 if views == 1 else out
    return out, torch.stack([y[:, :k].to(F64).mean(0) for y in out]).to(torch.float32).contiguous(), U, h


def _factors(k: int, restarts: int, seed: int, sub: int) -> torch.Tensor:
    return torch.stack([_haar(k, seed, 1000 * (sub + 1) + r).T for r in range(restarts)]).to(torch.float32).contiguous()


def _perms(n: int, passes: int, seed: int, sub: int, device) -> torch.Tensor:
    g = _gen(seed, 30 + sub, "cpu")
    return torch.stack([torch.randperm(n, generator=g) for _ in range(passes)]).to(device=device, dtype=torch.int32)


def _sketch_input(case, seed: int, device):
    """Sketch Q (orthonormal columns) and O = M2 Q of a moment of rank k with
    noise of both signs below it.  The eigenvalues keep apart, as those of
    sampled moments do."""
    d, k, m = case["d"], case["k"], case["width"]
    g = _gen(seed, 3, device)
    z = torch.randn((d, m), dtype=F64, generator=_gen(seed, 4, "cpu"))
    Q = torch.linalg.qr(z)[0].contiguous().to(device)
    R = _haar(m, seed, 5).to(device)
    lam = torch.empty(m, dtype=F64, device=device)
    jitter = 0.4 * (torch.rand(k, dtype=F64, device=device, generator=g) - 0.5)
    lam[:k] = 1.0 + 75.0 * ((torch.arange(k, dtype=F64, device=device) + 0.5 + jitter) / k) ** 2
    lam[k:] = 0.3 * (2.0 * torch.rand(m - k, dtype=F64, device=device, generator=g) - 1.0)
    M = (R * lam[None, :]) @ R.T
    O = Q @ (0.5 * (M + M.T)) + 0.05 / math.sqrt(d) * torch.randn((d, m), dtype=F64, device=device, generator=g)
    return Q, O.contiguous()


def _problem_table(case, seed: int) -> list[dict]:
    """Shapes of a batch: k from the set of the batched workload, n log-uniform,
    half the problems with three views.  The shapes belong to the case, the
    data to the seed."""
    g = _gen(77, 6, "cpu")
    ks, N = (16, 32, 64, 100, 128), case["problems"]
    out = []
    for i in range(N):
        u = torch.rand(2, dtype=F64, generator=g)
        n = int(math.exp(math.log(case["n_lo"]) + float(u[0]) * math.log(case["n_hi"] / case["n_lo"])))
        views = 3 if i % 2 == 0 else 1
        out.append(dict(n=n, k=ks[int(float(u[1]) * 5)], views=views,
                        alpha0=1.0 if views == 3 else (0.1 if n <= 10000 else 0.5)))
    return out


def _train_input(case, seed: int, device):
    dims = otm.ws_dims()
    P, B = dims["P"], case["batch"]
    g = _gen(seed, 7, device)
    ks = torch.tensor([10, 50, 100], dtype=torch.int32, device=device)[torch.randint(0, 3, (B,), device=device,
                                                                                     generator=g)]
    live = torch.arange(P, device=device)[None, :] < ks[:, None]
    block = (live[:, :, None] & live[:, None, :]).to(torch.float32)
    scale = 1.0 / ks.to(torch.float32)[:, None, None]
    X = torch.zeros((B, dims["n_in"]), dtype=torch.float32, device=device)
    for r in range(4):
        X[:, r * P * P:(r + 1) * P * P] = (torch.randn((B, P, P), device=device, generator=g) * block * scale).reshape(B, -1)
    X[:, 4 * P * P:] = (torch.randn((B, 4, P), device=device, generator=g) * live[:, None, :]).reshape(B, -1)
    tgt = (torch.randn((B, P, P), device=device, generator=g) * block * scale).reshape(B, P * P).contiguous()
    parts = []
    for rows, cols in ((dims["hidden"], dims["n_in"]), (dims["n_out"], dims["hidden"])):
        for count in (rows * cols, rows):
            parts.append((torch.rand(count, device=device, generator=g) * 2 - 1) / math.sqrt(cols))
    params = torch.cat(parts)
    m = 1e-7 * torch.randn(params.shape, device=device, generator=g)
    v = 1e-14 * (0.5 + torch.rand(params.shape, device=device, generator=g))
    return dict(ks=ks, X=X, target=tgt, params=params, m=m, v=v, live=int((ks.to(torch.int64) ** 2).sum()), t=100)


# ------------------------------------------------------------------ prepare
def prepare(case: dict, seed: int) -> dict:
    dev = torch.device("cuda")
    path = case["path"]
    s = dict(case=case)
    if path == "fit":
        k, n = case["k"], case["nodes"] // 2
        c = dict(n=n, d=case["nodes"] - n, k=k, alpha0=case["alpha0"], p=case["p"], q=case["q"])
        s["C"], s["CT"] = _graph(c, seed, dev)
        s["S"] = torch.randn((c["d"], 2 * k), dtype=F64, generator=_gen(seed, 8, "cpu")).to(dev)
        s["Phi0"] = _factors(k, 1, seed, 0).to(dev)
        s["perms"] = _perms(n, case["passes"], seed, 0, dev)
        s["cfg"] = pipeline.FitConfig(k=k, alpha0=case["alpha0"], passes=case["passes"], beta0=0.05, beta_tau=500.0)
    elif path == "sketch":
        s["C"], s["CT"] = _graph(case, seed, dev) if case["data"] == "graph" else _documents(case, seed, dev, False)
        s["S"] = torch.randn((case["d"], 2 * case["k"]), dtype=F64, generator=_gen(seed, 8, "cpu")).to(dev)
        s["infos"] = torch.zeros(2 * case["power"] + 1, dtype=torch.int32, device=dev)
    elif path == "whitener":
        s["Q"], s["O"] = _sketch_input(case, seed, dev)
        s["info"] = torch.zeros(1, dtype=torch.int32, device=dev)
    elif path == "whiten":
        s["views"] = [_graph(case, seed, dev, False)[0]] if case["data"] == "graph" else _documents(case, seed, dev, True)
        k, ld = case["k"], otm.default_ldw(case["k"], DTYPES[case["dtype"]])
        W = torch.zeros((case["d"], ld), dtype=F64, device=dev)
        W[:, :k] = torch.randn((case["d"], k), dtype=F64, device=dev, generator=_gen(seed, 9, dev)) / math.sqrt(case["d"])
        s["W"] = W.to(TORCH[case["dtype"]])[:, :k]
    elif path == "stgd":
        k, n = case["k"], case["n"]
        s["Y"], s["ybar"], _, _ = _rows(n, k, case["alpha0"], case["views"], case["dtype"], seed, 0, dev)
        s["Phi0"] = _factors(k, case["restarts"], seed, 0).to(dev)
        s["perms"] = _perms(n, case["passes"], seed, 0, dev)
        s["flag"] = torch.zeros(1, dtype=torch.int32, device=dev)
        s["p"] = otm.SgdParams(k=k, batch=case["batch"], passes=case["passes"], y_dtype=DTYPES[case["dtype"]],
                               compensated=case["compensated"], alpha0=case["alpha0"], beta0=case["beta0"],
                               beta_tau=2500.0)
    elif path == "batched":
        probs = []
        for i, t in enumerate(_problem_table(case, seed)):
            Y, ybar, _, _ = _rows(t["n"], t["k"], t["alpha0"], t["views"], "fp32", seed, 100 + i, dev)
            probs.append(otm.Problem(YA=Y[0], YB=Y[1], YC=Y[2], ybar3=ybar, k=t["k"], alpha0=t["alpha0"],
                                     Phi0=_factors(t["k"], case["restarts"], seed, i).to(dev),
                                     perms=_perms(t["n"], case["passes"], seed, i, dev)))
        p = otm.SgdParams(k=1, batch=100, passes=case["passes"], compensated=True, beta0=3e-4, beta_tau=2500.0)
        s["run"] = otm.BatchedRun(probs, case["restarts"], p)
    elif path == "train":
        s.update(_train_input(case, seed, dev))
        s["grads"] = torch.zeros_like(s["params"])
    else:
        n, k = case["n"], case["k"]
        Y, _, U, h = _rows(n, k, 0.5, 1, case["dtype"], seed, 0, dev)
        s["Y"], s["truth"] = Y[0], h.T.to(torch.float32).contiguous()
        noise = torch.randn((k, k), dtype=F64, generator=_gen(seed, 11, "cpu")) * 0.02 / math.sqrt(k)
        s["Phi"] = (k ** (1.0 / 6.0) * (U.T + noise)).to(torch.float32).contiguous().to(dev)
    torch.cuda.synchronize()
    return s


# ---------------------------------------------------------------------- run
def run(s: dict):
    case = s["case"]
    path = case["path"]
    if path == "fit":
        r = pipeline.fit([s["C"]], s["C"], s["CT"], s["S"], s["Phi0"].clone(), s["perms"], s["cfg"], pi_view=0)
        return dict(W=r.W, evals=r.evals, Y=r.Y[0], ybar=r.ybar3, Phi=r.Phi, Pi=r.Pi)
    if path == "sketch":
        Q, O = otm.power_sketch(s["C"], s["CT"], case["data"] == "docs", case["alpha0"], s["S"], case["power"],
                                infos=s["infos"])
        return dict(Q=Q, O=O)
    if path == "whitener":
        W, ev, lo = otm.whitener(s["O"], s["Q"], case["k"], w_lo_dtype=DTYPES[case["dtype"]], info=s["info"])
        return dict(W=W, evals=ev, W_lo=lo)
    if path == "whiten":
        return [otm.whiten(v, case["data"] == "docs", s["W"], y_dtype=DTYPES[case["dtype"]]) for v in s["views"]]
    if path == "stgd":
        Phi = s["Phi0"].clone()
        otm.sgd_run(s["p"], case["n"], *s["Y"], s["ybar"], s["perms"], Phi, restarts=case["restarts"],
                    nonfinite=s["flag"])
        return dict(Phi=Phi, nonfinite=s["flag"])
    if path == "batched":
        b = s["run"]
        b.run()
        return dict(Phi=b.Phi, scores=b.scores, best=b.best)
    if path == "train":
        H, out = otm.mlp_forward(s["params"], s["X"])
        loss, dout = otm.ws_mse(s["ks"], s["live"], out, s["target"])
        otm.mlp_backward(s["params"], s["X"], H, dout, s["grads"])
        s["t"] += 1
        otm.mlp_adam(s["params"], s["grads"], s["m"], s["v"], s["t"], 1e-3)
        return dict(loss=loss, out=out, grads=s["grads"], params=s["params"], m=s["m"], v=s["v"])
    Pi = otm.recover_pi(s["Y"], case["k"], s["Phi"])
    v = otm.validate(Pi, s["truth"])
    return dict(Pi=Pi, rho=v.rho, p=v.p, p_adj=v.p_adj, edges=v.edges, l1=v.l1, scores=v.scores)


# --------------------------------------------------------------------- work
def _stored(case) -> float:
    """Expected stored entries of a drawn data set."""
    if case["data"] == "graph":
        return case["n"] * case["d"] * (case["q"] + (case["p"] - case["q"]) / case["k"])
    return case["n"] * case["length"] * 0.96


def _sgd_work(n, k, views, size, batch, passes, restarts):
    steps = -(-n // batch) * passes
    flops = restarts * (steps * 4.0 * k ** 3 + n * passes * (6.0 if views == 3 else 4.0) * k * k)
    return restarts * passes * n * views * k * size + 4.0 * passes * n + 8.0 * restarts * k * k, flops


def work(case: dict) -> dict:
    path = case["path"]
    if path in ("fit", "sketch"):
        c = dict(case, data=case.get("data", "graph"), power=case.get("power", 3))
        if path == "fit":
            c["n"] = c["nodes"] // 2
            c["d"] = c["nodes"] - c["n"]
        nnz, m = _stored(c), 2 * c["k"]
        entry = 4 if c["data"] == "graph" else 8
        flops = (c["power"] + 1) * 4.0 * nnz * m + c["power"] * 8.0 * c["d"] * m * m
        nbytes = 2 * entry * nnz + 4.0 * (c["n"] + c["d"]) + 3 * 8.0 * c["d"] * m
        if path == "fit":
            b, f = _sgd_work(c["n"], c["k"], 1, 4, 100, c["passes"], 1)
            nbytes += b + 4.0 * c["n"] * c["k"] * 2
            flops += f + 2.0 * nnz * c["k"]
        return dict(bytes=nbytes, flops=flops)
    if path == "whitener":
        d, m, k = case["d"], case["width"], case["k"]
        return dict(bytes=8.0 * d * (2 * m + k) + (2 if case["dtype"] == "bf16" else 4) * d * k,
                    flops=2.0 * d * (m * m + m * k + 2 * k * k) + 9.0 * (m ** 3 + k ** 3))
    if path == "whiten":
        nnz, size = _stored(case), 2 if case["dtype"] == "bf16" else 4
        views = 1 if case["data"] == "graph" else 3
        entry = 4 if case["data"] == "graph" else 8
        return dict(bytes=entry * nnz + views * (4.0 * case["n"] + case["n"] * case["k"] * size) + case["d"] * case["k"] * size,
                    flops=2.0 * nnz * case["k"])
    if path == "stgd":
        b, f = _sgd_work(case["n"], case["k"], case["views"], 2 if case["dtype"] == "bf16" else 4, case["batch"],
                         case["passes"], case["restarts"])
        return dict(bytes=b, flops=f)
    if path == "batched":
        b = f = 0.0
        for t in _problem_table(case, 0):   # the updates and one scoring pass
            for passes in (case["passes"], 1):
                x, y = _sgd_work(t["n"], t["k"], t["views"], 4, 100, passes, case["restarts"])
                b, f = b + x, f + y
        return dict(bytes=b, flops=f)
    if path == "train":
        dims = otm.ws_dims()
        w = dims["hidden"] * (dims["n_in"] + dims["n_out"])
        return dict(bytes=4.0 * (8 * dims["n_params"] + case["batch"] * (dims["n_in"] + 3 * dims["n_out"])),
                    flops=2.0 * case["batch"] * (2 * w + dims["hidden"] * dims["n_out"]) + 12.0 * dims["n_params"])
    n, k = case["n"], case["k"]
    return dict(bytes=n * k * ((2 if case["dtype"] == "bf16" else 4) + 4.0 + 4.0 + 4.0), flops=7.0 * n * k * k)


# -------------------------------------------------------------------- exact
def _sparse64(C) -> torch.Tensor:
    vals = torch.ones(C.nnz, dtype=F64, device=C.device) if C.vals is None else C.vals.to(F64)
    rows = torch.repeat_interleave(torch.arange(C.n_rows, device=C.device), (C.rowptr[1:] - C.rowptr[:-1]).to(torch.int64))
    return torch.sparse_coo_tensor(torch.stack([rows, C.colidx.to(torch.int64)]), vals, (C.n_rows, C.n_cols)).coalesce()


def _power_sketch64(C, CT, normalize: bool, alpha0: float, S, q: int):
    A, At = _sparse64(C).to_sparse_csr(), _sparse64(CT).to_sparse_csr()
    n = C.n_rows
    one = torch.ones((n, 1), dtype=F64, device=S.device)
    length = (A @ torch.ones((C.n_cols, 1), dtype=F64, device=S.device)) if normalize else None
    w1 = 1.0 / length if normalize else one
    w2 = 1.0 / (length * (length - 1.0)) if normalize else one
    u, M1 = At @ w2, (At @ w1) / n

    def m2(V):
        return (alpha0 + 1.0) / n * (At @ (w2 * (A @ V)) - u * V) - alpha0 * M1 @ (M1.T @ V)

    Q = S
    for _ in range(q):
        z, r = torch.linalg.qr(m2(Q).cpu())
        Q = (z * torch.sign(torch.diagonal(r))[None, :]).to(S.device)
    return Q, m2(Q)


def _whitener64(O, Q, k: int):
    om = (Q.T @ O).cpu()
    lam, U = torch.linalg.eigh(0.5 * (om + om.T))
    at = torch.argsort(lam, descending=True)[:k]
    B = O @ (U[:, at] / torch.sqrt(lam[at])[None, :]).to(O.device)
    ev, V = torch.linalg.eigh((B.T @ B).cpu())
    at = torch.argsort(ev, descending=True)
    W = B @ (V[:, at] / ev[at][None, :]).to(O.device)
    top = W.gather(0, W.abs().argmax(0, keepdim=True))
    return W * torch.where(top < 0, -1.0, 1.0), ev[at].to(O.device)


def _sgd64(Y, ybar, Phi0, perms, batch: int, alpha0: float, beta0: float, tau: float, score: bool = False):
    """The update of all restarts in 64 bits: F[r] has phi_i as column i."""
    a, b, c = (alpha0 + 1) * (alpha0 + 2) / 2, alpha0 * (alpha0 + 1) / 2, alpha0 * alpha0
    k = Phi0.shape[-1]
    YA, YB, YC = (y[:, :k].to(F64) for y in Y)
    ya, yb, yc = ybar.to(F64)
    F = Phi0.to(F64).transpose(1, 2).contiguous()

    def direction(F, rows):
        A, B, C = YA[rows], YB[rows], YC[rows]
        mA, mB = (ya @ F)[:, None, :], (yb @ F)[:, None, :]
        PA, PB = A @ F, B @ F
        H = PA * PB
        D = C.T @ (a * H - b * (PA * mB + mA * PB)) / len(rows)
        return D + yc[None, :, None] * (c * mA * mB - b * H.mean(1, keepdim=True))

    t, n = 0, YA.shape[0]
    for order in perms.to(torch.int64):
        for s0 in range(0, n, batch):
            G = F.transpose(1, 2) @ F
            F = F + beta0 / (1.0 + t / tau) * (direction(F, order[s0:s0 + batch]) - F @ (G * G))
            t += 1
    Phi = F.transpose(1, 2).contiguous()
    if not score:
        return Phi
    G = F.transpose(1, 2) @ F
    T = (F * direction(F, torch.arange(n, device=F.device))).sum((1, 2))
    return Phi, (G ** 3).sum((1, 2)) - 2.0 * T


def _memberships64(Y, Phi):
    P = Phi.to(F64)
    nrm = P.norm(dim=1, keepdim=True)
    x = ((P / nrm / nrm ** 3) @ Y.to(F64).T).clamp_(min=0)
    s = x.sum(0, keepdim=True)
    return torch.where(s > 0, x / s, torch.zeros_like(x))


def exact(case: dict, seed: int):
    s = prepare(case, seed)
    path = case["path"]
    if path == "fit":
        cfg = s["cfg"]
        Q, O = _power_sketch64(s["C"], s["CT"], False, cfg.alpha0, s["S"], cfg.q_power)
        W, ev = _whitener64(O, Q, cfg.k)
        Y = torch.zeros((s["C"].n_rows, otm.default_ldy(cfg.k)), dtype=F64, device=W.device)
        Y[:, :cfg.k] = _sparse64(s["C"]) @ W
        ybar = Y[:, :cfg.k].mean(0).repeat(3, 1)
        Phi = _sgd64([Y] * 3, ybar, s["Phi0"], s["perms"], cfg.batch, cfg.alpha0, cfg.beta0, cfg.beta_tau)
        return dict(W=W, evals=ev, Y=Y, ybar=ybar.reshape(-1), Phi=Phi, Pi=_memberships64(Y[:, :cfg.k], Phi[0]))
    if path == "sketch":
        Q, O = _power_sketch64(s["C"], s["CT"], case["data"] == "docs", case["alpha0"], s["S"], case["power"])
        return dict(Q=Q, O=O)
    if path == "whitener":
        W, ev = _whitener64(s["O"], s["Q"], case["k"])
        return dict(W=W, evals=ev, W_lo=W)
    if path == "whiten":
        out, k = [], case["k"]
        for v in s["views"]:
            A = _sparse64(v)
            y = A @ s["W"].to(F64)
            if case["data"] == "docs":
                total = A @ torch.ones((v.n_cols, 1), dtype=F64, device=y.device)
                y = torch.where(total > 0, y / total, torch.zeros_like(y))
            Y = torch.zeros((v.n_rows, otm.default_ldy(k)), dtype=F64, device=y.device)
            Y[:, :k] = y
            out.append((Y, y.mean(0)))
        return out
    if path == "stgd":
        return dict(Phi=_sgd64(s["Y"], s["ybar"], s["Phi0"], s["perms"], case["batch"], case["alpha0"], case["beta0"],
                               2500.0), nonfinite=None)
    if path == "batched":
        Phi, scores = [], []
        for P in s["run"].problems:
            x, y = _sgd64([P.YA, P.YB, P.YC], P.ybar3, P.Phi0, P.perms, 100, P.alpha0, 3e-4, 2500.0, score=True)
            Phi.append(x)
            scores.append(y)
        return dict(Phi=Phi, scores=scores, best=None)
    if path == "train":
        dims = otm.ws_dims()
        ni, nh, no = dims["n_in"], dims["hidden"], dims["n_out"]
        p = s["params"].to(F64)
        W1, b1, W2, b2 = torch.split(p, [nh * ni, nh, no * nh, no])
        W1, W2, X = W1.reshape(nh, ni), W2.reshape(no, nh), s["X"].to(F64)
        H = (X @ W1.T + b1).clamp_(min=0)
        out = H @ W2.T + b2
        k = s["ks"].to(torch.int64)
        live = torch.arange(dims["P"], device=p.device)[None, :] < k[:, None]
        mask = (live[:, :, None] & live[:, None, :]).reshape(out.shape)
        diff = torch.where(mask, out - s["target"].to(F64), torch.zeros_like(out))
        dout = 2.0 * diff / s["live"]
        dZ = (dout @ W2) * (H > 0)
        grads = torch.cat([(dZ.T @ X).reshape(-1), dZ.sum(0), (dout.T @ H).reshape(-1), dout.sum(0)])
        t = s["t"] + 1
        m, v = 0.9 * s["m"].to(F64) + 0.1 * grads, 0.999 * s["v"].to(F64) + 0.001 * grads ** 2
        new = p - 1e-3 * (m / (1 - 0.9 ** t)) / (torch.sqrt(v / (1 - 0.999 ** t)) + 1e-8)
        return dict(loss=(diff ** 2).sum().reshape(1) / s["live"], out=out, grads=grads, params=new, m=m, v=v)
    Pi = _memberships64(s["Y"][:, :case["k"]], s["Phi"])
    X, T = Pi - Pi.mean(1, keepdim=True), s["truth"].to(F64)
    Z = T - T.mean(1, keepdim=True)
    rho = (X @ Z.T) / (X.norm(dim=1)[:, None] * Z.norm(dim=1)[None, :])
    l1 = torch.stack([(Pi[i][None, :] - T).abs().mean(1) for i in range(Pi.shape[0])])
    return dict(Pi=Pi, rho=rho, p=None, p_adj=None, edges=None, l1=l1, scores=None)
