"""Performance cases of the library: what its users run, through its public
entry points.

Each case is a dict of plain values; `prepare` makes what a program holds
before the call (queries, a built index with its filters and calibration, a
server), `run` is one pass.  The kinds:

  search     one batch of k-NN queries against a built index
  serve      a burst of requests through the continuous-batching server
  leaf_knn   node-wise nearest neighbours of training queries (filter targets)
  build      index construction from raw series
  mlp_infer, cnn_infer   dense filter predictions
  mlp_sgd, cnn_sgd       one SGD step of every filter on its own mini-batch

Collections are random walks or a Gaussian mixture drawn on the GPU, queries
are collection rows with noise, as in `workloads`.  Filters of the searches
are fitted here by ridge regression on random ReLU features of training
queries, so that they predict the leaves' distances the way trained filters do
and stay the same whatever the library's own training does.
"""
import math

import numpy as np
import torch

import paper_2502_01836_amd as leafi

SEGMENTS = 16
N_TRAIN = 1000   # training queries of the fitted filters
N_CALIB = 500    # calibration queries
NOISE = (0.05, 0.2)
CHUNK = 1 << 20  # collection rows drawn at a time


def listed():
    return [
        # a small collection searched exactly (rw20k of `workloads`): 100 queries, bound by launches
        dict(name="search_20k_exact", kind="search", data="walk", n=20_000, m=256, capacity=1_000, split="median",
             nq=100, ks="1", targets="", scan="bf16"),
        # one interactive query against 1M series with filters: latency
        dict(name="search_1m_one", kind="search", data="walk", n=1_000_000, m=256, capacity=10_000, split="median",
             nq=1, ks="10", targets="0.99", scan="bf16"),
        # the 1M learned-filter workload (rw1m): a batch of 1,000 queries, k = 1
        dict(name="search_1m_batch", kind="search", data="walk", n=1_000_000, m=256, capacity=10_000, split="median",
             nq=1_000, ks="1", targets="0.99", scan="bf16"),
        # the mixed serving batch (k and recall target per query) over 10M series: the largest search
        dict(name="search_10m_mixed", kind="search", data="walk", n=10_000_000, m=256, capacity=10_000,
             split="median", nq=1_024, ks="1,10,100", targets="0.9,0.95,0.99", scan="bf16"),
        # ragged leaves of short series (gm25m with rows and leaf capacity scaled down), many queries, mixed k
        dict(name="search_ragged_mixed", kind="search", data="mixture", n=2_500_000, m=96, capacity=2_000,
             split="midpoint", nq=4_096, ks="1,10,50", targets="0.99", scan="bf16"),
        # a burst of requests to the server over 1M series
        dict(name="serve_1m_burst", kind="serve", data="walk", n=1_000_000, m=256, capacity=10_000, split="median",
             nq=2_000, ks="1,10", targets="0.95,0.99", scan="bf16"),
        # distances of training queries to every leaf: the targets filters are trained on
        dict(name="leaf_knn_1m", kind="leaf_knn", data="walk", n=1_000_000, m=256, capacity=10_000, split="median",
             nq=500, k=1),
        # index construction over 1M raw series
        dict(name="build_1m", kind="build", data="walk", n=1_000_000, m=256, capacity=10_000, split="median"),
        # predictions of a 10M-series index's filters for the calibration queries
        dict(name="mlp_infer_1024f", kind="mlp_infer", f=1_024, m=256, h=256, nq=500),
        # one training step of the same filters, the paper's mini-batch
        dict(name="mlp_sgd_1024f", kind="mlp_sgd", f=1_024, m=256, h=256, batch=64),
        # CNN filters as wide as the series (length 96)
        dict(name="cnn_infer_128f", kind="cnn_infer", f=128, m=96, c=96, nq=200),
        # a training step of narrower CNN filters
        dict(name="cnn_sgd_128f", kind="cnn_sgd", f=128, m=96, c=32, batch=32),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["search"] * 5 + ["serve", "leaf_knn", "build", "mlp_infer", "mlp_infer", "mlp_sgd", "cnn_infer",
                                        "cnn_sgd"])
    if kind == "mlp_infer":
        m, h = (4 * rng.randint(8, 64) for _ in range(2)) if rng.random() < 0.5 else (rng.choice([96, 128, 256]),) * 2
        return dict(kind=kind, f=_log(rng, 1, 1_024), m=m, h=h, nq=_log(rng, 1, 500))
    if kind == "mlp_sgd":
        m, h = (4 * rng.randint(8, 64) for _ in range(2)) if rng.random() < 0.5 else (rng.choice([96, 128, 256]),) * 2
        return dict(kind=kind, f=_log(rng, 1, 1_024), m=m, h=h, batch=rng.randint(1, 64))
    if kind in ("cnn_infer", "cnn_sgd"):
        m, c = 4 * rng.randint(4, 24), 4 * rng.randint(1, 24 if kind == "cnn_infer" else 8)
        size = dict(nq=_log(rng, 1, 200)) if kind == "cnn_infer" else dict(batch=rng.randint(1, 32))
        return dict(kind=kind, f=_log(rng, 1, 128), m=m, c=c, **size)
    data = rng.choice(["walk", "walk", "mixture"])
    case = dict(kind=kind, data=data, n=_log(rng, 5_000, 1_000_000), m=32 * rng.randint(1, 8),
                capacity=0, split="median" if data == "walk" else "midpoint")
    case["capacity"] = max(200, case["n"] // rng.randint(16, 128))
    if kind in ("build", "leaf_knn"):
        case["split"] = "median"  # the number of leaves, and so the outputs' shape, follows from the sizes alone
    if kind == "build":
        return case
    if kind == "leaf_knn":
        return dict(case, nq=_log(rng, 1, 500), k=rng.choice([1, 1, 5, 10]))
    filtered = kind == "serve" or rng.random() < 0.6
    ks = rng.choice(["1", "10", "1,10", "1,10,50", "100", "7"])
    return dict(case, nq=_log(rng, 1, 2_000), ks=ks, targets=rng.choice(["0.99", "0.9,0.95,0.99"]) if filtered else "",
                scan="fp32" if kind == "search" and case["n"] < 50_000 and rng.random() < 0.3 else "bf16")


# ---- inputs ---------------------------------------------------------------------


def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1_000_003 + salt)
    return g


def _collection(case, seed):
    n, m = case["n"], case["m"]
    x = torch.empty((n, m), dtype=torch.float32, device="cuda")
    means = torch.randn((1_000, m), generator=_gen(seed, 1), device="cuda") if case["data"] == "mixture" else None
    for c, lo in enumerate(range(0, n, CHUNK)):
        g, rows = _gen(seed, 100 + c), min(CHUNK, n - lo)
        v = torch.randn((rows, m), generator=g, device="cuda")
        if means is None:
            torch.cumsum(v, dim=1, out=x[lo:lo + rows])
        else:
            pick = torch.randint(0, means.shape[0], (rows,), generator=g, device="cuda")
            torch.add(means[pick], v, alpha=0.3, out=x[lo:lo + rows])
    return x


def _noisy(x, nq, seed, salt, noise=NOISE):
    """Rows of the collection with noise relative to each row's deviation."""
    g = _gen(seed, salt)
    rows = torch.randint(0, x.shape[0], (nq,), generator=g, device="cuda")
    base = x[rows].double()
    level = noise[0] + (noise[1] - noise[0]) * torch.rand((nq, 1), generator=g, device="cuda", dtype=torch.float64)
    scale = base.std(dim=1, unbiased=False, keepdim=True) * level
    return (base + scale * torch.randn(base.shape, generator=g, device="cuda", dtype=torch.float64)).float()


def _znorm64(x):
    x = x.double()
    x = x - x.mean(dim=1, keepdim=True)
    sd = x.square().mean(dim=1, keepdim=True).sqrt()
    return torch.where(sd < 1e-8, torch.zeros_like(x), x / sd.clamp_min(1e-300))


def _fit_filters(index, x, case, seed):
    """One MLP per leaf: random first layer, output layer by ridge regression on
    the training queries' distances to the leaf.  The hidden units of filter f
    are rotated by f places, so no two filters hold the same weights."""
    m = h = case["m"]
    q = _noisy(x, N_TRAIN, seed, 11)
    d, _ = index.leaf_knn(q, 1)
    y = d[:, :, 0].double().cpu()
    n_leaves = y.shape[1]
    g = _gen(seed, 12)
    w1 = (2 * torch.rand((m, h), generator=g, device="cuda") - 1) / math.sqrt(m)
    b1 = (2 * torch.rand((h,), generator=g, device="cuda") - 1) / math.sqrt(m)
    phi = torch.relu(_znorm64(q).cpu() @ w1.double().cpu() + b1.double().cpu())
    phi = torch.cat([phi, torch.ones((N_TRAIN, 1), dtype=torch.float64)], dim=1)
    ridge = torch.eye(h + 1, dtype=torch.float64) * 1e-2 * N_TRAIN
    ridge[h, h] = 0.0
    out = torch.linalg.solve(phi.T @ phi + ridge, phi.T @ y).float().cuda()  # [h + 1, leaves]
    w = torch.empty((n_leaves, h * m + 2 * h + 1), dtype=torch.float32, device="cuda")
    at = (torch.arange(h, device="cuda")[None] + torch.arange(n_leaves, device="cuda")[:, None]) % h
    w[:, : h * m] = w1.T[at].transpose(1, 2).reshape(n_leaves, h * m)
    w[:, h * m: h * m + h] = b1[at]
    w[:, h * m + h: h * m + 2 * h] = torch.gather(out[:h].T, 1, at)
    w[:, -1] = out[h]
    index.set_filters(np.arange(n_leaves, dtype=np.int32), w, h)


def _numbers(text, kind):
    return [kind(v) for v in text.split(",") if v]


def _built(case, x):
    return leafi.Index().build(x, leaf_capacity=case["capacity"], n_segments=SEGMENTS, split_rule=case["split"])


def _mlp(f, m, h, seed, bias):
    g = _gen(seed, 21)
    w = 2 * torch.rand((f, h * m + 2 * h + 1), generator=g, device="cuda") - 1
    w[:, : h * m + h] /= math.sqrt(m)
    w[:, h * m + h:] /= math.sqrt(h)
    w[:, -1] += bias
    return w


def _cnn(f, c, seed, bias):
    g = _gen(seed, 22)
    w = 2 * torch.rand((f, 3 * c * c + 6 * c + 1), generator=g, device="cuda") - 1
    w[:, : 4 * c] /= math.sqrt(3)
    w[:, 4 * c: 5 * c + 3 * c * c] /= math.sqrt(3 * c)
    w[:, 5 * c + 3 * c * c:] /= math.sqrt(c)
    w[:, -1] += bias
    return w


def _series(rows, m, seed, salt):
    """z-normalised random walks."""
    return _znorm64(torch.cumsum(torch.randn((rows, m), generator=_gen(seed, salt), device="cuda"), dim=1)).float()


def _filter_inputs(case, seed):
    f, m = case["f"], case["m"]
    w = _mlp(f, m, case["h"], seed, 8.0) if case["kind"].startswith("mlp") else _cnn(f, case["c"], seed, 8.0)
    if "batch" not in case:
        return dict(w=w, x=_series(case["nq"], m, seed, 23))
    y = 8.0 + 2.0 * torch.randn((f, case["batch"]), generator=_gen(seed, 24), device="cuda")
    return dict(w=w, x=_series(f * case["batch"], m, seed, 23).reshape(f, case["batch"], m), y=y)


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("mlp_infer", "mlp_sgd", "cnn_infer", "cnn_sgd"):
        return dict(case=case, **_filter_inputs(case, seed))
    x = _collection(case, seed)
    if kind == "build":
        return dict(case=case, x=x)
    index = _built(case, x)
    q = _noisy(x, case["nq"], seed, 31, (0.1, 0.1))
    if kind == "leaf_knn":
        return dict(case=case, index=index, q=_noisy(x, case["nq"], seed, 31))
    ks, targets = _numbers(case["ks"], int), _numbers(case["targets"], float)
    g = _gen(seed, 32)
    k = torch.tensor(ks, dtype=torch.int32, device="cuda")[
        torch.randint(0, len(ks), (case["nq"],), generator=g, device="cuda")]
    if targets:
        _fit_filters(index, x, case, seed)
        index.calibrate(_noisy(x, N_CALIB, seed, 33), ks, targets)
        t = torch.tensor(targets, dtype=torch.float32, device="cuda")[
            torch.randint(0, len(targets), (case["nq"],), generator=g, device="cuda")]
    else:
        t = torch.ones((case["nq"],), dtype=torch.float32, device="cuda")
    state = dict(case=case, index=index, q=q, k=k, t=t, k_max=max(ks), filters=bool(targets))
    if kind == "serve":
        state.update(server=leafi.Server(index, k_max=max(ks), scan=case["scan"]), q=q.cpu().numpy(),
                     k=k.cpu().numpy(), t=t.cpu().numpy(), arrivals=np.zeros(case["nq"]))
    return state


# ---- one pass --------------------------------------------------------------------


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "search":
        return state["index"].search(state["q"], k=state["k"], target=state["t"], k_max=state["k_max"],
                                     scan=case["scan"], use_filters=state["filters"])
    if kind == "serve":
        ids, d, _, _ = state["server"].replay(state["q"], state["arrivals"], state["k"], state["t"])
        return ids, d
    if kind == "leaf_knn":
        return state["index"].leaf_knn(state["q"], case["k"])
    if kind == "build":
        index = _built(case, state["x"])
        offsets, members = index.leaves()
        return offsets, members, index.boxes()
    if kind == "mlp_infer":
        return leafi.mlp_infer(state["w"], case["m"], case["h"], state["x"])
    if kind == "cnn_infer":
        return leafi.cnn_infer(state["w"], case["m"], case["c"], state["x"])
    if kind == "mlp_sgd":
        return state["w"], leafi.mlp_sgd_step(state["w"], case["m"], case["h"], state["x"], state["y"], 0.01)
    return state["w"], leafi.cnn_sgd_step(state["w"], case["m"], case["c"], state["x"], state["y"], 0.01)


# ---- what a pass cannot do without ---------------------------------------------------

# Share of the collection's rows a query of a search scans after pruning (measured on the listed cases).
SCANNED = {"walk": 0.06, "mixture": 0.35}
SCANNED_EXACT = 0.15


def work(case):
    kind, m = case["kind"], case["m"]
    if kind in ("mlp_infer", "mlp_sgd"):
        f, h = case["f"], case["h"]
        params = f * (h * m + 2 * h + 1)
        rows = case["nq"] if kind == "mlp_infer" else case["batch"]
        if kind == "mlp_infer":
            return dict(bytes=4 * (params + rows * m + rows * f), flops=2 * f * rows * h * m)
        return dict(bytes=4 * (2 * params + f * rows * (m + 1) + f), flops=4 * f * rows * h * m)
    if kind in ("cnn_infer", "cnn_sgd"):
        f, c = case["f"], case["c"]
        params = f * (3 * c * c + 6 * c + 1)
        if kind == "cnn_infer":
            return dict(bytes=4 * (params + case["nq"] * (m + f)), flops=6 * f * case["nq"] * m * c * (c + 1))
        return dict(bytes=4 * (2 * params + f * case["batch"] * (m + 1) + f),
                    flops=18 * f * case["batch"] * m * c * (c + 1))
    n = case["n"]
    if kind == "build":  # raw rows read, both copies of the store written
        return dict(bytes=n * (4 * m + 6 * m + 8), flops=8 * n * m)
    if kind == "leaf_knn":
        leaves = n / case["capacity"]
        return dict(bytes=n * (2 * m + 4) + case["nq"] * (4 * m + leaves * case["k"] * 12),
                    flops=2.0 * case["nq"] * n * m)
    nq, k_max = case["nq"], max(_numbers(case["ks"], int))
    share = SCANNED[case["data"]] if case["targets"] else SCANNED_EXACT
    row = 2 * m + 4 if case["scan"] == "bf16" else 4 * m
    size = min(1.0, share * nq) * n * row + nq * (4 * m + 12 * k_max)
    return dict(bytes=size, flops=2.0 * nq * share * n * m)


# ---- the same in 64 bits ---------------------------------------------------------------


def _mlp64(w, m, h, x):
    """Hidden pre-activations and predictions of every filter: x [F or 1, rows, m]."""
    w1 = w[:, : h * m].reshape(-1, m, h)
    z = torch.matmul(x, w1) + w[:, None, h * m: h * m + h]
    w2 = w[:, h * m + h: h * m + 2 * h]
    return z, (z.relu() * w2[:, None]).sum(dim=2) + w[:, -1:]


def _cnn64(w, c, x):
    """Predictions [rows] of one CNN filter for x [rows, m]."""
    conv = torch.nn.functional.conv1d
    w1, b1 = w[: 3 * c].reshape(c, 1, 3), w[3 * c: 4 * c]
    w2, b2 = w[4 * c: 4 * c + 3 * c * c].reshape(c, c, 3), w[4 * c + 3 * c * c: 5 * c + 3 * c * c]
    h1 = conv(x[:, None], w1, b1, padding=1).relu()
    return conv(h1, w2, b2, padding=1).relu().mean(dim=2) @ w[5 * c + 3 * c * c: 6 * c + 3 * c * c] + w[-1]


def exact(case, seed):
    kind, m = case["kind"], case["m"]
    if kind in ("mlp_infer", "mlp_sgd"):
        s = _filter_inputs(case, seed)
        h, out = case["h"], []
        for lo in range(0, case["f"], 32):
            w = s["w"][lo:lo + 32].double()
            if kind == "mlp_infer":
                out.append(_mlp64(w, m, h, s["x"][None].double())[1].T)
                continue
            x, y = s["x"][lo:lo + 32].double(), s["y"][lo:lo + 32].double()
            w.requires_grad_(True)
            loss = (_mlp64(w, m, h, x)[1] - y).square().mean(dim=1)
            out.append((w.detach() - 0.01 * torch.autograd.grad(loss.sum(), w)[0], loss.detach()))
        if kind == "mlp_infer":
            return torch.cat(out, dim=1)
        return torch.cat([a for a, _ in out]), torch.cat([b for _, b in out])
    if kind in ("cnn_infer", "cnn_sgd"):
        # on the CPU: 64-bit convolutions there need no tuned library kernel
        s = {k: v.double().cpu() for k, v in _filter_inputs(case, seed).items()}
        if kind == "cnn_infer":
            return torch.stack([_cnn64(w, case["c"], s["x"]) for w in s["w"]], dim=1)
        new, losses = [], []
        for w, x, y in zip(s["w"], s["x"], s["y"]):
            w = w.clone().requires_grad_(True)
            loss = (_cnn64(w, case["c"], x) - y).square().mean()
            new.append(w.detach() - 0.01 * torch.autograd.grad(loss, w)[0])
            losses.append(loss.detach())
        return torch.stack(new), torch.stack(losses)
    if kind != "search" or case["targets"]:
        return None  # the leaves, and what the filters prune, are the library's own
    x = _collection(case, seed)
    q = _znorm64(_noisy(x, case["nq"], seed, 31, (0.1, 0.1)))
    ks = _numbers(case["ks"], int)
    pick = torch.randint(0, len(ks), (case["nq"],), generator=_gen(seed, 32), device="cuda")
    k = torch.tensor(ks, dtype=torch.int64, device="cuda")[pick]
    k_max, rows = max(ks), max(1, (1 << 27) // case["nq"])
    best = torch.full((case["nq"], 0), math.inf, dtype=torch.float64, device="cuda")
    for lo in range(0, case["n"], rows):
        z = _znorm64(x[lo:lo + rows])
        d2 = q.square().sum(1)[:, None] + z.square().sum(1)[None] - 2 * (q @ z.T)
        best = torch.cat([best, d2.clamp_min(0).sqrt()], dim=1).topk(min(k_max, best.shape[1] + z.shape[0]), dim=1,
                                                                     largest=False).values
    best = torch.nn.functional.pad(best, (0, k_max - best.shape[1]), value=math.inf)
    best[torch.arange(k_max, device="cuda")[None] >= k[:, None]] = math.inf
    return None, best
