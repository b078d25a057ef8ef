"""Series and queries with NaN or infinite values: such a series is nobody's
neighbour and hides none, and such a query finds nothing and leaves the other
queries' results as they are."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

N, M = 9000, 64


@pytest.fixture(scope="module")
def env():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_01836_amd as pkg
    pkg.load()
    raw = W.random_walk(N, M, seed=5)
    q = W.noisy_queries(raw, 60, 0.2, 3, 4)[0]
    bad = np.random.default_rng(0).choice(N, 400, replace=False)
    raw[bad[:200], 3] = np.nan
    raw[bad[200:300], 0] = np.inf
    raw[bad[300:]] = -np.inf
    fine = np.setdiff1d(np.arange(N), bad)
    ids, d = O.knn(O.znorm(raw[fine]), O.znorm(q), 50)
    return dict(pkg=pkg, raw=raw, q=q, bad=bad, ids=fine[ids], d=d)


@pytest.mark.parametrize("split_rule,capacity", [("median", 100), ("isax", 100), ("median", N)])
@pytest.mark.parametrize("scan", ["bf16", "fp32"])
def test_series_that_are_not_finite(env, split_rule, capacity, scan):
    pkg = env["pkg"]
    ix = pkg.Index().build(torch.from_numpy(env["raw"]).cuda(), leaf_capacity=capacity, n_segments=8,
                           split_rule=split_rule)
    q = torch.from_numpy(env["q"]).cuda()
    for k in (1, 10, 50):
        for schedule in ((1, 0), (4, 0), (1,)):
            ids, d = ix.search(q, k=k, scan=scan, use_filters=False, schedule=schedule)
            ids, d = ids.cpu().numpy(), d.cpu().numpy()
            assert np.allclose(d, env["d"][:, :k], rtol=1e-5, atol=1e-6), (k, schedule)
            assert not np.isin(ids, env["bad"]).any()


def test_a_leaf_of_few_finite_series(env):
    """More neighbours wanted than a leaf has: the others' slots are empty."""
    pkg = env["pkg"]
    raw = W.random_walk(40, M, seed=6)
    raw[5:] = np.nan
    ix = pkg.Index().build(torch.from_numpy(raw).cuda(), leaf_capacity=40, n_segments=8)
    q = W.random_walk(3, M, seed=7)
    want = np.sort(np.sqrt(((O.znorm(q).astype(np.float64)[:, None] - O.znorm(raw[:5])[None]) ** 2).sum(-1)), 1)
    qd = torch.from_numpy(q).cuda()
    for d, ids in (ix.search(qd, k=10, use_filters=False)[::-1], ix.search(qd, k=10, scan="fp32", use_filters=False)[::-1],
                   [t[:, 0] for t in ix.leaf_knn(qd, 10)]):
        d, ids = d.cpu().numpy(), ids.cpu().numpy()
        assert np.allclose(d[:, :5], want, rtol=1e-5) and np.isposinf(d[:, 5:]).all()
        assert (ids[:, 5:] == -1).all() and (np.sort(ids[:, :5], 1) == np.arange(5)).all()


@pytest.mark.parametrize("schedule", [(1, 0), (4, 0)])
def test_queries_that_are_not_finite(env, schedule):
    pkg = env["pkg"]
    ix = pkg.Index().build(torch.from_numpy(env["raw"]).cuda(), leaf_capacity=100, n_segments=8)
    want = [t.cpu().numpy() for t in ix.search(torch.from_numpy(env["q"]).cuda(), k=10, use_filters=False, schedule=schedule)]
    q = env["q"].copy()
    q[7, 3], q[20], q[41, 0] = np.nan, np.nan, np.inf
    ids, d = [t.cpu().numpy() for t in ix.search(torch.from_numpy(q).cuda(), k=10, use_filters=False, schedule=schedule)]
    bad, fine = [7, 20, 41], np.setdiff1d(np.arange(60), [7, 20, 41])
    assert np.array_equal(ids[fine], want[0][fine]) and np.array_equal(d[fine], want[1][fine])
    assert (ids[bad] == -1).all() and np.isposinf(d[bad]).all()
