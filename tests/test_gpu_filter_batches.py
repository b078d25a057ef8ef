"""A filter's prediction for a row depends on the filter and the row alone: not
on the rows beside it, on how many there are, or on whether the pair was
listed by a search.  Compared bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import workloads as W

pytestmark = pytest.mark.gpu


def _pkg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_01836_amd as pkg
    pkg.load()
    return pkg


def _rows(nq, m, seed):
    return np.random.default_rng(seed).standard_normal((nq, m)).astype(np.float32)


@pytest.mark.parametrize("F,m,h", [(300, 256, 256), (300, 96, 96), (260, 64, 32), (3, 256, 256)])
def test_rows_beside_rows_that_are_not_finite(F, m, h):
    pkg = _pkg()
    w = torch.from_numpy(W.mlp_weights(F, m, h, seed=F + m)).cuda()
    x = _rows(200, m, m)
    want = pkg.mlp_infer(w, m, h, torch.from_numpy(x).cuda()).cpu().numpy()
    odd = [3, 40, 41, 130, 199]
    y = x.copy()
    y[3, 0], y[40, m - 1], y[41], y[130, 5], y[199, 1] = np.nan, np.inf, np.nan, 3.4e38, -np.inf
    got = pkg.mlp_infer(w, m, h, torch.from_numpy(y).cuda()).cpu().numpy()
    same = np.setdiff1d(np.arange(200), odd)
    assert np.array_equal(got[same], want[same])
    # a NaN unit counts as 0: a row of NaN alone is left with the output bias
    assert np.array_equal(got[41], w[:, -1].cpu().numpy())


@pytest.mark.parametrize("F,m,h", [(3, 256, 256), (64, 128, 128), (128, 256, 256), (255, 96, 96), (256, 96, 96),
                                   (300, 100, 100), (300, 228, 144), (520, 256, 256), (1024, 32, 64),
                                   (300, 256, 64), (520, 160, 128), (300, 68, 36), (300, 128, 256)])
def test_rows_in_calls_of_any_size(F, m, h):
    pkg = _pkg()
    w = torch.from_numpy(W.mlp_weights(F, m, h, seed=F + h)).cuda()
    x = torch.from_numpy(_rows(500, m, h)).cuda()
    want = pkg.mlp_infer(w, m, h, x)
    for a, b in ((0, 1), (0, 17), (33, 65), (100, 333), (499, 500)):
        assert torch.equal(pkg.mlp_infer(w, m, h, x[a:b].clone()), want[a:b]), (a, b)


@pytest.mark.parametrize("arch,n_leaves,nq", [("mlp", 128, 300), ("mlp", 256, 300), ("mlp", 256, 2000), ("mlp", 512, 300),
                                              ("cnn", 128, 60), ("cnn", 512, 60)])
def test_listed_pairs_have_the_dense_predictions(arch, n_leaves, nq):
    """What a search subtracts its offsets from is what calibration fits them
    on.  Predictions of 1e9 and more stand a thousand apart, distances are
    below 50: with every offset the dense prediction itself no pair may be
    pruned, with the next float below it every pair that the search evaluates
    must be, for every query (each with a target, and so offsets, of its own)."""
    pkg = _pkg()
    m = 128 if arch == "mlp" else 32
    h = m if arch == "mlp" else 8
    raw = W.random_walk(n_leaves * 40, m, seed=n_leaves)
    ix = pkg.Index().build(torch.from_numpy(raw).cuda(), leaf_capacity=40, n_segments=8)
    F = ix.info()["n_leaves"]
    assert F == n_leaves
    g = np.random.default_rng(F)
    leaves = np.arange(F, dtype=np.int32)
    q = torch.from_numpy(W.noisy_queries(raw, nq, 0.4, 1, 2)[0]).cuda()
    if arch == "mlp":
        w = W.mlp_weights(F, m, h, seed=F)
        w[:, m * h + h: m * h + 2 * h] = g.uniform(1e9, 2e9, (F, h))
        ix.set_filters(leaves, torch.from_numpy(w).cuda(), h)
        y = pkg.mlp_infer(torch.from_numpy(w).cuda(), m, h, pkg.znorm(q))
    else:
        w = g.uniform(-0.5, 0.5, (F, 3 * h * h + 6 * h + 1)).astype(np.float32)
        w[:, 3 * h * h + 4 * h:3 * h * h + 5 * h] = 0.5  # the second layer's biases
        w[:, 3 * h * h + 5 * h:-1] = g.uniform(1e10, 2e10, (F, h))
        ix.set_cnn_filters(leaves, torch.from_numpy(w).cuda(), h)
        y = pkg.cnn_infer(torch.from_numpy(w).cuda(), m, h, pkg.znorm(q))
    y = y.cpu().numpy()
    assert y.min() > 1e9
    targets = ((np.arange(nq) + 1) / (nq + 1)).astype(np.float32)
    t = torch.from_numpy(targets).cuda()
    for offsets, share in ((y, 0), (np.nextafter(y, np.float32(0)), 1)):
        ix.set_offsets([1], targets, offsets)
        _, _, st = ix.search(q, k=1, target=t, k_max=1, schedule=(1, 0), with_stats=True)
        assert st["filter_evals"] > nq
        assert st["leaves_filter_pruned"] == share * st["filter_evals"]


@pytest.mark.parametrize("F,m,C", [(3, 96, 32), (256, 64, 64), (257, 64, 64), (300, 128, 32), (257, 96, 96), (1024, 36, 4)])
def test_cnn_rows_in_calls_of_any_size(F, m, C):
    pkg = _pkg()
    g = np.random.default_rng(F + m)
    w = torch.from_numpy(g.uniform(-0.5, 0.5, (F, 3 * C * C + 6 * C + 1)).astype(np.float32)).cuda()
    x = torch.from_numpy(_rows(70, m, C)).cuda()
    want = pkg.cnn_infer(w, m, C, x)
    for a, b in ((0, 1), (3, 5), (20, 37), (69, 70)):
        assert torch.equal(pkg.cnn_infer(w, m, C, x[a:b].clone()), want[a:b]), (a, b)
