"""Batches over more leaves than a wavefront's registers or LDS hold per query:
the filter pairs selected by the merge (256 leaves) or in a launch of their
own, the leaf counts and item slots taken per work-group of 16 queries,
indexes past the 4,096 leaves that the layout keeps in LDS, and visit orders
by bucket and rank, with bounds that crowd one bucket as well.  Results and
pruning counts against the FP64 oracle, and the host-driven rounds, the
planned launches and replayed graphs against each other."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
import workloads as W
from test_gpu_parity import assert_knn_parity

pytestmark = pytest.mark.gpu

M, S, H = 32, 8, 8


@pytest.mark.parametrize("n,capacity,leaves,nq,crowd", [(2500, 10, 256, 17, 0), (5000, 15, 512, 1, 0),
                                                       (5000, 15, 512, 33, 0), (20000, 4, 7712, 18, 0),
                                                       (6000, 15, 512, 9, 4000)])
def test_counts_slots_and_pairs(n, capacity, leaves, nq, crowd):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_01836_amd as pkg
    pkg.load()
    raw = W.random_walk(n, M, seed=n + 1)
    if crowd:  # the last rows are close copies of one series: their leaves' bounds crowd together
        raw[n - crowd:] = raw[n - 1] + 2e-3 * np.random.default_rng(n).standard_normal((crowd, M)).astype(np.float32)
    ix = pkg.Index().build(torch.from_numpy(raw).cuda(), leaf_capacity=capacity, n_segments=S)
    N = ix.info()["n_leaves"]
    assert N == leaves
    filtered = np.arange(0, N, 3, dtype=np.int32)  # every third leaf has a filter
    w = W.mlp_weights(len(filtered), M, H, seed=n + 2, out_bias=2.0)
    offs = np.random.default_rng(n + 3).uniform(0.0, 1.0, len(filtered)).astype(np.float32)
    ix.set_filters(filtered, torch.from_numpy(w).cuda(), H)
    ix.set_offsets([1], [0.9], offs[None])
    q, _, _ = W.noisy_queries(raw[:n - crowd], nq, (0.3, 0.6), n + 4, n + 5)
    xs, qs = O.znorm(raw), O.znorm(q)
    mu, sd = O.segment_stats(xs, S)
    t = O.build_tree(mu, sd, M, capacity, "median")
    lb = O.lower_bound(*O.query_stats(qs, S), O.leaf_boxes(mu, sd, t), M)
    if crowd:
        for b in lb:
            assert np.histogram(b, bins=1024)[0].max() > 128
    ld, li = O.leaf_knn(xs, t.leaves, qs, 1)
    dF = np.zeros((nq, N))
    dF[:, filtered] = np.stack([O.mlp_forward(w[f], qs, M, H) for f in range(len(filtered))], 1) - offs[None]
    has = np.zeros(N, dtype=bool)
    has[filtered] = True
    r = O.leafi_search(lb, O.visit_order(lb), ld, li, 1, has, dF, (1, 0))
    qd = torch.from_numpy(q).cuda()
    out = (torch.empty((nq, 1), dtype=torch.int64, device="cuda"), torch.empty((nq, 1), device="cuda"))
    seen = []
    for flags in (pkg.SEARCH_HOST_ROUNDS, pkg.SEARCH_NO_GRAPH, 0, 0, 0, 0):
        ids, d, st = ix.search(qd, k=1, target=0.9, use_filters=True, schedule=(1, 0), with_stats=True, flags=flags,
                               out=out)
        torch.cuda.synchronize()
        seen.append((ids.cpu().numpy().copy(), d.cpu().numpy().copy(), st))
    ids, d, st = seen[0]
    assert_knn_parity(ids, d, r.ids, r.dist, xs, qs)
    if not r.near_tie.any():
        assert st["leaves_filter_pruned"] == int(r.f_pruned.sum())
        assert nq == 1 or r.f_pruned.any()  # the batches reach the filter test
        assert st["leaves_scanned"] == int(r.scanned.sum())
    for i2, d2, s2 in seen[1:]:
        assert np.array_equal(i2, ids) and np.array_equal(d2, d)
        for key in ("leaves_scanned", "leaves_lb_pruned", "leaves_filter_pruned", "series_scanned"):
            assert s2[key] == st[key], key


@pytest.mark.parametrize("nq,k", [(1, 10), (40, 50), (40, 256), (9, 1), (330, 1)])
def test_bounds_skip_no_result(nq, k):
    """Exact batches on unstructured series (few leaves pruned, so every query
    meets most of the 256): items tested against their queries' bounds one to a
    wavefront, several to one, or listed first; bounds from the scan alone
    (k = 1) and from the k-th of the collected keys, up to more than fit."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_01836_amd as pkg
    pkg.load()
    rng = np.random.default_rng(31)
    raw = rng.standard_normal((8000, M)).astype(np.float32)
    q = (raw[rng.choice(8000, nq, replace=False)] + rng.standard_normal((nq, M))).astype(np.float32)
    ix = pkg.Index().build(torch.from_numpy(raw).cuda(), leaf_capacity=32, n_segments=S)
    ids, d, st = ix.search(torch.from_numpy(q).cuda(), k=k, k_max=k, use_filters=False, schedule=(1, 0),
                           with_stats=True)
    torch.cuda.synchronize()
    assert st["leaves_scanned"] > 128 * nq
    xs, qs = O.znorm(raw), O.znorm(q)
    ref_ids, ref_d = O.knn(xs, qs, k)
    assert_knn_parity(ids.cpu().numpy(), d.cpu().numpy(), ref_ids, ref_d, xs, qs)


@pytest.mark.parametrize("k,nq", [(40, 3), (256, 3), (5, 20)])
def test_lists_end_where_their_keys_do(k, nq):
    """Lists of far fewer keys than their slots, over a workspace whose slots
    hold an earlier batch's full lists: nothing past a list's end is read."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_01836_amd as pkg
    pkg.load()
    raw = W.random_walk(9000, 64, seed=77)
    q, _, _ = W.noisy_queries(raw, 40, 0.4, 78, 79)
    ix = pkg.Index().build(torch.from_numpy(raw).cuda(), leaf_capacity=100, n_segments=S)
    qd = torch.from_numpy(q).cuda()
    xs, qs = O.znorm(raw), O.znorm(q)
    want_ids, want_d = O.knn(xs, qs, 256)
    ix.search(qd, k=256, k_max=256, use_filters=False, schedule=(0,))  # tau +inf: full lists everywhere
    for schedule in ((1, 0), (2, 5, 0)):
        ids, d = ix.search(qd[:nq], k=k, k_max=k, use_filters=False, schedule=schedule)
        torch.cuda.synchronize()
        assert_knn_parity(ids.cpu().numpy(), d.cpu().numpy(), want_ids[:nq, :k], want_d[:nq, :k], xs, qs[:nq])
    ks = torch.from_numpy(np.resize([1, 40, 256], 40).astype(np.int32)).cuda()
    ids, d = ix.search(qd, k=ks, k_max=256, use_filters=False, schedule=(1, 0))
    torch.cuda.synchronize()
    for i, kk in enumerate(ks.cpu().tolist()):
        assert_knn_parity(ids[i:i + 1, :kk].cpu().numpy(), d[i:i + 1, :kk].cpu().numpy(), want_ids[i:i + 1, :kk],
                          want_d[i:i + 1, :kk], xs, qs[i:i + 1])
