"""Binary trees built on the device (large collections) against the oracle's:
the same leaves, member for member, and boxes that hold them.  Ties by the
thousand (few distinct series), midpoints with an empty side, segment counts
that are no power of two, chunks and nodes that end anywhere, capacity 1."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,S,capacity,rule,distinct", [
    (8192, 64, 16, 100, "median", 0), (8191, 64, 16, 100, "median", 0), (40001, 32, 5, 700, "median", 40),
    (33000, 32, 1, 9, "median", 0), (30011, 96, 12, 500, "midpoint", 0), (20000, 64, 32, 300, "midpoint", 7),
    (16500, 64, 64, 2, "median", 0)])
def test_device_tree_is_the_oracles(n, m, S, capacity, rule, distinct):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_01836_amd as pkg
    pkg.load()
    raw = W.random_walk(distinct or n, m, seed=n + S)
    if distinct:
        raw = raw[np.random.default_rng(n).integers(0, distinct, n)]
    ix = pkg.Index().build(torch.from_numpy(raw).cuda(), leaf_capacity=capacity, n_segments=S, split_rule=rule)
    offsets, members = ix.leaves()
    xs = O.znorm(raw)
    mu, sd = O.segment_stats(xs, S)
    t = O.build_tree(mu, sd, m, capacity, rule)
    assert np.array_equal(np.diff(offsets), [len(l) for l in t.leaves])
    assert np.array_equal(members, np.concatenate(t.leaves))
    boxes, want = ix.boxes(), O.leaf_boxes(mu, sd, t)
    # the summaries' own rounding (FP32 of FP64 sums) and the box's one ulp
    assert np.allclose(np.asarray(boxes).reshape(want.shape), want, rtol=1e-6, atol=1e-6)


@pytest.mark.parametrize("n,m,S,capacity,rule,distinct", [
    (9000, 32, 4, 1, "median", 0), (24000, 32, 4, 600, "midpoint", 0), (23999, 32, 4, 600, "midpoint", 0),
    (26000, 64, 32, 300, "midpoint", 7)])
def test_device_tree_of_single_series_and_at_the_midpoint_rules_edge(n, m, S, capacity, rule, distinct):
    test_device_tree_is_the_oracles(n, m, S, capacity, rule, distinct)
