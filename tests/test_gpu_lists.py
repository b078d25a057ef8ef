"""Candidate lists at the sizes where their cut and sort change form: lists of
up to 16, 64, 128, 256, 512 and more keys, kept whole or cut, on leaves smaller
and larger than a tile.  Exact search must equal FP64 brute force."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle as O
import workloads as W

from test_gpu_parity import assert_knn_parity

pytestmark = pytest.mark.gpu


def _pkg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_01836_amd as pkg
    pkg.load()
    return pkg


@pytest.fixture(scope="module")
def data():
    raw = W.random_walk(6000, 32, seed=81)
    q, _, _ = W.noisy_queries(raw, 40, 0.1, 82, 83)
    return raw, q, O.znorm(raw), O.znorm(q)


@pytest.mark.parametrize("capacity", [40, 900])
@pytest.mark.parametrize("k", [5, 16, 17, 33, 64, 130, 256])
def test_exact_search_at_list_sizes(data, capacity, k):
    pkg = _pkg()
    raw, q, xs, qs = data
    ix = pkg.Index().build(torch.from_numpy(raw).cuda(), leaf_capacity=capacity, n_segments=8)
    want_ids, want_d = O.knn(xs, qs, k)
    for tiling in ((128, 16), (2048, 64)):
        ix.set_tiling(*tiling)
        for scan in ("bf16", "fp32"):
            ids, d = ix.search(torch.from_numpy(q).cuda(), k=k, use_filters=False, scan=scan)
            assert_knn_parity(ids.cpu().numpy(), d.cpu().numpy(), want_ids, want_d, xs, qs)
