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
