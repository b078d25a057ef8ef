"""Tile shapes set by the caller: the default can be restored, and passes that
are no searches keep their own.  Seen by the device memory a fresh index takes
for the same calls, which follows the shape of its tiles."""
import pytest

torch = pytest.importorskip("torch")

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_01836_amd as pkg
    pkg.load()
    raw = W.random_walk(20000, 64, seed=1)
    q = W.noisy_queries(raw, 100, 0.1, 2, 3)[0]
    return pkg, torch.from_numpy(raw).cuda(), torch.from_numpy(q).cuda()


def _live(env, call, *shapes):
    pkg, raw, q = env
    alloc = pkg.TorchAllocator()
    ix = pkg.Index(allocator=alloc).build(raw, leaf_capacity=1500, n_segments=8)
    for s in shapes:
        ix.set_tiling(*s)
    call(ix, q)
    torch.cuda.synchronize()
    live = alloc.live_bytes
    ix.close()
    return live


def _search(ix, q):
    ix.search(q, k=10, use_filters=False, schedule=(1, 0))


def test_the_default_can_be_restored(env):
    want = _live(env, _search)
    assert _live(env, _search, (2048, 64)) != want  # the shape shows
    assert _live(env, _search, (2048, 64), (1024, 32)) == want


def test_passes_that_are_no_searches_keep_their_shape(env):
    def knn(ix, q):
        ix.leaf_knn(q, 3)
    want = _live(env, knn)
    assert _live(env, knn, (128, 16)) == want
