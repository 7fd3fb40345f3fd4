"""Index building on the GPU (dictionaries, leaf centers, encoding, layout) against the oracle, at the sizes where the
kernels' tiles and variants meet their edges."""
import numpy as np
import pytest

import oracle
from util import unit_rows

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
avq = pytest.importorskip("paper_1908_10396_amd")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# points around a workgroup's 256 and a tile's 64, exactly as many points as codewords; every specialised number of
# dimensions per subspace and others; sums too large for one workgroup's LDS (256 codewords of 96 dimensions)
@pytest.mark.parametrize("n,d,M,bits", [(16, 2, 1, 4), (257, 6, 6, 4), (255, 6, 3, 4), (1025, 105, 35, 4), (700, 20, 5, 4),
                                        (513, 35, 7, 4), (256, 10, 5, 8), (1000, 12, 3, 8), (2049, 24, 3, 8), (600, 36, 4, 8),
                                        (900, 96, 1, 8), (70_001, 4, 2, 4)])
@pytest.mark.parametrize("residual", [False, True])
def test_dictionaries_of_all_subspaces_match(n, d, M, bits, residual):
    rng = np.random.default_rng(n + d)
    x = unit_rows(rng, n, d)
    okw = {}
    leaves = 3 if residual else 0
    idx = avq.Index(d, M, bits, kmeans_iters=3, seed=5, n_leaves=leaves, leaf_kmeans_iters=2)
    idx.train(dev(x))
    if residual:
        okw = dict(leaf_centers=idx.get_leaf_centers())
        okw["leaf_assign"] = oracle.assign_nearest(x, okw["leaf_centers"])
    want = oracle.train_pq(x, M, 1 << bits, 3, 5, **okw)
    # fp64 means in another order, rounded to fp32: one unit in the last place of values below 1
    np.testing.assert_allclose(idx.get_codebooks(), want, rtol=0, atol=1.2e-7)
