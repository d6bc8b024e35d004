"""Tree scoring where the trees do not divide: leaf values added eight at a time after a chunk (tiles split over slices), and
eight trees side by side (one configuration per thread).  Bit for bit against the oracle, which adds in tree order."""
import numpy as np
import pytest
import torch

from paper_1905_12799_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rls():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_12799_amd import binding
    binding.lib()
    return binding


# small: slices, trees 1 .. two chunks and a remainder; large: groups of eight, the last one of 1, 7 or all
@pytest.mark.parametrize("N,d,T,D", [(1, 8, 1, 3), (65, 5, 7, 4), (1000, 8, 8, 6), (3001, 16, 9, 6), (4000, 8, 129, 8), (20001, 12, 65, 5), (50001, 16, 95, 9),
                                     (262145, 8, 8, 4), (300001, 16, 9, 6), (262145, 32, 23, 7), (270001, 5, 55, 8), (262145, 16, 25, 10), (262145, 8, 12, 7)])
def test_trees_that_do_not_divide(rls, orc, N, d, T, D):
    rng = np.random.default_rng(N + T)
    X = rng.standard_normal((N, d)).astype(np.float32)
    f = synth.random_forest(X, T, D, 0, rng)
    f.base = -0.0                                        # (and leaves of -0: a sum of nothing but these keeps its sign)
    f.leaf[::3] = -0.0
    f.leaf[T // 2, 0] = np.inf
    got = rls.gbt_score(rls.DeviceForest.from_host(f), torch.as_tensor(X).cuda()).cpu().numpy()
    want = orc.gbt_score(f, X)[0]
    np.testing.assert_array_equal(got.view(np.int32), want.view(np.int32))
