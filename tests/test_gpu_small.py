"""Sweeps of few points, one workgroup per run in one launch, against the same sweep launched round by round (the route of a
sweep that also returns the loss of every round), bit for bit, and against the oracle."""
import numpy as np
import pytest
import torch

from tests.test_gpu_ordered import make

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rls():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_12799_amd import binding
    binding.lib()
    return binding


# one block and less, odd numbers of blocks, the largest size and one more, every padded width, one to four tiles, exact ties
CASES = [("clusters", 1, 4, 1, 1), ("clusters", 31, 8, 1, 20), ("clusters", 33, 5, 1, 33), ("clusters", 2000, 8, 1, 16), ("noise", 1025, 16, 5, 64),
         ("clusters", 3001, 13, 1, 40), ("grid", 2049, 6, 1, 60), ("grid", 4095, 16, 30, 64), ("noise", 2560, 32, 1, 33), ("clusters", 1703, 29, 110, 128),
         ("clusters", 4096, 16, 1, 128), ("clusters", 6144, 16, 1, 40), ("clusters", 6145, 16, 1, 40), ("line", 4001, 1, 1, 128), ("same", 600, 8, 1, 33),
         ("wide", 1800, 7, 1, 40), ("wide", 2100, 20, 30, 64), ("clusters", 777, 17, 97, 128), ("grid", 853, 32, 128, 128), ("grid", 3072, 8, 3, 3)]


def step_launches(rls, sweep):
    """The sweep's results, and how many launches of the step it took: none when all rounds were one launch."""
    rls.profile_read()
    rls.profile_enable(True)
    try:
        result = sweep()
    finally:
        rls.profile_enable(False)
    return result, rls.profile_read()[0]


@pytest.mark.parametrize("kind,N,d,k_min,k_max", CASES)
def test_small_sweep_equals_launched_rounds(rls, kind, N, d, k_min, k_max):
    X = torch.as_tensor(make(kind, N, max(d, 2), N + d)[:, :d].copy()).cuda()
    for iters in (0, 1, 7):
        got, steps = step_launches(rls, lambda: rls.kmeans_sweep(X, k_min, k_max, iters, seed=3))
        assert steps == (iters if N == 6145 else 0)          # (the one that is too large)
        want = rls.kmeans_sweep(X, k_min, k_max, iters, seed=3, want_trace=True)
        assert torch.equal(got.labels, want.labels)
        assert torch.equal(got.centroids, want.centroids)
        assert torch.equal(got.inertia, want.inertia)


@pytest.mark.parametrize("N,d,k_min,k_max", [(2000, 8, 1, 16), (2555, 21, 8, 40), (853, 32, 120, 128)])
def test_small_sweep_against_the_oracle(rls, orc, N, d, k_min, k_max):
    X = make("clusters", N, d, 5)
    got, steps = step_launches(rls, lambda: rls.kmeans_sweep(torch.as_tensor(X).cuda(), k_min, k_max, 12, seed=9))
    assert steps == 0
    ref = orc.kmeans_sweep(X, k_min, k_max, 12, seed=9)
    np.testing.assert_array_equal(got.labels.cpu().numpy(), ref["labels"])
    np.testing.assert_array_equal(got.centroids.cpu().numpy(), ref["centroids"])
    np.testing.assert_allclose(got.inertia.cpu().numpy(), ref["inertia"], rtol=1e-12)


def test_small_batch_strides_and_repeats(rls):
    """Spaces of a batch with rows further apart than they are long; the same call again gives the same, losses included."""
    X = torch.stack([torch.as_tensor(make(k, 1500, 12, i)) for i, k in enumerate(("clusters", "noise", "grid", "wide"))]).cuda()
    got = rls.kmeans_sweep_batched(X, 2, 20, 6, seeds=[4, 5, 6, 7])
    again = rls.kmeans_sweep_batched(X, 2, 20, 6, seeds=[4, 5, 6, 7])
    assert torch.equal(got.inertia, again.inertia) and torch.equal(got.centroids, again.centroids)
    for b in range(4):
        wide = torch.zeros(1500, 17, device="cuda")
        wide[:, 3:15] = X[b]
        one = rls.kmeans_sweep(wide[:, 3:15], 2, 20, 6, seed=4 + b, want_trace=True)
        assert torch.equal(got.labels.reshape(4, 19, -1)[b], one.labels)
        assert torch.equal(got.centroids.reshape(4, -1)[b], one.centroids)


def test_small_sweep_turns_down_bad_data(rls):
    X = torch.as_tensor(make("clusters", 500, 8, 1)).cuda()
    X[17, 3] = float("nan")
    r = rls.kmeans_sweep(X, 1, 8, 3, seed=1, check_status=False)
    assert int(r.status.item()) != 0
