"""Sweeps on the spatially ordered copy of the points, whose blocks meet listed tiles of centroids only, against the same
sweep on the points as they come (taken with a workspace that holds nothing else, and by a sweep that also returns the loss of
every round), bit for bit, losses included, and against the oracle."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rls():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_12799_amd import binding
    binding.lib()
    return binding


def clustered(rng, N, d, spread=1.0):
    centres = rng.uniform(-40, 40, (24, d))
    return np.rint(centres[rng.integers(0, 24, N)] + spread * rng.standard_normal((N, d))).astype(np.float32)


def make(kind, N, d, seed):
    rng = np.random.default_rng(seed)
    if kind == "clusters":
        X = clustered(rng, N, d, 4.0)
    elif kind == "noise":                       # no structure: most units meet most tiles
        X = rng.standard_normal((N, d)).astype(np.float32)
    elif kind == "grid":                        # few distinct rows: exact ties between centroids, long buckets
        X = rng.integers(0, 3, (N, d)).astype(np.float32)
    elif kind == "line":                        # one column carries nearly all of the key
        X = clustered(rng, N, d, 0.01)
        X[:, 0] = rng.uniform(0, 1e4, N)
    elif kind == "same":                        # nothing to order by
        X = np.full((N, d), 3.25, np.float32)
    elif kind == "wide":                        # columns that span more bits than one accumulator keeps
        X = clustered(rng, N, d, 3.0)
        X[:, 1] = (rng.integers(1, 1 << 20, N) * 2.0 ** -30).astype(np.float32)
        X[::7, 1] = 2.0 ** 21
    elif kind == "islands":                     # every column spans 61 binary digits; whoever isolates the far rows has a tiny loss
        X = (rng.integers(0, 1 << 20, (N, d)) * 2.0 ** -40).astype(np.float32)
        X[::7] = 2.0 ** 21
    return X


def as_they_come(rls, X, k_min, k_max, iters, **kw):
    """The sweep with the least workspace.  Where the library would not take an order with a larger one either, there is nothing to
    compare with."""
    batch, (N, d) = (X.shape[0] if X.dim() == 3 else 1), X.shape[-2:]
    least = rls.kmeans_sweep_least_workspace_bytes(N, d, k_min, k_max, batch)
    assert least < rls.kmeans_sweep_workspace_bytes(N, d, k_min, k_max, batch), "this sweep is not an ordered one"
    workspace = torch.empty(least, dtype=torch.uint8, device="cuda")
    return (rls.kmeans_sweep_batched if X.dim() == 3 else rls.kmeans_sweep)(X, k_min, k_max, iters, workspace=workspace, **kw)


def equal(a, b):
    return torch.equal(a.labels, b.labels) and torch.equal(a.centroids, b.centroids) and torch.equal(a.inertia, b.inertia)


# units and chunks that end raggedly, every padded width, groups of 1, 2, 4 and 8 slots per run, groups with and without lists
CASES = [("clusters", 245760, 16, 1, 40), ("clusters", 86017, 13, 8, 63), ("clusters", 90011, 5, 1, 64), ("clusters", 60017, 32, 1, 100),
         ("clusters", 67000, 17, 97, 128), ("clusters", 50001, 8, 1, 110), ("clusters", 70001, 24, 10, 90), ("clusters", 66415, 3, 30, 90),
         ("noise", 86016, 32, 1, 64), ("noise", 96333, 12, 20, 64), ("grid", 99017, 6, 1, 60), ("grid", 96480, 16, 20, 64),
         ("line", 85000, 9, 1, 64), ("line", 86500, 1, 1, 64), ("same", 82400, 8, 1, 65), ("wide", 87000, 7, 1, 64), ("wide", 81000, 20, 10, 64),
         ("islands", 87003, 8, 1, 64), ("islands", 84001, 11, 8, 70), ("islands", 82000, 18, 2, 64)]


@pytest.mark.parametrize("kind,N,d,k_min,k_max", CASES)
def test_ordered_sweep_equals_plain_sweep(rls, kind, N, d, k_min, k_max):
    X = torch.as_tensor(make(kind, N, d, N + d)).cuda()
    got = rls.kmeans_sweep(X, k_min, k_max, 6, seed=3)
    assert equal(got, as_they_come(rls, X, k_min, k_max, 6, seed=3))
    assert equal(got, rls.kmeans_sweep(X, k_min, k_max, 6, seed=3, want_trace=True))
    without = rls.kmeans_sweep(X, k_min, k_max, 6, seed=3, want_labels=False)
    assert torch.equal(got.inertia, without.inertia)


@pytest.mark.parametrize("kind,N,d,k_min,k_max", [("clusters", 87999, 11, 9, 64), ("islands", 90001, 8, 1, 64), ("grid", 50003, 19, 10, 90),
                                                  ("grid", 95003, 16, 8, 64)])
def test_ordered_sweep_against_the_oracle(rls, orc, kind, N, d, k_min, k_max):
    X = make(kind, N, d, 5)
    got = rls.kmeans_sweep(torch.as_tensor(X).cuda(), k_min, k_max, 3, seed=9)
    as_they_come(rls, torch.as_tensor(X).cuda(), k_min, k_max, 1, seed=9)               # (an order is taken)
    ref = orc.kmeans_sweep(X, k_min, k_max, 3, seed=9)
    np.testing.assert_array_equal(got.labels.cpu().numpy(), ref["labels"])
    np.testing.assert_array_equal(got.centroids.cpu().numpy(), ref["centroids"])
    # (the oracle adds the N distances up one after the other: its sum may be N 2^-53 off, 1e-11, and is 1.2e-12)
    np.testing.assert_allclose(got.inertia.cpu().numpy(), ref["inertia"], rtol=N * 2.0 ** -53)


def test_knee_of_an_ordered_sweep_over_columns_of_many_digits(rls, orc):
    """The k at which Algorithm 1 stops, where the losses it compares are 2^-100 of the points' squares."""
    X = make("islands", 90001, 8, 12)
    k, n_done, r = rls.kmeans_sweep_until_knee(torch.as_tensor(X).cuda(), 1, 64, 64, 5, 1.05, seed=7)
    ref = orc.kmeans_sweep(X, 1, 64, 5, seed=7)
    assert n_done == 64
    np.testing.assert_allclose(r.inertia.cpu().numpy(), ref["inertia"], rtol=90001 * 2.0 ** -53)
    assert k == orc.pick_knee(ref["inertia"], 1, 64, 1.05)


def test_ordered_sweep_of_strided_rows_and_given_centres(rls):
    """Rows further apart than they are long, initial centres that name one point twice; the same call again gives the same."""
    full = torch.as_tensor(make("clusters", 100003, 16, 8)).cuda()
    X = full[:, 1:14]
    init = torch.arange(0, 100003, 1500, device="cuda", dtype=torch.int64)[:64].clone()
    init[7] = init[3]
    got = rls.kmeans_sweep(X, 1, 64, 5, init_idx=init)
    again = rls.kmeans_sweep(X, 1, 64, 5, init_idx=init)
    want = as_they_come(rls, X.contiguous(), 1, 64, 5, init_idx=init)
    assert equal(got, want) and equal(again, want)


# chunks of their own for every group, and the same chunks for all (19 and 5 spaces: a number of chunks that eight does not divide)
@pytest.mark.parametrize("batch,N,d,k_min,k_max", [(3, 82421, 10, 1, 40), (19, 20011, 9, 8, 50), (5, 20003, 27, 1, 100)])
def test_ordered_batch_and_smaller_workspace(rls, batch, N, d, k_min, k_max):
    """Spaces of a batch are ordered one by one; a workspace that only holds the sweep as it comes takes it without an order."""
    kinds = ("clusters", "noise", "grid")
    X = torch.stack([torch.as_tensor(make(kinds[i % 3], N, d, i)) for i in range(batch)]).cuda()
    seeds = [4 + i for i in range(batch)]
    got = rls.kmeans_sweep_batched(X, k_min, k_max, 5, seeds=seeds)
    assert equal(got, as_they_come(rls, X, k_min, k_max, 5, seeds=seeds))


def test_waves_until_the_knee_share_the_order(rls):
    X = torch.as_tensor(make("clusters", 500011, 14, 2)).cuda()
    init = rls.kmeanspp_chain(X, 60, 11)
    k, n_done, r = rls.kmeans_sweep_until_knee(X, 17, 60, 16, 5, 1e-9, seed=11)        # the knee never fires: all waves run
    assert n_done == 44
    for k_lo in (17, 33, 49):                                  # (the losses are added up by the plan of a wave)
        k_hi = min(k_lo + 15, 60)
        want = as_they_come(rls, X, k_lo, k_hi, 5, init_idx=init[:k_hi])
        rows = slice(14 * sum(range(17, k_lo)), 14 * sum(range(17, k_hi + 1)))
        assert torch.equal(r.labels[k_lo - 17:k_hi - 16], want.labels) and torch.equal(r.centroids[rows], want.centroids)
        assert torch.equal(r.inertia[k_lo - 17:k_hi - 16], want.inertia)


def test_last_wave_of_one_small_k_does_without_the_order(rls):
    X = torch.as_tensor(make("clusters", 480011, 5, 3)).cuda()
    init = rls.kmeanspp_chain(X, 32, 2)
    as_they_come(rls, X, 16, 31, 1, init_idx=init)             # (the first wave takes an order)
    k, n_done, r = rls.kmeans_sweep_until_knee(X, 16, 32, 16, 3, 1e-9, seed=2)
    assert n_done == 17
    want = rls.kmeans_sweep(X, 32, 32, 3, init_idx=init)
    assert torch.equal(r.labels[16:], want.labels) and torch.equal(r.centroids[-32 * 5:], want.centroids) and torch.equal(r.inertia[16:], want.inertia)


@pytest.mark.parametrize("N,d,k_min,k_max", [(3000, 8, 1, 20), (40003, 16, 1, 24), (90011, 12, 1, 64), (60017, 32, 1, 100)])
def test_rows_scaled_by_a_power_of_two(rls, N, d, k_min, k_max):
    """Nothing rounds differently, up to the largest floats and their differences (which no float holds)."""
    X = torch.as_tensor(make("clusters", N, d, 8)).cuda()
    X[0], X[1] = 63.0, -63.0
    want = rls.kmeans_sweep(X, k_min, k_max, 4, seed=3)
    for s in (-60, 90, 110, 112, 116, 122):
        got = rls.kmeans_sweep(X * 2.0 ** s, k_min, k_max, 4, seed=3)
        assert torch.equal(got.labels, want.labels)
        assert torch.equal(got.centroids, want.centroids * 2.0 ** s)
        assert torch.equal(got.inertia, want.inertia * 2.0 ** (2 * s))


def test_ordered_sweep_in_a_graph(rls):
    """Recorded once and replayed with eager work in between: every replay gives the eager result."""
    X = torch.as_tensor(make("clusters", 90011, 16, 4)).cuda()
    ws = torch.empty(rls.kmeans_sweep_workspace_bytes(90011, 16, 1, 64, 1) + 256, dtype=torch.uint8, device="cuda")
    init = rls.kmeanspp_chain(X, 64, 5)
    sweep = lambda: rls.kmeans_sweep(X, 1, 64, 5, init_idx=init, workspace=ws, check_status=False)
    want = [t.clone() for t in (lambda r: (r.labels, r.centroids, r.inertia))(sweep())]
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        sweep()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side):
            res = sweep()
    torch.cuda.current_stream().wait_stream(side)
    for rep in range(3):
        for t in (res.labels, res.centroids, res.inertia):
            t.zero_()
        rls.kmeans_sweep(X[:30000], 2, 20, 2, seed=rep)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert int(res.status.item()) == 0
        for got, exp in zip((res.labels, res.centroids, res.inertia), want):
            assert torch.equal(got, exp), f"replay {rep}"


@pytest.mark.parametrize("iters,want_trace", [(0, False), (1, False), (4, True)])
def test_sweeps_that_would_not_read_the_order_do_without(rls, iters, want_trace):
    """A loss trace, or fewer than two rounds: the same sweep, to the last bit of its losses, as without an order at hand."""
    X = torch.as_tensor(make("noise", 90011, 16, 6)).cuda()
    got = rls.kmeans_sweep(X, 1, 64, iters, seed=5, want_trace=want_trace)
    want = as_they_come(rls, X, 1, 64, iters, seed=5, want_trace=want_trace)
    assert equal(got, want)
    assert not want_trace or torch.equal(got.trace, want.trace)


def test_ordered_sweep_turns_down_bad_data(rls):
    X = torch.as_tensor(make("clusters", 90011, 16, 4)).cuda()
    X[80000, 3] = float("inf")
    assert int(rls.kmeans_sweep(X, 1, 64, 2, seed=1, check_status=False).status.item()) & rls.RLS_STATUS_NONFINITE


def list_lengths(rls, workspace, N, d, k_min, k_max):
    """How many tiles the units of the sweep that last used the workspace met in its last round, per group with lists."""
    at, words = ctypes.c_int64(0), ctypes.c_int64(0)
    assert rls.lib().rls_sweep_tile_lists(ctypes.c_int64(N), d, k_min, k_max, ctypes.byref(at), ctypes.byref(words)) == 0
    assert words.value > 0, "this sweep is not an ordered one"
    base = -workspace.data_ptr() % 256 + at.value
    lists = workspace[base:base + 4 * words.value].view(torch.int32).view(-1, 16).cpu().numpy().view(np.uint32)
    lengths = (lists[:, :8] >> 28) + 1
    assert np.all(lengths == lengths[:, :1])
    units = -(-N // (64 if d > 16 else 32))
    return lengths[:, 0].reshape(-1, units)


# `found`: lengths that have to occur.  (A unit that would leave out one tile of many meets them all: 15 of 16 are never listed.)
@pytest.mark.parametrize("kind,N,d,k_min,k_max,found", [("noise", 120017, 4, 20, 64, range(1, 14)), ("noise", 150001, 16, 25, 64, (12, 14, 16)),
                                                        ("clusters", 200001, 2, 33, 64, (1, 2)), ("noise", 60001, 30, 40, 90, (7, 8, 9))])
def test_lists_of_seven_and_more_tiles(rls, orc, kind, N, d, k_min, k_max, found):
    """Units that meet up to all sixteen tiles of a group: entries of a list's second word, and the sixteenth."""
    rows = make(kind, N, d, 21)
    X = torch.as_tensor(rows).cuda()
    workspace = torch.zeros(rls.kmeans_sweep_workspace_bytes(N, d, k_min, k_max) + 256, dtype=torch.uint8, device="cuda")
    got = rls.kmeans_sweep(X, k_min, k_max, 4, seed=6, workspace=workspace)
    lengths = list_lengths(rls, workspace, N, d, k_min, k_max)
    print([(int(n), int((lengths == n).sum())) for n in np.unique(lengths)])
    assert set(found) <= set(np.unique(lengths).tolist()) and lengths.max() <= 16
    assert equal(got, as_they_come(rls, X, k_min, k_max, 4, seed=6))
    ref = orc.kmeans_sweep(rows, k_min, k_max, 4, seed=6)
    np.testing.assert_array_equal(got.labels.cpu().numpy(), ref["labels"])
    np.testing.assert_array_equal(got.centroids.cpu().numpy(), ref["centroids"])
