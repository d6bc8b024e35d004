"""The bound within which two distances of the matrix pipeline are settled with the exact arithmetic (`pair_error_of` in
paper_1905_12799_amd/csrc/lloyd_device.h): what the instructions leave out, measured one by one and over the whole chain of a distance,
and labels of points whose two nearest centroids lie on either side of it."""
import ctypes

import numpy as np
import pytest
import torch

from tests.matrix_model import FAMILIES, UNIT, distances, exact_distances, near_ties, operands, padded, pair_error, point_norm, step_model

pytestmark = pytest.mark.gpu

LANE = np.arange(64)
ROWS = 8 * (np.arange(16) // 4) + 4 * (LANE[:, None] // 32) + np.arange(16) % 4
COLS = np.repeat(LANE[:, None] % 32, 16, 1)


@pytest.fixture(scope="module")
def rls():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_12799_amd import binding
    binding.lib()
    return binding


@pytest.fixture(scope="module")
def step(rls):
    fn = rls.lib().rls_matrix_step
    fn.restype = ctypes.c_int32
    fn.argtypes = [ctypes.c_int32] + [ctypes.c_void_p] * 4 + [ctypes.c_int32, ctypes.c_void_p]

    def half(v, bf16):                           # as 16-bit patterns; the values are ones that the type holds
        v = np.ascontiguousarray(v, np.float32)
        return (v.view(np.uint32) >> 16).astype(np.uint16) if bf16 else v.astype(np.float16).view(np.uint16)

    def run(A, B, acc, bf16):
        n = A.shape[0]
        assert A.shape == (n, 32, 16) and B.shape == (n, 16, 32) and acc.shape == (n, 32, 32)
        a = half(A, bf16).reshape(n, 32, 2, 8).swapaxes(1, 2)                           # [n][half of K][row][8]
        b = half(np.swapaxes(B, 1, 2), bf16).reshape(n, 32, 2, 8).swapaxes(1, 2)
        a, b = (torch.as_tensor(np.ascontiguousarray(v).view(np.int16)).cuda() for v in (a, b))
        c = torch.as_tensor(np.ascontiguousarray(acc[:, ROWS, COLS], np.float32)).cuda()
        assert a.numel() == n * 64 * 8 and b.numel() == n * 64 * 8 and c.numel() == n * 64 * 16
        out = torch.empty_like(c)
        assert fn(int(bf16), a.data_ptr(), b.data_ptr(), c.data_ptr(), out.data_ptr(), n, torch.cuda.current_stream().cuda_stream) == 0
        d = np.empty((n, 32, 32), np.float32)
        d[:, ROWS, COLS] = out.cpu().numpy()
        return d
    return run


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("spread", [0, 1, 3, 6])
def test_one_instruction(step, spread, bf16):
    """Against the model: equal, but for one result in a hundred at most, which has one of its two roundings the other way (where the
    accumulator is far above the products: a unit in the last place of the largest term)."""
    rng = np.random.default_rng(10 * spread + bf16)
    n = 16

    def values(shape):
        v = (rng.uniform(1, 2, shape) * 2.0 ** rng.integers(-spread, spread + 1, shape) * rng.choice([-1, 1], shape)).astype(np.float32)
        return (v.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32) if bf16 else v.astype(np.float16).astype(np.float32)

    A, B = values((n, 32, 16)), values((n, 16, 32))
    exact = np.matmul(A.astype(np.float64), B.astype(np.float64))
    twin = np.concatenate([A[:, :, :8], A[:, :, :8]], axis=2), np.concatenate([B[:, :8], -B[:, :8]], axis=1)     # halves that cancel
    noise = rng.standard_normal((n, 32, 32))
    for a, b, acc in [(A, B, noise * s) for s in (0.0, 2.0 ** -20, 2.0 ** -6, 1.0, 2.0 ** 10, 2.0 ** 22)] + \
                     [(A, B, -exact * (1 + 2.0 ** -12 * noise)), (*twin, noise * 2.0 ** -15)]:
        acc = acc.astype(np.float32)
        got, want = step(a, b, acc, bf16), step_model(a, b, acc)
        terms = np.abs(acc) + np.matmul(np.abs(a), np.abs(b))
        off = np.abs(got.astype(np.float64) - want) / np.spacing(terms)
        share, worst = float((got != want).mean()), float(off.max())
        assert share <= 0.01 and worst <= 1.0


@pytest.mark.parametrize("family", FAMILIES)
@pytest.mark.parametrize("dp", [8, 16, 32])
def test_distances_stay_within_half_of_the_bound(step, dp, family):
    """Half of the bound is for each of two distances; two units of it are for the centring, which these operands have behind them."""
    rng = np.random.default_rng(dp + FAMILIES.index(family))
    x, c = operands(family, dp, 64, rng)
    xnorm = point_norm(x)
    got = distances(x, c, xnorm, dp, step).astype(np.float64)
    S = (x.astype(np.float64) ** 2).sum(-1)[:, None, :] + (c.astype(np.float64) ** 2).sum(-1)[:, :, None]
    worst = float(((np.abs(got - exact_distances(x, c, xnorm)) - 0.0781 * dp) / (UNIT * S)).max())
    print(f"d_pad {dp}, {family}: {worst:.2f} units besides the floor")
    assert worst <= pair_error(dp) / 2 - 2


# every padded width and number of slots per run, the sweep of one launch (3000 rows, one round), an ordered one (90,011 rows, two rounds)
@pytest.mark.parametrize("N,d,k_min,k,iters", [(20003, 8, 2, 2, 0), (20003, 6, 16, 16, 0), (20003, 16, 2, 2, 0), (20003, 13, 64, 64, 0),
                                               (20003, 16, 9, 32, 0), (20003, 32, 2, 2, 0), (20003, 27, 100, 128, 0), (20003, 32, 40, 64, 0),
                                               (3001, 8, 2, 16, 1), (3001, 16, 2, 2, 1), (1201, 32, 2, 16, 1), (90011, 16, 8, 64, 2),
                                               (60017, 32, 20, 100, 2)])
def test_labels_of_points_near_the_bound(rls, orc, N, d, k_min, k, iters):
    rng = np.random.default_rng(N + d + k)
    X, gap, own = near_ties(rng, N, d, k)
    dp = padded(d)
    for lo, hi in ((0, 4), (4, pair_error(dp) / 2), (pair_error(dp) / 2, pair_error(dp)), (pair_error(dp), 3 * pair_error(dp))):
        assert ((np.abs(gap) >= lo) & (np.abs(gap) < hi)).sum() >= (N - k) // 100, "the distances differ by all of that"
    init = np.arange(k, dtype=np.int64)
    got = rls.kmeans_sweep(torch.as_tensor(X).cuda(), k_min, k, iters, init_idx=torch.as_tensor(init).cuda())
    ref = orc.kmeans_sweep(X, k_min, k, iters, init_idx=init)
    if iters == 0:
        near = ref["labels"][-1][k:] // 2 == own                                        # (the inputs are what they are meant to be)
        assert near.mean() > 0.999
        np.testing.assert_array_equal(ref["labels"][-1][k:][near], np.where(gap < 0, 2 * own, 2 * own + 1)[near])
    np.testing.assert_array_equal(got.labels.cpu().numpy(), ref["labels"])
    np.testing.assert_array_equal(got.centroids.cpu().numpy(), ref["centroids"])
