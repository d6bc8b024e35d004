"""Which path a rule on sizes takes, for the cases of the GPU tests that are there for one of the paths (no GPU needed)."""
import pytest

from paper_1905_12799_amd import binding as rls
from tests import test_gpu_parity as gpu


@pytest.mark.parametrize("batch,k,knobs,lanes", gpu.SNAP_ROWS)
def test_snap_lanes(batch, k, knobs, lanes):
    assert rls.lib().rls_snap_lanes(batch, k, knobs) == lanes


def test_snap_cases_lie_on_both_sides():
    assert {c[3] for c in gpu.SNAP_ROWS} == {1, 64}
    assert rls.lib().rls_snap_lanes(1, 0, 8) == rls.lib().rls_snap_lanes(1, 4, 33) == -1


@pytest.mark.parametrize("batch,N,d,k,limit,at_once", gpu.SPACES_IN_PARTS)
def test_seeding_in_parts(batch, N, d, k, limit, at_once):
    assert gpu.spaces_at_once(rls, batch, N, d, k) == at_once
    assert 0 < at_once < min(batch, 64)


@pytest.mark.parametrize("N,d,gap", gpu.MANY_SPACES)
def test_seeding_of_many_spaces_in_parts(N, d, gap):
    assert gpu.spaces_at_once(rls, 70, N, d, 6, gap) == 51
    assert gpu.spaces_at_once(rls, 6, N, d, 6, gap) == 6          # (what comes after the first 64)


@pytest.mark.parametrize("batch,N,d,gap,k", gpu.WALKED_SPACES)
def test_seeding_walked(batch, N, d, gap, k):
    assert gpu.spaces_at_once(rls, batch, N, d, k, gap) == 0


def test_seeding_on_smaller_chips():
    """The rule goes by the compute units at hand: what is one launch on 256 goes in parts on 64, and a space that fits no chip is walked."""
    assert gpu.spaces_at_once(rls, 8, 65536, 16, 32) == 8
    assert gpu.spaces_at_once(rls, 8, 65536, 16, 32, compute_units=64) == 4
    assert gpu.spaces_at_once(rls, 1, 1 << 20, 16, 32) == 1
    assert gpu.spaces_at_once(rls, 1, (1 << 20) + 1, 16, 32) == 0
    assert gpu.spaces_at_once(rls, 1, 1 << 20, 16, 32, compute_units=64) == 0


@pytest.mark.parametrize("N,d,T,D", gpu.SLICE_THAT_ADDS)
def test_score_with_a_slice_that_adds(N, d, T, D):
    tile, side, trees, apart = gpu.score_plan(rls, N, d, T, D)
    assert (tile, side, apart) == (256, 4, 1)
    assert 32 <= trees < T


def test_score_without_one():
    """One chunk, few trees a chunk, other tiles."""
    for N, d, T, D in ((60001, 8, 32, 8), (50000, 32, 256, 10), (1 << 20, 16, 256, 8), (2000, 8, 64, 6), (30000, 32, 256, 8)):
        assert gpu.score_plan(rls, N, d, T, D)[3] == 0
