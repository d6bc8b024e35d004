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
