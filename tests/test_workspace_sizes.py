"""Workspace queries (host only, no GPU): what fitted the fixed workspace of rls_kmeans_sweep_static goes on fitting it."""
import ctypes
import os

import pytest

from tests.test_zz_no_alloc import EDGE


@pytest.fixture(scope="module")
def query():
    from paper_1905_12799_amd import build
    if not os.path.exists(build.LIB):
        build.build_library()
    fn = ctypes.CDLL(build.LIB).rls_kmeans_sweep_workspace_bytes
    fn.restype = ctypes.c_int64
    fn.argtypes = [ctypes.c_int64] + [ctypes.c_int32] * 4
    return fn


@pytest.mark.parametrize("N,d,k_min,k_max", EDGE)
def test_fits_the_fixed_workspace(query, N, d, k_min, k_max):
    assert 0 < query(N, d, k_min, k_max, 1) <= 64 << 20
