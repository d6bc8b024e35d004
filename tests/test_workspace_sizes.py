"""Workspace queries (host only, no GPU): what fitted the fixed workspace of rls_kmeans_sweep_static goes on fitting it."""
import ctypes
import os

import pytest

from tests.test_zz_no_alloc import EDGE


@pytest.fixture(scope="module")
def library():
    from paper_1905_12799_amd import build
    if not os.path.exists(build.LIB):
        build.build_library()
    lib = ctypes.CDLL(build.LIB)
    for fn in (lib.rls_kmeans_sweep_workspace_bytes, lib.rls_kmeans_sweep_least_workspace_bytes):
        fn.restype = ctypes.c_int64
        fn.argtypes = [ctypes.c_int64] + [ctypes.c_int32] * 4
    return lib


@pytest.mark.parametrize("N,d,k_min,k_max", EDGE)
def test_fits_the_fixed_workspace(library, N, d, k_min, k_max):
    assert 0 < library.rls_kmeans_sweep_workspace_bytes(N, d, k_min, k_max, 1) <= 64 << 20


@pytest.mark.parametrize("N,d,k_min,k_max,batch,ordered", [
    (2000, 8, 1, 16, 1, False), (65536, 16, 1, 64, 1, False), (1048576, 16, 32, 32, 1, False),
    # what an order costs these is more than it saves: 4 to 13% over 10 to 22 rounds of knob configurations
    (17549, 32, 1, 106, 1, False), (134029, 16, 8, 15, 13, False), (880164, 32, 1, 20, 1, False), (55202, 21, 8, 48, 1, False),
    # many points and few tiles: 13 to 17% less with an order
    (8388608, 32, 1, 16, 1, True), (6000000, 12, 8, 19, 1, True),
    (300007, 13, 8, 63, 1, True), (1048576, 16, 1, 64, 1, True), (262144, 16, 1, 32, 64, True), (8388608, 32, 1, 128, 1, True)])
def test_least_workspace(library, N, d, k_min, k_max, batch, ordered):
    """Equal where the points are taken as they come anyway; less where the larger one holds a copy of the rows in order."""
    best = library.rls_kmeans_sweep_workspace_bytes(N, d, k_min, k_max, batch)
    least = library.rls_kmeans_sweep_least_workspace_bytes(N, d, k_min, k_max, batch)
    assert 0 < least <= best and least % 256 == 0 and best % 256 == 0
    assert best - least >= batch * N * d * 4 if ordered else best == least


def test_least_workspace_refuses_what_the_other_refuses(library):
    for shape in ((0, 8, 1, 16, 1), (1000, 33, 1, 16, 1), (1000, 8, 5, 4, 1), (10, 8, 1, 16, 1), (1000, 8, 1, 129, 1), (1000, 8, 1, 16, 0)):
        assert library.rls_kmeans_sweep_least_workspace_bytes(*shape) == library.rls_kmeans_sweep_workspace_bytes(*shape) == -1


def test_fixed_workspace_goes_by_the_least(library):
    """A shape that fits the fixed workspace as the points come, and not with their order."""
    assert library.rls_kmeans_sweep_least_workspace_bytes(300007, 13, 8, 63, 1) <= 64 << 20 < library.rls_kmeans_sweep_workspace_bytes(300007, 13, 8, 63, 1)
