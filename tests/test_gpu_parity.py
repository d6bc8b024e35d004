"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the same seeded inputs.

Bars: bit-exact for labels, snapped configurations, chosen k and seeding indices (labels except points whose
two nearest centroids differ by less than 1e-6 relative, in the oracle's fp64 distances); 1e-5 relative
for centroids (per column scale), inertia and tree scores (scores are also compared bit for bit with the
oracle's fp32 tree-order sum).
"""
import ctypes
import threading

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


def dev(a):
    return torch.as_tensor(a).cuda()


# ----------------------------------------------------------------------------------------------
def check_scores(rls, orc, forest, X):
    got = rls.gbt_score(rls.DeviceForest.from_host(forest), dev(X)).cpu().numpy()
    s32, s64 = orc.gbt_score(forest, X)
    np.testing.assert_array_equal(got, s32)
    scale = np.maximum(np.abs(s64), 1.0)
    assert np.all(np.abs(got.astype(np.float64) - s64) <= 1e-5 * scale * max(1.0, forest.n_trees ** 0.5))


def test_gbt_score_tiny(rls, orc):
    p = synth.make_problem(synth.WORKLOADS["tiny"])
    check_scores(rls, orc, p.forest, p.X)


@pytest.mark.parametrize("N,d,T,D", [(1, 8, 3, 1), (1025, 8, 5, 3), (3000, 16, 40, 8), (777, 32, 9, 10),
                                     (2049, 5, 7, 12), (4096, 16, 70, 6),
                                     # many shallow trees: more leaves per byte of forest than deep trees have
                                     (600, 32, 1200, 3), (700, 20, 4500, 1), (513, 32, 2300, 2), (1100, 16, 9000, 1),
                                     (300, 24, 3, 12), (900, 8, 300, 4),
                                     # tiles of 1024 and of 896 configurations, chunks of 4, 2 and 1 trees, chunks moved
                                     # four entries at a time and (a last chunk of 3 trees, 30 features) one at a time
                                     (2000, 32, 23, 10), (1800, 32, 24, 10), (1100, 32, 13, 9), (950, 32, 5, 11),
                                     (900, 32, 3, 12), (1030, 16, 7, 11), (1900, 30, 10, 10), (2100, 32, 64, 8)])
def test_gbt_score_shapes(rls, orc, N, d, T, D):
    rng = np.random.default_rng(N + d)
    X = rng.standard_normal((N, d)).astype(np.float32)
    f = synth.random_forest(X, T, D, 0, rng)
    f.base = 0.25
    # plant exact equality with a threshold: must go right
    f.thr[0, 0] = X[0, f.feat[0, 0]]
    check_scores(rls, orc, f, X)


@pytest.mark.parametrize("N,d,T,D", [
    # tiles of 64 ... 1024 configurations (by the number of rows), full and with one configuration more or less
    (63, 8, 64, 6), (64, 8, 65, 6), (2001, 7, 130, 6), (16385, 8, 33, 5), (32769, 16, 50, 7), (65535, 8, 256, 8), (131073, 5, 40, 4),
    (262145, 32, 12, 6),
    # trees that leave slices idle, fewer trees than slices, one tree, chunks that hold few deep trees
    (200, 8, 1, 3), (300, 16, 5, 1), (500, 32, 21, 9), (130, 32, 37, 11), (70, 24, 18, 12)])
def test_gbt_score_tiles_and_slices(rls, orc, N, d, T, D):
    rng = np.random.default_rng(N + T)
    X = rng.standard_normal((N, d)).astype(np.float32)
    f = synth.random_forest(X, T, D, 0, rng)
    f.base = -0.5
    check_scores(rls, orc, f, X)


# tiles of 256: a slice that adds while the others move (32 and more trees a chunk), last chunks of 6 and 3 trees, and the fewest nodes
SLICE_THAT_ADDS = [(60001, 8, 150, 8), (50003, 16, 99, 8), (65000, 8, 200, 6), (64999, 24, 130, 7)]


def score_plan(rls, N, d, T, D, batch=1):
    out = [ctypes.c_int32() for _ in range(4)]
    assert rls.lib().rls_score_plan(ctypes.c_int64(N), d, batch, T, D, *[ctypes.byref(o) for o in out]) == 0
    return [o.value for o in out]


@pytest.mark.parametrize("N,d,T,D", SLICE_THAT_ADDS)
def test_gbt_score_slice_that_adds(rls, orc, N, d, T, D):
    assert score_plan(rls, N, d, T, D)[3] == 1
    rng = np.random.default_rng(N + T)
    X = rng.standard_normal((N, d)).astype(np.float32)
    f = synth.random_forest(X, T, D, 0, rng)
    check_scores(rls, orc, f, X)


def test_gbt_score_batched_forests_of_different_shapes(rls, orc):
    """Spaces whose forests share a shape go into one launch (at most 64 of them), the others into launches of their own."""
    rng = np.random.default_rng(5)
    shapes = [(20, 5)] * 3 + [(20, 6)] + [(7, 6)] * 2 + [(20, 5)] * 66
    X = rng.standard_normal((len(shapes), 333, 9)).astype(np.float32)
    forests = [synth.random_forest(X[b], T, D, 0, rng) for b, (T, D) in enumerate(shapes)]
    got = rls.gbt_score_batched([rls.DeviceForest.from_host(f) for f in forests], dev(X)).cpu().numpy()
    for b, f in enumerate(forests):
        np.testing.assert_array_equal(got[b], orc.gbt_score(f, X[b])[0])


def test_gbt_score_feature_index_out_of_range_reads_the_border_column(rls, orc):
    """The library documents that a feature index outside [0, d) reads column 0 or d - 1 (the oracle rejects such a
    forest): the scores equal the oracle's on the forest with its indices brought inside."""
    rng = np.random.default_rng(17)
    X = rng.standard_normal((900, 12)).astype(np.float32)
    f = synth.random_forest(X, 20, 5, 0, rng)
    bad = synth.Forest(f.n_trees, f.depth, f.n_features, f.base, f.feat.copy(), f.thr, f.leaf)
    bad.feat[::3, ::2] = 12 + rng.integers(0, 1000, size=bad.feat[::3, ::2].shape)
    bad.feat[1::3, 1::2] = -1 - rng.integers(0, 1000, size=bad.feat[1::3, 1::2].shape)
    with pytest.raises(RuntimeError):
        orc.gbt_score(bad, X)
    inside = synth.Forest(f.n_trees, f.depth, f.n_features, f.base, np.clip(bad.feat, 0, 11), f.thr, f.leaf)
    got = rls.gbt_score(rls.DeviceForest.from_host(bad), dev(X)).cpu().numpy()
    np.testing.assert_array_equal(got, orc.gbt_score(inside, X)[0])


def test_gbt_score_forest_arrays_not_16_byte_aligned(rls, orc):
    """Forest arrays that start 4 bytes past a 16-byte boundary (views into larger buffers): same scores."""
    rng = np.random.default_rng(23)
    X = rng.standard_normal((1500, 32)).astype(np.float32)
    f = synth.random_forest(X, 16, 10, 0, rng)

    def shifted(a):
        buf = torch.empty(a.size + 1, dtype=torch.as_tensor(a).dtype, device="cuda")
        buf[1:] = torch.as_tensor(a).reshape(-1).cuda()
        v = buf[1:].view(a.shape)
        assert v.data_ptr() % 16 == 4
        return v

    F = rls.DeviceForest(f.n_trees, f.depth, f.n_features, f.base, shifted(f.feat), shifted(f.thr), shifted(f.leaf))
    assert F.feat.data_ptr() % 16 == 4 and F.thr.data_ptr() % 16 == 4 and F.leaf.data_ptr() % 16 == 4
    got = rls.gbt_score(F, dev(X)).cpu().numpy()
    np.testing.assert_array_equal(got, orc.gbt_score(f, X)[0])


def test_gbt_score_mid_subset(rls, orc):
    p = synth.make_problem(synth.WORKLOADS["mid"], N=20000)
    check_scores(rls, orc, p.forest, p.X)


def test_gbt_score_strided_rows(rls, orc):
    rng = np.random.default_rng(0)
    Xw = rng.standard_normal((1500, 20)).astype(np.float32)
    f = synth.random_forest(Xw[:, :16], 11, 5, 0, rng)
    got = rls.gbt_score(rls.DeviceForest.from_host(f), dev(Xw)[:, :16])   # ldx = 20
    s32, _ = orc.gbt_score(f, np.ascontiguousarray(Xw[:, :16]))
    np.testing.assert_array_equal(got.cpu().numpy(), s32)


def test_gbt_score_batched(rls, orc):
    w = synth.WORKLOADS["batched"]
    probs = synth.make_batched_problems(w, batch=3, N=5000)
    X = np.stack([p.X for p in probs])
    forests = [rls.DeviceForest.from_host(p.forest) for p in probs]
    got = rls.gbt_score_batched(forests, dev(X)).cpu().numpy()
    for b, p in enumerate(probs):
        np.testing.assert_array_equal(got[b], orc.gbt_score(p.forest, p.X)[0])


# ----------------------------------------------------------------------------------------------
def test_snap_matches_oracle(rls, orc):
    p = synth.make_problem(synth.WORKLOADS["mid"], N=64)
    rng = np.random.default_rng(1)
    C = (p.X + rng.uniform(-0.75, 0.75, size=p.X.shape)).astype(np.float32)
    C[:8, :8] = np.floor(C[:8, :8]) + 0.5          # exact half-way cases
    C[8:12, :8] = -3.0                              # below every domain
    C[12:16, :8] = 1e6                              # above every domain
    got = rls.snap_to_valid(dev(C), rls.DeviceDomains(p.dom_offsets, p.dom_values)).cpu().numpy()
    np.testing.assert_array_equal(got, orc.snap_to_valid(C, p.dom_offsets, p.dom_values))


def test_snap_irregular_domains_and_batched(rls, orc):
    rng = np.random.default_rng(2)
    sizes = [5, 1, 9, 3]
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    doms, Cs = [], []
    for b in range(3):
        values = np.concatenate([np.sort(rng.uniform(-5, 5, size=s)) for s in sizes]).astype(np.float32)
        doms.append((offsets, values))
        Cs.append(rng.uniform(-7, 7, size=(17, 6)).astype(np.float32))
    got = rls.snap_to_valid_batched(dev(np.stack(Cs)), [rls.DeviceDomains(o, v) for o, v in doms]).cpu().numpy()
    for b in range(3):
        np.testing.assert_array_equal(got[b], orc.snap_to_valid(Cs[b], *doms[b]))


# either side of the number of pairs that a wave each takes, one space and more than a launch holds; knobs that do not divide a workgroup;
# so many rows that a workgroup takes several turns, and a wave each would be a launch of 2^32 threads
SNAP_ROWS = [(1, 4096, 8, 64), (1, 4097, 8, 1), (1, 1025, 32, 1), (1, 32769, 1, 1), (64, 64, 8, 64), (66, 65, 8, 1), (3, 2999, 5, 1), (1, 1 << 23, 8, 1)]


@pytest.mark.parametrize("batch,k,knobs,lanes", SNAP_ROWS)
def test_snap_of_few_and_of_many_rows(rls, orc, batch, k, knobs, lanes):
    assert rls.lib().rls_snap_lanes(batch, k, knobs) == lanes
    rng = np.random.default_rng(k + knobs)
    doms = []
    for _ in range(batch):
        sizes = [2, 3, 9, 17] if k < 1 << 20 else [2, 3]
        sizes = (sizes * 8)[:knobs]
        parts = [rng.permutation(rng.integers(0, 2 * s, s)).astype(np.float32) for s in sizes]
        doms.append((np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32), np.concatenate(parts)))
    C = (rng.integers(-4, 36, size=(batch, k, min(knobs + 1, 32)), dtype=np.int8) * np.float32(0.5)).astype(np.float32)
    C[:, 0, 0], C[:, 1, 0], C[:, -1, 0] = np.nan, np.inf, -np.inf
    got = rls.snap_to_valid_batched(dev(C), [rls.DeviceDomains(*dom) for dom in doms]).cpu().numpy()
    for b in range(batch):
        np.testing.assert_array_equal(got[b], orc.snap_to_valid(C[b], *doms[b]))


# sizes around the lanes of a wave and the values it reads at a time; more knobs than are searched side by side; rows around a workgroup's
@pytest.mark.parametrize("sizes,n,order", [([1, 2, 3, 8, 9, 63, 64, 65, 127], 257, "sorted"), ([255, 256, 257, 300, 1000], 1023, "sorted"),
                                           ([511, 513, 5, 1, 70, 64, 33, 17, 9, 2, 40], 255, "shuffled"), ([64, 300, 9, 8], 131073, "repeats"), ([220], 1, "sorted"),
                                           # some knobs sorted and some not, in groups of eight and beyond; rows that are searched one knob after the other
                                           ([300, 9, 40, 2, 70, 5, 17, 64, 33, 220], 1025, "mixed"), ([300, 9, 40, 2, 70, 5, 17, 64, 33], (1 << 20) + 77, "mixed"),
                                           ([64, 300, 9, 8], (1 << 20) + 1, "repeats"), ([220, 40, 2], 1 << 20, "sorted")])
def test_nearest_entries_over_domain_sizes(rls, orc, sizes, n, order):
    """Snap, histogram and mode: nearest entry and first of equal ones, whichever lane or step has them."""
    rng = np.random.default_rng(sum(sizes) + n)
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    parts = [np.sort(rng.permutation(4 * s)[:s]).astype(np.float32) for s in sizes]
    if order == "repeats":
        parts = [np.sort(rng.integers(0, max(2, s // 3), s)).astype(np.float32) for s in sizes]
    if order in ("shuffled", "mixed"):
        parts = [rng.permutation(q) if order == "shuffled" or j % 3 == 1 else q for j, q in enumerate(parts)]
    values = np.concatenate(parts)
    X = (rng.integers(-4, 8 * np.array(sizes) + 4, size=(n, len(sizes))) * 0.5).astype(np.float32)      # half-way cases among them
    dom = rls.DeviceDomains(offsets, values)
    mode, hist = rls.knob_modes(dev(X), dom)
    mode_o, hist_o = orc.knob_modes(X, offsets, values)
    np.testing.assert_array_equal(hist.cpu().numpy().astype(np.int64), hist_o)
    np.testing.assert_array_equal(mode.cpu().numpy(), mode_o)
    C = X[:300].copy()
    C[:1, 0], C[1:2, 0], C[2:3, 0] = np.nan, np.inf, -np.inf
    np.testing.assert_array_equal(rls.snap_to_valid(dev(C), dom).cpu().numpy(), orc.snap_to_valid(C, offsets, values))


@pytest.mark.parametrize("k,knobs,n", [(1, 1, 1), (64, 3, 255), (65, 4, 257), (130, 5, 70001), (3, 9, 300000)])
def test_visited_over_samples_and_knobs(rls, orc, k, knobs, n):
    """Samples around those of a workgroup, rows of fewer and more knobs than are compared first, several rows per thread."""
    rng = np.random.default_rng(k + n)
    top = max(2, int(round(n ** (1.0 / knobs))) + 1)
    visited = rng.integers(0, top, (n, knobs)).astype(np.int32)
    cfg = rng.integers(0, top, (k, knobs)).astype(np.int32)
    cfg[-1] = visited[-1]
    mode = np.full(knobs, top, dtype=np.int32)
    got = dev(cfg)
    flags = rls.replace_visited(got, dev(visited), dev(mode)).cpu().numpy()
    want, want_flags = orc.replace_visited(cfg, visited, mode)
    np.testing.assert_array_equal(flags, want_flags)
    np.testing.assert_array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("k,knobs,n", [(64, 8, 100001), (130, 3, 5000), (7, 4, 300)])
def test_visited_rows_that_repeat(rls, orc, k, knobs, n):
    """Every other row is one configuration, which every third sample has: found by many waves, again and again."""
    rng = np.random.default_rng(k + n)
    visited = rng.integers(0, 40, (n, knobs)).astype(np.int32)
    cfg = rng.integers(40, 80, (k, knobs)).astype(np.int32)
    visited[::2] = 7
    cfg[::3] = 7
    cfg[1, :min(4, knobs)] = 7                   # (agrees in what is compared first)
    if knobs <= 4:
        cfg[1, -1] = 85
    mode = np.full(knobs, 90, dtype=np.int32)
    got = dev(cfg)
    flags = rls.replace_visited(got, dev(visited), dev(mode)).cpu().numpy()
    want, want_flags = orc.replace_visited(cfg, visited, mode)
    np.testing.assert_array_equal(flags, want_flags)
    np.testing.assert_array_equal(got.cpu().numpy(), want)
    assert want_flags.sum() == (k + 2) // 3


def test_visited_rows_that_repeat_form_no_queue(rls):
    """A history of one configuration that all samples have: some five times as long as one that none has (waves that all wrote to the
    samples' flags took 170 times as long)."""
    visited = torch.full((1000000, 8), 7, dtype=torch.int32, device="cuda")
    mode = torch.full((8,), 7, dtype=torch.int32, device="cuda")

    def shortest(value):
        cfg = torch.full((64, 8), value, dtype=torch.int32, device="cuda")
        times = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(8):
                flags = rls.replace_visited(cfg, visited, mode if value == 7 else cfg[0])
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
            assert bool((flags == (1 if value == 7 else 0)).all())
        return min(times)

    assert shortest(7) < 25 * shortest(9)


# ----------------------------------------------------------------------------------------------
@pytest.mark.parametrize("name,N", [("tiny", None), ("mid", 50001), ("large", 20000)])
def test_knob_modes_match_oracle(rls, orc, name, N):
    p = synth.make_problem(synth.WORKLOADS[name], N=N)
    mode, hist = rls.knob_modes(dev(p.X), rls.DeviceDomains(p.dom_offsets, p.dom_values))
    mode_o, hist_o = orc.knob_modes(p.X, p.dom_offsets, p.dom_values)
    np.testing.assert_array_equal(hist.cpu().numpy().astype(np.int64), hist_o)
    np.testing.assert_array_equal(mode.cpu().numpy(), mode_o)


def test_knob_modes_irregular_domains_ties_and_strided_rows(rls, orc):
    rng = np.random.default_rng(4)
    sizes = [5, 1, 9, 3]
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    values = np.concatenate([np.sort(rng.uniform(-5, 5, size=s)) for s in sizes]).astype(np.float32)
    X = rng.uniform(-7, 7, size=(3001, 6)).astype(np.float32)
    X[:40, 0] = (values[0] + values[1]) / 2          # half-way between two entries (where fp32 holds it exactly or not)
    wide = np.zeros((3001, 10), dtype=np.float32)
    wide[:, :6] = X
    Xd = dev(wide)[:, :6]                            # rows 10 floats apart
    mode, hist = rls.knob_modes(Xd, rls.DeviceDomains(offsets, values))
    mode_o, hist_o = orc.knob_modes(X, offsets, values)
    np.testing.assert_array_equal(hist.cpu().numpy().astype(np.int64), hist_o)
    np.testing.assert_array_equal(mode.cpu().numpy(), mode_o)
    # entries in no particular order, with a repeated value: the scan path, first of equal entries wins
    shuffled = values.copy()
    shuffled[offsets[2]:offsets[3]] = shuffled[offsets[2]:offsets[3]][::-1]
    shuffled[offsets[2] + 4] = shuffled[offsets[2] + 1]
    rep = values.copy()
    rep[offsets[2] + 3] = rep[offsets[2] + 2]                 # sorted with a repeated value: the bisection path
    for vals in (shuffled, rep):
        mode, hist = rls.knob_modes(Xd, rls.DeviceDomains(offsets, vals))
        mode_o, hist_o = orc.knob_modes(X, offsets, vals)
        np.testing.assert_array_equal(hist.cpu().numpy().astype(np.int64), hist_o)
        np.testing.assert_array_equal(mode.cpu().numpy(), mode_o)
    # equal counts: two entries of one knob, each taken by exactly half of the rows
    offs2 = np.array([0, 3], dtype=np.int32)
    vals2 = np.array([0.0, 1.0, 2.0], dtype=np.float32)
    X2 = np.zeros((1000, 2), dtype=np.float32)
    X2[::2, 0] = 2.0
    X2[1::2, 0] = 1.0
    mode, hist = rls.knob_modes(dev(X2), rls.DeviceDomains(offs2, vals2))
    assert hist.cpu().tolist() == [0, 500, 500]
    assert mode.cpu().tolist() == [1]


def test_replace_visited_matches_oracle(rls, orc):
    rng = np.random.default_rng(9)
    n_knobs = 8
    visited = rng.integers(0, 2, size=(5000, n_knobs)).astype(np.int32)          # 256 possible rows, most of them visited
    cfg = rng.integers(0, 2, size=(128, n_knobs)).astype(np.int32)
    cfg[:16, 0] = 7                                                               # certainly not visited
    mode = rng.integers(0, 9, size=n_knobs).astype(np.int32)
    want_cfg, want_flags = orc.replace_visited(cfg, visited, mode)
    assert 0 < want_flags.sum() < 128
    cfg_d = dev(cfg.copy())
    flags = rls.replace_visited(cfg_d, dev(visited), dev(mode))
    np.testing.assert_array_equal(flags.cpu().numpy(), want_flags)
    np.testing.assert_array_equal(cfg_d.cpu().numpy(), want_cfg)
    # nothing visited yet
    cfg_d = dev(cfg.copy())
    flags = rls.replace_visited(cfg_d, None, dev(mode))
    assert int(flags.sum()) == 0
    np.testing.assert_array_equal(cfg_d.cpu().numpy(), cfg)


def test_apply_actions_matches_oracle_and_feeds_scoring(rls, orc):
    """Configuration updater: a trajectory of agent steps, every configuration equal to the oracle's, then scored."""
    w = synth.WORKLOADS["tiny"]
    p = synth.make_problem(w)
    rng = np.random.default_rng(13)
    sizes = np.diff(p.dom_offsets)
    cfg = np.stack([rng.integers(0, s, size=4097) for s in sizes], axis=1).astype(np.int32)
    dom = rls.DeviceDomains(p.dom_offsets, p.dom_values)
    forest = rls.DeviceForest.from_host(p.forest)
    cur_d, cur_h = dev(cfg), cfg
    for step in range(4):
        act = rng.integers(-1, 2, size=cfg.shape).astype(np.int8)
        cur_d, feats_d = rls.apply_actions(cur_d, dev(act), dom)
        cur_h, feats_h = orc.apply_actions(cur_h, act, p.dom_offsets, p.dom_values)
        np.testing.assert_array_equal(cur_d.cpu().numpy(), cur_h)
        np.testing.assert_array_equal(feats_d.cpu().numpy(), feats_h)
        np.testing.assert_array_equal(rls.gbt_score(forest, feats_d).cpu().numpy(), orc.gbt_score(p.forest, feats_h)[0])


def test_apply_actions_in_place_and_out_of_range_input(rls, orc):
    """cfg_out may be cfg; a configuration outside its domain is first brought to the border and a direction beyond
    +-1 counts as +-1 (documented; the oracle rejects both): the result equals the oracle's on the input brought inside."""
    p = synth.make_problem(synth.WORKLOADS["tiny"])
    rng = np.random.default_rng(14)
    sizes = np.diff(p.dom_offsets)
    cfg = np.stack([rng.integers(-3, s + 3, size=3000) for s in sizes], axis=1).astype(np.int32)
    act = rng.integers(-4, 5, size=cfg.shape).astype(np.int8)
    with pytest.raises(RuntimeError):
        orc.apply_actions(cfg, act, p.dom_offsets, p.dom_values)
    want_cfg, want_feats = orc.apply_actions(np.clip(cfg, 0, sizes[None, :] - 1).astype(np.int32), np.clip(act, -1, 1),
                                             p.dom_offsets, p.dom_values)
    dom = rls.DeviceDomains(p.dom_offsets, p.dom_values)
    out_d, feats_d = rls.apply_actions(dev(cfg), dev(act), dom)
    np.testing.assert_array_equal(out_d.cpu().numpy(), want_cfg)
    np.testing.assert_array_equal(feats_d.cpu().numpy(), want_feats)
    # in place, straight through the C ABI: cfg_out_dev == cfg_dev
    import ctypes
    cfg_d, act_d = dev(cfg), dev(act)
    d_struct = dom.struct()
    rc = rls.lib().rls_apply_actions(cfg_d.data_ptr(), act_d.data_ptr(), cfg.shape[0], ctypes.byref(d_struct),
                                     cfg_d.data_ptr(), None, 0, rls._stream())
    assert rc == 0
    torch.cuda.synchronize()
    np.testing.assert_array_equal(cfg_d.cpu().numpy(), want_cfg)


# ----------------------------------------------------------------------------------------------
@pytest.mark.parametrize("name,N,k_max", [("tiny", None, 16), ("mid", 30000, 40), ("large", 5000, 24)])
def test_seeding_chain(rls, orc, name, N, k_max):
    p = synth.make_problem(synth.WORKLOADS[name], N=N)
    for seed in (12799, 7):
        got = rls.kmeanspp_chain(dev(p.X), k_max, seed).cpu().numpy()
        np.testing.assert_array_equal(got, orc.kmeanspp_chain(p.X, k_max, seed))


@pytest.mark.parametrize("N,d,span,stride", [(5000, 2, 6, None), (30011, 4, 3, None), (9000, 8, 2, 12), (7001, 5, 4, None),
                                             (20000, 16, 1, None), (3000, 32, 2, 40)])
def test_seeding_chain_lattice_points(rls, orc, N, d, span, stride):
    """Integer lattices: many duplicates, many equal distances; rows that are strided or no multiple of 16 bytes.  (Sizes that
    the chain in one launch takes; test_seeding_chain_walked_in_memory has the larger ones.)"""
    rng = np.random.default_rng(N + d)
    X = rng.integers(0, span + 1, size=(N, d)).astype(np.float32)
    Xd = dev(X)
    if stride is not None:
        wide = torch.zeros((N, stride), dtype=torch.float32, device="cuda")
        wide[:, :d] = Xd
        Xd = wide[:, :d]
    k_max = min(64, (span + 1) ** d + 3)          # more centres than distinct points where the lattice is small
    for seed in (1, 2):
        got = rls.kmeanspp_chain(Xd, k_max, seed).cpu().numpy()
        np.testing.assert_array_equal(got, orc.kmeanspp_chain(X, k_max, seed))


@pytest.mark.parametrize("N,d,span,stride", [
    # one size past the chain in one launch, per padded number of features; rows of 1 to 8 units of 16 bytes, dense and strided
    (2097153, 4, 3, None), (2097999, 8, 2, 12), (1048577, 12, 2, None), (1050001, 16, 1, 20), (524289, 20, 1, None), (530001, 24, 2, None),
    (525003, 28, 1, None), (524800, 32, 2, 40),
    # element by element: rows that are no multiple of 16 bytes, or too far apart for that; more centres than distinct points
    (2100001, 5, 4, None), (524300, 17, 2, None), (1049600, 12, 2, 13), (2097155, 2, 1, None)])
def test_seeding_chain_walked_in_memory(rls, orc, N, d, span, stride):
    """Chains with an update and a draw launch per centre.  Integer lattices: many duplicates, and many points exactly half way
    between two centres, where the bound that lets the update skip a row (D_i against a quarter of the squared distance
    between centres) is met with equality.  Drawn at once, and wave by wave from the distances, nearest centres and
    bounds that the waves before left (with no rounds the centroids of a run are the rows of its first centres)."""
    dp = 8 if d <= 8 else (16 if d <= 16 else 32)
    assert N > torch.cuda.get_device_properties(0).multi_processor_count * 1024 * (64 // dp)
    rng = np.random.default_rng(N + d)
    X = rng.integers(0, span + 1, size=(N, d)).astype(np.float32)
    Xd = dev(X)
    if stride is not None:
        wide = torch.zeros((N, stride), dtype=torch.float32, device="cuda")
        wide[:, :d] = Xd
        Xd = wide[:, :d]
    k_max = min(40, (span + 1) ** d + 3)
    ref = orc.kmeanspp_chain(X, k_max, 1)
    np.testing.assert_array_equal(rls.kmeanspp_chain(Xd, k_max, 1).cpu().numpy(), ref)
    for k_wave in (1, 4):
        _, n_done, part = rls.kmeans_sweep_until_knee(Xd, 1, 7, k_wave, 0, 1e-9, seed=1, want_labels=False)
        assert n_done == 7
        np.testing.assert_array_equal(part.centroids_of(7).cpu().numpy(), X[ref[:7]])


def spaces_at_once(rls, batch, N, d, k, gap=0, compute_units=256):
    """The route of the chains of the first 64 spaces: so many per launch, 0 where they are walked in memory."""
    quads = d % 4 == 0 and (batch == 1 or (N * d + gap) % 4 == 0)
    return rls.lib().rls_seed_spaces_at_once(ctypes.c_int64(N), d, min(batch, 64), k, int(quads), compute_units)


def compute_units():
    return torch.cuda.get_device_properties(0).multi_processor_count


def spaces_with_gaps(X, gap):
    batch, N, d = X.shape
    buf = torch.zeros((batch, N * d + gap), dtype=torch.float32, device="cuda")
    buf[:, :N * d] = dev(X).view(batch, -1)
    Xd = buf[:, :N * d].view(batch, N, d)
    assert Xd.stride(0) == N * d + gap
    return Xd


MANY_SPACES = [(17001, 16, 0), (33000, 7, 0), (8200, 20, 8), (8200, 20, 6)]


@pytest.mark.parametrize("N,d,gap", MANY_SPACES)
def test_seeding_chain_of_many_spaces(rls, orc, N, d, gap):
    """64 spaces that do not fit the chip together are drawn in parts, the six after them in one launch; rows that can
    and (spaces 2 floats off) cannot be read 16 bytes at a time in every space."""
    batch, k_max = 70, 6
    assert spaces_at_once(rls, batch, N, d, k_max, gap, compute_units()) == 51
    rng = np.random.default_rng(N + gap)
    X = rng.integers(0, 3, size=(batch, N, d)).astype(np.float32)
    Xd = spaces_with_gaps(X, gap)
    seeds = [100 + b for b in range(batch)]
    res = rls.kmeans_sweep_batched(Xd, k_max, k_max, 0, seeds=seeds)
    got = res.centroids.cpu().numpy().reshape(batch, k_max, d)
    for b in range(batch):
        np.testing.assert_array_equal(got[b], X[b][orc.kmeanspp_chain(X[b], k_max, seeds[b])], err_msg=f"space {b}")


# spaces too large for the chip one at a time, or too few centres for parts to pay; rows of 2, 4, 5 and 8 units of 16 bytes, rows that are no multiple
# of 16 bytes, spaces that begin 8 bytes off; 64 spaces, and six more that are one launch
WALKED_SPACES = [(6, 300000, 32, 0, 8), (2, 530001, 32, 0, 8), (2, 524300, 17, 0, 8), (3, 300000, 32, 2, 5), (2, 2097153, 8, 0, 5), (64, 17001, 16, 0, 4), (64, 8200, 20, 8, 4),
                 (70, 8200, 20, 6, 3), (64, 33000, 7, 0, 3), (64, 20011, 16, 0, 2)]


@pytest.mark.parametrize("batch,N,d,gap,k_max", WALKED_SPACES)
def test_seeding_chain_of_spaces_walked_in_memory(rls, orc, batch, N, d, gap, k_max):
    """The chains of a batch with an update and a draw launch per centre, from the third centre on with rows left out by the bound: integer
    lattices, where it is met with equality."""
    assert spaces_at_once(rls, batch, N, d, k_max, gap, compute_units()) == 0
    rng = np.random.default_rng(N + gap + k_max)
    X = rng.integers(0, 3, size=(batch, N, d), dtype=np.int8).astype(np.float32)
    seeds = [100 + b for b in range(batch)]
    res = rls.kmeans_sweep_batched(spaces_with_gaps(X, gap), k_max, k_max, 0, seeds=seeds, want_labels=False)
    got = res.centroids.cpu().numpy().reshape(batch, k_max, d)
    for b in range(batch):
        np.testing.assert_array_equal(got[b], X[b][orc.kmeanspp_chain(X[b], k_max, seeds[b])], err_msg=f"space {b}")


@pytest.mark.parametrize("N,d,k_max", [(1, 3, 1), (2, 8, 2), (1024, 8, 5), (1025, 16, 9), (2049, 32, 128), (4097, 5, 6), (70001, 7, 12),
                                       (300000, 17, 6), (1048577, 16, 4), (540000, 32, 4), (2000003, 6, 4)])
def test_seeding_chain_one_launch(rls, orc, N, d, k_max):
    """Edges of the chain that runs in one launch (one workgroup / several, points per thread, last sizes it takes and
    the first it does not), and the kernel that takes over when its workgroups stop waiting for each other."""
    rng = np.random.default_rng(N + d)
    X = (rng.integers(0, 9, (N, d)) + rng.integers(0, 2, (N, 1)) * 0.25).astype(np.float32)
    ref = orc.kmeanspp_chain(X, k_max, 21)
    Xd = dev(X)
    np.testing.assert_array_equal(rls.kmeanspp_chain(Xd, k_max, 21).cpu().numpy(), ref)
    try:
        rls.lib().rls_seed_wait_limit(ctypes.c_int64(0))
        np.testing.assert_array_equal(rls.kmeanspp_chain(Xd, k_max, 21).cpu().numpy(), ref)
    finally:
        rls.lib().rls_seed_wait_limit(ctypes.c_int64(-1))


@pytest.mark.parametrize("N,d", [(1, 8), (1500, 5), (4096, 8), (4096, 16), (2048, 32)])
def test_seeding_chain_of_one_workgroup(rls, orc, N, d):
    """Nothing is prepared for a chain that one workgroup draws: whatever the workspace holds, at once and wave by wave."""
    rng = np.random.default_rng(N + d)
    X = rng.integers(0, 7, (N, d)).astype(np.float32)
    Xd, k_max = dev(X), min(N, 11)
    ref = orc.kmeanspp_chain(X, k_max, 17)
    ws = torch.empty(1 << 24, dtype=torch.uint8, device="cuda")
    for content in (0, 1, 255):
        ws.fill_(content)
        np.testing.assert_array_equal(rls.kmeanspp_chain(Xd, k_max, 17, workspace=ws).cpu().numpy(), ref)
        ws.fill_(content)
        _, n_done, part = rls.kmeans_sweep_until_knee(Xd, 1, k_max, 3, 0, 1e-9, seed=17, workspace=ws, want_labels=False)
        assert n_done == k_max
        np.testing.assert_array_equal(part.centroids_of(k_max).cpu().numpy(), X[ref])


@pytest.mark.parametrize("d,points", [(d, n) for d in (1, 6, 8) for n in (1, 2, 4, 8)] + [(d, n) for d in (12, 13) for n in (1, 2, 4)] +
                         [(d, n) for d in (19, 28) for n in (1, 2)])
def test_seeding_chain_stages_every_kind_of_rows(rls, orc, d, points):
    """Every number of points per thread of the chain in one launch, a last workgroup with a few points: rows that follow each other, rows
    further apart, rows that can and cannot be read 16 bytes at a time."""
    N = 5001 if points == 1 else 1024 * (256 * points // 2 + 3) + 5
    rng = np.random.default_rng(N + d)
    X = (rng.integers(0, 9, (N, d)) + rng.integers(0, 2, (N, 1)) * 0.25).astype(np.float32)
    ref = orc.kmeanspp_chain(X, 5, 8)
    for lead, width in ((0, d), (1, d + 3), (4, (d + 11) // 4 * 4)):
        full = torch.full((N, width), float("nan"), device="cuda")        # (what lies between the rows is not read as a feature)
        full[:, lead:lead + d] = dev(X)
        rows = full[:, lead:lead + d]
        np.testing.assert_array_equal(rls.kmeanspp_chain(rows, 5, 8).cpu().numpy(), ref)
        try:                                     # (the kernel that takes over stages them as well)
            rls.lib().rls_seed_wait_limit(ctypes.c_int64(0))
            np.testing.assert_array_equal(rls.kmeanspp_chain(rows, 5, 8).cpu().numpy(), ref)
        finally:
            rls.lib().rls_seed_wait_limit(ctypes.c_int64(-1))


# spaces that fit the chip 25, 51, 3, 7 and one at a time, a last part that is shorter, two spaces after the first 64
SPACES_IN_PARTS = [(64, 40009, 13, 16, -1, 25), (64, 20011, 16, 24, -1, 51), (64, 20011, 16, 24, 0, 51), (5, 262145, 16, 12, -1, 3), (9, 70001, 32, 20, -1, 7),
                   (3, 600007, 13, 30, -1, 1), (66, 20011, 16, 9, -1, 51)]


@pytest.mark.parametrize("batch,N,d,k,limit,at_once", SPACES_IN_PARTS)
def test_seeding_of_more_spaces_than_fit_together(rls, batch, N, d, k, limit, at_once):
    """Chains of a batch, one part of its spaces after the other: every space draws what it draws on its own."""
    assert spaces_at_once(rls, batch, N, d, k, 0, compute_units()) == at_once
    gen = torch.Generator(device="cuda").manual_seed(N + k)
    X = torch.randint(0, 50, (batch, N, d), generator=gen, device="cuda").float()
    X[:, :, 0] += torch.arange(batch, device="cuda")[:, None]
    seeds = [1000 + 7 * b for b in range(batch)]
    try:
        rls.lib().rls_seed_wait_limit(ctypes.c_int64(limit))
        got = rls.kmeans_sweep_batched(X, k, k, 0, seeds=seeds, want_labels=False).centroids.view(batch, k, d)
    finally:
        rls.lib().rls_seed_wait_limit(ctypes.c_int64(-1))
    for b in range(batch):
        assert torch.equal(got[b], X[b][rls.kmeanspp_chain(X[b], k, seeds[b])]), b


@pytest.mark.parametrize("limit,words", [(-1, (0, 0)), (0, (1, 3))])
def test_seeding_in_parts_does_not_wait_for_a_held_chip_again(rls, limit, words):
    """Once the workgroups of a part have given up, those of the next one are told (and wait a twentieth of the time to begin with)."""
    batch, N, d, k = 64, 20011, 16, 5
    assert spaces_at_once(rls, batch, N, d, k, 0, compute_units()) == 51
    X = torch.randint(0, 50, (batch, N, d), generator=torch.Generator(device="cuda").manual_seed(4), device="cuda").float()
    ws = torch.zeros(rls.kmeans_sweep_least_workspace_bytes(N, d, k, k, batch) + 256, dtype=torch.uint8, device="cuda")
    per_space = (ws.numel() - 256) // batch
    try:
        rls.lib().rls_seed_wait_limit(ctypes.c_int64(limit))
        got = rls.kmeans_sweep_batched(X, k, k, 0, seeds=range(batch), want_labels=False, workspace=ws).centroids.view(batch, k, d)
    finally:
        rls.lib().rls_seed_wait_limit(ctypes.c_int64(-1))
    # word 37248 of a space's exchange area, which the column statistics of so few rows leave alone: 1 its workgroups gave up, 2 those of the part before did
    at = (-ws.data_ptr()) % 256
    quit = ws[at:at + batch * per_space].view(batch, per_space)[:, 37248 * 8:37248 * 8 + 8].contiguous().view(torch.int64).flatten().cpu().numpy()
    np.testing.assert_array_equal(quit, [words[0]] * 51 + [words[1]] * 13)
    for b in range(0, batch, 7):
        assert torch.equal(got[b], X[b][rls.kmeanspp_chain(X[b], k, b)]), b


def exchange_words(ws, k_max):
    """The words that the workgroups of a chain exchange, at the head of the workspace: the sums of step j are words
    256 j + workgroup, and a word nobody has written is -1."""
    base = (-ws.data_ptr()) % 256
    return ws[base:base + 256 * k_max * 8].view(torch.int64).view(k_max, 256).cpu().numpy()


def test_seeding_wait_limit_holds_for_one_host_thread(rls, orc):
    """A limit set by one thread leaves the chains of another alone: that one's workgroups wait for each other to the end."""
    rng = np.random.default_rng(31)
    X = rng.standard_normal((20000, 8)).astype(np.float32)
    Xd, k_max, groups = dev(X), 8, 20                       # 20 workgroups of 1024 points
    ref = orc.kmeanspp_chain(X, k_max, 5)
    seen = {}

    def chain(name):
        ws = torch.zeros(rls.kmeans_sweep_workspace_bytes(20000, 8, k_max, k_max) + 256, dtype=torch.uint8, device="cuda")
        got = rls.kmeanspp_chain(Xd, k_max, 5, workspace=ws)
        torch.cuda.synchronize()
        seen[name] = (got.cpu().numpy(), exchange_words(ws, k_max)[k_max - 1, :groups])

    try:
        rls.lib().rls_seed_wait_limit(ctypes.c_int64(0))
        chain("own")
        other = threading.Thread(target=chain, args=("other",))
        other.start()
        other.join()
    finally:
        rls.lib().rls_seed_wait_limit(ctypes.c_int64(-1))
    for name in ("own", "other"):
        np.testing.assert_array_equal(seen[name][0], ref)
    assert (seen["own"][1] == -1).any()                     # gave up before the last step
    assert (seen["other"][1] != -1).all()


@pytest.mark.parametrize("first", [0, 1, 5])
def test_seeding_resume_after_workgroups_gave_up(rls, orc, first):
    """Workgroups from `first` on give up in every step, those before wait: a workgroup may finish the last step of a call
    (its draw needs the others' sums only) while another has left without its distances.  The wave that goes on from there
    must still draw the oracle's centres.  The second centre is a point of workgroup 0, the third one is not."""
    rng = np.random.default_rng(8)
    N, d, k_max = 6000, 8, 5                                # six workgroups of 1024 points
    X = (rng.integers(0, 30, (N, d)) + rng.standard_normal((N, d))).astype(np.float32)
    chains = ((s, orc.kmeanspp_chain(X, k_max, s)) for s in range(1000))
    seeds = [s for s, c in chains if c[1] < 1024 <= c[2]][:4]
    assert len(seeds) == 4
    Xd = dev(X)
    ws = torch.empty(1 << 24, dtype=torch.uint8, device="cuda")
    for seed in seeds:
        ref = orc.kmeans_sweep(X, 1, k_max, 1, seed=seed)
        ws.zero_()                                          # distances that nobody has written read as zero
        try:
            rls.lib().rls_seed_wait_limit_from(first, ctypes.c_int64(0))
            _, n_done, part = rls.kmeans_sweep_until_knee(Xd, 1, k_max, 1, 1, 1e-9, seed=seed, workspace=ws)
        finally:
            rls.lib().rls_seed_wait_limit(ctypes.c_int64(-1))
        assert n_done == k_max
        compare_sweep(orc, X, part, ref, 1, k_max)


@pytest.mark.parametrize("N,d,k_max", [(1025, 8, 9), (65537, 16, 24), (300007, 13, 7), (1048576, 16, 5), (524288, 32, 5), (2097152, 3, 5)])
@pytest.mark.parametrize("kind", ["gauss", "lattice"])
def test_seeding_chain_done_again(rls, orc, N, d, k_max, kind):
    """The kernel that does a chain again when workgroups have given up, over the sizes that it can be asked for: two blocks
    of points up to 256, one to eight points per thread, ragged last blocks; every centre, and centres added to a chain that
    an earlier call began (the waves of a sweep until the knee)."""
    rng = np.random.default_rng(N + d)
    X = rng.standard_normal((N, d), dtype=np.float32) if kind == "gauss" else rng.integers(0, 4, (N, d)).astype(np.float32)
    Xd = dev(X)
    ref = orc.kmeanspp_chain(X, k_max, 3)
    try:
        rls.lib().rls_seed_wait_limit(ctypes.c_int64(0))
        for _ in range(3):
            np.testing.assert_array_equal(rls.kmeanspp_chain(Xd, k_max, 3).cpu().numpy(), ref)
        # no rounds: the centroids of a run are the rows of its first k centres
        _, n_done, part = rls.kmeans_sweep_until_knee(Xd, 1, k_max, 2, 0, 1e-9, seed=3, want_labels=False)
    finally:
        rls.lib().rls_seed_wait_limit(ctypes.c_int64(-1))
    assert n_done == k_max
    np.testing.assert_array_equal(part.centroids_of(k_max).cpu().numpy(), X[ref])


def test_seeding_done_again_uses_the_whole_chip(rls):
    """When workgroups of the one-launch chain give up (other streams hold compute units), what follows must not be a
    matter of one workgroup: measured 0.16 ms undisturbed and 0.8 ms done again, 150 ms in one workgroup."""
    X = torch.randn(1048576, 16, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    ws = torch.empty(rls.kmeans_sweep_workspace_bytes(1048576, 16, 16, 16) + 256, dtype=torch.uint8, device="cuda")

    def ms():
        times = []
        for _ in range(4):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            rls.kmeanspp_chain(X, 16, 3, workspace=ws)
            end.record()
            end.synchronize()
            times.append(begin.elapsed_time(end))
        return min(times)

    undisturbed = ms()
    try:
        rls.lib().rls_seed_wait_limit(ctypes.c_int64(0))
        again = ms()
    finally:
        rls.lib().rls_seed_wait_limit(ctypes.c_int64(-1))
    assert again < 100 * undisturbed, f"{again} ms against {undisturbed} ms"


def test_sweeps_on_two_streams_and_threads(rls, orc):
    """Two host threads sweep on streams of their own at the same time; the chains of each take the whole chip, if they can
    get it."""
    rng = np.random.default_rng(77)
    Xs = [rng.standard_normal((262147 + 64 * i, 16), dtype=np.float32) * (1 + i) for i in range(2)]
    refs = [orc.kmeans_sweep(X, 10, 12, 2, seed=6 + i) for i, X in enumerate(Xs)]
    results = [[], []]

    def work(i):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            Xd = dev(Xs[i])
            for _ in range(6):
                results[i].append(rls.kmeans_sweep(Xd, 10, 12, 2, seed=6 + i))
            stream.synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i in range(2):
        assert len(results[i]) == 6
        for res in results[i]:
            compare_sweep(orc, Xs[i], res, refs[i], 10, 12)


def test_seeding_all_points_equal(rls, orc):
    X = np.full((300, 8), 3.0, dtype=np.float32)
    got = rls.kmeanspp_chain(dev(X), 5, 11).cpu().numpy()
    np.testing.assert_array_equal(got, orc.kmeanspp_chain(X, 5, 11))


# ----------------------------------------------------------------------------------------------
def compare_sweep(orc, X, res, ref, k_min, k_max, expect_exempt=0):
    """res: binding.SweepResult (GPU); ref: oracle dict.  A label may differ from the oracle's only where the
    point's two nearest centroids lie within 1e-6 relative; the number of such differences must be the one the
    test names (none, unless it says otherwise), and without any the centroids must be bit-identical."""
    N, d = X.shape
    exempt = 0
    col_scale = np.abs(X).max(axis=0).astype(np.float64)
    col_scale[col_scale == 0] = 1.0
    gl = res.labels.cpu().numpy() if res.labels is not None else None
    gJ = res.inertia.cpu().numpy()
    for k in range(k_min, k_max + 1):
        r = k - k_min
        Cg = res.centroids_of(k).cpu().numpy()
        Co = orc.unpack_centroids(ref["centroids"], k_min, k, d)
        if gl is not None and ref["labels"] is not None:
            bad = np.flatnonzero(gl[r] != ref["labels"][r])
            for i in bad:
                d1, d2, _ = orc.two_nearest(X[i], Co)
                assert (d2 - d1) <= 1e-6 * d2, f"k={k} point {i}: label {gl[r][i]} vs {ref['labels'][r][i]}, d1={d1} d2={d2}"
                exempt += 1
        err = np.abs(Cg.astype(np.float64) - Co.astype(np.float64))
        tol = 1e-5 * np.maximum(np.abs(Co.astype(np.float64)), col_scale[None, :])
        assert np.all(err <= tol), f"k={k}: centroid error {err.max()}"
        assert abs(gJ[r] - ref["inertia"][r]) <= 1e-5 * max(ref["inertia"][r], 1e-300), f"k={k}: inertia"
        if exempt == 0:
            np.testing.assert_array_equal(Cg, Co, err_msg=f"k={k}: centroids not bit-identical")
    if res.trace is not None and ref["trace"] is not None:
        gt = res.trace.cpu().numpy()
        assert np.all(np.abs(gt - ref["trace"]) <= 1e-5 * np.maximum(ref["trace"], 1e-300))
    assert exempt == expect_exempt, f"{exempt} label differences inside the near-tie rule, {expect_exempt} expected"
    return exempt


def run_both(rls, orc, X, k_min, k_max, iters, seed=None, init=None, trace=True):
    Xd = dev(X)
    if init is not None:
        res = rls.kmeans_sweep(Xd, k_min, k_max, iters, init_idx=dev(init), want_trace=trace)
        ref = orc.kmeans_sweep(X, k_min, k_max, iters, init_idx=init, want_trace=trace)
    else:
        res = rls.kmeans_sweep(Xd, k_min, k_max, iters, seed=seed, want_trace=trace)
        ref = orc.kmeans_sweep(X, k_min, k_max, iters, seed=seed, want_trace=trace)
    torch.cuda.synchronize()
    if trace:
        # Without the loss trace the rounds after the first run a different kernel path (operands from a copy of the
        # points prepared once per sweep, rows read on demand): it must give the same sweep, bit for bit.
        if init is not None:
            plain = rls.kmeans_sweep(Xd, k_min, k_max, iters, init_idx=dev(init))
        else:
            plain = rls.kmeans_sweep(Xd, k_min, k_max, iters, seed=seed)
        torch.cuda.synchronize()
        assert torch.equal(plain.labels, res.labels), "labels differ between the sweep with and without trace"
        assert torch.equal(plain.centroids, res.centroids), "centroids differ between the sweep with and without trace"
        assert torch.equal(plain.inertia, res.inertia)
    return res, ref


def test_sweep_tiny_full(rls, orc):
    w = synth.WORKLOADS["tiny"]
    p = synth.make_problem(w)
    res, ref = run_both(rls, orc, p.X, w.k_min, w.k_max, w.iters, seed=w.seed)
    compare_sweep(orc, p.X, res, ref, w.k_min, w.k_max)
    for const in (1.01, 1.05, 1.1, 1.5, 2.0):
        assert rls.pick_knee(res.inertia.cpu().tolist(), w.k_min, w.k_max, const) == \
            orc.pick_knee(ref["inertia"], w.k_min, w.k_max, const)


def test_sweep_trace_is_monotone(rls):
    w = synth.WORKLOADS["tiny"]
    p = synth.make_problem(w)
    res = rls.kmeans_sweep(dev(p.X), 1, 16, 20, seed=3, want_trace=True)
    t = res.trace.cpu().numpy()
    assert np.all(t[:, 1:] <= t[:, :-1] * (1 + 1e-6))
    np.testing.assert_array_equal(t[:, -1], res.inertia.cpu().numpy())


@pytest.mark.parametrize("N,d,k_min,k_max,iters", [
    (257, 8, 1, 9, 3),        # ragged tail of one point
    (1000, 5, 2, 12, 4),      # d padded to 8
    (999, 12, 1, 20, 3),      # d padded to 16
    (640, 32, 1, 10, 3),      # d = 32 tiles
    (3000, 16, 8, 63, 2),     # the paper's range(8, 64)
    (2000, 20, 30, 40, 2),    # d padded to 32, mid k only
    (500, 16, 1, 8, 0),       # no Lloyd round: assignment against the seeds only
    (128, 8, 128, 128, 2),    # k = N = the largest k
    (1, 8, 1, 1, 2),          # a single point
    (2, 3, 1, 2, 3),          # two points, k up to N
    (33, 16, 1, 33, 2),       # one point past a 32-point block, k up to N
    (64, 32, 60, 64, 1),      # exactly one slab at d = 32... and a second, k close to N
])
def test_sweep_shapes(rls, orc, N, d, k_min, k_max, iters):
    rng = np.random.default_rng(N * 31 + d)
    centres = rng.uniform(-20, 20, size=(7, d))
    X = (centres[rng.integers(0, 7, size=N)] + rng.standard_normal((N, d))).astype(np.float32)
    res, ref = run_both(rls, orc, X, k_min, k_max, iters, seed=5)
    compare_sweep(orc, X, res, ref, k_min, k_max)


@pytest.mark.parametrize("d", [5, 16, 32])
@pytest.mark.parametrize("k_min,k_max", [(1, 1), (3, 3), (8, 8), (31, 31), (32, 32), (33, 33), (64, 64), (100, 100),
                                         (128, 128), (30, 33), (62, 64), (127, 128)])
def test_sweep_single_k_and_narrow_ranges(rls, orc, d, k_min, k_max):
    # a sweep over one k (plain k-means) or the last few k of a range: one run per group, or a group that is not full
    rng = np.random.default_rng(1000 * d + 7 * k_min + k_max)
    N = 2100
    centres = rng.uniform(-15, 15, size=(11, d))
    X = (centres[rng.integers(0, 11, size=N)] + rng.standard_normal((N, d))).astype(np.float32)
    X[::7] = np.round(X[::7])                       # some exact ties
    res, ref = run_both(rls, orc, X, k_min, k_max, 3, seed=k_min + d)
    compare_sweep(orc, X, res, ref, k_min, k_max)


def test_sweep_integer_ties_and_duplicates(rls, orc):
    # small-integer data with many duplicate rows: exact distance ties everywhere; lowest index must win
    rng = np.random.default_rng(3)
    X = rng.integers(0, 4, size=(1500, 8)).astype(np.float32)
    res, ref = run_both(rls, orc, X, 1, 24, 5, seed=9)
    assert compare_sweep(orc, X, res, ref, 1, 24) == 0
    # duplicate initial centres: clusters that never win a point keep their centroid
    init = np.zeros(6, dtype=np.int64)
    init[3:] = 7
    res, ref = run_both(rls, orc, X, 2, 6, 3, init=init)
    assert compare_sweep(orc, X, res, ref, 2, 6) == 0


def test_sweep_all_points_equal(rls, orc):
    X = np.full((700, 16), 2.5, dtype=np.float32)
    res, ref = run_both(rls, orc, X, 1, 5, 2, seed=1)
    assert compare_sweep(orc, X, res, ref, 1, 5) == 0
    assert float(res.inertia.abs().max()) == 0.0


def test_sweep_planted_clusters(rls, orc):
    X, truth = synth.planted_clusters(300, 9, 16, sep=40.0, sigma=0.5, seed=4)
    res, ref = run_both(rls, orc, X, 9, 9, 12, seed=2)
    compare_sweep(orc, X, res, ref, 9, 9)
    labels = res.labels.cpu().numpy()[0]
    mapping = {}
    for a, b in zip(labels.tolist(), truth.tolist()):
        assert mapping.setdefault(a, b) == b
    assert len(set(mapping.values())) == 9


def test_sweep_mid_full(rls, orc):
    w = synth.WORKLOADS["mid"]
    p = synth.make_problem(w)
    res, ref = run_both(rls, orc, p.X, w.k_min, w.k_max, w.iters, seed=w.seed, trace=False)
    compare_sweep(orc, p.X, res, ref, w.k_min, w.k_max)
    for const in (1.01, 1.05, 1.1):
        assert rls.pick_knee(res.inertia.cpu().tolist(), w.k_min, w.k_max, const) == \
            orc.pick_knee(ref["inertia"], w.k_min, w.k_max, const)


def test_sweep_large_features_subset(rls, orc):
    w = synth.WORKLOADS["large"]
    p = synth.make_problem(w, N=20000)
    res, ref = run_both(rls, orc, p.X, 1, 128, 4, seed=w.seed, trace=False)
    compare_sweep(orc, p.X, res, ref, 1, 128)


def test_sweep_batched(rls, orc):
    w = synth.WORKLOADS["batched"]
    probs = synth.make_batched_problems(w, batch=3, N=6000)
    X = np.stack([p.X for p in probs])
    seeds = [w.seed + b for b in range(3)]
    res = rls.kmeans_sweep_batched(dev(X), 1, 32, 5, seeds=seeds, want_trace=True)
    torch.cuda.synchronize()
    for b, p in enumerate(probs):
        ref = orc.kmeans_sweep(p.X, 1, 32, 5, seed=seeds[b], want_trace=True)
        one = rls.SweepResult(1, 32, 16, res.labels[b], res.centroids[b], res.inertia[b], res.trace[b], res.status[b:b + 1])
        compare_sweep(orc, p.X, one, ref, 1, 32)


@pytest.mark.parametrize("batch,N,d,k_max,iters", [(130, 700, 8, 6, 3), (1024, 300, 5, 4, 2)])
def test_sweep_many_spaces(rls, orc, batch, N, d, k_max, iters):
    """More spaces than one launch of the seeding kernels takes (they go 64 at a time), up to the largest batch the
    library accepts; every space against the oracle, the snapped centroids of one k as well."""
    rng = np.random.default_rng(batch)
    X = (rng.integers(0, 12, size=(batch, N, d)) + rng.standard_normal((batch, N, d)) * 0.25).astype(np.float32)
    seeds = [1000 + 7 * b for b in range(batch)]
    res = rls.kmeans_sweep_batched(dev(X), 1, k_max, iters, seeds=seeds)
    torch.cuda.synchronize()
    lab, cen, J, st = res.labels.cpu(), res.centroids.cpu(), res.inertia.cpu(), res.status.cpu()
    for b in range(batch):
        ref = orc.kmeans_sweep(X[b], 1, k_max, iters, seed=seeds[b])
        one = rls.SweepResult(1, k_max, d, lab[b], cen[b], J[b], None, st[b:b + 1])
        compare_sweep(orc, X[b], one, ref, 1, k_max)


@pytest.mark.parametrize("batch,N,d,k_min,k_max,iters", [(3, 70000, 16, 1, 64, 2), (5, 33000, 32, 1, 40, 2), (17, 4100, 5, 3, 17, 2)])
def test_sweep_batched_block_order(rls, orc, batch, N, d, k_min, k_max, iters):
    """The workgroups of a launch take the chunks of all spaces in blocks (all groups of a block of chunks, then the
    next block).  Shapes where the chunks of the batch do not fill a whole number of blocks, where a block spans
    several spaces, and where a space ends inside a block: every space against the oracle."""
    rng = np.random.default_rng(batch * 1000 + d)
    c = rng.uniform(-20, 20, size=(batch, 11, d))
    X = np.stack([c[b][rng.integers(0, 11, N)] + rng.standard_normal((N, d)) * 1.5 for b in range(batch)]).astype(np.float32)
    seeds = [77 + 13 * b for b in range(batch)]
    res = rls.kmeans_sweep_batched(dev(X), k_min, k_max, iters, seeds=seeds)
    torch.cuda.synchronize()
    lab, cen, J, st = res.labels.cpu(), res.centroids.cpu(), res.inertia.cpu(), res.status.cpu()
    for b in range(batch):
        ref = orc.kmeans_sweep(X[b], k_min, k_max, iters, seed=seeds[b])
        one = rls.SweepResult(k_min, k_max, d, lab[b], cen[b], J[b], None, st[b:b + 1])
        compare_sweep(orc, X[b], one, ref, k_min, k_max)


@pytest.mark.parametrize("d", [5, 16, 32])
@pytest.mark.parametrize("chunks", [1, 4, 8, 9, 16, 17, 24, 25])
def test_sweep_few_chunks_per_sum(rls, orc, d, chunks):
    """The centroid kernel's slices of one, two or more chunks each: one group whose chunks are one slab per wave."""
    per_chunk = 32 * (8 if d == 32 else 12)
    for N in (chunks * per_chunk, (chunks - 1) * per_chunk + 1):
        rng = np.random.default_rng(N + d)
        X = (rng.integers(0, 6, size=(N, d)) * 2.0 + rng.standard_normal((N, d))).astype(np.float32)
        k = min(3, N)
        res, ref = run_both(rls, orc, X, k, k, 3, seed=chunks)
        compare_sweep(orc, X, res, ref, k, k)


@pytest.mark.parametrize("d,k_min,k_max", [(16, 96, 96), (16, 97, 97), (8, 128, 128), (9, 15, 22), (32, 32, 32), (25, 33, 33), (16, 8, 15)])
def test_sweep_staging_of_small_groups(rls, orc, d, k_min, k_max):
    """A group whose operands and centroids are one and two loads per thread is staged at once, a larger one in batches: the
    last sizes of the one and the first of the other."""
    rng = np.random.default_rng(d + k_max)
    X = (rng.uniform(-15, 15, size=(11, d))[rng.integers(0, 11, 1500)] + rng.standard_normal((1500, d))).astype(np.float32)
    res, ref = run_both(rls, orc, X, k_min, k_max, 3, seed=k_min)
    compare_sweep(orc, X, res, ref, k_min, k_max)


@pytest.mark.parametrize("batch,N,d,k_min,k_max", [(128, 513, 5, 3, 3), (127, 513, 5, 3, 3), (43, 2049, 16, 8, 31), (42, 2049, 16, 8, 31),
                                                   (37, 4097, 6, 8, 63), (36, 4095, 6, 8, 63), (37, 65537, 5, 8, 63), (520, 300, 5, 2, 2)])
def test_sweep_batched_chunk_rule(rls, orc, batch, N, d, k_min, k_max):
    """Both sides of the rules by which a batch cuts its points: groups times spaces up to half of the compute units (chunks of
    equal cost per group), up to all of them, and more (one or two chunks per space, of 4096 points at least)."""
    rng = np.random.default_rng(batch + N)
    c = rng.uniform(-20, 20, size=(batch, 9, d)).astype(np.float32)
    X = np.stack([c[b][rng.integers(0, 9, N)] for b in range(batch)]) + rng.standard_normal((batch, N, d), dtype=np.float32)
    init = rng.integers(0, N, size=(batch, k_max))
    res = rls.kmeans_sweep_batched(dev(X), k_min, k_max, 2, init_idx=dev(init))
    lab, cen, J, st = res.labels.cpu(), res.centroids.cpu(), res.inertia.cpu(), res.status.cpu()
    for b in (0, batch // 2, batch - 1):
        for k in sorted({k_min, (k_min + k_max) // 2, k_max}):
            ref = orc.kmeans_sweep(X[b], k, k, 2, init_idx=init[b, :k])
            at = sum(range(k_min, k)) * d
            one = rls.SweepResult(k, k, d, lab[b, k - k_min:k - k_min + 1], cen[b, at:at + k * d], J[b, k - k_min:k - k_min + 1], None, st[b:b + 1])
            compare_sweep(orc, X[b], one, ref, k, k)


@pytest.mark.parametrize("N,d", [(769, 5), (24577, 16), (150001, 5), (300007, 13), (600011, 5), (600011, 32), (3200003, 5)])
def test_sweep_chunks_per_group(rls, orc, N, d):
    """k 1..128 over the sizes at which the step changes how it cuts the points: chunks of equal cost per group, one
    workgroup per compute unit; the same chunks for every group; chunks per group, several per compute unit; and the same
    chunks again.  A run does not depend on the others of its sweep: some k against the oracle."""
    rng = np.random.default_rng(N + d)
    centres = rng.uniform(-20, 20, size=(40, d)).astype(np.float32)
    X = centres[rng.integers(0, 40, size=N)] + rng.standard_normal((N, d), dtype=np.float32)
    Xd = dev(X)
    init = rls.kmeanspp_chain(Xd, 128, 9)
    res = rls.kmeans_sweep(Xd, 1, 128, 2, init_idx=init)
    lab, J, st = res.labels.cpu(), res.inertia.cpu(), res.status.cpu()
    for k in (1, 8, 63, 97, 128):
        ref = orc.kmeans_sweep(X, k, k, 2, init_idx=init.cpu().numpy()[:k])
        one = rls.SweepResult(k, k, d, lab[k - 1:k], res.centroids_of(k).cpu().reshape(-1), J[k - 1:k], None, st)
        compare_sweep(orc, X, one, ref, k, k)


def test_sweep_strided_unaligned_rows_and_small_d(rls, orc):
    # rows 11 floats apart and starting 4 bytes off a 16-byte boundary: the scalar load paths
    rng = np.random.default_rng(21)
    for d in (1, 3, 7, 8):
        X = (rng.integers(0, 5, size=(1100, d)) * 3.0 + rng.standard_normal((1100, d))).astype(np.float32)
        buf = torch.zeros(1100 * 11 + 1, dtype=torch.float32, device="cuda")
        Xd = buf[1:].view(1100, 11)[:, :d]
        Xd.copy_(torch.as_tensor(X))
        res = rls.kmeans_sweep(Xd, 1, 11, 4, seed=4, want_trace=True)
        ref = orc.kmeans_sweep(X, 1, 11, 4, seed=4, want_trace=True)
        torch.cuda.synchronize()
        assert compare_sweep(orc, X, res, ref, 1, 11) == 0


def test_sweep_wide_columns(rls, orc):
    # one column mixes values near 2^-10 and near 2^40 with full 24-bit significands: more binary digits than the
    # main fixed-point accumulator keeps, so the low-order accumulator is in play; sums must still be exact
    rng = np.random.default_rng(22)
    N = 3000
    X = rng.standard_normal((N, 8)).astype(np.float32)
    small = rng.integers(1, 1 << 24, size=N).astype(np.float64) * 2.0 ** -34
    big = rng.integers(1, 1 << 24, size=N).astype(np.float64) * 2.0 ** 16
    X[:, 2] = np.where(rng.random(N) < 0.5, small, big).astype(np.float32)
    X[:, 5] = (rng.integers(-(1 << 23), 1 << 23, size=N).astype(np.float64) * 2.0 ** -30).astype(np.float32)
    res, ref = run_both(rls, orc, X, 1, 9, 5, seed=6)
    assert int(res.status.item()) == 0
    assert compare_sweep(orc, X, res, ref, 1, 9) == 0


@pytest.mark.parametrize("case", ["scale_up", "scale_down", "offset", "mixed_columns", "small_next_to_big", "d32_offset",
                                  "tiny_magnitude"])
def test_sweep_value_ranges(rls, orc, case):
    """The matrix path works on centred data scaled by a power of two into 16-bit range: magnitudes far from 1, means
    far from the spread, and columns that all but vanish next to the largest one must give the oracle's results
    (within what the oracle's exact sums hold: |x| < 2^40, multiples of 2^-60)."""
    rng = np.random.default_rng(700 + len(case) * 13 + ord(case[0]))
    N, d = 4000, 16
    centres = rng.standard_normal((12, d)) * 3.0
    X = centres[rng.integers(0, 12, size=N)] + rng.standard_normal((N, d)) * 0.4
    if case == "scale_up":
        X = X * 2.0 ** 33 * 1.37
    elif case == "scale_down":
        X = X * 2.0 ** -14 * 0.81
    elif case == "offset":
        X = X * 1.0e-3 + 4096.5              # mean 4e6 times the spread: fp32 keeps about 12 bits of the spread
    elif case == "mixed_columns":
        X = X * (10.0 ** rng.integers(-5, 7, size=d))[None, :]
    elif case == "small_next_to_big":
        X[:, 0] *= 1.0e4                     # the other columns fall below the fp16 range after scaling
        X[:, 1:] *= 1.0e-4
        X[:, 0] = np.round(X[:, 0] / 2.0e4) * 2.0e4      # and decide between points that tie in the big column
    elif case == "d32_offset":
        d = 32
        centres = rng.standard_normal((12, d)) * 3.0
        X = centres[rng.integers(0, 12, size=N)] + rng.standard_normal((N, d)) * 0.4 + 1000.0
    elif case == "tiny_magnitude":
        # squared distances on both sides of 1e-30: below it the first, fp32 stage of the exact argmin hands over to
        # fp64 (fp32 may have lost such a distance); integers times 2^-54, so the exact sums still hold every value
        X = np.round(X * 16.0) * 2.0 ** -54
    X = X.astype(np.float32)
    res, ref = run_both(rls, orc, X, 1, 20, 6, seed=3)
    assert int(res.status.item()) == 0
    assert compare_sweep(orc, X, res, ref, 1, 20) == 0


def random_sweep_case(rng):
    """One random shape and data kind: clustered, small integers, duplicates, knob-like lattices, scaled, shifted."""
    d = int(rng.choice([1, 2, 3, 4, 5, 8, 9, 12, 16, 17, 24, 32]))
    N = int(rng.choice([65, 200, 513, 1000, 2049, 5000]))
    k_max = int(min(N, rng.choice([1, 3, 8, 9, 17, 33, 64, 65, 100, 128])))
    k_min = int(rng.integers(1, k_max + 1)) if rng.random() < 0.5 else 1
    iters = int(rng.integers(0, 6))
    kind = str(rng.choice(["gauss", "int", "dup", "mixed", "const_col", "scaled", "offset", "colmix", "knob"]))
    blobs = rng.uniform(-30, 30, size=(9, d))[rng.integers(0, 9, N)] + rng.standard_normal((N, d))
    if kind == "gauss":
        X = blobs
    elif kind == "int":
        X = rng.integers(0, 4, size=(N, d)).astype(np.float64)
    elif kind == "dup":
        base = rng.standard_normal((max(2, N // 50), d)) * 5
        X = base[rng.integers(0, len(base), N)]
    elif kind == "mixed":
        X = rng.standard_normal((N, d))
        X[:, 0] = rng.integers(0, 3, N)
        X *= rng.choice([1e-3, 1.0, 1e3])
    elif kind == "scaled":
        X = blobs * 2.0 ** int(rng.integers(-12, 30))
    elif kind == "offset":
        X = blobs * 0.1 * 2.0 ** int(rng.integers(-8, 4)) + float(rng.choice([100.0, 4096.5, -70000.25]))
    elif kind == "colmix":
        X = blobs * (2.0 ** rng.integers(-10, 20, size=d))[None, :]
    elif kind == "knob":
        sizes = rng.integers(2, 200, size=d)
        c = rng.uniform(0, 1, size=(12, d)) * sizes
        X = np.clip(np.round(c[rng.integers(0, 12, N)] + rng.standard_normal((N, d)) * np.maximum(0.5, 0.08 * sizes)), 0, sizes - 1)
    else:
        X = rng.standard_normal((N, d))
        X[:, -1] = 7.25
    return X.astype(np.float32), k_min, k_max, iters, kind, int(rng.integers(0, 1 << 30))


@pytest.mark.parametrize("seed", [11, 12, 13])
def test_sweep_randomized(rls, orc, seed):
    rng = np.random.default_rng(seed)
    for case in range(30):
        X, k_min, k_max, iters, kind, s = random_sweep_case(rng)
        print(f"case {case}: N={X.shape[0]} d={X.shape[1]} k={k_min}..{k_max} iters={iters} kind={kind} seed={s}", flush=True)
        res, ref = run_both(rls, orc, X, k_min, k_max, iters, seed=s)
        assert int(res.status.item()) == 0
        compare_sweep(orc, X, res, ref, k_min, k_max)


@pytest.mark.parametrize("name,N,k_min,k_max,k_wave,const", [
    ("tiny", None, 1, 16, 8, 1.05), ("tiny", None, 1, 16, 3, 1.5), ("tiny", None, 2, 16, 5, 1.0001),
    ("mid", 20000, 1, 40, 8, 1.05), ("mid", 20000, 8, 63, 16, 1.02), ("mid", 20000, 1, 24, 8, 1e9)])
def test_sweep_until_knee_equals_full_sweep_and_oracle(rls, orc, name, N, k_min, k_max, k_wave, const):
    """Algorithm 1's early exit: same chosen k and same outputs for the computed k as sweeping the whole range."""
    w = synth.WORKLOADS[name]
    p = synth.make_problem(w, N=N)
    Xd = dev(p.X)
    iters = 6
    k_star, n_done, part = rls.kmeans_sweep_until_knee(Xd, k_min, k_max, k_wave, iters, const, seed=w.seed)
    full = rls.kmeans_sweep(Xd, k_min, k_max, iters, seed=w.seed)
    ref = orc.kmeans_sweep(p.X, k_min, k_max, iters, seed=w.seed)
    assert k_star == orc.pick_knee(ref["inertia"], k_min, k_max, const)
    assert k_star == rls.pick_knee(full.inertia.cpu().tolist(), k_min, k_max, const)
    # a whole number of waves was computed, the last of them holds the chosen k (or everything was computed)
    assert n_done >= k_star - k_min + 1
    assert n_done == k_max - k_min + 1 or n_done % k_wave == 0
    assert n_done <= ((k_star - k_min) // k_wave + 1) * k_wave
    rows_done = sum(range(k_min, k_min + n_done))
    # the loss is a floating-point sum over chunks of points, and the chunking depends on how many k share a launch;
    # centroids come from integer sums and labels from exact comparisons, so they are identical
    np.testing.assert_allclose(part.inertia[:n_done].cpu().numpy(), full.inertia[:n_done].cpu().numpy(), rtol=1e-12)
    np.testing.assert_array_equal(part.centroids[:rows_done * w.d].cpu().numpy(), full.centroids[:rows_done * w.d].cpu().numpy())
    np.testing.assert_array_equal(part.labels[:n_done].cpu().numpy(), full.labels[:n_done].cpu().numpy())
    np.testing.assert_array_equal(part.labels[:n_done].cpu().numpy(), ref["labels"][:n_done])


def test_sweep_is_reproducible_run_to_run(rls):
    """Labels and centroids are exact; the fp64 loss sums are taken in a fixed order: two runs agree bit for bit."""
    p = synth.make_problem(synth.WORKLOADS["mid"], N=30011)
    Xd = dev(p.X)
    a = rls.kmeans_sweep(Xd, 1, 40, 5, seed=9, want_trace=True)
    b = rls.kmeans_sweep(Xd, 1, 40, 5, seed=9, want_trace=True)
    torch.cuda.synchronize()
    assert torch.equal(a.labels, b.labels) and torch.equal(a.centroids, b.centroids)
    assert torch.equal(a.inertia, b.inertia) and torch.equal(a.trace, b.trace)


def test_sweep_graph_capture_and_replay(rls):
    """A caller can record a whole sweep into a HIP graph (the sweep enqueues kernels only: no allocation, no host
    synchronisation, no memset nodes) and replay it; every replay, with eager work in between, gives the eager result."""
    p = synth.make_problem(synth.WORKLOADS["tiny"])
    Xd = dev(p.X)
    k_min, k_max, iters = 1, 16, 6
    ws = torch.empty(rls.kmeans_sweep_workspace_bytes(Xd.shape[0], Xd.shape[1], k_min, k_max, 1) + 256, dtype=torch.uint8, device="cuda")
    init = rls.kmeanspp_chain(Xd, k_max, 5)
    eager = rls.kmeans_sweep(Xd, k_min, k_max, iters, init_idx=init, workspace=ws, check_status=False)
    torch.cuda.synchronize()
    want = [t.clone() for t in (eager.labels, eager.centroids, eager.inertia)]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        rls.kmeans_sweep(Xd, k_min, k_max, iters, init_idx=init, workspace=ws, check_status=False)   # warm-up on this stream
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side):
            res = rls.kmeans_sweep(Xd, k_min, k_max, iters, init_idx=init, workspace=ws, check_status=False)
    torch.cuda.current_stream().wait_stream(side)
    for rep in range(3):
        for t in (res.labels, res.centroids, res.inertia):
            t.zero_()
        other = rls.kmeans_sweep(Xd, 2, 5, 2, seed=rep)        # eager work in between, with its own workspace
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert int(res.status.item()) == 0
        for got, exp in zip((res.labels, res.centroids, res.inertia), want):
            assert torch.equal(got, exp), f"replay {rep}"
        assert other.inertia.shape[0] == 4


def test_sweep_status_flags(rls):
    X = np.ones((600, 8), dtype=np.float32)
    X[5, 2] = np.inf
    res = rls.kmeans_sweep(dev(X), 1, 4, 2, seed=1, check_status=False)
    assert int(res.status.item()) & rls.RLS_STATUS_NONFINITE
    X[5, 2] = 1e-30        # column spans 100 binary orders of magnitude: no exact fixed-point sum
    res = rls.kmeans_sweep(dev(X), 1, 4, 2, seed=1, check_status=False)
    assert int(res.status.item()) & rls.RLS_STATUS_RANGE


# workgroups of either size over the columns: one space and few, long columns and short ones, rows that do not divide among the workgroups
@pytest.mark.parametrize("batch,N,d", [(1, 2000, 8), (1, 65537, 29), (1, 300007, 13), (64, 2000, 8), (8, 70001, 13), (3, 300007, 16), (4, 1048577, 5), (5, 262144, 32)])
def test_column_statistics_of_spaces_together(rls, batch, N, d):
    """Every space of a batch as on its own, and what a column must not hold is seen in the last row of the last space."""
    gen = torch.Generator(device="cuda").manual_seed(N + d)
    X = torch.randn(batch, N, d, generator=gen, device="cuda").mul_(20).round_().mul_(0.25).add_(3000.0)
    seeds = [5 + b for b in range(batch)]
    got = rls.kmeans_sweep_batched(X, 2, 4, 3, seeds=seeds)
    for b in {0, batch // 2, batch - 1}:
        own = rls.kmeans_sweep(X[b], 2, 4, 3, seed=seeds[b])
        for name in ("labels", "centroids", "inertia"):
            assert torch.equal(getattr(got, name)[b], getattr(own, name)), (b, name)
    for value, status in ((float("nan"), 1), (float("-inf"), 1), (1e-30, 2), (3e38, 2), (-1e-44, 2), (0.0, 0)):
        X[-1, -1, -1] = value
        res = rls.kmeans_sweep_batched(X, 2, 2, 1, seeds=seeds, want_labels=False, check_status=False)
        assert res.status.tolist() == [0] * (batch - 1) + [status], value


def test_end_to_end_chain_tiny(rls, orc):
    """score -> sweep -> knee -> snap on the tiny space, every stage against the oracle."""
    w = synth.WORKLOADS["tiny"]
    p = synth.make_problem(w)
    Xd = dev(p.X)
    scores = rls.gbt_score(rls.DeviceForest.from_host(p.forest), Xd)
    np.testing.assert_array_equal(scores.cpu().numpy(), orc.gbt_score(p.forest, p.X)[0])
    res = rls.kmeans_sweep(Xd, w.k_min, w.k_max, w.iters, seed=w.seed)
    ref = orc.kmeans_sweep(p.X, w.k_min, w.k_max, w.iters, seed=w.seed)
    k_gpu = rls.pick_knee(res.inertia.cpu().tolist(), w.k_min, w.k_max, 1.05)
    k_ref = orc.pick_knee(ref["inertia"], w.k_min, w.k_max, 1.05)
    assert k_gpu == k_ref
    cfg = rls.snap_to_valid(res.centroids_of(k_gpu), rls.DeviceDomains(p.dom_offsets, p.dom_values)).cpu().numpy()
    want = orc.snap_to_valid(orc.unpack_centroids(ref["centroids"], w.k_min, k_ref, w.d), p.dom_offsets, p.dom_values)
    np.testing.assert_array_equal(cfg, want)
    assert np.all(cfg >= 0) and np.all(cfg < p.space.sizes)
