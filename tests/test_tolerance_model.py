"""The Lloyd kernels compute distances from two fp16 pieces per operand and re-decide every comparison that falls inside an error
bound with the exact arithmetic.  The parts of that bound (comment at `pair_error_of` in paper_1905_12799_amd/csrc/lloyd_device.h), the
keys and lists that lean on it, and the exact arithmetic's own shortcuts are checked here on the CPU against models in numpy (no
GPU, no oracle); test_gpu_bound.py measures the instructions themselves."""
import numpy as np
import pytest

from tests.matrix_model import (FAMILIES, UNIT, distances, exact_distances, near_ties, operands, padded, pair_error, point_norm,
                                step_model)


def lost_below_normal(v):
    return np.where(np.abs(v) < 2.0 ** -14, 0.0, v).astype(np.float32)


@pytest.mark.parametrize("flush", [False, True])
def test_two_nearest_pieces_stay_inside_their_bound(flush):
    """Pieces rounded to the nearest (`split2_pair` in paper_1905_12799_amd/csrc/lloyd_device.h): what they leave out of a distance
    is at most 6.5 * 2^-23 * (|x'|^2 + |c'|^2) plus 0.0781 * d (comment at `pair_error_of`: 6 + 0.5)."""
    rng = np.random.default_rng(15 + int(flush))
    f64 = np.float64
    worst = 0.0
    for trial in range(80):
        d = int(rng.choice([8, 16, 32]))
        scale = 2.0 ** rng.integers(-24, 14)
        x = (rng.standard_normal((2048, d)) * scale).astype(np.float32)
        c = (rng.standard_normal((2048, d)) * scale * rng.choice([1.0, 0.01, 30.0])).astype(np.float32)
        if trial % 3 == 0:
            x[:, 0] *= 2.0 ** 10
            c[:, 0] *= 2.0 ** 10
        if trial % 4 == 0:                       # halfway between two pieces: the largest remainders
            x = (np.clip(x, -2.0 ** 12, 2.0 ** 12).astype(np.float16).astype(f64) * (1 + 2.0 ** -11 - 2.0 ** -22)).astype(np.float32)
        x = np.clip(x, -2.0 ** 13, 2.0 ** 13)
        C = (-2.0 * np.clip(c, -2.0 ** 13, 2.0 ** 13)).astype(np.float32)
        xh, Ch = (v.astype(np.float16).astype(np.float32) for v in (x, C))
        assert np.all((x - xh).astype(f64) == x.astype(f64) - xh.astype(f64))            # the remainder is exact in fp32
        xl, Cl = ((v - h).astype(np.float16).astype(np.float32) for v, h in ((x, xh), (C, Ch)))
        if flush:
            xh, xl, Ch, Cl = (lost_below_normal(a) for a in (xh, xl, Ch, Cl))
        approx = (xh.astype(f64) * Ch + xh.astype(f64) * Cl + xl.astype(f64) * Ch).sum(1)
        exact = (x.astype(f64) * C.astype(f64)).sum(1)
        S = (x.astype(f64) ** 2).sum(1) + (C.astype(f64) ** 2).sum(1) / 4
        worst = max(worst, float((np.abs(approx - exact) / (6.5 * 2.0 ** -23 * S + 0.0781 * d + d * 2.0 ** -27)).max()))
    assert 0.01 < worst <= 1.0


def model(A, B, acc, bf16):
    return step_model(A, B, acc)


@pytest.mark.parametrize("family", FAMILIES)
@pytest.mark.parametrize("dp", [8, 16, 32])
def test_whole_distances_stay_inside_their_bound(dp, family):
    """Pieces, instructions and norms together: 19.5 units per distance (22 at d_pad 32), which with two for the centring are half of
    43 (48) - and the bound is 48 (56).  Seen: 3.5."""
    assert pair_error(dp) == (56 if dp == 32 else 48)
    rng = np.random.default_rng(100 * dp + FAMILIES.index(family))
    x, c = operands(family, dp, 16, rng)
    xnorm = point_norm(x)
    S = (x.astype(np.float64) ** 2).sum(-1)[:, None, :] + (c.astype(np.float64) ** 2).sum(-1)[:, :, None]
    error = np.abs(distances(x, c, xnorm, dp, model) - exact_distances(x, c, xnorm)) - 0.0781 * dp
    assert (error / (UNIT * S)).max() <= (22 if dp == 32 else 19.5)


@pytest.mark.parametrize("d,k", [(8, 16), (6, 8), (13, 16), (32, 8), (27, 16)])
def test_order_of_two_distances_is_wrong_only_inside_the_bound(d, k):
    """Points with near ties, in the kernels' arithmetic up to the comparison: some of the nearer centroids come out as the farther ones
    (or the labels of such points would show nothing), all of them well inside the bound."""
    X, gap, own = near_ties(np.random.default_rng(d + k), 32 * 64 + k, d, k)
    mean = X.mean(axis=0, dtype=np.float64)
    scale = 2.0 ** (13 - np.ceil(np.log2(np.abs(X - mean).max())))
    centred = np.zeros((X.shape[0], padded(d)), np.float32)
    centred[:, :d] = (X.astype(np.float64) * scale - mean * scale).astype(np.float32)
    x = centred[k:].reshape(64, 32, padded(d))
    wrong = 0.0
    for i in range(k // 2):
        mine = (own == i).reshape(64, 32)
        c = np.zeros((64, 32, padded(d)), np.float32)
        c[:, :2] = centred[2 * i:2 * i + 2]
        got = distances(x, c, point_norm(x), padded(d), model)
        first = got[:, 0] < got[:, 1]
        off = mine & (first != (gap.reshape(64, 32) < 0)) & (got[:, 0] != got[:, 1])
        if off.any():
            wrong = max(wrong, np.abs(gap.reshape(64, 32)[off]).max())
    print(f"d {d}, k {k}: wrong up to {wrong:.2f} units apart")
    assert 0.1 < wrong < pair_error(padded(d)) / 4


@pytest.mark.parametrize("bits", range(8))
def test_keys_tell_no_more_than_the_distances(bits):
    """A key is a distance whose lowest `bits` bits gave way to an index.  The difference of two distances is at least
    g2 (1 - 2^(bits - 22)) - g1 (`key_shrink`), for keys g2 >= |g1| and with one rounding."""
    rng = np.random.default_rng(bits)
    v1 = (2.0 ** rng.uniform(-10, 30, 200000)).astype(np.float32)
    v2 = np.where(rng.random(v1.size) < 0.5, v1 * (1 + 2.0 ** rng.uniform(-24, -8, v1.size)), 2.0 ** rng.uniform(-10, 30, v1.size)).astype(np.float32)
    v1, v2 = np.minimum(v1, v2), np.maximum(v1, v2)

    def key(v):
        return ((v.view(np.uint32) >> bits << bits) | rng.integers(0, 1 << bits, v.size).astype(np.uint32)).view(np.float32)

    g = np.sort(np.stack([key(v1), key(v2)]), axis=0).astype(np.float64)
    shrink = np.array(0x3F800000 - (4 << bits), dtype=np.uint32).view(np.float32).astype(np.float64)
    assert shrink == 1 - 2.0 ** (bits - 22)
    told = (g[1] * shrink - g[0]).astype(np.float32).astype(np.float64)
    diff = v2.astype(np.float64) - v1.astype(np.float64)
    assert np.all((told <= diff) | (told <= 0))


def test_fp32_direct_form_first_stage_keeps_the_fp64_winner():
    """The exact argmin of the Lloyd step settles most calls in fp32: direct-form distances (difference, square, running
    sum with one rounding per multiply-add), then every centroid within 8 (d + 2) 2^-24 of the smallest stays a
    candidate and fp64 decides only among several.  Model of that stage in numpy: the relative error of the fp32 form
    against the exact distance is below (d + 2) 2^-24, and the fp64 winner (lowest index among equals) is always among
    the candidates - also with near-ties planted a few fp32 units apart."""
    rng = np.random.default_rng(41)
    worst = 0.0
    for trial in range(60):
        d = int(rng.choice([8, 16, 32]))
        k = int(rng.integers(2, 129))
        scale = 2.0 ** rng.integers(-30, 30)
        x = (rng.standard_normal(d) * scale).astype(np.float32)
        c = (rng.standard_normal((k, d)) * scale).astype(np.float32)
        if trial % 2 == 0:
            # near-ties: mirror a centroid in x along one feature (the same distance up to rounding), nudge another copy
            j, l = int(rng.integers(0, k - 1)), int(rng.integers(0, d))
            c[j + 1] = c[j]
            c[j + 1, l] = np.float32(2.0) * x[l] - c[j, l]
            if k > 3:
                c[(j + 2) % k] = np.nextafter(c[j], np.float32(np.inf))
        # fp32 stage: sequential multiply-adds (the product and the sum are rounded once together: emulate in fp64, round)
        acc = np.zeros(k, dtype=np.float32)
        for l in range(d):
            diff = (x[l] - c[:, l]).astype(np.float32)
            acc = (diff.astype(np.float64) * diff.astype(np.float64) + acc.astype(np.float64)).astype(np.float32)
        exact = ((x.astype(np.float64)[None, :] - c.astype(np.float64)) ** 2).sum(1)     # exact up to 2^-53 relative
        rel = np.abs(acc.astype(np.float64) - exact) / np.maximum(exact, 1e-300)
        worst = max(worst, float(rel.max() / ((d + 2) * 2.0 ** -24)))
        # the oracle's decision: fp64 direct form with separately rounded multiply and add, lowest index among equals
        d64 = np.zeros(k)
        for l in range(d):
            diff = x[l].astype(np.float64) - c[:, l].astype(np.float64)
            d64 = d64 + diff * diff
        winner = int(np.argmin(d64))
        wmin = acc.min()
        thr = np.float32(np.float64(wmin) * (8 * (d + 2)) * 2.0 ** -24 + np.float64(wmin))
        assert acc[winner] <= thr
    assert worst <= 1.0
    assert worst > 0.02


def test_seeding_skip_rule_never_skips_a_point_that_would_improve():
    """The seeding update leaves a point's row unread when D_i <= (1 - 2^-30) / 4 * |c_a - c_new|^2, a being the
    point's nearest earlier centre (triangle inequality).  Model of the rule in numpy, in the kernel's arithmetic
    (fp64 direct form on fp32 rows): no skipped point may have a strictly smaller distance to the new centre -
    on lattice data, where D_i = |c_a - c_new|^2 / 4 holds exactly for many points, on duplicates and on
    continuous data of very different scales."""
    rng = np.random.default_rng(77)
    cases = []
    for dims, span in ((2, 6), (3, 4), (8, 3), (16, 2)):
        cases.append(rng.integers(0, span + 1, size=(4000, dims)).astype(np.float32))
    cases.append((rng.standard_normal((4000, 16)) * 1e-6).astype(np.float32))
    cases.append((rng.standard_normal((4000, 32)) * 3e5 + 1e6).astype(np.float32))
    line = np.zeros((4001, 4), dtype=np.float32)
    line[:, 0] = np.arange(4001) * 0.5                         # midpoints between centres are data points
    cases.append(line)
    skipped_total = 0
    for X32 in cases:
        X = X32.astype(np.float64)
        n = X.shape[0]
        chain = [int(rng.integers(n))]
        D = ((X - X[chain[0]]) ** 2).sum(1)
        near = np.zeros(n, dtype=np.int64)
        for j in range(1, 24):
            pick = int(rng.integers(n))
            c = X[pick]
            dcc = ((X[chain] - c) ** 2).sum(1)
            thr = dcc * (0.25 * (1.0 - 2.0 ** -30))
            skip = D <= thr[near]
            dn = ((X - c) ** 2).sum(1)
            assert not np.any(skip & (dn < D))
            skipped_total += int(skip.sum())
            better = dn < D
            D = np.where(better, dn, D)
            near = np.where(better, j, near)
            chain.append(pick)
    assert skipped_total > 100000        # the rule does fire on these inputs


@pytest.mark.parametrize("kind", ["lattice", "gauss", "tight"])
def test_ball_rule_keeps_every_nearest_centroid(kind):
    """The tile lists of an ordered sweep: a centroid farther from a unit's centre than the nearest one plus twice the unit's
    radius is left out; distances enter with their error bound either way, and no point's nearest centroid may be missing."""
    rng = np.random.default_rng({"lattice": 1, "gauss": 2, "tight": 3}[kind])
    for _ in range(200):
        d, k = int(rng.integers(1, 33)), int(rng.integers(1, 129))
        if kind == "lattice":
            P, C = rng.integers(0, 4, (32, d)).astype(float), rng.integers(0, 4, (k, d)).astype(float)
        elif kind == "gauss":
            P, C = rng.standard_normal((32, d)) * 100, rng.standard_normal((k, d)) * 100
        else:
            P, C = 1000 + 1e-3 * rng.standard_normal((32, d)), 1000 + rng.standard_normal((k, d))
        b = P.mean(axis=0)
        err = pair_error(padded(d)) * UNIT * ((b ** 2).sum() + (C ** 2).sum(axis=1).max()) + 8
        v = ((C - b) ** 2).sum(axis=1) + err / 2 * rng.uniform(-1, 1, k)          # the matrix pipeline's distances
        radius = np.sqrt(((P - b) ** 2).sum(axis=1)).max()
        reach = np.sqrt(max(v.min(), 0.0) + err) + 2 * radius
        kept = v <= reach ** 2 + 2 * err
        D = ((P[:, None, :] - C[None]) ** 2).sum(axis=2)
        for i in range(32):
            assert kept[D[i] == D[i].min()].all()
