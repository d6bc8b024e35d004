"""The work a tuner gives this library, as cases to be timed.

A tuner's round scores the configurations of a trajectory with its boosted-tree cost model (gbt_score), clusters them
with k-means for every k of a range (kmeans_sweep), stops at the knee of the loss curve and hands the centroids on as
valid configurations (snap_to_valid), with configurations it has measured before replaced by the trajectory's modes
(knob_modes, replace_visited); the search agent moves its configurations on in between (apply_actions).

The inputs are conv2d knob spaces as in paper_1905_12799_amd.synth (8 knob indices, 8 log2 loop extents, up to 16
log-normal extent/stride columns), drawn on the GPU.  Sizes are those of synth.WORKLOADS, and odd ones between them.
"""
import functools

import torch

from paper_1905_12799_amd import binding as rls
from paper_1905_12799_amd import synth

KNEE_CONST = 1.05
N_VISITED = 65536
KNOBS = 8


def listed():
    return [
        # a small round (the `tiny` workload): dependent launches of a few microseconds, what a sweep costs at the least
        {"name": "sweep_tiny", "kind": "sweep", "n": 2000, "d": 8, "mixture": 6, "k_min": 1, "k_max": 16, "iters": 20},
        # an ordinary trajectory (the `mid` workload)
        {"name": "sweep_mid", "kind": "sweep", "n": 65536, "d": 16, "mixture": 32, "k_min": 1, "k_max": 64, "iters": 30},
        # a ragged one: odd number of rows, features that fill neither a register nor a row of 16 bytes, the paper's range of k
        {"name": "sweep_ragged", "kind": "sweep", "n": 300007, "d": 13, "mixture": 20, "k_min": 8, "k_max": 63, "iters": 17},
        # every configuration of a layer's sample (the `whole_layer` workload)
        {"name": "sweep_whole_layer", "kind": "sweep", "n": 1048576, "d": 16, "mixture": 0, "k_min": 1, "k_max": 64, "iters": 30},
        # the largest feature space (the `large` workload)
        {"name": "sweep_large", "kind": "sweep", "n": 8388608, "d": 32, "mixture": 128, "k_min": 1, "k_max": 128, "iters": 30},
        # all layers of a network at once (the `batched` workload)
        {"name": "sweep_batched", "kind": "sweep_batched", "batch": 64, "n": 262144, "d": 16, "mixture": 0, "k_min": 1, "k_max": 32,
         "iters": 30},
        # Algorithm 1 as it is written: k = 8, 9, ... 63 until the knee, in waves of 16
        {"name": "until_knee", "kind": "knee", "n": 1000003, "d": 16, "mixture": 0, "k_min": 8, "k_max": 63, "iters": 30},
        # one whole round of the tuner, host steps included, on a trajectory of ordinary size
        {"name": "round", "kind": "round", "n": 100003, "d": 16, "mixture": 32, "k_min": 1, "k_max": 32, "iters": 20, "trees": 256,
         "depth": 8},
        # the cost model on a small round: latency
        {"name": "score_tiny", "kind": "score", "n": 2000, "d": 8, "mixture": 6, "trees": 64, "depth": 6},
        # the cost model on the largest feature space
        {"name": "score_large", "kind": "score", "n": 8388608, "d": 32, "mixture": 128, "trees": 512, "depth": 10},
        # one cost model per layer of a network
        {"name": "score_batched", "kind": "score_batched", "batch": 64, "n": 262144, "d": 16, "mixture": 0, "trees": 256, "depth": 8},
        # a step of the search agent: its configurations move by one action each and are scored where they arrive
        {"name": "agent_step", "kind": "agent", "n": 65536, "d": 8, "mixture": 0, "trees": 256, "depth": 8},
    ]


def _between(rng, lo, hi):
    """A whole number in lo..hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    """Another case: any of the calls, sizes between the smallest and the largest listed."""
    kind = rng.choice(["sweep", "sweep", "sweep", "sweep_batched", "knee", "round", "score", "score", "score_batched", "agent"])
    case = {"kind": kind}
    top = 8388608
    if kind in ("sweep_batched", "score_batched"):
        case["batch"] = _between(rng, 2, 64)
        top = 16777216 // case["batch"]
    elif kind == "agent":
        top = 1048576
    case["n"] = _between(rng, 2000, min(top, 8388608))
    if kind == "agent":
        case["d"] = KNOBS
    else:
        case["d"] = rng.choice([8, 16, 32]) if rng.random() < 0.5 else rng.randint(5 if kind.startswith("sweep") else KNOBS, 32)
        if "batch" in case:
            case["d"] = min(case["d"], 16)
    case["mixture"] = rng.choice([0, 6, 32, 128])
    if kind in ("sweep", "sweep_batched", "knee", "round"):
        case["k_max"] = _between(rng, 4, {"sweep": 128, "sweep_batched": 32}.get(kind, 64))
        case["k_min"] = 1
        if case["k_max"] > 8 and rng.random() < 0.5:
            case["k_min"] = 8                            # the paper's range begins at 8
        if kind == "sweep" and rng.random() < 0.25:
            case["k_min"] = case["k_max"]                # a user with a fixed k
        case["iters"] = rng.randint(10, 30)
    if kind in ("round", "score", "score_batched", "agent"):
        case["trees"] = _between(rng, 64, 256 if "batch" in case else 512)
        case["depth"] = rng.randint(4, 8 if "batch" in case else 10)
    return case


# ---- inputs ------------------------------------------------------------------------------------------------------

_SHAPES = synth.batched_conv_shapes(128)


@functools.lru_cache(maxsize=None)
def _space(conv):
    """Knob domains of a conv2d template and, per knob, the loop extents that the derived columns look up."""
    space = synth.conv2d_knob_space(*conv)
    tables = []
    for j, cols in ((0, (0, 2)), (1, (0, 2)), (2, (0, 2)), (3, (1,)), (4, (1,)), (5, (1,))):
        entries = torch.tensor(space.entries[j], dtype=torch.float64)
        tables.append(torch.log2(entries[:, list(cols)]).float())
    return space, tables


def _knobs(space, n, mixture, gen):
    """Knob indices [n, 8] as floats: a Gaussian mixture in index space, rounded and clamped, or uniform draws; and the component."""
    sizes = torch.tensor(space.sizes, dtype=torch.float32, device="cuda")
    if mixture == 0:
        u = torch.rand(n, KNOBS, generator=gen, device="cuda")
        return torch.minimum((u * sizes).floor_(), sizes - 1), torch.zeros(n, dtype=torch.int64, device="cuda")
    means = torch.rand(mixture, KNOBS, generator=gen, device="cuda") * (sizes - 1)
    comp = torch.randint(mixture, (n,), generator=gen, device="cuda")
    v = torch.randn(n, KNOBS, generator=gen, device="cuda")
    v.mul_(torch.clamp(0.08 * sizes, min=0.5)).add_(means[comp]).round_()
    return torch.minimum(v.clamp_(min=0), sizes - 1), comp


def _rows(conv, n, d, mixture, gen):
    """Feature matrix [n, d] of one space."""
    space, tables = _space(conv)
    knobs, comp = _knobs(space, n, mixture, gen)
    cols = [knobs]
    if d > KNOBS:
        idx = knobs.long()
        looked = [t.cuda()[idx[:, j]] for j, t in enumerate(tables)]
        cols += looked[:4] + [looked[4] + looked[5]]
    if d > 16:
        centres = torch.randn(max(mixture, 1), d - 16, generator=gen, device="cuda").exp_()
        z = torch.randn(n, d - 16, generator=gen, device="cuda")
        cols.append(z.mul_(0.1).add_(1.0).mul_(centres[comp]))
    return torch.cat(cols, dim=1)[:, :d].contiguous()


def _forest(X, trees, depth, gen):
    """Random splits within the columns' ranges (half-integers on index columns), leaves N(0, 1)."""
    d, inner = X.shape[1], (1 << depth) - 1
    lo, hi = X.min(dim=0).values, X.max(dim=0).values
    feat = torch.randint(d, (trees, inner), generator=gen, device="cuda", dtype=torch.int32)
    at = feat.long()
    thr = lo[at] + torch.rand(trees, inner, generator=gen, device="cuda") * (hi - lo)[at]
    thr = torch.where(feat < KNOBS, thr.floor() + 0.5, thr)
    leaf = torch.randn(trees, 1 << depth, generator=gen, device="cuda")
    return rls.DeviceForest(trees, depth, d, 0.0, feat, thr, leaf)


def _domains(conv):
    return rls.DeviceDomains(*_space(conv)[0].domains_csr())


def prepare(case, seed):
    """Trajectory, cost models, knob domains, history and workspace: what a tuner holds when a round begins."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kind, n, d = case["kind"], case["n"], case["d"]
    batch = case.get("batch", 1)
    convs = [_SHAPES[(seed + b) % len(_SHAPES)] for b in range(batch)]
    if batch == 1:
        convs = [(256, 256, 14, 3) if d <= 16 else (512, 512, 28, 3)]
    s = {"case": case, "seed": seed, "kind": kind}
    if kind == "agent":
        space = _space(convs[0])[0]
        knobs, _ = _knobs(space, n, case["mixture"], gen)
        s["cfg"] = knobs.to(torch.int32).contiguous()
        s["action"] = torch.randint(-1, 2, (n, KNOBS), generator=gen, device="cuda", dtype=torch.int8)
        s["domains"] = _domains(convs[0])
        s["forest"] = _forest(knobs, case["trees"], case["depth"], gen)
        return s
    if "batch" in case:
        X = torch.empty(batch, n, d, device="cuda")
        for b in range(batch):
            X[b] = _rows(convs[b], n, d, case["mixture"], gen)
        s["X"] = X
        if kind == "score_batched":
            s["forests"] = [_forest(X[b], case["trees"], case["depth"], gen) for b in range(batch)]
            s["out"] = torch.empty(batch, n, device="cuda")
    else:
        s["X"] = X = _rows(convs[0], n, d, case["mixture"], gen)
        if kind in ("score", "round"):
            s["forest"] = _forest(X, case["trees"], case["depth"], gen)
            s["out"] = torch.empty(n, device="cuda")
    if kind in ("sweep", "sweep_batched", "round"):
        need = rls.kmeans_sweep_workspace_bytes(n, d, case["k_min"], case["k_max"], batch)
        s["workspace"] = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
    if kind == "round":
        s["domains"] = _domains(convs[0])
        half = torch.randint(n, (N_VISITED // 2,), generator=gen, device="cuda")
        rest, _ = _knobs(_space(convs[0])[0], N_VISITED - N_VISITED // 2, 0, gen)
        s["visited"] = torch.cat([X[half, :KNOBS], rest]).to(torch.int32).contiguous()
    return s


# ---- one pass ------------------------------------------------------------------------------------------------------

def run(s):
    case, kind = s["case"], s["kind"]
    if kind == "score":
        return rls.gbt_score(s["forest"], s["X"], out=s["out"])
    if kind == "score_batched":
        return rls.gbt_score_batched(s["forests"], s["X"], out=s["out"])
    if kind == "agent":
        cfg, features = rls.apply_actions(s["cfg"], s["action"], s["domains"])
        return {"cfg": cfg, "features": features, "scores": rls.gbt_score(s["forest"], features)}
    ks = (case["k_min"], case["k_max"])
    if kind == "sweep":
        r = rls.kmeans_sweep(s["X"], *ks, case["iters"], seed=s["seed"], workspace=s["workspace"])
        return {"labels": r.labels, "centroids": r.centroids, "inertia": r.inertia}
    if kind == "sweep_batched":
        seeds = [s["seed"] + b for b in range(case["batch"])]
        r = rls.kmeans_sweep_batched(s["X"], *ks, case["iters"], seeds=seeds, workspace=s["workspace"])
        return {"labels": r.labels, "centroids": r.centroids, "inertia": r.inertia}
    if kind == "knee":
        k, n_done, r = rls.kmeans_sweep_until_knee(s["X"], *ks, 16, case["iters"], KNEE_CONST, seed=s["seed"])
        rows = sum(range(ks[0], ks[0] + n_done))         # only the runs up to the knee are written
        return {"k": k, "n_done": n_done, "labels": r.labels[:n_done], "centroids": r.centroids[:rows * case["d"]],
                "inertia": r.inertia[:n_done]}
    # a tuner's round: the losses come to the host for the knee, everything else stays on the GPU
    scores = rls.gbt_score(s["forest"], s["X"], out=s["out"])
    r = rls.kmeans_sweep(s["X"], *ks, case["iters"], seed=s["seed"], workspace=s["workspace"], check_status=False)
    inertia = r.inertia.tolist()
    k = rls.pick_knee(inertia, *ks, KNEE_CONST)
    cfg = rls.snap_to_valid(r.centroids_of(k), s["domains"])
    mode, hist = rls.knob_modes(s["X"], s["domains"])
    replaced = rls.replace_visited(cfg, s["visited"], mode)
    return {"scores": scores, "labels": r.labels, "centroids": r.centroids, "inertia": r.inertia, "k": k, "cfg": cfg, "mode": mode,
            "hist": hist, "replaced": replaced}


# ---- what a pass cannot do without ---------------------------------------------------------------------------------

def work(case):
    """Rows, forests and history read once, outputs written once; the distances of every assignment and of the seeding
    (2 d flop per pair), a compare per tree level and an add per tree."""
    n, d, batch, kind = case["n"], case["d"], case.get("batch", 1), case["kind"]
    rows = float(batch) * n
    total_bytes, flops = 4.0 * d * rows, 0.0
    if kind in ("score", "score_batched", "agent", "round"):
        total_bytes += 4.0 * rows + batch * case["trees"] * 12.0 * (1 << case["depth"])
        flops += rows * case["trees"] * (case["depth"] + 1.0)
    if kind == "agent":
        total_bytes += rows * KNOBS * (4 + 1 + 4)        # configurations and actions in, configurations out (features: above)
    if kind in ("sweep", "sweep_batched", "round", "knee"):
        # (until the knee: at least the first wave of 16)
        k_last = case["k_max"] if kind != "knee" else min(case["k_max"], case["k_min"] + 15)
        runs, sum_k = k_last - case["k_min"] + 1, sum(range(case["k_min"], k_last + 1))
        total_bytes += rows * 4.0 * runs + batch * (sum_k * d * 4.0 + runs * 8.0)
        flops += 2.0 * d * rows * (sum_k * (case["iters"] + 1.0) + k_last - 1.0)
    if kind == "round":
        total_bytes += N_VISITED * KNOBS * 4.0
    return {"bytes": total_bytes, "flops": flops}


def tolerance(case):
    """Scores are fp32 sums in tree order, labels and configurations are defined exactly, centroids are exact means rounded
    to fp32, losses fp64 sums."""
    if case["kind"] in ("score", "score_batched", "agent"):
        return "exact"
    return {"rel": 1e-6, "differ": 0.0}
