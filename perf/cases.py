"""Performance cases: the work a user of this package has it do, through its public entry points.

Every case is one of these operations:

``tree``    one tree on a given gradient matrix: the sketch, then the level loop (``SplitSearch.step``);
``grow``    the level loop alone on a sketch in hand (``SplitSearch.grow``);
``sketch``  a random projection of a wide gradient matrix, dense or sparse (``SplitSearch.sketch``,
            ``sb_sketch_sparse_projection``);
``boost``   one boosting iteration: update, derivatives, sketch, tree, leaf values (``Booster.step``);
``level``   one level of a tree through the per-step calls, for callers with a level loop of their own
            (``sb_build_histograms``, ``sb_subtract_histograms``, ``sb_score_splits``, ``sb_partition_rows``);
``grad``    loss derivatives and column norms alone (``sb_gradients``);
``leaf``    leaf values of a grown tree with stored per-element hessians (``SplitSearch.leaf_values``).

Inputs are drawn on the GPU from the seed.  Features are quantile-binned (uniform bins), one feature in eight
with few levels as flags and categories have; labels depend on some of the features plus noise; gradients are those
of a softmax or sigmoid cross-entropy at random scores.
"""
import math

import torch

from paper_2211_12858_amd import _lib as L
from paper_2211_12858_amd.driver import Booster, SplitSearch, workspace

DEV = "cuda"
LAM = 1.0
LR = 0.01


def listed():
    return [
        # A small dataset: 10k rows, every output used.  A tree is a few dozen short kernels, so launches count.
        dict(name="tree_10k_identity", op="tree", n=10_000, m=10, bins=256, d=5, k=5, kind="identity", depth=3,
             loss="softmax"),
        # An ordinary multiclass dataset with coarse bins.
        dict(name="tree_200k_top5", op="tree", n=200_000, m=50, bins=64, d=20, k=5, kind="top_outputs", depth=6,
             loss="softmax"),
        # The synthetic timing experiment: 2M rows, 100 features, 100 classes, depth 6 (what bench.py times).
        dict(name="tree_2m_rs5", op="tree", n=2_000_000, m=100, bins=256, d=100, k=5, kind="random_sampling", depth=6,
             loss="softmax"),
        # A large multilabel dataset, deep trees: the histograms of many nodes weigh as much as the rows.
        dict(name="tree_1m_multilabel_top10", op="tree", n=1_000_000, m=200, bins=256, d=500, k=10, kind="top_outputs",
             depth=8, loss="sigmoid"),
        # The level loop at the widest sketch of the paper's experiments (k = 20), odd row and feature counts.
        dict(name="grow_1m_k20", op="grow", n=1_000_003, m=99, bins=256, k=20, depth=6),
        # Random projection of 1000 outputs to 20 columns: one pass over 8 GB of gradients.
        dict(name="sketch_2m_d1000_rp20", op="sketch", n=2_000_000, d=1000, k=20, s=0),
        # A boosting iteration on a small dataset (the smoke shape): many short launches.
        dict(name="boost_20k_rs5", op="boost", n=20_000, m=20, bins=256, d=10, k=5, kind="random_sampling", depth=4,
             loss="softmax"),
        # A boosting iteration on multilabel data, odd sizes.
        dict(name="boost_300k_multilabel", op="boost", n=300_001, m=61, bins=255, d=203, k=10, kind="top_outputs",
             depth=7, loss="sigmoid"),
        # A boosting iteration of the synthetic timing experiment.
        dict(name="boost_2m_rs5", op="boost", n=2_000_000, m=100, bins=256, d=100, k=5, kind="random_sampling", depth=6,
             loss="softmax"),
        # One level (8 nodes) through the per-step calls.
        dict(name="level_500k_8nodes", op="level", n=500_009, m=100, bins=256, k=5, nodes=8),
        # Derivatives of a many-class softmax (more classes than a row's registers hold).
        dict(name="grad_300k_d1000", op="grad", n=300_007, d=1000, loss="softmax", hess=False),
        # Leaf values from stored gradients and hessians.
        dict(name="leaf_1m_d100_hess", op="leaf", n=1_000_000, d=100, leaves=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges; none costs more than the largest listed ones."""
    op = rng.choice(["tree", "tree", "boost", "boost", "grow", "sketch", "level", "grad", "leaf"])
    if op in ("tree", "boost"):
        n, m, bins = _log_int(rng, 5_000, 2_000_000), _log_int(rng, 8, 200), rng.choice([64, 128, 255, 256])
        kind = rng.choice(["top_outputs", "random_sampling", "identity"])
        k = rng.randint(2, 10)
        d = k if kind == "identity" else _log_int(rng, k, 500)
        while n * max(d, m) > 200_000_000 or n * m * ((k + 6) // 6) > 200_000_000:
            n = n // 2 + 1
        return dict(op=op, n=n, m=m, bins=bins, d=d, k=k, kind=kind, depth=rng.randint(3, 7),
                    loss=rng.choice(["softmax", "sigmoid"]))
    if op == "grow":
        return dict(op=op, n=_log_int(rng, 20_000, 1_000_000), m=_log_int(rng, 8, 100), bins=rng.choice([128, 255, 256]),
                    k=rng.randint(6, 20), depth=rng.randint(3, 6))
    if op == "sketch":
        n, d = _log_int(rng, 50_000, 2_000_000), _log_int(rng, 50, 1000)
        return dict(op=op, n=n, d=d, k=rng.randint(2, 20), s=rng.choice([0, 0, 1, 2]))
    if op == "level":
        return dict(op=op, n=_log_int(rng, 20_000, 500_000), m=_log_int(rng, 8, 100), bins=rng.choice([64, 255, 256]),
                    k=rng.randint(2, 10), nodes=rng.choice([2, 4, 8, 16, 32]))
    if op == "grad":
        n, d = _log_int(rng, 20_000, 2_000_000), _log_int(rng, 5, 1000)
        while n * d > 300_000_000:
            n = n // 2 + 1
        return dict(op=op, n=n, d=d, loss=rng.choice(["softmax", "sigmoid"]), hess=rng.choice([False, True]))
    n, d = _log_int(rng, 20_000, 1_000_000), _log_int(rng, 5, 300)
    while n * d > 100_000_000:
        n = n // 2 + 1
    return dict(op="leaf", n=n, d=d, leaves=2 ** rng.randint(3, 9))


# ---------------------------------------------------------------- inputs
def _rng(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _bins(case, g):
    """(n, m) uint8 bins on the GPU, and a signal per row that depends on some of the features."""
    n, m, B = case["n"], case["m"], case["bins"]
    bins = torch.empty((n, m), dtype=torch.uint8, device=DEV)
    signal = 1.5 * torch.randn(n, generator=g, device=DEV)
    for f in range(m):
        u = torch.rand(n, generator=g, device=DEV)
        if f % 8 == 7:  # a feature with few levels
            u = (u * (2 + f % 5)).floor() / (2 + f % 5)
        bins[:, f] = (u * B).to(torch.uint8)
        if f < 6:
            signal += (1.0 if f % 2 else -1.0) * (1.0 - 0.1 * f) * (u - 0.5) * 3.4641016
    return bins, signal


def _labels(signal, d):
    """Class labels in [0, d): the signal's rank in d about equally large classes."""
    p = torch.special.ndtr(signal / 2.45)
    return (p * d).to(torch.int32).clamp_(0, d - 1)


def _targets(signal, d, n, loss, g):
    if loss == "softmax":
        return _labels(signal, d)
    # multilabel: about 5% positives, more of them for some outputs where the signal is high
    Y = torch.empty((d, n), dtype=torch.uint8, device=DEV)
    for j in range(d):
        Y[j] = torch.rand(n, generator=g, device=DEV) < 0.05 + 0.05 * torch.tanh(signal * (1.0 if j % 3 == 0 else 0.2))
    return Y


def _gradients(F, target, loss):
    """fp32 gradients of the loss at the scores F (d, n), in place, and the split-search weight h (n,)."""
    n = F.shape[1]
    if loss == "softmax":
        step = 1 << 18
        for a in range(0, n, step):
            b = min(n, a + step)
            p = torch.softmax(F[:, a:b], dim=0)
            p[target[a:b].long(), torch.arange(b - a, device=DEV)] -= 1.0
            F[:, a:b] = p
        return F, torch.ones(n, device=DEV)
    h = torch.zeros(n, device=DEV)
    for j in range(F.shape[0]):
        s = torch.sigmoid(F[j])
        h += s * (1.0 - s)
        F[j] = s - target[j]
    return F, h / F.shape[0]


def _given_gradients(case, g, signal):
    n, d, loss = case["n"], case["d"], case["loss"]
    F = torch.randn((d, n), generator=g, device=DEV)
    return _gradients(F, _targets(signal, d, n, loss, g), loss)


def _projection(case, g):
    """Pi dense (d, k), or row-sparse with s entries +-1/sqrt(s) per row in distinct columns."""
    d, k, s = case["d"], case["k"], case["s"]
    if s == 0:
        return torch.randn((d, k), generator=g, device=DEV) / math.sqrt(k)
    col = torch.rand((d, k), generator=g, device=DEV).argsort(dim=1)[:, :s].to(torch.int32).contiguous()
    val = (torch.randint(0, 2, (d, s), generator=g, device=DEV) * 2 - 1).to(torch.float32) / math.sqrt(s)
    return col, val


def _leaf_segments(n, leaves, g):
    """Row indices grouped by leaf (ascending inside a leaf, as the level loop leaves them), uneven leaves."""
    weight = torch.rand(leaves, generator=g, device=DEV) ** 2 + 0.02
    edges = torch.cumsum(weight / weight.sum(), 0)[:-1]
    leaf = torch.bucketize(torch.rand(n, generator=g, device=DEV), edges)
    rows = torch.argsort(leaf, stable=True).to(torch.int32)
    off = torch.zeros(leaves + 1, dtype=torch.int32, device=DEV)
    off[1:] = torch.cumsum(torch.bincount(leaf, minlength=leaves), 0).to(torch.int32)
    return leaf, rows, off


def _raw(case, seed):
    """The inputs of a case as tensors, from the seed alone."""
    g = _rng(seed)
    op, n = case["op"], case["n"]
    x = {}
    if op in ("tree", "boost", "grow", "level"):
        x["bins"], signal = _bins(case, g)
    if op == "tree":
        x["G"], x["h"] = _given_gradients(case, g, signal)
        x["u"] = torch.rand(case["k"], generator=g, device=DEV, dtype=torch.float64)
    elif op == "boost":
        x["target"] = _targets(signal, case["d"], n, case["loss"], g)
        x["F"] = torch.randn((case["d"], n), generator=g, device=DEV)
        x["u"] = torch.rand(case["k"], generator=g, device=DEV, dtype=torch.float64)
    elif op in ("grow", "level"):
        # a sketch of k columns: the gradients of k outputs stand for it
        x["G"], x["h"] = _given_gradients(dict(case, d=case["k"], loss="softmax"), g, signal)
        if op == "level":
            x["leaf"], x["rows"], x["off"] = _leaf_segments(n, case["nodes"], g)
    elif op == "sketch":
        signal = torch.randn(n, generator=g, device=DEV)
        x["G"], x["h"] = _given_gradients(dict(case, loss="softmax"), g, signal)
        x["Pi"] = _projection(case, g)
    elif op == "grad":
        signal = torch.randn(n, generator=g, device=DEV)
        x["target"] = _targets(signal, case["d"], n, case["loss"], g)
        x["F"] = 2.0 * torch.randn((case["d"], n), generator=g, device=DEV)
    else:
        x["F"] = torch.randn((case["d"], n), generator=g, device=DEV)
        x["leaf"], x["rows"], x["off"] = _leaf_segments(n, case["leaves"], g)
        p = torch.softmax(x["F"], dim=0)
        x["hess"] = p * (1.0 - p)
        y = torch.randint(0, case["d"], (n,), generator=g, device=DEV)
        p[y, torch.arange(n, device=DEV)] -= 1.0
        x["G"] = p
    return x


def prepare(case, seed):
    x = _raw(case, seed)
    op, n = case["op"], case["n"]
    st = {"case": case}
    if op in ("tree", "grow", "level"):
        depth = case.get("depth", 1)
        st["ss"] = ss = SplitSearch(x["bins"].cpu().numpy(), case["bins"], case["k"], depth, LAM, device=DEV)
    if op == "tree":
        st.update(G=x["G"], h=x["h"], u=x["u"])
        ss.norm2 = torch.zeros(case["d"], dtype=torch.float64, device=DEV)
    elif op in ("grow", "level"):
        ss.sketch("identity", x["G"], x["h"])
    if op == "level":
        m, B, k, nn = case["m"], case["bins"], case["k"], case["nodes"]
        off = x["off"]
        size = off[1:] - off[:-1]
        pair = torch.arange(0, nn, 2, dtype=torch.int32, device=DEV)
        build = pair + (size[0::2] > size[1::2]).to(torch.int32)
        shape = (nn, m, k + 1, B)
        st.update(rows=x["rows"], off=off, build=build, H=torch.zeros(shape, dtype=torch.float64, device=DEV),
                  Hp=torch.zeros((nn // 2,) + shape[1:], dtype=torch.float64, device=DEV),
                  bf=torch.zeros(nn, dtype=torch.int32, device=DEV), bb=torch.zeros(nn, dtype=torch.int32, device=DEV),
                  bs=torch.zeros(nn, dtype=torch.float64, device=DEV),
                  rows_out=torch.zeros(n, dtype=torch.int32, device=DEV),
                  off_out=torch.zeros(2 * nn + 1, dtype=torch.int32, device=DEV),
                  build_out=torch.zeros(nn, dtype=torch.int32, device=DEV),
                  ws_h=workspace(L.sb_workspace_bytes(L.SB_CALL_BUILD_HISTOGRAMS, n=n, m=m, n_bins=B, k=k, n_nodes=nn), DEV),
                  ws_s=workspace(L.sb_workspace_bytes(L.SB_CALL_SCORE_SPLITS, m=m, n_nodes=nn), DEV),
                  ws_p=workspace(L.sb_workspace_bytes(L.SB_CALL_PARTITION_ROWS, n=n, n_nodes=nn), DEV))
        # the level above, whose histograms a level loop has in hand
        L.sb_build_histograms(None, 0, ss.rec, ss.ld_rec, n, m, B, ss.GH, ss.ld_gh, k, ss.qexp, st["rows"],
                              off[::2].contiguous(), nn // 2, None, nn // 2, st["Hp"], st["ws_h"], st["ws_h"].numel())
    elif op == "boost":
        st["bst"] = bst = Booster(x["bins"].cpu().numpy(), case["bins"], case["d"], case["loss"], case["kind"],
                                  case["k"], case["depth"], LAM, LR, device=DEV, F0=x["F"])
        bst.set_target(x["target"])
        st["u"] = x["u"]
    elif op == "sketch":
        k = case["k"]
        # a projection needs no bins: the sketch call's own buffers are all a program keeps for it
        st.update(G=x["G"], h=x["h"], Pi=x["Pi"], ld=(k + 8) // 8 * 8, qexp=torch.zeros(k + 1, dtype=torch.int32, device=DEV))
        st["GH"] = torch.zeros((n, st["ld"]), device=DEV)
        st["ws"] = workspace(L.sb_workspace_bytes(L.SB_CALL_SKETCH, n=n, d=case["d"], k=k), DEV)
    elif op == "grad":
        d = case["d"]
        st.update(F=x["F"], target=x["target"], G=torch.empty_like(x["F"]),
                  hess=torch.empty_like(x["F"]) if case["hess"] else None,
                  h_row=torch.empty(n, device=DEV) if case["loss"] == "sigmoid" else None,
                  norm2=torch.zeros(d, dtype=torch.float64, device=DEV),
                  ws=workspace(L.sb_workspace_bytes(L.SB_CALL_GRADIENTS, n=n, d=d), DEV))
    elif op == "leaf":
        d, nl = case["d"], case["leaves"]
        st.update(G=x["G"], hess=x["hess"], rows=x["rows"], off=x["off"],
                  V=torch.zeros((nl, d), dtype=torch.float64, device=DEV),
                  ws=workspace(L.sb_workspace_bytes(L.SB_CALL_LEAF_VALUES, n=n, d=d, n_nodes=nl), DEV))
    return st


# ---------------------------------------------------------------- one pass
def _tree_outputs(ss):
    return {"feature": ss.tree_feature, "bin": ss.tree_bin, "score": ss.tree_score, "rows": ss.row_idx,
            "leaf_off": ss.leaf_off}


def run(st):
    case = st["case"]
    op, n = case["op"], case["n"]
    if op == "tree":
        ss = st["ss"]
        ss.step(case["kind"], st["G"], st["h"], u=st["u"])
        return dict(_tree_outputs(ss), norm2=ss.norm2, cols=ss.cols, scales=ss.scales)
    if op == "grow":
        st["ss"].grow()
        return _tree_outputs(st["ss"])
    if op == "boost":
        bst = st["bst"]
        bst.step(u=st["u"])
        return dict(_tree_outputs(bst.ss), G=bst.G, norm2=bst.norm2, V=bst.ss.V)
    if op == "sketch":
        d, k = case["d"], case["k"]
        if case["s"]:
            col, val = st["Pi"]
            L.sb_sketch_sparse_projection(st["G"], n, d, n, st["h"], k, case["s"], col, val, st["GH"], st["ld"],
                                          st["qexp"], st["ws"], st["ws"].numel())
        else:
            L.sb_sketch(L.SB_SKETCH_RANDOM_PROJECTION, st["G"], n, d, n, st["h"], k, None, st["Pi"], st["GH"],
                        st["ld"], None, None, None, st["qexp"], st["ws"], st["ws"].numel())
        return {"GH": st["GH"], "qexp": st["qexp"]}
    if op == "level":
        ss, m, B, k, nn = st["ss"], case["m"], case["bins"], case["k"], case["nodes"]
        L.sb_build_histograms(None, 0, ss.rec, ss.ld_rec, n, m, B, ss.GH, ss.ld_gh, k, ss.qexp, st["rows"], st["off"],
                              nn, st["build"], nn // 2, st["H"], st["ws_h"], st["ws_h"].numel())
        L.sb_subtract_histograms(st["Hp"], st["H"], nn // 2, m, B, k, st["build"])
        L.sb_score_splits(st["H"], nn, m, B, k, LAM, 0.0, st["bf"], st["bb"], st["bs"], st["ws_s"], st["ws_s"].numel())
        L.sb_partition_rows(ss.bins_cm, n, m, n, st["rows"], st["off"], nn, st["bf"], st["bb"], st["rows_out"],
                            st["off_out"], st["build_out"], st["ws_p"], st["ws_p"].numel())
        return {"H": st["H"], "feature": st["bf"], "bin": st["bb"], "score": st["bs"], "rows": st["rows_out"],
                "off": st["off_out"], "build": st["build_out"]}
    if op == "grad":
        soft = case["loss"] == "softmax"
        L.sb_gradients(L.LOSS[case["loss"]], st["F"], n, case["d"], n, st["target"] if soft else None,
                       None if soft else st["target"], n, st["G"], n, st["hess"], n, st["h_row"], st["norm2"],
                       st["ws"], st["ws"].numel())
        return {"G": st["G"], "hess": st["hess"], "h_row": st["h_row"], "norm2": st["norm2"]}
    L.sb_leaf_values(st["G"], n, case["d"], n, st["hess"], n, None, st["rows"], st["off"], case["leaves"], LAM, st["V"],
                     case["d"], st["ws"], st["ws"].numel())
    return {"V": st["V"]}


# ---------------------------------------------------------------- what a pass needs
def work(case):
    """Inputs read once, outputs written once; the adds of the histograms (the root's rows, and at most half of
    them on each further level) and the multiplies and adds of the other steps."""
    op, n = case["op"], case["n"]
    m, d, k = case.get("m", 0), case.get("d", 0), case.get("k", 0)
    c = k + 1
    tree_flops = n * m * c * (1 + 0.5 * (case.get("depth", 1) - 1))
    if op == "tree":
        return {"bytes": 4 * n * d + 4 * n + n * m + 4 * n, "flops": 2 * n * d + tree_flops}
    if op == "grow":
        return {"bytes": 4 * n * c + n * m + 4 * n, "flops": tree_flops}
    if op == "boost":
        # scores read and written, gradients written (they are read again by the leaf values: an output of the
        # step already), targets, bins, row order
        target = 4 * n if case["loss"] == "softmax" else n * d
        return {"bytes": 12 * n * d + target + n * m + 4 * n, "flops": 20 * n * d + tree_flops}
    if op == "sketch":
        s = case["s"] or k
        return {"bytes": 4 * n * d + 4 * n + 4 * n * c, "flops": 2 * n * d * s}
    if op == "level":
        H = case["nodes"] * m * c * case["bins"] * 8
        return {"bytes": n * (4 + m / 2 + 4 * c / 2) + 1.5 * H + 4 * n, "flops": n / 2 * m * c}
    if op == "grad":
        target = 4 * n if case["loss"] == "softmax" else n * d
        return {"bytes": (12 if case["hess"] else 8) * n * d + target + 8 * d, "flops": 20 * n * d}
    return {"bytes": 8 * n * d + 4 * n + 8 * case["leaves"] * d, "flops": 2 * n * d}


def tolerance(case):
    """About four times the error against ``exact`` (random projections 4e-7; gradients 4e-8 and row means 3.7e-7;
    histograms of 18-bit fixed-point values 1.4e-7; leaf values, exact to 41 bits, below 1e-10).  Trees follow from
    exact integer sums: whole values are the same, and the scales carry one fp32 rounding (3e-8)."""
    op = case["op"]
    if op in ("tree", "grow"):
        return {"rel": 1.5e-7, "differ": 0.0}
    if op == "boost":
        return {"rel": 2e-7, "differ": 0.0}
    if op == "sketch":
        return {"rel": 2e-6, "max": 1e-4, "differ": 0.0}
    if op == "level":
        return {"rel": 6e-7, "max": 1e-4, "differ": 0.0}
    if op == "grad":
        return {"rel": 1.5e-6, "max": 1e-4}
    return {"rel": 1e-9, "max": 1e-6}


def exact(case, seed):
    """The computed numbers in 64 bits.  A tree's split scores follow from its own earlier splits and have no value
    of their own here; the ``level`` cases check the histograms and scores."""
    x = _raw(case, seed)
    op, n = case["op"], case["n"]
    none_tree = {"feature": None, "bin": None, "score": None, "rows": None, "leaf_off": None}
    if op == "grow":
        return None
    if op == "tree":
        norm2 = torch.stack([col.double().square().sum() for col in x["G"]])
        return dict(none_tree, norm2=norm2, cols=None, scales=_exact_scales(case, norm2, x["u"]))
    if op == "boost":
        G, _, _ = _exact_gradients(x["F"], x["target"], case["loss"], False)
        return dict(none_tree, G=G, norm2=torch.stack([col.square().sum() for col in G]), V=None)
    if op == "grad":
        G, hess, h_row = _exact_gradients(x["F"], x["target"], case["loss"], True)
        return {"G": G, "hess": hess if case["hess"] else None, "h_row": h_row if case["loss"] == "sigmoid" else None,
                "norm2": torch.stack([col.square().sum() for col in G])}
    if op == "sketch":
        k, d = case["k"], case["d"]
        if case["s"]:
            col, val = x["Pi"]
            Pi = torch.zeros((d, k), dtype=torch.float64, device=DEV).scatter_add_(1, col.long(), val.double())
        else:
            Pi = x["Pi"].double()
        GH = torch.zeros((n, (k + 8) // 8 * 8), dtype=torch.float64, device=DEV)
        for a in range(0, n, 1 << 17):
            b = min(n, a + (1 << 17))
            GH[a:b, :k] = x["G"][:, a:b].double().t().contiguous() @ Pi
        GH[:, k] = x["h"].double()
        return {"GH": GH, "qexp": None}
    if op == "level":
        return _exact_level(case, x)
    nl, d = case["leaves"], case["d"]
    V = torch.zeros((nl, d), dtype=torch.float64, device=DEV)
    for j in range(d):
        sg = torch.zeros(nl, dtype=torch.float64, device=DEV).index_add_(0, x["leaf"], x["G"][j].double())
        sh = torch.zeros(nl, dtype=torch.float64, device=DEV).index_add_(0, x["leaf"], x["hess"][j].double())
        V[:, j] = -sg / (sh + LAM)
    return {"V": V}


def _exact_scales(case, norm2, u):
    if case["kind"] != "random_sampling":
        return torch.ones(case["k"], dtype=torch.float64, device=DEV)
    C = torch.cumsum(norm2, 0)
    cols = torch.searchsorted(C, u * C[-1], right=True).clamp_(0, case["d"] - 1)
    return torch.sqrt(C[-1] / (case["k"] * norm2[cols]))


def _exact_gradients(F, target, loss, want_hess):
    d, n = F.shape
    G = torch.empty((d, n), dtype=torch.float64, device=DEV)
    hess = torch.empty_like(G) if want_hess else None
    step = 1 << 17
    for a in range(0, n, step):
        b = min(n, a + step)
        z = F[:, a:b].double()
        p = torch.softmax(z, dim=0) if loss == "softmax" else torch.sigmoid(z)
        if want_hess:
            hess[:, a:b] = p * (1.0 - p)
        if loss == "softmax":
            p[target[a:b].long(), torch.arange(b - a, device=DEV)] -= 1.0
        else:
            p -= target[:, a:b]
        G[:, a:b] = p
    return G, hess, hess.mean(dim=0) if want_hess else None


def _exact_level(case, x):
    m, B, k, nn = case["m"], case["bins"], case["k"], case["nodes"]
    ch = torch.cat([x["G"], x["h"][None]]).double()
    H = torch.zeros((nn, m, k + 1, B), dtype=torch.float64, device=DEV)
    for f in range(m):
        at = x["leaf"] * B + x["bins"][:, f].long()
        for t in range(k + 1):
            H[:, f, t] = torch.zeros(nn * B, dtype=torch.float64, device=DEV).index_add_(0, at, ch[t]).view(nn, B)
    left = H.cumsum(-1)[..., :-1]
    right = H.sum(-1, keepdim=True) - left
    hl, hr = left[:, :, k], right[:, :, k]
    S = (left[:, :, :k].square().sum(2) / (hl + LAM)) + (right[:, :, :k].square().sum(2) / (hr + LAM))
    # a side without rows is no split
    S = torch.where((hl > 0.5) & (hr > 0.5), S, torch.full_like(S, -math.inf))
    return {"H": H, "feature": None, "bin": None, "score": S.view(nn, -1).max(dim=1).values, "rows": None, "off": None,
            "build": None}
