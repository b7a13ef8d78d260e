"""The work that a user of this framework has it do, as a list of cases: batches scored by forests
and linear models through the public entry points (`forest_load` / `predict` / `predict_leaves`,
`linear_load` / `predict`), with the model loaded and the rows in device memory beforehand.

A case is a dict of plain values.  Forest cases (kind "full" or "irregular"):
    trees, depth      number of trees; depth of every tree ("full") or the greatest one ("irregular")
    features, outputs columns of X; output columns K
    vector            a leaf holds K values (random forests of class probabilities) or one
    mean              the trees are averaged (random forests) or summed (boosting)
    transform         "none", "sigmoid" or "softmax"
    output            "scores", "both", or "leaves" (leaf ids, one per row and tree)
    grid              thresholds from 255 quantiles (histogram boosting) or drawn freely
    zeros             share of X that is exactly 0 (sparse features)
    rows              rows of the batch
An irregular tree stops growing at a node with probability 0.15 and keeps between an eighth and a
half of the leaves that a full tree of its depth has.  Linear cases (kind "linear"): features,
outputs, transform, output, rows.

Every model and every X comes from the seed: features of splits uniform, thresholds and X ~ N(0, 1),
leaves ~ U(0, 1) where averaged and ~ N(0, 0.1) where summed.
"""
from __future__ import annotations

import statistics

import numpy as np
import torch

import paper_2301_13441_amd as pk
from workloads import (AGG_MEAN, AGG_SUM, OUT_BOTH, OUT_SCORES, TRANSFORM_NONE, TRANSFORM_SIGMOID,
                       TRANSFORM_SOFTMAX, Forest, full_tree_arrays)
from workloads.linear import LinearModel

STOP = 0.15
TRANSFORM = {"none": TRANSFORM_NONE, "sigmoid": TRANSFORM_SIGMOID, "softmax": TRANSFORM_SOFTMAX}
MAX_X = 4_000_000 * 256              # values of X in the largest listed case
MAX_NODES = 4_000_000 * 120_000      # rows x internal nodes in the largest listed case


def _forest(name, kind, rows, trees, depth, features, outputs=1, vector=False, mean=False, transform="none",
            output="both", grid=False, zeros=0.0):
    return dict(name=name, kind=kind, rows=rows, trees=trees, depth=depth, features=features, outputs=outputs,
                vector=vector, mean=mean, transform=transform, output=output, grid=grid, zeros=zeros)


def _linear(name, rows, features, outputs=1, transform="none", output="scores"):
    return dict(name=name, kind="linear", rows=rows, features=features, outputs=outputs, transform=transform,
                output=output)


def listed():
    return [
        # one record at a time from a random forest: an online request, nothing but latency
        _forest("record", "full", 1, 500, 8, 28, mean=True),
        # the smallest batch anyone scores: a ten-tree forest over a thousand rows
        _forest("small_forest", "full", 1_000, 10, 4, 28, mean=True),
        # a micro-batch of a serving queue on a multiclass boosted model, an odd number of rows
        _forest("micro_batch", "full", 1_021, 2000, 6, 128, outputs=10, transform="softmax", zeros=0.3),
        # batch scoring with a random forest of deep full trees
        _forest("random_forest", "full", 1_000_000, 500, 8, 28, mean=True),
        # batch scoring with boosted regression trees, thresholds from quantiles
        _forest("boosted_regression", "full", 1_000_000, 1000, 6, 50, output="scores", grid=True),
        # batch scoring with multiclass boosting: one tree per class and round, softmax and argmax
        _forest("boosted_multiclass", "full", 500_000, 2000, 6, 128, outputs=10, transform="softmax", zeros=0.3),
        # the largest job: a forest of deep irregular trees over wide rows
        _forest("deep_forest", "irregular", 4_000_000, 128, 12, 256, outputs=2, vector=True, mean=True),
        # the inference share of YearPrediction (a fifth of 515 345 x 90): binary boosting, irregular trees
        _forest("boosted_binary", "irregular", 103_069, 300, 9, 90, transform="sigmoid"),
        # a medium batch below the size that fills the chip: multiclass boosting on irregular trees
        _forest("medium_multiclass", "irregular", 10_007, 250, 8, 64, outputs=5, transform="softmax"),
        # leaf ids as features of a second model (trees as feature encoders)
        _forest("leaf_ids", "full", 100_003, 200, 6, 50, output="leaves", grid=True),
        # linear regression at YearPrediction's width, and multinomial logistic regression
        _linear("linear_regression", 4_000_000, 90),
        _linear("logistic_multinomial", 2_000_000, 128, 10, "softmax", "both"),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    """One more case of the same ranges."""
    what = rng.choice(["full", "full", "full", "irregular", "irregular", "irregular", "leaves", "linear", "linear"])
    if what == "linear":
        features = _log_int(rng, 8, 300)
        outputs = rng.choice([1, 1, rng.randint(2, 12)])
        rows = min(_log_int(rng, 1_000, 8_000_000), 400_000_000 // features)
        transform = rng.choice(["none", "sigmoid"]) if outputs == 1 else "softmax"
        return {k: v for k, v in _linear("", rows, features, outputs, transform,
                                         rng.choice(["scores", "both"])).items() if k != "name"}
    kind = what if what != "leaves" else rng.choice(["full", "irregular"])
    features = _log_int(rng, 8, 128 if kind == "full" else 256)
    depth = rng.randint(4, 8) if kind == "full" else rng.randint(6, 12)
    trees = _log_int(rng, 10, 2000 if kind == "full" else 300)
    nodes = trees * ((1 << depth) - 1) // (1 if kind == "full" else 4)
    outputs = rng.choice([1, 1, rng.randint(2, 10)])
    mean = rng.random() < 0.4
    vector = outputs > 1 and kind == "irregular" and mean
    transform = "none" if mean else rng.choice(["none", "sigmoid"]) if outputs == 1 else "softmax"
    rows = min(_log_int(rng, 1, 4_000_000), MAX_X // features, max(1, MAX_NODES // nodes))
    if what == "leaves":
        rows = min(rows, 50_000_000 // trees)
    return {k: v for k, v in _forest("", kind, rows, trees, depth, features, outputs, vector, mean, transform,
                                     "leaves" if what == "leaves" else rng.choice(["scores", "both"]),
                                     rng.random() < 0.3, rng.choice([0.0, 0.0, 0.3])).items() if k != "name"}


def _irregular_shape(rng, depth):
    """(is_leaf, left, right) of one tree in level order, grown by random stopping."""
    lo, hi = (1 << depth) // 8, (1 << depth) // 2
    while True:
        levels, n = [], 1
        for d in range(depth + 1):
            leaf = rng.random(n) < STOP if d < depth else np.ones(n, bool)
            levels.append(leaf)
            n = 2 * int((~leaf).sum())
            if n == 0:
                break
        is_leaf = np.concatenate(levels)
        if lo <= int(is_leaf.sum()) <= hi:
            break
    left = np.full(len(is_leaf), -1, np.int32)
    inner = np.flatnonzero(~is_leaf)
    left[inner] = 1 + 2 * np.arange(len(inner), dtype=np.int32)   # children follow in level order, in pairs
    return is_leaf, left, np.where(is_leaf, -1, left + 1).astype(np.int32)


def _make_forest(case, seed):
    rng = np.random.default_rng(seed)
    trees, outputs = case["trees"], case["outputs"]
    if case["kind"] == "full":
        shape = full_tree_arrays(case["depth"])
        shapes = [shape] * trees
    else:
        shapes = [_irregular_shape(rng, case["depth"]) for _ in range(trees)]
    is_leaf, left, right = (np.concatenate([s[k] for s in shapes]) for k in range(3))
    offset = np.concatenate([[0], np.cumsum([len(s[0]) for s in shapes])]).astype(np.int64)
    n = len(is_leaf)
    feature = np.where(is_leaf, -1, rng.integers(0, case["features"], n)).astype(np.int32)
    if case["grid"]:
        dist = statistics.NormalDist()
        quantiles = np.asarray([dist.inv_cdf(k / 256) for k in range(1, 256)], np.float32)
        threshold = quantiles[rng.integers(0, 255, n)]
    else:
        threshold = rng.standard_normal(n, dtype=np.float32)
    threshold[is_leaf] = 0.0
    width = outputs if case["vector"] else 1
    if case["mean"]:
        leaf = rng.random((n, width), dtype=np.float32)
        if width > 1:
            leaf /= leaf.sum(axis=1, keepdims=True)
    else:
        leaf = rng.standard_normal((n, width), dtype=np.float32) * np.float32(0.1)
    leaf[~is_leaf] = 0.0
    column = np.zeros(trees, np.int32) if case["vector"] else (np.arange(trees) % outputs).astype(np.int32)
    return Forest(n_features=case["features"], n_outputs=outputs, leaf_width=width, tree_offset=offset,
                  feature=feature, threshold=threshold, left=left, right=right, leaf_value=leaf,
                  tree_output=column, aggregate=AGG_MEAN if case["mean"] else AGG_SUM,
                  base_score=None if case["mean"] else np.full(outputs, 0.5, np.float32),
                  transform=TRANSFORM[case["transform"]],
                  output=OUT_SCORES if case["output"] == "scores" else OUT_BOTH)


def _make_linear(case, seed):
    rng = np.random.default_rng(seed)
    weight = (rng.standard_normal((case["features"], case["outputs"])) / np.sqrt(case["features"])).astype(np.float32)
    bias = (rng.standard_normal(case["outputs"]) * 0.1).astype(np.float32)
    return LinearModel(case["features"], case["outputs"], weight, bias, TRANSFORM[case["transform"]],
                       OUT_SCORES if case["output"] == "scores" else OUT_BOTH)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    X = torch.empty((case["rows"], case["features"]), dtype=torch.float32, device="cuda").normal_(generator=gen)
    if case["kind"] == "linear":
        return {"model": pk.linear_load(_make_linear(case, seed)), "X": X, "leaves": False}
    if case["zeros"]:
        X[torch.rand(X.shape, device="cuda", generator=gen) < case["zeros"]] = 0.0
    return {"model": pk.forest_load(_make_forest(case, seed)), "X": X, "leaves": case["output"] == "leaves"}


def run(state):
    if state["leaves"]:
        return state["model"].predict_leaves(state["X"])
    return state["model"].predict(state["X"])


def work(case):
    """X and the model read once, the outputs written once; of a tree, the tests on one row's path
    and the addition of its leaf (the others do not change the answer)."""
    n, f, k = case["rows"], case["features"], case["outputs"]
    bytes_ = 4.0 * n * f
    if case["output"] == "leaves":
        bytes_ += 4.0 * n * case["trees"]
    else:
        bytes_ += 4.0 * n * k + (4.0 * n if case["output"] == "both" else 0.0)
    if case["kind"] == "linear":
        return {"bytes": bytes_ + 4.0 * f * k, "flops": 2.0 * n * f * k}
    t, d = case["trees"], case["depth"]
    if case["kind"] == "full":
        path, inner = float(d), (1 << d) - 1
    else:  # expected length of a path and size of a tree grown by random stopping
        path = sum((1 - STOP) ** (i + 1) for i in range(d))
        inner = sum((1 - STOP) * (2 * (1 - STOP)) ** i for i in range(d))
    width = k if case["vector"] else 1
    return {"bytes": bytes_ + t * (8.0 * inner + 4.0 * width * (inner + 1)),
            "flops": n * t * (path + width)}


def tolerance(case):
    """Leaf ids are exact.  Scores and linear outputs are accumulated in 64 bits and rounded to 32
    bits once: against a 64-bit result the rounding is at most 6e-8 of a value and 3e-8 in the
    2-norm; four times that."""
    if case["output"] == "leaves":
        return "exact"
    return {"rel": 1.2e-7, "max": 2.4e-7}
