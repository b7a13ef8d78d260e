"""What a call launches: batches longer than one launch may be, and the kernels that calls reach."""
import numpy as np
import pytest

import oracle
import workloads as wl
from test_gpu_parity import _full_forest

HIP_MAX_THREADS = 1 << 32  # threads per grid axis, exclusive


def _vector_forest(outputs, features=1, trees=5):
    return wl.random_forest(17 + outputs, n_trees=trees, n_features=features, max_depth=9, stop_prob=0.3, n_outputs=outputs,
                            leaf_width=outputs, aggregate=wl.AGG_MEAN, transform=wl.TRANSFORM_NONE)


@pytest.mark.parametrize("rows", [1, 8192, 1 << 27, (1 << 27) + 1, 1 << 28, 600_000_000, 10**9])
@pytest.mark.parametrize("what", ["vector3", "vector2", "columns", "one_column", "wide", "ranklds", "lds"])
def test_no_launch_asks_for_more_threads_than_hip_takes(what, rows):
    from paper_2301_13441_amd import binding
    f = {"vector3": lambda: _vector_forest(3), "vector2": lambda: _vector_forest(2),
         "columns": lambda: _full_forest(1, 12, 5, 4, n_outputs=2), "one_column": lambda: _full_forest(1, 12, 8, 2),
         "wide": lambda: _full_forest(1, 12, 5, 600), "ranklds": lambda: _vector_forest(17, 9),
         "lds": lambda: _vector_forest(20, 300, 96)}[what]()
    for leaves in (False, True):
        s = binding.forest_packed_launch(f, rows, leaves)
        assert s["workgroups"] * s["threads"] < HIP_MAX_THREADS
        assert s["launches"] * s["workgroups"] * s["rows_per_workgroup"] >= rows
        assert s["launches"] == 1 or s["shares"] == 1


@pytest.mark.gpu
@pytest.mark.parametrize("what,form,kernel", [("vector3", "walk", "deep"), ("full", "walk", "walk"), ("full", "dense", "rank")])
def test_batches_longer_than_a_launch(what, form, kernel):
    """268 million rows and a ragged rest: the first rows, the last ones and those on both sides of every border
    between two launches, scores, labels and leaf ids."""
    import torch
    from paper_2301_13441_amd import binding
    f = _vector_forest(3) if what == "vector3" else _full_forest(9, 3, 5, 1, n_outputs=2)
    n = (1 << 28) + 77
    xd = torch.empty((n, 1), dtype=torch.float32, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(3)
    for at in range(0, n, 1 << 26):
        xd[at:at + (1 << 26)].normal_(generator=gen)
    border = [b + i for b in (1 << 26, 1 << 27, 3 << 26, 1 << 28) for i in range(-70, 70) if b + i < n]
    pick = np.unique(np.concatenate([np.arange(300), border, np.arange(n - 300, n),
                                     np.random.default_rng(1).integers(0, n, 3000)]))
    idx = torch.from_numpy(pick).cuda()
    ref = oracle.predict(f, xd[idx].cpu().numpy(), want_leaves=True, n_threads=8)
    model = binding.forest_load_form(f, form)
    try:
        s = binding.forest_launch(model, n)
        assert s["launches"] == 3 and s["kernel"] == kernel
        scores, labels = model.predict(xd)
        np.testing.assert_array_equal(labels[idx].cpu().numpy(), ref.labels)
        np.testing.assert_allclose(scores[idx].cpu().numpy(), ref.scores, rtol=1e-5, atol=1e-6)
        del scores, labels
        np.testing.assert_array_equal(model.predict_leaves(xd)[idx].cpu().numpy(), ref.leaf_node_id)
    finally:
        model.close()


def test_shares_of_shallow_trees():
    """A copy of depth-3 trees is 16 of them: a wave with one copy has work enough, if three shares come of it."""
    from paper_2301_13441_amd import binding
    shares = lambda trees, depth: binding.forest_packed_launch(_full_forest(3, trees, depth, 10), 3000)["shares"]
    assert shares(1000, 3) == shares(1000, 1) == 3 and shares(768, 3) == 3
    assert shares(700, 3) == 1 and shares(300, 4) == 1 and shares(1000, 4) == 3


@pytest.mark.gpu
@pytest.mark.parametrize("trees,outputs", [(768, 1), (1000, 5), (2000, 3)])
def test_shares_of_shallow_trees_against_the_oracle(trees, outputs):
    from test_gpu_parity import _check
    rng = np.random.default_rng(trees)
    f = _full_forest(trees, trees, 3, 10, n_outputs=outputs)
    for rows in (517, 3000):
        _check(f, rng.standard_normal((rows, 10)).astype(np.float32), leaves=False)


def _mixed(stumps, outputs, features, depth):
    """Stumps and a few deep trees."""
    a = _full_forest(5, stumps, 1, features, n_outputs=outputs)
    b = wl.random_forest(7, n_trees=outputs, n_features=features, max_depth=depth, stop_prob=0.05, n_outputs=outputs)
    cat = {k: np.concatenate([getattr(a, k), getattr(b, k)]) for k in ("feature", "threshold", "left", "right", "leaf_value", "tree_output")}
    cat["tree_output"][:] = np.arange(stumps + outputs) % outputs
    return wl.Forest(**{**a.__dict__, **cat, "tree_offset": np.concatenate([a.tree_offset, a.tree_offset[-1] + b.tree_offset[1:]])})


def _vector_full(trees, depth, features, outputs):
    arrs = wl._full_forest(np.random.default_rng(depth), trees, depth, features, wl._normal_thr,
                           lambda r, s: r.standard_normal((s[0], s[1] * outputs), dtype=np.float32), leaf_width=outputs)
    return wl.Forest(n_features=features, n_outputs=outputs, leaf_width=outputs, tree_output=np.zeros(trees, np.int32),
                     aggregate=wl.AGG_MEAN, **arrs)


def test_shallow_trees_over_few_features_stay_with_the_dense_kernels():
    """The models that the walk kernels run slower than the dense ones did (by 1.3 to 3.4 at these sizes), and the ones
    they were written for."""
    from paper_2301_13441_amd import binding
    kernel = lambda f, rows, **kw: binding.forest_packed_launch(f, rows, **kw)["kernel"]
    infinite = _full_forest(1, 1000, 2, 10)
    infinite.threshold[0] = np.inf
    for f in (_vector_full(10, 3, 10, 10), _vector_full(100, 3, 10, 3), _full_forest(2, 10, 3, 10), infinite):
        assert kernel(f, 1_000_000) == kernel(f, 100_000) == "rank"
        # leaf ids: only with fewer trees than waves, and only where the deep walk kernel has the model
        few = f.n_trees < 16 and f.leaf_width > 1
        assert kernel(f, 1_000_000, leaves=True) == ("rank" if few else "walk" if f.n_trees == 10 else "deep")
        assert kernel(f, 100) in ("point", "deep")
        assert kernel(f, 1_000_000, form="walk") in ("walk", "deep")
    assert kernel(infinite, 20_000) == kernel(infinite, 5_000) == "rank" and kernel(infinite, 4_000) == "deep"
    few = wl.random_forest(312, n_trees=10, n_features=10, max_depth=3, stop_prob=0.15, n_outputs=12, leaf_width=12)
    assert kernel(few, 1_000_000) == "rank_lds" and kernel(few, 1_000) == "deep"
    assert kernel(_mixed(1000, 5, 10, 8), 1_000_000) == "rank_lds"
    for name, rows, want in (("c2", 1_000_000, "walk"), ("c3", 1_000_000, "walk"), ("c4", 500_000, "walk"), ("c5", 4_000_000, "deep")):
        f = wl.make_workload(name, n_rows=1).forest
        assert kernel(f, rows) == want and kernel(f, rows, form="dense").startswith("rank")


@pytest.mark.parametrize("what", ["walk", "deep", "vector"])
def test_padding_of_the_walk_programs_is_bounded(what):
    """Tens of thousands of stumps with one deep tree among them, and of stumps with vector leaves: the walk programs
    would be a hundred times the model."""
    import paper_2301_13441_amd as pk
    for trees, taken in ((1000, True), (40_000, False)):
        if what == "vector":
            f = _vector_full(trees, 1, 10, 3)
        else:
            f = _mixed(trees, 1, 10, 8 if what == "walk" else 9)
        v = pk.forest_pack(f)
        assert (v["walk_depth"] > 0 or v["deep_groups"] > 0) == taken
    full = pk.forest_pack(_full_forest(1, 20_000, 8, 10))                 # 82 MB, no padding in it
    assert full["walk_depth"] == 8


def test_leaf_ids_take_no_lds_for_sums():
    """Leaf ids of a model whose sums fill more than half a CU's LDS: two workgroups on a CU, counted as such."""
    from paper_2301_13441_amd import binding
    f = _vector_full(20, 4, 10, 16)                # 16 waves x 16 columns x 64 rows of sums: 128 KB
    lds = lambda leaves: binding.forest_packed_launch(f, 100_000, leaves, form="walk")["lds_bytes"]
    assert lds(False) > 128 << 10 and lds(True) <= 80 << 10


def test_row_groups_leave_every_cu_a_workgroup():
    """The most rows per workgroup of which there are 256 (of two groups and 100 trees: 128), and one group where trees
    are cut into shares.  Rounds of 512 workgroups, counted whole, chose one group for a batch of 66,000 or 150,000 rows."""
    from paper_2301_13441_amd import binding
    group = lambda f, rows: binding.forest_packed_launch(f, rows, form="walk")["rows_per_workgroup"] // 64
    few, many, deep = _full_forest(1, 10, 4, 10), _full_forest(1, 600, 8, 10), _vector_full(30, 4, 10, 2)
    for rows, want in ((9_000, 1), (16_257, 2), (33_000, 2), (65_280, 2), (65_281, 4), (66_000, 4), (150_000, 4), (10**6, 4)):
        less = want if rows != 16_257 else 1
        assert group(few, rows) == less and group(deep, rows) == min(less, 2)
        s = binding.forest_packed_launch(many, rows, form="walk")
        assert s["rows_per_workgroup"] == 64 * (want if s["shares"] == 1 else 1)


def test_a_row_of_many_tests_is_cut_into_shares():
    """One workgroup tests a row in the kernel with a lane per (row, tree): up to 12,000 tests, or trees of a line each."""
    from paper_2301_13441_amd import binding
    for trees, depth, kernel in ((2000, 6, "point"), (2001, 6, "walk"), (1500, 8, "point"), (1501, 8, "walk"), (2400, 5, "point"),
                                 (2401, 5, "walk"), (4000, 4, "point")):
        f = _full_forest(1, trees, depth, 10)
        s = binding.forest_packed_launch(f, 1)
        assert s["kernel"] == kernel and (s["shares"] > 1) == (kernel == "walk"), s
    # several columns make the reduction of the shares dearer, most against the fewest tests of a copy, or where they are many
    for trees, depth, outputs, rows, kernel in ((2800, 5, 3, 1, "point"), (2801, 5, 3, 1, "walk"), (2800, 5, 10, 40, "point"), (2001, 6, 10, 1, "walk"),
                                                (1750, 8, 20, 16, "point"), (1751, 8, 20, 16, "walk"), (1501, 8, 20, 17, "walk"), (1501, 8, 16, 1, "walk")):
        s = binding.forest_packed_launch(_full_forest(1, trees, depth, 10, n_outputs=outputs), rows)
        assert s["kernel"] == kernel, (trees, depth, outputs, rows)
    assert binding.forest_packed_launch(_full_forest(1, 2800, 5, 10, n_outputs=10), 1, leaves=True)["kernel"] == "walk"


def test_a_row_of_many_tests_without_a_workspace():
    """A call that finds every workspace taken cannot be cut into shares; one workgroup of the walk kernels would take all
    the trees.  Leaf ids need no workspace."""
    from paper_2301_13441_amd import binding
    for trees, depth, outputs in ((2001, 6, 1), (2001, 6, 10), (1501, 8, 1), (4000, 5, 1)):
        f = _full_forest(1, trees, depth, 10, n_outputs=outputs)
        for rows in (1, 40):
            plan = lambda **kw: binding.forest_packed_launch(f, rows, **kw)
            assert plan()["kernel"] == "walk" and plan()["shares"] > 1
            assert plan(workspace=False)["kernel"] == "point"
            assert plan(workspace=False, leaves=True) == plan(leaves=True)
    few = _full_forest(1, 100, 6, 10)
    assert binding.forest_packed_launch(few, 1, workspace=False)["kernel"] == "point"


@pytest.mark.gpu
@pytest.mark.parametrize("trees,depth,outputs", [(2001, 6, 10), (1501, 8, 1), (2803, 5, 32)])
def test_few_rows_of_many_tests(trees, depth, outputs):
    """The same through the reduction: shares of 1 to 40 rows, up to as many columns as a model may have; and 200 trees of
    the same shapes, which the kernel with a lane per (row, tree) takes and whose columns' first trees it counts."""
    from paper_2301_13441_amd import binding
    from test_gpu_parity import _check
    f = _full_forest(trees, trees, depth, 12, n_outputs=outputs, transform=wl.TRANSFORM_SOFTMAX if outputs > 1 else wl.TRANSFORM_SIGMOID)
    few = _full_forest(trees, 200, depth, 12, n_outputs=outputs, aggregate=wl.AGG_MEAN)
    X = np.random.default_rng(depth).standard_normal((40, 12)).astype(np.float32)
    for rows in (1, 3, 40):
        s = binding.forest_packed_launch(f, rows)
        assert s["kernel"] == "walk" and s["shares"] > 1 and binding.forest_packed_launch(few, rows)["kernel"] == "point"
        _check(f, X[:rows], leaves=True)
        _check(few, X[:rows], leaves=True)


@pytest.mark.gpu
def test_few_rows_of_many_tests_on_more_streams_than_workspaces():
    """Four streams have a workspace of the handle each, the others none; all of them get the same rows."""
    import torch
    import paper_2301_13441_amd as pk
    f = _full_forest(5, 2001, 6, 12, n_outputs=3)
    X = np.random.default_rng(6).standard_normal((3, 12)).astype(np.float32)
    ref = oracle.predict(f, X, want_leaves=True)
    model, xd = pk.forest_load(f), torch.from_numpy(X).cuda()
    streams, got = [torch.cuda.Stream() for _ in range(7)], []
    torch.cuda.synchronize()
    for s in streams:
        with torch.cuda.stream(s):
            got.append(model.predict(xd) + (model.predict_leaves(xd),))
    torch.cuda.synchronize()
    for scores, labels, leaves in got:
        np.testing.assert_array_equal(leaves.cpu().numpy(), ref.leaf_node_id)
        np.testing.assert_array_equal(labels.cpu().numpy(), ref.labels)
        np.testing.assert_allclose(scores.cpu().numpy(), ref.scores, rtol=2e-7, atol=1e-30)  # fp64 sums, one rounding apart
    model.close()


def _by_fours(f, rows):
    from paper_2301_13441_amd import binding
    return bool(binding.forest_packed_launch(f, rows, True, form="walk")["leaves_by_fours"])


def test_leaf_ids_of_few_trees_go_by_fours_where_workgroups_are_many():
    """Large batches of few trees over narrow rows, which the exchange of the ids made up to 1.5 times slower; sums never."""
    from paper_2301_13441_amd import binding
    walk = lambda trees, features, outputs=2: _full_forest(1, trees, 6, features, n_outputs=outputs)
    for trees, features, rows, want in ((1, 300, 9_000, True), (2, 300, 9_000, True), (5, 40, 16_000, False), (5, 40, 40_000, True), (5, 41, 700_000, False),
                                        (9, 40, 40_000, True), (8, 3, 40_000, False), (10, 40, 700_000, False), (12, 16, 70_000, False), (12, 16, 80_000, True), (12, 3, 700_000, False), (12, 33, 700_000, False),
                                        (16, 16, 350_000, False), (16, 16, 600_000, True), (17, 16, 10**6, False), (64, 16, 10**6, False)):
        assert _by_fours(walk(trees, features), rows) == want, (trees, features, rows)
    assert not _by_fours(walk(12, 16, 1), 10**6)  # 256 rows per workgroup
    assert _by_fours(walk(9, 16, 1), 10**6) and not _by_fours(_full_forest(1, 7, 7, 16), 10**6)
    for trees, features, outputs, rows, want in ((1, 200, 3, 9_000, True), (2, 64, 3, 30_000, False), (2, 64, 3, 40_000, True), (6, 3, 15, 130_000, True),
                                                 (20, 4, 15, 130_000, True), (20, 3, 15, 130_000, False), (20, 4, 15, 120_000, False), (21, 4, 15, 10**6, False),
                                                 (6, 32, 2, 200_000, True), (7, 32, 2, 10**6, False), (6, 33, 2, 10**6, False)):
        f = _vector_forest(outputs, features, trees)
        assert _by_fours(f, rows) == want, (trees, features, outputs, rows)
        assert binding.forest_packed_launch(f, rows, False, form="walk")["leaves_by_fours"] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("what,trees", [("walk", t) for t in (1, 2, 3, 5, 6, 7, 9, 10, 12, 13, 16, 17)] + [("deep", t) for t in (1, 2, 3, 5, 6, 7, 19, 20, 21)])
def test_leaf_ids_of_few_trees(what, trees):
    """Both sides of the rule, waves with one to four trees and with none, a ragged last workgroup."""
    import torch
    from paper_2301_13441_amd import binding
    rng = np.random.default_rng(trees)
    for depth in (3, 4, 5, 6, 7, 8) if what == "walk" else (9, 11):
        for outputs in (1, 2, 9):
            f = _full_forest(trees, trees, depth, 7, n_outputs=outputs) if what == "walk" else \
                wl.random_forest(trees, n_trees=trees, n_features=7, max_depth=depth, stop_prob=0.3, n_outputs=outputs, leaf_width=outputs, aggregate=wl.AGG_MEAN)
            model = binding.forest_load_form(f, "walk")
            for rows in (77, 40_001, 300_001):
                X = rng.standard_normal((rows, 7)).astype(np.float32)
                got = model.predict_leaves(torch.from_numpy(X).cuda()).cpu().numpy()
                np.testing.assert_array_equal(got, oracle.predict(f, X, want_leaves=True, n_threads=8).leaf_node_id)
            model.close()
