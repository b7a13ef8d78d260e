"""The walk kernels and their packed form: trees of depth up to 8 laid out as full trees, one node
per level and row.  Leaf ids and labels are exact; scores are fp64 sums rounded once on both sides,
at most one float32 rounding (6e-8) apart, well inside the bar used here."""
import numpy as np
import pytest

import oracle
import workloads as wl
from test_gpu_parity import _check, _full_forest


def _forest(seed, trees, depth, features, outputs=1, full=True):
    if full:
        return _full_forest(seed, trees, depth, features, n_outputs=outputs,
                            transform=wl.TRANSFORM_SOFTMAX if outputs > 1 else wl.TRANSFORM_SIGMOID)
    f = wl.random_forest(seed, n_trees=trees, n_features=features, max_depth=depth, stop_prob=0.2, n_outputs=outputs)
    return wl.Forest(**{**f.__dict__, "tree_output": (np.arange(trees) % outputs).astype(np.int32)})


def _special_rows(X, f, rng):
    """Rows on thresholds, signed zeros, NaN and infinities."""
    thr = f.threshold[f.feature >= 0]
    if thr.size:
        X[:40] = rng.choice(thr, (40, X.shape[1]))
    X[40:50] = np.float32(0.0)
    X[50:60] = np.float32(-0.0)
    X[60:70] = rng.choice(np.float32([np.nan, np.inf, -np.inf, 1e-45, -1e-45]), (10, X.shape[1]))
    return X


@pytest.mark.parametrize("depth,full", [(1, True), (3, True), (4, False), (6, True), (7, False), (8, True), (8, False)])
def test_walk_layout_reaches_the_oracles_leaves(depth, full):
    import paper_2301_13441_amd as pk
    rng = np.random.default_rng(depth)
    f = _forest(60 + depth, 11, depth, 5, outputs=3, full=full)
    f.threshold[np.flatnonzero(f.feature >= 0)[::5]] = np.float32(-0.0)
    v = pk.forest_pack(f)
    D, T = v["walk_depth"], f.n_trees
    assert D == max(3, int(v["tree_depth"].max())) and v["walk_trees"] >= T
    X = _special_rows(rng.standard_normal((100, 5)).astype(np.float32), f, rng)
    ref = oracle.predict(f, X, want_leaves=True).leaf_node_id
    x = np.where(np.isnan(X), np.float32(np.inf), X)
    seen = set()
    for i in range(T):
        thr = v["walk_node"][i, :, 0].view(np.float32)
        feat = v["walk_node"][i, :, 1] // (256 * v["walk_groups"])
        caller = int(v["walk_node"][i, 0, 1])
        assert int(v["walk_node"][i, 0, 0]) == f.tree_output[caller]
        seen.add(caller)
        at = np.zeros(len(X), np.int64)
        for l in range(D):
            h = (1 << l) + at
            with np.errstate(invalid="ignore"):
                right = np.signbit(thr[h] - x[np.arange(len(X)), feat[h]])     # the sign the kernel takes
            at |= right.astype(np.int64) << l
        np.testing.assert_array_equal(v["walk_leaf_node"][i, at], ref[:, caller])
        values = f.leaf_value[f.tree_offset[caller] + v["walk_leaf_node"][i, at], 0]
        np.testing.assert_array_equal(v["walk_leaf"][i, at], values)
    assert seen == set(range(T))
    assert (v["walk_leaf"][T:] == 0).all()


def test_walk_takes_what_it_is_built_for():
    import paper_2301_13441_amd as pk
    assert pk.forest_pack(_forest(1, 20, 8, 28))["walk_groups"] == 4
    assert pk.forest_pack(_forest(1, 20, 6, 128, outputs=10))["walk_groups"] == 2
    assert pk.forest_pack(_forest(1, 20, 6, 500))["walk_groups"] == 1
    assert pk.forest_pack(_forest(1, 20, 6, 700))["walk_depth"] == 0                    # X tile beyond the LDS
    assert pk.forest_pack(wl.random_forest(3, 9, 5, 9, stop_prob=0.0))["walk_depth"] == 0  # depth 9
    f = _forest(1, 20, 6, 9)
    f.threshold[np.flatnonzero(f.feature >= 0)[3]] = np.inf
    assert pk.forest_pack(f)["walk_depth"] == 0                                         # infinite threshold
    f = _forest(1, 100, 6, 9, outputs=8)
    assert pk.forest_pack(f)["walk_depth"] == 6
    f.tree_output[:] = np.sort(np.concatenate([np.arange(7), np.full(93, 7)])).astype(np.int32)
    assert pk.forest_pack(f)["walk_depth"] == 0                                         # 7 columns in one wave's run


def _launches(f, rows, kernel, rows_per_workgroup):
    """What a test is about: the walk kernels with this many rows per workgroup, for sums and for leaf ids."""
    from paper_2301_13441_amd import binding
    for leaves in (False, True):
        s = binding.forest_packed_launch(f, rows, leaves, form="walk")
        assert s["kernel"] == kernel and s["rows_per_workgroup"] == rows_per_workgroup and s["shares"] == 1, s


@pytest.mark.gpu
@pytest.mark.parametrize("rows,groups", [(12301, 1), (49152 - 13, 2), (131072 - 13, 4)])
@pytest.mark.parametrize("depth", [3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("features,outputs,full", [(3, 1, True), (40, 1, False), (9, 4, False), (90, 4, True)])
def test_walk_kernels_by_rows_per_lane(depth, features, outputs, full, rows, groups):
    """One, two and four row groups per workgroup with a ragged last one; few trees (waves without any) and more trees
    than waves, in numbers that are no multiple of four."""
    rng = np.random.default_rng(100 * depth + features)
    for trees in (5, 53):
        f = _forest(9 * depth + features, trees, depth, features, outputs, full)
        _launches(f, rows, "walk", 64 * min(groups, 4 if outputs == 1 else 2))
        _check(f, _special_rows(rng.standard_normal((rows, features)).astype(np.float32), f, rng), leaves=True)


@pytest.mark.gpu
@pytest.mark.parametrize("depth", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("features,outputs,full", [(3, 1, True), (40, 4, False), (61, 1, False), (130, 4, True), (300, 1, True)])
def test_walk_kernels(depth, features, outputs, full):
    """Every depth; tiles of 4, 2 and 1 row groups; one and several columns; few trees over few rows (a lane per row and
    tree) and more trees than waves; leaf ids of a tree count that is no multiple of four."""
    import paper_2301_13441_amd as pk
    rng = np.random.default_rng(100 * depth + features)
    for trees, rows in ((5, 517), (83, 65536 + 77)):
        f = _forest(9 * depth + features, trees, depth, features, outputs, full)
        assert pk.forest_pack(f)["walk_depth"] > 0
        if rows > 60000:
            _launches(f, rows, "walk", 64 * pk.forest_pack(f)["walk_groups"])
        X = _special_rows(rng.standard_normal((rows, features)).astype(np.float32), f, rng)
        _check(f, X, leaves=True)


@pytest.mark.gpu
@pytest.mark.parametrize("depth,trees,features,outputs", [(3, 1, 2, 1), (8, 500, 28, 1), (6, 2000, 128, 10), (7, 65, 300, 4), (4, 10, 9, 3),
                                                          (5, 10, 10, 5), (3, 5, 4, 32), (4, 40, 7, 31), (5, 300, 4, 32), (8, 104, 7, 31),
                                                          (6, 30, 5, 2), (6, 60, 5, 7)])
def test_smallest_batches_with_a_lane_per_row_and_tree(depth, trees, features, outputs):
    """One row, whole and ragged workgroups of rows, more pairs than threads, and the first batches beyond
    the kernel's limit on rows and on tests; one column up to as many as a model may have, whose first trees it counts.
    (More than four columns in a wave's run of trees: the deep walk kernel's.)"""
    from paper_2301_13441_amd import binding
    rng = np.random.default_rng(depth + trees)
    f = _forest(trees + depth, trees, depth, features, outputs, full=True)
    limit = min(8192, (1 << 20) // (trees * depth))
    for rows in sorted({1, 2, 15, 17, 70, limit, limit + 1}):
        assert binding.forest_packed_launch(f, rows)["kernel"] == ("deep" if trees < outputs * 2 and outputs > 30 else "point" if rows <= limit else "walk")
        X = rng.standard_normal((rows, features)).astype(np.float32)
        if rows >= 70:
            X = _special_rows(X, f, rng)
        _check(f, X, leaves=rows <= 70)


@pytest.mark.gpu
@pytest.mark.parametrize("features", [1, 2, 3, 4, 5, 15, 17, 35])
def test_tiles_of_rows_that_end_inside_a_piece(features):
    """Rows of fewer features than a lane loads at once, of just as many, and of one or three beyond a piece; a last
    workgroup of one row; both walk kernels, which fill their tiles with the same code."""
    rng = np.random.default_rng(features)
    scalar = _forest(features, 9, 6, features)
    vector = wl.random_forest(features, n_trees=9, n_features=features, max_depth=9, stop_prob=0.2, n_outputs=2, leaf_width=2,
                              aggregate=wl.AGG_MEAN)
    for f in (scalar, vector):
        for rows in (16385, 20011):
            _check(f, _special_rows(rng.standard_normal((rows, features)).astype(np.float32), f, rng), leaves=True)


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [9001, 49157, 131075])
@pytest.mark.parametrize("depth,trees", [(3, 1), (3, 4), (3, 5), (3, 65), (4, 63), (5, 16), (6, 33), (6, 64), (6, 130), (7, 49), (8, 17), (8, 129)])
def test_leaf_ids_by_rounds_of_trees(depth, trees, rows):
    """One, two and four row groups per workgroup (with shares of the trees at 9,001 rows); tree counts below, at and
    beyond a round of four trees for each of 16 waves, and rests of one to four trees per wave."""
    import torch
    from paper_2301_13441_amd import binding
    rng = np.random.default_rng(depth + trees)
    f = _forest(depth + trees, trees, depth, 7, full=depth != 7)
    s = binding.forest_packed_launch(f, rows, True, form="walk")
    assert s["kernel"] == "walk" and s["rows_per_workgroup"] == {9001: 64, 49157: 128, 131075: 256}[rows], s
    assert s["shares"] == (2 if rows == 9001 and trees >= 128 else 1), s
    X = _special_rows(rng.standard_normal((rows, 7)).astype(np.float32), f, rng)
    model = binding.forest_load_form(f, "walk")
    try:
        got = model.predict_leaves(torch.from_numpy(X).cuda()).cpu().numpy()
    finally:
        model.close()
    np.testing.assert_array_equal(got, oracle.predict(f, X, want_leaves=True, n_threads=8).leaf_node_id)


@pytest.mark.gpu
@pytest.mark.parametrize("depth", [3, 6, 8, 9])
@pytest.mark.parametrize("trees,rows", [(41, 9001), (300, 9001), (1000, 9001), (41, 70_001)])
def test_columns_without_trees_between_columns_with_some(depth, trees, rows):
    """A wave's run of trees that goes from one column to one further on leaves zeros for those between; odd tree
    counts, which end a pair of trees walked together; with and without shares of the trees."""
    from paper_2301_13441_amd import binding
    rng = np.random.default_rng(depth + trees)
    f = _forest(trees + depth, trees, min(depth, 8), 9, outputs=7) if depth < 9 else \
        wl.random_forest(trees, n_trees=trees, n_features=9, max_depth=9, stop_prob=0.3, n_outputs=7, aggregate=wl.AGG_SUM)
    f = wl.Forest(**{**f.__dict__, "tree_output": rng.choice([0, 3, 6], trees).astype(np.int32)})
    s = binding.forest_packed_launch(f, rows, form="walk")
    assert s["kernel"] == ("walk" if depth < 9 else "deep") and s["rows_per_workgroup"] == (64 if rows == 9001 else 128), s
    assert s["shares"] == (1 if trees == 41 or (trees, depth) == (300, 3) else 3), s
    _check(f, _special_rows(rng.standard_normal((rows, 9)).astype(np.float32), f, rng))


@pytest.mark.gpu
@pytest.mark.parametrize("what,rows,groups,last", [
    ("one", 65536 + 61 * 256 + 3, 4, 1), ("one", 65536 + 64 * 256, 4, 1), ("one", 65536 + 64 * 256 + 1, 4, 2),
    ("one", 65536 + 128 * 256 - 255, 4, 2), ("one", 65536 + 128 * 256 + 1, 4, 4), ("depth8", 65536 + 9 * 256 + 65, 4, 1),
    ("depth8", 65536 + 70 * 256 + 129, 4, 2), ("columns", 32768 + 50 * 128 + 1, 2, 1), ("columns", 32768 + 128 * 128 + 1, 2, 2),
    ("deep", 32768 + 7, 2, 1), ("deep", 3 * 32768 + 127 * 128 + 65, 2, 1), ("deep_alone", 32768 + 3 * 128 + 70, 2, 1),
    ("deep_alone", 21 * 32768 + 3 * 128, 2, 2), ("vector", 32768 + 40 * 128 + 64, 2, 1)])
def test_launches_that_end_in_smaller_workgroups(what, rows, groups, last):
    """The rest of a division by the CUs in workgroups of fewer rows: both smaller sizes, the first and last rests that
    take them, ragged ends, and leaf ids, which have the same rows per workgroup."""
    import torch
    from paper_2301_13441_amd import binding
    rng = np.random.default_rng(rows)
    f = {"one": lambda: _forest(5, 18, 5, 9), "depth8": lambda: _forest(6, 18, 8, 7), "columns": lambda: _forest(7, 31, 6, 9, outputs=4),
         "deep": lambda: wl.random_forest(8, n_trees=40, n_features=9, max_depth=10, stop_prob=0.25, aggregate=wl.AGG_SUM),
         "deep_alone": lambda: wl.random_forest(9, n_trees=33, n_features=200, max_depth=9, stop_prob=0.25, aggregate=wl.AGG_SUM),
         "vector": lambda: wl.random_forest(10, n_trees=35, n_features=9, max_depth=9, stop_prob=0.25, n_outputs=2, leaf_width=2,
                                            aggregate=wl.AGG_MEAN)}[what]()
    model = binding.forest_load_form(f, "walk")
    try:
        for leaves in (False, True):
            s = binding.forest_packed_launch(f, rows, leaves, form="walk")
            assert (s["rows_per_workgroup"], s["last_rows_per_workgroup"]) == (64 * groups, 64 * last) and s["shares"] == 1, s
        X = _special_rows(rng.standard_normal((rows, f.n_features)).astype(np.float32), f, rng)
        # the whole workgroups' last rows and everything after them, and the first rows
        pick = np.unique(np.concatenate([np.arange(300), np.arange(max(0, rows - 256 * 200), rows)]))
        ref = oracle.predict(f, X[pick], want_leaves=True, n_threads=8)
        xd, at = torch.from_numpy(X).cuda(), torch.from_numpy(pick).cuda()
        scores, labels = model.predict(xd)
        np.testing.assert_allclose(scores[at].cpu().numpy(), ref.scores, rtol=1e-5, atol=1e-6)
        np.testing.assert_array_equal(labels[at].cpu().numpy(), ref.labels)
        np.testing.assert_array_equal(model.predict_leaves(xd)[at].cpu().numpy(), ref.leaf_node_id)
    finally:
        model.close()


def test_only_whole_aligned_pieces_of_ids_go_past_the_l2():
    from paper_2301_13441_amd import binding
    for at in (1 << 20, (1 << 20) + 16, (1 << 20) + 4, (1 << 20) + 8, (1 << 20) + 12):
        for trees in (4, 8, 16, 17, 20, 32, 48, 50, 52, 64, 101, 128, 200, 1 << 20, (1 << 20) + 4):
            whole = trees % 4 == 0 and at % 16 == 0 and trees <= 1 << 20
            assert binding.forest_ids_go_through(trees, 1, at) == (whole and not 16 < trees <= 48), (trees, at)
    for bad in ((0, 1), (1, 0)):
        with pytest.raises(binding.ForestError):
            binding.forest_ids_go_through(*bad, 1 << 20)


@pytest.mark.parametrize("trees", [52, 64, 68, 84, 96, 100, 128, 132, 200, 300, 400])
def test_many_ids_go_past_the_l2_only_where_a_rows_runs_are_whole_pieces(trees):
    """Of more than 64 trees a row's ids leave in runs of 256 bytes: only of a multiple of 16 trees do they begin 64-byte pieces."""
    from paper_2301_13441_amd import binding
    few = (1 << 23) // trees
    for rows in (1, few, few + 1, 10**6):
        for at in (1 << 20, (1 << 20) + 16):
            through = trees <= 64 or rows <= few or (trees % 16 == 0 and at % 64 == 0)
            assert binding.forest_ids_go_through(trees, rows, at) == through, (rows, at)


@pytest.mark.gpu
@pytest.mark.parametrize("depth,trees,rows", [(6, 8, 9001), (6, 20, 5003), (6, 64, 9001), (7, 68, 40_001), (5, 101, 9001), (6, 128, 70_003),
                                              (9, 12, 9001), (9, 64, 5003), (10, 100, 9001), (9, 128, 40_001)])
def test_leaf_ids_to_any_address(depth, trees, rows):
    """The caller's buffer may begin at any id; nothing before or behind it is touched."""
    import torch
    from paper_2301_13441_amd import binding
    rng = np.random.default_rng(depth * trees)
    f = _forest(depth + trees, trees, depth, 9) if depth < 9 else \
        wl.random_forest(depth + trees, n_trees=trees, n_features=9, max_depth=depth, stop_prob=0.3, aggregate=wl.AGG_SUM)
    X = rng.standard_normal((rows, 9)).astype(np.float32)
    want = oracle.predict(f, X, want_leaves=True, n_threads=8).leaf_node_id
    model = binding.forest_load_form(f, "walk")
    try:
        xd = torch.from_numpy(X).cuda()
        for off in (0, 1, 2, 3, 4):
            buf = torch.full((rows * trees + 64,), -7, dtype=torch.int32, device="cuda")
            out = buf[16 + off:16 + off + rows * trees]
            assert out.data_ptr() % 16 == 4 * (off % 4)
            rc = model._lib.forest_predict_leaves(model._h, binding._p(xd.data_ptr()), rows, binding._p(out.data_ptr()),
                                                  binding._p(torch.cuda.current_stream().cuda_stream))
            assert rc == 0
            np.testing.assert_array_equal(out.view(rows, trees).cpu().numpy(), want)
            assert (buf[:16 + off] == -7).all() and (buf[16 + off + rows * trees:] == -7).all()
    finally:
        model.close()


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [9001, 40_001, 70_003])
@pytest.mark.parametrize("depth,trees", [(4, 12), (6, 20), (6, 68), (3, 76), (8, 96), (5, 128), (7, 204), (9, 12), (10, 36), (9, 68), (10, 128), (9, 133)])
def test_leaf_ids_past_the_l2(depth, trees, rows):
    """Tree counts that are multiples of four, whose ids go past the L2 by fours and by ones, and are kept there by twos and
    threes; one that is not; both walk kernels, with shares and without, whole workgroups and smaller ones at the end."""
    import torch
    from paper_2301_13441_amd import binding
    rng = np.random.default_rng(depth * trees)
    f = _forest(depth + trees, trees, depth, 9) if depth < 9 else \
        wl.random_forest(depth + trees, n_trees=trees, n_features=9, max_depth=depth, stop_prob=0.3, aggregate=wl.AGG_SUM)
    X = rng.standard_normal((rows, 9)).astype(np.float32)
    model = binding.forest_load_form(f, "walk")
    try:
        got = model.predict_leaves(torch.from_numpy(X).cuda()).cpu().numpy()
    finally:
        model.close()
    np.testing.assert_array_equal(got, oracle.predict(f, X, want_leaves=True, n_threads=8).leaf_node_id)


def test_lines_of_x_stay_in_the_l2_where_rows_share_them_and_the_trees_keep_their_place():
    from paper_2301_13441_amd import binding
    few, many = _forest(1, 40, 6, 16), _forest(2, 500, 8, 16)  # 30 KB and 1.5 MB of tables
    at = lambda f, features: wl.Forest(**{**f.__dict__, "n_features": features})
    for features in (32, 64, 96, 224):  # whole lines are asked for once
        assert not binding.forest_keeps_lines(at(few, features), 10**6)
        assert all(binding.forest_keeps_lines(at(few, features), 10**6, x=x) for x in (4, 64))
    for features, rows, keep_few, keep_many in ((16, 10**6, 0, 0), (17, 10**6, 1, 1), (127, 10**6, 1, 1), (200, 10**6, 1, 0), (300, 10**6, 1, 0),
                                                (500, 10**6, 1, 0), (300, 5000, 1, 1)):  # the last: shares of the trees read a tile several times
        assert binding.forest_keeps_lines(at(few, features), rows) == keep_few, (features, rows)
        assert binding.forest_keeps_lines(at(many, features), rows) == keep_many, (features, rows)
    assert not binding.forest_keeps_lines(few, 1, x=4)  # a lane per (row, tree)
    some = _forest(3, 500, 7, 16)  # 0.8 MB: too many where a CU has one row group
    assert [binding.forest_keeps_lines(at(some, features), 10**6) for features in (100, 129, 200, 300)] == [1, 1, 1, 0]
    assert binding.forest_keeps_lines(_forest(4, 33, 7, 285), 10**6)  # few trees beside 4.5 MB of X
    for bad in (0, 1 << 62):
        with pytest.raises(binding.ForestError):
            binding.forest_keeps_lines(few, bad)


@pytest.mark.gpu
@pytest.mark.parametrize("kind,trees,depth,features,rows,shift,keep", [
    ("walk", 500, 8, 201, 33_333, 0, 0), ("walk", 1600, 8, 31, 33_333, 0, 0), ("walk", 1600, 8, 31, 9_001, 0, 1), ("walk", 500, 8, 301, 33_333, 0, 0), ("walk", 40, 6, 64, 70_003, 1, 1), ("walk", 40, 6, 128, 33_333, 16, 1),
    ("walk", 500, 8, 256, 33_333, 3, 0), ("deep", 200, 12, 131, 3 * 32_768, 0, 0), ("deep", 200, 12, 225, 65_536 + 1, 0, 0),
    ("deep", 20, 9, 160, 3 * 32_768 - 3, 1, 1), ("deep", 200, 12, 95, 40_009, 0, 0)])
def test_tiles_by_how_x_is_loaded(kind, trees, depth, features, rows, shift, keep):
    """Rows that share lines, by their width or by X's address, loaded either way; tile after tile too."""
    import torch
    from paper_2301_13441_amd import binding
    rng = np.random.default_rng(features)
    f = _forest(features, trees, depth, features) if kind == "walk" else wl.random_forest(features, n_trees=trees, n_features=features, max_depth=depth, stop_prob=0.05 if trees > 20 else 0.25, aggregate=wl.AGG_SUM)
    X = _special_rows(rng.standard_normal((rows, features)).astype(np.float32), f, rng)
    flat = torch.zeros(X.size + 32, dtype=torch.float32, device="cuda")
    xd = flat[shift:shift + X.size].view(rows, features)
    xd.copy_(torch.from_numpy(X))
    assert xd.data_ptr() % 128 == 4 * shift
    s = binding.forest_packed_launch(f, rows)
    assert s["kernel"] == kind and s["tile_after_tile"] == (kind == "deep" and features > 96) and binding.forest_keeps_lines(f, rows, x=xd.data_ptr()) == keep
    model = binding.forest_load(f)
    try:
        scores, _ = model.predict(xd)
        np.testing.assert_allclose(scores.cpu().numpy(), oracle.predict(f, X, n_threads=8).scores, rtol=1e-5, atol=1e-6)
    finally:
        model.close()


@pytest.mark.gpu
@pytest.mark.parametrize("features", [16, 17, 31, 32, 33])
@pytest.mark.parametrize("outputs", [1, 2])
def test_narrow_tiles_of_few_trees(features, outputs):
    """Leaf ids by fours, whose narrow rows are loaded another way than those of more trees; four row groups and two."""
    import torch
    from paper_2301_13441_amd import binding
    rows = 70_003
    rng = np.random.default_rng(features)
    f = _forest(features, 7, 6, features, outputs)
    s = binding.forest_packed_launch(f, rows, True, form="walk")
    assert s["kernel"] == "walk" and s["leaves_by_fours"] == 1 and s["rows_per_workgroup"] == (256 if outputs == 1 else 128), s
    X = _special_rows(rng.standard_normal((rows, features)).astype(np.float32), f, rng)
    model = binding.forest_load_form(f, "walk")
    try:
        got = model.predict_leaves(torch.from_numpy(X).cuda()).cpu().numpy()
    finally:
        model.close()
    np.testing.assert_array_equal(got, oracle.predict(f, X, want_leaves=True, n_threads=8).leaf_node_id)


@pytest.mark.gpu
@pytest.mark.parametrize("features", [3, 4, 5, 15, 16, 17, 30, 31, 32, 33, 47, 61, 64])
@pytest.mark.parametrize("rows,groups", [(12_301, 1), (33_333, 2), (70_003, 4)])
def test_tiles_of_every_width(features, rows, groups):
    """Rows that are no multiple of a line or of a load's features, fewer features than a load takes and one more, a ragged
    last workgroup; walk kernels and the deep one, every size of workgroup."""
    import torch
    from paper_2301_13441_amd import binding
    rng = np.random.default_rng(features)
    for f in (_forest(features, 40, 6, features), wl.random_forest(features, n_trees=40, n_features=features, max_depth=9, stop_prob=0.25, aggregate=wl.AGG_SUM)):
        s = binding.forest_packed_launch(f, rows, True, form="walk")
        assert s["rows_per_workgroup"] == 64 * (groups if s["kernel"] == "walk" else min(groups, 2)) and s["shares"] == 1, s
        X = _special_rows(rng.standard_normal((rows, features)).astype(np.float32), f, rng)
        ref = oracle.predict(f, X, want_leaves=True, n_threads=8)
        model = binding.forest_load_form(f, "walk")
        try:
            xd = torch.from_numpy(X).cuda()
            np.testing.assert_array_equal(model.predict_leaves(xd).cpu().numpy(), ref.leaf_node_id)
            scores, _ = model.predict(xd)
            np.testing.assert_allclose(scores.cpu().numpy(), ref.scores, rtol=1e-5, atol=1e-6)
        finally:
            model.close()
