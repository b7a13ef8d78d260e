"""The deep walk kernels and their packed form: trees of any shape and depth, the top levels laid out
as a full tree and the rest as units.  Leaf ids and labels are exact; scores are fp64 sums rounded once
on both sides, at most one float32 rounding (6e-8) apart, well inside the bar used here."""
import numpy as np
import pytest

import oracle
import workloads as wl
from test_gpu_parity import _check
from test_walk import _launches, _special_rows


def _forest(seed, trees, depth, features, outputs=1, width=1, stop=0.2):
    f = wl.random_forest(seed, n_trees=trees, n_features=features, max_depth=depth, stop_prob=stop, n_outputs=outputs,
                         leaf_width=width, transform=wl.TRANSFORM_SOFTMAX if outputs > 1 else wl.TRANSFORM_SIGMOID)
    if width == 1:
        f = wl.Forest(**{**f.__dict__, "tree_output": (np.arange(trees) % outputs).astype(np.int32)})
    inner = np.flatnonzero(f.feature >= 0)
    f.threshold[inner[::7]] = np.float32(-0.0)
    f.threshold[inner[3::29]] = np.float32(np.inf)
    f.threshold[inner[5::31]] = np.float32(-np.inf)
    return f


@pytest.mark.parametrize("depth,outputs,width", [(9, 1, 1), (12, 3, 1), (13, 2, 2), (10, 5, 5), (3, 2, 2), (0, 3, 3)])
def test_deep_layout_reaches_the_oracles_leaves(depth, outputs, width):
    import paper_2301_13441_amd as pk
    rng = np.random.default_rng(depth)
    f = _forest(70 + depth, 9, depth, 6, outputs, width)
    v = pk.forest_pack(f)
    T = f.n_trees
    assert v["deep_groups"] > 0
    X = _special_rows(rng.standard_normal((120, 6)).astype(np.float32), f, rng)
    ref = oracle.predict(f, X, want_leaves=True).leaf_node_id
    lane = np.arange(len(X))
    units = v["deep_unit"]
    assert sorted(v["deep_position"]) == list(range(T))
    for caller in range(T):
        i = int(v["deep_position"][caller])
        base, column = (int(a) for a in v["deep_top"][i, 0])
        assert column == (f.tree_output[caller] if width == 1 else 0)
        thr, feat = v["deep_top"][i, :, 0].copy().view(np.float32), v["deep_top"][i, :, 1] // 256
        at = np.zeros(len(X), np.int64)
        for l in range(7):
            h = (1 << l) + at
            at |= (~(X[lane, feat[h]] <= thr[h])).astype(np.int64) << l
        np.testing.assert_array_equal(v["deep_top"][i, 128:], units[base:base + 128])
        at = base + at
        for _ in range(max(0, depth - 7)):
            w = units[at, 1]
            node = np.isnan(w.copy().view(np.float32))
            right = ~(X[lane, np.where(node, (w >> 14) & 511, 0)] <= units[at, 0].copy().view(np.float32))
            at = np.where(node, at + (w & 0x3fff) + right, at)
        assert not np.isnan(units[at, 1].copy().view(np.float32)).any()
        np.testing.assert_array_equal(v["deep_unit_node"][at], ref[:, caller])
        value = f.leaf_value[f.tree_offset[caller] + ref[:, caller]]
        if width <= 2:
            got = units[at, :width].copy().view(np.float32)
        else:
            got = v["deep_value"][units[at, 0], :width]
        np.testing.assert_array_equal(got, value)


def test_deep_takes_what_it_is_built_for():
    import paper_2301_13441_amd as pk
    assert pk.forest_pack(_forest(1, 20, 9, 96))["deep_groups"] == 2                    # two workgroups on a CU
    assert pk.forest_pack(_forest(1, 20, 9, 192))["deep_groups"] == 1                   # two workgroups on a CU
    assert pk.forest_pack(_forest(1, 20, 9, 256))["deep_groups"] == 2                   # one
    assert pk.forest_pack(_forest(1, 20, 9, 500))["deep_groups"] == 1
    assert pk.forest_pack(_forest(1, 20, 9, 513))["deep_groups"] == 0                   # 9 bits of feature
    assert pk.forest_pack(_forest(1, 20, 9, 9, 16, 16))["deep_groups"] == 1
    assert pk.forest_pack(_forest(1, 20, 9, 9, 17, 17))["deep_groups"] == 0
    f = wl.random_forest(3, 9, 5, 8, stop_prob=0.0)
    assert pk.forest_pack(f)["deep_groups"] == 0 and pk.forest_pack(f)["walk_depth"] == 8
    f = _forest(1, 20, 9, 9, 2, 2)
    f.leaf_value[np.flatnonzero(f.feature < 0)[0], 1] = np.nan                          # would read as a node
    assert pk.forest_pack(f)["deep_groups"] == 0
    f = _forest(1, 100, 9, 9, 8)
    f.tree_output[:] = np.sort(np.concatenate([np.arange(7), np.full(93, 7)])).astype(np.int32)
    assert pk.forest_pack(f)["deep_groups"] == 0                                        # 7 columns in one wave's run


@pytest.mark.gpu
@pytest.mark.parametrize("features", [3, 16, 61, 130, 256, 300])
@pytest.mark.parametrize("depth,outputs,width", [(9, 1, 1), (11, 4, 1), (12, 2, 2), (10, 3, 3), (9, 8, 8), (5, 10, 10)])
def test_deep_kernels(features, depth, outputs, width):
    """One and two row groups; every kind of sum; few trees (waves without any) and more trees than
    waves; leaf ids of a tree count that is no multiple of four."""
    import paper_2301_13441_amd as pk
    rng = np.random.default_rng(100 * depth + features)
    for trees, rows in ((5, 517), (37, 65536 + 77)):
        f = _forest(9 * depth + features, trees, depth, features, outputs, width, stop=0.3)
        assert pk.forest_pack(f)["deep_groups"] > 0
        X = _special_rows(rng.standard_normal((rows, features)).astype(np.float32), f, rng)
        _check(f, X, leaves=True)


@pytest.mark.gpu
@pytest.mark.parametrize("features", [3, 90, 256])
@pytest.mark.parametrize("depth,outputs,width", [(9, 1, 1), (11, 4, 1), (12, 2, 2)])
@pytest.mark.parametrize("rows,groups", [(12301, 1), (65536 - 13, 2)])
def test_deep_kernels_by_rows_per_lane(features, depth, outputs, width, rows, groups):
    """One and two row groups with a ragged last workgroup, two workgroups on a CU and one; one column, several, and
    vector leaves; trees in numbers that are no multiple of four or two."""
    rng = np.random.default_rng(100 * depth + features)
    for trees in (5, 29):
        f = _forest(9 * depth + features, trees, depth, features, outputs, width, stop=0.3)
        _launches(f, rows, "deep", 64 * groups)
        _check(f, _special_rows(rng.standard_normal((rows, features)).astype(np.float32), f, rng), leaves=True)


def _tiles(f, rows):
    """What a test is about: the kernel whose workgroups take tile after tile."""
    from paper_2301_13441_amd import binding
    for form in ("auto", "walk"):
        s = binding.forest_packed_launch(f, rows, form=form)
        assert s["kernel"] == "deep" and s["tile_after_tile"] == 1, s


def test_deep_sums_go_tile_after_tile_where_a_cu_holds_one_tile():
    from paper_2301_13441_amd import binding
    plan = lambda features, rows, outputs=1, width=1, leaves=False: binding.forest_packed_launch(_forest(1, 20, 9, features, outputs, width), rows, leaves, form="walk")
    for features, rows, outputs, width, leaves, want in (
            (96, 10**6, 1, 1, False, 0), (97, 65535, 1, 1, False, 0), (97, 65536, 1, 1, False, 1), (256, 65536, 2, 2, False, 1), (257, 10**6, 1, 1, False, 0),
            (192, 10**6, 2, 1, False, 0), (192, 10**6, 3, 3, False, 0), (192, 10**6, 1, 1, True, 0)):
        s = plan(features, rows, outputs, width, leaves)
        assert s["kernel"] == "deep" and s["tile_after_tile"] == want, (features, rows, outputs, width, leaves)
        if want:
            assert s["rows_per_workgroup"] == s["last_rows_per_workgroup"] == 128 and s["workgroups"] == -(-rows // 128)


@pytest.mark.parametrize("features", [97, 192, 193, 256])
def test_rounds_and_few_tiles_more_are_left_to_smaller_workgroups(features):
    """Where these share a CU, up to 192 features, and the rounds are few."""
    from paper_2301_13441_amd import binding
    rounds = 256 * 128
    for trees, most in ((20, 2), (199, 2), (200, 6)):
        f = _forest(1, trees, 9, features)
        for n in (2, 3, 6, 7):
            spread = features <= 192 and n <= most
            for rows, want in ((n * rounds, 1), (n * rounds + 1, not spread), (n * rounds + 128 * 128, not spread), (n * rounds + 128 * 128 + 1, 1)):
                s = binding.forest_packed_launch(f, rows, form="walk")
                assert s["kernel"] == "deep" and s["tile_after_tile"] == want, (trees, rows)
                assert want or s["rows_per_workgroup"] == 64


@pytest.mark.parametrize("features,trees", [(97, 1), (97, 16), (192, 16), (192, 17), (193, 16)])
def test_waves_with_one_tree_go_tile_after_tile_only_over_many(features, trees):
    """Where two smaller workgroups, with twice as many such waves, share a CU."""
    from paper_2301_13441_amd import binding
    f = _forest(1, trees, 9, features, stop=0.2 if trees > 1 else 0.0)
    for tiles, many in ((3 * 256, False), (16 * 256 - 1, False), (16 * 256, True)):
        s = binding.forest_packed_launch(f, 128 * tiles, form="walk")
        assert s["kernel"] == "deep" and s["tile_after_tile"] == (many or trees > 16 or features > 192), (tiles, s)


@pytest.mark.parametrize("features,waves", [(97, 8), (128, 8), (129, 10), (160, 10), (161, 12), (200, 14), (225, 16), (256, 16)])
def test_tiles_ahead_are_loaded_once(features, waves):
    """A wave per piece of 64 rows x 32 features; no wave asks for another's again."""
    from paper_2301_13441_amd import binding
    s = binding.forest_packed_launch(_forest(1, 20, 9, features), 10**6, form="walk")
    assert s["tile_after_tile"] == 1 and s["loading_waves"] == waves == 2 * -(-features // 32) <= s["threads"] // 64


@pytest.mark.gpu
@pytest.mark.parametrize("features", [97, 127, 130, 193, 224, 253, 256])
@pytest.mark.parametrize("depth,outputs,width", [(9, 1, 1), (12, 2, 2)])
@pytest.mark.parametrize("trees,rows", [(1, 65536), (17, 3 * 32768 + 1), (33, 3 * 32768 + 128 + 65), (48, 3 * 32768 - 3)])
def test_deep_kernels_tile_after_tile(features, depth, outputs, width, trees, rows):
    """Whole and ragged pieces of 32 features, a last tile of one row and of two row groups, CUs with two, three and four tiles; waves
    without trees, with one and with three.  A tree alone takes smaller workgroups up to 192 features."""
    rng = np.random.default_rng(100 * depth + features + trees)
    f = _forest(9 * depth + features, trees, depth, features, outputs, width, stop=0.3 if trees > 1 else 0.0)
    assert len(f.feature) > 200  # a tree alone reads features too
    if trees > 1 or features > 192:
        _tiles(f, rows)
    X = _special_rows(rng.standard_normal((rows, features)).astype(np.float32), f, rng)
    _check(f, X, leaves=False)


@pytest.mark.gpu
@pytest.mark.parametrize("aggregate,transform,outputs,output", [
    (wl.AGG_MEAN, wl.TRANSFORM_NONE, 1, wl.OUT_BOTH), (wl.AGG_MEAN, wl.TRANSFORM_NONE, 2, wl.OUT_BOTH), (wl.AGG_SUM, wl.TRANSFORM_NONE, 1, wl.OUT_LABELS),
    (wl.AGG_SUM, wl.TRANSFORM_NONE, 2, wl.OUT_SCORES), (wl.AGG_MEAN, wl.TRANSFORM_SIGMOID, 1, wl.OUT_SCORES), (wl.AGG_SUM, wl.TRANSFORM_SIGMOID, 2, wl.OUT_BOTH),
    (wl.AGG_MEAN, wl.TRANSFORM_SOFTMAX, 2, wl.OUT_LABELS)])
def test_tile_after_tile_finishes_rows_as_the_model_says(aggregate, transform, outputs, output):
    """Means and sums, base scores, every transform, scores or labels alone."""
    rows, features = 65536 + 65, 200
    rng = np.random.default_rng(outputs)
    f = wl.random_forest(5 + outputs, n_trees=37, n_features=features, max_depth=10, stop_prob=0.2, n_outputs=outputs, leaf_width=outputs,
                         aggregate=aggregate, transform=transform, output=output)
    f = wl.Forest(**{**f.__dict__, "base_score": np.float32([0.25, -0.5][:outputs])})
    _tiles(f, rows)
    _check(f, _special_rows(rng.standard_normal((rows, features)).astype(np.float32), f, rng), leaves=False)


@pytest.mark.gpu
@pytest.mark.parametrize("width", [9, 11, 12, 13, 16])
def test_deep_kernels_with_wide_leaves(width):
    """9 values: the sums leave room for two workgroups on a CU; 10 to 12 and 13 to 16: one workgroup."""
    rng = np.random.default_rng(width)
    f = _forest(width, 37, 9, 20, width, width)
    _launches(f, 70_001, "deep", 64)
    _check(f, _special_rows(rng.standard_normal((70_001, 20)).astype(np.float32), f, rng), leaves=True)


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [9001, 49157])
@pytest.mark.parametrize("trees", [1, 4, 5, 17, 33, 63, 64, 65, 130])
def test_deep_leaf_ids_by_rounds_of_trees(trees, rows):
    """One and two row groups per workgroup (with shares of the trees at 9,001 rows); tree counts below, at and beyond a
    round of four trees for each of 16 waves, and rests of one to four trees per wave."""
    import torch
    from paper_2301_13441_amd import binding
    rng = np.random.default_rng(trees)
    f = _forest(trees, trees, 9, 7, stop=0.3)
    s = binding.forest_packed_launch(f, rows, True, form="walk")
    assert s["kernel"] == "deep" and s["rows_per_workgroup"] == (64 if rows == 9001 else 128) and s["shares"] == (2 if rows == 9001 and trees >= 128 else 1), s
    X = _special_rows(rng.standard_normal((rows, 7)).astype(np.float32), f, rng)
    model = binding.forest_load_form(f, "walk")
    try:
        got = model.predict_leaves(torch.from_numpy(X).cuda()).cpu().numpy()
    finally:
        model.close()
    np.testing.assert_array_equal(got, oracle.predict(f, X, want_leaves=True, n_threads=8).leaf_node_id)
