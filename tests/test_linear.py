"""Linear-model family: ABI checks that need no GPU, and GPU parity against the CPU oracle
through the C ABI.  Bar: labels bit-exact, float32 scores within 1e-5 relative / 1e-6 absolute
(both sides accumulate in float64 and round once)."""
import ctypes
import os
import re

import numpy as np
import pytest

from oracle.linear_oracle import predict_linear
from paper_2301_13441_amd import linear_binding as lb
from workloads import OUT_BOTH, OUT_LABELS, OUT_SCORES, TRANSFORM_NONE, TRANSFORM_SIGMOID, TRANSFORM_SOFTMAX
from workloads.linear import LinearModel, make_linear_workload

RTOL, ATOL = 1e-5, 1e-6


def _rand_model(seed, F, K, transform, output=OUT_BOTH):
    rng = np.random.default_rng(seed)
    return LinearModel(F, K, (rng.standard_normal((F, K)) / np.sqrt(F)).astype(np.float32),
                       (rng.standard_normal(K) * 0.2).astype(np.float32), transform, output)


# ---------------------------------------------------------------- no GPU needed
def test_library_exports_every_declared_symbol():
    header = open(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                               "include", "linear.h")).read()
    declared = set(re.findall(r"\b(linear_[a-z_]+)\s*\(", header))
    assert declared == set(lb.LINEAR_EXPORTS)
    lib = lb._lib()
    for name in declared:
        assert hasattr(lib, name)


def test_validation_happens_before_any_device_call():
    lib = lb._lib()
    h = ctypes.c_void_p()

    def load(model):
        d, keep = lb.linear_desc(model)
        return lib.linear_load(ctypes.byref(d), ctypes.byref(h))

    good = _rand_model(0, 4, 3, TRANSFORM_SOFTMAX)
    assert lib.linear_load(None, ctypes.byref(h)) == -1
    assert load(LinearModel(0, 3, good.weight, good.bias, TRANSFORM_NONE)) == -1            # F < 1
    assert load(LinearModel(4, 1, good.weight[:, :1], good.bias[:1], TRANSFORM_SOFTMAX)) == -1  # softmax, K = 1
    assert load(LinearModel(4, 3, good.weight, good.bias, 7)) == -1                          # bad enum
    assert load(LinearModel(4, 33, np.zeros((4, 33), np.float32), None, TRANSFORM_NONE)) == -7  # K limit
    bad = good.weight.copy()
    bad[2, 1] = np.nan
    assert load(LinearModel(4, 3, bad, good.bias, TRANSFORM_NONE)) == -4
    assert h.value is None                                                                  # *out untouched
    assert lib.linear_out_bytes(None, 5) == -1
    assert lib.linear_predict(None, None, 5, None, None) == -1
    assert lib.linear_strerror(-7).decode().startswith("model exceeds")
    lib.linear_free(None)


def test_testing_header_declares_what_the_library_exports():
    header = open(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "linear_testing.h")).read()
    assert set(re.findall(r"\b(linear_[a-z_]+)\s*\(", header)) == set(lb.LINEAR_TESTING_EXPORTS)
    lib = lb._lib()
    assert all(hasattr(lib, name) for name in lb.LINEAR_TESTING_EXPORTS)
    for bad in ((0, 1, 1, -1), (4, 0, 1, -1), (4, 1, 0, -1), (65537, 1, 1, -7), (4, 33, 1, -7), (4, 1, 10**9 + 1, -7)):
        with pytest.raises(lb.LinearError) as e:
            lb.linear_launch_shape(*bad[:2], n_rows=bad[2])
        assert e.value.code == bad[3]


@pytest.mark.parametrize("F", [96, 104, 112, 128, 129, 130, 144, 150, 155, 156])
def test_whole_rows_only_where_their_tile_fits_the_workgroup(F):
    """64 KB of LDS, which a workgroup has anywhere, hold 127 features of two waves' rows at most: wider tiles need what
    the device says, and go by chunks where it says less."""
    most = lb.linear_launch_shape(F, 1)
    assert most["lds_bytes"] <= 160 * 1024 and most["whole_rows"] == (F % 32 != 0 or F <= 96)
    if most["whole_rows"]:
        assert most["lds_bytes"] >= 2 * 64 * 4 * F
        at, less = (lb.linear_launch_shape(F, 1, lds_limit=n) for n in (most["lds_bytes"], most["lds_bytes"] - 1))
        assert at == most
        assert (less["whole_rows"], less["padded"], less["lds_bytes"]) == (0, 0, 0)
        assert less["load_width"] == (4 if F % 4 == 0 else 2 if F % 2 == 0 else 1)
    assert lb.linear_launch_shape(F, 1, lds_limit=64 * 1024)["lds_bytes"] <= 64 * 1024


@pytest.mark.parametrize("rows", [64, 65, 70, 1000, 4096 + 16, 20_000_005])
@pytest.mark.parametrize("F", [8, 28, 48, 55])
def test_only_whole_pieces_of_one_value_a_row_go_past_the_l2(F, rows):
    """Labels lie behind the scores, and the buffer may begin at any float: where that leaves a wave's run of them off a
    64-byte boundary, two waves would write the same piece of memory past the L2 one after the other."""
    for at in (1 << 20, (1 << 20) + 4, (1 << 20) + 32, (1 << 20) + 64):
        for K in (1, 2, 7):
            labels = at + 4 * rows * K
            s = lb.linear_launch_shape(F, K, 1 << 12, at, labels)
            assert s["labels_past"] == (labels % 64 == 0), (at, K)
            assert s["scores_past"] == (K > 1 or at % 64 == 0), (at, K)
            assert lb.linear_launch_shape(F, K, 1 << 12, 0, at)["scores_past"] == 0
            assert lb.linear_launch_shape(F, K, 1 << 12, at, 0)["labels_past"] == 0


def test_rows_of_a_few_features_keep_both_or_neither_result_in_the_l2():
    at = 1 << 20
    for rows in (16, 17, 4_734_624, 4_734_629):
        for F in (1, 5, 6, 12):
            s = lb.linear_launch_shape(F, 1, 1 << 12, at, at + 4 * rows)
            assert (s["scores_past"], s["labels_past"]) == (rows % 16 == 0 or F > 5, rows % 16 == 0)
        assert lb.linear_launch_shape(1, 1, 1 << 12, at, 0)["scores_past"] == 1
        assert lb.linear_launch_shape(1, 2, 1 << 12, at, at + 8 * rows)["scores_past"] == 1


@pytest.mark.parametrize("rows", [64, 1000, 4_000_000, 4_000_005])
def test_one_score_of_a_wide_row_stays_out_of_the_way_of_its_label(rows):
    """From 64 features on the score is stored non-temporally with and without a label, and the label past the L2; below,
    and with several outputs, scores go past the L2."""
    at = 1 << 20
    for F, K in ((64, 1), (90, 1), (300, 1), (63, 1), (90, 7)):
        past = F < 64 or K > 1
        assert lb.linear_launch_shape(F, K, 1 << 12, at, 0)["scores_past"] == past
        s = lb.linear_launch_shape(F, K, 1 << 12, at, at + 4 * rows * K)
        assert s["scores_past"] == past and s["labels_past"] == (rows % 16 == 0 or (K == 1 and F >= 64))


def test_results_of_two_or_three_outputs_of_a_small_batch_of_wide_rows_are_kept_in_the_l2():
    past = lambda F, K, rows: lb.linear_launch_shape(F, K, 1 << 12, 1 << 20, 0, n_rows=rows)["scores_past"]
    for F in (56, 64, 90, 128, 300):
        most = (1 << 27) // F
        for K, kept in ((2, True), (3, True), (4, False), (10, False)):
            assert past(F, K, 1) == past(F, K, most - 1) == (not kept)
            assert lb.linear_launch_shape(F, K, 1 << 12, 1 << 20, 1 << 21, n_rows=most - 1)["labels_past"] == (not kept)
            assert past(F, K, most + 1) == past(F, K, 10**9) == 1
    assert past(55, 2, 1000) == past(28, 3, 1000) == 1


@pytest.mark.parametrize("F", [108, 112, 128, 130, 132, 160, 200, 201, 300])
def test_chunks_are_kept_in_the_caches_where_they_share_lines_and_outputs_are_few(F):
    for K in (2, 10, 16, 17, 20, 32):
        for x in (0, 4, 8, 16, 64, 128):
            s = lb.linear_launch_shape(F, K, (1 << 20) + x, n_rows=300_000)
            width = 4 if F % 4 == 0 and x % 16 == 0 else 2 if F % 2 == 0 and x % 8 == 0 else 1
            assert s["whole_rows"] == 0 and s["load_width"] == width
            assert s["once"] == (width == 4 and (K > 16 or (F % 32 == 0 and x % 128 == 0)))


@pytest.mark.parametrize("F", [112, 132, 200, 300])
def test_chunks_of_a_batch_with_a_cu_for_every_workgroup_are_not_kept_in_the_caches(F):
    once = lambda K, n, x=0: lb.linear_launch_shape(F, K, (1 << 20) + x, n_rows=n)["once"]
    few = (1 << 22) // F
    long = max(65_536, min(131_072, 7 * (1 << 21) // F))
    longest = 131_072 if F <= 160 else 262_144
    for K, most in ((2, 65_536), (6, 65_536), (7, long), (10, long), (11, 131_072), (12, 131_072), (13, longest), (16, longest)):
        assert once(K, 1) == once(K, few) == 0 and once(K, few + 1) == once(K, most) == 1 and once(K, most + 1) == 0
        assert once(K, most, x=8) == 0  # narrower loads
    assert once(17, 1) == once(17, 10**6) == 1


def test_where_rows_of_more_than_96_features_go_whole():
    """One round of row workgroups is 98,304 rows where three of them fit a CU; a rest behind it costs another round."""
    rows = lambda F, K, n: lb.linear_launch_shape(F, K, 1 << 20, n_rows=n)["whole_rows"]
    for F in (97, 98, 100, 103, 104):
        loose = F % 4 != 0
        for n in (1, 1000, 65_536, 65_537, 98_304, 98_305, 200_000, 1 << 18, (1 << 18) + 1, 2_000_000):
            assert rows(F, 1, n) == 1
            for K in (2, 3):
                assert rows(F, K, n) == (loose or n <= 98_304 or n > 1 << 18), (F, K, n)
            for K in (4, 6):
                assert rows(F, K, n) == (n <= 98_304 or n > 1 << 18), (F, K, n)
            for K in (7, 8):
                assert rows(F, K, n) == (65_536 < n <= 98_304), (F, K, n)
            for K in (9, 16):
                assert rows(F, K, n) == (n <= 98_304), (F, K, n)
            for K in (17, 32):
                assert rows(F, K, n) == (loose or n <= 98_304), (F, K, n)
    for F in (105, 108, 112, 120, 130, 136, 144, 152, 155, 156):
        for n in (1, 32_768, 32_769, 90_000, 1 << 19, (1 << 19) + 1, 4_000_000):
            assert rows(F, 1, n) == (F % 8 != 0 or n <= 32_768 or n > 1 << 19), (F, n)
            assert rows(F, 2, n) == 0
    for K in (1, 2, 10, 32):
        for n in (1, 90_000, 4_000_000):
            assert rows(96, K, n) == rows(64, K, n) == 1 and rows(128, K, n) == rows(157, K, n) == rows(160, K, n) == 0


# ---------------------------------------------------------------- GPU parity
def _run(model, X):
    import torch
    m = lb.linear_load(model)
    try:
        xd = torch.from_numpy(np.ascontiguousarray(X)).cuda()
        scores, labels = m.predict(xd)
        torch.cuda.synchronize()
        return (None if scores is None else scores.cpu().numpy(),
                None if labels is None else labels.cpu().numpy())
    finally:
        m.close()


def _check(model, X):
    ref = predict_linear(model, X)
    scores, labels = _run(model, X)
    if model.output != OUT_SCORES:
        np.testing.assert_array_equal(labels, ref.labels)
    else:
        assert labels is None
    if model.output != OUT_LABELS:
        np.testing.assert_allclose(scores, ref.scores, rtol=RTOL, atol=ATOL)
    else:
        assert scores is None


@pytest.mark.gpu
@pytest.mark.parametrize("name,rows", [("l1", 1000), ("l2", 70001), ("l3", 50003), ("l4", 65537)])
def test_configs(name, rows):
    w = make_linear_workload(name, n_rows=rows)
    _check(w.model, w.make_x())


@pytest.mark.gpu
@pytest.mark.parametrize("F", [1, 3, 31, 32, 33, 64, 90, 257])
@pytest.mark.parametrize("K,transform", [(1, TRANSFORM_NONE), (1, TRANSFORM_SIGMOID), (2, TRANSFORM_SOFTMAX),
                                          (7, TRANSFORM_SOFTMAX), (10, TRANSFORM_NONE), (17, TRANSFORM_SOFTMAX),
                                          (32, TRANSFORM_SIGMOID)])
def test_shapes_ragged_in_every_direction(F, K, transform):
    model = _rand_model(100 * F + K, F, K, transform)
    rng = np.random.default_rng(F + K)
    for rows in (1, 63, 64, 65, 300):
        _check(model, rng.standard_normal((rows, F)).astype(np.float32))


@pytest.mark.gpu
@pytest.mark.parametrize("F", [4, 8, 28, 100, 124, 128])
def test_rows_of_whole_16_byte_pieces(F):
    """Feature counts that are multiples of 4 on both sides of the whole-row / chunked kernel
    boundary, full and partial tiles."""
    for K, transform in ((1, TRANSFORM_SIGMOID), (10, TRANSFORM_SOFTMAX)):
        model = _rand_model(7 * F + K, F, K, transform)
        rng = np.random.default_rng(F * K)
        for rows in (1, 63, 64, 65, 129, 1000):
            _check(model, rng.standard_normal((rows, F)).astype(np.float32))


@pytest.mark.gpu
@pytest.mark.parametrize("F", [4, 15, 16, 32, 48, 80, 95, 96, 97, 100, 104, 105, 112, 128, 144, 155, 156, 157, 160, 200])
@pytest.mark.parametrize("K,rows", [(1, 64 * 130 + 3), (1, 1), (3, 64 * 70 + 63), (12, 64 * 5 + 1), (20, 130)])
def test_tiles_of_rows_with_and_without_padding(F, K, rows):
    """Rows of a multiple of 16 floats, whose tile has padding, and of others; the widest rows that go as whole tiles, for one
    output and several, and the narrowest by chunks; partial tiles, whose last floats are copied one by one."""
    m = _rand_model(5 * F + K, F, K, TRANSFORM_SOFTMAX if K > 1 else TRANSFORM_SIGMOID)
    _check(m, np.random.default_rng(F + rows).standard_normal((rows, F)).astype(np.float32))


@pytest.mark.gpu
@pytest.mark.parametrize("F,K,rows", [(100, 2, 98_304), (100, 2, 98_305), (98, 4, 98_369), (104, 8, 65_536), (104, 8, 65_537), (101, 12, 98_311),
                                      (97, 17, 98_305), (200, 2, 40_000), (200, 2, 65_537), (132, 16, 131_073), (112, 1, 32_768), (112, 1, 32_769), (152, 1, (1 << 19) + 1), (100, 3, (1 << 18) + 1)])
def test_both_sides_of_the_rows_that_a_round_of_workgroups_holds(F, K, rows):
    m = _rand_model(F + K, F, K, TRANSFORM_SOFTMAX if K > 1 else TRANSFORM_SIGMOID)
    _check(m, np.random.default_rng(rows).standard_normal((rows, F), dtype=np.float32))


@pytest.mark.gpu
@pytest.mark.parametrize("F", [28, 40, 64, 90, 100, 130])
def test_x_that_starts_off_a_16_byte_boundary_and_absent_bias(F):
    """X may start at any float: 4, 8 or 12 bytes past a 16-byte boundary the kernels fall back
    to narrower loads.  The bias pointer may be NULL (zeros)."""
    import torch
    rng = np.random.default_rng(F)
    model = LinearModel(F, 3, rng.standard_normal((F, 3)).astype(np.float32), None, TRANSFORM_SOFTMAX, OUT_BOTH)
    m = lb.linear_load(model)
    try:
        for off in (0, 1, 2, 3):
            for rows in (1, 65, 300):
                X = rng.standard_normal((rows, F)).astype(np.float32)
                buf = torch.empty(rows * F + 4, dtype=torch.float32, device="cuda")
                xd = buf[off:off + rows * F].view(rows, F)
                xd.copy_(torch.from_numpy(X))
                assert xd.data_ptr() % 16 == 4 * off
                scores, labels = m.predict(xd)
                torch.cuda.synchronize()
                ref = predict_linear(model, X)
                np.testing.assert_array_equal(labels.cpu().numpy(), ref.labels)
                np.testing.assert_allclose(scores.cpu().numpy(), ref.scores, rtol=RTOL, atol=ATOL)
    finally:
        m.close()


@pytest.mark.gpu
@pytest.mark.parametrize("F", [105, 112, 128, 130, 156, 160, 200])
@pytest.mark.parametrize("K", [1, 3, 20])
def test_chunks_of_x_at_every_alignment(F, K):
    """Rows that go by chunks wherever X begins, on and off the lines that chunks of 32 features are, and those of one output
    that go whole from a 16-byte boundary only; full and partial tiles, one of them with all its chunks whole."""
    import torch
    rng = np.random.default_rng(F + K)
    model = _rand_model(F * K, F, K, TRANSFORM_SOFTMAX if K > 1 else TRANSFORM_SIGMOID)
    m = lb.linear_load(model)
    try:
        for rows in (1, 64, 300):
            X = rng.standard_normal((rows, F)).astype(np.float32)
            ref = predict_linear(model, X)
            for off in (0, 1, 2, 4, 8, 16, 32):
                buf = torch.empty(rows * F + 32, dtype=torch.float32, device="cuda")
                xd = buf[off:off + rows * F].view(rows, F)
                xd.copy_(torch.from_numpy(X))
                assert xd.data_ptr() % 128 == 4 * (off % 32)
                scores, labels = m.predict(xd)
                torch.cuda.synchronize()
                np.testing.assert_array_equal(labels.cpu().numpy(), ref.labels)
                np.testing.assert_allclose(scores.cpu().numpy(), ref.scores, rtol=RTOL, atol=ATOL)
    finally:
        m.close()


@pytest.mark.gpu
@pytest.mark.parametrize("F", [12, 28, 64, 90, 128, 130])
@pytest.mark.parametrize("K", [1, 2, 3, 10, 20])
def test_results_that_start_off_a_16_byte_boundary(F, K):
    """The buffer of scores and labels may start at any float and labels follow the scores of any number of rows; nothing
    before or behind them is touched.  Full and ragged last tiles."""
    import torch
    model = _rand_model(F + K, F, K, TRANSFORM_SOFTMAX if K > 1 else TRANSFORM_SIGMOID)
    rng = np.random.default_rng(F * K)
    m = lb.linear_load(model)
    try:
        for rows in (1, 64, 129, 1000):
            X = rng.standard_normal((rows, F)).astype(np.float32)
            xd, ref = torch.from_numpy(X).cuda(), predict_linear(model, X)
            for off in (0, 1, 2, 3, 16):
                n = rows * (K + 1)
                buf = torch.full((n + 64,), -1, dtype=torch.int32, device="cuda")
                out = buf[off + 16:off + 16 + n]
                assert out.data_ptr() % 64 == 4 * (off % 16)
                scores, labels = m.predict(xd, out=out)
                torch.cuda.synchronize()
                np.testing.assert_allclose(scores.cpu().numpy(), ref.scores, rtol=RTOL, atol=ATOL)
                np.testing.assert_array_equal(labels.cpu().numpy(), ref.labels)
                guard = torch.cat([buf[:off + 16], buf[off + 16 + n:]]).cpu().numpy()
                assert (guard == -1).all()
    finally:
        m.close()


@pytest.mark.gpu
def test_output_kinds_ties_and_empty_batch():
    import torch
    X = np.random.default_rng(5).standard_normal((130, 6)).astype(np.float32)
    for output in (OUT_SCORES, OUT_LABELS, OUT_BOTH):
        _check(_rand_model(9, 6, 4, TRANSFORM_SOFTMAX, output), X)
    # exact ties between columns: the first maximum wins
    tie = LinearModel(6, 3, np.zeros((6, 3), np.float32), np.float32([0.5, 0.5, 0.25]), TRANSFORM_SOFTMAX, OUT_BOTH)
    _check(tie, X)
    m = lb.linear_load(tie)
    m.predict_raw(0, 0, 0, 0)   # n_rows == 0 is a successful no-op
    with pytest.raises(lb.LinearError) as e:   # more rows than one call takes
        m.predict_raw(256, 10**9 + 1, 256, 0)
    assert e.value.code == -7
    for bad in (torch.zeros((10, 5), dtype=torch.float32, device="cuda"),      # wrong feature count
                torch.zeros((10, 6), dtype=torch.float32),                     # host memory
                torch.zeros((10, 6), dtype=torch.float16, device="cuda")):     # wrong dtype
        with pytest.raises(ValueError):
            m.predict(bad)
    m.close()
    torch.cuda.synchronize()


@pytest.mark.gpu
def test_large_magnitudes_and_cancellation():
    """Float64 accumulation: sums that cancel to a small value keep their digits."""
    rng = np.random.default_rng(8)
    F = 64
    w = np.tile(np.float32([1.0, -1.0]), F // 2).reshape(F, 1)
    model = LinearModel(F, 1, w, np.float32([0.0]), TRANSFORM_NONE, OUT_SCORES)
    base = (rng.standard_normal((500, F // 2)) * 1e4).astype(np.float32)
    X = np.empty((500, F), np.float32)
    X[:, 0::2] = base
    X[:, 1::2] = base + rng.standard_normal((500, F // 2)).astype(np.float32) * np.float32(1e-3)
    _check(model, X)


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["l2", "l3", "l4"])
def test_full_size_sampled(name):
    """The bench's launch configuration at full size; the oracle checks sampled rows."""
    import torch
    w = make_linear_workload(name)
    m = lb.linear_load(w.model)
    try:
        n = w.n_rows
        xd = torch.empty((n, w.model.n_features), dtype=torch.float32, device="cuda")
        pos = 0
        keep = {}
        rng = np.random.default_rng(17)
        for ci, chunk in enumerate(w.x_chunks()):
            xd[pos:pos + len(chunk)].copy_(torch.from_numpy(chunk))
            if ci % 7 == 0 or pos + len(chunk) == n:
                idx = np.unique(np.concatenate([rng.integers(0, len(chunk), 200), [0, len(chunk) - 1]]))
                keep[pos] = (idx, chunk[idx].copy())
            pos += len(chunk)
        scores, labels = m.predict(xd)
        torch.cuda.synchronize()
        for start, (idx, rows) in keep.items():
            ref = predict_linear(w.model, rows)
            sel = torch.from_numpy(start + idx).cuda()
            np.testing.assert_allclose(scores[sel].cpu().numpy(), ref.scores, rtol=RTOL, atol=ATOL)
            if labels is not None:
                np.testing.assert_array_equal(labels[sel].cpu().numpy(), ref.labels)
    finally:
        m.close()


@pytest.mark.gpu
def test_input_larger_than_2_to_31_elements():
    """Row offsets past 2^31 elements of X in both kernels (whole-row tiles: 30 features;
    chunked: 130 features); the oracle checks the ends and seeded rows between."""
    import torch
    for F, K, n in ((30, 3, 75_000_000), (130, 2, 17_000_000)):
        assert n * F > 2**31
        model = _rand_model(F, F, K, TRANSFORM_SOFTMAX)
        gen = torch.Generator(device="cuda").manual_seed(F)
        xd = torch.empty((n, F), dtype=torch.float32, device="cuda")
        step = 5_000_000
        for pos in range(0, n, step):
            xd[pos:pos + step].normal_(generator=gen)
        rng = np.random.default_rng(F)
        pick = np.unique(np.concatenate([np.arange(200), np.arange(n - 200, n), rng.integers(0, n, 3000),
                                         rng.integers(2**31 // F, n, 3000)]))
        idx = torch.from_numpy(pick).cuda()
        xs = xd[idx].cpu().numpy()
        m = lb.linear_load(model)
        try:
            scores, labels = m.predict(xd)
            torch.cuda.synchronize()
            got_scores, got_labels = scores[idx].cpu().numpy(), labels[idx].cpu().numpy()
        finally:
            m.close()
        del xd, scores, labels
        ref = predict_linear(model, xs)
        np.testing.assert_array_equal(got_labels, ref.labels)
        np.testing.assert_allclose(got_scores, ref.scores, rtol=RTOL, atol=ATOL)
