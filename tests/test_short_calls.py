"""predict() with a buffer of its own against predict() into the caller's: same views, same bits; and linear
models with several outputs, whose scores leave a wave as one piece."""
import numpy as np
import pytest

import workloads as wl
from workloads.linear import LinearModel


@pytest.mark.gpu
@pytest.mark.parametrize("outputs", [1, 3])
@pytest.mark.parametrize("kind", [wl.OUT_SCORES, wl.OUT_LABELS, wl.OUT_BOTH])
@pytest.mark.parametrize("family", ["forest", "linear"])
def test_own_buffer_and_the_callers(family, kind, outputs):
    import torch
    import paper_2301_13441_amd as pk
    rng = np.random.default_rng(5)
    if family == "forest":
        model = pk.forest_load(wl.random_forest(4, 30, 9, 6, n_outputs=outputs, output=kind))
    else:
        model = pk.linear_load(LinearModel(9, outputs, rng.standard_normal((9, outputs)).astype(np.float32),
                                           np.zeros(outputs, np.float32), wl.TRANSFORM_NONE, kind))
    for rows in (0, 1, 77):
        X = torch.from_numpy(rng.standard_normal((rows, 9)).astype(np.float32)).cuda()
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            own = model.predict(X)
            callers = model.predict(X, out=torch.empty(max(model.out_bytes(rows), 4), dtype=torch.uint8, device="cuda"))
        side.synchronize()
        for a, b, shape, dtype in zip(own, callers, ((rows, outputs), (rows,)), (torch.float32, torch.int32)):
            assert (a is None) == (b is None)
            if a is not None:
                assert a.shape == b.shape == shape and a.dtype == b.dtype == dtype and a.is_contiguous()
                assert torch.equal(a, b)
    assert (own[0] is None) == (kind == wl.OUT_LABELS) and (own[1] is None) == (kind == wl.OUT_SCORES)
    with pytest.raises(ValueError):
        model.predict(X.double())
    model.close()


@pytest.fixture
def without_the_extension(monkeypatch):
    import sys
    import paper_2301_13441_amd as pk
    monkeypatch.delattr(pk, "_short_call", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2301_13441_amd._short_call", None)  # its import raises ImportError


def test_a_missing_extension_declines(without_the_extension):
    from paper_2301_13441_amd import binding
    with pytest.warns(RuntimeWarning, match="paper_2301_13441_amd.build"):
        call = binding.short_call()
    assert call(0, 0, None, 1, 1, 1, 1) is None


@pytest.mark.gpu
@pytest.mark.parametrize("family", ["forest", "linear"])
def test_models_load_and_predict_without_the_extension(family, without_the_extension):
    import torch
    import paper_2301_13441_amd as pk
    rng = np.random.default_rng(8)
    X = torch.from_numpy(rng.standard_normal((50, 9)).astype(np.float32)).cuda()
    with pytest.warns(RuntimeWarning):
        if family == "forest":
            model = pk.forest_load(wl.random_forest(4, 30, 9, 6, n_outputs=2))
        else:
            model = pk.linear_load(LinearModel(9, 2, rng.standard_normal((9, 2)).astype(np.float32), np.zeros(2, np.float32), wl.TRANSFORM_NONE, wl.OUT_BOTH))
    out = torch.empty(model.out_bytes(50), dtype=torch.uint8, device="cuda")
    got = model.predict(X)
    assert all(torch.equal(a, b) for a, b in zip(got, model.predict(X, out=out)))
    if family == "forest":
        assert torch.equal(model.predict_leaves(X), model.predict_leaves(X, stream=torch.cuda.current_stream()))
    model.close()


@pytest.mark.gpu
@pytest.mark.parametrize("features,outputs", [(2, 12), (12, 12), (7, 3), (90, 2), (96, 32), (97, 5), (128, 10), (130, 24)])
def test_linear_scores_of_whole_and_ragged_tiles(features, outputs):
    import torch
    import paper_2301_13441_amd as pk
    from oracle.linear_oracle import predict_linear
    rng = np.random.default_rng(features)
    model = LinearModel(features, outputs, (rng.standard_normal((features, outputs)) / 9).astype(np.float32),
                        rng.standard_normal(outputs).astype(np.float32), wl.TRANSFORM_SOFTMAX, wl.OUT_BOTH)
    f = pk.linear_load(model)
    for rows in (1, 63, 64, 65, 200, 1027):
        X = rng.standard_normal((rows, features)).astype(np.float32)
        out = torch.full((f.out_bytes(rows) + 64,), 0xAB, dtype=torch.uint8, device="cuda")
        scores, labels = f.predict(torch.from_numpy(X).cuda(), out=out)
        ref = predict_linear(model, X)
        np.testing.assert_array_equal(labels.cpu().numpy(), ref.labels)
        # fp64 sums rounded to fp32 once on both sides: one rounding apart at most (6e-8)
        np.testing.assert_allclose(scores.cpu().numpy(), ref.scores, rtol=2e-7, atol=1e-30)
        assert bool((out[f.out_bytes(rows):] == 0xAB).all())
    f.close()


@pytest.mark.gpu
@pytest.mark.parametrize("family", ["forest", "linear"])
def test_what_the_native_call_declines_goes_the_general_way(family):
    """Tensors it does not take are refused as before or give the same bits; a closed model is refused; leaf ids and
    sums follow the current stream; several threads on their own streams."""
    import threading

    import torch
    import paper_2301_13441_amd as pk
    rng = np.random.default_rng(8)
    if family == "forest":
        model = pk.forest_load(wl.random_forest(4, 30, 9, 6, n_outputs=2))
    else:
        model = pk.linear_load(LinearModel(9, 2, rng.standard_normal((9, 2)).astype(np.float32),
                                           np.zeros(2, np.float32), wl.TRANSFORM_NONE, wl.OUT_BOTH))
    X = torch.from_numpy(rng.standard_normal((500, 9)).astype(np.float32)).cuda()
    want = model.predict(X)
    for same in (torch.nn.Parameter(X), X.clone().requires_grad_(), torch.cat([X, X])[:500]):
        for a, b in zip(model.predict(same), want):
            assert torch.equal(a, b)
    for wrong in (X.double(), X.cpu(), X.half(), X[:, :8], X[::2].t(), X.t(), X[0], X.repeat(1, 2)[:, ::2], None, X.cpu().numpy()):
        calls = [model.predict] + ([model.predict_leaves] if family == "forest" else [])
        for call in calls:
            with pytest.raises(ValueError):
                call(wrong)
    got = [None] * 4

    def work(i):
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.default_stream())
        with torch.cuda.stream(side):
            Y = X * 1.0
            for _ in range(20):
                got[i] = model.predict(Y) + ((model.predict_leaves(Y),) if family == "forest" else ())
        side.synchronize()

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    leaves = (model.predict_leaves(X),) if family == "forest" else ()
    for result in got:
        assert all(torch.equal(a, b) for a, b in zip(result, want + leaves))
    model.close()
    with pytest.raises(RuntimeError):
        model.predict(X)
