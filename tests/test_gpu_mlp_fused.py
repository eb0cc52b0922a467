"""The surrogate's fused kernels at the edges of their tiles: 16- and 32-row query tiles,
walks of more than 256 workgroups, batches around the 64-row padding and the slice rule,
and the check of inputs and labels on the
host (short calls) and the device."""
import numpy as np
import pytest

from oracle import mlp as ref
from test_gpu_mlp import SCALE, SHIFT, _check_grad, _raw

pytestmark = pytest.mark.gpu


def _ctx(ft):
    import torch
    return ft.Context(0, torch.cuda.current_stream().cuda_stream)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 4096, 4097, 8191, 8193, 20000])
def test_predict_tiles(ft, n):
    rng = np.random.default_rng(n)
    theta = ref.init_params(3).astype(np.float32)
    raw = _raw(rng, n).astype(np.float32)
    logit, _ = ref.forward(theta.astype(np.float64), ref.features(raw.astype(np.float64), SHIFT, SCALE))
    with _ctx(ft) as c:
        net = ft.Mlp(c, SHIFT, SCALE, max_batch=64, params=theta)
        p = net.predict(raw)
        # a row's result does not depend on the rows beside it
        some = np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, 40)]))
        q = net.predict(raw[some])
        net.close()
    assert np.max(np.abs(p - ref.sigmoid(logit))) < 0.02  # BF16 operands, as for the unfused layers
    assert np.array_equal(p[some], q)


@pytest.mark.parametrize("n", [2, 63, 65, 255, 511, 513, 3000, 8192])
def test_gradient_tiles(ft, n):
    rng = np.random.default_rng(n)
    theta = ref.init_params(4).astype(np.float32)
    raw = _raw(rng, n).astype(np.float32)
    y = (rng.uniform(size=n) < 0.4).astype(np.float32)
    loss64, g64 = ref.loss_and_grad(theta.astype(np.float64), ref.features(raw.astype(np.float64), SHIFT, SCALE),
                                    y.astype(np.float64))
    with _ctx(ft) as c:
        net = ft.Mlp(c, SHIFT, SCALE, max_batch=8192, params=theta)
        full = _raw(rng, 8192).astype(np.float32)
        net.loss_grad(full, np.ones(8192, np.float32))  # rows a smaller batch must not see
        loss, g = net.loss_grad(raw, y)
        net.close()
    assert abs(loss - loss64) < 2e-2 * loss64
    _check_grad(g, g64)


@pytest.mark.parametrize("n", [1000, 5000])
@pytest.mark.parametrize("row,col,value,text", [
    (700, 0, 0.0, "input 700: amplitude must be > 0"), (700, 0, np.nan, "input 700: amplitude must be > 0"),
    (3, 0, np.inf, "inputs must be finite"), (999, 5, -np.inf, "inputs must be finite"),
    (0, 3, np.nan, "inputs must be finite")])
def test_check_reports_the_first_bad_input(ft, n, row, col, value, text):
    rng = np.random.default_rng(5)
    raw = _raw(rng, n).astype(np.float32)
    y = np.zeros(n, np.float32)
    with _ctx(ft) as c:
        net = ft.Mlp(c, SHIFT, SCALE, max_batch=1024, seed=1)
        before = net.params()
        bad = raw.copy()
        bad[row, col] = value
        if row < 900:
            bad[row + 90, 0] = -1.0  # a later one
        for call in (lambda: net.predict(bad), lambda: net.train(bad, y, batch=512, epochs=1, lr=1e-3)):
            with pytest.raises(ft.FtError, match=text) as e:
                call()
            assert e.value.status == ft.FT_E_INVALID
        for v in (-1e-6, 1.5, np.nan):
            yb = y.copy()
            yb[-1] = v
            with pytest.raises(ft.FtError, match="labels must lie"):
                net.train(raw, yb, batch=512, epochs=1, lr=1e-3)
        assert np.array_equal(net.params(), before)
        net.close()
