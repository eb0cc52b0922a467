"""The check of the surrogate's inputs on both of its sides: the host reads up to 16384 rows,
the device more.  The first bad row is the one reported, wherever it lies (either end, the
edges of the device's 256-row workgroups); nothing is changed or returned before.  And
queries around 2048 rows, where their tiles change from 8 to 16 rows."""
import numpy as np
import pytest

from oracle import mlp as ref
from test_gpu_mlp import SCALE, SHIFT, _raw

pytestmark = pytest.mark.gpu

BAD = [(0, 0.0, "input {r}: amplitude must be > 0"), (0, np.nan, "input {r}: amplitude must be > 0"),
       (0, -np.inf, "input {r}: amplitude must be > 0"), (0, np.inf, "inputs must be finite"),
       (3, np.nan, "inputs must be finite"), (5, -np.inf, "inputs must be finite")]


def _net(ft, **kw):
    import torch
    c = ft.Context(0, torch.cuda.current_stream().cuda_stream)
    return c, ft.Mlp(c, SHIFT, SCALE, **kw)


def _refused(ft, text, call):
    with pytest.raises(ft.FtError, match=text) as e:
        call()
    assert e.value.status == ft.FT_E_INVALID


@pytest.mark.parametrize("n", [16384, 16385, 40000])
@pytest.mark.parametrize("col,value,text", BAD)
def test_first_bad_input(ft, n, col, value, text):
    rng = np.random.default_rng(n)
    raw, y = _raw(rng, n).astype(np.float32), np.zeros(n, np.float32)
    c, net = _net(ft, max_batch=1024, seed=1)
    before = net.params()
    for row in (0, 255, 256, 16383, n - 1):
        bad = raw.copy()
        bad[row, col] = value
        # later rows that would read differently, and a label that is looked at last
        bad[row + 1:row + 2, 1] = np.nan
        bad[row + 300:, 0] = -1.0
        yb = y.copy()
        yb[0] = 2.0
        for call in (lambda: net.predict(bad), lambda: net.train(bad, yb, batch=1024, epochs=1, lr=1e-3)):
            _refused(ft, text.format(r=row), call)
    assert np.array_equal(net.params(), before)
    net.close()
    c.close()


@pytest.mark.parametrize("n", [16384, 16385, 40000])
def test_first_bad_label(ft, n):
    rng = np.random.default_rng(n)
    raw, y = _raw(rng, n).astype(np.float32), (rng.uniform(size=n) < 0.5).astype(np.float32)
    c, net = _net(ft, max_batch=1024, seed=1)
    before = net.params()
    for row in (0, 255, 256, n - 1):
        for v in (np.nextafter(np.float32(0), np.float32(-1)), np.nextafter(np.float32(1), np.float32(2)), np.nan, np.inf):
            bad = y.copy()
            bad[row] = v
            _refused(ft, "labels must lie", lambda: net.train(raw, bad, batch=1024, epochs=1, lr=1e-3))
    assert np.array_equal(net.params(), before)
    net.train(raw, y, batch=1024, epochs=1, lr=1e-3)  # nothing of the refused calls is left
    assert np.all(np.isfinite(net.params())) and not np.array_equal(net.params(), before)
    net.close()
    c.close()


@pytest.mark.parametrize("n", [2047, 2048, 2049])
def test_predict_where_the_tiles_change(ft, n):
    rng = np.random.default_rng(n)
    theta = ref.init_params(3).astype(np.float32)
    raw = _raw(rng, n).astype(np.float32)
    logit, _ = ref.forward(theta.astype(np.float64), ref.features(raw.astype(np.float64), SHIFT, SCALE))
    c, net = _net(ft, max_batch=64, params=theta)
    p = net.predict(raw)
    some = [0, n // 2, n - 1]
    q = net.predict(raw[some])
    net.close()
    c.close()
    assert np.max(np.abs(p - ref.sigmoid(logit))) < 0.02  # BF16 operands, as for the unfused layers
    assert np.array_equal(p[some], q)
