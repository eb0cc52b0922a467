"""Normaliser and moments of the sky-dependent weights at the SFT counts where their chain of
additions changes form (register groups of 32, chunks of 256): sums, critical ratios and
toplists are the oracle's bit for bit."""
import numpy as np
import pytest

from paper_2411_18370_amd import synth
from test_gpu_weighting import _assert_sky_tops, _ctx, _grid_eval, _sky_case, _want_tops, _weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_sft", [1, 31, 32, 33, 63, 64, 96, 255, 256, 257, 288, 511, 513])
@pytest.mark.parametrize("weighted", [False, True])
def test_sky_moments_sft_counts(ft, n_sft, weighted):
    w = synth.tiny_bank(24, 2, 9, 300)
    w.t_mid, w.v, w.arms, w.power = w.t_mid[:n_sft], w.v[:n_sft], w.arms[:n_sft], np.ascontiguousarray(w.power[:n_sft])
    w.n_sft_per_det = [n_sft]
    u = _weights(w, weighted)
    S, ms = _sky_case(w, u, 0)
    c = _ctx(ft, w, u)
    try:
        _, tops = _grid_eval(ft, c, w, weights=ft.FT_WEIGHTS_SKY)
    finally:
        c.close()
    _assert_sky_tops(tops, _want_tops(w, S), S, ms, w.f0.size * w.f1.size)
