"""Sequential FP64 sums formed 256 terms at a time: bit for bit the oracle's term-by-term sums
where that is hard -- ties at the sum's last bit, terms that cross many binades, runs of
zeros, terms far below and far above the sum, a sum that starts at zero."""
import numpy as np
import pytest

import oracle
from paper_2411_18370_amd import synth

pytestmark = pytest.mark.gpu


def _table(kind, shape, rng):
    if kind == "ties":      # odd 24-bit significands times odd 24-bit weights: 48-bit products
        return (1.0 + (2 * rng.integers(0, 2 ** 22, shape) + 1) * 2.0 ** -23).astype(np.float32)
    if kind == "binades":
        return np.exp2(rng.uniform(-60.0, 40.0, shape)).astype(np.float32)
    if kind == "zeros":
        return np.where(rng.uniform(size=shape) < 0.9, 0.0, rng.exponential(1.0, shape)).astype(np.float32)
    if kind == "tiny":      # the first rows large, then terms near and below half an ulp of the sum
        t = np.exp2(rng.integers(-56, -44, shape).astype(np.float64)).astype(np.float32)
        t[:3] = 3.0
        return t
    return np.full(shape, 2.0 ** -149, np.float32)  # "denormal"


@pytest.mark.parametrize("kind", ["ties", "binades", "zeros", "tiny", "denormal"])
@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("k", [30, 5000])
def test_chain_bits(ft, kind, weighted, k):
    import torch
    rng = np.random.default_rng(11)
    w = synth.tiny_bank(40, 1, 1, 1100)
    n, n_sft = (400 if k < 1000 else 6000), w.t_mid.size
    f0, f1, sky = rng.uniform(150.0, 150.02, n), rng.uniform(-3e-10, 2e-10, n), synth.isotropic_sky(n, rng)
    power = _table(kind, w.power.shape, rng)
    u = (0.5 + (2 * rng.integers(0, 2 ** 22, n_sft) + 1) * 2.0 ** -24).astype(np.float32) if weighted else None
    s64, bad = oracle.eval_list(w.t_mid, w.t_ref, w.t_sft, w.first_bin, power, u, w.v, f0, f1, sky)
    assert bad == -1
    with ft.Context(0, torch.cuda.current_stream().cuda_stream) as c:
        c.set_sfts(w.n_sft_per_det, w.t_mid, w.t_sft, w.first_bin, power, u)
        c.set_velocities(w.v)
        c.eval_templates(f0, f1, sky, w.t_ref, k, np.array([149.0, 151.0]), kind=ft.FT_BANK_LIST)
        top = c.toplist(0, k)
    assert len(top) == min(n, k)
    assert all(t.s64 == s64[t.index] for t in top)
    assert [t.index for t in top] == list(oracle.toplist(s64, np.zeros(n, np.int32), 1, k)[0])
