"""List banks through LDS windows: the statistics are, bit for bit, the blocked FP32 sums at
the canonical bins -- one workgroup and many, windows that fit and templates too far apart
for one, SFT counts around the summation blocks, data gaps, weights, equal f0, large
spindowns (bins a segment long) and tables that end at the outermost track."""
import numpy as np
import pytest

import oracle
from paper_2411_18370_amd import synth

pytestmark = pytest.mark.gpu


def _blocked(power, u, bins, first):
    """[n_sft][n] canonical bins -> FP32 sums of 32 SFTs in order, added in FP64."""
    n_sft, n = bins.shape
    tot, acc = np.zeros(n), np.zeros(n, np.float32)
    for k in range(n_sft):
        val = power[k, bins[k] - first]
        acc = acc + (val if u is None else val * u[k])
        if (k + 1) % 32 == 0:
            tot, acc = tot + acc.astype(np.float64), np.zeros(n, np.float32)
    return (tot + acc.astype(np.float64)).astype(np.float32)


def _bins(t, t_ref, t_sft, v, f0, f1, sky):
    dt = t - t_ref
    g = 1.0 + ((v[:, :1] * sky[:, 0] + v[:, 1:2] * sky[:, 1]) + v[:, 2:] * sky[:, 2])
    return np.floor((f0 + f1 * dt[:, None]) * g * t_sft + 0.5).astype(np.int64)


@pytest.mark.parametrize("n,width,n_sft,f1_max,weight,gap", [
    (1, 0.02, 40, 1e-9, False, False), (511, 0.02, 31, 1e-9, False, False), (513, 0.02, 32, 1e-9, True, False),
    (3000, 0.05, 33, 1e-9, False, True), (5000, 0.3, 700, 1e-9, True, True), (700, 0.6, 500, 1e-9, False, True),
    (20000, 0.5, 200, 0.0, False, False), (2000, 0.0, 1000, 2e-9, True, True), (4097, 0.1, 300, 3e-8, False, False)])
def test_list_statistics_are_blocked_sums(ft, n, width, n_sft, f1_max, weight, gap):
    import torch
    rng = np.random.default_rng(n + n_sft)
    w = synth.tiny_bank(4, 1, 1, 1200)
    t, v = w.t_mid[:n_sft].copy(), w.v[:n_sft]
    if gap:  # blocks across a gap, a run of missing SFTs
        t[n_sft // 2:] += 3.3e5
    f0 = 150.0 + rng.uniform(0.0, 1.0, n) * width
    f1 = rng.uniform(-1.0, 0.3, n) * f1_max
    sky = synth.isotropic_sky(n, rng)
    B = _bins(t, w.t_ref, w.t_sft, v, f0, f1, sky)
    lo, hi = int(B.min()) - 40, int(B.max()) + 41
    power = rng.exponential(1.0, (n_sft, hi - lo)).astype(np.float32)
    u = rng.uniform(0.3, 1.7, n_sft).astype(np.float32) if weight else None
    s64, bad = oracle.eval_list(t, w.t_ref, w.t_sft, lo, power, u, v, f0, f1, sky)
    assert bad == -1
    want = _blocked(power, u, B, lo)
    assert np.max(np.abs(want - s64) / s64) <= 41 * 2.0 ** -24  # the bins are the oracle's
    edges = np.array([149.0, 150.0 + 0.4 * width + 1e-9, 152.0])
    with ft.Context(0, torch.cuda.current_stream().cuda_stream) as c:
        c.set_sfts([n_sft], t, w.t_sft, lo, power, u)
        c.set_velocities(v)
        for mode in (ft.FT_SUM_BLOCKED, ft.FT_SUM_PLAIN_FP32):
            stats = torch.empty(n, dtype=torch.float32, device="cuda")
            c.eval_templates(f0, f1, sky, w.t_ref, 5, edges, kind=ft.FT_BANK_LIST, stats=stats, sum_mode=mode)
            c.sync()
            got = stats.cpu().numpy()
            if mode == ft.FT_SUM_BLOCKED:
                assert np.array_equal(got, want)
            assert np.max(np.abs(got - s64) / s64) <= (n_sft + 8) * 2.0 ** -24
            best = oracle.toplist(s64, oracle.subband(f0, edges), 2, 5)
            for s in range(2):
                assert [x.index for x in c.toplist(s, 5)] == list(best[s])


def test_list_range_errors_stay_errors(ft):
    """A table one column short of some track: the same error as ever, no window read."""
    import torch
    rng = np.random.default_rng(8)
    w = synth.tiny_bank(4, 1, 1, 200)
    n = 3000
    f0, f1, sky = 150.0 + rng.uniform(0, 0.05, n), rng.uniform(-1e-9, 0, n), synth.isotropic_sky(n, rng)
    B = _bins(w.t_mid, w.t_ref, w.t_sft, w.v, f0, f1, sky)
    edges = np.array([149.0, 152.0])
    for cut_lo, cut_hi, ok in ((0, 0, True), (1, 0, False), (0, 1, False)):
        lo, hi = int(B.min()) + cut_lo, int(B.max()) + 1 - cut_hi
        power = rng.exponential(1.0, (w.t_mid.size, hi - lo)).astype(np.float32)
        with ft.Context(0, torch.cuda.current_stream().cuda_stream) as c:
            c.set_sfts(w.n_sft_per_det, w.t_mid, w.t_sft, lo, power, None)
            c.set_velocities(w.v)
            c.eval_templates(f0, f1, sky, w.t_ref, 5, edges, kind=ft.FT_BANK_LIST)
            if ok:
                assert len(c.toplist(0, 5)) == 5
            else:
                with pytest.raises(ft.FtError) as e:
                    c.toplist(0, 5)
                assert e.value.status == ft.FT_E_RANGE
