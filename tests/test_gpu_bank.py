"""The LDS-window kernel of binary banks (eval_bank.hip) against the oracle and, bit for
bit, against the gather kernel (which the polynomial cosine mode selects): SFT counts
around its 32-SFT blocks, template counts around its workgroups and waves, bin ranges
around its row strides, data gaps that cut blocks, velocities no polynomial fits, tracks on
bin edges, weights and the number count."""
import numpy as np
import pytest

import oracle
from oracle import weighting
from paper_2411_18370_amd import synth

pytestmark = pytest.mark.gpu


def _workload(n_per_det, n_tmpl, width=0.125, trim=0, seed=51):
    w = synth.binary_band(seed=seed, n_tmpl=n_tmpl, n_per_det=n_per_det, width=width, n_sub=2)
    if trim:
        w.t_mid, w.v, w.power = w.t_mid[:-trim], w.v[:-trim], np.ascontiguousarray(w.power[:-trim])
        w.n_sft_per_det = [n_per_det, n_per_det - trim]
    return w


def _both(ft, w, k=8, weight=None, stat=0, sum_mode=0, s64=None):
    """Statistics of the bank kernel and of the gather kernel, equal bit for bit, and the
    toplists of the first against s64."""
    import torch
    out = []
    with ft.Context(0, torch.cuda.current_stream().cuda_stream) as c:
        c.set_sfts(w.n_sft_per_det, w.t_mid, w.t_sft, w.first_bin, w.power, weight)
        c.set_velocities(w.v)
        for mode in (0, 1):
            c.binary_cos_mode(mode)
            stats = torch.zeros(w.n_templates, dtype=torch.float32, device="cuda")
            c.eval_binary(w.f0, w.sky, w.ap, w.omega, w.phib, w.t_ref, k, w.sub_edges, stats=stats, statistic=stat,
                          sum_mode=sum_mode)
            tops = [[(t.index, t.s64) for t in c.toplist(j, k)] for j in range(2)]
            out.append((stats.cpu().numpy(), tops))
    assert np.array_equal(out[0][0].view(np.uint32), out[1][0].view(np.uint32))
    assert out[0][1] == out[1][1]
    if s64 is not None:
        bound = 40 * 2.0 ** -24 + 4 * w.n_sft * 2.0 ** -53
        assert np.max(np.abs(out[0][0].astype(np.float64) - s64) / np.maximum(s64, 1e-30)) <= bound
        want = oracle.toplist(s64, oracle.subband(w.f0, w.sub_edges), 2, k)
        assert [[i for i, _ in t] for t in out[0][1]] == [list(x) for x in want]
    return out[0][0]


def _oracle(w, weight=None, power=None):
    s64, bad = oracle.eval_binary(w.t_mid, w.t_ref, w.t_sft, w.first_bin, w.power if power is None else power, weight,
                                  w.v, w.f0, w.sky, w.ap, w.omega, w.phib)
    assert bad == -1
    return s64


# SFT counts 1, 31, 32, 33, 63, 64, 65 and 400 per detector (the last less one); template
# counts around a wave (64), a workgroup (512) and its multiples; widths for each row stride
# (128, 256, 512 columns) and past the widest, where the gather kernel runs either way
@pytest.mark.parametrize("n_per_det,trim,n_tmpl,width", [
    (1, 0, 1, 0.125), (16, 1, 63, 0.125), (16, 0, 64, 0.05), (17, 1, 65, 0.05), (32, 1, 511, 0.125),
    (32, 0, 512, 0.125), (33, 1, 513, 0.3), (200, 1, 1537, 0.3), (200, 0, 700, 0.062), (200, 0, 700, 0.07),
    (200, 0, 700, 0.19), (200, 0, 700, 0.42), (200, 0, 300, 0.6), (400, 1, 20_000, 0.125)])
def test_bank_kernel_shapes(ft, n_per_det, trim, n_tmpl, width):
    w = _workload(n_per_det, n_tmpl, width, trim)
    _both(ft, w, s64=_oracle(w))


@pytest.mark.parametrize("case", ["gaps", "unsorted", "rough_velocities", "half_bins", "no_orbit", "far_reference",
                                  "short_period"])
def test_bank_kernel_data(ft, case):
    """Blocks cut by week-long gaps and by times out of order; velocities that no smooth
    polynomial fits; every track on a bin edge; a_p = 0; t_ref 3 years off; periods of hours."""
    w = _workload(300, 900)
    rng = np.random.default_rng(7)
    if case == "gaps":
        w.t_mid = w.t_mid + 7 * synth.DAY * np.searchsorted([100, 117, 118, 333, 500], np.arange(600), side="right")
    elif case == "unsorted":
        order = np.concatenate([rng.permutation(150), 150 + np.arange(450)])
        w.t_mid, w.v = w.t_mid[order], w.v[order]
    elif case == "rough_velocities":
        w.v = w.v * (1.0 - 1e-2 * rng.random((600, 1)))
    elif case == "half_bins":
        w.v = np.zeros_like(w.v)
        w.ap = np.zeros_like(w.ap)
        w.f0 = (np.floor(w.f0 * w.t_sft) + 0.5) / w.t_sft
    elif case == "no_orbit":
        w.ap, w.omega = np.zeros_like(w.ap), np.zeros_like(w.omega)
    elif case == "far_reference":
        w.t_ref = w.t_ref - 3 * synth.SIDEREAL_YEAR
    elif case == "short_period":
        w.omega = w.omega * 20.0
        w.ap = w.ap / 40.0
    _both(ft, w, s64=_oracle(w))


@pytest.mark.parametrize("sum_mode", [0, 1])
def test_bank_kernel_weights_and_number_count(ft, sum_mode):
    w = _workload(150, 1300)
    u = np.random.default_rng(3).uniform(0.2, 2.0, w.n_sft).astype(np.float32)
    _both(ft, w, weight=u, sum_mode=sum_mode, s64=None if sum_mode else _oracle(w, u))
    if sum_mode == 0:
        ind = weighting.number_count_table(w.power)
        _both(ft, w, stat=ft.FT_STAT_NUMBER_COUNT, s64=_oracle(w, None, ind.astype(np.float32)))
