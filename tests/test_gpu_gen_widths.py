"""Generated tables at the widths and row counts where the generator's mapping of cells to
lanes changes: rows of fewer and more than 96 columns, groups of 16 and of 64 rows with
remainders, a signal at the table's edges, several signals.  Bit for bit the oracle's."""
import numpy as np
import pytest

from oracle import inject
from paper_2411_18370_amd import synth
from test_gpu_gen import _assert_tables_equal, _gen_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_sft,n_bins", [(1, 1), (15, 5), (16, 95), (17, 96), (33, 97), (64, 200), (65, 1), (200, 17),
                                          (270_000, 3)])
@pytest.mark.parametrize("signals", [0, 1, 2])
def test_generated_widths(ft, n_sft, n_bins, signals):
    if n_sft > 1000 and signals == 2:
        n_sft = 262_145
    w = synth.allsky_band(seed=31, n_sky=1, n_per_det=150)
    i = np.arange(n_sft) % w.t_mid.size
    w.t_mid = w.t_mid[i] + 1e6 * (np.arange(n_sft) // w.t_mid.size)
    w.v, w.arms, w.n_sft_per_det = w.v[i], w.arms[i], [n_sft]
    rng = np.random.default_rng(n_sft + n_bins)
    inj = [synth.injection_params(rng, 200.2, 200.2 + 1e-4, 0.5, 0.5, -1e-10, 0.0) for _ in range(signals)]
    w.first_bin = int(200.2 * w.t_sft) - n_bins // 2
    w.n_bins = n_bins
    assert w.n_sft == n_sft
    got = _gen_gpu(ft, w, 1234567, 9, inj if inj else None)
    want = inject.generate_table(1234567, 9, w.t_mid, w.t_ref, w.t_sft, w.v, w.arms, w.first_bin, n_bins, inj if inj else None)
    _assert_tables_equal(got, want)


@pytest.mark.parametrize("n_sft,n_bins,signals", [(3, 97, 1), (5, 200, 2), (2048, 9, 1), (2049, 97, 1), (2049, 3, 2),
                                                  (65_535, 2, 0), (65_536, 2, 1)])
def test_generated_row_counts(ft, n_sft, n_bins, signals):
    """The row counts where a workgroup takes 4, 16 and 64 rows."""
    test_generated_widths(ft, n_sft, n_bins, signals)
