"""The FP64 re-summation of toplist candidates at the sizes where its pipeline can go wrong:
SFT counts around its register groups (8, 32, 64) and its chunks of 768, one workgroup per
candidate and one wave per candidate (toplists of more than 4096 entries), plain calls and
batches.  The sums are the oracle's bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2411_18370_amd import synth

pytestmark = pytest.mark.gpu


def _load(ft, w, weight=None):
    import torch
    c = ft.Context(0, torch.cuda.current_stream().cuda_stream)
    c.set_sfts(w.n_sft_per_det, w.t_mid, w.t_sft, w.first_bin, w.power, weight)
    c.set_velocities(w.v)
    return c


def _list_bank(w, n, seed=3):
    rng = np.random.default_rng(seed)
    return rng.uniform(w.f0[0], w.f0[-1], n), rng.uniform(-3e-10, 2e-10, n), synth.isotropic_sky(n, rng)


def _check(c, w, s64, f0, k):
    want = oracle.toplist(s64, oracle.subband(f0, w.sub_edges), 1, k)[0]
    top = c.toplist(0, k)
    assert [t.index for t in top] == list(want)
    assert all(t.s64 == s64[t.index] for t in top)


@pytest.mark.parametrize("n_sft", [1, 7, 8, 31, 32, 33, 63, 64, 65, 95, 767, 768, 769, 1536, 1537, 2400])
@pytest.mark.parametrize("weighted", [False, True])
def test_rescore_sft_counts(ft, n_sft, weighted):
    w = synth.tiny_bank(40, 1, 1, 1200)
    w.t_mid, w.v, w.power = w.t_mid[:n_sft], w.v[:n_sft], np.ascontiguousarray(w.power[:n_sft])
    w.n_sft_per_det = [n_sft]
    u = np.random.default_rng(4).uniform(0.3, 1.7, n_sft).astype(np.float32) if weighted else None
    f0, f1, sky = _list_bank(w, 90)
    s64, bad = oracle.eval_list(w.t_mid, w.t_ref, w.t_sft, w.first_bin, w.power, u, w.v, f0, f1, sky)
    assert bad == -1
    with _load(ft, w, u) as c:
        c.eval_templates(f0, f1, sky, w.t_ref, 20, w.sub_edges, kind=ft.FT_BANK_LIST)
        _check(c, w, s64, f0, 20)


@pytest.mark.parametrize("k", [4000, 5000])
def test_rescore_long_toplists(ft, k):
    w = synth.tiny_bank(40, 1, 1, 60)
    f0, f1, sky = _list_bank(w, 6000)
    s64, _ = oracle.eval_list(w.t_mid, w.t_ref, w.t_sft, w.first_bin, w.power, None, w.v, f0, f1, sky)
    with _load(ft, w) as c:
        c.eval_templates(f0, f1, sky, w.t_ref, k, w.sub_edges, kind=ft.FT_BANK_LIST)
        _check(c, w, s64, f0, k)


@pytest.mark.parametrize("k,n_per_det", [(1024, 10), (1025, 10), (1024, 400), (1025, 400)])
def test_rescore_either_way(ft, k, n_per_det):
    """The longest toplist re-summed by a workgroup each and the shortest by a wave each."""
    w = synth.tiny_bank(40, 1, 1, n_per_det)
    f0, f1, sky = _list_bank(w, 3000)
    s64, _ = oracle.eval_list(w.t_mid, w.t_ref, w.t_sft, w.first_bin, w.power, None, w.v, f0, f1, sky)
    with _load(ft, w) as c:
        c.eval_templates(f0, f1, sky, w.t_ref, k, w.sub_edges, kind=ft.FT_BANK_LIST)
        _check(c, w, s64, f0, k)


def test_rescore_batch_groups(ft):
    """Runs of 5, 768 and 1537 SFTs, toplists of 1, 4 and 11 (groups of four candidates)."""
    import torch
    w = synth.tiny_bank(30, 2, 4, 1200)
    for k in (1, 4, 11):
        runs, want = [], []
        for i, n in enumerate((5, 768, 1537)):
            sl = slice(i, i + n)
            runs.append(dict(sft_begin=i, n_sft=n, n_bins=w.n_bins, first_bin=w.first_bin, table_offset=i * w.n_bins,
                             f0_begin=0, n_f0=30, f1_begin=0, n_f1=2, sky_begin=0, n_sky=4, t_ref=w.t_ref))
            s64, bad = oracle.eval_grid(w.t_mid[sl], w.t_ref, w.t_sft, w.first_bin, np.ascontiguousarray(w.power[sl]),
                                        None, w.v[sl], w.f0, w.f1, w.sky)
            assert bad == -1
            want.append(s64)
        with ft.Context(0, torch.cuda.current_stream().cuda_stream) as c:
            c.eval_batch(runs, w.t_mid, w.v, w.t_sft, w.f0, w.f1, w.sky, k, power=w.power)
            for r, s64 in enumerate(want):
                top = c.batch_toplist(r, k)
                order = sorted(range(s64.size), key=lambda t: (-s64[t], t))[:k]
                assert [t.index for t in top] == order
                assert all(t.s64 == s64[t.index] for t in top)
