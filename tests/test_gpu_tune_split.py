"""Tuning and the split over SFT blocks: a tuned call is launched, and was timed, as split as
an untuned one, and a batch splits the runs whose tiles can be, whatever the others' are."""
import numpy as np
import pytest

from paper_2411_18370_amd import synth
from test_gpu_batch import _key, _plain_run

pytestmark = pytest.mark.gpu


def _ctx(ft):
    import torch
    return ft.Context(0, torch.cuda.current_stream().cuda_stream)


def _best(run, time):
    run()
    ms = []
    for _ in range(7):
        run()
        ms.append(time())
    return min(ms)


# few workgroups and many SFTs: timed unsplit, these chose tiles of 1.6 to 15 times the time
@pytest.mark.parametrize("n_f0,n_f1,n_sky,n_per_det", [(437, 3, 60, 1500), (100, 4, 20, 2500), (900, 4, 20, 1000)])
def test_tuned_grid_is_as_fast_as_untuned(ft, n_f0, n_f1, n_sky, n_per_det):
    w = synth.tiny_bank(n_f0, n_f1, n_sky, n_per_det)
    with _ctx(ft) as c:
        c.load_workload(w)

        def run(tile=0):
            c.eval_templates(w.f0, w.f1, w.sky, w.t_ref, w.k, w.sub_edges, tile=tile)
            c.sync()

        untuned = _best(run, lambda: c.info().eval_ms)
        want = _key(c.toplist(0, w.k))
        run(ft.FT_TILE_TUNE)
        tuned = _best(run, lambda: c.info().eval_ms)
        assert _key(c.toplist(0, w.k)) == want
        rep, _ = c.tune_report()
    print("tuned %.3f ms, untuned %.3f ms" % (tuned, untuned))
    assert tuned < 1.3 * untuned, rep


def test_tuned_batch_is_as_fast_as_untuned(ft):
    cp = synth.campaign(16, seed=4, n_pool=2000, n_sft_range=(200, 2000), nt_range=(1e3, 1e5), k=5)
    with _ctx(ft) as c:
        untuned = _best(lambda: c.eval_campaign(cp), c.batch_time)
        want = [_key(c.batch_toplist(r, cp.k)) for r in range(16)]
        c.eval_campaign(cp, tile=ft.FT_TILE_TUNE)
        tuned = _best(lambda: c.eval_campaign(cp), c.batch_time)
        assert [_key(c.batch_toplist(r, cp.k)) for r in range(16)] == want
    print("tuned %.3f ms, untuned %.3f ms" % (tuned, untuned))
    assert tuned < 1.5 * untuned  # 2.8 times as long, timed and launched unsplit


@pytest.mark.parametrize("use_graph", [0, 1])
@pytest.mark.parametrize("tile", [4, 16, 18])  # L5_J4_W4_K16 and L3_J3_W4_K16 are never split, L5_J4_W4_K8_O4 is
def test_runs_split_beside_whole_ones(ft, tile, use_graph):
    """Grids that are not uniform leave the asked-for tile for one that can be split."""
    cp = synth.campaign(8, seed=47, n_pool=900, n_sft_range=(100, 800), width_range=(0.01, 0.1), nt_range=(300, 5000), k=5)
    rng = np.random.default_rng(1)
    for r in (1, 2, 5):
        R = cp.runs[r]
        f0 = cp.f0[R["f0_begin"]:R["f0_begin"] + R["n_f0"]]
        f0[1:-1] += rng.uniform(-0.2, 0.2, f0[1:-1].size) / cp.t_sft
    with _ctx(ft) as c:
        c.eval_campaign(cp, tile=tile, use_graph=use_graph)
        for _ in range(2 * use_graph):
            c.batch_replay()
        got = [_key(c.batch_toplist(r, cp.k)) for r in range(8)]
        assert got == [_key(_plain_run(ft, c, cp, r)[0]) for r in range(8)]
