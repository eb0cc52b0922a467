"""Batch runs with a local bank: f0 chunks of 5 and 8 with idle slots, one and several
workgroups of (f1, sky) pairs, SFT counts around the summation blocks, tables that end at
the outermost track (blocks at canonical bins), spindowns that move most of a window.  The
statistics equal a plain call's bit for bit, the toplists are the oracle's, and a table too
narrow by one column is a range error."""
import numpy as np
import pytest

import oracle
from paper_2411_18370_amd import synth

pytestmark = pytest.mark.gpu


def _patch(rng, n, radius):
    c = synth.isotropic_sky(1, rng)[0]
    s = c + rng.normal(size=(n, 3)) * radius
    return s / np.linalg.norm(s, axis=1, keepdims=True)


def _batch(shapes, tight, seed=5, f1_lo=-1e-9):
    pool = synth.campaign(1, seed=seed, n_pool=1300, n_sft_range=(80, 600))
    rng = np.random.default_rng(seed)
    T = pool.t_sft
    f0s, f1s, skys, runs, tables = [], [], [], [], []
    off = n0 = n1 = ns = 0
    for nf0, nf1, nsk, nsft in shapes:
        begin = int(rng.integers(0, len(pool.t_mid) - nsft + 1))
        sl = slice(begin, begin + nsft)
        t_ref = float(pool.t_mid[begin])
        f0 = float(rng.uniform(100.0, 300.0)) + np.arange(nf0) / T
        f1 = np.linspace(f1_lo, 0.0, nf1) if nf1 > 1 else np.array([-3e-10])
        sky = _patch(rng, nsk, 0.01)
        i, j, s = (x.ravel() for x in np.meshgrid(np.arange(nf0), np.arange(nf1), np.arange(nsk), indexing="ij"))
        B = oracle.bins_list(pool.t_mid[sl], t_ref, T, pool.v[sl], f0[i], f1[j], sky[s])
        lo, hi = int(B.min()) - (0 if tight else 9), int(B.max()) + (0 if tight else 9)
        runs.append(dict(sft_begin=begin, n_sft=nsft, first_bin=lo, n_bins=hi - lo + 1, table_offset=off, f0_begin=n0,
                         n_f0=nf0, f1_begin=n1, n_f1=nf1, sky_begin=ns, n_sky=nsk, t_ref=t_ref))
        tables.append(rng.exponential(2.0, (nsft, hi - lo + 1)).astype(np.float32))
        f0s.append(f0), f1s.append(f1), skys.append(sky)
        off += tables[-1].size
        n0, n1, ns = n0 + nf0, n1 + nf1, ns + nsk
    return pool, runs, tables, np.concatenate(f0s), np.concatenate(f1s), np.concatenate(skys)


FIVES = [(1, 1, 1, 1), (5, 11, 16, 517), (5, 60, 5, 100), (4, 3, 7, 31), (10, 2, 33, 32), (5, 7, 9, 1200)]
EIGHTS = [(8, 3, 16, 33), (16, 5, 13, 300), (31, 1, 48, 65), (7, 2, 9, 96), (24, 9, 29, 700)]


def _key(top):
    return [(t.index, t.s32, t.s64) for t in top]


@pytest.mark.parametrize("f1_lo", [-1e-9, -1e-8])
@pytest.mark.parametrize("tight", [False, True])
@pytest.mark.parametrize("shapes", [FIVES, EIGHTS], ids=["chunk5", "chunk8"])
def test_local_runs_match_plain_calls(ft, shapes, tight, f1_lo):
    import torch
    pool, runs, tables, f0, f1, sky = _batch(shapes, tight, f1_lo=f1_lo)
    k = 400
    power = np.concatenate([t.ravel() for t in tables])
    with ft.Context(0, torch.cuda.current_stream().cuda_stream) as c:
        for use_graph in (0, 1, 1):
            c.eval_batch(runs, pool.t_mid, pool.v, pool.t_sft, f0, f1, sky, k, power=power, use_graph=use_graph)
            tops = [c.batch_toplist(r, k) for r in range(len(runs))]
            if use_graph == 0:
                first = [_key(t) for t in tops]
            assert [_key(t) for t in tops] == first
        for R, table, top in zip(runs, tables, tops):
            sl = slice(R["sft_begin"], R["sft_begin"] + R["n_sft"])
            rf0 = f0[R["f0_begin"]:R["f0_begin"] + R["n_f0"]]
            rf1 = f1[R["f1_begin"]:R["f1_begin"] + R["n_f1"]]
            rsky = sky[R["sky_begin"]:R["sky_begin"] + R["n_sky"]]
            c.set_sfts([R["n_sft"]], pool.t_mid[sl], pool.t_sft, R["first_bin"], table)
            c.set_velocities(pool.v[sl])
            c.eval_templates(rf0, rf1, rsky, R["t_ref"], k, np.array([rf0[0] - 1.0, rf0[-1] + 1.0]))
            assert _key(top) == _key(c.toplist(0, k)), R
            s64, bad = oracle.eval_grid(pool.t_mid[sl], R["t_ref"], pool.t_sft, R["first_bin"], table, None, pool.v[sl],
                                        rf0, rf1, rsky)
            assert bad == -1
            assert [t.index for t in top] == sorted(range(s64.size), key=lambda t: (-s64[t], t))[:k]


@pytest.mark.parametrize("side", ["low", "high"])
def test_local_range_error(ft, side):
    import torch
    pool, runs, tables, f0, f1, sky = _batch(FIVES, True)
    power = np.concatenate([t.ravel() for t in tables])
    bad = [dict(R) for R in runs]
    if side == "low":
        bad[1]["first_bin"] += 1
    else:
        bad[1]["n_bins"] -= 1
    with ft.Context(0, torch.cuda.current_stream().cuda_stream) as c:
        c.eval_batch(bad, pool.t_mid, pool.v, pool.t_sft, f0, f1, sky, 5, power=power)
        with pytest.raises(ft.FtError) as e:
            c.batch_toplist(0, 5)
        assert e.value.status == ft.FT_E_RANGE
        c.eval_batch(runs, pool.t_mid, pool.v, pool.t_sft, f0, f1, sky, 5, power=power)
        assert len(c.batch_toplist(1, 5)) == 5
