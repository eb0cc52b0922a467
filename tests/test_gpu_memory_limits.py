"""Calls under a limit on the context's device memory (FT_FAULT=budget:<bytes>, read once a
process, so every case is a script of its own): what a failed call leaves behind."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEAD = """
import numpy as np, torch
from paper_2411_18370_amd import fasttracks as ft, synth
def refused(status, call):
    try:
        call()
    except ft.FtError as e:
        assert e.status == status, e
    else:
        raise AssertionError("accepted")
"""


def _run(ft, budget, body):
    env = dict(os.environ, FT_FAULT="budget:%d" % budget)
    r = subprocess.run([sys.executable, "-c", HEAD + body], cwd=ROOT, env=env, capture_output=True, text=True, timeout=90)
    assert r.returncode == 0, r.stdout[-500:] + r.stderr[-3000:]


def test_failed_batch_leaves_nothing_to_replay(ft):
    """The failed call has freed buffers that the captured graph before it refers to."""
    _run(ft, 64 << 20, """
small = synth.campaign(4, seed=1, n_pool=300, n_sft_range=(40, 100), nt_range=(1000, 2000), k=3)
large = synth.campaign(40, seed=2, n_pool=2000, n_sft_range=(1500, 2000), nt_range=(1000, 2000), k=3)
with ft.Context(0) as c:
    c.eval_campaign(small, use_graph=1)
    before = [[t.index for t in c.batch_toplist(r, 3)] for r in range(4)]
    c.batch_replay()
    assert [[t.index for t in c.batch_toplist(r, 3)] for r in range(4)] == before
    refused(ft.FT_E_NOMEM, lambda: c.eval_campaign(large))
    refused(ft.FT_E_STATE, c.batch_replay)
    refused(ft.FT_E_STATE, lambda: c.batch_toplist(0, 3))
    refused(ft.FT_E_STATE, lambda: c.batch_labels(9.5, 4))
    c.eval_campaign(small, use_graph=1)
    c.batch_replay()
    assert [[t.index for t in c.batch_toplist(r, 3)] for r in range(4)] == before
""")


def test_failed_evaluation_ends_the_one_before(ft):
    """Its buffers may be gone; a bank that is refused for what it holds leaves it whole."""
    _run(ft, 64 << 20, """
w = synth.tiny_bank(40, 1, 1, 20)
def bank(n):
    rng = np.random.default_rng(n)
    return rng.uniform(150.0, 150.02, n), rng.uniform(-1e-9, 0, n), synth.isotropic_sky(n, rng)
edges = np.array([149.0, 151.0])
with ft.Context(0) as c:
    c.set_sfts(w.n_sft_per_det, w.t_mid, w.t_sft, w.first_bin, w.power, None)
    c.set_velocities(w.v)
    def ev(n, k=4):
        f0, f1, sky = bank(n)
        c.eval_templates(f0, f1, sky, w.t_ref, k, edges, kind=ft.FT_BANK_LIST)
    def tops():
        return [t.index for t in c.toplist(0, 4)], c.toplist_number_count(0, 4)[0].tolist()
    ev(2000)
    before = tops()
    f0, f1, sky = bank(300000)
    f0[0] = np.nan
    refused(ft.FT_E_INVALID, lambda: c.eval_templates(f0, f1, sky, w.t_ref, 4, edges, kind=ft.FT_BANK_LIST))
    assert tops() == before
    many = np.linspace(149.0, 151.0, 301)
    f0, f1, sky = bank(200000)
    refused(ft.FT_E_NOMEM, lambda: c.eval_templates(f0, f1, sky, w.t_ref, 65536, many, kind=ft.FT_BANK_LIST))
    refused(ft.FT_E_STATE, lambda: c.toplist(0, 4))
    refused(ft.FT_E_STATE, lambda: c.toplist_number_count(0, 4))
    ev(2000)
    assert tops() == before
""")


LIST = """
w = synth.tiny_bank(40, 1, 1, 20)
edges = np.array([149.0, 151.0])
def bank(seed, n=200000):
    rng = np.random.default_rng(seed)
    return rng.uniform(150.0, 150.02, n), rng.uniform(-1e-9, 0, n), synth.isotropic_sky(n, rng)
def top(c, b):
    c.eval_templates(*b, w.t_ref, 4, edges, kind=ft.FT_BANK_LIST)
    return [(t.index, t.s64) for t in c.toplist(0, 4)]
def load(c):
    c.set_sfts(w.n_sft_per_det, w.t_mid, w.t_sft, w.first_bin, w.power, None)
    c.set_velocities(w.v)
"""


@pytest.mark.parametrize("mb", [14, 18, 64])
def test_list_without_room_for_a_second_copy(ft, mb):
    """200,000 templates take 8 MB a copy; the checks of a bank are the same either way."""
    _run(ft, mb << 20, LIST + """
import oracle
want = []
for s in (1, 2, 3):
    s64, bad = oracle.eval_list(w.t_mid, w.t_ref, w.t_sft, w.first_bin, w.power, None, w.v, *bank(s))
    want.append([(i, s64[i]) for i in oracle.toplist(s64, oracle.subband(bank(s)[0], edges), 1, 4)[0]])
with ft.Context(0) as c:
    load(c)
    assert [top(c, bank(s)) for s in (1, 2)] == want[:2]
    b = bank(3)
    b[2][777] *= 1.1
    refused(ft.FT_E_INVALID, lambda: top(c, b))
    assert [(t.index, t.s64) for t in c.toplist(0, 4)] == want[1]
    assert top(c, bank(3)) == want[2]
""")


def test_scratch_is_given_back_to_what_needs_it(ft):
    """The block sums a split grid keeps (15 MB) make way for a table, a bank and a batch."""
    _run(ft, 40 << 20, LIST + """
def grid(c):
    f0 = 150.0 + np.arange(200) / 1800.0
    sky = synth.isotropic_sky(100, np.random.default_rng(4))
    f1 = np.linspace(-1e-9, 0, 3)
    rng = np.random.default_rng(5)
    t = np.sort(synth.EPOCH + 1800.0 * rng.choice(2400, 2000, replace=False) + 900.0)
    v = synth.detector_velocity(t, synth.DETECTORS[0])
    vm = float(np.max(np.linalg.norm(v, axis=1)))
    first, nb = synth.table_range(f0[0], f0[-1], f1[0], f1[-1], t[0] - synth.EPOCH, t[-1] - synth.EPOCH, vm, 1800.0)
    c.set_sfts([2000], t, 1800.0, first, np.ones((2000, nb), np.float32))
    c.set_velocities(v)
    c.eval_templates(f0, f1, sky, synth.EPOCH, 4, np.array([149.0, 151.0]))
    c.toplist(0, 4)
with ft.Context(0) as c:
    grid(c)
    n = 2000
    rng = np.random.default_rng(6)
    t = np.sort(synth.EPOCH + 1800.0 * rng.choice(2400, n, replace=False) + 900.0)
    c.set_sfts([n], t, 1800.0, 270000, np.ones((n, 3500), np.float32))  # 28 MB
    c.set_velocities(synth.detector_velocity(t, synth.DETECTORS[0]))
with ft.Context(0) as c:
    grid(c)
    load(c)
    top(c, bank(1, 450000))  # 18 MB, with its statistics 22
with ft.Context(0) as c:
    grid(c)
    cp = synth.campaign(8, seed=2, n_pool=2000, n_sft_range=(1900, 2000), nt_range=(1000, 2000), k=3)
    c.eval_campaign(cp)
    c.batch_toplist(0, 3)
""")


def test_number_counts_of_a_bank_that_is_gone(ft):
    """Evaluations refused after their bank was uploaded (lists have no sky-dependent weights)
    free the last one's buffers where theirs need more: its toplists stay, its number counts
    can be read as long as its bank is there."""
    _run(ft, 1 << 40, LIST + """
def counts(c):
    return c.toplist_number_count(0, 4)[0].tolist()
def fail(c, seed, n):
    refused(ft.FT_E_UNSUPPORTED, lambda: c.eval_templates(*bank(seed, n), w.t_ref, 4, edges, kind=ft.FT_BANK_LIST,
                                                          weights=ft.FT_WEIGHTS_SKY))
with ft.Context(0) as c:
    load(c)
    want = top(c, bank(1, 2000))
    nc = counts(c)
    fail(c, 2, 3000)  # beside the evaluated bank, which stays
    assert counts(c) == nc
    fail(c, 3, 9000)  # into the evaluated bank's buffers, which are too small
    refused(ft.FT_E_STATE, lambda: counts(c))
    assert [(t.index, t.s64) for t in c.toplist(0, 4)] == want
    assert top(c, bank(1, 2000)) == want and counts(c) == nc
    c.eval_templates(w.f0, w.f1, w.sky, w.t_ref, 4, edges)
    nc = counts(c)
    assert len(nc) == 4
    fail(c, 4, 20000)
    fail(c, 5, 50000)
    refused(ft.FT_E_STATE, lambda: counts(c))
    assert len(c.toplist(0, 4)) == 4
""")
