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
