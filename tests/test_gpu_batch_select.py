"""Selection of a batch's runs where its mapping changes: candidates by groups of waves (as
many as groups, more than 1536 SFTs) and by waves, rounds of 16 and of 4 with remainders,
256-term steps with remainders, one group a run (many small runs, toplists of one or two).
Run by run the toplists of separate calls."""
import numpy as np
import pytest

from paper_2411_18370_amd import synth
from test_gpu_batch import _key, _plain_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_runs,n_sft,n_t,k", [
    (3, 1536, 3000, 1), (3, 1537, 3000, 1), (2, 1600, 3000, 4), (2, 1600, 3000, 5), (2, 2000, 40_000, 40),
    (3, 255, 2000, 16), (3, 256, 2000, 17), (3, 257, 2000, 100), (2, 90, 5000, 512),
    (257, 40, 1000, 1), (257, 40, 1000, 2), (257, 40, 3000, 2), (257, 60, 1000, 3), (300, 1540, 200, 1), (260, 257, 300, 2)])
def test_batch_selection(ft, n_runs, n_sft, n_t, k):
    import torch
    cp = synth.campaign(n_runs, seed=n_runs + n_sft + k, n_pool=n_sft + 100, n_sft_range=(n_sft, n_sft),
                        width_range=(0.01, 0.03), nt_range=(n_t, 1.02 * n_t), k=k)
    some = range(n_runs) if n_runs < 4 else [0, n_runs // 2, n_runs - 1]
    with ft.Context(0, torch.cuda.current_stream().cuda_stream) as c:
        c.eval_campaign(cp)
        got = {r: _key(c.batch_toplist(r, k)) for r in some}
        _, max_z = c.batch_labels(8.0, n_runs)
        assert np.all(np.isfinite(max_z))
        for r in some:
            assert got[r] == _key(_plain_run(ft, c, cp, r)[0]), r
