"""svt_process_batch captured in a graph that the caller owns and replays for batches of other sizes,
with eager passes on other buffers in between: with a kept list and in kept-only mode, of units that
are cut into slices and of units that are not."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import BATCH_KEYS, compare, gpu_cfg
from test_gpu_slices import heavy_words

from paper_1312_0917_amd import _lib as L
from paper_1312_0917_amd import pipeline as P

pytestmark = pytest.mark.gpu
CFG = oracle.make_config(chi2_cut=2**14)
KEPT = ("p0", "p1", "p2", "c0", "c1", "c2", "chi2")


@pytest.mark.parametrize("schedule", [0, L.SVT_SCHEDULE_EVENTS])
@pytest.mark.parametrize("kept_only", [False, True])
@pytest.mark.parametrize("most", [2, 8], ids=["whole", "sliced"])
def test_replays_for_batches_of_other_sizes(bank, most, kept_only, schedule):
    batches = []
    for units in (300, 40, 3):  # (the first needs the largest buffers)
        words = heavy_words(units, most, np.random.default_rng(units))
        batches.append((words, oracle.run(words, bank.f, bank.q, CFG)))
    words, ref = batches[0]

    def runner():
        return P.BatchRunner(gpu_cfg(CFG), P.device_bank(bank.f, bank.q), len(words),
                             ref["n_roads"], ref["n_combos"], kept_cap=ref["n_kept"] + 1, graph=False,
                             tune=L.make_tune(schedule=schedule), kept_only=kept_only)
    r, other = runner(), runner()
    r.load(P.words_tensor(words)).run()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=r.stream):
        r.run()  # (with the runner's own flags: a kept-only pass writes kept_cap records, others more)
    torch.cuda.synchronize()
    for i in (1, 0, 2, 0, 1):
        words, ref = batches[i]
        other.load(P.words_tensor(batches[2 - i][0])).run()
        r.load(P.words_tensor(words))
        torch.cuda.synchronize()
        with torch.cuda.stream(r.stream):
            g.replay()
        got = r.result()
        where = f"batch {i}, most {most}, kept only {kept_only}, schedule {schedule}"
        compare(ref, got, [k for k in BATCH_KEYS if not kept_only or k not in KEPT], where)
        if kept_only:
            kept = np.asarray(ref["kept"])
            for k in KEPT:
                assert np.array_equal(np.asarray(ref[k])[kept], got[f"kept_{k}"].cpu().numpy()), k
    del g
