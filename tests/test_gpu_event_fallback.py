"""Input with errors in the event schedule, whose pre-pass is the one with a look-back: with every wait
answered from the words themselves the error and the sizes are those of its own counting, in batches
of several groups of pre-pass blocks."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import gpu_cfg
from tiny import stream

from paper_1312_0917_amd import _lib as L
from paper_1312_0917_amd import pipeline as P

pytestmark = pytest.mark.gpu
CFG = oracle.make_config()
HOOK = "SVT_LOOKBACK_TIMEOUT_TICKS"  # read at every launch


@pytest.mark.parametrize("n_events", [120, 520])
def test_computed_look_back_keeps_required_sizes_of_bad_input(bank, monkeypatch, n_events):
    rng = np.random.default_rng(11)
    events = []
    for e in range(n_events):
        roads = []
        for r in range(40):
            kind = rng.integers(0, 10)
            if kind == 0:    # 9 hits on layer 2: over the limit
                hits = [(l, 1) for l in range(5)] + [(2, 3)] * 8
            elif kind == 1:  # 60 words: longer than 5 x 8
                hits = [(l % 5, l) for l in range(60)]
            else:
                hits = [(l, int(rng.integers(-4096, 4096))) for l in range(5)
                        for _ in range(int(rng.integers(1, 4)))]
            roads.append((int(rng.integers(0, 200)) if r % 2 else 1 + (r % 7),
                          [hits[i] for i in rng.permutation(len(hits))]))
        events.append(roads)
    words = stream(events)
    assert len(words) > (2 * 64 if n_events > 200 else 30) * 2048
    st, nr, ne, nc, ei = oracle.count(words, CFG)
    assert st == L.SVT_ERR_HITS
    out = {}
    for mode, ticks in (("own", "20000"), ("computed", "0")):
        monkeypatch.setenv(HOOK, ticks)
        r = P.BatchRunner(gpu_cfg(CFG), P.device_bank(bank.f, bank.q), len(words), nr + 8,
                          64 * len(words), graph=False,
                          tune=L.make_tune(schedule=L.SVT_SCHEDULE_EVENTS))
        r.load(P.words_tensor(words)).run()
        torch.cuda.synchronize()
        assert r.error() == (L.SVT_ERR_HITS, ei), mode
        out[mode] = r.sizes()
        assert out[mode]["n_roads"] == nr, mode
    # the oracle stops at the first error: the combinations are compared between the two ways
    assert out["own"] == out["computed"] and out["own"]["n_combos"] > 0
