"""A kept list that is too short, in batches whose units fall into several groups of the list
kernel's workgroups: the error and the required size, nothing written past the capacity (words of
another value lie before and after each array), and what the list holds: with records its first
kept_cap entries, in kept-only mode what it held before."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import caps_for, gpu_cfg, to_np

from paper_1312_0917_amd import _lib as L
from paper_1312_0917_amd import pipeline as P
from paper_1312_0917_amd import synth

pytestmark = pytest.mark.gpu
GUARD, FILL = 64, -77


@pytest.fixture(scope="module")
def samples(bank):
    out = {}
    for config, n_events in (("c2", 700), ("c3", 400)):
        s = synth.make_sample(config, bank=bank, n_events=n_events)
        assert len(s.words) > 2 * 256 * 256 or config == "c3", "several groups of 256 units"
        for cut in (synth.DEFAULT_CHI2_CUT, 2**40):
            out[config, cut] = (s.words, oracle.run(s.words, bank.f, bank.q,
                                                    oracle.make_config(chi2_cut=cut)))
    return out


def guarded(n, dtype):
    whole = torch.full((n + 2 * GUARD,), FILL, dtype=dtype, device="cuda")
    return whole, whole[GUARD:GUARD + n]


@pytest.mark.parametrize("kept_only", [False, True])
@pytest.mark.parametrize("cut", [synth.DEFAULT_CHI2_CUT, 2**40], ids=["cut", "open"])
@pytest.mark.parametrize("config", ["c2", "c3"])
def test_too_short_a_kept_list(samples, bank, config, cut, kept_only):
    words, ref = samples[config, cut]
    n_kept = ref["n_kept"]
    wc, rc, cc = caps_for(words, ref)
    w = P.words_tensor(words)
    for cap in (1, n_kept // 3, n_kept - 1):
        r = P.BatchRunner(gpu_cfg(oracle.make_config(chi2_cut=cut)), P.device_bank(bank.f, bank.q),
                          wc, rc, cc, kept_cap=cap, graph=False, kept_only=kept_only)
        arrays = dict(kept=guarded(cap, torch.int64))
        r.kept = arrays["kept"][1]
        if kept_only:
            for k, v in list(r.rec.items()):
                arrays[k] = guarded(cap, v.dtype)
                r.rec[k] = arrays[k][1]
        r._calls.clear()
        r._call = r._prepared(r.word_cap)
        for i in range(3):
            print(f"[kept overflow] {config} cut {cut} kept_only {kept_only} cap {cap} pass {i}",
                  flush=True)
            r.load(w).run()
            torch.cuda.synchronize()
            assert r.error() == (L.SVT_ERR_CAPACITY, 2)
            assert r.sizes()["n_kept"] == n_kept
            for k, (whole, _) in arrays.items():
                got = to_np(whole)
                want = np.full(cap, FILL)
                if not kept_only:
                    want = np.asarray(ref["kept"])[:cap].astype(np.int64)
                assert np.array_equal(got[GUARD:GUARD + cap], want), k
                assert np.all(got[:GUARD] == FILL) and np.all(got[GUARD + cap:] == FILL), k
