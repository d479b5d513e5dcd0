"""Units whose accepted combinations are found again from the accept flags, part by part: units of just
under and over one and two parts (4096 flags), with flags that start at any offset in a 4-byte word, in
batches that are cut finely and in batches that are not; and units of 2e5 combinations."""
import numpy as np
import pytest

import oracle
from gpu_util import BATCH_KEYS, caps_for, compare, gpu_cfg, run_batch
from tiny import stream

from paper_1312_0917_amd import pipeline as P

pytestmark = pytest.mark.gpu
CFGS = {"all": oracle.make_config(chi2_cut=2**62), "some": oracle.make_config(chi2_cut=2**17)}
KEPT = ("p0", "p1", "p2", "c0", "c1", "c2", "chi2")


def unit(big, ones):
    """Hits of the roads of 256 words: `big`, `ones` roads of a single combination, roads of one word."""
    hits = list(big) + [[1] * 5] * ones
    left = 256 - sum(map(sum, hits))
    assert left >= 0
    return hits + [[0, 1, 0, 0, 0]] * left


BIG = [[8, 8, 8, 8, 1]]                        # 4096 combinations in 33 words


def units(kind):
    out = []
    if kind == "parts":
        for lead in range(4):                  # the next unit's first combination modulo 4
            for extra in range(6):
                out += [unit([], 20 + lead), unit(BIG, extra), unit(BIG * 2, extra),
                        unit([[8, 8, 8, 7, 1]], 40)]
    else:                                      # 6 roads of 32768
        out = [unit([[8] * 5] * 6, 3), unit([], 7), unit([[8] * 5] * 6, 2)]
    return out


@pytest.mark.parametrize("cut", list(CFGS))
@pytest.mark.parametrize("kind,keep", [("parts", 16), ("parts", 96), ("giant", 3)])
def test_searched_units(bank, kind, keep, cut):
    rng = np.random.default_rng(keep)
    roads, tag = [], 0
    for hits in units(kind)[:keep]:
        for nh in hits:
            tag = (tag + int(rng.integers(1, 200))) % 256
            h = [(l, int(rng.integers(-4096, 4096))) for l in range(5) for _ in range(nh[l])]
            roads.append((tag, [h[i] for i in rng.permutation(len(h))]))
    words = stream([roads[i:i + 40] for i in range(0, len(roads), 40)])
    assert len(words) == 256 * keep
    cfg = CFGS[cut]
    ref = oracle.run(words, bank.f, bank.q, cfg)
    assert 0 < ref["n_kept"] and (cut == "all") == (ref["n_kept"] == ref["n_combos"])
    got, _ = run_batch(words, bank.f, bank.q, cfg, ref=ref, graph=False)
    compare(ref, got, BATCH_KEYS, f"{kind} {keep} {cut}")
    wc, rc, cc = caps_for(words, ref)
    r = P.BatchRunner(gpu_cfg(cfg), P.device_bank(bank.f, bank.q), wc, rc, cc, kept_cap=cc,
                      graph=False, kept_only=True)
    got = r.load(P.words_tensor(words)).run().result()
    compare(ref, got, [k for k in BATCH_KEYS if k not in KEPT], f"kept only {kind} {keep} {cut}")
    kept = np.asarray(ref["kept"])
    for k in KEPT:
        assert np.array_equal(np.asarray(ref[k])[kept], got[f"kept_{k}"].cpu().numpy()), k
