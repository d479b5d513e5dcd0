"""Batches on both sides of the sizes at which the slices that a unit is cut into get longer, of heavy
roads: every output against the oracle, and no step in the time of a pass."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import BATCH_KEYS, caps_for, compare, gpu_cfg, run_batch

from paper_1312_0917_amd import pipeline as P

pytestmark = pytest.mark.gpu
CFG = oracle.make_config(chi2_cut=2**14)
KEPT = ("p0", "p1", "p2", "c0", "c1", "c2", "chi2")


def heavy_words(units, most, rng):
    """256 * units words of roads with 1 to 4 hits a layer, a twentieth of the layers `most`."""
    n = 40 * units + 8
    nh = rng.integers(1, 5, size=(n, 5))
    nh[rng.random((n, 5)) < 0.05] = most
    layer = np.repeat(np.tile(np.arange(5), n), nh.reshape(-1))
    road = np.repeat(np.arange(n), nh.sum(1))
    tag = np.cumsum(rng.integers(1, 256, n)) % 256
    words = (rng.integers(0, 8192, len(layer)) | layer << 13 | tag[road] << 16
             | ((road // 50) % 256) << 24)
    return words[:256 * units].astype(np.uint32)


@pytest.mark.parametrize("want", ["records", "list", "kept_only"])
@pytest.mark.parametrize("units", [1, 32, 33, 63, 64, 65, 128, 129, 257, 512, 513, 1024, 1025])
def test_both_sides_of_a_slice_length(bank, units, want):
    words = heavy_words(units, 8, np.random.default_rng(units))
    ref = oracle.run(words, bank.f, bank.q, CFG)
    if want != "kept_only":
        got, _ = run_batch(words, bank.f, bank.q, CFG, ref=ref, graph=False, kept=want == "list")
        compare(ref, got, BATCH_KEYS, f"{units} units, {want}")
        return
    wc, rc, cc = caps_for(words, ref)
    r = P.BatchRunner(gpu_cfg(CFG), P.device_bank(bank.f, bank.q), wc, rc, cc,
                      kept_cap=ref["n_kept"] + 1, graph=False, kept_only=True)
    got = r.load(P.words_tensor(words)).run().result()
    compare(ref, got, [k for k in BATCH_KEYS if k not in KEPT], f"{units} units, kept only")
    kept = np.asarray(ref["kept"])
    for k in KEPT:
        assert np.array_equal(np.asarray(ref[k])[kept], got[f"kept_{k}"].cpu().numpy()), k


def best_of(bank, words, want):
    """The least time of ten passes over these words, in ms."""
    _, nr, _, nc, _ = oracle.count(words, CFG)
    r = P.BatchRunner(gpu_cfg(oracle.make_config()), P.device_bank(bank.f, bank.q), len(words),
                      nr + 1, nc + 4, kept_cap=0 if want == "records" else nc, graph=False,
                      with_c=False, kept_only=want == "kept_only")
    r.load(P.words_tensor(words))
    times = []
    for _ in range(12):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(r.stream)
        for _ in range(10):
            r.run()
        b.record(r.stream)
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    return min(times)


@pytest.mark.parametrize("want", ["records", "list", "kept_only"])
def test_one_more_unit_makes_no_step(bank, want):
    """A pass over 65 units took more than twice as long as one over 64 when the slices got 16 times as
    long there."""
    for units in (32, 64, 128, 256, 512, 1024):
        few, more = (best_of(bank, heavy_words(n, 8, np.random.default_rng(7)), want)
                     for n in (units, units + 1))
        assert more < 1.5 * few, units


def giant_words(n, rng):
    """n roads of 8^5 combinations."""
    layer = np.repeat(np.tile(np.arange(5), n), 8)
    road = np.repeat(np.arange(n), 40)
    return (rng.integers(0, 8192, 40 * n) | layer << 13 | (3 * road + 1) % 256 << 16).astype(np.uint32)


@pytest.mark.parametrize("units", [1, 3, 20])
@pytest.mark.parametrize("combo_cap", [None, 10**7, 2 * 10**8])
def test_units_of_as_many_slices_as_there_can_be(bank, units, combo_cap):
    """Roads of 8^5 combinations, seven to a unit, under a capacity of their number and far above it:
    what the slices of a unit share is counted by the words as well as by the capacity."""
    n = (256 * units + 39) // 40
    words = giant_words(n, np.random.default_rng(units))
    ref = oracle.run(words, bank.f, bank.q, CFG)
    assert ref["n_combos"] == 32768 * n
    r = P.BatchRunner(gpu_cfg(CFG), P.device_bank(bank.f, bank.q), len(words), n,
                      combo_cap or ref["n_combos"], kept_cap=ref["n_kept"] + 1, graph=False)
    for _ in range(2):
        got = r.load(P.words_tensor(words)).run().result()
        compare(ref, got, BATCH_KEYS, f"{units} units, capacity {combo_cap}")
