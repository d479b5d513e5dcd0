"""The unit kernels at their edges, against the oracle bit for bit: word counts around a unit (256
words) and its span (320), roads of one combination (groups of four combinations cut three
times), units cut into slices (finely in batches of up to 64 units, every 8192 combinations
above), units whose roads do not fit the tables together, many one-word roads, words at an
address that is only 4-byte aligned, and words in host memory."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import BATCH_KEYS, caps_for, compare, gpu_cfg, run_batch
from tiny import stream

from paper_1312_0917_amd import _lib as L
from paper_1312_0917_amd import pipeline as P
from paper_1312_0917_amd import synth

pytestmark = pytest.mark.gpu
CFG = oracle.make_config()
OPEN = oracle.make_config(chi2_cut=2**40)  # accepts most combinations


def roads(rng, hits, tags=200):
    """One road per row of hits (hits per layer), in events of 7 roads."""
    out, tag = [], 0
    for nh in hits:
        tag = (tag + int(rng.integers(1, tags))) % 256
        h = [(l, int(rng.integers(-4096, 4096))) for l in range(5) for _ in range(int(nh[l]))]
        out.append((tag, [h[i] for i in rng.permutation(len(h))]))
    return [out[i:i + 7] for i in range(0, len(out), 7)]


def mixture(rng, n):
    """Mostly small roads, some of a single combination, some empty on a layer, some of 8 hits."""
    hits = rng.integers(1, 4, size=(n, 5))
    kind = rng.integers(0, 12, size=n)
    hits[kind < 3] = 1
    hits[kind == 3, 2] = 0
    hits[kind == 4] = 8
    return hits


def check(words, bank, cfg, where, **kw):
    ref = oracle.run(words, bank.f, bank.q, cfg)
    got, runner = run_batch(words, bank.f, bank.q, cfg, ref=ref, graph=False, **kw)
    compare(ref, got, BATCH_KEYS, where)
    return ref, runner


@pytest.mark.parametrize("n", [1, 5, 255, 256, 257, 319, 320, 321, 511, 512, 513, 575, 576, 577,
                               4095, 4096, 4097, 4161])
def test_word_counts_around_units(bank, n):
    rng = np.random.default_rng(n)
    words = stream(roads(rng, rng.integers(1, 4, size=(460, 5))))[:n]
    assert len(words) == n
    check(words, bank, CFG, f"{n} words")


KINDS = ["ones", "mixture", "one_word", "giant", "wide_tables", "quads"]


def kind_words(kind, n):
    """n = 60 roads stay within the finely sliced batches; of 1500, "mixture" and "wide_tables"
    have more than 64 units and units of more than 8192 combinations; the units of "quads" hold
    about 2000."""
    rng = np.random.default_rng(n + len(kind))
    if kind == "ones":
        hits = np.ones((n, 5), int)
    elif kind == "mixture":
        hits = mixture(rng, min(n, 900))
    elif kind == "one_word":  # roads of one word, now and then one with a combination
        hits = np.zeros((6 * n, 5), int)
        hits[np.arange(6 * n), rng.integers(0, 5, size=6 * n)] = 1
        hits[::37] = 1
    elif kind == "giant":
        hits = np.full((n // 10, 5), 8) if n < 100 else rng.integers(1, 9, size=(n // 4, 5))
    elif kind == "quads":
        hits = rng.integers(1, 5, size=(n, 5))
    else:  # 128 table entries and few combinations
        hits = np.tile([8, 8, 1, 1, 1], (n, 1))
        hits[1::2] = [1, 1, 8, 8, 2]
    return stream(roads(rng, hits))


@pytest.mark.parametrize("cfg", [CFG, OPEN], ids=["cut", "open"])
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [60, 1500])
@pytest.mark.parametrize("kept", [True, False], ids=["kept", "no_list"])
def test_road_mixtures(bank, kind, n, cfg, kept):
    check(kind_words(kind, n), bank, cfg, f"{kind} {n}", kept=kept)


@pytest.mark.parametrize("cfg", [CFG, OPEN], ids=["cut", "open"])
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [60, 1500])
def test_road_mixtures_kept_only(bank, kind, n, cfg):
    """Kept-only mode fits groups of eight combinations; its accept flags here start at 4 bytes
    past a multiple of 8."""
    words = kind_words(kind, n)
    ref = oracle.run(words, bank.f, bank.q, cfg)
    wc, rc, cc = caps_for(words, ref)
    r = P.BatchRunner(gpu_cfg(cfg), P.device_bank(bank.f, bank.q), wc, rc, cc, kept_cap=cc,
                      graph=False, kept_only=True)
    r.accept = torch.zeros(r.accept.numel() + 4, dtype=torch.uint8, device="cuda")[4:]
    assert r.accept.data_ptr() % 8 == 4
    r._calls.clear()
    r._call = r._prepared(r.word_cap)
    got = r.load(P.words_tensor(words)).run().result()
    compare(ref, got, [k for k in BATCH_KEYS if k not in ("p0", "p1", "p2", "c0", "c1", "c2",
                                                          "chi2")], f"kept only {kind} {n}")
    kept = np.asarray(ref["kept"])
    for k in ("p0", "p1", "p2", "c0", "c1", "c2", "chi2"):
        assert np.array_equal(np.asarray(ref[k])[kept], got[f"kept_{k}"].cpu().numpy()), k


def test_unaligned_and_host_words(bank):
    rng = np.random.default_rng(3)
    words = stream(roads(rng, mixture(rng, 300)))
    ref, runner = check(words, bank, CFG, "resident")
    n = len(words)
    shifted = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    shifted[1:] = P.words_tensor(words)
    assert shifted[1:].data_ptr() % 16 == 4
    host = torch.empty(n, dtype=torch.int32, pin_memory=True)
    host.numpy().view(np.uint32)[:] = words
    for where, src in (("4-byte aligned", shifted[1:]), ("host", L.svt_mapped_pointer(host))):
        runner.accept.zero_()
        torch.cuda.synchronize()
        runner.run(words=src)
        compare(ref, runner.result(), BATCH_KEYS, where)


def test_kept_only_of_sliced_units(bank):
    """Kept-only mode over sliced units: the list, its records and the best tracks."""
    rng = np.random.default_rng(9)
    words = stream(roads(rng, mixture(rng, 500)))
    ref = oracle.run(words, bank.f, bank.q, CFG)
    wc, rc, cc = caps_for(words, ref)
    r = P.BatchRunner(gpu_cfg(CFG), P.device_bank(bank.f, bank.q), wc, rc, cc, kept_cap=cc,
                      graph=False, kept_only=True)
    got = r.load(P.words_tensor(words)).run().result()
    compare(ref, got, [k for k in BATCH_KEYS if k not in ("p0", "p1", "p2", "c0", "c1", "c2",
                                                          "chi2")], "kept only")
    kept = np.asarray(ref["kept"])
    for k in ("p0", "p1", "p2", "c0", "c1", "c2", "chi2"):
        assert np.array_equal(np.asarray(ref[k])[kept], got[f"kept_{k}"].cpu().numpy()), k


def test_event_schedule_with_computed_look_back(bank, monkeypatch):
    """The event schedule's pre-pass, several groups of blocks, with every wait of its look-back
    answered by the words themselves."""
    monkeypatch.setenv("SVT_LOOKBACK_TIMEOUT_TICKS", "0")
    s = synth.make_sample("c2", bank=bank, n_events=1000)
    cfg = oracle.make_config(chi2_cut=synth.config_chi2_cut("c2"))
    ref = oracle.run(s.words, bank.f, bank.q, cfg)
    got, _ = run_batch(s.words, bank.f, bank.q, cfg, ref=ref, graph=False,
                       tune=L.make_tune(schedule=L.SVT_SCHEDULE_EVENTS))
    compare(ref, got, BATCH_KEYS, "event schedule")
