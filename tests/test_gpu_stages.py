"""The combine, fit and select stages called on their own, against the oracle bit for bit: lists
that start at any 4-byte address, either list alone, tiles of more roads than are staged at once,
long runs of roads without combinations, and a list whose order says nothing about its roads."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import gpu_cfg
from test_gpu_units import roads
from tiny import stream

from paper_1312_0917_amd import _lib as L
from paper_1312_0917_amd import pipeline as P

pytestmark = pytest.mark.gpu
CFG = oracle.make_config(chi2_cut=2**20)


def batch(kind, rng):
    if kind == "ones":       # 2048 roads in a listing tile
        hits = np.ones((5000, 5), int)
    elif kind == "empty":    # runs of roads without combinations, longer than the staged roads
        hits = np.zeros((4000, 5), int)
        hits[:, 2] = 1
        hits[rng.integers(0, 4000, size=40)] = rng.integers(1, 5, size=(40, 5))
    else:
        hits = rng.integers(1, 4, size=(700, 5))
        hits[::50] = 8
    return stream(roads(rng, hits))


def shifted(n, dtype, off):
    """n elements that start `off` elements past an allocation's start."""
    return torch.zeros(n + off, dtype=dtype, device="cuda")[off:]


@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("kind", ["ones", "empty", "mixed"])
def test_stages_at_their_edges(bank, kind, off):
    rng = np.random.default_rng(len(kind) + off)
    words = batch(kind, rng)
    ref = oracle.run(words, bank.f, bank.q, CFG)
    n, nr, nc = len(words), ref["n_roads"], ref["n_combos"]
    cfg, dbank, w = gpu_cfg(CFG), P.device_bank(bank.f, bank.q), P.words_tensor(words)
    i32, i64 = torch.int32, torch.int64
    table = P._alloc_roads(nr, "cuda")
    coord, state = shifted(n, torch.int16, off), torch.zeros(3, dtype=i64, device="cuda")
    err = torch.zeros(1, dtype=i64, device="cuda")
    work = P._ws(max(L.svt_unpack_workspace(n), L.svt_combine_workspace(nr),
                     L.svt_select_workspace(nc)), "cuda")
    assert L.svt_unpack(w, n, cfg, table, nr, coord, state[0:1], err, work) == L.SVT_OK
    road, hits = shifted(nc, i32, off), shifted(nc, i32, off)
    for a, b in ((road, None), (None, hits)):  # either list alone, then both
        assert L.svt_combine(table, nr, cfg, a, b, nc, state[1:2], err, work) == L.SVT_OK
    same = [(road, "combo_road"), (hits, "combo_hits"), (coord, "hit_coord")]
    alone = [(t.clone(), k) for t, k in same]
    road.zero_()
    hits.zero_()
    assert L.svt_combine(table, nr, cfg, road, hits, nc, state[1:2], err, work) == L.SVT_OK
    torch.cuda.synchronize()
    assert state[:2].tolist() == [nr, nc] and int(err) == -1
    for t, k in same + alone:
        assert np.array_equal(t.cpu().numpy().astype(np.int64) & 0xFFFFFFFF,
                              np.asarray(ref[k]).astype(np.int64) & 0xFFFFFFFF), k
    # the list in order, and shuffled over the whole table
    for order in (np.arange(nc), rng.permutation(nc)):
        o = torch.from_numpy(order).cuda()
        lr, lh = shifted(nc, i32, off), shifted(nc, i32, off)
        lr.copy_(road[o])
        lh.copy_(hits[o])
        rec = {k: shifted(nc, i64 if k == "chi2" else i32, off)
               for k in ("p0", "p1", "p2", "c0", "c1", "c2", "chi2")}
        assert L.svt_fit(dbank, cfg, table, nr, coord, n, lr, lh, nc, rec, err) == L.SVT_OK
        for k, t in rec.items():
            assert np.array_equal(t.cpu().numpy(), np.asarray(ref[k])[order]), k
    # back in order for the selection
    inv = torch.from_numpy(np.argsort(order)).cuda()
    rec = {k: (v2 := shifted(nc, v.dtype, off)).copy_(v[inv]) for k, v in rec.items()}
    accept, best = shifted(nc, torch.uint8, off), P._alloc_best(nr, "cuda")
    kept = torch.zeros(nc, dtype=i64, device="cuda")
    assert L.svt_select(cfg, table, nr, road, rec, nc, accept, best, kept, nc, state[2:3], err,
                        work) == L.SVT_OK
    nk = int(state[2])
    assert int(err) == -1 and nk == ref["n_kept"]
    assert np.array_equal(accept.cpu().numpy(), np.asarray(ref["accept"]))
    assert np.array_equal(kept[:nk].cpu().numpy(), np.asarray(ref["kept"]))
    for k in ("k", "p0", "p1", "p2", "chi2"):
        assert np.array_equal(best[k].cpu().numpy()[:nr], np.asarray(ref[f"best_{k}"])), k
    assert np.array_equal(best["n_accept"].cpu().numpy()[:nr], np.asarray(ref["best_nacc"]))
