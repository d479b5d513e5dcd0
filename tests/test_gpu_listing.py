"""The combine stage's list, for tables and capacities that the generator's batches do not have."""
import numpy as np
import pytest
import torch

from paper_1312_0917_amd import _lib as L
from paper_1312_0917_amd import pipeline as P

pytestmark = pytest.mark.gpu


def expected(nh):
    """ncombo, combo_begin, combo_road, combo_hits of roads with hits nh (n, 5), by definition."""
    nh = np.asarray(nh, np.int64)
    n = nh.prod(1)
    begin = np.cumsum(n) - n
    road = np.repeat(np.arange(len(nh)), n)
    k = np.arange(int(n.sum())) - begin[road]
    hits = np.zeros(len(k), np.int64)
    for l in range(4, -1, -1):  # layer 0 most significant
        hits |= (k % nh[road, l]) << (4 * l)
        k = k // nh[road, l]
    return n, begin, road, hits


def combine(nh, cap=None, only=None):
    """svt_combine over a table that the caller filled; `cap`: the capacity it states."""
    nh = np.asarray(nh, np.int64)
    n, begin, road, hits = expected(nh)
    total = int(n.sum())
    table = P._alloc_roads(len(nh), "cuda")
    packed = sum(nh[:, l] << (4 * l) for l in range(5))
    table["nhits"].copy_(torch.from_numpy(packed.astype(np.uint32).view(np.int32)))
    got_road = torch.full((total,), -1, dtype=torch.int32, device="cuda")
    got_hits = torch.full((total,), -1, dtype=torch.int32, device="cuda")
    d_n = torch.zeros(1, dtype=torch.int64, device="cuda")
    err = torch.full((1,), -1, dtype=torch.int64, device="cuda")
    work = P._ws(L.svt_combine_workspace(len(nh)), "cuda")
    st = L.svt_combine(table, len(nh), L.make_config(), None if only == "hits" else got_road,
                       None if only == "road" else got_hits, total if cap is None else cap, d_n,
                       err, work)
    assert st == L.SVT_OK
    torch.cuda.synchronize()
    assert int(d_n) == total and int(err) == -1
    assert np.array_equal(table["ncombo"][:len(nh)].cpu().numpy(), n)
    assert np.array_equal(table["combo_begin"][:len(nh)].cpu().numpy(), begin)
    if only != "hits":
        assert np.array_equal(got_road.cpu().numpy(), road)
    if only != "road":
        assert np.array_equal(got_hits.cpu().numpy(), hits)


@pytest.mark.parametrize("only", [None, "road", "hits"])
@pytest.mark.parametrize("cap", [None, 10**7, 2**40, 2**63 - 1])
def test_the_capacity_may_be_any_size(cap, only):
    """A caller's capacity bounds the list and does not shape the launch: 2^63 - 1 says "no bound"."""
    combine(np.random.default_rng(1).integers(1, 4, size=(500, 5)), cap, only)


@pytest.mark.parametrize("n,cap", [(5000, None), (5000, 8192 * 2048), (5000, 8192 * 2048 + 1),
                                   (17000, None)])
def test_a_workgroup_per_tile_or_tiles_in_turn(n, cap):
    """2500 tiles of 2048 combinations at the largest capacity with a workgroup each and one above it,
    and 8500 tiles, more than the workgroups that take them in turn."""
    combine(np.full((n, 5), 4), cap)


@pytest.mark.parametrize("only", [None, "road", "hits"])
def test_tables_with_up_to_15_hits_on_a_layer(only):
    """A table that the caller filled may hold whatever 4 bits a layer can: 15^5 combinations a road."""
    nh = np.random.default_rng(2).integers(1, 16, size=(24, 5))
    nh[3], nh[11], nh[17] = 15, [9, 15, 15, 15, 1], [1, 15, 9, 1, 15]
    combine(nh, None, only)


def sparse(n, every, rng):
    """n roads of which one in `every` has combinations, the first of them after a run without."""
    nh = np.zeros((n, 5), np.int64)
    nh[:, 2] = 1
    at = np.arange(every - 1, n, every)
    nh[at] = rng.integers(1, 5, size=(len(at), 5))
    return nh


@pytest.mark.parametrize("n", [512, 513, 767, 768, 769, 1025, 70000, 300001])
@pytest.mark.parametrize("every", [500, 511, 513, 1000, 66000])
def test_runs_of_roads_without_combinations(n, every):
    if n >= every:
        combine(sparse(n, every, np.random.default_rng(n + every)))


def test_a_run_of_roads_without_combinations_costs_little():
    """The list of a million roads of which 200 have combinations, against that of those 200 alone: by
    steps of 512 roads it took 35 times as long, in one workgroup."""
    def best_of(nh):
        n = len(nh)
        table = P._alloc_roads(n, "cuda")
        packed = sum(nh[:, l] << (4 * l) for l in range(5))
        table["nhits"].copy_(torch.from_numpy(packed.astype(np.uint32).view(np.int32)))
        total = int(nh.prod(1).sum())
        road, hits = (torch.empty(total, dtype=torch.int32, device="cuda") for _ in range(2))
        d_n = torch.zeros(1, dtype=torch.int64, device="cuda")
        err = torch.full((1,), -1, dtype=torch.int64, device="cuda")
        work = P._ws(L.svt_combine_workspace(n), "cuda")
        times = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                L.svt_combine(table, n, L.make_config(), road, hits, total, d_n, err, work)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        assert int(err) == -1
        return min(times)
    nh = sparse(10**6, 5000, np.random.default_rng(3))
    assert best_of(nh) < 8 * best_of(nh[nh.prod(1) > 0])
