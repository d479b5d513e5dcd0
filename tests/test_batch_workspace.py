"""svt_process_batch takes a workspace of svt_batch_workspace bytes or more and refuses a smaller one on
the host, before any HIP call (the device addresses here are never used)."""
import ctypes

import pytest

from paper_1312_0917_amd import _lib as L

FAKE = 1 << 20


@pytest.mark.parametrize("schedule", [0, L.SVT_SCHEDULE_EVENTS, L.SVT_SCHEDULE_ONEPASS,
                                      L.SVT_SCHEDULE_TILES])
@pytest.mark.parametrize("caps", [(1, 1, 4), (4096, 512, 1 << 15), (1 << 21, 1 << 18, 1 << 23)])
def test_a_workspace_too_small_is_refused(caps, schedule):
    words, roads_cap, combos = caps
    lib, cfg, tune = L.load(), L.make_config(), L.make_tune(schedule=schedule)
    roads = L.svt_roads(*([FAKE] * 6))
    rec = L.svt_fitrec(*([FAKE] * 4), None, None, None)
    best = L.svt_best(*([FAKE] * 6))
    need = L.svt_batch_workspace(words, roads_cap, combos, tune)
    for size in (0, need // 2, need - 4 * words, need - 256, need - 1):
        assert lib.svt_process_batch(
            FAKE, ctypes.byref(cfg), ctypes.byref(tune), FAKE, FAKE, words, ctypes.byref(roads),
            roads_cap, ctypes.byref(rec), FAKE, combos, ctypes.byref(best), None, 0, FAKE, FAKE,
            None, FAKE, FAKE, max(size, 0), 0, None) == L.SVT_ERR_ARG, size
