"""How kernels read the error word, from their sources.  A kernel that reports errors changes the
word while its own workgroups start; if each wave of a workgroup read the word for itself, some could
leave at once and the others go on, through barriers and over LDS that the missing waves never wrote."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1312_0917_amd", "csrc")


def kernels():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        for m in re.finditer(r"__global__[^;{]*?\b(k_\w+)\s*\(", text):
            at = text.index("{", m.end())
            depth, end = 0, at
            for end in range(at, len(text)):
                depth += {"{": 1, "}": -1}.get(text[end], 0)
                if depth == 0:
                    break
            yield m.group(1), text[at:end]


KERNELS = dict(kernels())


def test_the_kernels_are_found():
    for k in ("k_unit_keep", "k_unit_fit", "k_fit_events", "k_scan", "k_best_finalize"):
        assert k in KERNELS


@pytest.mark.parametrize("name", sorted(KERNELS))
def test_reporting_kernels_with_barriers_read_the_word_once_per_workgroup(name):
    body = KERNELS[name]
    reports = "report(" in body
    barriers = re.search(r"__syncthreads\(|\bblock_\w+<|scan_column<", body)
    if not (reports and barriers):
        return
    own = re.findall(r"(?<!block_)\bhas_error\(", body)
    # (a lane may leave by itself where no barrier follows: k_best_finalize's workgroups of roads)
    after = body[body.rindex("has_error("):] if own else ""
    assert not own or not re.search(r"__syncthreads\(|\bblock_\w+<|scan_column<", after), name
