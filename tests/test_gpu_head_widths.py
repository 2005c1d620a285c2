"""The fused loss head at last hidden widths between its padded ones, for both networks and with mirrored rows, against the
oracle's own steps; widths outside its rule, which keep the per-layer launches."""
from dataclasses import replace

import pytest

from test_gpu_update import Case, check_forced_steps, rx  # noqa: F401
from workloads import WORKLOADS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("base,width,A", [("tiny", 68, 12), ("tiny", 100, 3), ("tiny", 124, 17), ("tiny", 132, 12), ("tiny", 252, 8), ("rough", 100, 12),
                                          ("tiny", 40, 12), ("tiny", 66, 12), ("tiny", 260, 12), ("rough", 98, 12)])
def test_head_between_padded_widths(rx, base, width, A):  # noqa: F811
    w = replace(WORKLOADS[base], N=50, hidden=(64, width)) if base == "tiny" else WORKLOADS[base].scaled(24)
    if base == "tiny":
        w = replace(w, A=A)
    else:
        w = replace(w, hidden=(64, width))
    check_forced_steps(rx, Case(w, 1, perturb=0.2))
