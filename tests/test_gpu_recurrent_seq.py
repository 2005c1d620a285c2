"""Memories of the width whose whole roll-out runs in one launch each way: against the oracle at row counts around that
launch's 16-row workgroups, one-step roll-outs, and weights that have no split for the bf16 matrix cores."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from test_gpu_recurrent import RCase, _call, _nets, check_forced_steps, rx  # noqa: F401
from workloads import WORKLOADS

pytestmark = pytest.mark.gpu


def _workload(N, T, cell, **kw):
    return replace(WORKLOADS["recurrent"].scaled(N), T=T, minibatches=2, hidden=(64, 32), memory_hidden=128, memory_cell=cell, **kw)


@pytest.mark.parametrize("cell", ["gru", "lstm"])
@pytest.mark.parametrize("N,T", [(2, 3), (30, 1), (34, 4), (64, 2)])
def test_whole_rollout_launch(rx, N, T, cell):
    case = RCase(_workload(N, T, cell, done_p=0.3), 1, perturb=0.1)
    # few samples per minibatch: statistics relative to their terms, as in test_recurrent_update_degenerate_shapes
    check_forced_steps(rx, case, floor=5e-2)


@pytest.mark.parametrize("cell", ["gru", "lstm"])
def test_weights_without_a_split_reach_only_their_own_unit(rx, cell):
    """A recurrent weight of 2^120 saturates the gates of one unit: the update stays finite wherever fp32 arithmetic does."""
    case = RCase(_workload(34, 2, cell, done_p=0.0), 1)
    tr = case.ref["trace"][0]
    b = tr["before"]
    w, out = case.w, []
    G, H = (4 if cell == "lstm" else 3), 128
    at = (w.Da + 1) * G * H + 5 * G * H + 7            # W_hh[5, gate 0, unit 7]
    for value in (2.0 ** 100, 2.0 ** 120):             # the first has a split
        actor = np.array(b["actor"])
        actor[at] = value
        nets = _nets(rx, w, actor, b["critic"], b["opt"])
        _call(rx, nets, case.gpu_rollout(rx, tr["envs"]), case.gpu_cfg(rx, 1, 1), 1, b["opt"]["step"])
        torch.cuda.synchronize()
        out.append([n.grads.cpu().numpy() for n in nets])
    # both saturate gate 0 of unit 7 to exactly 0 or 1, and its derivative to 0: everything else agrees
    for x, y in zip(*out):
        assert np.isfinite(x).all() and np.isfinite(y).all()
        assert np.linalg.norm(x - y) <= 1e-5 * np.linalg.norm(x)
