"""A workspace for more environments serves fewer, across the line up to which an update runs in one launch per step.  Host arithmetic only."""
import pytest
import torch

import paper_2509_10771_amd as rx


def _mlp(dims, log_std=False):
    n = sum(i * o + o for i, o in zip(dims[:-1], dims[1:])) + (dims[-1] if log_std else 0)
    return rx.Mlp(dims, torch.zeros(n), trainable=True, has_log_std=log_std)


@pytest.mark.parametrize("hidden,line", [((128, 128), 3072), ((256, 256, 128), 2048), ((32,), 3072)])
def test_update_workspace_serves_fewer_rows(hidden, line):
    D, A = 48, 12
    z = torch.zeros
    need = []
    for n in (16, line // 2, line - 1, line, line + 1, line + 64, 2 * line):
        ro = rx.Rollout(1, n, z(n, D), z(n, D), z(n, A), z(n), z(n), z(n, A), z(n, A), z(n), z(n))
        need.append(rx.rslx_ppo_update_workspace_bytes(_mlp((D,) + hidden + (A,), True), _mlp((D,) + hidden + (1,)), ro, rx.PpoCfg(minibatches=1)))
    assert need == sorted(need)


@pytest.mark.parametrize("hidden,line", [((128, 128), 6144), ((256, 256, 128), 4096)])
def test_regression_workspace_serves_fewer_rows(hidden, line):
    need = [rx.rslx_bc_update_workspace_bytes(_mlp((48,) + hidden + (12,)), None, n, rx.BcCfg(minibatches=1)) for n in (16, line - 1, line, line + 1, line + 64, 2 * line)]
    assert need == sorted(need)
