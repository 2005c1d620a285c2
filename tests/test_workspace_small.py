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


@pytest.mark.parametrize("D,hidden", [(256, (256, 256, 256)), (235, (256, 256, 128)), (256, (256, 128))])
def test_update_workspace_serves_fewer_rows_of_wide_networks(D, hidden):
    """Their line lies at fewer rows."""
    z, A = torch.zeros, 12
    need = []
    for n in range(16, 2049, 16):
        ro = rx.Rollout(1, n, z(n, D), z(n, D), z(n, A), z(n), z(n), z(n, A), z(n, A), z(n), z(n))
        need.append(rx.rslx_ppo_update_workspace_bytes(_mlp((D,) + hidden + (A,), True), _mlp((D,) + hidden + (1,)), ro, rx.PpoCfg(minibatches=1)))
    assert need == sorted(need)


@pytest.mark.parametrize("hidden,line", [((128, 128), 6144), ((256, 256, 128), 4096)])
def test_regression_workspace_serves_fewer_rows(hidden, line):
    need = [rx.rslx_bc_update_workspace_bytes(_mlp((48,) + hidden + (12,)), None, n, rx.BcCfg(minibatches=1)) for n in (16, line - 1, line, line + 1, line + 64, 2 * line)]
    assert need == sorted(need)


@pytest.mark.parametrize("cell,H,D", [(0, 128, 48), (0, 256, 513), (1, 64, 20), (1, 256, 235)])
def test_recurrent_inference_query_grows_with_the_environments(cell, H, D):
    """Also over the line from which the split weights of the memories are held."""
    G = 4 if cell == rx.CELL_LSTM else 3
    mem = rx.Memory(cell, D, H, torch.zeros(G * H * (D + H + 2)))
    net = rx.Mlp((H, 64, 1), torch.zeros(H * 64 + 64 + 64 + 1))
    rows = [1, 64, 1000, 1023, 1024, 1025, 2048, 2049, 4096, 8192, 16384, 32767, 32768, 65536]
    for query in (lambda n: rx.rslx_memory_step_workspace_bytes(mem, n), lambda n: rx.rslx_act_recurrent_workspace_bytes(mem, net, mem, net, n)):
        sizes = [query(n) for n in rows]
        assert sizes == sorted(sizes)


@pytest.mark.parametrize("H,D", [(64, 129), (128, 300), (256, 600)])
def test_no_split_weights_for_a_gru_whose_inputs_stay_apart(H, D):
    """Its step splits its weights itself: a row more costs the same on both sides of the line to the step on split operands."""
    mem = rx.Memory(rx.CELL_GRU, D, H, torch.zeros(3 * H * (D + H + 2)))
    line = (1 << 18) // H
    below, at, above = (rx.rslx_memory_step_workspace_bytes(mem, n) for n in (line - 64, line, line + 64))
    assert above - at == at - below
