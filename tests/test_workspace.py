"""Workspace queries: what a path does not read is not asked for, and a workspace serves smaller calls.  Host arithmetic only."""
import pytest
import torch

import paper_2509_10771_amd as rx


def _mlp(dims, log_std=False):
    n = sum(i * o + o for i, o in zip(dims[:-1], dims[1:])) + (dims[-1] if log_std else 0)
    return rx.Mlp(dims, torch.zeros(n), trainable=True, has_log_std=log_std)


def _bytes(cell, Ha, Hc, T, N):
    G, D, A, B = (4 if cell == "lstm" else 3), 8, 2, T * N
    memory = lambda H: rx.Memory(int(cell == "lstm"), D, H, torch.zeros(G * H * (D + H + 2)), trainable=True)  # noqa: E731
    z = torch.zeros
    ro = rx.Rollout(T, N, z(B, D), z(B, D), z(B, A), z(B), z(B), z(B, A), z(B, A), z(B), z(B))
    return rx.rslx_ppo_update_recurrent_workspace_bytes(memory(Ha), _mlp((Ha, 8, A), True), memory(Hc), _mlp((Hc, 8, 1)), ro,
                                                        rx.PpoCfg(minibatches=1))


@pytest.mark.parametrize("cell", ["gru", "lstm"])
@pytest.mark.parametrize("T,other", [(3, 64), (3, 124), (1, 128)])
def test_no_split_copies_where_nothing_reads_them(cell, T, other):
    """A memory of 128 beside one of another width, or for a single step, runs a launch per step, which reads fp32 weights: it asks
    for no more than the next wider memory."""
    assert _bytes(cell, 124, other, T, 2) < _bytes(cell, 128, other, T, 2) < _bytes(cell, 132, other, T, 2)


@pytest.mark.parametrize("cell", ["gru", "lstm"])
def test_no_buffers_of_the_path_not_taken(cell):
    """A launch per step stores 3 H (GRU) or 4 H (LSTM) hidden-side terms per row for the backward pass, the whole-roll-out kernels
    H or none: what a further row costs lies that much below the widths around."""
    T, rows = 24, 24 * 512
    per_row = lambda H: (_bytes(cell, H, H, T, 1024) - _bytes(cell, H, H, T, 512)) / rows  # noqa: E731
    per_step = 0.5 * (per_row(124) + per_row(132))
    saved = 2 * 4 * 128 * (2 if cell == "gru" else 4)          # two memories, bytes
    assert per_row(128) <= per_step - 0.95 * saved             # 5 %: the reduction's partial sums, which step with the width


def test_gae_workspace_serves_fewer_environments():
    need = [rx.rslx_gae_workspace_bytes(24, n) for n in (1, 64, 65, 4096, 16384, 16385, 20000, 32768, 65535)]
    assert need == sorted(need)


@pytest.mark.parametrize("B,per_bucket", [(98304, 8), (262144, 16), (1 << 20, 16), (1 << 24, 16), (1 << 25, 32), (1 << 26, 32)])
def test_permutation_buckets(B, per_bucket):
    """Keys and indices of eight permutations, and two words per bucket: large ones have fewer, fuller buckets."""
    slack = 8 * 5 * 256
    assert rx.rslx_permutation_workspace_bytes(B) <= 8 * (12 * B + 8 * (B // per_bucket)) + slack
