"""Inference behind memories takes the networks' weights split ahead of it: the bits of an inference call on the new states, whose workgroups
split them themselves, at widths around the column groups and contraction steps."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rx():
    import paper_2509_10771_amd as m
    m.rslx_device_check()
    return m


def _net(rx, dims, gen, log_std=False):
    parts = []
    for a, b in zip(dims[:-1], dims[1:]):
        parts += [torch.randn(a * b, generator=gen) / a ** 0.5, torch.randn(b, generator=gen) * 0.1]
    return rx.Mlp(dims, torch.cat(parts + ([0.3 * torch.randn(dims[-1], generator=gen)] if log_std else [])).cuda(), has_log_std=log_std)


@pytest.mark.parametrize("N,H,hidden,critic_hidden,A", [(4099, 64, (129,), (129,), 1), (1100, 256, (132, 1, 33), (200, 64), 12), (4100, 64, (512, 31), (64, 65, 512), 24), (2049, 128, (128, 128), (20,), 3),
                                                        (1025, 256, (256, 128), (64, 64), 12), (700, 252, (400, 200, 100), (130,) * 7, 33), (512, 36, (20,), (512, 300, 5), 64),
                                                        (511, 256, (512, 256, 128), (512, 256, 128), 12), (1000, 64, (64,), (128, 64), 12)])
@pytest.mark.parametrize("bad", [False, True])
def test_same_bits_as_inference_on_the_new_states(rx, N, H, hidden, critic_hidden, A, bad):
    gen, D = torch.Generator().manual_seed(N + H), 20
    mem = [rx.Memory(rx.CELL_GRU, D, H, ((torch.rand(3 * H * (D + H + 2), generator=gen) * 2 - 1) / H ** 0.5).cuda()) for _ in range(2)]
    actor, critic = _net(rx, (H,) + hidden + (A,), gen, True), _net(rx, (H,) + critic_hidden + (1,), gen)
    if bad:                               # weights without a split, in the first and the last layer
        actor.params[3 % (H * hidden[0])] = 2.0 ** 120
        critic.params[-2] = float("inf")
    x, states = torch.randn(N, D, generator=gen).cuda(), [(0.5 * torch.randn(N, H, generator=gen)).cuda() for _ in range(2)]
    e = lambda *s: torch.empty(*s, device="cuda")  # noqa: E731
    eps = torch.randn(N, A, generator=gen).cuda()
    a, b = (dict(actions=e(N, A), logp=e(N), values=e(N), mu=e(N, A), sigma=e(N, A)) for _ in range(2))
    ws = rx.workspace(rx.rslx_act_recurrent_workspace_bytes(mem[0], actor, mem[1], critic, N))
    rx.rslx_act_recurrent(mem[0], actor, mem[1], critic, x, x, N, states[0], states[1], None, None, None, 7, 3, eps, a["actions"], a["logp"], a["values"], a["mu"], a["sigma"], 0, ws)
    ws = rx.workspace(rx.rslx_act_workspace_bytes(actor, critic, N))
    rx.rslx_act(actor, critic, states[0], states[1], N, 7, 3, eps, b["actions"], b["logp"], b["values"], b["mu"], b["sigma"], 0, ws)
    torch.cuda.synchronize()
    for k in a:
        assert torch.equal(torch.nan_to_num(a[k], nan=0.125), torch.nan_to_num(b[k], nan=0.125)) and torch.equal(torch.isnan(a[k]), torch.isnan(b[k])), k


P, F, S = "fused_forward_packed", "fused_forward", "small_forward"


# Split weights are there from 512 rows, for all networks where the launch splits the memories' weights as well, else from 6 << 17 bytes
# of them; a network that the narrow kernel takes does not use them.
@pytest.mark.parametrize("N,H,hidden,critic_hidden,A,sites", [(4099, 64, (129,), (129,), 1, [P]), (1100, 256, (132, 1, 33), (200, 64), 12, [P]), (4100, 64, (512, 31), (64, 65, 512), 24, [P]),
                                                              (2049, 128, (128, 128), (20,), 3, [P]), (1025, 256, (256, 128), (64, 64), 12, [P, S]), (700, 252, (400, 200, 100), (130,) * 7, 33, [P]),
                                                              (512, 36, (20,), (512, 300, 5), 64, [S, P]), (511, 256, (512, 256, 128), (512, 256, 128), 12, [F]),
                                                              (1000, 64, (64,), (128, 64), 12, [S, S]), (600, 32, (256, 384), (256, 384), 12, [P]), (600, 32, (256, 352), (256, 352), 12, [F])])
def test_which_networks_take_split_weights(rx, N, H, hidden, critic_hidden, A, sites):
    rx.rslx_trace_begin(32)
    test_same_bits_as_inference_on_the_new_states(rx, N, H, hidden, critic_hidden, A, False)
    ran = [r[0] for r in rx.rslx_trace_end() if r[0] in (P, F, S)]
    assert ran[:len(sites)] == sites and P not in ran[len(sites):]                # behind them: act() on the new states
