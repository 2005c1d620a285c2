"""One step of a memory that forms the input-side gate terms in the same launch: against float64 at input widths around its chunks, inputs
aligned to four bytes only, infinite inputs and weights, and the line to a product of its own."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rx():
    import paper_2509_10771_amd as m
    m.rslx_device_check()
    return m


def _memory(rx, cell, D, H, gen):
    G = 4 if cell == "lstm" else 3
    return rx.Memory(rx.CELL_LSTM if cell == "lstm" else rx.CELL_GRU, D, H, ((torch.rand(G * H * (D + H + 2), generator=gen) * 2 - 1) / H ** 0.5).cuda())


def _reference(m, x, state):
    """The step in float64; sums of products, so that an infinite operand gives infinities of its column and sign."""
    D, H, GH = m.in_dim, m.hidden, m.gates * m.hidden
    p, x, h = m.params.double(), x.double(), state.double()[:, :m.hidden]
    o = D * GH + GH
    gi = torch.stack([(r[:, None] * p[:D * GH].view(D, GH)).sum(0) for r in x]) if not torch.isfinite(x).all() else x @ p[:D * GH].view(D, GH)
    gi, gh = gi + p[D * GH:o], h @ p[o:o + H * GH].view(H, GH) + p[o + H * GH:]
    if m.gates == 3:
        r, z = torch.sigmoid(gi[:, :H] + gh[:, :H]), torch.sigmoid(gi[:, H:2 * H] + gh[:, H:2 * H])
        return (1 - z) * torch.tanh(gi[:, 2 * H:] + r * gh[:, 2 * H:]) + z * h
    i, f, g, u = (gi + gh).split(H, 1)
    c = torch.sigmoid(f) * state.double()[:, H:] + torch.sigmoid(i) * torch.tanh(g)
    return torch.cat([torch.sigmoid(u) * torch.tanh(c), c], 1)


def _step(rx, m, x, state):
    s = state.clone()
    ws = rx.workspace(rx.rslx_memory_step_workspace_bytes(m, x.shape[0]))
    rx.rslx_trace_begin(16)
    rx.rslx_memory_step(m, x, x.shape[0], s, None, None, None, ws)
    torch.cuda.synchronize()
    return s, [r[0] for r in rx.rslx_trace_end()]


@pytest.mark.parametrize("cell,H,N", [("gru", 64, 4099), ("gru", 192, 1400), ("gru", 256, 1025), ("lstm", 128, 6145), ("lstm", 320, 2048)])
@pytest.mark.parametrize("D", [1, 3, 4, 31, 32, 33, 64, 65, 101, 128])
@pytest.mark.parametrize("shift", [0, 1])
def test_state_against_float64(rx, cell, H, N, D, shift):
    gen = torch.Generator().manual_seed(N + D)
    m = _memory(rx, cell, D, H, gen)
    x = torch.randn(N * D + shift, generator=gen).cuda()[shift:].view(N, D)
    state = (0.5 * torch.randn(N, m.state_width, generator=gen)).cuda()
    got, sites = _step(rx, m, x, state)
    assert sites == [cell + "_split"]
    # gates of D + H terms below 2^2 each in fp32: 2^-24 of the largest partial sum per 32 terms, far below 1e-5 after the sigmoid and tanh
    assert float((got.double() - _reference(m, x, state)).abs().max()) <= 1e-5


@pytest.mark.parametrize("cell,H,N", [("gru", 128, 2049), ("lstm", 128, 6145)])
def test_line_of_the_input_width(rx, cell, H, N):
    """Up to twice the memory's width in the step's launch, beyond it in a product of its own: the same states from one column of zeros more."""
    gen = torch.Generator().manual_seed(5)
    D, m = 2 * H, _memory(rx, cell, 2 * H, H, gen)
    x, state = torch.randn(N, D, generator=gen).cuda(), (0.5 * torch.randn(N, m.state_width, generator=gen)).cuda()
    wide = rx.Memory(m.cell, D + 1, H, torch.cat([m.params[:D * m.gates * H], torch.ones(m.gates * H, device="cuda"), m.params[D * m.gates * H:]]))
    a, sa = _step(rx, m, x, state)
    b, sb = _step(rx, wide, torch.cat([x, torch.zeros(N, 1, device="cuda")], 1), state)
    assert sa == [cell + "_split"] and len(sb) == 2 and sb[1] == cell + "_split"
    assert float((a - b).abs().max()) <= 1e-5


@pytest.mark.parametrize("cell,H,N", [("gru", 64, 4099), ("lstm", 128, 6145)])
@pytest.mark.parametrize("D", [5, 48])
def test_infinite_inputs_and_weights(rx, cell, H, N, D):
    """Infinities saturate the gates of their rows, NaN stays in its row, the other rows keep their bits; an infinite weight of the last
    input gives the float64 step's values."""
    gen = torch.Generator().manual_seed(7)
    m = _memory(rx, cell, D, H, gen)
    x, state = torch.randn(N, D, generator=gen).cuda(), (0.5 * torch.randn(N, m.state_width, generator=gen)).cuda()
    clean, _ = _step(rx, m, x, state)
    bad = x.clone()
    bad[7, 3], bad[64, D - 1], bad[N - 1, 0] = float("inf"), -float("inf"), float("nan")
    got, sites = _step(rx, m, bad, state)
    assert sites == [cell + "_split"] and bool(torch.isnan(got[N - 1, :H]).all())
    keep = torch.ones(N, dtype=torch.bool, device="cuda")
    keep[[7, 64, N - 1]] = False
    assert torch.equal(got[keep], clean[keep])
    ref = _reference(m, bad[[7, 64]], state[[7, 64]])
    assert bool(torch.isfinite(ref).all()) and float((got[[7, 64]].double() - ref).abs().max()) <= 1e-5
    m.params[(D - 1) * m.gates * H + 5] = float("inf")                   # the first gate of unit 5
    got, _ = _step(rx, m, x, state)
    ref = _reference(m, x, state)
    assert bool(torch.isfinite(ref).all()) and float((got.double() - ref).abs().max()) <= 1e-5


@pytest.mark.parametrize("cell,H,N", [("gru", 64, 4099), ("lstm", 256, 2048)])
def test_inputs_that_are_the_states(rx, cell, H, N):
    """The states as inputs, the other memory's and the own: read before any of them is written."""
    gen = torch.Generator().manual_seed(9)
    S = 2 * H if cell == "lstm" else H
    own, other = (_memory(rx, cell, S, H, gen) for _ in range(2))
    state, second = ((0.5 * torch.randn(N, S, generator=gen)).cuda() for _ in range(2))
    want, _ = _step(rx, own, state.clone(), state)
    got = state.clone()
    ws = rx.workspace(rx.rslx_memory_step_workspace_bytes(own, N))
    rx.rslx_trace_begin(16)
    rx.rslx_memory_step(own, got, N, got, None, None, None, ws)
    torch.cuda.synchronize()
    assert len(rx.rslx_trace_end()) == 2                   # a product for the inputs, and the step
    assert float((got - want).abs().max()) <= 1e-5
    net = lambda A, ls: rx.Mlp((H, 8, A), torch.randn(H * 8 + 8 + 8 * A + A + ls, generator=gen).cuda(), has_log_std=ls > 0)  # noqa: E731
    actor, critic, e = net(2, 2), net(1, 0), lambda *s: torch.empty(*s, device="cuda")  # noqa: E731
    a, c = state.clone(), second.clone()
    ws = rx.workspace(rx.rslx_act_recurrent_workspace_bytes(own, actor, other, critic, N))
    rx.rslx_act_recurrent(own, actor, other, critic, c, a, N, a, c, None, None, None, 1, 1, None, e(N, 2), e(N), e(N), e(N, 2), e(N, 2), 0, ws)
    torch.cuda.synchronize()
    assert float((a.double() - _reference(own, second, state)).abs().max()) <= 1e-5
    assert float((c.double() - _reference(other, state, second)).abs().max()) <= 1e-5


@pytest.mark.parametrize("cell,H,N", [("gru", 64, 4099), ("lstm", 256, 2048)])
def test_inputs_that_are_the_own_state_keep_the_bits(rx, cell, H, N):
    """Such inputs are copied ahead of the step, which then runs as for any other input."""
    gen, S = torch.Generator().manual_seed(9), 2 * H if cell == "lstm" else H
    m, state = _memory(rx, cell, S, H, gen), (0.5 * torch.randn(N, S, generator=gen)).cuda()
    want, _ = _step(rx, m, state.clone(), state)
    ws = rx.workspace(rx.rslx_memory_step_workspace_bytes(m, N))
    rx.rslx_trace_begin(16)
    rx.rslx_memory_step(m, state, N, state, None, None, None, ws)
    torch.cuda.synchronize()
    assert [r[0] for r in rx.rslx_trace_end()] == ["copy_input", cell + "_split"] and torch.equal(state, want)


@pytest.mark.parametrize("cell,H,N", [("gru", 64, 4099), ("gru", 256, 1025), ("lstm", 128, 6145)])
def test_values_by_themselves_from_inputs_that_are_a_state(rx, cell, H, N):
    """The bootstrap values keep the bits of a full call also where the critic's inputs lie in the actor's state, which a values-only
    call does not see, or in its own; with 4-byte alignment and a width that is no multiple of four as well."""
    gen, S = torch.Generator().manual_seed(11), 2 * H if cell == "lstm" else H
    net = lambda A, ls: rx.Mlp((H, 8, A), torch.randn(H * 8 + 8 + 8 * A + A + ls, generator=gen).cuda(), has_log_std=ls > 0)  # noqa: E731
    e = lambda *s: torch.empty(*s, device="cuda")  # noqa: E731
    actor, critic, ma = net(2, 2), net(1, 0), _memory(rx, cell, 5, H, gen)
    x = torch.randn(N, 5, generator=gen).cuda()
    for D, shift in ((S, 0), (S // 2 - 1, 1)):
        mc = _memory(rx, cell, D, H, gen)
        ws = rx.workspace(rx.rslx_act_recurrent_workspace_bytes(ma, actor, mc, critic, N))
        for own in (False, True):
            a, c = ((0.5 * torch.randn(N, S, generator=gen)).cuda() for _ in range(2))
            seen = (c if own else a).view(-1)[shift:shift + N * D].view(N, D)
            alone, full = e(N), e(N)
            rx.rslx_act_recurrent(None, None, mc, critic, None, seen, N, None, c, None, None, None, 1, 1, None, None, None, alone, None, None, rx.ACT_VALUES_ONLY, ws)
            want = _reference(mc, seen, c)
            rx.rslx_act_recurrent(ma, actor, mc, critic, x, seen, N, a, c, None, None, None, 1, 1, None, e(N, 2), e(N), full, e(N, 2), e(N, 2), 0, ws)
            torch.cuda.synchronize()
            assert torch.equal(alone, full), (D, own)
            assert float((c.double() - want).abs().max()) <= 1e-5


@pytest.mark.parametrize("cell,Ha,Hc,Da,Dc,N,site", [("gru", 128, 128, 20, 261, 2049, "gru_split"), ("lstm", 128, 128, 257, 33, 4099, "lstm_split"), ("gru", 64, 64, 129, 600, 4111, "gru_split"),
                                                    ("lstm", 192, 192, 385, 400, 2732, "lstm_split"), ("gru", 256, 64, 513, 130, 4097, "gru_uneven"), ("lstm", 256, 128, 513, 20, 4097, "lstm_uneven")])
def test_memories_of_which_one_or_none_takes_its_inputs(rx, cell, Ha, Hc, Da, Dc, N, site):
    """Beyond twice a memory's width its inputs go through a product of their own and a GRU's weights are split in the step: new states of
    both memories against float64, and the bits of the step of either by itself through a values-only call."""
    gen, k = torch.Generator().manual_seed(N + Da), 2 if cell == "lstm" else 1
    net = lambda H, A, ls: rx.Mlp((H, 8, A), torch.randn(H * 8 + 8 + 8 * A + A + ls, generator=gen).cuda(), has_log_std=ls > 0)  # noqa: E731
    e = lambda *s: torch.empty(*s, device="cuda")  # noqa: E731
    ma, mc, actor, critic = _memory(rx, cell, Da, Ha, gen), _memory(rx, cell, Dc, Hc, gen), net(Ha, 2, 2), net(Hc, 1, 0)
    x, y = torch.randn(N, Da, generator=gen).cuda(), torch.randn(N, Dc, generator=gen).cuda()
    a, c = (0.5 * torch.randn(N, k * Ha, generator=gen)).cuda(), (0.5 * torch.randn(N, k * Hc, generator=gen)).cuda()
    want_a, want_c, alone, full = _reference(ma, x, a), _reference(mc, y, c), e(N), e(N)
    ws = rx.workspace(rx.rslx_act_recurrent_workspace_bytes(ma, actor, mc, critic, N))
    rx.rslx_act_recurrent(None, None, mc, critic, None, y, N, None, c, None, None, None, 1, 1, None, None, None, alone, None, None, rx.ACT_VALUES_ONLY, ws)
    rx.rslx_trace_begin(16)
    rx.rslx_act_recurrent(ma, actor, mc, critic, x, y, N, a, c, None, None, None, 1, 1, None, e(N, 2), e(N), full, e(N, 2), e(N, 2), 0, ws)
    torch.cuda.synchronize()
    assert [r[0] for r in rx.rslx_trace_end() if r[0].startswith(cell)] == [site]
    assert float((a.double() - want_a).abs().max()) <= 1e-5 and float((c.double() - want_c).abs().max()) <= 1e-5
    assert torch.equal(alone, full)
