"""Calls in the least workspace that they take, which holds their general form only (a launch per layer, steps of memories on fp32
operands): the results of a call in a workspace of the queried size, nothing written behind the least one, a byte less refused."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rx():
    import paper_2509_10771_amd as m
    m.rslx_device_check()
    return m


def _net(rx, dims, gen, log_std=False, trainable=False):
    parts = []
    for a, b in zip(dims[:-1], dims[1:]):
        parts += [torch.randn(a * b, generator=gen) / a ** 0.5, torch.randn(b, generator=gen) * 0.1]
    return rx.Mlp(dims, torch.cat(parts + ([0.3 * torch.randn(dims[-1], generator=gen)] if log_std else [])).cuda(), trainable=trainable, has_log_std=log_std)


def _both(rx, query, least, fast, call):
    """Outputs of call(workspace) in the queried and in the least workspace; `fast`: launch site of the faster form."""
    assert query > least
    sites, out = [], []
    guard = 4096
    room = torch.full((query + guard,), 0xA5, dtype=torch.uint8, device="cuda")
    for nbytes in (query, least):
        room.fill_(0xA5)
        rx.rslx_trace_begin(4096)
        out.append(call(room[:nbytes]))
        torch.cuda.synchronize()
        sites.append({r[0] for r in rx.rslx_trace_end()})
        assert bool((room[nbytes:] == 0xA5).all())
    assert fast is None or (fast in sites[0] and fast not in sites[1])
    with pytest.raises(rx.RslxError, match="workspace"):
        call(room[:least - 1])
    # two orders of summation in fp32: 2^-24 per value times the root of the terms that meet, 6144 rows at most: 5e-6
    for a, b in zip(*out):
        assert bool(torch.isfinite(a).all()) and float((a - b).norm()) <= 1e-5 * float(b.norm())


@pytest.mark.parametrize("D,hidden,mb,minibatches,least,fast", [(48, (128, 128), 96, 4, 1592728, "small_step"), (48, (256, 128), 512, 1, 8200320, "small_step"), (45, (256, 256, 128), 2064, 1, 38499976, None)])
def test_update(rx, D, hidden, mb, minibatches, least, fast):
    A, N = 12, mb * minibatches
    def call(ws):
        gen = torch.Generator().manual_seed(mb)
        actor, critic = _net(rx, (D,) + hidden + (A,), gen, True, True), _net(rx, (D,) + hidden + (1,), gen, False, True)
        r = lambda *s: torch.randn(1, N, *s, generator=gen).cuda()  # noqa: E731
        mu = 0.1 * r(A)
        ro = rx.Rollout(1, N, r(D), r(D), mu + r(A), r() - 12, r(), mu, torch.ones_like(mu), r(), r())
        stats = torch.zeros(minibatches, rx.NSTATS, device="cuda")
        rx.rslx_ppo_update(actor, critic, ro, rx.PpoCfg(epochs=1, minibatches=minibatches, lr=1e-5), None, None, ctypes.c_int64(0), stats, ws)
        torch.cuda.synchronize()
        return actor.params, critic.params, critic.grads
    z = torch.zeros
    ro = rx.Rollout(1, N, z(N, D), z(N, D), z(N, A), z(N), z(N), z(N, A), z(N, A), z(N), z(N))
    gen = torch.Generator().manual_seed(0)
    query = rx.rslx_ppo_update_workspace_bytes(_net(rx, (D,) + hidden + (A,), gen, True, True), _net(rx, (D,) + hidden + (1,), gen, False, True), ro, rx.PpoCfg(epochs=1, minibatches=minibatches))
    _both(rx, query, least, fast, call)


@pytest.mark.parametrize("D,hidden,mb,minibatches,least,fast", [(48, (128, 128), 384, 4, 2452520, "small_step"), (45, (256, 256, 128), 6144, 1, 51641664, None)])
def test_regression(rx, D, hidden, mb, minibatches, least, fast):
    A, B = 12, mb * minibatches
    cfg = rx.BcCfg(epochs=1, minibatches=minibatches, lr=1e-5)
    def call(ws):
        gen = torch.Generator().manual_seed(mb)
        student = _net(rx, (D,) + hidden + (A,), gen, False, True)
        x, y, stats = torch.randn(B, D, generator=gen).cuda(), torch.randn(B, A, generator=gen).cuda(), torch.zeros(minibatches, rx.NSTATS, device="cuda")
        rx.rslx_bc_update(student, None, x, None, y, B, cfg, ctypes.c_int64(0), stats, ws)
        torch.cuda.synchronize()
        return student.params, student.grads, stats[:, 0]
    _both(rx, rx.rslx_bc_update_workspace_bytes(_net(rx, (D,) + hidden + (A,), torch.Generator(), False, True), None, B, cfg), least, fast, call)


def _memory(rx, cell, D, H, gen):
    G = 4 if cell == "lstm" else 3
    return rx.Memory(rx.CELL_LSTM if cell == "lstm" else rx.CELL_GRU, D, H, ((torch.rand(G * H * (D + H + 2), generator=gen) * 2 - 1) / H ** 0.5).cuda())


@pytest.mark.parametrize("cell,H,D,N,least", [("gru", 256, 48, 1025, 5248256), ("lstm", 128, 235, 8192, 33554688)])
def test_step_of_a_memory(rx, cell, H, D, N, least):
    gen = torch.Generator().manual_seed(N)
    m = _memory(rx, cell, D, H, gen)
    x, state = torch.randn(N, D, generator=gen).cuda(), (0.5 * torch.randn(N, m.state_width, generator=gen)).cuda()
    def call(ws):
        s = state.clone()
        rx.rslx_memory_step(m, x, N, s, None, None, None, ws)
        return (s,)
    _both(rx, rx.rslx_memory_step_workspace_bytes(m, N), least, cell + "_split", call)


@pytest.mark.parametrize("cell,H,D,hidden,N,least,fast", [("gru", 256, 48, (256, 128), 1025, 13698564, "gru_split"), ("lstm", 128, 20, (512, 256, 128), 512, 7891200, None)])
def test_inference_behind_memories(rx, cell, H, D, hidden, N, least, fast):
    gen, A = torch.Generator().manual_seed(N), 12
    mem = [_memory(rx, cell, D, H, gen) for _ in range(2)]
    actor, critic = _net(rx, (H,) + hidden + (A,), gen, True), _net(rx, (H,) + hidden + (1,), gen)
    x, state = torch.randn(N, D, generator=gen).cuda(), [(0.5 * torch.randn(N, mem[0].state_width, generator=gen)).cuda() for _ in range(2)]
    e = lambda *s: torch.empty(*s, device="cuda")  # noqa: E731
    def call(ws):
        h, out = [s.clone() for s in state], [e(N, A), e(N), e(N), e(N, A), e(N, A)]
        rx.rslx_act_recurrent(mem[0], actor, mem[1], critic, x, x, N, h[0], h[1], None, None, None, 7, 3, None, *out, 0, ws)
        return h + out
    _both(rx, rx.rslx_act_recurrent_workspace_bytes(mem[0], actor, mem[1], critic, N), least, fast, call)


@pytest.mark.parametrize("cell,H,D,N,least", [("gru", 256, 48, 1025, 13698564), ("lstm", 256, 33, 2049, None)])
def test_values_alone_are_those_of_a_full_call(rx, cell, H, D, N, least):
    """In one workspace, whichever form it holds: the bits of the full call's values; without the actor, in the room for the critic."""
    gen, A = torch.Generator().manual_seed(N), 12
    mem = [_memory(rx, cell, D, H, gen) for _ in range(2)]
    actor, critic = _net(rx, (H, 256, 128, A), gen, True), _net(rx, (H, 256, 128, 1), gen)
    x, state = torch.randn(N, D, generator=gen).cuda(), [(0.5 * torch.randn(N, mem[0].state_width, generator=gen)).cuda() for _ in range(2)]
    e = lambda *s: torch.empty(*s, device="cuda")  # noqa: E731
    def values(ws, flags, with_actor=True):
        h, out = [s.clone() for s in state], [e(N, A), e(N), e(N), e(N, A), e(N, A)]
        rx.rslx_trace_begin(64)
        rx.rslx_act_recurrent(mem[0] if with_actor else None, actor if with_actor else None, mem[1], critic, x, x, N, h[0], h[1], None, None, None, 7, 3,
                              None, *out, flags, ws)
        torch.cuda.synchronize()
        return out[2], {r[0] for r in rx.rslx_trace_end()}
    query = rx.rslx_act_recurrent_workspace_bytes(mem[0], actor, mem[1], critic, N)
    alone = rx.rslx_act_recurrent_workspace_bytes(None, None, mem[1], critic, N)
    room = torch.empty(query, dtype=torch.uint8, device="cuda")
    for nbytes in (query, query - 1) + ((least,) if least else ()):
        full, sites = values(room[:nbytes], 0)
        assert (cell + "_split" in sites) == (nbytes == query)
        only, sites = values(room[:nbytes], rx.ACT_VALUES_ONLY)
        assert (cell + "_split" in sites) == (nbytes == query) and torch.equal(only, full)
    full, _ = values(room, 0)
    only, sites = values(room[:alone], rx.ACT_VALUES_ONLY, with_actor=False)
    assert cell + "_split" in sites and torch.equal(only, full)
