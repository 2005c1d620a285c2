"""The optimiser keeps the split copies of the weights current within a call: two epochs in one call return the bits of two
calls of one epoch, each of which splits the weights anew."""
import ctypes as C

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
    p = torch.cat(parts + ([torch.full((dims[-1],), -0.3)] if log_std else []))
    return rx.Mlp(dims, p.cuda(), trainable=True, has_log_std=log_std)


def _memory(rx, cell, D, H, gen):
    G = 4 if cell else 3
    return rx.Memory(cell, D, H, (torch.randn(G * H * (D + H + 2), generator=gen) / H ** 0.5).cuda(), trainable=True)


@pytest.mark.parametrize("D,hidden,memory,cell", [(48, (64, 32), 0, 0), (45, (100, 36, 20), 0, 0), (21, (9, 130), 0, 0), (48, (512, 256, 128), 0, 0),
                                                  (20, (64, 32), 128, 0), (21, (72, 40), 128, 1), (23, (40,), 44, 0), (48, (64, 32), 256, 1)])
def test_two_epochs_in_one_call_or_two(rx, D, hidden, memory, cell):
    T, N, A, M = 4, 36, 5, 2
    gen = torch.Generator().manual_seed(3)
    r = lambda *s: torch.randn(*s, generator=gen).cuda()  # noqa: E731
    obs, act, mu = r(T, N, D), r(T, N, A), r(T, N, A)
    data = (act, r(T, N), r(T, N), mu, torch.full((T, N, A), 0.7).cuda(), r(T, N), r(T, N))
    dones = (torch.rand(T, N, generator=gen) < 0.2).to(torch.uint8).cuda()
    S = memory * (2 if cell else 1)
    h0 = (r(N, max(S, 1)), r(N, max(S, 1)))
    start = int(gen.initial_seed())
    out = []
    for calls in ((2,), (1, 1)):
        g = torch.Generator().manual_seed(start + 1)
        d = memory or D
        nets = [_net(rx, (d,) + hidden + (A,), g, True), _net(rx, (d,) + hidden + (1,), g)]
        if memory:
            nets = [_memory(rx, cell, D, memory, g), nets[0], _memory(rx, cell, D, memory, g), nets[1]]
        ro = rx.Rollout(T, N, obs, obs, *data)
        step, first = C.c_int64(0), 0
        for epochs in calls:
            cfg = rx.PpoCfg(epochs=epochs, minibatches=M, seed=3, epoch_offset=first, lr=1e-2)
            stats = torch.zeros(epochs * M, rx.NSTATS, device="cuda")
            if memory:
                ws = rx.workspace(rx.rslx_ppo_update_recurrent_workspace_bytes(*nets, ro, cfg))
                rx.rslx_ppo_update_recurrent(*nets, ro, dones, h0[0], h0[1], cfg, step, stats, ws)
            else:
                ws = rx.workspace(rx.rslx_ppo_update_workspace_bytes(nets[0], nets[1], ro, cfg))
                rx.rslx_ppo_update(nets[0], nets[1], ro, cfg, None, None, step, stats, ws)
            torch.cuda.synchronize()
            first += epochs
        out.append([t for n in nets for t in (n.params, n.grads, n.adam_m, n.adam_v)] + [stats[-M:]])
    for a, b in zip(*out):
        assert torch.isfinite(a).all() and torch.equal(a, b)


@pytest.mark.parametrize("kind", ["ppo", "rnd", "bc", "recurrent", "bc_recurrent"])
def test_last_step_leaves_the_split_copies(rx, kind):
    """Nothing of a call reads the copies after its last step, so that step does not write them: the workspace behind a call of one
    step does not depend on the learning rate."""
    rec = kind.endswith("recurrent")
    T, N, A, D, H = (3 if rec else 1), 1, 4, 20, 128       # one item to permute: its scratch depends on no atomics' order
    gen = torch.Generator().manual_seed(11)
    r = lambda *s: torch.randn(*s, generator=gen).cuda()  # noqa: E731
    obs, act, mu, tg = r(T, N, D), r(T, N, A), r(T, N, A), r(T, N, A)
    ro = rx.Rollout(T, N, obs, obs, act, r(T, N), r(T, N), mu, torch.full((T, N, A), 0.7).cuda(), r(T, N), r(T, N))
    dones, h0 = torch.zeros(T, N, dtype=torch.uint8, device="cuda"), (r(N, H), r(N, H))
    seen = []
    for lr in (0.0, 0.1):
        g = torch.Generator().manual_seed(5)
        d = H if rec else D
        actor, critic = _net(rx, (d, 64, 32, A), g, True), _net(rx, (d, 64, 32, 1), g)
        ma, mc = _memory(rx, 0, D, H, g), _memory(rx, 0, D, H, g)
        rnd = rx.RndTrain(_net(rx, (D, 16, 8), g), _net(rx, (D, 16, 8), g), lr=lr) if kind == "rnd" else None
        step, stats = C.c_int64(0), torch.zeros(1, rx.NSTATS, device="cuda")
        cfg = (rx.BcCfg if kind.startswith("bc") else rx.PpoCfg)(epochs=1, minibatches=1, lr=lr)
        student = _net(rx, (d, 64, 32, A), g)
        size = dict(ppo=lambda: rx.rslx_ppo_update_workspace_bytes(actor, critic, ro, cfg), rnd=lambda: rx.rslx_ppo_update_workspace_bytes(actor, critic, ro, cfg, None, rnd),
                    bc=lambda: rx.rslx_bc_update_workspace_bytes(student, None, T * N, cfg),
                    recurrent=lambda: rx.rslx_ppo_update_recurrent_workspace_bytes(ma, actor, mc, critic, ro, cfg),
                    bc_recurrent=lambda: rx.rslx_bc_update_recurrent_workspace_bytes(ma, student, T, N, cfg))[kind]()
        ws = rx.workspace(size).zero_()
        if kind in ("ppo", "rnd"):
            rx.rslx_ppo_update(actor, critic, ro, cfg, None, rnd, step, stats, ws)
        elif kind == "bc":
            rx.rslx_bc_update(student, None, obs, None, tg, T * N, cfg, step, stats, ws)
        elif kind == "recurrent":
            rx.rslx_ppo_update_recurrent(ma, actor, mc, critic, ro, dones, h0[0], h0[1], cfg, step, stats, ws)
        else:
            rx.rslx_bc_update_recurrent(ma, student, obs, tg, dones, h0[0], T, N, cfg, step, stats, ws)
        torch.cuda.synchronize()
        trained = student if kind.startswith("bc") else actor
        seen.append((ws, trained.params.clone()))
    assert torch.equal(seen[0][0], seen[1][0]) and not torch.equal(seen[0][1], seen[1][1])
