"""Inference of narrow networks, 16 rows per workgroup: against float64 at rows and widths around its tiles, the line to the wider kernel,
networks of one call that take different kernels, and values-only calls bit for bit."""
import ctypes

import pytest
import torch

from oracle import rng as orng

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


def _forward(net, x):
    o, p = 0, net.params.double()
    for i, (a, b) in enumerate(zip(net.dims[:-1], net.dims[1:])):
        x = x @ p[o:o + a * b].view(a, b) + p[o + a * b:o + a * b + b]
        o += a * b + b
        if i < len(net.dims) - 2:
            x = torch.where(x > 0, x, torch.expm1(torch.clamp(x, max=0.0)))
    return x


def _act(rx, actor, critic, x, flags=0, eps=None):
    N, A = x.shape[0], actor.dims[-1]
    e = lambda *s: torch.empty(*s, device="cuda")  # noqa: E731
    out = dict(actions=e(N, A), logp=e(N), values=e(N), mu=e(N, A), sigma=e(N, A))
    ws = rx.workspace(rx.rslx_act_workspace_bytes(actor, critic, N))
    rx.rslx_trace_begin(16)
    rx.rslx_act(actor, critic, x, x, N, 7, 3, eps, out["actions"], out["logp"], out["values"], out["mu"], out["sigma"], flags, ws)
    torch.cuda.synchronize()
    return out, [r[0] for r in rx.rslx_trace_end()]


@pytest.mark.parametrize("N,D,hidden,A", [(1, 1, (1,), 1), (15, 31, (16, 20), 3), (16, 32, (128, 128), 12), (17, 33, (36, 20), 17), (33, 64, (100, 36, 20), 33), (100, 65, (128,), 64),
                                          (40, 128, (127, 129 - 1), 32), (48, 129, (128, 9), 9), (31, 235, (9, 128, 30), 4), (80, 256, (128, 128, 128), 64), (2048, 48, (128, 128), 12)])
def test_outputs_against_float64(rx, N, D, hidden, A):
    gen = torch.Generator().manual_seed(N + D)
    actor, critic = _net(rx, (D,) + hidden + (A,), gen, True), _net(rx, (D,) + hidden + (1,), gen)
    x = torch.randn(N, D, generator=gen).cuda()
    out, sites = _act(rx, actor, critic, x)
    assert sites == ["small_forward"]
    mu, v = _forward(actor, x.double()), _forward(critic, x.double())[:, 0]
    # six roundings of 2^-24 per layer and value at most, amplified by weights of unit gain: 1e-5 of the largest value is ten times that
    for got, ref in ((out["mu"], mu), (out["values"], v)):
        assert float((got.double() - ref).abs().max()) <= 1e-5 * float(ref.abs().max() + 1)
    eps = torch.from_numpy(orng.act_noise(7, 3, N, A)).cuda()
    ls = actor.params[-A:].double()
    assert float((out["actions"].double() - (out["mu"].double() + torch.exp(ls) * eps)).abs().max()) <= 1e-5
    z = (out["actions"].double() - out["mu"].double()) / torch.exp(ls)
    logp = (-0.5 * z * z - ls - 0.9189385332046727).sum(-1)
    assert float((out["logp"].double() - logp).abs().max()) <= 1e-5 * float(logp.abs().max() + 1)
    assert torch.equal(out["sigma"], out["sigma"][:1].expand(N, A)) and float((out["sigma"][0].double() - torch.exp(ls)).abs().max()) <= 1e-6
    # the critic by itself: the same bits
    alone, ws = torch.empty(N, device="cuda"), rx.workspace(rx.rslx_act_workspace_bytes(None, critic, N))
    rx.rslx_act(None, critic, None, x, N, 0, 0, None, None, None, alone, None, None, rx.ACT_VALUES_ONLY, ws)
    assert torch.equal(alone, out["values"])
    det, _ = _act(rx, actor, critic, x, rx.ACT_DETERMINISTIC)
    assert torch.equal(det["actions"], out["mu"]) and torch.equal(det["mu"], out["mu"])
    own = torch.randn(N, A, generator=gen).cuda()
    given, _ = _act(rx, actor, critic, x, 0, own)
    assert float((given["actions"] - (out["mu"] + out["sigma"] * own)).abs().max()) <= 1e-5


@pytest.mark.parametrize("N,actor_hidden,critic_hidden,want", [(2048, (128, 64), (128, 64), ["small_forward"]), (2049, (128, 64), (128, 64), ["fused_forward"]),
                                                               (64, (132, 64), (132, 64), ["fused_forward"]), (64, (132, 64), (128, 64), ["fused_forward", "small_forward"]),
                                                               (64, (64,), (132, 64), ["small_forward", "fused_forward"]), (64, (64,), (64, 32), ["small_forward", "small_forward"])])
def test_which_kernel_a_network_takes(rx, N, actor_hidden, critic_hidden, want):
    """By the network and the row count alone: beside a network that takes the other kernel, or one of another depth, the values keep
    their bits."""
    gen = torch.Generator().manual_seed(N)
    actor, critic = _net(rx, (40,) + actor_hidden + (5,), gen, True), _net(rx, (40,) + critic_hidden + (1,), gen)
    x = torch.randn(N, 40, generator=gen).cuda()
    out, sites = _act(rx, actor, critic, x)
    assert sites == want
    mu, v = _forward(actor, x.double()), _forward(critic, x.double())[:, 0]
    assert float((out["mu"].double() - mu).abs().max()) <= 1e-5 * float(mu.abs().max() + 1) and float((out["values"].double() - v).abs().max()) <= 1e-5 * float(v.abs().max() + 1)
    alone, ws = torch.empty(N, device="cuda"), rx.workspace(rx.rslx_act_workspace_bytes(None, critic, N))
    rx.rslx_act(None, critic, None, x, N, 0, 0, None, None, None, alone, None, None, rx.ACT_VALUES_ONLY, ws)
    assert torch.equal(alone, out["values"])


def _launches(rx, call):
    """Kernel nodes of a captured call (which has run once before, so that nothing is set up inside the capture)."""
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    n = ctypes.c_size_t()
    assert rx.lib.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("N", [1, 40, 2048])
@pytest.mark.parametrize("Da,actor_hidden,Dc,critic_hidden", [(40, (132, 64), 40, (128, 64)), (40, (64,), 40, (132, 64)), (48, (128, 128), 300, (128, 128)), (40, (64,), 40, (64, 32)),
                                                              (130, (20, 128, 7), 33, (128,)), (7, (5, 6, 7), 200, (9,) * 4)])
def test_networks_that_differ_run_side_by_side(rx, N, Da, actor_hidden, Dc, critic_hidden):
    gen = torch.Generator().manual_seed(N + Dc)
    actor, critic = _net(rx, (Da,) + actor_hidden + (5,), gen, True), _net(rx, (Dc,) + critic_hidden + (1,), gen)
    x, y = torch.randn(N, Da, generator=gen).cuda(), torch.randn(N, Dc, generator=gen).cuda()
    e = lambda *s: torch.empty(*s, device="cuda")  # noqa: E731
    out = dict(actions=e(N, 5), logp=e(N), values=e(N), mu=e(N, 5), sigma=e(N, 5))
    ws = rx.workspace(rx.rslx_act_workspace_bytes(actor, critic, N))
    assert _launches(rx, lambda: rx.rslx_act(actor, critic, x, y, N, 7, 3, None, out["actions"], out["logp"], out["values"], out["mu"], out["sigma"], 0, ws)) == 1
    mu, v = _forward(actor, x.double()), _forward(critic, y.double())[:, 0]
    assert float((out["mu"].double() - mu).abs().max()) <= 1e-5 * float(mu.abs().max() + 1) and float((out["values"].double() - v).abs().max()) <= 1e-5 * float(v.abs().max() + 1)
    eps = torch.from_numpy(orng.act_noise(7, 3, N, 5)).cuda()
    assert float((out["actions"].double() - (out["mu"].double() + torch.exp(actor.params[-5:].double()) * eps)).abs().max()) <= 1e-5
    alone = e(N)
    rx.rslx_act(None, critic, None, y, N, 0, 0, None, None, None, alone, None, None, rx.ACT_VALUES_ONLY, ws)
    assert torch.equal(alone, out["values"])


def test_student_beside_a_wider_teacher(rx):
    gen, N, A = torch.Generator().manual_seed(4), 100, 6
    student, teacher = _net(rx, (30, 64, A), gen), _net(rx, (50, 512, 256, 128, A), gen)
    x, y = torch.randn(N, 30, generator=gen).cuda(), torch.randn(N, 50, generator=gen).cuda()
    s, t = torch.empty(N, A, device="cuda"), torch.empty(N, A, device="cuda")
    ws = rx.workspace(rx.rslx_bc_collect_workspace_bytes(student, teacher, N))
    assert _launches(rx, lambda: rx.rslx_bc_collect(student, teacher, x, y, N, s, t, ws)) == 1
    for net, inp, got in ((student, x, s), (teacher, y, t)):
        ref = _forward(net, inp.double())
        assert float((got.double() - ref).abs().max()) <= 1e-5 * float(ref.abs().max() + 1)


def test_rows_without_a_split_leave_the_others_alone(rx):
    gen = torch.Generator().manual_seed(2)
    actor, critic = _net(rx, (48, 128, 72, 12), gen, True), _net(rx, (48, 128, 72, 1), gen)
    critic.params[:128] *= 1e-36                      # weights of input 0
    x = torch.randn(50, 48, generator=gen).cuda()
    clean, _ = _act(rx, actor, critic, x)
    bad = x.clone()
    bad[3, 5], bad[20, 5], bad[33, 0] = float("nan"), float("inf"), 2e34
    out, _ = _act(rx, actor, critic, bad)
    keep = [i for i in range(50) if i not in (3, 20, 33)]
    assert all(torch.equal(out[k][keep], clean[k][keep]) for k in out)
    assert bool(torch.isnan(out["values"][3])) and not bool(torch.isfinite(out["values"][20]))
    ref = _forward(critic, bad[33:34].double())[0, 0]
    assert abs(float(out["values"][33]) - float(ref)) <= 1e-5 * (1 + abs(float(ref)))
