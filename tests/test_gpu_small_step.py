"""Optimiser steps of small networks over few rows, which run forward pass, loss and backward pass in one launch: against the oracle's
own steps at row counts around the 16 of a workgroup and widths around its tiles, on both sides of the line between this and the
launches per layer, and those launches at the sizes just above it."""
import ctypes
from dataclasses import replace

import pytest
import torch

import test_gpu_split
from test_gpu_update import Case, check_forced_steps, run_bc, rx  # noqa: F401
from workloads import WORKLOADS

pytestmark = pytest.mark.gpu


def _sites(rx, call):  # noqa: F811
    rx.rslx_trace_begin(1024)
    call()
    torch.cuda.synchronize()
    return {n[0] for n in rx.rslx_trace_end()}


@pytest.mark.parametrize("rows,Da,hidden,A", [(1, 1, (4,), 1), (15, 31, (16, 20), 3), (16, 32, (128, 128), 12), (17, 33, (36, 20), 17), (33, 45, (100, 36, 20), 5),
                                              (40, 256, (256, 256), 32), (48, 235, (250, 129), 9), (31, 129, (9, 130, 30), 4), (100, 21, (256, 1, 256), 16),
                                              (80, 20, (128, 128, 128), 31)])
def test_steps_against_the_oracle(rx, rows, Da, hidden, A):  # noqa: F811
    w = replace(WORKLOADS["tiny"], T=1, N=2 * rows, minibatches=2, Da=Da, Dc=Da, A=A, hidden=hidden)
    case = Case(w, 1, perturb=0.2)
    assert "small_step" in _sites(rx, lambda: check_forced_steps(rx, case))


@pytest.mark.parametrize("hidden,A,N", [((64, 96), 12, 130), ((128, 128), 16, 130), ((64, 256), 20, 90), ((100, 36, 20), 5, 130)])
def test_launches_per_layer_above_the_line(rx, hidden, A, N):  # noqa: F811
    """The small networks of the other tests, at rows that keep a launch per layer."""
    w = replace(WORKLOADS["tiny"], N=N, minibatches=1, hidden=hidden, A=A)
    case = Case(w, 1, perturb=0.2)
    assert "small_step" not in _sites(rx, lambda: check_forced_steps(rx, case))


@pytest.mark.parametrize("student,N", [((128, 64), 100), ((256, 256, 128), 60), ((30,), 7)])
def test_regression(rx, student, N):  # noqa: F811
    assert "small_step" in _sites(rx, lambda: run_bc(rx, replace(WORKLOADS["distill"].scaled(N), student_hidden=student), 1))


@pytest.mark.parametrize("rows,dims", [(100, (200, 128, 64, 8)), (61, (37, 100, 30, 5)), (384, (64, 256, 256, 32))])
def test_values_beyond_the_split(rx, rows, dims):  # noqa: F811
    test_gpu_split.test_update_with_values_beyond_the_split(rx, rows, dims)


@pytest.mark.parametrize("N,hidden", [(3072, (128, 32)), (2048, (132, 32))])
def test_steps_of_the_most_rows_against_the_oracle(rx, N, hidden):  # noqa: F811
    """As many workgroups, and splits of the partial gradients, as a step may have: 192 and 128 for each network."""
    case = Case(replace(WORKLOADS["tiny"], T=1, N=N, minibatches=1, Da=20, Dc=20, A=6, hidden=hidden), 1, perturb=0.2)
    assert "small_step" in _sites(rx, lambda: check_forced_steps(rx, case))


@pytest.mark.parametrize("hidden,rows", [((128,), 6144), ((132, 64), 4096)])
def test_regression_of_the_most_rows(rx, hidden, rows):  # noqa: F811
    """384 and 256 splits: loss and gradient of one step against float64."""
    g = torch.Generator().manual_seed(rows)
    r = lambda *s: torch.randn(*s, generator=g).cuda()  # noqa: E731
    dims = (20,) + hidden + (5,)
    flat = torch.cat([torch.cat([r(a * b) / a ** 0.5, 0.1 * r(b)]) for a, b in zip(dims[:-1], dims[1:])])
    student, obs, tg = rx.Mlp(dims, flat.clone(), trainable=True), r(rows, 20), r(rows, 5)
    p, x, o = flat.double().requires_grad_(True), obs.double(), 0
    for i, (a, b) in enumerate(zip(dims[:-1], dims[1:])):
        x = x @ p[o:o + a * b].view(a, b) + p[o + a * b:o + a * b + b]
        o += a * b + b
        x = x if i == len(dims) - 2 else torch.where(x > 0, x, torch.expm1(torch.clamp(x, max=0.0)))
    loss = ((x - tg.double()) ** 2).mean()
    loss.backward()
    loss = float(loss.detach())
    cfg, stats = rx.BcCfg(epochs=1, minibatches=1), torch.zeros(1, rx.NSTATS, device="cuda")
    ws = rx.workspace(rx.rslx_bc_update_workspace_bytes(student, None, rows, cfg))
    assert "small_step" in _sites(rx, lambda: rx.rslx_bc_update(student, None, obs, None, tg, rows, cfg, ctypes.c_int64(0), stats, ws))
    # sums of `rows` terms in fp32 that partly cancel: 2^-24 sqrt(rows) of the terms, 1e-5 of the gradient's norm with a factor of two
    assert abs(float(stats[0, 0]) - loss) <= 1e-6 * loss
    assert float((student.grads.double() - p.grad).norm()) <= 1e-5 * float(p.grad.norm())


def test_a_row_of_nan_leaves_other_minibatches_alone(rx):  # noqa: F811
    """A NaN observation makes the gradients of its minibatch NaN, as fp32 arithmetic does, and a value of 2^112 with small weights
    does not make those of another NaN."""
    g = torch.Generator().manual_seed(5)
    r = lambda *s: torch.randn(*s, generator=g).cuda()  # noqa: E731
    D, H, A, N = 20, 48, 3, 40
    for bad, finite in ((float("nan"), False), (6e33, True)):
        params = 0.1 * r(D * H + H + H * A + A + A)
        params[:H] *= 1e-36                               # the weights of input 0
        actor, critic = rx.Mlp((D, H, A), params, trainable=True, has_log_std=True), rx.Mlp((D, H, 1), 0.1 * r(D * H + H + H + 1), trainable=True)
        critic.params[:H] *= 1e-36
        obs = r(1, N, D)
        obs[0, 7, 0] = bad
        mu = r(1, N, A)
        ro = rx.Rollout(1, N, obs, obs, mu + r(1, N, A), r(1, N), r(1, N), mu, torch.ones_like(mu), r(1, N), r(1, N))
        cfg, stats = rx.PpoCfg(epochs=1, minibatches=1), torch.zeros(1, rx.NSTATS, device="cuda")
        ws = rx.workspace(rx.rslx_ppo_update_workspace_bytes(actor, critic, ro, cfg))
        rx.rslx_ppo_update(actor, critic, ro, cfg, None, None, ctypes.c_int64(0), stats, ws)
        torch.cuda.synchronize()
        upper = torch.cat([actor.grads[D * H:], critic.grads[D * H:]])
        assert bool(torch.isfinite(upper).all()) == finite, bad


def test_a_row_of_nan_leaves_the_minibatch_before_it_alone(rx):  # noqa: F811
    """A NaN observation makes the gradients of its minibatch NaN, as fp32 arithmetic does, and leaves those of the minibatch before it
    alone; a value of 2^112 with small weights does not make any NaN."""
    g = torch.Generator().manual_seed(5)
    r = lambda *s: torch.randn(*s, generator=g).cuda()  # noqa: E731
    D, H, A, N = 20, 48, 3, 40
    for bad, finite in ((float("nan"), False), (6e33, True)):
        params = 0.1 * r(D * H + H + H * A + A + A)
        params[:H] *= 1e-36                               # the weights of input 0
        value = 0.1 * r(D * H + H + H + 1)
        value[:H] *= 1e-36
        obs, mu, rest = r(1, N, D), r(1, N, A), [r(1, N) for _ in range(4)]
        action = mu + r(1, N, A)
        cfg = rx.PpoCfg(epochs=1, minibatches=2, lr=0.0)             # the small weights stay

        def update(x):
            actor, critic = rx.Mlp((D, H, A), params.clone(), trainable=True, has_log_std=True), rx.Mlp((D, H, 1), value.clone(), trainable=True)
            ro = rx.Rollout(1, N, x, x, action, rest[0], rest[1], mu, torch.ones_like(mu), rest[2], rest[3])
            stats = torch.zeros(2, rx.NSTATS, device="cuda")
            ws = rx.workspace(rx.rslx_ppo_update_workspace_bytes(actor, critic, ro, cfg))
            assert "small_step" in _sites(rx, lambda: rx.rslx_ppo_update(actor, critic, ro, cfg, None, None, ctypes.c_int64(0), stats, ws))
            return torch.cat([actor.grads[D * H:], critic.grads[D * H:]]), stats

        order = torch.empty(N, dtype=torch.int32, device="cuda")
        rx.rslx_permutation(cfg.c.seed, cfg.c.call_index, 0, N, order, rx.workspace(rx.rslx_permutation_workspace_bytes(N)))
        row = int(order[N // 2 + 3])                      # of the second minibatch
        _, clean = update(obs)
        obs[0, row, 0] = bad
        upper, stats = update(obs)
        assert bool(torch.isfinite(upper).all()) == finite, bad
        assert torch.equal(stats[0], clean[0]) and bool(torch.isfinite(stats[1]).all()) == finite


@pytest.mark.parametrize("width,rows,small", [(128, 3072, True), (128, 3073, False), (132, 2048, True), (132, 2049, False)])
def test_line_of_the_update(rx, width, rows, small):  # noqa: F811
    g = torch.Generator().manual_seed(rows)
    r = lambda *s: torch.randn(*s, generator=g).cuda()  # noqa: E731
    net = lambda out, ls: rx.Mlp((8, width, 32, out), 0.1 * r(9 * width + 33 * width - width + 32 + 33 * out + (out if ls else 0)), trainable=True, has_log_std=ls)  # noqa: E731
    actor, critic = net(6, True), net(1, False)
    obs, act, mu = r(1, rows, 8), r(1, rows, 6), r(1, rows, 6)
    ro = rx.Rollout(1, rows, obs, obs, act, r(1, rows), r(1, rows), mu, torch.ones_like(mu), r(1, rows), r(1, rows))
    cfg, stats = rx.PpoCfg(epochs=1, minibatches=1), torch.zeros(1, rx.NSTATS, device="cuda")
    ws = rx.workspace(rx.rslx_ppo_update_workspace_bytes(actor, critic, ro, cfg))
    sites = _sites(rx, lambda: rx.rslx_ppo_update(actor, critic, ro, cfg, None, None, ctypes.c_int64(0), stats, ws))
    assert ("small_step" in sites) == small and torch.isfinite(actor.params).all()


@pytest.mark.parametrize("D,hidden,A,rows,small", [(256, (256, 256, 256), 12, 480, True), (256, (256, 256, 256), 12, 512, False), (235, (256, 256, 256), 12, 816, True),
                                                   (235, (256, 256, 256), 12, 832, False), (256, (256, 128), 12, 1584, True), (256, (256, 128), 12, 1680, False),
                                                   (48, (256, 256, 128), 12, 2048, True), (256, (256, 256, 256), 17, 2048, True), (256, (256, 200, 128), 12, 2048, True),
                                                   (256, (128, 256), 12, 2048, True), (64, (256, 256), 12, 2048, True)])
def test_line_of_layers_that_fill_their_tiles(rx, D, hidden, A, rows, small):  # noqa: F811
    """Fewer rows where launches per layer are the faster form: both sides, and networks without that limit, against the oracle's step."""
    case = Case(replace(WORKLOADS["tiny"], T=1, N=rows, minibatches=1, Da=D, Dc=D, A=A, hidden=hidden), 1, perturb=0.2)
    assert ("small_step" in _sites(rx, lambda: check_forced_steps(rx, case))) == small


@pytest.mark.parametrize("width,rows,small", [(128, 6144, True), (128, 6145, False), (132, 4096, True), (132, 4097, False)])
def test_line_of_the_regression(rx, width, rows, small):  # noqa: F811
    g = torch.Generator().manual_seed(rows)
    r = lambda *s: torch.randn(*s, generator=g).cuda()  # noqa: E731
    student = rx.Mlp((8, width, 5), 0.1 * r(9 * width + 5 * width + 5), trainable=True)
    cfg, stats = rx.BcCfg(epochs=1, minibatches=1), torch.zeros(1, rx.NSTATS, device="cuda")
    ws = rx.workspace(rx.rslx_bc_update_workspace_bytes(student, None, rows, cfg))
    obs, tg = r(rows, 8), r(rows, 5)
    sites = _sites(rx, lambda: rx.rslx_bc_update(student, None, obs, None, tg, rows, cfg, ctypes.c_int64(0), stats, ws))
    assert ("small_step" in sites) == small and torch.isfinite(student.params).all()
