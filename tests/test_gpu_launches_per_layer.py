"""Small networks with a launch per layer, which they take in the least workspace (otherwise one launch runs the whole step): the padded loss
heads, the stand-alone loss kernel, staged and in-place inputs, values beyond the split and rounding offsets, against the references of
the tests that compare the step as it comes.  The trace says which launches ran."""
import ctypes
from dataclasses import replace

import pytest
import torch

import test_gpu_shapes
import test_gpu_split
import test_gpu_update as U
from gpu_util import host, least_workspace
from test_gpu_update import rx  # noqa: F401
from workloads import WORKLOADS

pytestmark = pytest.mark.gpu


@pytest.fixture
def sites(monkeypatch):
    """Updates of test_gpu_update's cases in the least workspace; the names of their launches."""
    seen = set()

    def call(rx, case, a, c, rnd, rollout, cfg, n_rows, step0):  # noqa: F811
        stats, step, sym = torch.zeros(n_rows, rx.NSTATS, device="cuda"), ctypes.c_int64(step0), case.gpu_sym(rx)
        run = lambda ws: rx.rslx_ppo_update(a, c, rollout, cfg, sym, rnd, step, stats, ws)  # noqa: E731
        ws = least_workspace(rx, run)
        rx.rslx_trace_begin(4096)
        run(ws)
        torch.cuda.synchronize()
        seen.update(r[0] for r in rx.rslx_trace_end())
        return host(stats), step.value

    monkeypatch.setattr(U, "_call", call)
    return seen


@pytest.mark.parametrize("width,A,site", [(68, 12, "ppo_head"), (100, 3, "ppo_head"), (124, 17, "ppo_head"), (132, 12, "ppo_head"), (252, 8, "ppo_head"), (40, 12, "ppo_loss"), (66, 12, "ppo_loss")])
def test_head_between_padded_widths(rx, sites, width, A, site):  # noqa: F811
    U.check_forced_steps(rx, U.Case(replace(WORKLOADS["tiny"], N=50, A=A, hidden=(64, width)), 1, perturb=0.2))
    assert site in sites and "small_step" not in sites


@pytest.mark.parametrize("N,A,hidden,site", [(40, 3, (64, 32), "ppo_head"), (50, 16, (128, 128), "ppo_head"), (36, 20, (64, 256), "ppo_head"), (50, 12, (64, 96), "ppo_head"), (50, 12, (64, 98), "ppo_loss")])
def test_head_widths_over_whole_updates(rx, sites, N, A, hidden, site):  # noqa: F811
    """A last hidden width that is no multiple of 4 takes the output layers' own launches and the stand-alone loss kernel."""
    case = U.Case(replace(WORKLOADS["tiny"].scaled(N), A=A, hidden=hidden), 1, perturb=0.2)
    U.check_free_running(rx, case, U.check_forced_steps(rx, case))
    assert site in sites and "small_step" not in sites


@pytest.mark.parametrize("i,shape", [(i, s) for i, s in enumerate(test_gpu_shapes._shapes(101, 10)) if i % 3])
def test_irregular_shapes(rx, sites, i, shape):  # noqa: F811
    """(Some of them in one launch here too, where that takes no more room.)"""
    w = replace(WORKLOADS["tiny"], N=shape["N"], T=shape["T"], Da=shape["D"], Dc=shape["D"], A=shape["A"], hidden=shape["hidden"], minibatches=shape["minibatches"], height_scan=0)
    U.check_forced_steps(rx, U.Case(w, 1, perturb=0.15))


@pytest.mark.parametrize("hidden,staged,site", [((64, 64), True, "ppo_head"), ((64,), False, "ppo_head")])
def test_staged_and_in_place_inputs(rx, sites, hidden, staged, site):  # noqa: F811
    """37 observations: copied into zero-padded rows, or read in place where the first layer is too small for the padded contraction.
    More rows than one launch for the step takes, which would need less room."""
    w = replace(WORKLOADS["tiny"], N=650, T=5, Da=37, Dc=37, A=4, hidden=hidden, minibatches=1, height_scan=0)
    U.check_forced_steps(rx, U.Case(w, 1, perturb=0.15))
    assert site in sites and "small_step" not in sites and ("stage_input" in sites) == staged


def _bc_grads(rx, dims, params, x, y):  # noqa: F811
    net = rx.Mlp(dims, params, trainable=True)
    cfg = rx.BcCfg(lr=1e-9, epochs=1, minibatches=1, max_grad_norm=0.0, seed=1, call_index=0)
    stats, step = torch.zeros(1, rx.NSTATS, device="cuda"), ctypes.c_int64(0)
    run = lambda ws: rx.rslx_bc_update(net, None, x, None, y, x.shape[0], cfg, step, stats, ws)  # noqa: E731
    ws = least_workspace(rx, run)
    rx.rslx_trace_begin(64)
    run(ws)
    torch.cuda.synchronize()
    assert "small_step" not in {r[0] for r in rx.rslx_trace_end()}
    return net.grads


@pytest.mark.parametrize("rows,dims", [(384, (200, 256, 8))])
def test_values_beyond_the_split(rx, monkeypatch, rows, dims):  # noqa: F811
    monkeypatch.setattr(test_gpu_split, "_bc_grads", _bc_grads)
    test_gpu_split.test_update_with_values_beyond_the_split(rx, rows, dims)


@pytest.mark.parametrize("rows", [128, 384])
@pytest.mark.parametrize("K", [16, 48])
def test_input_gradient_has_no_rounding_offset(rx, K, rows):  # noqa: F811
    """With the first layer zero its units are 0, their slope is one, and its bias gradient is the column sum of the input gradient.
    More inputs than one launch for the step takes."""
    gen = torch.Generator(device="cuda").manual_seed(K + rows)
    normal = lambda *s: torch.randn(*s, generator=gen, device="cuda")  # noqa: E731
    H, D, offset = 256, 272, []
    for _ in range(3):
        w, x, y = normal(H, K) / K ** 0.5, normal(rows, D), normal(rows, K)
        flat = torch.cat([torch.zeros(D * H + H, device="cuda"), w.ravel(), torch.zeros(K, device="cuda")])
        g = _bc_grads(rx, (D, H, K), flat, x, y).double()
        dz = (-2.0 * y.double() / (rows * K)) @ w.double().T.contiguous()
        offset.append((g[D * H:D * H + H] - dz.sum(0)) / (rows * dz.pow(2).mean().sqrt()))
    err = torch.stack(offset)
    # the mean of errors without an offset lies within six of its own standard errors
    assert abs(float(err.mean())) <= 6 * float(err.std()) / err.numel() ** 0.5
