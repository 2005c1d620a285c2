"""The fused loss head at last hidden widths between its padded ones, for both networks and with mirrored rows, against the
oracle's own steps; widths outside its rule, which keep the per-layer launches."""
import ctypes
from dataclasses import replace

import pytest
import torch

from test_gpu_update import Case, check_forced_steps, rx  # noqa: F401
from workloads import WORKLOADS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("base,width,A", [("tiny", 68, 12), ("tiny", 100, 3), ("tiny", 124, 17), ("tiny", 132, 12), ("tiny", 252, 8), ("rough", 100, 12),
                                          ("tiny", 40, 12), ("tiny", 66, 12), ("tiny", 260, 12), ("rough", 98, 12)])
def test_head_between_padded_widths(rx, base, width, A):  # noqa: F811
    w = replace(WORKLOADS[base], N=50, hidden=(64, width)) if base == "tiny" else WORKLOADS[base].scaled(24)
    if base == "tiny":
        w = replace(w, A=A)
    else:
        w = replace(w, hidden=(64, width))
    check_forced_steps(rx, Case(w, 1, perturb=0.2))


@pytest.mark.parametrize("widths,A,rows,site", [((132, 132), 12, 32768, "ppo_head"), ((132, 132), 12, 32769, "ppo_loss"), ((68, 200), 12, 32769, "ppo_loss"),
                                                ((256, 252), 20, 16384, "ppo_head"), ((256, 252), 20, 16385, "ppo_loss"),
                                                ((68, 68), 20, 49152, "ppo_head"), ((68, 128), 20, 49153, "ppo_loss"),
                                                ((68, 68), 12, 49153, "ppo_head"), ((132, 68), 3, 49153, "ppo_head"), ((132, 68), 8, 49152, "ppo_head"),
                                                ((132, 68), 8, 49153, "ppo_loss"), ((256, 256), 20, 49153, "ppo_head")])
def test_head_padded_widths_up_to_so_many_rows(rx, widths, A, rows, site):  # noqa: F811
    """Which loss launch an update takes, on both sides of the rows up to which padding a last hidden layer pays."""
    g = torch.Generator().manual_seed(rows)
    r = lambda *s: torch.randn(*s, generator=g).cuda()  # noqa: E731
    net = lambda H, out, ls: rx.Mlp((8, H, out), 0.1 * r(8 * H + H + H * out + out + (out if ls else 0)), trainable=True, has_log_std=ls)  # noqa: E731
    actor, critic = net(widths[0], A, True), net(widths[1], 1, False)
    obs, act, mu = r(1, rows, 8), r(1, rows, A), r(1, rows, A)
    ro = rx.Rollout(1, rows, obs, obs, act, r(1, rows), r(1, rows), mu, torch.ones_like(mu), r(1, rows), r(1, rows))
    cfg, stats = rx.PpoCfg(epochs=1, minibatches=1), torch.zeros(1, rx.NSTATS, device="cuda")
    ws = rx.workspace(rx.rslx_ppo_update_workspace_bytes(actor, critic, ro, cfg))
    rx.rslx_trace_begin(64)
    rx.rslx_ppo_update(actor, critic, ro, cfg, None, None, ctypes.c_int64(0), stats, ws)
    torch.cuda.synchronize()
    assert [n[0] for n in rx.rslx_trace_end() if n[0].startswith("ppo")] == [site]
    assert torch.isfinite(stats).all() and torch.isfinite(actor.params).all()
