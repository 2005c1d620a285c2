"""The memories' kernels on split operands against the oracle: the whole roll-out in one launch each way at row counts around
its 16-row workgroups, one-step roll-outs, weights without a split for the bf16 matrix cores, and act()'s step for many rows."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from gpu_util import assert_elementwise, dev, host, rel_l2
from oracle import rng as orng
from test_gpu_recurrent import SEED, RCase, _call, _cell, _flat, _nets, check_forced_steps, oracle_collect, rx  # noqa: F401
from workloads import WORKLOADS, make_inputs

pytestmark = pytest.mark.gpu


def _workload(N, T, cell, **kw):
    return replace(WORKLOADS["recurrent"].scaled(N), T=T, minibatches=2, hidden=(64, 32), memory_hidden=128, memory_cell=cell, **kw)


@pytest.mark.parametrize("cell", ["gru", "lstm"])
@pytest.mark.parametrize("N,T", [(2, 3), (30, 1), (34, 4), (64, 2)])
def test_whole_rollout_launch(rx, N, T, cell):
    case = RCase(_workload(N, T, cell, done_p=0.3), 1, perturb=0.1)
    # few samples per minibatch: statistics relative to their terms, as in test_recurrent_update_degenerate_shapes
    check_forced_steps(rx, case, floor=5e-2)


@pytest.mark.parametrize("cell", ["gru", "lstm"])
@pytest.mark.parametrize("T", [1, 2])
def test_one_step_takes_the_launch_per_step(rx, cell, T):
    """Which kernels an update of memories of 128 runs: the whole roll-out's from two steps on."""
    case = RCase(_workload(34, T, cell), 1)
    tr = case.ref["trace"][0]
    b = tr["before"]
    nets = _nets(rx, case.w, b["actor"], b["critic"], b["opt"])
    rx.rslx_trace_begin(256)
    _call(rx, nets, case.gpu_rollout(rx, tr["envs"]), case.gpu_cfg(rx, 1, 1), 1, b["opt"]["step"])
    torch.cuda.synchronize()
    names = [r[0] for r in rx.rslx_trace_end()]
    per_step = ["%s_step_%s" % (cell, d) for d in ("fwd", "bwd")]
    whole = ["%s_seq_%s" % (cell, d) for d in ("fwd", "bwd")]
    assert [names.count(n) for n in per_step + whole] == ([1, 1, 0, 0] if T == 1 else [0, 0, 1, 1]), names


@pytest.mark.parametrize("cell", ["gru", "lstm"])
def test_weights_without_a_split_reach_only_their_own_unit(rx, cell):
    """A recurrent weight of 2^120 saturates the gates of one unit: the update stays finite wherever fp32 arithmetic does."""
    case = RCase(_workload(34, 2, cell, done_p=0.0), 1)
    tr = case.ref["trace"][0]
    b = tr["before"]
    w, out = case.w, []
    G, H = (4 if cell == "lstm" else 3), 128
    at = (w.Da + 1) * G * H + 5 * G * H + 7            # W_hh[5, gate 0, unit 7]
    for value in (2.0 ** 100, 2.0 ** 120):             # the first has a split
        actor = np.array(b["actor"])
        actor[at] = value
        nets = _nets(rx, w, actor, b["critic"], b["opt"])
        _call(rx, nets, case.gpu_rollout(rx, tr["envs"]), case.gpu_cfg(rx, 1, 1), 1, b["opt"]["step"])
        torch.cuda.synchronize()
        out.append([n.grads.cpu().numpy() for n in nets])
    # both saturate gate 0 of unit 7 to exactly 0 or 1, and its derivative to 0: everything else agrees
    for x, y in zip(*out):
        assert np.isfinite(x).all() and np.isfinite(y).all()
        assert np.linalg.norm(x - y) <= 1e-5 * np.linalg.norm(x)


@pytest.mark.parametrize("cell,H,N", [("gru", 256, 1024), ("gru", 256, 1061), ("gru", 320, 1090), ("lstm", 256, 2050)])
def test_large_act_step(rx, cell, H, N):
    """act() at row counts that take the split-operand step kernel, around its tiles of 64 rows, against the fp64 oracle; the same
    values from a values-only call, and fp32 arithmetic for a state that has no split."""
    w = replace(WORKLOADS["recurrent"].scaled(N), T=1, hidden=(64, 32), memory_hidden=H, memory_cell=cell)
    inp = make_inputs(w)
    ref = oracle_collect(w, inp)
    nets = _nets(rx, w, _flat(inp, "actor"), _flat(inp, "critic"))
    ga, ma, gc, mc = nets
    ws = rx.workspace(rx.rslx_act_recurrent_workspace_bytes(ga, ma, gc, mc, N))
    A, S = w.A, _cell(w)[2]
    eps = dev(orng.act_noise(SEED, 0, N, A), torch.float32)
    obs, reset = dev(inp["obs"][0]), dev(inp["reset0"])

    def step(h_a, h_c):
        out = {k: torch.empty(N, A, device="cuda") for k in ("actions", "mu", "sigma")}
        out.update(logp=torch.empty(N, device="cuda"), values=torch.empty(N, device="cuda"), h_a=h_a, h_c=h_c)
        rx.rslx_act_recurrent(ga, ma, gc, mc, obs, obs, N, h_a, h_c, reset, None, None, SEED, 0, eps, out["actions"], out["logp"],
                              out["values"], out["mu"], out["sigma"], 0, ws)
        torch.cuda.synchronize()
        return out

    h0 = dev(inp["h_actor"]), dev(inp["h_critic"])
    last = torch.empty(N, device="cuda")
    rx.rslx_act_recurrent(None, None, gc, mc, None, obs, N, None, h0[1], reset, None, None, 0, 0, None, None, None, last, None, None,
                          rx.ACT_VALUES_ONLY, ws)
    out = step(h0[0].clone(), h0[1].clone())
    for k in ("actions", "mu", "logp", "values", "h_a", "h_c"):
        assert rel_l2(host(out[k]), ref[k][0]) <= 2e-5, k
        assert_elementwise(k, host(out[k]), ref[k][0])
    assert torch.equal(last, out["values"])
    # one huge entry in one state: its row saturates, all others keep their bits
    big = h0[0].clone()
    big[N - 1, 3] = 2.0 ** 120
    got = step(big, h0[1].clone())
    assert torch.isfinite(got["h_a"][:, :H]).all()
    assert torch.equal(got["h_a"][:N - 1], out["h_a"][:N - 1]) and torch.equal(got["h_c"], out["h_c"])


@pytest.mark.parametrize("cell,Ha,Hc,N,site", [("gru", 256, 64, 1100, "gru_uneven"), ("gru", 36, 256, 1100, "gru_uneven"), ("gru", 256, 128, 2050, "gru_uneven"),
                                               ("gru", 64, 64, 4099, "gru_split"), ("lstm", 128, 128, 4099, "lstm_split"),
                                               ("lstm", 512, 64, 1101, "lstm_uneven"), ("gru", 64, 36, 1100, "gru_step_fwd")])
def test_act_step_of_memories_of_different_widths(rx, cell, Ha, Hc, N, site):
    """Each memory takes the kernel of its own sizes, both in one launch: the oracle's values for either network, and the bits of a
    values-only call."""
    nets, refs = {}, {}
    for which, H in (("actor", Ha), ("critic", Hc)):
        w = replace(WORKLOADS["recurrent"].scaled(N), T=1, hidden=(64, 32), memory_hidden=H, memory_cell=cell)
        inp = make_inputs(w)
        inp["reset0"] = (np.random.default_rng(N).random(N) < 0.1).astype(np.uint8)
        got = _nets(rx, w, _flat(inp, "actor"), _flat(inp, "critic"))
        nets[which], refs[which] = got[:2] if which == "actor" else got[2:], (inp, oracle_collect(w, inp))
    (ga, ma), (gc, mc) = nets["actor"], nets["critic"]
    (ia, ra), (ic, rc) = refs["actor"], refs["critic"]
    A = w.A
    ws = rx.workspace(rx.rslx_act_recurrent_workspace_bytes(ga, ma, gc, mc, N))
    eps = dev(orng.act_noise(SEED, 0, N, A), torch.float32)
    obs_a, obs_c, reset = dev(ia["obs"][0]), dev(ic["obs"][0]), dev(ia["reset0"])
    h_a, h_c = dev(ia["h_actor"]), dev(ic["h_critic"])
    last = torch.empty(N, device="cuda")
    rx.rslx_act_recurrent(None, None, gc, mc, None, obs_c, N, None, h_c, reset, None, None, 0, 0, None, None, None, last, None, None,
                          rx.ACT_VALUES_ONLY, ws)
    out = {k: torch.empty(N, A, device="cuda") for k in ("actions", "mu", "sigma")}
    out.update(logp=torch.empty(N, device="cuda"), values=torch.empty(N, device="cuda"), h_a=h_a, h_c=h_c)
    rx.rslx_trace_begin(32)
    rx.rslx_act_recurrent(ga, ma, gc, mc, obs_a, obs_c, N, h_a, h_c, reset, None, None, SEED, 0, eps, out["actions"], out["logp"], out["values"],
                          out["mu"], out["sigma"], 0, ws)
    torch.cuda.synchronize()
    assert [r[0] for r in rx.rslx_trace_end() if r[0].startswith(cell)] == [site]
    for k, ref in (("actions", ra), ("mu", ra), ("logp", ra), ("h_a", ra), ("values", rc), ("h_c", rc)):
        assert rel_l2(host(out[k]), ref[k][0]) <= 2e-5, k
        assert_elementwise(k, host(out[k]), ref[k][0])
    assert torch.equal(last, out["values"])


@pytest.mark.parametrize("cell,H,N,site", [("gru", 256, 1024, "gru_step_fwd"), ("gru", 256, 1025, "gru_split"), ("gru", 128, 2048, "gru_step_fwd"),
                                           ("gru", 128, 2049, "gru_split"), ("lstm", 64, 16385, "lstm_step_fwd"), ("lstm", 128, 4096, "lstm_step_fwd"),
                                           ("lstm", 128, 6143, "lstm_step_fwd"), ("lstm", 128, 6144, "lstm_split"), ("lstm", 256, 2048, "lstm_split")])
def test_memory_step_sizes(rx, cell, H, N, site):
    """Which kernel a memory's own step takes, on both sides of the line; its states are those of calls with fewer rows, which run the
    fp32 kernel."""
    g = torch.Generator().manual_seed(N)
    G, S, D = (4 if cell == "lstm" else 3), (2 if cell == "lstm" else 1) * H, 20
    m = rx.Memory(rx.CELL_LSTM if cell == "lstm" else rx.CELL_GRU, D, H, ((torch.rand(G * H * (D + H + 2), generator=g) * 2 - 1) / H ** 0.5).cuda())
    obs, s0 = torch.randn(N, D, generator=g).cuda(), (0.5 * torch.randn(N, S, generator=g)).cuda()
    ws = rx.workspace(rx.rslx_memory_step_workspace_bytes(m, N))
    whole, parts = s0.clone(), s0.clone()
    rx.rslx_trace_begin(16)
    rx.rslx_memory_step(m, obs, N, whole, None, None, None, ws)
    torch.cuda.synchronize()
    assert [r[0] for r in rx.rslx_trace_end() if r[0].startswith(cell)] == [site]
    for i in range(0, N, 1000):
        rx.rslx_memory_step(m, obs[i:i + 1000], min(1000, N - i), parts[i:i + 1000], None, None, None, ws)
    torch.cuda.synchronize()
    assert rel_l2(host(whole), host(parts)) <= 2e-6
    assert_elementwise("state", host(whole), host(parts).astype(np.float64))


@pytest.mark.parametrize("cell", ["gru", "lstm"])
@pytest.mark.parametrize("Ha,Hc", [(128, 64), (44, 128)])
def test_update_of_memories_of_different_widths(rx, cell, Ha, Hc):
    """A memory of 128 beside one of another width runs a launch per step.  Without a norm clip the two networks' updates do not meet,
    so the oracle's runs of equal widths give the actor's and the critic's half."""
    cases = {}
    for H in (Ha, Hc):
        w = replace(WORKLOADS["recurrent"].scaled(34), T=4, minibatches=2, hidden=(64, 32), memory_hidden=H, memory_cell=cell, done_p=0.2, max_grad_norm=1e9)
        cases[H] = RCase(w, 2)
    ca, cc = cases[Ha], cases[Hc]
    assert np.array_equal(ca.oro["obs_a"], cc.oro["obs_a"]) and np.array_equal(ca.oro["dones"], cc.oro["dones"])
    na, nc = _nets(rx, ca.w, ca.actor0, ca.critic0), _nets(rx, cc.w, cc.actor0, cc.critic0)
    nets = na[:2] + nc[2:]
    ro_a, dones, h0_a, _ = ca.gpu_rollout(rx)
    ro_c, _, _, h0_c = cc.gpu_rollout(rx)
    ro_a.t.update({k: ro_c.t[k] for k in ("values", "returns")})
    rx.rslx_trace_begin(1024)
    stats, step = _call(rx, nets, (ro_a, dones, h0_a, h0_c), ca.gpu_cfg(rx, 2, 2), 4, 0)
    names = [r[0] for r in rx.rslx_trace_end()]
    assert names.count("%s_step_fwd" % cell) == names.count("%s_step_bwd" % cell) == 4 * 4 and not any("seq" in n for n in names)
    assert step == 4
    # the free-running bounds of test_recurrent_update_two_epochs
    np.testing.assert_allclose(stats[:, 0], ca.ref["stats"][:, 0], rtol=5e-2, atol=1e-2 * 5e-2)
    np.testing.assert_allclose(stats[:, 1], cc.ref["stats"][:, 1], rtol=5e-2)
    assert rel_l2(np.concatenate([host(n.params) for n in nets[:2]]), ca.ref["actor"]) <= 2e-4
    assert rel_l2(np.concatenate([host(n.params) for n in nets[2:]]), cc.ref["critic"]) <= 2e-4
