"""The contractions run on the bf16 matrix cores on operands split in three parts: the results must keep fp32 accuracy
over the whole exponent range, at every remainder of the tiles, and infinite inputs must give what fp32 arithmetic
gives.  More than 8192 rows take the tiled per-layer launches, fewer the layer-fused one."""
import ctypes as C

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
LAYERED, FUSED = 8193, 70


@pytest.fixture(scope="module")
def rx():
    import paper_2509_10771_amd as m
    m.rslx_device_check()
    return m


def _critic(rx, dims, seed):
    g = np.random.default_rng(seed)
    flat = np.concatenate([np.concatenate([(g.normal(size=a * b) / np.sqrt(a)), 0.1 * g.normal(size=b)]) for a, b in zip(dims, dims[1:])])
    flat = flat.astype(np.float32)
    return rx.Mlp(dims, torch.from_numpy(flat).cuda()), flat


def _values(rx, net, obs, N):
    out = torch.empty(N, device="cuda")
    ws = rx.workspace(rx.rslx_act_workspace_bytes(None, net, N))
    rx.rslx_act(None, net, None, torch.from_numpy(obs).cuda(), N, 0, 0, None, None, None, out, None, None, rx.ACT_VALUES_ONLY, ws)
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("N,A", [(FUSED, 1), (FUSED, 200), (LAYERED, 1), (LAYERED, 50), (LAYERED, 200), (LAYERED, 1400)])
@pytest.mark.parametrize("D", [1, 4, 31, 32, 33, 100, 512])
def test_linear_layer_keeps_fp32_accuracy_over_the_exponent_range(rx, D, N, A):
    """One linear layer without a bias on rows scaled by powers of ten from 1e-44 (where fp32 has four bits left) to 1e37;
    the output widths of the layered calls are one for each tile shape.  Bound: D + 1 roundings of fp32 (2^-24 each) and
    the 2^-24 of the products left out, against the sum of the terms' sizes (2^-150 each where the sum is subnormal); a
    sum of bf16 products would be off by 2^-9 of it, one without the third parts by 2^-17."""
    g = np.random.default_rng(D)
    w = (g.normal(size=(D, A)) / np.sqrt(D)).astype(np.float32)
    net = rx.Mlp((D, A), torch.from_numpy(np.concatenate([w.ravel(), np.zeros(A, np.float32)])).cuda())
    obs = torch.from_numpy((g.normal(size=(N, D)) * 10.0 ** g.integers(-44, 38, size=(N, 1))).astype(np.float32)).cuda()
    got, twin = torch.full((N, A), 7.0, device="cuda"), torch.empty(N, A, device="cuda")
    rx.rslx_bc_collect(net, net, obs, obs, N, got, twin, rx.workspace(rx.rslx_bc_collect_workspace_bytes(net, net, N)))
    w64, x64 = torch.from_numpy(w).cuda().double(), obs.double()
    ref, size = x64 @ w64, x64.abs() @ w64.abs()
    over = (got.double() - ref).abs() - (D + 3) * (2.0 ** -24 * size + 2.0 ** -150)
    worst = int(over.amax(1).argmax())
    assert bool((over <= 0).all()), (float(over[worst].max()), worst, float(obs[worst].abs().max()))
    assert torch.equal(got, twin)


@pytest.mark.parametrize("N", [FUSED, LAYERED])
@pytest.mark.parametrize("dims", [(13, 20, 1), (48, 128, 72, 1), (37, 100, 300, 12, 1), (64, 512, 512, 1), (5, 3, 2, 1)])
def test_networks_of_ragged_widths(rx, dims, N):
    """fp32 accuracy through several layers: each adds at most a few 1e-7 (sums of up to 512 terms, ELU)."""
    from oracle import mlp
    net, flat = _critic(rx, dims, 5)
    obs = np.random.default_rng(N).normal(size=(N, dims[0])).astype(np.float32)
    ref, _ = mlp.forward(mlp.unpack(flat, dims), obs)
    got = _values(rx, net, obs, N)
    assert np.linalg.norm(got - ref[:, 0]) <= 2e-6 * np.linalg.norm(ref)


@pytest.mark.parametrize("N", [FUSED, LAYERED])
def test_infinite_and_nan_inputs_give_what_fp32_gives(rx, N):
    D = 40
    net, flat = _critic(rx, (D, 1), 7)
    obs = np.random.default_rng(1).normal(size=(N, D)).astype(np.float32)
    big = np.float32(3.4e38)                       # finite, but rounds to infinity in bf16
    obs[3, 5], obs[20, 0], obs[33, 7], obs[69, 39], obs[40, 1] = np.inf, -np.inf, np.nan, big, np.inf
    obs[40, 2] = -np.inf * np.sign(flat[1] * flat[2])       # meets the other infinity with the opposite sign
    got = _values(rx, net, obs, N)
    with np.errstate(invalid="ignore", over="ignore"):
        ref = (obs * flat[:D]).astype(np.float64).sum(1) + float(flat[D])
    assert np.isnan(ref[33]) and np.isnan(ref[40]) and np.isinf(ref[3]) and np.isinf(ref[20]) and np.isfinite(ref[69])
    np.testing.assert_allclose(got, ref, rtol=2e-5, atol=1e-5)      # also compares NaN and infinity places


@pytest.mark.parametrize("cell", ["gru", "lstm"])
def test_infinite_observation_saturates_the_gates(rx, cell):
    """The input-side gates of an infinite observation are infinite, the new state is finite."""
    N, D, H = 100, 48, 64
    G = 4 if cell == "lstm" else 3
    g = np.random.default_rng(2)
    flat = g.uniform(-0.1, 0.1, size=G * H * (D + H + 2)).astype(np.float32)
    mem = rx.Memory(rx.CELL_LSTM if cell == "lstm" else rx.CELL_GRU, D, H, torch.from_numpy(flat).cuda())
    obs = g.normal(size=(N, D)).astype(np.float32)
    obs[7, 3], obs[64, 0] = np.inf, -np.inf
    S = 2 * H if cell == "lstm" else H
    h0 = (0.5 * g.normal(size=(N, S))).astype(np.float32)
    h = torch.from_numpy(h0).cuda()
    ws = rx.workspace(rx.rslx_memory_step_workspace_bytes(mem, N))
    rx.rslx_memory_step(mem, torch.from_numpy(obs).cuda(), N, h, None, None, None, ws)
    torch.cuda.synchronize()
    w_ih, o = flat[:D * G * H].reshape(D, G * H).astype(np.float64), (D + 1) * G * H
    gi = np.empty((N, G * H))
    with np.errstate(invalid="ignore"):
        for r in range(N):
            gi[r] = (obs[r].astype(np.float64)[:, None] * w_ih).sum(0)
    gi += flat[D * G * H:o]
    gh = h0[:, :H].astype(np.float64) @ flat[o:o + H * G * H].reshape(H, G * H) + flat[o + H * G * H:]
    sig = lambda a: np.where(a > 0, 1 / (1 + np.exp(-np.abs(a))), np.exp(-np.abs(a)) / (1 + np.exp(-np.abs(a))))
    if cell == "gru":
        r, z = sig(gi[:, :H] + gh[:, :H]), sig(gi[:, H:2 * H] + gh[:, H:2 * H])
        ref = (1 - z) * np.tanh(gi[:, 2 * H:] + r * gh[:, 2 * H:]) + z * h0
    else:
        a = gi + gh
        c = sig(a[:, H:2 * H]) * h0[:, H:] + sig(a[:, :H]) * np.tanh(a[:, 2 * H:3 * H])
        ref = np.concatenate([sig(a[:, 3 * H:]) * np.tanh(c), c], 1)
    got = h.cpu().numpy()
    assert np.isfinite(ref).all() and np.isfinite(got).all()
    assert np.abs(got - ref).max() < 1e-5


def test_layer_of_more_than_two_to_the_thirty_weights(rx):
    """A hidden layer [1040, 2^20]: its split weights take more than 2^32 bytes, forward and input gradient.  Gradients
    of the whole network against float64 on the GPU.  Bound: the input gradient's sums run over 2^20 terms in 6 x 65 536
    matrix instructions, each rounding by up to 2^-24 of the sum so far; with random signs sqrt(393 216) x 2^-24 = 4e-5 of
    the largest sum, and the bias gradient, a sum over rows with random signs, is smaller than its terms' sizes add up
    to by sqrt(48): 2.6e-4.  A part of the weights read at the wrong place is an error of order one."""
    dims, rows = (8, 1040, 1 << 20, 2), 48
    n = [a * b for a, b in zip(dims, dims[1:])]
    gen = torch.Generator(device="cuda").manual_seed(4)
    net = rx.Mlp(dims, torch.zeros(sum(n) + sum(dims[1:]), device="cuda"), trainable=True)
    views, o = [], 0
    for k, (a, b) in enumerate(zip(dims, dims[1:])):
        w = net.params[o:o + a * b].view(a, b)
        w.uniform_(-1, 1, generator=gen).mul_((3.0 / a) ** 0.5)
        views.append((w, net.params[o + a * b:o + a * b + b].uniform_(-0.1, 0.1, generator=gen), o))
        o += a * b + b
    x = torch.randn(rows, dims[0], generator=gen, device="cuda")
    y = torch.randn(rows, dims[-1], generator=gen, device="cuda")
    elu = lambda z: torch.where(z > 0, z, torch.expm1(torch.clamp(z, max=0.0)))  # noqa: E731
    hs = [x.double()]
    for k, (w, b, _) in enumerate(views):
        z = hs[-1] @ w.double() + b.double()
        hs.append(elu(z) if k < 2 else z)
    d = 2.0 * (hs[-1] - y.double()) / y.numel()
    ref = [None] * 3
    for k in (2, 1, 0):
        ref[k] = (hs[k].T.contiguous() @ d, d.sum(0))
        if k:
            d = (d @ views[k][0].double().T.contiguous()) * torch.where(hs[k] > 0, 1.0, hs[k] + 1.0)
    cfg = rx.BcCfg(lr=1e-9, epochs=1, minibatches=1, max_grad_norm=0.0, seed=1, call_index=0)
    stats, step = torch.zeros(1, rx.NSTATS, device="cuda"), C.c_int64(0)
    ws = rx.workspace(rx.rslx_bc_update_workspace_bytes(net, None, rows, cfg))
    rx.rslx_bc_update(net, None, x, None, y, rows, cfg, step, stats, ws)
    torch.cuda.synchronize()
    for k, (w, b, o) in enumerate(views):
        for name, r, o_ in (("W", ref[k][0], o), ("b", ref[k][1], o + w.numel())):
            got = net.grads[o_:o_ + r.numel()].view_as(r)
            err = float((got.double() - r).norm() / r.norm())
            assert err <= 2.6e-4, (k, name, err)


# Rounding must not have a direction: gradients are sums over minibatches, where an offset of 1e-8 of a result's size in
# every row adds up while random errors of 1e-7 cancel.  Bound: six standard deviations of a mean of independent errors.
def _mean_is_random(err, rms, what):
    mean, dev = float(err.mean() / rms), float(err.std() / rms)
    assert abs(mean) <= 6 * dev / err.numel() ** 0.5, (what, mean, dev)


@pytest.mark.parametrize("N", [8192, 16384])
@pytest.mark.parametrize("K,A", [(16, 200), (48, 256), (200, 40), (512, 12), (512, 200)])
def test_layer_outputs_have_no_rounding_offset(rx, K, A, N):
    gen = torch.Generator(device="cuda").manual_seed(K + A)
    for _ in range(3):
        w = torch.randn(K, A, generator=gen, device="cuda") / K ** 0.5
        x = torch.randn(N, K, generator=gen, device="cuda")
        net = rx.Mlp((K, A), torch.cat([w.ravel(), torch.zeros(A, device="cuda")]))
        got, twin = torch.empty(N, A, device="cuda"), torch.empty(N, A, device="cuda")
        rx.rslx_bc_collect(net, net, x, x, N, got, twin, rx.workspace(rx.rslx_bc_collect_workspace_bytes(net, net, N)))
        ref = x.double() @ w.double()
        _mean_is_random(got.double() - ref, ref.pow(2).mean().sqrt(), "forward")


def _bc_grads(rx, dims, params, x, y):
    net = rx.Mlp(dims, params, trainable=True)
    cfg = rx.BcCfg(lr=1e-9, epochs=1, minibatches=1, max_grad_norm=0.0, seed=1, call_index=0)
    stats, step = torch.zeros(1, rx.NSTATS, device="cuda"), C.c_int64(0)
    ws = rx.workspace(rx.rslx_bc_update_workspace_bytes(net, None, x.shape[0], cfg))
    rx.rslx_bc_update(net, None, x, None, y, x.shape[0], cfg, step, stats, ws)
    torch.cuda.synchronize()
    return net.grads


@pytest.mark.parametrize("rows", [128, 384, 24576])
@pytest.mark.parametrize("K", [16, 48, 512])
def test_gradients_have_no_rounding_offset(rx, K, rows):
    """Forward with packed weights: with zero targets the bias gradient is the column mean of the outputs.  Weight gradient:
    one, an odd and an even number of row splits.  Input gradient: with the first layer zero its units are 0, their slope
    is one, and its bias gradient is the column sum of the input gradient."""
    gen = torch.Generator(device="cuda").manual_seed(K + rows)
    normal = lambda *s: torch.randn(*s, generator=gen, device="cuda")  # noqa: E731
    H = 256
    offset = dict(forward=[], weight=[], input=[])
    for _ in range(3):
        w, x = normal(K, H) / K ** 0.5, normal(rows, K)
        g = _bc_grads(rx, (K, H), torch.cat([w.ravel(), torch.zeros(H, device="cuda")]), x, torch.zeros(rows, H, device="cuda")).double()
        d = 2.0 * (x.double() @ w.double()) / (rows * H)
        offset["forward"].append((g[K * H:] - d.sum(0)) / (rows * d.pow(2).mean().sqrt()))
        gw = x.double().T.contiguous() @ d
        offset["weight"].append((g[:K * H].view(K, H) - gw) / gw.pow(2).mean().sqrt())
        w, x, y = normal(H, K) / K ** 0.5, normal(rows, 32), normal(rows, K)
        flat = torch.cat([torch.zeros(32 * H + H, device="cuda"), w.ravel(), torch.zeros(K, device="cuda")])
        g = _bc_grads(rx, (32, H, K), flat, x, y).double()
        dz = (-2.0 * y.double() / (rows * K)) @ w.double().T.contiguous()
        offset["input"].append((g[32 * H:32 * H + H] - dz.sum(0)) / (rows * dz.pow(2).mean().sqrt()))
    for what, parts in offset.items():
        err = torch.stack(parts)
        assert abs(float(err.mean())) <= 6 * float(err.std()) / err.numel() ** 0.5, (what, float(err.mean()), float(err.std()))


@pytest.mark.parametrize("N,dims", [(FUSED, (48, 128, 72, 12)), (FUSED, (33, 512, 300, 7)), (LAYERED, (48, 128, 72, 12)), (LAYERED, (45, 300, 1400))])
def test_rows_without_a_split_leave_the_others_alone(rx, N, dims):
    """Rows with infinite, NaN or very large inputs are repeated in fp32; the rows beside them keep every bit."""
    g = np.random.default_rng(3)
    flat = np.concatenate([np.concatenate([g.normal(size=a * b) / np.sqrt(a), 0.1 * g.normal(size=b)]) for a, b in zip(dims, dims[1:])])
    net = rx.Mlp(dims, torch.from_numpy(flat.astype(np.float32)).cuda())
    obs = torch.from_numpy(g.normal(size=(N, dims[0])).astype(np.float32)).cuda()
    out = [torch.empty(N, dims[-1], device="cuda") for _ in range(3)]
    ws = rx.workspace(rx.rslx_bc_collect_workspace_bytes(net, net, N))
    rx.rslx_bc_collect(net, net, obs, obs, N, out[0], out[2], ws)
    odd = obs.clone()
    for row, col, v in ((3, 5, np.inf), (20, 0, -np.inf), (33, 7, np.nan), (47, 1, 3e38), (N - 2, 31, 6e33)):
        odd[row, col] = float(v)
    rx.rslx_bc_collect(net, net, odd, odd, N, out[1], out[2], ws)
    keep = torch.ones(N, dtype=torch.bool, device="cuda")
    keep[[3, 20, 33, 47, N - 2]] = False
    assert torch.equal(out[0][keep], out[1][keep])
    assert bool(torch.isnan(out[1][33]).all()) and bool(torch.isfinite(out[1][N - 2]).all())


@pytest.mark.parametrize("rows,dims", [(384, (200, 256, 8)), (384, (37, 300, 100, 5)), (384, (37, 301, 133, 70, 5)), (384, (1024, 1024, 16)), (11264, (64, 1024, 1024, 16))])
def test_update_with_values_beyond_the_split(rx, rows, dims):
    """Finite values of 2^112 and above in the observations, the weights and the loss gradient that meet small ones, so that
    every sum of fp32 products is finite: packed forward, input gradient and weight gradients (three row splits at 384 rows, even
    and odd counts at 11 264; 64 x 128 and 128 x 128 tiles, inside and at the edge, widths that allow 16-byte loads and
    others), against float64, element by element.
    Bound: 2^-24 of the terms' sizes for every index of the contraction, for each contraction on the way."""
    gen = torch.Generator(device="cuda").manual_seed(rows + dims[0])
    L, W, b, flat = len(dims) - 1, [], [], []
    for a, c in zip(dims, dims[1:]):
        W.append(torch.randn(a, c, generator=gen, device="cuda") / a ** 0.5)
        b.append(0.1 * torch.randn(c, generator=gen, device="cuda"))
    x = torch.randn(rows, dims[0], generator=gen, device="cuda")
    y = torch.randn(rows, dims[-1], generator=gen, device="cuda")
    # input column 3 of some rows is huge, its weights are tiny; output column 1 has tiny weights and huge targets
    x[5::70, 3] = 2e38
    W[0][3] *= 1e-39
    W[-1][:, 1] *= 1e-37
    y[11::50, 1] = 1e38
    for w, c in zip(W, b):
        flat += [w.ravel(), c]
    g = _bc_grads(rx, dims, torch.cat(flat), x, y).double()
    hs, size = [x.double()], []
    for k in range(L):
        z = hs[-1] @ W[k].double() + b[k].double()
        hs.append(torch.where(z > 0, z, torch.expm1(torch.clamp(z, max=0.0))) if k < L - 1 else z)
    d = 2.0 * (hs[-1] - y.double()) / y.numel()
    size, eps, o = d.abs() + 2.0 * hs[-1].abs() / y.numel(), 2.0 ** -24, sum(a * c + c for a, c in zip(dims, dims[1:]))
    terms = sum(dims[:-1])                                # roundings behind a value so far
    for k in range(L - 1, -1, -1):
        a, c = dims[k], dims[k + 1]
        o -= a * c + c
        for got, ref, s in ((g[o:o + a * c].view(a, c), hs[k].T.contiguous() @ d, hs[k].abs().T.contiguous() @ size),
                            (g[o + a * c:o + a * c + c], d.sum(0), size.sum(0))):
            assert bool(torch.isfinite(got).all())
            over = (got - ref).abs() / ((terms + rows) * eps * s + 1e-38)
            assert float(over.max()) <= 1.0, (k, float(over.max()), int(over.argmax()))
        if k:
            slope = torch.where(hs[k] > 0, 1.0, hs[k] + 1.0)
            d, size = (d @ W[k].double().T.contiguous()) * slope, (size @ W[k].double().abs().T.contiguous()) * slope
            terms += c


@pytest.mark.parametrize("gathered", [False, True])
def test_observations_of_more_than_four_gibibytes(rx, gathered):
    """2^24 + 77 rows of 64: layered inference reads them by offsets from each tile's first row, the update (gathered rows) by
    64-bit addresses.  Outputs of the last rows, and of some far apart, to fp32 accuracy; gradients against float64 sums to
    2e-5 (sums of 1.7e7 rows by 128 to 65 536 at a time)."""
    rows, dims = (1 << 24) + 77, (64, 8, 1)
    gen = torch.Generator(device="cuda").manual_seed(9)
    x = torch.empty(rows, 64, device="cuda").normal_(generator=gen)
    parts = []
    for a, c in zip(dims, dims[1:]):
        parts += [torch.randn(a, c, generator=gen, device="cuda") / a ** 0.5, 0.1 * torch.randn(c, generator=gen, device="cuda")]
    flat = torch.cat([p.ravel() for p in parts])
    if not gathered:
        net, out = rx.Mlp(dims, flat), torch.empty(rows, device="cuda")
        ws = rx.workspace(rx.rslx_act_workspace_bytes(None, net, rows))
        rx.rslx_act(None, net, None, x, rows, 0, 0, None, None, None, out, None, None, rx.ACT_VALUES_ONLY, ws)
        pick = torch.cat([torch.arange(0, rows, 99991, device="cuda"), torch.arange(rows - 200, rows, device="cuda")])
        h = x[pick].double() @ parts[0].double() + parts[1].double()
        ref = (torch.where(h > 0, h, torch.expm1(torch.clamp(h, max=0.0))) @ parts[2].double() + parts[3].double())[:, 0]
        assert float((out[pick].double() - ref).abs().max()) <= 2e-6 * float(ref.abs().max())
        return
    y = torch.empty(rows, 1, device="cuda").normal_(generator=gen)
    g, ref = _bc_grads(rx, dims, flat, x, y).double(), torch.zeros(flat.numel(), dtype=torch.float64, device="cuda")
    for s in range(0, rows, 1 << 21):
        xs = x[s:s + (1 << 21)].double()
        h = xs @ parts[0].double() + parts[1].double()
        e = torch.where(h > 0, h, torch.expm1(torch.clamp(h, max=0.0)))
        d = 2.0 * (e @ parts[2].double() + parts[3].double() - y[s:s + (1 << 21)].double()) / rows
        dz = (d @ parts[2].double().T.contiguous()) * torch.where(h > 0, 1.0, e + 1.0)
        ref += torch.cat([(xs.T.contiguous() @ dz).ravel(), dz.sum(0), (e.T.contiguous() @ d).ravel(), d.sum(0)])
    assert float((g - ref).norm() / ref.norm()) <= 2e-5
