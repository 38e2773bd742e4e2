"""Forwards of few rows run on tiles, larger ones as chains and streams: a row's
result is the same bits either way, also at the line between the two."""
from __future__ import annotations

import numpy as np
import pytest

from cases import log
from oracle import graph as og
from oracle import model as om
from synth import init_params

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_17164_amd import api as a
    return a


def forward(api, recv, send, n, pos, x, hidden, activation, agg, precision="fp32"):
    desc = om.Desc(hidden=hidden, layers=2, node_in=x.shape[1], activation=activation, aggregate=agg)
    params = torch.from_numpy(init_params(om.param_entries(desc), 5)).cuda()
    model = api.Model(hidden, 2, node_in=x.shape[1], activation=activation, precision=precision, aggregate=agg)
    norm = np.array([[0, 0, 0, 1], [1, 1, 1, 0.5]], dtype=np.float32)
    G = og.Graph(n, recv, send)
    ctx = api.Context(0)
    ps = api.Partset.halo(api.Graph.from_csr(G.row_ptr, G.col), pos, None, 2)
    out = torch.full((n, 4), float("nan"), device="cuda")
    free = torch.full_like(out, float("nan"))
    xd, pd = torch.from_numpy(x).cuda(), torch.from_numpy(pos).cuda()
    ctx.forward(model, params, ps, [0], xd, pd, norm, out)
    ctx.forward(model, params, ps, [0], xd, pd, norm, free, keep_tape=False)
    torch.cuda.synchronize()
    assert torch.equal(out, free)
    return out


@pytest.mark.parametrize("agg", ["message", "edge"])
@pytest.mark.parametrize("activation", ["silu", "relu"])
@pytest.mark.parametrize("precision,hidden,node_in", [("fp32", 128, 6), ("fp32", 256, 6), ("fp32", 256, 24), ("bf16", 128, 6),
                                                       ("bf16", 256, 6), ("bf16", 512, 6)])
@pytest.mark.parametrize("degrees", [[1, 0, 2], [6], [24, 3, 9, 0, 6, 15], [31, 30]])
def test_copies(api, precision, hidden, node_in, degrees, activation, agg):
    """A graph of 530 nodes alone and as so many disjoint copies (over 2^17 edges and
    8,192 nodes) that no kernel takes tiles."""
    n = 530
    rng = np.random.default_rng(len(degrees))
    deg = np.array([degrees[i % len(degrees)] for i in range(n)])
    recv = np.repeat(np.arange(n), deg)
    send = (recv + 1 + np.concatenate([rng.choice(n - 1, d, replace=False) for d in deg])) % n
    pos = rng.standard_normal((n, 3)).astype(np.float32)
    x = rng.standard_normal((n, node_in)).astype(np.float32)
    one = forward(api, recv, send, n, pos, x, hidden, activation, agg, precision)
    k = max(8193 // n, (1 << 17) // len(recv)) + 1
    shift = np.repeat(np.arange(k) * n, len(recv))
    many = forward(api, np.tile(recv, k) + shift, np.tile(send, k) + shift, n * k, np.tile(pos, (k, 1)),
                   np.tile(x, (k, 1)), hidden, activation, agg, precision)
    log(f"few rows {precision} H={hidden} E={len(recv)} x {k} {activation} {agg}")
    assert torch.isfinite(one).all()
    assert all(torch.equal(one, c) for c in many.view(k, n, 4))


@pytest.mark.parametrize("n", [31, 32, 33, 8191, 8192])
def test_line(api, n):
    """One more node without edges: around one tile, and from the most rows that tiles
    take at H = 256 to the first that stream."""
    rng = np.random.default_rng(n)
    recv = np.arange(n)
    send = (recv + rng.integers(1, n, n)) % n
    pos = rng.standard_normal((n + 1, 3)).astype(np.float32)
    x = rng.standard_normal((n + 1, 6)).astype(np.float32)
    a = forward(api, recv, send, n, pos[:n].copy(), x[:n].copy(), 256, "silu", "message")
    b = forward(api, recv, send, n + 1, pos, x, 256, "silu", "message")
    assert torch.isfinite(b).all() and torch.equal(a, b[:n])


@pytest.mark.parametrize("precision,hidden", [("fp32", 256), ("fp32", 128), ("bf16", 128), ("bf16", 512)])
@pytest.mark.parametrize("n", [40, 9000])
def test_params_anywhere(api, precision, hidden, n):
    """Parameters, inputs and results that begin at any element: the same bits."""
    rng = np.random.default_rng(n)
    recv = np.repeat(np.arange(n), 2)
    send = (recv + rng.integers(1, n, len(recv))) % n
    G = og.Graph(n, recv, send)
    pos = rng.standard_normal((n, 3)).astype(np.float32)
    desc = om.Desc(hidden=hidden, layers=1, node_in=6, activation="silu")
    model = api.Model(hidden, 1, node_in=6, activation="silu", precision=precision)
    norm = np.array([[0, 0, 0, 1], [1, 1, 1, 0.5]], dtype=np.float32)
    params, x = init_params(om.param_entries(desc), 5), rng.standard_normal((n, 6)).astype(np.float32)
    ps = api.Partset.halo(api.Graph.from_csr(G.row_ptr, G.col), pos, None, 1)
    got = []
    for off in (0, 1, 3):
        def at(a):
            room = torch.zeros(a.size + 8, device="cuda")
            room[off:off + a.size] = torch.from_numpy(a.reshape(-1)).cuda()
            return room[off:off + a.size].view(a.shape)
        ctx = api.Context(0)
        p, xd, pd = at(params), at(x), at(pos)
        out, grad, d_out = at(np.zeros((n, 4), np.float32)), at(np.zeros_like(params)), at(np.full((n, 4), 1e-3, np.float32))
        ctx.forward(model, p, ps, [0], xd, pd, norm, out)
        ctx.backward(model, p, d_out, grad)
        torch.cuda.synchronize()
        got.append((out.clone(), grad.clone()))
    assert torch.isfinite(got[0][1]).all()
    for out, grad in got[1:]:
        assert torch.equal(out, got[0][0]) and torch.equal(grad, got[0][1])
