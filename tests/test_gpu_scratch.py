"""A context's workspace holds whatever its last step left there: a step's
results are the same bits after a step that left NaNs in every buffer as after
an ordinary one, also where there are fewer rows than waves and some waves of
the only workgroup have none."""
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


def ring(n, degree):
    """Receiver i < n with the degree(i) nodes behind it as senders."""
    recv, send = [], []
    for i in range(n):
        s = sorted((i + k) % n for k in range(1, degree(i) + 1))
        recv += [i] * len(s)
        send += s
    return og.Graph(n, np.array(recv, dtype=np.int64), np.array(send, dtype=np.int64))


def step(api, ctx, G, hidden, layers, precision, activation, agg="message", bad=False):
    """One step on ctx; bad: with every parameter NaN.  Returns outputs and gradient."""
    rng = np.random.default_rng(G.n)
    pos = rng.standard_normal((G.n, 3)).astype(np.float32)
    x = rng.standard_normal((G.n, 6)).astype(np.float32)
    target = rng.standard_normal((G.n, 4)).astype(np.float32)
    norm = np.array([[0, 0, 0, 1], [1, 1, 1, 0.5]], dtype=np.float32)
    desc = om.Desc(hidden=hidden, layers=layers, node_in=6, activation=activation)
    params = init_params(om.param_entries(desc), 5)
    if bad:
        params = np.full_like(params, np.nan)
    model = api.Model(hidden, layers, node_in=6, activation=activation, precision=precision, aggregate=agg)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    ps = api.Partset.halo(api.Graph.from_csr(G.row_ptr, G.col), pos, None, layers)
    p, out = dev(params), torch.zeros(G.n, 4, device="cuda")
    d_out, loss, grad = torch.zeros_like(out), torch.zeros(1, device="cuda"), torch.zeros_like(p)
    xd, pd, td = dev(x), dev(pos), dev(target)
    ctx.forward(model, p, ps, [0], xd, pd, norm, out)
    ctx.mse_grad(out, td, G.n, d_out, loss)
    ctx.backward(model, p, d_out, grad)
    torch.cuda.synchronize()
    return out.cpu(), grad.cpu()


def check(api, G, hidden, layers, precision, activation, agg="message"):
    got = []
    for bad in (False, True):
        ctx = api.Context(0)
        step(api, ctx, ring(64, lambda i: 12), hidden, 2, precision, activation, agg, bad)  # larger in every buffer
        got.append(step(api, ctx, G, hidden, layers, precision, activation, agg))
    (out, grad), (out_bad, grad_bad) = got
    log(f"scratch {precision} H={hidden} L={layers} {activation} n={G.n} E={len(G.col)}: "
        f"{int((~torch.isfinite(grad_bad)).sum())} gradient entries not finite")
    assert torch.isfinite(grad).all()
    assert torch.equal(out, out_bad) and torch.equal(grad, grad_bad)


@pytest.mark.parametrize("activation", ["silu", "relu"])
@pytest.mark.parametrize("layers", [1, 2])
@pytest.mark.parametrize("n", [3, 5, 7])
@pytest.mark.parametrize("precision,hidden", [("bf16", 128), ("bf16", 256), ("bf16", 512), ("fp32", 128), ("fp32", 256)])
def test_fewer_nodes_than_waves(api, precision, hidden, n, layers, activation):
    check(api, ring(n, lambda i: n - 1), hidden, layers, precision, activation)


@pytest.mark.parametrize("activation", ["silu", "relu"])
@pytest.mark.parametrize("edges", [1, 3, 7])
@pytest.mark.parametrize("precision,hidden", [("bf16", 128), ("bf16", 256), ("bf16", 512), ("fp32", 128), ("fp32", 256)])
def test_fewer_edges_than_waves(api, precision, hidden, edges, activation):
    """(One layer: the buffer that takes the encoder's pre-activations is then
    not written by the layers.)"""
    check(api, ring(12, lambda i: int(i < edges)), hidden, 1, precision, activation)
