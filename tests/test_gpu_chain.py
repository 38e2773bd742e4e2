"""The edge and encoder kernels where their work split can go wrong: a wave
takes whole receiver segments 16 edges at a time, so segments that straddle
16-edge groups and tile ends, receivers without in-edges, and edge counts
around one group and one workgroup's share are held against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from cases import Case, log, oracle_refs, rel_l2
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


def degree_graph(n, degrees, seed):
    """Graph on n nodes whose receiver i has degrees[i % len(degrees)] random senders."""
    rng = np.random.default_rng(seed)
    recv, send = [], []
    for i in range(n):
        d = min(degrees[i % len(degrees)], n - 1)
        s = rng.choice(n - 1, size=d, replace=False)
        s = np.sort(np.where(s >= i, s + 1, s))
        recv.append(np.full(d, i, dtype=np.int64))
        send.append(s.astype(np.int64))
    return og.Graph(n, np.concatenate(recv), np.concatenate(send))


@pytest.mark.parametrize("act,agg", [("silu", "message"), ("silu", "edge"), ("relu", "message"), ("relu", "edge")])
@pytest.mark.parametrize("n,degrees", [
    (8, [1, 0]),                # less than one group
    (40, [16]),                 # every group exactly one segment
    (33, [15, 1, 17]),          # segments around a group's end
    (70, [31, 0, 0, 2, 32]),    # segments over three groups, runs of empty receivers
    (130, [1]),                 # a receiver per edge
    (515, [0, 9, 7, 0, 12]),    # a ragged last group in many workgroups
])
@pytest.mark.parametrize("hidden", [128, 256, 512])
def test_chain_edges(api, hidden, n, degrees, act, agg):
    """Outputs within 2e-2 of the oracle at the BF16-cast weights (the bar of
    the BF16 form), and under SiLU the whole gradient too (under ReLU a
    cloud this small has single kinks that BF16 rounding flips)."""
    case = Case(1, levels=(n,), hidden=hidden, layers=2, precision="bf16", activation=act, aggregate=agg)
    G = degree_graph(n, degrees, 7)
    case._graph = G
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    ctx = api.Context(0)
    ps = api.Partset.halo(api.Graph.from_csr(G.row_ptr, G.col), case.inp.pos, None, case.L)
    p, node_in, pos, target = dev(case.params), dev(case.inp.node_in), dev(case.inp.pos), dev(case.inp.targets)
    out = torch.full((n, 4), float("nan"), device="cuda")
    d_out, loss, grad = torch.zeros_like(out), torch.zeros(1, device="cuda"), torch.full_like(p, float("nan"))
    log(f"chain H={hidden} n={n} E={len(G.col)} {act} {agg}")
    ctx.forward(case.model(api), p, ps, [0], node_in, pos, case.inp.edge_norm, out)
    ctx.mse_grad(out, target, n, d_out, loss)
    ctx.backward(case.model(api), p, d_out, grad)
    torch.cuda.synchronize()
    _, (_, y, g) = oracle_refs(case)
    e_out, e_grad = rel_l2(out.cpu().numpy(), y), rel_l2(grad.cpu().numpy(), g)
    log(f"  out {e_out:.2e} grad {e_grad:.2e}")
    assert np.isfinite(grad.cpu().numpy()).all()
    assert e_out <= 2e-2
    if act == "silu":
        assert e_grad <= 2e-2
    # a forward without a tape gives the same bits
    free = torch.zeros_like(out)
    ctx.forward(case.model(api), p, ps, [0], node_in, pos, case.inp.edge_norm, free, keep_tape=False)
    torch.cuda.synchronize()
    assert torch.equal(free, out)


@pytest.mark.parametrize("agg", ["message", "edge"])
@pytest.mark.parametrize("n,degrees", [
    (8, [1, 0]),                # less than one group
    (70, [31, 0, 0, 2, 32]),    # segments over three groups, runs of empty receivers
    (1024, [12]),               # the most edges that four-wave workgroups take at H = 128
    (1025, [12]),               # and the first that eight waves take
])
@pytest.mark.parametrize("hidden", [128, 256])
def test_fp32_edges(api, hidden, n, degrees, agg):
    """The FP32 form under SiLU at its bar: outputs and whole gradient within
    1e-4 of the oracle."""
    case = Case(1, levels=(n,), hidden=hidden, layers=2, precision="fp32", activation="silu", aggregate=agg)
    G = degree_graph(n, degrees, 7)
    case._graph = G
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    ctx = api.Context(0)
    ps = api.Partset.halo(api.Graph.from_csr(G.row_ptr, G.col), case.inp.pos, None, case.L)
    p, node_in, pos, target = dev(case.params), dev(case.inp.node_in), dev(case.inp.pos), dev(case.inp.targets)
    out = torch.full((n, 4), float("nan"), device="cuda")
    d_out, loss, grad = torch.zeros_like(out), torch.zeros(1, device="cuda"), torch.full_like(p, float("nan"))
    log(f"fp32 H={hidden} n={n} E={len(G.col)} {agg}")
    ctx.forward(case.model(api), p, ps, [0], node_in, pos, case.inp.edge_norm, out)
    ctx.mse_grad(out, target, n, d_out, loss)
    ctx.backward(case.model(api), p, d_out, grad)
    torch.cuda.synchronize()
    (_, y, g), _ = oracle_refs(case)
    e_out, e_grad = rel_l2(out.cpu().numpy(), y), rel_l2(grad.cpu().numpy(), g)
    log(f"  out {e_out:.2e} grad {e_grad:.2e}")
    assert e_out <= 1e-4 and e_grad <= 1e-4


@pytest.mark.parametrize("precision,hidden", [("bf16", 128), ("bf16", 256), ("bf16", 512), ("fp32", 128), ("fp32", 256)])
def test_rows_in_several_steps(api, precision, hidden):
    """So many nodes that every wave takes its rows in two or more 16-row steps,
    the last one ragged, two layers (the lower layer's node adjoint starts from
    the sums of the upper layer's edges), SiLU, at the form's bar (outputs and
    whole gradient 2e-2 or 1e-4)."""
    n = 33001
    case = Case(1, levels=(n,), hidden=hidden, layers=2, precision=precision, activation="silu")
    rng = np.random.default_rng(2)
    case._graph = G = og.Graph(n, np.arange(n, dtype=np.int64), (np.arange(n) + rng.integers(1, n, n)) % n)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    ctx = api.Context(0)
    ps = api.Partset.halo(api.Graph.from_csr(G.row_ptr, G.col), case.inp.pos, None, case.L)
    p, out = dev(case.params), torch.full((n, 4), float("nan"), device="cuda")
    d_out, loss, grad = torch.zeros_like(out), torch.zeros(1, device="cuda"), torch.full_like(p, float("nan"))
    ctx.forward(case.model(api), p, ps, [0], dev(case.inp.node_in), dev(case.inp.pos), case.inp.edge_norm, out)
    ctx.mse_grad(out, dev(case.inp.targets), n, d_out, loss)
    ctx.backward(case.model(api), p, d_out, grad)
    torch.cuda.synchronize()
    log(f"steps {precision} H={hidden}: the oracle")
    base, amp = oracle_refs(case)
    _, y, g = amp or base
    e_out, e_grad = rel_l2(out.cpu().numpy(), y), rel_l2(grad.cpu().numpy(), g)
    log(f"  out {e_out:.2e} grad {e_grad:.2e}")
    bar = 2e-2 if precision == "bf16" else 1e-4
    assert e_out <= bar and e_grad <= bar


@pytest.mark.parametrize("hidden", [256, 512])
@pytest.mark.parametrize("node_in", [1, 8, 12, 32])
def test_stream_encoder_inputs(api, hidden, node_in):
    """The streamed encoders at every way they take the node inputs (1 and 8 in
    LDS, 12 and 32 from memory) and a ragged last group of rows, SiLU, held to
    the bar of the BF16 form (outputs and whole gradient 2e-2)."""
    inputs_step(api, "bf16", hidden, node_in, 77, 2e-2)


@pytest.mark.parametrize("precision,hidden,node_in,n", [
    ("bf16", 128, 12, 65), ("bf16", 128, 32, 127), ("bf16", 256, 24, 129), ("bf16", 512, 32, 64),
    ("fp32", 128, 12, 33), ("fp32", 128, 32, 31), ("fp32", 256, 20, 32), ("fp32", 128, 4, 2), ("bf16", 128, 8, 2),
])
def test_weight_gradient_rows(api, precision, hidden, node_in, n):
    """The weight-gradient products at row counts around one stage (64 rows,
    FP32 32), gathered node inputs of any width included, at the form's bar."""
    inputs_step(api, precision, hidden, node_in, n, 2e-2 if precision == "bf16" else 1e-4)


def inputs_step(api, precision, hidden, node_in, n, bar):
    rng = np.random.default_rng(node_in)
    G = degree_graph(n, [3, 5, 1], 3)
    pos = rng.standard_normal((n, 3)).astype(np.float32)
    x = rng.standard_normal((n, node_in)).astype(np.float32)
    target = rng.standard_normal((n, 4)).astype(np.float32)
    norm = np.array([[0, 0, 0, 1], [1, 1, 1, 0.5]], dtype=np.float32)
    desc = om.Desc(hidden=hidden, layers=1, node_in=node_in, activation="silu")
    params = init_params(om.param_entries(desc), 5)
    model = api.Model(hidden, 1, node_in=node_in, activation="silu", precision=precision)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    ctx = api.Context(0)
    ps = api.Partset.halo(api.Graph.from_csr(G.row_ptr, G.col), pos, None, 1)
    p, out = dev(params), torch.zeros(n, 4, device="cuda")
    d_out, loss, grad = torch.zeros_like(out), torch.zeros(1, device="cuda"), torch.zeros_like(p)
    xd, pd = dev(x), dev(pos)
    ctx.forward(model, p, ps, [0], xd, pd, norm, out)
    ctx.mse_grad(out, dev(target), n, d_out, loss)
    ctx.backward(model, p, d_out, grad)
    torch.cuda.synchronize()
    cast = om.amp_cast(desc, params) if precision == "bf16" else params.astype(np.float64)
    _, y, g = om.step_full(desc, cast, G, x, pos, norm, target)
    e_out, e_grad = rel_l2(out.cpu().numpy(), y), rel_l2(grad.cpu().numpy(), g)
    log(f"inputs {precision} H={hidden} node_in={node_in}: out {e_out:.2e} grad {e_grad:.2e}")
    assert e_out <= bar and e_grad <= bar
