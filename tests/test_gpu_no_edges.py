"""A batch without a single edge: every message is an empty sum, and the edge
MLPs' and the edge encoder's gradients are zero."""
from __future__ import annotations

import numpy as np
import pytest

from cases import log, rel_l2
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


@pytest.mark.parametrize("form", ["keep", "recompute", "split"])
@pytest.mark.parametrize("precision,hidden", [("bf16", 128), ("bf16", 256), ("bf16", 512), ("fp32", 128), ("fp32", 256)])
def test_no_edges(api, precision, hidden, form):
    """At the form's bar against the oracle (SiLU, outputs and whole gradient)."""
    n = 77
    none = np.zeros(0, dtype=np.int64)
    G = og.Graph(n, none, none)
    rng = np.random.default_rng(4)
    pos = rng.standard_normal((n, 3)).astype(np.float32)
    x = rng.standard_normal((n, 6)).astype(np.float32)
    target = rng.standard_normal((n, 4)).astype(np.float32)
    norm = np.array([[0, 0, 0, 1], [1, 1, 1, 0.5]], dtype=np.float32)
    desc = om.Desc(hidden=hidden, layers=2, node_in=6, activation="silu")
    params = init_params(om.param_entries(desc), 5)
    model = api.Model(hidden, 2, node_in=6, activation="silu", precision=precision)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    ctx = api.Context(0)
    ctx.set_tape(form != "recompute")
    ctx.set_edge_split(form == "split")
    ps = api.Partset.halo(api.Graph.from_csr(G.row_ptr, G.col), pos, None, 2)
    p, out = dev(params), torch.full((n, 4), float("nan"), device="cuda")
    d_out, loss, grad = torch.zeros_like(out), torch.zeros(1, device="cuda"), torch.full_like(p, float("nan"))
    xd, pd, td = dev(x), dev(pos), dev(target)
    ctx.forward(model, p, ps, [0], xd, pd, norm, out)
    ctx.mse_grad(out, td, n, d_out, loss)
    ctx.backward(model, p, d_out, grad)
    torch.cuda.synchronize()
    cast = om.amp_cast(desc, params) if precision == "bf16" else params.astype(np.float64)
    _, y, g = om.step_full(desc, cast, G, x, pos, norm, target)
    e_out, e_grad = rel_l2(out.cpu().numpy(), y), rel_l2(grad.cpu().numpy(), g)
    log(f"no edges {precision} H={hidden} {form}: out {e_out:.2e} grad {e_grad:.2e}")
    bar = 2e-2 if precision == "bf16" else 1e-4
    assert e_out <= bar and e_grad <= bar
    got, off = grad.cpu().numpy(), 0
    for b, _, s in om.layout(desc):
        cnt = int(np.prod(s))
        if b.startswith("edge") or b == "enc_edge":
            assert (got[off:off + cnt] == 0).all(), b
        off += cnt
