"""What a training step's device workspace grows by per node and edge: the
buffers of the layout, and nothing beside them."""
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


def step_memory(api, n, degree, precision, hidden, layers):
    idx = np.arange(n)
    G = og.Graph(n, np.repeat(idx, degree), (np.repeat(idx, degree) + np.tile(np.arange(1, degree + 1), n)) % n)
    rng = np.random.default_rng(1)
    pos = rng.standard_normal((n, 3)).astype(np.float32)
    norm = np.array([[0, 0, 0, 1], [1, 1, 1, 0.5]], dtype=np.float32)
    params = init_params(om.param_entries(om.Desc(hidden=hidden, layers=layers)), 5)
    model = api.Model(hidden, layers, precision=precision)
    ctx = api.Context(0)
    ps = api.Partset.halo(api.Graph.from_csr(G.row_ptr, G.col), pos, None, layers)
    p, out = torch.from_numpy(params).cuda(), torch.zeros(n, 4, device="cuda")
    grad, x, pd = torch.zeros_like(p), torch.randn(n, 6, device="cuda"), torch.from_numpy(pos).cuda()
    d_out = torch.full_like(out, 1e-3)
    ctx.forward(model, p, ps, [0], x, pd, norm, out)
    ctx.backward(model, p, d_out, grad)
    torch.cuda.synchronize()
    return ctx.memory()


@pytest.mark.parametrize("precision,hidden", [("bf16", 128), ("bf16", 256), ("fp32", 128)])
def test_workspace_per_node(api, precision, hidden):
    """From n to 2 n nodes of in-degree 8 (the per-workgroup buffers do not grow
    any more), one layer: tape h 2, m 1 (FP32), e and z 8 each; backward dh, dh_mid,
    dm, S_r, S_s (FP32), de twice 8 (FP32), four factors of 8; edge features, dy
    and the batch plan (under 200 bytes a node).  Rows of H."""
    n, k, L = 20_000, 8, 1
    grown = (step_memory(api, 2 * n, k, precision, hidden, L) - step_memory(api, n, k, precision, hidden, L)) / n
    s = 2 if precision == "bf16" else 4
    rows = hidden * (s * ((L + 1) + 2 * k * L + 4 * k) + 4 * (L + 5 + 2 * k))
    log(f"workspace {precision} H={hidden}: {grown:.0f} bytes a node, rows of the layout {rows}")
    assert rows <= grown <= rows + 16 * k + 64 + 200
