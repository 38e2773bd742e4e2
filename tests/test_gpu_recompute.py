"""The edge adjoint that recomputes z from the checkpoints, at every tile height
and wave count it has at each width: against the adjoint with z on the tape,
and under SiLU against the oracle."""
from __future__ import annotations

import functools

import numpy as np
import pytest

from cases import Case, check_step, log, oracle_refs, per_tensor_errors

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_17164_amd import api as a
    return a


@functools.lru_cache(maxsize=None)
def the_case(hidden, precision, activation, aggregate):
    cfg, levels = {128: (3, (500, 2000, 6000)), 256: (5, (400, 1600, 5000)), 512: (6, (200, 800, 2500))}[hidden]
    return Case(cfg, levels=levels, hidden=hidden, layers=3, precision=precision, activation=activation,
                aggregate=aggregate)


@functools.lru_cache(maxsize=None)
def the_refs(*key):
    return oracle_refs(the_case(*key))


def step(api, ctx, case):
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    p, node_in, pos = dev(case.params), dev(case.inp.node_in), dev(case.inp.pos)
    g = ctx.build_knn(pos, case.levels, case.k_intra, case.k_cross)
    ps = api.Partset.halo(g, case.inp.pos, None, case.L)
    out, loss = torch.zeros(case.N, 4, device="cuda"), torch.zeros(1, device="cuda")
    d_out, grad = torch.zeros_like(out), torch.full_like(p, float("nan"))
    ctx.forward(case.model(api), p, ps, [0], node_in, pos, case.inp.edge_norm, out)
    ctx.mse_grad(out, dev(case.inp.targets), case.N, d_out, loss)
    ctx.backward(case.model(api), p, d_out, grad)
    torch.cuda.synchronize()
    return out.cpu().numpy(), float(loss.item()), grad.cpu().numpy()


_kept = {}


@pytest.mark.parametrize("activation,aggregate", [("silu", "message"), ("relu", "message"), ("relu", "edge")])
@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("precision,hidden,rows,adjoint", [
    ("bf16", 128, 32, 0), ("bf16", 128, 64, 0), ("bf16", 128, 64, 32), ("bf16", 128, 32, 64),
    ("bf16", 256, 32, 0), ("bf16", 256, 64, 0), ("bf16", 256, 128, 64), ("bf16", 512, 32, 0),
    ("fp32", 128, 32, 0), ("fp32", 128, 64, 0), ("fp32", 256, 32, 0),
])
def test_recompute_tiles(api, precision, hidden, rows, adjoint, waves, activation, aggregate):
    """The forward is the same bits; every gradient tensor is within 5e-3 (FP32
    1e-5) of the tape's, the bars of the tape policy; the step meets its own."""
    key = (hidden, precision, activation, aggregate)
    case = the_case(*key)
    log(f"recompute {precision} H={hidden} rows {rows}/{adjoint} waves {waves} {activation} {aggregate}")
    if key not in _kept:
        _kept[key] = step(api, api.Context(0), case)
    ctx = api.Context(0)
    ctx.set_tape(False)
    ctx.set_tiles(rows, 0, 0, waves)
    ctx.set_bwd_tiles(adjoint, waves)
    got = step(api, ctx, case)
    assert (got[0] == _kept[key][0]).all()
    errs = per_tensor_errors(case, got[2], _kept[key][2])
    worst = sorted(errs.items(), key=lambda kv: -kv[1])[:3]
    log(f"  against the tape: {worst}")
    assert worst[0][1] <= (5e-3 if precision == "bf16" else 1e-5), worst
    if activation == "silu":
        log("  " + check_step(case, *got, the_refs(*key)))
