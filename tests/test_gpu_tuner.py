"""What the tuner chooses where no kernel of the step takes edge tiles, and what
it takes from a cache file."""
import numpy as np
import pytest

from cases import Case
from oracle import graph as og

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_17164_amd import api as a
    return a


@pytest.mark.parametrize("hidden", [128, 256])
@pytest.mark.parametrize("keep", [True, False])
def test_tuner_rows(api, tmp_path, hidden, keep):
    """With z on the tape and the gathered forward, edge rows and waves change no
    kernel: the tuner leaves them at the most rows and the default waves whatever
    the timing or a cache line says, so a graph of in-degree 40 runs afterwards.
    With checkpoints only, the adjoint takes them and the line counts."""
    n = 600
    case = Case(1, levels=(n,), hidden=hidden, layers=2, precision="bf16", activation="silu")
    idx = np.arange(n)
    graph = {k: og.Graph(n, np.repeat(idx, k), (np.repeat(idx, k) + np.tile(np.arange(1, k + 1), n)) % n) for k in (8, 40)}
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    ps = {k: api.Partset.halo(api.Graph.from_csr(G.row_ptr, G.col), case.inp.pos, None, case.L) for k, G in graph.items()}
    model, p, node_in, pos = case.model(api), dev(case.params), dev(case.inp.node_in), dev(case.inp.pos)
    out = torch.zeros(n, 4, device="cuda")
    d_out, grad = torch.full_like(out, 1e-3), torch.zeros_like(p)
    cache = tmp_path / "tiles.txt"

    def tune():
        ctx = api.Context(0)
        ctx.set_tape(keep)
        got = ctx.autotune(model, p, ps[8], [0], node_in, pos, case.inp.edge_norm, out, d_out, grad, str(cache))
        return ctx, got

    ctx, (er, nr, grid, wv, _) = tune()
    if keep:
        assert (er, wv) == (64, 4) and ctx.get_bwd_tiles() == (0, 0)
    else:
        assert er in (32, 64) and wv in (4, 8)
    key, _, nr, grid, _, _, _, ms = cache.read_text().split()
    cache.write_text(f"{key} 32 {nr} {grid} 8 64 4 {ms}\n")
    ctx, (er, nr2, grid2, wv, _) = tune()
    assert (nr2, grid2) == (int(nr), int(grid))
    if keep:
        assert (er, wv) == (64, 4) and ctx.get_bwd_tiles() == (0, 0)
        ctx.forward(model, p, ps[40], [0], node_in, pos, case.inp.edge_norm, out)
        torch.cuda.synchronize()
        assert torch.isfinite(out).all()
    else:
        assert (er, wv) == (32, 8) and ctx.get_bwd_tiles() == (64, 4)
