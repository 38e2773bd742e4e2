"""GPU: the optimizer step on arrays of any alignment and length.  Four
elements at a time or one at a time, each element's update is the same
arithmetic: without clipping the results are equal bit for bit; the clipping
norm is summed in FP64, so its FP32 value agrees to one unit in the last
place."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def api():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_17164_amd import api as a
    return a


@pytest.mark.parametrize("n", [1, 3, 4, 5, 1023, 262_147])
@pytest.mark.parametrize("off", [(0, 0, 0, 0), (1, 1, 1, 1), (0, 2, 0, 0), (0, 0, 0, 3)])
def test_adam_any_alignment(api, n, off):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    base = [torch.randn(n, device="cuda", generator=gen) for _ in range(4)]
    base[3] = base[3].abs() * 0.01
    ref = [t.clone() for t in base]
    odd = []
    for t, o in zip(base, off):
        room = torch.full((n + 8,), 7.0, device="cuda")
        room[o:o + n] = t
        odd.append(room)
    norms = [torch.zeros(1, device="cuda") for _ in range(2)]
    for clip in (0.0, 0.5):
        api.adam_step_noalloc(ref[0], ref[1], ref[2], ref[3], 3, 1e-3, clip_norm=clip, grad_norm=norms[0])
        view = [room[o:o + n] for room, o in zip(odd, off)]
        api.adam_step_noalloc(*view, 3, 1e-3, clip_norm=clip, grad_norm=norms[1])
        torch.cuda.synchronize()
        assert abs(norms[0].item() - norms[1].item()) <= 2.0 ** -23 * norms[0].item()
        if clip == 0.0:
            for a, b in zip(ref, view):
                assert torch.equal(a, b)
    for room, o in zip(odd, off):  # nothing outside the arrays was written
        assert (room[:o] == 7.0).all() and (room[o + n:] == 7.0).all()
