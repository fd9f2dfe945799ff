"""Workspaces of the TV prox: one that holds three dual buffers and not four takes
single steps inside its bounds, a smaller one is refused; and a solve whose
scratch does not fit with the fourth buffer runs without it."""
import numpy as np
import pytest

import synth
from gpu_common import leave_free, say, torch_cuda

pytestmark = pytest.mark.gpu


def _plan(nx, ny, nz, ns):
    import paper_2510_23739_amd as pk
    t0, taps = synth.random_table(nz, 1, 4, 2, np.random.default_rng(1), t0_lo=0, t0_hi=3)
    return pk.Plan(nx, ny, nz, 2, 4, 1, synth.phi_depth(nz), synth.species(ns), t0, taps, prec="bf16")


@pytest.mark.parametrize("shape", [(33, 27, 16, 2), (7, 5, 3, 1)])
def test_smaller_workspace_stays_in_bounds(shape):
    torch = torch_cuda()
    import paper_2510_23739_amd as pk
    p = _plan(*shape)
    n = int(np.prod(p.c_shape))
    z = torch.randn(p.c_shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    want = p.prox_tv(z, 0.1, 7)
    full = int(pk.load().psoam_prox_tv_ws_bytes(p.handle)) // 4
    for floats in (full, 10 * n + 256, 9 * n + 2 * 63):
        say(f"[workspace] {shape} {floats} of {full} floats")
        buf = torch.full((floats + 4 * n + 64,), 3.5, device="cuda")
        # (a storage of its own size: what the binding may use)
        ws = torch.tensor([], device="cuda").set_(buf.untyped_storage()[:4 * floats])
        assert torch.equal(p.prox_tv(z, 0.1, 7, ws=ws), want)
        assert (buf[floats:] == 3.5).all()
    with pytest.raises(pk.PsoamError):
        p.prox_tv(z, 0.1, 7, ws=torch.empty(9 * n - 1, device="cuda"))
    p.close()


def test_solve_without_room_for_the_fourth_buffer():
    """400 x 400 x 400 voxels, 2 species: scratch of 9.2 GB with the fourth dual
    buffer and of 7.7 GB without, on a card with 8.4 GB left."""
    torch = torch_cuda()
    shape, o = (400, 400, 400, 2), dict(lambda_tv=0.05, k1=2, k2=5, alpha1=0.3)
    g = torch.Generator(device="cuda").manual_seed(1)
    p = _plan(*shape)
    y = torch.randn(p.y_shape, device="cuda", generator=g)
    want, _ = p.solve(y, **o)
    p.close()
    p, c = _plan(*shape), torch.zeros(p.c_shape, device="cuda")
    rest = leave_free(torch, int(8.4e9))
    if rest is None:
        pytest.skip("the card is in use")
    say(f"[workspace] {torch.cuda.mem_get_info()[0] / 1e9:.2f} GB left")
    p.solve(y, c=c, **o)
    del rest
    assert torch.equal(c, want)
    p.close()
    torch.cuda.empty_cache()
