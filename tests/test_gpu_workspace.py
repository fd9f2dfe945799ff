"""Workspaces of the TV prox: one that holds three dual buffers and not four takes
single steps inside its bounds, a smaller one is refused."""
import numpy as np
import pytest

import synth
from gpu_common import say, torch_cuda

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
