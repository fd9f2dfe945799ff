"""The TV prox with several dual steps a launch (strips marched along y)
against one step a launch: the same expressions in the same order, so equal
bit for bit.  Volumes narrower than a strip, of one row, column or depth,
depths on either side of a thread's positions, step counts that leave every
remainder, warm starts, and inputs with infinities and NaN."""
import numpy as np
import pytest

import synth
from gpu_common import say, torch_cuda

pytestmark = pytest.mark.gpu

# ny, nx, nz, species
SHAPES = [(1, 1, 1, 1), (1, 9, 5, 2), (7, 1, 33, 1), (5, 40, 1, 3), (33, 27, 16, 2), (70, 19, 50, 3),
          (24, 67, 64, 1), (19, 41, 129, 2), (9, 30, 256, 1), (6, 5, 300, 1), (4, 3, 700, 1),
          (61, 300, 8, 1), (130, 90, 96, 2)]


def _plan(monkeypatch, shape, march):
    import paper_2510_23739_amd as pk
    ny, nx, nz, ns = shape
    monkeypatch.setenv("PSOAM_TV_MARCH", str(march))
    t0, taps = synth.random_table(nz, 1, 4, 2, np.random.default_rng(1), t0_lo=0, t0_hi=3)
    return pk.Plan(nx, ny, nz, 2, 4, 1, synth.phi_depth(nz), synth.species(ns), t0, taps, prec="bf16")


def _same(torch, a, b):
    return bool(((a == b) | (torch.isnan(a) & torch.isnan(b))).all())


@pytest.mark.parametrize("march", [2, 3, 4])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_equals_single_steps(shape, march, monkeypatch):
    torch = torch_cuda()
    ny, nx, nz, ns = shape
    say(f"[tv march] {shape} {march} steps")
    g = torch.Generator(device="cuda").manual_seed(7)
    z = torch.randn(ns, ny, nx, nz, device="cuda", generator=g)
    odd = z.clone()
    odd.view(-1)[:: max(1, odd.numel() // 5)] = float("nan")
    odd.view(-1)[odd.numel() // 2] = float("inf")
    one, many = _plan(monkeypatch, shape, 1), _plan(monkeypatch, shape, march)
    for n in (0, 1, 2, 3, 4, 5, 6, 9):
        for zz in (z, odd):
            a = one.prox_tv(zz, 0.1, n, nonneg=True)
            b = many.prox_tv(zz, 0.1, n, nonneg=True)
            assert _same(torch, a, b), n
            assert _same(torch, a, many.prox_tv_noalloc(zz, 0.1, n, nonneg=True)), n
    p = torch.randn(one.y_shape, device="cuda", generator=g)
    o = dict(lambda_tv=0.05, k1=4, k2=5, alpha1=0.3)
    for warm in (False, True):
        a, _ = one.solve(p, warm_inner=warm, **o)
        b, _ = many.solve(p, warm_inner=warm, **o)
        assert torch.equal(a, b), warm
    one.close()
    many.close()
