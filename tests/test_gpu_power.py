"""The power iteration's dot products and scaling: sizes below one workgroup,
at its edge, of several, and beyond one value a thread, against the same
iteration written with A, A^T and FP64 norms.  Lambda is a quotient of sums of
the same FP32 operator outputs: 1e-5 is ten times an FP32 operator's error."""
import numpy as np
import pytest

import synth
from gpu_common import say, torch_cuda

pytestmark = pytest.mark.gpu

# nx, ny, nz, species: 6, 255, 256, 257, 270000 values
SHAPES = [(3, 2, 1, 1), (17, 5, 3, 1), (16, 8, 2, 1), (257, 1, 1, 1), (90, 50, 30, 2)]


@pytest.mark.parametrize("n_power", [1, 5])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_lambda_equals_the_iteration(shape, n_power):
    torch = torch_cuda()
    import paper_2510_23739_amd as pk
    nx, ny, nz, ns = shape
    say(f"[power] {shape} {n_power} iterations")
    rng = np.random.default_rng(3)
    t0, taps = synth.random_table(nz, 3, 24, 4, rng, t0_lo=0, t0_hi=20)
    p = pk.Plan(nx, ny, nz, 3, 24, 3, synth.phi_depth(nz), synth.species(ns), t0, taps, prec="fp32")
    g = torch.Generator(device="cuda").manual_seed(5)
    v0 = torch.randn(p.c_shape, device="cuda", generator=g)
    y = torch.randn(p.y_shape, device="cuda", generator=g)
    _, st = p.solve(y, lambda_tv=0.0, k1=1, k2=1, n_power=n_power, v0=v0)
    v = (v0.double() / v0.double().norm()).float()
    for _ in range(n_power):
        w = p.apply_AT(p.apply_A(v))
        lam = float((v.double() * w.double()).sum())
        v = (w.double() / w.double().norm()).float()
    assert abs(st["lambda_max"] - lam) <= 1e-5 * abs(lam)
    p.close()
