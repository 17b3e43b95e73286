"""FP32 sums stay FP32 sums: the kernels of the shapes without instantiated ones (csrc/chain.hip) and the one-launch
step (csrc/step.hip) against the FP64 oracle at 1e-5, at the shapes of test_gpu_chain.py and test_gpu_step.py, whose
own bound (1e-4) holds both precisions.

The bound: a step passes six transform stages of at most 128 products each, whose FP32 rounding (2^-24 an addition)
adds up to sqrt(128) 2^-24 = 7e-7 of a stage's sum, sqrt(6) times that over a step's stages, 1.7e-6, and at most
linearly over the two or three steps of a sweep and its adjoint: 1e-5.  A product of split BF16 operands drops
2^-16 = 1.5e-5 of itself before any sum."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import Params  # noqa: E402
from oracle import deformation as D  # noqa: E402
from oracle.jacobi import forward, gradient, hessvec  # noqa: E402
from paper_1807_11560_amd import synth  # noqa: E402

CASES = [
    # grid, band, spectral
    ((8, 9, 11), (4, 6, 4), (5, 7, 6)),
    ((17, 33, 18), (14, 18, 16), (21, 27, 24)),
    ((35, 16, 34), (34, 16, 34), (51, 24, 49)),
    ((24, 40, 31), (24, 24, 24), (37, 36, 36)),
    ((64, 12, 65), (64, 4, 64), (94, 5, 96)),
    ((20, 66, 23), (18, 64, 20), (26, 97, 28)),
    ((8, 32, 32), (6, 32, 32), (9, 48, 48)),
    ((8, 32, 32), (6, 32, 32), (9, 48, 49)),
    ((8, 34, 34), (4, 34, 32), (6, 51, 48)),
    ((9, 32, 11), (4, 32, 4), (5, 47, 5)),
    ((18, 9, 33), (16, 4, 30), (25, 6, 45)),
]


def rel(t, ref):
    a = t.cpu().numpy().astype(np.complex128 if t.is_complex() else np.float64)
    return float(np.linalg.norm((a - ref).ravel()) / np.linalg.norm(ref.ravel()))


@pytest.mark.parametrize("grid,band,spectral", CASES)
def test_fp32_against_oracle(grid, band, spectral):
    from paper_1807_11560_amd import lddmm as L

    print(f"\n[{grid} {band} {spectral}]", flush=True)
    nt, s = 2, 2
    w = synth.workload(3, grid=grid, band=band)
    p = Params(grid=grid, band=band, nt=nt, alpha=synth.ALPHA, s=s, sigma=synth.SIGMA, spectral=spectral)
    vstar = synth.scale_to_displacement(w["v_star"], grid, 1.0)
    I0, v0, d = w["I0"], 0.5 * vstar, synth.random_direction(3, band)
    img = lambda x: torch.from_numpy(np.ascontiguousarray(x)).float().cuda()  # noqa: E731
    vec = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(torch.complex64).cuda()  # noqa: E731
    errs = {}
    for name, state, fwd, grad, hess in (("image", L.STATE_IMAGE, forward, gradient, hessvec),
                                         ("deformation", L.STATE_DEFORMATION, D.forward, D.gradient, D.hessvec)):
        prob = L.Problem(grid=grid, band=band, spectral=spectral, time_steps=nt, alpha=synth.ALPHA, s=s,
                         sigma=synth.SIGMA, state=state)
        ws = L.Workspace(prob)
        out = fwd(vstar, I0, p)
        m1 = out[2][-1] if state == L.STATE_IMAGE else out[2]
        errs[name + " m1"] = rel(L.shoot(prob, img(I0), vec(vstar), ws), m1)
        ref, _, cache = grad(v0, I0, m1, p)
        g, _ = L.gradient(prob, img(I0), img(m1), vec(v0), ws)
        errs[name + " gradient"] = rel(g, ref)
        errs[name + " hessvec"] = rel(L.hessvec(prob, vec(d), ws), hess(cache, d, p, "R1"))
    torch.cuda.synchronize()
    print(errs, flush=True)
    assert max(errs.values()) < 1e-5, errs
