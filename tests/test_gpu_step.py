"""Synthesis and products of a step in one launch (csrc/step.hip) at the edges of
its rule and its tiles: the largest half spectrum, k1 count and padded-grid row
that it takes and the first that it leaves to the two launches, rows of odd
length, rows shorter than the k1 count, one and several tiles per axis.

Every program it serves: shooting, gradient, the incremental sweeps with and
without coupling, the exact adjoint and the deformation chains.  Against the
FP64 oracle at the bounds of the other parity tests: 1e-4 in relative L2."""

import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import Params  # noqa: E402
from oracle import deformation as D  # noqa: E402
from oracle import exact  # noqa: E402
from oracle.jacobi import forward, gradient, hessvec  # noqa: E402
from paper_1807_11560_amd import synth  # noqa: E402

CASES = [
    # grid, band, spectral
    ((8, 32, 32), (6, 32, 32), (9, 48, 48)),
    ((8, 32, 32), (6, 32, 32), (9, 48, 49)),
    ((8, 34, 34), (4, 34, 32), (6, 51, 48)),
    ((8, 32, 34), (4, 32, 34), (6, 48, 51)),
    ((9, 32, 11), (4, 32, 4), (5, 47, 5)),
    ((18, 9, 33), (16, 4, 30), (25, 6, 45)),
]


def rel(t, ref):
    a = t.cpu().numpy().astype(np.complex128 if t.is_complex() else np.float64)
    return float(np.linalg.norm((a - ref).ravel()) / np.linalg.norm(ref.ravel()))


@pytest.mark.parametrize("bf16x3", [False, True])
@pytest.mark.parametrize("grid,band,spectral", CASES)
def test_programs_against_oracle(grid, band, spectral, bf16x3):
    from paper_1807_11560_amd import lddmm as L

    print(f"\n[{grid} {band} {spectral} bf16x3={bf16x3}]", flush=True)
    nt, s = 3, 2
    w = synth.workload(3, grid=grid, band=band)
    p = Params(grid=grid, band=band, nt=nt, alpha=synth.ALPHA, s=s, sigma=synth.SIGMA, spectral=spectral)
    vstar = synth.scale_to_displacement(w["v_star"], grid, 1.0)
    I0, v0, d = w["I0"], 0.5 * vstar, synth.random_direction(3, band)
    vs, _, ms = forward(vstar, I0, p)
    prob = L.Problem(grid=grid, band=band, spectral=spectral, time_steps=nt, alpha=synth.ALPHA, s=s,
                     sigma=synth.SIGMA, precision=L.FP32_BF16X3 if bf16x3 else L.FP32)
    img = lambda x: torch.from_numpy(np.ascontiguousarray(x)).float().cuda()  # noqa: E731
    vec = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(torch.complex64).cuda()  # noqa: E731
    errs = {}
    _, v1 = L.shoot(prob, img(I0), vec(vstar), L.Workspace(prob), want_v1=True)
    errs["v1"] = rel(v1, vs[-1])
    g_ref, _, cache = gradient(v0, I0, ms[-1], p)
    for name, mode, how in (("R1", "R1", L.GN_PAPER), ("R2", "R2", L.GN_CLASSICAL), ("FULL", "FULL", L.NEWTON)):
        q = dataclasses.replace(prob, hessian=how)
        ws = L.Workspace(q)
        g, _ = L.gradient(q, img(I0), img(ms[-1]), vec(v0), ws)
        errs["gradient " + name] = rel(g, g_ref)
        errs["hessvec " + name] = rel(L.hessvec(q, vec(d), ws), hessvec(cache, d, p, mode))
    _, _, ec = exact.gradient(v0, I0, ms[-1], p)
    ref = v0 + exact.adjoint_sweep(ec["vs"], ec["vgrid"], ec["ms"],
                                   2.0 / (p.sigma ** 2 * float(np.prod(p.grid))) * (ec["ms"][-1] - ms[-1]), p,
                                   decisions="fp32")[0]
    g, _ = L.gradient_exact(prob, img(I0), img(ms[-1]), vec(v0), L.Workspace(prob))
    errs["exact"] = rel(g, ref)
    q = dataclasses.replace(prob, state=L.STATE_DEFORMATION)
    ws = L.Workspace(q)
    I1 = D.forward(vstar, I0, p)[2]
    g_ref, _, cache = D.gradient(v0, I0, I1, p)
    g, _ = L.gradient(q, img(I0), img(I1), vec(v0), ws)
    errs["deformation gradient"] = rel(g, g_ref)
    errs["deformation hessvec"] = rel(L.hessvec(q, vec(d), ws), D.hessvec(cache, d, p, "R1"))
    torch.cuda.synchronize()
    print(errs, flush=True)
    assert max(errs.values()) < 1e-4, errs
