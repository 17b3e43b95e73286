"""The kernels of the shapes without instantiated ones (csrc/chain.hip) at the
edges of their tiles: bands around a multiple of 16 (4, 14, 16, 18, 34, 64 per
axis), padded grids around a multiple of 16 and of odd length (rows of odd
length end in a load that begins one value earlier), half spectra of one and of two tiles, grids
with a ragged last tile on every axis and rows that are not a multiple of four.

Oracle and bounds are those of the other parity tests: the FP64 oracle, 1e-4 in
relative L2 for shooting, gradient and Hessian-vector product."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import Params  # noqa: E402
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
]


def rel(t, ref):
    a = t.cpu().numpy().astype(np.complex128 if t.is_complex() else np.float64)
    return float(np.linalg.norm((a - ref).ravel()) / np.linalg.norm(ref.ravel()))


@pytest.mark.parametrize("bf16x3", [False, True])
@pytest.mark.parametrize("grid,band,spectral", CASES)
def test_tile_edges_against_oracle(grid, band, spectral, bf16x3):
    from paper_1807_11560_amd import lddmm as L

    print(f"\n[{grid} {band} {spectral} bf16x3={bf16x3}]", flush=True)
    nt, s = 2, 2
    w = synth.workload(3, grid=grid, band=band)
    p = Params(grid=grid, band=band, nt=nt, alpha=synth.ALPHA, s=s, sigma=synth.SIGMA, spectral=spectral)
    vstar = synth.scale_to_displacement(w["v_star"], grid, 1.0)
    I0 = w["I0"]
    vs, _, ms = forward(vstar, I0, p)
    v0, d = 0.5 * vstar, synth.random_direction(3, band)
    g_ref, _, cache = gradient(v0, I0, ms[-1], p)
    prob = L.Problem(grid=grid, band=band, spectral=spectral, time_steps=nt, alpha=synth.ALPHA, s=s,
                     sigma=synth.SIGMA, precision=L.FP32_BF16X3 if bf16x3 else L.FP32)
    ws = L.Workspace(prob)
    img = lambda x: torch.from_numpy(np.ascontiguousarray(x)).float().cuda()  # noqa: E731
    vec = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(torch.complex64).cuda()  # noqa: E731
    m1, v1 = L.shoot(prob, img(I0), vec(vstar), ws, want_v1=True)
    g, _ = L.gradient(prob, img(I0), img(ms[-1]), vec(v0), ws)
    h = L.hessvec(prob, vec(d), ws)
    torch.cuda.synchronize()
    errs = dict(m1=rel(m1, ms[-1]), v1=rel(v1, vs[-1]), gradient=rel(g, g_ref), hessvec=rel(h, hessvec(cache, d, p, "R1")))
    print(errs, flush=True)
    assert max(errs.values()) < 1e-4, errs
