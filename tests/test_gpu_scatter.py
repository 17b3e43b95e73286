"""The scatter of the exact derivative's state adjoint (csrc/source.hip) at the
edges of its bricks: grids of one and of two planes past a multiple of the
brick, rows that are not a multiple of 8 or 4 long, a grid narrower than the
window of a brick, bricks of four planes with fewer left, and displacements of up to
four voxels a step, so that cells fall inside and outside of the windows and
wrap around every axis.

Against the FP64 oracle with the kernels' own cell decisions, at the bound of the
other tests of the exact derivative, 1e-5 in relative L2."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import Params  # noqa: E402
from oracle import exact  # noqa: E402
from oracle.jacobi import forward  # noqa: E402
from paper_1807_11560_amd import synth  # noqa: E402

CASES = [
    # grid, band, displacement in voxels over two steps
    ((8, 8, 10), (4, 4, 4), 8.0),
    ((9, 17, 21), (6, 8, 6), 8.0),
    ((34, 23, 35), (8, 10, 8), 2.0),
    ((66, 129, 18), (8, 8, 6), 6.0),
]


@pytest.mark.parametrize("grid,band,dmax", CASES)
def test_scatter_against_oracle(grid, band, dmax):
    from paper_1807_11560_amd import lddmm as L

    print(f"\n[{grid} {band} {dmax}]", flush=True)
    nt, s = 2, 2
    w = synth.workload(3, grid=grid, band=band)
    p = Params(grid=grid, band=band, nt=nt, alpha=synth.ALPHA, s=s, sigma=synth.SIGMA)
    vstar = synth.scale_to_displacement(w["v_star"], grid, dmax)
    I0 = w["I0"]
    I1 = forward(0.5 * vstar, I0, p)[2][-1]
    _, _, cache = exact.gradient(vstar, I0, I1, p)
    ref = vstar + exact.adjoint_sweep(cache["vs"], cache["vgrid"], cache["ms"],
                                      2.0 / (p.sigma ** 2 * float(np.prod(p.grid))) * (cache["ms"][-1] - I1), p,
                                      decisions="fp32")[0]
    prob = L.Problem(grid=grid, band=band, time_steps=nt, alpha=synth.ALPHA, s=s, sigma=synth.SIGMA)
    img = lambda x: torch.from_numpy(np.ascontiguousarray(x)).float().cuda()  # noqa: E731
    v = torch.from_numpy(np.ascontiguousarray(vstar)).to(torch.complex64).cuda()
    g, _ = L.gradient_exact(prob, img(I0), img(I1), v, L.Workspace(prob))
    torch.cuda.synchronize()
    err = float(np.linalg.norm((g.cpu().numpy().astype(np.complex128) - ref).ravel()) / np.linalg.norm(ref.ravel()))
    print(err, flush=True)
    assert err < 1e-5
