"""The scatter of the exact derivative's state adjoint (csrc/source.hip) where a brick passes its rows in several
chunks of columns: the sums of forward stage 2 stay in registers over the chunks, the window moves with each, and
the table's loads end inside odd rows.  Rows of 65 (a second chunk of 25), 91 and 133 (odd, ragged last chunks) and
160 (even), half spectra of one and of two tiles, displacements of up to four voxels a step, which cross
chunk boundaries and the periodic edge.

Oracle and bound as for the single chunk (test_gpu_scatter.py): FP64 with the kernels' own cell decisions, 1e-5 in
relative L2."""

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
    ((9, 34, 91), (4, 8, 8), 8.0),
    ((8, 34, 133), (4, 8, 34), 6.0),
    ((10, 16, 65), (4, 6, 64), 8.0),
    ((8, 17, 160), (4, 8, 40), 4.0),
]


@pytest.mark.parametrize("hessian", [False, True])
@pytest.mark.parametrize("grid,band,dmax", CASES)
def test_chunks_against_oracle(grid, band, dmax, hessian):
    from paper_1807_11560_amd import lddmm as L

    print(f"\n[{grid} {band} {dmax} product={hessian}]", flush=True)
    nt, s = 2, 2
    w = synth.workload(3, grid=grid, band=band)
    p = Params(grid=grid, band=band, nt=nt, alpha=synth.ALPHA, s=s, sigma=synth.SIGMA)
    vstar = synth.scale_to_displacement(w["v_star"], grid, dmax)
    I0 = w["I0"]
    I1 = forward(0.5 * vstar, I0, p)[2][-1]
    img = lambda x: torch.from_numpy(np.ascontiguousarray(x)).float().cuda()  # noqa: E731
    vec = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(torch.complex64).cuda()  # noqa: E731
    _, _, cache = exact.gradient(vstar, I0, I1, p)
    kw = dict(grid=grid, band=band, time_steps=nt, alpha=synth.ALPHA, s=s, sigma=synth.SIGMA)
    if hessian:
        d = synth.random_direction(3, band)
        ref = exact.gauss_newton_hessvec(cache, d, p, decisions="fp32")
        prob = L.Problem(hessian=L.GN_EXACT, **kw)
        ws = L.Workspace(prob)
        L.gradient(prob, img(I0), img(I1), vec(vstar), ws)
        got = L.hessvec(prob, vec(d), ws)
    else:
        ref = vstar + exact.adjoint_sweep(cache["vs"], cache["vgrid"], cache["ms"],
                                          2.0 / (p.sigma ** 2 * float(np.prod(p.grid))) * (cache["ms"][-1] - I1), p,
                                          decisions="fp32")[0]
        prob = L.Problem(**kw)
        got, _ = L.gradient_exact(prob, img(I0), img(I1), vec(vstar), L.Workspace(prob))
    torch.cuda.synchronize()
    err = float(np.linalg.norm((got.cpu().numpy().astype(np.complex128) - ref).ravel()) / np.linalg.norm(ref.ravel()))
    print(err, flush=True)
    assert err < 1e-5
