"""The prod_rows field of the tile table (lddmm_tiles_set, lddmm_autotune) where the Lie products are a launch of
their own: every choice gives bitwise the built-in rule's gradient and products, at half spectra of one and of
two tiles past the rule of the one-launch step (Kh <= 16, K1 <= 32, M2 <= 48), rows that are no whole k-steps of
four, and the deformation state of a small band, whose products at t = 1 are such a launch; and where no launch
reads the field the autotuner does not time it."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1807_11560_amd import synth  # noqa: E402

CASES = [
    # grid, band, spectral, deformation state, precision, rows (at most 256 // M2)
    ((48, 48, 48), (40, 40, 40), (60, 60, 60), False, 0, (1, 2, 3)),
    ((48, 48, 48), (40, 40, 40), (60, 60, 60), True, 1, (1, 3)),
    ((32, 36, 31), (20, 34, 18), (29, 51, 25), False, 0, (1, 4, 9)),
    ((32, 36, 31), (20, 34, 18), (29, 51, 26), False, 1, (1, 4, 8)),
    ((24, 24, 66), (12, 12, 30), (18, 18, 49), False, 0, (1, 2, 4)),
    ((66, 20, 64), (64, 8, 64), (96, 12, 97), False, 0, (1,)),
    ((32, 32, 32), (16, 16, 16), (24, 24, 24), True, 0, (1, 3, 9)),
]


def setup(grid, band, spectral, deformation, precision, s=2):
    from paper_1807_11560_amd import lddmm as L

    w = synth.workload(3, grid=grid, band=band)
    prob = L.Problem(grid=grid, band=band, spectral=spectral, time_steps=3, alpha=synth.ALPHA, s=s, sigma=synth.SIGMA,
                     state=L.STATE_DEFORMATION if deformation else L.STATE_IMAGE, precision=precision)
    vec = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(torch.complex64).cuda()  # noqa: E731
    vstar = synth.scale_to_displacement(w["v_star"], grid, 2.0)
    ws = L.Workspace(prob)
    I0 = torch.from_numpy(w["I0"]).float().cuda()
    I1 = L.shoot(prob, I0, vec(vstar), ws)
    return prob, ws, I0, I1, vec(0.5 * vstar), vec(synth.random_direction(11, band, s=s))


def results(prob, ws, I0, I1, v0, d):
    from paper_1807_11560_amd import lddmm as L

    g, e = L.gradient(prob, I0, I1, v0, ws)
    h = L.hessvec(prob, d, ws)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in (g, e, h)]


@pytest.mark.parametrize("grid,band,spectral,deformation,precision,rows", CASES)
def test_every_row_count_is_bitwise_the_built_in_rule(grid, band, spectral, deformation, precision, rows):
    from paper_1807_11560_amd import lddmm as L

    print(f"\n[prod_rows {grid} {band} {spectral} {deformation} {precision}]", flush=True)
    args = setup(grid, band, spectral, deformation, precision)
    L.tiles_clear()
    try:
        want = results(*args)
        assert all(np.isfinite(x).all() and x.any() for x in want)
        for r in rows:
            assert r < 256 // spectral[2]
            L.tiles_set(args[0], dict(prod_rows=r))
            assert all(np.array_equal(a, b) for a, b in zip(results(*args), want)), r
    finally:
        L.tiles_clear()


@pytest.mark.parametrize("deformation,fields", [(False, 5), (True, 5 + 9)])
def test_autotune_times_the_field_only_where_a_launch_reads_it(deformation, fields):
    """Launches of the Lie products are counted: one gradient, and for the built-in rule (twice) and each
    candidate one product and `reps` more.  Candidates: two of sl_threads, three of col_split, and the nine
    row counts below the largest (M2 = 24) where the product launches k_prods."""
    from paper_1807_11560_amd import lddmm as L

    print(f"\n[autotune {deformation}]", flush=True)
    prob, ws, I0, I1, v0, d = setup((32, 32, 32), (16, 16, 16), (24, 24, 24), deformation, 0)

    def launches(call):
        L.kernel_timer(L.KF_PRODS, 1)
        call()
        torch.cuda.synchronize()
        return L.kernel_timer_read()[0]

    L.tiles_clear()
    try:
        n_grad = launches(lambda: L.gradient(prob, I0, I1, v0, ws))
        n_hvp = launches(lambda: L.hessvec(prob, d, ws))
        reps = 2
        tuned = []
        n = launches(lambda: tuned.append(L.autotune(prob, I0, I1, v0, ws, reps=reps)))
        assert n_grad > 0 and n_hvp > 0
        assert n == n_grad + (2 + fields) * (1 + reps) * n_hvp
        assert deformation or tuned[0][0]["prod_rows"] == 0
    finally:
        L.kernel_timer(0, 1)
        L.tiles_clear()
