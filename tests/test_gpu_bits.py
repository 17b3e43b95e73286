"""Outputs keep their bits: every sum is formed in a stated order (csrc/mfma.h), in FP32 and in the
compensated BF16 mode, so a kernel that replaces another returns the same values.

tests/golden/bits.json holds the SHA-256 of each output of the calls below, recorded on an MI355X from the
kernels that staged their tables in LDS (tests/golden/make_bit_records.py).  The inputs are whole numbers times
powers of two, the same on every host.  Shapes: instantiated band and grid kernels, an instantiated grid with a
generic band, one launch and two launches for synthesis and products, odd sizes."""

import hashlib
import json
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

RECORDS = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "bits.json")
CASES = {
    "64cubed_band16": ((64, 64, 64), (16, 16, 16)),
    "96cubed_band32": ((96, 96, 96), (32, 32, 32)),
    "96cubed_band18x24x24": ((96, 96, 96), (18, 24, 24)),
    "64cubed_band40": ((64, 64, 64), (40, 40, 40)),
    "41x44x37_band12x14x10": ((41, 44, 37), (12, 14, 10)),
}


def whole_numbers(shape, seed, n):
    """Integers 0 .. n - 1 from a multiplicative hash of the index."""
    i = np.arange(int(np.prod(shape)), dtype=np.uint64) + np.uint64(1 + 1000003 * seed)
    return ((i * np.uint64(0x9E3779B97F4A7C15)) >> np.uint64(40)).astype(np.int64).reshape(shape) % n


def image(grid, seed):
    return (whole_numbers(grid, seed, 256) / 256.0).astype(np.float32)


def band_field(band, seed, exponent):
    """Hermitian coefficients 2^(exponent - |k0| - |k1| - |k2|) times whole numbers in [-8, 8], no k = 0."""
    f = [np.where(np.arange(k) < k // 2, np.arange(k), np.arange(k) - k) for k in band]
    a = np.abs(f[0])[:, None, None] + np.abs(f[1])[None, :, None] + np.abs(f[2])[None, None, :]
    keep = (f[0] != -(band[0] // 2))[:, None, None] & (f[1] != -(band[1] // 2))[None, :, None] & \
        (f[2] != -(band[2] // 2))[None, None, :]
    flip = np.ix_(*[(-np.arange(k)) % k for k in band])
    out = []
    for c in range(3):
        x = whole_numbers(band, 10 * seed + c, 17) - 8 + 1j * (whole_numbers(band, 10 * seed + 3 + c, 17) - 8)
        x = 0.5 * (x + np.conj(x[flip])) * keep * np.ldexp(1.0, exponent - a)
        x[0, 0, 0] = 0
        out.append(x)
    return np.stack(out).astype(np.complex64)


def outputs(name, bf16x3):
    """name -> tensor: shooting by Euler and RK4 steps, energy, gradient and Hessian-vector products of both states."""
    from paper_1807_11560_amd import lddmm as L

    grid, band = CASES[name]
    kw = dict(grid=grid, band=band, time_steps=3, alpha=0.0025, s=2, sigma=0.03,
              precision=L.FP32_BF16X3 if bf16x3 else L.FP32)
    I0, I1 = (torch.from_numpy(image(grid, q)).cuda() for q in (1, 2))
    v0 = torch.from_numpy(band_field(band, 1, -9)).cuda()
    d = torch.from_numpy(band_field(band, 2, -4)).cuda()
    out = {}
    p = L.Problem(**kw)
    ws = L.Workspace(p)
    out["m1"], out["v1"] = L.shoot(p, I0, v0, ws, want_v1=True)
    out["energies"] = L.geodesic_energy(p, v0, ws)
    p = L.Problem(integrator=L.RK4, **kw)
    out["rk4 m1"], out["rk4 v1"] = L.shoot(p, I0, v0, L.Workspace(p), want_v1=True)
    for state, s in ((L.STATE_IMAGE, ""), (L.STATE_DEFORMATION, "deformation ")):
        for hessian, h in ((L.GN_PAPER, "paper"), (L.GN_CLASSICAL, "classical"), (L.NEWTON, "newton")):
            p = L.Problem(state=state, hessian=hessian, **kw)
            ws = L.Workspace(p)
            out[s + "gradient " + h], out[s + "energy " + h] = L.gradient(p, I0, I1, v0, ws)
            out[s + "hessvec " + h] = L.hessvec(p, d, ws)
    torch.cuda.synchronize()
    return out


def digests(name, bf16x3):
    out = {k: t.cpu().numpy() for k, t in outputs(name, bf16x3).items()}
    assert all(np.isfinite(v).all() and v.any() for v in out.values())
    return {k: hashlib.sha256(np.ascontiguousarray(v).tobytes()).hexdigest() for k, v in out.items()}


@pytest.mark.parametrize("bf16x3", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_outputs_keep_their_bits(name, bf16x3):
    print(f"\n[bits {name} bf16x3={bf16x3}]", flush=True)
    with open(RECORDS) as f:
        want = json.load(f)["bf16x3" if bf16x3 else "fp32"][name]
    got = digests(name, bf16x3)
    assert got.keys() == want.keys()
    changed = [k for k in want if got[k] != want[k]]
    assert not changed, changed
