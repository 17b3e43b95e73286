"""The size limit of lddmm_shoot_static (LDDMM_STATIC_SCRATCH_BYTES) where the transform tables are mostly
padding: four band frequencies against rows of 241 to 245 points, whose fragment tables take about 93 KB more
than plain ones.  The limit is that of the plain tables: what fits it is taken, whatever the padding.

On the host a problem past the limit returns LDDMM_E_WORKSPACE before the device is touched, and one within it
goes on and, without a device, returns LDDMM_E_HIP; on the GPU the latter gives lddmm_shoot's result."""

import ctypes

import numpy as np
import pytest
import torch

from paper_1807_11560_amd import lddmm as L

CASES = [
    # grid, band, spectral, workspace with plain tables less the limit (bytes)
    ((10, 174, 241), (4, 4, 4), (5, 241, 242), -25984),
    ((10, 163, 241), (4, 4, 4), (5, 243, 243), -14720),
    ((9, 177, 241), (4, 4, 4), (5, 242, 245), -16704),
    ((10, 175, 241), (4, 4, 4), (5, 241, 242), 98944),
    ((10, 164, 241), (4, 4, 4), (5, 243, 243), 111744),
]


@pytest.mark.skipif(torch.cuda.is_available(), reason="the pointers are not device memory")
@pytest.mark.parametrize("grid,band,spectral,over", CASES)
def test_padding_of_the_tables_is_not_counted(grid, band, spectral, over):
    prob = L.Problem(grid=grid, band=band, spectral=spectral, time_steps=1)
    assert prob.workspace_bytes() > L.STATIC_SCRATCH_BYTES
    fake, null = ctypes.c_void_p(0x1000), ctypes.c_void_p(0)  # never dereferenced
    rc = L.raw().lddmm_shoot_static(ctypes.byref(prob.c_params()), fake, fake, fake, null, null)
    assert rc == (L.E_WORKSPACE if over > 0 else L.E_HIP)


@pytest.mark.gpu
def test_the_largest_padded_problem_equals_shoot():
    grid, band, spectral, _ = CASES[0]
    prob = L.Problem(grid=grid, band=band, spectral=spectral, time_steps=1)
    print(f"\n[static {grid} {band} {spectral}]", flush=True)
    I0 = torch.from_numpy((np.arange(np.prod(grid)) * 7919 % 256 / 256.0).astype(np.float32).reshape(grid)).cuda()
    v0 = np.zeros((3,) + band, dtype=np.complex64)
    v0[:, 1, 1, 1], v0[:, -1, -1, -1] = 0.01 + 0.005j, 0.01 - 0.005j
    v0 = torch.from_numpy(v0).cuda()
    a, va = L.shoot_static(prob, I0, v0, want_v1=True)
    b, vb = L.shoot(prob, I0, v0, L.Workspace(prob), want_v1=True)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and torch.equal(va, vb) and bool(torch.isfinite(a).all())
