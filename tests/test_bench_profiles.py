"""bench.py's stored profile values: a line holds for the source files that its kernel is built from, and the
kernel families are named after kernels that exist.  And its initial velocity on another band (--band)."""

import hashlib
import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import numpy as np  # noqa: E402

import bench  # noqa: E402
from paper_1807_11560_amd import lddmm as L  # noqa: E402

CSRC = os.path.join(ROOT, "paper_1807_11560_amd", "csrc")


def digest(*data):
    return hashlib.sha256(b"".join(data)).hexdigest()[:16]


@pytest.mark.parametrize("changed,expect", [(None, (1.0, 2.0, 3.0)), ("kernels.hip", (None, 2.0, 3.0)),
                                            ("step.hip", (1.0, None, 3.0)), ("mfma.h", (1.0, None, 3.0)),
                                            ("chain.hip", (1.0, 2.0, None))])
def test_a_stored_value_follows_its_own_sources(tmp_path, changed, expect):
    files = {f: f.encode() for f in ("kernels.hip", "step.hip", "mfma.h", "chain.hip")}
    md = tmp_path / "p.md"
    md.write_text(f"| traffic | a | 1 | {digest(files['kernels.hip'])} |\n"
                  f"| traffic of step.hip mfma.h | b, c | 2 | {digest(files['step.hip'], files['mfma.h'])} |\n"
                  f"| trace of chain.hip | b, c | 9 | {digest(files['chain.hip'])} |\n"
                  f"| traffic of chain.hip | d | 3 | {digest(files['chain.hip'])} |\n")
    for f, data in files.items():
        (tmp_path / f).write_bytes(data + (b" changed" if f == changed else b""))
    got = tuple(bench.stored_value(str(md), "traffic", k, csrc=str(tmp_path)) for k in ("a", "b, c", "d"))
    assert got == expect
    assert bench.stored_value(str(md), "traffic", "e", csrc=str(tmp_path)) is None


def test_families_are_named_after_kernels():
    text = "".join(open(os.path.join(CSRC, f)).read() for f in os.listdir(CSRC) if f.endswith(".hip"))
    kernels = set(re.findall(r"__global__[^;{]*?\b(k_\w+)\(", text))
    for name in L.KERNEL_FAMILIES.values():
        for k in re.findall(r"k_\w+", name):
            # a kernel, or the stem of several
            assert k in kernels or sum(q.startswith(k + "_") for q in kernels) > 1, k


@pytest.mark.parametrize("band", [(4, 6, 8), (12, 10, 8), (8, 8, 8), (16, 4, 8)])
def test_a_velocity_on_another_band_keeps_the_common_frequencies(band):
    rng = np.random.default_rng(0)
    v = rng.standard_normal((3, 8, 8, 8)) + 1j * rng.standard_normal((3, 8, 8, 8))
    v[:, 4], v[:, :, 4], v[:, :, :, 4] = 0, 0, 0  # a band field holds nothing at -K/2
    got = bench.on_band(v, band)
    assert got.shape == (3,) + band
    for k in np.ndindex(*band):
        f = [q if q < n // 2 else q - n for q, n in zip(k, band)]
        common = all(abs(q) < min(n, 8) // 2 for q, n in zip(f, band))
        assert np.array_equal(got[(slice(None),) + k], v[(slice(None),) + tuple(f)] if common else np.zeros(3))
    if band == (8, 8, 8):
        assert np.array_equal(got, v)
