"""Writes the digests of tests/test_gpu_bits.py: python tests/golden/make_bit_records.py TREE OUT

TREE holds the built package whose outputs are recorded (an older checkout, to hold newer kernels to its bits)."""

import importlib.util
import json
import os
import sys

tree, out = os.path.abspath(sys.argv[1]), sys.argv[2]
sys.path.insert(0, tree)
import paper_1807_11560_amd.lddmm as lddmm  # noqa: E402

assert os.path.dirname(os.path.dirname(lddmm.__file__)) == tree
spec = importlib.util.spec_from_file_location(
    "bits", os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "test_gpu_bits.py"))
bits = importlib.util.module_from_spec(spec)
spec.loader.exec_module(bits)
doc = {p: {n: bits.digests(n, p == "bf16x3") for n in bits.CASES} for p in ("fp32", "bf16x3")}
again = {p: {n: bits.digests(n, p == "bf16x3") for n in bits.CASES} for p in ("fp32", "bf16x3")}
assert doc == again, "outputs differ between two runs"
with open(out, "w") as f:
    json.dump(doc, f, indent=1)
    f.write("\n")
print("written", out)
