"""The coefficients of the device's polynomials are those their generator gives."""
import importlib.util
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2312_16981_amd", "csrc")
NUMBER = r"-?0x1\.[0-9a-f]+p[+-]\d+"


def test_table_equals_its_generator():
    spec = importlib.util.spec_from_file_location("gen_math_tab", os.path.join(CSRC, "gen_math_tab.py"))
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    want = gen.coefficients()
    src = open(os.path.join(CSRC, "device_math.hpp")).read()
    body = src[src.index("g_math_tab = {") + len("g_math_tab = {"):]
    body = body[:body.index("\n};")]
    rows = [[float.fromhex(v) for v in re.findall(NUMBER, r)] for r in re.findall(r"\{([^{}]*)\}", body)]
    names = ["head", "weight", "L1", "L2", "L3", "L4", "ex", "one_ex", "w", "c2", "ln"]
    assert len(rows) == len(names) == len(want)
    for name, row in zip(names, rows):
        assert row == want[name], name
    # the logarithm's coefficients once more as literals, highest first
    fn = src[src.index("__device__ inline double neg_log_unit(double u)"):]
    literal = [float.fromhex(v) for v in re.findall(r"q = (?:fma\(q, z, )?(" + NUMBER + ")", fn[:fn.index("} else {")])]
    assert literal[::-1] == want["ln"]
