"""The polynomials of the device functions: coefficients as their generator gives them, and the
exponentials and quotients made of them as exact as libm and division."""
import importlib.util
import os
import re
import subprocess

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
    names = ["head", "weight", "L1", "L2", "L3", "L4", "ex", "exf", "one_ex", "w", "c2", "ln"]
    assert len(rows) == len(names) == len(want)
    for name, row in zip(names, rows):
        assert row == want[name], name
    # the logarithm's coefficients once more as literals, highest first
    fn = src[src.index("__device__ inline double neg_log_unit(double u)"):]
    literal = [float.fromhex(v) for v in re.findall(r"q = (?:fma\(q, z, )?(" + NUMBER + ")", fn[:fn.index("} else {")])]
    assert literal[::-1] == want["ln"]


def test_replacements_of_libm_are_as_exact(tmp_path):
    """The exponentials whose own rounding is a result's, compiled for the host: no further from
    quad precision than libm's on the same arguments (2% for the largest of 4e5 errors and its
    place, 1% for the mean), and the quotients by constants within half an ulp."""
    here = os.path.dirname(os.path.abspath(__file__))
    exe = str(tmp_path / "device_math_host")
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-w",
                    os.path.join(here, "helpers", "device_math_host.cpp"), "-o", exe, "-lquadmath"], check=True,
                   capture_output=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()
    err = {w[0]: (float(w[1]), float(w[2])) for w in (line.split() for line in out) if w[0] != "end"}
    for new, old in (("exp_neg_fine", "exp"), ("one_less_exp_neg", "expm1")):
        assert err[new][0] <= 1.02 * err[old][0], (new, err)
        assert err[new][1] <= 1.01 * err[old][1], (new, err)
    for name in ("sixth", "over_pi4_15"):
        assert err[name][0] <= 2.0 ** -53, (name, err)
    ends = [tuple(float(v) for v in line.split()[1:]) for line in out if line.startswith("end")]
    assert ends == [(0.0, 1.0, 0.0), (1e-300, 1.0, 1e-300), (800.0, 0.0, 1.0), (1e300, 0.0, 1.0), (float("inf"), 0.0, 1.0)]
