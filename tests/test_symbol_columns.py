"""The rule that sends several symbols to the column form, on the host: its lines in
n_sym and C, and the shapes whose byte offsets leave 32 bits, which stay with the
vector form."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIP = "/opt/rocm/include/hip/hip_runtime.h"

pytestmark = pytest.mark.skipif(not (shutil.which("g++") and os.path.exists(HIP)), reason="no g++ or HIP headers")

CASES = [  # U, n_sym, B, C, columns (T <= 8)
    (8, 14, 64, 8, False),
    (16, 3, 128, 8, False), (16, 4, 128, 8, True), (16, 4, 32, 2, False), (16, 4, 48, 3, True),
    (32, 4, 256, 8, False), (32, 5, 256, 8, True), (32, 5, 32, 1, False), (32, 5, 64, 2, True),
    (64, 2, 512, 8, False), (64, 3, 512, 8, True), (64, 3, 64, 1, True),
    # 7 B + S entries of eight bytes: up to 2^31 - 1
    (16, 8, 37_682_640, 16, True), (16, 8, 38_347_920, 16, False), (16, 8, 80_000_000, 16, False),
    # S rows of 8 U bytes
    (64, 3, 4_194_303, 1, True), (64, 3, 4_194_304, 1, False), (32, 5, 2 * 8_388_608, 2, False),
]

MANY = [(64, 3, 512, 8, False), (64, 4, 512, 8, True), (64, 3, 64, 1, True), (16, 4, 128, 8, True)]   # T = 9


def test_symbol_columns_rule(tmp_path):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    calls = "".join(f"  putchar(dbp::symbol_columns({u}, {n}, {b}, {b // c}, {c}, {t}) ? '1' : '0');\n"
                    for t, cases in ((8, CASES), (9, MANY)) for u, n, b, c, _ in cases)
    src.write_text('#include <cstdio>\n#include "dbp_launch.h"\nint main() {\n' + calls + "}\n")
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "paper_1702_04458_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    got = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    assert got == "".join("1" if want else "0" for *_, want in CASES + MANY)
