"""CPU check of the division by numbers the host knows (csrc/lcsa_quotient.h): exact for every non-negative 32-bit dividend."""
import ctypes
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("quotient")
    src, so = tmp / "q.cpp", tmp / "q.so"
    src.write_text('#include "lcsa_quotient.h"\n'
                   'extern "C" int quotient(int n, int d) { return lcsa::quotient_by(d)(n); }\n'
                   'extern "C" int first_wrong(int d, int n0, int count) {\n'
                   '    const lcsa::Quotient q = lcsa::quotient_by(d);\n'
                   '    for (int i = 0; i < count; ++i) if (q(n0 + i) != (n0 + i) / d) return n0 + i;\n'
                   '    return -1;\n}\n')
    subprocess.run(["g++", "-O2", "-Wall", "-Werror", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2510_12747_amd", "csrc"),
                    "-o", str(so), str(src)], check=True)
    return ctypes.CDLL(str(so))


def test_quotients_are_exact(lib):
    top = 2 ** 31 - 1
    rng = random.Random(0)
    divisors = list(range(1, 600)) + [2 ** e + o for e in range(9, 31) for o in (-1, 0, 1)] + [top] + [rng.randrange(1, top) for _ in range(500)]
    for d in divisors:
        assert lib.first_wrong(d, 0, 2000) == -1 and lib.first_wrong(d, top - 2000, 2001) == -1, d
        for _ in range(50):
            multiple = rng.randrange(0, top // d + 1) * d
            for n in (multiple - 1, multiple, multiple + 1, rng.randrange(0, top)):
                if 0 <= n <= top:
                    assert lib.quotient(n, d) == n // d, (n, d)
