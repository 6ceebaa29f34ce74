"""The refinement's whole-number helpers, built for the host with the undefined
behaviour sanitizer and run over the ends of their ranges."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_16576_amd", "csrc")


def run(tmp_path, body):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include "refine_keys.hpp"\n#include <cstdio>\nusing namespace polymh;\nint main() {\n' + body + "\n}\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC, "-o",
                    str(exe), str(src)], check=True, capture_output=True, text=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return r.stdout.split()


@pytest.mark.parametrize("x", [-2**31, -2**26, -1, 0, 1, 2**26, 2**31 - 1])
def test_vertex_key_orders_down_and_right(tmp_path, x):
    """Along an edge from (x, y) the key falls when it points down, or is
    horizontal and points right, whatever the signs."""
    ends = [(x2, y2) for x2 in (-2**31, -5, 0, 5, 2**31 - 1) for y2 in (-2**31, -1, 0, 1, 2**31 - 1)]
    body = "\n".join(f'printf("%d ", down_right_key((int32_t){a}LL, (int32_t){b}LL) < down_right_key((int32_t){x}LL, 0));'
                     for a, b in ends)
    got = run(tmp_path, body)
    assert got == [str(int(b < 0 or (b == 0 and a > x))) for a, b in ends]


@pytest.mark.parametrize("n,m", [(3, 3), (512, 256), (46340, 46341), (46341, 46341), (2**31 - 1, 2**31 - 1)])
def test_edge_pairs(tmp_path, n, m):
    assert run(tmp_path, f'printf("%lld", (long long)edge_pairs({n}, {m}));') == [str(n * m)]
