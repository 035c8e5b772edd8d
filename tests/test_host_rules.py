"""Rules of the kernels' launches that hold no device code, compiled with the
host compiler from the headers that the kernels include."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2609_29554_amd", "csrc")


def _run(tmp_path, header, body):
    """The lines that a C++ main() with this body prints, as lists of integers."""
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(f'#include <cstdio>\n#include "{header}"\nint main() {{\n{body}\nreturn 0;\n}}\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", f"-I{CSRC}", str(src), "-o",
                    str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    return [[int(x) for x in line.split()] for line in out.splitlines()]


@pytest.mark.parametrize("nc", [2, 3, 4])
def test_work_left_grows_with_the_order(tmp_path, nc):
    rows = _run(tmp_path, "batch_rules.hpp",
                f'for (long r = 1; r <= 1024; ++r) std::printf("%u\\n", ozb::work_left({nc}, r));')
    v = [r[0] for r in rows]
    assert v[0] >= 1 and all(a <= b for a, b in zip(v, v[1:]))
    # an order 1024 system ranks above every smaller order's next block
    assert v[1023] > v[1007] > v[511] > v[63]
    assert v[1023] == nc * nc * 2 ** 24 + 1
