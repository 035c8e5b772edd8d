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


def test_batch_tasks(tmp_path):
    """Workgroups that can work on one system: its owner alone where nothing is
    shared, and for an order 512 system of width 64 the 504 x 56 deferred
    elements in tasks of 512."""
    sizes = [(1, 32), (64, 64), (100, 32), (128, 64), (129, 64), (512, 64), (1024, 64), (1024, 256),
             (1024, 1), (90, 256)]
    rows = _run(tmp_path, "batch_rules.hpp",
                " ".join(f'std::printf("%ld\\n", (long)ozb::most_tasks({n}, {b}));'
                         for n, b in sizes))
    got = dict(zip(sizes, (r[0] for r in rows)))
    assert got[(1, 32)] == got[(64, 64)] == 1
    assert got[(100, 32)] == 6          # 68 trailing rows: 4 + 2 chunks, 2 x 2 tiles
    assert got[(128, 64)] == 14         # 120 x 56 deferred elements
    assert got[(512, 64)] == 56 and got[(1024, 64)] == 15 * 15
    assert got[(1024, 1)] == 16 * 16 and got[(90, 256)] == (82 * 82 + 511) // 512
    # four systems of order 64, or one of 512, leave most CUs alone
    assert 4 * got[(64, 64)] == 4 and got[(512, 64)] < 64


def test_panel_tags_do_not_come_again(tmp_path):
    """Over more than 2^32 tags: the tags of the panels between two clearings
    are disjoint ranges of 512, none of them 0."""
    panels = [1, 7, 1024, 1 << 20, 3, 400000, 65, 999999]
    body = """
  uint32_t end = 0;
  const uint32_t panels[] = {%s};
  for (int rep = 0; rep < 2000; ++rep) {
    const uint32_t n = panels[rep %% 8] / (rep < 1000 ? 1 : 7) + 1;
    const ozp::TagRange r = ozp::next_tags(end, n);
    end = r.end;
    std::printf("%%d %%u %%u %%u\\n", r.clear ? 1 : 0, n, ozp::panel_tag0(end, n - 1),
                ozp::panel_tag0(end, 0));
  }""" % ", ".join(map(str, panels))
    rows = _run(tmp_path, "panel_tags.hpp", body)
    top, clears = 0, 0
    for clear, n, lowest, highest in rows:
        if clear:
            top, clears = 0, clears + 1
        assert lowest > top and highest == lowest + 1024 * (n - 1)
        top = highest + 511
        assert top < 2 ** 32
    assert clears > 50
