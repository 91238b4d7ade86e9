"""Index arithmetic of launches over very many rows (csrc/ranges.h), compiled
for the host: no GPU is needed, and none could show an overflow safely."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_26164_amd", "csrc")


def _run(tmp_path, body):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include <stdio.h>\n#include "ranges.h"\nusing namespace chisao;\n'
                   "#define CHECK(c) do { if (!(c)) { printf(\"line %d: %s\\n\", __LINE__, #c); return 1; } } while (0)\n"
                   "int main() {\n" + body + "\nreturn 0;\n}\n")
    subprocess.run([cxx, "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC,
                    str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr


# rows of caller memory (one unit each) up to the largest int, and probes of a population beyond it
@pytest.mark.parametrize("jobs,centres", [(1, 1), (70000, 1), (2**31 - 16385, 1), (2**31 - 16384, 1), (2**31 - 1, 1),
                                          (2**26, 32), (2**27 + 5, 32)])
def test_every_wave_ends_at_the_last_unit(tmp_path, jobs, centres):
    """Each wave walks its units in steps of the grid; near the end of the range
    the next unit must lie past it, not wrap to a negative one."""
    _run(tmp_path, f"""
    const unsigned blocks = 4096; const int waves = 4;
    const unit_t total = units_of({jobs}, {centres});
    CHECK(total == {jobs * centres}ll);
    unit_t last = -1;
    for (unsigned b = 0; b < blocks; ++b) for (int w = 0; w < waves; ++w) {{
        unit_t u = first_unit(b, waves, w);
        if (u >= total) continue;
        u += (total - 1 - u) / ((unit_t)blocks * waves) * ((unit_t)blocks * waves);  // the wave's last unit
        CHECK(u >= 0 && u < total && u / {centres} < {jobs}ll);
        if (u > last) last = u;
        CHECK(next_unit(u, blocks, waves) >= total);
    }}
    CHECK(last == total - 1);""")


@pytest.mark.parametrize("rows", [1, 2**29 - 1, 2**29, 2**29 + 1, 2**30, 2**30 + 1, 2**31 - 64, 2**31 - 1])
def test_launches_cover_the_rows_within_hips_limit(tmp_path, rows):
    """Every row once, in parts of one size whose four threads a row stay below
    HIP's 2^32 threads a launch."""
    _run(tmp_path, f"""
    long long at = 0; int left = {rows}, first = launch_rows(left), n = 0;
    while (left > 0) {{
        const int r = launch_rows(left);
        CHECK(r > 0 && r <= left && first - r >= 0 && first - r <= 4);
        CHECK((unsigned long long)r * kThreadsPerRow + 1023 < 1ull << 32);
        at += r; left -= r; ++n;
    }}
    CHECK(at == {rows}ll && n == ({rows}ll + kLaunchRows - 1) / kLaunchRows);""")
