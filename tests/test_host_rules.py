"""Rules that choose kernels, checked on a machine without a GPU: tests/host_checks/rules_harness.cpp is built from the headers that
the library's launchers use."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CHECKS = os.path.join(ROOT, "tests", "host_checks")
SAN = ["-fsanitize=address,undefined", "-fno-sanitize-recover=all"]


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not found")
    exe = str(tmp_path_factory.mktemp("rules") / "rules_harness")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-Wall", "-Werror", *SAN, os.path.join(CHECKS, "rules_harness.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def _run(exe, mode, stdin=""):
    r = subprocess.run([exe, mode], input=stdin, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    return r.stdout


def test_a_thread_walks_over_few_rows_that_it_does_not_have(harness):
    """Beyond 16 rows per thread the N x H x W x C kernels load every row that they can hold: no more than seven of them for nothing, as
    long as the registers hold all, and no more than LDS holds beyond that."""
    table = {}
    for line in _run(harness, "rows").splitlines():
        V, backward, mixed, rows, regs, park = map(int, line.split())
        table.setdefault((V, backward, mixed), []).append((rows, regs, park))
    assert len(table) == 12
    for (V, backward, mixed), entries in table.items():
        most_regs = max(regs for _, regs, park in entries if park == 0)
        most = max(regs + park for _, regs, park in entries)
        for rows, regs, park in entries:
            if rows <= most:
                assert regs + park >= rows
            if V > 1 and 16 < rows <= most_regs:
                assert regs - rows <= 7 and park == 0, (V, backward, mixed, rows, regs)
            elif V > 1 and most_regs < rows <= most:
                assert regs + park - rows < park
