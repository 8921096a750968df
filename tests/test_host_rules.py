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


def test_members_of_a_tile_and_the_sums_they_read(harness):
    """No more members than the device holds, two rows per thread at least, 4096 pairs of sums at most unless that left more than four rows; every member's
    sums are added by one thread of those that share a channel, none of which has nothing to do, eight at a time at most."""
    seen = {"two": 0, "pairs": 0, "four": 0}
    for line in _run(harness, "tiles").splitlines():
        kind, *v = line.split()
        if kind == "m":
            groups, channels, most, members = map(int, v)
            two, four, pairs = -(-groups // 2), -(-groups // 4), 4096 // channels
            assert members == max(1, min(most, max(four, min(two, pairs))))
            if 1 < members < most:
                seen["two" if two <= pairs else "pairs" if pairs > four else "four"] += 1
            continue
        members, threads, groups, polled = map(int, v)
        each = -(-members // groups)
        assert 1 <= groups <= min(threads, members) and 1 <= polled <= 8
        assert (each - 1) * groups < members                # the last turn is not empty for the first thread
        assert groups == -(-members // -(-members // threads))
        assert -(-each // polled) == -(-each // 8) and polled == -(-each // -(-each // 8))
    assert min(seen.values()) > 100, seen


# One block per compute unit on 256 units: layers on both sides of each line, with what other kernels and these took (us).
# N, C, H, W, dtype, mode, n_s, patch_h, patch_w, n_v, backward, kernel (0 other, 1 dy (x) alone on chip, 2 x beside dy)
FULL, BS, FS = 0, 2, 3
LAYERS = [
    # forward
    (64, 256, 56, 56, 1, BS, 8, 0, 0, 0, 0, 1),             # 36.7 / 34.5
    (45, 48, 105, 105, 0, FULL, 0, 0, 0, 0, 0, 1),          # 0.91 of the registers: 42.9 / 40.9
    (42, 64, 90, 90, 0, BS, 4, 0, 0, 0, 0, 0),              # 0.85: 35.9 / 37.7
    (64, 256, 56, 56, 0, BS, 8, 0, 0, 0, 0, 0),             # two rounds, part: 71.9 / 75.6
    (64, 64, 112, 112, 0, FULL, 0, 0, 0, 0, 0, 1),          # two rounds, everything: 82.4 / 77.7
    (51, 256, 60, 60, 0, FULL, 0, 0, 0, 0, 0, 1),           # 84.1 / 75.0
    (33, 256, 55, 55, 0, BS, 4, 0, 0, 0, 0, 0),             # part of odd planes: 40.3 / 43.1
    (32, 256, 55, 55, 0, FULL, 0, 0, 0, 0, 0, 1),           # all of them: 46.5 / 42.9
    (64, 256, 55, 55, 1, FS, 0, 14, 14, 0, 0, 0),           # rows that are no whole number of vectors: 47.3 / 51.2
    # backward, dy alone on chip
    (64, 256, 56, 56, 1, FS, 0, 14, 14, 0, 1, 1),           # 64.9 / 49.4
    (64, 256, 56, 56, 0, BS, 8, 0, 0, 0, 1, 1),             # two rounds: 114.1 / 106.1
    (26, 384, 60, 60, 0, FS, 0, 15, 15, 0, 1, 1),           # 0.70 of the device: 94.6 / 81.3
    (64, 160, 56, 56, 0, BS, 1, 0, 0, 0, 1, 0),             # 0.62: 69.8 / 75.1
    (30, 320, 80, 80, 1, BS, 7, 0, 0, 0, 1, 0),             # 0.60: 74.0 / 77.2
    (48, 172, 64, 64, 1, FS, 0, 32, 32, 0, 1, 0),           # a thread meets the patch at one place: 49.1 / 60.0
    (93, 128, 64, 64, 1, BS, 2, 0, 0, 0, 1, 1),             # no patch: 62.1 / 49.3
    (64, 48, 96, 96, 0, FS, 0, 24, 24, 0, 1, 0),            # three places: 66.4 / 79.2
    (21, 192, 64, 64, 0, FS, 0, 16, 16, 0, 1, 1),           # two places, one round: 40.7 / 36.2
    (128, 128, 43, 45, 0, FS, 0, 21, 22, 0, 1, 0),          # rows that are no whole number of vectors: 81.4 / 96.1
    (33, 192, 55, 55, 0, FS, 0, 13, 13, 0, 1, 1),           # one round of them: 55.1 / 43.2
    (106, 240, 27, 27, 0, FS, 0, 6, 6, 0, 1, 2),            # 51.2 / 52.6 with dy alone, 51.0 with x beside it
    (97, 128, 64, 64, 0, BS, 12, 0, 0, 0, 1, 0),            # samples 2 MiB apart, two rounds: 112.7 / 154.9
    (64, 256, 56, 56, 0, BS, 32, 0, 0, 0, 1, 1),            # half of x is needed again: 114.7 / 113.5
    (64, 256, 56, 56, 0, BS, 48, 0, 0, 0, 1, 0),            # three quarters: 114.5 / 123.2
    (64, 256, 56, 56, 0, FS, 0, 53, 53, 0, 1, 0),           # 118.8 / 137.5
    (21, 250, 64, 64, 0, FS, 0, 28, 28, 0, 1, 1),           # two places, less than half of the rows: 53.7 / 45.0
    # backward, x beside dy
    (21, 250, 64, 64, 0, FS, 0, 35, 35, 0, 1, 2),           # two places, more than half: 53.5 / 50.2 (dy alone 55.0)
    (64, 256, 56, 56, 1, BS, 32, 0, 0, 0, 1, 2),            # half of x: 65.9 / 54.5 (57.2)
    (64, 256, 56, 56, 1, BS, 25, 0, 0, 0, 1, 1),            # 0.39: 65.3 / 52.9 (53.9)
    (94, 128, 64, 64, 1, FULL, 0, 0, 0, 0, 1, 0),           # samples 1 MiB apart, two rounds: 63.4 / 113.6
    (98, 112, 64, 64, 1, FULL, 0, 0, 0, 0, 1, 2),           # 62.5 / 49.6
    (128, 256, 32, 32, 1, BS, 1, 0, 0, 0, 1, 0),            # 39.6 / 49.1
    (64, 256, 56, 56, 1, FULL, 0, 0, 0, 0, 1, 2),           # 66.9 / 53.9
    (130, 128, 28, 28, 0, FS, 0, 7, 7, 2, 1, 2),            # Eq. 4
    (25, 128, 64, 64, 0, FS, 0, 16, 16, 0, 1, 2),           # one round: 37.2 / 26.7
    (60, 128, 27, 27, 0, BS, 4, 0, 0, 0, 1, 0),             # 0.44 of the registers: 15.5 / 17.4
    (34, 160, 35, 35, 0, BS, 4, 0, 0, 0, 1, 0),             # 0.53 of the device: 16.7 / 17.3
    (54, 96, 55, 55, 1, BS, 13, 0, 0, 0, 1, 0),             # bf16, odd planes, 0.60: 27.0 / 31.4
    (48, 128, 83, 83, 1, BS, 2, 0, 0, 0, 1, 0),             # two rounds of them, 0.81: 67.7 / 72.3
    (32, 96, 112, 112, 0, FULL, 0, 0, 0, 0, 1, 2),          # three rounds, teams of 8: 100.2 / 91.2
    (64, 64, 112, 112, 0, FULL, 0, 0, 0, 0, 1, 2),          # four, teams of 16: 124.6 / 119.5
    (64, 128, 80, 80, 0, FULL, 0, 0, 0, 0, 1, 0),           # four, teams of 8: 121.9 / 123.9
    (128, 128, 80, 80, 1, FULL, 0, 0, 0, 0, 1, 2),          # the same in bf16: 147.3 / 114.7
    (64, 256, 56, 56, 0, FULL, 0, 0, 0, 0, 1, 0),           # four, teams of 4: 115.5 / 119.6
    (8, 16, 8, 8, 0, BS, 2, 0, 0, 0, 1, 0),                 # small
]


def test_layers_on_both_sides_of_the_lines_of_one_block_per_unit(harness):
    lines = [" ".join(map(str, l[:10] + (0,) + l[10:11])) for l in LAYERS]
    got = [int(line.split()[0]) for line in _run(harness, "rule", "\n".join(lines) + "\n").splitlines()]
    assert len(got) == len(LAYERS)
    for layer, kernel in zip(LAYERS, got):
        assert kernel == layer[11], (layer, kernel)


def test_plans_of_one_block_per_unit_hold_every_vector_and_fit_the_device(harness):
    assert int(_run(harness, "sweep").split()[1]) > 100000
