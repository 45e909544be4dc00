"""Which single products take the kernel for few output tiles, and in which form: the rule itself, on the CPU."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CUS = 256


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("split") / "rule")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", os.path.join(HERE, "split_rule.cpp"), "-o", exe], check=True)

    def ask(calls):
        """(b, block rows, tokens, blocks per row, fullest row) -> waves, 0 for the other kernel"""
        lines = "".join(f"{b} {nbr} {t} {round(nbr * mean)} {full} 0 {CUS}\n" for b, nbr, t, mean, full in calls)
        res = subprocess.run([exe], input=lines, capture_output=True, text=True, check=True).stdout.split()
        assert all(once == "1" for once in res[1::2])
        return [int(w) for w in res[::2]]

    return ask


def tiles(call):
    return call[1] * (call[0] // 64) * ((call[2] + 63) // 64)


def test_narrow_outputs(rule):
    """One to a dozen block rows under many tokens: up to one tile of 64 x 64 per CU (128-wide blocks: two) the tile is shared by
    waves, whose eight chains of sums are more exact than the streaming kernel's one."""
    calls = [(b, nbr, t, mean, mean + extra) for b in (64, 128) for nbr in range(1, 13) for t in range(300, 20000, 450)
             for mean in (1, 3, 8, 20, 60) for extra in (0, 9)]
    calls = [c for c in calls if tiles(c) <= CUS * (2 if c[0] == 128 else 1)]
    assert len(calls) > 2000
    for call, waves in zip(calls, rule(calls)):
        assert waves in (4, 8), call


def test_form_by_load(rule):
    """Eight waves to a tile where each has a CU to itself and no row is long, and on few more tiles than CUs where a row is very long
    or much longer than the others; else four (there eight are a round more)."""
    for call, waves in (((128, 28, 513, 20, 20), 4), ((64, 32, 640, 44, 44), 4), ((64, 32, 640, 60, 60), 8), ((128, 32, 257, 34, 40), 8), ((64, 7, 2084, 5, 12), 8), ((128, 8, 900, 20, 20), 4),
                        ((64, 25, 384, 20, 20), 8), ((64, 25, 384, 31, 31), 4), ((64, 24, 800, 9, 9), 4), ((128, 10, 960, 4, 30), 8),
                        ((64, 60, 300, 2, 16), 8), ((64, 60, 300, 2, 9), 4)):
        assert rule([call])[0] == waves, call
    calls = [(b, nbr, t, mean, mean) for b in (64, 128) for nbr in range(1, 60) for t in range(300, 3000, 170) for mean in (1, 4, 9, 30)]
    for call, waves in zip(calls, rule(calls)):
        units = call[1] * call[0] // 64
        groups, padded = (call[2] + 63) // 64, (units + 7) // 8 * 8
        launched = (units if units < 12 and units != 8 and padded * groups > CUS else padded) * groups
        stages = call[3] * call[0] // 64
        assert waves in ((0, 8) if CUS < launched <= 1.75 * CUS and stages > 48 else (0, 4) if launched > CUS else
                         (8,) if stages <= 20 else (4,)), call


def test_line_to_the_streaming_kernel(rule):
    """Up to the line by tiles always waves; beyond it where they are faster: not for short equal rows, for long ones and for one
    row much fuller than the others (measured products, each at least 10 % apart)."""
    calls = [(b, nbr, t, mean, max(mean, full)) for b in (64, 128) for nbr in (1, 3, 4, 9, 16, 25, 50, 90) for t in range(257, 2600, 101)
             for mean in (1, 5, 30) for full in (0, 7, 40)]
    for call, waves in zip(calls, rule(calls)):
        if tiles(call) * 4 <= CUS * (8 if call[0] == 128 else 4 if call[4] < 8 else 5):
            assert waves in (4, 8), call
    for call, split in (((64, 25, 1189, 0.8, 1), False), ((64, 18, 1624, 2.3, 3), False), ((64, 33, 841, 4.3, 5), False),
                        ((64, 40, 906, 4.5, 5), False), ((128, 44, 421, 2, 2), False),
                        ((128, 52, 326, 5.7, 6), False), ((128, 23, 1022, 10, 10), False), ((128, 52, 261, 22, 22), True), ((64, 32, 700, 3.2, 7), True),
                        ((128, 32, 500, 3.2, 7), True), ((128, 64, 330, 1, 4), True),
                        ((64, 42, 1185, 10, 100), True), ((64, 79, 401, 5, 100), True), ((128, 47, 332, 12.8, 64), True),
                        ((128, 10, 2226, 4.8, 16), True)):
        assert (rule([call])[0] > 0) == split, call


def test_what_the_gpu_tests_run(rule):
    """The products of the GPU tests of either form are the rule's for that form."""
    from tests import test_gpu_parity as gpu

    for b, nbr, per_row, full, t in gpu.FOUR_WAVES:
        rows = gpu.rows_of_four_waves(nbr, per_row, full)
        assert rule([(b, nbr, t, sum(rows) / nbr, max(rows))]) == [4], (b, nbr, t)
    for b, nbr, per_row, few, many in gpu.EIGHT_AND_FOUR:
        rows = gpu.rows_of_eight_and_four(nbr, per_row)
        assert rule([(b, nbr, t, sum(rows) / nbr, max(rows)) for t in (few, many)]) == [8, 4], (b, nbr)


def test_workgroups_cover_every_tile_once(rule):
    rule([(64, units, t, 1, 1) for units in range(1, 70) for t in (33, 64, 65, 200, 2100)])
