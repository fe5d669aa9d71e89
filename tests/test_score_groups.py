"""How single-layer scoring cuts a batch into workgroups, on the CPU: the rule of csrc/score_groups.h compiled into a host program.
Batches of short sequences take single tiles (in groups they were up to twice as slow as in the kernel's first form), long runs of
tiles stay together."""
import os
import subprocess

import pytest

from tests.test_gpu_score_tiles import CASES

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def tiling(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("groups") / "score_groups_check")
    src = os.path.join(HERE, "host_check", "score_groups_check.cpp")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-o", exe, src], check=True)

    def ask(lens, Hkv, kernel):
        r = subprocess.run([exe], input=f"{len(lens)} {sum(lens)} {max(lens)} {Hkv} {kernel}\n", capture_output=True, text=True, check=True)
        waves, tiles, single = (int(x) for x in r.stdout.split())
        return waves, tiles, bool(single)
    return ask


@pytest.mark.parametrize("lens", [[1], [30], [100], [777], [100] * 64, [40] * 200, [1] * 256, [(i * 37) % 130 for i in range(70)]])
@pytest.mark.parametrize("Hkv", [1, 8, 32])
@pytest.mark.parametrize("kernel", [1, 3, 5, 7, 9])
def test_short_sequences_take_single_tiles(tiling, lens, Hkv, kernel):
    assert tiling(lens, Hkv, kernel) == (4, 1, True)


@pytest.mark.parametrize("lens,Hkv", [([32768], 32), ([4096] * 4, 32), ([4096] * 4, 8), ([16384], 16)])
@pytest.mark.parametrize("kernel", [5, 7, 9])
def test_long_runs_stay_together(tiling, lens, Hkv, kernel):
    waves, tiles, single = tiling(lens, Hkv, kernel)
    assert not single and tiles > 1 and waves == (4 if kernel == 5 else 8)


@pytest.mark.parametrize("case", CASES)
def test_gpu_cases_run_the_tiling_they_are_meant_for(tiling, case):
    _, Hkv, kernel, _, _, lens, expected = case
    assert tiling(lens, Hkv, kernel) == expected
