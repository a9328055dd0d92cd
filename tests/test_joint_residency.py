"""The most samplers that run beside the launch that streams their rows (CPU): by brute
force over every way to place them, streaming workgroups of the worst size that the launch
bounds allow keep as many places as there are CUs."""
import itertools
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def most(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("layout") / "layout_ref")
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", exe, os.path.join(HERE, "layout_ref.cpp")], check=True)

    def run(cus, lds):
        return int(subprocess.run([exe], input=f"{cus} {lds}\n", capture_output=True, text=True, check=True).stdout)

    return run


def places(lds):
    """Workgroups of 512 / 3 registers per lane (four waves, one per SIMD) and lds bytes on a CU."""
    return min(512 // (512 // 3 // 8 * 8), (160 << 10) // lds)


@pytest.mark.parametrize("cus", [1, 2, 3, 4])
@pytest.mark.parametrize("lds", [1, 40960, 47104, 54000, 60000, 81920, 100000, 163840])
def test_places_are_left(most, cus, lds):
    n, per_cu = most(cus, lds), places(lds)
    for split in itertools.product(range(per_cu + 1), repeat=cus):
        if sum(split) == n:
            assert sum(per_cu - x for x in split) >= cus
    assert cus * per_cu - (n + 1) < cus  # (one more would leave fewer)


def test_largest_batches(most):
    """256 CUs, a sampler's LDS at V = 256000 and at the largest vocabulary: 512 of the 768
    samplers that would be resident by themselves."""
    assert most(256, 30464 + 8000) == most(256, 30464 + 16384) == 512
