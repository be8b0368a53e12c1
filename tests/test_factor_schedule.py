"""The factorisation's schedule on the CPU: factor_replay.cpp runs the kernel's own schedule header with as many resident workgroups as asked."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BLOCKS = [1, 2, 3, 4, 5, 8, 9, 10, 13, 16, 17, 22, 33]


@pytest.fixture(scope="module")
def replay(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("replay") / "factor_replay")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2406_09904_amd", "csrc"),
                           os.path.join(ROOT, "tests", "factor_replay.cpp"), "-o", exe])
    return lambda nb, grid, slots, helps, seed: subprocess.run([exe, *map(str, (nb, grid, slots, helps, seed))], capture_output=True, text=True, timeout=60)


def _grid(nb):
    return 1 + min(nb * (nb - 1) // 2, 255)


@pytest.mark.parametrize("slots", [1, 2, 3, 4, 8, 256])
def test_waits_end_however_few_workgroups_are_resident(replay, slots):
    for nb in BLOCKS + ([64] if slots in (1, 2, 256) else []):
        for seed in range(4):
            r = replay(nb, _grid(nb), slots, 1, seed)
            assert r.returncode == 0, (nb, seed, r.stdout)


@pytest.mark.parametrize("grid", [1, 2, 3, 5])
def test_waits_end_with_a_small_grid(replay, grid):
    for nb in BLOCKS:
        for seed in range(3):
            r = replay(nb, min(grid, _grid(nb)), 256, 1, seed)
            assert r.returncode == 0, (nb, seed, r.stdout)


@pytest.mark.parametrize("slots,nb", [(1, 3), (1, 16), (2, 9), (2, 33)])
def test_a_chain_that_only_waits_needs_three(replay, slots, nb):
    """What the chain's own tasks are for."""
    assert replay(nb, _grid(nb), slots, 0, 1).returncode == 1
    assert replay(nb, _grid(nb), 3, 0, 1).returncode == 0


@pytest.mark.parametrize("nb", [1, 2])
def test_two_blocks_need_nobody(replay, nb):
    """Why the kernel's chain looks for no crew there."""
    assert replay(nb, _grid(nb), 1, 0, 1).returncode == 0
