"""Step launches at the runtime's limit (fewer than 2^32 threads in a
dimension), on the CPU: the library's own rule (csrc/plan.hpp) at products of
nodes and species around it. A candidate beyond it must not be offered: its
refused launch would be timed as a step of no length."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1303_2470_amd", "csrc")


@pytest.fixture(scope="module")
def launchable(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_limits")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", CSRC, os.path.join(HERE, "plan_limits.cpp"), "-o", exe])

    def ask(variant, K, gs, geoms, nq=4):
        line = f"{variant} {K} {gs} {nq} {len(geoms)} " + " ".join(
            f"{nx} {ny} {nz} {S} {nx * ny * nz} {nch} 2" for nx, ny, nz, S, nch in geoms)
        return subprocess.run([exe], input=line, capture_output=True, text=True, check=True).stdout.strip() == "1"
    return ask


def cube(S, nch=0):
    return (256, 256, 256, S, nch)  # 2^24 nodes, 65,536 tiles of 256


# nodes x species   9: K = 1, 2, 4   variant 0, one species a block, uptake's 9
CUBES = [(63, True, True, True, True, True),        # 2^30 - 2^24
         (64, False, True, True, True, True),       # 2^30: four quantity blocks a tile
         (127, False, True, True, True, True),
         (128, False, False, True, True, True),     # 2^31
         (254, False, False, True, True, True),
         (256, False, False, False, False, False)]  # 2^32


@pytest.mark.parametrize("row", CUBES, ids=lambda r: f"S{r[0]}")
def test_products_of_nodes_and_species(launchable, row):
    S, k1, k2, k4, direct, uptake = row
    assert [launchable(9, K, 1, [cube(S)]) for K in (1, 2, 4)] == [k1, k2, k4]
    assert launchable(0, 1, 1, [cube(S)]) == direct
    assert launchable(9, 1, 1, [cube(S)], nq=1) == uptake
    # blocks that walk several species are far from the limit
    assert launchable(0, 2, 64, [cube(S)]) and launchable(6, 2, 32, [cube(S)]) and launchable(7, 2, 32, [cube(S)])
    assert launchable(8, 2, 32, [cube(S, nch=2 ** 24 // 512)])


def test_the_limit_is_the_handle_s(launchable):
    """Two geometries, each well inside it."""
    assert launchable(9, 1, 1, [cube(32)]) and launchable(9, 1, 1, [cube(31), cube(32)])
    assert not launchable(9, 1, 1, [cube(32), cube(32)])


def test_recording_blocks_count(launchable):
    """Variant 0 on planes of 256 nodes: nz blocks, one more per pair and one
    per 2,048 tiles; 2^24 blocks of 256 threads are one too many."""
    for nz, ok in ((16769025, True), (16769026, False)):
        assert nz + 1 + -(-nz // 2048) == 2 ** 24 - (1 if ok else 0)
        assert launchable(0, 1, 1, [(16, 16, nz, 1, 0)]) == ok


def test_threads_of_larger_blocks(launchable):
    """Variant 6 with four planes: 1,024 threads, a quarter of the blocks."""
    assert launchable(6, 4, 1, [(64, 256, 1024, 255, 0)])       # 2^24 nodes, 255 species
    assert not launchable(6, 4, 1, [(64, 256, 1024, 256, 0)])
