"""Partition of the compact fluid nodes into gathered chunks, on the CPU: the
library's own rules (csrc/plan.hpp) over a host model of the order and of the
halos. Every chunk starts at a multiple of 64 and the last one ends at the last
fluid node, also where the last stretch, whose length is no multiple of 64, is
cut short by its halo."""
import os
import subprocess

import numpy as np
import pytest

from paper_1303_2470_amd import inputs

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1303_2470_amd", "csrc")


@pytest.fixture(scope="module")
def partition(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("chunks") / "chunk_partition")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", CSRC, os.path.join(HERE, "chunk_partition.cpp"), "-o", exe])

    def run(mask, nh):
        nz, ny, nx = mask.shape
        nf = int((mask == 0).sum())
        cap = 2 * -(-nf // 256)
        out = subprocess.run([exe, str(nx), str(ny), str(nz), str(256 * nh), str(cap)], input=mask.tobytes(),
                             capture_output=True, check=True).stdout.split()
        v = np.array(out, dtype=np.int64)
        assert v[0] == nf
        return nf, v[1:].reshape(-1, 2)
    return run


# (mask, nh: 256 nh nodes per chunk). The first seven have a last stretch that
# is cut short; the others are the shapes around it.
TAILS = {
    "random 79x52x13 seed 2": (lambda: inputs.random_mask(79, 52, 13, 0.05, seed=2), 2),
    "random 79x52x13 seed 5": (lambda: inputs.random_mask(79, 52, 13, 0.05, seed=5), 2),
    "random 79x52x13 seed 11": (lambda: inputs.random_mask(79, 52, 13, 0.05, seed=11), 2),
    "random 83x85x9 seed 0": (lambda: inputs.random_mask(83, 85, 9, 0.1, seed=0), 2),
    "bulk 97x12x13": (lambda: inputs.bulk_mask(97, 12, 13), 2),
    "spheres 65^3, 256": (lambda: inputs.sphere_pack(65, 6, 0.5, seed=1), 1),
    "bulk 97x12x13, 256": (lambda: inputs.bulk_mask(97, 12, 13), 1),
    "column": (lambda: inputs.slit_mask(1, 1, 34), 2),
    "bulk 33x5x9": (lambda: inputs.bulk_mask(33, 5, 9), 2),
    "random 40^3 0.6": (lambda: inputs.random_mask(40, 40, 40, 0.6, seed=4), 2),
    "spheres 50^3": (lambda: inputs.sphere_pack(50, 6, 0.4, seed=6), 2),
}


@pytest.mark.parametrize("name", TAILS)
def test_chunks_cover_the_fluid_nodes(partition, name):
    make, nh = TAILS[name]
    nf, ch = partition(np.ascontiguousarray(make(), dtype=np.uint8), nh)
    assert len(ch) > 0
    base, length = ch[:, 0], ch[:, 1]
    assert (base % 64 == 0).all() and (length > 0).all() and (length <= 256 * nh).all()
    assert base[0] == 0 and (base[1:] == base[:-1] + length[:-1]).all()
    assert base[-1] + length[-1] == nf


def test_ragged_lattices(partition):
    """Shapes at random: every remainder of the last stretch."""
    rng = np.random.default_rng(1)
    for _ in range(40):
        nx, ny, nz = (int(v) for v in rng.integers(3, 100, 3))
        nz = max(1, min(nz, 60000 // (nx * ny)))
        m = inputs.random_mask(nx, ny, nz, float(rng.choice([0.0, 0.05, 0.1, 0.4])), seed=int(rng.integers(1 << 30)))
        for nh in (1, 2):
            nf, ch = partition(np.ascontiguousarray(m, dtype=np.uint8), nh)
            if len(ch) == 0:  # not offered
                continue
            assert (ch[:, 0] % 64 == 0).all(), (nx, ny, nz, nh)
            assert (ch[:-1, :].sum(1) == ch[1:, 0]).all() and ch[-1].sum() == nf, (nx, ny, nz, nh)
