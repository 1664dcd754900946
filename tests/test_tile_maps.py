"""Index maps of the binary64 tile kernel, on the host: for every tile shape the
library uses or the tuner tries, and every operand layout, each operand value is
staged once, each lane's fragments meet at the same k and belong to the element
of C that the lane stores, and the epilogue touches every element of the tile
once and none outside it."""
import os
import subprocess

import pytest

from paper_2203_09353_amd import bgemm, tune

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2203_09353_amd", "csrc")


def test_every_shape_covers_its_tile_once(tmp_path):
    tuned = sorted({s for _, cands in tune.CANDIDATES.values() for s in cands})
    exe = str(tmp_path / "tile_maps")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC,
                    "-DTUNED_SHAPES=" + " ".join("SHAPE(%s)" % s for s in tuned),
                    os.path.join(HERE, "tile_maps.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.split() == ["ok", str(8 + len(tuned))], r.stdout


@pytest.mark.parametrize("shape,m,n,k,batch", [
    (2, 512, 512, 512, 5000), (3, 256, 190, 64, 1000), (7, 128, 48, 64, 530),
    (1, 500, 64, 8, 5000), (4, 60, 32, 40, 5000), (5, 32, 64, 40, 5000), (5, 65, 64, 64, 700),
    (0, 32, 32, 32, 1000), (0, 32, 32, 32, 1), (6, 9, 15, 16, 2100)])
def test_a_batch_of_each_shape(shape, m, n, k, batch):
    """Sizes that take each tile shape by default on 256 compute units: a change
    of the rule that leaves a shape to no one shows here."""
    assert bgemm.lib().bgi_pick_tile(1, m, n, k, batch, 256) == shape


def test_override_refuses_unknown_shapes_and_handles():
    L = bgemm.lib()
    assert L.bgi_force_tile(None, 0) == 5
