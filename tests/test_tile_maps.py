"""Index maps of the binary64 tile kernel, on the host: for every tile shape the
library uses or the tuner tries, and every operand layout, each operand value is
staged once, each lane's fragments meet at the same k and belong to the element
of C that the lane stores, and the epilogue touches every element of the tile
once and none outside it."""
import os
import subprocess

from paper_2203_09353_amd import tune

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
