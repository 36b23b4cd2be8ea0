"""The kernels in a CPU build that checks every access to memory and LDS (tests/lanes), against the oracle: layers, single
matrices, decompression, the device encoder and what goes before the matrix-core kernel at small odd sizes, every layout, numbering, grid and tile; and streams that are none,
which must stay inside their buffers whatever they decode to."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(HERE, "lanes"))


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    from cpu_build import build

    return build(str(tmp_path_factory.mktemp("lanes")))


@pytest.mark.parametrize("kind,count", [("layer", 60), ("layer_corrupt", 24), ("single", 60), ("single_corrupt", 18), ("encode", 60), ("blocks", 60), ("dispatch", 80)])
def test_every_access_is_inside(library, kind, count):
    cmd = [sys.executable, os.path.join(HERE, "lanes", "cases.py"), kind, "1", str(count)]
    r = subprocess.run(cmd, env={**os.environ, "QMOE_LIBRARY": library}, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.rstrip().endswith("done"), r.stdout[-3000:]
