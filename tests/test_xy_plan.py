"""How the iteration's xy pass is cut (host code): strips, chunks, workgroup sizes
and launch ranges, and which form the volumes of the GPU tests take."""
import os
import shutil
import subprocess

import pytest

from xy_forms import BATCHES, VOLUMES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = tmp_path_factory.mktemp("xyf") / "xyf_check"
    csrc = os.path.join(ROOT, "paper_2404_02813_amd", "csrc")
    subprocess.run([HIPCC, "-std=c++17", "-O1", "-x", "hip", "--offload-arch=gfx950",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "include"), "-I", csrc,
                    os.path.join(ROOT, "tests", "xyf_check.cpp"),
                    os.path.join(csrc, "rsf_split.hip"), "-o", str(exe)],
                   check=True, capture_output=True)

    def run(*args):
        r = subprocess.run([str(exe), *map(str, args)], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return r.stdout
    return run


def test_strips_chunks_and_launches(check):
    assert "xyf ok" in check()


@pytest.mark.parametrize("radius,shape,waves,chunks", VOLUMES)
def test_form_of_a_volume(check, radius, shape, waves, chunks):
    assert check(radius, 0, *shape).split() == [str(waves), str(chunks)]


@pytest.mark.parametrize("radius,shapes,waves", BATCHES)
def test_form_of_a_batch(check, radius, shapes, waves):
    assert check(radius, 0, *sum(shapes, ())).split()[0] == str(waves)


# strips times slices fill the CUs: a third chunk evens the SIMDs' loads, one of
# 128^3 or less is cut by their mean
@pytest.mark.parametrize("force,radius,shape,chunks", [
    (0, 6, (257, 301, 316), 3), (0, 6, (300, 300, 100), 3), (1, 9, (628, 601, 88), 3),
    (0, 3, (192, 320, 352), 2), (1, 3, (192, 320, 352), 2), (0, 6, (128, 128, 128), 6)])
def test_row_chunks(check, force, radius, shape, chunks):
    assert check(radius, force, *shape).split() == ["4", str(chunks)]
