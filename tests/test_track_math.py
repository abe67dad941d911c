"""The last step of a tracked image (image_close of sblm_math.h, compiled for the
host by track_check.cpp): what it accepts as an image solves the lens equation,
from any start -- far from the lenses, next to a critical curve, and where a step
at |det J| = 0 has thrown it."""
import json
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1208_4830_amd", "csrc")


@pytest.fixture(scope="module")
def families(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("track") / "track_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-Wall",
                    "-Wno-unknown-pragmas", "-I", CSRC, os.path.join(HERE, "track_check.cpp"),
                    "-o", exe], check=True)
    return json.loads(subprocess.run([exe, "500000"], check=True, capture_output=True,
                                     text=True).stdout)


@pytest.mark.parametrize("family", ["given", "far", "random", "critical"])
def test_accepted_images_solve_the_lens_equation(families, family):
    f = families[family]
    # most starts end at an image (some meet no image within their steps)
    assert f["accepted"] >= 0.3 * f["tried"], f
    # The bounds leave a position error of at most 1e-6 of the step, the step
    # being at most 1e-2 of the distance to a lens, and the residual (1 + |g|)
    # times that, the factor covered by the bound's own (1 + |g|^2)(3 + |g|^2):
    # |residual| <= 2e-8 (1 + |z|), and its square 4e-16 (1 + |z|)^2.
    assert f["worst"] <= 1e-15, f
