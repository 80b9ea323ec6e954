"""Host rules of the pass launches (lf2_rules.hpp), compiled with g++ (no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


def _run(tmp_path, name):
    exe = str(tmp_path / name)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-o", exe,
                           os.path.join(ROOT, "tests", "model", name + ".cpp")])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout


def test_grids_of_the_binned_passes(tmp_path):
    _run(tmp_path, "grid_check")


def test_autotuner_choice(tmp_path):
    _run(tmp_path, "tune_check")
