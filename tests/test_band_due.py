"""The prediction of a row's next band, left to the update kernel, in a host program."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_a_band_predicted_later_is_the_same(tmp_path):
    exe = str(tmp_path / "band_due")
    build = subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-Werror", "-Wno-format-extra-args", "-Wno-format-security",
                            "-I", os.path.join(ROOT, "paper_2402_11857_amd", "csrc"), "-o", exe,
                            os.path.join(ROOT, "tests", "host", "band_due.cpp")], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and "band due ok" in run.stdout, run.stdout + run.stderr
