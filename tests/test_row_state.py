"""The row descriptor's state changes, as the kernels run them, in a host program."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_a_block_that_starts_late_sees_the_same_work(tmp_path):
    """Block 0 of a row finishes the search on its own when a wait has run out (and whenever the list is short); blocks that
    start after that derive what they do from the descriptor it has written.  With the next step's band already in force
    there, such a block indexed a 256-bin histogram by keys relative to the wrong band."""
    exe = str(tmp_path / "row_state")
    build = subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-Werror",
                            "-I", os.path.join(ROOT, "paper_2402_11857_amd", "csrc"), "-o", exe,
                            os.path.join(ROOT, "tests", "host", "row_state.cpp")], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and "row state ok" in run.stdout, run.stdout + run.stderr
