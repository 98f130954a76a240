"""The neighbour search's walk over cells away from the box's faces visits the
rows of the general walk, in its order, for z-major and brick-ordered boxes:
both compiled for the CPU from the library's own header, under the
undefined-behaviour sanitizer."""
import os
import subprocess

from paper_1808_06381_amd import build

SRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host", "cell_order.hip")


def test_short_walk_is_the_general_one(tmp_path):
    exe = str(tmp_path / "cell_order")
    res = subprocess.run(["hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-ffp-contract=off",
                          "-I", build.CSRC, "-Xarch_host", "-fsanitize=undefined",
                          "-Xarch_host", "-fno-sanitize-recover=all", SRC, "-o", exe],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout
    run = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert run.returncode == 0 and "runtime error" not in run.stdout, run.stdout
    assert len(run.stdout.splitlines()) == 7
