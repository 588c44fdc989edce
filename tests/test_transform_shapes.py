"""The transforms in every shape that a kernel gives them (lanes, interleaved
groups, exchange areas), driven lane by lane on the CPU from the kernels' own
shape structs against double-precision DFTs, and bit for bit against each other."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = tmp_path_factory.mktemp("shapes") / "transform_shapes_check"
    src = os.path.join(ROOT, "tests", "native", "transform_shapes_check.cpp")
    inc = os.path.join(ROOT, "paper_0911_2889_amd", "csrc")
    subprocess.run(["/opt/rocm/bin/hipcc", "-O1", "-std=c++17", "-I", inc, src, "-o", str(out)], check=True,
                   capture_output=True)
    return out


@pytest.mark.parametrize("family,least", [("step", 30), ("adjoint", 30), ("averages", 8), ("resident", 60)])
def test_every_shape_of_a_transform(exe, family, least):
    res = subprocess.run([str(exe), family], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
    assert int(res.stdout.split()[-2]) >= least
