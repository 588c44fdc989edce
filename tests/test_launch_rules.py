"""The rules by which the library picks its launches, on a checked model of the
HIP calls (CPU only, with the host sanitizers): devices and kernels that the
model of test_host_sanitizers.py does not have."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NATIVE = os.path.join(ROOT, "tests", "native")
CSRC = os.path.join(ROOT, "paper_0911_2889_amd", "csrc")
FLAGS = ["-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", "-fsanitize=address,undefined",
         "-fno-sanitize-recover=undefined", "-I", os.path.join(NATIVE, "hipstub"), "-I", NATIVE, "-I", CSRC,
         "-I", os.path.join(ROOT, "include")]


@pytest.fixture(scope="module")
def drive(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("g++ is not available")
    exe = tmp_path_factory.mktemp("rules") / "launch_rules_check"
    subprocess.run([cxx] + FLAGS + [os.path.join(NATIVE, "launch_rules_check.cpp"), "-x", "c++",
                                    os.path.join(CSRC, "flame_api.hip"), "-o", str(exe)],
                   check=True, capture_output=True)

    def run(what):
        env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=1", UBSAN_OPTIONS="halt_on_error=1")
        res = subprocess.run([str(exe), what], capture_output=True, text=True, env=env, timeout=120)
        assert res.returncode == 0 and res.stdout.endswith("OK\n"), res.stderr[-3000:]

    return run


def test_persistent_grid_is_two_workgroups_per_compute_unit(drive):
    drive("persistent_default")


def test_resident_kernels_need_the_lds_they_ask_for(drive):
    drive("resident_lds")


def test_resident_paths_are_clean_under_sanitizers(drive):
    drive("resident_paths")


def test_averages_of_two_flames_share_no_counters(drive):
    drive("averages_apart")


def test_disabling_the_product_grid_gives_the_papers_grid(drive):
    drive("step_grids")


def test_autotuner_times_equal_kernels_once(drive):
    drive("autotune_equals")
