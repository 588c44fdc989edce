"""The mixed-radix product-grid transforms, driven lane by lane on the CPU
against numpy, for every number of lanes the kernels give them."""

import os
import struct
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = tmp_path_factory.mktemp("mixed") / "mixed_fft_check"
    src = os.path.join(ROOT, "tests", "native", "mixed_fft_check.cpp")
    inc = os.path.join(ROOT, "paper_0911_2889_amd", "csrc")
    subprocess.run(["/opt/rocm/bin/hipcc", "-O1", "-std=c++17", "-I", inc, src, "-o", str(out)], check=True,
                   capture_output=True)
    return out


@pytest.mark.parametrize("logn,full", [(n, 0) for n in range(6, 15)] + [(n, 1) for n in (4, 5, 6)])
def test_mixed_transforms_match_numpy(exe, logn, full):
    n = 1 << logn if full else 3 << (logn - 2)
    kept = n // 4 if full else n // 3
    for inv in (0, 1):
        for lanes in (0, 1, 2, 4):
            if lanes == 0 and logn == 4:
                continue  # one lane is the fewest
            rng = np.random.default_rng(100 * logn + 10 * inv + lanes)
            x = (rng.standard_normal(n) + 1j * rng.standard_normal(n)).astype(np.complex64)
            if inv:
                x[kept:n - kept] = 0
            out = subprocess.run([str(exe)], input=struct.pack("4i", logn, inv, lanes, full) + x.tobytes(),
                                 capture_output=True, check=True).stdout
            y = np.frombuffer(out, dtype=np.complex64)
            ref = np.fft.ifft(x.astype(np.complex128)) * n if inv else np.fft.fft(x.astype(np.complex128))
            # a transform of b bits rounds about 2 b times at 2^-24 / sqrt(3) each in the mean square: 2.6e-7 at 2^14
            assert np.linalg.norm(y - ref) / np.linalg.norm(ref) < 5e-7, (inv, lanes)
