"""The transforms' range of magnitudes, driven lane by lane on the CPU against
numpy: no intermediate is larger than the sums it stands for, up to the
butterflies' own roots (tan(3 pi/8) = 2.4), so that inputs far up the range of
float come out as exactly as inputs near one."""

import os
import struct
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def drivers(tmp_path_factory):
    out = tmp_path_factory.mktemp("range")
    inc = os.path.join(ROOT, "paper_0911_2889_amd", "csrc")
    exes = {name: str(out / name) for name in ("fft_engine_check", "mixed_fft_check")}
    builds = [subprocess.Popen(["/opt/rocm/bin/hipcc", "-O0", "-std=c++17", "-I", inc,
                                os.path.join(ROOT, "tests", "native", name + ".cpp"), "-o", exe])
              for name, exe in exes.items()]
    assert [b.wait() for b in builds] == [0, 0]

    def run(header, x):
        name = "fft_engine_check" if len(header) == 6 else "mixed_fft_check"
        res = subprocess.run([exes[name]], input=struct.pack(f"{len(header)}i", *header) + x.tobytes(),
                             capture_output=True, check=True)
        return np.frombuffer(res.stdout, dtype=np.complex64)

    return run


def inputs(n, kept, inv, kind):
    """White values of 1e33, or one mode of it: their sums stay below 16384 * 4e33 = 7e37."""
    rng = np.random.default_rng(n + inv)
    if kind == "white":
        x = 1e33 * (rng.standard_normal(n) + 1j * rng.standard_normal(n))
    else:
        k = int(rng.integers(1, kept))
        x = np.eye(1, n, k)[0] * 1e33 if inv else 1e33 * np.exp(2j * np.pi * k * np.arange(n) / n)
    x = x.astype(np.complex64)
    if inv:
        x[kept:n - kept] = 0
    return x


def check(y, x, inv):
    ref = np.fft.ifft(x.astype(np.complex128)) * len(x) if inv else np.fft.fft(x.astype(np.complex128))
    assert np.isfinite(y).all()
    # a transform of b bits rounds about 2 b times at 2^-24 / sqrt(3) each in the mean square: 2.6e-7 at 2^14
    y = y.astype(np.complex128)
    assert np.linalg.norm(y - ref) / np.linalg.norm(ref) < 5e-7


@pytest.mark.parametrize("kind", ["white", "mode"])
@pytest.mark.parametrize("inv", [0, 1])
@pytest.mark.parametrize("pts", [8, 16])
def test_power_of_two_lengths(drivers, pts, inv, kind):
    for logn in range(4, 15):
        n = 1 << logn
        x = inputs(n, n // 4, inv, kind)
        check(drivers((logn, inv, 1, 0, pts, 0), x), x, inv)


@pytest.mark.parametrize("kind", ["white", "mode"])
@pytest.mark.parametrize("inv", [0, 1])
def test_product_grid_lengths(drivers, inv, kind):
    for logn in range(6, 15):
        n = 3 << (logn - 2)
        x = inputs(n, n // 3, inv, kind)
        check(drivers((logn, inv, 1, 0), x), x, inv)
