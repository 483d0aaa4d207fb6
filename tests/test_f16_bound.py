"""The norm bound of the f16 screens (f16_bound.h, built for the host): the
largest scaled centroid norm is covered from the squared norm rounded to fp32,
whatever its size (normal, subnormal, vanished), exceeds it by no more than
the rounding it allows for, and the scale brings it below 2^8."""
import os
import subprocess

import numpy as np
import pytest

from test_emu_screen_i8 import CLANG, CSRC, HERE


@pytest.fixture(scope="module")
def f16_bound(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("clang++ of the ROCm toolchain not found")
    d = tmp_path_factory.mktemp("f16_bound")
    exe = str(d / "f16_bound_host")
    cmd = [CLANG, "-std=c++20", "-O1", "-I", os.path.join(HERE, "wave_emu"), "-I", CSRC,
           os.path.join(HERE, "wave_emu", "f16_bound_host.cpp"), "-o", exe, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]

    def go(n2):
        np.ascontiguousarray(n2, np.float32).tofile(d / "in.bin")
        subprocess.run([exe, str(d / "in.bin"), str(d / "out.bin")], check=True, timeout=60)
        v = np.fromfile(d / "out.bin", np.float64).reshape(-1, 2)
        return v[:, 0], v[:, 1]

    return go


def test_largest_norm_is_covered(f16_bound):
    r = np.random.default_rng(0)
    # every norm whose square is below FLT_MAX, many of them with a subnormal square or none left of it
    norm = 2.0 ** np.concatenate([r.uniform(-90.0, 63.9, 4000), r.uniform(-76.0, -62.0, 4000)])
    n2 = (norm * norm).astype(np.float32)
    assert (n2 == 0).sum() > 50 and ((n2 > 0) & (n2 < 2.0**-126)).sum() > 1000
    scale, top = f16_bound(n2)
    assert (top >= norm * scale).all()
    assert (top <= np.sqrt(norm * norm * (1 + 2.0**-18) + 2.0**-147) * scale).all()
    assert (norm * scale < 2.0**8 * (1 + 2.0**-20)).all()
    assert (np.log2(scale) == np.rint(np.log2(scale))).all()
