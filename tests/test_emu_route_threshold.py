"""The routing threshold of the planes (select.hip) built for the host against
the wave64 emulation (tests/wave_emu) and run under AddressSanitizer: tau is the
rank_j-th smallest group minimum, on the f16 plane at least the window above
the rank_safe-th, never infinite, and a window that reaches past the rank_max-th
minimum raises the batch's flag. Ranks below, at and above the ranks the f16
branch keeps, few and many groups, equal and infinite minima. No GPU is
involved."""
import os
import subprocess

import numpy as np
import pytest

from test_emu_screen_i8 import CLANG, CSRC, HERE, dynamic_lds

FLT_MAX = np.finfo(np.float32).max


@pytest.fixture(scope="module")
def emu_threshold(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("clang++ of the ROCm toolchain not found")
    d = tmp_path_factory.mktemp("wave_emu_threshold")
    with open(os.path.join(CSRC, "select.hip")) as f:
        src = dynamic_lds(f.read())
    with open(d / "select_host_src.hip", "w") as f:
        f.write(src)
    exe = str(d / "threshold_host")
    cmd = [CLANG, "-std=c++20", "-O1", "-g", "-fsanitize=address", "-fno-omit-frame-pointer",
           "-I", os.path.join(HERE, "wave_emu"), "-I", str(d), "-I", CSRC,
           os.path.join(HERE, "wave_emu", "threshold_host.cpp"), "-o", exe, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


def round_up(x):
    f = x.astype(np.float32)
    return np.where(f.astype(np.float64) < x, np.nextafter(f, np.float32(np.inf)), f)


@pytest.mark.parametrize("f16", [0, 1])
@pytest.mark.parametrize("G,rank,safe,top", [(64, 32, 20, 32), (300, 32, 31, 64), (300, 64, 31, 64), (300, 65, 31, 64),
                                             (257, 400, 9, 64), (33, 50, 12, 64), (4096, 3000, 31, 64)])
def test_threshold_ranks(emu_threshold, tmp_path, G, rank, safe, top, f16):
    r = np.random.default_rng(G + rank)
    Q = 6
    m = (r.normal(size=(Q, G)) - 20.0).astype(np.float32)
    m[1] += 40.0
    m[2] = -3.5
    m[3, :] = np.inf
    bound = (0.01 * r.random(Q)).astype(np.float32)
    bound[4] = 1e3  # past the rank_max-th minimum
    bound[5] = np.inf
    src, dst = tmp_path / "in.bin", tmp_path / "out.bin"
    for wide in (False, True):
        if not wide:
            bound[2], keep = 0.0, [0, 1, 2]
        else:
            keep = range(Q)
        with open(src, "wb") as f:
            f.write(np.array([len(keep), G, rank, safe, top, f16], np.int64).tobytes())
            f.write(m[keep].tobytes() + bound[keep].tobytes())
        env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:halt_on_error=1")
        p = subprocess.run([emu_threshold, str(src), str(dst)], capture_output=True, text=True, timeout=600, env=env)
        assert p.returncode == 0 and "AddressSanitizer" not in p.stderr, p.stderr[-4000:]
        raw = np.fromfile(dst, np.uint32)
        n = len(keep)
        tau, cnt, off = raw[:n].view(np.float32), raw[n:2 * n], raw[2 * n]
        assert (cnt == 0).all()
        s = np.sort(m[keep], axis=1)
        want = s[:, min(rank, G) - 1]
        if f16:
            last = min(top, G)
            cover = round_up(s[:, min(safe, last) - 1].astype(np.float64) + 2.0 * bound[keep].astype(np.float64))
            want = np.minimum(np.maximum(want, cover), FLT_MAX)
            # more equal minima than the branch keeps leave out which, not what, it keeps
            assert bool(off) == bool((cover > s[:, last - 1]).any())
        assert np.array_equal(tau.view(np.uint32), want.view(np.uint32))
