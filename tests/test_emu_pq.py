"""The PQ assignment's kernel (pq.hip) built for the host against the wave64
emulation (tests/wave_emu: the f16 MFMA's operand layout among others) and run
under AddressSanitizer: codes and labels equal to the oracle's for every padded
width, rows around the 64-row tile, a few undecided rows of a tile, tiles that
wait for the dense evaluation (in turns of eight, four and one, past 32 tiles of
a wave, whole words of codes and single bytes), tiles that skip the screen, and
subspaces that are dense from the start; no access leaves its allocation. No GPU
is involved."""
import os
import subprocess

import numpy as np
import pytest

from test_emu_screen_i8 import CLANG, CSRC, HERE
from test_gpu_pq_screen import data


@pytest.fixture(scope="module")
def emu_pq(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("clang++ of the ROCm toolchain not found")
    d = tmp_path_factory.mktemp("wave_emu_pq")
    with open(os.path.join(CSRC, "pq.hip")) as f:
        src = f.read()
    with open(d / "pq_host_src.hip", "w") as f:
        f.write(src)
    exe = str(d / "pq_host")
    cmd = [CLANG, "-std=c++20", "-O1", "-g", "-fsanitize=address", "-fno-omit-frame-pointer", "-ffp-contract=off",
           "-I", os.path.join(HERE, "wave_emu"), "-I", str(d), "-I", CSRC,
           os.path.join(HERE, "wave_emu", "pq_host.cpp"), "-o", exe, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


@pytest.mark.parametrize("kind,n,D,M", [
    ("plain", 1, 4, 1), ("plain", 65, 8, 1), ("plain", 70, 32, 4), ("plain", 70, 16, 1), ("plain", 64, 12, 4),
    ("plain", 70, 20, 4), ("plain", 20, 120, 30), ("range", 70, 16, 2), ("far30", 70, 16, 2),
    ("equal", 70, 32, 4), ("equal", 600, 16, 1), ("one", 1300, 8, 2), ("vanish", 70, 8, 1), ("vast", 70, 8, 8),
    ("blocks", 8 * 64 * 37 + 5, 4, 1), ("blocks", 8 * 64 * 9 + 5, 8, 4),
])
def test_emulated_codes(emu_pq, oracle_mod, tmp_path, kind, n, D, M):
    x, cb = data(kind, n, D, M, n + D + M)
    src, dst = tmp_path / "in.bin", tmp_path / "out.bin"
    with open(src, "wb") as f:
        f.write(np.array([n, D, M], np.int64).tobytes() + x.tobytes() + cb.tobytes())
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:halt_on_error=1")
    r = subprocess.run([emu_pq, str(src), str(dst), "1"], capture_output=True, text=True, timeout=900, env=env)
    assert r.returncode == 0 and "AddressSanitizer" not in r.stderr, r.stderr[-6000:]
    raw = np.fromfile(dst, np.uint8)
    want = oracle_mod.pq_encode(x, cb)
    assert (raw[:n * M].reshape(n, M) == want).all()
    assert (raw[n * M:].view(np.int32).reshape(M, n) == want.T).all()
