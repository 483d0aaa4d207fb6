"""The f16 kernels (screen_f16.hip: quantisation, the assignment screen, the
collecting pass, the routing sample and filter) and the resolving kernel
(resolve.hip) built for the host against the wave64 emulation (tests/wave_emu)
and run under AddressSanitizer: settled rows carry the oracle's labels and the
others are listed, on several dims, tables that are no multiple of a chunk, near
ties of two, a few and many, rows f16 cannot hold and a list that overflows; the
sample minima and the candidates agree with fp64 keys within the bound. No
access leaves its allocation. No GPU is involved."""
import os
import subprocess

import numpy as np
import pytest

from test_emu_screen_i8 import CLANG, CSRC, HERE, strip_fences
from test_gpu_screen_f16 import data

UNWRITTEN = 0x7F7F7F7F


@pytest.fixture(scope="module")
def emu_f16(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("clang++ of the ROCm toolchain not found")
    d = tmp_path_factory.mktemp("wave_emu_f16")
    for name in ("screen_f16", "resolve"):
        with open(os.path.join(CSRC, name + ".hip")) as f:
            src = strip_fences(f.read())
        with open(d / (name + "_host_src.hip"), "w") as f:
            f.write(src)
    exe = str(d / "screen_f16_host")
    cmd = [CLANG, "-std=c++20", "-O1", "-g", "-fsanitize=address", "-fno-omit-frame-pointer", "-ffp-contract=off",
           "-I", os.path.join(HERE, "wave_emu"), "-I", str(d), "-I", CSRC,
           os.path.join(HERE, "wave_emu", "screen_f16_host.cpp"), "-o", exe, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


def run(exe, tmp_path, x, c, tau, list_cap, duel_cap, collect, Cs, stride, L, cus):
    N, D = x.shape
    src, dst = tmp_path / "in.bin", tmp_path / "out.bin"
    n2 = np.zeros(c.shape[0])
    for d in range(D):  # fp64 in dimension order, as the library's norms
        n2 += c[:, d].astype(np.float64) ** 2
    with open(src, "wb") as f:
        f.write(np.array([N, c.shape[0], D, list_cap, duel_cap, collect, Cs, stride, L], np.int64).tobytes())
        f.write(x.tobytes() + c.tobytes() + np.float32(n2.astype(np.float32).max()).tobytes() + tau.tobytes())
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:halt_on_error=1")
    r = subprocess.run([exe, str(src), str(dst), str(cus)], capture_output=True, text=True, timeout=900, env=env)
    assert r.returncode == 0 and "AddressSanitizer" not in r.stderr, r.stderr[-6000:]
    raw = np.fromfile(dst, np.uint32)
    lab, raw = raw[:N].view(np.int32), raw[N:]
    cnt, raw = raw[:3].astype(int), raw[3:]
    left, raw = raw[:list_cap].view(np.int32), raw[list_cap:]
    g = N * (Cs // 16)
    kmin, raw = raw[:g].view(np.float32).reshape(N, -1), raw[g:]
    return lab, cnt, left, kmin, raw[:N], raw[N:].reshape(N, L, 2)


@pytest.mark.parametrize("kind,N,C,D,cap,duels,collect,cus", [
    ("plain", 70, 300, 36, 70, 70, 1, 1), ("plain", 540, 70, 64, 540, 540, 1, 2),
    ("plain", 40, 90, 160, 40, 40, 1, 2), ("plain", 33, 70, 256, 33, 33, 1, 1), ("plain", 5, 1, 4, 5, 5, 1, 1),
    ("ties", 100, 200, 96, 100, 100, 1, 2), ("ties", 100, 150, 128, 100, 20, 1, 2), ("ties", 200, 150, 32, 40, 200, 1, 1),
    ("ties", 60, 150, 64, 60, 60, 0, 1), ("range", 100, 100, 64, 100, 100, 1, 1), ("zero", 40, 50, 32, 40, 40, 1, 1),
])
def test_emulated_f16(emu_f16, oracle_mod, tmp_path, kind, N, C, D, cap, duels, collect, cus):
    x, c = data(kind, N, C, D, seed=N + C + D)
    Cs, stride = (64, max(1, C // 64)) if C >= 64 else (0, 1)
    # keys as -2 v in the plane's scaled units: |C|^2 - 2 X.C of the rows and centroids scaled by the table's power of two
    n2max = (c.astype(np.float64) ** 2).sum(1).max()
    scale = 2.0 ** (8 - ((np.floor(np.log2(np.float32(n2max))) + 2) // 2)) if n2max > 0 else 1.0
    xs, cs = x.astype(np.float64) * scale, c.astype(np.float64) * scale
    key = 0.5 * (cs * cs).sum(1)[None] - xs @ cs.T  # -v in fp64
    M = np.sqrt((cs * cs).sum(1).max())
    xl = np.linalg.norm(xs, axis=1)
    err = (2.0 ** -11 * 1.01 * 2 * xl * M + 2.0 ** -10 * M * np.sqrt(D) + 2.0 ** -10 * np.sqrt(D) * xl
           + (D + 4) * 2.0 ** -21 * (M * M + xl * M) + 1e-12)
    tau = np.sort(key, axis=1)[:, min(12, C - 1)].astype(np.float32)
    L = C + 3
    lab, cnt, left, kmin, ncand, cand = run(emu_f16, tmp_path, x, c, tau, cap, duels, collect, Cs, stride, L, cus)
    want = oracle_mod.assign(x, c)
    listed, nduel, nleft = cnt
    done = lab != UNWRITTEN
    assert (lab[done] == want[done]).all()
    if listed > cap:  # the next screen takes every row
        assert nleft == 0
    elif collect:
        rest = set(left[:nleft].tolist())
        assert len(rest) == nleft and rest == set(np.nonzero(~done)[0].tolist())
    else:
        assert listed == (~done).sum() and nleft == 0
    if kind == "plain":
        assert done.all()
    if kind == "ties":
        assert listed > 0 and nduel > 0
    held = np.isfinite(xl) & (np.abs(xs).max(1) <= 60000)
    if Cs:
        pos = np.concatenate([np.arange(64 * j * stride, 64 * j * stride + 64) for j in range(Cs // 64)])
        g = key[:, pos].reshape(N, Cs // 16, 16).min(2)
        assert (np.abs(kmin - g)[held] <= err[held, None]).all()
    for i in np.nonzero(held)[0]:
        n = int(ncand[i])
        assert n <= C
        ids = cand[i, :n, 1].astype(int)
        assert len(set(ids.tolist())) == n and (ids < C).all()
        assert set(np.nonzero(key[i] < tau[i] - err[i])[0].tolist()) <= set(ids.tolist())
        assert (key[i, ids] <= tau[i] + err[i]).all()
