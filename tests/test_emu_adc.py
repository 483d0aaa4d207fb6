"""The ADC scan's kernels (adc.hip) built for the host against the wave64
emulation (tests/wave_emu) and run under AddressSanitizer: results equal to the
oracle's bit for bit for every way a width is taken (codebooks in registers,
from memory in 1 to 8 dims, up to 16 and in blocks), one part per query, several,
and extra parts for a query far heavier than the others; no access leaves its
allocation. No GPU is involved."""
import os
import subprocess

import numpy as np
import pytest

import synth
from test_emu_screen_i8 import CLANG, CSRC, HERE


@pytest.fixture(scope="module")
def emu_adc(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("clang++ of the ROCm toolchain not found")
    d = tmp_path_factory.mktemp("wave_emu_adc")
    with open(os.path.join(CSRC, "adc.hip")) as f:
        src = f.read()
    with open(d / "adc_host_src.hip", "w") as f:
        f.write(src)
    exe = str(d / "adc_host")
    cmd = [CLANG, "-std=c++20", "-O1", "-g", "-fsanitize=address", "-fno-omit-frame-pointer", "-ffp-contract=off",
           "-I", os.path.join(HERE, "wave_emu"), "-I", str(d), "-I", CSRC,
           os.path.join(HERE, "wave_emu", "adc_host.cpp"), "-o", exe, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


def run(exe, tmp_path, q, c, probes, off, perm, codes, cb, k, num_cus):
    B, D = q.shape
    src, dst = tmp_path / "in.bin", tmp_path / "out.bin"
    with open(src, "wb") as f:
        f.write(np.array([B, D, c.shape[0], probes.shape[1], perm.size, codes.shape[1], k], np.int64).tobytes())
        for a in (q, c, probes, off, perm, codes, cb):
            f.write(np.ascontiguousarray(a).tobytes())
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:halt_on_error=1")
    r = subprocess.run([exe, str(src), str(dst), str(num_cus)], capture_output=True, text=True, timeout=900, env=env)
    assert r.returncode == 0 and "AddressSanitizer" not in r.stderr, r.stderr[-6000:]
    raw = np.fromfile(dst, np.uint32)
    n = B * k
    return raw[:n].reshape(B, k), raw[n:2 * n].view(np.float32).reshape(B, k), raw[2 * n:].astype(int)


def setup(seed, B, C, D, M, N, P, skew):
    rng = np.random.default_rng(seed)
    c = (rng.standard_normal((C, D)) * 2).astype(np.float32)
    q = (rng.standard_normal((B, D)) * 2).astype(np.float32)
    cb = rng.standard_normal((M, 256, D // M)).astype(np.float32)
    lab = synth.random_labels(N, C, seed=seed, skew=skew)
    perm = np.argsort(lab, kind="stable").astype(np.uint32)
    off = np.concatenate([[0], np.cumsum(np.bincount(lab, minlength=C))]).astype(np.int64)
    codes = rng.integers(0, 256, (N, M)).astype(np.uint8)
    probes = np.stack([rng.choice(C, P, replace=False) for _ in range(B)]).astype(np.int32)
    return q, c, probes, off, perm, codes, cb


@pytest.mark.parametrize("D,M", [(32, 4), (64, 16), (96, 24), (32, 2), (8, 8), (12, 6), (36, 12), (20, 4),
                                 (24, 4), (28, 4), (192, 24), (36, 4), (208, 13), (68, 2), (256, 1), (60, 60)])
def test_emulated_widths(emu_adc, oracle_mod, tmp_path, D, M):
    a = setup(D + M, 1, 9, D, M, 700, 5, 0.5)
    a[2][0, 1] = -1  # not a list
    ids, dist, parts = run(emu_adc, tmp_path, *a, 70, 1)
    oids, odist = oracle_mod.adc_scan(*a, 70)
    assert parts[0] == 1
    assert (ids == oids).all() and (dist.view(np.uint32) == odist.view(np.uint32)).all()


@pytest.mark.parametrize("B,C,N,P,k,cus,skew", [(1, 40, 3000, 40, 100, 4, 0.5), (6, 12, 120_000, 4, 30, 2, 3.0),
                                                (5, 10, 150_000, 2, 8, 1, 3.0)])
def test_emulated_parts(emu_adc, oracle_mod, tmp_path, B, C, N, P, k, cus, skew):
    """Several parts per query; a heavy list in some queries only, whose extra
    parts are more than there may be in the last case."""
    a = setup(B + N, B, C, 8, 2, N, P, skew)
    ids, dist, parts = run(emu_adc, tmp_path, *a, k, cus)
    oids, odist = oracle_mod.adc_scan(*a, k)
    assert (ids == oids).all() and (dist.view(np.uint32) == odist.view(np.uint32)).all()
    print(parts)
    if skew < 1:
        assert (parts > 1).all()
    else:
        assert parts.max() > 1 and parts.min() == 1 and (parts - 1).sum() <= 2 * cus
