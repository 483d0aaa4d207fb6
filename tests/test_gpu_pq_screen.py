"""The matrix-core screen of the PQ assignment where it can go wrong: groups of
subspaces that fill LDS or leave a short last group, every padded width, row
counts around the 64-row tile, and sub-vectors it must hand to the exact
evaluation (ties, equal codewords, rows beyond f16's range, tiny values, data
far from the origin), a few of a tile or so many that the tile waits for the
dense evaluation: one codeword far from the others, subspaces of a single
point, tiles of equal codewords among ordinary ones, values whose squares
vanish or overflow, and more tiles per wave than wait at a time. Codes equal
the oracle's."""
import numpy as np
import pytest

from test_gpu_pq import ivf_ctx, to_dev  # noqa: F401

pytestmark = pytest.mark.gpu


def data(kind, n, D, M, seed):
    r = np.random.default_rng(seed)
    x = r.normal(size=(n, D)).astype(np.float32)
    cb = (0.8 * r.normal(size=(M, 256, D // M))).astype(np.float32)
    if kind == "equal":  # every codeword four times, every row on one of them
        cb = np.repeat(cb[:, ::4], 4, axis=1)
        x = cb[np.arange(M)[None, :], r.integers(0, 256, (n, M))].reshape(n, D).copy()
    elif kind == "range":
        x[::5] *= np.float32(1e5)
        x[1::7] *= np.float32(1e-6)
    elif kind == "tiny":
        x, cb = x * np.float32(1e-15), cb * np.float32(1e-15)
    elif kind == "huge":
        x, cb = x * np.float32(1e15), cb * np.float32(1e15)
    elif kind == "offset":
        x, cb = x + np.float32(500.0), cb + np.float32(500.0)
    elif kind.startswith("far"):  # one codeword at so many times the others' radius
        cb[:, 77] *= np.float32(kind[3:])
    elif kind == "blocks":  # tiles of rows on one codeword each, and on three equal ones
        side = np.where(np.repeat(r.random((n + 63) // 64) < 0.5, 64)[:n], 30.0, -30.0).astype(np.float32)
        x += side[:, None]
        cb[:, :64] += np.float32(30.0)
        cb[:, 64:] = np.tile(cb[:, 64:128] - np.float32(30.0), (1, 3, 1))
    elif kind == "vanish":
        x, cb = x * np.float32(1e-24), cb * np.float32(1e-24)
    elif kind == "vast":  # squared norms below FLT_MAX, squared differences above it
        x, cb = np.clip(x, -1.4, 1.4) * np.float32(1e19), np.clip(cb, -1.4, 1.4) * np.float32(1e19)
    elif kind == "one":  # a single point: every codeword the same
        cb[:] = cb[:, :1]
    return np.ascontiguousarray(x), np.ascontiguousarray(cb)


@pytest.mark.parametrize("kind,n,D,M", [
    ("plain", 1, 4, 1), ("plain", 63, 128, 16), ("plain", 64, 128, 32), ("plain", 65, 256, 16), ("plain", 3000, 160, 20),
    ("plain", 2000, 256, 256), ("plain", 1500, 144, 9), ("plain", 700, 60, 5), ("plain", 900, 252, 84),
    ("plain", 20000, 128, 16), ("plain", 600, 12, 4), ("plain", 600, 136, 34),
    ("equal", 500, 128, 16), ("range", 999, 128, 16), ("range", 500, 64, 16), ("range", 500, 64, 4),
    ("far10", 3000, 128, 16), ("far30", 3000, 128, 16), ("far100", 3000, 128, 16), ("far100", 2000, 100, 20),
    ("far100", 2000, 128, 8), ("far30", 2000, 128, 32), ("far100", 700, 144, 12),
    ("blocks", 300_000, 8, 2), ("blocks", 300_000, 8, 4), ("blocks", 5000, 128, 8), ("blocks", 5000, 96, 32),
    ("vanish", 300, 64, 8), ("vast", 300, 4, 4), ("vast", 300, 8, 8),
    ("tiny", 500, 128, 16), ("huge", 500, 96, 6), ("offset", 1000, 128, 16), ("one", 130, 32, 4),
])
def test_codes_equal_the_oracle(ivf_ctx, oracle_mod, kind, n, D, M):  # noqa: F811
    import torch

    import paper_2608_08751_amd as ivf

    x, cb = data(kind, n, D, M, n + D + M)
    codes = ivf.ivf_pq_encode(ivf_ctx, to_dev(x), to_dev(cb))
    torch.cuda.synchronize()
    want = oracle_mod.pq_encode(x, cb)
    bad = np.argwhere(codes.cpu().numpy() != want)
    assert bad.size == 0, "%s %s: %d codes differ, first at %s" % (kind, (n, D, M), len(bad), bad[0])


@pytest.mark.parametrize("kind,D,M", [("blocks", 4, 1), ("far100", 4, 1), ("blocks", 4, 4)])
def test_more_tiles_than_wait_at_a_time(ivf_ctx, oracle_mod, kind, D, M):  # noqa: F811
    """About 38 tiles per wave; the labels of 20,000 rows compared, the last tile among them."""
    import torch

    import paper_2608_08751_amd as ivf

    n = 5_000_017
    x, cb = data(kind, n, D, M, 7)
    codes = ivf.ivf_pq_encode(ivf_ctx, to_dev(x), to_dev(cb))
    torch.cuda.synchronize()
    pick = np.r_[0:200, np.random.default_rng(1).integers(0, n, 19_600), n - 200:n]
    want = oracle_mod.pq_encode(x[pick], cb)
    bad = np.argwhere(codes.cpu().numpy()[pick] != want)
    assert bad.size == 0, "%d codes differ, first at row %d" % (len(bad), pick[bad[0][0]])
