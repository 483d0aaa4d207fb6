"""Routing by a kept key matrix (tables of up to 2,048 centroids, and the
smallest batches on larger ones) against the oracle, at the edges of its rules
and tiles and beside the general path: query counts around a tile and the
limit, table sizes around a block, a thread's keys and a kernel's range, few
and many neighbours, near and exact ties past the candidate window, values
whose keys overflow or vanish, forced scans, and two internal batches."""
import numpy as np
import pytest

from test_gpu_screen_f16 import data, ivf_ctx, to_dev  # noqa: F401

pytestmark = pytest.mark.gpu


def check(ctx, oracle_mod, q, c, k, pick=slice(None)):
    import torch

    import paper_2608_08751_amd as ivf

    print(q.shape, c.shape, k, flush=True)
    ids, dist = ivf.ivf_route(ctx, to_dev(q), to_dev(c), k)
    torch.cuda.synchronize()
    oids, odist = oracle_mod.route(q[pick], c, k)
    assert (ids.cpu().numpy()[pick] == oids).all() and (dist.cpu().numpy()[pick] == odist).all()
    return ctx.last_stats()


@pytest.mark.parametrize("Q,C,D,k", [
    (1, 1, 4, 1), (3, 2, 8, 2), (33, 31, 12, 31), (5, 33, 100, 7), (90, 256, 256, 256), (90, 257, 256, 200), (40, 300, 32, 300), (40, 512, 64, 400), (40, 513, 64, 100), (300, 1024, 128, 16), (64, 1025, 96, 128),
    (31, 1025, 64, 129), (70, 2048, 256, 1024), (32, 2048, 160, 1), (1, 2049, 128, 512), (32, 2049, 64, 513),
    (33, 2049, 64, 64), (16, 4000, 32, 9), (17, 4000, 32, 9), (32, 16384, 100, 64), (8, 16385, 96, 128),
    (4, 65536, 36, 100), (18, 65536, 36, 1), (3, 65537, 36, 100),
])
@pytest.mark.parametrize("integer", [False, True])
def test_direct_sizes(ivf_ctx, oracle_mod, Q, C, D, k, integer):  # noqa: F811
    q, c = data("plain", Q, C, D, seed=Q + C + D)
    if integer:  # many equal distances
        q, c = np.rint(q * 6).astype(np.float32), np.rint(c * 6).astype(np.float32)
    check(ivf_ctx, oracle_mod, q, c, k)


@pytest.mark.parametrize("C", [900, 2000, 5000, 20000])
@pytest.mark.parametrize("kind", ["ties", "offset", "range", "tiny", "huge", "zero"])
def test_direct_values(ivf_ctx, oracle_mod, kind, C):  # noqa: F811
    """The window covers a few centroids, every one, or has no finite bound."""
    q, c = data(kind, 20, C, 96, seed=C)
    st = check(ivf_ctx, oracle_mod, q, c, 40)
    assert st["candidates"] == 20 * C
    if kind == "zero":  # every centroid is a candidate: more than the window keeps, or all of them
        assert (st["fallback"] == 20) == (C > 2048)


@pytest.mark.parametrize("Q,C", [(40, 700), (30, 3000)])
def test_direct_forced_scan(ivf_ctx, oracle_mod, Q, C):  # noqa: F811
    import paper_2608_08751_amd as ivf

    q, c = data("plain", Q, C, 64, seed=1)
    ivf_ctx.set_option(ivf.IVF_OPT_FORCE_FALLBACK, 1)
    try:
        assert check(ivf_ctx, oracle_mod, q, c, 33)["fallback"] == Q
    finally:
        ivf_ctx.set_option(ivf.IVF_OPT_FORCE_FALLBACK, 0)


def test_direct_batches(ivf_ctx, oracle_mod):  # noqa: F811
    q, c = data("plain", 16384 + 70, 600, 16, seed=2)
    st = check(ivf_ctx, oracle_mod, q, c, 5, np.r_[0:64, 16384 - 40:16384 + 70])
    assert st["candidates"] == q.shape[0] * 600


@pytest.mark.parametrize("C", [6000, 20000])
def test_direct_neighbours_in_one_thread(ivf_ctx, oracle_mod, C):  # noqa: F811
    """The nearest centroids all among one thread's keys, the others at one
    distance: the minima let every key through, the selection over the keys
    themselves finds the neighbours, and one neighbour more takes the scan."""
    r = np.random.default_rng(C)
    c = np.full((C, 32), 40, np.float32)
    near = np.concatenate([np.arange(e, min(e + 4, C)) for e in range(0, C, 4096)])
    c[near] = r.integers(-1, 2, (near.size, 32))
    q = np.zeros((16, 32), np.float32)
    assert check(ivf_ctx, oracle_mod, q, c, near.size)["fallback"] == 0
    assert check(ivf_ctx, oracle_mod, q, c, near.size + 1)["fallback"] == 16
