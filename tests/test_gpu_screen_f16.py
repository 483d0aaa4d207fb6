"""The f16 screen of fp32 rows and queries (and the small calls beside it that
stay on fp32): labels, ids and distances equal the
oracle's on ordinary data, among near ties (two candidates, a few, more than
the collecting pass keeps), and where f16 cannot decide: data far from the
origin (its window covers every centroid), values beyond its range or below
its smallest normal number, and a zero table. IVF_OPT_FP32_SCREEN gives the
same."""
import numpy as np
import pytest

from test_gpu_screen_i8 import ivf_ctx, to_dev  # noqa: F401

pytestmark = pytest.mark.gpu


def data(kind, N, C, D, seed):
    r = np.random.default_rng(seed)
    c = r.normal(size=(C, D)).astype(np.float32)
    c /= np.linalg.norm(c, axis=1, keepdims=True)
    x = (c[r.integers(0, C, N)] + 0.3 / np.sqrt(D) * r.normal(size=(N, D))).astype(np.float32)
    if kind == "ties":  # groups of 1, 2, 3, 8 and 12 almost equal centroids
        size = np.resize([1, 2, 3, 8, 12], C)
        head = np.repeat(np.arange(C), size)[:C]
        c = (c[head] * (1.0 + 1e-6 * r.normal(size=(C, D)))).astype(np.float32)
    elif kind == "offset":
        c, x = c * np.float32(0.01) + np.float32(50.0), x * np.float32(0.01) + np.float32(50.0)
    elif kind == "range":  # some rows 1e4 times longer than any centroid, some 1e-6 times as long
        x[::7] *= np.float32(1e4)
        x[3::11] *= np.float32(1e-6)
    elif kind == "tiny":
        c, x = c * np.float32(1e-17), x * np.float32(1e-17)
    elif kind == "huge":
        c, x = c * np.float32(1e17), x * np.float32(1e17)
    elif kind == "zero":
        c[:] = 0
    return np.ascontiguousarray(x), np.ascontiguousarray(c)


@pytest.mark.parametrize("kind,N,C,D", [
    ("plain", 513, 257, 96), ("plain", 1, 1, 4), ("plain", 3000, 1000, 128), ("plain", 700, 65, 36),
    ("plain", 900, 130, 256), ("plain", 600, 300, 160), ("plain", 520, 700, 64),
    ("ties", 4000, 900, 100), ("ties", 2500, 600, 200), ("offset", 2000, 500, 96), ("range", 1500, 400, 128),
    ("tiny", 800, 200, 96), ("huge", 800, 200, 96), ("zero", 100, 70, 32),
    # small tables, which take f16 from 0.8 GFLOP on; the smallest calls above stay on fp32
    ("plain", 200_000, 65, 36), ("plain", 45_000, 257, 96), ("plain", 1_100_000, 3, 128), ("ties", 120_000, 33, 128),
    ("zero", 100_000, 70, 64), ("range", 60_000, 130, 64), ("tiny", 3000, 400, 96), ("huge", 3000, 400, 96),
])
def test_assign_equals_the_oracle(ivf_ctx, oracle_mod, kind, N, C, D):  # noqa: F811
    import torch

    import paper_2608_08751_amd as ivf

    x, c = data(kind, N, C, D, seed=N + D)
    olab = oracle_mod.assign(x, c)
    for fp32 in (0, 1):
        ivf_ctx.set_option(ivf.IVF_OPT_FP32_SCREEN, fp32)
        try:
            lab = ivf.ivf_assign_build(ivf_ctx, to_dev(x), to_dev(c))[0]
            torch.cuda.synchronize()
            print(kind, N, C, D, "fp32" if fp32 else "f16", ivf_ctx.last_stats(), flush=True)
        finally:
            ivf_ctx.set_option(ivf.IVF_OPT_FP32_SCREEN, 0)
        bad = np.nonzero(lab.cpu().numpy() != olab)[0]
        assert bad.size == 0, "labels differ at rows %s" % bad[:10]


def test_assign_stops_when_the_list_overflows(ivf_ctx, oracle_mod):  # noqa: F811
    """Rows far from the origin: every one is left undecided, and once a quarter
    of them is listed the f16 pass ends and the fp32 screen takes all of them."""
    import torch

    import paper_2608_08751_amd as ivf

    N, C = 700_000, 600
    x, c = data("plain", N, C, 32, seed=3)
    x, c = x + np.float32(30.0), c + np.float32(30.0)
    lab = ivf.ivf_assign_build(ivf_ctx, to_dev(x), to_dev(c))[0]
    torch.cuda.synchronize()
    st = ivf_ctx.last_stats()
    print(st, flush=True)
    assert N // 4 < st["rescreen"] < N // 2
    pick = np.r_[0:2000, np.random.default_rng(0).integers(0, N, 4000), N - 2000:N]
    assert (lab.cpu().numpy()[pick] == oracle_mod.assign(x[pick], c)).all()


@pytest.mark.parametrize("kind,Q,C,D,k", [
    ("plain", 513, 4096, 96, 16), ("plain", 1, 3000, 128, 5), ("plain", 40, 9001, 4, 128), ("plain", 300, 2049, 256, 64),
    ("plain", 65, 5000, 100, 1000), ("plain", 200, 2113, 160, 1), ("ties", 500, 4100, 64, 40),
    ("offset", 64, 3000, 96, 32), ("range", 100, 3000, 128, 16), ("tiny", 50, 2500, 96, 8), ("huge", 50, 2500, 96, 8),
])
def test_route_equals_the_oracle(ivf_ctx, oracle_mod, kind, Q, C, D, k):  # noqa: F811
    import torch

    import paper_2608_08751_amd as ivf

    q, c = data(kind, Q, C, D, seed=Q + D)
    if kind != "huge" and D >= 64:
        q[0] = c[C // 3]  # a planted query
    oids, odist = oracle_mod.route(q, c, k)
    ids, dist = ivf.ivf_route(ivf_ctx, to_dev(q), to_dev(c), k)
    torch.cuda.synchronize()
    print(kind, Q, C, D, k, ivf_ctx.last_stats(), flush=True)
    assert (ids.cpu().numpy() == oids).all() and (dist.cpu().numpy() == odist).all()


@pytest.mark.parametrize("kind,Q,C,D,k", [
    ("plain", 20000, 70000, 4, 128), ("plain", 2000, 20011, 128, 64), ("plain", 6000, 4097, 256, 5),
    ("ties", 9000, 9001, 64, 40), ("offset", 3000, 20000, 96, 32), ("range", 2500, 20000, 128, 16),
    ("tiny", 4000, 15000, 96, 8), ("huge", 4000, 15000, 96, 8), ("plain", 20000, 8300, 32, 8),
])
def test_large_route_equals_the_oracle(ivf_ctx, oracle_mod, kind, Q, C, D, k):  # noqa: F811
    """Calls of at least 10 GFLOP, which take the f16 plane; 120 queries compared."""
    import torch

    import paper_2608_08751_amd as ivf

    assert 2 * Q * C * D >= 1e10
    q, c = data(kind, Q, C, D, seed=Q + D)
    ids, dist = ivf.ivf_route(ivf_ctx, to_dev(q), to_dev(c), k)
    torch.cuda.synchronize()
    st = ivf_ctx.last_stats()
    print(kind, Q, C, D, k, st, flush=True)
    assert st["screen_f16"] == (0 if kind in ("offset", "range") else (Q + 16383) // 16384)
    pick = np.r_[0:60, Q - 60:Q]
    oids, odist = oracle_mod.route(q[pick], c, k)
    assert (ids.cpu().numpy()[pick] == oids).all() and (dist.cpu().numpy()[pick] == odist).all()


@pytest.mark.parametrize("rank", [1, 60, 65, 100, 400])
def test_threshold_ranks_on_the_f16_plane(ivf_ctx, oracle_mod, rank):  # noqa: F811
    """Ranks below and above the 64 minima the threshold keeps: the same
    candidates at every run, more of them at a higher rank, the same results."""
    import torch

    import paper_2608_08751_amd as ivf

    q, c = data("plain", 2000, 20011, 128, seed=31)
    qd, cd = to_dev(q), to_dev(c)
    ivf_ctx.set_option(ivf.IVF_OPT_SAMPLE_RANK, rank)
    try:
        runs = []
        for _ in range(2):
            ids, dist = ivf.ivf_route(ivf_ctx, qd, cd, 16)
            torch.cuda.synchronize()
            runs.append(ivf_ctx.last_stats())
            print(rank, runs[-1], flush=True)
    finally:
        ivf_ctx.set_option(ivf.IVF_OPT_SAMPLE_RANK, 0)
    assert runs[0] == runs[1]
    if rank > 1:  # a sample of 2,496 in 156 groups: eight centroids per sample key
        assert runs[0]["candidates"] > 2000 * min(rank, 156) * 6
    pick = np.r_[0:40, 1960:2000]
    oids, odist = oracle_mod.route(q[pick], c, 16)
    assert (ids.cpu().numpy()[pick] == oids).all() and (dist.cpu().numpy()[pick] == odist).all()


@pytest.mark.parametrize("odd,batches", [(None, 2), (5, 1), (16384 + 5, 1), ("both", 0)])
def test_route_batches_and_odd_queries(ivf_ctx, oracle_mod, odd, batches):  # noqa: F811
    """Two internal batches: where a query of one has no f16 bound, that batch
    alone goes to the fp32 kernels."""
    import torch

    import paper_2608_08751_amd as ivf

    Q, C, D = 16384 + 700, 9300, 32
    assert 2 * Q * C * D >= 1e10  # a call the f16 plane takes
    q, c = data("plain", Q, C, D, seed=9)
    for i in () if odd is None else (5, 16384 + 5) if odd == "both" else (odd,):
        q[i] *= np.float32(1e6)
    ids, dist = ivf.ivf_route(ivf_ctx, to_dev(q), to_dev(c), 8)
    torch.cuda.synchronize()
    st = ivf_ctx.last_stats()
    assert st["screen_f16"] == batches and st["screen_i8"] == 0
    pick = np.r_[0:64, 16384 - 8:16384 + 64, 16384 + 636:16384 + 700]
    oids, odist = oracle_mod.route(q[pick], c, 8)
    assert (ids.cpu().numpy()[pick] == oids).all() and (dist.cpu().numpy()[pick] == odist).all()


@pytest.mark.parametrize("kind", ["int8", "centroid", "query"])
def test_integer_queries_and_what_does_not_quantise(ivf_ctx, oracle_mod, kind):  # noqa: F811
    """uint8-valued queries in two batches: the int8 planes take them; one centroid
    outside their range sends both batches to the fp32 kernels (no f16 plane
    was built), one other query value both to the f16 plane."""
    import torch

    import paper_2608_08751_amd as ivf

    Q, C, D = 16384 + 700, 9300, 32
    r = np.random.default_rng(4)
    c = (255 * r.random((C, D))).astype(np.float32)
    q = r.integers(0, 256, (Q, D)).astype(np.float32)
    if kind == "centroid":
        c[77, 3] = 300.0
    elif kind == "query":
        q[16384 + 9, 1] = 17.5
    ids, dist = ivf.ivf_route(ivf_ctx, to_dev(q), to_dev(c), 8)
    torch.cuda.synchronize()
    st = ivf_ctx.last_stats()
    assert (st["screen_i8"], st["screen_f16"]) == {"int8": (1, 0), "centroid": (0, 0), "query": (0, 2)}[kind]
    pick = np.r_[0:64, 16384 - 8:16384 + 64, 16384 + 636:16384 + 700]
    oids, odist = oracle_mod.route(q[pick], c, 8)
    assert (ids.cpu().numpy()[pick] == oids).all() and (dist.cpu().numpy()[pick] == odist).all()
