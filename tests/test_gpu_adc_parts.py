"""The ADC scan's branches: every register layout of the codebooks (subspaces of
4, 8 and 16 dims) and every width read from memory (1 to 8 dims, up to 16, in
blocks of 16, whole and part last blocks), codes of one
to sixty bytes, batches cut into many parts, a few and one, lists of one code
and of many rounds, ties (equal codes, ids decide), and k from 1 to 1,024.
Bit for bit the oracle's."""
import numpy as np
import pytest

from test_gpu_adc import gpu_adc, ivf_ctx, setup  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,C,D,M,N,P,k", [
    (1, 64, 128, 16, 9000, 64, 512), (3, 9, 32, 4, 30000, 9, 1024), (70, 40, 64, 8, 4000, 7, 33),
    (300, 30, 96, 12, 3000, 5, 100), (1100, 20, 128, 16, 2000, 4, 50), (9, 30, 160, 20, 9000, 11, 300),
    (5, 20, 32, 8, 5000, 6, 64), (5, 20, 64, 16, 5000, 6, 64), (5, 20, 96, 24, 5000, 6, 64),
    (5, 20, 128, 32, 5000, 6, 64), (5, 20, 160, 40, 5000, 6, 64), (5, 20, 64, 4, 5000, 6, 64),
    (5, 20, 128, 8, 5000, 6, 64), (4, 20, 240, 60, 4000, 6, 64), (4, 20, 256, 32, 4000, 6, 64),
    (5, 20, 48, 12, 5000, 6, 64), (5, 20, 80, 20, 5000, 6, 64), (5, 20, 112, 28, 5000, 6, 64),
    (5, 20, 144, 36, 5000, 6, 64), (5, 20, 64, 32, 5000, 6, 64), (5, 20, 60, 60, 5000, 6, 64),
    (5, 20, 36, 12, 5000, 6, 64), (5, 20, 100, 20, 5000, 6, 64), (5, 20, 120, 20, 5000, 11, 64),
    (5, 20, 28, 4, 5000, 9, 64), (5, 20, 120, 10, 5000, 9, 64), (5, 20, 36, 4, 5000, 9, 64), (5, 20, 240, 12, 5000, 9, 64),
    (5, 20, 256, 8, 5000, 9, 64), (5, 20, 256, 1, 5000, 20, 64), (5, 20, 68, 2, 5000, 9, 64), (5, 20, 252, 28, 5000, 6, 64),
    (5, 20, 224, 28, 5000, 6, 64), (300, 60, 256, 16, 6000, 20, 31), (300, 60, 208, 13, 6000, 20, 31),
    (300, 60, 192, 24, 6000, 20, 31), (300, 60, 12, 12, 6000, 20, 31),
    (300, 60, 96, 12, 6000, 30, 100), (300, 60, 160, 10, 6000, 20, 31), (2, 60, 160, 10, 6000, 20, 31),
    (300, 60, 64, 4, 6000, 20, 31), (300, 60, 160, 40, 6000, 20, 31), (300, 60, 160, 20, 6000, 20, 31),
    (300, 60, 96, 24, 6000, 20, 31), (300, 60, 64, 8, 6000, 20, 31), (4, 20, 120, 15, 4000, 6, 64), (4, 20, 12, 3, 4000, 6, 1), (4, 300, 64, 8, 300, 256, 1000),
])
def test_branches_equal_the_oracle(ivf_ctx, oracle_mod, B, C, D, M, N, P, k):  # noqa: F811
    q, c, probes, off, perm, codes, cb = setup(B + C + D + M, B, C, D, M, N, P, 0.6)
    ids, dist = gpu_adc(ivf_ctx, q, c, probes, off, perm, codes, cb, k)
    oids, odist = oracle_mod.adc_scan(q, c, probes, off, perm, codes, cb, k)
    assert (ids == oids).all() and (dist.view(np.uint32) == odist.view(np.uint32)).all()


@pytest.mark.parametrize("B,C,D,M,N,P,k", [
    (300, 40, 64, 8, 400_000, 4, 300),   # a few heavy queries of many
    (700, 12, 32, 4, 300_000, 6, 1024),  # more extra parts wanted than there are: scaled down
    (1500, 30, 32, 4, 300_000, 2, 10),   # two probes, more queries than a round of the extra kernel takes
    (20, 200, 32, 8, 2_000_000, 40, 64),  # several parts each, more for some
    (260, 300, 32, 4, 200_000, 2, 1),
])
def test_skewed_lists_get_more_parts(ivf_ctx, oracle_mod, B, C, D, M, N, P, k):
    """Lists of very different lengths, so that some queries are cut into more
    parts than the others; the heaviest and the lightest queries are compared."""
    q, c, probes, off, perm, codes, cb = setup(B + N, B, C, D, M, N, P, 2.0)
    ids, dist = gpu_adc(ivf_ctx, q, c, probes, off, perm, codes, cb, k)
    n = (off[probes + 1] - off[probes]).sum(1)
    assert n.max() > 2 * 12 * 2048 and n.max() > 8 * n.min()  # (a part's least work: 12 lists, 2,048 codes each)
    order = np.argsort(n, kind="stable")
    pick = np.r_[order[:4], order[B // 2:B // 2 + 3], order[-5:]]
    oids, odist = oracle_mod.adc_scan(q[pick], c, probes[pick], off, perm, codes, cb, k)
    assert (ids[pick] == oids).all() and (dist[pick].view(np.uint32) == odist.view(np.uint32)).all()
    # a query's result does not depend on the others: alone it takes other parts
    one = order[-1:]
    ids1, dist1 = gpu_adc(ivf_ctx, q[one], c, probes[one], off, perm, codes, cb, k)
    assert (ids1 == ids[one]).all() and (dist1.view(np.uint32) == dist[one].view(np.uint32)).all()


@pytest.mark.parametrize("B", [2, 1100])
def test_equal_codes_rank_by_id(ivf_ctx, oracle_mod, B):  # noqa: F811
    q, c, probes, off, perm, codes, cb = setup(3, B, 6, 64, 8, 20000, 3)
    codes[:] = codes[:1]
    ids, dist = gpu_adc(ivf_ctx, q, c, probes, off, perm, codes, cb, 700)
    n = min(B, 4)
    oids, odist = oracle_mod.adc_scan(q[:n], c, probes[:n], off, perm, codes, cb, 700)
    assert (ids[:n] == oids).all() and (dist[:n].view(np.uint32) == odist.view(np.uint32)).all()
