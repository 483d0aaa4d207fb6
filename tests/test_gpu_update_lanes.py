"""Means of narrow rows with a list per group of lanes, against the oracle bit
for bit: every width it takes, both batch lengths (lists of 256 members on
average and just below), lists of none, one and most of the rows, and group
counts that are and are not spread over the compute dies."""
import numpy as np
import pytest

from test_gpu_pq import ivf_ctx, to_dev  # noqa: F401

pytestmark = pytest.mark.gpu


def skewed(n, D, seed):
    r = np.random.default_rng(seed)
    x = (r.standard_normal((n, D)) * 3).astype(np.float32)
    x[r.random(n) < 0.4] = x[0]  # one list holds 40 % of the rows
    return x


@pytest.mark.parametrize("ds", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("n", [1, 300, 65535, 65536])
def test_pq_means(ivf_ctx, oracle_mod, n, ds):  # noqa: F811
    import torch

    import paper_2608_08751_amd as ivf

    D = 48 if ds == 16 else 32
    M = D // ds
    x = skewed(n, D, n + ds)
    r = np.random.default_rng(ds)
    cb = x[r.choice(n, 256, replace=n < 256)].reshape(256, M, ds).transpose(1, 0, 2).copy()
    cb[:, 17] = 1e6  # an empty list
    out, cnt, obj = ivf.ivf_pq_train_step(ivf_ctx, to_dev(x), to_dev(cb), seed=5, it=1)
    torch.cuda.synchronize()
    oout, ocnt, oobj = oracle_mod.pq_train_step(x, cb, seed=5, it=1)
    assert (ocnt[:, 17] == 0).all() and (cnt.cpu().numpy() == ocnt).all()
    assert (out.cpu().numpy().view(np.uint32) == oout.view(np.uint32)).all()
    assert np.all(np.abs(obj.cpu().numpy() - oobj) <= 1e-12 * np.maximum(oobj, 1e-300))


@pytest.mark.parametrize("u8", [False, True])
@pytest.mark.parametrize("N,C,D", [(4000, 1030, 8), (262144, 1024, 8), (65000, 257, 32)])
def test_kmeans_means(ivf_ctx, oracle_mod, N, C, D, u8):  # noqa: F811
    import torch

    import paper_2608_08751_amd as ivf

    x = skewed(N, D, N)
    if u8:
        x = np.clip(np.rint(x * 20 + 128), 0, 255).astype(np.uint8)
    c = x[np.random.default_rng(1).choice(N, C, replace=False)].astype(np.float32)
    lab, cent, cnt, obj = ivf.ivf_kmeans_step(ivf_ctx, to_dev(x), to_dev(c), seed=3, it=2)
    torch.cuda.synchronize()
    olab, ocent, ocnt, oobj = oracle_mod.kmeans_step(x, c, seed=3, it=2)
    assert (lab.cpu().numpy() == olab).all() and (cnt.cpu().numpy() == ocnt).all()
    assert (cent.cpu().numpy().view(np.uint32) == ocent.view(np.uint32)).all()
    assert abs(float(obj[0]) - oobj) <= 1e-12 * oobj
