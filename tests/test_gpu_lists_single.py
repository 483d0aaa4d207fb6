"""The single-level list build (at most 256 lists): rows around its 12,288-row
tile, one list, all 256, skewed labels, and labels outside the lists, which are
left out. Equal to the oracle's build. (Several groups of labels at once are the
PQ training step's, which its own tests compare.)"""
import numpy as np
import pytest

import synth
from test_gpu_pq import ivf_ctx, to_dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,C,skew", [(1, 1, 0.0), (12287, 256, 0.0), (12288, 256, 0.0), (12289, 255, 0.5),
                                      (100000, 1, 0.0), (300001, 256, 1.5), (3_200_000, 200, 0.0), (70000, 257, 0.0)])
def test_build_equals_the_oracle(ivf_ctx, oracle_mod, N, C, skew):  # noqa: F811
    import torch

    import paper_2608_08751_amd as ivf

    lab = synth.random_labels(N, C, seed=N, skew=skew)
    cnt, off, perm = ivf.ivf_build_lists(ivf_ctx, to_dev(lab), C)
    torch.cuda.synchronize()
    ocnt, ooff, operm = oracle_mod.build_lists(lab, C)
    assert (cnt.cpu().numpy() == ocnt).all() and (off.cpu().numpy() == ooff).all()
    assert (perm.cpu().numpy().view(np.uint32) == operm).all()


@pytest.mark.parametrize("C", [1, 200, 256])
@pytest.mark.parametrize("kind", ["mixed", "tile", "all"])
def test_labels_outside_the_lists_are_left_out(ivf_ctx, oracle_mod, kind, C):  # noqa: F811
    """-1, C, 256 and the largest and smallest int32 among valid labels, a whole
    tile of them, nothing else: the lists of the other rows, and offsets to match."""
    import torch

    import paper_2608_08751_amd as ivf

    N = 3 * 12288 + 77
    r = np.random.default_rng(C)
    lab = r.integers(0, C, N).astype(np.int32)
    bad = np.array([-1, C, 256, 2**31 - 1, -2**31], np.int64).astype(np.int32)
    where = {"mixed": r.random(N) < 0.3, "tile": (np.arange(N) >= 12288) & (np.arange(N) < 2 * 12288),
             "all": np.ones(N, bool)}[kind]
    lab[where] = bad[r.integers(0, 5, int(where.sum()))]
    cnt, off, perm = ivf.ivf_build_lists(ivf_ctx, to_dev(lab), C)
    torch.cuda.synchronize()
    keep = np.nonzero((lab >= 0) & (lab < C))[0]
    ocnt, ooff, operm = oracle_mod.build_lists(lab[keep], C) if keep.size else (np.zeros(C), np.zeros(C + 1), keep)
    assert (cnt.cpu().numpy() == ocnt).all() and (off.cpu().numpy() == ooff).all()
    assert (perm.cpu().numpy().view(np.uint32)[:keep.size] == keep[operm.astype(np.int64)]).all()
