"""The single-level list build (at most 256 lists): rows around its 12,288-row
tile, one list, all 256, labels outside the lists, skewed labels, and several
groups of labels at once (the PQ training step). Equal to the oracle's build."""
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
