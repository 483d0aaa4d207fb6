"""Rows inside the single plane's window: two candidates (decided by the
resolving kernel, or by the screen when its list is full), three to eight
(collected by a second pass over the plane), more than eight (the fp64 scan
for few such rows, the two-plane screen for many), and a list that overflows
(the two-plane screen takes every row). Labels equal the oracle's in all of
them."""
import numpy as np
import pytest

import synth
from test_gpu_screen_i8 import gpu_assign, ivf_ctx  # noqa: F401

pytestmark = pytest.mark.gpu


def crowded(N, C, D, sizes, seed):
    """C centroids in groups of the given sizes, a quarter apart from each
    other, and rows around the groups' middles."""
    rng = np.random.default_rng(seed)
    groups, left = [], C
    while left > 0:
        groups.append(min(left, sizes[len(groups) % len(sizes)]))
        left -= groups[-1]
    mid = rng.integers(20, 236, size=(len(groups), D)).astype(np.float32)
    c = np.concatenate([m + rng.uniform(-0.5, 0.5, size=(n, D)) for m, n in zip(mid, groups)]).astype(np.float32)
    x, a = synth.mixture_rows_u8(mid, 0, N, seed=seed)
    return x, np.ascontiguousarray(c), np.asarray(groups)[a]


@pytest.mark.parametrize("N,C,D,sizes", [
    (767, 300, 128, [1, 2]),              # one ragged tile, duels
    (9000, 1025, 100, [2]),               # every row a duel: more than the list of duels holds
    (3000, 513, 36, [1, 1, 3, 4, 8]),     # collected, a ragged last chunk
    (5000, 700, 64, [1] * 20 + [9]),      # some rows with too many candidates
    (20000, 2000, 128, [1, 1, 1, 1, 1, 24]),  # many such rows: two planes
    (40000, 900, 96, [5]),                # every row listed: the list overflows
    (1, 9, 4, [9]),
])
def test_near_ties_equal_the_oracle(ivf_ctx, oracle_mod, N, C, D, sizes):  # noqa: F811
    x, c, crowd = crowded(N, C, D, sizes, seed=N + C)
    olab = oracle_mod.assign(x, c)
    lab, cnt, off, perm, st = gpu_assign(ivf_ctx, x, c)
    print(N, C, D, sizes, st, flush=True)
    bad = np.nonzero(lab != olab)[0]
    assert bad.size == 0, "labels differ at rows %s" % bad[:10]
    ocnt, ooff, operm = oracle_mod.build_lists(olab, C)
    assert (cnt == ocnt).all() and (off == ooff).all() and (perm == operm).all()
    assert st["screen_i8"] == 1
    if (crowd >= 2).any():
        assert st["refine2"] + st["rescreen"] > 0


def test_single_plane_lists_of_several_slices(ivf_ctx, oracle_mod):  # noqa: F811
    x, c, _ = crowded(6000, 640, 128, [1, 2, 3, 12], seed=5)
    olab = oracle_mod.assign(x, c)
    lab, _, _, _, _ = gpu_assign(ivf_ctx, x, c, IVF_OPT_ASSIGN_SLICE=1111)
    assert (lab == olab).all()
