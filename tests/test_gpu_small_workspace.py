"""Calls in the smallest workspace that they accept (no f16 plane, no lists of
undecided rows): the oracle's results, and nothing written past the workspace."""
import numpy as np
import pytest

from test_gpu_screen_f16 import data, ivf_ctx, to_dev  # noqa: F401

pytestmark = pytest.mark.gpu


def smallest(call, lib, h, need):
    """The least workspace that call() does not refuse, on a validation-only context."""
    import ctypes

    from paper_2608_08751_amd import _binding as B

    lo, hi = 0, need  # refused, accepted
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lib.ivf_set_workspace(h, ctypes.c_void_p(1 << 45), mid)
        lo, hi = (lo, mid) if call(h) != B.IVF_ENOMEM else (mid, hi)
    return hi


@pytest.mark.parametrize("op,u8,N,C,D,slice_rows", [
    ("route", False, 2000, 20011, 128, 0), ("assign", False, 3000, 1001, 96, 0), ("assign", True, 5000, 1001, 96, 0),
    ("assign", True, 2500, 700, 200, 0), ("assign", True, 5000, 1001, 96, 700), ("assign", False, 3000, 1001, 96, 700),
])
def test_smallest_workspace(ivf_ctx, oracle_mod, op, u8, N, C, D, slice_rows):  # noqa: F811
    import torch

    import paper_2608_08751_amd as ivf
    from paper_2608_08751_amd import _binding as B

    x, c = data("plain" if op == "route" else "ties", N, C, D, seed=N + C)
    if u8:
        x = np.clip(np.rint(x * 200 + 128), 0, 255).astype(np.uint8)
        c = np.clip(c * 200 + 128, 0, 255).astype(np.float32)
    xd, cd = to_dev(x), to_dev(c)
    lib, k = ivf_ctx.lib, 16
    dev = lambda n, dt: torch.empty(n, dtype=dt, device="cuda")
    if op == "route":
        outs = [dev((N, k), torch.int32), dev((N, k), torch.float32)]
        need = lib.ivf_workspace_bytes(B.IVF_OP_ROUTE, N, C, D, k)
        call = lambda h: lib.ivf_route(h, B._ptr(xd), N, B._ptr(cd), C, D, k, *map(B._ptr, outs))
    else:
        outs = [dev(N, torch.int32), dev(C, torch.int64), dev(C + 1, torch.int64), dev(N, torch.int32)]
        need = lib.ivf_workspace_bytes(B.IVF_OP_ASSIGN_BUILD, N, C, D, 0)
        call = lambda h: lib.ivf_assign_build(h, B._ptr(xd), B.IVF_U8 if u8 else B.IVF_F32, N, B._ptr(cd), C, D,
                                              *map(B._ptr, outs))
    vctx = B.Context(-1)
    least = smallest(call, lib, vctx.handle, need)
    print(op, u8, N, C, D, "least", least, "of", need, flush=True)
    assert least < need
    ctx = ivf.Context(0)
    ws = torch.full((least + 65536,), 0x5A, dtype=torch.uint8, device="cuda")
    ctx.bind_stream()
    ctx.set_option(ivf.IVF_OPT_ASSIGN_SLICE, slice_rows)
    assert lib.ivf_set_workspace(ctx.handle, B._ptr(ws), least) == B.IVF_OK
    assert call(ctx.handle) == B.IVF_OK
    torch.cuda.synchronize()
    print(ctx.last_stats(), flush=True)
    assert (ws[least:] == 0x5A).all()
    if op == "route":
        pick = np.r_[0:50, N - 50:N]
        oids, odist = oracle_mod.route(x[pick], c, k)
        assert (outs[0].cpu().numpy()[pick] == oids).all() and (outs[1].cpu().numpy()[pick] == odist).all()
    else:
        lab = outs[0].cpu().numpy()
        assert (lab == oracle_mod.assign(x, c)).all()
        cnt, off, perm = oracle_mod.build_lists(lab, C)
        assert (outs[1].cpu().numpy() == cnt).all() and (outs[2].cpu().numpy() == off).all()
        assert (outs[3].cpu().numpy().view(np.uint32) == perm).all()
