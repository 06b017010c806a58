"""Launch graphs: one for all batches of the same kernels, whatever their length bounds (which set the LDS and the block
size of the seeded kernels), and no more than a fixed number of them."""
import ctypes

import numpy as np
import pytest

import gpu_util as U
from test_gpu_seed import seeded_batch

pytestmark = pytest.mark.gpu


def graphs(ctx):
    from paper_1402_4876_amd import _lib
    built, held = ctypes.c_int64(), ctypes.c_int64()
    _lib.load().mica_ctx_graphs(ctx.handle, ctypes.byref(built), ctypes.byref(held))
    return built.value, held.value


@pytest.mark.parametrize("mode", [0, 1])
def test_one_graph_for_all_length_bounds(mode):
    import paper_1402_4876_amd as mica
    b = seeded_batch(2000, mode, 140, 160, 41)
    o = U.run_oracle(b)
    n = int(b.win_len.max())
    ctx = mica.Context(0)
    try:
        # LDS of the scan from one block size's to the next one's and back
        for win in (n, n + 200, 1500, 3000, n + 64, 8000, n):
            U.assert_same(U.run_gpu(ctx, b, max_win_len=win, min_read_len=140), o, what="windows of up to %d" % win)
        assert graphs(ctx) == (1, 1)
    finally:
        ctx.close()


def test_number_of_graphs_is_bounded():
    """Plain launches of every range of length classes: more sequences than are kept."""
    import paper_1402_4876_amd as mica
    b = seeded_batch(64, 0, 1, 250, 42)
    o = U.run_oracle(b)
    sizes = [(lo, hi) for lo in range(1, 250, 16) for hi in range(lo + 15, 272, 16)]
    ctx = mica.Context(0)
    try:
        for rep in range(2):
            for lo, hi in sizes[rep * 60:] if rep else sizes:
                pick = np.nonzero((b.read_len >= lo) & (b.read_len <= hi))[0]
                if len(pick) == 0:
                    continue
                g = U.run_gpu(ctx, b.subset(pick), plain=True, min_read_len=lo, max_read_len=hi,
                              max_win_len=int(b.win_len.max()))
                U.assert_same(g, {k: v[pick] for k, v in o.items()}, what="reads %d-%d" % (lo, hi))
        built, held = graphs(ctx)
        assert built > 64 and held == 64
    finally:
        ctx.close()
