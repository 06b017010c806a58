"""Contexts whose workspace cap is below what one block of waves needs: the batch runs in one block, and every pair
gets its result.  Compared with the oracle, element by element."""
import pytest

import gpu_util as U
from test_gpu_seed import seeded_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("workspace", [256, 65536, 400_000])
@pytest.mark.parametrize("mode,m_lo,m_hi", [(0, 150, 150), (1, 101, 160), (2, 30, 150), (0, 230, 420), (1, 24, 60)])
def test_small_workspace(mode, m_lo, m_hi, workspace):
    import paper_1402_4876_amd as mica
    b = seeded_batch(300, mode, m_lo, m_hi, 21)
    clip = 7 if mode == 2 else 0
    o = U.run_oracle(b, clip=clip)
    ctx = mica.Context(0, workspace_bytes=workspace)
    try:
        for trace in (True, False):
            g = U.run_gpu(ctx, b, trace=trace, clip=clip, max_ext_h0=80 if mode == 2 else 0)
            U.assert_same(g, o, trace=trace, what="workspace %d, mode %d, trace %s" % (workspace, mode, trace))
    finally:
        ctx.close()


def test_long_reads_in_a_small_workspace():
    """Reads of up to the length limit, whose band slots are the largest."""
    import paper_1402_4876_amd as mica
    b = seeded_batch(40, 0, 900, 1024, 22)
    o = U.run_oracle(b, cap=256)
    ctx = mica.Context(0, workspace_bytes=4096)
    try:
        U.assert_same(U.run_gpu(ctx, b, cap=256), o, cap=256, what="long reads")
    finally:
        ctx.close()
