"""Batches that are sampled before the seeded bands: modes that the sample leaves and modes that it does not, in one
batch and alone, with and without a traceback, and around the smallest sampled size.  Whatever the sample says, the
results are the full table's: compared with the oracle, element by element."""
import numpy as np
import pytest

import gpu_util as U
import synth
from test_gpu_seed import add_noise, seeded_batch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch

    import paper_1402_4876_amd as mica
    torch.cuda.set_device(0)
    c = mica.Context(0)
    yield c
    c.close()


def batch(modes, noisy, n):
    """n pairs each of some modes, reads of 60 to 110, those of the noisy modes with 15% errors."""
    parts = []
    for md in modes:
        p = seeded_batch(n, md, 60, 110, 31)
        if md in noisy:
            add_noise(p, 0.15)
        parts.append(p)
    ref = parts[0].ref
    size = np.cumsum([0] + [len(p.reads) for p in parts])
    b = synth.Batch(ref=np.concatenate([p.ref for p in parts]),
                    win_off=np.concatenate([p.win_off + i * len(ref) for i, p in enumerate(parts)]),
                    win_len=np.concatenate([p.win_len for p in parts]),
                    reads=np.concatenate([p.reads for p in parts]),
                    read_off=np.concatenate([p.read_off + s for p, s in zip(parts, size)]),
                    read_len=np.concatenate([p.read_len for p in parts]),
                    mode=np.concatenate([p.mode for p in parts]), name="sampled")
    if 2 in modes:
        b.h0 = np.concatenate([p.h0 if p.h0 is not None else np.zeros(p.n_pairs, np.int32) for p in parts])
    return b


@pytest.mark.parametrize("trace", [True, False])
@pytest.mark.parametrize("modes,noisy", [((0,), ()), ((0,), (0,)), ((1,), (1,)), ((0, 1), (0,)), ((0, 1), (1,)),
                                         ((0, 1, 2), (0, 1)), ((0, 1, 2), ())])
def test_sampled_modes(ctx, modes, noisy, trace):
    b = batch(modes, noisy, 1200)
    reps = -(-(33_000 if trace else 250_000) // b.n_pairs)
    kw = dict(clip=5 if 2 in modes else 0, trace=trace)
    o = {k: np.concatenate([v] * reps) for k, v in U.run_oracle(b, **kw).items()}
    big = b.subset(np.tile(np.arange(b.n_pairs), reps))
    g = U.run_gpu(ctx, big, max_ext_h0=80 if 2 in modes else 0, **kw)
    U.assert_same(g, o, trace=trace, what="modes %s, noisy %s" % (modes, noisy))


@pytest.mark.parametrize("int32", [False, True])
@pytest.mark.parametrize("n_pairs", [32_767, 32_768, 32_769])
def test_smallest_sampled_sizes(ctx, n_pairs, int32):
    b = batch((0, 1), (1,), 1000)
    pick = np.arange(n_pairs) % b.n_pairs
    o = {k: v[pick] for k, v in U.run_oracle(b).items()}
    U.assert_same(U.run_gpu(ctx, b.subset(pick), force_int32=int32), o, what="%d pairs" % n_pairs)
