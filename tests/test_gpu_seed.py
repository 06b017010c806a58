"""Seeded band kernels (seed.h): pairs whose answer provably lies in a narrow
band are finished without the full table.  Every output has to be the full
table's, so every batch here is compared with the oracle, element by element.

The batches hold what the proofs turn on: reads of lengths around whole
numbers of 12-base parts, with 0-12 substitutions and 0-3 indels of 1-20
bases anywhere (the last bases too); windows that begin or end inside the
read's place; tandem repeats and duplicated stretches (parts that occur
twice, equal parts, cores of several diagonals); unrelated reads; reads of
the one-wave classes; and the sizes of items and launches (8 pairs, one
block's planning, lists of one and of many)."""
import numpy as np
import pytest

import gpu_util as U
import synth

pytestmark = pytest.mark.gpu

SCORINGS = [(1, -4, 6, 1), (2, -4, 4, 2), (1, -3, 0, 1), (3, 0, 5, 2), (1, -1, 20, 1), (5, -11, 1, 7)]


@pytest.fixture(scope="module")
def ctx():
    import torch

    import paper_1402_4876_amd as mica
    torch.cuda.set_device(0)
    c = mica.Context(0)
    yield c
    c.close()


def add_noise(b, rate):
    rng = np.random.default_rng(913)
    flip = rng.random(len(b.reads)) < rate
    b.reads[flip] = (b.reads[flip] + rng.integers(1, 4, int(flip.sum())).astype(b.reads.dtype)) % 4


def seeded_batch(n_pairs, mode, m_lo, m_hi, seed):
    rng = np.random.default_rng([911, seed, mode, m_lo, m_hi])
    ref = synth.random_ref(rng, 60_000)
    unit = synth.random_ref(rng, 5)
    ref[10_000:11_500] = np.resize(unit, 1500)          # tandem repeat
    ref[20_000:22_000] = ref[20_300:22_300]             # copies 300 bases apart
    ref[30_000:30_040] = ref[30_003:30_043]             # and 3 apart
    m = rng.integers(m_lo, m_hi + 1, n_pairs).astype(np.int32)
    codes = np.zeros((n_pairs, m_hi), np.uint8)
    win_off = np.zeros(n_pairs, np.int64)
    win_len = np.zeros(n_pairs, np.int32)
    hot = [9_900, 11_400, 20_100, 21_900, 29_990]
    for p in range(n_pairs):
        mm = int(m[p])
        at = int(rng.choice(hot)) + int(rng.integers(-60, 60)) if rng.random() < 0.3 else int(rng.integers(100, 50_000))
        q = list(ref[at: at + mm + 80])
        for _ in range(int(rng.choice([0, 0, 1, 1, 2, 3]))):
            i = int(rng.integers(0, mm))
            k = int(rng.choice([1, 1, 2, 3, 7, 8, 15, 20]))
            if rng.random() < 0.5:
                del q[i: i + k]
            else:
                q[i:i] = list(rng.integers(0, 4, k))
        q = np.array(q[:mm], np.uint8)
        q = np.concatenate([q, rng.integers(0, 4, mm - len(q)).astype(np.uint8)])
        for _ in range(int(rng.choice([0, 0, 1, 2, 3, 5, 12]))):
            i = int(rng.integers(0, mm))
            q[i] = (q[i] + rng.integers(1, 4)) % 4
        r = rng.random()
        if r < 0.08:
            q = rng.integers(0, 4, mm).astype(np.uint8)
        elif r < 0.16:                                   # a random end
            i = int(rng.integers(0, mm))
            q[i:] = rng.integers(0, 4, mm - i)
        codes[p, :mm] = q
        if mode == 2:
            win_off[p], win_len[p] = at, mm + int(rng.integers(-mm // 2, 60))
        else:
            # the window may cut the read's place at either end
            left = int(rng.choice([0, 0, 1, 5, 30, 200])) if rng.random() < 0.8 else -int(rng.integers(0, mm))
            right = int(rng.choice([0, 1, 6, 40, 150])) if rng.random() < 0.8 else -int(rng.integers(0, mm))
            lo, hi = max(0, at - left), at + mm + right
            win_off[p], win_len[p] = lo, max(1, hi - lo)
    b = synth._finish("seeded", ref, win_off, np.maximum(win_len, 1), codes, m, np.full(n_pairs, mode))
    if mode == 2:
        b.h0 = rng.integers(0, 80, n_pairs).astype(np.int32)
    return b


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("m_lo,m_hi", [(1, 40), (24, 60), (71, 100), (150, 150), (230, 420)])
def test_seeded_bands_equal_the_full_table(ctx, mode, m_lo, m_hi):
    b = seeded_batch(1500, mode, m_lo, m_hi, 1)
    for sc in SCORINGS:
        for int32 in (False, True):
            clip = 7 if mode == 2 else 0
            o = U.run_oracle(b, sc, clip=clip)
            g = U.run_gpu(ctx, b, sc, force_int32=int32, clip=clip, max_ext_h0=80 if mode == 2 else 0)
            U.assert_same(g, o, what="seeded mode %d m %d-%d %s int32 %s" % (mode, m_lo, m_hi, sc, int32))


@pytest.mark.parametrize("n_pairs", [1, 7, 8, 9, 1024, 1025, 20_000])
def test_sizes_of_items_and_launches(ctx, n_pairs):
    """All modes in one batch, around the item size, the batches planned by one
    block and the lists that fill several rounds of waves."""
    parts = [seeded_batch(n_pairs // 3 + 1, md, 30, 160, 2) for md in (0, 1, 2)]
    ref = parts[0].ref
    b = synth.Batch(ref=np.concatenate([p.ref for p in parts]),
                    win_off=np.concatenate([p.win_off + i * len(ref) for i, p in enumerate(parts)])[:n_pairs],
                    win_len=np.concatenate([p.win_len for p in parts])[:n_pairs],
                    reads=np.concatenate([p.reads for p in parts]),
                    read_off=np.concatenate([p.read_off + s for p, s in zip(parts, np.cumsum(
                        [0] + [len(p.reads) for p in parts]))])[:n_pairs],
                    read_len=np.concatenate([p.read_len for p in parts])[:n_pairs],
                    mode=np.concatenate([p.mode for p in parts])[:n_pairs], name="seeded mix")
    b.h0 = np.concatenate([np.zeros(parts[0].n_pairs + parts[1].n_pairs, np.int32), parts[2].h0])[:n_pairs]
    for sc in SCORINGS[:2]:
        o = U.run_oracle(b, sc, cap=8, clip=3)
        U.assert_same(U.run_gpu(ctx, b, sc, cap=8, clip=3, max_ext_h0=80), o, cap=8, what="mix of %d" % n_pairs)


@pytest.mark.parametrize("noisy", [False, True])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_scores_alone_of_a_large_batch(ctx, mode, noisy):
    """Without a traceback the band kernels take batches of 65,536 pairs and 3e9 cells or more, and leave those of
    noisy reads."""
    b = seeded_batch(2000, mode, 100, 160, 3)
    if noisy:
        add_noise(b, 0.12)
    o = U.run_oracle(b, trace=False, clip=5)
    o = {k: np.tile(v, 100) for k, v in o.items() if k in U.KEYS_END + ("status",)}
    g = U.run_gpu(ctx, b.subset(np.tile(np.arange(2000), 100)), trace=False, clip=5, max_ext_h0=80 if mode == 2 else 0)
    U.assert_same(g, o, trace=False, what="scores alone, mode %d" % mode)


@pytest.mark.parametrize("mode", [0, 1])
def test_noisy_short_reads(ctx, mode):
    """Traced reads under 96 bases with many errors: the scan stops, some blocks have listed bands by then."""
    b = seeded_batch(3000, mode, 40, 90, 8)
    add_noise(b, 0.12)
    o = U.run_oracle(b)
    o = {k: np.concatenate([v] * 20) for k, v in o.items()}
    U.assert_same(U.run_gpu(ctx, b.subset(np.tile(np.arange(3000), 20))), o, what="noisy, mode %d" % mode)


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_unrelated_pairs(ctx, mode):
    """A batch without a related pair: the scan stops looking, the results stay."""
    rng = np.random.default_rng([912, mode])
    n = 30_000
    b = synth._finish("unrelated", synth.random_ref(rng, 200_000), rng.integers(0, 199_000, n).astype(np.int64),
                      np.full(n, 130), rng.integers(0, 4, (n, 90)).astype(np.uint8), np.full(n, 90, np.int32),
                      np.full(n, mode))
    if mode == 2:
        b.h0 = rng.integers(0, 80, n).astype(np.int32)
    o = U.run_oracle(b, clip=5)
    g = U.run_gpu(ctx, b, clip=5, max_ext_h0=80 if mode == 2 else 0)
    U.assert_same(g, o, what="unrelated, mode %d" % mode)
