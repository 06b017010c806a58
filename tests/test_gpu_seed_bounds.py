"""Seeded bands at the edge of their bounds: pairs whose best alignment lies just outside a band that a weaker bound
would accept.  Compared with the oracle, element by element."""
import numpy as np
import pytest

import gpu_util as U
import synth

pytestmark = pytest.mark.gpu

# (mode, scoring, read, window): insertions of more than 13 bases, which swallow whole parts of the read; local, the
# first and the last part (which clipping spoils for nothing) on a diagonal of their own
PAIRS = [
    (0, (2, -20, 40, 2),
     "TCAGTTTATGCCCCCGTAGGCCCTAGTAGTATGCCAAGGCGTGCTTTCCTCCTCCCTTACTATGCAAACGCTCTGCAGATTTCGTCCAGATGCATATTGCGTCCG",
     "GTATGAAACGTTGTTCAGTTTATGCCCCCGTAGGCCCTAGTAGTATGCCAAGGCGTGCTTTCCTCCTCCCTTACTATGCAAACGCGATGCATATTGCGTCCGGATGCATATTGC"
     "GTCCGGAAGACTCGAGTT"),
    (0, (1, -9, 16, 2),
     "CCGTCCGGGACTCGCTTCGAAGATTAGTCGCGTGGCCTCTGGTAAATAGATTAATGTAACCATGTCCGTAACTTTTTACCGTAACCCTTTTCTACCGTAACCCTT",
     "CGACCTCGGATCACATTGGAAGGTCCCGTCCGGGACTCGCTTCGAAGATTAGTCGCGTGGCCTCTGGTAAATAGATTAATGTAACCATGTCCGTAATTTTCTACCGTAACCCTT"
     "TCCTACCGTGTCCAATCATCTGTCAGTGACGCTAGAGTATTAT"),
    (0, (1, -23, 18, 2),
     "CTCGTCTAAATCATCTTCTCGTCTAAACGATATTTCTCCGGCTGAGTGGTCATAAGGCAGCTTTTGTTCGGAGTGTATGCCACCTCATACCGATAGTCTAGGGTGGGATAGATG"
     "CTTCGATGCTATAGCGAGCGTAACGGAGC",
     "CCGATGTATTCTAATACACCGCGAGTATCTCGACTAAATCATCTGCTCGTCTAAATGATATTTCTCCGGCTGAGTGGTCATAAGGCAGCTTTTGTTCGGAGTGTATGCCACCTC"
     "ATACCGATAGTCTAGGGTGGGATAGATGCTTCGATGCTATAGCGAGCGTAACGGAGCGAGAGCTTGGAC"),
    (1, (1, -4, 6, 1),
     "ATGTTGCGCCCGTGTAATCCTGGCTAAAAATATAGGACACACACCGCCAGGTCGGTGAACTCATCGCGACTGCGGATCTACCCTTTATCGTACCGTCTCTTATTTTGATATCGT"
     "ACCGTCCTG",
     "TAGACTTTCTATGCCTTCACAGGCCCTGGACCATGAGAAAGATAGCCATGTTGCGCCCGCTAATTGGAGGTTGTTGCGCCCGTGTAATCCTGGCTAAAAATATAGGACACACAC"
     "CGCCAGGTCGGTGAACTCATCGCGACTGCGGATCTACCCTTTATCGTACCGTCTCTTATTTTGATAGGATAATCGTACCGTCCTGAAACTAAGTGCGAACAG"),
]


@pytest.fixture(scope="module")
def ctx():
    import torch

    import paper_1402_4876_amd as mica
    torch.cuda.set_device(0)
    c = mica.Context(0)
    yield c
    c.close()


def codes(text):
    return np.array(["ACGT".index(x) for x in text], np.uint8)


def batch(reads, windows, mode):
    """Pairs of codes, each window a stretch of a reference of its own."""
    n = len(reads)
    win_len = np.array([len(w) for w in windows], np.int32)
    off = np.concatenate([[0], np.cumsum(win_len[:-1], dtype=np.int64)]).astype(np.int64)
    m = np.array([len(r) for r in reads], np.int32)
    table = np.zeros((n, int(m.max())), np.uint8)
    for p, r in enumerate(reads):
        table[p, :len(r)] = r
    return synth._finish("bounds", np.concatenate(windows), off, win_len, table, m, np.full(n, mode))


@pytest.mark.parametrize("int32", [False, True])
@pytest.mark.parametrize("mode,scoring,read,window", PAIRS, ids=["%d:%s" % (p[0], p[1]) for p in PAIRS])
def test_known_pairs(ctx, mode, scoring, read, window, int32):
    b = batch([codes(read)] * 3, [codes(window)] * 3, mode)
    U.assert_same(U.run_gpu(ctx, b, scoring, force_int32=int32), U.run_oracle(b, scoring), what="known pair")


@pytest.mark.parametrize("scoring", [(2, -20, 40, 2), (1, -9, 16, 2), (1, -8, 14, 1), (1, -10, 20, 1), (1, -4, 6, 1)])
def test_insertion_near_an_end_of_a_nearly_periodic_window(ctx, scoring):
    rng = np.random.default_rng([931, -scoring[1]])
    reads, windows = [], []
    for _ in range(1500):
        m, w = int(rng.integers(90, 160)), int(rng.integers(14, 26))
        q = rng.integers(0, 4, m).astype(np.uint8)
        t = int(rng.integers(12, 40))                      # the tail that the inserted bases lead to
        win = np.concatenate([rng.integers(0, 4, 30), q, rng.integers(0, 4, 40)]).astype(np.uint8)
        win[30 + m - t - w: 30 + m - w] = q[m - t:]        # the tail, w bases early
        for i in range(m - t, m, int(rng.integers(6, 13))):  # and its own place, its parts spoiled
            win[30 + i] = (win[30 + i] + rng.integers(1, 4)) % 4
        if rng.random() < 0.5:                             # the same at the head
            q, win = q[::-1].copy(), win[::-1].copy()
        reads.append(q)
        windows.append(win)
    b = batch(reads, windows, 0)
    U.assert_same(U.run_gpu(ctx, b, scoring), U.run_oracle(b, scoring), what="insertions %s" % (scoring,))


@pytest.mark.parametrize("scoring", [(1, -4, 6, 1), (1, -3, 5, 2), (2, -4, 4, 2)])
def test_local_end_parts_on_a_diagonal_of_their_own(ctx, scoring):
    rng = np.random.default_rng([932, -scoring[1]])
    reads, windows = [], []
    for _ in range(6000):
        m, d = int(rng.integers(72, 160)), int(rng.integers(1, 30)) * int(rng.choice([-1, 1]))
        q = rng.integers(0, 4, m).astype(np.uint8)
        last = 12 * (m // 12 - 1)
        # one end part as the read repeats it further in
        for i in (range(0, 12) if d > 0 else range(last, last + 12)):
            q[i + d] = q[i]
        win = np.concatenate([rng.integers(0, 4, 60), q, rng.integers(0, 4, 60)]).astype(np.uint8)
        for part in (0, last):                              # both spoiled in place
            i = 60 + part + int(rng.integers(0, 12))
            win[i] = (win[i] + rng.integers(1, 4)) % 4
        if d > 0:                                           # the other on the same diagonal
            win[60 + d + last: 60 + d + last + 12] = q[last: last + 12]
        else:
            win[60 + d: 60 + d + 12] = q[:12]
        past, cut = int(rng.integers(1, 13)) * int(rng.choice([-1, 1])), int(rng.integers(1, 5))
        if rng.random() < 0.5:                              # an end, without its part, a gap away
            win[60 + past + last + cut: 60 + past + m] = q[last + cut:]
        else:
            win[60 + past: 60 + past + 12 - cut] = q[:12 - cut]
        reads.append(q)
        windows.append(win)
    b = batch(reads, windows, 1)
    U.assert_same(U.run_gpu(ctx, b, scoring), U.run_oracle(b, scoring), what="end parts %s" % (scoring,))
