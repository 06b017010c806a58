"""The search's interval table: parts one base shorter, as long and longer than
the table's strings, references around the sizes at which the strings grow
(4^K entries of 8 bytes within twice the reference), matches at both ends of
the reference (strings the text ends inside), repeats above and below
max_occ, and the seeds of the parts."""
import numpy as np
import pytest
import torch

import oracle
from paper_1402_4876_amd import FmIndex, pack_codes

pytestmark = pytest.mark.gpu


def _string_bases(n):
    k = 0
    while k < 12 and 8 << (2 * (k + 1)) <= 2 * n:
        k += 1
    return k


@pytest.mark.parametrize("n", [15, 16, 63, 64, 1023, 1024, 16_383, 16_384, 70_000])
@pytest.mark.parametrize("k", [0, 1, 2])
def test_parts_around_the_table(n, k):
    rng = np.random.default_rng([5, n, k])
    ref = rng.integers(0, 4, n, dtype=np.uint8)
    if n >= 1000:
        ref[n // 2: n // 2 + 200] = np.resize(rng.integers(0, 4, 3, dtype=np.uint8), 200)
        ref[-40:] = ref[100:140]
    K = _string_bases(n)
    reads = []
    for d in (-1, 0, 1, 7):
        m = max(k + 1, (K + d) * (k + 1) + (1 if d == 7 else 0))
        if m > n:
            continue
        for p in [0, n - m] + [int(x) for x in rng.integers(0, n - m + 1, 40)]:
            q = ref[p: p + m].copy()
            for w in rng.integers(0, m, int(rng.integers(0, 3))):
                q[w] = (q[w] + 1) % 4
            reads.append(q)
    flat = np.concatenate(reads + [np.zeros(16, np.uint8)])
    ln = np.array([len(q) for q in reads], np.int32)
    off = np.concatenate([[0], np.cumsum(ln)[:-1]]).astype(np.int64)
    ix = FmIndex(pack_codes(ref), n)
    for max_occ in (1, 2, 64):
        out = ix.search(torch.from_numpy(pack_codes(flat).view(np.int32)).cuda(), torch.from_numpy(off).cuda(),
                        torch.from_numpy(ln).cuda(), k=k, max_occ=max_occ, reads_len=len(flat), cand=True)
        torch.cuda.synchronize()
        want = oracle.kmm_search(ref, flat, off, ln, k=k, max_occ=max_occ)
        for key in ("best_mm", "n_best", "n_hits", "pos", "status"):
            got = out[key].cpu().numpy().astype(np.int64)
            assert np.array_equal(got, want[key].astype(np.int64)), (key, n, k, max_occ)
        # seeds: the smallest placement of each part's occurrences
        text, cand = ref.tobytes(), out["cand"].cpu().numpy()
        for r, q in enumerate(reads):
            for j in range(k + 1):
                a, e = j * len(q) // (k + 1), (j + 1) * len(q) // (k + 1)
                part, at, found = q[a:e].tobytes(), -1, []
                while (at := text.find(part, at + 1)) >= 0:
                    found.append(at - a)
                seed = min(found) if found and len(found) <= max_occ else -2**63
                assert cand[r, j] == seed, (r, j, n, k, max_occ)
    ix.close()
