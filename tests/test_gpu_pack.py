"""Packing on the GPU: whole words by one 16-byte load where the codes are
aligned for it, byte by byte elsewhere and in the last word."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 1, 4, 8, 15, 16])
@pytest.mark.parametrize("n", [0, 1, 15, 16, 17, 31, 32, 4095, 4096, 4097, 70_001])
def test_pack_alignment_and_remainders(n, offset):
    import torch

    import paper_1402_4876_amd as mica
    from paper_1402_4876_amd.pack import pack_codes
    rng = np.random.default_rng([914, n, offset])
    codes = rng.integers(0, 256, n + offset).astype(np.uint8)  # only a code's low two bits count
    part = torch.from_numpy(codes).cuda()[offset:]
    assert n == 0 or part.data_ptr() % 16 == offset % 16
    got = mica.pack_2bit(part).cpu().numpy().view(np.uint32)
    assert np.array_equal(got, pack_codes(codes[offset:]))
