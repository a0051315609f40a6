"""The dense transcoders for every number of digits per word and code width, at the edges of a word, of a
thread's share and of a workgroup's, with the largest indices and with words that no stream of indices holds,
against the oracle byte for byte."""
import numpy as np
import pytest
import torch

import oracle
from paper_1904_01197_amd import ndq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("levels", [2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 16, 17, 24, 32, 33, 41, 64, 65, 85, 128, 129, 256])
def test_every_form_matches_oracle(levels):
    k, bits = oracle.dense_group(levels), oracle.code_bits(levels)
    for n in (1, k - 1, k, k + 1, 4 * k, 4 * k + 1, 8 * k - 1, 1024 * k - 1, 1024 * k, 1024 * k + 1, 2048 * k + 3, 5000 * k + 7):
        if n < 1:
            continue
        rng = np.random.default_rng(n)
        codes = rng.integers(0, levels, n).astype(np.uint8)
        codes[-min(n, 3 * k):] = levels - 1                  # full digits at the end
        ref = oracle.dense_pack(codes, levels)
        fixed = oracle.pack(codes, bits)
        fixed_d = torch.from_numpy(fixed).cuda()
        dense = torch.full((ref.size + 32,), 0x5A, dtype=torch.uint8, device="cuda")
        ndq.ndq_dense_pack(fixed_d, n, levels, dense[:ref.size])
        assert dense[:ref.size].cpu().numpy().tobytes() == ref.tobytes(), n
        back = torch.full((fixed.size + 32,), 0x5A, dtype=torch.uint8, device="cuda")
        ndq.ndq_dense_unpack(dense[:ref.size], n, levels, back[:fixed.size])
        assert back[:fixed.size].cpu().numpy().tobytes() == fixed.tobytes(), n
        assert bool((dense[ref.size:] == 0x5A).all()) and bool((back[fixed.size:] == 0x5A).all())


@pytest.mark.parametrize("levels", [3, 5, 6, 7, 10, 12, 20, 100])
def test_words_that_are_no_numbers_of_the_base_stay_in_bounds(levels):
    # a word from levels^k on: its lowest k digits, as repeated division gives them
    k, bits = oracle.dense_group(levels), oracle.code_bits(levels)
    rng = np.random.default_rng(levels)
    words = rng.integers(0, 1 << 32, 4096, dtype=np.uint64).astype(np.uint32)
    words[:4] = [0xFFFFFFFF, levels ** k - 1, min(levels ** k, 0xFFFFFFFF), 0]
    want, rest = np.empty((words.size, k), dtype=np.uint8), words.copy()
    for j in range(k):
        want[:, j] = rest % levels
        rest //= levels
    codes = ndq.ndq_dense_unpack(torch.from_numpy(words.view(np.uint8)).cuda(), words.size * k, levels)
    assert codes.cpu().numpy().tobytes() == oracle.pack(want.reshape(-1), bits).tobytes()
