"""The encoder's code widths that are known at compile time, in every form of a bucket (one step, a tile or
less, several buckets to a tile, several tiles to a bucket), on vectors that end inside a tile, a row, a
bucket and a group of four lanes: every step and every byte against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1904_01197_amd import ndq, workloads

pytestmark = pytest.mark.gpu

F = np.float32


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("bucket", [0, 512, 1024, 2048, 4096, 8192, 16384])
def test_every_code_width_matches_oracle(dtype, bucket):
    tile = 2048 if dtype == "f32" else 4096
    for n in (2 * tile, 3 * tile + 517, 9 * tile + 8, 8 * tile + 1, 4 * tile - 511):
        rng = np.random.default_rng(n + bucket)
        x = (rng.standard_t(3.0, n) * 0.01).astype(F)
        x[tile // 2:tile // 2 + 700] = 0                     # a bucket whose step is 0
        x[n // 2] = 5.0                                      # neighbours of very different steps
        g = workloads.f32_to_bf16_bits(x) if dtype == "bf16" else x
        t = torch.from_numpy(g)
        g_d = (t.view(torch.bfloat16) if dtype == "bf16" else t).cuda()
        d_o, d_g = oracle.dither(n, 3, 2, 8 * bucket), ndq.ndq_dither(n, 3, 2, 8 * bucket)
        for levels in (2, 3, 8, 16, 32):
            c_ref, s_ref = oracle.dq_encode(g, 0.0, levels, bucket, d_o)
            codes, steps = ndq.ndq_dq_encode(g_d, 0.0, levels, bucket, d_g)
            assert np.array_equal(steps.cpu().numpy(), s_ref), (n, levels)
            assert codes.cpu().numpy().tobytes() == c_ref.tobytes(), (n, levels)
        for M, alpha in ((2, 1.0), (4, 0.9), (8, 1.0), (16, 1.0), (3, 1.0), (7, 0.75), (12, 1.0)):
            c_ref, s_ref = oracle.nested_encode(g, 0.0, 16, M, bucket, d_o, alpha=alpha)
            codes, steps = ndq.ndq_nested_encode(g_d, 0.0, 16, M, alpha, bucket, d_g)
            assert np.array_equal(steps.cpu().numpy(), s_ref), (n, M)
            assert codes.cpu().numpy().tobytes() == c_ref.tobytes(), (n, M)
            if bucket == 0:                                  # a step that is handed over bounds nothing
                step = torch.tensor([s_ref[0]], device="cuda")
                codes, _ = ndq.ndq_nested_encode_with_step(g_d, step, M, alpha, d_g)
                assert codes.cpu().numpy().tobytes() == c_ref.tobytes(), (n, M, "handed over")
