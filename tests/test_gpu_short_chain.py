"""Short vectors through ndq_decode_chain, against the oracle bit for bit: the kernel that prepares all
workers of a row side by side, at the edges of its rows, of its code words and of its workgroup's shares,
and the lengths on both sides of the lines between it and the other kernels."""
import numpy as np
import pytest
import torch

import oracle
from oracle import pipeline as opipe
from paper_1904_01197_amd import ndq

pytestmark = pytest.mark.gpu

F = np.float32
# lines: plans that stream, from four workers on, 196,608 + 12,288 W elements, others 131,072 (W + 1), both up to a
# number of workers; one or two lengths are further up, where both sides of it go to the same kernel
PLANS = [
    ((("dq", 4), ("nested", 2)), 4, 0, 0.5, (294912,)),
    ((("dq", 16),) * 3, 16, 1024, 1.0, (311296,)),
    ((("dq", 4), ("nested", 2), ("nested", 2), ("nested", 2)), 4, 0, 0.25, (245760,)),
    ((("dq", 16),) + (("nested", 4),) * 7, 16, 1024, 1.0, (294912,)),
    ((("dq", 8), ("nested", 3), ("dq", 256), ("nested", 100), ("nested", 8)), 8, 0, 1.0, (786432,)),
    ((("dq", 5),) * 4 + (("nested", 3),) * 5, 5, 192, 1.0 / 9, (917504, 1048576)),      # nine workers: sixteen slots
    ((("dq", 2),) + (("nested", 4),) * 16, 4, 64, 1.0, (393216, 524288)),               # 17: thirty-two slots, every bucket in a row
    ((("dq", 3),) * 32, 3, 512, 1.0 / 32, ()),
]


@pytest.mark.parametrize("plan,fine,bucket,scale,lines", PLANS)
def test_short_chains_match_oracle(plan, fine, bucket, scale, lines):
    sizes = [1, 2, 7, 63, 64, 65, 511, 512, 513, 520, 1000, 1024 + 65, 40 * 512 - 3]
    sizes += [line + d for line in lines for d in (0, 1, 511)]
    for n in sizes:
        print(plan, bucket, n, flush=True)
        rng = np.random.default_rng(n)
        common = rng.standard_normal(n, dtype=F)
        host = [common + F(0.3) * rng.standard_normal(n, dtype=F) for _ in plan]
        for w in range(len(plan)):
            host[w][n // 3:n // 3 + 130] = 0                  # buckets whose step is 0
        W, offset = len(plan), 8 * (n % 513) + ((1 << 35) - 2048 if n == 1000 else 0)
        seeds = [11 + w for w in range(W)]
        ds = opipe.dithers(W, seeds, step=9, offset=offset)
        codes, steps, _ = opipe.encode_all(plan, fine, bucket, False, host, ds)
        ref = opipe.decode_chain(plan, bucket, n, codes, steps, ds, scale)
        workers = [(torch.from_numpy(codes[w]).cuda(), torch.from_numpy(steps[w]).cuda(),
                    ndq.NDQ_WORKER_DQ if kind == "dq" else ndq.NDQ_WORKER_NESTED, arg,
                    ndq.ndq_dither(seeds[w], 9, w, offset)) for w, (kind, arg) in enumerate(plan)]
        guarded = torch.full((n + 64,), 7.0, device="cuda")
        out = ndq.ndq_decode_chain(workers, n, bucket, scale, guarded[:n]).cpu().numpy()
        assert np.array_equal(out, ref), (n, np.nonzero(out != ref)[0][:5])
        assert bool((guarded[n:] == 7.0).all())               # nothing behind the vector


def test_a_short_chain_with_shrinkage_matches_oracle():
    n, bucket, alphas = 5000, 128, (1.0, 0.9, 0.75, 1.0)
    plan = (("dq", 16), ("nested", 4), ("nested", 3), ("nested", 8))
    rng = np.random.default_rng(3)
    common = rng.standard_normal(n, dtype=F)
    host = [common + F(0.2) * rng.standard_normal(n, dtype=F) for _ in plan]
    total, workers = None, []
    for w, ((kind, arg), alpha) in enumerate(zip(plan, alphas)):
        d = oracle.dither(5 + w, 2, w, 16)
        if kind == "dq":
            c, s = oracle.dq_encode(host[w], 0.0, arg, bucket, d)
            total = oracle.dq_decode(c, n, arg, bucket, s, d)
        else:
            c, s = oracle.nested_encode(host[w], 0.0, 16, arg, bucket, d, alpha=alpha)
            total = total + oracle.nested_decode(c, n, arg, bucket, s, d, total, side_scale=F(1.0) / F(w), alpha=alpha)
        workers.append((torch.from_numpy(c).cuda(), torch.from_numpy(s).cuda(),
                        ndq.NDQ_WORKER_DQ if kind == "dq" else ndq.NDQ_WORKER_NESTED, arg,
                        ndq.ndq_dither(5 + w, 2, w, 16), alpha))
    out = ndq.ndq_decode_chain(workers, n, bucket, 1.0).cpu().numpy()
    assert np.array_equal(out, total)
