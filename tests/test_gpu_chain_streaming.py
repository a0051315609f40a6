"""The persistent chain decoder at its real grid size, against the oracle bit for bit, at inputs
where its rearranged arithmetic has to give way: steps outside the range in which the fold
divided by M is exact, and dither indices whose block number crosses a 32-bit word."""
import numpy as np
import pytest
import torch

import oracle
from oracle import pipeline as opipe
from paper_1904_01197_amd import ndq

pytestmark = pytest.mark.gpu

F = np.float32
TILES = 2 * 6144                     # tiles of 1,024 elements from which the persistent launch is used


def _check(plan, fine, bucket, host, offset, scale=1.0):
    n, W = host[0].size, len(plan)
    seeds = [11 + w for w in range(W)]
    ds = opipe.dithers(W, seeds, step=9, offset=offset)
    codes, steps, _ = opipe.encode_all(plan, fine, bucket, False, host, ds)
    ref = opipe.decode_chain(plan, bucket, n, codes, steps, ds, scale)
    workers = [(torch.from_numpy(codes[w]).cuda(), torch.from_numpy(steps[w]).cuda(),
                ndq.NDQ_WORKER_DQ if kind == "dq" else ndq.NDQ_WORKER_NESTED, arg,
                ndq.ndq_dither(seeds[w], 9, w, offset)) for w, (kind, arg) in enumerate(plan)]
    out = ndq.ndq_decode_chain(workers, n, bucket, scale).cpu().numpy()
    assert np.array_equal(out, ref), np.nonzero(out != ref)[0][:5]


def _gradients(W, n, seed):
    rng = np.random.default_rng(seed)
    common = rng.standard_normal(n, dtype=F)
    return [common + F(0.3) * rng.standard_normal(n, dtype=F) for _ in range(W)]


@pytest.mark.parametrize("M", [2, 4])
@pytest.mark.parametrize("tail", [0, 517])
def test_steps_of_any_magnitude(M, tail):
    n, bucket = TILES * 1024 + tail, 4096
    host = _gradients(3, n, 3 + M)
    scale = np.ones(n // bucket + 1, dtype=F)
    scale[1::7] = F(2.0 ** 49)       # just inside and just outside of the exact range, and far outside
    scale[2::7] = F(2.0 ** 52)
    scale[3::7] = F(2.0 ** 120)
    scale[4::7] = F(2.0 ** -61)
    scale[5::7] = F(2.0 ** -95)
    scale[6::21] = F(0.0)
    for w, g in enumerate(host):
        g *= np.repeat(scale, bucket)[:n]
        g[7 * bucket * (w + 1):7 * bucket * (w + 1) + bucket] *= F(2.0 ** 70)    # one worker's step alone
    _check((("dq", 4), ("nested", M), ("nested", M)), 4, bucket, host, 64)


@pytest.mark.parametrize("n,offset", [
    (TILES * 1024 + 1024, 5 << 35),                 # a high word that is not zero
    (TILES * 1024 + 8, (1 << 35) - 8 * 4096),       # the block number's low word wraps inside the call
    (5000, (1 << 35) - 2048), (4096, (1 << 35) - 4096), (1024, (3 << 35) - 1032)])
def test_dither_indices_beyond_32_bits(n, offset):
    _check((("dq", 4), ("nested", 2), ("nested", 2)), 4, 0, _gradients(3, n, 8), offset, 0.5)


@pytest.mark.parametrize("plan,fine,bucket", [
    ((("dq", 8), ("nested", 4), ("nested", 3), ("dq", 256), ("nested", 100)), 8, 0),    # every fetch width of the general kernel
    ((("dq", 4), ("nested", 2), ("nested", 2)), 4, 0),
    ((("dq", 16),) * 3, 16, 1024),
    ((("dq", 3),), 3, 512)])
def test_short_vectors_take_one_row_per_wave(plan, fine, bucket):
    # edges of a row (512 elements) and of the 64-bit code loads at the stream's end, and the
    # lengths at which the tile grows from one row to two (2,048 and 4,096 tiles of 1,024)
    for n in (1, 7, 8, 63, 511, 512, 513, 520, 575, 1024 + 65, 2047 * 1024 + 1023, 2048 * 1024, 4096 * 1024 - 8,
              4096 * 1024 + 1):
        _check(plan, fine, bucket, _gradients(len(plan), n, n), 8 * (n % 513), 0.25)


@pytest.mark.parametrize("plan,fine,bucket,sizes", [
    # one tile per wave, of one row and of two, on both sides of the plans whose lanes put results in order before
    # the store: whole tiles, a row more, ragged ends
    ((("dq", 16),), 16, 0, (1024 * 700, 1024 * 700 + 517)),
    ((("dq", 4), ("dq", 16)), 16, 0, (1, 512, 515, 1024 * 700 + 5, 1024 * 2047 + 513, 1024 * 2100, 1024 * 2100 + 1)),
    ((("dq", 4), ("nested", 2)), 4, 2048, (7, 513, 1024 * 700 + 520, 1024 * 2100 + 1023)),
    ((("dq", 16),) * 3, 16, 0, (1024 * 700 + 511, 1024 * 2100 + 512)),
    ((("dq", 4), ("nested", 4), ("nested", 4)), 16, 0, (1024 * 700 + 8, 1024 * 2100 + 8)),
    # the general kernel's code loads at the stream's end, a worker of every width it has alone
    ((("dq", 8),), 8, 0, (1, 7, 8, 63, 511, 513, 520, 575, 1089)), ((("dq", 32),), 32, 0, (1, 7, 8, 63, 511, 513, 520, 575, 1089)),
    ((("dq", 64),), 64, 0, (1, 7, 8, 63, 511, 513, 520, 575, 1089)), ((("dq", 128),), 128, 0, (1, 7, 8, 63, 511, 513, 520, 575, 1089)),
    ((("dq", 256),), 256, 0, (1, 7, 8, 63, 511, 513, 520, 575, 1089)),
    # the general kernel's form for two workers in tiles of two rows, whole and ragged
    ((("dq", 32),) * 2, 32, 0, (1024 * 4200, 1024 * 4200 + 517)), ((("dq", 32),) * 2, 32, 512, (1024 * 4200, 1024 * 4200 + 517)),
    ((("dq", 100), ("nested", 64)), 100, 3072, (1024 * 4203, 1024 * 4200 + 8)),
    # (3-bit codes are the general kernel's where buckets are neither rows nor tiles; with one row per wave and with two)
    ((("dq", 8),), 8, 192, (1, 7, 8, 63, 511, 513, 520, 575, 1089, 1024 * 4200 + 3, 1024 * 4200 + 513))])
def test_few_workers_match_oracle(plan, fine, bucket, sizes):
    for n in sizes:
        print(plan, bucket, n, flush=True)
        _check(plan, fine, bucket, _gradients(len(plan), n, n), 8 * (n % 513), 0.75)


@pytest.mark.parametrize("kind", ["dq", "nested"])
@pytest.mark.parametrize("first", [2, 4, 16])
@pytest.mark.parametrize("other", [2, 4, 16])
def test_one_tile_forms_of_every_pair_of_widths_match_oracle(kind, first, other):
    # one row per wave and two, whole tiles and a ragged end
    for n in (1024 * 700, 1024 * 700 + 517, 1024 * 2100, 1024 * 2100 + 517):
        print(kind, first, other, n, flush=True)
        _check((("dq", first),) + ((kind, other),) * 2, 16, 0, _gradients(3, n, n + other), 64, 0.5)


def test_buckets_of_a_row_with_a_ratio_that_is_no_power_of_two():
    n = 2050 * 1024 + 77
    _check((("dq", 4), ("nested", 3)), 4, 512, _gradients(2, n, 5), 8, 0.5)


@pytest.mark.parametrize("last", [[(ndq.NDQ_WORKER_NESTED, 3, 1.0), (ndq.NDQ_WORKER_DQ, 32, 1.0)], [(ndq.NDQ_WORKER_NESTED, 4, 0.9), (ndq.NDQ_WORKER_NESTED, 4, 1.0)],
                                  [(ndq.NDQ_WORKER_NESTED, 4, 1.0), (ndq.NDQ_WORKER_DQ, 32, 1.0)]])
def test_the_last_two_of_34_workers_in_a_launch_of_their_own(last):
    # long enough for tiles of two rows; against the single calls, which other tests compare with the oracle
    n = 1024 * 4200 + 517
    gen = torch.Generator(device="cuda").manual_seed(len(last))
    workers, out = [], torch.empty(n, device="cuda")
    for w, (kind, arg, alpha) in enumerate([(ndq.NDQ_WORKER_DQ, 32, 1.0)] * 32 + last):
        # (codes below M: 3 of 4 two-bit values, by clearing the high bit of the fourth)
        codes = torch.randint(0, 256, (ndq.ndq_packed_bytes(n, oracle.code_bits(arg)),), dtype=torch.uint8, device="cuda", generator=gen)
        if arg == 3:
            codes = codes & ~((codes << 1) & 0xAA)
        d = ndq.ndq_dither(7 + w, 3, w, 64)
        step = torch.full((1,), 0.01 * (w + 1), device="cuda")
        workers.append((codes, step, kind, arg, d, alpha))
        if kind == ndq.NDQ_WORKER_DQ:
            ndq.ndq_dq_decode(codes, n, arg, 0, step, d, out, accumulate=w > 0)
        else:
            ndq.ndq_nested_decode(codes, n, arg, alpha, 0, step, d, out, float(F(1) / F(w)), out, accumulate=True)
    got = ndq.ndq_decode_chain(workers, n, 0, 1.0)
    assert torch.equal(got, out)
