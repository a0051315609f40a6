"""Chain decoder, plans with several DQSG workers before the nested ones, with 3-bit codes, with ratios that are no
powers of two and with buckets of one row, in the streaming kernel's forms (one row or one tile per wave, persistent),
against the oracle bit for bit: whole and ragged last tiles, codes up to the last byte of a stream, buckets of whole
tiles, steps that are 0 or far from 1."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import launch_recording as lr
import oracle
from oracle import pipeline as opipe
from paper_1904_01197_amd import ndq

F = np.float32
DQ, NESTED = "dq", "nested"
PLANS = {
    "1 of 8": [(DQ, 8)], "2 of 5": [(DQ, 5)] * 2, "8 and 5 of 3 bits": [(DQ, 8), (DQ, 5)] * 4, "8, M 4": [(DQ, 8), (NESTED, 4)],
    "5, M 2": [(DQ, 5), (NESTED, 2)], "16, M 8": [(DQ, 16)] + [(NESTED, 8)] * 2, "3 and 4, M 2": [(DQ, 3), (DQ, 4), (NESTED, 2), (NESTED, 2)],
    "4, M 4": [(DQ, 4)] * 2 + [(NESTED, 4)], "4, M 8": [(DQ, 4)] * 3 + [(NESTED, 8)], "8, M 2": [(DQ, 8)] * 2 + [(NESTED, 2)] * 3,
    "8, M 8": [(DQ, 8)] * 2 + [(NESTED, 8)], "16, M 2": [(DQ, 16)] * 2 + [(NESTED, 2)] * 2, "16, M 4": [(DQ, 16)] * 8 + [(NESTED, 4)] * 8,
    "5, M 3": [(DQ, 5)] * 4 + [(NESTED, 3)] * 4, "16, M 7": [(DQ, 16), (NESTED, 7)], "4, M 5": [(DQ, 4)] * 2 + [(NESTED, 5)],
    "3, M 3": [(DQ, 3)] + [(NESTED, 3)] * 7, "8, M 6": [(DQ, 8)] * 2 + [(NESTED, 6)], "4 of 8": [(DQ, 8)] * 4,
    "16, 15 of M 8": [(DQ, 16)] + [(NESTED, 8)] * 15,
}
# with buckets of one row (also plans whose other kernels are not the rarer plans')
ROW_PLANS = dict(PLANS, **{"2": [(DQ, 2)] * 2, "2, M 2": [(DQ, 2), (NESTED, 2)], "4, M 2": [(DQ, 4)] + [(NESTED, 2)] * 3, "16": [(DQ, 16)] * 3,
                           "16, M 16": [(DQ, 16), (NESTED, 16)], "16 and M 4": [(DQ, 16)] + [(NESTED, 4)] * 2})


def _tight(n):
    """The next length whose 3-bit stream ends with one byte, and with two, of the last lane's three."""
    out = []
    for left in (1, 2):
        m = n
        while oracle.packed_bytes(m, 3) - m // 8 * 3 != left or m % 8 == 0:
            m += 1
        out.append(m)
    return out


def _tiles_from(plan):
    """Tiles of 1,024 elements from which a wave takes two rows (fewer where the persistent form comes first)."""
    W, dq = len(plan), sum(kind == DQ for kind, _ in plan)
    if W < 4:
        return {1: 2048, 2: 1280, 3: 1536}[W]
    if dq == W:
        return 4864 if W < 8 else 2048
    any_ratio = plan[-1][1] in (3, 5, 6, 7)
    if any_ratio and W - dq >= 7:
        return 2048
    return 4096 if plan[-1][1] == 8 and W >= 12 else 2600


ROWS = [513, 512 * 2, 512 * 9 + 1, 512 * 40 - 1, 1024 * 15 + 8, 1024 * 33 + 512] + _tight(530) + _tight(1024 * 8)
# (up to 786,432 elements several workers are the kernel for short chains': rows of them from there on)
LONG_ROWS = [1024 * 772 + 513, 1024 * 772 + 512 * 9 + 8] + _tight(1024 * 773 + 530)
TILES = [1024 * 12, 1024 * 40, 1024 * 37 + 100, 1024 * 3 + 8, 1024 * 13 + 1, 1024 * 24 + 1023, 1025] + _tight(1024 * 14) + _tight(1024 * 25 + 640)


def _check(plan, n, bucket, offset, scale):
    """Any codes and steps are a message."""
    rng = np.random.default_rng(n + bucket + len(plan))
    ds_o = opipe.dithers(len(plan), [7 + w for w in range(len(plan))], step=3, offset=offset)
    codes, steps, workers = [], [], []
    for w, (kind, arg) in enumerate(plan):
        codes.append(oracle.pack(rng.integers(0, arg, n).astype(np.uint32), oracle.code_bits(arg)))
        s = (F(0.01) * (F(1) + rng.random(oracle.num_buckets(n, bucket), dtype=F))).astype(F)
        if s.size > 3:
            s[rng.integers(0, s.size, 3)] = [F(0), F(2.0 ** 52), F(2.0 ** -62)]      # outside the range of the fold divided by M
        steps.append(s)
        workers.append((torch.from_numpy(codes[w]).cuda(), torch.from_numpy(s).cuda(),
                        ndq.NDQ_WORKER_DQ if kind == DQ else ndq.NDQ_WORKER_NESTED, arg, ndq.ndq_dither(7 + w, 3, w, offset)))
    ref = opipe.decode_chain(plan, bucket, n, codes, steps, ds_o, scale)
    out = torch.full((n + 16,), -3.0, device="cuda")
    ndq.ndq_decode_chain(workers, n, bucket, scale, out[:n])
    got = out[:n].cpu().numpy()
    assert np.array_equal(got, ref), (plan, n, bucket, np.nonzero(got != ref)[0][:5])
    assert bool((out[n:] == -3.0).all())


def _sweep(sizes):
    for name, plan in ROW_PLANS.items():
        for i, n in enumerate(sizes):
            bucket = (0, 1024, 2048, 8192)[(i + len(plan)) % 4]
            print(name, n, bucket, flush=True)
            _check(plan, n, bucket, 8 * (n % 4099), 1.0 if i % 2 else 0.25)
            _check(plan, n, 512, 0, 1.0)
            if bucket:
                _check(plan, n, 0, 0, 1.0)


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(PLANS))
def test_rows_and_tiles_match_oracle(name):
    plan = PLANS[name]
    long = 1024 * _tiles_from(plan)
    rows = ROWS + (LONG_ROWS if len(plan) > 1 else [])
    for n, bucket in [(n, b) for n in rows for b in (0, 1024)] + [(long - 1, 0), (long, 0), (long + 1, 2048), (long + 4 * 1024 + 700, 0)] + [
            (n, 0) for n in _tight(long + 300)[:1 if len(plan) > 8 else 2]]:
        _check(plan, n, bucket, 8 * (n % 129), 1.0 / len(plan))


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(ROW_PLANS))
def test_buckets_of_a_row_match_oracle(name):
    plan = ROW_PLANS[name]
    rows = ROWS + (LONG_ROWS if len(plan) > 1 else [])
    for n in rows + [1024 * 2048 - 1, 1024 * 2048 + 513, 1024 * 2100]:
        _check(plan, n, 512, 8 * (n % 129), 1.0 / len(plan))


# DQSG and nested workers, 3-bit codes up to the stream's last byte, a ratio that is no power of two, a step per row
@pytest.mark.gpu
@pytest.mark.parametrize("plan,tiles,bucket", [
    ([(DQ, 16)] * 2 + [(NESTED, 4)], 10240, 4096), ([(DQ, 8), (NESTED, 2)], 10240, 0), ([(DQ, 8), (DQ, 5)] * 4, 2048, 2048),
    ([(DQ, 3)] + [(NESTED, 3)] * 7, 2048, 1024), ([(DQ, 5)] * 2 + [(NESTED, 3)], 10240, 0),
    ([(DQ, 4), (NESTED, 2)], 8192, 512), ([(DQ, 16)] * 2, 8192, 512), ([(DQ, 5), (NESTED, 3)], 8192, 512), ([(DQ, 8)] * 2 + [(NESTED, 8)], 8192, 512)])
def test_persistent_form_matches_oracle_on_its_own_grid(plan, tiles, bucket):
    for n in (1024 * tiles, _tight(1024 * tiles + 530)[0]):
        print(plan, n, bucket, flush=True)
        _check(plan, n, bucket, 8 * (n % 129), 1.0 / len(plan))


@pytest.mark.gpu
def test_persistent_form_matches_oracle_on_short_vectors():
    # (the library reads the thresholds once per process)
    env = dict(os.environ, NDQ_STREAM_MIN_TILES_PER_WAVE="0", NDQ_STREAM_MAX_BLOCKS="3", PYTHONPATH=os.pathsep.join(sys.path))
    code = "import sys; sys.path.insert(0, %r); import test_gpu_chain_plans as t; t._sweep(t.TILES); print('PLANS_OK')" % os.path.dirname(
        os.path.abspath(__file__))
    res = subprocess.run([sys.executable, "-u", "-c", code], env=env, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True,
                         timeout=300)
    assert res.returncode == 0 and "PLANS_OK" in res.stdout, "\n".join(res.stdout.splitlines()[-15:])


@pytest.mark.gpu
@pytest.mark.parametrize("plan", [[(DQ, 5)] * 4 + [(NESTED, 3)] * 4, [(DQ, 3)] + [(NESTED, 3)] * 7, [(DQ, 16), (NESTED, 7)]])
def test_sums_beyond_binary32_do_not_depend_on_the_kernel(plan):
    # an infinite running mean: a nested worker whose ratio is no power of two makes it NaN.  Short chains, the general kernel
    # (buckets of 64), one row and one tile per wave, persistent tiles, buckets of a row in both forms
    for n, bucket in ((5000, 0), (5000, 512), (5000, 64), (1024 * 1100 + 5, 1024), (1024 * 2200 + 5, 2048), (1024 * 2200 + 5, 512),
                      (1024 * 10300 + 5, 4096), (1024 * 8300 + 5, 512)):
        print(plan, n, bucket, flush=True)
        rng = np.random.default_rng(n + bucket)
        ds = opipe.dithers(len(plan), [7 + w for w in range(len(plan))], step=3, offset=0)
        codes, steps, workers = [], [], []
        for w, (kind, arg) in enumerate(plan):
            codes.append(oracle.pack(rng.integers(0, arg, n).astype(np.uint32), oracle.code_bits(arg)))
            s = np.full(oracle.num_buckets(n, bucket), 0.01, dtype=F)
            s[::3] = F(1.5 * 2.0 ** 126)
            steps.append(s)
            workers.append((torch.from_numpy(codes[w]).cuda(), torch.from_numpy(s).cuda(),
                            ndq.NDQ_WORKER_DQ if kind == DQ else ndq.NDQ_WORKER_NESTED, arg, ndq.ndq_dither(7 + w, 3, w, 0)))
        ref = opipe.decode_chain(plan, bucket, n, codes, steps, ds, 1.0)
        assert np.isnan(ref).sum() > n // 100
        got = ndq.ndq_decode_chain(workers, n, bucket, 1.0).cpu().numpy()
        assert np.array_equal(got, ref, equal_nan=True), (plan, n, bucket, np.nonzero(~((got == ref) | (np.isnan(got) & np.isnan(ref))))[0][:5])


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return lr.build(tmp_path_factory.mktemp("recorder"))


@pytest.mark.parametrize("name", list(PLANS))
def test_plans_reach_the_streaming_kernel(recorder, name):
    plan = PLANS[name]
    workers = [{"codes": 0x20000000, "steps": 0x30000000, "kind": 0 if kind == DQ else 1, "levels_or_M": arg, "alpha": 1.0,
                "dither": [1, 2, 3, 0]} for kind, arg in plan]
    line = _tiles_from(plan)
    sizes = [1024 * (line - 1) + 1023, 1024 * line, 1024 * 12288]
    calls = [["ndq_decode_chain", workers, len(plan), n, 0, 1.0, 0x40000000, None] for n in sizes]
    calls.append(["ndq_decode_chain", [dict(w, alpha=0.9) for w in workers], len(plan), sizes[1], 0, 1.0, 0x40000000, None])
    got = lr.record(recorder, calls)
    # (eight DQSG workers of 3 bits and seven nested ones with such a ratio: persistent from 2,048 tiles on)
    for (rc, launches), form in zip(got, (2, 0 if name in ("8 and 5 of 3 bits", "3, M 3") else 1, 0)):
        assert rc == 0 and len(launches) == 1 and "chain_stream_kernel" in launches[0][0], launches
        assert launches[0][0].endswith("ELi%dEEEvNS_9ChainArgsE" % form), launches
    # a worker that shrinks: the general kernel
    assert ("chain_stream_kernel" in got[3][1][0][0]) == all(kind == DQ for kind, _ in plan)


@pytest.mark.parametrize("name,tiles,form", [("16", 8191, 2), ("16", 8192, 0), ("4, M 2", 8192, 0), ("2", 8192, 2), ("16, M 16", 20000, 2),
                                             ("5, M 3", 8191, 2), ("5, M 3", 8192, 0), ("1 of 8", 8192, 0)])
def test_form_for_buckets_of_a_row(recorder, name, tiles, form):
    workers = [{"codes": 0x20000000, "steps": 0x30000000, "kind": 0 if kind == DQ else 1, "levels_or_M": arg, "alpha": 1.0,
                "dither": [1, 2, 3, 0]} for kind, arg in ROW_PLANS[name]]
    (rc, launches), = lr.record(recorder, [["ndq_decode_chain", workers, len(workers), 1024 * tiles + 1, 512, 1.0, 0x40000000, None]])
    assert rc == 0 and len(launches) == 1 and launches[0][0].endswith("ELi%dEEEvNS_9ChainArgsE" % form), launches


# (the stream's block numbers go no further than 2^35 elements)
@pytest.mark.parametrize("n", [(1 << 35) - 2048, (1 << 35) - 2047, 1 << 35])
@pytest.mark.parametrize("name", ["2", "16, M 16", "16"])
def test_longest_vectors_with_buckets_of_a_row_fit_a_grid(recorder, name, n):
    workers = [{"codes": 0x20000000, "steps": 0x30000000, "kind": 0 if kind == DQ else 1, "levels_or_M": arg, "alpha": 1.0,
                "dither": [1, 2, 3, 0]} for kind, arg in ROW_PLANS[name]]
    (rc, launches), = lr.record(recorder, [["ndq_decode_chain", workers, len(workers), n, 512, 1.0, 0x40000000, None]])
    # (workgroups of 256 threads, fewer than 2^32 threads)
    assert rc == 0 and len(launches) == 1 and launches[0][1] * 256 < 1 << 32, launches


# (that their values match the oracle: test_gpu_chain_streaming.py and streaming_cases.py, every pair of widths)
@pytest.mark.parametrize("first,other", [(a, b) for a in (2, 4, 16) for b in (2, 4, 16) if a != b])
@pytest.mark.parametrize("others", [1, 2, 4])
def test_quantizers_of_two_widths_reach_the_streaming_kernel(recorder, first, other, others):
    workers = [{"codes": 0x20000000, "steps": 0x30000000, "kind": 0, "levels_or_M": arg, "alpha": 1.0, "dither": [1, 2, 3, 0]}
               for arg in [first] + [other] * others]
    sizes = [(512, 0), (1024 * 1024, 0), (1024 * 2048, 2048), (1024 * 12288, 0), (1024 * 12288 + 1, 1024), (1024 * 2048, 512)]
    calls = [["ndq_decode_chain", workers, len(workers), n, bucket, 1.0, 0x40000000, None] for n, bucket in sizes]
    calls.append(["ndq_decode_chain", workers + [dict(workers[0])], len(workers) + 1, 1024 * 2048, 0, 1.0, 0x40000000, None])   # the first width again
    got = lr.record(recorder, calls)
    short = others >= 3                               # (the kernel for short chains: four workers and more)
    for (n, bucket), (rc, launches), form in zip(sizes, got, (2, 2, 1, 0, 0)):
        assert rc == 0 and len(launches) == 1, launches
        if short and n == 512:
            assert "chain_short_kernel" in launches[0][0]
            continue
        assert "chain_stream_kernel" in launches[0][0] and launches[0][0].endswith("ELi%dEEEvNS_9ChainArgsE" % form), (n, launches)
    assert all(rc == 0 and len(launches) == 1 and "12chain_kernel" in launches[0][0] for rc, launches in got[5:]), got[5:]
