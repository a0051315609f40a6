"""Calls whose workgroups meet in memory that nobody has cleared: the histogram with its entropy and the sum
of squared differences.  Whatever lies in the results and the workspace, in eager calls and in replays of a
graph, on one stream and on several; and the collector that gives up waiting."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_1904_01197_amd import ndq

pytestmark = pytest.mark.gpu
# codes: one workgroup, two, an uneven share, a full grid
SIZES = [1, 31, 60001, 32 * 1024, 32 * 1024 + 32, (1 << 20) + 64, 3000001, 32 * 1024 * 256 + 63]


def _stream(bits, n, seed=0):
    rng = np.random.default_rng(seed + n + bits)
    codes = np.minimum(rng.geometric(0.4, size=n) - 1, (1 << bits) - 1).astype(np.uint32)
    return torch.from_numpy(oracle.pack(codes, bits)).cuda(), np.bincount(codes, minlength=1 << bits)


def _entropy(counts):
    p = counts[counts > 0] / counts.sum()
    return float(-(p * np.log2(p)).sum())


@pytest.mark.parametrize("bits", range(1, 9))
def test_histogram_into_memory_that_holds_anything(bits):
    rng = np.random.default_rng(bits)
    for n in SIZES:
        packed, ref = _stream(bits, n)
        hist = torch.empty(1 << bits, dtype=torch.int64, device="cuda")
        ent = torch.empty(1, dtype=torch.float64, device="cuda")
        # zeros, ones, any bits, then twice over the call's own results
        for fill in (np.int64(0), np.int64(-1), None, "own", "own"):
            if fill is None:
                hist.copy_(torch.from_numpy(rng.integers(-2**63, 2**63 - 1, hist.numel())))
                ent.view(torch.int64).copy_(torch.from_numpy(rng.integers(-2**63, 2**63 - 1, 1)))
            elif not isinstance(fill, str):
                hist.fill_(int(fill))
                ent.view(torch.int64).fill_(int(fill))
            ndq.ndq_code_entropy(packed, n, bits, hist, ent)
            assert np.array_equal(hist.cpu().numpy(), ref), (n, fill)
            # (at most 256 terms, each to a few units in the last place)
            assert abs(float(ent.item()) - _entropy(ref)) <= 1e-12, (n, fill)


@pytest.mark.parametrize("bits,n", [(1, 160 * 8192 * 128 + 77), (1, 400000007), (2, 159 * 8192 * 64 - 5), (2, 160 * 8192 * 64 + 31), (2, 200000003)])
def test_histogram_of_long_streams(bits, n):
    # (both ways of clearing the bins; eager, then replays that find their own results)
    gen = torch.Generator(device="cuda").manual_seed(n)
    packed = torch.randint(0, 256, (ndq.ndq_packed_bytes(n, bits),), dtype=torch.uint8, device="cuda", generator=gen)
    hist = torch.full((1 << bits,), -7, dtype=torch.int64, device="cuda")
    ent = torch.full((1,), -7.0, dtype=torch.float64, device="cuda")
    per, whole = 8 // bits, n * bits // 8
    ndq.ndq_code_entropy(packed, n, bits, hist, ent)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ndq.ndq_code_entropy(packed, n, bits, hist, ent)
    for rep in range(4):
        if rep:
            packed.bitwise_and_(torch.randint(0, 256, packed.shape, dtype=torch.uint8, device="cuda", generator=gen))
            torch.cuda.synchronize()
            graph.replay()
        torch.cuda.synchronize()
        bytes_ = torch.bincount(packed[:whole], minlength=256).cpu().numpy()
        ref = np.zeros(1 << bits, dtype=np.int64)
        for byte, count in enumerate(bytes_):
            for k in range(per):
                ref[byte >> k * bits & (1 << bits) - 1] += count
        for k in range(n - whole * per):
            ref[int(packed[whole]) >> k * bits & (1 << bits) - 1] += 1
        assert np.array_equal(hist.cpu().numpy(), ref), (n, rep)
        assert abs(float(ent.item()) - _entropy(ref)) <= 1e-12, (n, rep)


def test_histograms_of_several_streams_at_once():
    streams = [torch.cuda.Stream() for _ in range(4)]
    calls = [(bits, n) + _stream(bits, n, seed=s) for s, (bits, n) in
             enumerate([(4, 3000001), (2, 30000001), (7, 4000000), (3, 70001), (1, 60000001), (8, 2000000), (5, 33000), (4, 9000000)])]
    out = [(torch.full((1 << bits,), -5, device="cuda", dtype=torch.int64), torch.full((1,), 3.0, device="cuda", dtype=torch.float64))
           for bits, *_ in calls]
    torch.cuda.synchronize()
    for _ in range(20):
        for i, (bits, n, packed, _) in enumerate(calls):
            with torch.cuda.stream(streams[i % 4]):
                ndq.ndq_code_entropy(packed, n, bits, *out[i])
    torch.cuda.synchronize()
    for (bits, n, _, ref), (hist, ent) in zip(calls, out):
        assert np.array_equal(hist.cpu().numpy(), ref) and abs(float(ent.item()) - _entropy(ref)) <= 1e-12


def test_replays_of_a_graph_follow_their_inputs():
    n = 1000003
    streams = {bits: _stream(bits, n) for bits in (1, 4, 7)}
    packed = {bits: s[0] for bits, s in streams.items()}
    hist = {bits: torch.empty(1 << bits, dtype=torch.int64, device="cuda") for bits in packed}
    ent = {bits: torch.empty(1, dtype=torch.float64, device="cuda") for bits in packed}
    a, b = torch.randn(n, device="cuda"), torch.randn(n, device="cuda")
    work = torch.empty(ndq.ndq_sqdiff_workspace() // 8, dtype=torch.float64, device="cuda")
    sq = torch.empty(1, dtype=torch.float64, device="cuda")

    def run():
        for bits in packed:
            ndq.ndq_code_entropy(packed[bits], n, bits, hist[bits], ent[bits])
        ndq.ndq_sqdiff(a, b, work, sq)

    run()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    for rep in range(4):
        refs = {}
        for bits in packed:                         # (nothing is overwritten: each replay finds the last one's results)
            new, refs[bits] = _stream(bits, n, seed=10 * (rep + 1))
            packed[bits].copy_(new)
        a.copy_(torch.randn(n, device="cuda") * (rep + 1))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for bits in packed:
            assert np.array_equal(hist[bits].cpu().numpy(), refs[bits]), (rep, bits)
            assert abs(float(ent[bits].item()) - _entropy(refs[bits])) <= 1e-12, (rep, bits)
        replayed = sq.clone()
        ndq.ndq_sqdiff(a, b, work, sq)
        assert torch.equal(replayed, sq), rep


def _sqdiff_cases():
    """-> for some lengths the sum from workspaces that hold anything, its bits as text"""
    got = []
    for n in (1, 3, 2047, 4 * 512 * 512, 1000003, 11173962):
        gen = torch.Generator(device="cuda").manual_seed(n)
        a, b = torch.randn(n, device="cuda", generator=gen), torch.randn(n, device="cuda", generator=gen)
        ref = float((a.double() - b.double()).square().sum().item())
        work = torch.empty(ndq.ndq_sqdiff_workspace() // 8 + 1, dtype=torch.float64, device="cuda")
        sums = []
        for fill in (0, -1, None):
            if fill is None:
                work.view(torch.int64).random_(-2**62, 2**62, generator=gen)
            else:
                work.view(torch.int64).fill_(fill)
            sums.append(ndq.ndq_sqdiff(a, b, work[:-1]).clone())
            inside = work[fill:][:1] if fill == 0 else work[77:78]         # a result that lies in the workspace
            sums.append(ndq.ndq_sqdiff(a, b, work[1:] if n % 2 else work[:-1], inside).clone())
        for s in sums:
            assert abs(float(s.item()) - ref) <= n * 2.0 ** -52 * ref, n
            assert torch.equal(s, sums[0]), n
        got.append(float(sums[0].item()).hex())
    return got


def test_squared_differences_with_and_without_a_patient_collector():
    here = _sqdiff_cases()
    code = "import sys; sys.path.insert(0, %r); import test_gpu_one_launch as t; print('SUMS', *t._sqdiff_cases())" % os.path.dirname(__file__)
    res = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, NDQ_COLLECT_POLLS="0", PYTHONPATH=os.pathsep.join(sys.path)),
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:]
    assert res.stdout.split("SUMS")[1].split() == here


def _impatient_replays():
    """A collector that looks once or never: replays of a call with other inputs, and what the call leaves in the workspace."""
    for n in (5, 3000, 4 * 512 * 512, 1000003, 11173962):
        a, b = torch.zeros(n, device="cuda"), torch.randn(n, device="cuda")
        slots = torch.empty(ndq.ndq_sqdiff_workspace() // 8, dtype=torch.int64, device="cuda").random_(-2**62, 2**62)
        work = slots.view(torch.float64)
        for inside in (None, 78, 79):                # (a result in the workspace; else its last slot is not used)
            out = torch.empty(1, dtype=torch.float64, device="cuda") if inside is None else work[inside:inside + 1]
            ndq.ndq_sqdiff(a, b, work, out)
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                ndq.ndq_sqdiff(a, b, work, out)
            unused = slice(1022, 1024) if inside is None else slice(78, 80)
            for rep in range(8):
                print("replay", n, inside, rep, flush=True)
                a.copy_(torch.randn(n, device="cuda") * (rep + 1))
                torch.cuda.synchronize()
                graph.replay()
                torch.cuda.synchronize()
                got, left = float(out.item()), slots.clone()
                ref = float((a.double() - b.double()).square().sum().item())
                assert abs(got - ref) <= n * 2.0 ** -52 * ref, (n, inside, rep, got, ref)
                left[unused] = 0
                assert not bool(left.any()), (n, inside, rep, int((left != 0).sum()))


@pytest.mark.parametrize("polls", ["0", "1", "3"])
def test_replays_after_a_collector_that_gave_up(polls):
    code = "import sys; sys.path.insert(0, %r); import test_gpu_one_launch as t; t._impatient_replays(); print('REPLAYS_OK')" % os.path.dirname(__file__)
    res = subprocess.run([sys.executable, "-u", "-c", code], env=dict(os.environ, NDQ_COLLECT_POLLS=polls, PYTHONPATH=os.pathsep.join(sys.path)),
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=100)
    assert res.returncode == 0 and "REPLAYS_OK" in res.stdout, res.stdout[-1500:]
