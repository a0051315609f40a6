"""Short vectors of several quantizers in one encoder launch, and steps that the encoder's workgroups find
from their own copies of the max-norm pass's parts: every step and every byte against the oracle, on lengths
around whole tiles and workgroups, where the last share of the codes is shortest and around the lines to the
other kernels; nothing is written behind a stream."""
import numpy as np
import pytest
import torch

import launch_recording as lr
import oracle
from paper_1904_01197_amd import ndq, workloads

F = np.float32
DQ, NESTED = ndq.NDQ_WORKER_DQ, ndq.NDQ_WORKER_NESTED
PLANS = {                                                    # (kind, levels or M, alpha)
    "one": [(DQ, 3, 1.0)],
    "two": [(DQ, 8, 1.0), (NESTED, 4, 1.0)],
    "mixed": [(DQ, 5, 1.0), (DQ, 16, 1.0), (NESTED, 3, 1.0), (NESTED, 2, 0.9), (NESTED, 8, 1.0), (NESTED, 7, 1.0)],
    "narrow": [(DQ, 2, 1.0), (NESTED, 2, 1.0)],
    "wide": [(DQ, 16, 1.0), (NESTED, 100, 1.0)],             # a width that takes a launch per quantizer
    "sixteen": [(DQ, 3, 1.0)] * 9 + [(NESTED, 4, 1.0)] * 9,  # more than a launch holds
}


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name", list(PLANS))
@pytest.mark.parametrize("bucket,shared", [(0, False), (0, True), (512, False), (1024, False), (4096, False), (8192, False),
                                           (192, False), (2048, False)])
def test_short_vectors_match_oracle(dtype, name, bucket, shared):
    plan = PLANS[name]
    tile = 2048 if dtype == "f32" else 4096
    sizes = [1, 63, 512, tile, 4 * tile + 1, 5 * tile - 8, 9 * tile + 70, 33 * tile + 7, 131 * tile + 300]
    if name == "narrow" and bucket == 0:
        sizes += [813 * tile - 1700, 1024 * tile + 8, 1537 * tile]       # the last share, the copies and the tiles bound it
    for n in sizes:
        rng = np.random.default_rng(n)
        common = rng.standard_normal(n, dtype=F)
        jobs, want, keep = [], [], []
        first_step = None
        for w, (kind, arg, alpha) in enumerate(plan):
            x = (common + F(0.3) * rng.standard_normal(n, dtype=F)) * F(0.01)
            x[(7 * n) // 8] = F(0.2 + w)                                  # the maximum, near the end, its own per vector
            g = workloads.f32_to_bf16_bits(x) if dtype == "bf16" else x
            t = torch.from_numpy(g)
            g_d = (t.view(torch.bfloat16) if dtype == "bf16" else t).cuda()
            d_o, d_g = oracle.dither(w, 3, w, 8 * w), ndq.ndq_dither(w, 3, w, 8 * w)
            given = first_step if shared and w > 0 else 0.0
            if kind == DQ:
                ref = oracle.dq_encode(g, given, arg, bucket, d_o)
            else:
                ref = oracle.nested_encode(g, given, 16, arg, bucket, d_o, alpha=alpha)
            if w == 0:
                first_step = float(ref[1][0])
            want.append(ref)
            size = ndq.ndq_packed_bytes(n, ndq.ndq_code_bits(arg))
            codes = torch.full((size + 64,), 0xA5, dtype=torch.uint8, device="cuda")
            steps = torch.full((ref[1].size + 1,), -1.0, device="cuda")
            keep.append((codes, steps, size))
            jobs.append((g_d, kind, arg if kind == DQ else 16, 0 if kind == DQ else arg, alpha, d_g, codes[:size],
                         steps[:-1], keep[0][1][:-1] if shared and w > 0 else None))
        ndq.ndq_encode_workers(jobs, 0.0, bucket)
        for w, ((c_ref, s_ref), (codes, steps, size)) in enumerate(zip(want, keep)):
            assert np.array_equal(steps[:-1].cpu().numpy(), s_ref), (n, w)
            assert codes[:size].cpu().numpy().tobytes() == c_ref.tobytes(), (n, w)
            assert bool((codes[size:] == 0xA5).all()) and steps[-1].item() == -1.0, (n, w)


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return lr.build(tmp_path_factory.mktemp("recorder"))


def _jobs(plan, shared):
    return [{"g": 0x10000000 + 0x4000000 * w, "codes_out": 0x80000000 + 0x1000000 * w, "steps_out": 0x30000000 + 0x10000 * w,
             "step_in": 0x30000000 if shared and w else None, "kind": kind, "levels": arg if kind == 0 else 16,
             "M": arg if kind else 0, "alpha": 1.0, "dither": [1, 2, 3, 0]} for w, (kind, arg) in enumerate(plan)]


# launches of a call: m a max-norm kernel, an encoder's number of vectors
@pytest.mark.parametrize("plan,n,bucket,shared,expected", [
    ([(0, 3)], 65536, 0, False, "m1"), ([(0, 3)], 4096 * 2048 + 1, 0, False, "mm1"),
    ([(0, 8), (1, 4)], 1 << 20, 0, True, "m2"), ([(0, 8), (1, 4)], 1 << 20, 0, False, "m2"),
    ([(0, 16)] + [(1, 4)] * 15, 11173962, 0, True, "mm10"), ([(0, 16), (1, 100)], 70000, 0, False, "mm11"),
    ([(0, 5)] * 4 + [(1, 3)] * 4, 266610, 0, False, "m8"), ([(0, 5)] * 4 + [(1, 3)] * 4, 266610, 2048, False, "8"),
    ([(0, 5)] * 4 + [(1, 3)] * 4, 16384 * 256 + 1, 2048, False, "44"), ([(0, 5)] * 8, 266610, 1024, False, "8"),
    # three workgroups of the encoder for one of the max-norm pass; more than eight vectors that are handed a step
    ([(0, 3)], 1663370, 0, False, "m1"), ([(0, 3)], 2200000, 0, False, "mm1"), ([(0, 3)] * 4, 800000, 0, False, "m4"),
    ([(0, 3)] * 4, 1300000, 0, False, "mm4"), ([(0, 3)] * 4, 1 << 20, 0, False, "m4"), ([(0, 16)] * 8, 800000, 0, False, "mm8"),
    ([(0, 16)] + [(1, 4)] * 7, 266610, 0, True, "m8"), ([(0, 16)] + [(1, 4)] * 8, 266610, 0, True, "mm9")])
def test_launches_of_short_calls(recorder, plan, n, bucket, shared, expected):
    (rc, launches), = lr.record(recorder, [["ndq_encode_workers", _jobs(plan, shared), len(plan), 0, n, 0.0, bucket, None]])
    text = "".join("m" if "absmax" in name else "%x" % y for name, _, y in launches)
    assert rc == 0 and text == expected, launches


def test_copies_of_the_parts_stay_inside_every_share(recorder):
    # 4 bytes for each workgroup of the pass at the start of every encoder workgroup's codes; the last one's
    # share ends with the vector
    seen = 0
    for dt, tile in ((0, 2048), (1, 4096)):
        for levels, bits in ((2, 1), (3, 2), (5, 3), (16, 4)):
            sizes = [tile * k + d for k in (0, 1, 2, 3, 4, 5, 8, 9, 131, 203, 812, 1023, 1024, 2000) for d in (1, 64, 700, tile - 1)]
            calls = [["ndq_encode_workers", [_jobs([(0, levels)], False)[0]], 1, dt, n, 0.0, 0, None] for n in sizes]
            for n, (rc, launches) in zip(sizes, lr.record(recorder, calls)):
                assert rc == 0
                parts = [x for name, x, _ in launches if "absmax_copies" in name]
                if not parts:
                    continue
                seen += 1
                tiles = -(-n // tile)
                groups = -(-tiles // 4)
                assert [x for name, x, _ in launches if "encode_short" in name] == [groups]
                first = (groups - 1) * (tiles // groups) + min(groups - 1, tiles % groups)
                assert parts[0] <= 256 and 4 * parts[0] <= oracle.packed_bytes(n, bits) - first * tile // 8 * bits, n
    assert seen > 200


@pytest.mark.gpu
def test_a_short_iteration_replayed_from_a_graph():
    # copies of the parts, encoders of all quantizers and the short chain, with eager work between the replays
    plan, n = [(DQ, 8), (NESTED, 4), (NESTED, 3)], 70001
    gen = torch.Generator(device="cuda").manual_seed(5)
    grads = [torch.empty(n, device="cuda") for _ in plan]
    codes = [torch.empty(ndq.ndq_packed_bytes(n, ndq.ndq_code_bits(arg)), dtype=torch.uint8, device="cuda") for _, arg in plan]
    steps = [torch.empty(1, device="cuda") for _ in plan]
    out = torch.empty(n, device="cuda")
    ds = [ndq.ndq_dither(w, 1, w, 0) for w in range(3)]

    def iteration():
        ndq.ndq_encode_workers([(grads[w], kind, arg if kind == DQ else 16, 0 if kind == DQ else arg, 1.0, ds[w], codes[w],
                                 steps[w], steps[0] if w else None) for w, (kind, arg) in enumerate(plan)], 0.0, 0)
        ndq.ndq_decode_chain([(codes[w], steps[w], kind, arg, ds[w]) for w, (kind, arg) in enumerate(plan)], n, 0, 0.5, out)

    def draw():
        for g in grads:
            g.copy_(torch.randn(n, device="cuda", generator=gen))

    draw()
    iteration()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        iteration()
    for _ in range(4):
        draw()
        iteration()
        torch.cuda.synchronize()
        want = [t.clone() for t in codes + steps + [out]]
        for t in codes + steps + [out]:
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(codes + steps + [out], want))
