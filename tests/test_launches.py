"""Properties of the launches a call makes that need no GPU to check: how much scratch
they use, their order, and that a refused call makes none."""
import pytest

import launch_recording as lr
import oracle


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return lr.build(tmp_path_factory.mktemp("recorder"))


D = {"dither": [1, 2, 3, 0]}


def _job(**kw):
    base = {"g": 0x10000000, "codes_out": 0x20000000, "steps_out": 0x30000000, "step_in": None, "kind": 0,
            "levels": 2, "M": 0, "alpha": 1.0, "dither": [1, 2, 3, 0]}
    base.update(kw)
    return base


@pytest.mark.parametrize("dt", [0, 1])
def test_the_max_norm_pass_keeps_its_parts_inside_the_code_stream(recorder, dt):
    # one float per workgroup of absmax_span_kernel lies in codes_out until the encoder overwrites it;
    # the tightest streams: 1-bit codes, vectors much shorter than their one bucket, ragged last buckets
    cases = [(n, bucket, W) for bucket in (0, 65536, 1 << 17, 1 << 20, 1 << 24, 1 << 31)
             for n in (1, 64, 1000, 4097, 5000, 16 * 4096 - 64, 65535, 65537, 70000, 131073, 400001)
             for W in (1, 3, 16)]
    calls = []
    for n, bucket, W in cases:
        if W == 1:
            calls.append(["ndq_dq_encode", 0x10000000, dt, n, 0.0, 2, bucket, D, 0x20000000, 0x30000000, None])
        else:
            jobs = [_job(codes_out=0x20000000 + 0x100000 * w, steps_out=0x30000000 + 0x1000 * w) for w in range(W)]
            calls.append(["ndq_encode_workers", jobs, W, dt, n, 0.0, bucket, None])
    spans = 0
    for (n, bucket, W), (rc, launches) in zip(cases, lr.record(recorder, calls)):
        assert rc == 0
        if not any("absmax_finish" in name for name, _, _ in launches):
            continue                                  # atomics: no parts
        for name, x, _ in launches:
            if "absmax_span" in name:
                spans += 1
                assert 4 * x <= oracle.packed_bytes(n, 1), (n, bucket, W, x)
    assert spans > 20                                 # (the sizes do reach that form)


def _kinds(launches):
    """A letter per launch: the max-norm pass (any of its kernels: m), an encoder (its number of vectors)."""
    text = ""
    for name, _, y in launches:
        if "absmax" in name or "fill_zero" in name:
            text += "" if text.endswith("m") else "m"
        else:
            assert "encode" in name
            text += str(y)
    return text


# steps of the workers: S[w]; a worker is (its steps_out, the step it is handed or None)
ORDERS = [
    # every worker handed the first one's step, which a max-norm pass finds: one batch
    ([(0, None), (1, 0), (2, 0)], 0.0, "m12"),
    # the same where every worker keeps it in place
    ([(0, None), (0, 0), (0, 0)], 0.0, "m12"),
    # a preset step is there only after its worker's encoder
    ([(0, None), (1, 0), (2, 0)], 0.5, "12"),
    # handed over along a chain
    ([(0, None), (1, 0), (2, 1)], 0.0, "m111"),
    # a LATER worker writes over the step an earlier one was handed: by its max-norm pass, by its encoder
    ([(1, 0), (0, None)], 0.0, "1m1"),
    ([(1, 0), (0, None)], 0.5, "11"),
    ([(2, 3), (1, 0), (0, 3)], 0.0, "21"),
    # two workers leave their steps in the same place
    ([(0, None), (0, None), (1, 0)], 0.0, "m1m11"),
    ([(0, None), (0, None)], 0.5, "11"),
]


@pytest.mark.parametrize("workers,preset,expected", ORDERS)
def test_workers_that_share_a_step_are_launched_in_the_order_given(recorder, workers, preset, expected):
    for n in (1000, 70000):
        jobs = [_job(codes_out=0x20000000 + 0x100000 * w, levels=16, steps_out=0x30000000 + 4 * out,
                     step_in=None if handed is None else 0x30000000 + 4 * handed)
                for w, (out, handed) in enumerate(workers)]
        (rc, launches), = lr.record(recorder, [["ndq_encode_workers", jobs, len(jobs), 0, n, preset, 0, None]])
        assert rc == 0 and _kinds(launches) == expected, launches


# byte offsets of out and of the reconstructions; n = 1000 floats are 4,000 bytes
@pytest.mark.parametrize("out,decoded,accepted", [
    (0, [4000], True), (0, [0], True), (4000, [0, 8000, 12000], True), (8000, [0, 8000, 12000], True),
    (0, [4000, 4000], True), (0, [3984], False), (3984, [0], False), (16000, [0, 8000, 11984], False),
    (8016, [0, 8000, 12000], False), (0, [4000 * (w + 1) for w in range(33)], True),
    (4000 * 7, [4000 * (w + 1) for w in range(33)], False), (4000 * 32, [4000 * w for w in range(32)], True),
    (4000 * 34, [4000 * w for w in range(32)] + [4000 * 32 - 16], False)])
def test_the_mean_refuses_vectors_that_overlap_by_a_part(recorder, out, decoded, accepted):
    base = 0x10000000
    workers = [{"codes": 0x20000000, "steps": 0x30000000, "kind": 0, "levels_or_M": 4, "alpha": 1.0,
                "dither": [1, 2, 3, 0]}] * len(decoded)
    (rc, launches), = lr.record(recorder, [["ndq_decode_mean", workers, [base + x for x in decoded], len(decoded), 1000,
                                            0, 1.0, base + out, None]])
    assert rc == (0 if accepted else -1) and len(launches) == ((len(decoded) + 31) // 32 if accepted else 0)


# form of the chain decoder: 0 persistent, 1 one tile (two rows) per wave, 2 one row per wave; lines in
# tiles of 1,024 elements (6,144 wave slots), DQSG workers and nested ones
@pytest.mark.parametrize("dq,nested,lines", [
    (1, 0, [(2047, 2), (2048, 0)]), (2, 0, [(2047, 2), (2048, 1), (6143, 1), (6144, 0)]),
    (3, 0, [(6143, 1), (6144, 0), (6527, 0), (6528, 1), (9215, 1), (9216, 0)]),
    (7, 0, [(6528, 1), (9216, 0)]), (8, 0, [(6143, 1), (6144, 0), (7000, 0)]),
    (1, 1, [(2048, 1), (6144, 0), (6528, 1), (12287, 1), (12288, 0)]), (1, 2, [(12287, 1), (12288, 0)]),
    (1, 3, [(6143, 1), (6144, 0), (7000, 0)]), (1, 7, [(2047, 2), (2048, 0)]), (1, 31, [(2047, 2), (2048, 0)])])
def test_form_of_the_chain_decoder(recorder, dq, nested, lines):
    worker = {"codes": 0x20000000, "steps": 0x30000000, "kind": 0, "levels_or_M": 16, "alpha": 1.0,
              "dither": [1, 2, 3, 0]}
    workers = [worker] * dq + [dict(worker, kind=1, levels_or_M=4)] * nested
    calls = [["ndq_decode_chain", workers, len(workers), 1024 * tiles + 1023, 0, 1.0, 0x40000000, None]
             for tiles, _ in lines]
    for (tiles, form), (rc, launches) in zip(lines, lr.record(recorder, calls)):
        assert rc == 0 and len(launches) == 1
        assert launches[0][0].startswith("_ZN3ndq19chain_stream_kernel"), launches
        assert launches[0][0].endswith("ELi%dEEEvNS_9ChainArgsE" % form), (tiles, form, launches)


def test_a_streaming_threshold_from_the_environment_reaches_the_persistent_encoder(recorder):
    # the calls streaming_cases.py makes with bfloat16 vectors in buckets of a tile, and sixteen vectors in a call
    tile, calls = 4096, []
    for n in (12 * tile, 37 * tile + 100, 121 * tile + 64, 3 * tile + 8):
        for kind, levels, M in ((0, 2, 0), (0, 4, 0), (0, 16, 0), (1, 4, 2), (1, 16, 4), (1, 64, 16)):
            jobs = [_job(kind=kind, levels=levels, M=M, codes_out=0x20000000 + 0x1000000 * w,
                         steps_out=0x30000000 + 0x10000 * w) for w in range(16)]
            calls += [["ndq_encode_workers", jobs[:W], W, 1, n, 0.0, tile, None] for W in (1, 16)]
    # (more than one quantizer)
    mixed = [_job(levels=16), _job(kind=1, levels=16, M=4, codes_out=0x28000000, steps_out=0x38000000)]
    calls.append(["ndq_encode_workers", mixed, 2, 1, 37 * tile + 100, 0.0, tile, None])
    env = {"NDQ_STREAM_MIN_TILES_PER_WAVE": "0", "NDQ_STREAM_MAX_BLOCKS": "3"}
    for call, (rc, launches) in zip(calls, lr.record(recorder, calls, env)):
        encoders = [(name, x) for name, x, _ in launches if "absmax" not in name and "fill_zero" not in name]
        assert rc == 0 and encoders and all("encode_stream_kernel" in name and x <= 3 for name, x in encoders), (call, launches)


# longest vector that the kernel for short chains takes, by its plan: (kind, levels or M) of every worker
@pytest.mark.parametrize("plan,most", [
    ([(0, 16)] * 3, 0), ([(0, 16), (1, 4)], 0), ([(0, 16)] * 4, 245760), ([(0, 4)] + [(1, 2)] * 7, 294912),
    ([(0, 16)] + [(1, 4)] * 15, 393216), ([(0, 16)] * 32, 393216), ([(0, 5)], 0),
    # the rarer plans of the streaming kernel
    ([(0, 8), (1, 4)], 131072), ([(0, 5)] * 2, 131072), ([(0, 16)] * 2 + [(1, 4)], 262144), ([(0, 5)] * 2 + [(1, 3)] * 2, 393216),
    ([(0, 5)] * 7, 393216), ([(0, 5)] * 8, 655360), ([(0, 16)] * 8 + [(1, 4)] * 8, 393216), ([(0, 16)] * 8 + [(1, 8)] * 3, 393216),
    ([(0, 16)] * 8 + [(1, 8)] * 4, 786432), ([(0, 5)] + [(1, 3)] * 15, 655360), ([(0, 5)] * 17, 393216), ([(0, 8)] + [(1, 8)] * 31, 393216),
    # and those of the general kernel
    ([(0, 100), (1, 4)], 393216), ([(0, 32)] * 2 + [(1, 3)] * 2, 655360), ([(0, 32)] * 5, 786432), ([(0, 16)] * 8 + [(1, 4)] * 7 + [(1, 2)], 917504),
    ([(0, 8)] + [(1, 8)] * 30 + [(1, 2)], 786432)])
def test_longest_vector_of_the_short_chain_kernel(recorder, plan, most):
    workers = [{"codes": 0x20000000, "steps": 0x30000000, "kind": kind, "levels_or_M": arg, "alpha": 1.0,
                "dither": [1, 2, 3, 0]} for kind, arg in plan]
    sizes = [most, most + 1] if most else [1, 512, 65536]
    calls = [["ndq_decode_chain", workers, len(workers), n, 0, 1.0, 0x40000000, None] for n in sizes]
    for n, (rc, launches) in zip(sizes, lr.record(recorder, calls)):
        assert rc == 0 and len(launches) == 1
        assert ("chain_short_kernel" in launches[0][0]) == (n <= most), (n, launches)


@pytest.mark.parametrize("dt,M,bucket,width", [(1, 3, 64, 0), (1, 3, 448, 0), (1, 3, 512, 2), (1, 3, 4096, 2), (1, 7, 64, 3), (0, 3, 64, 2),
                                               (1, 4, 64, 2)])
def test_encoders_that_know_their_code_width(recorder, dt, M, bucket, width):
    call = ["ndq_nested_encode", 0x10000000, dt, 100000, 0.0, 16, M, 1.0, bucket, D, 0x20000000, 0x30000000, None]
    (rc, launches), = lr.record(recorder, [call])
    assert rc == 0 and len(launches) == 1
    assert ("ELi%dEEEvNS_11EncodeBatch" % width) in launches[0][0], launches


# (counting workgroups of 1- and 2-bit codes take 8,192 vectors of 16 bytes at a time; from 160 of them on a launch of its own clears the bins)
@pytest.mark.parametrize("bits,n,kernels,grid", [
    (1, 159 * 8192 * 128, 1, 160), (1, 159 * 8192 * 128 + 128, 2, 160), (2, 159 * 8192 * 64, 1, 160), (2, 159 * 8192 * 64 + 64, 2, 160),
    (2, 1500000000, 2, 256), (4, 1500000000, 1, 257), (2, 8192 * 64, 1, 1), (2, 8192 * 64 + 64, 1, 3)])
def test_launches_of_the_entropy(recorder, bits, n, kernels, grid):
    (rc, launches), = lr.record(recorder, [["ndq_code_entropy", 0x10000000, n, bits, 0x20000000, 0x30000000, None]])
    assert rc == 0 and len(launches) == kernels and launches[-1][1] == grid, launches
    assert kernels == 1 or "clear_histogram" in launches[0][0]


@pytest.mark.parametrize("plan,bucket", [([(0, 8), (1, 4)], 0), ([(0, 5)] * 4 + [(1, 3)] * 4, 0), ([(0, 16)] * 8 + [(1, 8)] * 8, 1024),
                                         ([(0, 16)] * 2 + [(1, 4)] * 2, 512), ([(0, 8)] * 5, 512), ([(0, 16)] + [(1, 7)], 512)])
def test_a_streaming_threshold_from_the_environment_reaches_the_persistent_chain_decoder(recorder, plan, bucket):
    workers = [{"codes": 0x20000000, "steps": 0x30000000, "kind": kind, "levels_or_M": arg, "alpha": 1.0, "dither": [1, 2, 3, 0]}
               for kind, arg in plan]
    calls = [["ndq_decode_chain", workers, len(workers), n, bucket, 1.0, 0x40000000, None] for n in (1025, 12 * 1024, 40 * 1024 + 7)]
    for rc, launches in lr.record(recorder, calls, {"NDQ_STREAM_MIN_TILES_PER_WAVE": "0", "NDQ_STREAM_MAX_BLOCKS": "3"}):
        assert rc == 0 and len(launches) == 1 and launches[0][1] <= 3, launches
        assert "chain_stream_kernel" in launches[0][0] and launches[0][0].endswith("ELi0EEEvNS_9ChainArgsE"), launches


@pytest.mark.parametrize("plan,bucket,name", [
    ([(0, 32)] * 2, 0, "ILb0ELb0ELi2E"), ([(0, 100), (1, 64)], 2048, "ILb0ELb0ELi2E"), ([(0, 32), (1, 32)], 512, "ILb1ELb0ELi2E"),
    ([(0, 32)] * 3, 512, "ILb1ELb1ELi2E"),
    ([(0, 32), (1, 3)], 0, "ILb0ELb1ELi2E"), ([(0, 32)] * 3, 0, "ILb0ELb1ELi2E"), ([(0, 32)] * 34, 0, "ILb0ELb1ELi2E")])
def test_forms_of_the_general_chain_kernel(recorder, plan, bucket, name):
    workers = [{"codes": 0x20000000, "steps": 0x30000000, "kind": kind, "levels_or_M": arg, "alpha": 1.0, "dither": [1, 2, 3, 0]}
               for kind, arg in plan]
    (rc, launches), = lr.record(recorder, [["ndq_decode_chain", workers, len(workers), 6600000, bucket, 1.0, 0x40000000, None]])
    assert rc == 0 and ("chain_kernel" + name) in launches[0][0], launches


@pytest.mark.parametrize("last,name", [([(0, 32), (1, 4)], "ILb0ELb0ELi2E"), ([(1, 4), (0, 32)], "ILb0ELb0ELi2E"), ([(1, 3), (0, 32)], "ILb0ELb1ELi2E"),
                                       ([(0, 32), (1, 3)], "ILb0ELb1ELi2E"), ([(1, 4, 0.9), (1, 4)], "ILb0ELb1ELi2E"), ([(1, 4), (1, 4, 0.9)], "ILb0ELb1ELi2E")])
def test_the_last_two_of_34_workers(recorder, last, name):
    # the second launch of a call begins with any worker
    workers = [{"codes": 0x20000000, "steps": 0x30000000, "kind": w[0], "levels_or_M": w[1], "alpha": w[2] if len(w) > 2 else 1.0,
                "dither": [1, 2, 3, 0]} for w in [(0, 32)] * 32 + last]
    (rc, launches), = lr.record(recorder, [["ndq_decode_chain", workers, 34, 6600000, 0, 1.0, 0x40000000, None]])
    assert rc == 0 and len(launches) == 2 and ("chain_kernel" + name) in launches[1][0], launches
