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
