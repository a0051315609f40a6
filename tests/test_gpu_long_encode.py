"""Long binary32 vectors of several quantizers with one step each, which share an encoder launch: every mode and code
width that launch has, with steps of their own and with a shared one, on a length that ends in a ragged tile."""
import numpy as np
import pytest
import torch

import launch_recording as lr
import oracle
from paper_1904_01197_amd import ndq

F = np.float32
DQ, NESTED = ndq.NDQ_WORKER_DQ, ndq.NDQ_WORKER_NESTED
OWN = [(DQ, 2, 1.0), (DQ, 3, 1.0), (DQ, 5, 1.0), (DQ, 16, 1.0), (NESTED, 2, 0.9), (NESTED, 4, 1.0), (NESTED, 8, 1.0),
       (NESTED, 16, 1.0), (NESTED, 3, 1.0), (NESTED, 7, 1.0)]
SHARED = [(DQ, 16, 1.0), (DQ, 2, 1.0), (DQ, 3, 1.0), (DQ, 8, 1.0), (NESTED, 2, 1.0), (NESTED, 4, 0.9), (NESTED, 8, 1.0),
          (NESTED, 16, 1.0)]
CASES = [(OWN, False, 650 * 2048 + 77), (SHARED, True, 900 * 2048 + 2041), (OWN[:2], False, 4000 * 2048 + 1)]


@pytest.mark.gpu
@pytest.mark.parametrize("plan,shared,n", CASES)
def test_long_vectors_of_several_quantizers_match_oracle(plan, shared, n):
    rng = np.random.default_rng(n)
    common = rng.standard_normal(n, dtype=F)
    jobs, want, keep, step = [], [], [], None
    for w, (kind, arg, alpha) in enumerate(plan):
        g = (common + F(0.3) * rng.standard_normal(n, dtype=F)) * F(0.01)
        g[n - 3] = F(0.1 + 0.02 * w)                              # the maximum, in the ragged tile, its own per vector
        d_o, d_g = oracle.dither(w, 3, w, 8 * w), ndq.ndq_dither(w, 3, w, 8 * w)
        given = step if shared and w > 0 else 0.0
        ref = oracle.dq_encode(g, given, arg, 0, d_o) if kind == DQ else oracle.nested_encode(g, given, 16, arg, 0, d_o, alpha=alpha)
        step = float(ref[1][0]) if w == 0 else step
        want.append(ref)
        size = ndq.ndq_packed_bytes(n, ndq.ndq_code_bits(arg))
        keep.append((torch.full((size + 64,), 0xA5, dtype=torch.uint8, device="cuda"), torch.full((2,), -1.0, device="cuda"), size))
        jobs.append((torch.from_numpy(g).cuda(), kind, arg if kind == DQ else 16, 0 if kind == DQ else arg, alpha, d_g,
                     keep[w][0][:size], keep[w][1][:1], keep[0][1][:1] if shared and w > 0 else None))
    ndq.ndq_encode_workers(jobs, 0.0, 0)
    for w, ((c_ref, s_ref), (codes, steps, size)) in enumerate(zip(want, keep)):
        assert steps[0].item() == s_ref[0] and steps[1].item() == -1.0, w
        assert codes[:size].cpu().numpy().tobytes() == c_ref.tobytes(), w
        assert bool((codes[size:] == 0xA5).all()), w


def test_those_vectors_share_a_launch(tmp_path):
    recorder = lr.build(tmp_path)
    for plan, shared, n in CASES:
        jobs = [{"g": 0x10000000 + 0x4000000 * w, "codes_out": 0x80000000 + 0x1000000 * w, "steps_out": 0x60000000 + 0x10000 * w,
                 "step_in": 0x60000000 if shared and w else None, "kind": kind, "levels": arg if kind == DQ else 16,
                 "M": arg if kind == NESTED else 0, "alpha": alpha, "dither": [1, 2, 3, 0]}
                for w, (kind, arg, alpha) in enumerate(plan)]
        (rc, launches), = lr.record(recorder, [["ndq_encode_workers", jobs, len(jobs), 0, n, 0.0, 0, None]])
        encoders = [(name, y) for name, _, y in launches if "absmax" not in name]
        assert rc == 0 and len(encoders) == 1 and encoders[0][1] == len(plan), launches
        assert "encode_short_kernelILi0ELi4E" in encoders[0][0], launches
