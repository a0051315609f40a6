"""Calls that take several workers at once, against the oracle: codes and steps bit for bit
(they are defined by the same IEEE operations on both sides, so there is no tolerance)."""
import numpy as np
import pytest
import torch

import oracle
from oracle import pipeline as opipe
from paper_1904_01197_amd import ndq, workloads

pytestmark = pytest.mark.gpu

F = np.float32


def _host(W, n, dtype, seed):
    rng = np.random.default_rng(seed)
    common = rng.standard_normal(n) * 0.01
    out = [(common + rng.standard_normal(n) * 0.003).astype(F) for _ in range(W)]
    return [workloads.f32_to_bf16_bits(x) for x in out] if dtype == "bf16" else out


def _dev(g):
    t = torch.from_numpy(g)
    return (t.view(torch.bfloat16) if g.dtype == np.uint16 else t).cuda()


def _encode(plan, fine, bucket, shared, host, seeds, preset=0.0):
    n = host[0].size
    codes = [torch.full((ndq.ndq_packed_bytes(n, ndq.ndq_code_bits(arg)) + 64,), 0xA5, dtype=torch.uint8,
                        device="cuda") for _, arg in plan]
    steps = [torch.full((ndq.ndq_num_buckets(n, bucket),), -1.0, device="cuda") for _ in plan]
    jobs = []
    for w, (kind, arg) in enumerate(plan):
        step_in = steps[0] if shared and w > 0 else None
        d = ndq.ndq_dither(seeds[w], 3, w, 0)
        jobs.append((_dev(host[w]), ndq.NDQ_WORKER_DQ if kind == "dq" else ndq.NDQ_WORKER_NESTED,
                     arg if kind == "dq" else fine, arg, 1.0, d, codes[w], steps[w], step_in))
    ndq.ndq_encode_workers(jobs, preset, bucket)
    return codes, steps


def _compare(plan, fine, bucket, shared, host, preset=0.0):
    n = host[0].size
    seeds = [7 + w for w in range(len(plan))]
    ds = opipe.dithers(len(plan), seeds, step=3)
    c_ref, s_ref, _ = opipe.encode_all(plan, fine, bucket, shared, host, ds, preset)
    codes, steps = _encode(plan, fine, bucket, shared, host, seeds, preset)
    for w in range(len(plan)):
        got = codes[w].cpu().numpy()
        assert np.array_equal(steps[w].cpu().numpy(), s_ref[w]), (n, bucket, w)
        assert got[:c_ref[w].size].tobytes() == c_ref[w].tobytes(), (n, bucket, w)
        assert (got[c_ref[w].size:] == 0xA5).all(), "written past the stream"


# tile edges (2,048 binary32 / 4,096 bfloat16 elements), the length from which the max-norm
# pass leaves parts instead of using atomics (16 tiles), and more than one workgroup of parts
SIZES = [1, 2047, 2049, 4097, 16 * 2048 - 1, 16 * 4096 + 1, 70001, 300007]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("bucket,shared", [(0, False), (0, True), (1024, False), (4096, False), (8192, False),
                                           (6400, False), (32768, False)])
def test_several_workers_in_one_call_match_oracle(dtype, bucket, shared):
    plan = (("dq", 5), ("nested", 3), ("dq", 5), ("nested", 4), ("dq", 16), ("nested", 4))
    for n in SIZES:
        _compare(plan, 7, bucket, shared, _host(len(plan), n, dtype, n))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_vectors_much_shorter_than_their_bucket_stay_inside_their_streams(dtype):
    # the max-norm pass keeps its parts in the code stream: 1-bit codes are the least memory there is
    guard = 1 << 14
    for n, bucket in ((64, 65536), (1000, 1 << 20), (5000, 1 << 24), (16 * 4096 + 5, 1 << 17), (65600, 1 << 20)):
        host = _host(3, n, dtype, n)
        size = ndq.ndq_packed_bytes(n, 1)
        for together in (False, True):
            codes = [torch.full((size + guard,), 0xA5, dtype=torch.uint8, device="cuda") for _ in host]
            steps = [torch.full((1,), -1.0, device="cuda") for _ in host]
            ds = [ndq.ndq_dither(7 + w, 3, w, 0) for w in range(3)]
            if together:
                ndq.ndq_encode_workers([(_dev(host[w]), ndq.NDQ_WORKER_DQ, 2, 0, 1.0, ds[w], codes[w], steps[w], None)
                                        for w in range(3)], 0.0, bucket)
            else:
                for w in range(3):
                    ndq.ndq_dq_encode(_dev(host[w]), 0.0, 2, bucket, ds[w], codes[w], steps[w])
            for w in range(3):
                ref, s_ref = oracle.dq_encode(host[w], 0.0, 2, bucket, oracle.dither(7 + w, 3, w))
                got = codes[w].cpu().numpy()
                assert steps[w].item() == s_ref[0], (n, bucket, w)
                assert got[:size].tobytes() == ref.tobytes(), (n, bucket, w)
                assert (got[size:] == 0xA5).all(), "written past the stream"


@pytest.mark.parametrize("preset", [0.0, 0.004])
def test_more_workers_than_one_launch_holds_and_a_step_from_an_earlier_worker(preset):
    # preset: the shared step exists only after the first worker's encoder, not after a max-norm pass
    W = 35
    plan = (("dq", 16),) + (("nested", 4),) * (W - 1)
    host = _host(W, 5000, "f32", 1)
    if preset == 0.0:
        _compare(plan, 16, 0, True, host)
        return
    n, seeds = 5000, list(range(W))
    codes = [torch.empty(ndq.ndq_packed_bytes(n, 4), dtype=torch.uint8, device="cuda") for _ in plan]
    steps = [torch.full((1,), -1.0, device="cuda") for _ in plan]
    jobs = [(_dev(host[w]), ndq.NDQ_WORKER_DQ if w == 0 else ndq.NDQ_WORKER_NESTED, 16, 4, 1.0,
             ndq.ndq_dither(seeds[w], 3, w, 0), codes[w], steps[w], steps[w - 1] if w % 3 else None)
            for w in range(W)]
    ndq.ndq_encode_workers(jobs, preset, 0)
    for w in range(W):
        d = oracle.dither(seeds[w], 3, w)
        ref, s_ref = (oracle.dq_encode(host[w], preset, 16, 0, d) if w == 0
                      else oracle.nested_encode(host[w], preset, 16, 4, 0, d))
        assert steps[w].item() == s_ref[0]
        assert codes[w].cpu().numpy()[:ref.size].tobytes() == ref.tobytes(), w


@pytest.mark.parametrize("preset", [0.0, 0.02])
def test_a_step_that_a_later_worker_writes_over(preset):
    # (steps_out, step_in) as indices into the steps: the bytes are those of one call after the other
    n = 70001
    for workers in ([(1, 0), (0, None)], [(0, None), (0, None), (1, 0)], [(2, 3), (1, 0), (0, 3), (3, None), (2, 3)],
                    [(0, None), (1, 0), (0, 1), (0, None), (2, 0), (2, 2)]):
        host = _host(len(workers), n, "f32", 3)
        first = [0.01, 0.02, 0.03, 0.04]
        steps, codes, jobs = torch.tensor(first, device="cuda"), [], []
        for w, (to, given) in enumerate(workers):
            codes.append(torch.empty(ndq.ndq_packed_bytes(n, 4), dtype=torch.uint8, device="cuda"))
            jobs.append((_dev(host[w]), ndq.NDQ_WORKER_DQ, 16, 0, 1.0, ndq.ndq_dither(w, 3, w, 0), codes[w],
                         steps[to:to + 1], None if given is None else steps[given:given + 1]))
        ndq.ndq_encode_workers(jobs, preset, 0)
        held = list(first)
        for w, (to, given) in enumerate(workers):
            ref, s_ref = oracle.dq_encode(host[w], preset if given is None else float(F(held[given])), 16, 0,
                                          oracle.dither(w, 3, w))
            held[to] = float(s_ref[0])
            assert codes[w].cpu().numpy().tobytes() == ref.tobytes(), (workers, w)
        assert steps.cpu().numpy().tolist() == [float(F(x)) for x in held], workers


@pytest.mark.parametrize("bucket,shared", [(4096, False), (0, True)])
def test_streaming_encoder_over_several_vectors(bucket, shared):
    # together two tiles per wave slot (8,192 tiles of 4,096 elements) and a ragged end each:
    # waves walk from one vector into the next
    plan = (("dq", 4), ("nested", 2), ("nested", 2), ("nested", 2), ("nested", 2))
    _compare(plan, 4, bucket, shared, _host(len(plan), 2050 * 4096 + 77, "bf16", 5))


def test_bad_workers_are_reported_and_nothing_is_launched():
    g = torch.zeros(4096, device="cuda")
    codes, steps = torch.full((4096,), 7, dtype=torch.uint8, device="cuda"), torch.full((1,), -1.0, device="cuda")
    d = ndq.ndq_dither(1, 1, 1, 0)
    good = (g, ndq.NDQ_WORKER_DQ, 4, 0, 1.0, d, codes, steps, None)
    bad_M = (g, ndq.NDQ_WORKER_NESTED, 4, 1, 1.0, d, codes, steps, None)
    other = (g[:1024], ndq.NDQ_WORKER_NESTED, 4, 1, 1.0, d, codes, steps, None)     # needs a library call of its own
    for jobs in ([good, bad_M], [good, other]):
        with pytest.raises(ndq.NdqError) as e:
            ndq.ndq_encode_workers(jobs, 0.0, 0)
        assert e.value.rc == ndq.NDQ_EINVAL
        torch.cuda.synchronize()
        assert steps.item() == -1.0 and (codes == 7).all()


@pytest.mark.parametrize("W", [1, 3, 33, 70])
def test_decode_mean_keeps_every_reconstruction_and_their_sum(W):
    # tile edges (512 elements), partial vectors of four, levels of every code width, more workers
    # than one launch holds; sums in the same order as the oracle's, so bit for bit
    levels = [3, 5, 16, 2, 100, 256, 9]
    for n, bucket in ((1, 0), (511, 0), (1, 64), (513, 64), (513, 320), (4097, 192), (20001, 448), (2048 + 6, 512),
                      (20000, 2112), (1000, 1 << 20)):
        seeds = list(range(W))
        msgs, decoded = [], [torch.full((n,), 7.0, device="cuda") for _ in range(W)]
        host = _host(W, n, "f32", n)
        refs = []
        for w in range(W):
            d = oracle.dither(seeds[w], 2, w, 64)
            c, s = oracle.dq_encode(host[w], 0.0, levels[w % 7], bucket, d)
            refs.append(oracle.dq_decode(c, n, levels[w % 7], bucket, s, d))
            msgs.append((torch.from_numpy(c).cuda(), torch.from_numpy(s).cuda(), ndq.NDQ_WORKER_DQ, levels[w % 7],
                         ndq.ndq_dither(seeds[w], 2, w, 64)))
        out = ndq.ndq_decode_mean(msgs, decoded, n, bucket, 1.0 / W)
        for w in range(W):
            assert np.array_equal(decoded[w].cpu().numpy(), refs[w]), (n, bucket, w)
        assert np.array_equal(out.cpu().numpy(), oracle.aggregate(refs, 1.0 / W)), (n, bucket)
    if W <= 32:      # the sum in the place of one reconstruction; the others stay
        total = ndq.ndq_decode_mean(msgs, decoded, n, bucket, 1.0 / W, decoded[W // 2])
        assert np.array_equal(total.cpu().numpy(), oracle.aggregate(refs, 1.0 / W))
        for w in range(W):
            assert w == W // 2 or np.array_equal(decoded[w].cpu().numpy(), refs[w])
    bad = list(msgs[0])
    bad[2] = ndq.NDQ_WORKER_NESTED
    with pytest.raises(ndq.NdqError):
        ndq.ndq_decode_mean([tuple(bad)], decoded[:1], n, bucket)


def test_workers_of_different_length_type_and_bucket():
    # neighbours that do not agree are encoded by calls of their own: mixed types and lengths, and
    # handed-over steps (one for the whole vector) among bucketed vectors
    bucket = 2048
    host = [_host(1, n, dtype, n)[0] for n, dtype in ((9001, "f32"), (9001, "f32"), (9001, "bf16"), (70, "bf16"),
                                                      (70, "f32"))]
    outs, jobs, refs = [], [], []
    for w, g in enumerate(host):
        handed = w in (1, 4)
        codes = torch.full((ndq.ndq_packed_bytes(g.size, 4),), 0xA5, dtype=torch.uint8, device="cuda")
        steps = torch.full((1 if handed else ndq.ndq_num_buckets(g.size, bucket),), -1.0, device="cuda")
        outs.append((codes, steps))
        jobs.append((_dev(g), ndq.NDQ_WORKER_DQ, 16, 0, 1.0, ndq.ndq_dither(w, 3, w, 0), codes, steps,
                     outs[0][1][:1] if handed else None))
        d = oracle.dither(w, 3, w)
        refs.append(oracle.dq_encode(g, float(refs[0][1][0]) if handed else 0.0, 16, 0 if handed else bucket, d))
    ndq.ndq_encode_workers(jobs, 0.0, bucket)
    for w, (codes, steps) in enumerate(outs):
        assert np.array_equal(steps.cpu().numpy(), refs[w][1]), w
        assert codes.cpu().numpy().tobytes() == refs[w][0].tobytes(), w


def _bucket_maxima(g, bucket):
    g = g.float().abs()
    if bucket == 0:
        return g.max().reshape(1)
    whole = g.numel() // bucket * bucket
    parts = [g[:whole].view(-1, bucket).amax(1)] if whole else []
    return torch.cat(parts + ([g[whole:].max().reshape(1)] if whole < g.numel() else []))


# every form of the max-norm pass: an atomic per tile (under 16 tiles per bucket), per workgroup, a
# workgroup with a bucket to itself (129 buckets on), a bucket longer than the vector; cached loads and
# streaming ones (binary32 from 256 MB, bfloat16 from 32 MB on)
@pytest.mark.parametrize("dtype,n,bucket", [
    ("f32", 70001, 0), ("f32", 70001, 1 << 20), ("f32", 300007, 2048 * 15), ("f32", 128 * 32768, 32768),
    ("f32", 129 * 32768 - 5, 32768), ("f32", 700 * 32768 + 1, 32768), ("f32", (1 << 26) + 5, 0),
    ("f32", (1 << 26) + 5, 2048), ("bf16", 129 * 65536 + 9, 65536), ("bf16", (1 << 24) + 1, 0),
    ("bf16", 300 * 65536 + 3, 65536), ("bf16", (1 << 24) + 1, 4096)])
def test_max_norms_are_exact_in_every_form(dtype, n, bucket):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    g = torch.randn(n, device="cuda", generator=gen)
    g = g.to(torch.bfloat16) if dtype == "bf16" else g
    kappa = torch.full((ndq.ndq_num_buckets(n, bucket),), -1.0, device="cuda")
    ndq.ndq_absmax(g, bucket, kappa)
    assert torch.equal(kappa, _bucket_maxima(g, bucket))


@pytest.mark.parametrize("dtype,W,n,bucket", [
    ("f32", 16, 65 * 32768 + 77, 32768),      # more buckets in the batch than workgroups: one each
    ("f32", 3, 4 * 32768 + 77, 32768),        # parts, reduced by a kernel of their own
    ("bf16", 4, (1 << 22) + 9, 0),            # together above 32 MB: streaming loads
    ("f32", 2, 101000003, 0)])                # together above 768 MiB
def test_steps_of_a_batch_in_every_form_of_the_max_norm_pass(dtype, W, n, bucket):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    grads = [torch.randn(n, device="cuda", generator=gen) for _ in range(W)]
    grads = [g.to(torch.bfloat16) if dtype == "bf16" else g for g in grads]
    codes = [torch.empty(ndq.ndq_packed_bytes(n, 1), dtype=torch.uint8, device="cuda") for _ in grads]
    steps = [torch.full((ndq.ndq_num_buckets(n, bucket),), -1.0, device="cuda") for _ in grads]
    ndq.ndq_encode_workers([(grads[w], ndq.NDQ_WORKER_DQ, 2, 0, 1.0, ndq.ndq_dither(w, 3, w, 0), codes[w], steps[w],
                             None) for w in range(W)], 0.0, bucket)
    for w in range(W):       # two levels: Delta = 2 kappa, exactly
        assert torch.equal(steps[w], 2.0 * _bucket_maxima(grads[w], bucket)), w
    m = min(n, 1 << 20)      # the codes of the first elements
    ref, _ = oracle.dq_encode(grads[W - 1][:m].float().cpu().numpy(), steps[W - 1][0].item(), 2, 0,
                              oracle.dither(W - 1, 3, W - 1))
    if bucket == 0:
        assert codes[W - 1][:m // 8].cpu().numpy().tobytes() == ref[:m // 8].tobytes()


@pytest.mark.parametrize("kind,arg,bucket", [("dq", 3, 2048), ("nested", 4, 512), ("dq", 2, 8192), ("dq", 3, 0), ("nested", 2, 0)])
def test_codes_stored_through_the_cache_or_not_are_the_same(kind, arg, bucket):
    # narrow codes of binary32 vectors in buckets: stored through the L2 when a launch has 120 M bits of them, else plainly; sixteen
    # vectors in one call against one call each, and the last one against the oracle
    bits = ndq.ndq_code_bits(arg)
    n, W = (1 << 23) // bits + 77, 16
    gen = torch.Generator(device="cuda").manual_seed(arg)
    grads = [torch.randn(n, device="cuda", generator=gen) for _ in range(W)]
    ds = [ndq.ndq_dither(w, 3, w, 0) for w in range(W)]

    def encode(which):
        codes = [torch.full((ndq.ndq_packed_bytes(n, bits),), 0xA5, dtype=torch.uint8, device="cuda") for _ in which]
        steps = [torch.empty(ndq.ndq_num_buckets(n, bucket), device="cuda") for _ in which]
        ndq.ndq_encode_workers([(grads[w], ndq.NDQ_WORKER_DQ if kind == "dq" else ndq.NDQ_WORKER_NESTED,
                                 arg if kind == "dq" else 16, 0 if kind == "dq" else arg, 1.0, ds[w], c, s, None)
                                for w, c, s in zip(which, codes, steps)], 0.0, bucket)
        return codes, steps

    codes, steps = encode(range(W))
    for w in range(W):
        (c,), (s,) = encode([w])
        assert torch.equal(codes[w], c) and torch.equal(steps[w], s), w
    d = oracle.dither(W - 1, 3, W - 1)
    host = grads[-1].cpu().numpy()
    ref = oracle.dq_encode(host, 0.0, arg, bucket, d) if kind == "dq" else oracle.nested_encode(host, 0.0, 16, arg, bucket, d)
    assert codes[-1].cpu().numpy().tobytes() == ref[0].tobytes() and np.array_equal(steps[-1].cpu().numpy(), ref[1])
