"""The work this library is measured on.

Each case is one use of the public entry points at one size: an iteration's
communication (every worker encodes its gradient, the server decodes and sums), or
one of the calls around it (a message and its entropy, the dense base-L stream, a
worker that shrinks against side information).  ``listed`` are the fixed
cases, ``draw`` gives further ones of the same kinds and ranges.

Sizes are those of the benchmark configurations (``workloads.CONFIGS``) and of the
networks the raw bit counts of the paper's tables are given for (266,610 and 1,663,370
parameters); the others are round or random numbers.
"""
import math

import torch

from paper_1904_01197_amd import ndq, pipeline
from paper_1904_01197_amd.workloads import Workload

# Total elements (workers x length) a drawn case may have.
DRAW_ELEMENTS = 1 << 27


def _iteration(n, workers, dtype, bucket, levels, ratio=0, nested=0, fine=None, shared=False,
               heavy=False, mean=True, server="fused"):
    """One training iteration: ``workers - nested`` DQSG workers of ``levels`` levels, then
    ``nested`` workers that send the fine index modulo ``ratio``.

    server: "fused"     all messages in hand, one call decodes and sums them
            "arrivals"  a message is decoded into the running sum when it arrives
            "separate"  every gradient is reconstructed for itself, then averaged
    """
    return {"kind": "iteration", "n": n, "workers": workers, "dtype": dtype, "bucket": bucket,
            "levels": levels, "ratio": ratio, "nested": nested, "fine": fine or levels,
            "shared": shared, "heavy": heavy, "mean": mean, "server": server}


def listed():
    return [
        # the smallest call: one worker, one step for the whole vector, three levels, there and
        # back (benchmark configuration 1); launches and host work count
        {"name": "roundtrip_64k", **_iteration(65536, 1, "f32", 0, 3, mean=False)},
        # two workers that share a step, the second one nested (configuration 2): 3-bit codes
        {"name": "pair_1m", **_iteration(1 << 20, 2, "f32", 0, 8, 4, 1, shared=True, mean=False)},
        # the paper's own nested experiment on the network of 266,610 parameters: half the
        # workers DQSG with five levels, half nested with ratio 3 and fine step 1/3
        {"name": "small_net_w8_m3", **_iteration(266610, 8, "f32", 0, 5, 3, 4, fine=7)},
        # Algorithm 1 as printed, every gradient reconstructed for itself, on the network of
        # 1,663,370 parameters with three levels
        {"name": "separate_w4_1663k", **_iteration(1663370, 4, "f32", 0, 3, server="separate")},
        # bucketed DQSG of eight workers, averaged (configuration 3)
        {"name": "bucketed_w8_25m", **_iteration(25557032, 8, "f32", 2048, 16)},
        # one DQSG worker and fifteen nested ones at the same step (configuration 4)
        {"name": "chain_w16_11m", **_iteration(11173962, 16, "f32", 0, 16, 4, 15, shared=True)},
        # the largest: heavy-tailed bfloat16 gradients, 2-bit DQSG and three 1-bit nested
        # workers (configuration 5)
        {"name": "heavy_tail_w4_128m",
         **_iteration(1 << 27, 4, "bf16", 4096, 4, 2, 3, heavy=True, mean=False)},
        # the same plan on a server that decodes each message when it arrives, ragged length
        {"name": "arrivals_w4_100m",
         **_iteration(100000007, 4, "bf16", 4096, 4, 2, 3, heavy=True, mean=False, server="arrivals")},
        # bfloat16 with buckets smaller than a wave's tile, ragged length
        {"name": "bf16_bucket1024_w4_11m", **_iteration(11173962, 4, "bf16", 1024, 16)},
        # a worker's message and how far it could still be compressed: 4-bit codes of bucketed
        # gradients, their histogram and entropy
        {"name": "entropy_b4_25m", "kind": "entropy", "n": 25557032, "levels": 16},
        # the dense stream of 1.6 bits per index, packed and unpacked again
        {"name": "dense_l3_25m", "kind": "dense", "n": 25557032, "levels": 3},
        # a worker that shrinks: its distance from the side information, its message, and the
        # server's value
        {"name": "shrink_m4_11m", "kind": "shrink", "n": 11173962, "dtype": "f32", "bucket": 0,
         "levels": 16, "ratio": 4, "alpha": 0.9},
    ]


def _log_int(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    """One more case of the ranges above; ``rng``: a random.Random."""
    kind = rng.choice(["iteration"] * 6 + ["entropy", "dense", "shrink"])
    if kind == "entropy":
        return {"kind": kind, "n": _log_int(rng, 60000, 100000000),
                "levels": rng.choice([2, 3, 4, 5, 8, 16, 32, 100, 256])}
    if kind == "dense":
        return {"kind": kind, "n": _log_int(rng, 60000, 50000000),
                "levels": rng.choice([3, 3, 5, 6, 7, 9, 12])}
    if kind == "shrink":
        return {"kind": kind, "n": _log_int(rng, 60000, 50000000), "dtype": rng.choice(["f32", "bf16"]),
                "bucket": rng.choice([0, 2048, 4096]), "levels": rng.choice([4, 8, 16]),
                "ratio": rng.choice([2, 3, 4, 8]), "alpha": rng.choice([0.75, 0.9, 0.97])}
    workers = rng.choice([1, 2, 4, 8, 16])
    n = _log_int(rng, 60000, DRAW_ELEMENTS // workers)
    if rng.random() < 0.3:
        n = max(4096, n // 4096 * 4096)         # whole tiles, as padded parameter buffers have
    dtype = rng.choice(["f32", "bf16"])
    bucket = rng.choice([0, 0, 512, 1024, 2048, 4096, 8192])
    levels = rng.choice([3, 4, 5, 8, 16])
    nested = 0 if workers == 1 else rng.choice([0, workers // 2, workers - 1])
    ratio = rng.choice([2, 3, 4, 4, 8]) if nested else 0
    shared = bool(nested) and bucket == 0 and rng.random() < 0.5
    server = rng.choice(["fused", "fused", "arrivals"] if nested else ["fused", "fused", "arrivals", "separate"])
    return _iteration(n, workers, dtype, bucket, levels, ratio, nested, shared=shared,
                      heavy=rng.random() < 0.3, mean=rng.random() < 0.5, server=server)


def _law(n, heavy, gen):
    """Unit normal, or Student t with three degrees of freedom."""
    x = torch.randn(n, device="cuda", generator=gen)
    if heavy:
        chi2 = torch.zeros(n, device="cuda")
        for _ in range(3):
            chi2.add_(torch.randn(n, device="cuda", generator=gen).square_())
        x.div_(chi2.div_(3.0).sqrt_())
    return x


def _gradients(n, workers, dtype, heavy, gen):
    """A common vector plus noise of each worker's own (the gradient model of the paper)."""
    scale, own = (1e-3, 5e-4) if heavy else (0.01, 0.003)
    common = _law(n, heavy, gen).mul_(scale)
    out = []
    for _ in range(workers):
        g = _law(n, heavy, gen).mul_(own).add_(common)
        out.append(g.to(torch.bfloat16) if dtype == "bf16" else g)
    return out


def _workload(case):
    plan = (("dq", case["levels"]),) * (case["workers"] - case["nested"])
    plan += (("nested", case["ratio"]),) * case["nested"]
    return Workload("iteration", 0, case["workers"], case["n"], case["dtype"],
                    "student_t3" if case["heavy"] else "normal", 1.0, 1.0, case["bucket"], case["fine"], plan,
                    1.0 / case["workers"] if case["mean"] else 1.0, shared_step=case["shared"],
                    seed_per_worker=True)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    n, kind = case["n"], case["kind"]
    state = {"case": case, "iteration": seed % 100000}
    if kind == "iteration":
        wl = _workload(case)
        state["workload"] = wl
        state["grads"] = _gradients(n, wl.W, wl.dtype, case["heavy"], gen)
        state["buffers"] = pipeline.allocate(wl, n, separate=case["server"] == "separate")
        return state
    if kind == "shrink":
        side, g = _gradients(n, 2, "f32", False, gen)
        state["side"] = side
        state["own"] = g
        state["grad"] = g.to(torch.bfloat16) if case["dtype"] == "bf16" else g
        state["codes"] = torch.empty(ndq.ndq_packed_bytes(n, ndq.ndq_code_bits(case["ratio"])),
                                     dtype=torch.uint8, device="cuda")
        state["steps"] = torch.empty(ndq.ndq_num_buckets(n, case["bucket"]), device="cuda")
        state["out"] = torch.empty(n, device="cuda")
        state["workspace"] = torch.empty(ndq.ndq_sqdiff_workspace() // 8, dtype=torch.float64, device="cuda")
        state["distance"] = torch.empty(1, dtype=torch.float64, device="cuda")
        return state
    levels = case["levels"]
    (g,) = _gradients(n, 1, "f32", False, gen)
    codes, steps = ndq.ndq_dq_encode(g, 0.0, levels, 2048, ndq.ndq_dither(seed, state["iteration"], 0, 0))
    state["codes"] = codes
    if kind == "entropy":
        state["grad"], state["steps"] = g, steps
        state["counts"] = torch.empty(1 << ndq.ndq_code_bits(levels), dtype=torch.int64, device="cuda")
        state["entropy"] = torch.empty(1, dtype=torch.float64, device="cuda")
    else:
        state["dense"] = torch.empty(ndq.ndq_dense_bytes(n, levels), dtype=torch.uint8, device="cuda")
        state["back"] = torch.empty_like(codes)
    return state


def run(state):
    case = state["case"]
    n, kind = case["n"], case["kind"]
    if kind == "iteration":
        wl, grads, bufs = state["workload"], state["grads"], state["buffers"]
        ds = pipeline.dithers(wl, state["iteration"])      # the iteration number is part of the dither
        out = {"codes": bufs.codes, "steps": bufs.steps}
        if case["server"] == "fused":
            out["total"] = pipeline.step_fused(wl, grads, bufs, ds)
        elif case["server"] == "arrivals":
            out["total"] = pipeline.step(wl, grads, bufs, ds)
        else:
            pipeline.encode_all(wl, grads, bufs, ds)
            out["total"] = pipeline.decode_separately(wl, n, bufs, ds)
            out["decoded"] = bufs.decoded
        return out
    if kind == "entropy":
        d = ndq.ndq_dither(0, state["iteration"], 0, 0)
        codes, steps = ndq.ndq_dq_encode(state["grad"], 0.0, case["levels"], 2048, d, state["codes"],
                                         state["steps"])
        counts, entropy = ndq.ndq_code_entropy(codes, n, ndq.ndq_code_bits(case["levels"]),
                                               state["counts"], state["entropy"])
        return {"codes": codes, "steps": steps, "counts": counts, "entropy": entropy}
    if kind == "dense":
        dense = ndq.ndq_dense_pack(state["codes"], n, case["levels"], state["dense"])
        return {"dense": dense, "back": ndq.ndq_dense_unpack(dense, n, case["levels"], state["back"])}
    d = ndq.ndq_dither(1, state["iteration"], 1, 0)
    distance = ndq.ndq_sqdiff(state["own"], state["side"], state["workspace"], state["distance"])
    codes, steps = ndq.ndq_nested_encode(state["grad"], 0.0, case["levels"], case["ratio"], case["alpha"],
                                         case["bucket"], d, state["codes"], state["steps"])
    out = ndq.ndq_nested_decode(codes, n, case["ratio"], case["alpha"], case["bucket"], steps, d,
                                state["side"], 1.0, state["out"])
    return {"distance": distance, "codes": codes, "steps": steps, "out": out}


def work(case):
    """Bytes: inputs read once, outputs written once (messages written by the workers and
    read by the server).  Operations: the floating-point ones of the definitions per
    element -- dither 2, quantizer 4, DQSG value 3, nested value 13 -- without the
    generator's integer rounds."""
    n, kind = case["n"], case["kind"]
    bits = ndq.ndq_code_bits(case["levels"])
    if kind == "entropy":
        message = n * bits / 8 + 4 * ndq.ndq_num_buckets(n, 2048)
        return {"bytes": 4 * n + 2 * message + 8 * 2 ** bits + 8, "flops": 6 * n}
    if kind == "dense":
        dense = ndq.ndq_dense_bytes(n, case["levels"])
        return {"bytes": 2 * (n * bits / 8 + dense), "flops": 0}
    size = 4 if case["dtype"] == "f32" else 2
    steps = 4 * ndq.ndq_num_buckets(n, case["bucket"])
    if kind == "shrink":
        message = n * ndq.ndq_code_bits(case["ratio"]) / 8 + steps
        gradient = n * 4 if size == 4 else n * 6          # bfloat16: the binary32 original is compared
        return {"bytes": gradient + 4 * n + 2 * message + 4 * n, "flops": n * (3 + 6 + 16)}
    nested, first = case["nested"], case["workers"] - case["nested"]
    messages = first * (n * bits / 8 + steps)
    if nested:
        messages += nested * (n * ndq.ndq_code_bits(case["ratio"]) / 8 + steps)
    moved = case["workers"] * n * size + 2 * messages + 4 * n
    if case["server"] == "arrivals":
        moved += (case["workers"] - 1) * 8 * n             # every later message updates the sum in memory
    if case["server"] == "separate":
        moved += case["workers"] * 8 * n                   # written by the decoders, read by the mean
    return {"bytes": moved, "flops": n * (case["workers"] * 6 + first * 6 + nested * 16)}


def tolerance(case):
    """The interface fixes every operation and its rounding, so codes, steps and values of two
    correct implementations agree in every bit.  The exceptions are sums in binary64 whose
    order is free: summed pairwise and one after the other, a squared distance of 11 to 50
    million normal terms differs by 1e-13 to 3e-13, an entropy of at most 256 terms by 1e-15."""
    if case["kind"] == "shrink":
        return {"rel": 1e-12}
    if case["kind"] == "entropy":
        return {"rel": 4e-15}
    return "exact"
