"""Calls of the binding that must raise, run in a process of their own by test_binding.py
(a failure of this kind can end the process).  There is no GPU: tensors are fake ones on the device,
and torch's current device and stream are stood in for, so that a call gets as far as
the addresses of its tensors."""
import sys

import torch
from torch._subclasses.fake_tensor import FakeTensorMode

torch._C._cuda_getDevice = lambda: 0
torch._C._cuda_getCurrentRawStream = lambda device: 0

from paper_1904_01197_amd import ndq  # noqa: E402

ndq.lib()
N, W = 64, 3


def every_call():
    """(name, function of a gradient, codes, steps, values and a binary64 number)"""
    d = ndq.ndq_dither(1, 1, 1, 0)
    job = lambda g, c, s: (g, ndq.NDQ_WORKER_DQ, 4, 0, 1.0, d, c, s, None)
    message = lambda c, s: (c, s, ndq.NDQ_WORKER_DQ, 4, d)
    return [
        ("absmax", lambda g, c, s, o, e, h: ndq.ndq_absmax(g, 0, s)),
        ("dq_encode", lambda g, c, s, o, e, h: ndq.ndq_dq_encode(g, 0.0, 4, 0, d, c, s)),
        ("dq_encode_with_step", lambda g, c, s, o, e, h: ndq.ndq_dq_encode_with_step(g, s, 4, d, c, s)),
        ("nested_encode", lambda g, c, s, o, e, h: ndq.ndq_nested_encode(g, 0.0, 4, 4, 1.0, 0, d, c, s)),
        ("nested_encode_with_step", lambda g, c, s, o, e, h: ndq.ndq_nested_encode_with_step(g, s, 4, 1.0, d, c, s)),
        ("encode_workers", lambda g, c, s, o, e, h: ndq.ndq_encode_workers([job(g, c, s)], 0.0, 0)),
        ("dq_decode", lambda g, c, s, o, e, h: ndq.ndq_dq_decode(c, N, 4, 0, s, d, o)),
        ("dq_decode_half", lambda g, c, s, o, e, h: ndq.ndq_dq_decode_half(c, N, 4, 0, s, o)),
        ("nested_decode", lambda g, c, s, o, e, h: ndq.ndq_nested_decode(c, N, 4, 1.0, 0, s, d, o, 1.0, o)),
        ("aggregate", lambda g, c, s, o, e, h: ndq.ndq_aggregate([g], 1.0, o)),
        ("decode_chain", lambda g, c, s, o, e, h: ndq.ndq_decode_chain([message(c, s)], N, 0, 1.0, o)),
        ("decode_mean", lambda g, c, s, o, e, h: ndq.ndq_decode_mean([message(c, s)], [o], N, 0, 1.0, g)),
        ("code_entropy", lambda g, c, s, o, e, h: ndq.ndq_code_entropy(c, N, 2, h, e)),
        ("dense_pack", lambda g, c, s, o, e, h: ndq.ndq_dense_pack(c, N, 4, c)),
        ("dense_unpack", lambda g, c, s, o, e, h: ndq.ndq_dense_unpack(c, N, 4, c)),
        ("sqdiff", lambda g, c, s, o, e, h: ndq.ndq_sqdiff(g, o, e, e)),
        ("sqdiff_static", lambda g, c, s, o, e, h: ndq.ndq_sqdiff_static(g, o, e)),
    ]


def tensors_without_storage():
    with FakeTensorMode():
        args = (torch.empty(W, N, device="cuda"), torch.empty(W, 64, dtype=torch.uint8, device="cuda"),
                torch.empty(W, 1, device="cuda"), torch.empty(W, N, device="cuda"),
                torch.empty(W, 1, dtype=torch.float64, device="cuda"),
                torch.empty(W, 4, dtype=torch.int64, device="cuda"))
        for name, call in every_call():
            print(name, flush=True)

            def one(g, c, s, o, e, h):
                call(g, c, s, o, e, h)
                return g

            try:
                torch.vmap(one)(*args)
            except RuntimeError as error:
                assert "data pointer" in str(error) and "#1 " not in str(error), str(error)
            else:
                raise AssertionError("%s took a tensor without storage" % name)
            # the interpreter is still whole
            assert sum(i * i for i in range(1000)) == 332833500


def a_refused_job_among_several_calls():
    """The binding over stand-ins for the library's functions: jobs of two lengths need two calls, the
    second of which is refused; the first must not have been made."""
    import ctypes as C
    made = []

    def answer(jobs, W, *rest):
        return ndq.NDQ_EINVAL if any(jobs[i].M == 1 for i in range(W)) else ndq.NDQ_OK

    @C.CFUNCTYPE(C.c_int, C.POINTER(ndq.ndq_encode_job), C.c_uint32, C.c_int, C.c_size_t, C.c_float, C.c_uint32,
                 C.c_void_p)
    def workers(jobs, W, *rest):
        rc = answer(jobs, W)
        if rc == ndq.NDQ_OK:
            made.append(W)
        return rc

    @C.CFUNCTYPE(C.c_int, C.POINTER(ndq.ndq_encode_job), C.c_uint32, C.c_int, C.c_size_t, C.c_float, C.c_uint32)
    def check(jobs, W, *rest):
        return answer(jobs, W)

    lib = ndq.lib()
    addresses = {name: C.cast(getattr(lib, name), C.c_void_p).value for name in ndq.EXPORTS}
    addresses["ndq_encode_workers"] = C.cast(workers, C.c_void_p).value
    addresses["ndq_encode_check"] = C.cast(check, C.c_void_p).value
    ndq._native.bind(addresses, ndq.ndq_dither, torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream)
    with FakeTensorMode():
        d = ndq.ndq_dither(1, 1, 1, 0)

        def job(n, M):
            return (torch.empty(n, device="cuda"), ndq.NDQ_WORKER_NESTED, 4, M, 1.0, d,
                    torch.empty(n, dtype=torch.uint8, device="cuda"), torch.empty(1, device="cuda"), None)

        ndq.ndq_encode_workers([job(64, 4), job(64, 4), job(128, 4)], 0.0, 0)
        assert made == [2, 1], made
        for jobs in ([job(64, 4), job(128, 1)], [job(64, 4)] * 1024 + [job(64, 1)], [job(64, 1)]):
            del made[:]
            try:
                ndq.ndq_encode_workers(jobs, 0.0, 0)
            except ndq.NdqError as error:
                assert error.rc == ndq.NDQ_EINVAL and made == [], made
            else:
                raise AssertionError("the refusal was lost")


def forms_of_a_message():
    """What a server may pass as a worker's message, over a stand-in for the library's function."""
    import ctypes as C
    seen = []

    @C.CFUNCTYPE(C.c_int, C.POINTER(ndq.ndq_worker), C.c_uint32, C.c_size_t, C.c_uint32, C.c_float, C.c_void_p,
                 C.c_void_p)
    def chain(workers, W, *rest):
        seen.append([(w.kind, w.levels_or_M, w.alpha, w.dither.seed, w.dither.step, w.dither.worker, w.dither.offset)
                     for w in workers[:W]])
        return ndq.NDQ_OK if W else ndq.NDQ_EINVAL

    lib = ndq.lib()
    addresses = {name: C.cast(getattr(lib, name), C.c_void_p).value for name in ndq.EXPORTS}
    addresses["ndq_decode_chain"] = C.cast(chain, C.c_void_p).value
    ndq._native.bind(addresses, ndq.ndq_dither, torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream)
    with FakeTensorMode():
        c, s = torch.empty(64, dtype=torch.uint8, device="cuda"), torch.empty(1, device="cuda")
        out = torch.empty(N, device="cuda")
        d = ndq.ndq_dither(1 << 40, 2, 3, 64)
        for message in ((c, s, 0, 4, d), [c, s, 0, 4, d], (c, s, 0, 4, (1 << 40, 2, 3, 64)), (c, s, 0, 4, d, 1.0, "more")):
            ndq.ndq_decode_chain([message], N, 0, 1.0, out)
            assert seen.pop() == [(0, 4, 1.0, 1 << 40, 2, 3, 64)], message
        ndq.ndq_decode_chain([(c, s, 0, 4, (9,)), (c, s, 1, 3, d, 0.5)], N, 0, 1.0, out)
        assert seen.pop() == [(0, 4, 1.0, 9, 0, 0, 0), (1, 3, 0.5, 1 << 40, 2, 3, 64)]
        for workers, kind in (([], ndq.NdqError), ([(c, s, 0, 4, [1, 2, 3, 0])], TypeError),
                              ([(c, s, 0, 4, (1, 2, 3, 0, 5))], TypeError), ([(c, s, 0, 4, None)], TypeError)):
            try:
                ndq.ndq_decode_chain(workers, N, 0, 1.0, out)
            except kind:
                continue
            raise AssertionError(workers)
        from paper_1904_01197_amd import pipeline, workloads
        wl = workloads.CONFIGS[1]
        empty = type(wl)(**dict(vars(wl), plan=(), W=0))
        pipeline.encode_all(empty, [], None, [])       # nobody to encode for: nothing happens


def refusals():
    """What the binding checks before the library is called: tensors on the device, contiguous, of the
    right type and large enough (the library never learns their sizes)."""
    d = ndq.ndq_dither(1, 1, 1, 0)
    with FakeTensorMode():
        n = 130                                                     # 130 codes of 2 bits: 33 bytes, so 48
        g, c, s = torch.empty(n, device="cuda"), torch.empty(48, dtype=torch.uint8, device="cuda"), \
            torch.empty(3, device="cuda")                           # three buckets of 64
        o, e = torch.empty(n, device="cuda"), torch.empty(1, dtype=torch.float64, device="cuda")
        host, strided = torch.empty(n), torch.empty(n, 2, device="cuda")[:, 0]
        job = lambda g=g, c=c, s=s, step=None, d=d, M=4: (g, ndq.NDQ_WORKER_NESTED, 4, M, 1.0, d, c, s, step)
        enc = lambda g=g, c=c, s=s, d=d: ndq.ndq_dq_encode(g, 0.0, 4, 64, d, c, s)
        nes = lambda g=g, c=c, s=s, d=d: ndq.ndq_nested_encode(g, 0.0, 4, 4, 1.0, 64, d, c, s)
        dec = lambda c=c, s=s, o=o, d=d: ndq.ndq_dq_decode(c, n, 4, 64, s, d, o)
        half = lambda c=c, s=s, o=o: ndq.ndq_dq_decode_half(c, n, 4, 64, s, o)
        ndec = lambda c=c, s=s, o=o, side=o, d=d: ndq.ndq_nested_decode(c, n, 4, 1.0, 64, s, d, side, 1.0, o)
        msg = lambda c=c, s=s, d=d: (c, s, ndq.NDQ_WORKER_DQ, 4, d)
        chain = lambda *m, o=o: ndq.ndq_decode_chain(list(m), n, 64, 1.0, o)
        mean = lambda m, dec, o=o: ndq.ndq_decode_mean(m, dec, n, 64, 1.0, o)
        workers = lambda *j: ndq.ndq_encode_workers(list(j), 0.0, 64)
        small_c, small_s, small_o = c[:32], s[:2], o[:129]
        cases = []
        for f in (enc, nes, lambda **k: workers(job(**k))):
            cases += [(TypeError, lambda f=f: f(g=host)), (TypeError, lambda f=f: f(g=strided)),
                      (TypeError, lambda f=f: f(g=[1.0])), (TypeError, lambda f=f: f(g=g.double())),
                      (TypeError, lambda f=f: f(c=c.cpu())), (TypeError, lambda f=f: f(s=s.cpu())),
                      (ValueError, lambda f=f: f(c=small_c)), (ValueError, lambda f=f: f(s=small_s)),
                      (TypeError, lambda f=f: f(d=(1, 1, 1, 0))), (TypeError, lambda f=f: f(d=None))]
        for f in (dec, ndec, half, lambda **k: chain(msg(**{x: k[x] for x in k if x != "o"}), o=k.get("o", o)),
                  lambda **k: mean([msg(**{x: k[x] for x in k if x != "o"})], [o], k.get("o", o)),
                  lambda **k: mean([msg(**{x: k[x] for x in k if x != "o"})], [k.get("o", o)])):
            cases += [(TypeError, lambda f=f: f(c=c.cpu())), (TypeError, lambda f=f: f(s=s.cpu())),
                      (TypeError, lambda f=f: f(o=o.cpu())), (TypeError, lambda f=f: f(o=strided)),
                      (ValueError, lambda f=f: f(c=small_c)), (ValueError, lambda f=f: f(s=small_s)),
                      (ValueError, lambda f=f: f(s=s.double())), (ValueError, lambda f=f: f(o=small_o)),
                      (ValueError, lambda f=f: f(o=o.double()))]
            if f is not half:
                cases.append((TypeError, lambda f=f: f(d=7)))
        cases += [
            (ValueError, lambda: workers()), (ValueError, lambda: workers(job()[:8])), (TypeError, lambda: workers(5)),
            (ValueError, lambda: workers(job(step=s.double()))), (ValueError, lambda: workers(job(step=s[:0]))),
            (ValueError, lambda: ndq.ndq_dq_encode_with_step(g, s.double(), 4, d, c, s)),
            (ValueError, lambda: ndq.ndq_nested_encode_with_step(g, s[:0], 4, 1.0, d, c, s)),
            (ValueError, lambda: ndq.ndq_nested_encode_with_step(g, s, 4, 1.0, d, small_c, s)),
            (ValueError, lambda: ndec(side=small_o)), (ValueError, lambda: ndec(side=o.double())),
            (TypeError, lambda: ndec(side=host)),
            (ValueError, lambda: chain(msg()[:4])), (ValueError, lambda: chain(msg(), msg(c=small_c))),
            (ValueError, lambda: mean([msg()], [])), (ValueError, lambda: mean([msg(), msg()], [o])),
            (ValueError, lambda: ndq.ndq_dq_decode(c, n, 4, 64, s, d, None, True)),
            (TypeError, lambda: ndq.ndq_absmax(host, 64, s)), (TypeError, lambda: ndq.ndq_absmax(g, 64, s.cpu())),
            (TypeError, lambda: ndq.ndq_absmax(g.half(), 64, s)), (TypeError, lambda: ndq.ndq_absmax(g, 64.0, s)),
            (ValueError, lambda: ndq.ndq_aggregate([g, g[:64]], 1.0, o)),
            (ValueError, lambda: ndq.ndq_aggregate([g.double()], 1.0, o)),
            (TypeError, lambda: ndq.ndq_aggregate([host], 1.0, o)), (TypeError, lambda: ndq.ndq_aggregate([g], "x", o)),
            (ValueError, lambda: ndq.ndq_code_entropy(small_c, n, 2)),
            (TypeError, lambda: ndq.ndq_code_entropy(c.cpu(), n, 2)),
            (ValueError, lambda: ndq.ndq_dense_pack(c, n, 3, c[:8])),
            (ValueError, lambda: ndq.ndq_dense_unpack(c, n, 3, small_c)),
            (ValueError, lambda: ndq.ndq_sqdiff(g, o[:64], e, e)), (ValueError, lambda: ndq.ndq_sqdiff(g, e, e, e)),
            (ValueError, lambda: ndq.ndq_sqdiff_static(g, o, s)), (ValueError, lambda: ndq.ndq_sqdiff_static(g, o, e[:0])),
        ]
        for i, (kind, call) in enumerate(cases):
            try:
                call()
            except kind as error:
                assert type(error) is kind, (i, error)
                continue
            raise AssertionError("case %d was not refused" % i)
        # what passes these checks reaches the library, which refuses the null addresses of fake tensors
        for call in (enc, nes, dec, half, ndec, lambda: chain(msg()), lambda: mean([msg()], [o]),
                     lambda: workers(job())):
            try:
                call()
            except ndq.NdqError as error:
                assert error.rc == ndq.NDQ_EINVAL
                continue
            raise AssertionError("null addresses were accepted")


if __name__ == "__main__":
    {"refusals": refusals, "messages": forms_of_a_message, "storage": tensors_without_storage, "refused": a_refused_job_among_several_calls}[sys.argv[1]]()
    print("BINDING_ERRORS_OK", flush=True)
