"""ctypes binding of libndq (include/ndq.h): argument marshalling only.

Every function has the name and the argument order of its C entry point and
takes torch CUDA tensors where the C function takes device pointers; kernels
are enqueued on torch's current stream.  Output tensors may be passed in
(to reuse memory) or are allocated with torch.  There is no CPU fallback: if
``libndq.so`` has not been built, loading raises.
"""
import ctypes as C
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
_SO = os.environ.get("NDQ_LIBRARY", os.path.join(_HERE, "libndq.so"))   # override: another build

NDQ_F32, NDQ_BF16 = 0, 1
NDQ_OK, NDQ_EINVAL, NDQ_EALIGN, NDQ_EUNSUPPORTED, NDQ_ELAUNCH = 0, -1, -2, -3, -4

EXPORTS = ("ndq_code_bits", "ndq_packed_bytes", "ndq_num_buckets", "ndq_absmax", "ndq_dq_encode",
           "ndq_dq_encode_with_step", "ndq_nested_encode_with_step", "ndq_encode_workers",
           "ndq_dq_decode", "ndq_dq_decode_half", "ndq_nested_encode", "ndq_nested_decode", "ndq_aggregate",
           "ndq_decode_chain", "ndq_code_entropy", "ndq_dense_group", "ndq_dense_bytes",
           "ndq_dense_pack", "ndq_dense_unpack", "ndq_alpha_for_equal_variance",
           "ndq_decode_error_bound", "ndq_nesting_ratio_for_error", "ndq_sqdiff_workspace", "ndq_sqdiff", "ndq_sqdiff_static",
           "ndq_strerror")


class ndq_dither(C.Structure):
    """Mirror of the C struct: (seed, step, worker, offset)."""
    _fields_ = [("seed", C.c_uint64), ("step", C.c_uint32), ("worker", C.c_uint32),
                ("offset", C.c_uint64)]


NDQ_WORKER_DQ, NDQ_WORKER_NESTED = 0, 1


class ndq_worker(C.Structure):
    """Mirror of the C struct: one worker's message as the server holds it."""
    _fields_ = [("codes", C.c_void_p), ("steps", C.c_void_p), ("kind", C.c_uint32),
                ("levels_or_M", C.c_uint32), ("alpha", C.c_float), ("dither", ndq_dither)]


class ndq_encode_job(C.Structure):
    """Mirror of the C struct: one worker's vector to encode."""
    _fields_ = [("g", C.c_void_p), ("codes_out", C.c_void_p), ("steps_out", C.c_void_p),
                ("step_in", C.c_void_p), ("kind", C.c_uint32), ("levels", C.c_uint32),
                ("M", C.c_uint32), ("alpha", C.c_float), ("dither", ndq_dither)]


class NdqError(RuntimeError):
    def __init__(self, rc, what):
        self.rc = rc
        super().__init__("%s failed: %s (%d)" % (what, ndq_strerror(rc), rc))


_lib = None


def lib():
    """The loaded shared library (loads it on first use)."""
    global _lib
    if _lib is None:
        if not os.path.exists(_SO):
            raise RuntimeError(
                "libndq.so is not built (%s); run `python -m paper_1904_01197_amd.build` or "
                "__graft_entry__.build() first -- there is no fallback path" % _SO)
        L = C.CDLL(_SO)
        vp, sz, u32, f32, ci = C.c_void_p, C.c_size_t, C.c_uint32, C.c_float, C.c_int
        dp = C.POINTER(ndq_dither)
        L.ndq_code_bits.argtypes, L.ndq_code_bits.restype = [u32], u32
        L.ndq_packed_bytes.argtypes, L.ndq_packed_bytes.restype = [sz, u32], sz
        L.ndq_num_buckets.argtypes, L.ndq_num_buckets.restype = [sz, u32], sz
        L.ndq_absmax.argtypes, L.ndq_absmax.restype = [vp, ci, sz, u32, vp, vp], ci
        L.ndq_dq_encode.argtypes = [vp, ci, sz, f32, u32, u32, dp, vp, vp, vp]
        L.ndq_dq_encode.restype = ci
        L.ndq_dq_decode.argtypes = [vp, sz, u32, u32, vp, dp, vp, ci, vp]
        L.ndq_dq_decode.restype = ci
        L.ndq_dq_decode_half.argtypes = [vp, sz, u32, u32, vp, vp, ci, vp]
        L.ndq_dq_decode_half.restype = ci
        L.ndq_nested_encode.argtypes = [vp, ci, sz, f32, u32, u32, f32, u32, dp, vp, vp, vp]
        L.ndq_nested_encode.restype = ci
        L.ndq_dq_encode_with_step.argtypes = [vp, ci, sz, vp, u32, dp, vp, vp, vp]
        L.ndq_dq_encode_with_step.restype = ci
        L.ndq_nested_encode_with_step.argtypes = [vp, ci, sz, vp, u32, f32, dp, vp, vp, vp]
        L.ndq_nested_encode_with_step.restype = ci
        L.ndq_encode_workers.argtypes = [C.POINTER(ndq_encode_job), u32, ci, sz, f32, u32, vp]
        L.ndq_encode_workers.restype = ci
        L.ndq_nested_decode.argtypes = [vp, sz, u32, f32, u32, vp, dp, vp, f32, vp, ci, vp]
        L.ndq_nested_decode.restype = ci
        L.ndq_aggregate.argtypes, L.ndq_aggregate.restype = [vp, u32, sz, f32, vp, vp], ci
        L.ndq_decode_chain.argtypes = [C.POINTER(ndq_worker), u32, sz, u32, f32, vp, vp]
        L.ndq_decode_chain.restype = ci
        L.ndq_alpha_for_equal_variance.argtypes = [C.c_double, C.c_double]
        L.ndq_alpha_for_equal_variance.restype = C.c_double
        L.ndq_decode_error_bound.argtypes = [C.c_double, u32, C.c_double, C.c_double]
        L.ndq_decode_error_bound.restype = C.c_double
        L.ndq_nesting_ratio_for_error.argtypes = [C.c_double, C.c_double, C.c_double, C.c_double]
        L.ndq_nesting_ratio_for_error.restype = u32
        L.ndq_sqdiff_workspace.argtypes, L.ndq_sqdiff_workspace.restype = [], sz
        L.ndq_sqdiff.argtypes, L.ndq_sqdiff.restype = [vp, vp, sz, vp, vp, vp], ci
        L.ndq_sqdiff_static.argtypes, L.ndq_sqdiff_static.restype = [vp, vp, sz, vp, vp], ci
        L.ndq_dense_group.argtypes, L.ndq_dense_group.restype = [u32], u32
        L.ndq_dense_bytes.argtypes, L.ndq_dense_bytes.restype = [sz, u32], sz
        L.ndq_dense_pack.argtypes, L.ndq_dense_pack.restype = [vp, sz, u32, vp, vp], ci
        L.ndq_dense_unpack.argtypes, L.ndq_dense_unpack.restype = [vp, sz, u32, vp, vp], ci
        L.ndq_code_entropy.argtypes, L.ndq_code_entropy.restype = [vp, sz, u32, vp, vp, vp], ci
        L.ndq_strerror.argtypes, L.ndq_strerror.restype = [ci], C.c_char_p
        _lib = L
    return _lib


def _stream():
    return C.c_void_p(torch.cuda.current_stream().cuda_stream)


def _dt(g):
    if g.dtype == torch.float32:
        return NDQ_F32
    if g.dtype == torch.bfloat16:
        return NDQ_BF16
    raise TypeError("gradient must be float32 or bfloat16")


def _dev(t, what):
    if not (isinstance(t, torch.Tensor) and t.is_cuda and t.is_contiguous()):
        raise TypeError("%s must be a contiguous CUDA tensor" % what)
    return C.c_void_p(t.data_ptr())


def _check(rc, what):
    if rc != NDQ_OK:
        raise NdqError(rc, what)


def ndq_strerror(rc):
    return lib().ndq_strerror(rc).decode()


def ndq_code_bits(levels_or_M):
    return lib().ndq_code_bits(levels_or_M)


def ndq_packed_bytes(n, bits):
    return lib().ndq_packed_bytes(n, bits)


def ndq_num_buckets(n, bucket):
    return lib().ndq_num_buckets(n, bucket)


def ndq_absmax(g, bucket, kappa_out=None):
    n = g.numel()
    if kappa_out is None:
        kappa_out = torch.empty(ndq_num_buckets(n, bucket), dtype=torch.float32, device=g.device)
    _check(lib().ndq_absmax(_dev(g, "g"), _dt(g), n, bucket, _dev(kappa_out, "kappa_out"),
                            _stream()), "ndq_absmax")
    return kappa_out


def _bits(levels_or_M):
    # ndq_code_bits and the two size rules below without a call into the library: they are
    # evaluated several times per call, and a foreign call costs as much as a launch's half
    return (levels_or_M - 1).bit_length() if 2 <= levels_or_M <= 256 else 0


def _packed(n, bits):
    return ((n * bits + 7) // 8 + 15) // 16 * 16


def _buckets(n, bucket):
    return (n + bucket - 1) // bucket if bucket else 1


def _enc_outputs(g, bits, bucket, codes_out, steps_out):
    n = g.numel()
    if codes_out is None:
        codes_out = torch.empty(_packed(n, bits), dtype=torch.uint8, device=g.device)
    if steps_out is None:
        steps_out = torch.empty(_buckets(n, bucket), dtype=torch.float32, device=g.device)
    if codes_out.numel() * codes_out.element_size() < _packed(n, bits):
        raise ValueError("codes_out too small")
    if steps_out.numel() < _buckets(n, bucket):
        raise ValueError("steps_out too small")
    return codes_out, steps_out


def ndq_dq_encode(g, delta, levels, bucket, d, codes_out=None, steps_out=None):
    """-> (codes uint8 tensor, steps float32 tensor)"""
    codes_out, steps_out = _enc_outputs(g, _bits(levels), bucket, codes_out, steps_out)
    _check(lib().ndq_dq_encode(_dev(g, "g"), _dt(g), g.numel(), delta, levels, bucket, C.byref(d),
                               _dev(codes_out, "codes_out"), _dev(steps_out, "steps_out"),
                               _stream()), "ndq_dq_encode")
    return codes_out, steps_out


def ndq_nested_encode(g, delta, levels, M, alpha, bucket, d, codes_out=None, steps_out=None):
    codes_out, steps_out = _enc_outputs(g, _bits(M), bucket, codes_out, steps_out)
    _check(lib().ndq_nested_encode(_dev(g, "g"), _dt(g), g.numel(), delta, levels, M, alpha, bucket,
                                   C.byref(d), _dev(codes_out, "codes_out"),
                                   _dev(steps_out, "steps_out"), _stream()), "ndq_nested_encode")
    return codes_out, steps_out


def _step_in(step_in):
    ptr = _dev(step_in, "step_in")
    if step_in.dtype != torch.float32 or step_in.numel() < 1:
        raise ValueError("step_in must hold one float32")
    return ptr


def ndq_dq_encode_with_step(g, step_in, levels, d, codes_out=None, steps_out=None):
    """-> (codes, steps); the step is read from the device tensor step_in"""
    codes_out, steps_out = _enc_outputs(g, _bits(levels), 0, codes_out, steps_out)
    _check(lib().ndq_dq_encode_with_step(_dev(g, "g"), _dt(g), g.numel(), _step_in(step_in), levels,
                                         C.byref(d), _dev(codes_out, "codes_out"),
                                         _dev(steps_out, "steps_out"), _stream()),
           "ndq_dq_encode_with_step")
    return codes_out, steps_out


def ndq_nested_encode_with_step(g, step_in, M, alpha, d, codes_out=None, steps_out=None):
    codes_out, steps_out = _enc_outputs(g, _bits(M), 0, codes_out, steps_out)
    _check(lib().ndq_nested_encode_with_step(_dev(g, "g"), _dt(g), g.numel(), _step_in(step_in), M, alpha,
                                             C.byref(d), _dev(codes_out, "codes_out"),
                                             _dev(steps_out, "steps_out"), _stream()),
           "ndq_nested_encode_with_step")
    return codes_out, steps_out


def ndq_encode_workers(jobs, delta, bucket):
    """jobs: sequence of (g, kind, levels, M, alpha, ndq_dither, codes_out, steps_out, step_in) with
    vectors of one length and type; M and alpha count for nested workers, step_in is None or a
    device tensor holding one float32 step (bucket 0)."""
    g0 = jobs[0][0]
    n, dt = g0.numel(), _dt(g0)
    arr = (ndq_encode_job * len(jobs))()
    for a, (g, kind, levels, M, alpha, d, codes_out, steps_out, step_in) in zip(arr, jobs):
        if g.numel() != n or g.dtype != g0.dtype:
            raise ValueError("all gradients must have one length and type")
        bits = _bits(M if kind == NDQ_WORKER_NESTED else levels)
        _enc_outputs(g, bits, bucket, codes_out, steps_out)
        a.g = _dev(g, "g").value
        a.codes_out = _dev(codes_out, "codes_out").value
        a.steps_out = _dev(steps_out, "steps_out").value
        a.step_in = None if step_in is None else _step_in(step_in).value
        a.kind, a.levels, a.M, a.alpha, a.dither = kind, levels, M, alpha, d
    _check(lib().ndq_encode_workers(arr, len(jobs), dt, n, delta, bucket, _stream()), "ndq_encode_workers")


def _check_message(codes, steps, n, bits, bucket):
    """A worker's message must be as large as the call will read."""
    if codes.numel() * codes.element_size() < _packed(n, bits):
        raise ValueError("codes hold fewer than ndq_packed_bytes(n, bits) bytes")
    if steps.dtype != torch.float32 or steps.numel() < _buckets(n, bucket):
        raise ValueError("steps must hold ndq_num_buckets(n, bucket) float32")


def ndq_dq_decode(codes, n, levels, bucket, steps, d, out=None, accumulate=False):
    _check_message(codes, steps, n, _bits(levels), bucket)
    if out is None:
        if accumulate:
            raise ValueError("accumulate needs an existing out")
        out = torch.empty(n, dtype=torch.float32, device=codes.device)
    if out.dtype != torch.float32 or out.numel() < n:
        raise ValueError("out must hold n float32")
    _check(lib().ndq_dq_decode(_dev(codes, "codes"), n, levels, bucket, _dev(steps, "steps"),
                               C.byref(d), _dev(out, "out"), int(bool(accumulate)), _stream()),
           "ndq_dq_decode")
    return out


def ndq_dq_decode_half(codes, n, levels, bucket, steps, out=None, accumulate=False):
    _check_message(codes, steps, n, _bits(levels), bucket)
    if out is None:
        if accumulate:
            raise ValueError("accumulate needs an existing out")
        out = torch.empty(n, dtype=torch.float32, device=codes.device)
    if out.dtype != torch.float32 or out.numel() < n:
        raise ValueError("out must hold n float32")
    _check(lib().ndq_dq_decode_half(_dev(codes, "codes"), n, levels, bucket, _dev(steps, "steps"),
                                    _dev(out, "out"), int(bool(accumulate)), _stream()),
           "ndq_dq_decode_half")
    return out


def ndq_nested_decode(codes, n, M, alpha, bucket, steps, d, side, side_scale=1.0, out=None,
                      accumulate=False):
    _check_message(codes, steps, n, _bits(M), bucket)
    if out is None:
        if accumulate:
            raise ValueError("accumulate needs an existing out")
        out = torch.empty(n, dtype=torch.float32, device=codes.device)
    if out.dtype != torch.float32 or out.numel() < n or side.dtype != torch.float32 or side.numel() < n:
        raise ValueError("out and side must hold n float32")
    _check(lib().ndq_nested_decode(_dev(codes, "codes"), n, M, alpha, bucket, _dev(steps, "steps"),
                                   C.byref(d), _dev(side, "side"), side_scale, _dev(out, "out"),
                                   int(bool(accumulate)), _stream()), "ndq_nested_decode")
    return out


def ndq_aggregate(gs, scale=1.0, out=None):
    n = gs[0].numel()
    for g in gs:
        if g.dtype != torch.float32 or g.numel() != n:
            raise ValueError("all inputs must be float32 of equal length")
    if out is None:
        out = torch.empty(n, dtype=torch.float32, device=gs[0].device)
    ptrs = (C.c_void_p * len(gs))(*[_dev(g, "gs[w]").value for g in gs])
    _check(lib().ndq_aggregate(C.cast(ptrs, C.c_void_p), len(gs), n, scale, _dev(out, "out"),
                               _stream()), "ndq_aggregate")
    return out


def ndq_decode_chain(workers, n, bucket, scale=1.0, out=None):
    """workers: sequence of (codes, steps, kind, levels_or_M, ndq_dither[, alpha]) in decoding
    order; alpha (nested workers only) defaults to 1."""
    arr = (ndq_worker * len(workers))()
    for i, wk in enumerate(workers):
        codes, steps, kind, arg, d = wk[:5]
        _check_message(codes, steps, n, _bits(arg), bucket)
        arr[i].codes = _dev(codes, "codes").value
        arr[i].steps = _dev(steps, "steps").value
        arr[i].kind = kind
        arr[i].levels_or_M = arg
        arr[i].alpha = wk[5] if len(wk) > 5 else 1.0
        arr[i].dither = d
    if out is None:
        out = torch.empty(n, dtype=torch.float32, device=workers[0][0].device)
    if out.dtype != torch.float32 or out.numel() < n:
        raise ValueError("out must hold n float32")
    _check(lib().ndq_decode_chain(arr, len(workers), n, bucket, scale, _dev(out, "out"),
                                  _stream()), "ndq_decode_chain")
    return out


def ndq_code_entropy(codes, n, bits, hist_out=None, entropy_out=None, want_entropy=True):
    """-> (histogram int64 tensor of 2^bits counts, entropy float64 tensor of 1 element;
    None with want_entropy=False: the C call then gets a null entropy_out)"""
    dev = codes.device
    if n and codes.numel() * codes.element_size() < _packed(n, bits):
        raise ValueError("codes hold fewer than ndq_packed_bytes(n, bits) bytes")
    if hist_out is None:
        hist_out = torch.empty(1 << bits, dtype=torch.int64, device=dev)
    if not want_entropy:
        entropy_out = None
    elif entropy_out is None:
        entropy_out = torch.empty(1, dtype=torch.float64, device=dev)
    cptr = _dev(codes, "codes") if n else C.c_void_p(0)
    eptr = _dev(entropy_out, "entropy_out") if want_entropy else C.c_void_p(0)
    _check(lib().ndq_code_entropy(cptr, n, bits, _dev(hist_out, "hist_out"), eptr, _stream()),
           "ndq_code_entropy")
    return hist_out, entropy_out


def ndq_dense_group(levels):
    return lib().ndq_dense_group(levels)


def ndq_dense_bytes(n, levels):
    return lib().ndq_dense_bytes(n, levels)


def ndq_dense_pack(codes, n, levels, dense_out=None):
    if dense_out is None:
        dense_out = torch.empty(ndq_dense_bytes(n, levels), dtype=torch.uint8, device=codes.device)
    if dense_out.numel() * dense_out.element_size() < ndq_dense_bytes(n, levels):
        raise ValueError("dense_out too small")
    if n:
        _check(lib().ndq_dense_pack(_dev(codes, "codes"), n, levels, _dev(dense_out, "dense_out"),
                                    _stream()), "ndq_dense_pack")
    return dense_out


def ndq_dense_unpack(dense, n, levels, codes_out=None):
    nbytes = _packed(n, _bits(levels))
    if codes_out is None:
        codes_out = torch.empty(nbytes, dtype=torch.uint8, device=dense.device)
    if codes_out.numel() * codes_out.element_size() < nbytes:
        raise ValueError("codes_out too small")
    if n:
        _check(lib().ndq_dense_unpack(_dev(dense, "dense"), n, levels, _dev(codes_out, "codes_out"),
                                      _stream()), "ndq_dense_unpack")
    return codes_out


def ndq_alpha_for_equal_variance(delta1, sigma_z2):
    return lib().ndq_alpha_for_equal_variance(delta1, sigma_z2)


def ndq_decode_error_bound(delta1, M, alpha, sigma_z2):
    return lib().ndq_decode_error_bound(delta1, M, alpha, sigma_z2)


def ndq_nesting_ratio_for_error(delta1, alpha, sigma_z2, p_max):
    return lib().ndq_nesting_ratio_for_error(delta1, alpha, sigma_z2, p_max)


def ndq_sqdiff_workspace():
    return lib().ndq_sqdiff_workspace()


def ndq_sqdiff(a, b, workspace=None, out=None):
    """sum_i (a_i - b_i)^2 in binary64 -> 1-element float64 tensor"""
    if a.dtype != torch.float32 or b.dtype != torch.float32 or a.numel() != b.numel():
        raise ValueError("a and b must be float32 of equal length")
    if workspace is None:
        workspace = torch.empty(ndq_sqdiff_workspace() // 8, dtype=torch.float64, device=a.device)
    if out is None:
        out = torch.empty(1, dtype=torch.float64, device=a.device)
    _check(lib().ndq_sqdiff(_dev(a, "a"), _dev(b, "b"), a.numel(), _dev(workspace, "workspace"),
                            _dev(out, "out"), _stream()), "ndq_sqdiff")
    return out


def ndq_sqdiff_static(a, b, out):
    """ndq_sqdiff with the library's own static partial-sum array: allocates nothing,
    so `out` (1-element float64 tensor) must be passed in."""
    if a.dtype != torch.float32 or b.dtype != torch.float32 or a.numel() != b.numel():
        raise ValueError("a and b must be float32 of equal length")
    if out.dtype != torch.float64 or out.numel() < 1:
        raise ValueError("out must hold one float64")
    _check(lib().ndq_sqdiff_static(_dev(a, "a"), _dev(b, "b"), a.numel(), _dev(out, "out"),
                                   _stream()), "ndq_sqdiff_static")
    return out
