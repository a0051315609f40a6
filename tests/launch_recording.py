"""The launches a library call makes, recorded on the CPU (see launch_recorder.cpp).

    recorder = build(tmp_path)
    (rc, launches), ... = record(recorder, [["ndq_dq_encode", arguments...], ...])

The calls run in a process of their own, because the library of this process has long been
bound to the real runtime; device pointers are plain numbers that nobody dereferences."""
import ctypes as C
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
LIBRARY = os.environ.get("NDQ_LIBRARY", os.path.join(os.path.dirname(HERE), "paper_1904_01197_amd", "libndq.so"))


class Dither(C.Structure):
    _fields_ = [("seed", C.c_uint64), ("step", C.c_uint32), ("worker", C.c_uint32), ("offset", C.c_uint64)]


class Job(C.Structure):
    _fields_ = [("g", C.c_void_p), ("codes_out", C.c_void_p), ("steps_out", C.c_void_p),
                ("step_in", C.c_void_p), ("kind", C.c_uint32), ("levels", C.c_uint32),
                ("M", C.c_uint32), ("alpha", C.c_float), ("dither", Dither)]


class Worker(C.Structure):
    _fields_ = [("codes", C.c_void_p), ("steps", C.c_void_p), ("kind", C.c_uint32),
                ("levels_or_M", C.c_uint32), ("alpha", C.c_float), ("dither", Dither)]


def build(tmp_path):
    so = str(tmp_path / "launch_recorder.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", os.path.join(HERE, "launch_recorder.cpp"),
                           "-o", so])
    return so


def record(recorder, calls, env=None):
    """calls: list of [function, arguments...] as plain values -> list of (status, launches),
    a launch being (kernel's mangled name, grid x, grid y).  A list of dicts among the arguments
    is an array of jobs (with "g") or of workers; a list of numbers an array of pointers; None NULL;
    {"dither": [seed, step, worker, offset]} a dither; a float a float."""
    res = subprocess.run([sys.executable, os.path.abspath(__file__), recorder], input=json.dumps(calls), text=True,
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, env=dict(os.environ, **(env or {})),
                         timeout=120)
    assert res.returncode == 0, res.stdout[-2000:]
    return [(rc, [(name, int(x), int(y)) for name, x, y in (line.split() for line in text.splitlines())])
            for rc, text in json.loads(res.stdout.splitlines()[-1])]


def _structure(cls, values):
    s = cls()
    for key, v in values.items():
        setattr(s, key, Dither(*v) if key == "dither" else v)
    return s


def _argument(a):
    if a is None:
        return C.c_void_p(None)
    if isinstance(a, dict):
        return C.byref(Dither(*a["dither"]))
    if isinstance(a, list) and a and isinstance(a[0], dict):
        cls = Job if "g" in a[0] else Worker
        return (cls * len(a))(*[_structure(cls, v) for v in a])
    if isinstance(a, list):
        return (C.c_void_p * len(a))(*a)
    if isinstance(a, float):
        return C.c_float(a)
    return C.c_size_t(a)


def _child(recorder):
    r = C.CDLL(recorder, mode=C.RTLD_GLOBAL)
    r.recorder_log.restype = C.c_char_p
    lib = C.CDLL(LIBRARY)
    out = []
    for name, *args in json.load(sys.stdin):
        r.recorder_clear()
        rc = getattr(lib, name)(*[_argument(a) for a in args])
        out.append((rc, r.recorder_log().decode()))
    print(json.dumps(out))


if __name__ == "__main__":
    _child(sys.argv[1])
