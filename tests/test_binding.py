"""The Python binding's refusals, on the CPU."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))


def _run(case):
    env = dict(os.environ, PYTHONPATH=os.path.dirname(HERE))
    res = subprocess.run([sys.executable, "-u", os.path.join(HERE, "binding_errors.py"), case], env=env,
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    tail = "\n".join(res.stdout.splitlines()[-15:])
    assert res.returncode == 0 and "BINDING_ERRORS_OK" in res.stdout, (res.returncode, tail)


def test_a_tensor_without_storage_raises_and_the_process_goes_on():
    _run("storage")


def test_nothing_is_enqueued_when_one_of_several_calls_is_refused():
    _run("refused")


def test_the_forms_of_a_workers_message():
    _run("messages")


def test_tensors_of_the_wrong_kind_or_size_are_refused():
    _run("refusals")
