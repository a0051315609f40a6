"""Calls whose workgroups meet in memory that nobody has cleared: the sum of squared differences, whatever lies in
the result and the workspace; and the collector that gives up waiting."""
import os
import subprocess
import sys

import pytest
import torch

from paper_1904_01197_amd import ndq

pytestmark = pytest.mark.gpu


def _sqdiff_cases():
    """-> for some lengths the sum from workspaces that hold anything, its bits as text"""
    got = []
    for n in (1, 3, 2047, 4 * 512 * 512, 1000003, 11173962):
        gen = torch.Generator(device="cuda").manual_seed(n)
        a, b = torch.randn(n, device="cuda", generator=gen), torch.randn(n, device="cuda", generator=gen)
        ref = float((a.double() - b.double()).square().sum().item())
        work = torch.empty(ndq.ndq_sqdiff_workspace() // 8 + 1, dtype=torch.float64, device="cuda")
        sums = []
        for fill in (0, -1, None):
            if fill is None:
                work.view(torch.int64).random_(-2**62, 2**62, generator=gen)
            else:
                work.view(torch.int64).fill_(fill)
            sums.append(ndq.ndq_sqdiff(a, b, work[:-1]).clone())
            inside = work[fill:][:1] if fill == 0 else work[77:78]         # a result that lies in the workspace
            sums.append(ndq.ndq_sqdiff(a, b, work[1:] if n % 2 else work[:-1], inside).clone())
        for s in sums:
            assert abs(float(s.item()) - ref) <= n * 2.0 ** -52 * ref, n
            assert torch.equal(s, sums[0]), n
        got.append(float(sums[0].item()).hex())
    return got


def test_squared_differences_with_and_without_a_patient_collector():
    here = _sqdiff_cases()
    code = "import sys; sys.path.insert(0, %r); import test_gpu_one_launch as t; print('SUMS', *t._sqdiff_cases())" % os.path.dirname(__file__)
    res = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, NDQ_COLLECT_POLLS="0", PYTHONPATH=os.pathsep.join(sys.path)),
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:]
    assert res.stdout.split("SUMS")[1].split() == here
