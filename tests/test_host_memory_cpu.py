"""Out of host memory inside a batched entry point: the status of a failed
call, not a C++ exception across the C ABI (which ends the process).  A child
with little address space left passes a job count whose lists cannot be
allocated; the jobs themselves are not read before that."""
import subprocess
import sys

import pytest

from conftest import ROOT
from paper_2608_03057_amd import _lib

CHILD = """
import ctypes, resource
from paper_2608_03057_amd import _lib
L = _lib.lib()
pages = int(open("/proc/self/statm").read().split()[0])
limit = pages * resource.getpagesize() + (256 << 20)
resource.setrlimit(resource.RLIMIT_AS, (limit, limit))
print(L.{name}((_lib.{job} * 1)(), 1 << 30, None))
"""


@pytest.mark.parametrize("name,job", [("tasq_quantize_activations_batch", "ActJob"),
                                      ("tasq_quantize_weights_batch", "WeightJob")])
def test_batch_without_host_memory(name, job):
    r = subprocess.run([sys.executable, "-c", CHILD.format(name=name, job=job)], cwd=ROOT,
                       stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-500:]
    assert int(r.stdout.split()[-1]) == _lib.TASQ_ERR_HIP
