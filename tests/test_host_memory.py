"""Host memory that runs out inside a C entry comes back as BILU_ERR_ALLOC, not
as an exception through the C boundary."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import resource, sys
from paper_1703_01325_amd import synth, _native as N
Ap, Aj = synth.stencil7_pattern(40, 60, 50)
ctx = N.bilu_analyze(Ap.size - 1, 3, Ap, Aj, 0, N.WANT_TRANSPOSE)
held = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
old = resource.getrlimit(resource.RLIMIT_AS)
resource.setrlimit(resource.RLIMIT_AS, (held + (1 << 20), old[1]))
try:
    N.bilu_validate(ctx)
    code = 0
except N.BiluError as e:
    code = e.code
resource.setrlimit(resource.RLIMIT_AS, old)
N.bilu_validate(ctx)                       # nothing half built is left
print("code", code)
"""


@pytest.mark.skipif(sys.platform != "linux", reason="reads /proc")
def test_validate_without_memory():
    r = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-500:]
    assert r.stdout.split()[-2:] == ["code", "-2"], r.stdout
