"""CPU test of the compile calls where host memory runs out: a status, not an exception that leaves the C boundary (which
ends the process)."""
import subprocess
import sys
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SCRIPT = """
import ctypes, resource
import gamegen as gg
import paper_2609_11923_amd as cfr
lib = cfr.load()
d = cfr.GameDesc(gg.kuhn())
games = (cfr.cfr_game_desc * 1)(d.desc)
used = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (used + (1 << 30),) * 2)
h = ctypes.c_void_p(1)
# the games' host layouts are the first thing allocated: their array alone is above the limit
status = lib.cfr_compile_batch(games, {n}, None, ctypes.byref(h))
print("status", status, "handle", h.value, lib.cfr_last_error().decode(), flush=True)
"""


@pytest.mark.parametrize("n", [1 << 24, (1 << 31) - 1])
def test_no_host_memory_is_a_status(n):
    r = subprocess.run([sys.executable, "-c", SCRIPT.replace("{n}", str(n))], capture_output=True, text=True, cwd=ROOT,
                       timeout=300)
    assert r.returncode == 0, (r.returncode, r.stderr[-500:])
    import paper_2609_11923_amd as cfr
    assert r.stdout.startswith(f"status {cfr.CFR_ENOMEM} handle None host compile failed"), r.stdout
