"""A package whose extension module cannot be loaded: the calls that need it say so, the others take their memory from PyTorch's allocator all
the same (no GPU: the allocator is stood in for)."""
import subprocess
import sys
from pathlib import Path

ROOT = Path(__file__).resolve().parent.parent

SCRIPT = """
import ctypes, sys
sys.modules["paper_2204_02662_amd._binding"] = None  # (import: ImportError)
import torch
import paper_2204_02662_amd as epp

try:
    epp.epp_backward_aggregate(None, None, None)
except FileNotFoundError:
    pass
else:
    raise SystemExit("no binding, and no error")

room, given = ctypes.create_string_buffer(4096), []

def alloc(nbytes):
    if nbytes > 4096:
        raise torch.OutOfMemoryError("as PyTorch says it")
    return ctypes.addressof(room)

torch.cuda.caching_allocator_alloc, torch.cuda.caching_allocator_delete = alloc, given.append
handed = ctypes.cast(epp._allocator(True), ctypes.POINTER(epp._Alloc)).contents
assert handed.alloc and handed.free, "the library would take memory of its own"
assert epp._allocator(False) is None
assert handed.alloc(4097, None) is None
p = handed.alloc(1000, None)
assert p == ctypes.addressof(room) and dict(epp.alloc_stats) == {"allocs": 1, "frees": 0, "bytes": 1000, "live": 1}, epp.alloc_stats
handed.free(p, None)
assert given == [p] and epp.alloc_stats == {"allocs": 1, "frees": 1, "bytes": 1000, "live": 0}, epp.alloc_stats
print("as before")
"""


def test_memory_still_comes_from_pytorch():
    out = subprocess.run([sys.executable, "-c", SCRIPT], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and "as before" in out.stdout, out.stdout[-500:] + out.stderr[-2000:]
