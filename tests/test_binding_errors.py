"""The CPython entry points with tensors that PyTorch cannot give sizes or memory for: an exception, never the
end of the process (no GPU involved: nothing is launched)."""
import subprocess
import sys
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent

SCRIPT = """
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
from torch.fx.experimental.symbolic_shapes import ShapeEnv
import paper_2204_02662_amd as epp

class Handle:
    _h, _n, n = 16, 5, 5

env = ShapeEnv()
with FakeTensorMode(shape_env=env):
    t = torch.empty((env.create_unbacked_symint(), 3), device="cuda")
    b = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
for call in (lambda: epp.epp_backward_aggregate(Handle(), t, t), lambda: epp.epp_full_aggregate(Handle(), t, t),
             lambda: epp.epp_weight_gradient(Handle(), 0, t, t, t, b),
             lambda: epp.epp_weight_gradient_static(Handle(), 0, t, t, t),
             lambda: epp.epp_input_gradient(Handle(), 0, t, t, t)):
    try:
        call()
    except Exception:
        continue
    raise SystemExit("a tensor without sizes was accepted")
print("all refused")
"""


def test_tensors_of_unknown_shape_are_refused():
    import paper_2204_02662_amd as epp
    from paper_2204_02662_amd import build
    if not build.BINDING.exists():
        pytest.skip("binding not built")
    out = subprocess.run([sys.executable, "-c", SCRIPT], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and "all refused" in out.stdout, out.stdout[-500:] + out.stderr[-2000:]
