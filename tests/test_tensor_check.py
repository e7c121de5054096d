"""The binding's native argument check: it accepts exactly what the Python checks
accept, and leaves everything else (with the error to raise) to them."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2609_24456_amd import _tensor_check
from paper_2609_24456_amd import conduit as cd


def test_left_to_python_on_the_host():
    t = torch.zeros(8)
    for x in (t, t[::2], None, 3, "t", np.zeros(8), torch.empty(4, device="meta"), torch.nn.Parameter(t)):
        assert _tensor_check.address(x, torch.float32, None, None) is None
    with pytest.raises(TypeError):
        _tensor_check.address(t)
    with pytest.raises(ValueError, match="on a HIP device"):
        cd._ptr(t, torch.float32, "t")


def test_build_without_it(tmp_path, monkeypatch):
    from paper_2609_24456_amd import build as B
    old = tmp_path / "_tensor_check.so"
    old.write_bytes(b"an earlier build's")
    monkeypatch.setattr(B, "TENSOR_CHECK", str(old))
    monkeypatch.setattr(B, "CSRC", str(tmp_path))  # no source: the compiler fails
    with pytest.warns(UserWarning, match="checks in Python"):
        assert B.try_tensor_check() is None
    assert not old.exists()


@pytest.mark.parametrize("version", [None, "0.1"])
def test_module_of_another_torch_is_not_used(version):
    prog = f"""
import sys, types
m = types.ModuleType("paper_2609_24456_amd._tensor_check")
m.address = lambda *a: 1 / 0
if {version!r}: m.torch_version = {version!r}
sys.modules[m.__name__] = m
import paper_2609_24456_amd
from paper_2609_24456_amd import conduit as cd
assert cd._address(None, None, None, None) is None
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", prog], cwd=root, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]


def test_module_in_use_is_of_this_torch():
    assert _tensor_check.torch_version == torch.__version__
    assert cd._address is _tensor_check.address


@pytest.mark.gpu
def test_agrees_with_the_python_checks(monkeypatch):
    base = torch.zeros(24, dtype=torch.int32, device="cuda")
    tensors = [base, base[1:], base[:0], base.view(4, 6).t(), base.view(4, 6)[:, :3], base.view(torch.uint8), base.cpu(),
               torch.nn.Parameter(torch.zeros(24, device="cuda")), base.as_subclass(type("Sub", (torch.Tensor,), {})), "x"]
    dtypes = [None, torch.int32, torch.float32, torch.uint8, (torch.int32, torch.float32), (torch.int64, torch.uint64)]
    sizes = [(None, None), (96, None), (97, None), (None, 24), (None, 25), (np.int64(8), None), (0, 0)]

    def outcome(*a, **k):
        try:
            return cd._ptr(*a, **k)
        except (TypeError, ValueError) as e:
            return type(e), str(e)

    cases = [(t, d, s) for t in tensors for d in dtypes for s in sizes]
    native = [outcome(t, d, "t", nbytes=s[0], numel=s[1]) for t, d, s in cases]
    monkeypatch.setattr(cd, "_address", lambda *a: None)
    python = [outcome(t, d, "t", nbytes=s[0], numel=s[1]) for t, d, s in cases]
    assert native == python
    assert any(isinstance(x, int) for x in native) and any(isinstance(x, tuple) for x in native)
