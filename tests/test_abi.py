"""The C-ABI library loads and exports every function include/tsp.h declares (no GPU needed)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_functions():
    text = open(os.path.join(ROOT, "include", "tsp.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = re.findall(r"^\s*(?:const\s+char\s*\*\s*|int\s+)(tsp_\w+)\s*\(", text, flags=re.M)
    assert len(names) >= 14
    return names


def test_library_exports_every_declared_symbol():
    from paper_2009_14600_amd import tsp
    if not os.path.exists(tsp.LIB_PATH):
        from paper_2009_14600_amd.build import build_library
        build_library()
    lib = ctypes.CDLL(tsp.LIB_PATH)
    declared = _declared_functions()
    for name in declared:
        assert hasattr(lib, name), f"{name} is declared in tsp.h but not exported"
    assert sorted(declared) == sorted(tsp.EXPORTS)


def test_strerror_needs_no_gpu():
    from paper_2009_14600_amd import tsp
    lib = tsp.load_library()
    assert lib.tsp_strerror(0) == b"success"
    assert b"canonical" in lib.tsp_strerror(-3)
    assert lib.tsp_strerror(-99) == b"unknown status"


def test_binding_refuses_to_run_without_gpu():
    import torch
    from paper_2009_14600_amd import tsp
    if torch.cuda.is_available():
        pytest.skip("a GPU is present")
    with pytest.raises(RuntimeError):
        tsp.Handle()


def test_bench_refuses_more_than_one_gpu():
    """The path has no multi-GPU part: bench.py says so instead of running."""
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"],
                         capture_output=True, text=True, timeout=120)
    assert res.returncode == 2
    assert "one GPU" in res.stderr


def test_every_result_is_a_tensor_of_its_own():
    """Views of one block for results of one length share memory and nothing else: what a caller does to the shape or the
    flags of one in place does not show in the next."""
    import torch
    from paper_2009_14600_amd import tsp
    h = object.__new__(tsp.Handle)                # (the views alone: no library, no GPU)
    h._h = None
    h._torch, h._typed = torch, {}
    block = torch.zeros(4096, dtype=torch.uint8)
    h._blocks = {block.data_ptr(): block}
    first = h._view(block.data_ptr(), 100, torch.float32)
    first.fill_(2.0)
    first.requires_grad_(True)
    with torch.no_grad():
        first.unsqueeze_(0)
    second = h._view(block.data_ptr(), 100, torch.float32)
    assert second is not first and second.shape == (100,) and not second.requires_grad
    assert second.data_ptr() == first.data_ptr() and bool((second == 2.0).all())
    second.resize_(10)
    assert h._view(block.data_ptr(), 100, torch.float32).shape == (100,)
    assert h._view(block.data_ptr(), 7, torch.int64).shape == (7,)


def test_a_handle_is_destroyed_once(monkeypatch):
    """Also where a program that ends has lost the modules: __del__ closes again what a close before it did not come through."""
    from paper_2009_14600_amd import tsp
    destroyed = []

    class Lib:
        def tsp_destroy(self, handle):
            destroyed.append(handle)
            return 0
    h = object.__new__(tsp.Handle)
    h._lib, h._h, h._blocks, h._typed = Lib(), ctypes.c_void_p(16), {1: 2}, {}
    with monkeypatch.context() as gone:
        gone.setattr(tsp, "ctypes", None)
        try:
            h.close()
        except AttributeError:
            pass
        h.__del__()
    h.close()
    assert len(destroyed) == 1 and not h._blocks
