"""What the Python binding refuses before anything reaches the library (no GPU: tensors and library are stand-ins)."""
import os
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")


class Tensor:
    """A 2-D row-major tensor as far as the binding looks at one."""
    def __init__(self, rows, cols, ld=None, dtype=torch.float64, is_cuda=True, unit=1):
        self.shape, self.dtype, self.is_cuda, self.device = (rows, cols), dtype, is_cuda, "cuda"
        self.strides = (cols if ld is None else ld, unit)

    def dim(self):
        return 2

    def stride(self, i=None):
        return self.strides if i is None else self.strides[i]

    def data_ptr(self):
        return 4096

    def numel(self):
        return 1 << 40


@pytest.fixture
def oz(monkeypatch):
    from paper_2409_13313_amd import ozimmu

    class Library:
        calls = []

        def __getattr__(self, name):
            return lambda *args: self.calls.append((name, args)) or 0

    library = Library()
    library.calls.clear()
    monkeypatch.setattr(ozimmu, "_lib", library)
    monkeypatch.setattr(ozimmu, "_stream", lambda: 0)
    return ozimmu


CALLS = {"dgemm": lambda oz, A, B, D, ws: oz.dgemm(A, B, 8, D=D, workspace=ws),
         "dgemm_variant": lambda oz, A, B, D, ws: oz.dgemm_variant(A, B, 8, D=D, workspace=ws),
         "dgemm_profiled": lambda oz, A, B, D, ws: oz.dgemm_profiled(A, B, 8, D, ws, [None] * 3),
         "dgemm_resident": lambda oz, A, B, D, ws: oz.dgemm_resident(A, B, 8, 0, D=D, workspace=ws)}


@pytest.mark.parametrize("call", list(CALLS))
def test_an_output_that_cannot_hold_the_product_is_refused(oz, call):
    # (it would be written out of range)
    A, B, ws = Tensor(20, 30), Tensor(30, 40), Tensor(1, 1)
    for D in (Tensor(19, 40), Tensor(20, 39), Tensor(20, 39, ld=64), Tensor(40, 20), Tensor(20, 40, dtype=torch.float32),
              Tensor(20, 40, is_cuda=False), Tensor(20, 40, ld=40, unit=2)):
        with pytest.raises(ValueError):
            CALLS[call](oz, A, B, D, ws)
        assert oz._lib.calls == []


@pytest.mark.parametrize("call", list(CALLS))
def test_an_output_of_the_size_or_larger_is_taken_with_its_leading_dimension(oz, call):
    A, B, ws = Tensor(20, 30, ld=31), Tensor(30, 40), Tensor(1, 1)
    for D, ldd in ((Tensor(20, 40), 40), (Tensor(20, 40, ld=48), 48), (Tensor(25, 44), 44)):
        oz._lib.calls.clear()
        CALLS[call](oz, A, B, D, ws)
        (_, args), = oz._lib.calls
        assert args[:3] == (20, 30, 40) and args[4] == 31 and args[6] == 40 and args[8] == ldd


def test_the_functions_of_the_host_need_no_torch_with_a_gpu():
    code = ("import torch\n"
            "for name in ('_cuda_getDevice', '_cuda_getCurrentRawStream'):\n"
            "    if hasattr(torch._C, name): delattr(torch._C, name)\n"
            "from paper_2409_13313_amd import ozimmu\n"
            "assert ozimmu.params(1024) == (7, 128) and ozimmu.num_chunks(1024, 8) == 8\n")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    pr = subprocess.run([sys.executable, "-c", code], cwd=root, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert pr.returncode == 0, pr.stdout
