"""The native argument marshalling reads a torch.Tensor itself and anything else through its methods: both ways have to see the
same pointers, sizes, strides, types and byte counts, and to refuse the same objects.  Every call here is refused before a launch."""
import ctypes
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")
import torch.overrides  # noqa: E402

from paper_2601_12212_amd import _dtcall, binding  # noqa: E402
from tests.conftest import ROOT  # noqa: E402


class Duck:
    """A tensor's methods, and not its type."""

    def __init__(self, t):
        self._t = t

    def __getattr__(self, name):
        return getattr(self._t, name)


class Derived(torch.Tensor):
    pass


@pytest.fixture
def call():
    binding._native()
    reader = binding._tensor_reader(torch.__version__)
    assert reader is not None                       # else both ways are one
    _dtcall.set_reader(reader)
    _dtcall.setup(torch.float32, torch.bfloat16, lambda: 0, lambda device: 0)
    yield _dtcall
    _dtcall.setup(torch.float32, torch.bfloat16, torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream)


def _rows(**kw):
    """Arguments of topk_rows: refused for want of a workspace unless something else is wrong first."""
    a = dict(logits=torch.zeros(4, 64), k=3, val=torch.zeros(4, 3), id=torch.zeros(4, 3, dtype=torch.int32), lse=torch.zeros(4),
             ws=torch.zeros(1024, dtype=torch.uint8))
    a.update(kw)
    return list(a.values())


aligned = torch.zeros(4096, dtype=torch.uint8)
aligned = aligned[-aligned.data_ptr() % 256:][:1024]
CASES = {
    "a workspace too small": _rows(ws=aligned[:256], logits=torch.zeros(2, 40000, dtype=torch.bfloat16)),
    "a misaligned workspace": _rows(ws=aligned[1:], logits=torch.zeros(2, 40000)),
    "no workspace": _rows(ws=None, logits=torch.zeros(2, 40000)),
    "rows that overlap": _rows(logits=torch.zeros(512).as_strided((4, 64), (32, 1))),
    "no output": _rows(val=None),
    "too many of a row": _rows(k=400),
    "an integer type": _rows(logits=torch.zeros(4, 64, dtype=torch.int32)),
    "half precision": _rows(logits=torch.zeros(4, 64, dtype=torch.float16)),
    "one dimension": _rows(logits=torch.zeros(64)),
    "three dimensions": _rows(logits=torch.zeros(2, 4, 64)),
    "no dimension": _rows(logits=torch.zeros(())),
    "no storage": _rows(logits=torch.zeros(4, 64).to_sparse()),
    "not a tensor": _rows(logits=7),
}


def _outcome(call, args):
    try:
        return call.topk_rows(*args)
    except Exception as e:  # noqa: BLE001
        return type(e), str(e)


@pytest.mark.parametrize("name", CASES)
def test_tensors_and_other_objects_are_read_alike(call, name):
    args = CASES[name]
    want = _outcome(call, [Duck(a) if isinstance(a, torch.Tensor) else a for a in args])
    assert want != 0
    assert _outcome(call, args) == want
    assert _outcome(call, [a.as_subclass(Derived) if isinstance(a, torch.Tensor) and a.layout == torch.strided else a
                           for a in args]) == want


class Redirected(torch.overrides.TorchFunctionMode):
    """Sees every tensor function that the marshalling calls and answers data_ptr() itself."""

    def __init__(self):
        super().__init__()
        self.seen = set()

    def __torch_function__(self, func, types, args=(), kwargs=None):
        self.seen.add(getattr(func, "__name__", str(func)))
        if func is torch.Tensor.data_ptr:
            return 0
        return func(*args, **(kwargs or {}))


def test_an_active_torch_function_mode_is_asked(call):
    args = CASES["a misaligned workspace"]
    plain = _outcome(call, args)
    no_pointers = _outcome(call, [None if isinstance(a, torch.Tensor) and a is not args[0] else a for a in args])
    with Redirected() as mode:
        got = _outcome(call, args)
    assert {"data_ptr", "stride"} <= mode.seen, mode.seen
    assert got != plain and got == no_pointers     # the mode's answers went into the call
    assert _outcome(call, args) == plain


def test_the_marshalling_needs_no_torch():
    code = ("import sys\n"
            "from paper_2601_12212_amd import _dtcall\n"
            "assert 'torch' not in sys.modules\n"
            "class T:\n"
            "    shape, dtype, nbytes = (4, 64), 'bf16', 512\n"
            "    def data_ptr(self): return 0\n"
            "    def stride(self, dim): return 64\n"
            "_dtcall.setup('f32', 'bf16', lambda: 0, lambda device: 0)\n"
            "print(_dtcall.topk_rows(T(), 3, T(), T(), T(), None))\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    assert r.stdout.split() == ["-1"]               # null pointers


def test_another_torch_is_named_and_its_tensors_read_through_their_methods(call):
    with pytest.warns(RuntimeWarning, match="no tensor reader for torch 0.0.0"):
        reader = binding._tensor_reader("0.0.0")
    assert reader is None
    want = {name: _outcome(call, args) for name, args in CASES.items()}
    call.set_reader(None)
    for name, args in CASES.items():
        assert _outcome(call, args) == want[name], name


def test_what_is_not_a_reader_is_refused(call):
    with pytest.raises(ValueError):
        call.set_reader(7)


PyObject, Int, Long, LL = ctypes.py_object, ctypes.c_int, ctypes.c_long, ctypes.c_longlong
READER = [("overridden", ctypes.PYFUNCTYPE(Int)),
          ("data_ptr", ctypes.PYFUNCTYPE(Int, PyObject, ctypes.POINTER(ctypes.c_void_p))),
          ("sizes", ctypes.PYFUNCTYPE(Int, PyObject, Int, Int, ctypes.POINTER(LL))),
          ("stride", ctypes.PYFUNCTYPE(Int, PyObject, Long, ctypes.POINTER(LL))),
          ("dtype", ctypes.PYFUNCTYPE(Int, PyObject, ctypes.POINTER(Int))),
          ("nbytes", ctypes.PYFUNCTYPE(Int, PyObject, ctypes.POINTER(ctypes.c_size_t)))]


class Table(ctypes.Structure):
    _fields_ = READER


@pytest.fixture
def table():
    get = ctypes.PYFUNCTYPE(ctypes.c_void_p, PyObject, ctypes.c_char_p)(("PyCapsule_GetPointer", ctypes.pythonapi))
    capsule = binding._tensor_reader(torch.__version__)
    t = Table.from_address(get(capsule, b"paper_2601_12212_amd.tensor_reader"))
    t.capsule = capsule
    return t


base = torch.zeros(6, 8, 10)
TENSORS = {
    "whole": base,
    "a view with an offset": base[2:, 3:5],
    "transposed": base.permute(2, 0, 1),
    "every third column": base[..., ::3],
    "expanded": base[:1].expand(5, 8, 10),
    "an empty one": base[:, :0],
    "no dimension": torch.zeros(()),
    "one dimension": torch.zeros(7, dtype=torch.bfloat16)[1:],
    "bfloat16, strided": torch.zeros(4, 64, dtype=torch.bfloat16).as_strided((3, 16), (20, 2), 5),
    "with a gradient": torch.zeros(3, 4, requires_grad=True),
    "integers": torch.zeros(3, 4, dtype=torch.int32),
    "half precision": torch.zeros(3, 4, dtype=torch.float16),
    "more than 2^31 bytes": torch.zeros(1).expand(3, 1 << 30),
}


@pytest.mark.parametrize("name", TENSORS)
def test_the_reader_says_what_the_methods_say(table, name):
    x = TENSORS[name]
    p, v, n, bf16 = ctypes.c_void_p(), LL(), ctypes.c_size_t(), Int(-1)
    assert table.overridden() == 0
    assert table.data_ptr(x, p) == 1 and (p.value or 0) == x.data_ptr()
    assert table.nbytes(x, n) == 1 and n.value == x.nbytes
    for dim in range(-x.dim(), x.dim()):
        assert table.stride(x, dim, v) == 1 and v.value == x.stride(dim)
    assert table.stride(x, x.dim(), v) == 0                   # the method says what is wrong
    for want in range(x.dim() + 2):
        out = (LL * 8)(*[-7] * 8)
        assert table.sizes(x, want, 1, out) == (want == x.dim())
        assert list(out) == (list(x.shape) if want == x.dim() else []) + [-7] * (8 - x.dim() * (want == x.dim()))
        assert table.sizes(x, want, 0, out) == (want <= x.dim())
        if want <= x.dim():
            assert list(out)[:want] == list(x.shape)[:want]
    assert table.dtype(x, bf16) == (x.dtype in (torch.float32, torch.bfloat16))
    if x.dtype in (torch.float32, torch.bfloat16):
        assert bf16.value == (x.dtype == torch.bfloat16)


@pytest.mark.parametrize("x", [7, None, Duck(base), base.as_subclass(Derived), torch.nn.Parameter(torch.zeros(3))],
                         ids=["int", "None", "duck", "derived", "parameter"])
def test_the_reader_leaves_other_objects_to_their_methods(table, x):
    p, v, n, bf16 = ctypes.c_void_p(), LL(), ctypes.c_size_t(), Int()
    assert table.data_ptr(x, p) == table.nbytes(x, n) == table.stride(x, 0, v) == table.dtype(x, bf16) == 0
    assert table.sizes(x, 1, 0, v) == 0
