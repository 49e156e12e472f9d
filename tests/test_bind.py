"""The native argument marshalling (_rv_bind): the same addresses, and the same refusals, as
the checks written in Python."""
import ctypes

import pytest
import torch

from paper_2609_23286_amd import rv

SHAPE = (5, 2, 64)


def outcome(f, *args):
    try:
        return f(*args)
    except Exception as e:  # the type and the words are what a caller sees
        return type(e), str(e)


class Sub(torch.Tensor):
    pass


FORMS = {
    "none": lambda d: None,
    "address": lambda d: 4096,
    "not a tensor": lambda d: "K",
    "ctypes pointer": lambda d: ctypes.c_void_p(64),
    "bf16": lambda d: torch.zeros(SHAPE, dtype=torch.bfloat16, device=d),
    "int16": lambda d: torch.zeros(SHAPE, dtype=torch.int16, device=d),
    "fp32": lambda d: torch.zeros(SHAPE, device=d),
    "other shape": lambda d: torch.zeros((5, 64, 2), dtype=torch.int16, device=d),
    "fewer dims": lambda d: torch.zeros((10, 64), dtype=torch.int16, device=d),
    "empty": lambda d: torch.zeros((0, 2, 64), dtype=torch.int16, device=d),
    "offset view": lambda d: torch.zeros((6, 2, 64), dtype=torch.int16, device=d)[1:],
    "transposed": lambda d: torch.zeros((2, 5, 64), dtype=torch.int16, device=d).transpose(0, 1),
    "strided": lambda d: torch.zeros((5, 2, 128), dtype=torch.int16, device=d)[..., ::2],
    "subclass": lambda d: torch.zeros(SHAPE, dtype=torch.int16, device=d).as_subclass(Sub),
    "parameter": lambda d: torch.nn.Parameter(torch.zeros(SHAPE, dtype=torch.bfloat16, device=d)),
    "meta": lambda d: torch.zeros(SHAPE, dtype=torch.int16, device="meta"),
    "sparse": lambda d: torch.zeros(SHAPE, dtype=torch.bfloat16, device=d).to_sparse(),
}


def check_form(form, device):
    x = FORMS[form](device)
    want = outcome(rv._ptr_python, x, SHAPE, 2, "K")
    assert outcome(rv._ptr, x, SHAPE, 2, "K") in ((want, 0) if want is None else (want,))
    want3 = outcome(rv._ptr_python, x, SHAPE, 2, "K[1]")
    got = outcome(rv._ptrs, [None, x], 3, SHAPE, 2, "K")
    if isinstance(want3, tuple):
        assert got == want3
    else:
        assert list((ctypes.c_uint64 * 3).from_buffer_copy(got)) == [0, want3 or 0, 0]


@pytest.mark.parametrize("form", FORMS)
def test_address_and_refusals_cpu(form):
    check_form(form, "cpu")


@pytest.mark.gpu
@pytest.mark.parametrize("form", FORMS)
def test_address_and_refusals_gpu(form):
    check_form(form, "cuda")


def test_lists():
    assert outcome(rv._ptrs, [1, 2, 3], 2, SHAPE, 2, "K") == (IndexError, "invalid index")
    assert outcome(rv._ptrs, (7,), 1, SHAPE, 2, "K") == (7).to_bytes(8, "little")
    assert outcome(rv._ptrs, 7, 1, SHAPE, 2, "K")[0] is TypeError
    assert outcome(rv._ptrs, (x for x in (7, 9)), 2, SHAPE, 2, "K") == (7 + (9 << 64)).to_bytes(16, "little")


def test_closed_memory_is_refused():
    m = rv.Memory.__new__(rv.Memory)
    m.handle, m.n_heads = None, 2
    want = outcome(rv.Memory.view, m)
    assert want[0] is rv.RVError and outcome(rv._mem_state, m) == want


def test_another_torch_or_a_broken_module_is_refused(tmp_path, monkeypatch):
    assert torch.__version__.startswith(rv._load_bind().built_for[0])
    with monkeypatch.context() as m:
        m.setattr(torch, "__version__", "1.0.0+rocm7.0")
        with pytest.raises(ImportError, match=r"built for another torch.*1\.0\.0.*build\(\)"):
            rv._load_bind()
    (tmp_path / "_rv_bind.so").write_bytes(b"not a module")
    monkeypatch.setattr(rv, "BIND_PATH", str(tmp_path / "_rv_bind.so"))
    with pytest.raises(ImportError, match=r"build\(\)"):
        rv._load_bind()


@pytest.mark.gpu
def test_default_stream_is_the_current_one(monkeypatch):
    s = torch.cuda.Stream()
    for raw in (rv._raw_stream, None):      # (with and without the short way)
        monkeypatch.setattr(rv, "_raw_stream", raw)
        assert rv._stream(None) == torch.cuda.current_stream().cuda_stream
        with torch.cuda.stream(s):
            assert rv._stream(None) == s.cuda_stream
