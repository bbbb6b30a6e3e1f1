"""The native call path leaves to the Python checks every call that they would not pass,
here on the CPU: no tensor is on a GPU, so nothing may be taken, and the errors are those
of the Python path."""
import pytest
import torch

from paper_2607_09207_amd import DecodeAttention, RldaError


def layer(kv="bf16"):
    return DecodeAttention(8, 2, 128, 4, 8, "bf16", kv, "f32")


def args():
    q = torch.zeros((2, 8, 128), dtype=torch.bfloat16)
    k = torch.zeros((5, 2, 16, 128), dtype=torch.bfloat16)
    return q, k, k.clone(), torch.zeros((2, 8), dtype=torch.int32), torch.ones(2, dtype=torch.int32)


def test_cpu_tensors_and_other_objects_are_not_taken():
    h = layer()
    q, k, v, bt, sl = args()
    for a in [(q, k, v, bt, sl), (None,) * 5, (1, "k", v, bt, sl), (q[0], k, v, bt, sl)]:
        assert h._fast.run(*a, None, None, None, None, None, None) is None
        assert h._fast.noalloc(*a, None, None, None, None, None, None) is None
        assert h._fast.grouped(*a, None, None, None, None, None, None, 2, sl, -1) is None
        assert h._fast.multi(*a, None, None, None, None, None, None, sl, 0) is None
        assert h._fast.append(a[0], *a[1:], None, None, None, None, q, None) is None
    with pytest.raises(TypeError):
        h._fast.run(q)


def test_errors_are_those_of_the_python_checks():
    h = layer()
    q, k, v, bt, sl = args()
    for call in (lambda: h(q, k, v, bt, sl), lambda: h.run_noalloc(q, k, v, bt, sl),
                 lambda: h.multi(q, k, v, bt, sl, torch.zeros(3, dtype=torch.int32)),
                 lambda: h.append(q[:, :2].contiguous(), q[:, :2].contiguous(), k, v, bt, sl)):
        with pytest.raises(RldaError, match="must be on a GPU"):
            call()


def test_without_the_native_path_the_python_path_takes_every_call(monkeypatch):
    import sys

    import paper_2607_09207_amd as pkg
    from paper_2607_09207_amd import _abi
    monkeypatch.setattr(_abi, "_fast", None)
    monkeypatch.delattr(pkg, "_fastcall", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2607_09207_amd._fastcall", None)   # the import fails
    with pytest.warns(RuntimeWarning, match="native call path"):
        h = layer()
    layer()   # warned once
    q, k, v, bt, sl = args()
    for call in (lambda: h(q, k, v, bt, sl), lambda: h.run_noalloc(q, k, v, bt, sl),
                 lambda: h(q, k, v, bt, sl, group_size=2, prefix_pages=sl),
                 lambda: h.multi(q, k, v, bt, sl, torch.zeros(3, dtype=torch.int32)),
                 lambda: h.append(q[:, :2].contiguous(), q[:, :2].contiguous(), k, v, bt, sl)):
        with pytest.raises(RldaError, match="must be on a GPU"):
            call()


def test_a_destroyed_layer_keeps_no_handle_in_the_native_path():
    from paper_2607_09207_amd import _abi
    h = layer()
    assert isinstance(h._fast, _abi.fastcall().Layer)
    h.__del__()
    assert h._h is None and h._fast is _abi.LEFT_TO_PYTHON
