"""The native part of the binding: what it takes itself and what it leaves to the Python form."""
import os
import shutil
import subprocess
import sys

import pytest
import torch

from paper_2505_14201_amd import flashd

NATIVE = flashd._native


def tensors(device="cpu", dtype=torch.bfloat16, d=64):
    return [torch.zeros(1, h, n, d, dtype=dtype, device=device) for h, n in ((4, 3), (2, 40), (2, 40), (4, 3))]


def test_the_native_part_is_built_for_this_torch_and_python():
    assert NATIVE.built_for == f"torch {torch.__version__} and Python 3.{sys.version_info[1]}"


def test_anything_but_gpu_tensors_is_left_to_the_python_form():
    q, k, v, o = tensors()
    assert NATIVE.attn_fwd(q, k, v, o, True, 1.0) is None
    assert NATIVE.attn_fwd(1, "k", None, [], True, 1.0) is None
    assert NATIVE.attn_fwd(q, k, v) is None
    assert NATIVE.attn_fwd_kv8(q, k, v, o, True, 1.0, 1.0, 1.0) is None
    assert NATIVE.attn_fwd_state(q, k, v, True, 1.0, o, None, None, None) is None
    for call in (lambda: flashd.attn_fwd(q, k, v, o, True, 1.0),
                 lambda: flashd.attn_fwd_kv8(q, k, v, o, True, 1.0, 1.0, 1.0),
                 lambda: flashd.attn_fwd_state(q, k, v, True, 1.0, o=o)):
        with pytest.raises(ValueError, match="GPU"):
            call()


@pytest.mark.parametrize("there", [False, True])
def test_the_package_works_without_its_native_part(tmp_path, there):
    """Missing, or there and not loadable (built for another Python or torch): a warning that says which,
    and the same calls, checks and messages through ctypes."""
    pkg = os.path.dirname(flashd.__file__)
    shutil.copytree(pkg, tmp_path / "paper_2505_14201_amd", ignore=shutil.ignore_patterns(
        "csrc", "__pycache__", "_flashd_binding*", "libflashd.so"))
    os.symlink(os.path.join(pkg, "libflashd.so"), tmp_path / "paper_2505_14201_amd" / "libflashd.so")
    if there:
        (tmp_path / "paper_2505_14201_amd" / "_flashd_binding.so").write_bytes(b"not a shared object")
    code = """
import warnings
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    from paper_2505_14201_amd import flashd
assert [w for w in seen if w.category is RuntimeWarning and "ctypes" in str(w.message)], seen
import torch
q = torch.zeros(1, 4, 3, 64)
for call in (lambda: flashd.attn_fwd(q, q, q, q, True, 1.0),
             lambda: flashd.attn_fwd_kv8(q, q, q, q, True, 1.0, 1.0, 1.0),
             lambda: flashd.attn_fwd_state(q, q, q, True, 1.0, o=q)):
    try:
        call()
    except ValueError as e:
        assert "GPU" in str(e)
    else:
        raise AssertionError
assert flashd.version() >= 100
"""
    subprocess.run([sys.executable, "-c", code], check=True, cwd=tmp_path)


@pytest.mark.gpu
def test_arguments_out_of_the_ordinary_are_refused_or_taken_as_before():
    q, k, v, o = tensors("cuda")
    bad = [(q.float(), k, v, o), (q, k.half(), v, o), (q, k, v[:, :, :39], o), (q, k, v, o[:, :2]),
           (q[0], k, v, o), (q.cpu(), k, v, o), (q, k.transpose(2, 3), v, o), (q, k, v, o.to(torch.float64))]
    for args in bad:
        assert NATIVE.attn_fwd(*args, True, 1.0) is None
        with pytest.raises(ValueError):
            flashd.attn_fwd(*args, True, 1.0)
    assert NATIVE.attn_fwd(q, k, v, o, True, "1") is None
    # the library's own refusals come through as statuses
    d32 = tensors("cuda", d=32)
    assert NATIVE.attn_fwd(*d32, True, 1.0) == -4
    with pytest.raises(flashd.FlashdError) as e:
        flashd.attn_fwd(*d32, True, 1.0)
    assert e.value.status == -4
    assert NATIVE.attn_fwd_state(q, k, v, True, 1.0, o, None, None, 2.5) is None
    assert NATIVE.attn_fwd_state(q, k, v, True, 1.0, o, o, None, None) is None


@pytest.mark.gpu
def test_both_forms_make_the_same_call():
    gen = torch.Generator().manual_seed(5)
    q, k, v, o = [torch.randn(t.shape, generator=gen).to(torch.bfloat16).cuda() for t in tensors()]
    side = torch.cuda.Stream()
    want = torch.empty_like(o)
    flashd.attn_fwd(q, k, v, want, True, 0.1, stream=torch.cuda.current_stream())   # the Python form
    torch.cuda.synchronize()
    flashd.attn_fwd(q, k, v, o, 1, 0.1)
    torch.cuda.synchronize()
    assert torch.equal(o, want)
    o.zero_()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):                       # the current stream is asked for on every call
        flashd.attn_fwd(q, k, v, o, True, 0.1)
    side.synchronize()
    assert torch.equal(o, want)
    st = torch.empty(1, 4, 3, 66, device="cuda")
    st2 = torch.empty_like(st)
    flashd.attn_fwd_state(q, k, v, True, 0.1, state_out=st, causal_shift=5)
    flashd.attn_fwd_state(q, k, v, True, 0.1, state_out=st2, causal_shift=5, stream=torch.cuda.current_stream())
    k8, v8 = k.to(torch.float8_e4m3fn), v.to(torch.float8_e4m3fn)
    o2 = torch.empty_like(o)
    flashd.attn_fwd_kv8(q, k8, v8, o, True, 0.1, 0.5, 2.0)
    flashd.attn_fwd_kv8(q, k8, v8, o2, True, 0.1, 0.5, 2.0, stream=torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert torch.equal(st, st2) and torch.equal(o, o2)
