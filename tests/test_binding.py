"""The native argument marshalling of the per-chunk calls against the Python functions it stands for (no launch: the library
refuses these calls, or the arguments never reach it)."""
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2405_05329_amd import build, kvra


class Strange(torch.Tensor):
    pass


def _append(t, **other):
    args = dict(k_in=t, v_in=4096, q_inout=None, k_cache=4096, v_cache=4096, prefix_len=0, chunk_len=1, capacity=1,
                n_q_heads=1, n_kv_heads=1, head_dim=63, rope_base=1e4, stream=None, check=False)
    args.update(other)
    return kvra.kvra_append_kv(**args)


@pytest.mark.parametrize("make", [lambda: torch.zeros(4, 4), lambda: torch.nn.Parameter(torch.zeros(4)),
                                  lambda: torch.zeros(4, 4).t()[1:], lambda: torch.zeros(4).as_subclass(Strange),
                                  lambda: torch.zeros(4, 4).as_subclass(Strange).t()[1:]])
def test_tensors_that_may_not_be_passed_are_refused_as_by_the_python_function(make):
    t = make()
    with pytest.raises(ValueError) as want:
        kvra._ptr(t)
    with pytest.raises(ValueError) as got:
        _append(t)
    assert str(got.value) == str(want.value)


def test_numbers_addresses_and_streams():
    assert _append(4096) == kvra.KVRA_EUNSUPPORTED                       # (head_dim 63)
    assert _append(None) == kvra.KVRA_EINVAL
    assert _append(4096, prefix_len=np.int64(5), capacity=torch.tensor(3), head_dim=64.0) == kvra.KVRA_ERANGE
    assert _append(4096, rope_base=float("nan"), head_dim=64) == kvra.KVRA_EINVAL
    assert _append(4096, rope_base=np.float32("nan"), head_dim=True * 64) == kvra.KVRA_EINVAL
    assert _append(4096, chunk_len=(1 << 64) + 1) == kvra.KVRA_EUNSUPPORTED   # cut to 64 bits, as ctypes does

    class Stream:
        cuda_stream = 0

    assert _append(4096, stream=Stream()) == _append(4096, stream=0) == kvra.KVRA_EUNSUPPORTED
    with pytest.raises(kvra.KvraError):
        _append(4096, check=True)
    for bad in (dict(stream="x"), dict(chunk_len="x"), dict(chunk_len=None), dict(rope_base="x"), dict(k_cache="x")):
        with pytest.raises((TypeError, ValueError, AttributeError)):
            _append(4096, **bad)


def test_every_entry_point_reads_its_arguments_in_order():
    a = [4096 * (i + 1) for i in range(6)]
    assert kvra.kvra_chunk_attn(a[0], a[1], a[2], 0, 1, 3, 2, 64, 0.1, a[3], check=False) == kvra.KVRA_EINVAL
    assert kvra.kvra_chunk_attn(a[0], a[1], a[2], 0, 1, 2, 2, 60, 0.1, a[3], check=False) == kvra.KVRA_EUNSUPPORTED
    assert kvra.kvra_chunk_attn(a[0], a[1], a[2], 0, 1, 2, 2, 64, 0.1, None, check=False) == kvra.KVRA_EINVAL

    def code(call, *args):
        with pytest.raises(kvra.KvraError) as e:
            call(*args)
        return e.value.code

    assert code(kvra.kvra_rms_norm, a[0], a[1], a[2], 3, 60, 1e-6) == kvra.KVRA_EUNSUPPORTED
    assert code(kvra.kvra_rms_norm, a[0], a[1], a[2], 3, 64, -1.0) == kvra.KVRA_EINVAL
    assert code(kvra.kvra_linear, a[0], a[1], None, None, a[2], 8, 33, 64) == kvra.KVRA_EUNSUPPORTED
    assert code(kvra.kvra_linear, a[0], a[1], a[2], a[3], a[4], 8, 32, 64) == kvra.KVRA_EINVAL
    assert code(kvra.kvra_qkv_proj, a[0], a[1], a[2], a[3], a[4], 8, 2, 1, 64, 65) == kvra.KVRA_EUNSUPPORTED
    assert code(kvra.kvra_qkv_proj, a[0], a[1], a[2], a[3], None, 8, 2, 1, 64, 64) == kvra.KVRA_EINVAL
    layer = kvra.make_layer(64, 64, 1, 1, 64, 1e-6, 1e4, 0.1, *a, 4096)
    assert code(kvra.kvra_layer_chunk, layer, a[0], a[1], a[2], a[3], 5, 1, 5, a[4], 1 << 20) == kvra.KVRA_ERANGE
    assert code(kvra.kvra_layer_chunk, layer, a[0], a[1], a[2], a[3], 0, 1, 5, a[4], 8) == kvra.KVRA_EINVAL
    with pytest.raises(TypeError):
        kvra.kvra_layer_chunk(4096, a[0], a[1], a[2], a[3], 0, 1, 5, a[4], 1 << 20)


def test_the_native_module_is_the_one_in_use():
    assert os.path.exists(build.binding_path()), "build it with `python -m paper_2405_05329_amd.build`"
    assert kvra._call.__name__.endswith("._kvra_call") and kvra._call.__file__ == build.binding_path()


def test_ctypes_does_the_same(monkeypatch):
    monkeypatch.setattr(kvra, "_call", kvra._CtypesCalls)
    for make in (lambda: torch.zeros(4, 4), lambda: torch.zeros(4, 4).t()[1:], lambda: torch.zeros(4).as_subclass(Strange)):
        test_tensors_that_may_not_be_passed_are_refused_as_by_the_python_function(make)
    test_numbers_addresses_and_streams()
    test_every_entry_point_reads_its_arguments_in_order()


def test_a_package_without_a_module_for_this_torch_works_through_ctypes(tmp_path):
    """libkvra.so alone is enough, and a module that was built for another torch or Python is not loaded."""
    package = tmp_path / "paper_2405_05329_amd"
    package.mkdir()
    here = os.path.dirname(kvra.__file__)
    for name in ("__init__.py", "build.py", "kvra.py", "libkvra.so"):
        shutil.copy(os.path.join(here, name), package / name)
    for other in ("_kvra_call.so", os.path.basename(build.binding_path()).replace("torch-", "torch-9."),
                  os.path.basename(build.binding_path()).replace("cpython-3", "cpython-9")):
        (package / other).write_bytes(b"not for this interpreter")
    code = ("from paper_2405_05329_amd import kvra; print(kvra.__file__, kvra._call.__name__, "
            "kvra.kvra_append_kv(4096, 4096, None, 4096, 4096, 0, 1, 1, 1, 1, 63, 1e4, check=False))")
    r = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.split() == [str(package / "kvra.py"), "_CtypesCalls", str(kvra.KVRA_EUNSUPPORTED)]
