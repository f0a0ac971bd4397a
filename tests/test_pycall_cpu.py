"""The C module behind the binding: what it reads from its arguments and what it refuses, without a GPU (a null handle makes
every entry point answer before it looks at the device)."""

import ctypes
import os
import subprocess
import sys
import sysconfig

import numpy as np
import pytest
import torch

import paper_2603_02883_amd as F
from paper_2603_02883_amd import binding as B

X = torch.zeros((4, 64), dtype=torch.bfloat16)


def calls(o, x):
    c, m = torch.zeros((4, 32), dtype=torch.uint8), torch.zeros((4, 2), dtype=torch.int16)
    tg, sub = torch.zeros(4, dtype=torch.int32), torch.zeros((1, 8), dtype=torch.uint8)
    sal = torch.zeros(1, dtype=torch.int32)
    return {
        "quantize": lambda h: B._call.quantize(h, o, x, c, m, 0),
        "quantize_seda": lambda h: B._call.quantize_seda(h, o, x, tg, sub, c, m, 0),
        "quantize_decompose": lambda h: B._call.quantize_decompose(h, o, x, sal, tg, sub, c, m, c, m, 0),
        "dequantize": lambda h: B._call.dequantize(h, c, m, 32, None, None, None, x, 0, 0),
        "repack_mxfp8": lambda h: B._call.repack_mxfp8(h, c, m, 32, x.view(torch.uint8), m, 0),
        "layernorm_quantize": lambda h: B._call.layernorm_quantize(h, o, x, None, None, 1e-6, tg, sub, c, m, None, 0),
        "gelu_quantize": lambda h: B._call.gelu_quantize(h, o, x, 1, tg, sub, c, m, 0),
    }


def test_a_null_handle_is_an_invalid_argument():
    for handle in (None, 0, ctypes.c_void_p(None)):
        for name, call in calls(F.opts(), X).items():
            assert call(handle) == F.ERR_INVALID_ARG, name
    # two dimensions are what the matrices have, three what the scores' operands have
    q = torch.zeros((1, 0, 8), dtype=torch.bfloat16)
    assert B._call.attention_scores(q, q, 0, None, 0) == F.OK
    assert B._call.attention_scores(q, q, 2, None, 0) == F.ERR_INVALID_ARG


@pytest.mark.parametrize("x,error", [(torch.zeros(64), ValueError), (torch.zeros((1, 4, 64)), ValueError), (object(), AttributeError), (None, AttributeError)])
def test_what_is_no_matrix_is_refused(x, error):
    c = torch.zeros((4, 32), dtype=torch.uint8)
    with pytest.raises(error):
        B._call.quantize(None, F.opts(), x, c, c, 0)
    with pytest.raises(error):
        B._call.attention_scores(x if x is None or not isinstance(x, torch.Tensor) or x.dim() != 3 else x[0], x, 0, c, 0)


class Wider(B.fb4_opts):
    _fields_ = [("more", ctypes.c_int32)]


def test_handles_options_and_counts_are_checked():
    """By type, as ctypes checks the same arguments: neither any four or eight bytes are a handle nor any sixteen options."""
    for name, call in calls(F.opts(), X).items():
        for wrong in (ctypes.c_int32(1), ctypes.c_int64(0), ctypes.c_double(0.0), np.zeros(1, np.int64), np.int64(0), 0.0, X):
            with pytest.raises(ctypes.ArgumentError):
                call(wrong)
        for null in (False, ctypes.POINTER(ctypes.c_int)()):
            assert call(null) == F.ERR_INVALID_ARG, name
    for wrong, error in ((bytes(16), TypeError), (np.zeros(4, np.int32), TypeError), (None, TypeError), (ctypes.byref(F.opts()), TypeError),
                         ((ctypes.c_int32 * 4)(), ctypes.ArgumentError), (ctypes.pointer(F.opts()), ctypes.ArgumentError)):
        for name, call in calls(wrong, X).items():
            if name not in ("dequantize", "repack_mxfp8"):
                with pytest.raises(error):
                    call(None)
    for name, call in calls(Wider(32, F.SEL_LUT, 8, 0, 5), X).items():
        assert call(None) == F.ERR_INVALID_ARG, name
    with pytest.raises(TypeError):
        B._call.quantize(None, F.opts(), X)
    for call in (lambda h: B._call.quantize_seda(h, F.opts(), X, None, None, None, None, 0),
                 lambda h: B._call.quantize_decompose(h, F.opts(), X, None, None, None, None, None, None, None, 0)):
        with pytest.raises(AttributeError):  # these lists have to be there
            call(None)


class Like:
    """What has a tensor's methods."""

    def __init__(self, shape):
        self.shape = shape

    def data_ptr(self):
        return 64

    def stride(self, dim):
        return 64


def test_numbers_and_shapes_are_read_as_before():
    c, m = torch.zeros((4, 32), dtype=torch.uint8), torch.zeros((4, 2), dtype=torch.int16)
    for block, error in ((32, None), (np.int64(32), None), (2**70, None), (32.0, ctypes.ArgumentError), (None, ctypes.ArgumentError)):
        for call in (lambda: B._call.dequantize(None, c, m, block, None, None, None, X, 0, 0), lambda: B._call.repack_mxfp8(None, c, m, block, c, m, 0)):
            if error is None:
                assert call() == F.ERR_INVALID_ARG
            else:
                with pytest.raises(error):
                    call()
    for eps in (1, 1e-6, "1e-6", np.float32(1e-6), torch.tensor(1e-6)):
        assert B._call.layernorm_quantize(None, F.opts(), X, None, None, eps, None, None, c, m, None, 0) == F.ERR_INVALID_ARG
    for shape in ((4, 64), [4, 64], np.array([4, 64])):
        assert B._call.quantize(None, F.opts(), Like(shape), c, m, 0) == F.ERR_INVALID_ARG
    with pytest.raises(ctypes.ArgumentError):
        B._call.quantize(None, F.opts(), Like((4.0, 64)), c, m, 0)


def test_the_module_is_this_interpreters_and_not_needed(tmp_path):
    """Its file carries the interpreter's tag; without it and without what builds it the same calls go through ctypes, and the
    library that is there is not compiled again."""
    assert os.path.basename(B._build.CALL) == "_fb4call" + sysconfig.get_config_var("EXT_SUFFIX") != "_fb4call.so"
    assert B._call.__name__.endswith("_fb4call") and B._call.__file__ == B._build.CALL
    package = os.path.dirname(B.__file__)
    root = tmp_path / "paper_2603_02883_amd"
    root.mkdir()
    for f in ("__init__.py", "binding.py", "build.py", "csrc", "libfb4.so"):
        os.symlink(os.path.join(package, f), root / f)
    os.symlink(os.path.join(os.path.dirname(package), "include"), tmp_path / "include")
    (root / "_fb4call.so").write_bytes(b"another interpreter's")
    program = ("import torch, paper_2603_02883_amd as F; from paper_2603_02883_amd import binding as B; "
               "print(B._call is B.CtypesCall, B._call.quantize(None, F.opts(), torch.zeros((2, 32)), None, None, 0))")
    for env, through_ctypes in (({"CC": "no-such-compiler"}, True), ({"CC": "false"}, True), ({}, False)):
        r = subprocess.run([sys.executable, "-c", program], cwd=tmp_path, capture_output=True, text=True,
                           env=dict(os.environ, PYTHONPATH=str(tmp_path), HIPCC="false", **env))
        assert r.returncode == 0 and r.stdout.split() == [str(through_ctypes), str(F.ERR_INVALID_ARG)], r.stderr
    assert not (root / "_build").exists() and sorted(f.name for f in root.iterdir() if f.name.startswith("_fb4call")) == [
        os.path.basename(B._build.CALL), "_fb4call.so"]


def test_calls_through_ctypes_answer_like_the_modules():
    for o, h in ((F.opts(), None), (F.opts(), ctypes.c_void_p(1)), (F.opts(block=5), ctypes.c_void_p(1))):
        for name, call in calls(o, X).items():
            if h is None or (name not in ("dequantize", "repack_mxfp8") and o.block == 5):
                got = call(h)
                try:
                    B._call, module = B.CtypesCall, B._call
                    assert call(h) == got == F.ERR_INVALID_ARG, name
                finally:
                    B._call = module
