"""The C module behind the binding: what it reads from its arguments and what it refuses, without a GPU (a null handle makes
every entry point answer before it looks at the device)."""

import ctypes
import importlib.machinery
import importlib.util
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


class Stream:
    cuda_stream = 0


@pytest.mark.parametrize("through_ctypes", [False, True])
def test_the_refresh_refuses_by_the_same_errors_with_outputs_given(monkeypatch, through_ctypes):
    if through_ctypes:
        monkeypatch.setattr(B, "_call", B.CtypesCall)
    gh, gw, frames, heads, dim = 4, 6, 3, 5, 16
    sc, ts = torch.zeros((frames, heads, gh * gw)), torch.zeros((gh * gw, heads, frames))
    qt, cand = torch.zeros((gh * gw, heads, frames, dim), dtype=torch.bfloat16), torch.zeros((frames, 2), dtype=torch.int32)
    main, s = torch.zeros(2, dtype=torch.int32), Stream()
    for out in (None, cand):
        for th, tw, error in ((0, 4, ZeroDivisionError), (4, 0, ZeroDivisionError), (None, 4, TypeError), (4, "4", TypeError)):
            with pytest.raises(error):
                B.fb4_select_salient_tokens(sc, gh, gw, th, tw, rows_out=out, stream=s)
            for kw in (dict(main_anchor=None if out is None else main, kept=out), dict(main_anchor=main), dict(kept=cand)):
                with pytest.raises(error):
                    B.fb4_seda_main_anchor(ts, qt, qt, cand, gh, gw, th, tw, stream=s, **kw)
        with pytest.raises(B.Fb4Error):
            B.fb4_select_salient_tokens(sc, gh, gw, -1, 4, rows_out=cand, stream=s)
        for kw in (dict(kept=out), dict(main_anchor=main, kept=out)):
            with pytest.raises(AssertionError):
                B.fb4_seda_main_anchor(ts, qt, qt, cand[1:], gh, gw, stream=s, **kw)
            with pytest.raises(AttributeError):
                B.fb4_seda_main_anchor(ts, qt, qt, None, gh, gw, stream=s, **kw)


RECORDER = r"""
#include <stdint.h>
#include "fb4.h"
int64_t seen[20];
#define P(i, v) seen[i] = (int64_t)(uintptr_t)(v)
#define N(i, v) seen[i] = (int64_t)(v)
#define OPTIONS(o) N(18, (((o)->block * 100 + (o)->selector) * 100 + (o)->num_groups) * 100 + (o)->flags)
int fb4_quantize(const fb4_luts* l, const fb4_opts* o, const void* x, int64_t r, int64_t c, int64_t st, uint8_t* co, uint16_t* m, void* s)
{ P(0, x); N(1, r); N(2, c); N(3, st); P(4, co); P(5, m); P(16, s); P(17, l); OPTIONS(o); return 0; }
int fb4_quantize_seda(const fb4_luts* l, const fb4_opts* o, const void* x, int64_t r, int64_t c, int64_t st, const int32_t* tg, const uint8_t* sub, int g,
                      uint8_t* co, uint16_t* m, void* s)
{ P(0, x); N(1, r); N(2, c); N(3, st); P(4, tg); P(5, sub); N(6, g); P(7, co); P(8, m); P(16, s); P(17, l); OPTIONS(o); return 0; }
int fb4_quantize_decompose(const fb4_luts* l, const fb4_opts* o, const void* x, int64_t r, int64_t c, int64_t st, const int32_t* tg, const uint8_t* sub, int g,
                           const int32_t* sal, int64_t n, uint8_t* c1, uint16_t* m1, uint8_t* c2, uint16_t* m2, void* s)
{ P(0, x); N(1, r); N(2, c); N(3, st); P(4, tg); P(5, sub); N(6, g); P(7, sal); N(8, n); P(9, c1); P(10, m1); P(11, c2); P(12, m2); P(16, s); P(17, l); OPTIONS(o); return 0; }
int fb4_dequantize(const fb4_luts* l, const uint8_t* c1, const uint16_t* m1, int64_t r, int64_t c, int b, const uint8_t* c2, const uint16_t* m2,
                   const int32_t* sal, int64_t n, void* out, int dt, int64_t st, void* s)
{ P(0, c1); P(1, m1); N(2, r); N(3, c); N(4, b); P(5, c2); P(6, m2); P(7, sal); N(8, n); P(9, out); N(10, dt); N(11, st); P(16, s); P(17, l); return 0; }
int fb4_repack_mxfp8(const fb4_luts* l, const uint8_t* co, const uint16_t* m, int64_t r, int64_t c, int b, uint8_t* e, int64_t st, uint8_t* sc, void* s)
{ P(0, co); P(1, m); N(2, r); N(3, c); N(4, b); P(5, e); N(6, st); P(7, sc); P(16, s); P(17, l); return 0; }
int fb4_layernorm_quantize(const fb4_luts* l, const fb4_opts* o, const void* x, int64_t r, int64_t c, int64_t st, const float* ga, const float* be, float eps,
                           const int32_t* tg, const uint8_t* sub, int g, uint8_t* co, uint16_t* m, void* y, void* s)
{ P(0, x); N(1, r); N(2, c); N(3, st); P(4, ga); P(5, be); P(6, tg); P(7, sub); N(8, g); P(9, co); P(10, m); P(11, y); P(16, s); P(17, l); OPTIONS(o); N(19, eps * 1099511627776.0f); return 0; }
int fb4_gelu_quantize(const fb4_luts* l, const fb4_opts* o, const void* x, int64_t r, int64_t c, int64_t st, int a, const int32_t* tg, const uint8_t* sub, int g,
                      uint8_t* co, uint16_t* m, void* s)
{ P(0, x); N(1, r); N(2, c); N(3, st); N(4, a); P(5, tg); P(6, sub); N(7, g); P(8, co); P(9, m); P(16, s); P(17, l); OPTIONS(o); return 0; }
int fb4_attention_scores(const void* q, const void* k, int64_t g, int64_t t, int64_t d, int mode, float* out, void* s)
{ P(0, q); P(1, k); N(2, g); N(3, t); N(4, d); N(5, mode); P(6, out); P(16, s); return 0; }
int fb4_select_salient_tokens(const float* sc, int64_t f, int h, int gh, int gw, int th, int tw, int32_t* out, void* s)
{ P(0, sc); N(1, f); N(2, h); N(3, gh); N(4, gw); N(5, th); N(6, tw); P(7, out); P(16, s); return 0; }
int fb4_seda_assign(const void* q, const void* k, int j, int64_t f, int h, int gh, int gw, int64_t d, const int32_t* an, int64_t n, int th, int tw, int w,
                    int wt, float t, int32_t* tg, int32_t* ag, float* sc, void* s)
{ P(0, q); P(1, k); N(2, j); N(3, f); N(4, h); N(5, gh * 1000 + gw); N(6, d); P(7, an); N(8, n); N(9, th * 1000 + tw); N(10, w * 1000 + wt);
  N(11, t * 4096); P(12, tg); P(13, ag); P(14, sc); P(16, s); return 0; }
int fb4_seda_main_anchor(const float* ts, const void* q, const void* k, int64_t f, int h, int gh, int gw, int64_t d, const int32_t* c, int n, int th, int tw,
                         float t, int32_t* m, int32_t* kept, float* ps, void* s)
{ P(0, ts); P(1, q); P(2, k); N(3, f); N(4, h); N(5, gh); N(6, gw); N(7, d); P(8, c); N(9, n); N(10, th); N(11, tw); N(12, t * 4096); P(13, m);
  P(14, kept); P(15, ps); P(16, s); return 0; }
int fb4_seda_profile(const fb4_luts* l, const uint16_t* m, int64_t r, int64_t nb, const int32_t* ag, int g, uint32_t* c, uint8_t* sub, void* s)
{ P(0, m); N(1, r); N(2, nb); P(3, ag); N(4, g); P(5, c); P(6, sub); P(16, s); P(17, l); return 0; }
"""


@pytest.fixture(scope="module")
def recorder(tmp_path_factory, request):
    """The module on a library that notes down what its calls get: (module, function that returns and clears the notes)."""
    if not hasattr(torch.Tensor, "__dlpack_c_exchange_api__") or not B._build.can_build_call():
        pytest.skip("tensors without a reader, or nothing to build the module with")
    d = tmp_path_factory.mktemp("recorder")
    (d / "recorder.c").write_text(RECORDER)
    lib, so = d / "libfb4_recorder.so", d / "_fb4call_recorder.so"
    include = os.path.join(os.path.dirname(os.path.dirname(B.__file__)), "include")
    cc = B._build.HOST_CC.split()
    subprocess.run(cc + ["-shared", "-fPIC", "-I" + include, "-o", str(lib), str(d / "recorder.c")], check=True)
    subprocess.run(cc + ["-O1", "-shared", "-fPIC", "-I" + B._build.PYTHON_INCLUDE, "-o", str(so), B._build.CALL_SOURCE, "-L" + str(d),
                         "-l:" + lib.name, "-Wl,-rpath,$ORIGIN"], check=True)
    loader = importlib.machinery.ExtensionFileLoader("_fb4call", str(so))
    module = importlib.util.module_from_spec(importlib.util.spec_from_file_location("_fb4call", str(so), loader=loader))
    loader.exec_module(module)
    module.bind(B.fb4_opts, ctypes.c_void_p, B.CtypesCall)
    recording = ctypes.CDLL(str(lib))
    seen = (ctypes.c_int64 * 20).in_dll(recording, "seen")
    for call in B.EXPORTS:   # (what the module hands over to ctypes gets there too)
        if hasattr(recording, call):
            getattr(recording, call).argtypes = getattr(B.lib(), call).argtypes
    real, B._lib = B._lib, recording
    request.addfinalizer(lambda: setattr(B, "_lib", real))

    def notes():
        out = list(seen)
        ctypes.memset(seen, 0xEE, ctypes.sizeof(seen))
        return out

    return module, notes


def matrices():
    big = torch.zeros((6, 192), dtype=torch.bfloat16)
    return {"plain": big, "columns": big[:, 64:128], "rows": big[1:5], "every other row": big[::2], "one row": big[2:3], "one row, strided": big[::6],
            "no rows": big[:0], "no columns": big[:, :0], "transposed": big.t(), "stride 0": big[:1].expand(6, 192), "gradient": torch.zeros((4, 64), requires_grad=True),
            "parameter": torch.nn.Parameter(torch.zeros((4, 64))), "lazy copy": torch._lazy_clone(big), "float8": torch.zeros((4, 64), dtype=torch.float8_e4m3fn),
            "conjugate": torch.zeros((4, 64), dtype=torch.complex64).conj(), "meta": torch.zeros((4, 64), device="meta")}


@pytest.mark.parametrize("name", list(matrices()))
def test_tensors_are_read_as_by_their_methods(recorder, name):
    module, notes = recorder
    x = matrices()[name]
    o, h = F.opts(), ctypes.c_void_p(64)
    c, m = torch.zeros((4, 32), dtype=torch.uint8), torch.zeros((9, 2), dtype=torch.int16)[3:]
    tg, sub, sal = torch.zeros(4, dtype=torch.int32), torch.zeros((3, 8), dtype=torch.uint8), torch.zeros((2, 3), dtype=torch.int32)
    cube = x[None].expand(2, *x.shape)
    calls = [lambda: module.quantize(h, o, x, c, x, 0), lambda: module.quantize_seda(h, o, x, tg, sub, c, m, 0), lambda: module.quantize_seda(h, o, x, tg, x, c, m, 0),
             lambda: module.quantize_decompose(h, o, x, sal, None, None, c, m, c[1:], m, 0), lambda: module.quantize_decompose(h, o, x, x, tg, sub, c, m, c, m, 0),
             lambda: module.dequantize(h, c, m, 32, None, None, None, x, 0, 0), lambda: module.dequantize(h, x, m, 16, c, m, sal, x, 1, 0),
             lambda: module.repack_mxfp8(h, x, m, 32, x, c, 0), lambda: module.repack_mxfp8(h, c, m, 32, x, c, 0),
             lambda: module.layernorm_quantize(h, o, x, tg[1:], None, 1e-6, tg, sub, c, m, x, 0),
             lambda: module.gelu_quantize(h, o, x, 1, None, None, c, m, 0), lambda: module.attention_scores(cube, cube, 1, x, 0)]

    def results():
        notes()
        return [(call(), notes()) for call in calls]

    assert not module.read_through(torch.Tensor, None)
    want = results()
    assert module.read_through(torch.Tensor, torch.Tensor.__dlpack_c_exchange_api__)
    assert results() == want


def test_tensors_without_storage_are_refused_as_before(recorder):
    module, _ = recorder
    c = torch.zeros((4, 32), dtype=torch.uint8)
    for through in (None, torch.Tensor.__dlpack_c_exchange_api__):
        module.read_through(torch.Tensor, through)
        for transform in (torch.vmap, lambda f: torch.func.grad(lambda x: f(x).sum())):
            with pytest.raises(RuntimeError, match="data pointer"):
                transform(lambda x: (module.quantize(ctypes.c_void_p(64), F.opts(), x, c, c, 0), x)[1])(torch.zeros((2, 4, 64))[0] if transform is not torch.vmap else torch.zeros((2, 4, 64)))
        with pytest.raises(ValueError):
            module.quantize(ctypes.c_void_p(64), F.opts(), torch.zeros((1, 4, 64)), c, c, 0)


def refresh_calls(module, kind):
    """The refresh's calls with tensors and numbers of one kind."""
    frames, heads, gh, gw, dim = 3, 5, 4, 6, 16
    sc, ts = torch.zeros((frames, heads, gh * gw)), torch.zeros((gh * gw, heads, frames))
    q, qt = torch.zeros((frames, heads, gh * gw, dim), dtype=torch.bfloat16), torch.zeros((gh * gw, heads, frames, dim), dtype=torch.bfloat16)
    qj = torch.zeros((heads, frames * gh * gw, dim), dtype=torch.bfloat16)
    cand, out, meta = torch.zeros((frames, 2), dtype=torch.int32), torch.zeros(72, dtype=torch.int32), torch.zeros((72, 9), dtype=torch.int16)
    t, joint, i = 1.5, (False, True), int
    if kind == "views":
        sc, ts, q, qt, cand, meta = sc.transpose(0, 1).contiguous().transpose(0, 1), ts[1:2].expand(gh * gw, heads, frames), q.transpose(1, 2).contiguous().transpose(1, 2), qt.flip(0), cand[:, :1], meta[:, 3:]
    elif kind == "parameters":
        sc, ts, q, qj, qt = (torch.nn.Parameter(v) for v in (sc, ts, q, qj, qt))
    elif kind == "numbers":
        t, joint, i = np.float32(1.5), (0, 1), np.int32
    elif kind == "no scores":
        sc, ts, q, qt, qj, cand, meta = sc[:0], ts[:, :, :0], q[:0], qt[:, :, :0], qj[:, :0], cand[:0], meta[:0]
        frames = 0
    h = ctypes.c_void_p(64)
    return [lambda: module.select_salient_tokens(sc, i(gh), gw, 4, i(2), out, 0), lambda: module.select_salient_tokens(sc, gh, gw, 4, 4, None, None),
            lambda: module.seda_assign(q, q, joint[0], frames, gh, i(gw), cand, 4, 2, 5, i(1), t, out, out, None, 0),
            lambda: module.seda_assign(qj, q, joint[1], i(frames), gh, gw, out, 4, 4, 3, 2, 2, out, out[1:], ts, 0),
            lambda: module.seda_main_anchor(ts, qt, qt, cand, gh, gw, i(4), 2, t, out, cand, None, 0),
            lambda: module.seda_main_anchor(ts, qt, q, cand, gh, gw, 4, 4, 3, out, cand, sc, 0),
            lambda: module.seda_profile(h, meta, out, i(7), out, cand, 0), lambda: module.seda_profile(h, q[0, 0], out, 7, out, cand, 0) if frames else None,
            # sizes and shapes that are refused
            lambda: module.select_salient_tokens(sc, gh, gw + 1, 4, 4, out, 0), lambda: module.select_salient_tokens(q, gh, gw, 4, 4, out, 0),
            lambda: module.seda_main_anchor(ts, qt, qt, torch.zeros((9, 2), dtype=torch.int32), gh, gw, 4, 2, t, out, cand, None, 0),
            lambda: module.seda_main_anchor(ts, qj, qt, cand, gh, gw, 4, 2, t, out, cand, None, 0),
            lambda: module.seda_assign(qj, q, False, 3, gh, gw, cand, 4, 2, 5, 1, t, out, out, None, 0),
            lambda: module.seda_assign(q, q, False, 3, gh, gw, None, 4, 2, 5, 1, t, out, out, None, 0),
            lambda: module.seda_assign(q, q, False, 3, gh, gw, cand, 4, 2, 5, 1, None, out, out, None, 0),
            lambda: module.seda_profile(h, meta, out, 7.5, out, cand, 0), lambda: module.seda_profile(h, sc, out, 7, out, cand, 0)]


@pytest.mark.parametrize("kind", ["plain", "views", "parameters", "numbers", "no scores"])
def test_the_refresh_is_called_as_through_ctypes(recorder, kind):
    module, notes = recorder

    def results(calls):
        out = []
        for call in calls:
            notes()
            try:
                out.append((call(), notes()))
            except Exception as e:
                out.append((type(e), str(e)))
        return out

    # (the same tensors on both sides: the module to ask is looked up at the call)
    class Asked:
        which = B.CtypesCall

        def __getattr__(self, name):
            return getattr(Asked.which, name)

    calls = refresh_calls(Asked(), kind)
    want = results(calls)
    Asked.which = module
    assert module.read_through(torch.Tensor, torch.Tensor.__dlpack_c_exchange_api__)
    assert results(calls) == want
    assert not module.read_through(torch.Tensor, None)
    assert results(calls) == want


@pytest.mark.parametrize("call", ["select_salient_tokens", "seda_assign", "seda_main_anchor", "seda_profile"])
def test_sizes_are_those_at_the_start_of_a_call(recorder, call):
    # (an argument's method that resizes an earlier argument: what another thread can do while the library runs)
    module, notes = recorder
    frames, heads, gh, gw, dim = 3, 5, 4, 6, 16

    class Resizes:
        def __init__(self, *tensors):
            self.tensors = tensors

        def data_ptr(self):
            for t in self.tensors:
                t.resize_([n // 2 for n in t.shape])
            return 64

    def result(which):
        sc, out, meta = torch.zeros((frames, heads, gh * gw)), torch.zeros(72, dtype=torch.int32), torch.zeros((72, 9), dtype=torch.int16)
        q, qt = torch.zeros((frames, heads, gh * gw, dim), dtype=torch.bfloat16), torch.zeros((gh * gw, heads, frames, dim), dtype=torch.bfloat16)
        cand, h = torch.zeros((frames, 2), dtype=torch.int32), ctypes.c_void_p(64)
        args = {"select_salient_tokens": (sc, gh, gw, 4, 4, Resizes(sc), 0),
                "seda_assign": (q, Resizes(q), False, frames, gh, gw, cand, 4, 2, 5, 1, 1.5, out, out, None, 0),
                "seda_main_anchor": (sc, qt, qt, cand, gh, gw, 4, 2, 1.5, out, out, Resizes(qt, cand), 0),
                "seda_profile": (h, meta, out, 7, out, Resizes(meta), 0)}[call]
        notes()
        rc = getattr(which, call)(*args)
        known = {a.data_ptr(): i for i, a in enumerate(args) if isinstance(a, torch.Tensor)}   # (addresses differ from call to call)
        return rc, [known.get(v, v) for v in notes()]

    assert module.read_through(torch.Tensor, torch.Tensor.__dlpack_c_exchange_api__)
    assert result(module) == result(B.CtypesCall)


def all_calls(module, x, stream, handle, o, eps):
    """A call of every entry point with tensors and numbers of its own in every place."""
    c, m, c2, m2 = (torch.zeros((4, 32), dtype=torch.uint8) for _ in range(4))
    tg, sub, sal, ag = torch.zeros(4, dtype=torch.int32), torch.zeros((3, 8), dtype=torch.uint8), torch.zeros((2, 3), dtype=torch.int32), torch.zeros(4, dtype=torch.int32)
    ga, be, y = torch.zeros(64), torch.zeros(64), torch.zeros((4, 64), dtype=torch.bfloat16)
    frames, heads, gh, gw, dim = 3, 5, 4, 6, 16
    sc, ts, ps = torch.zeros((frames, heads, gh * gw)), torch.zeros((gh * gw, heads, frames)), torch.zeros((frames, 4))
    q, k = (torch.zeros((frames, heads, gh * gw, dim), dtype=torch.bfloat16) for _ in range(2))
    qt, kt = (torch.zeros((gh * gw, heads, frames, dim), dtype=torch.bfloat16) for _ in range(2))
    cand, kept, main = torch.zeros((frames, 2), dtype=torch.int32), torch.zeros((frames, 2), dtype=torch.int32), torch.zeros(4, dtype=torch.int32)
    return {"quantize": lambda: module.quantize(handle, o, x, c, m, stream),
            "quantize_seda": lambda: module.quantize_seda(handle, o, x, tg, sub, c, m, stream),
            "quantize_decompose": lambda: module.quantize_decompose(handle, o, x, sal, tg, sub, c, m, c2, m2, stream),
            "dequantize": lambda: module.dequantize(handle, c, m, 32, c2, m2, sal, y, 1, stream),
            "repack_mxfp8": lambda: module.repack_mxfp8(handle, c, m, 32, c2, m2, stream),
            "layernorm_quantize": lambda: module.layernorm_quantize(handle, o, x, ga, be, eps, tg, sub, c, m, y, stream),
            "gelu_quantize": lambda: module.gelu_quantize(handle, o, x, 1, tg, sub, c, m, stream),
            "attention_scores": lambda: module.attention_scores(q[0], k[0], 1, sc, stream),
            "select_salient_tokens": lambda: module.select_salient_tokens(sc, gh, gw, 2, 3, main, stream),
            "seda_assign": lambda: module.seda_assign(q, k, False, frames, gh, gw, cand, 2, 3, 5, 1, 1.5, tg, ag, ps, stream),
            "seda_main_anchor": lambda: module.seda_main_anchor(ts, qt, kt, cand, gh, gw, 2, 3, 1.5, main, kept, ps, stream),
            "seda_profile": lambda: module.seda_profile(handle, m, ag, 7, main, sub, stream)}


@pytest.mark.parametrize("reader", [False, True])
def test_streams_handles_options_and_eps_arrive(recorder, reader):
    module, notes = recorder
    module.read_through(torch.Tensor, torch.Tensor.__dlpack_c_exchange_api__ if reader else None)

    class Asked:
        which = None

        def __getattr__(self, name):
            return getattr(Asked.which, name)

    untouched = -0x1111111111111112   # (what a place holds that a call does not write)
    calls = all_calls(Asked(), X, 0x7001, ctypes.c_void_p(0x640), F.opts(16, F.SEL_SSE, 32, F.FLAG_TWO_STAGE), 0.25)
    assert set(calls) == {n for n in dir(B.CtypesCall) if not n.startswith("_")}
    options = ((16 * 100 + F.SEL_SSE) * 100 + 32) * 100 + F.FLAG_TWO_STAGE
    for name, call in calls.items():
        got = []
        for Asked.which in (module, B.CtypesCall):
            notes()
            assert call() == 0
            got.append(notes())
        assert got[0] == got[1], name
        with_handle = name not in ("attention_scores", "select_salient_tokens", "seda_assign", "seda_main_anchor")
        with_options = "quantize" in name and name != "dequantize"
        assert got[0][16:] == [0x7001, 0x640 if with_handle else untouched, options if with_options else untouched,
                               1 << 38 if name == "layernorm_quantize" else untouched], name


def test_a_copy_on_write_tensor_is_read_as_its_own(recorder):
    # (a fresh lazy copy for every place, which the table's reader is the first to look at)
    module, notes = recorder
    assert module.read_through(torch.Tensor, torch.Tensor.__dlpack_c_exchange_api__)
    c, o, h = torch.zeros((4, 32), dtype=torch.uint8), F.opts(), ctypes.c_void_p(64)
    source = torch.zeros((2, 4, 64), dtype=torch.bfloat16)
    for call in (lambda x: module.quantize(h, o, x[0], c, c, 0), lambda x: module.attention_scores(x, c, 0, c, 0), lambda x: module.seda_profile(h, x[0], c, 1, c, c, 0),
                 lambda x: module.dequantize(h, x[0], c, 32, None, None, None, c, 0, 0), lambda x: module.repack_mxfp8(h, x[0], c, 32, c, c, 0),
                 lambda x: module.select_salient_tokens(x, 8, 8, 4, 4, c, 0)):
        x = torch._lazy_clone(source)
        notes()
        assert call(x) == 0
        assert notes()[0] == x.data_ptr() != source.data_ptr()
    x = torch._lazy_clone(source)
    notes()
    assert module.quantize(h, o, source[0], x, c, 0) == 0   # (an address alone)
    assert notes()[4] == x.data_ptr() != source.data_ptr()
