"""The calls without ctypes (csrc/pycall.c): arguments arrive as through ctypes, matrices are looked over as in Python."""
import ctypes as C
import sysconfig

import numpy as np
import pytest
import torch

import paper_2507_16099_amd.build as build
import paper_2507_16099_amd.fp8 as fp8

pytestmark = pytest.mark.skipif(fp8._pycall is None, reason="built without the interpreter's headers")


class Pointer:
    def __init__(self, address):
        self.address = address

    def data_ptr(self):
        return self.address


@pytest.mark.parametrize("n", range(1, 19))
def test_every_argument_arrives(n):
    got = []
    f = C.CFUNCTYPE(C.c_int, *([C.c_int64] * n))(lambda *a: got.append(a) or -7)
    values = [(-1) ** i * (1 << 40) + i for i in range(n)]
    call = fp8._pycall.Call(C.cast(f, C.c_void_p).value, "l" * n)
    assert call(*values) == -7 and got == [tuple(values)]
    assert fp8._pycall.Call(C.cast(f, C.c_void_p).value, "t" * n)(*[Pointer(0x7FFF00000000 + i) if i % 3 else None for i in range(n)]) == -7
    assert got[1] == tuple(0x7FFF00000000 + i if i % 3 else 0 for i in range(n))
    for wrong in (values + [0], values[:-1], [1.5] * n, ["a"] * n, [None] * n):
        with pytest.raises(TypeError):
            call(*wrong)
    assert len(got) == 2


def test_narrow_arguments_and_results_of_the_library():
    """A call that the library refuses before any device: the code and the message of ctypes."""
    L = fp8.load_library()
    for bad in (dict(M=-1), dict(gran=5), dict(fmt=9), dict(ldw=3)):
        M, fmt, gran, ldw = bad.get("M", 2), bad.get("fmt", 0), bad.get("gran", 1), bad.get("ldw", 16)
        args = (4096, M, 16, fmt, gran, 0, 4096, ldw, 0, 4096, 1, 8, 4096, 8, 4096, 16, 0)
        tensors = [Pointer(a) if a == 4096 else a for a in args]
        want = L.fp8_linear_fwd_prequantized(*args), fp8.fp8_last_error()
        assert want[0] != 0
        assert (L.fast_linear_fwd_prequantized(*tensors), fp8.fp8_last_error()) == want, bad
    for i in (0, 6, 9, 12, 14):
        for wrong in (object(), 4096, 1, True, 1.0):      # a number is no tensor, although it would pass for an address
            with pytest.raises(AttributeError):
                L.fast_linear_fwd_prequantized(*tensors[:i], wrong, *tensors[i + 1:])


class Index:
    def __init__(self, value):
        self.value = value

    def __index__(self):
        return self.value


class Parameter:
    def __init__(self, value):
        self._as_parameter_ = value


@pytest.mark.parametrize("number", [np.int64, np.int32, np.uint8, torch.tensor, Index, Parameter, bool, lambda v: v + (1 << 32)], ids=lambda f: getattr(f, "__name__", "f"))
def test_whatever_ctypes_takes_for_an_integer(number):
    """Sizes, formats, granularities and flags that are no ints: the code and the message that the same numbers give as ints (calls that
    the library refuses before any device; the refused argument comes last, so that the others have been read)."""
    L = fp8.load_library()
    args = [Pointer(4096), 2, 16, 0, 1, 0, Pointer(4096), 16, 0, Pointer(4096), 1, 8, Pointer(4096), 8, Pointer(4096 + 64), 16, 0]      # (workspace not on 256 bytes)
    want = L.fast_linear_fwd_prequantized(*args), fp8.fp8_last_error()
    assert want[0] != 0 and "256" in want[1]
    plain = [a.address if isinstance(a, Pointer) else a for a in args]
    wide = number is not bool and number(1) == (1 << 32) + 1
    for i in (1, 2, 3, 4, 5, 7, 8, 10, 11, 13, 15):
        if isinstance(args[i], Pointer) or (number is bool and args[i] > 1) or (wide and i not in (3, 4, 5, 8, 10)):
            continue
        values = [number(a) if k == i else a for k, a in enumerate(args)]
        assert (L.fp8_linear_fwd_prequantized(*[number(a) if k == i else a for k, a in enumerate(plain)]), fp8.fp8_last_error()) == want, i
        assert (L.fast_linear_fwd_prequantized(*values), fp8.fp8_last_error()) == want, i
    for i in (1, 3, 15):
        for wrong in (1.0, np.float32(1), "1", None, torch.tensor(1.5)):
            errors = []
            for call, rest in ((L.fp8_linear_fwd_prequantized, plain), (L.fast_linear_fwd_prequantized, args)):
                with pytest.raises(Exception) as e:
                    call(*rest[:i], wrong, *rest[i + 1:])
                errors.append((e.type, str(e.value)))
            assert errors[0] == errors[1], (i, wrong)


class Tensor:
    """What a tensor on the GPU answers."""
    is_cuda, dtype, device = True, "x", "y"

    def __init__(self, t):
        self.t = t
        self.shape = t.shape

    def element_size(self):
        return self.t.element_size()

    def stride(self):
        return self.t.stride()


def test_matrices_are_looked_over_as_in_python():
    base = torch.zeros((40, 48), dtype=torch.bfloat16)
    for t in (base, base[:1], base[:1, :8], base[:, :1], base[3:4, 5:6], base[::2], base[:0], base[:, :0], base[:, ::2], base.t(), base[0], base[None], base.view(torch.int16),
              base.float(), base[:1, ::2], base.t()[:1], base.expand(2, 40, 48)[0], base[:1].expand(5, 48), base[:, :1].expand(40, 9)):
        for size in (1, 2, 4):
            results = []
            for mat in (fp8._mat_any, fp8._mat):
                try:
                    results.append(mat(Tensor(t), size))
                except AssertionError as e:
                    results.append(str(e))
                except (ValueError, TypeError) as e:
                    results.append(type(e))
            assert results[0] == results[1], (t.shape, t.stride(), size, results)
    with pytest.raises(AssertionError):
        fp8._mat(base, 2)                  # not on a GPU
    with pytest.raises(AttributeError):
        fp8._mat(3, 2)


def test_without_the_module(monkeypatch):
    monkeypatch.setattr(fp8, "_pycall", None)
    seen = []

    class Function:
        argtypes = [C.c_void_p, C.c_int64, C.c_void_p, C.c_void_p]

        def __call__(self, *a):
            seen.append(a)
            return 0

    t = torch.zeros(3)
    call = fp8._fast(Function())
    assert call(t, 5, None, 9) == 0 and seen == [(t.data_ptr(), 5, None, 9)]
    with pytest.raises(AttributeError):
        call(4096, 5, None, 9)


def test_built_for_one_interpreter(tmp_path, monkeypatch, capfd):
    """The file names the interpreter; a build that cannot make it goes on without it and leaves no older one."""
    assert build.PYCALL.endswith(sysconfig.get_config_var("EXT_SUFFIX")) and fp8._pycall.__file__ == build.PYCALL
    out = tmp_path / "_pycall.so"
    for cc in ("false", "no-such-compiler", ""):
        monkeypatch.setenv("CC", cc)
        out.write_bytes(b"old")
        build._compile_pycall(str(out))
        assert not out.exists() and "calls go through ctypes" in capfd.readouterr().err
    monkeypatch.setenv("CC", "gcc -g0")
    build._compile_pycall(str(out))
    assert out.stat().st_size > 1000
