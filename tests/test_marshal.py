"""The native marshalling of the launches hands the library exactly what ctypes would, and leaves to ctypes what it does not know.

No GPU: it is bound to recorders in place of the library's functions."""
import ctypes as C
import os
import subprocess
import sys
import sysconfig
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from paper_2602_20656_amd import binding as lg

GEMM = C.CFUNCTYPE(C.c_int, C.c_void_p, C.c_void_p, C.c_void_p, C.c_int64, C.c_int64, C.c_int64, C.c_int, C.c_int, C.c_void_p)
COMM = C.CFUNCTYPE(C.c_int, C.c_int, C.c_int, C.POINTER(C.c_void_p), C.c_int, C.POINTER(C.c_void_p), C.c_int, C.c_int64, C.POINTER(lg.lagom_cfg), C.c_void_p)
STEPS = C.CFUNCTYPE(C.c_int, C.c_int, C.POINTER(lg.lagom_comm_step), C.c_int, C.c_int64, C.POINTER(lg.lagom_cfg), C.c_void_p)


@pytest.fixture
def calls():
    lib = lg.lib()
    got, code = [], [0]
    cfg = lambda c: (c[0].nc, c[0].nt, c[0].chunk_bytes)

    def gemm(*a):
        got.append(a)
        return code[0]

    def comm(op, dt, s, ns, d, nd, count, c, st):
        got.append((op, dt, s[:ns], d[:nd], count, cfg(c), st))
        return code[0]

    def steps(dt, t, n, count, c, st):
        got.append((dt, [(t[i].op, t[i].srcs[:t[i].nsrc], t[i].dsts[:t[i].ndst]) for i in range(n)], count, cfg(c), st))
        return code[0]

    keep = (GEMM(gemm), COMM(comm), STEPS(steps))
    address = lambda f: C.cast(f, C.c_void_p).value
    lg._launch.bind(*map(address, keep), lg.lagom_cfg)
    yield SimpleNamespace(got=got, code=code)
    lg._launch.bind(*(address(f) for f in (lib.lagom_gemm, lib.lagom_comm_kernel, lib.lagom_comm_steps)), lg.lagom_cfg)


T = [torch.zeros(8) for _ in range(3)]
P = [t.data_ptr() for t in T]
STREAM = SimpleNamespace(cuda_stream=0x7F0000001230)


@pytest.mark.parametrize("stream,handle", [(None, None), (0, None), (STREAM, 0x7F0000001230), (0xFFFFFFFFFFFFFFF0, 0xFFFFFFFFFFFFFFF0)])
def test_gemm(calls, stream, handle):
    lg.lagom_gemm(T[0], P[1], T[2], 5, 1 << 40, 7, stream=stream)
    lg.lagom_gemm(P[0], T[1], P[2], True, -3, 2**63 - 1, [], lg.LAGOM_F32, stream)
    assert calls.got == [(P[0], P[1], P[2], 5, 1 << 40, 7, 1, lg.LAGOM_BF16, handle), (P[0], P[1], P[2], 1, -3, 2**63 - 1, 0, lg.LAGOM_F32, handle)]


@pytest.mark.parametrize("cfg", [(8, 256, 1 << 40), [8, 256, 1 << 40], (8, 256, 1 << 40, "more"), lg.lagom_cfg(8, 256, 1 << 40)])
def test_comm_kernel(calls, cfg):
    lg.lagom_comm_kernel(1, 0, [T[0], P[1]] * 8, (T[2],), 1 << 35, cfg, STREAM)
    lg.lagom_comm_kernel(0, 1, [], [], 0, cfg)
    assert calls.got == [(1, 0, P[:2] * 8, P[2:], 1 << 35, (8, 256, 1 << 40), STREAM.cuda_stream), (0, 1, [], [], 0, (8, 256, 1 << 40), None)]


def test_comm_steps(calls):
    ring = [(0, [P[0], T[1]], [P[2], P[0]])] * 7 + [(1, (T[0],), (P[1], T[2]))] * 25
    lg.lagom_comm_steps(1, ring, 99, (1, 64, 16), STREAM)
    assert calls.got == [(1, [(0, [P[0], P[1]], [P[2], P[0]])] * 7 + [(1, [P[0]], [P[1], P[2]])] * 25, 99, (1, 64, 16), STREAM.cuda_stream)]


def test_codes_become_errors(calls):
    calls.code[0] = lg.LAGOM_EALIGN
    for call in (lambda: lg.lagom_gemm(*P, 1, 1, 8), lambda: lg.lagom_comm_kernel(0, 0, P[:1], P[1:2], 1, (1, 64, 16)), lambda: lg.lagom_comm_steps(0, [], 1, (1, 64, 16))):
        with pytest.raises(lg.LagomError) as e:
            call()
        assert e.value.code == lg.LAGOM_EALIGN
    assert len(calls.got) == 3


class Raises:
    def data_ptr(self):
        raise RuntimeError("no storage")


@pytest.mark.parametrize("args", [
    (*P, np.int64(4), 4, 8, True, 1, None), (*P, 4.0, 4, 8, True, 1, None), (*P, 4, 4, 1 << 64, True, 1, None), (*P, 4, 4, 8, True, 1 << 31, None),
    (np.int64(64), P[1], P[2], 4, 4, 8, True, 1, None), (-1, P[1], P[2], 4, 4, 8, True, 1, None), (1 << 64, P[1], P[2], 4, 4, 8, True, 1, None),
    (*P, 4, 4, 8, True, 1, "0"), (*P, 4, 4, 8, True, 1, SimpleNamespace(cuda_stream=-1)), (Raises(), P[1], P[2], 4, 4, 8, True, 1, None), (None,) * 9])
def test_gemm_leaves_the_rest_to_ctypes(calls, args):
    assert lg._launch.gemm(*args) is None and calls.got == []


@pytest.mark.parametrize("args", [
    (0, 0, iter(P[:1]), P[1:2], 1, (1, 64, 16), None), (0, 0, P[:1], T[0], 1, (1, 64, 16), None), (0, 0, P[:1], ["x"], 1, (1, 64, 16), None),
    (0, 0, P[:1], P[1:2], 1, (1, 64), None), (0, 0, P[:1], P[1:2], 1, (1.5, 64, 16), None), (0, 0, P[:1], P[1:2], 1, (1 << 31, 64, 16), None),
    (0, 0, P[:1], P[1:2], 1, {0: 1, 1: 64, 2: 16}, None), (0, 0, [P[0]] * 65, P[1:2], 1, (1, 64, 16), None), (0.0, 0, P[:1], P[1:2], 1, (1, 64, 16), None)])
def test_comm_kernel_leaves_the_rest_to_ctypes(calls, args):
    assert lg._launch.comm_kernel(*args) is None and calls.got == []


@pytest.mark.parametrize("steps", [iter([]), [[0, P[:1], P[1:2]]], [(0, P[:1])], [(0, P[0], P[1:2])], [(np.int32(0), P[:1], P[1:2])],
                                   [(0, P[:1], P[1:2])] * 65, [(0, [P[0]] * 512, [P[1]] * 513)], [(0, [P[0]] * 1000, [P[1]] * 24), (0, [P[0]], [])]])
def test_comm_steps_leaves_the_rest_to_ctypes(calls, steps):
    assert lg._launch.comm_steps(0, steps, 1, (1, 64, 16), None) is None and calls.got == []


class Interrupted:
    calls = 0

    def data_ptr(self):
        Interrupted.calls += 1
        raise KeyboardInterrupt

    cuda_stream = property(data_ptr)


@pytest.mark.parametrize("call", [
    lambda x: lg.lagom_gemm(x, P[1], P[2], 4, 4, 8), lambda x: lg.lagom_gemm(*P, 4, 4, 8, stream=x), lambda x: lg.lagom_comm_kernel(0, 0, [P[0], x], P[1:2], 1, (1, 64, 16)),
    lambda x: lg.lagom_comm_steps(0, [(0, P[:1], [x])], 1, (1, 64, 16)), lambda x: lg.lagom_comm_steps(0, [(0, P[:1], P[1:2])], 1, (1, 64, 16), x)])
def test_an_interrupt_is_no_wrong_argument(calls, call):
    """It ends the call where it comes up, and the object is not asked again through ctypes."""
    before = Interrupted.calls
    with pytest.raises(KeyboardInterrupt):
        call(Interrupted())
    assert Interrupted.calls == before + 1 and calls.got == []


class Shrinks:
    """data_ptr() empties the list it is in."""
    def __init__(self, inside):
        self.inside = inside

    def data_ptr(self):
        self.inside.clear()
        return P[0]


def test_a_list_that_changes_under_the_call(calls):
    xs = []
    xs += [Shrinks(xs), P[1], P[2]]
    lg.lagom_comm_kernel(0, 0, xs, P[2:], 1, (1, 64, 16))
    assert calls.got == [(0, 0, P[:1], P[2:], 1, (1, 64, 16), None)]


def test_what_ctypes_refused_is_refused():
    """Through the entry points, with the library bound: nothing is launched."""
    with pytest.raises(C.ArgumentError):
        lg.lagom_gemm(*P, 4, 4, 8, True, "bf16")
    with pytest.raises(RuntimeError, match="no storage"):
        lg.lagom_gemm(Raises(), P[1], P[2], 4, 4, 8)
    with pytest.raises(TypeError):
        lg.lagom_comm_kernel(0, 0, P[:1], 7, 1, (1, 64, 16))
    with pytest.raises(IndexError):
        lg.lagom_comm_kernel(0, 0, P[:1], P[1:2], 1, (1, 64))
    with pytest.raises(lg.LagomError) as e:
        lg.lagom_comm_kernel(0, 0, [P[0]] * 65, P[1:2], 1, (1, 64, 16))
    assert e.value.code == lg.LAGOM_EINVAL


def test_the_module_is_for_this_interpreter_only():
    assert lg._launches().__file__.endswith("_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))


def test_without_the_module_the_error_names_the_build():
    code = ("import sys; sys.modules['paper_2602_20656_amd._marshal'] = None\n"
            "from paper_2602_20656_amd import binding\n"
            "try: binding.lib()\n"
            "except ImportError as e: assert 'python -m paper_2602_20656_amd.build' in str(e), e\n"
            "else: raise AssertionError('loaded')")
    subprocess.run([sys.executable, "-c", code], check=True, timeout=120, cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
