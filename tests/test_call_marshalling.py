"""The step's calls reach the library with the same arguments through native code (csrc/pt_call.cpp) as through ctypes, in every form that
either takes.  The entry points are stand-ins that write their arguments down; no GPU."""
import ctypes as C
import importlib.machinery
import os
import sys

import pytest
import torch

from paper_2406_08334_amd import binding as B

VP, U32, U64, PP = C.c_void_p, C.c_uint32, C.c_uint64, C.POINTER(C.c_void_p)
HP = C.POINTER(B.pt_hparams)
N = 3                                                        # pointers read of every array
PROTOTYPES = {
    "pt_chunk_pack_grads": (VP, VP, PP, VP), "pt_chunk_unpack": (VP, VP, PP, VP),
    "pt_chunk_accum_grads": (VP, VP, PP, C.c_int, C.c_int, VP), "pt_chunk_grad_sqnorm": (VP, PP, U32, U32, C.c_int, VP),
    "pt_chunk_adamw_step": (VP, HP, U32, U32, PP, PP, PP, PP, PP, VP), "pt_step_end": (VP, VP),
    "pt_chunk_grad_sqnorm_noalloc": (VP, C.c_int, U64, U32, C.c_double, VP, VP, VP)}


@pytest.fixture
def calls(monkeypatch):
    """Everything that reaches an entry point, as plain values; the real library is bound again afterwards."""
    B.lib()
    seen, keep, L = [], {}, type("Stub", (), {})()

    def plain(x):
        if isinstance(x, C.POINTER(C.c_void_p)):
            return [x[i] for i in range(N if x[0] else 1)] if x else None
        return bytes(x.contents) if isinstance(x, HP) else x

    for name, args in PROTOTYPES.items():
        keep[name] = C.CFUNCTYPE(C.c_int, *args)(lambda *a, name=name: seen.append((name, [plain(x) for x in a])) or 0)
        setattr(L, name, keep[name])
    L.pt_last_error = lambda ctx: b""
    monkeypatch.setattr(B, "_lib", L)
    order = ["pt_chunk_pack_grads", "pt_chunk_unpack", "pt_chunk_accum_grads", "pt_chunk_grad_sqnorm", "pt_chunk_adamw_step", "pt_step_end",
             "pt_chunk_grad_sqnorm_noalloc"]
    B._native.bind([C.cast(keep[n], VP).value for n in order], VP, B.pt_hparams, torch.cuda.is_initialized, None, None)
    yield seen
    monkeypatch.undo()
    B._lib = None
    B.lib()


T = [torch.zeros(4 + k) for k in range(N)]
LISTS = [T, [T[0], None, T[2]], [T[0], 4096, 2 ** 63 + 16], tuple(T), [T[0], T[1], T[2].double()], torch.nn.ParameterList(T)]
CTX, PLAN = C.c_void_p(0x1230), C.c_void_p(0x4560)


class Nothing:                                               # native code that takes no call
    def __getattr__(self, name):
        return lambda *a: None


def both(calls, monkeypatch, call):
    call()
    with monkeypatch.context() as m:
        m.setattr(B, "_native", Nothing())
        call()
    assert len(calls) == 2 and calls[0] == calls[1], calls
    calls.clear()


@pytest.mark.parametrize("rows", LISTS, ids=range(len(LISTS)))
@pytest.mark.parametrize("ctx", [CTX, 0x1230, None])
def test_lists_and_handles(calls, monkeypatch, rows, ctx):
    hp = B.hparams(1e-4, 0.9, 0.95, 1e-8, 0.1, 1.0)
    for stream in (0, 0x7777, 2 ** 63 + 8):
        both(calls, monkeypatch, lambda: B.pt_chunk_pack_grads(ctx, PLAN, rows, stream))
        both(calls, monkeypatch, lambda: B.pt_chunk_unpack(ctx, PLAN, rows, stream))
        both(calls, monkeypatch, lambda: B.pt_chunk_accum_grads(ctx, PLAN, rows, 0, 3, stream))
        both(calls, monkeypatch, lambda: B.pt_chunk_grad_sqnorm(ctx, rows, 0, N, True, stream))
        both(calls, monkeypatch, lambda: B.pt_chunk_adamw_step(ctx, hp, 1, N, rows, T, rows, T, rows, stream))
        both(calls, monkeypatch, lambda: B.pt_step_end(ctx, stream))


def test_numbers_and_nothing(calls, monkeypatch):
    for first, n, how in [(0, 0, 0), (2, 5, B.PT_FINALIZE_CARRY), (1.0, 2.0, False), (2 ** 32 - 1, 2 ** 32 + 7, 1), (-1, 3, -1), (True, 3, 2 ** 31 - 1)]:
        for rows in (None, [], T):
            both(calls, monkeypatch, lambda: B.pt_chunk_grad_sqnorm(CTX, rows, first, n, how, 8))
    for arena, out in [(T[0], T[1]), (0x1000, T[1]), (T[0], None)]:
        for scale in (1.0, 1024, True):
            both(calls, monkeypatch, lambda: B.pt_chunk_grad_sqnorm_noalloc(arena, B.PT_FP16, 2 ** 40, 3, scale, out, T[2], 8))


def test_refused_forms_are_refused_as_before(calls, monkeypatch):
    hp = B.hparams(1e-4, 0.9, 0.95, 1e-8, 0.1, 1.0)
    for call in (lambda: B.pt_chunk_pack_grads(CTX, PLAN, [T[0], "x"], 0), lambda: B.pt_chunk_pack_grads(object(), PLAN, T, 0),
                 lambda: B.pt_chunk_adamw_step(CTX, None, 0, 1, T, T, T, T, T, 0), lambda: B.pt_chunk_grad_sqnorm(CTX, None, "zero", 1, 1, 0),
                 lambda: B.pt_chunk_adamw_step(CTX, hp, 0, 1, T, T, T, T, None, object())):
        raised = []
        for native in (B._native, Nothing()):
            with monkeypatch.context() as m:
                m.setattr(B, "_native", native)
                with pytest.raises(Exception) as e:
                    call()
                raised.append(type(e.value))
        assert raised[0] is raised[1] and not calls


def test_hyper_parameters_of_another_layout_are_refused(calls):
    class Short(C.Structure):                                # as an extension module would see that another header was built with
        _fields_ = B.pt_hparams._fields_[:-1]

    entries = [C.cast(C.CDLL(None).abs, VP).value] * 7
    with pytest.raises(ValueError):
        B._native.bind(entries, VP, Short, torch.cuda.is_initialized, None, None)
    B.pt_step_end(CTX, 8)                                    # still bound to the stand-ins
    assert len(calls) == 1


class Stream:                                                # torch.cuda.Stream as the binding looks at it
    cuda_stream = 0x7770


class Counted:
    """A tensor as the binding looks at it, which counts how often its address is taken."""

    def __init__(self, at):
        self.at, self.asked = at, 0

    def data_ptr(self):
        self.asked += 1
        return self.at


STEP_CALLS = {
    "pack": lambda hp, x, st: B.pt_chunk_pack_grads(CTX, PLAN, x, st), "unpack": lambda hp, x, st: B.pt_chunk_unpack(CTX, PLAN, x, st),
    "accum": lambda hp, x, st: B.pt_chunk_accum_grads(CTX, PLAN, x, 0, 1, st), "norm": lambda hp, x, st: B.pt_chunk_grad_sqnorm(CTX, x, 0, N, 1, st),
    "update": lambda hp, x, st: B.pt_chunk_adamw_step(CTX, hp, 0, N, x, x, x, x, x, st), "end": lambda hp, x, st: B.pt_step_end(CTX, st),
    "noalloc": lambda hp, x, st: B.pt_chunk_grad_sqnorm_noalloc(x[0], B.PT_FP16, 8, 3, 1.0, x[1], x[2], st)}


@pytest.mark.parametrize("name", STEP_CALLS)
def test_stream_objects(calls, monkeypatch, name):
    hp = B.hparams(1e-4, 0.9, 0.95, 1e-8, 0.1, 1.0)
    both(calls, monkeypatch, lambda: STEP_CALLS[name](hp, T, Stream()))


@pytest.mark.parametrize("name,how", [(name, how) for name in STEP_CALLS for how in ("object", "handle", "large")])
def test_an_address_is_taken_once(calls, monkeypatch, name, how):
    """With a stream object in native code; a call that is left to ctypes because of its handle or stream has not been through its lists before."""
    hp = B.hparams(1e-4, 0.9, 0.95, 1e-8, 0.1, 1.0)
    x = [Counted(0x1000 * (k + 1)) for k in range(N)]
    stream = {"object": Stream(), "handle": 0x10, "large": 2 ** 64 + 16}[how]      # ctypes cuts the last one off
    if how == "handle":
        monkeypatch.setitem(globals(), "CTX", 0x1230)        # a form that ctypes takes
    STEP_CALLS[name](hp, x, stream)
    times = {"update": 5, "end": 0}.get(name, 1)
    assert len(calls) == 1 and [t.asked for t in x] == [times] * N, [t.asked for t in x]


def test_lists_of_other_forms_are_found_first(calls, monkeypatch):
    hp = B.hparams(1e-4, 0.9, 0.95, 1e-8, 0.1, 1.0)
    x = [Counted(0x1000 * (k + 1)) for k in range(N)]
    B.pt_chunk_adamw_step(CTX, hp, 0, N, x, x, x, x, tuple(x), 0)
    assert [t.asked for t in x] == [5] * N


def test_without_the_extension_module(monkeypatch):
    """The library serves a Python that the module was not built for: its calls go by ctypes."""
    with monkeypatch.context() as m:
        m.setitem(sys.modules, B.__package__ + "._ptcall", None)        # as if it were not there
        m.setattr(B, "_lib", None)
        segs, chunks = B.pt_layout_dense([5, 11], 8)
        assert chunks == 2 and len(segs) == 3
        with pytest.raises(B.PtError) as e:                  # reaches the library, which refuses it
            B.pt_chunk_pack_grads(None, None, T, 0)
        assert e.value.status == B.PT_ERR_INVALID_ARG
    B._lib = None
    B.lib()
    if B._native is not B._Ctypes:                           # a module of this interpreter alone
        assert os.path.basename(B._native.__file__) == "_ptcall" + importlib.machinery.EXTENSION_SUFFIXES[0]


def test_a_module_that_does_not_load_says_why(monkeypatch):
    def broken(*args):
        raise ImportError("undefined symbol")

    with monkeypatch.context() as m:
        m.setattr(B, "_lib", None)
        m.setattr(B.importlib, "import_module", broken)
        with pytest.raises(ImportError, match="undefined symbol"):
            B.lib()
