"""The per-iteration calls marshalled in C against the binding's general path, over the forms that arguments come in: the same
values reach the library, the same exceptions come back, a failing status raises.  The library is a stub that records."""
import contextlib
import ctypes as C
import shutil
import subprocess

import numpy as np
import pytest
import torch

from paper_2502_11058_amd import binding as B

# entry point -> letters of its arguments behind the context: i int, p pointer, P peers, o options
ENTRIES = {"ddp_pack": "ipp", "ddp_unpack": "ipp", "ddp_pack_wire16": "ipp", "ddp_partial_average": "ipPiippp",
           "ddp_partial_average_wire16": "ipPiippp", "ddp_local_update": "op", "ddp_local_update_layers": "iiop",
           "ddp_fused_sync_update": "iPiipop", "ddp_fused_sync_update_wire16": "iPiipop", "ddp_fused_sync_update_layers": "iiiPiiiipop"}


def _stub():
    c = {"i": "int", "p": "void *", "P": "void **", "o": "void *"}
    src = "long rec[16], peers[4]; float lr; int status;\n"
    for name, sig in ENTRIES.items():
        src += f"int {name}(void *ctx, {', '.join(f'{c[k]} a{j}' for j, k in enumerate(sig))}) {{ rec[0] = (long)ctx;"
        for j, k in enumerate(sig):
            if k == "P":
                src += f" rec[{j + 1}] = a{j} != 0; for (int q = 0; q < 3; ++q) peers[q] = a{j} ? (long)a{j}[q] : 0;"
            elif k == "o":
                src += f" lr = ((float *)a{j})[1];"
            else:
                src += f" rec[{j + 1}] = (long)a{j};"
        src += " return status; }\n"
    src += 'int ddp_create(void **p, int d) { *p = rec; return 0; }\nint ddp_destroy(void *p) { return 0; }\n'
    src += 'const char *ddp_last_error(void *p) { return "stub"; }\n'
    done = set(ENTRIES) | {"ddp_create", "ddp_destroy", "ddp_last_error"}
    return src + "".join(f"int {n}(void) {{ return 0; }}\n" for n in B.EXPORTS if n not in done)


class _Stream:
    cuda_stream = 4096 + 64


@contextlib.contextmanager
def _stubbed(tmp_path, monkeypatch):
    """The binding on a recording library and a stream query of its own; what was there before is back afterwards, in the
    extension module as well."""
    if not shutil.which("gcc"):
        pytest.skip("no host compiler")
    real, query = B.lib(), B._raw_stream
    if isinstance(B._calls, B._NoCalls):
        pytest.skip("the extension module is not built")
    (tmp_path / "s.c").write_text(_stub())
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", str(tmp_path / "s.so"), str(tmp_path / "s.c")], check=True)
    monkeypatch.setattr(B, "LIB_PATH", str(tmp_path / "s.so"))
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_raw_stream", (lambda: False, lambda: 0, lambda d: 77))
    try:
        l = B.lib()
        B._calls.set_stream_query(*B._raw_stream)
        yield l
    finally:
        B._load_calls(real)
        B._calls.set_stream_query(*(query or (None, None, None)))


@pytest.fixture
def stub(tmp_path, monkeypatch):
    with _stubbed(tmp_path, monkeypatch) as l:
        yield l


def test_nothing_of_the_stub_is_left(tmp_path, monkeypatch):
    t = torch.zeros(8)
    with monkeypatch.context() as m, _stubbed(tmp_path, m):
        assert B._calls.pack(0, 1, t, None) == 0
    # (the library refuses a null context; without a stream query the call is the general path's)
    assert B._calls.pack(0, 1, t, 9) == 1
    assert (B._calls.pack(0, 1, t, None) is None) == (B._raw_stream is None)


def _both(l, monkeypatch, call):
    """(outcome, what the library saw) of a call, marshalled in C and on the general path."""
    got = []
    for calls in (B._calls, B._NoCalls()):
        with monkeypatch.context() as m:
            m.setattr(B, "_calls", calls)
            for name, n in (("rec", 16), ("peers", 4)):
                C.memset(C.addressof((C.c_long * n).in_dll(l, name)), 0, 8 * n)
            try:
                out = ("returns", call())
            except Exception as e:  # noqa: BLE001  (the two paths are compared, whatever they raise)
                out = (type(e).__name__, getattr(e, "code", None))
            got.append((out, list((C.c_long * 16).in_dll(l, "rec")), list((C.c_long * 4).in_dll(l, "peers")), C.c_float.in_dll(l, "lr").value))
    return got


def _forms():
    t, s = torch.zeros(8), torch.zeros(4, dtype=torch.float64)
    lists = [torch.zeros(4) for _ in range(3)]
    opt = B.make_opt("sgdm", 0.25, 3, momentum=0.9)
    peers = [lists, tuple(lists), B.device_pointer_array(lists), (C.c_void_p * 3)(1, None, 3), [lists[0], None, 12345], [lists[0], True, 7], [], (), None,
             [object()], "abc", [t] * 65]
    for stream in (None, 0, 5, _Stream(), True, 1.5, "x", np.int64(3)):
        yield "ddp_pack", (2, t, stream)
        yield "ddp_local_update", (opt, stream)
    for slot in (0, -1, 2 ** 31 - 1, 2 ** 31, -2 ** 40, 2 ** 70, True, 1.0, None, np.int32(3)):
        yield "ddp_unpack", (slot, t, 9)
        yield "ddp_fused_sync_update_layers", (1, slot, 2, lists, 0, 1, 4, 3, s, opt, 9)
    for buf in (t, t[3:], t.numpy(), None, 64):
        yield "ddp_pack_wire16", (1, buf, 9)
        yield "ddp_partial_average", (1, t, lists, 4, 0, buf, None, 9)
    for p in peers:
        yield "ddp_partial_average", (1, t, p, 4, 2, t, s, 9)
        yield "ddp_partial_average_wire16", (1, t, p, 4, 2, t, None, 9)
        yield "ddp_fused_sync_update", (1, p, 4, 2, s, opt, 9)
        yield "ddp_fused_sync_update_wire16", (1, p, 4, 2, None, opt, 9)
        yield "ddp_fused_sync_update_layers", (1, 0, 2, p, 0, 1, 4, 3, s, opt, 9)

    class Own(B.ddp_opt):
        pass

    for o in (opt, Own(0, 0.5), None, C.create_string_buffer(64), 7):
        yield "ddp_local_update_layers", (0, 2, o, 9)
        yield "ddp_fused_sync_update", (1, lists, 4, 2, s, o, None)


def test_same_as_the_general_path(stub, monkeypatch):
    ctx = B.Context(0)
    for name, args in _forms():
        fast, general = _both(stub, monkeypatch, lambda: getattr(ctx, name)(*args))
        assert fast == general, (name, args)
    t = torch.zeros(8)
    fast, general = _both(stub, monkeypatch, lambda: ctx.ddp_pack(slot=3, flat_local=t))
    assert fast == general and fast[0] == ("returns", None) and fast[1][1:4] == [3, t.data_ptr(), 77]
    C.c_int.in_dll(stub, "status").value = 3
    for name, args in list(_forms())[:4]:
        fast, general = _both(stub, monkeypatch, lambda: getattr(ctx, name)(*args))
        assert fast == general and fast[0] == ("DdpError", 3)
    C.c_int.in_dll(stub, "status").value = 0
    ctx.close()
    fast, general = _both(stub, monkeypatch, lambda: ctx.ddp_pack(1, t, 9))
    assert fast == general and fast[1][0] == 0


def test_the_calls_are_taken(stub):
    """Arguments as programs pass them every iteration do not fall back to the general path, which the comparison would not see."""
    at, t, s = B.Context(0)._at, torch.zeros(8), torch.zeros(4, dtype=torch.float64)
    lists, opt, calls = [torch.zeros(4) for _ in range(3)], B.make_opt("sgdm", 0.25, 3), B._calls
    for stream in (None, 0, 5, _Stream()):
        assert [c(at, 1, t, stream) for c in (calls.pack, calls.unpack, calls.pack16)] == [0] * 3
        assert calls.update(at, opt, stream) == 0 and calls.update_layers(at, 0, 2, opt, stream) == 0
        for peers in (lists, tuple(lists), B.device_pointer_array(lists)):
            for stats in (s, None):
                assert [c(at, 1, t, peers, 4, 0, t, stats, stream) for c in (calls.average, calls.average16)] == [0] * 2
                assert [c(at, 1, peers, 4, 0, stats, opt, stream) for c in (calls.fused, calls.fused16)] == [0] * 2
                assert calls.fused_layers(at, 1, 0, 2, peers, 0, 1, 4, 0, stats, opt, stream) == 0


def _short_forms(n):
    """Fewer than N - 1 peers, in every form that peers come in."""
    few = [torch.zeros(4) for _ in range(n)]
    return [few, tuple(few), iter(few), B.device_pointer_array(few), (C.c_char * (8 * n)).from_buffer_copy(B.device_pointer_array(few))], few


@pytest.mark.parametrize("n", [1, 2])
def test_missing_peers_are_null(stub, monkeypatch, n):
    """The library reads N - 1 pointers: those that a caller left out arrive as null, which it refuses, not as whatever lies behind
    the last one (the previous call's peers).  The same on both paths, and where N is none that the library takes."""
    ctx, t, s, opt = B.Context(0), torch.zeros(8), torch.zeros(4, dtype=torch.float64), B.make_opt("sgdm", 0.25, 3)
    full = [torch.zeros(4) for _ in range(3)]
    calls = {"ddp_partial_average": lambda p, N: (1, t, p, N, 0, t, s, 9), "ddp_partial_average_wire16": lambda p, N: (1, t, p, N, 0, t, None, 9),
             "ddp_fused_sync_update": lambda p, N: (1, p, N, 0, s, opt, 9), "ddp_fused_sync_update_wire16": lambda p, N: (1, p, N, 0, s, opt, 9),
             "ddp_fused_sync_update_layers": lambda p, N: (1, 0, 2, p, 0, 1, N, 0, s, opt, 9)}
    for name, args in calls.items():
        for i in range(5):
            for fast in (True, False):
                with monkeypatch.context() as m:
                    if not fast:
                        m.setattr(B, "_calls", B._NoCalls())
                    getattr(ctx, name)(*args(full, 4))
                    forms, few = _short_forms(n)
                    getattr(ctx, name)(*args(forms[i], 4))
                    seen = list((C.c_long * 4).in_dll(stub, "peers"))[:3]
                    assert seen == [q.data_ptr() for q in few] + [0] * (3 - n), (name, i, fast)
        for N in (0, -5, -2 ** 31, 65, 2 ** 31, 2 ** 32 + 4, 2 ** 70, True, np.int32(4), 4.0, None):
            fast, general = _both(stub, monkeypatch, lambda: getattr(ctx, name)(*args(full, N)))
            assert fast[0] == general[0] and fast[1] == general[1], (name, N)


class _Once:
    """A tensor (or a stream) whose address cannot be had the first time."""

    def __init__(self, error, value=64):
        self.error, self.value = error, value

    def _get(self):
        error, self.error = self.error, None
        if error:
            raise error("first")
        return self.value

    data_ptr = _get
    cuda_stream = property(_get)


@pytest.mark.parametrize("error", [KeyboardInterrupt, RuntimeError, AttributeError])
def test_an_argument_s_own_exception_comes_back(stub, monkeypatch, error):
    """What an argument raises when it is asked for its address ends the call, as on the general path; it is not asked again."""
    ctx, t, opt = B.Context(0), torch.zeros(8), B.make_opt("sgdm", 0.25, 3)
    once = lambda: _Once(error)  # noqa: E731
    calls = [lambda: ctx.ddp_pack(1, once(), 9), lambda: ctx.ddp_unpack(1, t, once()), lambda: ctx.ddp_pack_wire16(1, once(), once()),
             lambda: ctx.ddp_partial_average(1, once(), [t] * 3, 4, 0, t, t, 9), lambda: ctx.ddp_partial_average(1, t, [t, once(), t], 4, 0, t, t, 9),
             lambda: ctx.ddp_partial_average_wire16(1, t, (once(), t, t), 4, 0, once(), t, 9),
             lambda: ctx.ddp_partial_average(1, t, [t] * 3, 4, 0, once(), None, 9), lambda: ctx.ddp_partial_average(1, t, [t] * 3, 4, 0, t, once(), 9),
             lambda: ctx.ddp_local_update(opt, once()), lambda: ctx.ddp_local_update_layers(0, 2, opt, once()),
             lambda: ctx.ddp_fused_sync_update(1, [t] * 3, 4, 0, once(), opt, 9), lambda: ctx.ddp_fused_sync_update_wire16(1, [once()] * 3, 4, 0, None, opt, 9),
             lambda: ctx.ddp_fused_sync_update_layers(1, 0, 2, [t] * 3, 0, 1, 4, 0, None, opt, once()),
             # (two that cannot be used: the one that the general path looks at first decides)
             lambda: ctx.ddp_local_update(None, once()), lambda: ctx.ddp_fused_sync_update(1, [t] * 3, 4, 0, None, 7, once()),
             lambda: ctx.ddp_partial_average(1, once(), [t] * 3, 4, 2 ** 40, t, None, "x"), lambda: ctx.ddp_pack(None, once(), 9)]
    for k, call in enumerate(calls):
        got = []
        for path in (B._calls, B._NoCalls()):
            with monkeypatch.context() as m:
                m.setattr(B, "_calls", path)
                try:
                    got.append(("returns", call()))
                except BaseException as e:  # noqa: BLE001
                    got.append((type(e), str(e)))
        assert got[0] == got[1], k
        assert got[0] == (error, "first") or k in (13, 14), k


def test_forked_child_takes_the_general_path(stub, monkeypatch):
    ctx, t = B.Context(0), torch.zeros(8)
    B._calls.set_stream_query(lambda: True, lambda: 0, lambda d: 78)
    assert B._calls.pack(ctx._at, 1, t, None) is None and B._calls.pack(ctx._at, 1, t, 5) == 0


@pytest.mark.parametrize("missing", ["compiler", "headers"])
def test_build_without_compiler_or_headers(tmp_path, monkeypatch, capfd, missing):
    """hipcc alone builds the library: without the module the calls take the general path, and no stale module stays behind."""
    from paper_2502_11058_amd import build
    stale = tmp_path / "_calls.so"
    stale.write_bytes(b"stale")
    monkeypatch.setattr(build, "CALLS", str(stale))
    monkeypatch.setattr(build, "_run", lambda cmd, verbose: pytest.fail("nothing to run"))
    if missing == "compiler":
        monkeypatch.setenv("PATH", str(tmp_path))
    else:
        monkeypatch.setattr(build.sysconfig, "get_path", lambda name: str(tmp_path))
    build.build_calls()
    assert not stale.exists() and "marshalled in Python" in capfd.readouterr().err
