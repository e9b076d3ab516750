"""The native part of the binding (csrc/marshal.cpp) against its general way through ctypes, on the CPU: the library's functions are
replaced by ones that write down what they are given.  A regular call hands over the same arguments either way; a call that is not
regular in any one respect is left alone."""
import ctypes
import dis
import importlib.util
import os
import shutil
import subprocess
import sys
from types import SimpleNamespace

import pytest
import torch

from paper_2601_15498_amd import binding as M

B, N, V, H = 2, 5, 16, 128
PTR = ctypes.c_void_p


@pytest.fixture
def recorder(monkeypatch):
    real = M.lib()
    got, keep = [], []

    def stub(fn):
        types = [PTR if not hasattr(t, "_type_") or not isinstance(t._type_, str) else t for t in fn.argtypes]

        def run(*args):
            vals = list(args)
            if fn is real.mars_margin_stats:   # two host arrays
                vals[7] = tuple((ctypes.c_float * 6).from_address(vals[7]))
                vals[8] = tuple((ctypes.c_int32 * 3).from_address(vals[8]))
            elif fn is not real.mars_verify:   # the options
                o = M.VerifyOptionsStruct.from_address(vals[-1])
                vals[-1] = tuple(getattr(o, f) for f, _ in o._fields_)
            got.append(tuple(vals))
            return 0

        c = ctypes.CFUNCTYPE(ctypes.c_int, *types)(run)
        keep.append(c)
        return c

    names = ("mars_verify", "mars_verify_ex", "mars_margin_stats", "mars_lmhead_verify", "mars_lmhead_verify_sampling")
    stubs = {n: stub(getattr(real, n)) for n in names}
    native = M._calls()
    if "MARSHAL_UNDER_TEST" in os.environ:   # a build of the module other than the package's
        spec = importlib.util.spec_from_file_location("_marshal", os.environ["MARSHAL_UNDER_TEST"])
        native = importlib.util.module_from_spec(spec)
        monkeypatch.setattr(M, "_native", native)
    native.bind(*(ctypes.cast(stubs[n], PTR).value for n in names))
    # the general way: the same stubs behind ctypes
    general = {n: (lambda c, k: lambda *a: c(*[ctypes.cast(x, PTR) if isinstance(x, (ctypes.Array, type(ctypes.byref(ctypes.c_int()))))
                                               else x for x in a]))(c, n) for n, c in stubs.items()}
    monkeypatch.setattr(M, "_stream", lambda: 0x7F)
    yield got, native, SimpleNamespace(**general)
    native.bind(*(ctypes.cast(getattr(real, n), PTR).value for n in names))


def inputs(dtype=torch.bfloat16, K=1, commit=False, sampling=True, dense=torch.float32, stats=True):
    d = dict(logits=torch.zeros(B, N, V).to(dtype), tok=torch.zeros(B, N, dtype=torch.int32), par=torch.zeros(B, N, dtype=torch.int32),
             theta=torch.ones((K, B) if K > 1 else (B,)), u=torch.zeros(B, N + 1) if sampling else None,
             q=None if dense is None else torch.zeros(B, N, V).to(dense), T=0.7 if sampling else 0,
             out=M.VerifyOutputs(B, N, "cpu", want_stats=stats, want_diag=sampling, n_theta=K, want_commit=commit),
             ws=torch.zeros(1000, dtype=torch.uint8), hidden=torch.zeros(B, N, H).to(torch.bfloat16),
             weight=torch.zeros(V, H).to(torch.bfloat16), lo=torch.zeros(B, N, V).to(torch.bfloat16), K=K, commit=commit,
             rows=torch.zeros(B * N, 4), counts=torch.zeros(12 + 6 + 4, dtype=torch.int32))
    return SimpleNamespace(**d)


ENTRIES = {
    "verify": lambda s: M.mars_verify(s.logits, s.tok, s.par, s.theta, s.T, s.u, s.q, s.out, s.ws),
    "verify_ex": lambda s: M.mars_verify_ex(s.logits, s.tok, s.par, s.theta, s.T, s.u, s.q, s.out, s.ws, indicator=1, n_theta=s.K,
                                            want_commit=s.commit, spin_limit=3, stages=2),
    "margin_stats": lambda s: M.mars_margin_stats(s.logits, s.theta, s.T, (0.0, 1.0, 0.25, 2.0, 0, 1), (3, 4, 5), s.rows, s.counts, s.ws),
    "lmhead_verify": lambda s: M.mars_lmhead_verify(s.hidden, s.weight, s.tok, s.par, s.theta, s.out, s.ws, indicator=2, n_theta=s.K,
                                                    want_commit=s.commit, stages=1),
    "lmhead_verify_sampling": lambda s: M.mars_lmhead_verify_sampling(s.hidden, s.weight, s.tok, s.par, s.theta, s.T, s.u, s.q, s.lo,
                                                                      s.out, s.ws, n_theta=s.K, want_commit=s.commit, spin_limit=9),
}
FORMS = [dict(), dict(dtype=torch.float32, dense=torch.bfloat16), dict(dtype=torch.int16, dense=None), dict(dtype=torch.uint16, stats=False),
         dict(commit=True), dict(K=3, commit=True)]


@pytest.mark.parametrize("entry", ENTRIES)
@pytest.mark.parametrize("form", range(len(FORMS)))
def test_a_regular_call_hands_over_the_same_either_way(recorder, monkeypatch, entry, form):
    got, native, general = recorder
    if FORMS[form].get("K", 1) > 1 and entry in ("verify", "margin_stats"):
        return
    s = inputs(**FORMS[form])
    ENTRIES[entry](s)
    assert len(got) == 1
    monkeypatch.setattr(M, "_lib", general)
    monkeypatch.setattr(M, "_native", SimpleNamespace(**{e: lambda *a: None for e in ENTRIES}))
    ENTRIES[entry](s)
    assert len(got) == 2 and got[0] == got[1]


class Sub(torch.Tensor):
    pass


IRREGULAR = {
    "not contiguous": ("logits", lambda t: torch.zeros(B, V, N, dtype=t.dtype).transpose(1, 2)),
    "type of the logits": ("logits", lambda t: t.double()),
    "rank of the logits": ("logits", lambda t: t[0]),
    "shape of the tokens": ("tok", lambda t: t[:, 1:].contiguous()),
    "type of the tokens": ("tok", lambda t: t.long()),
    "strides of the parents": ("par", lambda t: torch.zeros(N, B, dtype=torch.int32).t()),
    "thresholds": ("theta", lambda t: t[:1]),
    "type of the thresholds": ("theta", lambda t: t.double()),
    "uniforms": ("u", lambda t: t[:, :-1].contiguous()),
    "type of the draft distribution": ("q", lambda t: t.double()),
    "shape of the draft distribution": ("q", lambda t: t[:, :, 1:].contiguous()),
    "a subclass": ("logits", lambda t: t.as_subclass(Sub)),
    "no tensor": ("logits", lambda t: t.float().numpy()),
    "a temperature of another kind": ("T", lambda t: "0.7"),
    "an output that is not there": ("out", lambda o: SimpleNamespace(**{**o.__dict__, "path_idx": None})),
    "no memory": ("theta", lambda t: t.to_sparse()),   # (mars_verify: found where its address is asked for)
}


@pytest.mark.parametrize("what", IRREGULAR)
def test_a_call_that_is_not_regular_is_left_alone(recorder, what):
    got, native, _ = recorder
    s = inputs()
    name, change = IRREGULAR[what]
    setattr(s, name, change(getattr(s, name)))
    assert native.verify(s.logits, s.tok, s.par, s.theta, s.T, s.u, s.q, s.out, s.ws, lambda: 0) is None
    assert native.verify_ex(s.logits, s.tok, s.par, s.theta, s.T, s.u, s.q, s.out, s.ws, 0, 1, 0, 0, lambda: 0) is None
    assert native.verify(s.logits) is None and not got


class Slot(M.VerifyOutputs):
    """Outputs whose attributes are made when they are asked for: views of slot 1 of larger buffers that nobody else holds, and a
    number of thresholds that is worked out."""

    def __init__(self, like):
        self.buf = {k: (torch.stack([v, v]) if isinstance(v, torch.Tensor) else v) for k, v in like.__dict__.items()}

    def __getattr__(self, name):
        if name == "buf" or name not in self.buf:
            raise AttributeError(name)
        v = self.buf[name]
        return v[1] if isinstance(v, torch.Tensor) else v


class Made(Slot):
    accept_mask = property(lambda self: self.buf["accept_mask"][1])
    n_theta = property(lambda self: int("1000000") - 1000000 + self.buf["n_theta"])


@pytest.mark.parametrize("kind", [Slot, Made])
@pytest.mark.parametrize("entry", [e for e in ENTRIES if e != "margin_stats"])
def test_outputs_that_are_made_when_they_are_asked_for(recorder, monkeypatch, kind, entry):
    got, native, general = recorder
    s = inputs(commit=entry != "verify")
    s.out = kind(s.out)
    monkeypatch.setattr(M, "_lib", None)   # the general way is not taken
    ENTRIES[entry](s)
    assert len(got) == 1 and s.out.accept_mask.data_ptr() in got[0] and s.out.path_idx.data_ptr() in got[0]
    monkeypatch.setattr(M, "_lib", general)
    monkeypatch.setattr(M, "_native", SimpleNamespace(**{e: lambda *a: None for e in ENTRIES}))
    ENTRIES[entry](s)
    assert len(got) == 2 and got[0] == got[1]


def test_no_object_is_looked_at_once_it_has_been_given_back(tmp_path):
    # the calls above with the module built under AddressSanitizer, in a process of its own
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    from paper_2601_15498_amd import build
    lib = str(tmp_path / "_marshal.so")
    build.build_marshal(out=lib, extra=["-O1", "-g", "-fsanitize=address"])
    asan = subprocess.run(["g++", "-print-file-name=libasan.so"], capture_output=True, text=True).stdout.strip()
    env = dict(os.environ, MARSHAL_UNDER_TEST=lib, LD_PRELOAD=" ".join([asan, os.environ.get("LD_PRELOAD", "")]).strip(), PYTHONMALLOC="malloc",
               ASAN_OPTIONS="verify_asan_link_order=0:detect_leaks=0:allocator_may_return_null=1")
    run = subprocess.run([sys.executable, "-m", "pytest", "-x", "-q", "-s", "-p", "no:cacheprovider", os.path.abspath(__file__),
                          "-k", "made_when_they_are_asked_for or either_way"], capture_output=True, text=True, env=env, timeout=600,
                         cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    said = (run.stdout + run.stderr)
    assert run.returncode == 0 and "AddressSanitizer" not in said, said[:2000]


@pytest.mark.parametrize("why", ["missing", "another PyTorch"])
def test_without_the_native_module_calls_go_through_ctypes(recorder, monkeypatch, why):
    got, native, general = recorder
    if why == "missing":
        monkeypatch.setitem(sys.modules, "paper_2601_15498_amd._marshal", None)   # its import fails
        monkeypatch.delattr("paper_2601_15498_amd._marshal", raising=False)
    else:
        monkeypatch.setattr(native, "torch_version", "0.4.1")
    monkeypatch.setattr(M, "_lib", None)
    monkeypatch.setattr(M, "_native", None)
    with pytest.warns(RuntimeWarning, match="through ctypes"):
        assert M.mars_version() > 0
    monkeypatch.setattr(M, "_lib", general)
    s = inputs()
    for entry in ENTRIES:
        ENTRIES[entry](s)
    assert len(got) == len(ENTRIES)


def test_the_calls_are_there_before_the_library_is():
    # (another thread's first call may come between the two)
    order = [i.argval for i in dis.get_instructions(M.lib) if i.opname == "STORE_GLOBAL"]
    assert order == ["_native", "_lib"]


def test_errors_come_from_the_general_way():
    s = inputs()
    for name, change, error in (("logits", lambda t: t.double(), TypeError), ("tok", lambda t: t.long(), AssertionError),
                                ("theta", lambda t: t[:1], AssertionError)):
        bad = SimpleNamespace(**{**s.__dict__, name: change(getattr(s, name))})
        with pytest.raises(error):
            ENTRIES["verify"](bad)
    with pytest.raises(M.MarsError):   # refused by the library
        M._stream, stream = (lambda: 0), M._stream
        try:
            M.mars_verify(s.logits, s.tok, s.par, s.theta, -1.0, s.u, s.q, s.out, s.ws)
        finally:
            M._stream = stream
