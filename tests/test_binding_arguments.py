"""What the Python binding looks at before it hands a pointer to the library.  On the CPU, with a library in whose place every call is
written down: a call that has to be refused must not reach it."""
import pytest
import torch

from paper_2402_02320_amd import spin


class Record:
    """In place of the loaded library: every entry point returns `answers` of its name (0 otherwise) and is written down."""

    def __init__(self, **answers):
        self.answers, self.launched = answers, []

    def __getattr__(self, name):
        def entry(*args):
            if not name.endswith(("_bytes", "_string", "_error")):
                self.launched.append(name)
            return self.answers.get(name, 1024 if name.endswith("_bytes") else b"" if name.endswith(("_string", "_error")) else 0)
        return entry


@pytest.fixture
def record(monkeypatch):
    r = Record()
    monkeypatch.setattr(spin, "_lib", r)
    monkeypatch.setattr(spin, "_fast", None)
    monkeypatch.setattr(spin, "_dev", lambda t, name: t.data_ptr())
    monkeypatch.setattr(spin, "_dev32", lambda t, name: t.data_ptr())
    monkeypatch.setattr(spin, "_stream", lambda: 0)
    return r


class Workspace:
    """A workspace that says it is on the GPU."""
    is_cuda = True

    def is_contiguous(self): return True
    def data_ptr(self): return 256
    def numel(self): return 1024
    def element_size(self): return 1


def w(*shape, words=1):
    return torch.zeros(shape + ((2,) if words == 2 else ()), dtype=torch.int64)


WS = Workspace()
MM, MM2 = [w(2, 1, 4, 4)] * 5, [w(2, 1, 4, 4, words=2)] * 5
# name -> words of the result, call with `out`
CALLS = {
    "share": (24, lambda o: spin.share(w(8), 3, 1, 1, out=o)),
    "bshare": (24, lambda o: spin.bshare(w(8), 3, 1, 1, out=o)),
    "mul": (24, lambda o: spin.beaver_mul(*[w(3, 8)] * 5, out=o)),
    "and": (24, lambda o: spin.beaver_and(*[w(3, 8)] * 5, out=o)),
    "mul_trunc": (24, lambda o: spin.beaver_mul_trunc(*[w(3, 8)] * 8, 16, out=o)),
    "mul_bcast": (48, lambda o: spin.beaver_mul_bcast(w(3, 2, 4), w(3, 2, 4, 2), w(3, 2, 4), *[w(3, 2, 4, 2)] * 2, True, out=o)),
    "trunc": (24, lambda o: spin.trunc(*[w(3, 8)] * 4, 16, out=o)),
    "lincomb": (24, lambda o: spin.lincomb_trunc([w(3, 8)] * 2, [1, 2], out=o)),
    "square": (24, lambda o: spin.completed_square_trunc(w(3, 8), 1, 2, 3, 4, [(w(3, 8),) * 3] * 2, [(w(3, 8),) * 3] * 2, (14, 15), out=o)),
    "matmul": (32, lambda o: spin.beaver_matmul(*MM, out=o, workspace=WS)),
    "grouped": (32, lambda o: spin.beaver_matmul_grouped([dict(zip("XYABC", MM)), dict(zip("XYABC", MM), out=o)], workspace=WS)),
    "share128": (48, lambda o: spin.ring128.share(w(8, 2), 3, 1, 1, out=o)),
    "mul128": (48, lambda o: spin.ring128.beaver_mul(*[w(3, 8, 2)] * 5, out=o)),
    "trunc128": (48, lambda o: spin.ring128.trunc(*[w(3, 8, 2)] * 4, 16, out=o)),
    "matmul128": (64, lambda o: spin.ring128.beaver_matmul(*MM2, out=o, workspace=WS)),
    "cast32": (24, lambda o: spin.ring32.cast_from_64(w(3, 8), out=o)),
    "share32": (24, lambda o: spin.ring32.share(w(8), 3, 1, 1, out=o)),
    "mul32": (24, lambda o: spin.ring32.beaver_mul(*[w(3, 8)] * 5, out=o)),
    "trunc32": (24, lambda o: spin.ring32.trunc(*[w(3, 8)] * 4, 16, out=o)),
    "matmul32": (32, lambda o: spin.ring32.beaver_matmul(*MM, out=o, workspace=WS)),
    "probe": (512, lambda o: spin.probe_mfma(w(24 * 128), 2, 1, sink=o)),
}
OPENS = {
    "open": (8, lambda o: spin.open(w(3, 8), out=o)), "bopen": (8, lambda o: spin.bopen(w(3, 8), out=o)),
    "open128": (16, lambda o: spin.ring128.open(w(3, 8, 2), out=o)), "open32": (8, lambda o: spin.ring32.open(w(3, 8), out=o)),
}


@pytest.mark.parametrize("name", sorted(CALLS) + sorted(OPENS))
def test_an_out_that_is_too_short_reaches_no_kernel(name, record):
    words, call = (CALLS.get(name) or OPENS[name])
    two = 2 if name.endswith("128") else 1               # words of an element
    for short in (words - two, two):
        with pytest.raises(spin.SpinError):
            call(w(short // two, words=two))
    assert record.launched == []
    call(w(words // two, words=two))
    assert len(record.launched) == 1


@pytest.mark.parametrize("name", sorted(CALLS))
def test_a_longer_out_holds_the_result_in_front(name, record):
    words, call = CALLS[name]
    two = 2 if name.endswith("128") else 1
    call(w(words // two + 1, words=two))
    assert len(record.launched) == 1


@pytest.mark.parametrize("name", sorted(OPENS))
def test_a_longer_out_of_an_opening_would_read_past_the_shares(name, record):
    words, call = OPENS[name]
    two = 2 if name.endswith("128") else 1
    with pytest.raises(spin.SpinError):
        call(w(words // two + 1, words=two))
    assert record.launched == []


def replaced(operands, i, other):
    return operands[:i] + [other] + operands[i + 1:]


@pytest.mark.parametrize("words", [14, 18])
@pytest.mark.parametrize("ring,call,count", [(ring, call, count) for ring in ("ring128", "ring32") for call, count in (("beaver_mul", 5), ("trunc", 4))]
                         + [("ring128", "open", 2), ("ring32", "open", 2)])
def test_operands_of_another_size_reach_no_kernel(ring, call, count, words, record):
    entry, two = getattr(getattr(spin, ring), call), 2 if ring == "ring128" else 1
    more = [16] if call == "trunc" else []
    same = [w(2, 8, words=two)] * count
    for i in range(1, count):
        with pytest.raises(spin.SpinError):
            entry(*replaced(same, i, w(2, words // 2, words=two)), *more)
    assert record.launched == []
    entry(*same, *more)
    assert len(record.launched) == 1


@pytest.mark.parametrize("workspace", [torch.zeros(4096, dtype=torch.uint8), "expanded"])
@pytest.mark.parametrize("call", [lambda ws: spin.beaver_matmul(*MM, workspace=ws),
                                  lambda ws: spin.beaver_matmul_grouped([dict(zip("XYABC", MM))], workspace=ws),
                                  lambda ws: spin.ring128.beaver_matmul(*MM2, workspace=ws), lambda ws: spin.ring32.beaver_matmul(*MM, workspace=ws)])
def test_a_workspace_on_the_host_or_of_repeated_bytes_reaches_no_kernel(call, workspace, record, monkeypatch):
    if isinstance(workspace, str):
        workspace = Workspace()
        monkeypatch.setattr(workspace, "is_contiguous", lambda: False, raising=False)
    with pytest.raises(spin.SpinError):
        call(workspace)
    assert record.launched == []


@pytest.mark.parametrize("status", [1, 2, 3, 4])
def test_a_call_that_failed_is_not_made_again(status, record, monkeypatch):
    # a launch may fail with earlier ones of the same call under way, and out may be C: a second call would add their parts twice
    class Failing:
        @staticmethod
        def matmul(*args):
            return status
    monkeypatch.setattr(spin, "_fast", Failing)
    with pytest.raises(spin.SpinError):
        spin.beaver_matmul(*MM, out=MM[4], workspace=WS)
    assert record.launched == []


def test_the_dimensions_of_a_refused_product_are_named(record, monkeypatch):
    class Failing:
        @staticmethod
        def matmul(*args):
            return 2
    asked = []
    monkeypatch.setattr(spin, "_fast", Failing)
    monkeypatch.setattr(spin, "beaver_matmul_workspace_bytes", lambda *dims: asked.append(dims) or 0)
    with pytest.raises(spin.SpinError, match="invalid matmul dimensions"):
        spin.beaver_matmul(w(2, 3, 4, 5), w(2, 3, 5, 6), w(2, 3, 4, 5), w(2, 3, 5, 6), w(2, 3, 4, 6))
    assert asked == [(2, 3, 4, 6, 5, spin.LIMB_MFMA)]


@pytest.mark.parametrize("content", [None, b"not a shared object"])
def test_a_binding_that_does_not_load_raises_every_time(content, monkeypatch, tmp_path):
    if content is not None:
        (tmp_path / "_binding.so").write_bytes(content)
    monkeypatch.setattr(spin, "_lib", None)
    monkeypatch.setattr(spin, "_fast", None)
    monkeypatch.setattr(spin, "BINDING_PATH", str(tmp_path / "_binding.so"))
    for _ in range(2):
        with pytest.raises(spin.SpinError, match="_binding.so"):
            spin.lib()
    assert spin._lib is None and spin._fast is None
