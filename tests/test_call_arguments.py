"""What the collectives' Python entry points take: lists and tuples of tensors and of addresses, which go
through the native module, and everything else through ctypes, with the same outcome.  Calls on
an empty payload look at no buffer.  No GPU."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

import paper_1910_04940_amd as bl
import synth_inputs as si
from paper_1910_04940_amd import binding, build

torch = pytest.importorskip("torch")


class Buffer:
    def __init__(self, at):
        self.at = at

    def data_ptr(self):
        return self.at


class Broken:
    def data_ptr(self):
        raise RuntimeError("no storage")


class Row(list):
    pass


def _schedule(n=0, op=bl.BLINK_OP_ALLREDUCE):
    t = si.complete_graph(4)
    return bl.blink_make_schedule(bl.blink_pack_trees(t.k, t.src, t.dst, t.cap, 0), op, n, 16)


FORMS = {
    "addresses": [16, 32, 48, 64],
    "tuple": (16, 32, 48, 64),
    "objects": [Buffer(16 * i) for i in range(1, 5)],
    "tensors": [torch.zeros(8) for _ in range(4)],
    "numpy integers": [np.int64(16 * i) for i in range(1, 5)],
    "numpy addresses in objects": [Buffer(np.int64(16 * i)) for i in range(1, 5)],
    "a list of one's own": Row([16, 32, 48, 64]),
    "an array": np.array([16, 32, 48, 64]),
    "mixed": [16, Buffer(32), torch.zeros(8), np.uint64(64)],
    "negative": [-16, -32, -48, -64],
}


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("native", [True, False])
def test_forms_of_buffers(form, native, monkeypatch):
    s = _schedule()
    if not native:
        monkeypatch.setattr(binding, "_call", lambda *a: None)
    for stream in (0, None, 1 << 63):
        bl.blink_allreduce(FORMS[form], 0, bl.BLINK_FP32, s, stream)
    bl.blink_allreduce(bufs=FORMS[form], n_elems=0, dtype=bl.BLINK_INT32, schedule=s)
    bl.blink_allreduce_op(FORMS[form], 0, bl.BLINK_INT32, bl.BLINK_MAX, s, stream=0)
    bl.blink_broadcast(FORMS[form], np.int64(0) if not native else 0, True, _schedule(op=bl.BLINK_OP_BROADCAST))


@pytest.mark.parametrize("native", [True, False])
@pytest.mark.parametrize("arguments,error,status", [
    (([16] * 17, 0, 1), bl.BlinkError, bl.BLINK_EMISMATCH), (([16] * 3, 0, 1), bl.BlinkError, bl.BLINK_EMISMATCH),
    (([], 0, 1), bl.BlinkError, bl.BLINK_EMISMATCH), (([16, 32, 48, 64], 0, 7), bl.BlinkError, bl.BLINK_EINVAL),
    (([16, 32, 48, 64], -1, 1), bl.BlinkError, bl.BLINK_EMISMATCH), (([16, 32, 48, 64], 0, -1), bl.BlinkError, bl.BLINK_EINVAL),
    (([16, 32, 48, 64], 8, 1), bl.BlinkError, bl.BLINK_EMISMATCH), (([16, 32, "x", 64], 0, 1), ValueError, None),
    (([16, None, 48, 64], 0, 1), TypeError, None), ((None, 0, 1), TypeError, None), ((16, 0, 1), TypeError, None),
    (([16, 32, 48, 64], 0.5, 1), ctypes.ArgumentError, None), (([16, Broken(), 48, 64], 0, 1), RuntimeError, None)])
def test_what_is_refused(arguments, error, status, native, monkeypatch):
    s = _schedule()
    if not native:
        monkeypatch.setattr(binding, "_call", lambda *a: None)
    with pytest.raises(error) as e:
        bl.blink_allreduce(*arguments, s)
    if status is not None:
        assert e.value.status == status
    with pytest.raises(AttributeError):
        bl.blink_allreduce([16, 32, 48, 64], 0, 1, None)


def test_a_list_that_shrinks_while_it_is_read():
    row = []

    class Shrinks:
        def data_ptr(self):
            row.clear()
            return 16

    row += [Shrinks() for _ in range(4)]
    with pytest.raises(bl.BlinkError):
        bl.blink_allreduce(row, 0, bl.BLINK_FP32, _schedule())


def test_the_usual_call_is_native(monkeypatch):
    s = _schedule()
    monkeypatch.setattr(binding, "_pointers", lambda bufs: pytest.fail("through ctypes"))
    bl.blink_allreduce([torch.zeros(8) for _ in range(4)], 0, bl.BLINK_FP32, s, 0)
    bl.blink_reduce([16, 32, 48, 64], 0, bl.BLINK_FP32, bl.BLINK_SUM, _schedule(op=bl.BLINK_OP_REDUCE))


def test_without_the_native_module():
    """Packing, scheduling and calls work on the library alone."""
    code = """
import sys
sys.modules["paper_1910_04940_amd._blinkcall"] = None     # what importing it then raises is an ImportError
import paper_1910_04940_amd as bl
import synth_inputs as si
t = si.complete_graph(4)
s = bl.blink_make_schedule(bl.blink_pack_trees(t.k, t.src, t.dst, t.cap, 0), bl.BLINK_OP_ALLREDUCE, 0, 16)
bl.blink_allreduce([16, 32, 48, 64], 0, bl.BLINK_FP32, s)
try:
    bl.blink_allreduce([16, 32, 48], 0, bl.BLINK_FP32, s)
except bl.BlinkError as e:
    print("status", e.status == bl.BLINK_EMISMATCH)
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = subprocess.run([sys.executable, "-c", code], cwd=root, check=True, capture_output=True, text=True).stdout
    assert out.split() == ["status", "True"]


def test_a_module_that_cannot_be_built_is_said_and_left_out(tmp_path, monkeypatch, capfd):
    to = str(tmp_path / "_blinkcall.so")
    assert build.build_call(to) and os.path.exists(to)
    for compiler in ("false", str(tmp_path / "no such compiler")):
        monkeypatch.setenv("CC", compiler)
        assert not build.build_call(to) and not os.path.exists(to)
        assert "ctypes" in capfd.readouterr().err
