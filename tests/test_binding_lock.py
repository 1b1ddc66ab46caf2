"""An exception inside a call of the compiled binding (a runtime that does not answer, memory that runs out in the library) is answered with the
interpreter's lock held.  The binding's own code with one more function, whose library call throws; in a process of its own, which
the touch of the interpreter without its lock would end.  Without a GPU the question for the stream throws first, from the same place."""
import os
import subprocess
import sys

from paper_2402_02320_amd import build

HARNESS = r"""
#include "%s"
static PyObject *throws(PyObject *, PyObject *)
{
    return guarded([&]() -> PyObject * { return run(at::Tensor(), [](spin_stream) -> spin_status { throw std::bad_alloc(); }); });
}
static PyMethodDef harness_methods[] = {{"throws", throws, METH_NOARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
static PyModuleDef harness = {PyModuleDef_HEAD_INIT, "harness", nullptr, -1, harness_methods, nullptr, nullptr, nullptr, nullptr};
PyMODINIT_FUNC PyInit_harness() { return PyModule_Create(&harness); }
"""


def test_an_exception_in_a_call_is_answered_with_the_lock_held(tmp_path):
    source = tmp_path / "harness.cpp"
    source.write_text(HARNESS % os.path.join(build.CSRC, "binding.cpp"))
    build.build_binding(source=str(source), target=str(tmp_path / "harness.so"))
    code = ("import torch, harness, threading\n"
            "for _ in range(100): assert harness.throws() is None\n"
            "t = threading.Thread(target=lambda: [harness.throws() for _ in range(100)]); t.start()\n"
            "for _ in range(100): assert harness.throws() is None\n"
            "t.join(); print('answered')")
    res = subprocess.run([sys.executable, "-c", code], cwd=str(tmp_path), stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300,
                         env=dict(os.environ, PYTHONPATH=str(tmp_path)))
    assert res.returncode == 0 and "answered" in res.stdout, res.stdout[-3000:]
