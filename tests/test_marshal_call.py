"""without_gil of the binding's extension (csrc/marshal_call.h, host code):
the call runs without the interpreter's lock, and a C++ exception of the call
becomes a Python exception with the lock taken again. The interpreter runs in
a process of its own: without the lock it ends in an abort or a crash."""
import os
import subprocess
import sys
import sysconfig

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1906_05936_amd", "csrc")

MODULE = r"""
#include "marshal_call.h"
#include <stdexcept>
static PyObject* call(PyObject*, PyObject* arg) {
    const long what = PyLong_AsLong(arg);
    return without_gil([&]() -> int {
        if (PyGILState_Check()) throw std::logic_error("called with the lock");
        if (what == 1) throw std::bad_alloc();
        if (what == 2) throw std::runtime_error("from the library");
        if (what == 3) throw 5;
        return 7;
    });
}
static PyMethodDef methods[] = {{"call", call, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
static PyModuleDef def = {PyModuleDef_HEAD_INIT, "probe", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};
PyMODINIT_FUNC PyInit_probe() { return PyModule_Create(&def); }
"""

SCRIPT = r"""
import gc, probe
assert probe.call(0) == 7
for what, kind, text in ((1, MemoryError, ""), (2, RuntimeError, "from the library"), (3, RuntimeError, "unknown")):
    for _ in range(100):
        try:
            probe.call(what)
        except kind as e:
            assert text in str(e), e
        else:
            raise AssertionError(what)
    gc.collect()
print("ok")
"""


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    d = tmp_path_factory.mktemp("marshal_call")
    (d / "probe.cpp").write_text(MODULE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + CSRC, "-isystem",
                    sysconfig.get_paths()["include"], str(d / "probe.cpp"), "-o", str(d / "probe.so")], check=True)
    return d


def test_exceptions_of_the_call_become_python_exceptions(probe):
    r = subprocess.run([sys.executable, "-c", SCRIPT], cwd=probe, capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stderr
