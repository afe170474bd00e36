"""The binding takes its native calls only from a module that was built from these sources, against this torch."""
import os
import subprocess
import sysconfig
import warnings

import pytest

from paper_2605_13907_amd import binding as B

# A module as an earlier build may have left it: it loads, and takes another table of entry points.
OTHER = r"""
#include <Python.h>
static PyObject* init(PyObject*, PyObject* args) {
  if (PyTuple_GET_SIZE(args) != 3) { PyErr_SetString(PyExc_TypeError, "init: three addresses"); return nullptr; }
  Py_RETURN_NONE;
}
static PyMethodDef methods[] = {{"init", init, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
static PyModuleDef def = {PyModuleDef_HEAD_INIT, "_ais_fast", nullptr, -1, methods};
PyMODINIT_FUNC PyInit__ais_fast(void) {
  PyObject* m = PyModule_Create(&def);
#ifdef STAMP
  PyModule_AddStringConstant(m, "stamp", STAMP);
#endif
  return m;
}
"""


def load(monkeypatch, path):
    monkeypatch.setattr(B, "FAST_PATH", str(path))
    monkeypatch.setattr(B, "_FAST", None)
    return B._load_fast()


def test_module_of_this_tree(monkeypatch):
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        fast = load(monkeypatch, B.FAST_PATH)
        assert fast is not None and fast.stamp == B.fast_stamp() and B._load_fast() is fast
        assert load(monkeypatch, "/nowhere/_ais_fast.so") is None


@pytest.mark.parametrize("stamp", [None, "0" * 64])
def test_module_of_another_build(monkeypatch, tmp_path, stamp):
    src, so = tmp_path / "other.cpp", tmp_path / "_ais_fast.so"
    src.write_text(OTHER)
    define = [] if stamp is None else [f'-DSTAMP="{stamp}"']
    subprocess.run([os.environ.get("CXX", "g++"), "-shared", "-fPIC", "-std=c++17", *define,
                    f"-I{sysconfig.get_paths()['include']}", str(src), "-o", str(so)], check=True)
    with pytest.warns(RuntimeWarning, match="other sources"):
        assert load(monkeypatch, so) is None


def test_file_that_does_not_load(monkeypatch, tmp_path):
    so = tmp_path / "_ais_fast.so"
    so.write_bytes(b"not a module")
    with pytest.warns(RuntimeWarning):
        assert load(monkeypatch, so) is None


def test_stamp_follows_what_it_depends_on(monkeypatch):
    before = B.fast_stamp()
    monkeypatch.setattr(B.torch, "__version__", "0.0")
    assert B.fast_stamp() != before
