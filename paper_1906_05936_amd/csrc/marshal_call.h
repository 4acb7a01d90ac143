// Runs a call of the library without the interpreter's lock, for the
// extension _marshal.
#pragma once

#include <Python.h>

#include <exception>
#include <new>

// Gives the interpreter lock up for a scope; taken again on every way out of it.
class WithoutGil {
public:
    WithoutGil() : state_(PyEval_SaveThread()) {}
    ~WithoutGil() { PyEval_RestoreThread(state_); }
    WithoutGil(const WithoutGil&) = delete;
    WithoutGil& operator=(const WithoutGil&) = delete;

private:
    PyThreadState* state_;
};

// The status `call` returns, as a Python int. A C++ exception of the call (the
// library's host tables may fail to allocate) becomes a Python one: work may
// have been enqueued by then, so the call must not be made again.
template <typename Call>
PyObject* without_gil(const Call& call) {
    long status;
    try {
        const WithoutGil unlocked;
        status = static_cast<long>(call());
    } catch (const std::bad_alloc&) {
        return PyErr_NoMemory();
    } catch (const std::exception& e) {
        PyErr_SetString(PyExc_RuntimeError, e.what());
        return nullptr;
    } catch (...) {
        PyErr_SetString(PyExc_RuntimeError, "unknown C++ exception");
        return nullptr;
    }
    return PyLong_FromLong(status);
}
