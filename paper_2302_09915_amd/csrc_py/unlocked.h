// Work without the interpreter lock.
#pragma once

#include <cxxabi.h>

#include <Python.h>

// Runs a C entry point or an allocation without the interpreter lock, as ctypes and torch's own binding do (another
// thread may need the lock to leave the allocator).  The lock is not taken again in a destructor: once
// the interpreter ends, taking it ends a daemon thread by unwinding its stack, which a function that may
// not throw turns into an abort of the process.
template <class F>
auto unlocked(F call) {
    PyThreadState* state = PyEval_SaveThread();
    try {
        auto r = call();
        PyEval_RestoreThread(state);
        return r;
    } catch (abi::__forced_unwind&) {
        throw;
    } catch (...) {
        PyEval_RestoreThread(state);
        throw;
    }
}
