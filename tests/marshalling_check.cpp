// csrc/va_host.cpp as it is, but for CPU tensors and a current stream that the test sets, so that its checks, allocations and
// errors can be looked at without a GPU; and a CPU allocator that says whether it was called with the interpreter's lock
// held, and can be told to be out of memory.
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/core/CPUAllocator.h>
#include <c10/hip/HIPStream.h>

namespace c10::hip {
void* test_stream = nullptr;
struct TestStream {
    void* stream() const { return test_stream; }
};
TestStream test_current_stream(int = -1) { return {}; }
}  // namespace c10::hip

#define is_cuda is_cpu
#define getCurrentHIPStream test_current_stream
#define PyInit__varlen_attn_host init_native
#include "../paper_2605_08962_amd/csrc/va_host.cpp"

namespace {

int with_lock = 0, without_lock = 0, out_of_memory = 0;

struct Watched : c10::Allocator {
    c10::Allocator* base = c10::GetDefaultCPUAllocator();
    c10::DataPtr allocate(size_t n) override {
        ++(PyGILState_Check() ? with_lock : without_lock);
        TORCH_CHECK_WITH(OutOfMemoryError, !out_of_memory, "the test has no memory");
        return base->allocate(n);
    }
    c10::DeleterFnPtr raw_deleter() const override { return base->raw_deleter(); }
    void copy_data(void* to, const void* from, size_t n) const override { base->copy_data(to, from, n); }
} watched;

// watch(out of memory from here on) -> allocations so far with and without the lock, counted from zero again
PyObject* watch(PyObject*, PyObject* fail) {
    c10::SetCPUAllocator(&watched, 255);
    out_of_memory = PyObject_IsTrue(fail);
    PyObject* r = Py_BuildValue("ii", with_lock, without_lock);
    with_lock = without_lock = 0;
    return r;
}
PyObject* set_current_stream(PyObject*, PyObject* handle) {
    c10::hip::test_stream = PyLong_AsVoidPtr(handle);
    if (PyErr_Occurred()) return nullptr;
    Py_RETURN_NONE;
}
PyMethodDef more[] = {{"watch", watch, METH_O, nullptr},
                      {"set_current_stream", set_current_stream, METH_O, nullptr},
                      {nullptr, nullptr, 0, nullptr}};

}  // namespace

PyMODINIT_FUNC PyInit_marshalling_check() {
    PyObject* m = init_native();
    if (m && PyModule_AddFunctions(m, more) < 0) Py_CLEAR(m);
    return m;
}
