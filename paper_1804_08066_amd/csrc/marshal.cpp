// The binding's argument tables in native code: the checks of a list of tensors and the pointer and item tables
// that the C ABI takes.  A model's batched step names about a hundred tensors, and four attribute reads, two
// size calls and an address for each took 90 of the 98 us of the small CNN's iteration (4 workers, two launches).
//
// Every function returns None for anything but plain tensors of the right kind and size (subclasses, wrapped or
// storage-less tensors, other containers, values out of range); the binding then runs its own checks, which
// accept it or raise.  Nothing is kept between calls.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <cstring>
#include <vector>

#include "mqgrad.h"

namespace {

struct Reject {};

// a contiguous CUDA tensor of `type`
const at::Tensor& plain(PyObject* o, at::ScalarType type) {
    if (!THPVariable_CheckExact(o)) throw Reject{};
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.defined() || !t.is_cuda() || t.scalar_type() != type || !t.is_contiguous()) throw Reject{};
    return t;
}
void* address(PyObject* o, at::ScalarType type, uint64_t least, bool exactly = false) {
    const at::Tensor& t = plain(o, type);
    const uint64_t n = (uint64_t)t.numel();
    if (exactly ? n != least : n < least) throw Reject{};
    return t.data_ptr();
}

// a list or tuple, whose items are borrowed
struct Items {
    PyObject** at;
    Py_ssize_t count;
    explicit Items(PyObject* o) {
        if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) throw Reject{};
        at = PySequence_Fast_ITEMS(o);
        count = PySequence_Fast_GET_SIZE(o);
    }
    Items(PyObject* o, Py_ssize_t want) : Items(o) {
        if (count != want) throw Reject{};
    }
};

uint64_t whole(PyObject* o) {
    const unsigned long long v = PyLong_Check(o) ? PyLong_AsUnsignedLongLong(o) : (unsigned long long)-1;
    if (v == (unsigned long long)-1) {
        PyErr_Clear();
        throw Reject{};
    }
    return v;
}
uint64_t words_of(uint64_t n, uint64_t bits) { return (n >> 5) * bits + (((n & 31u) * bits + 31u) >> 5); }
// floats that describe the ranges of n elements: one scale per bucket, a (min, max) pair per bucket, or one pair
uint64_t ranges_of(uint64_t n, uint64_t bucket, uint64_t kind) {
    if (kind == 2u) return 2u;
    const uint64_t nb = (n + bucket - 1u) / bucket;
    return kind == 1u ? 2u * nb : nb;
}
void check_format(uint64_t bits, uint64_t bucket, uint64_t kind) {
    if (bits < 1u || bits > 8u || kind > 2u || (kind != 2u && (bucket < 32u || bucket > 16384u || bucket % 32u != 0u))) throw Reject{};
}

PyObject* as_bytes(const void* p, size_t bytes) { return PyBytes_FromStringAndSize(static_cast<const char*>(p), (Py_ssize_t)bytes); }

template <class F>
PyObject* guarded(F f) {
    try {
        return f();
    } catch (...) {   // Reject, or what a tensor without storage throws
        PyErr_Clear();
        Py_RETURN_NONE;
    }
}

// pointers(packed, ranges, n, bits, bucket, kind) -> (W, bytes, bytes): the W workers' streams
PyObject* pointers(PyObject*, PyObject* const* a, Py_ssize_t argc) {
    return guarded([&]() -> PyObject* {
        if (argc != 6) throw Reject{};
        const Items packed(a[0]), ranges(a[1], packed.count);
        const uint64_t n = whole(a[2]), bits = whole(a[3]), bucket = whole(a[4]), kind = whole(a[5]);
        check_format(bits, bucket, kind);
        if (packed.count > MQG_MAX_WORKERS) throw Reject{};
        const uint64_t words = words_of(n, bits), floats = ranges_of(n, bucket, kind);
        void *p[MQG_MAX_WORKERS + 1] = {}, *r[MQG_MAX_WORKERS + 1] = {};
        for (Py_ssize_t w = 0; w < packed.count; ++w) {
            p[w] = address(packed.at[w], at::kInt, words);
            r[w] = address(ranges.at[w], at::kFloat, floats);
        }
        const size_t bytes = sizeof(void*) * (size_t)(packed.count > 0 ? packed.count : 1);
        return Py_BuildValue("nNN", packed.count, as_bytes(p, bytes), as_bytes(r, bytes));
    });
}

// stream(grad, packed, ranges, bits, bucket, kind) -> (n, grad, packed, ranges): one encoder call
PyObject* stream(PyObject*, PyObject* const* a, Py_ssize_t argc) {
    return guarded([&]() -> PyObject* {
        if (argc != 6) throw Reject{};
        const uint64_t bits = whole(a[3]), bucket = whole(a[4]), kind = whole(a[5]);
        check_format(bits, bucket, kind);
        const at::Tensor& g = plain(a[0], at::kFloat);
        const uint64_t n = (uint64_t)g.numel();
        void* p = address(a[1], at::kInt, words_of(n, bits));
        void* r = address(a[2], at::kFloat, ranges_of(n, bucket, kind));
        return Py_BuildValue("KKKK", (unsigned long long)n, (unsigned long long)(uintptr_t)g.data_ptr(),
                             (unsigned long long)(uintptr_t)p, (unsigned long long)(uintptr_t)r);
    });
}

// quantize_items(grads, outputs, bases or None, bits, bucket, kind) -> bytes: mqg_quantize_item[count]
PyObject* quantize_items(PyObject*, PyObject* const* a, Py_ssize_t argc) {
    return guarded([&]() -> PyObject* {
        if (argc != 6) throw Reject{};
        const Items grads(a[0]), outputs(a[1], grads.count);
        const uint64_t bits = whole(a[3]), bucket = whole(a[4]), kind = whole(a[5]);
        check_format(bits, bucket, kind);
        std::vector<mqg_quantize_item> items((size_t)grads.count + 1);
        for (Py_ssize_t i = 0; i < grads.count; ++i) {
            const Items out(outputs.at[i], 2);
            const at::Tensor& g = plain(grads.at[i], at::kFloat);
            const uint64_t n = (uint64_t)g.numel();
            mqg_quantize_item& t = items[(size_t)i];
            t.grad = static_cast<const float*>(g.data_ptr());
            t.n = n;
            t.elem_base = a[2] == Py_None ? 0u : whole(Items(a[2], grads.count).at[i]);
            t.packed_out = static_cast<uint32_t*>(address(out.at[0], at::kInt, words_of(n, bits)));
            t.scales_out = static_cast<float*>(address(out.at[1], at::kFloat, ranges_of(n, bucket, kind)));
            t.scales_in = nullptr;
        }
        return as_bytes(items.data(), sizeof(mqg_quantize_item) * items.size());
    });
}

// update_items(layers, W, bits, bucket, kind) -> bytes: mqg_update_item[count + 1], then the pointer tables that the
// items name (by their addresses inside the bytes object, which does not move)
PyObject* update_items(PyObject*, PyObject* const* a, Py_ssize_t argc) {
    static PyObject *k_params, *k_raw, *k_packed, *k_scales;
    if (k_scales == nullptr) {   // under the interpreter's lock; interned names live as long as the interpreter
        k_params = PyUnicode_InternFromString("params");
        k_raw = PyUnicode_InternFromString("raw");
        k_packed = PyUnicode_InternFromString("packed");
        k_scales = PyUnicode_InternFromString("scales");
    }
    return guarded([&]() -> PyObject* {
        if (argc != 5) throw Reject{};
        const Items layers(a[0]);
        const uint64_t W = whole(a[1]), bits = whole(a[2]), bucket = whole(a[3]), kind = whole(a[4]);
        check_format(bits, bucket, kind);
        if (W < 1u || W > MQG_MAX_WORKERS) throw Reject{};
        const auto entry = [](PyObject* d, PyObject* k) {
            PyObject* v = PyDict_GetItemWithError(d, k);   // borrowed
            if (v == nullptr) throw Reject{};
            return v;
        };
        const size_t count = (size_t)layers.count;
        std::vector<mqg_update_item> items(count + 1);
        std::vector<void*> tables(count * 2u * W);
        for (size_t i = 0; i < count; ++i) {
            PyObject* layer = layers.at[i];
            if (!PyDict_CheckExact(layer)) throw Reject{};
            const at::Tensor& params = plain(entry(layer, k_params), at::kFloat);
            const uint64_t n = (uint64_t)params.numel();
            mqg_update_item& t = items[i];
            t = {};
            t.n = n;
            t.params = static_cast<float*>(params.data_ptr());
            void** first = tables.data() + i * 2u * W;
            PyObject* raw = PyDict_GetItemWithError(layer, k_raw);
            if (raw != nullptr) {
                const Items g(raw, (Py_ssize_t)W);
                for (uint64_t w = 0; w < W; ++w) first[w] = address(g.at[w], at::kFloat, n, true);
                t.raw = reinterpret_cast<decltype(t.raw)>(first);   // the marker of a raw layer; placed below
            } else {
                const Items p(entry(layer, k_packed), (Py_ssize_t)W), r(entry(layer, k_scales), (Py_ssize_t)W);
                const uint64_t words = words_of(n, bits), floats = ranges_of(n, bucket, kind);
                for (uint64_t w = 0; w < W; ++w) {
                    first[w] = address(p.at[w], at::kInt, words);
                    first[W + w] = address(r.at[w], at::kFloat, floats);
                }
            }
        }
        const size_t head = sizeof(mqg_update_item) * items.size(), tail = sizeof(void*) * tables.size();
        PyObject* out = PyBytes_FromStringAndSize(nullptr, (Py_ssize_t)(head + tail));
        if (out == nullptr) return nullptr;
        char* base = PyBytes_AS_STRING(out);
        for (size_t i = 0; i < count; ++i) {
            char* first = base + head + sizeof(void*) * (i * 2u * W);
            mqg_update_item& t = items[i];
            if (t.raw != nullptr) {
                t.raw = reinterpret_cast<decltype(t.raw)>(first);
            } else {
                t.packed = reinterpret_cast<decltype(t.packed)>(first);
                t.scales = reinterpret_cast<decltype(t.scales)>(first + sizeof(void*) * W);
            }
        }
        memcpy(base, items.data(), head);
        if (tail != 0) memcpy(base + head, tables.data(), tail);
        return out;
    });
}

PyMethodDef methods[] = {
    {"pointers", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(pointers)), METH_FASTCALL, nullptr},
    {"stream", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(stream)), METH_FASTCALL, nullptr},
    {"quantize_items", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(quantize_items)), METH_FASTCALL, nullptr},
    {"update_items", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(update_items)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
