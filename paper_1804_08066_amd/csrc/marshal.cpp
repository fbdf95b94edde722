// The binding's argument tables in native code: the checks of a list of tensors and the pointer and item tables
// that the C ABI takes.  A model's batched step names about a hundred tensors, and four attribute reads, two
// size calls and an address for each took 90 of the 98 us of the small CNN's iteration (4 workers, two launches).
//
// The calls of a training iteration go on from there: the library's entry is called from here, with the interpreter's lock
// released, and its status is returned.  Through the foreign-function layer a call of a dozen arguments cost 1.3 us of 4.5
// (65,536 elements quantized and the server's update: 10.8 -> 8.5 us for both; 7.6 to 8.6 from machine to machine).
//
// Every function returns None for anything but plain tensors of the right kind and size (subclasses, wrapped or
// storage-less tensors, other containers, values out of range); the binding then runs its own checks, which
// accept it or raise.  Nothing is kept between calls but the entries' addresses.
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

// numbers as the foreign-function layer passes them: whole ones modulo the type's range, a float rounded once
uint64_t masked(PyObject* o) {
    if (!PyLong_CheckExact(o)) throw Reject{};
    const unsigned long long v = PyLong_AsUnsignedLongLongMask(o);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) {
        PyErr_Clear();
        throw Reject{};
    }
    return v;
}
float real(PyObject* o) {
    if (!PyFloat_CheckExact(o)) throw Reject{};
    return (float)PyFloat_AS_DOUBLE(o);
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

// the W workers' streams
struct Streams {
    Py_ssize_t W;
    void *packed[MQG_MAX_WORKERS + 1] = {}, *ranges[MQG_MAX_WORKERS + 1] = {};
    Streams(PyObject* p, PyObject* r, uint64_t n, uint64_t bits, uint64_t bucket, uint64_t kind) {
        const Items ps(p), rs(r, ps.count);
        W = ps.count;
        if (W > MQG_MAX_WORKERS) throw Reject{};
        const uint64_t words = words_of(n, bits), floats = ranges_of(n, bucket, kind);
        for (Py_ssize_t w = 0; w < W; ++w) {
            packed[w] = address(ps.at[w], at::kInt, words);
            ranges[w] = address(rs.at[w], at::kFloat, floats);
        }
    }
    const uint32_t* const* words() const { return reinterpret_cast<const uint32_t* const*>(packed); }
    const float* const* floats() const { return reinterpret_cast<const float* const*>(ranges); }
};

// pointers(packed, ranges, n, bits, bucket, kind) -> (W, bytes, bytes): the W workers' streams
PyObject* pointers(PyObject*, PyObject* const* a, Py_ssize_t argc) {
    return guarded([&]() -> PyObject* {
        if (argc != 6) throw Reject{};
        const uint64_t n = whole(a[2]), bits = whole(a[3]), bucket = whole(a[4]), kind = whole(a[5]);
        check_format(bits, bucket, kind);
        const Streams s(a[0], a[1], n, bits, bucket, kind);
        const size_t bytes = sizeof(void*) * (size_t)(s.W > 0 ? s.W : 1);
        return Py_BuildValue("nNN", s.W, as_bytes(s.packed, bytes), as_bytes(s.ranges, bytes));
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

std::vector<mqg_quantize_item> encoder_items(PyObject* const* a, uint64_t bits, uint64_t bucket, uint64_t kind) {
    const Items grads(a[0]), outputs(a[1], grads.count);
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
    return items;
}
// quantize_items(grads, outputs, bases or None, bits, bucket, kind) -> bytes: mqg_quantize_item[count]
PyObject* quantize_items(PyObject*, PyObject* const* a, Py_ssize_t argc) {
    return guarded([&]() -> PyObject* {
        if (argc != 6) throw Reject{};
        const std::vector<mqg_quantize_item> items = encoder_items(a, whole(a[3]), whole(a[4]), whole(a[5]));
        return as_bytes(items.data(), sizeof(mqg_quantize_item) * items.size());
    });
}

// the layers of a server step: their items, then the pointer tables that the items name.  An item's table is given by
// its index; place() turns the indices into addresses.
struct LayerItems {
    std::vector<mqg_update_item> items;
    std::vector<void*> tables;
    size_t W;
    LayerItems(PyObject* list, uint64_t workers, uint64_t bits, uint64_t bucket, uint64_t kind) : W((size_t)workers) {
        static PyObject *k_params, *k_raw, *k_packed, *k_scales;
        if (k_scales == nullptr) {   // under the interpreter's lock; interned names live as long as the interpreter
            k_params = PyUnicode_InternFromString("params");
            k_raw = PyUnicode_InternFromString("raw");
            k_packed = PyUnicode_InternFromString("packed");
            k_scales = PyUnicode_InternFromString("scales");
        }
        const Items layers(list);
        check_format(bits, bucket, kind);
        if (W < 1u || W > MQG_MAX_WORKERS) throw Reject{};
        const auto entry = [](PyObject* d, PyObject* k) {
            PyObject* v = PyDict_GetItemWithError(d, k);   // borrowed
            if (v == nullptr) throw Reject{};
            return v;
        };
        const size_t count = (size_t)layers.count;
        items.resize(count + 1);
        tables.resize(count * 2u * W);
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
                for (size_t w = 0; w < W; ++w) first[w] = address(g.at[w], at::kFloat, n, true);
                t.raw = reinterpret_cast<decltype(t.raw)>(first);   // the marker of a raw layer; placed below
            } else {
                const Items p(entry(layer, k_packed), (Py_ssize_t)W), r(entry(layer, k_scales), (Py_ssize_t)W);
                const uint64_t words = words_of(n, bits), floats = ranges_of(n, bucket, kind);
                for (size_t w = 0; w < W; ++w) {
                    first[w] = address(p.at[w], at::kInt, words);
                    first[W + w] = address(r.at[w], at::kFloat, floats);
                }
            }
        }
    }
    void place(char* first_table) {
        for (size_t i = 0; i + 1 < items.size(); ++i) {
            char* first = first_table + sizeof(void*) * (i * 2u * W);
            mqg_update_item& t = items[i];
            if (t.raw != nullptr) {
                t.raw = reinterpret_cast<decltype(t.raw)>(first);
            } else {
                t.packed = reinterpret_cast<decltype(t.packed)>(first);
                t.scales = reinterpret_cast<decltype(t.scales)>(first + sizeof(void*) * W);
            }
        }
    }
};
// update_items(layers, W, bits, bucket, kind) -> bytes: mqg_update_item[count + 1], then the pointer tables that the
// items name (by their addresses inside the bytes object, which does not move)
PyObject* update_items(PyObject*, PyObject* const* a, Py_ssize_t argc) {
    return guarded([&]() -> PyObject* {
        if (argc != 5) throw Reject{};
        LayerItems l(a[0], whole(a[1]), whole(a[2]), whole(a[3]), whole(a[4]));
        const size_t head = sizeof(mqg_update_item) * l.items.size(), tail = sizeof(void*) * l.tables.size();
        PyObject* out = PyBytes_FromStringAndSize(nullptr, (Py_ssize_t)(head + tail));
        if (out == nullptr) return nullptr;
        char* base = PyBytes_AS_STRING(out);
        l.place(base + head);
        memcpy(base, l.items.data(), head);
        if (tail != 0) memcpy(base + head, l.tables.data(), tail);
        return out;
    });
}

// ---- calls ------------------------------------------------------------------------------------------
// The library is loaded by the binding, which hands its entries over: bind(current_raw_stream, current_device, address, ...),
// the addresses in this order.
struct Entries {
    decltype(&mqg_quantize_mode) quantize_mode;
    decltype(&mqg_quantize_minmax) quantize_minmax;
    decltype(&mqg_quantize_minmax_tensor) quantize_minmax_tensor;
    decltype(&mqg_aggregate_update_from) aggregate_update_from;
    decltype(&mqg_aggregate_update_minmax) aggregate_update_minmax;
    decltype(&mqg_aggregate_update_minmax_tensor) aggregate_update_minmax_tensor;
    decltype(&mqg_aggregate_requantize_mode) aggregate_requantize_mode;
    decltype(&mqg_aggregate_requantize_minmax) aggregate_requantize_minmax;
    decltype(&mqg_aggregate_requantize_minmax_tensor) aggregate_requantize_minmax_tensor;
    decltype(&mqg_dequantize_update) dequantize_update;
    decltype(&mqg_quantize_tensors_mode) quantize_tensors_mode;
    decltype(&mqg_quantize_minmax_tensors) quantize_minmax_tensors;
    decltype(&mqg_aggregate_update_tensors) aggregate_update_tensors;
    decltype(&mqg_aggregate_update_minmax_tensors) aggregate_update_minmax_tensors;
};
constexpr Py_ssize_t kEntries = sizeof(Entries) / sizeof(void*);
Entries lib;

PyObject *current_raw_stream, *current_device;   // torch's functions; None: not to be had

PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t argc) {
    if (argc != 2 + kEntries) {
        PyErr_SetString(PyExc_TypeError, "bind: two functions and one address per entry");
        return nullptr;
    }
    void* at[kEntries];
    for (Py_ssize_t i = 0; i < kEntries; ++i) {
        at[i] = PyLong_AsVoidPtr(a[2 + i]);
        if (at[i] == nullptr) {
            if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind: no address");
            return nullptr;
        }
    }
    memcpy(&lib, at, sizeof lib);
    Py_INCREF(a[0]);
    Py_INCREF(a[1]);
    Py_XSETREF(current_raw_stream, a[0]);
    Py_XSETREF(current_device, a[1]);
    Py_RETURN_NONE;
}
// a call's stream argument: a torch stream, or None for the current one.  After the tensors' checks: they say that there is
// a GPU to ask.
void* stream_of(PyObject* o) {
    static PyObject* k_stream;
    if (k_stream == nullptr) k_stream = PyUnicode_InternFromString("cuda_stream");
    PyObject* h = nullptr;
    if (o != Py_None) {
        h = PyObject_GetAttr(o, k_stream);
    } else if (current_raw_stream != nullptr && current_raw_stream != Py_None) {
        PyObject* device = PyObject_CallNoArgs(current_device);
        if (device != nullptr) h = PyObject_CallOneArg(current_raw_stream, device);
        Py_XDECREF(device);
    }
    if (h == nullptr) throw Reject{};
    void* p = PyLong_Check(h) ? PyLong_AsVoidPtr(h) : nullptr;
    const bool bad = !PyLong_Check(h) || PyErr_Occurred() != nullptr;
    Py_DECREF(h);
    if (bad) throw Reject{};
    return p;
}
// f() without the interpreter's lock, as the foreign-function layer calls; f touches no Python object
template <class F>
PyObject* status_of(F f) {
    if (lib.quantize_mode == nullptr) throw Reject{};
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = (int)f();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
}

// quantize(grad, packed, scales, bits, bucket, mode, seed, iteration, worker, elem_base, stream) -> status
PyObject* quantize(PyObject*, PyObject* const* a, Py_ssize_t argc) {
    return guarded([&]() -> PyObject* {
        if (argc != 11) throw Reject{};
        const uint64_t bits = whole(a[3]), bucket = whole(a[4]), mode = whole(a[5]), seed = masked(a[6]), base = masked(a[9]);
        const uint32_t iteration = (uint32_t)masked(a[7]), worker = (uint32_t)masked(a[8]);
        check_format(bits, bucket, 0u);
        if (mode > 1u) throw Reject{};
        const at::Tensor& g = plain(a[0], at::kFloat);
        const uint64_t n = (uint64_t)g.numel();
        uint32_t* p = static_cast<uint32_t*>(address(a[1], at::kInt, words_of(n, bits)));
        float* r = static_cast<float*>(address(a[2], at::kFloat, ranges_of(n, bucket, 0u)));
        const float* grad = static_cast<const float*>(g.data_ptr());
        void* stream = stream_of(a[10]);
        return status_of([=] {
            return lib.quantize_mode(grad, n, (uint32_t)bits, (uint32_t)bucket, (mqg_scale_mode)mode, seed, iteration, worker, base, p, r, stream);
        });
    });
}
// quantize_minmax(grad, packed, ranges, bits, bucket, stream) -> status; bucket 0: one range
PyObject* quantize_minmax(PyObject*, PyObject* const* a, Py_ssize_t argc) {
    return guarded([&]() -> PyObject* {
        if (argc != 6) throw Reject{};
        const uint64_t bits = whole(a[3]), bucket = whole(a[4]), kind = bucket == 0u ? 2u : 1u;
        check_format(bits, bucket, kind);
        const at::Tensor& g = plain(a[0], at::kFloat);
        const uint64_t n = (uint64_t)g.numel();
        uint32_t* p = static_cast<uint32_t*>(address(a[1], at::kInt, words_of(n, bits)));
        float* r = static_cast<float*>(address(a[2], at::kFloat, ranges_of(n, bucket, kind)));
        const float* grad = static_cast<const float*>(g.data_ptr());
        void* stream = stream_of(a[5]);
        return status_of([=] {
            return kind == 2u ? lib.quantize_minmax_tensor(grad, n, (uint32_t)bits, p, r, stream)
                              : lib.quantize_minmax(grad, n, (uint32_t)bits, (uint32_t)bucket, p, r, stream);
        });
    });
}
// update(packed, ranges, n, bits, bucket, kind, lr, params, origin, stream) -> status
PyObject* update(PyObject*, PyObject* const* a, Py_ssize_t argc) {
    return guarded([&]() -> PyObject* {
        if (argc != 10) throw Reject{};
        const uint64_t n = whole(a[2]), bits = whole(a[3]), bucket = whole(a[4]), kind = whole(a[5]), origin = whole(a[8]);
        check_format(bits, bucket, kind);
        if (origin > 1u) throw Reject{};
        const Streams s(a[0], a[1], n, bits, bucket, kind);
        const float lr = real(a[6]);
        float* params = static_cast<float*>(address(a[7], at::kFloat, n, true));
        void* stream = stream_of(a[9]);
        return status_of([&] {
            const uint32_t W = (uint32_t)s.W, b = (uint32_t)bits, bu = (uint32_t)bucket;
            if (kind == 0u) return lib.aggregate_update_from(s.words(), s.floats(), W, n, b, bu, lr, params, (mqg_codes_origin)origin, stream);
            if (kind == 1u) return lib.aggregate_update_minmax(s.words(), s.floats(), W, n, b, bu, lr, params, stream);
            return lib.aggregate_update_minmax_tensor(s.words(), s.floats(), W, n, b, lr, params, stream);
        });
    });
}
// requantize(packed, ranges, n, bits, bucket, kind, mode, seed, iteration, worker, elem_base, packed_out, ranges_out, stream) -> status
PyObject* requantize(PyObject*, PyObject* const* a, Py_ssize_t argc) {
    return guarded([&]() -> PyObject* {
        if (argc != 14) throw Reject{};
        const uint64_t n = whole(a[2]), bits = whole(a[3]), bucket = whole(a[4]), kind = whole(a[5]), mode = whole(a[6]), seed = masked(a[7]), base = masked(a[10]);
        const uint32_t iteration = (uint32_t)masked(a[8]), worker = (uint32_t)masked(a[9]);
        check_format(bits, bucket, kind);
        if (mode > 1u) throw Reject{};
        const Streams s(a[0], a[1], n, bits, bucket, kind);
        if (s.W == 0) throw Reject{};
        uint32_t* p = static_cast<uint32_t*>(address(a[11], at::kInt, words_of(n, bits)));
        float* r = static_cast<float*>(address(a[12], at::kFloat, ranges_of(n, bucket, kind)));
        void* stream = stream_of(a[13]);
        return status_of([&] {
            const uint32_t W = (uint32_t)s.W, b = (uint32_t)bits, bu = (uint32_t)bucket;
            if (kind == 0u) return lib.aggregate_requantize_mode(s.words(), s.floats(), W, n, b, bu, (mqg_scale_mode)mode, seed, iteration, worker, base, p, r, stream);
            if (kind == 1u) return lib.aggregate_requantize_minmax(s.words(), s.floats(), W, n, b, bu, p, r, stream);
            return lib.aggregate_requantize_minmax_tensor(s.words(), s.floats(), W, n, b, p, r, stream);
        });
    });
}
// dequantize_update(packed, scales, n, bits, bucket, lr, params, stream) -> status
PyObject* dequantize_update(PyObject*, PyObject* const* a, Py_ssize_t argc) {
    return guarded([&]() -> PyObject* {
        if (argc != 8) throw Reject{};
        const uint64_t n = whole(a[2]), bits = whole(a[3]), bucket = whole(a[4]);
        check_format(bits, bucket, 0u);
        const uint32_t* p = static_cast<const uint32_t*>(address(a[0], at::kInt, words_of(n, bits)));
        const float* s = static_cast<const float*>(address(a[1], at::kFloat, ranges_of(n, bucket, 0u)));
        const float lr = real(a[5]);
        float* params = static_cast<float*>(address(a[6], at::kFloat, n, true));
        void* stream = stream_of(a[7]);
        return status_of([=] { return lib.dequantize_update(p, s, n, (uint32_t)bits, (uint32_t)bucket, lr, params, stream); });
    });
}
// quantize_tensors(grads, outputs, bases or None, bits, bucket, kind, mode, seed, iteration, worker, stream) -> status
PyObject* quantize_tensors(PyObject*, PyObject* const* a, Py_ssize_t argc) {
    return guarded([&]() -> PyObject* {
        if (argc != 11) throw Reject{};
        const uint64_t bits = whole(a[3]), bucket = whole(a[4]), kind = whole(a[5]), mode = whole(a[6]), seed = masked(a[7]);
        const uint32_t iteration = (uint32_t)masked(a[8]), worker = (uint32_t)masked(a[9]);
        if (mode > 1u) throw Reject{};
        const std::vector<mqg_quantize_item> items = encoder_items(a, bits, bucket, kind);
        void* stream = stream_of(a[10]);
        return status_of([&] {
            const uint32_t count = (uint32_t)items.size() - 1u;
            if (kind == 0u) return lib.quantize_tensors_mode(items.data(), count, (uint32_t)bits, (uint32_t)bucket, (mqg_scale_mode)mode, seed, iteration, worker, stream);
            return lib.quantize_minmax_tensors(items.data(), count, (uint32_t)bits, (uint32_t)bucket, stream);
        });
    });
}
// update_tensors(layers, W, bits, bucket, kind, lr, stream) -> status
PyObject* update_tensors(PyObject*, PyObject* const* a, Py_ssize_t argc) {
    return guarded([&]() -> PyObject* {
        if (argc != 7) throw Reject{};
        const uint64_t W = whole(a[1]), bits = whole(a[2]), bucket = whole(a[3]), kind = whole(a[4]);
        const float lr = real(a[5]);
        LayerItems l(a[0], W, bits, bucket, kind);
        l.place(reinterpret_cast<char*>(l.tables.data()));
        void* stream = stream_of(a[6]);
        return status_of([&] {
            const uint32_t count = (uint32_t)l.items.size() - 1u;
            if (kind == 0u) return lib.aggregate_update_tensors(l.items.data(), count, (uint32_t)W, (uint32_t)bits, (uint32_t)bucket, lr, stream);
            return lib.aggregate_update_minmax_tensors(l.items.data(), count, (uint32_t)W, (uint32_t)bits, (uint32_t)bucket, lr, stream);
        });
    });
}

template <class F>
PyCFunction fast(F f) { return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)); }
PyMethodDef methods[] = {
    {"pointers", fast(pointers), METH_FASTCALL, nullptr},
    {"stream", fast(stream), METH_FASTCALL, nullptr},
    {"quantize_items", fast(quantize_items), METH_FASTCALL, nullptr},
    {"update_items", fast(update_items), METH_FASTCALL, nullptr},
    {"bind", fast(bind), METH_FASTCALL, nullptr},
    {"quantize", fast(quantize), METH_FASTCALL, nullptr},
    {"quantize_minmax", fast(quantize_minmax), METH_FASTCALL, nullptr},
    {"update", fast(update), METH_FASTCALL, nullptr},
    {"requantize", fast(requantize), METH_FASTCALL, nullptr},
    {"dequantize_update", fast(dequantize_update), METH_FASTCALL, nullptr},
    {"quantize_tensors", fast(quantize_tensors), METH_FASTCALL, nullptr},
    {"update_tensors", fast(update_tensors), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
