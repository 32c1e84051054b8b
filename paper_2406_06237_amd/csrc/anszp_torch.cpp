// The binding's short calls in native code: results allocated through torch and the library called without a trip through
// ctypes.  Such a call takes 3 to 20 us on the GPU, and its Python took longer: dequantising a few hundred thousand
// symbols 7.2 us, packing one layer 28 (4.6 and 11.3 here).  Host work only; every kernel is behind the C ABI (include/anszp.h).
//
// The functions take what the binding has checked (devices, ranges of small integers) and the raw stream, and return their
// tensors, the library's error code, or None: for arguments that are no plain integers of the usual ranges and for failed
// allocations, which the binding's own path then accepts or refuses.  Allocations and the library's calls may wait (for
// memory to come free, for room in a queue): the interpreter lock is held only while Python objects are read and made.
#include <ATen/ATen.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <torch/csrc/utils/pybind.h>

#include <algorithm>
#include <climits>
#include <vector>

#include "anszp.h"

namespace {

constexpr int kDeclined = INT_MIN;                          // (no code of the library's)
py::object none() { return py::none(); }
py::object failed(int rc) { return rc == kDeclined ? none() : py::object(py::int_(rc)); }
void* stream_of(uint64_t raw) { return reinterpret_cast<void*>(static_cast<uintptr_t>(raw)); }
template <class T>
T* data(const at::Tensor& t) { return static_cast<T*>(t.data_ptr()); }

py::object dequant_zp(const at::Tensor& symbols, uint32_t zero_point, float scale, int out_code, uint32_t channel_len,
                      const std::optional<at::Tensor>& channel_scales, uint64_t stream) {
    static constexpr at::ScalarType kTypes[] = {at::kByte, at::kFloat, at::kBFloat16};
    const int64_t n = symbols.numel();
    at::Tensor out;
    int rc = 0;
    {
        py::gil_scoped_release unlocked;
        try {
            out = at::empty({std::max<int64_t>(n, 8)}, symbols.options().dtype(kTypes[out_code]));
        } catch (...) {
            rc = kDeclined;
        }
        const anszp_layer_t lay = {scale, zero_point, 8u, channel_len, 0u, 0u};
        if (!rc)
            rc = anszp_dequant_zp(data<uint8_t>(symbols), uint64_t(n), &lay, channel_scales ? data<float>(*channel_scales) : nullptr,
                                  channel_scales ? uint64_t(channel_scales->numel()) : 0u, out.data_ptr(), out_code, stream_of(stream));
    }
    if (rc) return failed(rc);
    return py::cast(n >= 8 ? out : out.narrow(0, 0, n));
}

py::object build_tables_device(const at::Tensor& freqs, int n_tables, int table_log, int64_t words, const std::optional<at::Tensor>& status, uint64_t stream) {
    at::Tensor tables;
    int rc = 0;
    {
        py::gil_scoped_release unlocked;
        try {
            tables = at::empty({words}, freqs.options().dtype(at::kInt));
        } catch (...) {
            rc = kDeclined;
        }
        if (!rc)
            rc = anszp_build_tables_device(data<uint32_t>(freqs), n_tables, table_log, data<uint32_t>(tables), status ? data<uint32_t>(*status) : nullptr,
                                           stream_of(stream));
    }
    return rc ? failed(rc) : py::cast(tables);
}

// A list or tuple of plain integers in [least, most], or one for all.
template <class T>
bool integers(py::handle from, size_t count, long long least, long long most, std::vector<T>& to) {
    auto one = [&](PyObject* o, T& v) {
        if (!PyLong_Check(o)) return false;
        int beyond = 0;
        const long long x = PyLong_AsLongLongAndOverflow(o, &beyond);
        if (beyond || x < least || x > most) return false;
        v = static_cast<T>(x);
        return true;
    };
    PyObject* const o = from.ptr();
    if (PyLong_Check(o)) {
        T v;
        if (!one(o, v)) return false;
        to.assign(count, v);
        return true;
    }
    const bool list = PyList_Check(o);
    if (!list && !PyTuple_Check(o)) return false;
    const size_t there = static_cast<size_t>(list ? PyList_GET_SIZE(o) : PyTuple_GET_SIZE(o));
    if (there < count) return false;
    to.resize(count);
    for (size_t i = 0; i < count; ++i)
        if (!one(list ? PyList_GET_ITEM(o, i) : PyTuple_GET_ITEM(o, i), to[i])) return false;
    return true;
}

// The payload is as long as the set can need; record: the inputs' memory is kept for this stream.
py::object pack_set(const at::Tensor& symbols, const at::Tensor& freqs, py::handle layer_symbols, py::handle chunk_sizes, uint32_t table_log, uint32_t n_streams,
                    uint32_t single, uint32_t layer_id, uint64_t out_offset, uint64_t payload_word_offset, uint32_t stream_offset, bool record,
                    uint64_t stream) {
    PyObject* const o = layer_symbols.ptr();
    if (!PyList_Check(o) && !PyTuple_Check(o)) return none();
    const size_t count = static_cast<size_t>(PyList_Check(o) ? PyList_GET_SIZE(o) : PyTuple_GET_SIZE(o));
    std::vector<uint64_t> sizes;
    std::vector<uint32_t> chunks_of;
    constexpr long long kMost = 1ll << 40;
    if (count == 0 || count > (1u << 20) || !integers(layer_symbols, count, 0, kMost, sizes) || !integers(chunk_sizes, count, 1, (1ll << 32) - 1, chunks_of)) return none();
    uint64_t n_chunks = 0, bound = 0;
    for (size_t l = 0; l < count; ++l) {
        uint64_t c = 0, words = 0;
        if (anszp_pack_bound(sizes[l], int(table_log), int(n_streams), chunks_of[l], &c, &words) != ANSZP_OK) return none();
        n_chunks += c;
        bound += words;
        if (n_chunks >= (1ull << 31)) return none();
    }
    const uint64_t chunk_count = std::max<uint64_t>(n_chunks, 1u), hdr_words = std::max<uint64_t>(n_chunks * n_streams, 4u), payload_words = std::max<uint64_t>(bound, 4u);
    const uint64_t scratch_bytes = anszp_pack_scratch_bytes(uint32_t(count), int(table_log));
    at::Tensor chunks, hdr, payload, used, status, scratch;
    int rc = 0;
    {
        py::gil_scoped_release unlocked;
        try {
            const at::TensorOptions bytes = symbols.options().dtype(at::kByte), ints = bytes.dtype(at::kInt);
            scratch = at::empty({int64_t(scratch_bytes)}, bytes);
            chunks = at::empty({int64_t(chunk_count * sizeof(anszp_chunk_t))}, bytes);
            hdr = at::empty({int64_t(hdr_words)}, ints);
            payload = at::empty({int64_t(payload_words)}, ints);
            used = at::empty({1}, bytes.dtype(at::kLong));
            status = at::empty({2}, ints);
            if (record) {                                   // (the tensors may come from another stream)
                const c10::Stream current = c10::impl::VirtualGuardImpl(symbols.device().type()).getStream(symbols.device());
                symbols.record_stream(current);
                freqs.record_stream(current);
            }
        } catch (...) {
            rc = kDeclined;
        }
        if (!rc) {
            anszp_pack_set_t a = {};
            a.symbols = data<uint8_t>(symbols); a.freqs = data<uint32_t>(freqs); a.layer_symbols = sizes.data(); a.chunk_sizes = chunks_of.data();
            a.n_layers = uint32_t(count); a.table_log = table_log; a.n_streams = n_streams;
            a.single = single; a.layer_id = layer_id; a.stream_offset = stream_offset; a.clear = 1u;
            a.out_offset = out_offset; a.payload_word_offset = payload_word_offset;
            a.chunks = data<anszp_chunk_t>(chunks); a.stream_hdr = data<uint32_t>(hdr); a.payload = data<uint32_t>(payload); a.payload_cap_words = bound;
            a.clear_chunks = chunk_count; a.clear_stream_hdr = hdr_words; a.clear_payload_words = payload_words;
            a.payload_words_used = data<uint64_t>(used); a.status = data<uint32_t>(status); a.scratch = scratch.data_ptr(); a.scratch_bytes = scratch_bytes;
            rc = anszp_pack_set_device(&a, stream_of(stream));
        }
    }
    if (rc) return failed(rc);
    return py::make_tuple(chunks, hdr, payload, used, status);
}

}  // namespace

PYBIND11_MODULE(_anszp_torch, m) {
    m.def("dequant_zp", &dequant_zp);
    m.def("build_tables_device", &build_tables_device);
    m.def("pack_set", &pack_set);
}
