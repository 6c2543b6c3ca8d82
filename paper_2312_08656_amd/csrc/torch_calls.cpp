// Marshalling of torch tensors for the calls of a pass: what binding.py does with ctypes, and the two halves of one aggregation with
// their buffers.  Host code only; the calls themselves are libmaxk's, whose addresses come from binding.py.
//
// Bound by the host on small graphs: a call took 4.8 to 5.1 us from Python, 1.2 of them checks and 0.8 ctypes, an empty tensor 1.5, and
// the backward half of a pass runs in a thread of its own, where the same Python is slower still.
//
// Every function returns false (None) on anything but plain device tensors of the shapes and types that the call takes; binding.py then makes
// the call itself, which raises what is to be raised.  A call that was made and failed is not made again: its status goes to binding.py's check.
#include <c10/hip/HIPStream.h>
#include <torch/extension.h>

#include <utility>

#include "../../include/maxk.h"

namespace {

decltype(&maxk_topk_cbsr_narrow) topk_call;
decltype(&maxk_spgemm_fwd_narrow) forward_call;
decltype(&maxk_spgemm_fwd_noalloc) forward_noalloc_call;
decltype(&maxk_sspmm_bwd_narrow) backward_call;
decltype(&maxk_cbsr_scatter) scatter_call;

PyObject* check;  // (status, name of the call): raises; held for good

void bind(const std::vector<uintptr_t>& at, const py::function& raise)
{
    TORCH_CHECK(at.size() == 5, "five addresses");
    topk_call = reinterpret_cast<decltype(topk_call)>(at[0]);
    forward_call = reinterpret_cast<decltype(forward_call)>(at[1]);
    forward_noalloc_call = reinterpret_cast<decltype(forward_noalloc_call)>(at[2]);
    backward_call = reinterpret_cast<decltype(backward_call)>(at[3]);
    scatter_call = reinterpret_cast<decltype(scatter_call)>(at[4]);
    Py_XDECREF(std::exchange(check, py::function(raise).release().ptr()));
}

// The tensor in `x`, where it is a plain one in device memory: no subclass with a dispatch of its own, no functorch wrapper
const at::Tensor* plain(const py::handle& x)
{
    if (!THPVariable_Check(x.ptr())) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(x.ptr());
    if (!t.defined() || !t.is_cuda() || !t.has_storage() || t.layout() != at::kStrided) return nullptr;
    const auto keys = t.key_set();
    if (keys.has_any(c10::DispatchKeySet({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::FuncTorchBatched,
                                          c10::DispatchKey::Functionalize})))
        return nullptr;
    return &t;
}

const at::Tensor* matrix(const py::handle& x, int64_t rows, int64_t cols)  // contiguous; -1: any
{
    const at::Tensor* t = plain(x);
    if (!t || t->dim() != 2 || !t->is_contiguous()) return nullptr;
    return (rows < 0 || t->size(0) == rows) && (cols < 0 || t->size(1) == cols) ? t : nullptr;
}

int index_bytes(const at::Tensor& t)
{
    switch (t.scalar_type()) {
        case at::kByte: return 1;
        case at::kUInt16:
        case at::kShort: return 2;
        case at::kInt: return 4;
        default: return 0;
    }
}

int value_type(const at::Tensor& t)
{
    return t.scalar_type() == at::kFloat ? MAXK_VALUE_F32 : t.scalar_type() == at::kBFloat16 ? MAXK_VALUE_BF16 : t.scalar_type() == at::kHalf ? MAXK_VALUE_F16 : -1;
}

bool takes(const at::Tensor& t, bool narrow) { return narrow ? value_type(t) >= 0 : t.scalar_type() == at::kFloat; }

void* stream() { return c10::hip::getCurrentHIPStream().stream(); }

maxk_graph* graph(uintptr_t g) { return reinterpret_cast<maxk_graph*>(g); }

template <typename F>
bool made(const char* what, F&& call)  // call() may change `what` to the call that failed
{
    maxk_status st;
    {
        py::gil_scoped_release released;  // a first call may build tables
        st = call(what);
    }
    if (st != MAXK_OK) py::reinterpret_borrow<py::function>(check)(st, what);
    return true;
}

bool topk(const py::handle& H_, int64_t k, const py::handle& data_, const py::handle& index_, bool narrow)
{
    const at::Tensor* H = matrix(H_, -1, -1);
    if (!H || H->scalar_type() != at::kFloat) return false;
    const int64_t N = H->size(0), dim = H->size(1);
    const at::Tensor *data = matrix(data_, N, k), *index = matrix(index_, N, k);
    if (!data || !index || !takes(*data, narrow) || !index_bytes(*index)) return false;
    return made(narrow ? "maxk_topk_cbsr_narrow" : "maxk_topk_cbsr", [&, s = stream()](const char*) {
        return topk_call(static_cast<const float*>(H->data_ptr()), N, (int32_t)dim, (int32_t)k, data->data_ptr(), value_type(*data), index->data_ptr(),
                         index_bytes(*index), s);
    });
}

bool forward(uintptr_t g, int64_t N, const py::handle& data_, const py::handle& index_, int64_t dim, const py::handle& Y_, bool narrow)
{
    const at::Tensor *data = matrix(data_, N, -1), *Y = matrix(Y_, N, dim);
    if (!g || !data || !Y || !takes(*data, narrow) || Y->scalar_type() != at::kFloat) return false;
    const int64_t k = data->size(1);
    const at::Tensor* index = matrix(index_, N, k);
    if (!index || !index_bytes(*index)) return false;
    return made(narrow ? "maxk_spgemm_fwd_narrow" : "maxk_spgemm_fwd", [&, s = stream()](const char*) {
        return forward_call(graph(g), data->data_ptr(), value_type(*data), index->data_ptr(), index_bytes(*index), (int32_t)dim, (int32_t)k,
                            static_cast<float*>(Y->data_ptr()), s);
    });
}

bool forward_noalloc(uintptr_t g, int64_t N, const py::handle& data_, const py::handle& index_, int64_t dim, const py::handle& Y_)
{
    const at::Tensor *data = matrix(data_, N, -1), *Y = matrix(Y_, N, dim);
    if (!g || !data || !Y || data->scalar_type() != at::kFloat || Y->scalar_type() != at::kFloat) return false;
    const int64_t k = data->size(1);
    const at::Tensor* index = matrix(index_, N, k);
    if (!index || !index_bytes(*index)) return false;
    return made("maxk_spgemm_fwd_noalloc", [&, s = stream()](const char*) {
        return forward_noalloc_call(graph(g), static_cast<const float*>(data->data_ptr()), index->data_ptr(), index_bytes(*index), (int32_t)dim,
                                    (int32_t)k, static_cast<float*>(Y->data_ptr()), s);
    });
}

bool backward(uintptr_t g, int64_t N, const py::handle& dY_, const py::handle& index_, const py::handle& dXs_, bool narrow)
{
    const at::Tensor *dY = matrix(dY_, N, -1), *index = matrix(index_, N, -1);
    if (!g || !dY || !index || !takes(*dY, narrow) || !index_bytes(*index)) return false;
    const int64_t k = index->size(1);
    const at::Tensor* dXs = matrix(dXs_, N, k);
    if (!dXs || dXs->scalar_type() != at::kFloat) return false;
    return made(narrow ? "maxk_sspmm_bwd_narrow" : "maxk_sspmm_bwd", [&, s = stream()](const char*) {
        return backward_call(graph(g), dY->data_ptr(), value_type(*dY), index->data_ptr(), index_bytes(*index), (int32_t)dY->size(1), (int32_t)k,
                             static_cast<float*>(dXs->data_ptr()), s);
    });
}

bool scatter(const py::handle& values_, const py::handle& index_, const py::handle& dense_)
{
    const at::Tensor* values = matrix(values_, -1, -1);
    if (!values || values->scalar_type() != at::kFloat) return false;
    const int64_t N = values->size(0), k = values->size(1);
    const at::Tensor *index = matrix(index_, N, k), *dense = matrix(dense_, N, -1);
    if (!index || !dense || !index_bytes(*index) || dense->scalar_type() != at::kFloat) return false;
    return made("maxk_cbsr_scatter", [&, s = stream()](const char*) {
        return scatter_call(static_cast<const float*>(values->data_ptr()), index->data_ptr(), index_bytes(*index), N, (int32_t)dense->size(1), (int32_t)k,
                            static_cast<float*>(dense->data_ptr()), s);
    });
}

at::ScalarType index_type(int ib) { return ib == 1 ? at::kByte : ib == 2 ? at::kUInt16 : at::kInt; }

// (Y, sp_index) of one aggregation: top-k, then the forward pass
py::object aggregate_forward(uintptr_t g, int64_t N, const py::handle& H_, int64_t k, int ib)
{
    const at::Tensor* H = matrix(H_, N, -1);
    if (!g || !H || H->scalar_type() != at::kFloat || k < 1 || (ib != 1 && ib != 2 && ib != 4)) return py::none();
    const int64_t dim = H->size(1);
    if (k > dim) return py::none();
    at::Tensor data, index, Y;
    try {
        data = at::empty({N, k}, H->options());
        index = at::empty({N, k}, H->options().dtype(index_type(ib)));
        Y = at::empty({N, dim}, H->options());
    } catch (const c10::Error&) {  // no memory: said by the calls from Python
        return py::none();
    }
    made("maxk_topk_cbsr", [&, s = stream()](const char*& what) {
        const maxk_status st = topk_call(static_cast<const float*>(H->data_ptr()), N, (int32_t)dim, (int32_t)k, data.data_ptr(), MAXK_VALUE_F32,
                                         index.data_ptr(), ib, s);
        if (st != MAXK_OK) return st;
        what = "maxk_spgemm_fwd";
        return forward_call(graph(g), data.data_ptr(), MAXK_VALUE_F32, index.data_ptr(), ib, (int32_t)dim, (int32_t)k, static_cast<float*>(Y.data_ptr()), s);
    });
    return py::make_tuple(Y, index);
}

// dH of one aggregation: the backward pass at the columns kept, then back to dense rows
py::object aggregate_backward(uintptr_t g, int64_t N, const py::handle& dY_, const py::handle& index_, int64_t dim, int64_t k)
{
    const at::Tensor *dY = matrix(dY_, N, dim), *index = matrix(index_, N, k);
    if (!g || !dY || !index || dY->scalar_type() != at::kFloat || !index_bytes(*index)) return py::none();
    const int ib = index_bytes(*index);
    at::Tensor dXs, dH;
    try {
        dXs = at::empty({N, k}, dY->options());
        dH = at::empty({N, dim}, dY->options());
    } catch (const c10::Error&) {
        return py::none();
    }
    made("maxk_sspmm_bwd", [&, s = stream()](const char*& what) {
        const maxk_status st = backward_call(graph(g), dY->data_ptr(), MAXK_VALUE_F32, index->data_ptr(), ib, (int32_t)dim, (int32_t)k,
                                             static_cast<float*>(dXs.data_ptr()), s);
        if (st != MAXK_OK) return st;
        what = "maxk_cbsr_scatter";
        return scatter_call(static_cast<const float*>(dXs.data_ptr()), index->data_ptr(), ib, N, (int32_t)dim, (int32_t)k, static_cast<float*>(dH.data_ptr()), s);
    });
    return py::cast(dH);
}

}  // namespace

PYBIND11_MODULE(_torch_calls, m)
{
    m.def("bind", &bind);
    m.def("topk", &topk);
    m.def("forward", &forward);
    m.def("forward_noalloc", &forward_noalloc);
    m.def("backward", &backward);
    m.def("scatter", &scatter);
    m.def("aggregate_forward", &aggregate_forward);
    m.def("aggregate_backward", &aggregate_backward);
}
