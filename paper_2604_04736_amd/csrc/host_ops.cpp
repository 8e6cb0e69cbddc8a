// Host side of the calls that BayesianLinear and hot_stats_whole make: metadata checks, output and scratch allocation and
// the C call in one native function each, since a small layer's call is bound by the interpreter (a forecast of one row through
// three layers with 16 samples 69 -> 41 us, of which the GPU works 23; a training pass on 64 rows 456 -> 330).  Every function answers None where an argument is not what it takes without
// a copy or a conversion; the caller then goes through binding.py, whose checks name what is wrong.  No arithmetic here.
#include <torch/csrc/utils/pybind.h>

#include <ATen/ATen.h>

#include "hot.h"

namespace py = pybind11;
using at::Tensor;
typedef std::optional<Tensor> MaybeTensor;

namespace {

// A dense float32 tensor with memory of its own on the current device (no subclass, no transform's wrapper, no lazy negation).
bool plain(const Tensor &t, int64_t device)
{
    return t.is_cuda() && t.get_device() == device && t.scalar_type() == at::kFloat && t.layout() == at::kStrided && t.has_storage() &&
           !t.key_set().has(c10::DispatchKey::Python) && !t.is_neg() && t.is_contiguous();
}

bool is_vector(const MaybeTensor &t, int64_t n, int64_t device) { return t && plain(*t, device) && t->dim() == 1 && t->size(0) == n; }

const float *data(const Tensor &t) { return t.const_data_ptr<float>(); }
const float *data(const MaybeTensor &t) { return t ? t->const_data_ptr<float>() : nullptr; }

// the layer's description, if the arrays are as the C calls want them and have the layer's sizes (its draws and offsets are by these:
// with more outputs than that, the weights' eps would be those of its biases and of the next layer)
bool describe(const Tensor &x, const Tensor &mu_w, const Tensor &sigma_w, const MaybeTensor &mu_b, const MaybeTensor &sigma_b, int64_t in_features,
              int64_t out_features, int64_t s_local, int64_t weight_offset, int64_t bias_offset, int64_t device, hot_linear_desc &d)
{
    if (!plain(x, device) || !plain(mu_w, device) || !plain(sigma_w, device) || s_local < 1 || s_local > INT32_MAX) return false;
    if ((x.dim() != 2 && x.dim() != 3) || mu_w.dim() != 2 || mu_w.sizes() != sigma_w.sizes()) return false;
    const int64_t rows = x.size(-2), k = x.size(-1), o = mu_w.size(0);
    if (k != in_features || o != out_features || mu_w.size(1) != k || (x.dim() == 3 && x.size(0) != s_local)) return false;
    if (mu_b.has_value() != sigma_b.has_value() || (mu_b && !(is_vector(mu_b, o, device) && is_vector(sigma_b, o, device)))) return false;
    d.rows = rows;
    d.in_features = k;
    d.out_features = o;
    d.ldx = k;
    d.weight_offset = weight_offset;
    d.bias_offset = bias_offset;
    d.s_local = (int32_t)s_local;
    d.reserved = 0;
    d.x_sample_stride = x.dim() == 3 ? rows * k : 0;
    return true;
}

// Scratch memory: `bytes`, or the `least` where the device has no room for so much, which only buys time.
Tensor scratch(int64_t &bytes, int64_t least, const Tensor &like)
{
    const auto options = like.options().dtype(at::kByte);
    if (bytes > least) {
        try {
            return at::empty({bytes}, options);
        } catch (const c10::OutOfMemoryError &) {
            bytes = least;
        }
    }
    return bytes > 0 ? at::empty({bytes}, options) : Tensor();
}

// y, or the error code, or None
py::object linear_forward(const Tensor &x, const Tensor &mu_w, const Tensor &sigma_w, const MaybeTensor &mu_b, const MaybeTensor &sigma_b, uint64_t seed,
                          uint32_t step, uint32_t first_sample, int64_t in_features, int64_t out_features, int64_t s_local, int64_t weight_offset,
                          int64_t bias_offset, int64_t scratch_bytes, int64_t device, uintptr_t stream)
{
    hot_linear_desc d;
    if (!describe(x, mu_w, sigma_w, mu_b, sigma_b, in_features, out_features, s_local, weight_offset, bias_offset, device, d)) return py::none();
    Tensor y;
    int code;
    {
        py::gil_scoped_release others_run;
        y = at::empty({s_local, d.rows, d.out_features}, x.options());
        const Tensor ws = scratch(scratch_bytes, 0, x);
        const hot_rng rng = {seed, step, first_sample};
        code = hot_linear_forward_rng_ws(&d, &rng, data(x), data(mu_w), data(sigma_w), data(mu_b), data(sigma_b), y.mutable_data_ptr<float>(),
                                         scratch_bytes > 0 ? ws.mutable_data_ptr() : nullptr, scratch_bytes, reinterpret_cast<void *>(stream));
    }
    if (code != HOT_OK) return py::int_(code);
    return py::cast(y);
}

// (dx or None, grad mu_w, grad sigma_w, grad mu_b or None, grad sigma_b or None), or the error code, or None
py::object linear_backward(const Tensor &x, const Tensor &grad_y, const Tensor &mu_w, const Tensor &sigma_w, const MaybeTensor &mu_b, const MaybeTensor &sigma_b,
                           bool want_dx, uint64_t seed, uint32_t step, uint32_t first_sample, int64_t in_features, int64_t out_features, int64_t s_local,
                           double dataset_size, int64_t weight_offset, int64_t bias_offset, int64_t scratch_bytes, int64_t least_scratch, int64_t device,
                           uintptr_t stream)
{
    hot_linear_desc d;
    if (!describe(x, mu_w, sigma_w, mu_b, sigma_b, in_features, out_features, s_local, weight_offset, bias_offset, device, d)) return py::none();
    if (!plain(grad_y, device) || grad_y.dim() != 3 || grad_y.size(0) != s_local || grad_y.size(1) != d.rows || grad_y.size(2) != d.out_features)
        return py::none();
    Tensor dx, gmw, gsw, gmb, gsb;
    int code;
    {
        py::gil_scoped_release others_run;
        gmw = at::empty(mu_w.sizes(), x.options());
        gsw = at::empty(mu_w.sizes(), x.options());
        if (mu_b) {
            gmb = at::empty({d.out_features}, x.options());
            gsb = at::empty({d.out_features}, x.options());
        }
        if (want_dx) dx = at::empty({s_local, d.rows, d.in_features}, x.options());
        const Tensor ws = scratch(scratch_bytes, least_scratch, x);
        const hot_rng rng = {seed, step, first_sample};
        code = hot_linear_backward_rng_ws(&d, (int32_t)s_local, dataset_size, HOT_REDUCE_NONE, &rng, data(x), data(grad_y), data(mu_w), data(sigma_w),
                                          data(mu_b), data(sigma_b), gmw.mutable_data_ptr<float>(), gsw.mutable_data_ptr<float>(),
                                          mu_b ? gmb.mutable_data_ptr<float>() : nullptr, mu_b ? gsb.mutable_data_ptr<float>() : nullptr,
                                          want_dx ? dx.mutable_data_ptr<float>() : nullptr, scratch_bytes > 0 ? ws.mutable_data_ptr() : nullptr,
                                          scratch_bytes > 0 ? scratch_bytes : 0, reinterpret_cast<void *>(stream));
    }
    if (code != HOT_OK) return py::int_(code);
    auto maybe = [](const Tensor &t) -> py::object { return t.defined() ? py::cast(t) : py::none(); };
    return py::make_tuple(maybe(dx), gmw, gsw, maybe(gmb), maybe(gsb));
}

// the KL term (a float64 of no dimensions), or the error code, or None
py::object kl_layer(const Tensor &mu_w, const Tensor &sigma_w, const MaybeTensor &mu_b, const MaybeTensor &sigma_b, int64_t n_w, int64_t n_b,
                    int64_t device, uintptr_t stream)
{
    if (!plain(mu_w, device) || !plain(sigma_w, device) || mu_w.numel() != n_w || sigma_w.numel() != n_w) return py::none();
    if (n_b > 0 && !(is_vector(mu_b, n_b, device) && is_vector(sigma_b, n_b, device))) return py::none();
    Tensor out;
    int code;
    {
        py::gil_scoped_release others_run;
        out = at::empty({}, mu_w.options().dtype(at::kDouble));
        code = hot_kl_layer(n_w, data(mu_w), data(sigma_w), n_b, n_b > 0 ? data(mu_b) : nullptr, n_b > 0 ? data(sigma_b) : nullptr,
                            out.mutable_data_ptr<double>(), reinterpret_cast<void *>(stream));
    }
    if (code != HOT_OK) return py::int_(code);
    return py::cast(out);
}

// the error code, or None
py::object stats_whole(const Tensor &yhat, int32_t ddof, const Tensor &mean, const Tensor &std, int64_t device, uintptr_t stream)
{
    if (!plain(yhat, device) || yhat.dim() != 2 || yhat.size(0) < 1 || yhat.size(0) > INT32_MAX) return py::none();
    const int64_t m = yhat.size(1);
    if (!is_vector(mean, m, device) || !is_vector(std, m, device)) return py::none();
    int code;
    {
        py::gil_scoped_release others_run;
        code = hot_stats_whole(data(yhat), m, m, (int32_t)yhat.size(0), ddof, mean.mutable_data_ptr<float>(), std.mutable_data_ptr<float>(),
                               reinterpret_cast<void *>(stream));
    }
    return py::int_(code);
}

}  // namespace

PYBIND11_MODULE(_hot_host, m)
{
    m.def("linear_forward", &linear_forward);
    m.def("linear_backward", &linear_backward);
    m.def("kl_layer", &kl_layer);
    m.def("stats_whole", &stats_whole);
}
