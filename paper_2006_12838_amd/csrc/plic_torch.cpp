// The package's torch functions in native code: plain CUDA tensors in, the C
// ABI's kernels on the current stream, autograd nodes that need no Python in
// the backward. A small call is bound by the host, which the interpreter's part
// had three quarters of: 1,003 offsets 13.2 -> 5.7 us, forward and backward of
// 4,000,037 rows 106 -> 54 us, of 2,000 112 -> 63 us, of a 192^3 lattice's
// curvature 113 -> 66 us.
// Anything out of the ordinary (other types and layouts, subclasses, broadcast
// shapes) is left to the Python path: these functions then return None.
#include <ATen/ATen.h>
#include <c10/core/DeviceGuard.h>
#include <c10/hip/HIPStream.h>
#include <hip/hip_runtime_api.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/csrc/utils/pybind.h>

#include "../../include/plic.h"

namespace {

using at::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::tensor_list;

// the current stream of t's device (in a backward, the forward's)
void* stream_of(const Tensor& t) {
    return c10::hip::getCurrentHIPStream(t.device().index()).stream();
}

void check(int rc, const char* name) {
    if (rc == PLIC_EHIP) TORCH_CHECK(false, name, ": ", plic_status_string(rc), " (hipError ", plic_last_hip_error(), ")");
    TORCH_CHECK(rc == PLIC_OK, name, ": ", plic_status_string(rc));
}

// exactly a torch.Tensor or Parameter, contiguous, float32 or float64 on a GPU
bool plain(const py::handle& h, Tensor* t) {
    if (!THPVariable_CheckExact(h.ptr())) return false;
    *t = THPVariable_Unpack(h.ptr());
    return t->is_cuda() && t->layout() == at::kStrided && (t->scalar_type() == at::kFloat || t->scalar_type() == at::kDouble) &&
           t->is_contiguous() && !t->is_neg();
}

bool alike(const Tensor& a, const Tensor& b) { return a.scalar_type() == b.scalar_type() && a.device() == b.device(); }

// n: one row (x, y, z) per element of x
bool rows_of(const Tensor& n, const Tensor& x) {
    if (!alike(n, x) || n.dim() != x.dim() + 1 || n.size(-1) != 3) return false;
    for (int64_t k = 0; k < x.dim(); ++k)
        if (n.size(k) != x.size(k)) return false;
    return true;
}

// whether a node will be made: the forward then keeps what its backward needs
template <class... T> bool will_differentiate(const T&... t) {
    return at::GradMode::is_enabled() && (t.requires_grad() || ...);
}

// what a backward gets: its gradient has the result's type, device and shape, and
// saved tensors (which a caller's saved-tensor hooks may have replaced) match it
void check_grad(const Tensor& g, const Tensor& saved, int64_t per = 1) {
    TORCH_CHECK(alike(saved, g) && saved.is_cuda() && saved.layout() == at::kStrided && saved.is_contiguous() &&
                    saved.numel() == g.numel() * per,
                "a saved tensor or the gradient is not of the result's type, device, layout or size");
}

template <class S> S* ptr(const Tensor& t) { return static_cast<S*>(t.data_ptr()); }

// ---- offsets -------------------------------------------------------------------
// The backward works on a copy of n that the forward's kernel writes beside d0,
// so n may change in between.
struct OffsetRows : torch::autograd::Function<OffsetRows> {
    static Tensor forward(AutogradContext* ctx, const Tensor& n, const Tensor& V0, int64_t solver, int64_t precision,
                          bool keep) {
        const c10::DeviceGuard device(V0.device());
        const Tensor d0 = at::empty_like(V0), copy = keep ? at::empty_like(n) : Tensor();
        void* st = stream_of(V0);
        void* c = keep ? copy.data_ptr() : nullptr;
        if (V0.scalar_type() == at::kDouble)
            check(plic_offset_rows_f64(ptr<double>(n), ptr<double>(V0), ptr<double>(d0), static_cast<double*>(c), V0.numel(),
                                       static_cast<int>(solver), st), "plic_offset_rows_f64");
        else
            check(plic_offset_rows_f32(ptr<float>(n), ptr<float>(V0), ptr<float>(d0), static_cast<float*>(c), V0.numel(),
                                       static_cast<int>(solver), static_cast<int>(precision), st), "plic_offset_rows_f32");
        if (keep) {
            ctx->save_for_backward({copy, V0});
            ctx->saved_data["o"] = solver * 8 + precision;
        }
        return d0;
    }

    static tensor_list backward(AutogradContext* ctx, const tensor_list& grads) {
        const auto saved = ctx->get_saved_variables();
        const Tensor &n = saved[0], &V0 = saved[1], g = grads[0].contiguous();
        const int64_t o = ctx->saved_data["o"].toInt();
        const c10::DeviceGuard device(V0.device());
        check_grad(g, V0);
        check_grad(g, n, 3);
        const Tensor gn = at::empty_like(n), gv = at::empty_like(V0);
        void* st = stream_of(V0);
        const int solver = static_cast<int>(o / 8), precision = static_cast<int>(o % 8);
        if (V0.scalar_type() == at::kDouble)
            check(plic_offset_backward_rows_f64(ptr<double>(n), ptr<double>(V0), ptr<double>(g), ptr<double>(gn),
                                                ptr<double>(gv), V0.numel(), solver, st), "plic_offset_backward_rows_f64");
        else
            check(plic_offset_backward_rows_f32(ptr<float>(n), ptr<float>(V0), ptr<float>(g), ptr<float>(gn), ptr<float>(gv),
                                                V0.numel(), solver, precision, st), "plic_offset_backward_rows_f32");
        return {gn, gv, Tensor(), Tensor(), Tensor()};
    }
};

struct OffsetParts : torch::autograd::Function<OffsetParts> {
    static Tensor forward(AutogradContext* ctx, const Tensor& nx, const Tensor& ny, const Tensor& nz, const Tensor& V0,
                          int64_t solver, int64_t precision) {
        const c10::DeviceGuard device(V0.device());
        const Tensor d0 = at::empty_like(V0);
        void* st = stream_of(V0);
        if (V0.scalar_type() == at::kDouble)
            check(plic_offset_f64(ptr<double>(nx), ptr<double>(ny), ptr<double>(nz), ptr<double>(V0), ptr<double>(d0),
                                  V0.numel(), static_cast<int>(solver), st), "plic_offset_f64");
        else
            check(plic_offset_f32(ptr<float>(nx), ptr<float>(ny), ptr<float>(nz), ptr<float>(V0), ptr<float>(d0), V0.numel(),
                                  static_cast<int>(solver), static_cast<int>(precision), st), "plic_offset_f32");
        ctx->save_for_backward({nx, ny, nz, V0});
        ctx->saved_data["o"] = solver * 8 + precision;
        return d0;
    }

    static tensor_list backward(AutogradContext* ctx, const tensor_list& grads) {
        const auto saved = ctx->get_saved_variables();
        const Tensor &nx = saved[0], &ny = saved[1], &nz = saved[2], &V0 = saved[3], g = grads[0].contiguous();
        const int64_t o = ctx->saved_data["o"].toInt();
        const c10::DeviceGuard device(V0.device());
        for (const Tensor& t : saved) check_grad(g, t);
        const Tensor gx = at::empty_like(V0), gy = at::empty_like(V0), gz = at::empty_like(V0), gv = at::empty_like(V0);
        void* st = stream_of(V0);
        const int solver = static_cast<int>(o / 8), precision = static_cast<int>(o % 8);
        if (V0.scalar_type() == at::kDouble)
            check(plic_offset_backward_f64(ptr<double>(nx), ptr<double>(ny), ptr<double>(nz), ptr<double>(V0), ptr<double>(g),
                                           ptr<double>(gx), ptr<double>(gy), ptr<double>(gz), ptr<double>(gv), V0.numel(),
                                           solver, st), "plic_offset_backward_f64");
        else
            check(plic_offset_backward_f32(ptr<float>(nx), ptr<float>(ny), ptr<float>(nz), ptr<float>(V0), ptr<float>(g),
                                           ptr<float>(gx), ptr<float>(gy), ptr<float>(gz), ptr<float>(gv), V0.numel(), solver,
                                           precision, st), "plic_offset_backward_f32");
        return {gx, gy, gz, gv, Tensor(), Tensor()};
    }
};

py::object wrap(const Tensor& t) { return py::reinterpret_steal<py::object>(THPVariable_Wrap(t)); }

py::object offset_rows(const py::handle& hn, const py::handle& hv, int64_t solver, int64_t precision) {
    Tensor n, v;
    if (!plain(hn, &n) || !plain(hv, &v) || !rows_of(n, v)) return py::none();
    return wrap(OffsetRows::apply(n, v, solver, precision, will_differentiate(n, v)));
}

py::object offset_parts(const py::handle& hx, const py::handle& hy, const py::handle& hz, const py::handle& hv, int64_t solver,
                        int64_t precision) {
    Tensor x, y, z, v;
    if (!plain(hx, &x) || !plain(hy, &y) || !plain(hz, &z) || !plain(hv, &v)) return py::none();
    for (const Tensor* t : {&x, &y, &z})
        if (!alike(*t, v) || !t->sizes().equals(v.sizes())) return py::none();
    return wrap(OffsetParts::apply(x, y, z, v, solver, precision));
}

py::object volume_rows(const py::handle& hn, const py::handle& hd, int64_t precision) {
    Tensor n, d;
    if (!plain(hn, &n) || !plain(hd, &d) || !rows_of(n, d)) return py::none();
    const c10::DeviceGuard device(d.device());
    const at::NoGradGuard no_grad;
    const Tensor v = at::empty_like(d);
    void* st = stream_of(d);
    if (d.scalar_type() == at::kDouble)
        check(plic_volume_rows_f64(ptr<double>(n), ptr<double>(d), ptr<double>(v), d.numel(), st), "plic_volume_rows_f64");
    else
        check(plic_volume_rows_f32(ptr<float>(n), ptr<float>(d), ptr<float>(v), d.numel(), static_cast<int>(precision), st),
              "plic_volume_rows_f32");
    return wrap(v);
}

// ---- curvature -----------------------------------------------------------------
// The forward's workspace is kept for the backward, which reuses its interface
// scan (the saved phi is checked for changes in place) and lets it go; a second
// backward of the same node scans.
struct Curvature : torch::autograd::Function<Curvature> {
    struct Options {
        int solver, precision, normal, neighbours;
        explicit Options(int64_t o)
            : solver(static_cast<int>(o & 255)), precision(static_cast<int>(o >> 8 & 255)),
              normal(static_cast<int>(o >> 16 & 255)), neighbours(static_cast<int>(o >> 24 & 1)) {}
    };

    static Tensor workspace(const Tensor& phi, size_t bytes) {
        return at::empty({static_cast<int64_t>(bytes > 0 ? bytes : 1)}, phi.options().dtype(at::kByte).requires_grad(false));
    }

    static Tensor forward(AutogradContext* ctx, const Tensor& phi, int64_t o, bool keep) {
        const Options opt(o);
        const c10::DeviceGuard device(phi.device());
        const int64_t X = phi.size(2), Y = phi.size(1), Z = phi.size(0);
        const Tensor kappa = at::empty_like(phi);
        const Tensor ws = workspace(phi, plic_curvature_workspace_bytes_ex(X, Y, Z, opt.neighbours));
        check(plic_curvature_ex_f32(ptr<float>(phi), X, Y, Z, ptr<float>(kappa), opt.solver, opt.precision, opt.normal,
                                    opt.neighbours, ws.data_ptr(), static_cast<size_t>(ws.numel()), stream_of(phi)),
              "plic_curvature_ex_f32");
        if (keep) {
            ctx->save_for_backward({phi});
            ctx->saved_data["o"] = o;
            ctx->saved_data["ws"] = ws;
        }
        return kappa;
    }

    static tensor_list backward(AutogradContext* ctx, const tensor_list& grads) {
        const Tensor phi = ctx->get_saved_variables()[0], g = grads[0].contiguous();
        const Options opt(ctx->saved_data["o"].toInt());
        const c10::DeviceGuard device(phi.device());
        check_grad(g, phi);
        TORCH_CHECK(phi.sizes().equals(g.sizes()), "the saved lattice is not of the result's shape");
        const int64_t X = phi.size(2), Y = phi.size(1), Z = phi.size(0);
        const Tensor gp = at::empty_like(phi);
        void* st = stream_of(phi);
        Tensor ws;
        const auto kept = ctx->saved_data.find("ws");
        if (kept != ctx->saved_data.end()) {
            ws = kept->second.toTensor();
            ctx->saved_data.erase(kept);
        }
        bool reuse = ws.defined();
        if (!reuse) ws = workspace(phi, plic_curvature_workspace_bytes_ex(X, Y, Z, opt.neighbours));
        for (int attempt = 0; attempt < 2; ++attempt, reuse = false) {
            const auto f = reuse ? plic_curvature_backward_reuse_f32 : plic_curvature_backward_ex_f32;
            check(f(ptr<float>(phi), X, Y, Z, ptr<float>(g), ptr<float>(gp), opt.solver, opt.precision, opt.normal,
                    opt.neighbours, ws.data_ptr(), static_cast<size_t>(ws.numel()), st),
                  reuse ? "plic_curvature_backward_reuse_f32" : "plic_curvature_backward_ex_f32");
            // neighbour normals have no fallback for rows that do not fit: asked
            // (which waits for the stream, so not under capture), and again with
            // a workspace that holds them all
            if (!opt.neighbours || phi.numel() == 0) break;
            hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
            if (hipStreamIsCapturing(static_cast<hipStream_t>(st), &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) break;
            int64_t cells = 0;
            size_t need = 0;
            const int rc = plic_curvature_status(ws.data_ptr(), static_cast<size_t>(ws.numel()), X, Y, Z, 1, &cells, &need, st);
            if (rc == PLIC_OK) break;
            TORCH_CHECK(rc == PLIC_EWORKSPACE && attempt == 0, "plic_curvature_backward_ex_f32: ", plic_status_string(rc), " (",
                        cells, " interface cells need ", need, " bytes, workspace has ", ws.numel(), ")");
            ws = workspace(phi, need);
        }
        return {gp, Tensor(), Tensor()};
    }
};

py::object curvature(const py::handle& hp, int64_t solver, int64_t precision, int64_t normal, bool neighbours) {
    Tensor phi;
    if (!plain(hp, &phi) || phi.scalar_type() != at::kFloat || phi.dim() != 3) return py::none();
    for (const int64_t v : {solver, precision, normal})
        if (v < 0 || v > 255) return py::none();
    const int64_t o = solver | precision << 8 | normal << 16 | static_cast<int64_t>(neighbours) << 24;
    return wrap(Curvature::apply(phi, o, will_differentiate(phi)));
}

}  // namespace

PYBIND11_MODULE(_native, m) {
    m.def("offset_rows", &offset_rows);
    m.def("offset_parts", &offset_parts);
    m.def("volume_rows", &volume_rows);
    m.def("curvature", &curvature);
}
