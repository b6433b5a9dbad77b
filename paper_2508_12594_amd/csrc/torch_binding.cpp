// Native half of the Python binding: checks torch tensors, makes the outputs and the workspace that the caller did
// not bring, and calls libflare.so on the current (or the given) stream.  No arithmetic of the operator is here.
//
// Why native: with argument checks, allocations and the C call marshalled in Python (ctypes) a forward cost the host
// 27 us and a training step through torch.autograd 215-230 us, while the kernels of four meshes of 16384 tokens
// (H = 8, d = 16, M = 64, bf16) need 31 and 84 us: every small or medium call was bound by the interpreter.
#include <torch/csrc/autograd/function.h>
#include <torch/csrc/autograd/functions/utils.h>
#include <torch/csrc/autograd/saved_variable.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/jit/frontend/tracer.h>
#include <torch/csrc/utils/pybind.h>

#include <ATen/ATen.h>
#include <ATen/core/LegacyTypeDispatch.h>
#include <ATen/hip/EmptyTensor.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <c10/hip/HIPStream.h>
#include <dlfcn.h>

#include <optional>
#include <stdexcept>
#include <string>

#include "flare.h"

namespace py = pybind11;
using at::Tensor;
using OptTensor = std::optional<Tensor>;

namespace {

struct Error : std::runtime_error {
    using std::runtime_error::runtime_error;
};
py::object *error_class = nullptr;   // what an Error surfaces as in Python

// The entry points of the libflare.so that the package loaded (see load_library).
struct Library {
    decltype(&flare_strerror) strerror = nullptr;
    decltype(&flare_workspace_bytes) workspace_bytes = nullptr;
    decltype(&flare_encode) encode = nullptr;
    decltype(&flare_decode) decode = nullptr;
    decltype(&flare_forward) forward = nullptr;
    decltype(&flare_forward_static) forward_static = nullptr;
    decltype(&flare_forward_project) forward_project = nullptr;
    decltype(&flare_backward) backward = nullptr;
    decltype(&flare_backward_cast) backward_cast = nullptr;
} lib;

template <typename F>
void resolve(void *handle, const char *name, F &fn)
{
    fn = reinterpret_cast<F>(dlsym(handle, name));
    if (!fn) throw Error(std::string("libflare.so does not export ") + name);
}

void load_library(const std::string &path)
{
    void *h = dlopen(path.c_str(), RTLD_NOW | RTLD_LOCAL);
    if (!h) throw Error(std::string("cannot load libflare.so: ") + dlerror());
    resolve(h, "flare_strerror", lib.strerror);
    resolve(h, "flare_workspace_bytes", lib.workspace_bytes);
    resolve(h, "flare_encode", lib.encode);
    resolve(h, "flare_decode", lib.decode);
    resolve(h, "flare_forward", lib.forward);
    resolve(h, "flare_forward_static", lib.forward_static);
    resolve(h, "flare_forward_project", lib.forward_project);
    resolve(h, "flare_backward", lib.backward);
    resolve(h, "flare_backward_cast", lib.backward_cast);
}

void check(int code, const char *what)
{
    if (code != FLARE_OK)
        throw Error(std::string(what) + " failed: " + std::to_string(code) + " (" + lib.strerror(code) + ")");
}

flare_dtype dtype_code(const Tensor &t)
{
    switch (t.scalar_type()) {
        case at::kFloat: return FLARE_F32;
        case at::kBFloat16: return FLARE_BF16;
        case at::kHalf: return FLARE_F16;
        default: throw Error(std::string("dtype must be float32, bfloat16 or float16, got ") + c10::toString(t.scalar_type()));
    }
}

at::ScalarType scalar_type(flare_dtype dt)
{
    return dt == FLARE_F32 ? at::kFloat : dt == FLARE_BF16 ? at::kBFloat16 : at::kHalf;
}

flare_shape shape_of(const Tensor &q, const Tensor &k, int layout, bool y_f32)
{
    if ((q.dim() != 2 && q.dim() != 3) || k.dim() != 4)
        throw Error("expected q_lat[H,M,d] (or [M,d]: one latent sequence shared by all heads) and "
                    "k[B,H,N,d] (layout 'bhnd') or k[B,N,H,d] (layout 'bnhd')");
    const bool shared = q.dim() == 2;
    const auto ks = k.sizes(), qs = q.sizes();
    const bool heads_first = layout == FLARE_BHND;
    const int64_t Hk = ks[heads_first ? 1 : 2], N = ks[heads_first ? 2 : 1];
    const int64_t H = shared ? Hk : qs[0], M = qs[shared ? 0 : 1], d = qs[shared ? 1 : 2];
    if (Hk != H || ks[3] != d || q.scalar_type() != k.scalar_type())
        throw Error("q_lat and k disagree on H, d or dtype");
    if (!k.is_cuda()) throw Error("k must be a contiguous device tensor");   // before anything asks for a stream
    flare_shape s{};
    s.B = (int)ks[0];
    s.H = (int)H;
    s.N = (int)N;
    s.M = (int)M;
    s.d = (int)d;
    s.dtype = dtype_code(k);
    s.layout = (flare_layout)layout;
    s.shared_latents = shared ? 1 : 0;
    s.y_f32 = y_f32 ? 1 : 0;
    return s;
}

std::string text(at::IntArrayRef s)
{
    std::string r = "(";
    for (size_t i = 0; i < s.size(); ++i) r += (i ? ", " : "") + std::to_string(s[i]);
    return r + ")";
}

void *dev(const Tensor &t, const char *name)
{
    if (!t.is_cuda() || !t.is_contiguous()) throw Error(std::string(name) + " must be a contiguous device tensor");
    return t.data_ptr();
}
void *dev(const Tensor &t, const char *name, at::ScalarType dt, at::IntArrayRef shape)
{
    void *p = dev(t, name);
    if (t.scalar_type() != dt) throw Error(std::string(name) + " must have dtype " + c10::toString(dt));
    if (t.sizes() != shape) throw Error(std::string(name) + " must have shape " + text(shape) + ", got " + text(t.sizes()));
    return p;
}
void *dev(const OptTensor &t, const char *name, at::ScalarType dt, at::IntArrayRef shape)
{
    return t ? dev(*t, name, dt, shape) : nullptr;
}
float *f32(void *p) { return static_cast<float *>(p); }

// A new device tensor, from the caching allocator (without the dispatcher: 0.7 instead of 1.7 us)
Tensor new_empty(at::IntArrayRef shape, at::ScalarType dt, const Tensor &like)
{
    return at::detail::empty_cuda(shape, dt, like.device(), std::nullopt);
}
// An output the caller brought, or a new one.
Tensor out_or_new(const OptTensor &t, at::IntArrayRef shape, at::ScalarType dt, const Tensor &like)
{
    return t ? *t : new_empty(shape, dt, like);
}

// Where a call is enqueued: torch's current stream, or the one that was handed in (a torch.cuda.Stream, or with a
// workspace of the caller's anything that has a cuda_stream).
struct Target {
    void *stream;
    std::optional<c10::Stream> other;   // set when it is not the current stream and a temporary has to be recorded there
};
// (called with the GIL; what follows it in the entry points, allocations and launches, runs without)
Target target(const py::object &stream, bool temporaries)
{
    const c10::hip::HIPStream cur = c10::hip::getCurrentHIPStream();
    if (stream.is_none()) return Target{cur.stream(), std::nullopt};
    void *const handle = reinterpret_cast<void *>(stream.attr("cuda_stream").cast<uintptr_t>());
    if (handle == cur.stream() || !temporaries) return Target{handle, std::nullopt};
    const c10::Stream s = c10::Stream::unpack3(stream.attr("stream_id").cast<int64_t>(),
                                               (c10::DeviceIndex)stream.attr("device_index").cast<int64_t>(),
                                               (c10::DeviceType)stream.attr("device_type").cast<int64_t>());
    return Target{handle, s};
}

struct Workspace {
    Tensor hold;
    void *ptr;
    size_t bytes;
};
Workspace workspace_for(size_t need, const OptTensor &given, const Tensor &like, const Target &to)
{
    Tensor t;
    if (given) {
        t = *given;
        if (t.scalar_type() != at::kByte) throw Error("workspace must be a uint8 tensor");
    } else {
        // A temporary block: the kernels are only enqueued when the call returns, so the caching allocator must
        // learn on which stream they run, or it could hand the block to other work on the allocating stream
        // while kernels on `stream` still use it.
        t = new_empty({(int64_t)(need < 256 ? 256 : need)}, at::kByte, like);
        if (to.other) t.record_stream(*to.other);
    }
    return Workspace{t, t.data_ptr(), (size_t)t.numel()};
}
size_t fwd_bytes(const flare_shape &s)
{
    size_t n = 0;
    check(lib.workspace_bytes(&s, &n, nullptr), "flare_workspace_bytes");
    return n;
}
size_t bwd_bytes(const flare_shape &s)
{
    size_t n = 0;
    check(lib.workspace_bytes(&s, nullptr, &n), "flare_workspace_bytes");
    return n;
}

// flare_shape.y_f32: asked for, or implied by an fp32 y next to 16-bit token tensors.
bool wants_f32_y(const OptTensor &y, const Tensor &k, bool asked)
{
    return asked || (y && y->scalar_type() == at::kFloat && k.scalar_type() != at::kFloat);
}

struct Dims {
    std::array<int64_t, 4> z;
    std::array<int64_t, 3> lse_enc, lse_dec;
    explicit Dims(const flare_shape &s) : z{s.B, s.H, s.M, s.d}, lse_enc{s.B, s.H, s.M}, lse_dec{s.B, s.H, s.N} {}
};

std::tuple<Tensor, Tensor> encode(const Tensor &q, const Tensor &k, const Tensor &v, double scale, const OptTensor &z_in,
                                  const OptTensor &le_in, const OptTensor &ws_in, const py::object &stream, int layout)
{
    const flare_shape s = shape_of(q, k, layout, false);
    const Dims dim(s);
    const Target to = target(stream, !ws_in);
    const py::gil_scoped_release no_gil;
    Tensor z = out_or_new(z_in, dim.z, at::kFloat, k), le = out_or_new(le_in, dim.lse_enc, at::kFloat, k);
    const Workspace ws = workspace_for(fwd_bytes(s), ws_in, k, to);
    check(lib.encode(&s, dev(q, "q_lat"), dev(k, "k"), dev(v, "v", k.scalar_type(), k.sizes()),
                     f32(dev(z, "z", at::kFloat, dim.z)), f32(dev(le, "lse_enc", at::kFloat, dim.lse_enc)), (float)scale,
                     ws.ptr, ws.bytes, to.stream),
          "flare_encode");
    return {z, le};
}

Tensor decode(const Tensor &q, const Tensor &k, const Tensor &z, double scale, const OptTensor &y_in,
              const OptTensor &ld, const OptTensor &ws_in, const py::object &stream, int layout, bool y_f32)
{
    const bool wide = wants_f32_y(y_in, k, y_f32);
    const flare_shape s = shape_of(q, k, layout, wide);
    const Dims dim(s);
    const Target to = target(stream, !ws_in);
    const py::gil_scoped_release no_gil;
    const at::ScalarType ydt = wide ? at::kFloat : k.scalar_type();
    Tensor y = out_or_new(y_in, k.sizes(), ydt, k);
    const Workspace ws = workspace_for(fwd_bytes(s), ws_in, k, to);
    check(lib.decode(&s, dev(q, "q_lat"), dev(k, "k"), f32(dev(z, "z", at::kFloat, dim.z)),
                     dev(y, "y", ydt, k.sizes()), f32(dev(ld, "lse_dec", at::kFloat, dim.lse_dec)), (float)scale, ws.ptr,
                     ws.bytes, to.stream),
          "flare_decode");
    return y;
}

std::tuple<Tensor, Tensor, Tensor> forward(const Tensor &q, const Tensor &k, const Tensor &v, double scale,
                                           const OptTensor &y_in, const OptTensor &z_in, const OptTensor &le_in,
                                           const OptTensor &ld, const OptTensor &ws_in, const py::object &stream,
                                           int layout, bool y_f32)
{
    const bool wide = wants_f32_y(y_in, k, y_f32);
    const flare_shape s = shape_of(q, k, layout, wide);
    const Dims dim(s);
    const Target to = target(stream, !ws_in);
    const py::gil_scoped_release no_gil;
    const at::ScalarType ydt = wide ? at::kFloat : k.scalar_type();
    Tensor y = out_or_new(y_in, k.sizes(), ydt, k), z = out_or_new(z_in, dim.z, at::kFloat, k),
           le = out_or_new(le_in, dim.lse_enc, at::kFloat, k);
    const Workspace ws = workspace_for(fwd_bytes(s), ws_in, k, to);
    check(lib.forward(&s, dev(q, "q_lat"), dev(k, "k"), dev(v, "v", k.scalar_type(), k.sizes()),
                      dev(y, "y", ydt, k.sizes()), f32(dev(z, "z", at::kFloat, dim.z)),
                      f32(dev(le, "lse_enc", at::kFloat, dim.lse_enc)), f32(dev(ld, "lse_dec", at::kFloat, dim.lse_dec)),
                      (float)scale, ws.ptr, ws.bytes, to.stream),
          "flare_forward");
    return {y, z, le};
}

void forward_static(const Tensor &q, const Tensor &k, const Tensor &v, double scale, const Tensor &y, const Tensor &z,
                    const Tensor &le, const OptTensor &ld, const py::object &stream, int layout)
{
    const bool wide = wants_f32_y(y, k, false);
    const flare_shape s = shape_of(q, k, layout, wide);
    const Dims dim(s);
    const Target to = target(stream, false);
    const py::gil_scoped_release no_gil;
    check(lib.forward_static(&s, dev(q, "q_lat"), dev(k, "k"), dev(v, "v", k.scalar_type(), k.sizes()),
                             dev(y, "y", wide ? at::kFloat : k.scalar_type(), k.sizes()),
                             f32(dev(z, "z", at::kFloat, dim.z)), f32(dev(le, "lse_enc", at::kFloat, dim.lse_enc)),
                             f32(dev(ld, "lse_dec", at::kFloat, dim.lse_dec)), (float)scale, to.stream),
          "flare_forward_static");
}

std::tuple<Tensor, Tensor, Tensor> forward_project(const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &w,
                                                   double scale, const OptTensor &bias, const OptTensor &out_in,
                                                   const OptTensor &y_in, const OptTensor &z_in, const OptTensor &le_in,
                                                   const OptTensor &ld, const OptTensor &ws_in, const py::object &stream,
                                                   bool keep_y)
{
    const flare_shape s = shape_of(q, k, FLARE_BNHD, false);
    const Dims dim(s);
    const Target to = target(stream, !ws_in);
    const py::gil_scoped_release no_gil;
    const int64_t C = (int64_t)s.H * s.d;
    const at::ScalarType dt = k.scalar_type();
    const std::array<int64_t, 3> out_dim{s.B, s.N, C};
    const std::array<int64_t, 2> w_dim{C, C};
    const std::array<int64_t, 1> b_dim{C};
    Tensor out = out_or_new(out_in, out_dim, dt, k), z = out_or_new(z_in, dim.z, at::kFloat, k),
           le = out_or_new(le_in, dim.lse_enc, at::kFloat, k);
    OptTensor y = y_in;
    if (!y && keep_y) y = new_empty(k.sizes(), dt, k);
    const Workspace ws = workspace_for(fwd_bytes(s), ws_in, k, to);
    check(lib.forward_project(&s, dev(q, "q_lat"), dev(k, "k"), dev(v, "v", dt, k.sizes()), dev(w, "w_out", dt, w_dim),
                              f32(dev(bias, "bias", at::kFloat, b_dim)), dev(out, "out", dt, out_dim),
                              dev(y, "y", dt, k.sizes()), f32(dev(z, "z", at::kFloat, dim.z)),
                              f32(dev(le, "lse_enc", at::kFloat, dim.lse_enc)),
                              f32(dev(ld, "lse_dec", at::kFloat, dim.lse_dec)), (float)scale, ws.ptr, ws.bytes,
                              to.stream),
          "flare_forward_project");
    return {out, z, le};
}

std::tuple<Tensor, Tensor, Tensor> backward(const Tensor &q, const Tensor &k, const Tensor &v, const Tensor &dy,
                                            const Tensor &z, const Tensor &le, double scale, const OptTensor &y,
                                            const OptTensor &ld, const OptTensor &dq_in, const OptTensor &dk_in,
                                            const OptTensor &dv_in, const OptTensor &ws_in, const py::object &stream,
                                            int layout, int variant)
{
    const bool wide = wants_f32_y(y, k, false);
    flare_shape s = shape_of(q, k, layout, wide);
    s.variant = variant;
    const Dims dim(s);
    const Target to = target(stream, !ws_in);
    const py::gil_scoped_release no_gil;
    const at::ScalarType dt = k.scalar_type();
    Tensor dq = out_or_new(dq_in, q.sizes(), at::kFloat, k), dk = out_or_new(dk_in, k.sizes(), dt, k),
           dv = out_or_new(dv_in, k.sizes(), dt, k);
    const Workspace ws = workspace_for(bwd_bytes(s), ws_in, k, to);
    check(lib.backward(&s, dev(q, "q_lat"), dev(k, "k"), dev(v, "v", dt, k.sizes()),
                       dev(y, "y", wide ? at::kFloat : dt, k.sizes()), f32(dev(ld, "lse_dec", at::kFloat, dim.lse_dec)),
                       dev(dy, "dy", dt, k.sizes()), f32(dev(z, "z", at::kFloat, dim.z)),
                       f32(dev(le, "lse_enc", at::kFloat, dim.lse_enc)), f32(dev(dq, "dq_lat", at::kFloat, q.sizes())),
                       dev(dk, "dk", dt, k.sizes()), dev(dv, "dv", dt, k.sizes()), (float)scale, ws.ptr, ws.bytes,
                       to.stream),
          "flare_backward");
    return {dq, dk, dv};
}

// ---- the differentiable mixer ------------------------------------------------------------------------------
// z, lse_enc and lse_dec are never seen by the caller: they share one allocation (offsets in bytes, 256-aligned).
struct Saved {
    size_t lse_enc, lse_dec, bytes;
    explicit Saved(const flare_shape &s)
    {
        const auto pad = [](size_t x) { return (x + 255) & ~(size_t)255; };
        const size_t bh = (size_t)s.B * s.H;
        lse_enc = pad(bh * s.M * s.d * 4);
        lse_dec = lse_enc + pad(bh * s.M * 4);
        bytes = lse_dec + pad(bh * s.N * 4);
    }
};

// The autograd node, written out (a torch::autograd::Function costs several microseconds more in both directions).
struct MixerBackward : torch::autograd::Node {
    torch::autograd::SavedVariable q, k, v, y, stats;
    flare_shape shape{};
    float scale = 0.f;

    std::string name() const override { return "FlareMixerBackward"; }
    void release_variables() override
    {
        std::lock_guard<std::mutex> lock(mutex_);
        for (auto *t : {&q, &k, &v, &y, &stats}) t->reset_data();
    }
    torch::autograd::variable_list apply(torch::autograd::variable_list &&grads) override
    {
        std::lock_guard<std::mutex> lock(mutex_);
        try {
            return gradients(std::move(grads[0]));
        } catch (const Error &e) {   // (the engine would turn it into a plain RuntimeError)
            const py::gil_scoped_acquire gil;
            PyErr_SetString(error_class->ptr(), e.what());
            python_error raised;
            raised.persist();
            throw raised;
        }
    }
    torch::autograd::variable_list gradients(Tensor &&dy)
    {
        const Tensor tq = q.unpack(), tk = k.unpack(), tv = v.unpack(), ty = y.unpack(shared_from_this()),
                     ts = stats.unpack();
        // The kernels go by the forward's shape, and a saved-tensor hook may have handed back anything: everything is
        // held against that shape before anything is allocated or launched.
        const at::ScalarType dt = scalar_type(shape.dtype);
        const bool heads_first = shape.layout == FLARE_BHND;
        const std::array<int64_t, 4> tok{shape.B, heads_first ? shape.H : shape.N, heads_first ? shape.N : shape.H, shape.d};
        const std::array<int64_t, 3> lat{shape.H, shape.M, shape.d};
        const at::IntArrayRef lat_dim = at::IntArrayRef(lat).slice(shape.shared_latents ? 1 : 0);
        const Saved off(shape);
        const std::array<int64_t, 1> stats_dim{(int64_t)off.bytes};
        const void *const pq = dev(tq, "q_lat", dt, lat_dim), *const pk = dev(tk, "k", dt, tok),
                   *const pv = dev(tv, "v", dt, tok), *const py = dev(ty, "y", shape.y_f32 ? at::kFloat : dt, tok);
        char *const st = static_cast<char *>(dev(ts, "saved statistics", at::kByte, stats_dim));
        if (!dy.defined()) dy = at::zeros(tok, ty.options().requires_grad(false));   // nothing came back to y
        // (with an fp32 y autograd hands over an fp32 dY: the library takes it in the storage type)
        if (dy.scalar_type() != dt) dy = dy.to(dt);
        dy = dy.contiguous();
        const Target to{c10::hip::getCurrentHIPStream().stream(), std::nullopt};
        Tensor dq = new_empty(lat_dim, dt, tk), dk = new_empty(tok, dt, tk), dv = new_empty(tok, dt, tk);
        const Workspace ws = workspace_for(bwd_bytes(shape), std::nullopt, tk, to);
        check(lib.backward_cast(&shape, pq, pk, pv, py, f32(st + off.lse_dec), dev(dy, "dy", dt, tok), f32(st),
                                f32(st + off.lse_enc), dq.data_ptr(), dk.data_ptr(), dv.data_ptr(), scale, ws.ptr, ws.bytes,
                                to.stream),
              "flare_backward_cast");
        return {dq, dk, dv};
    }
};

// Nothing under torch.jit.trace: y is made behind the dispatcher, so a trace would hold it as a constant (the caller then
// records the step as an operation, see autograd.py).
OptTensor mixer(const Tensor &q_in, const Tensor &k_in, const Tensor &v_in, double scale, int layout, bool y_f32)
{
    if (torch::jit::tracer::isTracing()) return std::nullopt;
    for (const Tensor *t : {&q_in, &k_in, &v_in})   // a tangent would be lost without a word
        if (t->_fw_grad(0).defined()) throw Error("flare_mixer has no forward-mode derivative");
    std::shared_ptr<MixerBackward> node;
    if (at::GradMode::is_enabled() && (q_in.requires_grad() || k_in.requires_grad() || v_in.requires_grad())) {
        node = std::shared_ptr<MixerBackward>(new MixerBackward(), torch::autograd::deleteNode);
        node->set_next_edges(torch::autograd::collect_next_edges(q_in, k_in, v_in));
    }
    Tensor q = q_in, k = k_in, v = v_in;
    {
        const at::AutoDispatchBelowADInplaceOrView below;   // not around the saving: saved-tensor hooks run there
        q = q.contiguous();
        k = k.contiguous();
        v = v.contiguous();
    }
    const flare_shape s = shape_of(q, k, layout, y_f32);
    const Saved off(s);
    const Target to{c10::hip::getCurrentHIPStream().stream(), std::nullopt};
    Tensor y = new_empty(k.sizes(), y_f32 ? at::kFloat : k.scalar_type(), k);
    Tensor stats = new_empty({(int64_t)off.bytes}, at::kByte, k);
    const Workspace ws = workspace_for(fwd_bytes(s), std::nullopt, k, to);
    char *const st = static_cast<char *>(stats.data_ptr());
    check(lib.forward(&s, dev(q, "q_lat"), dev(k, "k"), dev(v, "v", k.scalar_type(), k.sizes()), y.data_ptr(), f32(st),
                      f32(st + off.lse_enc), f32(st + off.lse_dec), (float)scale, ws.ptr, ws.bytes, to.stream),
          "flare_forward");
    if (node) {
        node->shape = s;
        node->scale = (float)scale;
        node->q = torch::autograd::SavedVariable(q, false);
        node->k = torch::autograd::SavedVariable(k, false);
        node->v = torch::autograd::SavedVariable(v, false);
        node->stats = torch::autograd::SavedVariable(stats, false);
        torch::autograd::set_history(y, node);
        node->y = torch::autograd::SavedVariable(y, true);
    }
    return y;
}

}  // namespace

PYBIND11_MODULE(_native, m)
{
    m.def("load_library", &load_library);
    // errors surface as the package's own exception class
    m.def("set_error_class", [](py::object cls) {
        if (error_class) return;
        error_class = new py::object(std::move(cls));
        py::register_exception_translator([](std::exception_ptr p) {
            try {
                if (p) std::rethrow_exception(p);
            } catch (const Error &e) {
                PyErr_SetString(error_class->ptr(), e.what());
            }
        });
    });
    m.def("encode", &encode);
    m.def("decode", &decode);
    m.def("forward", &forward);
    m.def("forward_static", &forward_static);
    m.def("forward_project", &forward_project);
    m.def("backward", &backward);
    m.def("mixer", &mixer, py::call_guard<py::gil_scoped_release>());
}
