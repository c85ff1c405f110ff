// The host path of the Python entry points that sit in a model's inner loop: argument checks, output and
// workspace allocation, the call into the library and the autograd nodes, in native code.  A short solve takes the
// device about 10 us; checks, allocations and ctypes marshalling in Python took 15 us of host time on top of the call.
// No arithmetic here, and no device code: everything runs in the kernels behind pararnn.h.
#include <ATen/ATen.h>
#include <c10/hip/HIPCachingAllocator.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/utils/pybind.h>
#include <torch/custom_class.h>

#include <algorithm>
#include <array>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "pararnn.h"

namespace py = pybind11;
using at::Tensor;
using OptTensor = c10::optional<Tensor>;

namespace {

// Entry points of a cell: the built-in ones with the cell number bound, or those of a library made with
// PARARNN_DEFINE_CELL (addresses).
struct Cell : torch::CustomClassHolder {
    using Ws = size_t (*)(int, int, int, int, int);
    using Fwd = int (*)(int, const float *, const void *, const void *, int, int, int, float, int, void *, int *, float *,
                        void *, size_t, void *);
    using Bwd = int (*)(int, const float *, const void *, const void *, const void *, const void *, int, int, int, void *,
                        float *, void *, void *, size_t, void *);
    using Parts = size_t (*)(int, int, int, int, int, int, size_t *);
    int number = -1, G = 0, S = 0;
    std::string what;
    Ws ws_fn = nullptr, ws_fused_fn = nullptr;
    Parts parts_fn = nullptr;      // not in a library built before there was one
    Fwd fwd_fn = nullptr;
    Bwd bwd_fn = nullptr;

    size_t ws(int dt, int B, int L, int H, int back) const
    {
        return number >= 0 ? pararnn_workspace_bytes(number, dt, B, L, H, back) : ws_fn(dt, B, L, H, back);
    }
    size_t ws_fused(int dt, int B, int L, int H, int n) const
    {
        return number >= 0 ? pararnn_workspace_bytes_fused(number, dt, B, L, H, n) : ws_fused_fn(dt, B, L, H, n);
    }
    size_t parts(int dt, int B, int L, int H, int back, int n, size_t *rest) const
    {
        if (number >= 0) return pararnn_workspace_parts(number, dt, B, L, H, back, n, rest);
        return parts_fn ? parts_fn(dt, B, L, H, back, n, rest) : 0;
    }
};
using CellPtr = c10::intrusive_ptr<Cell>;

const char *type_name(at::ScalarType t)
{
    return t == at::kFloat ? "torch.float32" : t == at::kBFloat16 ? "torch.bfloat16" : t == at::kInt ? "torch.int32" : c10::toString(t);
}

std::string shape_str(at::IntArrayRef s)
{
    std::string r = "(";
    for (size_t i = 0; i < s.size(); ++i) r += (i ? ", " : "") + std::to_string(s[i]);
    return r + (s.size() == 1 ? ",)" : ")");
}

void check(const Tensor &t, const char *name, at::ScalarType dtype)
{
    if (!t.is_cuda()) throw py::value_error(std::string(name) + " must be a CUDA tensor");
    if (t.scalar_type() != dtype)
        throw py::value_error(std::string(name) + " must be " + type_name(dtype) + ", got " + type_name(t.scalar_type()));
    if (!t.is_contiguous()) throw py::value_error(std::string(name) + " must be contiguous");
}
void check(const Tensor &t, const char *name, at::ScalarType dtype, at::IntArrayRef shape)
{
    check(t, name, dtype);
    if (t.sizes() != shape)
        throw py::value_error(std::string(name) + " must have shape " + shape_str(shape) + ", got " + shape_str(t.sizes()));
}

int dtype_code(at::ScalarType t)
{
    if (t == at::kFloat) return PARARNN_F32;
    if (t == at::kBFloat16) return PARARNN_BF16;
    throw py::key_error(type_name(t));
}

bool has(const OptTensor &t) { return t.has_value() && t->defined(); }
void *ptr(const OptTensor &t) { return has(t) ? t->data_ptr() : nullptr; }
void *stream_ptr(const c10::optional<int64_t> &stream)
{
    return stream ? reinterpret_cast<void *>(*stream) : static_cast<void *>(c10::hip::getCurrentHIPStream().stream());
}
void raise_if(int code, const std::string &what)
{
    if (code != 0)
        throw std::runtime_error(what + " failed: " + pararnn_status_string(code) + " (" + std::to_string(code) + ")");
}
Tensor workspace_of(size_t bytes, const Tensor &like, const OptTensor &given)
{
    return has(given) ? *given : at::empty({(int64_t)(bytes > 256 ? bytes : 256)}, like.options().dtype(at::kByte));
}

struct Dims { int B, L, H; };

// ------------------------------------------------------------------ kept workspaces
// The carry records of a solve or a backward pass have to be cleared unless the library knows what they hold: 1.3 GB for
// 2^30 timestep-channels (0.25 ms of a forward solve, 0.05 of a backward pass and, in small passes, a launch of 5 us).  So
// the fronts of the workspaces (control block and records) of the diagonal cells' calls are kept between calls, per device,
// stream and problem, under the library's per-workspace promise; what nothing reads after the call (boundary rows, the fp32
// iterate of bf16 storage, sums of parameter gradients: three quarters of a bf16 solve's workspace) is allocated for each
// call as before.  A call takes a front out while it enqueues its work, and the next one that gets it is behind it in the
// same stream; calls of several threads find different ones.  Bounds per device: kMost fronts and a thirty-second of its
// memory, the least recently used go first, and all of them when torch's allocator would take more memory (GiveBack).  Under stream
// capture, with a workspace or a stream of the caller's, for small problems (0.5 us of host time to look would show there)
// and for kernels without records nothing is kept.
using WsKey = std::array<int64_t, 8>;
constexpr size_t kMost = 16;
constexpr double kSmall = 1 << 20;       // timestep-channels; below, most calls take kernels without records and 10-20 us
struct KeptWs { WsKey key; Tensor ws; };
struct DevicePool {
    std::vector<KeptWs> free;          // least recently used first
    size_t bytes = 0, cap = 0;
};
std::mutex &pool_mutex()
{
    static std::mutex &m = *new std::mutex;
    return m;
}
std::map<int, DevicePool> &pools()
{
    static std::map<int, DevicePool> &p = *new std::map<int, DevicePool>;     // never destroyed: the runtime may be gone by then
    return p;
}

// Part of a workspace, allocated while its size is known to GiveBack.
thread_local size_t t_allocating = 0;
Tensor own_memory(size_t bytes, const Tensor &like)
{
    struct Note {
        explicit Note(size_t n) { t_allocating = n; }
        ~Note() { t_allocating = 0; }
    } note(bytes);
    return workspace_of(bytes, like, {});
}

// Gives a kept workspace up; the device is the current one.  The library has to know before the memory goes.
void give_up(Tensor &ws)
{
    pararnn_workspace_keep(ws.data_ptr(), 0);
    ws.reset();
}

class Workspace {
public:
    // n_iters: of a fixed-count solve, else 0; bytes: of a whole workspace
    Workspace(const Cell &c, bool back, int code, const Dims &d, int64_t n_iters, size_t bytes, const Tensor &like,
              const OptTensor &given, const c10::optional<int64_t> &stream)
    {
        size_t rest = 0;
        const size_t front = has(given) || stream ? 0 : look(c, back, code, d, n_iters, like, &rest);
        if (device_ < 0) { ws_ = workspace_of(bytes, like, given); return; }
        if (!kept_) {
            ws_ = own_memory(front, like);
            kept_ = pararnn_workspace_keep(ws_.data_ptr(), 1) == PARARNN_OK;
        }
        try {
            rest_ = own_memory(rest, like);
        } catch (...) {
            if (kept_) give_up(ws_);         // no destructor runs for an object that was not constructed
            throw;
        }
        pararnn_workspace_rest(ws_.data_ptr(), rest_.data_ptr(), (size_t)rest_.numel());
    }
    Workspace(const Workspace &) = delete;
    Workspace &operator=(const Workspace &) = delete;
    // after a call that failed, or one without carry records
    ~Workspace() { if (kept_) give_up(ws_); }

    void *data() const { return ws_.data_ptr(); }
    size_t size() const { return (size_t)ws_.numel(); }
    // the call's work is enqueued
    void done()
    {
        if (!kept_ || !pararnn_workspace_known(ws_.data_ptr())) return;
        std::vector<KeptWs> old;
        {
            std::lock_guard<std::mutex> lock(pool_mutex());
            DevicePool &p = pools()[device_];
            p.bytes += (size_t)ws_.numel();
            p.free.push_back({key_, std::move(ws_)});
            kept_ = false;
            while (p.free.size() > kMost || p.bytes > p.cap) {
                p.bytes -= (size_t)p.free.front().ws.numel();
                old.push_back(std::move(p.free.front()));
                p.free.erase(p.free.begin());
            }
        }
        for (KeptWs &k : old) give_up(k.ws);
    }

private:
    // Whether this call's front is one to keep (device_), and a kept one if there is one (ws_, kept_).  Returns its size.
    size_t look(const Cell &c, bool back, int code, const Dims &d, int64_t n_iters, const Tensor &like, size_t *rest)
    {
        if ((double)d.B * d.L * d.H < kSmall) return 0;
        const auto cur = c10::hip::getCurrentHIPStream();
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (cur.device_index() != like.get_device() || hipStreamIsCapturing(cur.stream(), &cap) != hipSuccess ||
            cap != hipStreamCaptureStatusNone)
            return 0;
        const size_t front = c.parts(code, d.B, d.L, d.H, back, (int)n_iters, rest);
        if (front == 0) return 0;
        key_ = {reinterpret_cast<int64_t>(cur.stream()), c.number >= 0 ? c.number : reinterpret_cast<int64_t>(c.fwd_fn),
                back ? -1 : n_iters, code, d.B, d.L, d.H, (int64_t)front};
        std::lock_guard<std::mutex> lock(pool_mutex());
        DevicePool &p = pools()[cur.device_index()];
        if (p.cap == 0) {
            size_t avail = 0, total = 0;
            p.cap = hipMemGetInfo(&avail, &total) == hipSuccess ? total / 32 : 1;
        }
        if (front > p.cap) return 0;
        device_ = cur.device_index();
        for (size_t i = p.free.size(); i-- > 0;)
            if (p.free[i].key == key_) {
                ws_ = std::move(p.free[i].ws);
                p.free.erase(p.free.begin() + (long)i);
                p.bytes -= (size_t)ws_.numel();
                kept_ = true;
                break;
            }
        return front;
    }

    Tensor ws_, rest_;
    WsKey key_{};
    int device_ = -1;
    bool kept_ = false;
};

// Gives up what is kept on the current device; returns its bytes.
int64_t release_on_device(int device)
{
    std::vector<KeptWs> old;
    int64_t bytes = 0;
    {
        std::lock_guard<std::mutex> lock(pool_mutex());
        const auto p = pools().find(device);
        if (p == pools().end()) return 0;
        bytes = (int64_t)p->second.bytes;
        p->second.bytes = 0;
        old.swap(p->second.free);
    }
    for (KeptWs &k : old) give_up(k.ws);
    return bytes;
}

int64_t release_workspaces()
{
    std::vector<int> devices;
    {
        std::lock_guard<std::mutex> lock(pool_mutex());
        for (auto &p : pools()) devices.push_back(p.first);
    }
    int64_t bytes = 0;
    for (int d : devices) {
        const c10::DeviceGuard guard(c10::Device(c10::DeviceType::CUDA, (c10::DeviceIndex)d));
        bytes += release_on_device(d);
    }
    return bytes;
}

// torch's allocator asks before it takes more memory from the device, and so before an allocation fails; it does not say
// how much it needs.  It gets everything kept on the device it allocates on: the current one, and no other, whose allocator
// may be locked by a thread that waits for this one.  Only a workspace of this thread's own call does not push out the kept
// ones while there is memory for both: forward and backward pass of one training step would otherwise take turns with the
// same memory for good.  The allocator's lock is held here and taken again by what is freed, which it allows; the pool's own
// lock is never held while memory is allocated or freed.
struct GiveBack : c10::FreeMemoryCallback {
    bool Execute() override
    {
        int device = -1;
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(c10::hip::getCurrentHIPStream().stream(), &cap) != hipSuccess || cap != hipStreamCaptureStatusNone)
            return false;
        if (hipGetDevice(&device) != hipSuccess) return false;
        size_t avail = 0, total = 0;
        if (t_allocating > 0 && hipMemGetInfo(&avail, &total) == hipSuccess) {
            namespace alloc = c10::hip::HIPCachingAllocator;
            const double need = (double)t_allocating + (32 << 20);        // the allocator rounds up
            const double mine = (double)alloc::getDeviceStats(device).reserved_bytes[0].current;
            if (need <= (double)avail && mine + need <= (double)total * alloc::getMemoryFraction(device)) return false;
        }
        return release_on_device(device) > 0;
    }
};

Dims dims4(const Tensor &u, const char *name)
{
    if (u.dim() != 4) throw py::value_error(std::string(name) + " must have four dimensions");
    return {(int)u.size(0), (int)u.size(1), (int)u.size(3)};
}

struct Solve { Tensor h, iters, trace; };

Solve solve(const Cell &c, const Tensor &params, const Tensor &u, const OptTensor &h0, double tol, int64_t max_iter, bool trace,
            const OptTensor &workspace, const c10::optional<int64_t> &stream, const OptTensor &out)
{
    const Dims d = dims4(u, "u");
    const auto dt = u.scalar_type();
    const int code = dtype_code(dt);
    check(u, "u", dt, {d.B, d.L, c.G, d.H});
    check(params, "params", at::kFloat);
    if (has(h0)) check(*h0, "h0", dt, {d.B, c.S, d.H});
    Solve r;
    r.h = has(out) ? *out : at::empty({d.B, d.L, c.S, d.H}, u.options());
    check(r.h, "h", dt, {d.B, d.L, c.S, d.H});
    r.iters = at::empty({2}, u.options().dtype(at::kInt));
    if (trace) r.trace = at::zeros({max_iter > 1 ? max_iter : 1}, u.options().dtype(at::kFloat));
    const size_t need = tol < 0 ? c.ws_fused(code, d.B, d.L, d.H, (int)max_iter) : c.ws(code, d.B, d.L, d.H, 0);
    Workspace ws(c, false, code, d, tol < 0 ? max_iter : 0, need, u, workspace, stream);
    float *tr = trace ? static_cast<float *>(r.trace.data_ptr()) : nullptr;
    const float *p = static_cast<const float *>(params.data_ptr());
    int *it = static_cast<int *>(r.iters.data_ptr());
    const int rc = c.number >= 0
                       ? pararnn_forward(c.number, code, p, u.data_ptr(), ptr(h0), d.B, d.L, d.H, (float)tol, (int)max_iter,
                                         r.h.data_ptr(), it, tr, ws.data(), ws.size(), stream_ptr(stream))
                       : c.fwd_fn(code, p, u.data_ptr(), ptr(h0), d.B, d.L, d.H, (float)tol, (int)max_iter, r.h.data_ptr(), it,
                                  tr, ws.data(), ws.size(), stream_ptr(stream));
    raise_if(rc, c.what + "_forward");
    ws.done();
    return r;
}

struct Grads { Tensor du, dparams, dh0; };

Grads adjoint(const Cell &c, const Tensor &params, const Tensor &u, const OptTensor &h0, const Tensor &h, const Tensor &g,
              bool want_dh0, const OptTensor &workspace, const c10::optional<int64_t> &stream, const Grads *out)
{
    const Dims d = dims4(u, "u");
    const auto dt = u.scalar_type();
    const int code = dtype_code(dt);
    check(u, "u", dt, {d.B, d.L, c.G, d.H});
    check(params, "params", at::kFloat);
    check(h, "h", dt, {d.B, d.L, c.S, d.H});
    check(g, "dL_dh", dt, {d.B, d.L, c.S, d.H});
    if (has(h0)) check(*h0, "h0", dt, {d.B, c.S, d.H});
    Grads r;
    if (out) {
        r = *out;
        check(r.du, "dL_du", dt, u.sizes());
        check(r.dparams, "dL_dparams", at::kFloat, params.sizes());
        if (r.dh0.defined()) check(r.dh0, "dL_dh0", dt, {d.B, c.S, d.H});
    } else {
        r.du = at::empty(u.sizes(), u.options());
        r.dparams = at::empty(params.sizes(), params.options());
        if (want_dh0) r.dh0 = at::empty({d.B, c.S, d.H}, u.options());
    }
    Workspace ws(c, true, code, d, 0, c.ws(code, d.B, d.L, d.H, 1), u, workspace, stream);
    const float *p = static_cast<const float *>(params.data_ptr());
    float *dp = static_cast<float *>(r.dparams.data_ptr());
    void *dh = r.dh0.defined() ? r.dh0.data_ptr() : nullptr;
    const int rc = c.number >= 0
                       ? pararnn_backward(c.number, code, p, u.data_ptr(), ptr(h0), h.data_ptr(), g.data_ptr(), d.B, d.L, d.H,
                                          r.du.data_ptr(), dp, dh, ws.data(), ws.size(), stream_ptr(stream))
                       : c.bwd_fn(code, p, u.data_ptr(), ptr(h0), h.data_ptr(), g.data_ptr(), d.B, d.L, d.H, r.du.data_ptr(),
                                  dp, dh, ws.data(), ws.size(), stream_ptr(stream));
    raise_if(rc, c.what + "_backward");
    ws.done();
    return r;
}

struct ProjDims { int B, L, H, G; };
ProjDims proj_dims(const Tensor &x, const Tensor &Wx, int64_t n_heads)
{
    if (x.dim() != 3) throw py::value_error("x must have three dimensions");
    if (Wx.dim() < 1) throw py::value_error("Wx must have three dimensions");
    const ProjDims d = {(int)x.size(0), (int)x.size(1), (int)x.size(2), (int)Wx.size(0)};
    check(x, "x", x.scalar_type(), {d.B, d.L, d.H});
    if (n_heads == 0) throw py::value_error("n_heads must be positive");
    check(Wx, "Wx", at::kFloat, {d.G, d.H, d.H / n_heads});
    return d;
}

Tensor project(const Tensor &x, const Tensor &Wx, const OptTensor &bias, int64_t n_heads, const OptTensor &workspace,
               const c10::optional<int64_t> &stream, const OptTensor &out)
{
    const ProjDims d = proj_dims(x, Wx, n_heads);
    const auto dt = x.scalar_type();
    const int code = dtype_code(dt);
    if (has(bias)) check(*bias, "bias", at::kFloat, {d.G, d.H});
    Tensor u = has(out) ? *out : at::empty({d.B, d.L, d.G, d.H}, x.options());
    check(u, "u", dt, {d.B, d.L, d.G, d.H});
    const Tensor ws = workspace_of(pararnn_input_projection_workspace_bytes(code, d.B, d.L, d.H, d.G, (int)n_heads, 0), x, workspace);
    raise_if(pararnn_input_projection(code, x.data_ptr(), static_cast<const float *>(Wx.data_ptr()),
                                      static_cast<const float *>(ptr(bias)), d.B, d.L, d.H, d.G, (int)n_heads, u.data_ptr(),
                                      ws.data_ptr(), (size_t)ws.numel(), stream_ptr(stream)),
             "pararnn_input_projection");
    return u;
}

struct ProjGrads { Tensor dx, dW, db; };

ProjGrads project_backward(const Tensor &x, const Tensor &Wx, const Tensor &du, int64_t n_heads, bool want_dx, bool want_dw,
                           bool want_db, const OptTensor &workspace, const c10::optional<int64_t> &stream)
{
    const ProjDims d = proj_dims(x, Wx, n_heads);
    const auto dt = x.scalar_type();
    const int code = dtype_code(dt);
    check(du, "du", dt, {d.B, d.L, d.G, d.H});
    ProjGrads r;
    if (want_dx) r.dx = at::empty(x.sizes(), x.options());
    if (want_dw) r.dW = at::empty(Wx.sizes(), Wx.options());
    if (want_db) r.db = at::empty({d.G, d.H}, Wx.options());
    const Tensor ws = workspace_of(pararnn_input_projection_workspace_bytes(code, d.B, d.L, d.H, d.G, (int)n_heads, 1), x, workspace);
    auto p = [](const Tensor &t) { return t.defined() ? t.data_ptr() : nullptr; };
    raise_if(pararnn_input_projection_backward(code, x.data_ptr(), static_cast<const float *>(Wx.data_ptr()), du.data_ptr(), d.B,
                                               d.L, d.H, d.G, (int)n_heads, p(r.dx), static_cast<float *>(p(r.dW)),
                                               static_cast<float *>(p(r.db)), ws.data_ptr(), (size_t)ws.numel(),
                                               stream_ptr(stream)),
             "pararnn_input_projection_backward");
    return r;
}

// ------------------------------------------------------------------ autograd
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

// Numbers the defined tensors among a function's inputs as the graph does.
struct Edges {
    AutogradContext *ctx;
    size_t next = 0;
    bool operator()(bool defined) { return defined && ctx->needs_input_grad(next++); }
};

Tensor or_none(const OptTensor &t) { return has(t) ? *t : Tensor(); }

// h = RNN(u): pararnn_forward with pararnn_backward as its gradient (Eq. (6)).
struct Recurrence : torch::autograd::Function<Recurrence> {
    static variable_list forward(AutogradContext *ctx, Tensor params, Tensor u, OptTensor h0, CellPtr cell, double tol, int64_t max_iter)
    {
        Solve s = solve(*cell, params, u, h0, tol, max_iter, false, {}, {}, {});
        ctx->save_for_backward({params, u, or_none(h0), s.h});
        ctx->saved_data["cell"] = c10::IValue::make_capsule(cell);
        ctx->mark_non_differentiable({s.iters});
        ctx->set_materialize_grads(false);
        return {s.h, s.iters};
    }
    static variable_list backward(AutogradContext *ctx, variable_list grads)
    {
        variable_list out(6);
        if (!grads[0].defined()) return out;
        const auto v = ctx->get_saved_variables();
        const auto cell = c10::static_intrusive_pointer_cast<Cell>(ctx->saved_data["cell"].toCapsule());
        Edges need{ctx};
        need(true); need(true);
        Grads g = adjoint(*cell, v[0], v[1], v[2], v[3], grads[0].contiguous(), need(v[2].defined()), {}, {}, nullptr);
        out[0] = g.dparams; out[1] = g.du; out[2] = g.dh0;
        return out;
    }
};

// u = B x + b for all gates
struct Projection : torch::autograd::Function<Projection> {
    static variable_list forward(AutogradContext *ctx, Tensor x, Tensor Wx, OptTensor bias, int64_t n_heads)
    {
        Tensor u = project(x, Wx, bias, n_heads, {}, {}, {});
        ctx->save_for_backward({x, Wx});
        ctx->saved_data["n_heads"] = n_heads;
        ctx->saved_data["bias"] = has(bias);
        ctx->set_materialize_grads(false);
        return {u};
    }
    static variable_list backward(AutogradContext *ctx, variable_list grads)
    {
        variable_list out(4);
        if (!grads[0].defined()) return out;
        const auto v = ctx->get_saved_variables();
        Edges need{ctx};
        const bool nx = need(true), nw = need(true), nb = need(ctx->saved_data["bias"].toBool());
        ProjGrads g = project_backward(v[0], v[1], grads[0].contiguous(), ctx->saved_data["n_heads"].toInt(), nx, nw || nb, nb, {}, {});
        out[0] = g.dx;
        if (nw) out[1] = g.dW;
        out[2] = g.db;
        return out;
    }
};

// The projection followed by the recurrence, as one node.
struct Layer : torch::autograd::Function<Layer> {
    static variable_list forward(AutogradContext *ctx, Tensor x, Tensor Wx, OptTensor bias, Tensor params, OptTensor h0, CellPtr cell,
                                 int64_t n_heads, double tol, int64_t max_iter)
    {
        Tensor u = project(x, Wx, bias, n_heads, {}, {}, {});
        Solve s = solve(*cell, params, u, h0, tol, max_iter, false, {}, {}, {});
        ctx->save_for_backward({x, Wx, params, or_none(h0), u, s.h});
        ctx->saved_data["cell"] = c10::IValue::make_capsule(cell);
        ctx->saved_data["n_heads"] = n_heads;
        ctx->saved_data["bias"] = has(bias);
        ctx->mark_non_differentiable({s.iters});
        ctx->set_materialize_grads(false);
        return {s.h, s.iters};
    }
    static variable_list backward(AutogradContext *ctx, variable_list grads)
    {
        variable_list out(9);
        if (!grads[0].defined()) return out;
        const auto v = ctx->get_saved_variables();
        const auto cell = c10::static_intrusive_pointer_cast<Cell>(ctx->saved_data["cell"].toCapsule());
        Edges need{ctx};
        const bool nx = need(true), nw = need(true), nb = need(ctx->saved_data["bias"].toBool());
        need(true);
        Grads g = adjoint(*cell, v[2], v[4], v[3], v[5], grads[0].contiguous(), need(v[3].defined()), {}, {}, nullptr);
        out[3] = g.dparams;
        out[4] = g.dh0;
        if (nx || nw || nb) {
            ProjGrads p = project_backward(v[0], v[1], g.du, ctx->saved_data["n_heads"].toInt(), nx, nw || nb, nb, {}, {});
            out[0] = p.dx;
            if (nw) out[1] = p.dW;
            out[2] = p.db;
        }
        return out;
    }
};

// Runs a call into the library without the interpreter lock: it may allocate, and wait for a place in a full launch queue.
template <class F> auto unlocked(F &&f)
{
    const py::gil_scoped_release unlock;
    return f();
}

py::object object_of(const Tensor &t) { return t.defined() ? py::cast(t) : py::none(); }

}  // namespace

namespace c10 {
C10_REGISTER_CLASS(FreeHipMemoryCallbacksRegistry, pararnn_kept_workspaces, GiveBack)
}

PYBIND11_MODULE(_host, m)
{
    py::class_<Cell, CellPtr>(m, "Cell");
    m.def("builtin_cell", [](int number, std::string what) {
        auto c = c10::make_intrusive<Cell>();
        c->number = number;
        c->G = pararnn_cell_gates(number);
        c->S = pararnn_cell_state(number);
        c->what = std::move(what);
        return c;
    });
    m.def("library_cell", [](std::string what, int G, int S, size_t ws, size_t ws_fused, size_t fwd, size_t bwd, size_t parts) {
        auto c = c10::make_intrusive<Cell>();
        c->G = G;
        c->S = S;
        c->what = std::move(what);
        c->ws_fn = reinterpret_cast<Cell::Ws>(ws);
        c->ws_fused_fn = reinterpret_cast<Cell::Ws>(ws_fused);
        c->fwd_fn = reinterpret_cast<Cell::Fwd>(fwd);
        c->bwd_fn = reinterpret_cast<Cell::Bwd>(bwd);
        c->parts_fn = reinterpret_cast<Cell::Parts>(parts);
        return c;
    }, py::arg("what"), py::arg("G"), py::arg("S"), py::arg("ws"), py::arg("ws_fused"), py::arg("fwd"), py::arg("bwd"), py::arg("parts") = 0);
    m.def("forward", [](const CellPtr &c, const Tensor &params, const Tensor &u, const OptTensor &h0, double tol, int64_t max_iter,
                        bool trace, const OptTensor &workspace, const c10::optional<int64_t> &stream, const OptTensor &out) {
        Solve s = unlocked([&] { return solve(*c, params, u, h0, tol, max_iter, trace, workspace, stream, out); });
        return py::make_tuple(s.h, s.iters, object_of(s.trace));
    });
    m.def("backward", [](const CellPtr &c, const Tensor &params, const Tensor &u, const OptTensor &h0, const Tensor &h, const Tensor &g,
                         bool want_dh0, const OptTensor &workspace, const c10::optional<int64_t> &stream, const OptTensor &du,
                         const OptTensor &dparams, const OptTensor &dh0) {
        Grads given;
        if (has(du)) given = {*du, or_none(dparams), or_none(dh0)};
        Grads r = unlocked([&] { return adjoint(*c, params, u, h0, h, g, want_dh0, workspace, stream, has(du) ? &given : nullptr); });
        return py::make_tuple(r.du, r.dparams, object_of(r.dh0));
    });
    m.def("input_projection", [](const Tensor &x, const Tensor &Wx, const OptTensor &bias, int64_t n_heads, const OptTensor &workspace,
                                 const c10::optional<int64_t> &stream, const OptTensor &out) {
        return unlocked([&] { return project(x, Wx, bias, n_heads, workspace, stream, out); });
    });
    m.def("input_projection_backward", [](const Tensor &x, const Tensor &Wx, const Tensor &du, int64_t n_heads, bool want_dx,
                                          bool want_dw, bool want_db, const OptTensor &workspace,
                                          const c10::optional<int64_t> &stream) {
        ProjGrads r = unlocked([&] { return project_backward(x, Wx, du, n_heads, want_dx, want_dw, want_db, workspace, stream); });
        return py::make_tuple(object_of(r.dx), object_of(r.dW), object_of(r.db));
    });
    m.def("release_workspaces", &release_workspaces, py::call_guard<py::gil_scoped_release>());
    m.def("rnn_apply", [](const CellPtr &c, const Tensor &params, const Tensor &u, const OptTensor &h0, double tol, int64_t max_iter) {
        variable_list r = unlocked([&] { return Recurrence::apply(params, u, h0, c, tol, max_iter); });
        return py::make_tuple(r[0], r[1]);
    });
    m.def("input_projection_apply", [](const Tensor &x, const Tensor &Wx, const OptTensor &bias, int64_t n_heads) {
        return unlocked([&] { return Projection::apply(x, Wx, bias, n_heads)[0]; });
    });
    m.def("rnn_layer", [](const CellPtr &c, const Tensor &x, const Tensor &Wx, const OptTensor &bias, const Tensor &params,
                          const OptTensor &h0, int64_t n_heads, double tol, int64_t max_iter) {
        variable_list r = unlocked([&] { return Layer::apply(x, Wx, bias, params, h0, c, n_heads, tol, max_iter); });
        return py::make_tuple(r[0], r[1]);
    });
}
