// Autograd nodes of the library's kernels in C++: the same calls as the Python Functions of autograd.py,
// without the interpreter between the launches.
//
// A small call is bound by the host: one forward and backward of a 1024-ray coarse render keeps the GPU
// busy for about 40 us, while the Python Functions took 170 us to issue it, half of that in the engine's
// thread (taking over the interpreter lock, building the argument structs); with these nodes 78 us, and a
// colour head on 2,160 samples 222 -> 107 us.  Every entry point here checks
// what the Python path checks and returns None where a check or the library refuses the call, so that the
// Python path then raises its own error for it; it never launches in that case.
#include <torch/extension.h>
#include <torch/csrc/Exceptions.h>

#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>

#include <array>
#include <optional>
#include <string>
#include <vector>

#include "dvgo.h"

namespace {

using at::Tensor;
using torch::autograd::AutogradContext;
using torch::autograd::variable_list;
using Vec3 = std::array<double, 3>;

void *stream() { return (void *)c10::hip::getCurrentHIPStreamMasqueradingAsCUDA().stream(); }

// a dense float32 (or int32) array on the GPU, as the library's pointers need it
bool fits(const Tensor &t, at::ScalarType dt = at::kFloat) {
    return t.defined() && t.is_cuda() && t.layout() == at::kStrided && t.scalar_type() == dt && t.is_contiguous();
}
bool fits(const Tensor &t, int64_t numel, at::ScalarType dt = at::kFloat) { return fits(t, dt) && t.numel() == numel; }

std::string dtype_of(const Tensor &t) {
    pybind11::gil_scoped_acquire gil;
    return pybind11::str(pybind11::cast(t).attr("dtype"));
}

// The checks of a backward on what it hands to the library, with the Python path's errors.  A tensor that
// comes back from a saved-tensor hook has the values, the sizes, the type and the device of the one that
// went in, if the hook keeps to its contract, but not its strides; and not every hook keeps to it.
void expect(const Tensor &t, const char *name, at::ScalarType dt = at::kFloat) {
    TORCH_CHECK_VALUE(t.defined() && t.is_cuda(), name, " must live on the GPU (libdvgo has no CPU path)");
    TORCH_CHECK_TYPE(t.scalar_type() == dt, name, " must be ",
                     dt == at::kFloat ? "torch.float32" : (dt == at::kInt ? "torch.int32" : "torch.uint8"), ", got ", dtype_of(t));
    TORCH_CHECK_VALUE(t.layout() == at::kStrided && t.has_storage() && t.is_contiguous(), name, " must be contiguous");
}
void expect(const Tensor &t, const char *name, int64_t numel, at::ScalarType dt = at::kFloat) {
    expect(t, name, dt);
    TORCH_CHECK_VALUE(t.numel() == numel, name, " has ", t.numel(), " elements, expected ", numel);
}
void expect_grid(const Tensor &t) {
    expect(t, "grid data");
    TORCH_CHECK_VALUE(t.dim() == 4, "grid data must be [nx, ny, nz, ch_stride]");
}

// the library said no although the forward had gone through: the binding's DvgoError, with its code
void check(int rc, const char *fn) {
    if (rc == DVGO_OK) return;
    const std::string detail = dvgo_last_error();
    pybind11::gil_scoped_acquire gil;
    const pybind11::object type = pybind11::module_::import("paper_2206_05085_amd._lib").attr("DvgoError");
    PyErr_SetObject(type.ptr(), type(fn, rc, detail).ptr());
    python_error e;
    e.persist();
    throw e;
}

Tensor floats(at::IntArrayRef shape, const Tensor &like) { return at::empty(shape, like.options().dtype(at::kFloat)); }
Tensor bytes(size_t n, const Tensor &like) { return at::empty({(int64_t)n}, like.options().dtype(at::kByte)); }
float *f(const Tensor &t) { return t.defined() ? t.data_ptr<float>() : nullptr; }

dvgo_grid grid_of(const Tensor &data, const Vec3 &lo, const Vec3 &hi, int channels, const Tensor &grad = Tensor()) {
    dvgo_grid g{};
    g.struct_size = sizeof(g);
    g.nx = (int32_t)data.size(0);
    g.ny = (int32_t)data.size(1);
    g.nz = (int32_t)data.size(2);
    g.ch_stride = (int32_t)data.size(3);
    g.channels = channels > 0 ? channels : g.ch_stride;
    for (int a = 0; a < 3; ++a) {
        g.xyz_min[a] = (float)lo[a];
        g.xyz_max[a] = (float)hi[a];
    }
    g.data = f(data);
    g.grad = f(grad);
    g.warp = DVGO_WARP_NONE;
    g.warp_b = 1.f;
    return g;
}
bool grid_fits(const Tensor &t) {
    return fits(t) && t.dim() == 4 && t.size(0) < INT32_MAX && t.size(1) < INT32_MAX && t.size(2) < INT32_MAX &&
           t.size(3) < INT32_MAX;
}

// ------------------------------------------------------------------------------ render

struct RenderCall : torch::CustomClassHolder {
    Tensor offs, xyz, delta, s_mid, s_len;
    int64_t n_rays, n_samples;
    Vec3 lo, hi;
    bool grid_color, want_dist;
    double act_shift, halt_T;
    Vec3 bg;
    bool refused = false;  // the forward found that the library does not take the call

    void expect_samples() const {
        expect(offs, "ray_offsets", n_rays + 1, at::kInt);
        expect(xyz, "xyz", 3 * n_samples);
        expect(delta, "delta", n_samples);
        expect(s_mid, "s_mid", n_samples);
        expect(s_len, "s_len", n_samples);
    }
    dvgo_samples samples() const {
        return {sizeof(dvgo_samples), (int32_t)n_rays, n_samples, offs.data_ptr<int32_t>(), f(xyz), f(delta), f(s_mid), f(s_len)};
    }
    dvgo_render_params params() const {
        dvgo_render_params p{};
        p.struct_size = sizeof(p);
        p.act_shift = (float)act_shift;
        p.halt_T = (float)halt_T;
        for (int a = 0; a < 3; ++a) p.bg[a] = (float)bg[a];
        p.color_mode = grid_color ? DVGO_COLOR_GRID : DVGO_COLOR_SAMPLES;
        p.want_dist = want_dist;
        return p;
    }
};
using RenderPtr = c10::intrusive_ptr<RenderCall>;

struct RenderNode : torch::autograd::Function<RenderNode> {
    static variable_list forward(AutogradContext *ctx, const Tensor &density, const Tensor &colour, const RenderPtr &c) {
        const Tensor rgb = floats({c->n_rays, 3}, c->xyz), T = floats({c->n_rays}, c->xyz), dist = floats({c->n_rays}, c->xyz);
        size_t need = 0;
        int rc = dvgo_render_state_size((int32_t)c->n_rays, c->n_samples, &need);
        const Tensor state = bytes(need, c->xyz);
        const dvgo_samples s = c->samples();
        const dvgo_render_params p = c->params();
        const dvgo_grid gd = grid_of(density, c->lo, c->hi, 0);
        dvgo_grid gc{};
        if (c->grid_color) gc = grid_of(colour, c->lo, c->hi, 3);
        if (rc == DVGO_OK)
            rc = dvgo_render_forward(&p, &s, &gd, c->grid_color ? &gc : nullptr, c->grid_color ? nullptr : f(colour), f(rgb),
                                     f(T), c->want_dist ? f(dist) : nullptr, nullptr, state.data_ptr(), need, stream());
        c->refused = rc != DVGO_OK;
        if (!c->want_dist && !c->refused) dist.zero_();
        ctx->set_materialize_grads(false);  // three outputs: the backward knows what to leave out
        ctx->save_for_backward({density, colour, T, state});
        ctx->saved_data["call"] = c10::IValue::make_capsule(c);
        return {rgb, T, dist};
    }

    static variable_list backward(AutogradContext *ctx, variable_list g) {
        const auto saved = ctx->get_saved_variables();
        const Tensor &density = saved[0], &colour = saved[1], &T = saved[2], &state = saved[3];
        const auto c = c10::static_intrusive_pointer_cast<RenderCall>(ctx->saved_data["call"].toCapsule());
        c->expect_samples();
        expect_grid(density);
        if (c->grid_color) expect_grid(colour);
        else expect(colour, "sample_rgb", 3 * c->n_samples);
        expect(T, "T_final", c->n_rays);
        expect(state, "state", at::kByte);
        const Tensor g_rgb = g[0].defined() ? g[0].contiguous() : at::zeros({c->n_rays, 3}, T.options());
        const Tensor g_T = g[1].defined() ? g[1].contiguous() : Tensor();
        const Tensor g_dist = g[2].defined() && c->want_dist ? g[2].contiguous() : Tensor();
        const Tensor gden = at::zeros_like(density);
        const Tensor gcol = c->grid_color ? at::zeros_like(colour) : floats({c->n_samples, 3}, c->xyz);
        const dvgo_samples s = c->samples();
        const dvgo_render_params p = c->params();
        const dvgo_grid gd = grid_of(density, c->lo, c->hi, 0, gden);
        dvgo_grid gc{};
        if (c->grid_color) gc = grid_of(colour, c->lo, c->hi, 3, gcol);
        check(dvgo_render_backward(&p, &s, &gd, c->grid_color ? &gc : nullptr, c->grid_color ? nullptr : f(colour), f(T),
                                   state.data_ptr(), (size_t)state.numel(), f(g_rgb), f(g_dist), f(g_T),
                                   c->grid_color ? nullptr : f(gcol), nullptr, stream()),
              "dvgo_render_backward");
        return {gden, gcol, Tensor()};
    }
};

std::optional<variable_list> render(const Tensor &density, const Tensor &colour, const Tensor &offs, const Tensor &xyz,
                                    const Tensor &delta, const Tensor &s_mid, const Tensor &s_len, int64_t n_rays,
                                    int64_t n_samples, const Vec3 &lo, const Vec3 &hi, bool grid_color, double act_shift,
                                    double halt_T, const Vec3 &bg, bool want_dist) {
    if (n_rays < 0 || n_rays >= INT32_MAX || n_samples < 0 || !fits(offs, n_rays + 1, at::kInt) || !fits(xyz, 3 * n_samples) ||
        !fits(delta, n_samples) || !fits(s_mid, n_samples) || !fits(s_len, n_samples) || !grid_fits(density) ||
        !(grid_color ? grid_fits(colour) : fits(colour, 3 * n_samples)) || (!grid_color && colour.dim() != 2))
        return std::nullopt;
    auto c = c10::make_intrusive<RenderCall>();
    c->offs = offs;
    c->xyz = xyz;
    c->delta = delta;
    c->s_mid = s_mid;
    c->s_len = s_len;
    c->n_rays = n_rays;
    c->n_samples = n_samples;
    c->lo = lo;
    c->hi = hi;
    c->grid_color = grid_color;
    c->want_dist = want_dist;
    c->act_shift = act_shift;
    c->halt_T = halt_T;
    c->bg = bg;
    auto out = RenderNode::apply(density, colour, c);
    if (c->refused) return std::nullopt;
    return out;
}

// -------------------------------------------------------------------------- distortion

struct DistortionNode : torch::autograd::Function<DistortionNode> {
    static Tensor forward(AutogradContext *ctx, const Tensor &w, const Tensor &offs, const Tensor &sm, const Tensor &sl,
                          bool *refused) {
        const Tensor wc = w.contiguous(), loss = floats({offs.numel() - 1}, w);
        *refused = dvgo_distortion_loss((int32_t)(offs.numel() - 1), offs.data_ptr<int32_t>(), wc.numel(), f(wc), f(sm), f(sl),
                                        f(loss), nullptr, nullptr, nullptr, 0, stream()) != DVGO_OK;
        ctx->save_for_backward({w, offs, sm, sl});
        return loss;
    }
    static variable_list backward(AutogradContext *ctx, variable_list g) {
        const auto saved = ctx->get_saved_variables();
        const Tensor w = saved[0].contiguous(), &offs = saved[1], &sm = saved[2], &sl = saved[3];
        expect(offs, "ray_offsets", at::kInt);
        expect(w, "w");
        expect(sm, "s_mid", w.numel());
        expect(sl, "s_len", w.numel());
        const int32_t R = (int32_t)(offs.numel() - 1);
        size_t need = 0;
        check(dvgo_distortion_workspace_size(R, w.numel(), &need), "dvgo_distortion_workspace_size");
        const Tensor gl = g[0].contiguous(), loss = floats({R}, w), gw = at::zeros({w.numel()}, w.options()), ws = bytes(need, w);
        check(dvgo_distortion_loss(R, offs.data_ptr<int32_t>(), w.numel(), f(w), f(sm), f(sl), f(loss), f(gl), f(gw),
                                   ws.data_ptr(), need, stream()),
              "dvgo_distortion_loss");
        return {gw, Tensor(), Tensor(), Tensor(), Tensor()};
    }
};

std::optional<Tensor> distortion(const Tensor &w, const Tensor &offs, const Tensor &sm, const Tensor &sl) {
    if (!fits(offs, at::kInt) || offs.numel() < 1 || offs.numel() > INT32_MAX || !fits(w) || w.dim() != 1 || !fits(sm, w.numel()) ||
        !fits(sl, w.numel()))
        return std::nullopt;
    bool refused = false;
    const Tensor loss = DistortionNode::apply(w, offs, sm, sl, &refused);
    if (refused) return std::nullopt;
    return loss;
}

// ------------------------------------------------------------------------------ gather

struct BoxCall : torch::CustomClassHolder {
    Vec3 lo, hi;
    bool refused = false;
};
using BoxPtr = c10::intrusive_ptr<BoxCall>;

struct GatherNode : torch::autograd::Function<GatherNode> {
    static Tensor forward(AutogradContext *ctx, const Tensor &grid, const Tensor &xyz, const BoxPtr &c) {
        const int64_t S = xyz.numel() / 3;
        const Tensor out = floats({S, grid.size(3)}, xyz);
        const dvgo_grid g = grid_of(grid, c->lo, c->hi, 0);
        c->refused = dvgo_grid_gather(&g, S, f(xyz), f(out), stream()) != DVGO_OK;
        ctx->save_for_backward({grid, xyz});
        ctx->saved_data["call"] = c10::IValue::make_capsule(c);
        return out;
    }
    static variable_list backward(AutogradContext *ctx, variable_list g) {
        const auto saved = ctx->get_saved_variables();
        const Tensor &grid = saved[0], &xyz = saved[1];
        const auto c = c10::static_intrusive_pointer_cast<BoxCall>(ctx->saved_data["call"].toCapsule());
        expect_grid(grid);
        expect(xyz, "xyz", g[0].size(0) * 3);
        const Tensor gg = at::zeros_like(grid), go = g[0].contiguous();
        const dvgo_grid dg = grid_of(grid, c->lo, c->hi, 0, gg);
        check(dvgo_grid_scatter(&dg, xyz.numel() / 3, f(xyz), f(go), stream()), "dvgo_grid_scatter");
        return {gg, Tensor(), Tensor()};
    }
};

std::optional<Tensor> gather(const Tensor &grid, const Tensor &xyz, const Vec3 &lo, const Vec3 &hi) {
    if (!grid_fits(grid) || !fits(xyz) || xyz.numel() % 3) return std::nullopt;
    auto c = c10::make_intrusive<BoxCall>();
    c->lo = lo;
    c->hi = hi;
    const Tensor out = GatherNode::apply(grid, xyz, c);
    if (c->refused) return std::nullopt;
    return out;
}

// --------------------------------------------------------------------------- colour head

dvgo_color_mlp head_of(const Tensor &feat, const Tensor *W, const Tensor *b, int64_t n_freq, const Tensor *gW = nullptr,
                       const Tensor *gb = nullptr) {
    dvgo_color_mlp m{};
    m.struct_size = sizeof(m);
    m.in_feat = (int32_t)feat.size(1);
    m.n_freq = (int32_t)n_freq;
    m.hidden = (int32_t)W[1].size(0);
    m.W1 = f(W[0]);
    m.W2 = f(W[1]);
    m.W3 = f(W[2]);
    m.b1 = f(b[0]);
    m.b2 = f(b[1]);
    m.b3 = f(b[2]);
    if (gW) {
        m.gW1 = f(gW[0]);
        m.gW2 = f(gW[1]);
        m.gW3 = f(gW[2]);
        m.gb1 = f(gb[0]);
        m.gb2 = f(gb[1]);
        m.gb3 = f(gb[2]);
    }
    m.precision = DVGO_MLP_SPLIT_F16;
    return m;
}

struct HeadCall : torch::CustomClassHolder {
    int64_t n_freq;
    bool refused = false;
};
using HeadPtr = c10::intrusive_ptr<HeadCall>;

struct HeadNode : torch::autograd::Function<HeadNode> {
    static Tensor forward(AutogradContext *ctx, const Tensor &feat, const Tensor &W1, const Tensor &b1, const Tensor &W2,
                          const Tensor &b2, const Tensor &W3, const Tensor &b3, const Tensor &offs, const Tensor &dirs,
                          const HeadPtr &c) {
        const Tensor W[3] = {W1, W2, W3}, b[3] = {b1, b2, b3};
        const int32_t R = (int32_t)(offs.numel() - 1);
        const int64_t S = feat.size(0);
        const dvgo_color_mlp m = head_of(feat, W, b, c->n_freq);
        const Tensor rgb = floats({S, 3}, feat);
        size_t need = 0;
        int rc = dvgo_mlp_workspace_size(&m, R, S, &need);
        if (rc == DVGO_OK) {
            const Tensor ws = bytes(need, feat);
            rc = dvgo_mlp_forward(&m, R, offs.data_ptr<int32_t>(), f(dirs), S, f(feat), f(rgb), ws.data_ptr(), need, stream());
        }
        c->refused = rc != DVGO_OK;
        ctx->save_for_backward({feat, W1, b1, W2, b2, W3, b3, offs, dirs});
        ctx->saved_data["call"] = c10::IValue::make_capsule(c);
        return rgb;
    }
    static variable_list backward(AutogradContext *ctx, variable_list g) {
        const auto v = ctx->get_saved_variables();
        const auto c = c10::static_intrusive_pointer_cast<HeadCall>(ctx->saved_data["call"].toCapsule());
        const Tensor &feat = v[0], &offs = v[7], &dirs = v[8];
        const Tensor W[3] = {v[1], v[3], v[5]}, b[3] = {v[2], v[4], v[6]};
        for (int i = 0; i < 3; ++i) {
            expect(W[i], ("W" + std::to_string(i + 1)).c_str());
            expect(b[i], ("b" + std::to_string(i + 1)).c_str());
        }
        expect(feat, "feat");
        expect(offs, "ray_offsets", at::kInt);
        expect(dirs, "dirs", 3 * (offs.numel() - 1));
        Tensor gW[3], gb[3];
        std::vector<Tensor> all;
        for (int i = 0; i < 3; ++i) {
            all.push_back(gW[i] = at::empty_like(W[i]));
            all.push_back(gb[i] = at::empty_like(b[i]));
        }
        at::_foreach_zero_(all);  // one launch for the six
        const int32_t R = (int32_t)(offs.numel() - 1);
        const int64_t S = feat.size(0);
        const dvgo_color_mlp m = head_of(feat, W, b, c->n_freq, gW, gb);
        const Tensor go = g[0].contiguous(), gf = floats({S, feat.size(1)}, feat);
        size_t need = 0;
        check(dvgo_mlp_workspace_size(&m, R, S, &need), "dvgo_mlp_workspace_size");
        const Tensor ws = bytes(need, feat);
        check(dvgo_mlp_backward(&m, R, offs.data_ptr<int32_t>(), f(dirs), S, f(feat), f(go), f(gf), ws.data_ptr(), need, stream()),
              "dvgo_mlp_backward");
        return {gf, gW[0], gb[0], gW[1], gb[1], gW[2], gb[2], Tensor(), Tensor(), Tensor()};
    }
};

std::optional<Tensor> color_mlp(const Tensor &feat, const std::array<Tensor, 3> &W, const std::array<Tensor, 3> &b,
                                const Tensor &offs, const Tensor &dirs, int64_t n_freq) {
    if (!fits(feat) || feat.dim() != 2 || feat.size(1) >= INT32_MAX || n_freq < 0 || n_freq >= INT32_MAX || !fits(offs, at::kInt) ||
        offs.numel() < 1 || offs.numel() > INT32_MAX || !fits(dirs, 3 * (offs.numel() - 1)))
        return std::nullopt;
    for (int i = 0; i < 3; ++i)
        if (!fits(W[i]) || !fits(b[i]) || W[i].dim() < 1 || W[i].size(0) >= INT32_MAX) return std::nullopt;
    auto c = c10::make_intrusive<HeadCall>();
    c->n_freq = n_freq;
    const Tensor rgb = HeadNode::apply(feat, W[0], b[0], W[1], b[1], W[2], b[2], offs, dirs, c);
    if (c->refused) return std::nullopt;
    return rgb;
}

}  // namespace

PYBIND11_MODULE(TORCH_EXTENSION_NAME, m) {
    TORCH_CHECK(dvgo_abi_version() == DVGO_ABI_VERSION, "libdvgo ABI version does not match this module's");
    // other Python threads run meanwhile, as in the ctypes calls
    const auto free_gil = pybind11::call_guard<pybind11::gil_scoped_release>();
    m.def("render", &render, free_gil);
    m.def("distortion", &distortion, free_gil);
    m.def("gather", &gather, free_gil);
    m.def("color_mlp", &color_mlp, free_gil);
}
