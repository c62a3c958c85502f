// Host side of the emulator calls declared in include/emu.h: workspace
// carving, the layer sequence of the forward and backward passes, and Adam's
// step bookkeeping.  Every arithmetic step runs in the kernels of
// emu_kernels.hip.
#include <cmath>
#include <cstring>
#include <new>
#include <string>

#include "../../include/emu.h"
#include "cpm_internal.hpp"
#include "emu_internal.hpp"

using namespace cpm::emu;

namespace {

constexpr int kMaxBatch = 1 << 20;

size_t align_up(size_t v) { return (v + 255) & ~(size_t)255; }

int64_t pad_rows(int64_t n) { return (n + kRows - 1) / kRows * kRows; }

struct EmuLayout {
    size_t params, grad, m, v, norm, loss;
    size_t w[kLayers], wt[kLayers];  // bf16 operand copies of the weights
    size_t work;                     // end of what starts at zero
    size_t in_t[kLayers], dz_t[kLayers], loss_part, part;
    size_t total;
};

EmuLayout layout_for(int64_t max_batch)
{
    const int64_t np = pad_rows(max_batch);
    const int64_t splits = (np + kSplitK - 1) / kSplitK;
    EmuLayout l{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = align_up(off + bytes);
        return at;
    };
    l.params = take(kParams * 4);
    l.grad = take(kParams * 4);
    l.m = take(kParams * 4);
    l.v = take(kParams * 4);
    l.norm = take(EMU_NORM * 4);
    l.loss = take(4);
    const size_t in_pad[kLayers] = {kInPad, kHidden, kHidden, kHidden};
    const size_t out_rows[kLayers] = {kHidden, kHidden, kHidden, kTile};
    for (int i = 0; i < kLayers; ++i) l.w[i] = take(out_rows[i] * in_pad[i] * 2);
    for (int i = 1; i < kLayers; ++i) l.wt[i] = take((size_t)kHidden * (i == 3 ? kOutPad : kHidden) * 2);
    l.work = off;
    for (int i = 0; i < kLayers; ++i) {
        l.in_t[i] = take((size_t)(i == 0 ? kTile : kHidden) * np * 2);
        l.dz_t[i] = take((size_t)(i == 3 ? kTile : kHidden) * np * 2);
    }
    l.loss_part = take(np * 4);
    l.part = take(splits > 1 ? (size_t)splits * kParams * 4 : 0);
    l.total = off;
    return l;
}

int fail(int code, const std::string &msg) { return cpm::report_error(code, msg.c_str()); }

int device_fail(hipError_t e, const char *where)
{
    return fail(CPM_EDEVICE, std::string(where) + ": " + hipGetErrorString(e));
}

hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

}  // namespace

struct emu_handle {
    int32_t max_batch = 0;
    int64_t steps = 0;
    char *base = nullptr;
    EmuLayout l{};
    template <typename T> T *at(size_t off) const { return reinterpret_cast<T *>(base + off); }
    float *params() const { return at<float>(l.params); }
    float *grad() const { return at<float>(l.grad); }
    float *norm() const { return at<float>(l.norm); }
};

namespace {

Copies copies(const emu_handle *h)
{
    Copies c{};
    for (int i = 0; i < kLayers; ++i) {
        c.w[i] = h->at<uint16_t>(h->l.w[i]);
        c.wt[i] = i ? h->at<uint16_t>(h->l.wt[i]) : nullptr;
    }
    return c;
}

// Adam's arguments for step t (1 based).
AdamArgs adam_args(const emu_handle *h, float lr, int64_t t)
{
    AdamArgs a{};
    a.param = h->params();
    a.m = h->at<float>(h->l.m);
    a.v = h->at<float>(h->l.v);
    a.lr = lr;
    a.beta1 = 0.9f;
    a.beta2 = 0.999f;
    a.one_minus_beta1 = 0.1f;
    a.one_minus_beta2 = 0.001f;
    a.eps = 1e-8f;
    a.c1 = (float)(1.0 - std::pow(0.9, (double)t));
    a.c2 = (float)(1.0 - std::pow(0.999, (double)t));
    a.c = copies(h);
    return a;
}

int check_batch(const emu_handle *h, int32_t n)
{
    if (!h) return fail(CPM_EINVAL, "null handle");
    if (n < 1 || n > h->max_batch)
        return fail(CPM_EINVAL, "batch of " + std::to_string(n) + " points outside [1, " +
                                    std::to_string(h->max_batch) + "]");
    return CPM_OK;
}

RowArgs row_args(const emu_handle *h, const float *d_x, int n)
{
    RowArgs r{};
    r.x = d_x;
    r.norm = h->norm();
    r.params = h->params();
    r.c = copies(h);
    r.n = n;
    r.n_pad = (int)pad_rows(n);
    return r;
}

// Gradient of the loss over n points into the gradient buffer, the loss, the
// caller's copies of them (nullable), and (adam not NULL) the step with it.
hipError_t gradients(emu_handle *h, const float *d_x, const float *d_targets, int n, float *d_grad, float *d_loss,
                     const AdamArgs *adam, hipStream_t st)
{
    RowArgs r = row_args(h, d_x, n);
    r.targets = d_targets;
    GradArgs g{};
    for (int i = 0; i < kLayers; ++i) {
        g.in_t[i] = r.in_t[i] = h->at<uint16_t>(h->l.in_t[i]);
        g.dz_t[i] = r.dz_t[i] = h->at<uint16_t>(h->l.dz_t[i]);
    }
    g.loss_part = r.loss_part = h->at<float>(h->l.loss_part);
    const hipError_t e = launch_rows(r, true, &g.loss_parts, st);
    if (e != hipSuccess) return e;
    g.n = n;
    g.n_pad = r.n_pad;
    g.splits = (g.n_pad + kSplitK - 1) / kSplitK;
    g.part = h->at<float>(h->l.part);
    g.grad = h->grad();
    g.loss = h->at<float>(h->l.loss);
    g.grad_out = d_grad;
    g.loss_out = d_loss;
    g.update = adam != nullptr;
    if (adam) g.adam = *adam;
    return launch_grads(g, st);
}

}  // namespace

extern "C" {

int emu_param_count(int64_t *count)
{
    if (!count) return fail(CPM_EINVAL, "null count");
    *count = kParams;
    return CPM_OK;
}

int emu_workspace_bytes(int32_t max_batch, size_t *bytes)
{
    if (!bytes) return fail(CPM_EINVAL, "null bytes");
    if (max_batch < 1 || max_batch > kMaxBatch) return fail(CPM_EINVAL, "max_batch outside [1, 2^20]");
    *bytes = layout_for(max_batch).total;
    return CPM_OK;
}

int emu_init(int32_t max_batch, void *d_workspace, size_t workspace_bytes, void *stream, emu_handle **out)
{
    if (!out || !d_workspace) return fail(CPM_EINVAL, "null pointer");
    *out = nullptr;
    if (max_batch < 1 || max_batch > kMaxBatch) return fail(CPM_EINVAL, "max_batch outside [1, 2^20]");
    if (reinterpret_cast<uintptr_t>(d_workspace) % 256 != 0) return fail(CPM_EINVAL, "workspace not 256-byte aligned");
    const EmuLayout l = layout_for(max_batch);
    if (workspace_bytes < l.total)
        return fail(CPM_ENOMEM, "workspace of " + std::to_string(workspace_bytes) + " bytes, need " +
                                    std::to_string(l.total));
    emu_handle *h = new (std::nothrow) emu_handle;
    if (!h) return fail(CPM_ENOMEM, "host allocation");
    h->max_batch = max_batch;
    h->base = static_cast<char *>(d_workspace);
    h->l = l;
    hipStream_t st = as_stream(stream);
    hipError_t e;
    // parameters, Adam state and every bf16 copy (with its zero padding) start at zero
    if ((e = launch_fill_f32(h->params(), 0.f, (int64_t)(l.work - l.params) / 4, st)) != hipSuccess) {
        delete h;
        return device_fail(e, "emu_init");
    }
    float *norm = h->norm();
    if ((e = launch_fill_f32(norm + kIn, 1.f, kIn, st)) != hipSuccess ||
        (e = launch_fill_f32(norm + 2 * kIn + kOut, 1.f, kOut, st)) != hipSuccess) {
        delete h;
        return device_fail(e, "emu_init");
    }
    *out = h;
    return CPM_OK;
}

int emu_set_params(emu_handle *h, const float *d_params, void *stream)
{
    if (!h || !d_params) return fail(CPM_EINVAL, "null pointer");
    hipStream_t st = as_stream(stream);
    hipError_t e = hipMemcpyAsync(h->params(), d_params, kParams * 4, hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess) e = launch_fill_f32(h->at<float>(h->l.m), 0.f, kParams, st);
    if (e == hipSuccess) e = launch_fill_f32(h->at<float>(h->l.v), 0.f, kParams, st);
    if (e == hipSuccess) e = launch_copies(copies(h), h->params(), st);
    if (e != hipSuccess) return device_fail(e, "emu_set_params");
    h->steps = 0;
    return CPM_OK;
}

int emu_get_params(emu_handle *h, float *d_params, void *stream)
{
    if (!h || !d_params) return fail(CPM_EINVAL, "null pointer");
    hipError_t e = hipMemcpyAsync(d_params, h->params(), kParams * 4, hipMemcpyDeviceToDevice, as_stream(stream));
    return e == hipSuccess ? CPM_OK : device_fail(e, "emu_get_params");
}

int emu_set_norm(emu_handle *h, const float *d_norm, void *stream)
{
    if (!h || !d_norm) return fail(CPM_EINVAL, "null pointer");
    hipError_t e = hipMemcpyAsync(h->norm(), d_norm, EMU_NORM * 4, hipMemcpyDeviceToDevice, as_stream(stream));
    return e == hipSuccess ? CPM_OK : device_fail(e, "emu_set_norm");
}

int emu_get_norm(emu_handle *h, float *d_norm, void *stream)
{
    if (!h || !d_norm) return fail(CPM_EINVAL, "null pointer");
    hipError_t e = hipMemcpyAsync(d_norm, h->norm(), EMU_NORM * 4, hipMemcpyDeviceToDevice, as_stream(stream));
    return e == hipSuccess ? CPM_OK : device_fail(e, "emu_get_norm");
}

int emu_fit_norm(emu_handle *h, const float *d_x, const float *d_targets, int32_t n, int32_t log_mask, void *stream)
{
    if (!h || !d_x || !d_targets) return fail(CPM_EINVAL, "null pointer");
    if (n < 1) return fail(CPM_EINVAL, "empty data set");
    if (log_mask < 0 || log_mask > 0xFF) return fail(CPM_EINVAL, "log_mask has bits beyond the 8 outputs");
    hipError_t e = launch_fit_norm(d_x, d_targets, n, log_mask, h->norm(), as_stream(stream));
    return e == hipSuccess ? CPM_OK : device_fail(e, "emu_fit_norm");
}

int emu_forward(emu_handle *h, const float *d_x, int32_t n, float *d_y, void *stream)
{
    int rc = check_batch(h, n);
    if (rc != CPM_OK) return rc;
    if (!d_x || !d_y) return fail(CPM_EINVAL, "null pointer");
    hipStream_t st = as_stream(stream);
    RowArgs r = row_args(h, d_x, n);
    r.y = d_y;
    const hipError_t e = launch_rows(r, false, nullptr, st);
    return e == hipSuccess ? CPM_OK : device_fail(e, "emu_forward");
}

int emu_grads(emu_handle *h, const float *d_x, const float *d_targets, int32_t n, float *d_grad, float *d_loss,
              void *stream)
{
    int rc = check_batch(h, n);
    if (rc != CPM_OK) return rc;
    if (!d_x || !d_targets) return fail(CPM_EINVAL, "null pointer");
    hipStream_t st = as_stream(stream);
    const hipError_t e = gradients(h, d_x, d_targets, n, d_grad, d_loss, nullptr, st);
    return e == hipSuccess ? CPM_OK : device_fail(e, "emu_grads");
}

int emu_adam(emu_handle *h, const float *d_grad, float lr, void *stream)
{
    if (!h) return fail(CPM_EINVAL, "null handle");
    if (!(lr > 0.f) || !std::isfinite(lr)) return fail(CPM_EINVAL, "learning rate must be positive and finite");
    const int64_t t = h->steps + 1;
    const hipError_t e = launch_adam(adam_args(h, lr, t), d_grad ? d_grad : h->grad(), as_stream(stream));
    if (e != hipSuccess) return device_fail(e, "emu_adam");
    h->steps = t;
    return CPM_OK;
}

int emu_train_step(emu_handle *h, const float *d_x, const float *d_targets, int32_t n, float lr, float *d_loss,
                   void *stream)
{
    if (!(lr > 0.f) || !std::isfinite(lr)) return fail(CPM_EINVAL, "learning rate must be positive and finite");
    int rc = check_batch(h, n);
    if (rc != CPM_OK) return rc;
    if (!d_x || !d_targets) return fail(CPM_EINVAL, "null pointer");
    hipStream_t st = as_stream(stream);
    const AdamArgs adam = adam_args(h, lr, h->steps + 1);
    const hipError_t e = gradients(h, d_x, d_targets, n, nullptr, d_loss, &adam, st);
    if (e != hipSuccess) return device_fail(e, "emu_train_step");
    h->steps += 1;
    return CPM_OK;
}

int emu_step_count(emu_handle *h, int64_t *steps)
{
    if (!h || !steps) return fail(CPM_EINVAL, "null pointer");
    *steps = h->steps;
    return CPM_OK;
}

int emu_destroy(emu_handle *h)
{
    delete h;
    return CPM_OK;
}

}  // extern "C"
