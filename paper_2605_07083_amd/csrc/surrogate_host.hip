// surrogate_host.hip -- host side of the surrogate C ABI (include/surrogate.h):
// workspace layout, weight packing, the forward pass into the caller's output
// (one launch) and the launch sequence of the training step (forward pass with
// the loss, one backward kernel per layer for the input and weight gradients,
// Adam with re-quantisation).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../../include/pic.h"
#include "../../include/surrogate.h"

extern "C" {
int surx_net_train_blocks(int X, int B);
hipError_t surx_net_train(const __bf16 *const *wf, const float *const *bias, const float *params, const float *target,
                          float *const *y, __bf16 *feat, __bf16 *dz, double *loss, int *blocks, int X, int B,
                          hipStream_t s);
hipError_t surx_conv_bwd(int layer, const __bf16 *dz, const float *yin, const __bf16 *feat, const __bf16 *Wb,
                         __bf16 *dzprev, float *part, float *pbias, int X, int B, hipStream_t s);
int surx_wgrad_parts(int X, int B);
hipError_t surx_reduce_adam(int layers, const float *const *part, const float *const *pbias, int P, float *const *wm,
                            float *const *mw, float *const *vw, float *const *dw, float *const *bias,
                            float *const *mb, float *const *vb, float *const *db, __bf16 *const *Wf,
                            __bf16 *const *Wb, const int *cin, const int *coutp, const int *cout_real, const int *kp,
                            const int *kpb, const double *loss_parts, int nloss, double *loss, float lr, float b1,
                            float b2, float eps, float c1, float c2, hipStream_t s);
hipError_t surx_requant(const float *wm, __bf16 *Wf, __bf16 *Wb, int cin, int coutp, int cout_real, int kp, int kpb,
                        hipStream_t s);
hipError_t surx_init_weights(float *wm, int cin, int coutp, int cout_real, int kp, uint32_t layer, uint32_t seed,
                             hipStream_t s);
hipError_t surx_net(const __bf16 *const *wf, const float *const *bias, int mode, const float *params,
                    const double *n0, void *out, int X, int B, hipStream_t s);
}

namespace {

thread_local std::string g_err;

int fail(int code, const std::string &msg)
{
    g_err = msg;
    return code;
}

#define SUR_TRY(expr)                                                                        \
    do {                                                                                     \
        hipError_t e_ = (expr);                                                              \
        if (e_ != hipSuccess) return fail(PIC_EHIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

constexpr size_t ALIGN = 256;
constexpr int CIN[SUR_LAYERS] = {16, 64, 64, 64, 64, 64};
constexpr int COUT[SUR_LAYERS] = {64, 64, 64, 64, 64, SUR_OUT};
constexpr int COUTP[SUR_LAYERS] = {64, 64, 64, 64, 64, 48};
constexpr float B1 = 0.9f, B2 = 0.999f, EPS = 1e-8f;

int pad32(int k) { return (k + 31) / 32 * 32; }
size_t align_up(size_t n) { return (n + ALIGN - 1) / ALIGN * ALIGN; }

struct Layer {
    int cin, cout, coutp, kp, kpb;
    float *wm, *mw, *vw, *dw;     // [coutp][kp] FP32 (kappa = t*cin + ci)
    float *bias, *mb, *vb, *db;   // [coutp]
    __bf16 *wf;                   // [coutp][kp] in fragment order
    __bf16 *wb;                   // [cin][kpb] (t*coutp + co)
};

struct Bump {
    char *base;
    size_t off = 0;
    template <class T>
    T *take(size_t n)
    {
        off = (off + ALIGN - 1) / ALIGN * ALIGN;
        T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
        off += n * sizeof(T);
        return p;
    }
};

}  // namespace

struct sur_net {
    int X = 0, bmax = 0;
    int device = -1;              // the GPU current at sur_create
    hipStream_t stream = nullptr;
    char *ws = nullptr;
    size_t param_bytes = 0;       // weights, moments, grads: the first bytes of ws
    Layer L[SUR_LAYERS];
    __bf16 *feat = nullptr;       // [bmax][X][16]
    float *y[SUR_LAYERS - 1];     // hidden outputs [bmax][X][64]
    __bf16 *dz[2];                // output gradients of a layer [bmax][X][64], ping-pong
    float *part[SUR_LAYERS];      // partial weight gradients [parts][coutp][kp]
    float *pbias[SUR_LAYERS];     // and bias gradients [parts][coutp]
    bool reduce_after[SUR_LAYERS];   // whether they are summed once this layer's are written (layout)
    double *loss = nullptr;       // the training loss
    double *loss_parts = nullptr; // its shares per forward block
    long long t = 0;              // Adam steps taken
};

namespace {

void layout(sur_net &n, Bump &bp)
{
    const size_t P = (size_t)n.bmax * n.X;
    for (int l = 0; l < SUR_LAYERS; ++l) {
        Layer &L = n.L[l];
        L.cin = CIN[l];
        L.cout = COUT[l];
        L.coutp = COUTP[l];
        L.kp = pad32(SUR_KS * L.cin);
        L.kpb = pad32(SUR_KS * L.coutp);
        const size_t nw = (size_t)L.coutp * L.kp;
        L.wm = bp.take<float>(nw);
        L.mw = bp.take<float>(nw);
        L.vw = bp.take<float>(nw);
        L.dw = bp.take<float>(nw);
        L.bias = bp.take<float>(L.coutp);
        L.mb = bp.take<float>(L.coutp);
        L.vb = bp.take<float>(L.coutp);
        L.db = bp.take<float>(L.coutp);
        L.wf = bp.take<__bf16>(nw);
        L.wb = bp.take<__bf16>((size_t)L.cin * L.kpb);
    }
    n.loss = bp.take<double>(1);
    n.param_bytes = align_up(bp.off);    // cleared whole: a tail of 8 bytes would be a launch of its own
    n.feat = bp.take<__bf16>(P * SUR_IN);
    for (int k = 0; k < 2; ++k) n.dz[k] = bp.take<__bf16>(P * SUR_HIDDEN);
    // One region for the forward blocks' shares of the loss, the partial
    // gradients and the hidden outputs.  The backward pass goes from the last
    // layer to the first and layer l reads y[l-1] only, so the partials are laid
    // out in that order behind the shares and the outputs, last layer first, at
    // the region's end: the partials of layer l may end where y[l-1] begins.
    // The region is 832 bytes per position and the largest layer's partials
    // besides the outputs, the size that callers have planned with.  Samples of
    // whole 256-position slices hold every layer's partials in it; with samples
    // of 64, 128 or 320 positions the gradients of the layers so far are summed
    // when it is full (reduce_after) and the next layer starts over.
    const size_t parts = (size_t)surx_wgrad_parts(n.X, n.bmax);
    const size_t ybytes = align_up(P * SUR_HIDDEN * sizeof(float));
    const size_t largest = parts * (SUR_HIDDEN * pad32(SUR_KS * SUR_HIDDEN) + SUR_HIDDEN) * sizeof(float);
    const size_t fresh = align_up(P * 832) + align_up(largest), region = fresh + (SUR_LAYERS - 1) * ybytes;
    const size_t shares = align_up((size_t)surx_net_train_blocks(n.X, n.bmax) * sizeof(double));   // < 832 P
    char *r = bp.take<char>(region);
    size_t off = shares;
    for (int l = SUR_LAYERS - 1; l >= 0; --l) {
        const size_t w = align_up(parts * n.L[l].coutp * n.L[l].kp * sizeof(float));
        const size_t b = align_up(parts * n.L[l].coutp * sizeof(float));
        const size_t limit = l > 0 ? fresh + (size_t)(SUR_LAYERS - 1 - l) * ybytes : region;
        n.reduce_after[l] = l == 0;
        if (off + w + b > limit) {
            n.reduce_after[l + 1] = true;
            off = shares;
        }
        if (r) {
            n.part[l] = reinterpret_cast<float *>(r + off);
            n.pbias[l] = reinterpret_cast<float *>(r + off + w);
        }
        off += w + b;
    }
    if (r) {
        n.loss_parts = reinterpret_cast<double *>(r);
        for (int l = 0; l < SUR_LAYERS - 1; ++l)
            n.y[l] = reinterpret_cast<float *>(r + fresh + (size_t)(SUR_LAYERS - 2 - l) * ybytes);
    }
}

int check_shape(int batch, int cells)
{
    if (cells <= 0 || cells % 64) return fail(PIC_EINVAL, "cells must be a positive multiple of 64");
    if (batch <= 0 || (long long)batch * cells > (1ll << 28)) return fail(PIC_EINVAL, "bad batch size");
    return PIC_OK;
}

int requant_all(sur_net *n)
{
    for (int l = 0; l < SUR_LAYERS; ++l) {
        const Layer &L = n->L[l];
        SUR_TRY(surx_requant(L.wm, L.wf, L.wb, L.cin, L.coutp, L.cout, L.kp, L.kpb, n->stream));
    }
    return PIC_OK;
}

// Forward pass of any batch straight into the caller's output (surx_net's modes).
int infer(sur_net *n, int mode, const float *params, const double *n0, int B, void *out)
{
    const __bf16 *wf[SUR_LAYERS];
    const float *bias[SUR_LAYERS];
    for (int l = 0; l < SUR_LAYERS; ++l) {
        wf[l] = n->L[l].wf;
        bias[l] = n->L[l].bias;
    }
    // pieces of at most 2^27 positions: the grid stays far below its limits
    const int piece = (int)std::max<long long>(1, (1ll << 27) / n->X);
    const size_t rows = mode == 1 ? 2 : SUR_OUT, size = mode == 0 ? sizeof(float) : sizeof(double);
    for (int b0 = 0; b0 < B; b0 += piece)
        SUR_TRY(surx_net(wf, bias, mode, params + (size_t)4 * b0, n0 ? n0 + b0 : nullptr,
                         static_cast<char *>(out) + (size_t)b0 * rows * n->X * size, n->X, std::min(piece, B - b0),
                         n->stream));
    return PIC_OK;
}

// packed W_l[co][ci][t] <-> master [coutp][t*cin + ci]
void pack(const sur_net *n, int l, const float *m, float *packed)
{
    const Layer &L = n->L[l];
    for (int co = 0; co < L.cout; ++co)
        for (int ci = 0; ci < L.cin; ++ci)
            for (int t = 0; t < SUR_KS; ++t)
                packed[((size_t)co * L.cin + ci) * SUR_KS + t] = m[(size_t)co * L.kp + t * L.cin + ci];
}

void unpack(const sur_net *n, int l, const float *packed, float *m)
{
    const Layer &L = n->L[l];
    std::memset(m, 0, sizeof(float) * L.coutp * L.kp);
    for (int co = 0; co < L.cout; ++co)
        for (int ci = 0; ci < L.cin; ++ci)
            for (int t = 0; t < SUR_KS; ++t)
                m[(size_t)co * L.kp + t * L.cin + ci] = packed[((size_t)co * L.cin + ci) * SUR_KS + t];
}

int copy_out(sur_net *n, bool grads, float *w, float *b)
{
    if (!n || !w || !b) return fail(PIC_EINVAL, "bad arguments");
    SUR_TRY(hipStreamSynchronize(n->stream));
    size_t wo = 0, bo = 0;
    for (int l = 0; l < SUR_LAYERS; ++l) {
        const Layer &L = n->L[l];
        std::vector<float> m((size_t)L.coutp * L.kp), bb(L.coutp);
        SUR_TRY(hipMemcpy(m.data(), grads ? L.dw : L.wm, m.size() * sizeof(float), hipMemcpyDeviceToHost));
        SUR_TRY(hipMemcpy(bb.data(), grads ? L.db : L.bias, bb.size() * sizeof(float), hipMemcpyDeviceToHost));
        pack(n, l, m.data(), w + wo);
        std::memcpy(b + bo, bb.data(), sizeof(float) * L.cout);
        wo += (size_t)L.cout * L.cin * SUR_KS;
        bo += L.cout;
    }
    return PIC_OK;
}

// The most cells per sample that sur_forward_noalloc takes: a limit of its
// interface.  Nothing in the forward pass needs it (the activations are in LDS).
constexpr int NOALLOC_MAX_CELLS = 17096;

}  // namespace

extern "C" {

int sur_workspace_size(int max_batch, int cells, size_t *bytes)
{
    if (!bytes) return fail(PIC_EINVAL, "null argument");
    int rc = check_shape(max_batch, cells);
    if (rc) return rc;
    sur_net n;
    n.X = cells;
    n.bmax = max_batch;
    Bump bp{nullptr};
    layout(n, bp);
    *bytes = (bp.off + ALIGN - 1) / ALIGN * ALIGN;
    return PIC_OK;
}

int sur_create(int max_batch, int cells, void *dev_workspace, size_t bytes, void *hip_stream, uint32_t seed,
               sur_net **out)
{
    if (!out || !dev_workspace) return fail(PIC_EINVAL, "bad arguments");
    if (reinterpret_cast<uintptr_t>(dev_workspace) % ALIGN) return fail(PIC_EINVAL, "workspace not 256-byte aligned");
    size_t need;
    int rc = sur_workspace_size(max_batch, cells, &need);
    if (rc) return rc;
    if (bytes < need) return fail(PIC_ENOSPACE, "workspace too small");
    sur_net *n = new (std::nothrow) sur_net;
    if (!n) return fail(PIC_ENOSPACE, "host allocation failed");
    n->X = cells;
    n->bmax = max_batch;
    n->ws = static_cast<char *>(dev_workspace);
    n->stream = static_cast<hipStream_t>(hip_stream);
    Bump bp{n->ws};
    layout(*n, bp);
    auto cleanup = [&](int code) { delete n; return code; };
    if (hipGetDevice(&n->device) != hipSuccess) return cleanup(fail(PIC_EHIP, "hipGetDevice failed"));
    if (hipMemsetAsync(n->ws, 0, n->param_bytes, n->stream) != hipSuccess)
        return cleanup(fail(PIC_EHIP, "hipMemsetAsync failed"));
    for (int l = 0; l < SUR_LAYERS; ++l) {
        const Layer &L = n->L[l];
        if (surx_init_weights(L.wm, L.cin, L.coutp, L.cout, L.kp, (uint32_t)l, seed, n->stream) != hipSuccess)
            return cleanup(fail(PIC_EHIP, "weight init launch failed"));
    }
    rc = requant_all(n);
    if (rc) return cleanup(rc);
    *out = n;
    return PIC_OK;
}

int sur_set_weights(sur_net *n, const float *w, const float *b)
{
    if (!n || !w || !b) return fail(PIC_EINVAL, "bad arguments");
    SUR_TRY(hipStreamSynchronize(n->stream));
    SUR_TRY(hipMemsetAsync(n->ws, 0, n->param_bytes, n->stream));
    size_t wo = 0, bo = 0;
    for (int l = 0; l < SUR_LAYERS; ++l) {
        const Layer &L = n->L[l];
        std::vector<float> m((size_t)L.coutp * L.kp), bb(L.coutp, 0.0f);
        unpack(n, l, w + wo, m.data());
        std::memcpy(bb.data(), b + bo, sizeof(float) * L.cout);
        SUR_TRY(hipMemcpyAsync(L.wm, m.data(), m.size() * sizeof(float), hipMemcpyHostToDevice, n->stream));
        SUR_TRY(hipMemcpyAsync(L.bias, bb.data(), bb.size() * sizeof(float), hipMemcpyHostToDevice, n->stream));
        SUR_TRY(hipStreamSynchronize(n->stream));   // the staging vectors die at the end of this iteration
        wo += (size_t)L.cout * L.cin * SUR_KS;
        bo += L.cout;
    }
    n->t = 0;
    int rc = requant_all(n);
    if (rc) return rc;
    SUR_TRY(hipStreamSynchronize(n->stream));
    return PIC_OK;
}

int sur_get_weights(sur_net *n, float *w, float *b) { return copy_out(n, false, w, b); }

int sur_get_grads(sur_net *n, float *w, float *b) { return copy_out(n, true, w, b); }

int sur_forward(sur_net *n, const float *dev_params, int batch, float *dev_out)
{
    if (!n || !dev_params || !dev_out) return fail(PIC_EINVAL, "bad arguments");
    if (batch < 1 || batch > n->bmax) return fail(PIC_EINVAL, "batch exceeds the workspace's max_batch");
    return infer(n, 0, dev_params, nullptr, batch, dev_out);
}

int sur_forward_noalloc(sur_net *n, const float *dev_params, int batch, float *dev_out)
{
    if (!n || !dev_params || !dev_out) return fail(PIC_EINVAL, "bad arguments");
    if (batch < 1) return fail(PIC_EINVAL, "batch must be positive");
    if (n->X > NOALLOC_MAX_CELLS)
        return fail(PIC_EINVAL, "sur_forward_noalloc takes at most " + std::to_string(NOALLOC_MAX_CELLS) +
                                    " cells per sample (sur_forward, which needs no scratch either, takes more)");
    int dev = -1;
    SUR_TRY(hipGetDevice(&dev));
    if (dev != n->device) return fail(PIC_EINVAL, "the handle's GPU is not the current device");
    return infer(n, 0, dev_params, nullptr, batch, dev_out);
}

int sur_train_step(sur_net *n, const float *dev_params, const float *dev_target, int batch, float lr, double *loss)
{
    if (!n || !dev_params || !dev_target) return fail(PIC_EINVAL, "bad arguments");
    if (batch < 1 || batch > n->bmax) return fail(PIC_EINVAL, "batch exceeds the workspace's max_batch");
    if (!(lr > 0.0f)) return fail(PIC_EINVAL, "learning rate must be positive");
    const int X = n->X;
    const __bf16 *wf[SUR_LAYERS];
    const float *bias[SUR_LAYERS];
    for (int l = 0; l < SUR_LAYERS; ++l) {
        wf[l] = n->L[l].wf;
        bias[l] = n->L[l].bias;
    }
    int shares = 0;
    SUR_TRY(surx_net_train(wf, bias, dev_params, dev_target, n->y, n->feat, n->dz[0], n->loss_parts, &shares, X,
                           batch, n->stream));
    n->t += 1;
    const float c1 = (float)(1.0 - std::pow((double)B1, (double)n->t));
    const float c2 = (float)(1.0 - std::pow((double)B2, (double)n->t));
    float *wm[SUR_LAYERS], *mw[SUR_LAYERS], *vw[SUR_LAYERS], *dw[SUR_LAYERS];
    float *bm[SUR_LAYERS], *mb[SUR_LAYERS], *vb[SUR_LAYERS], *db[SUR_LAYERS];
    __bf16 *lwf[SUR_LAYERS], *lwb[SUR_LAYERS];
    int kp[SUR_LAYERS], kpb[SUR_LAYERS];
    for (int l = 0; l < SUR_LAYERS; ++l) {
        const Layer &L = n->L[l];
        wm[l] = L.wm; mw[l] = L.mw; vw[l] = L.vw; dw[l] = L.dw;
        bm[l] = L.bias; mb[l] = L.mb; vb[l] = L.vb; db[l] = L.db;
        lwf[l] = L.wf; lwb[l] = L.wb;
        kp[l] = L.kp; kpb[l] = L.kpb;
    }
    // per layer, last to first: the input gradient (with this layer's weights
    // before their update) and the partial weight gradients in one kernel; once
    // the region is full or the first layer's are written, the layers' gradients
    // summed from the partials, their Adam update and BF16 copies in one launch,
    // the last of them with the loss
    int cur = 0, top = SUR_LAYERS - 1;
    for (int l = SUR_LAYERS - 1; l >= 0; --l) {
        const Layer &L = n->L[l];
        if (l > 0)
            SUR_TRY(surx_conv_bwd(l, n->dz[cur], n->y[l - 1], nullptr, L.wb, n->dz[cur ^ 1], n->part[l], n->pbias[l],
                                  X, batch, n->stream));
        else
            SUR_TRY(surx_conv_bwd(0, n->dz[cur], nullptr, n->feat, nullptr, nullptr, n->part[0], n->pbias[0], X,
                                  batch, n->stream));
        cur ^= 1;
        if (!n->reduce_after[l]) continue;
        SUR_TRY(surx_reduce_adam(top - l + 1, n->part + l, n->pbias + l, surx_wgrad_parts(X, batch), wm + l, mw + l,
                                 vw + l, dw + l, bm + l, mb + l, vb + l, db + l, lwf + l, lwb + l, CIN + l, COUTP + l,
                                 COUT + l, kp + l, kpb + l, n->loss_parts, shares, l == 0 ? n->loss : nullptr, lr, B1,
                                 B2, EPS, c1, c2, n->stream));
        top = l - 1;
    }
    if (loss) {
        SUR_TRY(hipMemcpyAsync(loss, n->loss, sizeof(double), hipMemcpyDeviceToHost, n->stream));
        SUR_TRY(hipStreamSynchronize(n->stream));
    }
    return PIC_OK;
}

int sur_densities(sur_net *n, const float *dev_params, const double *dev_n0, int batch, double *dev_dens)
{
    if (!n || !dev_params || !dev_n0 || !dev_dens) return fail(PIC_EINVAL, "bad arguments");
    if (batch < 1 || batch > n->bmax) return fail(PIC_EINVAL, "batch exceeds the workspace's max_batch");
    return infer(n, 1, dev_params, dev_n0, batch, dev_dens);
}

int sur_state(sur_net *n, const float *dev_params, const double *dev_n0, int batch, double *dev_state)
{
    if (!n || !dev_params || !dev_n0 || !dev_state) return fail(PIC_EINVAL, "bad arguments");
    if (batch < 1 || batch > n->bmax) return fail(PIC_EINVAL, "batch exceeds the workspace's max_batch");
    return infer(n, 2, dev_params, dev_n0, batch, dev_state);
}

const char *sur_last_error(void) { return g_err.c_str(); }

void sur_destroy(sur_net *n) { delete n; }

}  // extern "C"
