// Host runtime of the learned warm start (C ABI of pic_unet.h): layer table,
// workspace carving, and the order of the forward / backward launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "../../include/pic_unet.h"
#include "ctx_view.h"
#include "unet_internal.h"

using namespace unet;

namespace {

struct Layer {
    int cin, cout, level;
    long long w_off, b_off;
    // inputs: full-resolution source and optional half-resolution source (upsampled)
    int src_act, up_act;         // activation index, -1 = network input / none, -2 = pooled of level
};

// Network order: encoder level 0..3 (two convolutions each, the first of
// levels 1..3 reading the pooled output of the level above), then decoder
// levels 2, 1, 0 (the first reading [upsampled deeper output, skip]).
struct Net {
    Layer L[kNConv];
    long long head_off = 0, count = 0;
    Net()
    {
        const int ch[kLevels] = {16, 32, 64, 128};
        long long off = 0;
        int k = 0;
        int cin = kInCh;
        for (int l = 0; l < kLevels; l++) {
            for (int r = 0; r < 2; r++) {
                Layer &y = L[k];
                y.cin = r == 0 ? cin : ch[l];
                y.cout = ch[l];
                y.level = l;
                y.up_act = -1;
                y.src_act = r == 1 ? k - 1 : (l == 0 ? -1 : -2);
                k++;
            }
            cin = ch[l];
        }
        for (int l = kLevels - 2; l >= 0; l--) {
            for (int r = 0; r < 2; r++) {
                Layer &y = L[k];
                y.cin = r == 0 ? cin + ch[l] : ch[l];
                y.cout = ch[l];
                y.level = l;
                y.up_act = r == 0 ? k - 1 : -1;
                y.src_act = r == 0 ? 2 * l + 1 : k - 1;   // skip: second encoder conv of level l
                k++;
            }
            cin = ch[l];
        }
        for (int q = 0; q < kNConv; q++) {
            L[q].w_off = off;
            off += (long long)L[q].cout * 9 * L[q].cin;
            L[q].b_off = off;
            off += L[q].cout;
        }
        head_off = off;
        count = off + 17;
    }
};

const Net &net()
{
    static Net n;
    return n;
}

struct Carve {
    size_t off = 0;
    char *base = nullptr;
    template <class T> T *take(size_t count)
    {
        off = (off + 255) & ~size_t(255);
        T *p = base ? reinterpret_cast<T *>(base + off) : nullptr;
        off += count * sizeof(T);
        return p;
    }
};

// 32-channel chunks and 16-channel groups of c channels.
int chunks(int c) { return (c + 31) >> 5; }
int groups(int c) { return (c + 15) >> 4; }

} // namespace

struct pic_unet {
    int B = 0, H = 0, W = 0;
    long long P0 = 0;
    hipStream_t stream = nullptr;
    float *params = nullptr, *grads = nullptr, *m = nullptr, *v = nullptr;
    uint16_t *wf[kNConv] = {}, *wd[kNConv] = {};
    uint16_t *x = nullptr;
    uint16_t *act[kNConv] = {};
    uint16_t *pooled[kLevels] = {};
    float *out = nullptr, *target = nullptr, *mask = nullptr, *gout = nullptr;
    float *G[kLevels - 1] = {};                  // gradient of the skip connections
    uint16_t *gy[2] = {};                        // gradients of layer outputs, in turn
    float *part[kNConv] = {}, *bpart[kNConv] = {};
    PrepArgs prep{};
    ReduceArgs red{};
    double *dpart = nullptr, *scal = nullptr;   // scal[0] mask sum, scal[1] loss
    int ndpart = 0;
    int adam_t = 0;
    int pw = 0;                                  // circular padding along W
    bool dirty = true;
    bool timing = false;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    double timed_ms = 0.0;
    int timed_n = 0;
    std::string err;
};

namespace {

pic_status ufail(pic_unet *u, pic_status st, const std::string &msg)
{
    if (u) u->err = msg;
    return st;
}

#define UCHK(u, call)                                                                        \
    do {                                                                                     \
        hipError_t e_ = (call);                                                              \
        if (e_ != hipSuccess)                                                                \
            return ufail(u, PIC_ERR_HIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

int chan(int level) { return 16 << level; }

// Lays out every buffer of a network over B x H x W; base == nullptr only measures.
size_t carve(pic_unet *u, char *base, int B, int H, int W)
{
    const Net &N = net();
    Carve cv;
    cv.base = base;
    const long long P0 = (long long)B * H * W;
    auto P = [&](int l) { return (long long)B * (H >> l) * (W >> l); };
    uint16_t *wf[kNConv], *wd[kNConv], *act[kNConv], *pooled[kLevels] = {};
    float *part[kNConv], *bpart[kNConv];
    int ns[kNConv];
    for (int k = 0; k < kNConv; k++) {
        const int ci = N.L[k].cin, co = N.L[k].cout;
        wf[k] = cv.take<uint16_t>((size_t)chunks(ci) * groups(co) * 9 * 512);
        wd[k] = cv.take<uint16_t>((size_t)chunks(co) * groups(ci) * 9 * 512);
    }
    uint16_t *x = cv.take<uint16_t>((size_t)P0 * kInCh);
    for (int k = 0; k < kNConv; k++) act[k] = cv.take<uint16_t>((size_t)P(N.L[k].level) * N.L[k].cout);
    for (int l = 1; l < kLevels; l++) pooled[l] = cv.take<uint16_t>((size_t)P(l) * chan(l - 1));
    float *out = cv.take<float>(P0), *target = cv.take<float>(P0), *mask = cv.take<float>(P0);
    float *gout = cv.take<float>(P0);
    float *G[kLevels - 1];
    for (int l = 0; l < kLevels - 1; l++) G[l] = cv.take<float>((size_t)P(l) * chan(l));
    uint16_t *gy[2];
    for (int q = 0; q < 2; q++) gy[q] = cv.take<uint16_t>((size_t)P0 * 16);
    for (int k = 0; k < kNConv; k++) {
        const Layer &y = N.L[k];
        ns[k] = wgrad_splits(B, H >> y.level, W >> y.level, y.cin, y.cout);
        part[k] = cv.take<float>((size_t)ns[k] * (y.cout / 16) * groups(y.cin) * 9 * 256);
        bpart[k] = cv.take<float>((size_t)ns[k] * y.cout);
    }
    const int nd = std::max(17 * head_bwd_blocks(P0), loss_blocks(P0));
    double *dpart = cv.take<double>((size_t)nd);
    double *scal = cv.take<double>(8);
    if (u) {
        int first = 0, block0 = 0;
        for (int k = 0; k < kNConv; k++) {
            const Layer &y = N.L[k];
            u->wf[k] = wf[k];
            u->wd[k] = wd[k];
            u->act[k] = act[k];
            u->part[k] = part[k];
            u->bpart[k] = bpart[k];
            PrepArgs &pa = u->prep;
            pa.first[2 * k] = first;
            first += chunks(y.cin) * groups(y.cout) * 9 * 64;
            pa.first[2 * k + 1] = first;
            first += chunks(y.cout) * groups(y.cin) * 9 * 64;
            pa.Cin[k] = y.cin;
            pa.Cout[k] = y.cout;
            pa.w_off[k] = y.w_off;
            pa.wf[k] = wf[k];
            pa.wd[k] = wd[k];
            const int frags = (y.cout / 16) * groups(y.cin) * 9;
            u->red.L[k] = ReduceLayer{part[k], bpart[k], ns[k], frags, groups(y.cin), y.cin, y.cout, block0,
                                      y.w_off, y.b_off};
            block0 += frags;
        }
        u->prep.first[2 * kNConv] = first;
        u->red.wblocks = block0;
        for (int l = 0; l < kLevels; l++) u->pooled[l] = pooled[l];
        for (int l = 0; l < kLevels - 1; l++) u->G[l] = G[l];
        u->x = x;
        u->out = out;
        u->target = target;
        u->mask = mask;
        u->gout = gout;
        u->gy[0] = gy[0];
        u->gy[1] = gy[1];
        u->dpart = dpart;
        u->ndpart = nd;
        u->scal = scal;
    }
    return cv.off + 256;
}

// Full- and half-resolution inputs of convolution k.
void conv_inputs(const pic_unet *u, int k, const uint16_t **src, int *Cs, const uint16_t **up, int *Cu)
{
    const Layer &y = net().L[k];
    *up = nullptr;
    *Cu = 0;
    if (y.up_act >= 0) {
        *up = u->act[y.up_act];
        *Cu = net().L[y.up_act].cout;
    }
    if (y.src_act == -1) {
        *src = u->x;
        *Cs = kInCh;
    } else if (y.src_act == -2) {
        *src = u->pooled[y.level];
        *Cs = chan(y.level - 1);
    } else {
        *src = u->act[y.src_act];
        *Cs = net().L[y.src_act].cout;
    }
}

void enqueue_forward(pic_unet *u)
{
    const Net &N = net();
    hipStream_t s = u->stream;
    if (u->dirty) {
        launch_wprep(u->params, u->prep, s);
        u->dirty = false;
    }
    for (int k = 0; k < kNConv; k++) {
        const Layer &y = N.L[k];
        const int l = y.level;
        ConvArgs a{};
        a.B = u->B;
        a.H = u->H >> l;
        a.W = u->W >> l;
        conv_inputs(u, k, &a.src, &a.Cs, &a.up, &a.Cu);
        a.nchunk = chunks(y.cin);
        a.wt = u->wf[k];
        a.bias = u->params + y.b_off;
        a.Cout = y.cout;
        a.nct = y.cout / 16;
        a.out = u->act[k];
        a.pw = u->pw;
        // the second convolution of encoder levels 0 .. 2 feeds the pooled input of the next level
        if (k < 2 * kLevels - 2 && (k & 1)) a.pool = u->pooled[l + 1];
        if (k == kNConv - 1) {
            a.wh = u->params + N.head_off;
            a.hout = u->out;
        }
        launch_conv(a, EP_FWD, s);
    }
}

// Weight-gradient partial sums of convolution k from gy (its output gradient).
void conv_wgrad(pic_unet *u, int k, const uint16_t *gy)
{
    const Layer &y = net().L[k];
    const ReduceLayer &r = u->red.L[k];
    WgradArgs w{};
    w.B = u->B;
    w.H = u->H >> y.level;
    w.W = u->W >> y.level;
    w.gy = gy;
    w.Cout = y.cout;
    conv_inputs(u, k, &w.src, &w.Cs, &w.up, &w.Cu);
    w.ncs = r.ncs;
    w.nsplit = r.nsplit;
    w.frags = r.frags;
    w.part = u->part[k];
    w.bpart = u->bpart[k];
    w.pw = u->pw;
    launch_wgrad(w, u->stream);
}

// The input gradient of convolution k from gy, up to its epilogue.
ConvArgs dgrad_args(const pic_unet *u, int k, const uint16_t *gy)
{
    const Layer &y = net().L[k];
    ConvArgs a{};
    a.B = u->B;
    a.H = u->H >> y.level;
    a.W = u->W >> y.level;
    a.src = gy;
    a.Cs = y.cout;
    a.nchunk = chunks(y.cout);
    a.wt = u->wd[k];
    a.Cout = y.cin;
    a.nct = y.cin / 16;
    a.pw = u->pw;
    return a;
}

void enqueue_backward(pic_unet *u)
{
    const Net &N = net();
    hipStream_t s = u->stream;
    const int nb = head_bwd_blocks(u->P0);
    int cur = 0;
    launch_head_bwd(u->act[13], u->params + N.head_off, u->gout, u->gy[cur], u->dpart, u->P0, s);
    launch_head_finalize(u->dpart, nb, u->grads + N.head_off, s);
    // gy[cur] -> the masked gradient of the layer before, in the other buffer
    auto step = [&](int k, int ep, const uint16_t *mask, float *skip, int Cup) {
        conv_wgrad(u, k, u->gy[cur]);
        ConvArgs a = dgrad_args(u, k, u->gy[cur]);
        a.out = u->gy[1 - cur];
        a.mask = mask;
        a.skip = skip;
        a.Cup = Cup;
        launch_conv(a, ep, s);
        cur = 1 - cur;
    };
    // decoder, finest level first: convs 13,12 (level 0), 11,10 (level 1), 9,8 (level 2)
    for (int l = 0; l < kLevels - 1; l++) {
        const int kb = 13 - 2 * l, ka = kb - 1;
        step(kb, EP_MASK, u->act[ka], nullptr, 0);
        // the upsampled part goes to the deeper output (conv ka - 1), the rest waits for the encoder
        step(ka, EP_UP, u->act[ka - 1], u->G[l], chan(l + 1));
    }
    // encoder, deepest level first: convs 7,6 (level 3), 5,4 (2), 3,2 (1), 1,0 (0)
    for (int l = kLevels - 1; l >= 0; l--) {
        const int kb = 2 * l + 1, ka = 2 * l;
        step(kb, EP_MASK, u->act[ka], nullptr, 0);
        // the pooling adjoint joins the skip gradient of the finer level
        if (l > 0) step(ka, EP_DOWN, u->act[ka - 1], u->G[l - 1], 0);
        else conv_wgrad(u, ka, u->gy[cur]);
    }
    launch_wgrad_reduce(u->red, u->grads, s);
}

} // namespace

extern "C" {

int64_t pic_unet_param_count(void) { return net().count; }

pic_status pic_unet_layer_info(int32_t k, pic_unet_layer *out)
{
    if (!out || k < 0 || k > kNConv) return PIC_ERR_ARG;
    const Net &N = net();
    if (k == kNConv) {
        *out = pic_unet_layer{16, 1, 0, 0, N.head_off, N.head_off + 16};
        return PIC_OK;
    }
    const Layer &y = N.L[k];
    *out = pic_unet_layer{y.cin, y.cout, y.level, 0, y.w_off, y.b_off};
    return PIC_OK;
}

static bool shape_ok(int B, int H, int W)
{
    return B >= 1 && B <= 64 && H >= 8 && W >= 8 && H % 8 == 0 && W % 8 == 0 && H <= 8192 && W <= 8192;
}

pic_status pic_unet_workspace_size(int32_t batch, int32_t H, int32_t W, size_t *bytes)
{
    if (!bytes || !shape_ok(batch, H, W)) return PIC_ERR_ARG;
    *bytes = carve(nullptr, nullptr, batch, H, W);
    return PIC_OK;
}

pic_status pic_unet_create(int32_t batch, int32_t H, int32_t W, float *params, float *grads,
                           float *adam_m, float *adam_v, void *workspace, size_t workspace_bytes,
                           void *stream, pic_unet **out)
{
    if (!out) return PIC_ERR_ARG;
    *out = nullptr;
    if (!shape_ok(batch, H, W) || !params || !grads || !adam_m || !adam_v || !workspace) return PIC_ERR_ARG;
    if ((reinterpret_cast<uintptr_t>(workspace) & 255) != 0) return PIC_ERR_ARG;
    if (workspace_bytes < carve(nullptr, nullptr, batch, H, W)) return PIC_ERR_ARG;
    pic_unet *u = new pic_unet();
    u->B = batch;
    u->H = H;
    u->W = W;
    u->P0 = (long long)batch * H * W;
    u->stream = static_cast<hipStream_t>(stream);
    u->params = params;
    u->grads = grads;
    u->m = adam_m;
    u->v = adam_v;
    carve(u, static_cast<char *>(workspace), batch, H, W);
    *out = u;
    return PIC_OK;
}

pic_status pic_unet_io_buffers(pic_unet *u, pic_unet_io *io)
{
    if (!u || !io) return PIC_ERR_ARG;
    *io = pic_unet_io{u->x, u->out, u->target, u->mask, u->gout};
    return PIC_OK;
}

pic_status pic_unet_params_changed(pic_unet *u)
{
    if (!u) return PIC_ERR_ARG;
    u->dirty = true;
    return PIC_OK;
}

pic_status pic_unet_forward(pic_unet *u)
{
    if (!u) return PIC_ERR_ARG;
    if (u->timing) UCHK(u, hipEventRecord(u->e0, u->stream));
    enqueue_forward(u);
    if (u->timing) {
        UCHK(u, hipEventRecord(u->e1, u->stream));
        UCHK(u, hipEventSynchronize(u->e1));
        float ms = 0.f;
        UCHK(u, hipEventElapsedTime(&ms, u->e0, u->e1));
        u->timed_ms += ms;
        u->timed_n++;
    }
    UCHK(u, hipGetLastError());
    return PIC_OK;
}

pic_status pic_unet_loss(pic_unet *u, double *loss)
{
    if (!u) return PIC_ERR_ARG;
    const int nb = loss_blocks(u->P0);
    launch_mask_sum(u->mask, u->dpart, u->P0, u->stream);
    launch_sum_parts(u->dpart, nb, u->scal, u->stream);
    launch_loss(u->out, u->target, u->mask, u->scal, u->gout, u->dpart, u->P0, u->stream);
    launch_sum_parts(u->dpart, nb, u->scal + 1, u->stream);
    UCHK(u, hipGetLastError());
    double h = 0.0;
    UCHK(u, hipMemcpyAsync(&h, u->scal + 1, sizeof(double), hipMemcpyDeviceToHost, u->stream));
    UCHK(u, hipStreamSynchronize(u->stream));
    if (loss) *loss = h;
    return PIC_OK;
}

pic_status pic_unet_backward(pic_unet *u)
{
    if (!u) return PIC_ERR_ARG;
    if (u->dirty) return ufail(u, PIC_ERR_STATE, "pic_unet_backward: no forward pass with the current parameters");
    enqueue_backward(u);
    UCHK(u, hipGetLastError());
    return PIC_OK;
}

pic_status pic_unet_adam(pic_unet *u, float lr, float beta1, float beta2, float eps)
{
    if (!u || !(lr > 0.f) || !(beta1 >= 0.f && beta1 < 1.f) || !(beta2 >= 0.f && beta2 < 1.f) || !(eps > 0.f))
        return ufail(u, PIC_ERR_ARG, "pic_unet_adam: bad hyper-parameters");
    u->adam_t++;
    const float c1 = 1.f - (float)std::pow((double)beta1, u->adam_t);
    const float c2 = 1.f - (float)std::pow((double)beta2, u->adam_t);
    launch_adam(u->params, u->grads, u->m, u->v, net().count, lr, beta1, beta2, eps, c1, c2, u->stream);
    u->dirty = true;
    UCHK(u, hipGetLastError());
    return PIC_OK;
}

pic_status pic_unet_snapshot(pic_unet *u, int32_t slot, const double *b, const double *phi,
                             const uint8_t *node_cond, int32_t NX, int32_t NY, float s_rho,
                             float s_v, float s_phi)
{
    if (!u) return PIC_ERR_ARG;
    if (slot < 0 || slot >= u->B || !b || !node_cond || NX < u->H || NY < u->W || (phi && !(s_phi != 0.f)))
        return ufail(u, PIC_ERR_ARG, "pic_unet_snapshot: bad slot, pointer or grid smaller than the network");
    const long long off = (long long)slot * u->H * u->W;
    launch_snapshot(b, phi, node_cond, NX, NY, u->H, u->W, s_rho, s_v, s_phi, u->x + off * kInCh,
                    u->target + off, u->mask + off, u->stream);
    UCHK(u, hipGetLastError());
    return PIC_OK;
}

pic_status pic_unet_guess(pic_unet *u, int32_t slot, const double *b, const uint8_t *node_cond,
                          int32_t NX, int32_t NY, float s_phi, double *guess)
{
    if (!u) return PIC_ERR_ARG;
    if (slot < 0 || slot >= u->B || !b || !node_cond || !guess || NX < u->H || NY < u->W)
        return ufail(u, PIC_ERR_ARG, "pic_unet_guess: bad slot, pointer or grid smaller than the network");
    launch_guess(u->out + (long long)slot * u->H * u->W, b, node_cond, NX, NY, u->H, u->W, s_phi, guess,
                 u->stream);
    UCHK(u, hipGetLastError());
    return PIC_OK;
}

// The network's stream waits for the work queued so far on `other`.
static pic_status after_stream(pic_unet *u, hipStream_t other)
{
    if (other == u->stream) return PIC_OK;
    hipEvent_t ev = nullptr;
    UCHK(u, hipEventCreateWithFlags(&ev, hipEventDisableTiming));
    hipError_t e = hipEventRecord(ev, other);
    if (e == hipSuccess) e = hipStreamWaitEvent(u->stream, ev, 0);
    (void)hipEventDestroy(ev);
    UCHK(u, e);
    return PIC_OK;
}

pic_status pic_solve_learned(pic_ctx *ctx, pic_unet *u, const double *b, float s_rho, float s_v,
                             float s_phi, double *guess, pic_solve_info *info)
{
    if (!ctx || !u) return PIC_ERR_ARG;
    const uint8_t *nc = nullptr;
    int32_t NX = 0, NY = 0;
    pic_status st = pic_node_map(ctx, 0, &nc, nullptr, &NX, &NY);
    if (st != PIC_OK) return st;
    PicCtxView v;
    if ((st = pic_ctx_view(ctx, 0, &v)) != PIC_OK) return st;
    // b was assembled on the context's stream
    if ((st = after_stream(u, v.stream)) != PIC_OK) return st;
    if ((st = pic_unet_snapshot(u, 0, b, nullptr, nc, NX, NY, s_rho, s_v, s_phi)) != PIC_OK) return st;
    if ((st = pic_unet_forward(u)) != PIC_OK) return st;
    if ((st = pic_unet_guess(u, 0, b, nc, NX, NY, s_phi, guess)) != PIC_OK) return st;
    UCHK(u, hipStreamSynchronize(u->stream));
    return pic_solve(ctx, 2, guess, info);
}

pic_status pic_unet_set_periodic(pic_unet *u, int32_t periodic_w)
{
    if (!u || (periodic_w != 0 && periodic_w != 1)) return ufail(u, PIC_ERR_ARG, "periodic_w must be 0 or 1");
    u->pw = periodic_w;
    return PIC_OK;
}

pic_status pic_unet_residual_sample_work_bytes(int32_t H, int32_t W, size_t *bytes)
{
    if (!bytes || H < 1 || W < 1) return PIC_ERR_ARG;
    *bytes = (size_t)rsample_blocks(H, W) * 3 * sizeof(double);
    return PIC_OK;
}

pic_status pic_unet_residual_sample(const double *b, const double *phi_1, const double *phi_2,
                                    const double *phi_t, const uint8_t *node_cond, int32_t NX, int32_t NY,
                                    int32_t periodic_x, int32_t periodic_y, int32_t H, int32_t W, float s_r,
                                    float s_v, float s_d, uint16_t *x, uint16_t *t, double *stats,
                                    void *work, size_t work_bytes, void *stream)
{
    if (!b || !phi_1 || !node_cond || !x || H < 1 || W < 1 || H > NX || W > NY || (t && !phi_t)) return PIC_ERR_ARG;
    if (stats && (!work || work_bytes < (size_t)rsample_blocks(H, W) * 3 * sizeof(double))) return PIC_ERR_ARG;
    launch_rsample(b, phi_1, phi_2, phi_t, node_cond, NX, NY, periodic_x ? 1 : 0, periodic_y ? 1 : 0, H, W,
                   s_r, s_v, s_d, x, t, stats, static_cast<double *>(work), static_cast<hipStream_t>(stream));
    return hipGetLastError() == hipSuccess ? PIC_OK : PIC_ERR_HIP;
}

pic_status pic_unet_residual_sample_noalloc(const double *b, const double *phi_1, const double *phi_2,
                                            const double *phi_t, const uint8_t *node_cond, int32_t NX,
                                            int32_t NY, int32_t periodic_x, int32_t periodic_y, int32_t H,
                                            int32_t W, float s_r, float s_v, float s_d, uint16_t *x, uint16_t *t,
                                            double *stats, void *stream)
{
    if (!b || !phi_1 || !node_cond || !x || H < 1 || W < 1 || H > NX || W > NY || (t && !phi_t)) return PIC_ERR_ARG;
    if (stats && (long long)H * W > rsample_static_max_pixels()) return PIC_ERR_CAPACITY;
    hipError_t e = launch_rsample_static(b, phi_1, phi_2, phi_t, node_cond, NX, NY, periodic_x ? 1 : 0,
                                         periodic_y ? 1 : 0, H, W, s_r, s_v, s_d, x, t, stats,
                                         static_cast<hipStream_t>(stream));
    if (e == hipErrorInvalidDevice) return PIC_ERR_ARG;
    return e == hipSuccess ? PIC_OK : PIC_ERR_HIP;
}

pic_status pic_unet_load(pic_unet *u, int32_t slot, const uint16_t *x, const uint16_t *t)
{
    if (!u) return PIC_ERR_ARG;
    if (slot < 0 || slot >= u->B || !x) return ufail(u, PIC_ERR_ARG, "pic_unet_load: bad slot or null input");
    const long long P = (long long)u->H * u->W, off = (long long)slot * P;
    launch_load(x, t, P, u->x + off * kInCh, u->target + off, u->mask + off, u->stream);
    UCHK(u, hipGetLastError());
    return PIC_OK;
}

pic_status pic_unet_extrapolate(const double *const *phi, const double *coef, int32_t K, int64_t n, double *out,
                                void *stream)
{
    if (!phi || !coef || !out || K < 1 || K > kExtrapMax || n < 0) return PIC_ERR_ARG;
    ExtrapArgs a{};
    for (int k = 0; k < K; ++k) {
        if (!phi[k]) return PIC_ERR_ARG;
        a.p[k] = phi[k];
        a.c[k] = coef[k];
    }
    a.K = K;
    a.n = n;
    a.out = out;
    launch_extrapolate(a, static_cast<hipStream_t>(stream));
    return hipGetLastError() == hipSuccess ? PIC_OK : PIC_ERR_HIP;
}

pic_status pic_unet_residual_guess(pic_unet *u, int32_t slot, const double *phi_1, const double *phi_2,
                                   const uint8_t *node_cond, int32_t NX, int32_t NY, float s_d,
                                   int32_t use_output, double *guess)
{
    if (!u) return PIC_ERR_ARG;
    if (slot < 0 || slot >= u->B || !phi_1 || !node_cond || !guess || NX < u->H || NY < u->W || !(s_d != 0.f))
        return ufail(u, PIC_ERR_ARG, "pic_unet_residual_guess: bad slot, pointer, scale or grid");
    launch_rguess(u->out + (long long)slot * u->H * u->W, phi_1, phi_2, node_cond, NX, NY, u->H, u->W, s_d,
                  use_output ? 1 : 0, guess, u->stream);
    UCHK(u, hipGetLastError());
    return PIC_OK;
}

pic_status pic_solve_learned_residual(pic_ctx *ctx, pic_unet *u, float s_r, float s_v, float s_d,
                                      double *guess, pic_solve_info *info)
{
    if (!ctx || !u) return PIC_ERR_ARG;
    if (u->B < 1) return PIC_ERR_ARG;
    PicCtxView v;
    pic_status st = pic_ctx_view(ctx, 0, &v);
    if (st != PIC_OK) return st;
    if (!guess || v.NX < u->H || v.NY < u->W) return ufail(u, PIC_ERR_ARG, "pic_solve_learned_residual: grid or guess");
    // the right-hand side and the potentials were written on the context's stream
    if ((st = after_stream(u, v.stream)) != PIC_OK) return st;
    launch_rsample(v.b, v.phi, v.phi_prev, nullptr, v.node_cond, v.NX, v.NY, v.px, v.py, u->H, u->W, s_r, s_v,
                   s_d, u->x, nullptr, nullptr, nullptr, u->stream);
    if ((st = pic_unet_forward(u)) != PIC_OK) return st;
    launch_rguess(u->out, v.phi, v.phi_prev, v.node_cond, v.NX, v.NY, u->H, u->W, s_d, 1, guess, u->stream);
    UCHK(u, hipGetLastError());
    UCHK(u, hipStreamSynchronize(u->stream));
    return pic_solve(ctx, 4, guess, info);
}

static bool coarse_factor_ok(int f) { return f == 1 || f == 2 || f == 4 || f == 8 || f == 16; }

pic_status pic_unet_coarse_sample_work_bytes(int32_t f, int32_t H, int32_t W, size_t *bytes)
{
    if (!bytes || !coarse_factor_ok(f) || H < 1 || W < 1) return PIC_ERR_ARG;
    *bytes = (size_t)csample_blocks(f, H, W) * 3 * sizeof(double);
    return PIC_OK;
}

pic_status pic_unet_coarse_sample(const double *b, const double *phi_1, const double *phi_2, const double *phi_t,
                                  const uint8_t *node_cond, int32_t NX, int32_t NY, int32_t periodic_x,
                                  int32_t periodic_y, int32_t f, int32_t H, int32_t W, float s_r, float s_v,
                                  float s_d, uint16_t *x, uint16_t *t, double *stats, void *work,
                                  size_t work_bytes, void *stream)
{
    if (!b || !phi_1 || !node_cond || !x || !coarse_factor_ok(f) || H < 1 || W < 1 || (long long)H * f > NX ||
        (long long)W * f > NY || (t && !phi_t))
        return PIC_ERR_ARG;
    if (stats && (!work || work_bytes < (size_t)csample_blocks(f, H, W) * 3 * sizeof(double))) return PIC_ERR_ARG;
    launch_csample(b, phi_1, phi_2, phi_t, node_cond, NX, NY, periodic_x ? 1 : 0, periodic_y ? 1 : 0, f, H, W, s_r,
                   s_v, s_d, x, t, stats, static_cast<double *>(work), static_cast<hipStream_t>(stream));
    return hipGetLastError() == hipSuccess ? PIC_OK : PIC_ERR_HIP;
}

pic_status pic_unet_coarse_guess(pic_unet *u, int32_t slot, const double *phi_1, const double *phi_2,
                                 const uint8_t *node_cond, int32_t NX, int32_t NY, int32_t periodic_x,
                                 int32_t periodic_y, int32_t f, float s_d, int32_t use_output, double *guess)
{
    if (!u) return PIC_ERR_ARG;
    if (slot < 0 || slot >= u->B || !phi_1 || !node_cond || !guess || !coarse_factor_ok(f) ||
        (long long)u->H * f > NX || (long long)u->W * f > NY || !(s_d != 0.f))
        return ufail(u, PIC_ERR_ARG, "pic_unet_coarse_guess: bad slot, pointer, factor, scale or grid");
    launch_cguess(u->out + (long long)slot * u->H * u->W, phi_1, phi_2, node_cond, NX, NY, periodic_x ? 1 : 0,
                  periodic_y ? 1 : 0, f, u->H, u->W, s_d, use_output ? 1 : 0, guess, u->stream);
    UCHK(u, hipGetLastError());
    return PIC_OK;
}

pic_status pic_solve_learned_coarse(pic_ctx *ctx, pic_unet *u, int32_t f, float s_r, float s_v, float s_d,
                                    double *guess, pic_solve_info *info)
{
    if (!ctx || !u) return PIC_ERR_ARG;
    if (u->B < 1) return PIC_ERR_ARG;
    PicCtxView v;
    pic_status st = pic_ctx_view(ctx, 0, &v);
    if (st != PIC_OK) return st;
    if (!guess || !coarse_factor_ok(f) || (long long)u->H * f > v.NX || (long long)u->W * f > v.NY)
        return ufail(u, PIC_ERR_ARG, "pic_solve_learned_coarse: factor, grid or guess");
    // the right-hand side and the potentials were written on the context's stream
    if ((st = after_stream(u, v.stream)) != PIC_OK) return st;
    launch_csample(v.b, v.phi, v.phi_prev, nullptr, v.node_cond, v.NX, v.NY, v.px, v.py, f, u->H, u->W, s_r, s_v,
                   s_d, u->x, nullptr, nullptr, nullptr, u->stream);
    if ((st = pic_unet_forward(u)) != PIC_OK) return st;
    launch_cguess(u->out, v.phi, v.phi_prev, v.node_cond, v.NX, v.NY, v.px, v.py, f, u->H, u->W, s_d, 1, guess,
                  u->stream);
    UCHK(u, hipGetLastError());
    UCHK(u, hipStreamSynchronize(u->stream));
    return pic_solve(ctx, 4, guess, info);
}

pic_status pic_unet_set_timing(pic_unet *u, int32_t on)
{
    if (!u) return PIC_ERR_ARG;
    if (on && !u->e0) {
        UCHK(u, hipEventCreate(&u->e0));
        UCHK(u, hipEventCreate(&u->e1));
    }
    u->timing = on != 0;
    return PIC_OK;
}

pic_status pic_unet_forward_timing(pic_unet *u, double *avg_ms, int32_t *passes)
{
    if (!u) return PIC_ERR_ARG;
    if (avg_ms) *avg_ms = u->timed_n ? u->timed_ms / u->timed_n : 0.0;
    if (passes) *passes = u->timed_n;
    u->timed_ms = 0.0;
    u->timed_n = 0;
    return PIC_OK;
}

void pic_unet_destroy(pic_unet *u)
{
    if (!u) return;
    if (u->e0) (void)hipEventDestroy(u->e0);
    if (u->e1) (void)hipEventDestroy(u->e1);
    delete u;
}

const char *pic_unet_last_error(const pic_unet *u) { return u ? u->err.c_str() : "null network"; }

} // extern "C"
