// Stage handle and launch sequencing: a pipeline stage T_i is a run of
// consecutive encoder layers applied to one micro-batch (paper section 3.1);
// each layer is LayerNorm -> q|k|v projection -> multi-head attention ->
// output projection + residual -> LayerNorm -> MLP with GELU + residual
// (section 2.1).  ep_stage_forward only enqueues kernels on the caller's
// stream; all device memory is obtained in ep_stage_create.
//
// Workspace per stage (R = max_batch * T rows):
//   x    fp32 [R, D]            residual stream
//   a    act  [R, D]            LayerNorm output, later the attention output
//   big  act  [R, max(3D, M)]   q|k|v, later the MLP hidden activations
//   part fp32 [S, R, D]         bf16 path, small R only: the second MLP layer's sums over S ranges of K
// where act is bf16 on the bf16 path and fp32 on the fp32 path.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "edgepipe.h"
#include "ep_error.h"
#include "ep_kernels.h"
#include "ep_launch.h"
#include "ep_stage.h"

namespace {

struct LayerDev {
    const void *w_qkv, *w_o, *w_fc1, *w_fc2;                       // param dtype
    const float *ln1_g, *ln1_b, *b_qkv, *b_o, *ln2_g, *ln2_b, *b_fc1, *b_fc2;   // always fp32
};

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// A layer's parameters in a stage's block: dense weights, q|k|v, projection, second and first MLP layer (so that what attention touches,
// touch_weights, is one range), then fp32 vectors.  n: elements, off: bytes from where the layer begins; weights are indexed q|k|v,
// projection, first and second MLP layer
struct LayerLayout { size_t n_w[4], off_w[4], n_v[8], off_v[8], bytes; };

LayerLayout layer_layout(const ep_vit_config &c)
{
    const size_t D = c.d_model, M = c.d_mlp, wsz = c.param_dtype == EP_BF16 ? 2 : 4;
    LayerLayout l = {{3 * D * D, D * D, M * D, D * M}, {}, {D, D, 3 * D, D, D, D, M, D}, {}, 0};
    for (int i : {0, 1, 3, 2}) { l.off_w[i] = l.bytes; l.bytes += align_up(l.n_w[i] * wsz, 256); }
    for (int i = 0; i < 8; ++i) { l.off_v[i] = l.bytes; l.bytes += align_up(l.n_v[i] * 4, 256); }
    return l;
}

inline float bf16_bits_to_float(uint16_t h)
{
    uint32_t u = (uint32_t)h << 16;
    float f;
    std::memcpy(&f, &u, 4);
    return f;
}

}  // namespace

// where a forward keeps its intermediates (see the file header)
struct Workspace {
    float *x;
    void *a;
    void *big;
    float *part;
    size_t part_bytes;
    int32_t ranges_of = 0;                 // a group: the images of a micro-batch, whose K ranges it uses; 0: no group
};

struct ep_stage {
    ep_vit_config cfg;
    int32_t begin, end, max_batch;
    int device;
    bool bf16;
    char *params = nullptr;
    size_t params_bytes = 0;
    char *ws = nullptr;
    size_t ws_bytes = 0;
    Workspace own = {nullptr, nullptr, nullptr, nullptr, 0, 0};   // inside ws
    std::vector<LayerDev> layers;
    // per-kernel timing (ep_stage_trace_begin / _end)
    int trace_kernel = -1;
    size_t trace_used = 0;
    std::vector<hipEvent_t> trace_ev;      // pairs: start, stop
};

#define EP_HIP(call)                                                                         \
    do {                                                                                     \
        hipError_t e_ = (call);                                                              \
        if (e_ != hipSuccess)                                                                \
            return ep_fail(EP_ERR_HIP, "%s failed: %s", #call, hipGetErrorString(e_));       \
    } while (0)

namespace {

ep_status check_config(const ep_vit_config *c)
{
    if (c->n_layers < 1 || c->d_model < 1 || c->n_heads < 1 || c->d_mlp < 1 || c->n_tokens < 1)
        return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_create: non-positive shape in config");
    if (c->d_model % c->n_heads)
        return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_create: d_model %d not divisible by n_heads %d",
                       c->d_model, c->n_heads);
    if (!(c->ln_eps >= 0.f))
        return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_create: ln_eps must be >= 0");
    auto is_dt = [](int32_t d) { return d == EP_F32 || d == EP_BF16; };
    if (!is_dt(c->param_dtype) || !is_dt(c->in_dtype) || !is_dt(c->out_dtype))
        return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_create: unknown dtype");
    if (c->param_dtype == EP_F32) {
        if (c->in_dtype != EP_F32 || c->out_dtype != EP_F32)
            return ep_fail(EP_ERR_UNSUPPORTED, "fp32 parameters require fp32 input and output");
        if (c->n_tokens > 8192)
            return ep_fail(EP_ERR_UNSUPPORTED, "fp32 path supports at most 8192 tokens");
    } else {
        const int dh = c->d_model / c->n_heads;
        if (c->d_model % 64 || c->d_mlp % 64)
            return ep_fail(EP_ERR_UNSUPPORTED, "bf16 path needs d_model and d_mlp divisible by 64");
        if (c->d_model > 2048)
            return ep_fail(EP_ERR_UNSUPPORTED, "bf16 path supports d_model <= 2048");
        if (!ep_bf16_attention_supported(c->n_tokens, dh))
            return ep_fail(EP_ERR_UNSUPPORTED,
                           "bf16 attention supports d_head in {64, 80} and n_tokens <= 4096 (got %d, %d)",
                           dh, c->n_tokens);
    }
    return EP_OK;
}

// the bf16 dense layers index R rows with 32 bits
bool bf16_rows_fit(const ep_vit_config &c, int64_t R)
{
    const int64_t D = c.d_model, M = c.d_mlp, wide = 3 * D > M ? 3 * D : M, deep = D > M ? D : M;
    return R * wide < (1ll << 31) && R * deep * 2 < 0x7FFFFFF0ll && wide * deep * 2 < 0x7FFFFFF0ll;
}

// K ranges of the second MLP layer at `batch` images (1: the layer runs uncut) and the bytes their sums take
int fc2_splits(const ep_vit_config &c, int64_t batch)
{
    return c.param_dtype == EP_BF16 ? ep_bf16_gemm_splits(batch * c.n_tokens, c.d_model, c.d_mlp) : 1;
}

size_t part_bytes(const ep_vit_config &c, int64_t batch)
{
    const int sp = fc2_splits(c, batch);
    return sp > 1 ? align_up((size_t)sp * batch * c.n_tokens * c.d_model * 4, 256) : 0;
}

// Workspace of a forward: x | a | big for `batch` images, then `part_b` bytes for the sums over K ranges;
// each part 256-byte aligned.
struct WorkspaceLayout { size_t x_bytes, a_bytes, big_bytes, part_b; };

WorkspaceLayout workspace_layout(const ep_vit_config &c, int64_t batch, size_t part_b)
{
    const size_t asz = c.param_dtype == EP_BF16 ? 2 : 4;     // bytes per activation-operand element
    const size_t R = (size_t)batch * c.n_tokens, D = c.d_model, M = c.d_mlp;
    const size_t wide = 3 * D > M ? 3 * D : M;
    return {align_up(R * D * 4, 256), align_up(R * D * asz, 256), align_up(R * wide * asz, 256), part_b};
}

size_t workspace_bytes(const ep_vit_config &c, int64_t batch, size_t part_b)
{
    const WorkspaceLayout l = workspace_layout(c, batch, part_b);
    return l.x_bytes + l.a_bytes + l.big_bytes + l.part_b;
}

Workspace carve_workspace(char *base, const ep_vit_config &c, int64_t batch, size_t part_b)
{
    const WorkspaceLayout l = workspace_layout(c, batch, part_b);
    char *part = base + l.x_bytes + l.a_bytes + l.big_bytes;
    return {(float *)base, base + l.x_bytes, base + l.x_bytes + l.a_bytes, part_b ? (float *)part : nullptr, part_b, 0};
}

// Brackets one kernel of the layer with an event pair when that kernel is traced.  For a dense
// layer traced under its _MAIN id the closing event is handed to the GEMM dispatcher, which
// records it right after its first launch.
struct TraceScope {
    ep_stage *st; hipStream_t s; bool on, main_only;
    TraceScope(ep_stage *st_, int kernel, int main_id, hipStream_t s_) : st(st_), s(s_), on(false), main_only(false)
    {
        const bool hit = st->trace_kernel == kernel || (main_id >= 0 && st->trace_kernel == main_id);
        if (hit && st->trace_used + 2 <= st->trace_ev.size()) {
            on = hipEventRecord(st->trace_ev[st->trace_used], s) == hipSuccess;
            main_only = on && st->trace_kernel == main_id;
        }
    }
    hipEvent_t after_main() const { return main_only ? st->trace_ev[st->trace_used + 1] : nullptr; }
    ~TraceScope()
    {
        if (on) {
            if (!main_only) (void)hipEventRecord(st->trace_ev[st->trace_used + 1], s);
            st->trace_used += 2;
        }
    }
};
#define EP_TRACED(kernel, call) do { TraceScope ts_(st, kernel, -1, s); EP_HIP(call); } while (0)
// `call` may use ts_.after_main()
#define EP_TRACED_GEMM(kernel, main_id, call) do { TraceScope ts_(st, kernel, main_id, s); EP_HIP(call); } while (0)

// of weights that attention touches: half of the memory-side cache, and see touch_weights
constexpr size_t TOUCH_MOST_BYTES = (size_t)128 << 20, TOUCH_LARGE_BYTES = (size_t)32 << 20;
constexpr double TOUCH_ROWS_PER_MB = 27.0, TOUCH_RANGES_ROWS_PER_MB = 45.0, TOUCH_ALL_ROWS_PER_MB = 110.0;
enum Touch { TOUCH_NONE, TOUCH_LONG, TOUCH_ALL };       // LONG: the projection and the second MLP layer

// What a layer whose second MLP layer ran cut into K ranges has left for its successor: the residual stream
// in w.x still lacks ((part[0] + ... + part[splits-1]) + bias).
struct PendingSum { int splits; const float *bias; };

// Whether attention of a forward over R rows touches the weights of the launches behind it (why and how: ep_attn_bf16.hip).  Whether a call's weights
// come from memory or are still in the memory-side cache is not known here, so both count.  A layer's time over that with nothing touched,
// resident / from memory (all of 160 shapes in profiles/weights_touched.md):
//
//   rows to a MB of weights             projection, second MLP layer     all of them
//   ViT-Base   1 x 197    14            1.011 / 1.012                    1.026 / 1.010       nothing: attention is too short for it
//              2 x 197    28            1.006 / 0.997                    1.021 / 0.976
//              4 x 197    56            0.987 / 0.956                    1.000 / 0.923
//              2 x 577    82            1.011 / 0.989                    1.020 / 0.974
//             16 x 197   223            0.995 / 0.976                    0.999 / 0.906
//   DeiT-Small 8 x 197   445            0.994 / 0.951                    0.993 / 0.906
//             32 x 197  1781            0.999 / 0.948                    0.994 / 0.875
//   512 wide   1 x 197    31            0.998 / 1.001                    1.017 / 1.012
//              4 x 197   125            0.996 / 0.978                    0.990 / 0.947
//   ViT-Large  5 x 197    39            1.007 / 1.005                    1.023 / 0.992       nothing: FC2 in ranges of K waits less
//              6 x 197    47            0.991 / 0.972                    1.008 / 0.988
//             14 x 197   110            0.995 / 0.976                    1.007 / 0.979
//             16 x 197   125            0.994 / 0.944                    0.999 / 0.927
//             32 x 197   250            1.005 / 1.008                    0.989 / 0.996       LayerNorm with dense layers
//   ViT-Huge   8 x 197    40            1.003 / 0.933                    1.026 / 0.927
//             12 x 257    78            1.004 / 1.002                    1.017 / 1.003       nothing: a persistent first MLP layer
//             16 x 257   105            1.014 / 1.014                    1.025 / 1.039       nothing: higher tiles in FC2
//             64 x 257   418            1.004 / 0.999                    1.014 / 1.004       nothing: a persistent FC2
//
//   Up to 768 wide therefore all from 27 rows to a MB on, which costs 1.4 to 2.1 % of a layer with resident weights below 41 rows to a MB and at
// 2 x 577 and 4 x 257 of ViT-Base, and up to 1 % elsewhere (DeiT-Tiny, whose passes wait for the host, 1.9).  Past 768 wide only where LayerNorm goes
// with a dense layer or the second MLP layer waits for its weights, and below 110 rows to a MB only that layer's and the projection's, 40 % of the
// bytes: at most 0.8 % with resident weights.  256 x 192 tiles of more than 32 MB of weights (ViT-Huge on 25 x 257 0.97 / 0.98, 32 x 197 1.00 / 1.00,
// 32 x 257 0.98 / 0.99) are left alone: on another card they lost 1.5 %.  Images of 50 tokens gain more, and pay less, than as many rows of 197 to 577,
// so the line is not in tokens.
//   Dense layers that go with their LayerNorm touch their weights themselves otherwise, which takes them longer: ViT-Base on 32 images 1.015, ViT-Large
// on 28 180.7 us and 178.6, 40 232.6 and 226.5, with its touching left out.
// ranges: whether the second MLP layer may be cut into ranges of K; ranges_of: of a group, the images of a micro-batch (0: no group)
Touch touch_weights(const ep_vit_config &c, int32_t B, bool ranges, int32_t ranges_of)
{
    const int64_t R = (int64_t)B * c.n_tokens, D = c.d_model, M = c.d_mlp;
    const size_t bytes = 2 * (size_t)(4 * D * D + 2 * D * M);       // of a layer
    const double rows_per_mb = (double)R * 1e6 / (double)bytes;
    if (c.param_dtype != EP_BF16 || bytes > TOUCH_MOST_BYTES || rows_per_mb < TOUCH_ROWS_PER_MB) return TOUCH_NONE;
    if (!ep_bf16_attention_touches((int64_t)B * c.n_heads, c.n_tokens)) return TOUCH_NONE;
    const Touch most = D <= 768 || rows_per_mb >= TOUCH_ALL_ROWS_PER_MB ? TOUCH_ALL : TOUCH_LONG;
    if (D <= 768 || ep_bf16_ln_gemm_supported(R, 3 * D, D, EPI_BIAS, false) || ep_bf16_ln_gemm_supported(R, M, D, EPI_BIAS_GELU, false)) return most;
    const bool group = ranges_of != 0;
    const EpWeightWait fc2 = ep_bf16_gemm_weight_wait(R, D, M, EPI_BIAS_RESID, ranges ? fc2_splits(c, group ? ranges_of : B) : 1, group);
    if (fc2 == EP_WAITS_PERSISTENT || fc2 == EP_WAITS_HIGH) return TOUCH_NONE;
    if (fc2 == EP_WAITS_LARGE && bytes > TOUCH_LARGE_BYTES) return TOUCH_NONE;
    if (fc2 == EP_WAITS_RANGES && rows_per_mb < TOUCH_RANGES_ROWS_PER_MB) return TOUCH_NONE;
    if (fc2 != EP_WAITS_LARGE && ep_bf16_gemm_weight_wait(R, M, D, EPI_BIAS_GELU, 1, group) == EP_WAITS_PERSISTENT) return TOUCH_NONE;
    return most;
}

// Where that range ends, in bytes from where the layer begins (it begins with the projection); `next`: a layer follows in the block
size_t touch_end(const LayerLayout &l, Touch touch, bool next)
{
    switch (touch) {
    case TOUCH_LONG: return l.off_w[3] + l.n_w[3] * 2;
    case TOUCH_ALL: return next ? l.bytes + l.off_w[0] + l.n_w[0] * 2 : l.off_w[2] + l.n_w[2] * 2;
    default: return l.off_w[1];
    }
}

// What attention of a layer touches: `bytes` from its projection's weights on; before: the layer in front touched this one's first dense layer
struct TouchHere { Touch what; uint32_t bytes; bool before; };

// One layer on R = B*T rows.  `xin` is the residual stream read by this layer
// (may be the caller's fp32 input), the layer leaves its result in `xout`.
// `before`: the layer in front left its sums over K ranges in w.part (xin is w.x then); this layer's first
// LayerNorm adds them.  `after`: if non-null the layer may leave its own in the same way (then xout must be
// w.x, and *after says so with splits > 1); if null it finishes its output itself.
// `xin16`: the stage's bf16 input in place of xin (which is w.x then and gets it as fp32).  `xout16`: where the layer
// may leave its output as bf16 in place of xout; it says so in *narrowed.
ep_status run_layer(ep_stage *st, const Workspace &w, const LayerDev &L, const float *xin, float *xout, int B,
                    hipStream_t s, const PendingSum *before, PendingSum *after, const uint16_t *xin16 = nullptr,
                    uint16_t *xout16 = nullptr, bool *narrowed = nullptr, TouchHere touch = {TOUCH_NONE, 0, false})
{
    const ep_vit_config &c = st->cfg;
    const int T = c.n_tokens, D = c.d_model, M = c.d_mlp, H = c.n_heads;
    const int64_t R = (int64_t)B * T;
    if (after) *after = {1, nullptr};
    if (st->bf16) {
        uint16_t *a = (uint16_t *)w.a, *big = (uint16_t *)w.big;
        const bool one_order = w.ranges_of != 0;                // several micro-batches: each as it would be alone
        // a LayerNorm done inside the dense layer behind it leaves its own bracket empty
        const bool plain1 = !xin16 && !(before && before->splits > 1);
        const bool fuse1 = plain1 && ep_bf16_ln_gemm_supported(R, 3 * D, D, EPI_BIAS, false);
        const bool fuse2 = ep_bf16_ln_gemm_supported(R, M, D, EPI_BIAS_GELU, touch.what == TOUCH_ALL);
        if (xin16)
            EP_TRACED(EP_K_LN1, ep_bf16_layernorm_widen(xin16, w.x, L.ln1_g, L.ln1_b, c.ln_eps, a, R, D, s));
        else if (!plain1)
            EP_TRACED(EP_K_LN1, ep_bf16_layernorm_sum(w.x, w.part, before->splits, before->bias, L.ln1_g, L.ln1_b,
                                                      c.ln_eps, a, R, D, s));
        else
            EP_TRACED(EP_K_LN1, fuse1 ? hipSuccess : ep_bf16_layernorm(xin, D, L.ln1_g, L.ln1_b, c.ln_eps, a, R, D, s));
        EP_TRACED_GEMM(EP_K_QKV, EP_K_QKV_MAIN,
                       fuse1 ? ep_bf16_ln_gemm(xin, L.ln1_g, L.ln1_b, c.ln_eps, (const uint16_t *)L.w_qkv, L.b_qkv, big, R,
                                               3 * D, D, EPI_BIAS, touch.before, ts_.after_main(), s)
                             : ep_bf16_gemm(a, (const uint16_t *)L.w_qkv, L.b_qkv, nullptr, big, R, 3 * D, D, EPI_BIAS,
                                            one_order, ts_.after_main(), s));
        EP_TRACED(EP_K_ATTN, ep_bf16_attention(big, a, B, T, D, H, EpTouch{L.w_o, touch.bytes}, s));
        EP_TRACED_GEMM(EP_K_PROJ, EP_K_PROJ_MAIN,
                       ep_bf16_gemm(a, (const uint16_t *)L.w_o, L.b_o, xin, w.x, R, D, D, EPI_BIAS_RESID,
                                    one_order, ts_.after_main(), s));
        EP_TRACED(EP_K_LN2, fuse2 ? hipSuccess : ep_bf16_layernorm(w.x, D, L.ln2_g, L.ln2_b, c.ln_eps, a, R, D, s));
        EP_TRACED_GEMM(EP_K_FC1, EP_K_FC1_MAIN,
                       fuse2 ? ep_bf16_ln_gemm(w.x, L.ln2_g, L.ln2_b, c.ln_eps, (const uint16_t *)L.w_fc1, L.b_fc1, big, R, M, D,
                                               EPI_BIAS_GELU, touch.what == TOUCH_ALL, ts_.after_main(), s)
                             : ep_bf16_gemm(a, (const uint16_t *)L.w_fc1, L.b_fc1, nullptr, big, R, M, D, EPI_BIAS_GELU,
                                            one_order, ts_.after_main(), s));
        int sp = w.part ? fc2_splits(c, w.ranges_of ? w.ranges_of : B) : 1;
        if ((size_t)sp * R * D * 4 > w.part_bytes) sp = 1;      // never beyond what the workspace holds
        if (sp > 1 && one_order && ep_query_ranges_height(R, D, M, sp) > 0) {
            // a group: the ranges of a micro-batch one after the other in one launch
            TraceScope ts_(st, EP_K_FC2, EP_K_FC2_MAIN, s);
            EP_HIP(ep_bf16_gemm_ranges(big, (const uint16_t *)L.w_fc2, L.b_fc2, w.x, xout, R, D, M, sp, s));
            if (ts_.after_main()) EP_HIP(hipEventRecord(ts_.after_main(), s));
        } else if (sp > 1) {
            // few tiles and a long K: one workgroup per (K range, tile); the sums are added by the next
            // layer's first LayerNorm, or here when nobody follows
            TraceScope ts_(st, EP_K_FC2, EP_K_FC2_MAIN, s);
            EP_HIP(ep_bf16_gemm_partial(big, (const uint16_t *)L.w_fc2, w.part, R, D, M, sp, s));
            if (ts_.after_main()) EP_HIP(hipEventRecord(ts_.after_main(), s));
            if (after && xout == w.x) {
                *after = {sp, L.b_fc2};
            } else {
                EP_HIP(ep_f32_residual_sum(w.x, w.part, sp, L.b_fc2, xout16 ? (void *)xout16 : (void *)xout, xout16 != nullptr,
                                           R, D, s));
                if (xout16) *narrowed = true;
            }
        } else {
            EP_TRACED_GEMM(EP_K_FC2, EP_K_FC2_MAIN,
                           ep_bf16_gemm(big, (const uint16_t *)L.w_fc2, L.b_fc2, w.x, xout, R, D, M, EPI_BIAS_RESID,
                                        one_order, ts_.after_main(), s));
        }
    } else {
        float *a = (float *)w.a, *big = (float *)w.big;
        const bool fuse1 = ep_f32_ln_gemm_supported(xin, (const float *)L.w_qkv, R, 3 * D, D);
        const bool fuse2 = ep_f32_ln_gemm_supported(w.x, (const float *)L.w_fc1, R, M, D);
        EP_TRACED(EP_K_LN1, fuse1 ? hipSuccess : ep_f32_layernorm(xin, D, L.ln1_g, L.ln1_b, c.ln_eps, a, R, D, s));
        EP_TRACED(EP_K_QKV, fuse1 ? ep_f32_ln_gemm(xin, L.ln1_g, L.ln1_b, c.ln_eps, (const float *)L.w_qkv, L.b_qkv, big, R, 3 * D, D, EPI_BIAS, s)
                                  : ep_f32_gemm(a, (const float *)L.w_qkv, L.b_qkv, nullptr, big, R, 3 * D, D, EPI_BIAS, s));
        EP_TRACED(EP_K_ATTN, ep_f32_attention(big, a, B, T, D, H, s));
        EP_TRACED(EP_K_PROJ, ep_f32_gemm(a, (const float *)L.w_o, L.b_o, xin, w.x, R, D, D, EPI_BIAS_RESID, s));
        EP_TRACED(EP_K_LN2, fuse2 ? hipSuccess : ep_f32_layernorm(w.x, D, L.ln2_g, L.ln2_b, c.ln_eps, a, R, D, s));
        EP_TRACED(EP_K_FC1, fuse2 ? ep_f32_ln_gemm(w.x, L.ln2_g, L.ln2_b, c.ln_eps, (const float *)L.w_fc1, L.b_fc1, big, R, M, D, EPI_BIAS_GELU, s)
                                  : ep_f32_gemm(a, (const float *)L.w_fc1, L.b_fc1, nullptr, big, R, M, D, EPI_BIAS_GELU, s));
        EP_TRACED(EP_K_FC2, ep_f32_gemm(big, (const float *)L.w_fc2, L.b_fc2, w.x, xout, R, D, M, EPI_BIAS_RESID, s));
    }
    return EP_OK;
}

}  // namespace

// ---- the library's own workspace for callers that cannot allocate -------------------------------
// One array per device, part of the loaded code object, held until the process ends.  In host code
// the array's name stands for the symbol, not for device memory: its device address is looked up
// once per device (with that device current) and only that address is handed to kernels.
static __device__ __align__(256) unsigned char scratch[EP_STATIC_SCRATCH_BYTES];

namespace {

std::atomic<unsigned char *> g_scratch_ptr[EP_MAX_DEVICES];      // zero-initialised

// device address of `scratch` on the current device `dev`
ep_status static_scratch(int dev, unsigned char **out)
{
    if (dev < 0 || dev >= EP_MAX_DEVICES)
        return ep_fail(EP_ERR_UNSUPPORTED, "device index %d outside the %d the library keeps a workspace for", dev,
                       EP_MAX_DEVICES);
    unsigned char *p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        EP_HIP(hipGetSymbolAddress((void **)&p, HIP_SYMBOL(scratch)));
        if (!p) return ep_fail(EP_ERR_HIP, "hipGetSymbolAddress returned a null address");
        g_scratch_ptr[dev].store(p, std::memory_order_release);    // every thread stores the same address
    }
    *out = p;
    return EP_OK;
}

}  // namespace

extern "C" ep_status ep_stage_create(const ep_vit_config *cfg, int32_t layer_begin, int32_t layer_end,
                                     const ep_layer_weights *layers, int32_t max_batch, ep_stage_t **out)
{
    ep_clear_error();
    if (!cfg || !layers || !out) return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_create: null argument");
    *out = nullptr;
    ep_status rc = check_config(cfg);
    if (rc != EP_OK) return rc;
    if (layer_begin < 0 || layer_end <= layer_begin || layer_end > cfg->n_layers)
        return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_create: layer range [%d, %d) not inside [0, %d)",
                       layer_begin, layer_end, cfg->n_layers);
    if (max_batch < 1) return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_create: max_batch must be >= 1");
    const int nl = layer_end - layer_begin;
    const int64_t D = cfg->d_model, M = cfg->d_mlp, T = cfg->n_tokens;
    if ((int64_t)max_batch * T > (1ll << 24))
        return ep_fail(EP_ERR_UNSUPPORTED, "ep_stage_create: max_batch * n_tokens exceeds 2^24 rows");
    {
        // what the kernels of a forward over max_batch images index with 32 bits (or a 16-bit grid
        // dimension): refuse here rather than in the middle of a forward
        const int64_t R = (int64_t)max_batch * T;
        const bool fits = cfg->param_dtype == EP_BF16 ? bf16_rows_fit(*cfg, R)
                                                      : (R + 63) / 64 <= 65535 && max_batch <= 65535 && cfg->n_heads <= 65535;
        if (!fits)
            return ep_fail(EP_ERR_UNSUPPORTED,
                           "ep_stage_create: max_batch %d gives %lld rows, more than the dense layers of this "
                           "width can index", max_batch, (long long)R);
    }
    for (int l = 0; l < nl; ++l) {
        const ep_layer_weights &w = layers[l];
        if (!w.ln1_g || !w.ln1_b || !w.w_qkv || !w.b_qkv || !w.w_o || !w.b_o || !w.ln2_g || !w.ln2_b ||
            !w.w_fc1 || !w.b_fc1 || !w.w_fc2 || !w.b_fc2)
            return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_create: null parameter pointer in layer %d", l);
    }

    ep_stage *st = new (std::nothrow) ep_stage();
    if (!st) return ep_fail(EP_ERR_OOM, "ep_stage_create: host allocation failed");
    st->cfg = *cfg;
    st->begin = layer_begin; st->end = layer_end; st->max_batch = max_batch;
    st->bf16 = cfg->param_dtype == EP_BF16;
    const size_t wsz = st->bf16 ? 2 : 4;     // bytes per dense-weight element

    auto fail = [&](ep_status s) { ep_stage_destroy(st); return s; };
    hipError_t e = hipGetDevice(&st->device);
    if (e != hipSuccess) return fail(ep_fail(EP_ERR_HIP, "hipGetDevice failed: %s", hipGetErrorString(e)));
    {
        // set-up for ep_stage_forward_static on this device: the address of the library's own workspace
        unsigned char *unused = nullptr;
        const ep_status src = static_scratch(st->device, &unused);
        if (src != EP_OK) return fail(src);
    }

    const LayerLayout layout = layer_layout(*cfg);
    const size_t layer_bytes = layout.bytes;
    const auto &n_w = layout.n_w, &off_w = layout.off_w;
    const auto &n_v = layout.n_v, &off_v = layout.off_v;
    st->params_bytes = layer_bytes * nl;
    e = hipMalloc((void **)&st->params, st->params_bytes);
    if (e != hipSuccess) {
        st->params = nullptr;
        return fail(ep_fail(EP_ERR_OOM, "hipMalloc of %zu parameter bytes failed: %s", st->params_bytes,
                            hipGetErrorString(e)));
    }

    // ---- workspace; the sums over K ranges only exist at small micro-batches, sized for the micro-batch that
    // needs most
    size_t part_max = 0;
    for (int64_t b = 1; b <= max_batch && b * T <= EP_RANGE_SUM_ROWS; ++b) {
        const size_t pb = part_bytes(st->cfg, b);
        if (pb > part_max) part_max = pb;
    }
    st->ws_bytes = workspace_bytes(st->cfg, max_batch, part_max);
    e = hipMalloc((void **)&st->ws, st->ws_bytes);
    if (e != hipSuccess) {
        st->ws = nullptr;
        return fail(ep_fail(EP_ERR_OOM, "hipMalloc of %zu workspace bytes failed: %s", st->ws_bytes,
                            hipGetErrorString(e)));
    }
    st->own = carve_workspace(st->ws, st->cfg, max_batch, part_max);

    // ---- upload, one layer at a time through a host staging block
    std::vector<char> stage_buf;
    try {
        stage_buf.resize(layer_bytes);
    } catch (...) {
        return fail(ep_fail(EP_ERR_OOM, "ep_stage_create: host staging allocation failed"));
    }
    st->layers.resize(nl);
    // Layers of the bf16 path arrive, dense weights row by row, in a block of their own and are put in fragment order from
    // there: in the workspace where that holds a layer (allocating and freeing a block cost 3 ms a stage of six
    // ViT-Large layers)
    struct Arrival { char *p = nullptr; bool mine = false; ~Arrival() { if (mine) (void)hipFree(p); } } rows;
    if (st->bf16 && st->ws_bytes >= layer_bytes) {
        rows.p = st->ws;
    } else if (st->bf16) {
        if ((e = hipMalloc((void **)&rows.p, layer_bytes)) != hipSuccess)
            return fail(ep_fail(EP_ERR_OOM, "hipMalloc of %zu bytes for a layer's weights failed: %s", layer_bytes, hipGetErrorString(e)));
        rows.mine = true;
    }
    const int dim_n[4] = {(int)(3 * D), (int)D, (int)M, (int)D}, dim_k[4] = {(int)D, (int)D, (int)D, (int)M};
    for (int l = 0; l < nl; ++l) {
        const ep_layer_weights &w = layers[l];
        const void *src_w[4] = {w.w_qkv, w.w_o, w.w_fc1, w.w_fc2};
        const void *src_v[8] = {w.ln1_g, w.ln1_b, w.b_qkv, w.b_o, w.ln2_g, w.ln2_b, w.b_fc1, w.b_fc2};
        std::memset(stage_buf.data(), 0, layer_bytes);
        for (int i = 0; i < 4; ++i) std::memcpy(stage_buf.data() + off_w[i], src_w[i], n_w[i] * wsz);
        for (int i = 0; i < 8; ++i) {
            float *dst = reinterpret_cast<float *>(stage_buf.data() + off_v[i]);
            if (st->bf16) {
                const uint16_t *sv = static_cast<const uint16_t *>(src_v[i]);
                for (size_t k = 0; k < n_v[i]; ++k) dst[k] = bf16_bits_to_float(sv[k]);   // exact widening
            } else {
                std::memcpy(dst, src_v[i], n_v[i] * 4);
            }
        }
        char *base = st->params + (size_t)l * layer_bytes;
        if (st->bf16) {
            // in order on the null stream: each upload behind what still reads the block for the layer before
            e = hipMemcpy(rows.p, stage_buf.data(), layer_bytes, hipMemcpyHostToDevice);
            for (int i = 0; i < 4 && e == hipSuccess; ++i)
                e = ep_bf16_pack_weights((const uint16_t *)(rows.p + off_w[i]), (uint16_t *)(base + off_w[i]), dim_n[i], dim_k[i], nullptr);
            if (e == hipSuccess)
                e = hipMemcpyAsync(base + off_v[0], rows.p + off_v[0], layer_bytes - off_v[0], hipMemcpyDeviceToDevice, nullptr);
        } else {
            e = hipMemcpy(base, stage_buf.data(), layer_bytes, hipMemcpyHostToDevice);
        }
        if (e != hipSuccess)
            return fail(ep_fail(EP_ERR_HIP, "parameter upload failed: %s", hipGetErrorString(e)));
        LayerDev &d = st->layers[l];
        d.w_qkv = base + off_w[0]; d.w_o = base + off_w[1]; d.w_fc1 = base + off_w[2]; d.w_fc2 = base + off_w[3];
        d.ln1_g = (const float *)(base + off_v[0]); d.ln1_b = (const float *)(base + off_v[1]);
        d.b_qkv = (const float *)(base + off_v[2]); d.b_o = (const float *)(base + off_v[3]);
        d.ln2_g = (const float *)(base + off_v[4]); d.ln2_b = (const float *)(base + off_v[5]);
        d.b_fc1 = (const float *)(base + off_v[6]); d.b_fc2 = (const float *)(base + off_v[7]);
    }
    // forwards run on streams of their own
    if (st->bf16 && (e = hipStreamSynchronize(nullptr)) != hipSuccess)
        return fail(ep_fail(EP_ERR_HIP, "parameter upload failed: %s", hipGetErrorString(e)));
    *out = st;
    return EP_OK;
}

namespace {

// the launches of a forward over B images with the intermediates in `w`
ep_status forward_on(ep_stage *st, const Workspace &w, const void *x_in, int32_t B, void *x_out, hipStream_t s)
{
    const ep_vit_config &c = st->cfg;
    const int64_t n = (int64_t)B * c.n_tokens * c.d_model;
    const int nl = st->end - st->begin;

    // the first layer reads the caller's buffer directly, or widens it into w.x
    const uint16_t *in16 = c.in_dtype == EP_BF16 ? (const uint16_t *)x_in : nullptr;
    const float *cur = in16 ? w.x : (const float *)x_in;
    uint16_t *out16 = c.out_dtype == EP_BF16 ? (uint16_t *)x_out : nullptr;
    bool narrowed = false;
    PendingSum pending = {1, nullptr};
    const LayerLayout layout = layer_layout(c);
    const Touch touch = touch_weights(c, B, w.part != nullptr, w.ranges_of);
    for (int l = 0; l < nl; ++l) {
        const bool last = l + 1 == nl;
        float *dst = (last && c.out_dtype == EP_F32) ? (float *)x_out : w.x;
        const PendingSum before = pending;
        const TouchHere here = {touch, (uint32_t)(touch_end(layout, touch, !last) - layout.off_w[1]), touch == TOUCH_ALL && l > 0};
        ep_status rc = run_layer(st, w, st->layers[l], cur, dst, B, s, &before, last ? nullptr : &pending,
                                 l == 0 ? in16 : nullptr, last ? out16 : nullptr, &narrowed, here);
        if (rc != EP_OK) return rc;
        cur = dst;
    }
    if (out16 && !narrowed) EP_HIP(ep_f32_to_bf16(w.x, out16, n, s));
    return EP_OK;
}

}  // namespace

extern "C" void ep_query_touch_plan(const ep_vit_config *cfg, int32_t batch, int32_t ranges_of, int32_t next, EpTouchPlan *out)
{
    const LayerLayout l = layer_layout(*cfg);
    const Touch touch = touch_weights(*cfg, batch, true, ranges_of);
    *out = {touch, (int64_t)l.off_w[1], (int64_t)touch_end(l, touch, next != 0), (int64_t)l.bytes, {}, {}};
    for (int i = 0; i < 4; ++i) {
        out->weights[i] = (int64_t)l.off_w[i];
        out->weight_ends[i] = (int64_t)(l.off_w[i] + l.n_w[i] * (cfg->param_dtype == EP_BF16 ? 2 : 4));
    }
}

extern "C" ep_status ep_stage_forward(ep_stage_t *st, const void *x_in, int32_t B, void *x_out, void *stream)
{
    if (!st || !x_in || !x_out) return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_forward: null argument");
    if (B < 1 || B > st->max_batch)
        return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_forward: B=%d outside [1, max_batch=%d]", B, st->max_batch);
    int dev = -1;
    EP_HIP(hipGetDevice(&dev));
    if (dev != st->device)
        return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_forward: stage lives on device %d, current device is %d",
                       st->device, dev);
    return forward_on(st, st->own, x_in, B, x_out, (hipStream_t)stream);
}

extern "C" ep_status ep_stage_forward_static(ep_stage_t *st, const void *x_in, int32_t B, void *x_out, void *stream)
{
    if (!st || !x_in || !x_out) return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_forward_static: null argument");
    if (B < 1) return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_forward_static: B=%d, must be >= 1", B);
    // the sums over K ranges are an optimisation of small micro-batches: where they do not fit next to the rest,
    // the second MLP layer runs uncut (same result up to the order of the fp32 additions over K)
    const size_t need = workspace_bytes(st->cfg, B, 0);
    size_t part_b = part_bytes(st->cfg, B);
    if (need + part_b > (size_t)EP_STATIC_SCRATCH_BYTES) part_b = 0;
    if (need > (size_t)EP_STATIC_SCRATCH_BYTES)
        return ep_fail(EP_ERR_UNSUPPORTED,
                       "ep_stage_forward_static: a micro-batch of %d images needs %zu workspace bytes, the library's "
                       "own workspace holds %zu", B, need, (size_t)EP_STATIC_SCRATCH_BYTES);
    int dev = -1;
    EP_HIP(hipGetDevice(&dev));
    if (dev != st->device)
        return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_forward_static: stage lives on device %d, current device is %d",
                       st->device, dev);
    unsigned char *base = nullptr;
    const ep_status rc = static_scratch(dev, &base);      // looked up when the stage was created: a table read
    if (rc != EP_OK) return rc;
    return forward_on(st, carve_workspace((char *)base, st->cfg, B, part_b), x_in, B, x_out, (hipStream_t)stream);
}

// ---- several micro-batches at once: rows are independent of each other, and every kernel of the bf16 path adds up a row
// in the same order whatever the rows beside it, but for two things: the K ranges of the second MLP layer, which stay the
// micro-batch's, and the narrow tiles of a persistent launch, which a group's dense layers do without; a micro-batch that
// has them on its own is not grouped
namespace {

// Micro-batches of up to MICRO_ROWS rows; a group of up to GROUP_ROWS rows, GROUP_ELEMS activations of the widest
// kind and GROUP_SUM_BYTES of sums over K ranges.  Runs of a pipeline, one by one and in groups: eight micro-batches of 8
// ViT-Base images (1576 rows, 12 layers) 4.86 and 3.18 ms, of 4 DeiT-Tiny ones 2.69 and 0.59, four of 2 ViT-Large ones
// 0.96 and 0.54, of 24 3.56 and 3.17, eight of 64 DeiT-Tiny ones (12672 rows) 4.04 and 3.61; past the lines, twice as many
// activations to a group: four of 64 ViT-Large ones 8.67 and 8.31, of 24 3.17 and 3.42, eight of 64 ViT-Base ones 11.1 both.
constexpr int64_t MICRO_ROWS = 1 << 14, GROUP_ROWS = 1 << 15, GROUP_ELEMS = 1 << 26;
constexpr size_t GROUP_SUM_BYTES = (size_t)128 << 20;

// for any count, also those whose ranges follow each other in one launch (ViT-Base, micro-batches of 8: 3, 4 and 6 to 13 of them): a run's
// groups may be smaller
size_t group_part_bytes(const ep_vit_config &c, int32_t micro, int32_t count)
{
    const int sp = fc2_splits(c, micro);
    return sp > 1 ? align_up((size_t)sp * micro * count * c.n_tokens * c.d_model * 4, 256) : 0;
}

}  // namespace

namespace {

// whether a dense layer of a micro-batch on its own has narrow tiles, or past 384 wide would have if LayerNorm did not go with it
bool has_narrow_rows(const ep_vit_config &c, int32_t micro)
{
    const int64_t R = (int64_t)micro * c.n_tokens;
    const int D = c.d_model, M = c.d_mlp;
    const int sp = fc2_splits(c, micro);
    // q|k|v goes without its LayerNorm behind a bf16 input and behind sums over K ranges; wider models run it, and the first
    // MLP layer, in one launch with LayerNorm between two numbers of rows only, which is not asked here: 33, 42 and 55 images of
    // ViT-Base are not grouped though neither launch has narrow tiles
    const bool narrow = D <= 384;
    const bool qkv = !narrow || !ep_bf16_ln_gemm_supported(R, 3 * D, D, EPI_BIAS, false) || c.in_dtype == EP_BF16 || sp > 1;
    return (qkv && ep_bf16_gemm_narrow_rows(R, 3 * D, D, EPI_BIAS) > 0) || ep_bf16_gemm_narrow_rows(R, D, D, EPI_BIAS_RESID) > 0 ||
           (!(narrow && ep_bf16_ln_gemm_supported(R, M, D, EPI_BIAS_GELU, false)) && ep_bf16_gemm_narrow_rows(R, M, D, EPI_BIAS_GELU) > 0) ||
           (sp == 1 && ep_bf16_gemm_narrow_rows(R, D, M, EPI_BIAS_RESID) > 0);
}

int32_t group_limit(const ep_vit_config &c, int32_t micro)
{
    const int64_t rows = (int64_t)micro * c.n_tokens, wide = std::max(3 * (int64_t)c.d_model, (int64_t)c.d_mlp);
    if (c.param_dtype != EP_BF16 || rows > MICRO_ROWS || has_narrow_rows(c, micro)) return 1;
    int64_t n = std::min(GROUP_ROWS, GROUP_ELEMS / wide) / rows;
    while (n > 1 && (!bf16_rows_fit(c, n * rows) || group_part_bytes(c, micro, (int32_t)n) > GROUP_SUM_BYTES)) --n;
    return n < 1 ? 1 : (int32_t)n;
}

}  // namespace

int32_t ep_stage_group_limit(const ep_stage_t *st, int32_t micro) { return group_limit(st->cfg, micro); }

extern "C" int32_t ep_query_group_limit(const ep_vit_config *cfg, int32_t micro) { return group_limit(*cfg, micro); }

size_t ep_stage_group_bytes(const ep_stage_t *st, int32_t micro, int32_t count)
{
    return workspace_bytes(st->cfg, (int64_t)micro * count, group_part_bytes(st->cfg, micro, count));
}

ep_status ep_stage_forward_group(ep_stage_t *st, const void *x_in, int32_t micro, int32_t count, void *x_out, void *ws,
                                 hipStream_t stream)
{
    int dev = -1;
    EP_HIP(hipGetDevice(&dev));
    if (dev != st->device)
        return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_forward: stage lives on device %d, current device is %d", st->device, dev);
    Workspace w = carve_workspace((char *)ws, st->cfg, (int64_t)micro * count, group_part_bytes(st->cfg, micro, count));
    w.ranges_of = micro;
    return forward_on(st, w, x_in, micro * count, x_out, stream);
}

extern "C" ep_status ep_stage_profile(ep_stage_t *st, int32_t B, int32_t iters, void *stream,
                                      double *per_layer_seconds)
{
    if (!st || !per_layer_seconds) return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_profile: null argument");
    if (B < 1 || B > st->max_batch || iters < 1)
        return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_profile: need 1 <= B <= max_batch and iters >= 1");
    int dev = -1;
    EP_HIP(hipGetDevice(&dev));
    if (dev != st->device)
        return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_profile: stage lives on device %d, current device is %d",
                       st->device, dev);
    hipStream_t s = (hipStream_t)stream;
    const ep_vit_config &c = st->cfg;
    const int64_t n = (int64_t)B * c.n_tokens * c.d_model;
    const int nl = st->end - st->begin;
    hipEvent_t t0, t1;
    EP_HIP(hipEventCreate(&t0));
    hipError_t e = hipEventCreate(&t1);
    if (e != hipSuccess) {
        (void)hipEventDestroy(t0);
        return ep_fail(EP_ERR_HIP, "hipEventCreate failed: %s", hipGetErrorString(e));
    }
    ep_status rc = EP_OK;
    for (int l = 0; l < nl && rc == EP_OK; ++l) {
        // fresh, bounded input for every layer so that repeated application cannot drift
        if ((e = ep_fill_pattern(st->own.x, n, s)) != hipSuccess) { rc = ep_fail(EP_ERR_HIP, "fill failed: %s", hipGetErrorString(e)); break; }
        rc = run_layer(st, st->own, st->layers[l], st->own.x, st->own.x, B, s, nullptr, nullptr);          // untimed
        if (rc != EP_OK) break;
        if ((e = ep_fill_pattern(st->own.x, n, s)) != hipSuccess) { rc = ep_fail(EP_ERR_HIP, "fill failed: %s", hipGetErrorString(e)); break; }
        if ((e = hipEventRecord(t0, s)) != hipSuccess) { rc = ep_fail(EP_ERR_HIP, "hipEventRecord failed: %s", hipGetErrorString(e)); break; }
        for (int it = 0; it < iters && rc == EP_OK; ++it) rc = run_layer(st, st->own, st->layers[l], st->own.x, st->own.x, B, s, nullptr, nullptr);
        if (rc != EP_OK) break;
        if ((e = hipEventRecord(t1, s)) != hipSuccess) { rc = ep_fail(EP_ERR_HIP, "hipEventRecord failed: %s", hipGetErrorString(e)); break; }
        if ((e = hipEventSynchronize(t1)) != hipSuccess) { rc = ep_fail(EP_ERR_HIP, "hipEventSynchronize failed: %s", hipGetErrorString(e)); break; }
        float ms = 0.f;
        if ((e = hipEventElapsedTime(&ms, t0, t1)) != hipSuccess) { rc = ep_fail(EP_ERR_HIP, "hipEventElapsedTime failed: %s", hipGetErrorString(e)); break; }
        per_layer_seconds[l] = (double)ms * 1e-3 / iters;
    }
    (void)hipEventDestroy(t0);
    (void)hipEventDestroy(t1);
    return rc;
}

extern "C" ep_status ep_stage_trace_begin(ep_stage_t *st, int32_t kernel, int32_t max_launches)
{
    if (!st) return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_trace_begin: null stage");
    if (kernel < 0 || kernel >= EP_K_TRACE_COUNT || max_launches < 1 || max_launches > (1 << 20))
        return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_trace_begin: bad kernel id or max_launches");
    if (kernel >= EP_K_COUNT && !st->bf16)
        return ep_fail(EP_ERR_UNSUPPORTED, "ep_stage_trace_begin: the _MAIN ids exist on the bf16 path only");
    if (st->trace_kernel >= 0) return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_trace_begin: a trace is already active");
    st->trace_ev.clear();
    st->trace_ev.reserve((size_t)max_launches * 2);
    for (int i = 0; i < max_launches * 2; ++i) {
        hipEvent_t ev;
        hipError_t e = hipEventCreate(&ev);
        if (e != hipSuccess) {
            for (hipEvent_t x : st->trace_ev) (void)hipEventDestroy(x);
            st->trace_ev.clear();
            return ep_fail(EP_ERR_HIP, "hipEventCreate failed: %s", hipGetErrorString(e));
        }
        st->trace_ev.push_back(ev);
    }
    st->trace_used = 0;
    st->trace_kernel = kernel;
    return EP_OK;
}

extern "C" ep_status ep_stage_trace_end(ep_stage_t *st, int32_t *launches, double *seconds)
{
    if (!st || !launches || !seconds) return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_trace_end: null argument");
    if (st->trace_kernel < 0) return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_trace_end: no active trace");
    ep_status rc = EP_OK;
    double total = 0.0;
    for (size_t i = 0; i + 1 < st->trace_used && rc == EP_OK; i += 2) {
        hipError_t e = hipEventSynchronize(st->trace_ev[i + 1]);
        float ms = 0.f;
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, st->trace_ev[i], st->trace_ev[i + 1]);
        if (e != hipSuccess) rc = ep_fail(EP_ERR_HIP, "reading trace events failed: %s", hipGetErrorString(e));
        total += (double)ms * 1e-3;
    }
    for (hipEvent_t x : st->trace_ev) (void)hipEventDestroy(x);
    st->trace_ev.clear();
    if (rc == EP_OK) { *launches = (int32_t)(st->trace_used / 2); *seconds = total; }
    st->trace_used = 0;
    st->trace_kernel = -1;
    return rc;
}

extern "C" ep_status ep_stage_gemm_main_rows(const ep_stage_t *st, int32_t B, int32_t kernel, int64_t *rows)
{
    if (!st || !rows) return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_gemm_main_rows: null argument");
    if (B < 0 || B > st->max_batch) return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_gemm_main_rows: batch out of range");
    const ep_vit_config &c = st->cfg;
    const int64_t R = (int64_t)B * c.n_tokens;
    int N = 0, K = 0;
    switch (kernel) {
    case EP_K_QKV: case EP_K_QKV_MAIN: N = 3 * c.d_model; K = c.d_model; break;
    case EP_K_PROJ: case EP_K_PROJ_MAIN: N = c.d_model; K = c.d_model; break;
    case EP_K_FC1: case EP_K_FC1_MAIN: N = c.d_mlp; K = c.d_model; break;
    case EP_K_FC2: case EP_K_FC2_MAIN: N = c.d_model; K = c.d_mlp; break;
    default: return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_gemm_main_rows: kernel %d is not a dense layer", kernel);
    }
    *rows = st->bf16 && R > 0 ? ep_bf16_gemm_main_rows(R, N, K) : R;
    return EP_OK;
}

extern "C" ep_status ep_stage_info(const ep_stage_t *st, ep_vit_config *cfg, int32_t *layer_begin, int32_t *layer_end,
                                   int32_t *max_batch)
{
    if (!st) return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_info: null stage");
    if (cfg) *cfg = st->cfg;
    if (layer_begin) *layer_begin = st->begin;
    if (layer_end) *layer_end = st->end;
    if (max_batch) *max_batch = st->max_batch;
    return EP_OK;
}

extern "C" ep_status ep_stage_device_bytes(const ep_stage_t *st, uint64_t *bytes)
{
    if (!st || !bytes) return ep_fail(EP_ERR_INVALID_ARG, "ep_stage_device_bytes: null argument");
    *bytes = (uint64_t)st->params_bytes + (uint64_t)st->ws_bytes;
    return EP_OK;
}

extern "C" void ep_stage_destroy(ep_stage_t *st)
{
    if (!st) return;
    if (st->params) (void)hipFree(st->params);
    if (st->ws) (void)hipFree(st->ws);
    for (hipEvent_t x : st->trace_ev) (void)hipEventDestroy(x);
    delete st;
}
