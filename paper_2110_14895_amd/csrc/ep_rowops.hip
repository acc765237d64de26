// HBM-bound row kernels of the bf16 path: LayerNorm over the fp32 residual
// stream producing the bf16 GEMM operand (paper section 2.1: the two layer
// normalisations of a layer), with the widening of a stage's bf16 input on the
// way, and narrowing at the stage's end.
//
// LayerNorm: one wavefront (of narrow rows half or a quarter) per row, the whole
// row held in registers (float4 loads), mean then centred variance (two passes over
// registers, one pass over memory), fp32 statistics, round-to-nearest-even
// narrowing.  Algorithmic traffic per row: 4*D bytes read, 2*D written.
#include "ep_kernels.h"
#include "ep_device.h"

namespace {

// What a dense layer whose K was cut into ranges left to do: ((part[0] + ... + part[splits-1]) + bias) + resid,
// the ranges in index order (the same association as the epilogue of the uncut layer: sum, bias, residual).
// The number of ranges is a template argument (2, 4 or 8) so that all loads of a lane are in flight together:
// these kernels run on a few hundred rows, where latency is all there is.
template <int S>
__device__ inline float4 ranges_bias_resid(const float4 *part, size_t range_stride4, float4 bias, float4 resid)
{
    float4 p[S];
#pragma unroll
    for (int r = 0; r < S; ++r) p[r] = part[(size_t)r * range_stride4];
    float4 a = p[0];
#pragma unroll
    for (int r = 1; r < S; ++r) { a.x += p[r].x; a.y += p[r].y; a.z += p[r].z; a.w += p[r].w; }
    a.x += bias.x; a.y += bias.y; a.z += bias.z; a.w += bias.w;
    return make_float4(a.x + resid.x, a.y + resid.y, a.z + resid.z, a.w + resid.w);
}

// SUM == WIDEN: the rows come from bf16 `src` [rows, D] and are left in x as fp32 (the first layer of a stage)
constexpr int WIDEN = -1;

__device__ inline float4 widen4(uint2 p)
{
    return make_float4(__uint_as_float(p.x << 16), __uint_as_float(p.x & 0xFFFF0000u), __uint_as_float(p.y << 16),
                       __uint_as_float(p.y & 0xFFFF0000u));
}

// LPR = lanes to a row, NV = number of float4 per lane (D = 4 * LPR * NV exactly, or ragged when GUARD).  Rows of up to
// 512 elements share a wave: 384 are three float4 to each of 32 lanes, where a wave to a row had half its lanes idle
// in the second of two (DeiT-Small, images to logits on 32: 1021 -> 998 us).  SUM > 0: x is first brought up to
// date in place from the SUM K ranges of the dense layer before it (src: fp32 [SUM, rows, D], bias), then normalised.
// Bound by memory from a few thousand rows on (4.4 to 6 TB/s), by its launch below; so what else a row needs while it
// passes is done here.  Widening a stage's bf16 input in a launch of its own cost 2 us a stage on 197 rows of 1024
// and 4 us on 6304.
template <int LPR, int NV, bool GUARD, int SUM>
__global__ __launch_bounds__(256) void ln_bf16_kernel(float *__restrict__ x, int ldx, int rows, int D, float eps,
                                                      const float *__restrict__ g, const float *__restrict__ b,
                                                      uint16_t *__restrict__ y, const void *__restrict__ src,
                                                      const float *__restrict__ bias)
{
    const int lane = threadIdx.x & (LPR - 1);
    const int64_t row = (int64_t)blockIdx.x * (256 / LPR) + threadIdx.x / LPR;
    if (row >= rows) return;
    float4 *xr = reinterpret_cast<float4 *>(x + row * ldx);
    const int nvec = D >> 2;
    float4 v[NV], gg[NV], bb[NV];
    auto in = [&](int i) { return !GUARD || lane + i * LPR < nvec; };
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = lane + i * LPR;
        v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (!in(i)) continue;
        if (SUM == WIDEN)
            v[i] = widen4(reinterpret_cast<const uint2 *>(static_cast<const uint16_t *>(src) + row * D)[c]);
        else
            v[i] = xr[c];
        if (SUM > 0)
            v[i] = ranges_bias_resid<SUM >= 1 ? SUM : 1>(reinterpret_cast<const float4 *>(static_cast<const float *>(src) + row * D) + c,
                                                        (size_t)rows * D / 4, reinterpret_cast<const float4 *>(bias)[c], v[i]);
    }
    // gain and shift come behind the row and in front of its sums, behind which they would be one more trip to memory; the compiler moves plain
    // loads there, and buffer loads not past the empty assembly, or, where there is nothing else to fetch, past a scheduling barrier (a layer of ViT-Huge on
    // 1 image 51.1 -> 50.8 us, of ViT-Large on 24 160.3 -> 159.2; with the loads of K ranges in front of it too, ViT-Large on 1 to 5 takes 0.3 % more)
#if defined(__HIP_DEVICE_COMPILE__)
    const __amdgpu_buffer_rsrc_t g_rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(g), 0, D * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t b_rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(b), 0, D * 4, 0x00020000);
#pragma unroll
    for (int i = 0; i < NV; ++i) {                     // past the row: zeros
        gg[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(g_rs, (lane + i * LPR) * 16, 0, 0));
        bb[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(b_rs, (lane + i * LPR) * 16, 0, 0));
    }
    if (SUM <= 0) __builtin_amdgcn_sched_barrier(0);
#endif
    asm volatile("" ::: "memory");
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i)
        if (in(i)) {
            if (SUM != 0) xr[lane + i * LPR] = v[i];
            s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
        }
    const float mean = lanes_sum<LPR>(s) / (float)D;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = lane + i * LPR;
        if (!GUARD || c < nvec) {
            v[i].x -= mean; v[i].y -= mean; v[i].z -= mean; v[i].w -= mean;
            // which products are rounded is not left to the compiler, here and below: ep_gemm_bf16_rows.hip gives the same bits
            q += __builtin_fmaf(v[i].x, v[i].x, v[i].y * v[i].y) + __builtin_fmaf(v[i].z, v[i].z, v[i].w * v[i].w);
        }
    }
    const float inv = 1.0f / sqrtf(lanes_sum<LPR>(q) / (float)D + eps);
    uint2 *yr = reinterpret_cast<uint2 *>(y + row * D);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int c = lane + i * LPR;
        if (!GUARD || c < nvec) {
            uint2 o;
            o.x = pack_bf16x2(__builtin_fmaf(v[i].x * inv, gg[i].x, bb[i].x), __builtin_fmaf(v[i].y * inv, gg[i].y, bb[i].y));
            o.y = pack_bf16x2(__builtin_fmaf(v[i].z * inv, gg[i].z, bb[i].z), __builtin_fmaf(v[i].w * inv, gg[i].w, bb[i].w));
            yr[c] = o;
        }
    }
}

// OUT16: the sum leaves as bf16 (a stage's last layer handing over to the next stage)
template <int S, bool OUT16>
__global__ __launch_bounds__(256) void residual_sum_kernel(const float *resid, const float *__restrict__ part,
                                                           const float *__restrict__ bias, void *out,
                                                           int64_t n4, int d4)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n4) return;
    const float4 v =
        ranges_bias_resid<S>(reinterpret_cast<const float4 *>(part) + i, (size_t)n4,
                             reinterpret_cast<const float4 *>(bias)[i % d4], reinterpret_cast<const float4 *>(resid)[i]);
    if (OUT16)
        static_cast<uint2 *>(out)[i] = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
    else
        static_cast<float4 *>(out)[i] = v;
}

__global__ __launch_bounds__(256) void f32_to_bf16_kernel(const float *__restrict__ in,
                                                          uint16_t *__restrict__ out, int64_t n4)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n4) return;
    const float4 v = reinterpret_cast<const float4 *>(in)[i];
    uint2 o;
    o.x = pack_bf16x2(v.x, v.y);
    o.y = pack_bf16x2(v.z, v.w);
    reinterpret_cast<uint2 *>(out)[i] = o;
}

// mode 0: plain LayerNorm of x (which is then only read); WIDEN or a number of K ranges: see ln_bf16_kernel
template <int LPR, int NV>
hipError_t launch_ln(float *x, int64_t ldx, const void *src, int mode, const float *bias, const float *g, const float *b,
                     float eps, uint16_t *y, int64_t rows, int D, hipStream_t s)
{
    constexpr int RPB = 256 / LPR;                     // rows per workgroup
    const unsigned grid = (unsigned)((rows + RPB - 1) / RPB);
    const bool ragged = D != 4 * LPR * NV;
#define EP_LN_LAUNCH(GUARD, SUM) \
    hipLaunchKernelGGL((ln_bf16_kernel<LPR, NV, GUARD, SUM>), dim3(grid), dim3(256), 0, s, x, (int)ldx, (int)rows, D, eps, g, b, y, src, bias)
#define EP_LN_LAUNCH_SUM(SUM) do { if (ragged) EP_LN_LAUNCH(true, SUM); else EP_LN_LAUNCH(false, SUM); } while (0)
    switch (mode) {
    case WIDEN: EP_LN_LAUNCH_SUM(WIDEN); break;
    case 0: EP_LN_LAUNCH_SUM(0); break;
    case 2: EP_LN_LAUNCH_SUM(2); break;
    case 4: EP_LN_LAUNCH_SUM(4); break;
    case 8: EP_LN_LAUNCH_SUM(8); break;
    default: return hipErrorInvalidValue;
    }
#undef EP_LN_LAUNCH_SUM
#undef EP_LN_LAUNCH
    return hipGetLastError();
}

// mode: 0, WIDEN or the number of K ranges
hipError_t layernorm_any(float *x, int64_t ldx, const void *src, int mode, const float *bias, const float *g, const float *b,
                         float eps, uint16_t *y, int64_t rows, int D, hipStream_t s)
{
    if (rows <= 0) return hipSuccess;
    if (D % 4 != 0 || ldx % 4 != 0 || D <= 0 || D > 8 * 256 || rows > 0x7FFFFFFF || ldx > 0x7FFFFFFF) return hipErrorInvalidValue;
    // the fewest lanes to a row that keep it to four float4 a lane
#define EP_LN(LPR, NV) return launch_ln<LPR, NV>(x, ldx, src, mode, bias, g, b, eps, y, rows, D, s)
    if (D <= 256) {
        switch ((D + 63) / 64) {
        case 1: EP_LN(16, 1);
        case 2: EP_LN(16, 2);
        case 3: EP_LN(16, 3);
        default: EP_LN(16, 4);
        }
    }
    if (D <= 512) {
        if (D <= 384) EP_LN(32, 3);
        EP_LN(32, 4);
    }
    switch ((D + 255) / 256) {
    case 3: EP_LN(64, 3);
    case 4: EP_LN(64, 4);
    case 5: EP_LN(64, 5);
    case 6: EP_LN(64, 6);
    case 7: EP_LN(64, 7);
    default: EP_LN(64, 8);
    }
#undef EP_LN
}

}  // namespace

hipError_t ep_bf16_layernorm(const float *x, int64_t ldx, const float *g, const float *b, float eps,
                             uint16_t *y, int64_t rows, int D, hipStream_t s)
{
    // without ranges to add the kernel only reads x
    return layernorm_any(const_cast<float *>(x), ldx, nullptr, 0, nullptr, g, b, eps, y, rows, D, s);
}

hipError_t ep_bf16_layernorm_sum(float *x, const float *part, int splits, const float *bias, const float *g,
                                 const float *b, float eps, uint16_t *y, int64_t rows, int D, hipStream_t s)
{
    if (!part || !bias || (splits != 2 && splits != 4 && splits != 8)) return hipErrorInvalidValue;
    return layernorm_any(x, D, part, splits, bias, g, b, eps, y, rows, D, s);
}

hipError_t ep_bf16_layernorm_widen(const uint16_t *in, float *x, const float *g, const float *b, float eps, uint16_t *y,
                                   int64_t rows, int D, hipStream_t s)
{
    if (!in) return hipErrorInvalidValue;
    return layernorm_any(x, D, in, WIDEN, nullptr, g, b, eps, y, rows, D, s);
}

hipError_t ep_f32_residual_sum(const float *resid, const float *part, int splits, const float *bias, void *out,
                               bool out_bf16, int64_t rows, int D, hipStream_t s)
{
    if (rows <= 0) return hipSuccess;
    if (!part || !bias || D <= 0 || D % 4 != 0) return hipErrorInvalidValue;
    const int64_t n4 = rows * D / 4;
    const dim3 grid((unsigned)((n4 + 255) / 256));
#define EP_SUM_LAUNCH(S) do { if (out_bf16) EP_SUM_LAUNCH_AS(S, true); else EP_SUM_LAUNCH_AS(S, false); } while (0)
#define EP_SUM_LAUNCH_AS(S, OUT16) \
    hipLaunchKernelGGL((residual_sum_kernel<S, OUT16>), grid, dim3(256), 0, s, resid, part, bias, out, n4, D / 4)
    switch (splits) {
    case 2: EP_SUM_LAUNCH(2); break;
    case 4: EP_SUM_LAUNCH(4); break;
    case 8: EP_SUM_LAUNCH(8); break;
    default: return hipErrorInvalidValue;
    }
#undef EP_SUM_LAUNCH_AS
#undef EP_SUM_LAUNCH
    return hipGetLastError();
}

hipError_t ep_f32_to_bf16(const float *in, uint16_t *out, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    if (n % 4) return hipErrorInvalidValue;
    const int64_t n4 = n / 4;
    hipLaunchKernelGGL(f32_to_bf16_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, in, out, n4);
    return hipGetLastError();
}
