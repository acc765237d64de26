// LayerNorm and the dense layer behind it in one launch, narrow models: the q|k|v projection and the first MLP layer
// (paper section 2.1) where K = d_model is at most 384.
//
//   C[M, N] = LN(x)[M, K] . W[N, K]^T + bias[N]   (+ erf GELU), bf16 out
//
// A workgroup brings 64 or 128 rows of the fp32 residual stream in, normalises them (the arithmetic and the order of the
// sums of ln_bf16_kernel, so the same bits) and keeps them in LDS as bf16, all K of them: 96 KB for 128 rows at K = 384.
// Behind that one barrier its eight waves have nothing to wait for: each takes 32 columns at a time, the weights straight
// into registers (fragment order, a ring of R slices that runs on from one set of columns to the next), the rows from
// LDS, the result out through a staging area of its own.
//
// What bounds it: bringing the rows in (196 KB of fp32 for 128 rows at K = 384, 1.5 us at the 57 bytes a clock of a
// compute unit), then the matrix instructions, 2.6 us a set of columns for 128 rows of them.  A K of two to twelve slices
// is too short for a tile with a prologue and an epilogue of its own, and LayerNorm was a launch and two trips through
// memory.  LayerNorm and the dense layer, then this, in us: 1576 x 576 x 192 6.0 and 4.7, 6304 x 576 x 192 9.6 and 6.5,
// 12672 x 768 x 192 with GELU 18.7 and 12.8, 6304 x 1536 x 384 with GELU 21.8 and 15.4, 4728 x 1152 x 384 14.9 and 10.4,
// 50688 x 1152 x 384 72.9 and 64.5.
#include <cstdint>
#include "ep_gemm_bf16_tile.h"
#include "ep_launch.h"

namespace {

using namespace ep_tile;

constexpr int NW = 8, UC = 32, NI = UC / 16;         // waves, columns of a wave at a time

// The sum over LPR lanes, added up as the exchanges of ln_bf16_kernel add it (lane ^ LPR / 2, ... lane ^ 1): from 16 lanes on
// rotations of a row of 16 do what they do, as the values repeat every 8, 4 and 2 lanes by then, and need no LDS (1576
// x 1152 x 384 in panels of 128 rows 11.8 -> 11.2 us).
template <int LPR>
__device__ inline float lanes_sum(float v)
{
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(LPR == 16 || LPR == 32, "");
    if (LPR == 32) v += __shfl_xor(v, 16, 64);
    auto add = [&](auto n) EP_INLINE {
        v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + decltype(n)::value, 0xF, 0xF, false));
    };
    add(std::integral_constant<int, 8>{});
    add(std::integral_constant<int, 4>{});
    add(std::integral_constant<int, 2>{});
    add(std::integral_constant<int, 1>{});
#endif
    return v;
}

// K = 32 KS
template <int KS>
struct Rows {
    static constexpr int K = KS * 32, CH = KS * 4;                     // chunks of a row
    static constexpr int R = KS % 6 == 0 ? 6 : KS % 5 == 0 ? 5 : KS % 4 == 0 ? 4 : KS;   // slices of weights in registers
    static constexpr int LPR = K <= 256 ? 16 : 32, NV = (K + 4 * LPR - 1) / (4 * LPR);   // as ln_bf16_kernel's
    // chunk c of row r, so that the 16-byte reads of 16 rows meet no bank twice: rows of whole 256 bytes all begin at
    // the same bank, others at every second one
    __device__ static int slot(int r, int c) { return K % 128 == 0 ? (c & ~15) | ((c ^ r) & 15) : (c & ~7) | ((c & 7) ^ swz(r)); }
};

template <int KS, int BM, int EPI>
__global__ __launch_bounds__(NW * 64, 2) void gemm_bf16_rows_kernel(const float *x, const float *__restrict__ ln_g,
                                                                    const float *__restrict__ ln_b, float eps, const uint16_t *W,
                                                                    const float *bias, void *Cout, int M, int N, int units, int per,
                                                                    int groups, int panels)
{
#if defined(__HIP_DEVICE_COMPILE__)
    using S = Rows<KS>;
    constexpr int MI = BM / 16;
    typedef WaveOut<MI, NI, EPI> Out;
    extern __shared__ uint4 lds[];                   // BM rows, then the waves' staging areas
    // consecutive workgroups go to different XCDs: each takes a contiguous run of (panel, group)
    const int total = panels * groups, run = (total + NUM_XCD - 1) / NUM_XCD;
    const int id = (int)(blockIdx.x % NUM_XCD) * run + (int)(blockIdx.x / NUM_XCD);
    if ((int)(blockIdx.x / NUM_XCD) >= run || id >= total) return;
    const int m0 = id / groups * BM, u0 = id % groups * per, u1 = min(u0 + per, units);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l15 = lane & 15, g4 = lane >> 4;

    // ---- weights: slice s of columns 32 u .. + 31, two fragments; sets past the last read an empty buffer
    const int nb = N / 16;
    constexpr int block = S::K * 32;                 // bytes of the fragments of 16 columns
    bf16x8 wf[S::R][NI];
    auto load_w = [&](int u, int s, int r) EP_INLINE {
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(W, u < u1 ? (uint32_t)nb * (uint32_t)block : 0u);
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
            wf[r][ni] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16 + (u * NI + ni) * block, s * FRAG_BYTES, 0));
        asm volatile("" ::: "memory");
    };

    // ---- rows in, normalised: LPR lanes to a row, this wave's BM / NW rows all at once
    {
        constexpr int LPR = S::LPR, NV = S::NV, AT = 64 / LPR, IT = BM / NW / AT;
        const int lr = lane & (LPR - 1);
        const __amdgpu_buffer_rsrc_t x_rs = make_rsrc(x + (size_t)m0 * S::K, (uint32_t)(min(BM, M - m0) * S::K * 4));
        f32x4 v[IT][NV], gg[NV], bb[NV];
        auto in = [&](int i) { return (lr + i * LPR) * 4 < S::K; };
#pragma unroll
        for (int t = 0; t < IT; ++t)
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int r = (t * NW + wave) * AT + lane / LPR;
                v[t][i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(x_rs, in(i) ? (r * S::K + (lr + i * LPR) * 4) * 4 : OOB, 0, 0));
            }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            gg[i] = in(i) ? reinterpret_cast<const f32x4 *>(ln_g)[lr + i * LPR] : f32x4{0.f, 0.f, 0.f, 0.f};
            bb[i] = in(i) ? reinterpret_cast<const f32x4 *>(ln_b)[lr + i * LPR] : f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int s = 0; s < S::R; ++s) load_w(u0 + wave, s, s);
#pragma unroll
        for (int t = 0; t < IT; ++t) {
            const int r = (t * NW + wave) * AT + lane / LPR;
            float s = 0.f;
#pragma unroll
            for (int i = 0; i < NV; ++i)
                if (in(i)) s += (v[t][i][0] + v[t][i][1]) + (v[t][i][2] + v[t][i][3]);
            const float mean = lanes_sum<LPR>(s) / (float)S::K;
            float q = 0.f;
#pragma unroll
            for (int i = 0; i < NV; ++i)
                if (in(i)) {
                    v[t][i] -= mean;
                    // which products are rounded is not left to the compiler, here and below: as in ln_bf16_kernel
                    q += __builtin_fmaf(v[t][i][0], v[t][i][0], v[t][i][1] * v[t][i][1]) + __builtin_fmaf(v[t][i][2], v[t][i][2], v[t][i][3] * v[t][i][3]);
                }
            const float inv = 1.0f / sqrtf(lanes_sum<LPR>(q) / (float)S::K + eps);
#pragma unroll
            for (int i = 0; i < NV; ++i)
                if (in(i)) {
                    f32x4 y;
#pragma unroll
                    for (int j = 0; j < 4; ++j) y[j] = __builtin_fmaf(v[t][i][j] * inv, gg[i][j], bb[i][j]);
                    const int c = lr + i * LPR;      // float4 c of the row: half of chunk c / 2
                    reinterpret_cast<uint2 *>(lds + r * S::CH + S::slot(r, c >> 1))[c & 1] = make_uint2(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]));
                }
        }
    }
    __syncthreads();

    // ---- columns
    char *stg = reinterpret_cast<char *>(lds + BM * S::CH) + wave * Out::LDS_BYTES;
    bf16x8 af[MI];
    auto read_a = [&](int s, int mi) EP_INLINE {
        af[mi] = __builtin_bit_cast(bf16x8, lds[(mi * 16 + l15) * S::CH + S::slot(l15, s * 4 + kchunk(g4))]);
    };
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) read_a(0, mi);
    for (int u = u0 + wave; u < u1; u += NW) {
        Out out;
        out.init(Cout, nullptr, bias, m0, BM, 0, u * UC, M, N, 0, lane);
        f32x4 acc[NI][MI];
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) acc[ni][mi] = f32x4{0.f, 0.f, 0.f, 0.f};
        EP_SCHED_FENCE();
        static_for<KS>([&](auto s_c) EP_INLINE {
            constexpr int s = decltype(s_c)::value, r = s % S::R, ahead = s + S::R;
            static_for<MI>([&](auto m_c) EP_INLINE {
                constexpr int mi = decltype(m_c)::value;
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    acc[ni][mi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[r][ni], af[mi], acc[ni][mi], 0, 0, 0);
                EP_SCHED_FENCE();
                read_a(s + 1 == KS ? 0 : s + 1, mi);
                EP_SCHED_FENCE();
            });
            if constexpr (ahead < KS) load_w(u, ahead, r);
            else load_w(u + NW, ahead - KS, r);
            EP_SCHED_FENCE();
        });
        out.template store<0>(acc, stg);
    }
#endif
}

template <int KS, int BM, int EPI>
hipError_t launch_rows(const float *x, const float *g, const float *b, float eps, const uint16_t *W, const float *bias, void *C,
                       int M, int N, int groups, hipStream_t s)
{
    auto kern = gemm_bf16_rows_kernel<KS, BM, EPI>;
    constexpr size_t smem = (size_t)BM * Rows<KS>::CH * 16 + NW * WaveOut<BM / 16, NI, EPI>::LDS_BYTES;
    static_assert(smem <= 160 * 1024, "LDS of a compute unit");
    static EpSmemLimit smem_limit;
    const hipError_t e = smem_limit.ensure(reinterpret_cast<const void *>(kern), (int)smem);
    if (e != hipSuccess) return e;
    const int64_t panels = (M + BM - 1) / BM;
    const int units = (N + UC - 1) / UC;
    const int per = (units + groups - 1) / groups;
    groups = (units + per - 1) / per;
    const int64_t total = panels * groups;
    hipLaunchKernelGGL(kern, dim3((unsigned)((total + NUM_XCD - 1) / NUM_XCD * NUM_XCD)), dim3(NW * 64), smem, s, x, g, b, eps, W, bias,
                       C, M, N, units, per, groups, (int)panels);
    return hipGetLastError();
}

// Rows of a panel and the column groups that share one: rounds of workgroups, each of them as long as the sets of columns
// a wave takes and one more, for bringing the rows in; 64 rows take half as long at twice the weights from L2 (0.48
// for 0.55: 6304 x 1152 x 384 14.7 -> 12.9 us, but 18912 x 1152 x 384 28.1 -> 34.1, 50688 x 1152 x 384 65 -> 77).
struct RowsPlan { int bm, groups; double cost; };

RowsPlan plan_rows(int64_t M, int N, int cus)
{
    const int units = (N + UC - 1) / UC;
    RowsPlan best = {0, 0, 1e30};
    for (int bm : {128, 64})
        for (int n = 1; n * NW < units + NW; ++n) {
            const int64_t panels = (M + bm - 1) / bm;
            const double c = (bm == 128 ? 1.0 : 0.55) * ((panels * n + cus - 1) / cus) * ((units + n * NW - 1) / (n * NW) + 1);
            if (c < best.cost) best = {bm, n, c};
        }
    return best;
}

template <int EPI>
hipError_t launch_k(const float *x, const float *g, const float *b, float eps, const uint16_t *W, const float *bias, void *C,
                    int M, int N, int K, int cus, hipStream_t s)
{
    const RowsPlan p = plan_rows(M, N, cus);
#define EP_ROWS(KS) \
    return p.bm == 128 ? launch_rows<KS, 128, EPI>(x, g, b, eps, W, bias, C, M, N, p.groups, s) \
                       : launch_rows<KS, 64, EPI>(x, g, b, eps, W, bias, C, M, N, p.groups, s)
    switch (K) {
    case 64: EP_ROWS(2);
    case 128: EP_ROWS(4);
    case 192: EP_ROWS(6);
    case 256: EP_ROWS(8);
    case 320: EP_ROWS(10);
    case 384: EP_ROWS(12);
    }
#undef EP_ROWS
    return hipErrorInvalidValue;
}

}  // namespace

// Wider rows take longer to bring in than a few of them are worth (LayerNorm and its dense layer, then this: 394 x 1152 x 384
// 6.3 and 6.7 us, 788 x 960 x 320 7.1 and 7.3, 1182 x 1152 x 384 7.5 and 7.0; 394 x 576 x 192 5.5 and 4.5).
bool ep_bf16_ln_gemm_supported(int64_t M, int N, int K)
{
    return K % 64 == 0 && K >= 64 && K <= 384 && N % 16 == 0 && N < MAX_TILE_N && M * N < (1ll << 31) && (int64_t)N * K * 2 < 0x7FFFFFF0ll &&
           (K <= 256 || M >= 1024);
}

hipError_t ep_bf16_ln_gemm(const float *x, const float *g, const float *b, float eps, const uint16_t *W, const float *bias, void *C,
                           int64_t M, int N, int K, int epi, hipEvent_t after_main, hipStream_t s)
{
    if (M <= 0 || N <= 0) return hipSuccess;
    if (!ep_bf16_ln_gemm_supported(M, N, K) || (epi != EPI_BIAS && epi != EPI_BIAS_GELU)) return hipErrorInvalidValue;
    int cus = 0;
    hipError_t e = ep_device_cu_count(&cus);
    if (e != hipSuccess) return e;
    e = epi == EPI_BIAS ? launch_k<EPI_BIAS>(x, g, b, eps, W, bias, C, (int)M, N, K, cus, s)
                        : launch_k<EPI_BIAS_GELU>(x, g, b, eps, W, bias, C, (int)M, N, K, cus, s);
    if (e != hipSuccess) return e;
    if (after_main) e = hipEventRecord(after_main, s);
    return e;
}
