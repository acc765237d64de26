// LayerNorm and the dense layer behind it in one launch: the q|k|v projection and the first MLP layer (paper section 2.1)
// of models that are 64 to 384 wide in steps of 64, 512, 768 or 1024, between the limits of one_launch_pays.
//
//   C[M, N] = LN(x)[M, K] . W[N, K]^T + bias[N]   (+ erf GELU), bf16 out
//
// A workgroup brings 64 to 128 rows (32 where there are few: launch_few) of the fp32 residual stream in, normalises them (the
// arithmetic and the order of the sums of ln_bf16_kernel, so the same bits) and keeps them in LDS as bf16, all K of them: 96 KB
// for 128 rows at K = 384, 128 KB for 64 at K = 1024.  Behind that one barrier its eight waves have nothing to wait for: each takes 32 columns at a
// time, the weights straight into registers (fragment order, a ring of R slices that runs on from one set of columns to
// the next), the rows from LDS, the result out through a staging area of its own.
//
// What bounds it: bringing the rows in (196 KB of fp32 for 128 rows at K = 384, 1.5 us at the 57 bytes a clock of a
// compute unit), then the matrix instructions, 2.6 us a set of columns for 128 rows of them; from K = 512 on, with fewer rows,
// the weights on their way into the registers (64 bytes a clock of a unit for 64 rows at the matrix pipe's rate, of the 42
// that arrive from L2).  All workgroups go through the columns in the same order, so what an XCD has under way of weights that are
// not in its L2 is no more than what one or two workgroups have, and the launch waits for memory with every set; where few
// groups share a panel the workgroups of an XCD therefore touch all weights between them while their rows come in, a line to a lane
// (weights from memory: 12608 x 2304 x 768 65.5 -> 51.1 us, 7880 x 3072 x 1024 63.9 -> 54.4; over 2500 launches 0.79 of the time at 768
// wide in one group and at 1024 in two, 0.87, 0.92 and 0.97 at 768 in two, three and four, 1.00 at 384 in one, 0.98 and 1.03 at 512 in
// one and two), unless attention in front has touched them (ep_attn_bf16.hip): then it only costs, 2 to 4 % of a ViT-Base layer on
// 20 to 96 images.  A K of two to twelve slices is too short for a tile with a prologue and an epilogue of its own, and LayerNorm was a launch and two trips through
// memory.  LayerNorm and the dense layer, then this, in us, launches back to back with weights from memory: 6304 x 576 x 192 9.0 and 6.0,
// 12672 x 768 x 192 with GELU 18.0 and 12.4, 6304 x 1536 x 384 with GELU 21.3 and 15.4 (17.3 inside a DeiT-Small stage), 4728 x 1152 x 384
// 14.0 and 9.9, 50688 x 1152 x 384 72.6 and 67.3, 6344 x 1536 x 512 22.6 and 16.4, 3172 x 2304 x 768 21.4 and 18.8, 12608 x 3072 x 768
// with GELU 70.7 and 70.2, 7880 x 3072 x 1024 59.5 and 54.4.
#include <cstdint>
#include "ep_gemm_bf16_tile.h"
#include "ep_launch.h"

namespace {

using namespace ep_tile;

constexpr int NW = 8, UC = 32;                       // waves, columns of a wave at a time (16 for few rows)

// K = 32 KS
template <int KS>
struct Rows {
    static constexpr int K = KS * 32, CH = KS * 4;                     // chunks of a row
    // slices of weights in registers
    static constexpr int R = KS >= 16 && KS % 8 == 0 ? 8 : KS % 6 == 0 ? 6 : KS % 5 == 0 ? 5 : KS % 4 == 0 ? 4 : KS;
    static constexpr int LPR = K <= 256 ? 16 : K <= 512 ? 32 : 64, NV = (K + 4 * LPR - 1) / (4 * LPR);   // as ln_bf16_kernel's
    // chunk c of row r, so that the 16-byte reads of 16 rows meet no bank twice: rows of whole 256 bytes all begin at
    // the same bank, others at every second one
    __device__ static int slot(int r, int c) { return K % 128 == 0 ? (c & ~15) | ((c ^ r) & 15) : (c & ~7) | ((c & 7) ^ swz(r)); }
};

// the staging areas of the waves take what LDS the rows leave: passes of 32 rows, or of 16
template <int KS, int BM, int NI, int EPI>
struct RowsOut {
    static constexpr size_t ROWS = (size_t)BM * Rows<KS>::CH * 16;
    static constexpr int PASS = ROWS + NW * WaveOut<BM / 16, NI, EPI>::LDS_BYTES <= 160 * 1024 ? 32 : 16;
    typedef WaveOut<BM / 16, NI, EPI, PASS> Out;
    static constexpr size_t LDS_BYTES = ROWS + NW * Out::LDS_BYTES;
    static_assert(LDS_BYTES <= 160 * 1024, "LDS of a compute unit");
};

// TOUCH: the workgroups of an XCD bring the weights into its L2 between them (a template argument: as a branch it cost the
// launches that do not touch 2 % of twelve DeiT layers)
template <int KS, int BM, int NI, int R, int EPI, bool TOUCH>
__global__ __launch_bounds__(NW * 64, 2) void gemm_bf16_rows_kernel(const float *x, const uint16_t *W, int M, int N, int per, int groups,
                                                                    const float *__restrict__ ln_g, const float *__restrict__ ln_b,
                                                                    float eps, const float *bias, void *Cout)
{
#if defined(__HIP_DEVICE_COMPILE__)
    using S = Rows<KS>;
    constexpr int MI = BM / 16, COLS = 16 * NI;
    const int units = (N + COLS - 1) / COLS, panels = (M + BM - 1) / BM;
    typedef typename RowsOut<KS, BM, NI, EPI>::Out Out;
    extern __shared__ uint4 lds[];                   // BM rows, then the waves' staging areas
    // consecutive workgroups go to different XCDs: each takes a contiguous run of (panel, group)
    const int total = panels * groups, run = (total + NUM_XCD - 1) / NUM_XCD;
    const int id = (int)(blockIdx.x % NUM_XCD) * run + (int)(blockIdx.x / NUM_XCD);
    if ((int)(blockIdx.x / NUM_XCD) >= run || id >= total) return;
    const int m0 = id / groups * BM, u0 = id % groups * per, u1 = min(u0 + per, units);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l15 = lane & 15, g4 = lane >> 4;

    // ---- weights: slice s of columns COLS u .. + COLS - 1; sets past the last read an empty buffer
    const int nb = N / 16;
    constexpr int block = S::K * 32;                 // bytes of the fragments of 16 columns
    bf16x8 wf[R][NI];
    auto load_w = [&](int u, int s, int r) EP_INLINE {
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(W, u < u1 ? (uint32_t)nb * (uint32_t)block : 0u);
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
            wf[r][ni] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16 + (u * NI + ni) * block, s * FRAG_BYTES, 0));
        asm volatile("" ::: "memory");
    };

    // ---- weights, touched: 128 bytes to a lane, behind the rows and the first slices, so that nothing waits for them but the
    // slices after those; what is past NT loads of a wave comes in as it is needed
    constexpr int NT = !TOUCH ? 1 : S::K >= 1024 ? 6 : S::K >= 512 ? 4 : 2;
    int touched[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) touched[i] = 0;
    auto touch_weights = [&]() EP_INLINE {
        const int xcd = (int)(blockIdx.x % NUM_XCD), wgs = min(run, total - xcd * run);       // workgroups on this XCD
        const uint32_t bytes = (uint32_t)nb * (uint32_t)block, lines = (bytes + 127) / 128;
        const uint32_t mine = (lines + wgs * NW - 1) / (wgs * NW), first = ((blockIdx.x / NUM_XCD) * NW + wave) * mine;
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(W, bytes);
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const uint32_t l = (uint32_t)(i * 64 + lane);
            touched[i] = (int)__builtin_amdgcn_raw_buffer_load_b32(rs, l < mine && first + l < lines ? (int)((first + l) * 128) : OOB, 0, 0);
        }
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
        for (int s = 0; s < R; ++s) load_w(u0 + wave, s, s);
        if constexpr (TOUCH) touch_weights();
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
    // rows of the slices ahead: one where it has eight products to land, more where it has two
    constexpr int AD = NI * MI >= 8 ? 1 : KS % 4 ? 2 : 4;
    static_assert(KS % AD == 0, "a set of columns begins with the first register");
    bf16x8 af[AD][MI];
    auto read_a = [&](int s, int mi) EP_INLINE {
        af[s % AD][mi] = __builtin_bit_cast(bf16x8, lds[(mi * 16 + l15) * S::CH + S::slot(l15, s * 4 + kchunk(g4))]);
    };
#pragma unroll
    for (int s = 0; s < AD; ++s)
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) read_a(s, mi);
    for (int u = u0 + wave; u < u1; u += NW) {
        Out out;
        out.init(Cout, nullptr, bias, m0, BM, 0, u * COLS, M, N, 0, lane);
        f32x4 acc[NI][MI];
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int mi = 0; mi < MI; ++mi) acc[ni][mi] = f32x4{0.f, 0.f, 0.f, 0.f};
        EP_SCHED_FENCE();
        static_for<KS>([&](auto s_c) EP_INLINE {
            constexpr int s = decltype(s_c)::value, r = s % R, ahead = s + R;
            static_for<MI>([&](auto m_c) EP_INLINE {
                constexpr int mi = decltype(m_c)::value;
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    acc[ni][mi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[r][ni], af[s % AD][mi], acc[ni][mi], 0, 0, 0);
                EP_SCHED_FENCE();
                read_a((s + AD) % KS, mi);
                EP_SCHED_FENCE();
            });
            if constexpr (ahead < KS) load_w(u, ahead, r);
            else load_w(u + NW, ahead - KS, r);
            EP_SCHED_FENCE();
        });
        out.template store<0>(acc, stg);
    }
#pragma unroll
    for (int i = 0; i < (TOUCH ? NT : 0); ++i) asm volatile("" ::"v"(touched[i]));      // here at the latest they have to have arrived
#endif
}

template <int KS, int BM, int NI, int R, int EPI, bool TOUCH>
hipError_t launch_as(const float *x, const float *g, const float *b, float eps, const uint16_t *W, const float *bias, void *C,
                     int M, int N, int per, int groups, hipStream_t s)
{
    auto kern = gemm_bf16_rows_kernel<KS, BM, NI, R, EPI, TOUCH>;
    constexpr size_t smem = RowsOut<KS, BM, NI, EPI>::LDS_BYTES;
    static EpSmemLimit smem_limit;
    const hipError_t e = smem_limit.ensure(reinterpret_cast<const void *>(kern), (int)smem);
    if (e != hipSuccess) return e;
    const int64_t panels = (M + BM - 1) / BM, total = panels * groups;
    hipLaunchKernelGGL(kern, dim3((unsigned)((total + NUM_XCD - 1) / NUM_XCD * NUM_XCD)), dim3(NW * 64), smem, s, x, W, M, N, per, groups, g, b,
                       eps, bias, C);
    return hipGetLastError();
}

template <int KS, int BM, int EPI>
hipError_t launch_rows(const float *x, const float *g, const float *b, float eps, const uint16_t *W, const float *bias, void *C,
                       int M, int N, int groups, bool touched, hipStream_t s)
{
    const int units = (N + UC - 1) / UC, per = (units + groups - 1) / groups;
    groups = (units + per - 1) / per;
    // Touching pays where a workgroup goes through many columns behind few others' (figures above; when it was introduced, without and
    // with: 3152 x 4096 x 1024 in four groups 43.4 and 39.4 us, in five 38.0 and 39.5, 3152 x 2304 x 768 in six 18.8 and 19.8,
    // 6304 x 1152 x 384, 442 KB to a workgroup, in two 12.1 and 12.4) and every XCD has all groups.  Weights that are in the memory-side cache are
    // not touched again (a layer of ViT-Base on 32 images 133.7 us with both, 130.3 without, ViT-Large on 40 232.6 and 226.5).
    if constexpr (KS > 8)
        if (!touched && groups <= 4 && (int64_t)per * UC * KS * 64 >= 600 * 1024 && M / BM >= NUM_XCD)
            return launch_as<KS, BM, UC / 16, Rows<KS>::R, EPI, true>(x, g, b, eps, W, bias, C, M, N, per, groups, s);
    return launch_as<KS, BM, UC / 16, Rows<KS>::R, EPI, false>(x, g, b, eps, W, bias, C, M, N, per, groups, s);
}

// Rows of a panel, 64 or as many as LDS holds, by the modelled microseconds of a launch: rounds of workgroups, each of them
// bringing the rows in, then the sets of columns that a wave takes (matrix instructions) and the columns of the workgroup
// (weights on their way).  Fitted to 4700 launches of 217 to 39440 rows, K = 64 to 1024, N = 3 K and 4 K: 8 % off a launch.  A panel is shared
// by as many column groups as leave one round of workgroups.  The choice is 0.9 to 1.1 % off the fastest of all heights and groups up to
// 16000 rows of narrow models and 0 to 1 % off from 512 wide on.  (Rounds times sets, below, takes 128 rows in five groups for 6344 x 1152 x 384,
// 14.3 us, where 64 in two take 12.7; and groups of a whole set of columns at least, 1025 x 1152 x 384 7.3 us, where 64 rows in fifteen
// groups take 6.5.)
struct RowsPlan { int bm, groups; double us; };

double rows_us(int64_t M, int N, int K, bool gelu, int bm, int groups, int cus)
{
    const int units = (N + UC - 1) / UC, per = (units + groups - 1) / groups;
    const int64_t wgs = (M + bm - 1) / bm * ((units + per - 1) / per);
    const double rounds = (double)((wgs + cus - 1) / cus), sets = (per + NW - 1) / NW, part = (double)per / NW;
    const double k = K / 1024.0, b = bm / 64.0;
    return 3.3 + 0.32e-6 * M * N + 0.75 * wgs / cus * k * b +
           rounds * (0.2 + b * k * (2.1 + 5.8 * k) + part * k * (1.24 + 2.29 * b) + sets * k * (0.69 * b + 0.49 * k) +
                     (gelu ? b * (0.14 * part + 0.38 * sets) : 0.0));
}

// Narrow models from 2^14 rows on: rounds of workgroups times the sets of columns that a wave takes and one more, for the rows; 64 rows at
// 0.55.  There the one round of 128-row panels that the model above is held to leaves up to half of the units without work, and several
// groups in two rounds are the faster way (with GELU 21814 x 2048 x 256 44.5 us and, in two groups, 37.4, 20037 x 1536 x 384 in three
// 44.4 and 41.8; 23279 x 960 x 320 27.6 and 25.4), which the model, 10 to 20 % short for 128 rows, does not rank.  Of 478 layers from
// 2^14 rows to 60000 this rule is 1.7 % off the fastest of all heights and groups, the model 2.1; below, 1 to 8 % and 1 %.
RowsPlan plan_many_narrow_rows(int64_t M, int N, int cus)
{
    const int units = (N + UC - 1) / UC;
    RowsPlan best = {0, 0, 1e30};
    for (int bm : {128, 64})
        for (int n = 1; n * NW < units + NW; ++n) {
            const int64_t rounds = ((M + bm - 1) / bm * n + cus - 1) / cus, sets = (units + n * NW - 1) / (n * NW);
            const double cost = (bm == 128 ? 1.0 : 0.55) * rounds * (sets + 1);
            if (cost < best.us) best = {bm, n, cost};
        }
    return best;
}

// First MLP layers (the ones with GELU, N from 4 K on) of up to FEW_ROWS rows and models up to 384 wide in panels of 32, one round of workgroups.
// A layer inside a stage, microseconds, in panels of 64 rows or two launches and so: DeiT-Small on 1 image 30.2 and 28.2, 4 32.9 and 31.2, 8 37.4
// and 36.3, 12 40.4 and 39.8; DeiT-Tiny on 1 image 22.4 and 21.8, 8 25.3 and 24.7, 12 26.3 and 25.9.  With q|k|v in them too another 0.4 to 1.4 us of
// DeiT-Small on 4 and 8 images; it keeps its panels of 64 rows and its two launches.  Past the line, 16 images 46.2 and 46.5, 24 51.8 and 61.1,
// DeiT-Tiny on 16 level, 24 31.6 and 34.5; by outputs, 384 wide with an MLP of 8 K 3.0 million 35.4 and 34.6, 4.8 level, 7.3 43.9 and 46.0, of 16 K
// 3.6 36.1 and 35.4, 6.1 41.4 and 42.0, 256 wide of 16 K 2.4 30.2 and 29.2, 4.0 31.5 and 31.8.  320 and 384 wide not past 16 K (384 of 32 K on 1
// image 36.9 in two launches and 38.8).  Narrower first layers keep what they had, though 1 to 3.5 K on 197 to 2364 rows would take 0.92 to 1.00 of it.
constexpr int FEW_BM = 32, FEW_ROWS = 2560;
constexpr int64_t FEW_OUTPUTS = 3800000;

bool few_rows(int64_t M, int N, int K)
{
    return K <= 384 && N >= 4 * K && M <= FEW_ROWS && M * N <= FEW_OUTPUTS && (K <= 256 || N <= 16 * K);
}

RowsPlan plan_rows(int64_t M, int N, int K, bool gelu, int cus)
{
    if (gelu && few_rows(M, N, K)) {
        const int64_t n = cus / ((M + FEW_BM - 1) / FEW_BM), units = N / 16;
        return {FEW_BM, (int)(n < 1 ? 1 : n < units ? n : units), 0.0};
    }
    // 384 wide, the model's plan is still the faster one where a round of 128 rows takes two thirds of the units (22458 and 24428 rows of
    // DeiT-Small, a layer: 141 and 146 us; lower panels, which read the weights twice as often, 149 and 153) and, but for MLPs of 8 K and
    // more, past that round (33884 rows: 245 and 249 us)
    const int64_t tall = (M + 127) / 128;
    const bool model = K > 320 && 3 * tall >= 2 * cus && (tall <= cus || N <= 4 * K);
    if (K <= 384 && M >= 1 << 14 && !model) return plan_many_narrow_rows(M, N, cus);
    RowsPlan best = {0, 0, 1e30};
    for (int bm : {K <= 384 ? 128 : K <= 512 ? 96 : K <= 768 ? 80 : 0, 64}) {
        if (!bm) continue;
        const int64_t n = cus / ((M + bm - 1) / bm), units = (N + UC - 1) / UC;
        const int groups = (int)(n < 1 ? 1 : n < units ? n : units);
        const double us = rows_us(M, N, K, gelu, bm, groups, cus);
        if (us < best.us) best = {bm, groups, us};
    }
    return best;
}

// Few rows of narrow models: panels of 32 rows, and 16 columns to a wave, so that a wave has few sets of them (one or two of the named models, up
// to five: 257 x 14784 x 256).  The weights of the first, all K of them, are under way while the rows come in.
template <int KS, int EPI>
hipError_t launch_few(const float *x, const float *g, const float *b, float eps, const uint16_t *W, const float *bias, void *C,
                      int M, int N, int groups, hipStream_t s)
{
    const int units = N / 16, per = (units + groups - 1) / groups;
    return launch_as<KS, FEW_BM, 1, KS, EPI, false>(x, g, b, eps, W, bias, C, M, N, per, (units + per - 1) / per, s);
}

template <int EPI>
hipError_t launch_k(const float *x, const float *g, const float *b, float eps, const uint16_t *W, const float *bias, void *C,
                    int M, int N, int K, int cus, bool touched, hipStream_t s)
{
    const RowsPlan p = plan_rows(M, N, K, EPI == EPI_BIAS_GELU, cus);
#define EP_FEW(KS) if (K == KS * 32 && p.bm == FEW_BM) return launch_few<KS, EPI>(x, g, b, eps, W, bias, C, M, N, p.groups, s)
    if constexpr (EPI == EPI_BIAS_GELU) { EP_FEW(2); EP_FEW(4); EP_FEW(6); EP_FEW(8); EP_FEW(10); EP_FEW(12); }
#undef EP_FEW
#define EP_ROWS(KS, BM) \
    if (K == KS * 32 && p.bm == BM) return launch_rows<KS, BM, EPI>(x, g, b, eps, W, bias, C, M, N, p.groups, touched, s)
    EP_ROWS(2, 128); EP_ROWS(2, 64);
    EP_ROWS(4, 128); EP_ROWS(4, 64);
    EP_ROWS(6, 128); EP_ROWS(6, 64);
    EP_ROWS(8, 128); EP_ROWS(8, 64);
    EP_ROWS(10, 128); EP_ROWS(10, 64);
    EP_ROWS(12, 128); EP_ROWS(12, 64);
    EP_ROWS(16, 96); EP_ROWS(16, 64);
    EP_ROWS(24, 80); EP_ROWS(24, 64);
    EP_ROWS(32, 64);
#undef EP_ROWS
    return hipErrorInvalidValue;
}

// The depths there are, and where the one launch is the faster one.  Few rows take longer to bring in than a launch is worth; wide layers
// are matrix work that tiles of 256 columns do with a quarter of the weights' traffic, and so are many rows; and the launch itself loses
// where its panels just begin another round.  A layer's time inside a stage, with FC1 in two launches against one
// (profiles/layernorm_dense_one_launch.md):
//   K = 384    N = 12 K at 505 rows 1.03, 32 K 0.96, from 1010 rows on 1.00 and more
//   K = 512    N = 4 K at 505 rows 0.99, at 2525 1.07; 12 K at 505 rows 0.97, at 1010 1.06; 16 K at 505 and 1010 0.95 and 1.01; 32 K at 8080 0.95
//   K = 768    weights touched, two launches and one, us: N = 4 K 58.0 and 57.1 at 1773 rows, 61.9 and 58.9 at 1970, 70.7 and 67.8 at 2561; 6 K 69.7
//              and 67.6 at 1970, 83.5 and 81.8; 8 K 75.0 and 75.2 at 1773, 76.3 and 75.4, 97.3 and 92.1; 12 K 89.4 and 89.9 at 1773, 97.7 and 95.1,
//              120.1 and 115.1.  Over 4 to 12 K, eight counts of rows from 1970 to 2561, weights resident and from memory, 0.94 to 0.99 (10 K at 1970
//              1.005), 3.5 K 0.96 to 0.99 but not taken; q|k|v 68.1 and 69.9 at 1970
//              N = 4 K at 2626 rows 1.04 and at 10302 (129 panels of 80 rows: one group, half the chip) 0.97, 8 K 1.06 and 0.93, 12 K 1.03 and 0.89,
//              8 K at 12625 1.00, 12 K at 11110 0.92, 16 K at 9595 0.98; two launches 139 us and one 147 at 25256 rows of 4 K
//   K = 1024   N = 4 K at 5555 rows 0.97, at 6161 1.02; 5 K at 6363 0.96, 8 K 0.94, 12 K 0.89; two launches 85 us and one 106 at 9456 rows of 4 K
// At 1024, layers past 2304 columns lose where tiles of 256 rows on their own are one nearly whole round: q|k|v at 6161 rows 0.99 and at 6565
// 1.02, N = 2.75 K at 5757 0.97 and at 5959 1.01.
// Below 5500 rows of 1024 the one launch takes 0.93 to 1.08 of the time of two with no line in rows, but for a first MLP layer whose weights
// attention has touched and whose own launch would be one round of 256 x 256 tiles that fills more than three quarters and up to 13 sixteenths
// of the units: 193 to 208 tiles (many others of so many run as 256 x 192 or 192 x 256).  A layer's time, one launch over two, N = 3.06 to 4.25 K,
// 2885 to 4050 rows, weights resident and from memory: 0.963 to 0.988 at 28 points, 0.98 to 1.00 at another three, 3300 rows (ViT-Large on 16
// images 107.5 -> 105.2 us and 111.3 -> 108.4).  210 to 225 tiles 0.975 to 1.01, more 0.93 to 1.04 without a line; tiles of 192 rows or
// columns 0.97 to 1.02.  Where attention has not touched the weights 1.01 to 1.05 (6 to 8 images of 577 tokens).
bool tiles_leave_units(int64_t M, int N, int K)
{
    const int64_t cus = ep_bf16_gemm_persistent_workgroups(), tiles = (M + 255) / 256 * ((N + 255) / 256);
    if (4 * tiles <= 3 * cus || 16 * tiles > 13 * cus) return false;
    EpDensePlan p;
    ep_query_dense_plan(M, N, K, EPI_BIAS_GELU, &p);
    return !p.persistent && p.bm == 256 && p.bn == 256;
}

bool one_launch_pays(int64_t M, int N, int K, bool gelu, bool touched)
{
    const double wide = (double)N / K;
    switch (K) {
    case 64: case 128: case 192: case 256: return true;
    case 320: case 384: return M >= 1024 || (M >= 500 && wide <= 16.0) || (gelu && few_rows(M, N, K));
    case 512: return M <= 20000 && ((M >= 500 && wide <= 8.0) || (M >= 1000 && wide <= 16.0));
    case 768: return M >= (wide >= 4.0 ? 1900 : 2600) && M <= 20000 && (M <= 10240 ? wide <= 12.0 : wide <= 3.0 || (M > 10752 && wide <= 8.0));
    case 1024:
        if (gelu && touched && M < 5500 && wide > 3.0 && wide <= 4.25 && tiles_leave_units(M, N, K)) return true;
        break;
    default: return false;
    }
    if (M < 5500 || M > 8192 || wide > 4.0 || (wide > 3.5 && M <= 5888)) return false;
    const int64_t cus = ep_bf16_gemm_persistent_workgroups(), rows = (M + 255) / 256;
    for (int bn : {256, 320}) {
        const int64_t tiles = rows * ((N + bn - 1) / bn);
        if (N > 2304 && tiles <= cus && 8 * tiles >= 7 * cus) return false;
    }
    return true;
}

}  // namespace

bool ep_bf16_ln_gemm_supported(int64_t M, int N, int K, int epi, bool touched)
{
    return one_launch_pays(M, N, K, epi == EPI_BIAS_GELU, touched) && N % 16 == 0 && N < MAX_TILE_N && M * N < (1ll << 31) && (int64_t)N * K * 2 < 0x7FFFFFF0ll;
}

extern "C" int32_t ep_query_ln_gemm_plan(int64_t M, int32_t N, int32_t K, int32_t epi, int32_t cus, int32_t *groups)
{
    if (M <= 0 || N <= 0 || !ep_bf16_ln_gemm_supported(M, N, K, epi, false)) return 0;
    const RowsPlan p = plan_rows(M, N, K, epi == EPI_BIAS_GELU, cus);
    *groups = p.groups;
    return p.bm;
}

extern "C" int32_t ep_query_ln_gemm_touched_mlp(int64_t M, int32_t N, int32_t K) { return ep_bf16_ln_gemm_supported(M, N, K, EPI_BIAS_GELU, true); }

hipError_t ep_bf16_ln_gemm(const float *x, const float *g, const float *b, float eps, const uint16_t *W, const float *bias, void *C,
                           int64_t M, int N, int K, int epi, bool touched, hipEvent_t after_main, hipStream_t s)
{
    if (M <= 0 || N <= 0) return hipSuccess;
    if (!ep_bf16_ln_gemm_supported(M, N, K, epi, touched) || (epi != EPI_BIAS && epi != EPI_BIAS_GELU)) return hipErrorInvalidValue;
    int cus = 0;
    hipError_t e = ep_device_cu_count(&cus);
    if (e != hipSuccess) return e;
    e = epi == EPI_BIAS ? launch_k<EPI_BIAS>(x, g, b, eps, W, bias, C, (int)M, N, K, cus, touched, s)
                        : launch_k<EPI_BIAS_GELU>(x, g, b, eps, W, bias, C, (int)M, N, K, cus, touched, s);
    if (e != hipSuccess) return e;
    if (after_main) e = hipEventRecord(after_main, s);
    return e;
}
