// bf16 dense layers of small and middling batches (paper section 2.1; a pipeline's micro-batches are such, section 3.1):
//
//   C[M, N] = A[M, K] . W[N, K]^T + bias[N]   (+ erf GELU | + fp32 residual | bare sum over a K range)
//
// One BM x BN tile of C to a workgroup of four multiplying waves, side by side along N, and two loader waves.
//   - The loaders bring the panels of A, 64 of K at a time, into a ring of S stages in LDS (buffer_load ... lds)
//     and do nothing else: a wave that issues such a load is held until the address pipe takes it, 16 clocks for each
//     1 KB of the compute unit, and whoever multiplies in between waits with it.
//   - Weights are in fragment order (ep_gemm_bf16_tile.h): a multiplying wave reads the fragments of its own columns
//     straight into registers, D steps ahead.  They pass LDS neither way, no two waves read the same ones, and A is
//     all that LDS holds, so the ring is deep where tiles are small.
//   - A wave keeps one fragment of A a 16-row block and re-reads each as soon as it has been multiplied with, one
//     slice ahead; one barrier per K step, after the first block of its second slice: by then every wave has
//     read the stage for the last time and the next one has landed.
// Loads to LDS and loads to registers are never outstanding in the same wave: no wait counts one kind among the other.
//
// What bounds it: a compute unit takes in 64 bytes a clock (57 with all of them at it), (BM + BN) * 128 bytes a K step,
// 575 clocks for 128 x 128 next to 512 of matrix instructions; with every wave loading through LDS for itself
// a step took 780 to 880.  Then launch, first panel (1 us) and epilogue, half of a launch of a dozen K steps.
// Against tiles of the same shape whose waves all load both operands through LDS and store from their accumulators,
// microseconds a launch with weights from memory: 197 rows of ViT-Large 6.8 -> 5.9 (q|k|v), 6.7 -> 5.6 (projection),
// 7.4 -> 6.4 and 7.7 -> 6.6 (MLP); 985 rows 12.2 -> 10.6, 7.7 -> 7.0, 13.3 -> 12.4, 15.5 -> 13.2; 1576 rows of
// ViT-Base 9.9 -> 8.8, 8.8 -> 6.9, second MLP layer 16.5 -> 13.8; 3152 x 1024 x 4096 38.6 -> 33.9 (780 TFLOP/s);
// 6304 x 384 x 1536 17.1 -> 14.1.  The same sums in the same order.  Deeper rings than these gain nothing, nor do
// one loader or four.
//
// RANGES: K is gone through in ranges of k_len, each with a sum of its own that is added to those before it: the bits of
// EPI_PARTIAL and of whoever adds its ranges up, without their way through memory, at twice the accumulators.
//
// Rows past M and columns past N read as zeros and are never stored.  K % 64 == 0 and N % 16 == 0.
#include "ep_gemm_bf16_tile.h"
#include "ep_launch.h"

namespace {

using namespace ep_tile;

constexpr int NW = 4, NL = 2;                        // multiplying waves, loader waves

template <int BM, int BN, int S, int D, int WAVES_PER_SIMD, int EPI, bool RANGES>
__global__ __launch_bounds__((NW + NL) * 64, WAVES_PER_SIMD) void gemm_bf16_stream_kernel(
    int M, int N, int K, int k_len, const uint16_t *A, const uint16_t *W, const float *bias, const float *resid, void *Cout)
{
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int MI = BM / 16, NI = BN / NW / 16;   // 16 x 16 accumulators of a wave
    constexpr int STAGE = BM * CPR;                  // uint4 of a stage
    constexpr int L = BM / 8 / NL;                   // loads of a loader and stage, 8 rows each
    static_assert(BM % (8 * NL) == 0 && BN % (16 * NW) == 0 && S >= 2 && (S - 1) * L <= 63, "whole loads, vmcnt is six bits");
    extern __shared__ uint4 lds[];

    const TileOf t = tile_of((M + BM - 1) / BM, (N + BN - 1) / BN, EPI == EPI_PARTIAL ? K / k_len : 1);
    if (!t.live) return;
    const int m0 = t.m * BM, n0 = t.n * BN, k0 = t.range * k_len, KT = (RANGES ? K : k_len) / BK;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    if (wave >= NW) {
        // ---- loaders: load i fills rows (i * NL + lw) * 8 .. + 7 of a stage; lane l lands at row l / 8, slot l % 8 and
        // fetches chunk slot ^ swz(row)
        const int lw = wave - NW;
        __builtin_amdgcn_s_setprio(3);               // a load issued late is a load landed late
        const __amdgpu_buffer_rsrc_t a_rs = make_rsrc(A, (uint32_t)((size_t)M * K * 2));
        int off[L];
#pragma unroll
        for (int i = 0; i < L; ++i) {
            const int r = (i * NL + lw) * 8 + (lane >> 3);
            off[i] = m0 + r < M ? ((m0 + r) * K + k0 + ((lane & 7) ^ swz(r)) * 8) * 2 : OOB;
        }
        auto issue = [&](int kt, int slot) EP_INLINE {
#pragma unroll
            for (int i = 0; i < L; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rs, (lds_ptr)(lds + slot * STAGE + (i * NL + lw) * 64), 16, off[i], kt * (BK * 2), 0, 0);
        };
        auto landed = [&](int newer) EP_INLINE {               // all but the `newer` youngest stages
            static_for<S - 1>([&](auto n) EP_INLINE {
                if (newer == decltype(n)::value) EP_WAIT_VMCNT(decltype(n)::value * L);
            });
            if (newer < 0) EP_WAIT_VMCNT(0);
        };
        int issued = 0, slot = 0;
        for (; issued < min(S, KT); ++issued) issue(issued, issued);
        if (issued == S) EP_WAIT_VMCNT((S - 1) * L);
        else landed(issued - 1);
        __builtin_amdgcn_s_barrier();                // stage 0 is there
        for (int j = 0; j < KT; ++j) {
            landed(issued - 2 - j);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();            // stage j + 1 is there; stage j has been read
            asm volatile("" ::: "memory");
            if (issued < KT) issue(issued++, slot);
            slot = slot + 1 == S ? 0 : slot + 1;
        }
        __builtin_amdgcn_s_barrier();                // the ring becomes the staging area of the epilogue
        return;
    }

    // ---- multiplying waves
    const int wn0 = n0 + wave * (NI * 16);
    const int l15 = lane & 15, g4 = lane >> 4;
    const int nb = N / 16, nb0 = wn0 / 16;
    const int block = K * 32;                        // bytes of the fragments of 16 columns
    const char *w_base = reinterpret_cast<const char *>(W) + (size_t)min(nb0, nb) * block;
    const uint32_t w_bytes = nb0 < nb ? (uint32_t)(nb - nb0) * (uint32_t)block : 0u;
    // fragments of A: RA of them, each sent for RA blocks ahead; RA divides the fragments of a step
    constexpr int RA = RANGES && MI == 10 ? 4 : MI <= 13 ? MI : MI == 15 ? 10 : MI / 2;
    static_assert(NS * MI % RA == 0, "a step's fragments end with the registers");
    bf16x8 wf[D][NS][NI], af[RA];
    // fragment (slice, ni) of step kt.  Steps past the last read an empty buffer.  The empty assembly keeps the loads
    // in their places, which the compiler would otherwise move down to where the loop closes.
    auto load_w = [&](int kt, int d, int slice, int ni) EP_INLINE {
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(w_base, kt < KT ? w_bytes : 0u);
        wf[d][slice][ni] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16 + ni * block, (k0 / 32 + kt * NS + slice) * FRAG_BYTES, 0));
        asm volatile("" ::: "memory");
    };
    int a_rd[NS];
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) a_rd[sl] = l15 * CPR + ((sl * 4 + kchunk(g4)) ^ swz(l15));
    auto read_a = [&](const uint4 *stage, int f) EP_INLINE {        // block f of the step: slice f / MI, rows f % MI
        af[f % RA] = __builtin_bit_cast(bf16x8, stage[a_rd[f / MI] + f % MI * 16 * CPR]);
    };

    typedef WaveOut<MI, NI, EPI> Out;
    // the residual is fetched ahead of the K loop where registers hold it (a launch of a dozen steps would otherwise end
    // with one more trip to memory), a pass of rows of it otherwise
    constexpr int FREE = (WAVES_PER_SIMD == 3 ? 128 : 216) - (RANGES ? 2 : 1) * NI * MI * 4 - MI * 4 - D * NS * NI * 4;     // registers
    constexpr int FIT = FREE > 0 ? FREE / (Out::PP * 4) : 0, AHEAD = !Out::RES ? 0 : FIT < Out::NPASS ? FIT : Out::NPASS;
    Out out;
    out.init(Cout, resid, bias, m0, BM, 0, wn0, M, N, (size_t)t.range * M, lane);
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
        for (int sl = 0; sl < NS; ++sl)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
                if (d < D - 1 || sl == 0) load_w(d, d, sl, ni);     // the loop's first step sends for the rest
    static_for<AHEAD>([&](auto p) EP_INLINE { out.fetch(decltype(p)::value); });
    asm volatile("" ::: "memory");
    f32x4 acc[NI][MI];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) acc[ni][mi] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 sum[RANGES ? NI : 1][RANGES ? MI : 1];     // of the ranges that are over
    int left = k_len / BK;                           // steps of the range

    __builtin_amdgcn_s_barrier();
    EP_SCHED_FENCE();
#pragma unroll
    for (int f = 0; f < RA; ++f) read_a(lds, f);
    EP_SCHED_FENCE();
    int slot = 0;
    auto step = [&](int kt, auto d_c) EP_INLINE {
        constexpr int d = decltype(d_c)::value, prev = (d + D - 1) % D;
        const int next = slot + 1 == S ? 0 : slot + 1;
        const uint4 *cur_stage = lds + slot * STAGE, *next_stage = lds + next * STAGE;
        static_for<NS * MI>([&](auto f_c) EP_INLINE {
            constexpr int f = decltype(f_c)::value, sl = f / MI, mi = f % MI;
            constexpr bool last = sl == NS - 1;
            static_for<NI>([&](auto n_c) EP_INLINE {
                constexpr int q = mi * NI + decltype(n_c)::value, Q = MI * NI;
                constexpr int ni = (mi & 1) ? NI - 1 - decltype(n_c)::value : decltype(n_c)::value;
                acc[ni][mi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[d][sl][ni], af[f % RA], acc[ni][mi], 0, 0, 0);
                EP_SCHED_FENCE();
                // the weights of the slice before this one have been used: those D steps on take their registers
                static_for<NI>([&](auto j_c) EP_INLINE {
                    constexpr int j = decltype(j_c)::value;
                    if constexpr (j * Q / NI + Q / NI / 2 == q) {
                        if constexpr (last) load_w(kt + D, d, 0, j);
                        else load_w(kt + D - 1, prev, 1, j);
                        EP_SCHED_FENCE();
                    }
                });
            });
            if constexpr (f + RA == NS * MI) {
                EP_WAIT_LGKMCNT0();
                __builtin_amdgcn_s_barrier();
                EP_SCHED_FENCE();
            }
            if constexpr (f + RA < NS * MI) read_a(cur_stage, f + RA);
            else read_a(next_stage, f + RA - NS * MI);
            EP_SCHED_FENCE();
        });
        slot = next;
        if constexpr (RANGES)
            if (--left == 0) {
                left = k_len / BK;
                const bool first = kt < left;
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                    for (int mi = 0; mi < MI; ++mi) {
                        sum[ni][mi] = first ? acc[ni][mi] : sum[ni][mi] + acc[ni][mi];
                        acc[ni][mi] = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
                EP_SCHED_FENCE();
            }
    };
    int kt = 0;
    for (; kt + D <= KT; kt += D)
        static_for<D>([&](auto d_c) EP_INLINE { step(kt + decltype(d_c)::value, d_c); });
    static_for<D - 1>([&](auto d_c) EP_INLINE {
        if (kt + decltype(d_c)::value < KT) step(kt + decltype(d_c)::value, d_c);
    });

    EP_WAIT_LGKMCNT0();
    __builtin_amdgcn_s_barrier();                    // everyone is done with the ring
    if constexpr (RANGES) out.template store<AHEAD>(sum, reinterpret_cast<char *>(lds) + wave * Out::LDS_BYTES);
    else out.template store<AHEAD>(acc, reinterpret_cast<char *>(lds) + wave * Out::LDS_BYTES);
#endif
}

template <int BM, int BN, int S, int D, int WAVES_PER_SIMD, int EPI, bool RANGES = false>
hipError_t launch_cfg(const uint16_t *A, const uint16_t *W, const float *bias, const float *resid, void *C, int M, int N,
                      int K, int splits, hipStream_t s)
{
    auto kern = gemm_bf16_stream_kernel<BM, BN, S, D, WAVES_PER_SIMD, EPI, RANGES>;
    constexpr size_t ring = (size_t)S * BM * CPR * sizeof(uint4), stage = NW * WaveOut<BM / 16, BN / NW / 16, EPI>::LDS_BYTES;
    constexpr size_t smem = ring > stage ? ring : stage;
    static_assert(smem <= 160 * 1024, "LDS of a compute unit");
    static EpSmemLimit smem_limit;
    const hipError_t e = smem_limit.ensure(reinterpret_cast<const void *>(kern), (int)smem);
    if (e != hipSuccess) return e;
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN, total = tiles_m * tiles_n * (RANGES ? 1 : splits);
    hipLaunchKernelGGL(kern, dim3((total + NUM_XCD - 1) / NUM_XCD * NUM_XCD), dim3((NW + NL) * 64), smem, s, M, N, K, K / splits,
                       A, W, bias, resid, C);
    return hipGetLastError();
}

template <int BM, int BN, int S, int D, int WAVES_PER_SIMD>
hipError_t launch_epi(const uint16_t *A, const uint16_t *W, const float *bias, const float *resid, void *C, int M, int N,
                      int K, int splits, int epi, hipStream_t s)
{
    switch (epi) {
    case EPI_BIAS: return launch_cfg<BM, BN, S, D, WAVES_PER_SIMD, EPI_BIAS>(A, W, bias, resid, C, M, N, K, 1, s);
    case EPI_BIAS_GELU:
        if constexpr (BM <= 128) return launch_cfg<BM, BN, S, D, WAVES_PER_SIMD, EPI_BIAS_GELU>(A, W, bias, resid, C, M, N, K, 1, s);
        break;
    case EPI_BIAS_RESID: return launch_cfg<BM, BN, S, D, WAVES_PER_SIMD, EPI_BIAS_RESID>(A, W, bias, resid, C, M, N, K, 1, s);
    case EPI_PARTIAL: return launch_cfg<BM, BN, S, D, WAVES_PER_SIMD, EPI_PARTIAL>(A, W, bias, resid, C, M, N, K, splits, s);
    }
    return hipErrorInvalidValue;
}

// one 16-byte piece of the fragments to a thread
__global__ __launch_bounds__(256) void pack_weights_kernel(const uint16_t *__restrict__ w, uint16_t *__restrict__ p, int N, int K)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)N * K / 8) return;
    const int lane = (int)(i & 63);
    const int64_t frag = i >> 6;
    const int ks = K / 32;
    const int64_t n = frag / ks * 16 + (lane & 15);
    const int k = (int)(frag % ks) * 32 + kchunk(lane >> 4) * 8;
    reinterpret_cast<uint4 *>(p)[i] = *reinterpret_cast<const uint4 *>(w + n * K + k);
}

}  // namespace

hipError_t ep_bf16_pack_weights(const uint16_t *w, uint16_t *p, int N, int K, hipStream_t s)
{
    if (N <= 0 || K <= 0 || N % 16 || K % 32) return hipErrorInvalidValue;
    const int64_t n = (int64_t)N * K / 8;
    hipLaunchKernelGGL(pack_weights_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, w, p, N, K);
    return hipGetLastError();
}

// bm x bn: a tile shape of the dispatcher's table, 128 columns or fewer, or one of the heights between.  Up to 128 x 128 two
// workgroups fit a compute unit (three waves to a SIMD, 168 registers).
hipError_t ep_bf16_gemm_stream(int bm, int bn, const uint16_t *A, const uint16_t *W, const float *bias, const float *resid,
                               void *C, int64_t M, int N, int K, int splits, int epi, hipStream_t s)
{
    if (bm == 64 && bn == 64) return launch_epi<64, 64, 8, 4, 3>(A, W, bias, resid, C, (int)M, N, K, splits, epi, s);
    if (bm == 64 && bn == 128) return launch_epi<64, 128, 6, 4, 3>(A, W, bias, resid, C, (int)M, N, K, splits, epi, s);
    if (bm == 80 && bn == 128) return launch_epi<80, 128, 6, 4, 3>(A, W, bias, resid, C, (int)M, N, K, splits, epi, s);
    if (bm == 96 && bn == 128) return launch_epi<96, 128, 5, 3, 3>(A, W, bias, resid, C, (int)M, N, K, splits, epi, s);
    if (bm == 128 && bn == 128) return launch_epi<128, 128, 4, 3, 3>(A, W, bias, resid, C, (int)M, N, K, splits, epi, s);
    if (epi == EPI_BIAS_GELU) return hipErrorInvalidValue;
    if (bm == 144 && bn == 128) return launch_epi<144, 128, 6, 3, 2>(A, W, bias, resid, C, (int)M, N, K, splits, epi, s);
    if (bm == 160 && bn == 128) return launch_epi<160, 128, 6, 3, 2>(A, W, bias, resid, C, (int)M, N, K, splits, epi, s);
    if (bm == 176 && bn == 128) return launch_epi<176, 128, 5, 3, 2>(A, W, bias, resid, C, (int)M, N, K, splits, epi, s);
    if (bm == 192 && bn == 128) return launch_epi<192, 128, 5, 3, 2>(A, W, bias, resid, C, (int)M, N, K, splits, epi, s);
    if (bm == 208 && bn == 128) return launch_epi<208, 128, 5, 3, 2>(A, W, bias, resid, C, (int)M, N, K, splits, epi, s);
    if (bm == 224 && bn == 128) return launch_epi<224, 128, 5, 3, 2>(A, W, bias, resid, C, (int)M, N, K, splits, epi, s);
    if (bm == 240 && bn == 128) return launch_epi<240, 128, 4, 3, 2>(A, W, bias, resid, C, (int)M, N, K, splits, epi, s);
    if (bm == 256 && bn == 128) return launch_epi<256, 128, 4, 3, 2>(A, W, bias, resid, C, (int)M, N, K, splits, epi, s);
    return hipErrorInvalidValue;
}

// heights whose second set of sums the registers hold (160 rows with a longer ring of fragments, and 80 two to a unit, spill); 64 were
// modelled to be the fastest for one of 3500 layers
hipError_t ep_bf16_gemm_stream_ranges(int bm, const uint16_t *A, const uint16_t *W, const float *bias, const float *resid, float *C,
                                      int64_t M, int N, int K, int splits, hipStream_t s)
{
    if (bm == 128) return launch_cfg<128, 128, 6, 3, 2, EPI_BIAS_RESID, true>(A, W, bias, resid, C, (int)M, N, K, splits, s);
    if (bm == 160) return launch_cfg<160, 128, 6, 3, 2, EPI_BIAS_RESID, true>(A, W, bias, resid, C, (int)M, N, K, splits, s);
    return hipErrorInvalidValue;
}
